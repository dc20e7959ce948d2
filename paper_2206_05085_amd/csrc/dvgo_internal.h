// Internal helpers shared by the gfx950 kernels of libdvgo (not part of the C-ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dvgo.h"

namespace dvgo {

// ----------------------------------------------------------------------------- wave64

// All scans run across the 64 lanes of one wavefront (CDNA wave64).
__device__ __forceinline__ int lane() { return (int)__lane_id(); }

// inclusive prefix sum: lane l gets sum of lanes 0..l
__device__ __forceinline__ float wave_incl(float v) {
    const int l = lane();
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        float t = __shfl_up(v, d, 64);
        if (l >= d) v += t;
    }
    return v;
}

// exclusive prefix from an inclusive one (lane 0 gets 0); exact, no subtraction
__device__ __forceinline__ float wave_excl(float incl) {
    float t = __shfl_up(incl, 1, 64);
    return lane() == 0 ? 0.f : t;
}

// inclusive suffix sum: lane l gets sum of lanes l..63
__device__ __forceinline__ float wave_incl_rev(float v) {
    const int l = lane();
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        float t = __shfl_down(v, d, 64);
        if (l + d < 64) v += t;
    }
    return v;
}

// exclusive suffix from an inclusive suffix (lane 63 gets 0)
__device__ __forceinline__ float wave_excl_rev(float incl_rev) {
    float t = __shfl_down(incl_rev, 1, 64);
    return lane() == 63 ? 0.f : t;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

__device__ __forceinline__ float bcast(float v, int src) { return __shfl(v, src, 64); }

// --------------------------------------------------------------------------- math

__device__ __forceinline__ float softplusf(float z) {
    return z > 0.f ? z + log1pf(expf(-z)) : log1pf(expf(z));
}

__device__ __forceinline__ float sigmoidf(float z) {
    if (z >= 0.f) return 1.f / (1.f + expf(-z));
    float e = expf(z);
    return e / (1.f + e);
}

// --------------------------------------------------------------------------- grids

// Device view of a dvgo_grid.  The world->index map u = x*s + o per axis is carried as
// double-float pairs (hi + lo) so the cell index and the fractional position are exact to
// float32 precision of the fraction itself, not of u (u reaches 319 on a 320^3 grid).
struct DevGrid {
    const float *data;
    float *grad;
    int n[3];
    int cs;  // floats per vertex
    int C;   // channels used
    int sx, sy;  // strides (floats) of x and y; z stride is cs
    float s_hi[3], s_lo[3], o_hi[3], o_lo[3];
    int warp;              // DVGO_WARP_*: 0 = points index the box directly
    double wb;             // b of Eq. 4
    double s_d[3], o_d[3]; // the index map u = x*s + o in double, for warped points
};

struct Tri {
    int base;     // float offset of corner (0,0,0)
    float w[8];   // corner c = 4dx + 2dy + dz
};

// Cell index i0 in [0, n-2] and fraction f in [0, 1] of coordinate x on one axis.
__device__ __forceinline__ void axis_coord(float x, float shi, float slo, float ohi, float olo, int n, int &i0,
                                           float &f) {
    // The error-free transforms below need each operation rounded on its own: an FMA
    // formed from x*shi + ohi would break the two-sum.
#pragma clang fp contract(off)
    // x*shi exactly as p + pe (FMA), then p + ohi exactly as u + e (two-sum)
    float p = x * shi;
    float pe = fmaf(x, shi, -p);
    float u = p + ohi;
    float bb = u - p;
    float e = (p - (u - bb)) + (ohi - bb);
    float lo = e + pe + fmaf(x, slo, olo);
    float fl = floorf(u);
    float fr = (u - fl) + lo;  // u - fl is exact
    if (fr < 0.f) { fl -= 1.f; fr += 1.f; }
    else if (fr >= 1.f) { fl += 1.f; fr -= 1.f; }
    const float top = (float)(n - 2);
    if (!(fl >= 0.f)) { i0 = 0; f = 0.f; }               // below the box (or NaN)
    else if (fl > top) { i0 = n - 2; f = 1.f; }          // on or above the upper face
    else { i0 = (int)fl; f = fr; }
}

// Cell index and fraction of a point addressed through the unbounded-scene contraction
// (Eq. 4, p = inf or 2).  The contraction and the index map run in double, so the fraction
// is accurate to float32 although the contracted point is a derived value; the clamping
// matches axis_coord.  Every rounding is written out (explicit FMAs, no contraction): the binning and the
// scatter of the bins each form a point's cell, and an LDS tile has room only for cells that agree.
__device__ __forceinline__ void warped_coords(const DevGrid &g, float x, float y, float z, int (&i)[3],
                                              float (&f)[3]) {
#pragma clang fp contract(off)
    double p[3] = {(double)x, (double)y, (double)z};
    double n;
    if (g.warp == DVGO_WARP_CONTRACT_INF) {
        n = fabs(p[0]);
        n = fabs(p[1]) > n ? fabs(p[1]) : n;
        n = fabs(p[2]) > n ? fabs(p[2]) : n;
    } else {
        n = sqrt(__builtin_fma(p[2], p[2], __builtin_fma(p[0], p[0], p[1] * p[1])));
    }
    const double r = 1.0 / n;  // the one division of the contraction
    const double s = n > 1.0 ? __builtin_fma(-g.wb, r, 1.0 + g.wb) * r : 1.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double u = __builtin_fma(p[a] * s, g.s_d[a], g.o_d[a]);
        const double fl = floor(u);
        if (!(fl >= 0.0)) { i[a] = 0; f[a] = 0.f; }              // below the box (or NaN)
        else if (fl > (double)(g.n[a] - 2)) { i[a] = g.n[a] - 2; f[a] = 1.f; }
        else { i[a] = (int)fl; f[a] = (float)(u - fl); }
    }
}

// W: the kernel was built for grids with a warp (the double-precision contraction path costs
// registers, so kernels for plain grids leave it out).
template <bool W>
__device__ __forceinline__ void grid_coords(const DevGrid &g, float x, float y, float z, int (&i)[3], float (&f)[3]) {
    if (W && g.warp) {
        warped_coords(g, x, y, z, i, f);
        return;
    }
    axis_coord(x, g.s_hi[0], g.s_lo[0], g.o_hi[0], g.o_lo[0], g.n[0], i[0], f[0]);
    axis_coord(y, g.s_hi[1], g.s_lo[1], g.o_hi[1], g.o_lo[1], g.n[1], i[1], f[1]);
    axis_coord(z, g.s_hi[2], g.s_lo[2], g.o_hi[2], g.o_lo[2], g.n[2], i[2], f[2]);
}

template <bool W = false>
__device__ __forceinline__ Tri trilinear(const DevGrid &g, float x, float y, float z) {
    int i[3];
    float fr[3];
    grid_coords<W>(g, x, y, z, i, fr);
    const int ix = i[0], iy = i[1], iz = i[2];
    const float fx = fr[0], fy = fr[1], fz = fr[2];
    Tri t;
    t.base = ix * g.sx + iy * g.sy + iz * g.cs;
    const float wx[2] = {1.f - fx, fx}, wy[2] = {1.f - fy, fy}, wz[2] = {1.f - fz, fz};
#pragma unroll
    for (int c = 0; c < 8; ++c) t.w[c] = (wx[(c >> 2) & 1] * wy[(c >> 1) & 1]) * wz[c & 1];
    return t;
}

// Cell and fractions of a point (the inputs of the trilinear weights), kept for the
// aggregated scatter below.
struct Cell {
    int ix, iy, iz;
    float fx, fy, fz;
};

template <bool W = false>
__device__ __forceinline__ Cell cell_of(const DevGrid &g, float x, float y, float z) {
    int i[3];
    float fr[3];
    grid_coords<W>(g, x, y, z, i, fr);
    return Cell{i[0], i[1], i[2], fr[0], fr[1], fr[2]};
}

__device__ __forceinline__ float corner_weight(const Cell &c, int dx, int dy, int dz) {
    return ((dx ? c.fx : 1.f - c.fx) * (dy ? c.fy : 1.f - c.fy)) * (dz ? c.fz : 1.f - c.fz);
}

// Orders the calling wave's LDS accesses (for the compiler and the hardware) without waiting
// for its outstanding global stores and atomics, which stay in flight.
__device__ __forceinline__ void lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup", "local"); }

// Adjoint of trilinear interpolation along a run of consecutive samples: the slot walk.
//
// Consecutive samples lie along a ray, so they share vertices with their neighbours.  A cell has
// exactly one vertex of each parity class (x mod 2, y mod 2, z mod 2), and a vertex keeps its class
// for as long as the walk stays in its cells: eight accumulators, one per class, hold the vertices of
// the current cell, and one leaves (a single global atomic) only when the walk moves to a cell that
// has another vertex of its class.  A group of GL = (8 / SL) NC adjacent lanes walks one run of samples,
// lane = (classes, channel) with SL of the eight classes in registers; the lanes of one class hold
// consecutive channels and those of the two z parities follow each other, so vertices of one column
// that leave together leave as one contiguous span.  64 / GL groups per wave walk side by side.
//
// A sample's cell is a float4 (stage_cell): the offset of the cell's low corner and the three
// fractions, each with the parity of its cell index in the (otherwise clear) sign bit.  Where a group
// has more than one lane the cells are staged in LDS, one lane per sample.
__device__ __forceinline__ float4 stage_cell(int low, const Cell &c) {
    const auto tag = [](float f, int i) {
        return __builtin_bit_cast(float, (__builtin_bit_cast(unsigned, f) & 0x7fffffffu) | ((unsigned)i << 31));
    };
    return make_float4(__builtin_bit_cast(float, low), tag(c.fx, c.ix), tag(c.fy, c.iy), tag(c.fz, c.iz));
}
__device__ __forceinline__ float4 stage_cell(const DevGrid &g, const Cell &c) {
    return stage_cell(c.ix * g.sx + c.iy * g.sy + c.iz * g.cs, c);
}

// where a finished vertex sum goes: base[offset] in global memory or in LDS
struct GlobalSum {
    float *base;
    __device__ __forceinline__ void operator()(int at, float v) const { unsafeAtomicAdd(base + at, v); }
};
// LDS sums are kept in double: on gfx950 an LDS atomic add of 64 floats occupies the CU's LDS for about 80
// ns, one of 64 doubles for 4 to 9.
struct LdsSum {
    double *base;
    __device__ __forceinline__ void operator()(int at, float v) const { atomicAdd(base + at, (double)v); }
};

template <int NC, int SL>
struct SlotWalk {
    static constexpr int GL = (8 / SL) * NC;  // lanes of a group
    static constexpr int NG = 64 / GL;        // groups of a wave
    static_assert(GL <= 64 && (SL == 1 || SL == 2 || SL == 4 || SL == 8), "a group fits a wave");
    int cur[SL];    // offset (without the channel) of the vertex each slot holds
    float acc[SL];  // its sum so far; 0 when nothing is held
    int group, ch, hi;

    __device__ __forceinline__ SlotWalk() {
        group = lane() / GL;
        const int r = lane() - group * GL;
        hi = r / NC;
        ch = r - hi * NC;
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            cur[s] = 0;
            acc[s] = 0.f;
        }
    }
    // fraction weight and vertex offset of parity class p on one axis
    static __device__ __forceinline__ void axis(float tagged, int p, int stride, float &w, int &off) {
        const int bits = __builtin_bit_cast(int, tagged);
        const float f = __builtin_bit_cast(float, bits & 0x7fffffff);
        const bool up = (bits < 0) != (p != 0);  // the cell's vertex of this class is its upper one
        w = up ? f : 1.f - f;
        off = up ? stride : 0;
    }
    // one sample: its cell and this lane's channel value; sx, sy, sz: vertex strides of the target
    template <class Sum>
    __device__ __forceinline__ void step(int sx, int sy, int sz, const float4 &rec, float v, const Sum &sum) {
        constexpr int NX = SL > 1 ? 2 : 1, NY = SL > 2 ? 2 : 1, NZ = SL > 4 ? 2 : 1;  // classes in registers
        float wx[NX], wy[NY], wz[NZ];
        int ox[NX], oy[NY], oz[NZ];
#pragma unroll
        for (int p = 0; p < NX; ++p) axis(rec.y, NX > 1 ? p : (hi >> 2) & 1, sx, wx[p], ox[p]);
#pragma unroll
        for (int p = 0; p < NY; ++p) axis(rec.z, NY > 1 ? p : (hi >> 1) & 1, sy, wy[p], oy[p]);
#pragma unroll
        for (int p = 0; p < NZ; ++p) axis(rec.w, NZ > 1 ? p : hi & 1, sz, wz[p], oz[p]);
        const int base = __builtin_bit_cast(int, rec.x);
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            const int ix = s & 1, iy = (s >> 1) & 1, iz = s >> 2;
            const int at = base + ox[ix] + oy[iy] + oz[iz];
            const float w = (wx[ix] * wy[iy]) * wz[iz];
            if (at != cur[s]) {
                if (acc[s] != 0.f) sum(cur[s], acc[s]);
                cur[s] = at;
                acc[s] = w * v;
            } else {
                acc[s] = __builtin_fmaf(w, v, acc[s]);
            }
        }
    }
    // group g (a multiple of 2 K) takes over the sums of group g + K on the vertices both hold; whether any did (wave-uniform)
    template <int K>
    __device__ __forceinline__ bool join_at() {
        const int r = group & (2 * K - 1);
        const bool take = r == 0 && group + K < NG, give = r == K && group < NG;
        const int other = lane() + (take ? K * GL : (give ? -K * GL : 0));
        bool same[SL], any = false;
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            const int at = __shfl(cur[s], other, 64);
            same[s] = (take || give) && at == cur[s];
            any |= same[s] && acc[s] != 0.f;
        }
        if (!__any(any)) return false;
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            const float v = __shfl(acc[s], other, 64);
            acc[s] = same[s] ? (take ? acc[s] + v : 0.f) : acc[s];
        }
        return true;
    }
    // Groups of the wave that end on the same vertices join their sums: neighbours first, then, if any two of
    // them agreed, groups two and four apart.  Costs a wave on ordinary rays one look (no difference measured);
    // where a wave's samples all lie in one cell (rays behind the box's face, a small grid) its groups would
    // otherwise each send the same eight vertices: render_bwd of 491,520 samples at one point 786 -> 111 us,
    // of 300,000 samples along rays through an 8^3 grid 123 -> 67.  All 64 lanes must call it.
    __device__ __forceinline__ void join() {
        static_assert(NG <= 8, "three distances");
        if (!join_at<1>()) return;
        if constexpr (NG > 2) join_at<2>();
        if constexpr (NG > 4) join_at<4>();
    }
    template <class Sum>
    __device__ __forceinline__ void finish(const Sum &sum) {
#pragma unroll
        for (int s = 0; s < SL; ++s)
            if (acc[s] != 0.f) sum(cur[s], acc[s]);
    }
};

// The slot walk over one chunk of at most 64 samples of a wave: lane l holds sample l (the first n
// are real), its cell and its value; channel c of sample l takes val scaled by f0, f1, f2.  rec and
// vals: this wave's LDS (64 entries each).  All lanes must call it.
template <int NC, int SL>
__device__ __forceinline__ void walk_chunk(const DevGrid &g, int n, const Cell &cl, float val, float f0, float f1,
                                           float f2, float4 *rec, float *vals) {
    static_assert(NC <= 3, "three scale factors");
    using Walk = SlotWalk<NC, SL>;
    constexpr int T = (64 + Walk::NG - 1) / Walk::NG;  // samples of a group
    const int ln = lane();
    rec[ln] = stage_cell(g, cl);
    vals[ln] = val;
    lds_fence();
    Walk wk;
    const int b = wk.group * T;
    const int cnt = wk.group < Walk::NG ? min(min(n, 64) - b, T) : 0;
    const float fc = wk.ch == 0 ? f0 : (wk.ch == 1 ? f1 : f2);
    const GlobalSum sum{g.grad + wk.ch};
    for (int t = 0; t < cnt; ++t) wk.step(g.sx, g.sy, g.cs, rec[b + t], vals[b + t] * fc, sum);
    wk.join();
    wk.finish(sum);
    lds_fence();
}
constexpr int WALK_LDS_PER_WAVE = 64 * 20;  // bytes walk_chunk needs for each wave of a block

__device__ __forceinline__ Tri tri_from_cell(const DevGrid &g, const Cell &c) {
    Tri t;
    t.base = c.ix * g.sx + c.iy * g.sy + c.iz * g.cs;
#pragma unroll
    for (int k = 0; k < 8; ++k) t.w[k] = corner_weight(c, (k >> 2) & 1, (k >> 1) & 1, k & 1);
    return t;
}

__device__ __forceinline__ int corner_off(const DevGrid &g, int c) {
    return ((c >> 2) & 1) * g.sx + ((c >> 1) & 1) * g.sy + (c & 1) * g.cs;
}

// Channels c0..c0+3 of a trilinear lookup (rows 16-byte aligned, c0 % 4 == 0): corners in the
// order 0..7, one FMA each, so every kernel that interpolates this way gets the same bits.
__device__ __forceinline__ float4 interp4(const DevGrid &g, const Tri &t, int c0) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const float4 v = *reinterpret_cast<const float4 *>(g.data + t.base + corner_off(g, c) + c0);
        acc.x = __builtin_fmaf(t.w[c], v.x, acc.x);
        acc.y = __builtin_fmaf(t.w[c], v.y, acc.y);
        acc.z = __builtin_fmaf(t.w[c], v.z, acc.z);
        acc.w = __builtin_fmaf(t.w[c], v.w, acc.w);
    }
    return acc;
}

__device__ __forceinline__ float interp_ch(const DevGrid &g, const Tri &t, int ch) {
    float acc = 0.f;
#pragma unroll
    for (int c = 0; c < 8; ++c) acc += t.w[c] * g.data[t.base + corner_off(g, c) + ch];
    return acc;
}

// ------------------------------------------------------------------------------ Adam

// The update of one element (section 3's fused Adam): every kernel that applies Adam uses these
// expressions, so they agree bit for bit on the same gradient.
struct AdamArgs {
    float *p, *g, *m, *v;
    int64_t n;
    float lr_t;          // lr / (1 - beta1^t)
    float inv_sqrt_bc2;  // 1 / sqrt(1 - beta2^t)
    float b1, b2, eps, lr;
    const int *step_dev;  // when set, t is read here and lr_t / inv_sqrt_bc2 are recomputed
    int skip, zero;
};

__device__ __forceinline__ void adam_bias(AdamArgs &a) {
    if (a.step_dev) {
        const int t = *a.step_dev;
        const double bc1 = 1.0 - pow((double)a.b1, t), bc2 = 1.0 - pow((double)a.b2, t);
        a.lr_t = (float)((double)a.lr / bc1);
        a.inv_sqrt_bc2 = (float)(1.0 / sqrt(bc2));
    }
}

// Each operation rounded as written (explicit FMAs, no contraction), so every kernel that inlines
// this gets the same bits whatever code surrounds it.
__device__ __forceinline__ void adam_one(const AdamArgs &a, float g, float &p, float &m, float &v) {
#pragma clang fp contract(off)
    m = __builtin_fmaf(a.b1, m, (1.f - a.b1) * g);
    v = __builtin_fmaf(a.b2, v, (1.f - a.b2) * (g * g));
    p = p - (a.lr_t * m) / __builtin_fmaf(sqrtf(v), a.inv_sqrt_bc2, a.eps);
}

typedef float nt_f4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 ld_nt(const float4 *p) {
    const nt_f4 v = __builtin_nontemporal_load(reinterpret_cast<const nt_f4 *>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st_nt(float4 *p, float4 a) {
    const nt_f4 v = {a.x, a.y, a.z, a.w};
    __builtin_nontemporal_store(v, reinterpret_cast<nt_f4 *>(p));
}


// ------------------------------------------------------------------------ wave runs

// Runs of equal keys among the lanes of a wave: the head of each run (key >= 0) learns the run
// length; every lane learns its run's head.
struct Run {
    bool head;
    int len, head_lane;
};

__device__ __forceinline__ Run wave_runs(int key) {
    const int ln = lane();
    const int prev = __shfl_up(key, 1, 64);
    const bool head = key >= 0 && (ln == 0 || prev != key);
    const bool start = ln == 0 || prev != key;  // a run boundary (invalid lanes start runs too)
    const unsigned long long starts = __ballot(start);
    const unsigned long long after = ln == 63 ? 0ull : starts & (~0ull << (ln + 1));
    const int next = after ? __ffsll((long long)after) - 1 : 64;
    const unsigned long long upto = starts & (ln == 63 ? ~0ull : ((2ull << ln) - 1));
    Run r;
    r.head = head;
    r.len = next - ln;
    r.head_lane = 63 - __clzll((long long)upto);
    return r;
}

// ------------------------------------------------------------------------- host side

int set_error(int code, const char *fmt, ...);
int check_hip(hipError_t e, const char *what);
int make_dev_grid(const dvgo_grid *g, const char *name, DevGrid *out, bool need_grad);

// Debug mode (dvgo_set_debug, or DVGO_DEBUG=1 in the environment): the entry points that take a
// ragged batch first check it on the device with validate_batch (synchronous).
bool debug_mode();
int validate_batch(int32_t n_rays, int64_t n_samples, const int32_t *ray_offsets, const float *s_mid, hipStream_t st);

// The distortion loss on given weights (render.hip): argument checks, the bytes of its per-chunk
// checkpoint scratch, and the launch with a caller-chosen scratch pointer.
int distortion_check(int32_t n_rays, const int32_t *ray_offsets, int64_t n_samples, const float *w, const float *s_mid,
                     const float *s_len, const float *loss, const float *grad_loss, const float *grad_w);
size_t distortion_scratch_bytes(int32_t n_rays, int64_t n_samples);
int launch_distortion(int32_t n_rays, const int32_t *ray_offsets, int64_t n_samples, const float *w, const float *s_mid,
                      const float *s_len, float *loss, const float *grad_loss, float *grad_w, void *ckpt,
                      hipStream_t st);

// Largest batch the per-sample kernels address: 3 * n_samples (the xyz and colour rows) stays
// below 2^31 in their int32 indices.
constexpr int64_t MAX_SAMPLES = ((int64_t)1 << 31) / 3 - 1;

// checkpoint slot of the chunk starting at sample c0 of ray r (rays own disjoint slot ranges)
__host__ __device__ __forceinline__ int64_t ckpt_slot(int64_t beg, int r, int64_t c0) {
    return beg / 64 + r + (c0 - beg) / 64;
}
__host__ __device__ __forceinline__ int64_t ckpt_count(int32_t n_rays, int64_t n_samples) {
    return n_samples / 64 + n_rays + 1;
}

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

}  // namespace dvgo

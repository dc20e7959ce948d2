// Colour MLP of the hybrid representation (Table 1): [features, view encoding] -> 128 ->
// 128 -> RGB, forward and backward on gfx950 FP16 matrix cores with FP32-grade products.
//
// Split precision.  Every matrix operand v is held as two FP16 parts scaled by a power of
// two, v 2^e = hi + lo with hi = fp16(v 2^e) and lo = fp16(v 2^e - hi), and a product is
// taken as hi*hi' + hi*lo' + lo*hi' (three FP16 matrix instructions into one FP32
// accumulator).  The dropped lo*lo' term and the rounding of lo leave a relative error near
// 2^-22 per product.  The power of two keeps operands inside the FP16 normal range: weight
// matrices use one exponent each (largest entry just under 2^14); an activation column (one
// sample) uses an exponent from a bound on its magnitude that every wave can evaluate on
// its own (infinity norms of the weights times the sample's input or upstream gradient).
// Accumulators are brought back to true scale with v_ldexp, which is exact.
//
// Layout.  The forward works on 32x32 accumulator tiles (see its section).  In the backward a 16x16
// accumulator tile holds 16 hidden units (rows) x 16 samples (columns); lane (q = lane/16, j = lane%16)
// owns rows 4q..4q+3 of column j.  A K-step of 32 reads the lane's 8 operand slots (q, e) as logical
// index k(kk, q, e) = 32 kk + 4 q + e (e < 4) or 32 kk + 16 + 4 q + (e - 4) (e >= 4), so two
// consecutive row tiles of one layer's output are the next layer's B operand without any data movement.
// Weight rows are stored with their columns in that slot order ("phys" order), so an A operand is one
// 16-byte read per part.
//
// Backward: a block's waves own slices of 32 hidden units for the block's 32-sample tiles and keep their
// rows of W1, W2 or W2^T in registers (two roles, see the backward section); activations are exchanged
// through sample-major LDS planes.  The weight gradients reduce over samples, so their unit-major
// operands are read from those planes with transposing LDS reads; their accumulators carry a
// power-of-two frame that only ever decreases (rescaled when a tile needs it), and a sample's operands
// are scaled so that the product lands in that frame.
#include <string.h>

#include "dvgo_internal.h"

using namespace dvgo;

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));

constexpr int H = 128;      // hidden width
constexpr int KX = 64;      // padded input width: features 0..11, view encoding 12..47, zeros 48..63
constexpr int PEW = 36;     // per-ray encoding row (input columns 12..47)
constexpr int RBW = H + 4;  // per-ray layer-1 bias row: H biases, their largest magnitude, padding
constexpr int RS1 = 72;     // row stride (halves) of a 64-wide operand row
constexpr int RS2 = 136;    // row stride (halves) of a 128-wide operand row
constexpr int MAXE = 100;   // clamp of scaling exponents
constexpr int FRAME_NONE = 1 << 20;
constexpr int MAX_BLOCKS = 256;

// ---- weight image (written by mlp_prep_kernel into the workspace) ----
// W2 comes first so that every W2 read of the forward kernel reaches its LDS copy with one
// base register and a 16-bit immediate offset.
constexpr int IMG_W2H = 0;
constexpr int IMG_W2L = IMG_W2H + H * RS2 * 2;
constexpr int IMG_W1H = IMG_W2L + H * RS2 * 2;   // start of the part the backward kernel stages
constexpr int IMG_W1L = IMG_W1H + H * RS1 * 2;
constexpr int IMG_B1 = IMG_W1L + H * RS1 * 2;
constexpr int IMG_B2 = IMG_B1 + H * 4;
constexpr int IMG_W3 = IMG_B2 + H * 4;
constexpr int IMG_B3 = IMG_W3 + 3 * H * 4;
constexpr int IMG_META = IMG_B3 + 16;
constexpr int IMG_FWD_END = IMG_META + 48;  // end of the forward kernel's LDS image
constexpr int IMG_W2TH = IMG_FWD_END;
constexpr int IMG_W2TL = IMG_W2TH + H * RS2 * 2;
constexpr int IMG_W1FH = IMG_W2TL + H * RS2 * 2;
constexpr int IMG_W1FL = IMG_W1FH + 16 * RS2 * 2;
constexpr int IMG_BYTES = IMG_W1FL + 16 * RS2 * 2;
static_assert(IMG_W1H % 16 == 0 && IMG_FWD_END % 16 == 0 && IMG_BYTES % 16 == 0, "image alignment");

struct Meta {
    int sw1, sw2;           // weight exponents of W1 and W2 (W2^T shares sw2, W1F shares sw1)
    float n1, b1max;        // max_i sum_k |W1[i][k]|, max |b1|
    float n2t, n3t;         // max_in sum_out |W2[out][in]|, max_h sum_o |W3[o][h]|
    float n1f;              // max_i sum over the feature columns k of |W1[i][k]|
    int pad[5];
};
static_assert(sizeof(Meta) == 48, "meta size");

__host__ __device__ constexpr int kidx(int kk, int q, int e) {
    return 32 * kk + (e < 4 ? 4 * q + e : 16 + 4 * q + (e - 4));
}

__device__ __forceinline__ v4f mfma16(h8 a, h8 b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// exponent e with |v| 2^e < 2^14 for every |v| <= m
__device__ __forceinline__ int scale_exp(float m) {
    int k;
    frexpf(m, &k);
    const int e = 14 - k;
    return e < -MAXE ? -MAXE : (e > MAXE ? MAXE : e);
}

// exponent k with m < 2^k (FRAME_NONE - style "no constraint" handled by callers for m == 0)
__device__ __forceinline__ int ceil_exp(float m) {
    int k;
    frexpf(m, &k);
    return k;
}

// hi and lo parts of two values in packed halves: hi = fp16(t0), fp16(t1) from one packed
// conversion (round to nearest even, as every float -> half conversion here), lo = fp16(t - hi)
// of each from one mixed-precision FMA that writes its half of the register directly (t - hi is
// exact in FP32, so each equals (_Float16)(t - (float)hi)).  The compiler's hazard tracking does
// not see these as vector-ALU writes, and a matrix instruction may read a vector register only two
// wait states after a vector-ALU instruction wrote it: with MM (the results feed a product
// directly) the block ends with those two (s_nop 1); results that only go to LDS stores need none.
template <bool MM>
__device__ __forceinline__ void split2(float t0, float t1, unsigned &hi, unsigned &lo) {
    if (MM)
        asm("v_cvt_pk_f16_f32 %0, %2, %3\n\t"
            "v_fma_mixlo_f16 %1, %2, 1.0, -%0 op_sel_hi:[0,0,1]\n\t"
            "v_fma_mixhi_f16 %1, %3, 1.0, -%0 op_sel:[0,0,1] op_sel_hi:[0,0,1]\n\t"
            "s_nop 1"
            : "=&v"(hi), "=&v"(lo)
            : "v"(t0), "v"(t1));
    else
        asm("v_cvt_pk_f16_f32 %0, %2, %3\n\t"
            "v_fma_mixlo_f16 %1, %2, 1.0, -%0 op_sel_hi:[0,0,1]\n\t"
            "v_fma_mixhi_f16 %1, %3, 1.0, -%0 op_sel:[0,0,1] op_sel_hi:[0,0,1]"
            : "=&v"(hi), "=&v"(lo)
            : "v"(t0), "v"(t1));
}

// MM: the parts feed a matrix product directly (see split2)
template <bool MM>
__device__ __forceinline__ void split4(const float v[4], float sc, h4 &hi, h4 &lo) {
    uint2 h, l;
    split2<MM>(v[0] * sc, v[1] * sc, h.x, l.x);
    split2<MM>(v[2] * sc, v[3] * sc, h.y, l.y);
    hi = __builtin_bit_cast(h4, h);
    lo = __builtin_bit_cast(h4, l);
}

__device__ __forceinline__ h8 cat(h4 a, h4 b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7); }

// logistic function with the hardware exponential and reciprocal (about 1e-7 relative; the
// limits are exact: 1/(1 + inf) = 0 and 1/(1 + 0) = 1)
__device__ __forceinline__ float fast_sigmoid(float z) { return __builtin_amdgcn_rcpf(1.f + __expf(-z)); }

// Reductions over aligned lane groups with DPP moves (no LDS round trip).  quad_perm [1,0,3,2]
// and [2,3,0,1] reduce each quad; row_half_mirror (lane i of an 8-lane half-row reads lane
// 7 - i) joins the two quads of a half-row; row_mirror (15 - i) joins the halves of a row.
template <int CTRL>
__device__ __forceinline__ int dpp_mov(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp_movf(float v) {
    return __builtin_bit_cast(float, dpp_mov<CTRL>(__builtin_bit_cast(int, v)));
}
// min over the 16 lanes of each row
__device__ __forceinline__ int row16_min(int v) {
    v = min(v, dpp_mov<0xB1>(v));
    v = min(v, dpp_mov<0x4E>(v));
    v = min(v, dpp_mov<0x141>(v));
    return min(v, dpp_mov<0x140>(v));
}
// max over each aligned group of 8 lanes
__device__ __forceinline__ float group8_max(float v) {
    v = fmaxf(v, dpp_movf<0xB1>(v));
    v = fmaxf(v, dpp_movf<0x4E>(v));
    return fmaxf(v, dpp_movf<0x141>(v));
}

// the lower half-wave's values of a and b in the first result, the upper half-wave's in the second, each
// a's then b's; and the same with the even and odd rows of 16 lanes
struct Pair {
    float a, b;
};
__device__ __forceinline__ Pair swap32(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b),
                                                    false, false);
    const unsigned x = r[0], y = r[1];
    return {__builtin_bit_cast(float, x), __builtin_bit_cast(float, y)};
}
__device__ __forceinline__ Pair swap16(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b),
                                                    false, false);
    const unsigned x = r[0], y = r[1];
    return {__builtin_bit_cast(float, x), __builtin_bit_cast(float, y)};
}

__device__ __forceinline__ float pow2(int e) { return __builtin_amdgcn_ldexpf(1.f, e); }
__device__ __forceinline__ float ldx(float v, int e) { return __builtin_amdgcn_ldexpf(v, e); }

struct MlpArgs {
    const float *W1, *b1, *W2, *b2, *W3, *b3;
    int in_feat, n_in;  // n_in = in_feat + 3 + 6 F (columns of W1)
    int n_freq;
    int n_rays;
    const int *offs;
    const float *dirs;
    int S;
    const float *feat;
    int feat_vec;        // in_feat == 12 and feat 16-byte aligned: rows load as float4
    float *rgb;
    unsigned char *img;  // weight image (workspace)
    float *pe;           // [R][PEW] view encodings (workspace)
    float *rb;           // [R][RBW] layer-1 biases of the rays, b1 + W1 (view encoding), and their largest magnitude;
                         // NULL where the batch has none (ray_rows)
    int *tile_ray;       // [ceil(S/32)] ray of the first sample of each 32-sample tile (workspace)
    int n_tiles;         // ceil(S/32)
    const float *grad_rgb;
    float *grad_feat;
    float *partial;  // [blocks][n_params] (workspace)
    int n_params;
    float *gW1, *gb1, *gW2, *gb2, *gW3, *gb3;
    int nblocks;
    // fused feature gather: the feature grid the forward looks the features up in, and the
    // sample points
    DevGrid fg;
    const float *xyz;
    float *feat_out;  // forward with the gather: the features it used, [S][in_feat] (may be NULL)
};

// padded input column k -> column of W1 (or -1 for padding)
__host__ __device__ __forceinline__ int w1_col(int in_feat, int n_freq, int k) {
    if (k < 12) return k < in_feat ? k : -1;
    const int p = k - 12;
    return p < 3 + 6 * n_freq ? in_feat + p : -1;
}

// ------------------------------------------------------------------ preparation

constexpr int TILE = 32;   // samples per wave tile (forward) and per block tile (backward)

// ray of sample s: the last r with offs[r] <= s (rays may be empty)
__device__ __forceinline__ int find_ray(const int *offs, int R, int s) {
    int lo = 0, hi = R - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (offs[mid] <= s) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// The ray of each of the 8 consecutive samples sbase + (lane >> 3) of a wave (sbase wave-uniform and
// at or after offs[r0]), where lane l holds w = offs[min(r0 + l, R)]: per sample, a ballot counts the window entries at or before it
// (a prefix, as offs is non-decreasing), so no lane-to-lane round trips are needed.  All 64
// lanes must call it.
__device__ __forceinline__ int ray_of_group8(const int *offs, int R, int r0, int w, int sbase) {
    const int k = lane() >> 3;
    int cnt = __popcll(__ballot(w <= sbase));
    if (cnt != __popcll(__ballot(w <= sbase + 7))) {  // not all on one ray
#pragma unroll
        for (int i = 1; i < 8; ++i) {
            const int c = __popcll(__ballot(w <= sbase + i));
            cnt = k >= i ? c : cnt;
        }
    }
    const int s = sbase + k;
    if (cnt == 64 && r0 + 64 <= R && offs[r0 + 64] <= s) return find_ray(offs, R, s);
    return r0 + cnt - 1;
}

__device__ __forceinline__ int window_entry(const int *offs, int R, int r0) {
    const int i = r0 + lane();
    return offs[i < R ? i : R];
}

__device__ float block_max(float v, float *red) {
    // blockDim.x is a multiple of 64 and at most 1024
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    __syncthreads();
    if (lane() == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float m = 0.f;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) m = fmaxf(m, red[i]);
    return m;
}

__device__ __forceinline__ void put_split(unsigned char *img, int off_h, int off_l, int idx, float v, float sc) {
    const float t = v * sc;
    const _Float16 h = (_Float16)t;
    reinterpret_cast<_Float16 *>(img + off_h)[idx] = h;
    reinterpret_cast<_Float16 *>(img + off_l)[idx] = (_Float16)(t - (float)h);
}

// logical index of phys slot p of a 128- or 64-wide operand row
__device__ __forceinline__ int phys_to_k(int p) { return kidx(p >> 5, (p >> 3) & 3, p & 7); }

constexpr int PREP_THREADS = 512;
constexpr int PREP_W2_BLOCKS = 16;  // 8 rows of W2 and of W2^T each
constexpr int PREP_W1_BLOCKS = 4;   // 32 rows of W1 each (block 0 of them also W1F, b1, b3)
constexpr int PREP_FIXED_BLOCKS = PREP_W2_BLOCKS + PREP_W1_BLOCKS + 1;

// blocks [0, 16): W2 and W2^T planes; every one of them also reduces max|W2| and the column
// sums of |W2| from the same loads (block 0 stores sw2 and n2t).  Blocks [16, 20): W1 planes,
// max|W1| and the row sums of |W1| (block 16 stores sw1, n1, b1max and writes W1F, b1, b3).
// Block 20: W3, b2, n3t.  Then the rays and the tile start rays.  Where the batch has bias rows (ray_rows) a
// block takes PREP_RAYS rays: view encodings, one entry per thread, and the layer-1 biases that follow from
// them, one unit per thread; otherwise PREP_THREADS entries of the encodings, one per thread.
constexpr int PREP_RAYS = 16;

// blocks of the preparation that serve the rays
__host__ __device__ __forceinline__ int ray_blocks(const MlpArgs &a) {
    return a.rb ? (a.n_rays + PREP_RAYS - 1) / PREP_RAYS
                : (int)(((int64_t)a.n_rays * PEW + PREP_THREADS - 1) / PREP_THREADS);
}

// entry e of the view encoding of ray r (0 past its 3 + 6 F entries)
__device__ __forceinline__ float encoding(const MlpArgs &a, int r, int e) {
    const int F = a.n_freq;
    if (e >= 3 + 6 * F) return 0.f;
    const int q = e < 3 ? e : (e - 3) % (3 * F), ax = e < 3 ? e : q % 3;
    const float d = a.dirs[3 * (int64_t)r + ax];
    const float t = ldexpf(d, e < 3 ? 0 : q / 3);
    return e < 3 ? d : (e < 3 + 3 * F ? sinf(t) : cosf(t));
}

__global__ __launch_bounds__(PREP_THREADS) void mlp_prep_kernel(MlpArgs a) {
    __shared__ float red[PREP_THREADS / 64];
    __shared__ float sums[PREP_THREADS];
    __shared__ float enc[PREP_RAYS][PEW];
    __shared__ float w1[H * 39];  // the ray blocks' copy of W1 (at most 39 columns)
    unsigned char *img = a.img;
    Meta *meta = reinterpret_cast<Meta *>(img + IMG_META);
    const int tid = threadIdx.x, b = blockIdx.x;
    const int pe_blocks = ray_blocks(a);
    if (b < PREP_W2_BLOCKS) {
        // element i = tid + 512 k sits in column tid % 128 (512 is a multiple of H)
        float m = 0.f, cs = 0.f;
#pragma unroll
        for (int i = 0; i < H * H / PREP_THREADS; ++i) {  // all the loads in flight at once
            const float v = fabsf(a.W2[tid + i * PREP_THREADS]);
            m = fmaxf(m, v);
            cs += v;
        }
        sums[tid] = cs;
        const int sw = scale_exp(block_max(m, red));  // its barriers also order the sums
        float n2t = 0.f;
        if (b == 0) {
            const float col = tid < H ? sums[tid] + sums[tid + H] + sums[tid + 2 * H] + sums[tid + 3 * H] : 0.f;
            n2t = block_max(col, red);
        }
        const float sc = pow2(sw);
        for (int i = tid; i < 8 * RS2; i += PREP_THREADS) {
            const int row = 8 * b + i / RS2, p = i % RS2;
            const int k = p < H ? phys_to_k(p) : -1;
            put_split(img, IMG_W2H, IMG_W2L, row * RS2 + p, k >= 0 ? a.W2[row * H + k] : 0.f, sc);
            put_split(img, IMG_W2TH, IMG_W2TL, row * RS2 + p, k >= 0 ? a.W2[k * H + row] : 0.f, sc);
        }
        if (b == 0 && tid == 0) {
            meta->sw2 = sw;
            meta->n2t = n2t;
        }
    } else if (b < PREP_W2_BLOCKS + PREP_W1_BLOCKS) {
        const int wb = b - PREP_W2_BLOCKS;
        // four threads per row, every fourth column each: the row sums of |W1| over all columns and over the
        // feature columns
        float m = 0.f, all = 0.f, fs = 0.f;
        const int row = tid >> 2;
#pragma unroll
        for (int i = 0; i < 10; ++i) {  // at most 39 columns
            const int c = (tid & 3) + 4 * i;
            const float v = c < a.n_in ? fabsf(a.W1[row * a.n_in + c]) : 0.f;
            m = fmaxf(m, v);
            all += v;
            fs += c < a.in_feat ? v : 0.f;
        }
        all += __shfl_xor(all, 1, 64);
        fs += __shfl_xor(fs, 1, 64);
        all += __shfl_xor(all, 2, 64);
        fs += __shfl_xor(fs, 2, 64);
        const int sw = scale_exp(block_max(m, red));
        const float sc = pow2(sw);
        for (int i = tid; i < 32 * RS1; i += PREP_THREADS) {
            const int row = 32 * wb + i / RS1, p = i % RS1;
            const int c = p < KX ? w1_col(a.in_feat, a.n_freq, phys_to_k(p)) : -1;
            put_split(img, IMG_W1H, IMG_W1L, row * RS1 + p, c >= 0 ? a.W1[row * a.n_in + c] : 0.f, sc);
        }
        if (wb == 0) {
            const float n1 = block_max(all, red), n1f = block_max(fs, red);
            const float b1max = block_max(tid < H ? fabsf(a.b1[tid]) : 0.f, red);
            // W1F[c][phys over hidden] = W1[hidden][c] for the feature columns c < in_feat
            for (int i = tid; i < 16 * RS2; i += PREP_THREADS) {
                const int c = i / RS2, p = i % RS2;
                const int h = p < H ? phys_to_k(p) : -1;
                put_split(img, IMG_W1FH, IMG_W1FL, i, (h >= 0 && c < a.in_feat) ? a.W1[h * a.n_in + c] : 0.f, sc);
            }
            float *b1 = reinterpret_cast<float *>(img + IMG_B1);
            float *b3 = reinterpret_cast<float *>(img + IMG_B3);
            if (tid < H) b1[tid] = a.b1[tid];
            if (tid < 4) b3[tid] = tid < 3 ? a.b3[tid] : 0.f;
            if (tid == 0) {
                meta->sw1 = sw;
                meta->n1 = n1;
                meta->n1f = n1f;
                meta->b1max = b1max;
            }
        }
    } else if (b == PREP_FIXED_BLOCKS - 1) {
        float *w3 = reinterpret_cast<float *>(img + IMG_W3);
        float *b2 = reinterpret_cast<float *>(img + IMG_B2);
        float cs = 0.f;
        for (int i = tid; i < 3 * H; i += PREP_THREADS) w3[i] = a.W3[i];
        if (tid < H) {
            b2[tid] = a.b2[tid];
            cs = fabsf(a.W3[tid]) + fabsf(a.W3[H + tid]) + fabsf(a.W3[2 * H + tid]);
        }
        const float n3t = block_max(cs, red);
        if (tid == 0) meta->n3t = n3t;
    } else if (b >= PREP_FIXED_BLOCKS + pe_blocks) {
        const int t = (b - PREP_FIXED_BLOCKS - pe_blocks) * PREP_THREADS + tid;
        if (t < a.n_tiles) a.tile_ray[t] = find_ray(a.offs, a.n_rays, TILE * t);
    } else if (!a.rb) {
        const int64_t i = (int64_t)(b - PREP_FIXED_BLOCKS) * PREP_THREADS + tid;
        const int r = (int)(i / PEW);
        if (r < a.n_rays) a.pe[i] = encoding(a, r, (int)(i - (int64_t)r * PEW));
    } else {
        const int r0 = (b - PREP_FIXED_BLOCKS) * PREP_RAYS, nr = min(PREP_RAYS, a.n_rays - r0);
        float wl[10];  // W1, read with coalesced loads before the encodings are formed
#pragma unroll
        for (int i = 0; i < 10; ++i) {
            const int k = tid + i * PREP_THREADS;
            wl[i] = k < H * a.n_in ? a.W1[k] : 0.f;
        }
        for (int i = tid; i < PREP_RAYS * PEW; i += PREP_THREADS) {
            const int r = i / PEW, e = i - r * PEW;
            const float v = r < nr ? encoding(a, r0 + r, e) : 0.f;
            enc[r][e] = v;
            if (r < nr) a.pe[(int64_t)r0 * PEW + i] = v;
        }
#pragma unroll
        for (int i = 0; i < 10; ++i)
            if (tid + i * PREP_THREADS < H * 39) w1[tid + i * PREP_THREADS] = wl[i];
        __syncthreads();
        const int u = tid & (H - 1), NE = 3 + 6 * a.n_freq;
        const float *w = w1 + u * a.n_in + a.in_feat;
        const float bu = a.b1[u];
        float acc[PREP_RAYS * H / PREP_THREADS];
#pragma unroll
        for (int i = 0; i < PREP_RAYS * H / PREP_THREADS; ++i) acc[i] = bu;
        for (int e = 0; e < NE; ++e) {
            const float we = w[e];
#pragma unroll
            for (int i = 0; i < PREP_RAYS * H / PREP_THREADS; ++i)
                acc[i] = fmaf(we, enc[i * (PREP_THREADS / H) + tid / H][e], acc[i]);
        }
#pragma unroll
        for (int i = 0; i < PREP_RAYS * H / PREP_THREADS; ++i) {
            const int r = i * (PREP_THREADS / H) + tid / H;
            float m = fabsf(acc[i]);  // largest magnitude over the wave's 64 units, then over the ray's two waves
            for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
            __syncthreads();
            if (lane() == 0) red[tid >> 6] = m;
            __syncthreads();
            if (r < nr) {
                float *row = a.rb + (int64_t)(r0 + r) * RBW;
                row[u] = acc[i];
                if (u == 0) row[H] = fmaxf(red[tid >> 6], red[(tid >> 6) + 1]);
            }
        }
    }
}

// Pointer into a kernel's LDS block at byte offset `off`, with the offset hidden from the
// optimiser: accesses then share one base register and use the 16-bit immediate offset of
// ds_read/ds_write instead of one materialised address per constant offset above 64 KB.
__device__ __forceinline__ unsigned char *lds_region(unsigned char *sm, int off) {
    asm volatile("" : "+s"(off));
    return sm + off;
}

// A lane index the optimiser must treat as new in every loop iteration, so that address
// arithmetic built from it is recomputed next to its use (and folded into instruction
// offsets) instead of being hoisted out of the loop into long-lived registers.
__device__ __forceinline__ int fresh(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

__device__ __forceinline__ float4 feat4(const MlpArgs &a, int s, int c0) {
    const float *fp = a.feat + (int64_t)s * a.in_feat;
    if (a.feat_vec) return *reinterpret_cast<const float4 *>(fp + c0);
    return make_float4(c0 < a.in_feat ? fp[c0] : 0.f, c0 + 1 < a.in_feat ? fp[c0 + 1] : 0.f,
                       c0 + 2 < a.in_feat ? fp[c0 + 2] : 0.f, c0 + 3 < a.in_feat ? fp[c0 + 3] : 0.f);
}

// The 8 inputs of operand slot group (kk, q) of a valid sample s on ray `ray`, features read
// from a.feat: logical columns k(kk, q, 0..7).  For kk = 0 these are features 4q..4q+3 (view
// encoding 0..3 when q = 3) and view encoding 4+4q..7+4q; for kk = 1 view encoding 20+4q..23+4q
// and padding.  (The kernels use it only for feature rows that cannot be read as float4.)
__device__ __forceinline__ void load_x8(const MlpArgs &a, int s, int ray, int kk, int q, float v[8]) {
    const float *pe = a.pe + (int64_t)ray * PEW;
    float4 lo, hi;
    if (kk == 0) {
        lo = q < 3 ? feat4(a, s, 4 * q) : *reinterpret_cast<const float4 *>(pe);
        hi = *reinterpret_cast<const float4 *>(pe + 4 + 4 * q);
    } else {
        lo = *reinterpret_cast<const float4 *>(pe + 20 + 4 * q);
        hi = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    v[0] = lo.x; v[1] = lo.y; v[2] = lo.z; v[3] = lo.w;
    v[4] = hi.x; v[5] = hi.y; v[6] = hi.z; v[7] = hi.w;
}

__device__ __forceinline__ void copy_to_lds(unsigned char *dst, const unsigned char *src, int bytes) {
    for (int i = threadIdx.x * 16; i < bytes; i += blockDim.x * 16)
        *reinterpret_cast<uint4 *>(dst + i) = *reinterpret_cast<const uint4 *>(src + i);
}

// ------------------------------------------------------------------ forward
//
// Wave tiles of 32 samples x 128 units on v_mfma_f32_32x32x16_f16: lane (hf = lane / 32, j = lane % 32)
// of a 32 x 32 accumulator tile owns units 8 i + 4 hf + r (i, r < 4) of sample j, and a K-step of 16
// reads the lane's 8 operand slots (hf, e) as logical index 16 ks + 8 (e / 4) + 4 hf + e % 4, so a row
// tile of one layer's output is two K-steps of the next layer's B operand without any data movement.  W1
// and W2 sit in LDS (both parts), their columns in that slot order; three waves per SIMD (12 per block,
// at most 168 registers).  With ROWS (split mode, batches that have bias rows) layer 1 multiplies the features
// only (one K-step): the view encoding is the same for all samples of a ray, and its part of layer 1 is the
// ray's bias row, made once per ray by the preparation.  Otherwise the encoding stays in the product, K = 48.
// (So it does in the FP16 mode: its operands are rounded, and so is its encoding.)
//
// Bound by the matrix and vector units together, which overlap by about half on this chip (measured: eight
// 32 x 32 x 16 products and 56 FMAs of two waves take 188 ns where the products alone take 145 and the FMAs
// 82), and by the clock, which falls to 1.8-1.9 GHz under them; with the lookup inside also by its loads.
// 981,900 samples without the lookup 136 -> 104 us against 16 x 16 x 32 tiles of 16 samples: the larger tiles (half
// the weight reads and matrix instructions, K = 48 instead of 64) and the ray search by ray starts (instead of six
// dependent lane shuffles) gave 136 -> 117, the rays' bias rows 117 -> 104.  3,926,000 along rays with the lookup
// 550 -> 458.
constexpr int FRS2 = 136;  // halves per W2 row in the forward's LDS (128 used)
constexpr int FWD_WAVES = 12, FWD_THREADS = 64 * FWD_WAVES;

// LDS row strides: a 16-byte read of 32 rows at one column runs without bank conflicts when the stride is
// an odd multiple of 16 bytes.
template <bool SPLIT, bool ROWS>
struct FwdLds {
    static constexpr int K1 = ROWS ? 1 : 3;          // K-steps of layer 1
    static constexpr int RS1 = ROWS ? 24 : 56;       // halves per W1 row
    static constexpr int W2H = 0, W2L = W2H + H * FRS2 * 2, W1H = W2L + (SPLIT ? H * FRS2 * 2 : 0),
                         W1L = W1H + H * RS1 * 2,
                         SMALL = W1L + (SPLIT ? H * RS1 * 2 : 0),  // b1, b2, W3, b3, meta, laid out as in the image
                         END = SMALL + (IMG_FWD_END - IMG_B1);
    static_assert((FRS2 * 2) % 32 == 16 && (RS1 * 2) % 32 == 16 && SMALL % 16 == 0 && END <= 160 * 1024, "strides");
};

typedef float v16f __attribute__((ext_vector_type(16)));

__device__ __forceinline__ v16f mfma32(h8 a, h8 b, v16f c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// Copies the first 4 * GROUPS columns of the image's weight rows (stride sstride bytes) to LDS, from the
// image's slot order to the forward's: both keep groups of four consecutive columns together, column
// group u (columns 4 u ..) at group 8 (u / 8) + 2 (u % 4) + (u / 4) % 2 there and at 4 (u / 4) + 2 (u % 2)
// + (u / 2) % 2 here.
template <int GROUPS>
__device__ __forceinline__ void copy_rows_to_lds(unsigned char *dst, int dstride, const unsigned char *src,
                                                 int sstride) {
    for (int i = threadIdx.x; i < H * GROUPS; i += FWD_THREADS) {
        const int r = i / GROUPS, u = i - r * GROUPS;
        const int from = 8 * (u >> 3) + 2 * (u & 3) + ((u >> 2) & 1), to = 4 * (u >> 2) + 2 * (u & 1) + ((u >> 1) & 1);
        *reinterpret_cast<uint2 *>(dst + r * dstride + 8 * to) =
            *reinterpret_cast<const uint2 *>(src + r * sstride + 8 * from);
    }
}

// the value of the lane of the other half of the wave (lane l of lane l + 32 and the other way round)
__device__ __forceinline__ float other_half(float v) { return __shfl_xor(v, 32, 64); }

// The ray of sample s of the 32-sample tile whose first sample lies on ray r0, where lane l holds w =
// offs[min(r0 + l, R)]: only rays with samples matter, and those that start inside the tile are mostly few, so
// they are taken one by one (wave-uniform); more than 8 by a binary search over the window, six dependent lane
// shuffles.  All 64 lanes must call it.
__device__ __forceinline__ int ray_in_tile(const int *offs, int R, int r0, int w, int tile0, int s) {
    const int after = __shfl_down(w, 1, 64);
    const bool starts = lane() < 63 && w > tile0 && w < tile0 + TILE && after > w;
    int ray = r0;
    unsigned long long b = __ballot(starts);
    if (__popcll(b) > 8) {
        int at = 0;  // the last window entry at or before s
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) {
            const int v = __shfl(w, at + d, 64);
            if (v <= s) at += d;
        }
        ray = r0 + at;
        b = 0;
    }
    for (; b; b &= b - 1) {
        const int l = __ffsll((long long)b) - 1;
        if (s >= __builtin_amdgcn_readlane(w, l)) ray = r0 + l;
    }
    // the window's last entry: a ray whose end is not in it, or a later one
    if (s >= __builtin_amdgcn_readlane(w, 63)) ray = find_ray(offs, R, s);
    return ray;
}

// Channels c0 .. c0 + 3 and c1 .. c1 + 3 of a lookup, the bits of interp4 for each.  A corner's two loads
// follow each other: they mostly touch the same line, which the L1 does not keep until a second pass of eight
// loads where neighbouring samples share no cells, as on rays of few samples: 300,000 samples, 6 a ray, split
// 61 us in two passes, 57 this way, FP16 54 and 49.  Where they do share them the L1 keeps the lines, and the
// upper half-wave's loads of the second part are for nothing: batches with bias rows (ray_rows) take two passes
// (3,926,000 samples split 571 us, 575 this way, FP16 343 and 348; a training iteration on 981,504 1150 and 1158).
__device__ __forceinline__ void interp4_pair(const DevGrid &g, const Tri &t, int c0, int c1, float4 &a, float4 &b) {
    const auto fma4 = [](float4 &acc, float w, const float4 &v) {
        acc.x = __builtin_fmaf(w, v.x, acc.x);
        acc.y = __builtin_fmaf(w, v.y, acc.y);
        acc.z = __builtin_fmaf(w, v.z, acc.z);
        acc.w = __builtin_fmaf(w, v.w, acc.w);
    };
    a = b = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const float *p = g.data + t.base + corner_off(g, c);
        const float4 u = *reinterpret_cast<const float4 *>(p + c0), v = *reinterpret_cast<const float4 *>(p + c1);
        fma4(a, t.w[c], u);
        fma4(b, t.w[c], v);
    }
}

template <bool SPLIT, int GM, bool ROWS>
__global__ __launch_bounds__(FWD_THREADS) void mlp_fwd_kernel(MlpArgs a) {
    static_assert(SPLIT || !ROWS, "the FP16 mode rounds the encoding");
    using L = FwdLds<SPLIT, ROWS>;
    constexpr int K1 = L::K1, FRS1 = L::RS1;
    __shared__ __attribute__((aligned(16))) unsigned char sm[L::END];
    copy_rows_to_lds<32>(sm + L::W2H, FRS2 * 2, a.img + IMG_W2H, RS2 * 2);
    copy_rows_to_lds<4 * K1>(sm + L::W1H, FRS1 * 2, a.img + IMG_W1H, RS1 * 2);
    if (SPLIT) {
        copy_rows_to_lds<32>(sm + L::W2L, FRS2 * 2, a.img + IMG_W2L, RS2 * 2);
        copy_rows_to_lds<4 * K1>(sm + L::W1L, FRS1 * 2, a.img + IMG_W1L, RS1 * 2);
    }
    copy_to_lds(sm + L::SMALL, a.img + IMG_B1, IMG_FWD_END - IMG_B1);
    __syncthreads();
    const int ln = lane(), j = ln & 31, hf = ln >> 5;
    const _Float16 *W2 = reinterpret_cast<const _Float16 *>(sm) + j * FRS2 + 8 * hf;
    const unsigned char *r1 = lds_region(sm, L::W1H);
    const _Float16 *W1 = reinterpret_cast<const _Float16 *>(r1) + j * FRS1 + 8 * hf;
    constexpr int LO2 = (L::W2L - L::W2H) / 2, LO1 = (L::W1L - L::W1H) / 2;  // hi -> lo part, in halves
    const unsigned char *rs = r1 + (L::SMALL - L::W1H);
    const float *b1 = reinterpret_cast<const float *>(rs) + 4 * hf;
    const float *b2 = reinterpret_cast<const float *>(rs + (IMG_B2 - IMG_B1)) + 4 * hf;
    const float *W3 = reinterpret_cast<const float *>(rs + (IMG_W3 - IMG_B1)) + 4 * hf;
    const float *b3 = reinterpret_cast<const float *>(rs + (IMG_B3 - IMG_B1));
    const Meta meta = *reinterpret_cast<const Meta *>(rs + (IMG_META - IMG_B1));
    const int nwt = a.n_tiles;
    // neighbouring tiles go to neighbouring blocks: a small batch spreads over the CUs
    const int wt0 = blockIdx.x + (int)gridDim.x * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wstep = gridDim.x * FWD_WAVES;
    if (wt0 >= nwt) return;
    // First ray of a tile (past the last tile, the last tile's ray), read through the scalar cache: the
    // index is wave-uniform and the table is read-only here.
    const __attribute__((address_space(4))) int *tray = (const __attribute__((address_space(4))) int *)a.tile_ray;
    auto first_ray = [&](int wt) { return tray[wt < nwt ? wt : nwt - 1]; };
    // The ray window entry and the sample points of the next tile are loaded one tile ahead, so their
    // latency runs behind the products of the tile before.  The output of a tile is stored at the head of
    // the next one (after that tile's wait for its prefetched values), so that the wait does not include
    // the store.
    int r0 = first_ray(wt0);
    int win = window_entry(a.offs, a.n_rays, r0);
    int r0n = first_ray(wt0 + wstep);
    float pt[3] = {0.f, 0.f, 0.f};
    auto points = [&](int wt) {  // the point of this lane's sample (the last sample's past the end)
        const int sp = min(wt * TILE + j, a.S - 1);
#pragma unroll
        for (int d = 0; d < 3; ++d) pt[d] = a.xyz[3 * (int64_t)sp + d];
    };
    if (GM) points(wt0);
    float zout = 0.f, zout2 = 0.f;
    int sout = -1;
    auto store_out = [&]() {  // colours 0 and 2 from the lower half of the wave, 1 from the upper
        if (sout >= 0) {
            a.rgb[(int64_t)sout * 3 + hf] = zout;
            if (hf == 0) a.rgb[(int64_t)sout * 3 + 2] = zout2;
        }
    };
    const float4 none = make_float4(0.f, 0.f, 0.f, 0.f);
    const bool f0 = 4 * hf < a.in_feat, f1 = hf == 0 && 8 < a.in_feat;
    for (int wt = wt0; wt < nwt; wt += wstep) {
        const int s = wt * TILE + j;
        const bool sv = s < a.S;
        const int sc = sv ? s : a.S - 1;
        const int ray = min(ray_in_tile(a.offs, a.n_rays, r0, win, wt * TILE, s), a.n_rays - 1);
        // This lane's inputs, slot groups (ks, i) = columns 16 ks + 8 i + 4 hf ..: features 4 hf .. and
        // (hf = 0) 8 .. 11, view encoding 0..3 (hf = 1), then encoding 4 + 4 hf, 12 + 4 hf, 20 + 4 hf,
        // 28 + 4 hf.  ROWS: the ray's bias row instead of the encoding.
        float4 in[2 * K1], rb[ROWS ? 16 : 1];
        float rbmax = 0.f;
        const float *pe = a.pe + (int64_t)ray * PEW + 4 * hf;
        auto bias_row = [&]() {
            const float *row = a.rb + (int64_t)ray * RBW;
            rbmax = row[H];
#pragma unroll
            for (int i = 0; i < 16; ++i) rb[ROWS ? i : 0] = *reinterpret_cast<const float4 *>(row + 8 * i + 4 * hf);
        };
        if (ROWS && !GM) bias_row();
        if (!ROWS) {
#pragma unroll
            for (int i = 2; i < 2 * K1; ++i) in[i] = *reinterpret_cast<const float4 *>(pe + 8 * i - 12);
        }
        store_out();  // the previous tile's output
        if (GM) {
            const Tri t = trilinear<GM == 2>(a.fg, pt[0], pt[1], pt[2]);
            if ((SPLIT ? !ROWS : !a.rb) && a.in_feat > 8) {
                interp4_pair(a.fg, t, 4 * hf, 8, in[0], in[1]);
            } else {
                in[0] = interp4(a.fg, t, f0 ? 4 * hf : 0);
                in[1] = none;
                if (hf == 0) in[1] = interp4(a.fg, t, f1 ? 8 : 0);
            }
            if (a.feat_out && sv) {
                float *fo = a.feat_out + (int64_t)s * a.in_feat;
                if (f0) *reinterpret_cast<float4 *>(fo + 4 * hf) = in[0];
                if (f1) *reinterpret_cast<float4 *>(fo + 8) = in[1];
            }
            if (ROWS) {  // after the corner rows: both at once do not fit the registers
                __builtin_amdgcn_sched_barrier(0);
                bias_row();
            }
            points(wt + wstep);
        } else if (a.feat_vec) {
            const float *fp = a.feat + (int64_t)sc * 12;
            in[0] = *reinterpret_cast<const float4 *>(fp + 4 * hf);
            in[1] = *reinterpret_cast<const float4 *>(fp + 8);
        } else {
            in[0] = f0 ? feat4(a, sc, 4 * hf) : none;
            in[1] = f1 ? feat4(a, sc, 8) : none;
        }
        if (!f0) in[0] = none;
        if (!f1) in[1] = none;
        if (!ROWS && hf) in[1] = *reinterpret_cast<const float4 *>(pe - 4);
        // the next tile's first ray and window entry (the scalar load of the one after goes ahead)
        r0 = r0n;
        r0n = first_ray(wt + 2 * wstep);
        win = window_entry(a.offs, a.n_rays, r0);
        h8 xh[K1], xl[K1];
        float un1, sc1, un2;
        {
            float m = 0.f;
#pragma unroll
            for (int g = 0; g < 2 * K1; ++g) {
                if (!sv) in[g] = none;
                m = fmaxf(m, fmaxf(fmaxf(fabsf(in[g].x), fabsf(in[g].y)), fmaxf(fabsf(in[g].z), fabsf(in[g].w))));
            }
            m = fmaxf(m, other_half(m));
            const int ex = scale_exp(m), e1 = scale_exp(ROWS ? meta.n1f * m + rbmax : meta.n1 * m + meta.b1max);
            const float sx = pow2(ex);
#pragma unroll
            for (int ks = 0; ks < K1; ++ks) {
                h4 h0, l0, h1, l1;
                const float v0[4] = {in[2 * ks].x, in[2 * ks].y, in[2 * ks].z, in[2 * ks].w};
                const float v1[4] = {in[2 * ks + 1].x, in[2 * ks + 1].y, in[2 * ks + 1].z, in[2 * ks + 1].w};
                split4<true>(v0, sx, h0, l0);
                split4<true>(v1, sx, h1, l1);
                xh[ks] = cat(h0, h1);
                xl[ks] = cat(l0, l1);
            }
            un1 = pow2(-(meta.sw1 + ex));
            sc1 = pow2(e1);
            un2 = pow2(-(meta.sw2 + e1));
        }
        // Eight stages, one row tile each: 0..3 layer 1 (K1 K-steps), 4..7 layer 2 (8).  The products of a
        // stage run with the vector work that ends the stage before it (bias, ReLU, split; or bias, ReLU
        // and the output layer), in four pieces of four units, so that a wave keeps both units busy.  The
        // weight operands of the K-steps come from LDS one step ahead (two register sets).  Each K-step is fenced for the scheduler, which otherwise puts every read right before its
        // products and the vector work after them.
        constexpr int G1 = 4 * K1, G = G1 + 32;
        h8 wh[2], wl[2];
        auto fetch = [&](int g) {
            const int m = g < G1 ? g / K1 : (g - G1) / 8, ks = g < G1 ? g % K1 : (g - G1) % 8;
            const _Float16 *w = g < G1 ? W1 + 32 * m * FRS1 + 16 * ks : W2 + 32 * m * FRS2 + 16 * ks;
            wh[g % 2] = *reinterpret_cast<const h8 *>(w);
            if (SPLIT) wl[g % 2] = *reinterpret_cast<const h8 *>(w + (g < G1 ? LO1 : LO2));
        };
        v16f acc[2];
        auto products = [&](int g, h8 bh, h8 bl, v16f &c) {
            if (g + 1 < G) fetch(g + 1);
            if (SPLIT) {
                c = mfma32(wl[g % 2], bh, c);
                c = mfma32(wh[g % 2], bl, c);
            }
            c = mfma32(wh[g % 2], bh, c);
        };
        // piece i of the end of layer 1's row tile m: half i % 2 of h1's K-step 2 m + i / 2
        h4 hh[16], hl[16];
        auto end1 = [&](int m, int i, const v16f &c) {
            const float4 bb = ROWS ? rb[ROWS ? 4 * m + i : 0] : *reinterpret_cast<const float4 *>(b1 + 32 * m + 8 * i);
            const int r = 4 * i;
            const float v[4] = {fmaxf(fmaf(c[r], un1, bb.x), 0.f), fmaxf(fmaf(c[r + 1], un1, bb.y), 0.f),
                                fmaxf(fmaf(c[r + 2], un1, bb.z), 0.f), fmaxf(fmaf(c[r + 3], un1, bb.w), 0.f)};
            split4<true>(v, sc1, hh[4 * m + i], hl[4 * m + i]);
        };
        // piece i of the end of layer 2's row tile m: z3 += W3 relu(W2 h1 + b2), output rows on VALU
        float z[3] = {0.f, 0.f, 0.f};
        auto end2 = [&](int m, int i, const v16f &c) {
            const int u = 32 * m + 8 * i;
            const float4 bb = *reinterpret_cast<const float4 *>(b2 + u);
            const float4 w0 = *reinterpret_cast<const float4 *>(W3 + u);
            const float4 w1 = *reinterpret_cast<const float4 *>(W3 + H + u);
            const float4 w2 = *reinterpret_cast<const float4 *>(W3 + 2 * H + u);
            const float bv[4] = {bb.x, bb.y, bb.z, bb.w};
            const float wv[3][4] = {{w0.x, w0.y, w0.z, w0.w}, {w1.x, w1.y, w1.z, w1.w}, {w2.x, w2.y, w2.z, w2.w}};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float h2 = fmaxf(fmaf(c[4 * i + r], un2, bv[r]), 0.f);
#pragma unroll
                for (int o = 0; o < 3; ++o) z[o] += wv[o][r] * h2;
            }
        };
        fetch(0);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            v16f &c = acc[m & 1];
            const v16f &prev = acc[(m & 1) ^ 1];
            c = v16f{};
#pragma unroll
            for (int ks = 0; ks < K1; ++ks) {
                products(K1 * m + ks, xh[ks], xl[ks], c);
                if (m > 0) {
#pragma unroll
                    for (int i = ks * 4 / K1; i < (ks + 1) * 4 / K1; ++i) end1(m - 1, i, prev);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            v16f &c = acc[m & 1];
            const v16f &prev = acc[(m & 1) ^ 1];
            c = v16f{};
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {
                products(G1 + 8 * m + ks, cat(hh[2 * ks], hh[2 * ks + 1]), cat(hl[2 * ks], hl[2 * ks + 1]), c);
                if (m == 0 && ks < 4) end1(3, ks, prev);
                if (m > 0 && (ks & 1)) end2(m - 1, ks >> 1, prev);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) end2(3, i, acc[1]);
#pragma unroll
        for (int o = 0; o < 3; ++o) z[o] += other_half(z[o]);
        zout = fast_sigmoid((hf ? z[1] : z[0]) + b3[hf]);
        zout2 = fast_sigmoid(z[2] + b3[2]);
        sout = sv ? s : -1;
    }
    store_out();
}

// ------------------------------------------------------------------ backward
//
// Block = 2 BWD_RW waves in two roles (8 waves of 32 units each).  P waves (0..RW-1) own units 32 p .. of
// both hidden layers for the forward recompute and hold those rows of W1 and W2 in registers; C waves
// (RW..2RW-1) own the same units for the backward chain and hold those rows of W2^T.  Two phases per
// iteration t, with a block barrier after each:
//   1  P: layer 1 of t -> h1 plane, mask bits;           C: dz3, exponents, dz2 of t-1 -> the dz2 plane and
//         feature gradient of t-2; stage the inputs of      the dz2 frame plane; dW3 of t-1
//         t+1, loads of t+2
//   2  P: dW2 += dz2^T h1 of t-1; layer 2 of t -> h2,     C: dz1 of t-1 -> the wave's dz1 frame rows;
//         logit partials                                    dW1 += dz1^T x, dfeat partials of t-1
// What bounds it: registers hold two waves to a SIMD, so each wave's chains of dependent instructions show;
// the phases therefore hold independent work of up to three tiles.  dW1 reads only frame rows that its own
// wave wrote, so it needs no barrier of its own; the sums over three outputs (logits, dz2, dW3) go to FP32
// matrix instructions, since the vector ALU is the busier pipe (some 800 instructions a tile and SIMD, 1,400
// before); and the C waves run dz1, the longest chain of phase 2, at a raised wave priority.  981,504 samples, the
// launch repeated back to back: 543 us with four phases a tile, each a layer or a gradient, and the outputs' sums
// on the vector ALU; 437 this way (FP16 418 and 309).  Between other kernels, which leave other clocks and caches,
// the same launch takes longer: 596 and 500 in an autograd pass, 480 to 500 in a training step.
// The recompute of layer 1 multiplies the view encoding too (K = 64, split products), also where the forward took
// the ray's bias row: the two agree to FP32 rounding, not bit for bit, so a unit within rounding of its kink may
// be on here and off there.
// Both roles run the same number of barriers, so s_barrier stays matched.

constexpr int BWD_MP = 2;                   // 16-unit row tiles of one layer per wave
constexpr int BWD_RW = 8 / BWD_MP;          // waves per role: BWD_RW x 16 BWD_MP = 128 units
constexpr int BWD_RT = 64 * BWD_RW;         // threads per role
constexpr int BWD_WAVES = 2 * BWD_RW, BWD_THREADS = 64 * BWD_WAVES;
static_assert(BWD_MP == 2 && BWD_RW == 4, "the P threads stage 8 inputs each");
constexpr int NT = TILE;  // samples per block tile (two 16-sample column tiles)

// LDS of the backward kernel (bytes); the small image part is staged at offset 0
constexpr int BS = IMG_FWD_END - IMG_B1;             // b1, b2, W3, b3, meta
constexpr int BSL(int img_off) { return img_off - IMG_B1; }
// Every activation plane is sample-major ([NT samples][row stride] hi, then lo), written with 8-byte
// stores of a lane's four units; the weight-gradient products read their unit-major operands from
// the same planes with transposing LDS reads (see tr_operand).
constexpr int XB_BYTES = 2 * NT * RS1 * 2;           // x B operand [NT][RS1] hi, lo
constexpr int HB_BYTES = 2 * NT * RS2 * 2;           // one [NT][RS2] hi, lo plane
constexpr int B_XB0 = BS;                            // x: three buffers (t-1, t, t+1)
constexpr int B_HB = B_XB0 + 3 * XB_BYTES;           // h1: layer-2 and dW2 B operand, two (parity)
constexpr int B_DB = B_HB + 2 * HB_BYTES;            // dz2: dz1 B operand (per-sample scale)
constexpr int B_D2S = B_DB + HB_BYTES;               // dz2 in the dW2 frame: dW2 A operand
constexpr int B_D1S = B_D2S + HB_BYTES;              // dz1 in the dW1 frame: dW1 A operand
constexpr int B_Z3P = B_D1S + HB_BYTES;              // logit partials [RW][NT][4] f32
constexpr int DFS = 12;                              // row of dfeat partials (features)
constexpr int B_DFP = B_Z3P + BWD_RW * NT * 4 * 4;   // dfeat partials [RW][NT][DFS] f32
constexpr int H2S = H + 4;                           // row stride (floats) of the h2 plane
constexpr int B_H2 = B_DFP + BWD_RW * NT * DFS * 4;  // h2 [NT][H2S] f32, written by P, read by C
constexpr int B_MASK = B_H2 + NT * H2S * 4;          // h1 > 0 bits per lane [2][RW waves][64 lanes] u16
constexpr int B_EXP = B_MASK + 2 * BWD_RW * 64 * 2;  // exponents of x and of h1 per sample [3][NT][2]
constexpr int B_GR = B_EXP + 3 * NT * 8;             // grad_rgb [3][NT][4]
constexpr int B_DZ3 = B_GR + 3 * NT * 16;            // dz3 [RW waves][NT][4], each C wave its own
constexpr int B_F2 = B_DZ3 + BWD_RW * NT * 16;       // frame of dW2
constexpr int B_END = B_F2 + 16;
static_assert(B_END <= 160 * 1024, "backward LDS");
static_assert(B_XB0 % 16 == 0 && B_HB % 16 == 0 && B_DB % 16 == 0 && B_D2S % 16 == 0 && B_D1S % 16 == 0 &&
                  B_Z3P % 16 == 0 && B_DFP % 16 == 0 && B_H2 % 16 == 0 && B_MASK % 8 == 0 && B_EXP % 8 == 0,
              "LDS alignment");

// exponent that moves a gradient column into the accumulator frame F (operand scale e of
// the other factor); a zero column stays zero for any shift, so the clamp only guards range
__device__ __forceinline__ int frame_shift(int F, int e) {
    const int d = F - e;
    return d < -300 ? -300 : (d > 300 ? 300 : d);
}

__device__ __forceinline__ h8 lds_h8(const unsigned char *base, int off, int idx) {
    return *reinterpret_cast<const h8 *>(reinterpret_cast<const _Float16 *>(base + off) + idx);
}

__device__ __forceinline__ h8 glb_h8(const unsigned char *img, int off, int idx) {
    return *reinterpret_cast<const h8 *>(reinterpret_cast<const _Float16 *>(img + off) + idx);
}

// four values of one sample (a lane's units u0..u0+3), each moved by 2^e (exact; a zero stays zero
// for any e), split and stored at element idx of a sample-major plane (lo plane only in split mode)
template <bool SPLIT>
__device__ __forceinline__ void put_split4(unsigned char *plane, int idx, const float v[4], int e) {
    uint2 hi, lo;
    split2<false>(ldx(v[0], e), ldx(v[1], e), hi.x, lo.x);
    split2<false>(ldx(v[2], e), ldx(v[3], e), hi.y, lo.y);
    *reinterpret_cast<uint2 *>(reinterpret_cast<_Float16 *>(plane) + idx) = hi;
    if (SPLIT) *reinterpret_cast<uint2 *>(reinterpret_cast<_Float16 *>(plane) + NT * RS2 + idx) = lo;
}

// 64 bits per lane through the transposing LDS read: within each group of 16 lanes, the four
// 16-bit elements that lane t' addresses go to lanes 4 (t' mod 4) .. 4 (t' mod 4) + 3, each into
// element slot t' / 4.
__device__ __forceinline__ h4 lds_tr4(const unsigned char *p) {
    typedef short s4 __attribute__((ext_vector_type(4)));
    const s4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4 *)(p));
    return __builtin_bit_cast(h4, r);
}

// Unit-major MFMA operand (16 units U0..U0+15 as rows, the tile's 32 samples as K) from a
// sample-major plane [NT][RS] in which unit U0 + 4a + r sits at column cb + 8a + r (cb = the
// column of U0; phys slot order, U0 a multiple of 16): lane (q, j) gets unit U0 + j, its K slot
// 4h + e (h = read, e = element) holding sample 16h + 4e + q.  (The weight-gradient products sum
// over K, so any slot order serves as long as both operands use this one.)  Lane j of group q
// addresses the four units U0 + 4 (j mod 4) .. + 3 of sample 4 (j / 4) + q (+16 in the second
// read), so the four rows one 16-lane group reads lie 4 rows apart: with the 136-half row stride
// they start 16 banks apart and the group's 8-byte reads hit distinct banks.  The lane offset, in
// halves, is tr_lane<RS>(), taken once by the caller so that every read of a phase shares one
// address register.
template <int RS>
__device__ __forceinline__ int tr_lane(int j, int q) { return (4 * (j >> 2) + q) * RS + 8 * (j & 3); }
template <int RS>
__device__ __forceinline__ h8 tr_operand(const unsigned char *plane, int tl, int cb) {
    const _Float16 *p = reinterpret_cast<const _Float16 *>(plane) + tl + cb;
    return cat(lds_tr4(reinterpret_cast<const unsigned char *>(p)),
               lds_tr4(reinterpret_cast<const unsigned char *>(p + 16 * RS)));
}
// column of unit (or logical input) 16 n in the phys slot order of a 128- or 64-wide row
__device__ __forceinline__ int unit_col(int n) { return 32 * (n >> 1) + 4 * (n & 1); }

__device__ __forceinline__ void store_h4(unsigned char *base, int off, int idx, h4 v) {
    *reinterpret_cast<h4 *>(reinterpret_cast<_Float16 *>(base + off) + idx) = v;
}

// Block barrier that orders LDS only: the waves' outstanding global stores (the feature
// gradient rows) stay in flight across it instead of being drained at every phase.
// No global memory is exchanged between the waves of a block inside the backward kernel.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Orders a wave's LDS writes before its own later LDS reads of other lanes' values (the LDS keeps a wave's
// operations in order, so this only binds the compiler).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Feature gradient of a finished tile: the partials of the C waves, summed in a fixed order; t =
// the calling thread's index within its role.
template <bool VEC>
__device__ __forceinline__ void feat_grad_out(const MlpArgs &a, const float *dfp, int pbase, int t) {
    if constexpr (VEC) {  // four features to a thread
        const int sl = t / 3, c = 4 * (t - 3 * sl), s = pbase + sl;
        if (sl >= NT || s >= a.S) return;
        const float *p = dfp + sl * DFS + c;
        float4 g = *reinterpret_cast<const float4 *>(p);
#pragma unroll
        for (int ww = 1; ww < BWD_RW; ++ww) {
            const float4 v = *reinterpret_cast<const float4 *>(p + ww * NT * DFS);
            g.x += v.x, g.y += v.y, g.z += v.z, g.w += v.w;
        }
        *reinterpret_cast<float4 *>(a.grad_feat + (int64_t)s * 12 + c) = g;
        return;
    }
    for (int i = t; i < NT * a.in_feat; i += BWD_RT) {
        const int sl = i / a.in_feat, c = i % a.in_feat;
        const int s = pbase + sl;
        if (s < a.S) {
            float g = dfp[sl * DFS + c];
#pragma unroll
            for (int ww = 1; ww < BWD_RW; ++ww) g += dfp[(ww * NT + sl) * DFS + c];
            a.grad_feat[(int64_t)s * a.in_feat + c] = g;
        }
    }
}

// exponents of x (.x) and h1 (.y) of this lane's two samples 16c + j
struct SampleExp {
    int ex[2], e1[2];
};

__device__ __forceinline__ SampleExp sample_exp(const int2 *exps, int j) {
    const int2 a = exps[j], b = exps[16 + j];
    return {{a.x, b.x}, {a.y, b.y}};
}

// Output-layer gradient of a tile and the exponents that follow from it, the same in every wave.  Lane
// (q, j) forms output q (none for q = 3) of samples j and 16 + j, and the exponents of one sample,
// 16 (q / 2) + j, which two swaps hand to the lanes that scale with them.
struct GradExp {
    float dz3[2];      // dz3[q] of sample 16c + j
    int g2[2], g1[2];  // of sample 16c + j
    int k2, k1;        // of sample 16 (q / 2) + j
};

// slot of output o in a row of logit partials: the writing lanes hold outputs o and o + 2
__device__ __forceinline__ int z3_slot(int o) { return 2 * (o & 1) + (o >> 1); }

__device__ __forceinline__ GradExp grad_exp(const float *z3p, const float *gr_s, float b3q, const Meta &meta, int j,
                                            int q) {
    GradExp g;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int sl = 16 * c + j;
        float z = b3q;
#pragma unroll
        for (int ww = 0; ww < BWD_RW; ++ww) z += z3p[(ww * NT + sl) * 4 + z3_slot(q)];
        const float y = fast_sigmoid(z);
        g.dz3[c] = gr_s[sl * 4 + q] * y * (1.f - y);  // (the fourth upstream value is zero)
    }
    // max |dz3| over the outputs
    const Pair h = swap32(fabsf(g.dz3[0]), fabsf(g.dz3[1]));
    const float m = fmaxf(h.a, h.b);
    const Pair p = swap16(m, m);
    const float mx = fmaxf(p.a, p.b);
    // |dz2| <= n3t max|dz3| and |dz1| <= n2t |dz2| (infinity norms of W3^T and W2^T)
    const float bnd2 = meta.n3t * mx, bnd1 = meta.n2t * bnd2;
    g.k2 = bnd2 > 0.f ? ceil_exp(bnd2) : -FRAME_NONE;
    g.k1 = bnd1 > 0.f ? ceil_exp(bnd1) : -FRAME_NONE;
    const int e2 = scale_exp(bnd2), e1 = scale_exp(bnd1);
    const auto w2 = __builtin_amdgcn_permlane32_swap(e2, e2, false, false);
    const auto w1 = __builtin_amdgcn_permlane32_swap(e1, e1, false, false);
    g.g2[0] = w2[0];
    g.g2[1] = w2[1];
    g.g1[0] = w1[0];
    g.g1[1] = w1[1];
    return g;
}

// smallest frame the tile allows: F <= 14 + (other operand's exponent) - ceil_exp(bound), both of sample
// 16 (q / 2) + j
__device__ __forceinline__ int tile_frame(int other_e, int k) {
    const int f = row16_min(14 + other_e - k);  // over the 16 samples of the row
    // scalar, so the (rare) rescale is a real branch
    return min(__builtin_amdgcn_readlane(f, 0), __builtin_amdgcn_readlane(f, 32));
}

// dz2 = mask(h2) W3^T dz3 of one 16-unit row tile (FP32 products, K = the three outputs): w3t = W3[q][unit j
// of the tile], h = the lane's h2; added to db2, stored at its per-sample scale (the dz1 operand plane) and
// in the dW2 frame
template <bool SPLIT>
__device__ __forceinline__ void dz2_tile(float w3t, float dz3, float4 hv, int g2, int fs, int at, unsigned char *db,
                                         unsigned char *d2s, float (&db2)[4]) {
    const v4f d = __builtin_amdgcn_mfma_f32_16x16x4f32(w3t, dz3, v4f{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    const float h[4] = {hv.x, hv.y, hv.z, hv.w};
    float dz2[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        dz2[r] = h[r] > 0.f ? d[r] : 0.f;
        db2[r] += dz2[r];
    }
    h4 hi, lo;
    split4<false>(dz2, pow2(g2), hi, lo);
    store_h4(db, 0, at, hi);
    if (SPLIT) store_h4(db, NT * RS2 * 2, at, lo);
    put_split4<SPLIT>(d2s, at, dz2, fs);  // exact for any shift
}

template <int M, int N>
__device__ __forceinline__ void rescale(v4f (&acc)[M][N], int &F, int f) {
    if (f < F) {
        const int d = max(f - F, -300);
#pragma unroll
        for (int mp = 0; mp < M; ++mp)
#pragma unroll
            for (int n = 0; n < N; ++n)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[mp][n][r] = ldx(acc[mp][n][r], d);
        F = f;
    }
}

// VEC: 12 features, feat and grad_feat 16-byte aligned (rows move as float4); a template argument, since the
// general path's loads in one branch made the compiler wait for those of the other
template <bool SPLIT, bool VEC>
__global__ __launch_bounds__(BWD_THREADS) void mlp_bwd_kernel(MlpArgs a) {
    __shared__ __attribute__((aligned(16))) unsigned char sm[B_END];
    copy_to_lds(sm, a.img + IMG_B1, BS);
    const int tid = threadIdx.x, ln = lane(), j = ln & 15, q = ln >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Meta meta = *reinterpret_cast<const Meta *>(a.img + IMG_META);
    const float *b1 = reinterpret_cast<const float *>(sm + BSL(IMG_B1));
    const float *b2 = reinterpret_cast<const float *>(sm + BSL(IMG_B2));
    const float *W3 = reinterpret_cast<const float *>(sm + BSL(IMG_W3));
    const float *b3 = reinterpret_cast<const float *>(sm + BSL(IMG_B3));
    unsigned char *db = lds_region(sm, B_DB);    // dz2 (per-sample scale)
    unsigned char *d2s = lds_region(sm, B_D2S);  // dz2 in the dW2 frame
    unsigned char *d1s = lds_region(sm, B_D1S);  // dz1 in the dW1 frame
    unsigned char *rB = lds_region(sm, B_Z3P);   // partials, h2, masks, per-sample values
    float *z3p = reinterpret_cast<float *>(rB);
    float *dfp = reinterpret_cast<float *>(rB + (B_DFP - B_Z3P));
    float *h2s = reinterpret_cast<float *>(rB + (B_H2 - B_Z3P));
    // bit 15 - ((c MP + mp) 4 + r) of lane (j, q) of wave w: h1 > 0 for unit 16 (MP w + mp) + 4q + r,
    // sample 16c + j; the P wave and the C wave of the same w use the same lane -> (unit, sample) map
    uint16_t *mask_b = reinterpret_cast<uint16_t *>(rB + (B_MASK - B_Z3P));
    int2 *exp_b = reinterpret_cast<int2 *>(rB + (B_EXP - B_Z3P));
    float *gr_b = reinterpret_cast<float *>(rB + (B_GR - B_Z3P));
    float *dz3s = reinterpret_cast<float *>(rB + (B_DZ3 - B_Z3P));
    int *frame2 = reinterpret_cast<int *>(rB + (B_F2 - B_Z3P));
    const int ntiles = a.n_tiles;
    // tiles blockIdx.x + t gridDim.x, t < n
    const int n = (ntiles - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;
    float *P = a.partial + (int64_t)blockIdx.x * a.n_params;
    float *pW1 = P, *pb1 = pW1 + H * a.n_in, *pW2 = pb1 + H, *pb2 = pW2 + H * H, *pW3 = pb2 + H, *pb3 = pW3 + 3 * H;

    if (wave < BWD_RW) {
        // ================================================================ P waves
        const int w = wave;
        h8 w2h[BWD_MP][4], w2l[BWD_MP][4], w1h[BWD_MP][2], w1l[BWD_MP][2];
#pragma unroll
        for (int mp = 0; mp < BWD_MP; ++mp) {
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const int o = (16 * (BWD_MP * w + mp) + j) * RS2 + 32 * kk + 8 * q;
                w2h[mp][kk] = glb_h8(a.img, IMG_W2H, o);
                w2l[mp][kk] = glb_h8(a.img, IMG_W2L, o);
            }
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const int o = (16 * (BWD_MP * w + mp) + j) * RS1 + 32 * kk + 8 * q;
                w1h[mp][kk] = glb_h8(a.img, IMG_W1H, o);
                w1l[mp][kk] = glb_h8(a.img, IMG_W1L, o);
            }
        }
        v4f dW2[BWD_MP][8];
#pragma unroll
        for (int mp = 0; mp < BWD_MP; ++mp)
#pragma unroll
            for (int n = 0; n < 8; ++n) dW2[mp][n] = v4f{0.f, 0.f, 0.f, 0.f};
        int F2 = FRAME_NONE;
        // inputs of a tile: global loads, in three steps spread over phases so that their
        // latency overlaps other work (ray window; ray search and feature loads; staging)
        // The loaded values stay raw until stage_tile (phase 1 of the next iteration), where lanes past the last
        // sample and the padding columns are zeroed, so that nothing consumes the loads before then.
        float4 xlo = make_float4(0.f, 0.f, 0.f, 0.f), xhi = xlo;
        float grv = 0.f;
        unsigned xok = 0;  // bit 0: xlo is real, bit 1: xhi is real, bit 2: grv is real
        // (lane l of wave w: sample 8 w + l / 8, slot group xg = l mod 8)
        auto load_tile = [&](int t, int r0, int win) {
            const int ln = fresh(lane()), xg = ln & 7;
            const int s = t * NT + 8 * w + (ln >> 3);
            const bool sv = s < a.S;
            // all lanes take part; this wave's samples are t NT + 8 w + (lane >> 3).  Lanes past the
            // last sample load from the last sample and its ray (kept in range).
            const int ray = min(ray_of_group8(a.offs, a.n_rays, r0, win, t * NT + 8 * w), a.n_rays - 1);
            const int sc = sv ? s : a.S - 1;
            const int kk = xg >> 2, q = xg & 3;
            if constexpr (VEC) {
                // every lane issues the same two 16-byte loads and one 4-byte load, with no divergent
                // branch around them (divergent branches would make one group's loads wait for the
                // other's, as both write the same registers)
                const float *pe = a.pe + (int64_t)ray * PEW;
                const float *pl = kk == 0 && q < 3 ? a.feat + (int64_t)sc * 12 + 4 * q : pe + (kk == 0 ? 0 : 20 + 4 * q);
                xlo = *reinterpret_cast<const float4 *>(pl);
                xhi = *reinterpret_cast<const float4 *>(pe + 4 + 4 * q);
                grv = a.grad_rgb[(int64_t)sc * 3 + (xg < 3 ? xg : 2)];
                xok = (sv ? 1u : 0u) | (sv && kk == 0 ? 2u : 0u) | (sv && xg < 3 ? 4u : 0u);
            } else {
                float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                float g = 0.f;
                if (sv) {
                    load_x8(a, s, ray, kk, q, v);
                    if (xg < 3) g = a.grad_rgb[(int64_t)s * 3 + xg];
                }
                xlo = make_float4(v[0], v[1], v[2], v[3]);
                xhi = make_float4(v[4], v[5], v[6], v[7]);
                grv = g;
                xok = 7u;
            }
        };
        // ... and their split into the x plane of buffer xs (layer-1 B operand, read transposed by
        // dW1), the sample's exponents and grad_rgb
        auto stage_tile = [&](int xs) {
            const int ln = fresh(lane()), xg = ln & 7, xsl = 8 * w + (ln >> 3);
            const bool l = xok & 1u, h = xok & 2u;
            const float xv[8] = {l ? xlo.x : 0.f, l ? xlo.y : 0.f, l ? xlo.z : 0.f, l ? xlo.w : 0.f,
                                 h ? xhi.x : 0.f, h ? xhi.y : 0.f, h ? xhi.z : 0.f, h ? xhi.w : 0.f};
            float m = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(xv[e]));
            m = group8_max(m);  // over the 8 slot groups xg of this sample
            const int ex = scale_exp(m);
            const float sc = pow2(ex);
            h4 h0, l0, h1, l1;
            split4<false>(&xv[0], sc, h0, l0);
            split4<false>(&xv[4], sc, h1, l1);
            const int xb = B_XB0 + xs * XB_BYTES;
            *reinterpret_cast<h8 *>(reinterpret_cast<_Float16 *>(sm + xb) + xsl * RS1 + 8 * xg) = cat(h0, h1);
            if (SPLIT)
                *reinterpret_cast<h8 *>(reinterpret_cast<_Float16 *>(sm + xb + NT * RS1 * 2) + xsl * RS1 + 8 * xg) =
                    cat(l0, l1);
            if (xg == 0) exp_b[xs * NT + xsl] = make_int2(ex, scale_exp(meta.n1 * m + meta.b1max));
            if (xg < 4) gr_b[(xs * NT + xsl) * 4 + xg] = (xok & 4u) ? grv : 0.f;
        };
        // First rays of this block's tiles, 64 iterations at a time: lane l holds that of iteration
        // wb + l (wb a multiple of 64; indices past the last tile repeat the last tile's ray, a
        // valid ray).  One load per 64 tiles instead of a dependent load at the head of every tile.
        auto ray_window = [&](int wb) {
            const int t = (int)blockIdx.x + (wb + lane()) * (int)gridDim.x;
            return a.tile_ray[t < ntiles ? t : ntiles - 1];
        };
        int trw = ray_window(0);
        auto load_ahead = [&](int t, int r0, int win) { load_tile((int)blockIdx.x + t * (int)gridDim.x, r0, win); };
        for (int t = 0; t < 2; ++t) {  // (a second tile that is not there loads the last sample, unused)
            const int r0 = __builtin_amdgcn_readlane(trw, t);
            load_ahead(t, r0, window_entry(a.offs, a.n_rays, r0));
            if (t == 0) stage_tile(0);
        }
        lds_barrier();  // staged image and the first tile's inputs
        // dW2 += dz2^T h1 of a finished tile (K = its 32 samples; both operands read transposed from
        // the sample-major planes: the dz2 frame plane and that tile's h1 plane)
        auto dw2_step = [&](const unsigned char *h1p) {
            const int ln = fresh(lane()), j = ln & 15, q = ln >> 4;
            const int tl = tr_lane<RS2>(j, q);
            h8 ah[BWD_MP], al[BWD_MP];
#pragma unroll
            for (int mp = 0; mp < BWD_MP; ++mp) {
                const int cb = unit_col(BWD_MP * w + mp);
                ah[mp] = tr_operand<RS2>(d2s, tl, cb);
                al[mp] = SPLIT ? tr_operand<RS2>(d2s + NT * RS2 * 2, tl, cb) : ah[mp];
            }
            // the reads of step n + 1 beside the products of step n, and no further ahead (registers)
            h8 bh = tr_operand<RS2>(h1p, tl, unit_col(0)), bl = SPLIT ? tr_operand<RS2>(h1p + NT * RS2 * 2, tl, unit_col(0)) : bh;
#pragma unroll
            for (int n = 0; n < 8; ++n) {
                const h8 ch = bh, cl = bl;
                if (n < 7) {
                    bh = tr_operand<RS2>(h1p, tl, unit_col(n + 1));
                    bl = SPLIT ? tr_operand<RS2>(h1p + NT * RS2 * 2, tl, unit_col(n + 1)) : bh;
                }
                if (SPLIT) {
#pragma unroll
                    for (int mp = 0; mp < BWD_MP; ++mp) dW2[mp][n] = mfma16(al[mp], ch, dW2[mp][n]);
#pragma unroll
                    for (int mp = 0; mp < BWD_MP; ++mp) dW2[mp][n] = mfma16(ah[mp], cl, dW2[mp][n]);
                }
#pragma unroll
                for (int mp = 0; mp < BWD_MP; ++mp) dW2[mp][n] = mfma16(ah[mp], ch, dW2[mp][n]);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        int xs = 0, xn = 1;  // input buffers of t and t+1
        for (int it = 0; it <= n; ++it) {
            const int ln = fresh(lane()), j = ln & 15, q = ln >> 4;
            const int pb = it & 1;
            unsigned char *hb = lds_region(sm, B_HB + pb * HB_BYTES);
            const int2 *exps = exp_b + xs * NT;
            const int xb = B_XB0 + xs * XB_BYTES;
            uint16_t *mask1 = mask_b + pb * (BWD_RW * 64);
            // ---- 1: ray window of tile t+2 (consumed at the end of the phase)
            if (((it + 2) & 63) == 0) trw = ray_window(it + 2);
            const int r0n = __builtin_amdgcn_readlane(trw, (it + 2) & 63);
            const int winn = window_entry(a.offs, a.n_rays, r0n);
            //      layer 1 for this wave's units; h1 -> the h1 plane, mask bits
            if (it < n) {
                const SampleExp se = sample_exp(exps, j);
                v4f acc[2][BWD_MP];  // [c][mp]
                unsigned mbits = 0;
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int mp = 0; mp < BWD_MP; ++mp) acc[c][mp] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) {
                    h8 bh[2], bl[2];
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        bh[c] = lds_h8(sm, xb, (16 * c + j) * RS1 + 32 * kk + 8 * q);
                        bl[c] = lds_h8(sm, xb + NT * RS1 * 2, (16 * c + j) * RS1 + 32 * kk + 8 * q);
                    }
                    if (SPLIT) {
#pragma unroll
                        for (int c = 0; c < 2; ++c)
#pragma unroll
                            for (int mp = 0; mp < BWD_MP; ++mp) acc[c][mp] = mfma16(w1l[mp][kk], bh[c], acc[c][mp]);
#pragma unroll
                        for (int c = 0; c < 2; ++c)
#pragma unroll
                            for (int mp = 0; mp < BWD_MP; ++mp) acc[c][mp] = mfma16(w1h[mp][kk], bl[c], acc[c][mp]);
                    }
#pragma unroll
                    for (int c = 0; c < 2; ++c)
#pragma unroll
                        for (int mp = 0; mp < BWD_MP; ++mp) acc[c][mp] = mfma16(w1h[mp][kk], bh[c], acc[c][mp]);
                }
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const float un = pow2(-(meta.sw1 + se.ex[c]));
                    const float sc = pow2(se.e1[c]);
#pragma unroll
                    for (int mp = 0; mp < BWD_MP; ++mp) {
                        const float4 bb = *reinterpret_cast<const float4 *>(b1 + 16 * (BWD_MP * w + mp) + 4 * q);
                        const float bv[4] = {bb.x, bb.y, bb.z, bb.w};
                        float h1[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            h1[r] = fmaxf(fmaf(acc[c][mp][r], un, bv[r]), 0.f);
                            // shift in the sign of 0 - h1 (as integers: set unless h1 is zero)
                            mbits = __builtin_amdgcn_alignbit(mbits, 0u - __builtin_bit_cast(unsigned, h1[r]), 31);
                        }
                        h4 hi, lo;
                        split4<false>(h1, sc, hi, lo);
                        const int ob = (16 * c + j) * RS2 + unit_col(BWD_MP * w + mp) + 8 * q;
                        store_h4(hb, 0, ob, hi);
                        if (SPLIT) store_h4(hb, NT * RS2 * 2, ob, lo);
                    }
                }
                mask1[w * 64 + ln] = (uint16_t)mbits;
            }
            //      feature gradient of the tile whose partials the last phase 2 left
            if (it > 1) feat_grad_out<VEC>(a, dfp, ((int)blockIdx.x + (it - 2) * (int)gridDim.x) * NT, 64 * w + ln);
            //      the next tile's inputs, loaded an iteration ago; the loads of the one after
            if (it + 1 < n) stage_tile(xn);
            if (it + 2 < n) load_ahead(it + 2, r0n, winn);
            lds_barrier();
            // ---- 2: dW2 of the previous tile; layer 2 for this wave's units, logit partials
            if (it > 0) {
                const int f = __builtin_amdgcn_readfirstlane(*frame2);  // as the dz2 frame plane was written
                rescale(dW2, F2, f);
                dw2_step(lds_region(sm, B_HB + (pb ^ 1) * HB_BYTES));
            }
            if (it < n) {
                const SampleExp se = sample_exp(exps, j);
                v4f acc[2][BWD_MP], zp[2];  // [c][mp]; logits of sample 16c + j over this lane's units
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    zp[c] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int mp = 0; mp < BWD_MP; ++mp) acc[c][mp] = v4f{0.f, 0.f, 0.f, 0.f};
                }
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    h8 bh[2], bl[2];
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        bh[c] = lds_h8(hb, 0, (16 * c + j) * RS2 + 32 * kk + 8 * q);
                        bl[c] = lds_h8(hb, NT * RS2 * 2, (16 * c + j) * RS2 + 32 * kk + 8 * q);
                    }
                    if (SPLIT) {
#pragma unroll
                        for (int c = 0; c < 2; ++c)
#pragma unroll
                            for (int mp = 0; mp < BWD_MP; ++mp) acc[c][mp] = mfma16(w2l[mp][kk], bh[c], acc[c][mp]);
#pragma unroll
                        for (int c = 0; c < 2; ++c)
#pragma unroll
                            for (int mp = 0; mp < BWD_MP; ++mp) acc[c][mp] = mfma16(w2h[mp][kk], bl[c], acc[c][mp]);
                    }
#pragma unroll
                    for (int c = 0; c < 2; ++c)
#pragma unroll
                        for (int mp = 0; mp < BWD_MP; ++mp) acc[c][mp] = mfma16(w2h[mp][kk], bh[c], acc[c][mp]);
                }
                // W3 of output ln % 4 and this lane's units (a fourth row repeats the first: its logit is formed and
                // read as one, and its gradient is zero, as its upstream value is)
                float4 wa[BWD_MP];
#pragma unroll
                for (int mp = 0; mp < BWD_MP; ++mp)
                    wa[mp] = *reinterpret_cast<const float4 *>(W3 + ((ln & 3) < 3 ? (ln & 3) * H : 0) +
                                                               16 * (BWD_MP * w + mp) + 4 * q);
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const float un = pow2(-(meta.sw2 + se.e1[c]));
#pragma unroll
                    for (int mp = 0; mp < BWD_MP; ++mp) {
                        const int u0 = 16 * (BWD_MP * w + mp) + 4 * q;
                        const float4 bb = *reinterpret_cast<const float4 *>(b2 + u0);
                        const float bv[4] = {bb.x, bb.y, bb.z, bb.w}, w3a[4] = {wa[mp].x, wa[mp].y, wa[mp].z, wa[mp].w};
                        float h2[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            h2[r] = fmaxf(fmaf(acc[c][mp][r], un, bv[r]), 0.f);
                            // four outputs x four samples in each of 16 blocks, this lane's unit as K
                            zp[c] = __builtin_amdgcn_mfma_f32_4x4x1f32(w3a[r], h2[r], zp[c], 0, 0, 0);
                        }
                        *reinterpret_cast<float4 *>(h2s + (16 * c + j) * H2S + u0) =
                            make_float4(h2[0], h2[1], h2[2], h2[3]);
                    }
                }
                // over the four unit groups q: lane (q, j) ends with outputs q % 2 and q % 2 + 2 of sample
                // 16 (q / 2) + j
                float t[2][2];
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const Pair p = swap16(zp[c][2 * h], zp[c][2 * h + 1]);
                        t[c][h] = p.a + p.b;
                    }
                const Pair p0 = swap32(t[0][0], t[1][0]), p1 = swap32(t[0][1], t[1][1]);
                *reinterpret_cast<float2 *>(z3p + (w * NT + 16 * (q >> 1) + j) * 4 + 2 * (q & 1)) =
                    make_float2(p0.a + p0.b, p1.a + p1.b);
            }
            lds_barrier();
            xs = xn;
            xn = xn == 2 ? 0 : xn + 1;
        }
        feat_grad_out<VEC>(a, dfp, ((int)blockIdx.x + (n - 1) * (int)gridDim.x) * NT, tid);
        // ---- partial gradient of the P role: W2
        const int u2 = F2 == FRAME_NONE ? 0 : -F2;
#pragma unroll
        for (int mp = 0; mp < BWD_MP; ++mp)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int hrow = 16 * (BWD_MP * w + mp) + 4 * q + r;
#pragma unroll
                for (int n = 0; n < 8; ++n) pW2[hrow * H + 16 * n + j] = ldx(dW2[mp][n][r], u2);
            }
    } else {
        // ================================================================ C waves
        const int w = wave - BWD_RW;
        h8 w2th[BWD_MP][4], w2tl[BWD_MP][4];
#pragma unroll
        for (int mp = 0; mp < BWD_MP; ++mp)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const int o = (16 * (BWD_MP * w + mp) + j) * RS2 + 32 * kk + 8 * q;
                w2th[mp][kk] = glb_h8(a.img, IMG_W2TH, o);
                w2tl[mp][kk] = glb_h8(a.img, IMG_W2TL, o);
            }
        // W1's feature columns, transposed (rows = features), over this wave's units as K
        const int ofF = j * RS2 + unit_col(BWD_MP * w) + 8 * q;
        const h8 w1fh = glb_h8(a.img, IMG_W1FH, ofF), w1fl = glb_h8(a.img, IMG_W1FL, ofF);
        v4f dW1[BWD_MP][3];
#pragma unroll
        for (int mp = 0; mp < BWD_MP; ++mp)
#pragma unroll
            for (int n = 0; n < 3; ++n) dW1[mp][n] = v4f{0.f, 0.f, 0.f, 0.f};
        // lane-local sums over this lane's samples; reduced over the 16 sample lanes at the end (db3 of
        // output q)
        float db1[BWD_MP][4], db2[BWD_MP][4], db3 = 0.f;
#pragma unroll
        for (int mp = 0; mp < BWD_MP; ++mp)
#pragma unroll
            for (int r = 0; r < 4; ++r) db1[mp][r] = db2[mp][r] = 0.f;
        // element i of dw3[g], lane l: output i, unit 32 w + 8 (l % 4) + g, samples l / 4 and 16 + l / 4
        v4f dw3[8];
#pragma unroll
        for (int g = 0; g < 8; ++g) dw3[g] = v4f{0.f, 0.f, 0.f, 0.f};
        int F1 = FRAME_NONE, F2 = FRAME_NONE;
        // dW1 += dz1^T x of a finished tile (its x buffer xs; both operands read transposed from the
        // sample-major planes; logical inputs 0..47 in the three 16-column blocks)
        auto dw1_step = [&](int xs) {
            const int ln = fresh(lane()), j = ln & 15, q = ln >> 4;
            const int t2 = tr_lane<RS2>(j, q), t1 = tr_lane<RS1>(j, q);
            const unsigned char *xp = lds_region(sm, B_XB0 + xs * XB_BYTES);
#pragma unroll
            for (int mp = 0; mp < BWD_MP; ++mp) {
                const int cb = unit_col(BWD_MP * w + mp);
                const h8 dh = tr_operand<RS2>(d1s, t2, cb);
                const h8 dl = SPLIT ? tr_operand<RS2>(d1s + NT * RS2 * 2, t2, cb) : dh;
#pragma unroll
                for (int n = 0; n < 3; ++n) {
                    const h8 bh = tr_operand<RS1>(xp, t1, unit_col(n));
                    const h8 bl = SPLIT ? tr_operand<RS1>(xp + NT * RS1 * 2, t1, unit_col(n)) : bh;
                    if (SPLIT) {
                        dW1[mp][n] = mfma16(dl, bh, dW1[mp][n]);
                        dW1[mp][n] = mfma16(dh, bl, dW1[mp][n]);
                    }
                    dW1[mp][n] = mfma16(dh, bh, dW1[mp][n]);
                }
            }
        };
        // dW3 += dz3 h2^T of the current tile for this wave's units: 4x4x1 FP32 products, a sample per block
        // (outputs x four units), so every product is an FMA into the lane's own sum
        auto dw3_step = [&](int ln) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float d = dz3s[w * NT * 4 + 64 * c + ln];  // output ln % 4 of sample 16c + ln / 4
                const float4 *hp = reinterpret_cast<const float4 *>(h2s + (16 * c + (ln >> 2)) * H2S +
                                                                    16 * BWD_MP * w + 8 * (ln & 3));
                const float4 h0 = hp[0], h1 = hp[1];
                const float h[8] = {h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w};
#pragma unroll
                for (int g = 0; g < 8; ++g) dw3[g] = __builtin_amdgcn_mfma_f32_4x4x1f32(d, h[g], dw3[g], 0, 0, 0);
            }
        };
        // dz1 = mask(h1) W2^T dz2 of a tile (its mask bits, exponents g2 and ex), kept in registers and written to
        // the frame rows in the dW1 frame
        auto dz1_step = [&](const int g2[2], const int ex[2], unsigned mbits, float (&dz1)[BWD_MP][2][4]) {
            const int ln = fresh(lane()), j = ln & 15, q = ln >> 4;
            v4f acc[2][BWD_MP];  // [c][mp]
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int mp = 0; mp < BWD_MP; ++mp) acc[c][mp] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                h8 bh[2], bl[2];
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    bh[c] = lds_h8(db, 0, (16 * c + j) * RS2 + 32 * kk + 8 * q);
                    bl[c] = lds_h8(db, NT * RS2 * 2, (16 * c + j) * RS2 + 32 * kk + 8 * q);
                }
                if (SPLIT) {
#pragma unroll
                    for (int c = 0; c < 2; ++c)
#pragma unroll
                        for (int mp = 0; mp < BWD_MP; ++mp) acc[c][mp] = mfma16(w2tl[mp][kk], bh[c], acc[c][mp]);
#pragma unroll
                    for (int c = 0; c < 2; ++c)
#pragma unroll
                        for (int mp = 0; mp < BWD_MP; ++mp) acc[c][mp] = mfma16(w2th[mp][kk], bl[c], acc[c][mp]);
                }
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int mp = 0; mp < BWD_MP; ++mp) acc[c][mp] = mfma16(w2th[mp][kk], bh[c], acc[c][mp]);
            }
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float un = pow2(-(meta.sw2 + g2[c]));
                const int fs = frame_shift(F1, ex[c]);  // exact for any shift; 0 stays 0
#pragma unroll
                for (int mp = 0; mp < BWD_MP; ++mp) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        // all ones where h1 > 0
                        int on = __builtin_amdgcn_sbfe((int)mbits, 15 - ((c * BWD_MP + mp) * 4 + r), 1);
                        asm("" : "+v"(on));  // kept as a mask: one AND, where a select takes a compare too
                        dz1[mp][c][r] = __builtin_bit_cast(float, __builtin_bit_cast(int, acc[c][mp][r] * un) & on);
                        db1[mp][r] += dz1[mp][c][r];
                    }
                    put_split4<SPLIT>(d1s, (16 * c + j) * RS2 + unit_col(BWD_MP * w + mp) + 8 * q, dz1[mp][c], fs);
                }
            }
        };
        // dfeat partial of that tile over this wave's units: rows = feature 4q + r, column = sample
        auto dfeat_step = [&](const int g1[2], const float (&dz1)[BWD_MP][2][4]) {
            const int ln = fresh(lane()), j = ln & 15, q = ln >> 4;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float sc = pow2(g1[c]);
                v4f df = v4f{0.f, 0.f, 0.f, 0.f};
                h4 h0, l0, h1v, l1v;
                split4<true>(dz1[0][c], sc, h0, l0);
                split4<true>(dz1[1][c], sc, h1v, l1v);
                const h8 bh = cat(h0, h1v), bl = cat(l0, l1v);
                if (SPLIT) {
                    df = mfma16(w1fl, bh, df);
                    df = mfma16(w1fh, bl, df);
                }
                df = mfma16(w1fh, bh, df);
                const float un = pow2(-(meta.sw1 + g1[c]));
                if (q < DFS / 4)
                    *reinterpret_cast<float4 *>(dfp + (w * NT + 16 * c + j) * DFS + 4 * q) =
                        make_float4(df[0] * un, df[1] * un, df[2] * un, df[3] * un);
            }
        };
        lds_barrier();  // staged image and the first tile's inputs
        // W3 as the operand of dz2: output q of unit j of a row tile
        const float w3t[BWD_MP] = {q < 3 ? W3[q * H + 16 * BWD_MP * w + j] : 0.f,
                                   q < 3 ? W3[q * H + 16 * (BWD_MP * w + 1) + j] : 0.f};
        const float b3q = b3[q];
        int xs = 0, xp = 2;  // input buffers of t and t-1
        for (int it = 0; it <= n; ++it) {
            const int ln = fresh(lane()), j = ln & 15, q = ln >> 4;
            int g2[2] = {0, 0}, g1[2] = {0, 0}, ex[2] = {0, 0};  // exponents of the previous tile
            // ---- 1: output gradient and exponents of the previous tile, the frames, db3 += dz3; dz2; dW3
            if (it > 0) {
                const SampleExp se = sample_exp(exp_b + xp * NT, j);
                const GradExp ge = grad_exp(z3p, gr_b + xp * NT * 4, b3q, meta, j, q);
                rescale(dW1, F1, tile_frame(q < 2 ? se.ex[0] : se.ex[1], ge.k1));
                F2 = min(F2, tile_frame(q < 2 ? se.e1[0] : se.e1[1], ge.k2));
                if (tid == BWD_RT) *frame2 = F2;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    g2[c] = ge.g2[c];
                    g1[c] = ge.g1[c];
                    ex[c] = se.ex[c];
                    db3 += ge.dz3[c];
                    dz3s[(w * NT + 16 * c + j) * 4 + q] = ge.dz3[c];
                }
                wave_lds_fence();
#pragma unroll
                for (int mp = 0; mp < BWD_MP; ++mp)
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const float4 hv = *reinterpret_cast<const float4 *>(h2s + (16 * c + j) * H2S +
                                                                            16 * (BWD_MP * w + mp) + 4 * q);
                        dz2_tile<SPLIT>(w3t[mp], ge.dz3[c], hv, ge.g2[c], frame_shift(F2, se.e1[c]),
                                        (16 * c + j) * RS2 + unit_col(BWD_MP * w + mp) + 8 * q, db, d2s, db2[mp]);
                    }
                dw3_step(ln);
            }
            lds_barrier();
            // ---- 2: dz1, dW1 and dfeat of the previous tile
            if (it > 0) {
                __builtin_amdgcn_s_setprio(3);  // 490 -> 473 us
                float dz1[BWD_MP][2][4];
                dz1_step(g2, ex, mask_b[((it - 1) & 1) * (BWD_RW * 64) + w * 64 + ln], dz1);
                // the raised priority is for the chain up to here, and the feature partials cover the way of
                // the frame rows through LDS: 457 -> 440 us
                __builtin_amdgcn_s_setprio(0);
                wave_lds_fence();
                dfeat_step(g1, dz1);
                dw1_step(xp);
            }
            lds_barrier();
            xp = xs;
            xs = xs == 2 ? 0 : xs + 1;
        }
        // ---- partial gradients of the C role: W1, b1, b2, W3, b3
        const int u1 = F1 == FRAME_NONE ? 0 : -F1;
#pragma unroll
        for (int mp = 0; mp < BWD_MP; ++mp)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int hrow = 16 * (BWD_MP * w + mp) + 4 * q + r;
#pragma unroll
                for (int n = 0; n < 3; ++n) {
                    const int c = w1_col(a.in_feat, a.n_freq, 16 * n + j);
                    if (c >= 0) pW1[hrow * a.n_in + c] = ldx(dW1[mp][n][r], u1);
                }
                float s1 = db1[mp][r], s2 = db2[mp][r];
#pragma unroll
                for (int o = 1; o < 16; o <<= 1) {
                    s1 += __shfl_xor(s1, o, 64);
                    s2 += __shfl_xor(s2, o, 64);
                }
                if (j == 0) {
                    pb1[hrow] = s1;
                    pb2[hrow] = s2;
                }
            }
#pragma unroll
        for (int g = 0; g < 8; ++g)
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                float s3 = dw3[g][i];
#pragma unroll
                for (int o = 4; o < 64; o <<= 1) s3 += __shfl_xor(s3, o, 64);
                if (ln < 4) pW3[i * H + 16 * BWD_MP * w + 8 * ln + g] = s3;
            }
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) db3 += __shfl_xor(db3, o, 64);
        if (w == 0 && j == 0 && q < 3) pb3[q] = db3;
    }
}

// gradient += sum of the per-block partials: 64 parameters per block, the four waves sum
// interleaved quarters of the partials and are combined in a fixed order
constexpr int RED_THREADS = 256;

__global__ __launch_bounds__(RED_THREADS) void mlp_reduce_kernel(MlpArgs a) {
    __shared__ float part[RED_THREADS / 64][64];
    const int wv = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int i = blockIdx.x * 64 + l;
    float acc = 0.f;
    if (i < a.n_params) {
#pragma unroll 8
        for (int b = wv; b < a.nblocks; b += RED_THREADS / 64) acc += a.partial[(int64_t)b * a.n_params + i];
    }
    part[wv][l] = acc;
    __syncthreads();
    if (wv != 0 || i >= a.n_params) return;
    acc = (part[0][l] + part[1][l]) + (part[2][l] + part[3][l]);
    const int nW1 = H * a.n_in;
    int k = i;
    if (k < nW1) { a.gW1[k] += acc; return; }
    k -= nW1;
    if (k < H) { a.gb1[k] += acc; return; }
    k -= H;
    if (k < H * H) { a.gW2[k] += acc; return; }
    k -= H * H;
    if (k < H) { a.gb2[k] += acc; return; }
    k -= H;
    if (k < 3 * H) { a.gW3[k] += acc; return; }
    k -= 3 * H;
    a.gb3[k] += acc;
}

int check_mlp(const dvgo_color_mlp *m, bool bwd) {
    if (!m) return set_error(DVGO_ERR_NULL, "mlp is NULL");
    if (m->struct_size != sizeof(dvgo_color_mlp)) return set_error(DVGO_ERR_ABI, "dvgo_color_mlp.struct_size mismatch");
    if (m->hidden != H) return set_error(DVGO_ERR_UNSUPPORTED, "hidden must be %d", H);
    if (m->in_feat < 1 || m->in_feat > 12) return set_error(DVGO_ERR_UNSUPPORTED, "in_feat must be in [1, 12]");
    if (m->precision != DVGO_MLP_SPLIT_F16 && m->precision != DVGO_MLP_F16)
        return set_error(DVGO_ERR_UNSUPPORTED, "unknown precision %d", m->precision);
    if (m->n_freq < 0 || m->n_freq > 4) return set_error(DVGO_ERR_UNSUPPORTED, "n_freq must be in [0, 4]");
    if (!m->W1 || !m->b1 || !m->W2 || !m->b2 || !m->W3 || !m->b3) return set_error(DVGO_ERR_NULL, "a weight is NULL");
    if (bwd && (!m->gW1 || !m->gb1 || !m->gW2 || !m->gb2 || !m->gW3 || !m->gb3))
        return set_error(DVGO_ERR_NULL, "a weight gradient is NULL");
    return DVGO_OK;
}

int n_in_of(const dvgo_color_mlp *m) { return m->in_feat + 3 + 6 * m->n_freq; }
int n_params_of(const dvgo_color_mlp *m) { return H * n_in_of(m) + H + H * H + H + 3 * H + 3; }
int bwd_blocks(int64_t S) {
    int64_t t = (S + NT - 1) / NT;
    return (int)(t < MAX_BLOCKS ? (t < 1 ? 1 : t) : MAX_BLOCKS);
}

// Whether the preparation makes the rays' bias rows, which the split forward then reads: a rule on the batch
// alone, since one preparation serves every call on it.  A row costs its ray 128 x 39 FMAs and 528 bytes, and
// saves two of layer 1's three K-steps on each of the ray's samples.  300,000 samples, preparation and forward
// without rows and with them, us: 6 samples a ray 51 and 64, 12 49 and 53, 20 48.5 and 47.6, 40 47 and 44, 100
// 47 and 43.  Up to a few thousand rays the row blocks run beside those of the weights (0.7 us at 7,500).
bool ray_rows(int32_t R, int64_t S) { return R <= 8192 || S >= 24 * (int64_t)R; }

size_t ws_layout(const dvgo_color_mlp *m, int32_t R, int64_t S, size_t *off_pe, size_t *off_rb, size_t *off_tr,
                 size_t *off_part) {
    size_t o = align_up((size_t)IMG_BYTES, 256);
    *off_pe = o;
    o += align_up((size_t)R * PEW * 4, 256);
    *off_rb = o;
    if (ray_rows(R, S)) o += align_up((size_t)R * RBW * 4, 256);
    *off_tr = o;
    o += align_up((size_t)((S + TILE - 1) / TILE) * 4, 256);
    *off_part = o;
    o += (size_t)bwd_blocks(S) * n_params_of(m) * 4;
    return o;
}

int setup(const dvgo_color_mlp *m, int32_t R, const int32_t *offs, const float *dirs, int64_t S, const float *feat,
          void *ws, size_t ws_bytes, bool bwd, MlpArgs &a, bool need_feat = true) {
    int rc = check_mlp(m, bwd);
    if (rc) return rc;
    if (R < 0 || S < 0) return set_error(DVGO_ERR_SHAPE, "negative n_rays or n_samples");
    if (S >= ((int64_t)1 << 31) / 16) return set_error(DVGO_ERR_RANGE, "n_samples too large");
    if (S > 0 && (R == 0 || !offs || !dirs || (need_feat && !feat)))
        return set_error(DVGO_ERR_NULL, "ray_offsets, dirs or feat is NULL");
    size_t off_pe, off_rb, off_tr, off_part;
    const size_t need = ws_layout(m, R, S, &off_pe, &off_rb, &off_tr, &off_part);
    if (!ws || ws_bytes < need) return set_error(DVGO_ERR_WORKSPACE, "workspace too small (%zu < %zu)", ws_bytes, need);
    if (((uintptr_t)ws & 255) != 0) return set_error(DVGO_ERR_SHAPE, "workspace must be 256-byte aligned");
    memset(&a, 0, sizeof(a));
    a.W1 = m->W1; a.b1 = m->b1; a.W2 = m->W2; a.b2 = m->b2; a.W3 = m->W3; a.b3 = m->b3;
    a.gW1 = m->gW1; a.gb1 = m->gb1; a.gW2 = m->gW2; a.gb2 = m->gb2; a.gW3 = m->gW3; a.gb3 = m->gb3;
    a.in_feat = m->in_feat;
    a.n_freq = m->n_freq;
    a.n_in = n_in_of(m);
    a.n_params = n_params_of(m);
    a.n_rays = R;
    a.offs = offs;
    a.dirs = dirs;
    a.S = (int)S;
    a.feat = feat;
    a.feat_vec = m->in_feat == 12 && ((uintptr_t)feat & 15) == 0;
    a.img = (unsigned char *)ws;
    a.pe = (float *)((char *)ws + off_pe);
    a.rb = ray_rows(R, S) ? (float *)((char *)ws + off_rb) : nullptr;
    a.tile_ray = (int *)((char *)ws + off_tr);
    a.n_tiles = (int)((S + TILE - 1) / TILE);
    a.partial = (float *)((char *)ws + off_part);
    a.nblocks = bwd_blocks(S);
    return DVGO_OK;
}

template <int GM>
int launch_fwd(const MlpArgs &a, const dvgo_color_mlp *m, hipStream_t st) {
    const dim3 grid(a.n_tiles < MAX_BLOCKS ? a.n_tiles : MAX_BLOCKS);
    if (m->precision == DVGO_MLP_F16)
        hipLaunchKernelGGL((mlp_fwd_kernel<false, GM, false>), grid, dim3(FWD_THREADS), 0, st, a);
    else if (a.rb)
        hipLaunchKernelGGL((mlp_fwd_kernel<true, GM, true>), grid, dim3(FWD_THREADS), 0, st, a);
    else
        hipLaunchKernelGGL((mlp_fwd_kernel<true, GM, false>), grid, dim3(FWD_THREADS), 0, st, a);
    return check_hip(hipGetLastError(), "mlp_fwd_kernel launch");
}

int launch_prep(const MlpArgs &a, hipStream_t st) {
    const int n = PREP_FIXED_BLOCKS + ray_blocks(a) + (a.n_tiles + PREP_THREADS - 1) / PREP_THREADS;
    hipLaunchKernelGGL(mlp_prep_kernel, dim3(n), dim3(PREP_THREADS), 0, st, a);
    return check_hip(hipGetLastError(), "mlp_prep_kernel launch");
}

}  // namespace

extern "C" int dvgo_mlp_workspace_size(const dvgo_color_mlp *m, int32_t n_rays, int64_t n_samples, size_t *bytes) {
    int rc = check_mlp(m, false);
    if (rc) return rc;
    if (!bytes) return set_error(DVGO_ERR_NULL, "bytes is NULL");
    if (n_rays < 0 || n_samples < 0) return set_error(DVGO_ERR_SHAPE, "negative size");
    size_t a, b, c, d;
    *bytes = ws_layout(m, n_rays, n_samples, &a, &b, &c, &d);
    return DVGO_OK;
}

extern "C" int dvgo_mlp_prepare(const dvgo_color_mlp *m, int32_t n_rays, const int32_t *ray_offsets,
                                const float *dirs, int64_t n_samples, void *ws, size_t ws_bytes, void *stream) {
    MlpArgs a;
    int rc = setup(m, n_rays, ray_offsets, dirs, n_samples, nullptr, ws, ws_bytes, false, a, false);
    if (rc) return rc;
    if (n_samples == 0) return DVGO_OK;
    return launch_prep(a, (hipStream_t)stream);
}

extern "C" int dvgo_mlp_forward(const dvgo_color_mlp *m, int32_t n_rays, const int32_t *ray_offsets,
                                const float *dirs, int64_t n_samples, const float *feat, float *rgb, void *ws,
                                size_t ws_bytes, void *stream) {
    MlpArgs a;
    int rc = setup(m, n_rays, ray_offsets, dirs, n_samples, feat, ws, ws_bytes, false, a);
    if (rc) return rc;
    if (n_samples == 0) return DVGO_OK;
    if (!rgb) return set_error(DVGO_ERR_NULL, "rgb is NULL");
    a.rgb = rgb;
    hipStream_t st = (hipStream_t)stream;
    if (!m->prepared) {
        rc = launch_prep(a, st);
        if (rc) return rc;
    }
    return launch_fwd<0>(a, m, st);
}

extern "C" int dvgo_mlp_forward_gather(const dvgo_color_mlp *m, int32_t n_rays, const int32_t *ray_offsets,
                                       const float *dirs, int64_t n_samples, const dvgo_grid *feat_grid,
                                       const float *xyz, float *feat_out, float *rgb, void *ws, size_t ws_bytes,
                                       void *stream) {
    MlpArgs a;
    int rc = setup(m, n_rays, ray_offsets, dirs, n_samples, nullptr, ws, ws_bytes, false, a, false);
    if (rc) return rc;
    rc = make_dev_grid(feat_grid, "feature grid", &a.fg, false);
    if (rc) return rc;
    if (feat_grid->channels != m->in_feat)
        return set_error(DVGO_ERR_SHAPE, "feature grid channels (%d) != in_feat (%d)", feat_grid->channels, m->in_feat);
    if ((m->in_feat & 3) || (feat_grid->ch_stride & 3) || ((uintptr_t)feat_grid->data & 15) ||
        ((uintptr_t)feat_out & 15))
        return set_error(DVGO_ERR_UNSUPPORTED,
                         "the fused gather needs in_feat and ch_stride multiples of 4 and 16-byte aligned data and "
                         "feat_out");
    if (n_samples == 0) return DVGO_OK;
    if (!rgb || !xyz) return set_error(DVGO_ERR_NULL, "rgb or xyz is NULL");
    a.rgb = rgb;
    a.xyz = xyz;
    a.feat_out = feat_out;
    hipStream_t st = (hipStream_t)stream;
    if (!m->prepared) {
        rc = launch_prep(a, st);
        if (rc) return rc;
    }
    return a.fg.warp ? launch_fwd<2>(a, m, st) : launch_fwd<1>(a, m, st);
}

namespace {

int launch_reduce(const MlpArgs &a, hipStream_t st) {
    hipLaunchKernelGGL(mlp_reduce_kernel, dim3((a.n_params + 63) / 64), dim3(RED_THREADS), 0, st, a);
    return check_hip(hipGetLastError(), "mlp_reduce_kernel launch");
}

int mlp_backward_impl(const dvgo_color_mlp *m, int32_t n_rays, const int32_t *ray_offsets, const float *dirs,
                      int64_t n_samples, const float *feat, const float *grad_rgb, float *grad_feat, void *ws,
                      size_t ws_bytes, void *stream, bool reduce) {
    MlpArgs a;
    int rc = setup(m, n_rays, ray_offsets, dirs, n_samples, feat, ws, ws_bytes, true, a);
    if (rc) return rc;
    if (n_samples == 0) return DVGO_OK;
    if (!grad_rgb || !grad_feat) return set_error(DVGO_ERR_NULL, "grad_rgb or grad_feat is NULL");
    a.grad_rgb = grad_rgb;
    a.grad_feat = grad_feat;
    hipStream_t st = (hipStream_t)stream;
    if (!m->prepared) {
        rc = launch_prep(a, st);
        if (rc) return rc;
    }
    const bool vec = a.feat_vec && ((uintptr_t)grad_feat & 15) == 0;
    const dim3 grid(a.nblocks), block(BWD_THREADS);
    if (m->precision == DVGO_MLP_F16) {
        if (vec)
            hipLaunchKernelGGL((mlp_bwd_kernel<false, true>), grid, block, 0, st, a);
        else
            hipLaunchKernelGGL((mlp_bwd_kernel<false, false>), grid, block, 0, st, a);
    } else if (vec) {
        hipLaunchKernelGGL((mlp_bwd_kernel<true, true>), grid, block, 0, st, a);
    } else {
        hipLaunchKernelGGL((mlp_bwd_kernel<true, false>), grid, block, 0, st, a);
    }
    rc = check_hip(hipGetLastError(), "mlp_bwd_kernel launch");
    if (rc || !reduce) return rc;
    return launch_reduce(a, st);
}

}  // namespace

extern "C" int dvgo_mlp_backward(const dvgo_color_mlp *m, int32_t n_rays, const int32_t *ray_offsets,
                                 const float *dirs, int64_t n_samples, const float *feat, const float *grad_rgb,
                                 float *grad_feat, void *ws, size_t ws_bytes, void *stream) {
    return mlp_backward_impl(m, n_rays, ray_offsets, dirs, n_samples, feat, grad_rgb, grad_feat, ws, ws_bytes,
                             stream, true);
}

extern "C" int dvgo_mlp_backward_partials(const dvgo_color_mlp *m, int32_t n_rays, const int32_t *ray_offsets,
                                          const float *dirs, int64_t n_samples, const float *feat,
                                          const float *grad_rgb, float *grad_feat, void *ws, size_t ws_bytes,
                                          void *stream) {
    return mlp_backward_impl(m, n_rays, ray_offsets, dirs, n_samples, feat, grad_rgb, grad_feat, ws, ws_bytes,
                             stream, false);
}

extern "C" int dvgo_mlp_reduce_grads(const dvgo_color_mlp *m, int32_t n_rays, int64_t n_samples, void *ws,
                                     size_t ws_bytes, void *stream) {
    int rc = check_mlp(m, true);
    if (rc) return rc;
    if (n_rays < 0 || n_samples < 0) return set_error(DVGO_ERR_SHAPE, "negative n_rays or n_samples");
    if (n_samples >= ((int64_t)1 << 31) / 16) return set_error(DVGO_ERR_RANGE, "n_samples too large");
    size_t off_pe, off_rb, off_tr, off_part;
    const size_t need = ws_layout(m, n_rays, n_samples, &off_pe, &off_rb, &off_tr, &off_part);
    if (!ws || ws_bytes < need) return set_error(DVGO_ERR_WORKSPACE, "workspace too small (%zu < %zu)", ws_bytes, need);
    if (((uintptr_t)ws & 255) != 0) return set_error(DVGO_ERR_SHAPE, "workspace must be 256-byte aligned");
    if (n_samples == 0) return DVGO_OK;
    MlpArgs a;
    memset(&a, 0, sizeof(a));
    a.gW1 = m->gW1; a.gb1 = m->gb1; a.gW2 = m->gW2; a.gb2 = m->gb2; a.gW3 = m->gW3; a.gb3 = m->gb3;
    a.in_feat = m->in_feat;
    a.n_freq = m->n_freq;
    a.n_in = n_in_of(m);
    a.n_params = n_params_of(m);
    a.partial = (float *)((char *)ws + off_part);
    a.nblocks = bwd_blocks(n_samples);
    return launch_reduce(a, (hipStream_t)stream);
}

"""Interval counts of the guarded resampling where its running sums are at their edges (GPU)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def sequential(prob, occ, n_base, n_extra):
    """The allotment in bin order, one running double sum per ray."""
    out = np.zeros(prob.shape, np.int32)
    for r in range(len(prob)):
        tot = 0.0
        for b in range(64):
            tot += float(prob[r, b]) if occ[r, b] else 0.0
        even = not tot > 0.0
        tot = float(occ[r].sum()) if even else tot
        s = 0.0
        for b in range(64):
            if occ[r, b]:
                lo = np.floor(n_extra * (s / tot) + 0.5)
                s += 1.0 if even else float(prob[r, b])
                out[r, b] = n_base + int(np.floor(n_extra * (s / tot) + 0.5) - lo)
    return out


@pytest.mark.parametrize("n_base,n_extra", [(4, 0), (4, 32), (1, 1), (1, 1000)])
def test_guarded_counts(n_base, n_extra):
    from paper_2206_05085_amd import ops
    rng = np.random.default_rng(n_extra)
    R = 37  # a last block with one ray
    prob = rng.random((R, 64)).astype(np.float32) ** 8
    w = np.where(rng.random((R, 64)) < 0.2, 1.0, 0.0).astype(np.float32)
    prob[1] = 0.0                      # no probability at all: equal shares
    w[2] = 0.0                         # nothing occupied
    w[3] = 1.0                         # everything occupied
    prob[4], w[4] = 0.0, 0.0
    prob[4, 40], w[4, 3] = 1.0, 1.0    # probability on unoccupied bins only
    prob[5] = 2e-38                    # a tiny total
    prob[6, ::2], w[6] = 0.0, 1.0      # occupied bins without probability
    near = np.maximum(w, np.maximum(np.pad(w, ((0, 0), (1, 0)))[:, :-1], np.pad(w, ((0, 0), (0, 1)))[:, 1:]))
    t = lambda x: torch.as_tensor(np.ascontiguousarray(x, np.float32)).cuda()
    d = rng.standard_normal((R, 3))
    tn, tf = np.full(R, 0.5), np.full(R, 2.5)
    tf[7] = tn[7]                      # misses the box
    entropy = np.zeros(R)
    entropy[8] = 9.0                   # above the threshold: plain sampling
    rays = ops.RayBatch.from_arrays(rng.standard_normal((R, 3)).astype(np.float32), d.astype(np.float32), tn.astype(np.float32),
                                    tf.astype(np.float32))
    print(f"[case] guarded counts n_base {n_base} n_extra {n_extra}", flush=True)
    offs, counts = ops.resample_guarded_offsets(rays, t(prob), t(w), t(entropy), 5.0, n_base, n_extra, 0.5)[:2]
    torch.cuda.synchronize()
    want = sequential(prob, near >= 0.5, n_base, n_extra)
    want[7], want[8] = 0, n_base
    assert np.array_equal(counts.cpu().numpy().reshape(R, 64), want)
    assert np.array_equal(offs.cpu().numpy(), np.concatenate([[0], np.cumsum(want.sum(1))]))

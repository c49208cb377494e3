"""GPU: sums whose order the results hang on.  Gram-Schmidt on a nearly singular factor magnifies the rounding of its sums
by the factor's condition number, so these kernels promise an order, and it is pinned here to the last bit."""
import numpy as np
import pytest

from paper_2506_17974_amd import binding as B
from tests import parity_utils as pu

pytestmark = pytest.mark.gpu
f32 = np.float32


def _say(*a):
    print(*a, flush=True)


def _fma(a, b, c):
    """float32 a * b + c, rounded once (the product of two floats is exact in the 64 bits of a long double)."""
    return (np.asarray(a, np.longdouble) * np.asarray(b, np.longdouble) + np.asarray(c, np.longdouble)).astype(f32)


def _butterfly(x):
    """Sum over 64 lanes, the axis before the last: partners 32, 16, .. 1 apart."""
    for off in (32, 16, 8, 4, 2, 1):
        x = (x[..., :off, :] + x[..., off:2 * off, :]).astype(f32)
    return x[..., 0, :]


def _gram_schmidt(p, threads, pairs):
    """Modified Gram-Schmidt with its sums over `threads` rows-on-lanes threads: rows t, t + threads, .. in a chain, a
    butterfly per 64 threads, then the wavefronts one after the other (or in pairs)."""
    rows, r = p.shape
    v = np.zeros((-(-rows // threads) * threads, r), f32)
    v[:rows] = p
    for j in range(r):
        w = v.reshape(-1, threads, r)
        s = np.zeros((threads, r), f32)
        for i in range(w.shape[0]):
            s = _fma(w[i][:, j:j + 1], w[i], s)
        s = _butterfly(s.reshape(-1, 64, r))
        if pairs:
            t = (s[0] + s[1]) + (s[2] + s[3])
        else:
            t = s[0]
            for x in s[1:]:
                t = t + x
        inv = f32(1) / np.sqrt(t[j]) if t[j] > np.finfo(f32).tiny else f32(0)
        q = v[:, j] * inv
        v[:, j + 1:] = _fma(-(t[j + 1:] * inv), q[:, None], v[:, j + 1:])
        v[:, j] = q
    return v[:rows]


# first and last height of every form with columns on lanes
HEIGHTS = [(3, (40, 512, 513, 1024, 1025, 1792)), (7, (256, 257, 513, 1025, 1792)), (16, (128, 129, 257, 512, 513, 1025, 1792)),
           (20, (64, 65, 129, 257, 512, 513, 1024, 1025, 1792)), (50, (64, 65, 129, 257, 512, 513, 1024))]


@pytest.mark.parametrize("rank,rows", [(r, n) for r, heights in HEIGHTS for n in heights])
def test_gram_schmidt_sums_in_the_order_of_rows_on_lanes(rank, rows):
    _say("case: order of sums", rank, rows)
    rng = np.random.default_rng(rank * 7919 + rows)
    layers, W = [(rows, 200), (rank, 300)], 2          # (the second one's factor is square: its last columns are mostly rounding)
    comp = B.Compressor(B.layer_list(layers, ()), rank, 8, 8, W)
    for l, (n, c) in enumerate(layers):
        comp.set_q(l, rng.standard_normal((c, min(rank, n, c))).astype(f32))
    comp.compress(B.PHASE_P, pu.to_device([[(rng.standard_normal(s) * 1e-3).astype(f32) for s in layers] for _ in range(W)]))
    assert comp.launched_kernel(B.KERNEL_ORTH).startswith("orth_col")
    for l in range(len(layers)):
        for w in range(W):
            want = _gram_schmidt(comp.get_factor(B.FACTOR_P_PRE, l, w), 256, rank > 8 and rows > 512)
            assert np.array_equal(comp.get_factor(B.FACTOR_P_ORTH, l, w), want), (l, w)
    comp.close()


@pytest.mark.parametrize("rank,rows", [(3, 1793), (3, 2048), (3, 2049), (3, 4096), (3, 4097), (3, 8193), (3, 11264), (8, 1793), (8, 2049), (8, 4096)])
def test_gram_schmidt_sums_of_many_tall_factors(rank, rows):
    """Enough (layer, worker) pairs that each is left to one workgroup."""
    import torch
    _say("case: order of sums, many factors", rank, rows)
    rng = np.random.default_rng(rank * 7919 + rows)
    layers, W = [(rows, 12)] * 64, 2
    comp = B.Compressor(B.layer_list(layers, ()), rank, 8, 8, W)
    for l, (n, c) in enumerate(layers):
        comp.set_q(l, rng.standard_normal((c, min(rank, n, c))).astype(f32))
    G = [(rng.standard_normal(s) * 1e-3).astype(f32) for s in layers[:4]]
    D = [torch.from_numpy(g).cuda() for g in G]
    comp.compress(B.PHASE_P, [[D[(l + w) % 4] for l in range(len(layers))] for w in range(W)])
    assert comp.launched_kernel(B.KERNEL_ORTH).startswith("orth_col")
    for l, w in ((0, 0), (63, 1)):
        want = _gram_schmidt(comp.get_factor(B.FACTOR_P_PRE, l, w), 256 if rows <= 2048 else 1024, False)
        assert np.array_equal(comp.get_factor(B.FACTOR_P_ORTH, l, w), want), (l, w)
    comp.close()

"""GPU parity at the edges of the kernels' tiles: row widths around multiples of four, 64 and 256, widths below four
columns, heights around multiples of 8 and 32, ranks below their register pad, and the G-hat / parameter outputs'
neighbours in memory.  Needs a real MI355X."""
import zlib

import numpy as np
import pytest

from paper_2506_17974_amd import binding as B
from tests import parity_utils as pu

pytestmark = pytest.mark.gpu
f32 = np.float32


def _say(*a):
    print(*a, flush=True)


# (factors at least twice as tall as wide, or one column: Gram-Schmidt in 32 bits is off by about 6e-8 times the condition
# number of its input, which for a square normal matrix can be hundreds; the staged check's bar is for well-conditioned ones)
WIDTHS = [
    [(9, 1), (8, 2), (7, 3), (33, 4), (16, 5), (31, 7)],
    [(101, 255), (103, 257), (130, 259), (1, 6), (128, 254)],
    [(105, 1025), (103, 1283), (135, 1026)],
    [(129, 63), (130, 65), (161, 129), (136, 513), (1, 515)],
]


@pytest.mark.parametrize("rank,bits,W", [(1, 8, 2), (3, 8, 3), (4, 4, 2), (7, 8, 2), (8, 0, 2), (12, 8, 2), (20, 8, 3), (32, 8, 1), (50, 8, 2)])
@pytest.mark.parametrize("layers", WIDTHS, ids=lambda ls: "+".join("%dx%d" % s for s in ls))
def test_ragged_shapes(layers, rank, bits, W):
    """Two staged iterations against the oracle, then deferred and eager schedules bit for bit, with sentinels behind
    every output (rows of any width are written up to their last element and not one further)."""
    import torch
    _say("case: ragged", layers, rank, bits, W)
    rng = np.random.default_rng(zlib.crc32(str((layers, rank, bits, W)).encode()) % 1000)
    ll = B.layer_list(layers, ())
    ml = list(range(len(layers)))
    Q0 = [rng.standard_normal((c, min(rank, r, c))).astype(f32) for r, c in layers]
    Gs = [[[(rng.standard_normal(s) * 1e-3).astype(f32) for s in layers] for _ in range(W)] for _ in range(3)]
    comp = B.Compressor(ll, rank, bits, bits, W)
    for l in ml:
        comp.set_q(l, Q0[l])
    E = [[np.zeros(s, f32) for s in layers] for _ in range(W)]
    Q = [q.copy() for q in Q0]
    rep = pu.StageReport()
    for t in range(2):
        E, Q = pu.staged_iteration(comp, Gs[t], pu.to_device(Gs[t]), E, Q, ml, rep)
    comp.close()
    _say("  ", rep)

    outs = []
    for flags in (0, B.FLAG_EAGER_RESIDUAL):
        comp = B.Compressor(ll, rank, bits, bits, W, 255.0, flags)
        for l in ml:
            comp.set_q(l, Q0[l])
        bufs = [torch.full((r * c + 8,), 7.0, device="cuda") for r, c in layers]
        views = [b[:r * c].view(r, c) for b, (r, c) in zip(bufs, layers)]
        got = []
        for t in range(3):
            comp.step(pu.to_device(Gs[t]), views)
            torch.cuda.synchronize()
            got += [v.cpu().numpy().copy() for v in views]
            assert all(bool((b[-8:] == 7.0).all()) for b in bufs)
        got += [comp.get_state(l, w)[0] for l in ml for w in range(W)]
        before = [v.clone() for v in views]
        comp.step_update(pu.to_device(Gs[0]), views, 0.5)
        torch.cuda.synchronize()
        assert all(bool((b[-8:] == 7.0).all()) for b in bufs)
        got += [(v - w).cpu().numpy() for v, w in zip(views, before)]
        outs.append(got)
        comp.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("rank", [3, 7, 20])
def test_ragged_bf16_gradients(rank):
    """Rows of bfloat16 gradients that start at any even address give what the same values in float32 give."""
    import torch
    _say("case: ragged bfloat16", rank)
    layers, W = WIDTHS[1] + WIDTHS[3], 2
    rng = np.random.default_rng(rank)
    ll = B.layer_list(layers, (33,))
    shapes = layers + [(33,)]
    g16 = [[torch.from_numpy((rng.standard_normal(s) * 1e-3).astype(f32)).cuda().bfloat16() for s in shapes] for _ in range(W)]
    res = []
    for flags, g in ((B.FLAG_BF16_GRADIENTS, g16), (0, [[t.float() for t in gw] for gw in g16])):
        comp = B.Compressor(ll, rank, 8, 8, W, 255.0, flags)
        q = np.random.default_rng(1)
        for l, (r, c) in enumerate(layers):
            comp.set_q(l, q.standard_normal((c, min(rank, r, c))).astype(f32))
        out = [torch.zeros(s, device="cuda") for s in shapes]
        for _ in range(2):
            comp.step(g, out)
        torch.cuda.synchronize()
        res.append([t.cpu().numpy() for t in out])
        comp.close()
    for a, b in zip(*res):
        assert np.array_equal(a, b)


# heights at the edges of the one-workgroup Gram-Schmidt's forms (rows per lane x wavefronts x groups of rows), and the
# first heights beyond them
ORTH = [(3, (33, 512, 513, 1025)), (8, (257, 512, 1024)), (12, (128, 129, 513)), (16, (256, 1025)),
        (20, (64, 65, 1024)), (32, (129, 512, 513, 1500)), (50, (128, 257)), (64, (256, 513, 1024, 1025, 1500))]


@pytest.mark.parametrize("rank,rows", [(r, n) for r, heights in ORTH for n in heights])
def test_gram_schmidt_heights(rank, rows):
    _say("case: Gram-Schmidt", rank, rows)
    rng = np.random.default_rng(rank * 7919 + rows)
    layers, W = [(rows, 140), (2 * rank + 1, 160)], 2
    comp = B.Compressor(B.layer_list(layers, ()), rank, 8, 8, W)
    Q = [rng.standard_normal((c, min(rank, r, c))).astype(f32) for r, c in layers]
    for l, q in enumerate(Q):
        comp.set_q(l, q)
    E = [[np.zeros(s, f32) for s in layers] for _ in range(W)]
    rep = pu.StageReport()
    G = [[(rng.standard_normal(s) * 1e-3).astype(f32) for s in layers] for _ in range(W)]
    pu.staged_iteration(comp, G, pu.to_device(G), E, Q, [0, 1], rep)
    _say("  ", comp.launched_kernel(B.KERNEL_ORTH), rep)
    assert comp.launched_kernel(B.KERNEL_ORTH).startswith("orth_chol" if rank > 32 and rows > 1024 else "orth_col")
    comp.close()


@pytest.mark.parametrize("alpha", [1e-3, 0.0625, 1.0, 255.0, 1e6])
@pytest.mark.parametrize("scale", [1e-3, 3e-20, 1e17])      # (squares of factor columns stay in the range of floats: 1e-35 .. 1e38)
def test_quantiser_ranges(alpha, scale):
    """Codes on both sides of the quantiser's fast form: estimates further than a level away (small alpha) and factors
    whose absmax is far from one, where a reciprocal or a remainder could leave the normal range (Q_w carries the
    gradients' scale; P_w is orthonormal)."""
    _say("case: quantiser", alpha, scale)
    rng = np.random.default_rng(17)
    layers, W, rank = [(96, 130), (64, 27)], 3, 5
    for bits in (8, 3):
        comp = B.Compressor(B.layer_list(layers, ()), rank, bits, bits, W, alpha)
        Q = [rng.standard_normal((c, rank)).astype(f32) for r, c in layers]
        for l, q in enumerate(Q):
            comp.set_q(l, q)
        G = [[(rng.standard_normal(s) * scale).astype(f32) for s in layers] for _ in range(W)]
        comp.step(pu.to_device(G))
        comp.synchronize()
        for phase, factor in ((B.PHASE_P, B.FACTOR_P_ORTH), (B.PHASE_Q, B.FACTOR_Q_W)):
            for l in range(len(layers)):
                for w in range(W):
                    x = comp.get_factor(factor, l, w)
                    k, s, sc = comp.get_packet(phase, l, w)
                    assert sc == np.abs(x).max() and sc > 0
                    u = (np.abs(x) / sc).astype(f32)                     # correctly rounded, as the device's
                    lv = (1 << bits) - 1
                    thr = (np.expm1((np.arange(lv) + 0.5) / lv * np.log1p(float(f32(alpha)))) / float(f32(alpha))).astype(f32)
                    want = np.searchsorted(thr, u, side="right")         # thresholds <= u
                    assert np.array_equal(k, want), np.abs(k.astype(int) - want).max()
                    assert np.array_equal(s.astype(bool), (x < 0) & (want > 0))
        comp.close()


@pytest.mark.parametrize("rank,bits,W", [(20, 8, 2), (32, 0, 2)])
def test_rounds_of_256_columns(rank, bits, W):
    """Sweep 0 at rank pad 32 goes by rounds of 32 rows x 256 columns: one and several whole rounds, a partial one behind them and
    alone, one to three rows more or less than a round has, more than one column segment."""
    test_ragged_shapes([(96, 256), (65, 512), (95, 768), (97, 300), (66, 1028), (128, 2305), (161, 64)], rank, bits, W)


@pytest.mark.parametrize("rank,bits,W", [(12, 8, 2), (16, 0, 2)])
def test_rounds_of_256_columns_at_rank_pad_16(rank, bits, W):
    """The same rounds at rank pad 16, where a wavefront's 64 columns are one sum."""
    test_ragged_shapes([(96, 256), (65, 512), (95, 768), (97, 300), (66, 1028), (128, 2305), (161, 64)], rank, bits, W)


NARROW = [(64, 64), (33, 100), (96, 252), (31, 255), (70, 68), (32, 130), (65, 192), (37, 77), (128, 4), (61, 129), (3, 253), (40, 40)]


@pytest.mark.parametrize("rank,bits,W", [(12, 8, 2), (16, 0, 3), (20, 8, 2), (32, 0, 3)])
def test_layers_narrower_than_a_round(rank, bits, W):
    """Rank pads 16 and 32: the rows of an item of fewer than 256 columns are moved as one run of memory, rows of any width and
    number, the last items' sizes a multiple of four and not."""
    test_ragged_shapes(NARROW, rank, bits, W)


TAILS = [(96, 257), (64, 258), (65, 300), (32, 511), (33, 770), (70, 2305), (128, 320), (31, 600), (64, 512)]


@pytest.mark.parametrize("layers", [NARROW, TAILS])
@pytest.mark.parametrize("rank", [12, 20])
def test_bfloat16_gradients_of_narrow_layers_and_partial_rounds(rank, layers):
    """Items narrower than a round, and partial rounds behind whole ones, in bfloat16: the bits that the same values give as float32,
    in first and later iterations."""
    import torch
    _say("case: bfloat16 against float32", rank, layers)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rank)
    W = 2
    Q0 = [torch.randn((c, min(rank, n, c)), generator=gen, device="cuda").cpu().numpy() for n, c in layers]
    Gs = [[[(torch.randn(s, generator=gen, device="cuda") * 1e-3).to(torch.bfloat16) for s in layers] for _ in range(W)] for _ in range(3)]
    got = []
    for flags in (0, B.FLAG_BF16_GRADIENTS):
        comp = B.Compressor(B.layer_list(layers, ()), rank, 8, 8, W, 255.0, flags)
        for l, q in enumerate(Q0):
            comp.set_q(l, q)
        out, res = [torch.zeros(s, device="cuda") for s in layers], []
        for G in Gs:
            g = G if flags else [[x.float() for x in w] for w in G]
            comp.step(g, out)
            comp.synchronize()
            res += [o.clone() for o in out]
        comp.close()
        got.append(res)
    for a, b in zip(*got):
        assert torch.isfinite(a).all() and torch.equal(a, b)

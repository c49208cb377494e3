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


def _gram_schmidt_slices(p, single):
    """The same over slices of 256 rows: products, a butterfly per 64 of them, four wavefronts in pairs, the slices one after the other.
    With one column in all, a product meets that of the row 32 further on before it is rounded."""
    rows, r = p.shape
    n = -(-rows // 256)
    v = np.zeros((n * 256, r), f32)
    v[:rows] = p
    for j in range(r):
        s = (v[:, j:j + 1] * v).reshape(-1, 64, r)
        if single:
            low = v.reshape(-1, 64, 1)[:, :32]
            s = np.concatenate([_fma(low, low, s[:, 32:]), np.zeros_like(low)], 1)
        s = _butterfly(s).reshape(n, 4, r)
        t = np.zeros(r, f32)
        for x in (s[:, 0] + s[:, 1]) + (s[:, 2] + s[:, 3]):
            t = t + x
        inv = f32(1) / np.sqrt(t[j]) if t[j] > np.finfo(f32).tiny else f32(0)
        q = v[:, j] * inv
        v[:, j + 1:] = _fma(-(t[j + 1:] * inv), q[:, None], v[:, j + 1:])
        v[:, j] = q
    return v[:rows]


# few tall factors at rank pads 1 to 4: the sums of slices, by one workgroup each up to the height that it holds, by the slices
# beyond (or where a bound of their waits is set), in one launch and in several
@pytest.mark.parametrize("rank,rows", [(1, 1793), (1, 4097), (1, 11264), (2, 2049), (2, 8200), (3, 1793), (3, 4097), (3, 8191), (3, 11264), (4, 2048), (4, 8191), (4, 8192),
                                       (1, 11265), (2, 11265), (2, 16384), (3, 11265)])
def test_gram_schmidt_sums_of_few_tall_factors(monkeypatch, rank, rows):
    _say("case: order of sums, few tall factors", rank, rows)
    rng = np.random.default_rng(rank * 7919 + rows)
    layers, W = [(rows, 1100), (40, 12), (rows - 300, 2)], 2
    Q = [rng.standard_normal((c, min(rank, n, c))).astype(f32) for n, c in layers]
    G = pu.to_device([[(rng.standard_normal(s) * 1e-3).astype(f32) for s in layers] for _ in range(W)])
    for flags, polls in ((0, ""), (B.FLAG_NO_COOPERATIVE_LAUNCH, ""), (0, str(1 << 20))):
        monkeypatch.setenv("LQSGD_TABLE_POLLS", polls)
        comp = B.Compressor(B.layer_list(layers, ()), rank, 8, 8, W, 255.0, flags)
        for l, q in enumerate(Q):
            comp.set_q(l, q)
        comp.compress(B.PHASE_P, G)
        name = "orth_tall" if rows <= 11264 and not polls else "orth_wide" if flags else "orth_coop"
        assert comp.launched_kernel(B.KERNEL_ORTH).startswith(name)
        for l in range(len(layers)):
            for w in range(W):
                want = _gram_schmidt_slices(comp.get_factor(B.FACTOR_P_PRE, l, w), rank == 1)
                assert np.array_equal(comp.get_factor(B.FACTOR_P_ORTH, l, w), want), (l, w, flags, polls)
        comp.close()


# in place on the aggregate (whose padded copy the sweeps then read), and on caller-held state
@pytest.mark.parametrize("rank", [1, 2, 3])
def test_gram_schmidt_of_a_tall_aggregate(rank):
    import torch
    _say("case: tall aggregate", rank)
    layers, W = [(2500, 300), (40, 12), (1800, 2)], 3
    rng = np.random.default_rng(rank)
    Q = [rng.standard_normal((c, min(rank, n, c))).astype(f32) for n, c in layers]
    G = pu.to_device([[(rng.standard_normal(s) * 1e-3).astype(f32) for s in layers] for _ in range(W)])
    comp = B.Compressor(B.layer_list(layers, ()), rank, 0, 0, W, 255.0, B.FLAG_AGGREGATE_FIRST)
    for l, q in enumerate(Q):
        comp.set_q(l, q)
    out = [torch.zeros(s, device="cuda") for s in layers]
    comp.step(G, out)
    assert comp.launched_kernel(B.KERNEL_ORTH).startswith("orth_tall")
    for l in range(len(layers)):
        p, q = comp.get_factor(B.FACTOR_P_BAR, l), comp.get_factor(B.FACTOR_Q_BAR, l).astype(np.float64)
        assert np.array_equal(p, _gram_schmidt_slices(comp.get_factor(B.FACTOR_P_MEAN, l), rank == 1)), l
        mean = sum(g[l].cpu().numpy().astype(np.float64) for g in G) / W
        assert pu.rel_fro(q, mean.T @ p.astype(np.float64)) < pu.FP_TOL
        assert pu.rel_fro(out[l].cpu().numpy(), p.astype(np.float64) @ q.T) < pu.FP_TOL
    comp.close()
    layers_c = B.layer_list(layers, ())
    info = B.plan_query(layers_c, rank, 0, 0, W, 255.0, B.FLAG_AGGREGATE_FIRST)
    residual = torch.zeros((W, info.residual_stride), device="cuda")
    warm = torch.zeros(info.warm_q_floats, device="cuda")
    at = 0
    for q in Q:
        warm[at:at + q.size].copy_(torch.from_numpy(q).reshape(-1))
        at += -(-q.size // 64) * 64
    same = [torch.zeros(s, device="cuda") for s in layers]
    B.step_static(layers_c, rank, 0, 0, W, 255.0, B.FLAG_AGGREGATE_FIRST, G, residual, warm, same)
    torch.cuda.synchronize()
    for x, y in zip(out, same):
        assert torch.equal(x, y)


# the same beside layers of many columns: planes of 2^17 rows together by one workgroup, of more by the slices
@pytest.mark.parametrize("rank,rows,cols,name", [(1, 2048, 65536, "orth_tall"), (1, 2048, 65537, "orth_coop"), (4, 4097, 32000, "orth_coop"),
                                                 (3, 4000, 32768, "orth_tall")])
def test_gram_schmidt_of_many_planes(rank, rows, cols, name):
    import torch
    _say("case: order of sums, many planes", rank, rows, cols)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows)
    layers = [(rows, cols), (70, 30)]
    comp = B.Compressor(B.layer_list(layers, ()), rank, 8, 8, 1)
    for l, (n, c) in enumerate(layers):
        comp.set_q(l, np.random.default_rng(l).standard_normal((c, rank)).astype(f32))
    comp.compress(B.PHASE_P, [[torch.randn(s, generator=gen, device="cuda") * 1e-3 for s in layers]])
    assert comp.launched_kernel(B.KERNEL_ORTH).startswith(name)
    for l in range(len(layers)):
        want = _gram_schmidt_slices(comp.get_factor(B.FACTOR_P_PRE, l, 0), rank == 1)
        assert np.array_equal(comp.get_factor(B.FACTOR_P_ORTH, l, 0), want), l
    comp.close()


# more factors than CUs (a workgroup each then has fewer wavefronts, or columns on lanes), odd ranks, which leave a wavefront's
# block of columns half empty, and layers narrower than the rank beside them
@pytest.mark.parametrize("rank,rows", [(7, 500), (8, 1500), (9, 128), (13, 256), (15, 300), (16, 1000), (11, 1500), (17, 64), (31, 65),
                                       (25, 400), (33, 50), (64, 64), (41, 128), (63, 300), (49, 1000)])
def test_gram_schmidt_sums_of_more_factors_than_cus(rank, rows):
    import torch
    _say("case: order of sums, more factors than CUs", rank, rows)
    rng = np.random.default_rng(rank * 7919 + rows)
    layers, W = [(rows, rank + 8)] * 34 + [(rows, 1), (rows - 1, 3), (5, rank + 8)], 8
    comp = B.Compressor(B.layer_list(layers, ()), rank, 8, 8, W)
    for l, (n, c) in enumerate(layers):
        comp.set_q(l, rng.standard_normal((c, min(rank, n, c))).astype(f32))
    D = [torch.from_numpy((rng.standard_normal(rows * (rank + 8)) * 1e-3).astype(f32)).cuda() for _ in range(3)]
    comp.compress(B.PHASE_P, [[D[(l + w) % 3][:n * c].view(n, c) for l, (n, c) in enumerate(layers)] for w in range(W)])
    assert comp.launched_kernel(B.KERNEL_ORTH).startswith("orth_col")
    for l, w in ((0, 0), (20, 3), (33, 7), (34, 1), (35, 2), (36, 5)):
        want = _gram_schmidt(comp.get_factor(B.FACTOR_P_PRE, l, w), 256, rank > 8 and rows > 512)
        assert np.array_equal(comp.get_factor(B.FACTOR_P_ORTH, l, w), want), (l, w)
    comp.close()


@pytest.mark.parametrize("rank", [2, 4, 7, 20, 50])
def test_gram_schmidt_of_a_column_whose_squared_norm_overflows(rank):
    """Finite values whose squares leave the range of floats: the column becomes zero and the others, whose products with it
    are finite, stay what they are without it.  Nothing of it reaches G-hat or the residual."""
    import torch
    _say("case: overflowing column", rank)
    rng = np.random.default_rng(rank)
    layers, W = [(300, 210)], 2
    comp = B.Compressor(B.layer_list(layers, ()), rank, 0, 0, W)
    q = rng.standard_normal((210, rank)).astype(f32)
    q[:, rank // 2] *= f32(1e22)
    comp.set_q(0, q)
    G = [[(rng.standard_normal(s) * 1e-3).astype(f32) for s in layers] for _ in range(W)]
    out = [torch.zeros(s, device="cuda") for s in layers]
    comp.step(pu.to_device(G), out)
    for w in range(W):
        pre, got = comp.get_factor(B.FACTOR_P_PRE, 0, w), comp.get_factor(B.FACTOR_P_ORTH, 0, w)
        assert np.isfinite(pre).all() and np.abs(pre).max() > 1e19
        assert not got[:, rank // 2].any() and np.isfinite(got).all()
        with np.errstate(over="ignore"):
            want = _gram_schmidt(pre, 256, False)
        assert pu.rel_fro(got, want) < pu.FP_TOL if rank <= 2 else np.array_equal(got, want)
        assert np.isfinite(comp.get_state(0, w)[0]).all()
    assert bool(torch.isfinite(out[0]).all())
    comp.close()


@pytest.mark.parametrize("rank", [1, 2, 3, 7, 8, 12, 20, 32, 50])
@pytest.mark.parametrize("eager", [False, True])
def test_narrow_rows_sums_and_reconstructions(rank, eager):
    """Rows of at most 64 columns, no multiple of four of them: products added by a butterfly over the columns, the
    reconstruction in the order of the ranks, in a first and in a second iteration (whose residual is the deferred or the
    finished one)."""
    import torch
    _say("case: narrow rows", rank, eager)
    rng = np.random.default_rng(rank)
    layers, W = [(70, 27), (64, 63), (33, 1), (41, 2), (9, 3), (65, 5), (100, 33), (300, 64), (64, 200)], 2
    comp = B.Compressor(B.layer_list(layers, ()), rank, 8, 8, W, 255.0, B.FLAG_EAGER_RESIDUAL if eager else 0)
    Q = [rng.standard_normal((c, min(rank, n, c))).astype(f32) for n, c in layers]
    for l, q in enumerate(Q):
        comp.set_q(l, q)
    out = [torch.zeros(s, device="cuda") for s in layers]
    E = [[np.zeros(s, f32) for s in layers] for _ in range(W)]
    for _ in range(2):
        G = [[(rng.standard_normal(s) * 1e-3).astype(f32) for s in layers] for _ in range(W)]
        comp.step(pu.to_device(G), out)
        for l, (n, c) in enumerate(layers):
            if c % 4 == 0 or c > 64:
                continue
            k = Q[l].shape[1]
            P, Qn = comp.get_factor(B.FACTOR_P_BAR, l), comp.get_factor(B.FACTOR_Q_BAR, l)
            hat = np.zeros((n, c), f32)
            for j in range(k):
                hat = _fma(P[:, j:j + 1], Qn[:, j], hat)
            assert np.array_equal(out[l].cpu().numpy(), hat), (l, "G-hat")
            for w in range(W):
                M = G[w][l] + E[w][l]
                lanes = np.zeros((n, 64, k), f32)
                lanes[:, :c] = M[:, :, None] * Q[l][None]
                assert np.array_equal(comp.get_factor(B.FACTOR_P_PRE, l, w), _butterfly(lanes)), (l, w)
                E[w][l] = M - hat
            Q[l] = Qn
    for l, (n, c) in enumerate(layers):
        if c % 4 and c <= 64:
            for w in range(W):
                assert np.array_equal(comp.get_state(l, w)[0], E[w][l]), (l, w)
    comp.close()


@pytest.mark.parametrize("rank", [1, 2, 7, 12])
def test_tall_layers_of_few_columns(rank):
    """Several row blocks and several groups of rows per item, one column per lane and four: two staged iterations against
    the oracle, deferred and finished residuals bit for bit."""
    import torch
    _say("case: tall layers of few columns", rank)
    rng = np.random.default_rng(rank)
    layers, W = [(5003, 21), (2600, 7), (3001, 16), (40000, 3), (9000, 9), (1100, 61)], 2
    ll, ml = B.layer_list(layers, ()), list(range(len(layers)))
    Q0 = [rng.standard_normal((c, min(rank, n, c))).astype(f32) for n, c in layers]
    Gs = [[[(rng.standard_normal(s) * 1e-3).astype(f32) for s in layers] for _ in range(W)] for _ in range(3)]
    comp = B.Compressor(ll, rank, 8, 8, W)
    for l in ml:
        comp.set_q(l, Q0[l])
    E, Q, rep = [[np.zeros(s, f32) for s in layers] for _ in range(W)], [q.copy() for q in Q0], pu.StageReport()
    for t in range(2):
        E, Q = pu.staged_iteration(comp, Gs[t], pu.to_device(Gs[t]), E, Q, ml, rep)
    comp.close()
    _say("  ", rep)
    outs = []
    for flags in (0, B.FLAG_EAGER_RESIDUAL):
        comp = B.Compressor(ll, rank, 8, 8, W, 255.0, flags)
        for l in ml:
            comp.set_q(l, Q0[l])
        got, out = [], [torch.zeros(s, device="cuda") for s in layers]
        for t in range(3):
            comp.step(pu.to_device(Gs[t]), out)
            got += [v.cpu().numpy() for v in out]
        outs.append(got + [comp.get_state(l, w)[0] for l in ml for w in range(W)])
        comp.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("rank", [3, 20])
def test_factors_set_layer_by_layer(rank):
    """Q and P-bar set for single layers, in any order, in a list whose 1-D tensors shift the matrix layers: the sweeps read
    what was set (ranks below their pad: from copies)."""
    import torch
    _say("case: factors set layer by layer", rank)
    rng = np.random.default_rng(rank)
    layers, W = [(7, 1, B.LAYER_VECTOR), (200, 100, 0), (33, 1, B.LAYER_VECTOR), (64, 27, 0), (300, 130, 0)], 2
    ml = [1, 3, 4]
    comp = B.Compressor(layers, rank, 0, 0, W)
    G = [[(rng.standard_normal((n, c)[:1 if f else 2]) * 1e-3).astype(f32) for n, c, f in layers] for _ in range(W)]
    for rep in range(2):
        Q = {l: rng.standard_normal((layers[l][1], min(rank, *layers[l][:2]))).astype(f32) for l in ml}
        for l in (4, 1, 3):
            comp.set_q(l, Q[l])
        E = {(l, w): comp.get_state(l, w)[0] for l in ml for w in range(W)}
        comp.compress(B.PHASE_P, pu.to_device(G))
        for l in ml:
            for w in range(W):
                assert pu.rel_fro(comp.get_factor(B.FACTOR_P_PRE, l, w), (G[w][l] + E[l, w]) @ Q[l]) < pu.FP_TOL
        comp.decompress(B.PHASE_P)
        P = {l: rng.standard_normal((layers[l][0], Q[l].shape[1])).astype(f32) for l in ml}
        for l in (3, 4, 1):
            comp.set_factor(B.FACTOR_P_BAR, l, P[l])
        comp.compress(B.PHASE_Q)
        for l in ml:
            for w in range(W):
                assert pu.rel_fro(comp.get_factor(B.FACTOR_Q_W, l, w), (G[w][l] + E[l, w]).T @ P[l]) < pu.FP_TOL
        comp.decompress(B.PHASE_Q)
    comp.close()


@pytest.mark.parametrize("tensors,W", [(130, 2), (300, 7)])
def test_pointer_lists_that_change_from_step_to_step(tensors, W):
    """Other buffers in every step, in lists that go to the device in stream order and in lists (of 2100 pointers) that are
    copied after a wait, give what the same values in the same buffers give."""
    import torch
    _say("case: pointer lists", tensors, W)
    rng = np.random.default_rng(tensors)
    layers = [(16 + i % 5, 12 + i % 7) for i in range(tensors)]
    Q = [rng.standard_normal((c, 3)).astype(f32) for _, c in layers]
    G = [[[(rng.standard_normal(s) * 1e-3).astype(f32) for s in layers] for _ in range(W)] for _ in range(3)]
    outs = []
    for change in (False, True):
        comp = B.Compressor(B.layer_list(layers, ()), 3, 8, 8, W)
        for l, q in enumerate(Q):
            comp.set_q(l, q)
        bufs, out = pu.to_device(G[0]), [torch.zeros(s, device="cuda") for s in layers]
        keep, got = [bufs, out], []
        for t in range(3):
            if change:
                bufs, out = pu.to_device(G[t]), [torch.zeros(s, device="cuda") for s in layers]
                keep += [bufs, out]
            else:
                for w in range(W):
                    for b, g in zip(bufs[w], G[t][w]):
                        b.copy_(torch.from_numpy(g))
            comp.step(bufs, out)
            got.append(torch.cat([o.reshape(-1) for o in out]))
        outs.append([g.cpu().numpy() for g in got])
        comp.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("rank,layers", [(3, [(200, 100), (64, 27)]), (7, [(300, 130), (97, 515)]), (2, [(40, 60), (1, 9)])])
def test_capture_below_the_rank_pad_and_with_other_pointers(rank, layers):
    """A step of the vector sweeps with padded operand copies, recorded and replayed with eager work in between; a recording
    call with other pointers is refused, and neither the capture nor the bound list suffers."""
    import torch
    _say("case: capture", rank, layers)
    rng, W = np.random.default_rng(rank), 2
    ll = B.layer_list(layers, ())
    s = torch.cuda.Stream()
    rec, ref = B.Compressor(ll, rank, 8, 8, W, 255.0, 0, stream=s.cuda_stream), B.Compressor(ll, rank, 8, 8, W)
    for l, (n, c) in enumerate(layers):
        q = rng.standard_normal((c, min(rank, n, c))).astype(f32)
        rec.set_q(l, q)
        ref.set_q(l, q)

    def values():
        return [[(rng.standard_normal(sh) * 1e-3).astype(f32) for sh in layers] for _ in range(W)]

    buf, out, out_ref = pu.to_device(values()), [torch.zeros(sh, device="cuda") for sh in layers], [torch.zeros(sh, device="cuda") for sh in layers]
    other = pu.to_device(values())
    torch.cuda.synchronize()
    for _ in range(2):
        rec.step(buf, out)
        ref.step(buf, out_ref)
        rec.synchronize()
        ref.synchronize()
    import ctypes as C
    tab, tab_other, gt = rec.pointer_table(buf), rec.pointer_table(other), (C.c_void_p * len(layers))(*[t.data_ptr() for t in out])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        with pytest.raises(B.LqsgdError) as ei:
            rec.step_raw(tab_other, gt)
        assert ei.value.code == B.EHIP
        rec.step_raw(tab, gt)
    torch.cuda.synchronize()
    for _ in range(3):
        for b, g in zip(buf, values()):
            for x, y in zip(b, g):
                x.copy_(torch.from_numpy(y))
        torch.randn(1 << 16, device="cuda").sum()          # unrelated eager work between replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        ref.step(buf, out_ref)
        ref.synchronize()
        for a, b in zip(out, out_ref):
            assert torch.equal(a, b)
    rec.close()
    ref.close()


@pytest.mark.parametrize("rank,layers", [(2, [(300, 260), (40, 1)]), (3, [(1232, 160), (64, 224)]), (7, [(600, 130), (64, 5)]),
                                         (20, [(1000, 140), (64, 27)]), (50, [(700, 160), (64, 35)]), (50, [(1500, 60), (64, 40)]), (7, [(2600, 30)])])
@pytest.mark.parametrize("eager", [False, True])
def test_aggregate_first_below_the_rank_pad(rank, layers, eager):
    """The sweeps read the orthonormalised aggregate, from the copy that Gram-Schmidt or a launch after it has written: G-hat,
    the Q products and the residuals are those of the P-bar that the factor tap shows."""
    import torch
    _say("case: aggregate-first", rank, layers, eager)
    rng, W = np.random.default_rng(rank), 3
    comp = B.Compressor(B.layer_list(layers, ()), rank, 8, 0, W, 255.0, B.FLAG_AGGREGATE_FIRST | (B.FLAG_EAGER_RESIDUAL if eager else 0))
    for l, (n, c) in enumerate(layers):
        comp.set_q(l, rng.standard_normal((c, min(rank, n, c))).astype(f32))
    out = [torch.zeros(s, device="cuda") for s in layers]
    E = [[np.zeros(s, f32) for s in layers] for _ in range(W)]
    for _ in range(3):
        G = [[(rng.standard_normal(s) * 1e-3).astype(f32) for s in layers] for _ in range(W)]
        comp.step(pu.to_device(G), out)
        for l in range(len(layers)):
            P, Q = comp.get_factor(B.FACTOR_P_BAR, l).astype(np.float64), comp.get_factor(B.FACTOR_Q_BAR, l).astype(np.float64)
            hat = P @ Q.T
            assert pu.rel_fro(out[l].cpu().numpy(), hat) < 1e-5
            for w in range(W):
                M = G[w][l] + E[w][l]
                assert pu.rel_fro(comp.get_factor(B.FACTOR_Q_W, l, w), M.T @ P) < pu.FP_TOL
                E[w][l] = (M - hat).astype(f32)
    for l in range(len(layers)):
        for w in range(W):
            assert np.abs(comp.get_state(l, w)[0] - E[w][l]).max() <= 1e-5 * np.abs(G[w][l]).max()
    comp.close()


@pytest.mark.parametrize("rank", [1, 3, 8, 12])
def test_rows_of_any_width_in_sets_of_many_items(rank):
    """Enough work items that rows which are no multiple of four take the wide segments and chunks (small sets, as in the
    other tests, take narrower ones): a staged iteration against the oracle, deferred and finished residuals bit for bit."""
    import torch
    _say("case: many ragged layers", rank)
    rng = np.random.default_rng(rank)
    layers, W = [(72, 1283)] * 12 + [(130, 257)] * 40 + [(9, 65)] * 8, 2
    tiles = B.plan_tiles(B.layer_list(layers, ()), rank, 8, 8, W, 1)
    assert tiles[:, 5].max() == 256 and B.plan_tiles(B.layer_list(layers, ()), rank, 8, 8, W, 0)[:, 5].max() > 256
    ll, ml = B.layer_list(layers, ()), list(range(len(layers)))
    Q0 = [rng.standard_normal((c, min(rank, n, c))).astype(f32) for n, c in layers]
    Gs = [[[(rng.standard_normal(s) * 1e-3).astype(f32) for s in layers] for _ in range(W)] for _ in range(2)]
    comp = B.Compressor(ll, rank, 8, 8, W)
    for l in ml:
        comp.set_q(l, Q0[l])
    E, Q, rep = [[np.zeros(s, f32) for s in layers] for _ in range(W)], [q.copy() for q in Q0], pu.StageReport()
    for t in range(2):
        E, Q = pu.staged_iteration(comp, Gs[t], pu.to_device(Gs[t]), E, Q, ml, rep)
    comp.close()
    _say("  ", rep)
    outs = []
    for flags in (0, B.FLAG_EAGER_RESIDUAL):
        comp = B.Compressor(ll, rank, 8, 8, W, 255.0, flags)
        for l in ml:
            comp.set_q(l, Q0[l])
        got, out = [], [torch.zeros(s, device="cuda") for s in layers]
        for t in range(2):
            comp.step(pu.to_device(Gs[t]), out)
            got.append(torch.cat([v.reshape(-1) for v in out]).cpu().numpy())
        outs.append(got + [comp.get_state(l, 1)[0] for l in ml])
        comp.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("bf16", [False, True])
def test_sixty_four_row_items_add_in_the_order_of_thirty_two_row_ones(bf16):
    """Rank pad 64: sweep 0 takes items of 64 rows where there are more than 32-row ones for every CU.  The same layers alone (32
    rows) and in a long list (64 rows), heights around 32 and 64, whole and partial rounds of 256 columns: the same bits."""
    import torch
    shapes, W, rank = [(64, 300), (33, 1000), (40, 1023), (64, 256), (32, 770), (31, 700), (63, 516), (64, 61), (64, 1024)], 2, 50
    _say("case: 64-row items", shapes, bf16)
    rng = np.random.default_rng(64)
    Q0 = [rng.standard_normal((c, min(rank, n, c))).astype(f32) for n, c in shapes]
    Gs = [[[(rng.standard_normal(s) * 1e-3).astype(f32) for s in shapes] for _ in range(W)] for _ in range(3)]
    got = []
    for fill in (0, 60):
        layers = shapes + [(64, 260)] * fill
        comp = B.Compressor(B.layer_list(layers, ()), rank, 8, 8, W, 255.0, B.FLAG_BF16_GRADIENTS if bf16 else 0)
        for l, (n, c) in enumerate(layers):
            comp.set_q(l, Q0[l] if l < len(shapes) else rng.standard_normal((c, min(rank, n, c))).astype(f32))
        out = [torch.zeros(s, device="cuda") for s in layers]
        res, names = [], set()
        comp.timing_enable(True)
        for G in Gs:
            g = [[torch.from_numpy(x).cuda() for x in w] + [torch.ones(64, 260, device="cuda").normal_()] * fill for w in G]
            if bf16:
                g = [[x.to(torch.bfloat16) for x in w] for w in g]
            comp.step(g, out)
            res += [o.cpu().numpy() for o in out[:len(shapes)]]
            names.add(comp.launched_kernel(0).split("<")[0])
        res += [comp.get_state(l, w)[0] for l in range(len(shapes)) for w in range(W)]
        res += [comp.get_factor(B.FACTOR_P_PRE, l, w) for l in range(len(shapes)) for w in range(W)]
        assert names == {"mfma_pair_kernel" if fill else "mfma_sweep_kernel"}
        comp.close()
        got.append(res)
    for a, b in zip(*got):
        assert np.array_equal(a, b)


def _schedules(layers, rank, W, kernel, bf16=False, bits=8, iterations=3):
    """Deferred and eager residuals give the same bits (the eager schedule's sweeps are the ones that the staged tests hold
    against the oracle); `kernel` is what sweep 0 of the deferred one runs from its second iteration on."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rank + W)
    Q0 = [torch.randn((c, min(rank, n, c)), generator=gen, device="cuda").cpu().numpy() for n, c in layers]
    Gs = [[[(torch.randn(s, generator=gen, device="cuda") * 1e-3).to(torch.bfloat16 if bf16 else torch.float32) for s in layers]
           for _ in range(W)] for _ in range(iterations)]
    got = []
    for flags in (0, B.FLAG_EAGER_RESIDUAL):
        comp = B.Compressor(B.layer_list(layers, ()), rank, bits, bits, W, 255.0, flags | (B.FLAG_BF16_GRADIENTS if bf16 else 0))
        for l, q in enumerate(Q0):
            comp.set_q(l, q)
        out, res = [torch.full(s, 7.0, device="cuda") for s in layers], []
        for G in Gs:
            comp.step(G, out)
            res += [o.clone() for o in out]
        if not flags:
            assert comp.launched_kernel(0).startswith(kernel), comp.launched_kernel(0)
        res += [torch.from_numpy(comp.get_state(l, w)[0]) for l in range(len(layers)) for w in range(W)]
        res += [torch.from_numpy(comp.get_factor(B.FACTOR_P_PRE, l, w)) for l in range(len(layers)) for w in range(W)]
        comp.close()
        got.append(res)
    for i, (a, b) in enumerate(zip(*got)):
        assert torch.isfinite(a).all() and torch.equal(a, b), "tensor %d" % i
    return got[0]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("layers,W,kernel", [
    # 64-row items: the last one of a layer of any height, several segments, layers of one short item
    ([(161, 2305), (200, 1100), (20, 2100), (32, 300), (65, 516), (64, 61), (128, 1024), (97, 63)], 8, "mfma_pair_kernel<1"),
    # few of them: 32 rows a workgroup
    ([(161, 1305), (20, 300), (32, 512), (65, 131), (64, 61), (33, 65)], 2, "mfma_sweep_kernel<64, 1"),
])
def test_rank_pad_64_items_of_any_height(layers, W, kernel, bf16):
    _say("case: 64-row items, deferred and eager", layers, W, bf16)
    _schedules(layers, 50, W, kernel, bf16)


def test_sweep_one_row_blocks_of_any_height_at_rank_pad_64():
    """Sweep 1 at rank pad 64: row blocks of less than one group of 16 rows, of whole groups and a rest, around the 128 rows from which
    items are long, of 256 and a rest; strips without columns beside strips that share the rows of P-bar."""
    layers = [(h, 300) for h in (9, 16, 17, 31, 32, 33, 65, 100, 127, 128, 129, 144, 150, 255, 256, 257, 300, 520)] + [(80, 520), (200, 1030)]
    rank, W = 40, 20
    _say("case: row blocks of sweep 1", layers, rank, W)
    rng = np.random.default_rng(1)
    tiles = B.plan_tiles(B.layer_list(layers, ()), rank, 8, 8, W, 1)
    assert tiles[:, 3].max() == 256 and {9, 127, 128, 129, 255} <= set(tiles[:, 3].tolist())
    comp = B.Compressor(B.layer_list(layers, ()), rank, 8, 8, W)
    Q = [rng.standard_normal((c, min(rank, n, c))).astype(f32) for n, c in layers]
    ml = list(range(len(layers)))
    for l in ml:
        comp.set_q(l, Q[l])
    E = [[np.zeros(s, f32) for s in layers] for _ in range(W)]
    rep = pu.StageReport()
    G = [[(rng.standard_normal(s) * 1e-3).astype(f32) for s in layers] for _ in range(W)]
    pu.staged_iteration(comp, G, pu.to_device(G), E, Q, ml, rep, layers_to_check=ml, workers_to_check=[0, 7, 19])
    comp.close()
    _say("  ", rep)


@pytest.mark.parametrize("bits", [8, 0])
def test_sweep_zero_by_blocks_adds_like_sweep_zero_by_rounds(bits):
    """Rank pad 16: sets of many half-empty rounds go by 64-column blocks per wavefront.  The same layers beside wide ones, by
    rounds: the same bits."""
    import torch
    shapes, W, rank = [(96, 320), (70, 384), (64, 64), (33, 448), (40, 576), (128, 256), (65, 300), (31, 129), (5, 61)], 3, 13
    _say("case: blocks and rounds", shapes, bits)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    Q0 = [torch.randn((c, min(rank, n, c)), generator=gen, device="cuda").cpu().numpy() for n, c in shapes]
    Gs = [[[torch.randn(s, generator=gen, device="cuda") * 1e-3 for s in shapes] for _ in range(W)] for _ in range(3)]
    got = []
    for wide in (0, 2):
        layers = shapes + [(200, 1024)] * wide
        comp = B.Compressor(B.layer_list(layers, ()), rank, bits, bits, W)
        for l, (n, c) in enumerate(layers):
            comp.set_q(l, Q0[l] if l < len(shapes) else torch.randn((c, rank), generator=gen, device="cuda").cpu().numpy())
        out, res = [torch.zeros(s, device="cuda") for s in layers], []
        for G in Gs:
            comp.step([w + [torch.randn(200, 1024, generator=gen, device="cuda")] * wide for w in G], out)
            res += [o.clone() for o in out[:len(shapes)]]
        assert comp.launched_kernel(0).startswith("mfma_round_kernel<16, 1" if wide else "mfma_sweep_kernel<16, 1"), comp.launched_kernel(0)
        res += [torch.from_numpy(comp.get_factor(B.FACTOR_P_PRE, l, w)) for l in range(len(shapes)) for w in range(W)]
        comp.close()
        got.append(res)
    for a, b in zip(*got):
        assert torch.isfinite(a).all() and torch.equal(a, b)


def test_sweep_zero_by_blocks_in_both_schedules():
    layers = [(96, 320), (70, 384), (64, 64), (33, 448), (65, 320), (128, 64), (3, 320)]
    _say("case: blocks, deferred and eager", layers)
    _schedules(layers, 16, 3, "mfma_sweep_kernel<16, 1")


# (At most 64 rows and 1024 columns: one row block and one segment, however long the list.)
EVEN = [(64, 256), (64, 512), (32, 1024), (64, 768), (40, 700)]
UNEVEN = [(64, 320), (60, 640), (33, 1020), (25, 988), (1, 1024), (63, 300), (64, 128), (31, 255), (40, 40), (37, 77), (5, 61), (64, 572)]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("layers,first,later", [(EVEN, "sweep32", "round"), (UNEVEN, "sweep32", "sweep32"),
                                                ([(64, 320), (60, 640), (33, 300), (64, 576)], "sweep32", "sweep32"),
                                                ([(64, 320), (64, 1024)], "sweep32", "round"),
                                                ([(64, 64), (33, 100), (57, 192), (31, 129), (60, 68)], "sweep32", "sweep32")])
def test_sweep_zero_of_a_cu_an_item_adds_like_sweep_zero_by_rounds(layers, first, later, bf16):
    """Rank pad 32: lists of at most 256 items go by 32 x 32 blocks per wavefront, with the deferred residual if they are uneven.
    The same layers in a long list, by rounds: the same bits."""
    import torch
    W, rank = 3, 27
    _say("case: blocks and rounds at rank pad 32", layers, bf16)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    dt = torch.bfloat16 if bf16 else torch.float32
    Q0 = [torch.randn((c, min(rank, n, c)), generator=gen, device="cuda").cpu().numpy() for n, c in layers]
    Gs = [[[(torch.randn(s, generator=gen, device="cuda") * 1e-3).to(dt) for s in layers] for _ in range(W)] for _ in range(3)]
    more, got = (64, 512), []
    for longer in (0, 48):
        ls = layers + [more] * longer
        comp = B.Compressor(B.layer_list(ls, ()), rank, 8, 8, W, 255.0, B.FLAG_BF16_GRADIENTS if bf16 else 0)
        for l, (n, c) in enumerate(ls):
            comp.set_q(l, Q0[l] if l < len(layers) else torch.randn((c, rank), generator=gen, device="cuda").cpu().numpy())
        out, res = [torch.zeros(s, device="cuda") for s in ls], []
        fill = [(torch.randn(more, generator=gen, device="cuda") * 1e-3).to(dt) for _ in range(longer)]
        for it, G in enumerate(Gs):
            comp.step([w + fill for w in G], out)
            res += [o.clone() for o in out[:len(layers)]]
            kernel = "round" if longer else first if it == 0 else later
            assert comp.launched_kernel(0).startswith("mfma_%s_kernel<" % kernel), comp.launched_kernel(0)
        res += [torch.from_numpy(comp.get_state(l, w)[0]) for l in range(len(layers)) for w in range(W)]
        res += [torch.from_numpy(comp.get_factor(B.FACTOR_P_PRE, l, w)) for l in range(len(layers)) for w in range(W)]
        comp.close()
        got.append(res)
    for i, (a, b) in enumerate(zip(*got)):
        assert torch.isfinite(a).all() and torch.equal(a, b), "tensor %d" % i


@pytest.mark.parametrize("layers,kernel", [([(512, 320)] * 9 + [(70, 96)], "mfma_round_kernel<32, 1"),
                                           (UNEVEN + [(161, 2305)], "mfma_sweep32_kernel<1"),
                                           (UNEVEN + [(161, 2305), (3000, 512)], "mfma_round_kernel<32, 1")])
def test_sweep_zero_by_rounds_and_blocks_at_rank_pad_32_in_both_schedules(layers, kernel):
    """Also a long list whose first iterations alone go by blocks."""
    _say("case: rank pad 32, deferred and eager", layers)
    _schedules(layers, 32, 3, kernel)


# Slabs of W workers in MB (2^20 bytes): the store policy of sweep 0 turns on them and on how the elements' rows start.
@pytest.mark.parametrize("layers,rank,first,later", [
    ([(2048, 2048)] * 9, 16, "false>", "false>"),                          # 288 MB
    ([(2048, 2048)] * 11, 16, "false>", "true>"),                          # 352 MB: with the deferred residual only
    ([(2048, 2048)] * 11, 20, "false>", "true>"),
    ([(2048, 2048)] * 11, 50, "false>", "false>"),                         # rank pads 64 and 8 wait for 640 MB
    ([(2048, 2048)] * 11, 7, "false>", "false>"),
    ([(2048, 2048)] * 6 + [(2048, 2049)] * 5, 16, "false>", "true>"),      # most elements in rows of whole 64 bytes
    ([(2048, 2048)] * 5 + [(2048, 2049)] * 6, 16, "false>", "false>"),     # most not
    ([(2048, 2048)] * 12 + [(2048, 2052)] * 9, 32, "true>", "true>"),      # 672 MB
    ([(2048, 2048)] * 9 + [(2048, 2052)] * 12, 50, "false>", "false>"),
])
def test_store_policy_of_mixed_sets(layers, rank, first, later):
    """The first iteration and the later ones of the deferred schedule follow their own line; the eager schedule, which takes the
    former's throughout, gives the same bits."""
    import torch
    _say("case: store policy", len(layers), rank, first, later)
    comp = B.Compressor(B.layer_list(layers, ()), rank, 8, 8, 2)
    G = [[torch.zeros(s, device="cuda") for s in layers]] * 2
    for want in (first, later):
        comp.step(G)
        assert comp.launched_kernel(0).endswith(want), comp.launched_kernel(0)
    comp.close()
    _schedules(layers, rank, 2, "", iterations=2)


# the G-hat pass of rank pads 16 to 64 beside the eager schedule's, which takes G-hat from the residual sweep: edges of its 32 rows and
# 64 and 256 columns, rows that are no multiple of four, one column a lane (21), and sets whose items are 64 and 128 rows
GHAT_EDGES = [(1, 300), (31, 63), (32, 64), (33, 65), (97, 255), (64, 256), (70, 257), (130, 513), (40, 21), (300, 1), (65, 4)]


@pytest.mark.parametrize("update", [False, True])
@pytest.mark.parametrize("rank,layers", [(r, GHAT_EDGES) for r in (9, 16, 27, 32, 41, 64)] +
                         [(r, [(2111, 4100), (65, 130)]) for r in (12, 32, 50)] + [(r, [(4097, 8200)]) for r in (20, 64)])
def test_ghat_pass_writes_what_the_residual_sweep_subtracts(rank, layers, update):
    import torch
    _say("case: G-hat pass", rank, layers[:3], update)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rank)
    G = [[torch.randn(s, generator=gen, device="cuda") * 1e-3 for s in layers]]
    Q = [np.random.default_rng(rank).standard_normal((c, min(rank, r, c))).astype(f32) for r, c in layers]
    start = [torch.randn(s, generator=gen, device="cuda") for s in layers]
    got = []
    for flags in (0, B.FLAG_EAGER_RESIDUAL):
        comp = B.Compressor(B.layer_list(layers, ()), rank, 8, 8, 1, 255.0, flags)
        for l, q in enumerate(Q):
            comp.set_q(l, q)
        flat = torch.full((sum(t.numel() + 128 for t in start) + 64,), 7.0, device="cuda")
        out, at = [], 64
        for t in start:                          # (with untouched values around every layer's)
            out.append(flat[at:at + t.numel()].view(t.shape))
            out[-1].copy_(t)
            at += -(-t.numel() // 64) * 64 + 64
        for _ in range(2):
            comp.step_update(G, out, 0.1) if update else comp.step(G, out)
        comp.synchronize()
        if flags == 0:
            assert comp.launched_kernel(B.KERNEL_RESIDUAL).startswith("mfma_ghat_kernel")
        got.append(flat.cpu().numpy())
        comp.close()
    assert np.array_equal(got[0], got[1])


# rank pads 32 and 64: layers of one row block, whose sums and absmax sweep 1 stores itself, beside taller ones; strips of 128 columns that
# end early, ranks clipped by a layer; lists of few items and of many
SWEEP_ONE = [(5, 640), (64, 130), (63, 1), (100, 300), (128, 512), (256, 257), (300, 1025), (97, 60)]


@pytest.mark.parametrize("rank,copies,W", [(20, 1, 2), (32, 1, 1), (32, 12, 4), (33, 1, 2), (50, 1, 2), (50, 12, 4), (64, 1, 1)])
def test_sweep_one_stores_sums_and_absmax(rank, copies, W):
    import torch
    _say("case: sweep 1, sums and absmax", rank, copies, W)
    layers = SWEEP_ONE * copies
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rank + copies)
    comp = B.Compressor(B.layer_list(layers, ()), rank, 8, 8, W)
    rng = np.random.default_rng(rank)
    for l, (r, c) in enumerate(layers):
        comp.set_q(l, rng.standard_normal((c, min(rank, r, c))).astype(f32))
    G = [[torch.randn(s, generator=gen, device="cuda") * 1e-3 for s in layers] for _ in range(W)]
    comp.compress(B.PHASE_P, G)
    comp.decompress(B.PHASE_P)
    comp.compress(B.PHASE_Q)
    for l in list(range(8)) + list(range(len(layers) - 8, len(layers))):
        p = comp.get_factor(B.FACTOR_P_BAR, l).astype(np.float64)
        for w in range(W):
            q = comp.get_factor(B.FACTOR_Q_W, l, w)
            m = G[w][l].cpu().numpy().astype(np.float64)
            bound = (np.abs(m).T @ np.abs(p)) * (m.shape[0] + 2) * 2.0 ** -24          # a sum of that many terms, in any order
            assert (np.abs(q - m.T @ p) <= bound + 1e-30).all(), (l, w)
            assert comp.get_packet(B.PHASE_Q, l, w)[2] == np.abs(q).max(), (l, w)
    comp.close()


@pytest.mark.parametrize("rank,copies", [(50, 20), (50, 42), (20, 20)])
def test_matrix_layers_beside_many_vectors(rank, copies):
    """Sweep 1 of lists of up to two items a CU and more, with hundreds of 1-D tensors' workgroups in the same launch and without: the
    same bits, and the vectors' means."""
    import torch
    _say("case: sweep 1 beside vectors", rank, copies)
    layers, W, n = [(100, 300), (64, 600)] * copies, 8, 300
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rank)
    D = [torch.randn(64 * 600, generator=gen, device="cuda") * 1e-3 for _ in range(3)]
    V = [torch.randn(1500, generator=gen, device="cuda") for _ in range(W)]
    got = []
    for vectors in ((), (1500,) * n):
        comp = B.Compressor(B.layer_list(layers, vectors), rank, 8, 8, W)
        for l, (r, c) in enumerate(layers):
            comp.set_q(l, np.random.default_rng(l).standard_normal((c, min(rank, r, c))).astype(f32))
        G = [[D[(l + w) % 3][:r * c].view(r, c) for l, (r, c) in enumerate(layers)] + [V[w]] * len(vectors) for w in range(W)]
        out = [torch.zeros(s, device="cuda") for s in layers] + [torch.zeros(1500, device="cuda") for _ in vectors]
        for _ in range(2):
            comp.step(G, out)
        comp.synchronize()
        got.append([t.cpu().numpy() for t in out])
        comp.close()
    for x, y in zip(got[0], got[1]):
        assert np.array_equal(x, y)
    mean = sum(v.cpu().numpy().astype(np.float64) for v in V) / W
    assert all(np.allclose(x, mean, rtol=0, atol=1e-6) for x in got[1][len(layers):])

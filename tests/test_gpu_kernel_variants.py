"""The kernel variants that the library picks by size, each at the edges of its tiles and of the sizes it is picked for,
against the CPU oracle and with the tolerances of tests/util.py."""
import numpy as np
import pytest
import torch

import oracle
import s24_inputs as si
from util import F32_TOL, assert_close, dev, dev_bf16, host_bits, host_f64, joint_run, mask_tiles_run, slices_run, tiles_run, tol_for, torch_dtype

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def s24():
    import paper_2404_01847_amd as lib
    lib.lib()
    return lib


def compressed(W):
    """Oracle's compressed operands of a weight, in the library's storage, on the GPU: (vals, meta), (valsT, metaT)."""
    c = oracle.compress(W, oracle.transposable_mask(W))
    (v, m), (vt, mt) = oracle.pack(c[0], c[1]), oracle.pack(c[2], c[3])
    return c, (dev_bf16(v), dev(m)), (dev_bf16(vt), dev(mt))


# ------------------------------------------------------------------ fp32 on the matrix cores
F32_NT = [
    # (p, q, r): four slices of a 32-tile; eight slices (deep, few tiles); four slices of a 64-tile; ragged edges of each
    (33, 64, 48), (31, 128, 2064), (40, 576, 80), (1, 1024, 16), (1040, 64, 2064), (1057, 192, 2000),
    # r a multiple of 32, so that the gated forward runs too: its 64-tile in four slices and in eight, the 32 features of a
    # tile ragged (48, 80, 16, 528, 1008)
    (33, 64, 96), (40, 576, 160), (1, 1024, 32), (300, 512, 1056), (1057, 192, 2016)]


@pytest.mark.parametrize("pqr", F32_NT)
def test_f32_products_and_their_epilogues(s24, pqr):
    p, q, r = pqr
    r64 = (r + 63) // 64 * 64                # compress needs multiples of 64; the product takes the first r rows
    W = si.random_matrix(40 + r, (r64, q), 0.02, "f32")
    X = si.random_matrix(41 + p, (p, q), 1.0, "f32")
    bias = si.random_matrix(42 + r, (1, r), 0.5, "f32")[0]
    mask = oracle.transposable_mask(W)
    cv, cm = (a[:r] for a in oracle.compress(W, mask)[:2])
    v, m = oracle.pack(np.ascontiguousarray(cv), np.ascontiguousarray(cm))
    v, m, x = dev(v), dev(m), dev(X)
    ref = oracle.spmm_fwd(X, cv, cm)
    Y, Z, H = (torch.full((p, r), 7.0, device="cuda") for _ in range(3))
    s24.spmm_fwd(x, v, m, Y)
    assert_close(host_f64(Y), ref, F32_TOL, f"spmm_fwd {pqr}")
    s24.spmm_fwd_act(x, v, m, dev(bias), Z, H, s24.ACT_GELU_ERF)
    assert_close(host_f64(Z), ref + bias.astype(np.float64), F32_TOL, f"spmm_fwd_act {pqr}")
    two = torch.empty_like(H)
    s24.act_fwd(Z, two, s24.ACT_GELU_ERF)
    assert_close(host_f64(H), host_f64(two), F32_TOL, f"act {pqr}")
    assert torch.equal(H.view(torch.int32), two.view(torch.int32))           # the bits of the two calls
    s24.spmm_bwd_dx(x, v, m, Y, beta=1.0)    # the same product on top of itself
    assert_close(host_f64(Y), 2 * ref, F32_TOL, f"accumulate {pqr}")
    Wd = np.ascontiguousarray(W[:r])
    s24.dense_gemm(x, dev(Wd), Y)
    assert_close(host_f64(Y), X.astype(np.float64) @ Wd.astype(np.float64).T, F32_TOL, f"dense_gemm {pqr}")
    if r % 32 == 0:                          # the same weight as a stacked [gate; up]
        f, GU, Hg = r // 2, torch.full((p, r), 7.0, device="cuda"), torch.full((p, r // 2), 7.0, device="cuda")
        for gate in (s24.GATE_SILU, s24.GATE_GELU_ERF):
            s24.spmm_fwd_glu(x, v, m, dev(bias), GU, Hg, gate)
            assert torch.equal(GU.view(torch.int32), Z.view(torch.int32))    # the order of the sum is the plain product's
            two = torch.empty_like(Hg)
            s24.glu_fwd(Z, two, gate)
            assert_close(host_f64(Hg), host_f64(two), F32_TOL, f"glu {pqr} f={f}")
            assert torch.equal(Hg.view(torch.int32), two.view(torch.int32))


@pytest.mark.parametrize("case", [
    # (p, q, r, beta): 32-tiles; slices of less than one token; an odd token count; 64-tiles with ragged edges
    # (up to 7 tokens are one chain, here beside a second problem of 12 or fewer)
    (1, 16, 16, 0.0), (2, 1552, 2064, 0.0), (5, 80, 144, 0.0), (8, 48, 80, 1.0), (7, 48, 80, 1.0), (129, 80, 144, 0.0), (131, 1552, 2064, 1.0), (64, 1552, 2064, 0.0), (192, 48, 80, 1.0)])
def test_f32_weight_gradients(s24, case):
    p, q, r, beta = case
    lam = 2e-4
    dY, X = si.random_matrix(50 + p, (p, r), 1e-2, "f32"), si.random_matrix(51 + p, (p, q), 1.0, "f32")
    W, dW0 = si.random_matrix(52 + p, (r, q), 0.02, "f32"), si.random_matrix(53 + p, (r, q), 1e-3, "f32")
    mask = oracle.transposable_mask(W)
    decay = oracle.masked_decay(np.zeros((r, q), np.float32), W, mask, lam)
    dY2, X2 = si.random_matrix(54, (p + 5, 32), 1e-2, "f32"), si.random_matrix(55, (p + 5, 48), 1.0, "f32")
    a, b = dev(dW0).clone(), torch.zeros((32, 48), device="cuda")
    s24.dense_dw_batch([(dev(dY), dev(X), a, dev(W), dev(mask), lam), (dev(dY2), dev(X2), b, None, None, 0.0)], beta=beta)
    ref = dY.astype(np.float64).T @ X.astype(np.float64) + beta * dW0.astype(np.float64) + decay
    assert_close(host_f64(a), ref, F32_TOL, f"dense_dw_batch {case}")
    assert_close(host_f64(b), dY2.astype(np.float64).T @ X2.astype(np.float64), F32_TOL, f"second problem {case}")
    if p % 64 == 0:
        vz, mz = oracle.mvue24(dY, 99)
        vp, mp = oracle.pack(vz, mz)
        c = dev(dW0).clone()
        s24.spmm_dw(dev(vp), dev(mp), dev(X), c, beta=beta, W=dev(W), mask=dev(mask), lam=lam)
        ref = oracle.spmm_fwd(np.ascontiguousarray(X.T), vz, mz).T + beta * dW0.astype(np.float64) + decay
        assert_close(host_f64(c), ref, F32_TOL, f"spmm_dw {case}")


@pytest.mark.parametrize("p,q,r", [(7, 48, 80), (129, 48, 80), (131, 1552, 2064)])
def test_f32_weight_gradient_of_an_odd_token_count_with_an_infinity_in_the_last_token(s24, p, q, r):
    dY, X = si.random_matrix(150, (p, r), 1e-2, "f32"), si.random_matrix(151, (p, q), 1.0, "f32")
    X[p - 1, 5] = np.inf
    dW = torch.zeros((r, q), device="cuda")
    s24.dense_dw(dev(dY), dev(X), dW)
    got = dW.cpu().numpy()
    assert np.array_equal(got[:, 5], np.copysign(np.float32(np.inf), dY[p - 1]))    # dY has no zero
    rest = np.arange(q) != 5
    assert_close(got[:, rest].astype(np.float64), dY.astype(np.float64).T @ X[:, rest].astype(np.float64), F32_TOL)


@pytest.mark.parametrize("q,r", [(16, 16), (48, 80), (1552, 2064)])
def test_f32_weight_gradients_of_few_tokens_are_chains(s24, q, r):
    """3 and 7 tokens: the bits of fused multiply-adds in token order, alone and in one grid with a problem in slices."""
    long_ = (dev(si.random_matrix(62, (64, 32), 1e-2, "f32")), dev(si.random_matrix(63, (64, 48), 1.0, "f32")))
    for p in (3, 7):
        dY, X = si.random_matrix(64 + p, (p, r), 1e-2, "f32"), si.random_matrix(65 + p, (p, q), 1.0, "f32")
        chain = np.zeros((r, q), np.float32)
        for t in range(p):    # the product of two floats is exact in fp64; one rounding of it plus the sum, but for double rounding
            chain = (dY[t][:, None].astype(np.float64) * X[t][None, :] + chain).astype(np.float32)
        alone, shared, other = (torch.zeros(s, device="cuda") for s in ((r, q), (r, q), (32, 48)))
        s24.dense_dw(dev(dY), dev(X), alone)
        s24.dense_dw_batch([(dev(dY), dev(X), shared, None, None, 0.0), (*long_, other, None, None, 0.0)])
        assert torch.equal(alone.view(torch.int32), shared.view(torch.int32))
        assert (alone.cpu().numpy() != chain).mean() <= 1e-5, p    # a double rounding is rarer than one in 2^20 additions


def test_f32_weight_gradients_that_depend_on_their_order(s24):
    """Two problems that add to one gradient, and one whose operand is another's gradient, act one after the other."""
    p, q, r = 130, 48, 80
    dY = [dev(si.random_matrix(56 + i, (p, r), 1e-2, "f32")) for i in range(2)]
    X = [dev(si.random_matrix(58 + i, (p, q), 1.0, "f32")) for i in range(2)]
    dZ, start = dev(si.random_matrix(60, (r, 32), 1.0, "f32")), dev(si.random_matrix(61, (r, q), 1e-3, "f32"))
    sum_, chain = start.clone(), torch.zeros((32, q), device="cuda")
    problems = [(dY[0], X[0], sum_, None, None, 0.0), (dY[1], X[1], sum_, None, None, 0.0), (dZ, sum_, chain, None, None, 0.0)]
    s24.dense_dw_batch(problems, beta=1.0)
    sum1, chain1 = start.clone(), torch.zeros((32, q), device="cuda")
    for d, x, w in ((dY[0], X[0], sum1), (dY[1], X[1], sum1), (dZ, sum1, chain1)):
        s24.dense_dw(d, x, w, beta=1.0)
    assert torch.equal(sum_.view(torch.int32), sum1.view(torch.int32)) and torch.equal(chain.view(torch.int32), chain1.view(torch.int32))
    ref = host_f64(start) + sum(host_f64(d).T @ host_f64(x) for d, x in zip(dY, X))
    assert_close(host_f64(sum_), ref, F32_TOL, "two additions")
    assert_close(host_f64(chain), host_f64(dZ).T @ ref, F32_TOL, "chained")


# ------------------------------------------------------------------ infinities and NaNs beside pruned elements
def _cells(mask, shape):
    i, j = np.indices(shape)
    return ((mask[i // 4, j // 4] >> (4 * (i % 4) + j % 4)) & 1).astype(bool)


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
# fp32: four slices of a 32-tile, eight, four of a 64-tile; 16-bit: slices and the 256 x 128 tile
@pytest.mark.parametrize("pqr", [(33, 128, 96), (40, 576, 160), (1057, 192, 2016)])
def test_pruned_elements_never_reach_a_product(s24, dtype, pqr):
    p, q, r = pqr
    r64 = (r + 63) // 64 * 64
    W, X = si.random_matrix(130 + r, (r64, q), 0.02, dtype), si.random_matrix(131, (p, q), 1.0, dtype)
    mask = oracle.transposable_mask(W)
    v, m = oracle.pack(*(np.ascontiguousarray(a[:r]) for a in oracle.compress(W, mask)[:2]))
    kept = np.where(_cells(mask, W.shape)[:r], si.to_f32(W)[:r], 0).astype(np.float64)
    x = dev_bf16(X).clone()
    clean, hit = x.clone(), np.zeros((p, r), bool)
    for t, k, value in ((3, 17, np.inf), (7, 64, np.nan), (8, 100, -np.inf), (p - 1, q - 1, np.inf)):
        x[t, k], clean[t, k] = value, 0
        hit[t] |= kept[:, k] != 0
    ref, (v, m) = host_f64(clean) @ kept.T, (dev_bf16(v), dev(m))
    new = lambda n: torch.full((p, n), 1.0, dtype=torch_dtype(dtype), device="cuda")
    Y, Z, H, GU, Hg, dX = new(r), new(r), new(r), new(r), new(r // 2), new(r)
    s24.spmm_fwd(x, v, m, Y)
    s24.spmm_fwd_act(x, v, m, None, Z, H, s24.ACT_RELU)
    s24.spmm_fwd_glu(x, v, m, None, GU, Hg, s24.GATE_SILU)
    s24.spmm_bwd_dx(x, v, m, dX, beta=1.0)
    for got, want, what in ((Y, ref, "fwd"), (Z, ref, "act"), (GU, ref, "glu"), (dX, ref + 1, "accumulate")):
        got = host_f64(got)
        assert np.array_equal(~np.isfinite(got), hit), what
        assert_close(np.where(hit, 0, got), np.where(hit, 0, want), tol_for(dtype), what)


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("p,q,r", [(192, 48, 80), (64, 1552, 2064)])
def test_pruned_tokens_never_reach_a_weight_gradient(s24, dtype, p, q, r):
    dY, X = si.random_matrix(140, (p, r), 1e-2, dtype), si.random_matrix(141, (p, q), 1.0, dtype)
    vz, mz = oracle.mvue24(dY, 99)
    kept = np.zeros((r, p), bool)
    for g in range(p // 4):
        nib = (mz[:, g // 4].astype(np.uint32) >> (4 * (g % 4))) & 15
        kept[np.arange(r), 4 * g + (nib & 3)] = kept[np.arange(r), 4 * g + (nib >> 2)] = True
    v, m = oracle.pack(vz, mz)
    x, hit = dev_bf16(X).clone(), np.zeros((r, q), bool)
    clean = x.clone()
    for t, n, value in ((3, 17, np.inf), (50, 40, np.nan), (p - 1, q - 1, -np.inf)):
        x[t, n], clean[t, n] = value, 0
        hit[:, n] |= kept[:, t]
    got, want = torch.zeros((r, q), device="cuda"), torch.zeros((r, q), device="cuda")
    s24.spmm_dw(dev_bf16(v), dev(m), x, got)
    s24.spmm_dw(dev_bf16(v), dev(m), clean, want)
    got, want = host_f64(got), host_f64(want)
    assert np.array_equal(~np.isfinite(got), hit)
    assert_close(np.where(hit, 0, got), np.where(hit, 0, want), F32_TOL)


# ------------------------------------------------------------------ mask search, compress and L1 gap by matrix size
def _search_and_compress(s24, W):
    r, q = W.shape
    Wd, dt = dev_bf16(W), torch_dtype({np.uint16: "bf16", np.float16: "f16", np.float32: "f32"}[W.dtype.type])
    new = lambda shape, t: torch.zeros(shape, dtype=t, device="cuda")
    out = [new((q // 64, r, 32), dt), new((q // 64, r, 4), torch.int16), new((r // 64, q, 32), dt), new((r // 64, q, 4), torch.int16)]
    alone, fused = new((r // 4, q // 4), torch.int16), new((r // 4, q // 4), torch.int16)
    s24.transposable_mask(Wd, alone)
    s24.compress(Wd, None, *out, mask_out=fused)
    given = [torch.zeros_like(o) for o in out]
    s24.compress(Wd, alone, *given)
    return alone, fused, out, given


def _mask_tile(dtype, call, shapes):
    """The tile that a search alone, a search with compression ("fused") or a compression with given masks takes, by the number of
    tiles of 32 x 32 blocks of all weights."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rounds = sum(-(-r // 128) * -(-q // 128) for r, q in shapes) / cus
    if call == "alone":
        return (32, 32) if dtype == "bf16" and rounds >= 8 else (16, 16)
    if call == "fused":
        return (32, 32) if dtype != "f32" and rounds >= 4 else (16, 16)
    return (16, 16) if rounds < (1 if dtype == "f32" else 4) else (32, 32) if dtype == "f32" and rounds >= 4 else (32, 16)


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
# one 16 x 16 tile and its edges; both sides of the lines between the tile shapes (256, 1024 and 2048 tiles of 32 x 32 blocks: 16 x 16 and
# 15 x 17; 32 x 31 and 32 x 32; 64 x 65, in fp32 32 x 65) and between them, ragged
@pytest.mark.parametrize("rq", [(64, 64), (192, 320), (1920, 2112), (2048, 1984), (2240, 2048), (2368, 2048), (1984, 4160), (4096, 3904), (4032, 4032),
                                (8128, 8256)])
def test_mask_and_compress_tile_shapes(s24, dtype, rq):
    if rq[0] > 4096 and dtype == "f32":
        rq = (rq[0] // 128 * 64, rq[1])
    W = si.random_matrix(60 + rq[0], rq, 0.02, dtype)
    result = []
    assert mask_tiles_run(lambda: result.extend(_search_and_compress(s24, W))) == [_mask_tile(dtype, c, [rq]) for c in ("alone", "fused", "given")]
    alone, fused, out, given = result
    mask = oracle.transposable_mask(W)
    assert np.array_equal(host_bits(alone), mask) and np.array_equal(host_bits(fused), mask)
    c = oracle.compress(W, mask)
    for got, again, want in zip(out, given, oracle.pack(c[0], c[1]) + oracle.pack(c[2], c[3])):
        g, w = host_bits(got), want
        assert np.array_equal(g.view(np.uint8), w.reshape(g.shape).view(np.uint8))
        assert torch.equal(got.view(torch.uint8), again.view(torch.uint8))


def _repeated(a, r, q):
    """`a` over and over along both axes, cut to r x q: what a block is worth does not depend on where it lies."""
    return np.ascontiguousarray(np.tile(a, (-(-r // a.shape[0]), -(-q // a.shape[1])))[:r, :q])


def _search_in_tiles(s24, W, mask, ids, dtype, compress):
    """Masks and pattern ids of a search alone, and the masks of the search that compresses, in the tiles that the size asks for."""
    r, q = W.shape
    new = lambda *shape, t=torch.int16: torch.full(shape, 7, dtype=t, device="cuda")
    Wd, alone, index = dev_bf16(W), new(r // 4, q // 4), new(r // 4, q // 4, t=torch.uint8)
    assert mask_tiles_run(lambda: s24.transposable_mask(Wd, alone, index)) == [_mask_tile(dtype, "alone", [(r, q)])]
    assert np.array_equal(host_bits(alone), mask) and np.array_equal(index.cpu().numpy(), ids)
    if compress:
        fused, td = new(r // 4, q // 4), torch_dtype(dtype)
        out = [new(q // 64, r, 32, t=td), new(q // 64, r, 4), new(r // 64, q, 32, t=td), new(r // 64, q, 4)]
        assert mask_tiles_run(lambda: s24.compress(Wd, None, *out, mask_out=fused)) == [_mask_tile(dtype, "fused", [(r, q)])]
        assert np.array_equal(host_bits(fused), mask)


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("kind", ["few", "equal", "tiny", "range", "subnormal", "window", "zeros"])
# the small tile, and 46 x 46 tiles of 32 x 32 blocks, the last ones half empty (and, of the search alone, a block column and row less)
@pytest.mark.parametrize("rq", [(192, 320), (2432, 2048), (5824, 5824), (5820, 5820)])
def test_wide_blocks_in_both_tile_shapes(s24, dtype, kind, rq):
    """Ties, and blocks too wide for the fast paths, many per wave: the wave-cooperative paths of fp32, the integer scores of bf16 in the
    large tile with their queue and what the small one does instead, the fp64 scores of the fused search in either."""
    r, q = rq
    one = si.tie_matrix(61, *((192, 320) if r > 4096 else rq), dtype, kind)      # the large ones are it over and over: one oracle's worth
    mask, ids = oracle.transposable_mask(one, want_index=True)
    _search_in_tiles(s24, _repeated(one, r, q), _repeated(mask, r // 4, q // 4), _repeated(ids, r // 4, q // 4), dtype, r % 64 == 0)


@pytest.mark.parametrize("big_exp", [9, 10, 11, 12, 26, 40, 47, 60, 100])
@pytest.mark.parametrize("rq", [(64, 320), (5824, 5824)])
def test_margins_below_an_fp64_sum_in_both_tile_shapes(s24, legal_blocks, big_exp, rq):
    """Best patterns that are one unit in the last place of a small element ahead of an earlier one.  In every fourth block elements ten
    binades below the largest stand for the zeros, so that up to 2^10 the integer scores take it."""
    from util import absorbed_margin_blocks
    one, _ = absorbed_margin_blocks(legal_blocks, "bf16", big_exp)
    f = si.to_f32(one)
    full = np.where((f == 0) & (np.arange(f.shape[1]) // 4 % 4 == 0)[None, :], np.float32(2.0 ** (big_exp - 10)), f)
    one = si.f32_to_bf16_bits(torch.from_numpy(np.ascontiguousarray(full)))
    mask, ids = oracle.transposable_mask(one, want_index=True)
    r, q = rq
    _search_in_tiles(s24, _repeated(one, r, q), _repeated(mask, r // 4, q // 4), _repeated(ids, r // 4, q // 4), "bf16", True)


# 35 binades: fp64 sums; 60: fixed point.  Few or many of a wave's 64 blocks, all of them among them
@pytest.mark.parametrize("spread", [(35, 35), (60, 60), (35, 60)])
@pytest.mark.parametrize("share", [0.01, 0.2, 0.45, 0.95, 1.0])
def test_bf16_search_of_some_wide_blocks(s24, spread, share):
    """The small tile: wide blocks leave the common path and are scored by the wave together or by a lane each."""
    r, q = 208, 336
    rng = np.random.default_rng(63)
    scale = np.ones((r // 4, q // 4, 16))
    wide, at = rng.random((r // 4, q // 4)) < share, rng.integers(0, 16, (r // 4, q // 4))
    i, j = np.nonzero(wide)
    scale[i, j, at[i, j]] = 2.0 ** -np.where(rng.random(i.size) < 0.5, *spread)
    W = rng.standard_normal((r, q)) * 0.02 * scale.reshape(r // 4, q // 4, 4, 4).transpose(0, 2, 1, 3).reshape(r, q)
    W = si.f32_to_bf16_bits(torch.from_numpy(W.astype(np.float32)))
    mask, index = torch.zeros((r // 4, q // 4), dtype=torch.int16, device="cuda"), torch.zeros((r // 4, q // 4), dtype=torch.uint8, device="cuda")
    assert mask_tiles_run(lambda: s24.transposable_mask(dev_bf16(W), mask, index)) == [(16, 16)]
    want, ids = oracle.transposable_mask(W, want_index=True)
    assert np.array_equal(host_bits(mask), want) and np.array_equal(index.cpu().numpy(), ids)


def test_f32_search_beside_infinities_and_nans(s24, legal_blocks):
    """Blocks of values above 2^102 with an infinity or a NaN go through the fp64 sums: patterns that hold a NaN never win, and
    the first of the largest does, wherever in the wave the block lies."""
    W = si.random_matrix(170, (64, 256), 2.0 ** 110, "f32")
    W = np.where(np.abs(W) < 2.0 ** 104, 2.0 ** 104, W).astype(np.float32)
    for n in range(16):
        W[4 * (n % 4) + n // 4, 8 * n + (5 * n) % 8] = np.nan if n % 3 else np.inf
    a = np.abs(W).astype(np.float64).reshape(16, 4, 64, 4).transpose(0, 2, 1, 3).reshape(16, 64, 1, 16)
    legal = np.array([[(m >> t) & 1 for t in range(16)] for m in legal_blocks], bool)
    sums = np.where(legal, a, 0).sum(-1)
    want = np.array(legal_blocks, np.uint16)[np.where(np.isnan(sums), -1, sums).argmax(-1)]
    alone, fused, _, _ = _search_and_compress(s24, W)
    assert np.array_equal(host_bits(alone), want) and np.array_equal(host_bits(fused), want)


@pytest.mark.parametrize("dtype,r,q", [("f16", 4, 2 ** 30 + 1028), ("f16", 2 ** 30 + 1028, 4), ("f32", 4, 2 ** 30 + 1028)])
def test_mask_search_in_more_tiles_than_a_launch_holds(s24, dtype, r, q):
    """2^24 and some tiles of 16 x 16 blocks: the masks that searches of a part each give."""
    W = torch.empty((r, q), dtype=torch_dtype(dtype), device="cuda").normal_(generator=torch.Generator(device="cuda").manual_seed(q))
    new = lambda: torch.full((r // 4, q // 4), -1, dtype=torch.int16, device="cuda")
    index = torch.full((r // 4, q // 4), 255, dtype=torch.uint8, device="cuda")
    whole, parts = new(), new()
    s24.transposable_mask(W, whole, index)
    step = 2 ** 28
    for i in range(0, r, step):
        for j in range(0, q, step):
            part = torch.empty((min(step, r - i) // 4, min(step, q - j) // 4), dtype=torch.int16, device="cuda")
            s24.transposable_mask(W[i:i + step, j:j + step], part)
            parts[i // 4:(i + step) // 4, j // 4:(j + step) // 4] = part
    assert torch.equal(whole, parts)
    assert int(index.max()) == 89
    rows, cols = min(r, 1028), min(q, 1028)
    for i, j in ((0, 0), (r - rows, q - cols)):
        want, ids = oracle.transposable_mask(host_bits(W[i:i + rows, j:j + cols].contiguous()), want_index=True)
        at = (slice(i // 4, (i + rows) // 4), slice(j // 4, (j + cols) // 4))
        assert np.array_equal(host_bits(whole[at].contiguous()), want) and np.array_equal(index[at].cpu().numpy(), ids)


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("kind", ["few", "equal", "zeros", "tiny", "window", "normal"])
def test_l1_norm_gap_by_classes(s24, dtype, kind):
    """Ties for the best and for the second best across and inside the classes, ragged sizes; blocks inside the exact window
    match the oracle's 90 sums bit for bit."""
    W = si.random_matrix(62, (204, 260), 0.02, dtype) if kind == "normal" else si.tie_matrix(62, 204, 260, dtype, kind)
    gap = torch.full((51, 65), -1.0, dtype=torch.float64, device="cuda")
    s24.l1_norm_gap(dev_bf16(W), gap)
    a = np.abs(si.to_f32(W)).reshape(51, 4, 65, 4).transpose(0, 2, 1, 3).reshape(51, 65, 16).astype(np.float64)
    e = np.frexp(np.where(a > 0, a, np.nan))[1]
    exact = np.nanmax(np.where(np.isnan(e), -1e9, e), -1) - np.nanmin(np.where(np.isnan(e), 1e9, e), -1) <= {"bf16": 42, "f16": 39, "f32": 26}[dtype]
    got, ref = gap.cpu().numpy(), oracle.l1_norm_gap(W)
    assert exact.mean() > 0.5 or kind == "tiny"
    assert np.array_equal(got[exact], ref[exact]), kind
    # beyond it both carry fp64 rounding: eight additions, each 2^-53 of the block's kept norm, in either sum
    assert np.all(np.abs(got - ref)[~exact] <= 16 * 2.0 ** -53 * a.sum(-1)[~exact])


# one block column up to more than a wave's 64; as many rows of blocks as a grid of one workgroup per four could not hold
@pytest.mark.parametrize("r,q", [(1028, 4), (1012, 12), (516, 28), (132, 36), (68, 128), (36, 260), (4, 1028), (2 ** 28 + 1028, 4)])
def test_l1_norm_gap_by_width(s24, r, q):
    W = torch.empty((r, q), dtype=torch.bfloat16, device="cuda").normal_(generator=torch.Generator(device="cuda").manual_seed(r))
    gap = torch.full((r // 4, q // 4), -1.0, dtype=torch.float64, device="cuda")
    s24.l1_norm_gap(W, gap)
    for first in sorted({0, r // 8 * 4, max(0, r - 1028)}):      # the oracle on the first, middle and last rows
        rows = min(r - first, 1028)
        ref = oracle.l1_norm_gap(host_bits(W[first:first + rows]))
        assert np.array_equal(gap[first // 4:(first + rows) // 4].cpu().numpy(), ref), first
    assert (gap >= 0).all()


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
def test_l1_norm_gap_of_infinities_and_nans(s24, dtype, legal_blocks):
    """The gap is what best and second best of the 90 sums give when they are compared one by one, also where a block holds
    nothing but NaNs (a weight that has diverged must not look like one whose patterns tie)."""
    w = dev_bf16(si.random_matrix(160, (32, 512), 0.02, dtype)).clone()
    nan, inf = float("nan"), float("inf")
    w[0:4, 0:4], w[0:4, 4:8], w[4, 0] = nan, inf, nan
    w[8:12, 0:4], w[8:12, 4:8] = 3e4, 3e4
    w[9, 2], w[9, 5] = nan, inf
    w[12:16, 8:12], w[13, 9] = nan, 1.0
    if dtype != "f16":
        w[16:20, 0:4], w[16:20, 4:8] = 2.0 ** 127, 2.0 ** 127
        w[17, 1], w[17, 6] = nan, inf
    gap = torch.full((8, 128), -1.0, dtype=torch.float64, device="cuda")
    s24.l1_norm_gap(w, gap)
    a = np.abs(host_f64(w)).reshape(8, 4, 128, 4).transpose(0, 2, 1, 3).reshape(8, 128, 16)
    want = np.empty((8, 128))
    with np.errstate(invalid="ignore"):
        for at in np.ndindex(8, 128):
            sums = [sum(a[at][t] for t in range(16) if (m >> t) & 1) for m in legal_blocks]
            first, second = sums[0], 0.0
            for k, v in enumerate(sums[1:], 1):
                if v > first:
                    first, second = v, first
                elif k == 1 or v > second:
                    second = v
            want[at] = first - second
    got = gap.cpu().numpy()
    assert np.isnan(want[0, :2]).all() and np.isnan(want).sum() < 10
    assert np.array_equal(got, want, equal_nan=True)


# ------------------------------------------------------------------ sparse products on the 256 x 128 tile
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
# (p, q, r): one, two, three and four chunks of the ring, ragged in both directions (136 tiles, for the gated epilogue; the
# others take 128 x 128 tiles at so short a contraction); the same from 17 chunks on, for all of them; a strip of such
# tiles after a slab of large ones (51 rows of tiles, then 27 of half their height)
@pytest.mark.parametrize("pqr", [(2050, 64, 2016), (2050, 128, 2016), (2049, 192, 2048), (2061, 256, 2016), (16390, 64, 1248),
                                 (2050, 1088, 2016), (2049, 1152, 2048), (2061, 1216, 2016), (16390, 1088, 1248)])
def test_medium_tile_and_its_epilogues(s24, dtype, pqr):
    p, q, r = pqr
    r64 = (r + 63) // 64 * 64
    W, X = si.random_matrix(70 + q, (r64, q), 0.02, dtype), si.random_matrix(71 + p, (p, q), 1.0, dtype)
    bias, Zin = si.random_matrix(72, (1, r), 0.5, dtype)[0], si.random_matrix(73, (p, r), 1.0, dtype)
    cv, cm = (np.ascontiguousarray(a[:r]) for a in oracle.compress(W, oracle.transposable_mask(W))[:2])
    v, m = oracle.pack(cv, cm)
    v, m, x, b = dev_bf16(v), dev(m), dev_bf16(X), dev_bf16(bias)
    rows = np.unique(np.concatenate([[0, 1, 127, 128, 255, 256, p - 2, p - 1], np.random.default_rng(p).integers(0, p, 40)]))
    at = torch.from_numpy(rows).cuda()
    ref = oracle.spmm_fwd(X, cv, cm, rows=rows)
    tol, new = tol_for(dtype), lambda n: torch.full((p, n), 7.0, dtype=torch_dtype(dtype), device="cuda")
    Y, Z, H, dZ = new(r), new(r), new(r), new(r)
    plain = [(4, 4), (4, 2)] if q >= 1088 and r == 1248 else [(4, 2)] if q >= 1088 else [(2, 2)]
    assert tiles_run(lambda: s24.spmm_fwd(x, v, m, Y)) == plain
    assert_close(host_f64(Y[at]), ref, tol, f"spmm_fwd {pqr}")
    Y2 = Y.clone()
    s24.spmm_bwd_dx(x, v, m, Y2, beta=1.0)
    assert_close(host_f64(Y2[at]), ref + host_f64(Y[at]), tol, f"accumulate {pqr}")
    s24.spmm_fwd_act(x, v, m, b, Z, H, s24.ACT_GELU_ERF)
    assert_close(host_f64(Z[at]), ref + host_f64(b), tol, f"spmm_fwd_act {pqr}")
    two = torch.empty_like(H)
    s24.act_fwd(Z, two, s24.ACT_GELU_ERF)
    assert torch.equal(H.view(torch.int16), two.view(torch.int16))
    s24.spmm_bwd_dx_act(x, v, m, dev_bf16(Zin), dZ, s24.ACT_GELU_ERF)
    s24.act_bwd(Y, dev_bf16(Zin), two, s24.ACT_GELU_ERF)
    assert torch.equal(dZ.view(torch.int16), two.view(torch.int16))
    GU, Hg, two = new(r), new(r // 2), new(r // 2)
    assert tiles_run(lambda: s24.spmm_fwd_glu(x, v, m, b, GU, Hg, s24.GATE_SILU)) == [(4, 4) if r == 1248 else (4, 2)]
    s24.glu_fwd(GU, two, s24.GATE_SILU)
    assert torch.equal(GU.view(torch.int16), Z.view(torch.int16)) and torch.equal(Hg.view(torch.int16), two.view(torch.int16))


# ------------------------------------------------------------------ sparse products in slices of the contraction
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
# (p, q, r) and the tile: one chunk (seven idle slices), one feature block; a slice more or less than the others and the load pipeline's
# remainders (9, 31, 65 and 68 chunks); each of the smaller four tiles, ragged along both axes
@pytest.mark.parametrize("pqr, tile", [((1, 64, 16), (1, 1)), ((16, 576, 48), (1, 1)), ((15, 1984, 4112), (2, 1)), ((3, 4160, 272), (1, 1)), ((33, 4352, 2080), (2, 1)), ((17, 640, 4128), (4, 1)),
                                       ((130, 2112, 1040), (4, 1)), ((257, 512, 1056), (4, 2)), ((61, 1088, 4112), (4, 2))])
def test_sliced_products_and_their_epilogues(s24, dtype, pqr, tile):
    sliced_products_and_their_epilogues(s24, dtype, pqr, tile)


def sliced_products_and_their_epilogues(s24, dtype, pqr, tile):
    p, q, r = pqr
    r64 = (r + 63) // 64 * 64
    W, X = si.random_matrix(80 + q, (r64, q), 0.02, dtype), si.random_matrix(81 + p, (p, q), 1.0, dtype)
    bias, Zin = si.random_matrix(82, (1, r), 0.5, dtype)[0], si.random_matrix(83, (p, r), 1.0, dtype)
    cv, cm = (np.ascontiguousarray(a[:r]) for a in oracle.compress(W, oracle.transposable_mask(W))[:2])
    v, m = oracle.pack(cv, cm)
    v, m, x, b = dev_bf16(v), dev(m), dev_bf16(X), dev_bf16(bias)
    ref, tol = oracle.spmm_fwd(X, cv, cm), tol_for(dtype)
    new = lambda n: torch.full((p, n), 7.0, dtype=torch_dtype(dtype), device="cuda")
    bits = lambda t: t.view(torch.int16)
    Y, Yb, Z, H, dZ, two = (new(r) for _ in range(6))
    assert slices_run(lambda: s24.spmm_fwd(x, v, m, Y)) == [(*tile, False)]
    assert_close(host_f64(Y), ref, tol, f"spmm_fwd {pqr}")
    Y2 = Y.clone()
    s24.spmm_bwd_dx(x, v, m, Y2, beta=1.0)
    assert_close(host_f64(Y2), ref + host_f64(Y), tol, f"accumulate {pqr}")
    s24.spmm_fwd_bias(x, v, m, b, Yb)
    assert_close(host_f64(Yb), ref + host_f64(b), tol, f"bias {pqr}")
    for act in (s24.ACT_RELU, s24.ACT_GELU_ERF):   # the fused epilogues give the bits of the separate calls
        s24.spmm_fwd_act(x, v, m, b, Z, H, act)
        s24.act_fwd(Yb, two, act)
        assert torch.equal(bits(Z), bits(Yb)) and torch.equal(bits(H), bits(two))
        s24.spmm_bwd_dx_act(x, v, m, dev_bf16(Zin), dZ, act)
        s24.act_bwd(Y, dev_bf16(Zin), two, act)
        assert torch.equal(bits(dZ), bits(two))
    if r % 32 == 0:
        GU, Hg, two = new(r), new(r // 2), new(r // 2)
        for gate in (s24.GATE_SILU, s24.GATE_GELU_ERF):
            s24.spmm_fwd_glu(x, v, m, b, GU, Hg, gate)
            s24.glu_fwd(Yb, two, gate)
            assert torch.equal(bits(GU), bits(Yb)) and torch.equal(bits(Hg), bits(two))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
# (p, q, r) of the 64 x 64 tile: of three to five chunks to a wave, and of one or two; ragged along both axes, by one token and by 16 features
@pytest.mark.parametrize("pqr", [(513, 1984, 1040), (193, 2112, 3104), (500, 576, 1616)])
def test_sliced_products_in_the_largest_tile(s24, dtype, pqr):
    sliced_products_and_their_epilogues(s24, dtype, pqr, (4, 4))


@pytest.mark.parametrize("q", [1984, 2048])     # slices; the tiles' kernel from 384 tiles of 128 x 128 and this contraction on
def test_few_tokens_of_many_features_on_either_kernel(s24, q):
    few_tokens(s24, 13, q, 49152)


# below 48 MB of values and index words, from there on, and 101 MB in the lowest tile
@pytest.mark.parametrize("q, r, variant", [(4096, 10880, (4, 1, False)), (4096, 10944, (4, 1, True)), (22016, 4096, (1, 1, False))])
def test_weights_of_few_tokens_past_the_caches_and_through_them(s24, q, r, variant):
    assert few_tokens(s24, 13, q, r) == [variant]


def few_tokens(s24, p, q, r):
    """The forward products of p tokens against a reference and each other; the variants of the sliced kernel that the plain one ran in."""
    gen = torch.Generator(device="cuda").manual_seed(q)
    rnd = lambda *shape: torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
    W, x, b = rnd(r, q) * 0.02, rnd(p, q), rnd(r)
    new = lambda *shape, t=torch.bfloat16: torch.empty(shape, dtype=t, device="cuda")
    v, m, vt, mt = new(q // 64, r, 32), new(q // 64, r, 4, t=torch.int16), new(r // 64, q, 32), new(r // 64, q, 4, t=torch.int16)
    mask = new(r // 4, q // 4, t=torch.int16)
    s24.compress(W, None, v, m, vt, mt, mask_out=mask)
    rows = np.unique(np.concatenate([[0, 63, 64, 255, 256, r - 1], np.random.default_rng(q).integers(0, r, 200)]))
    bits = host_bits(mask)[rows[:, None] // 4, np.arange(q)[None] // 4] >> (4 * (rows[:, None] % 4) + np.arange(q)[None] % 4)
    kept = np.where(bits & 1, host_f64(W[torch.from_numpy(rows).cuda()]), 0)
    Y, Z, H, two, GU = new(p, r), new(p, r), new(p, r), new(p, r), new(p, r)
    variants = slices_run(lambda: s24.spmm_fwd_bias(x, v, m, b, Y))
    assert_close(host_f64(Y)[:, rows], host_f64(x) @ kept.T + host_f64(b)[rows], tol_for("bf16"), f"spmm_fwd_bias {q}")
    s24.spmm_fwd_act(x, v, m, b, Z, H, s24.ACT_GELU_ERF)
    s24.act_fwd(Y, two, s24.ACT_GELU_ERF)
    assert torch.equal(Z.view(torch.int16), Y.view(torch.int16)) and torch.equal(H.view(torch.int16), two.view(torch.int16))
    Hg, two = new(p, r // 2), new(p, r // 2)
    s24.spmm_fwd_glu(x, v, m, b, GU, Hg, s24.GATE_SILU)
    s24.glu_fwd(Y, two, s24.GATE_SILU)
    assert torch.equal(GU.view(torch.int16), Y.view(torch.int16)) and torch.equal(Hg.view(torch.int16), two.view(torch.int16))
    return variants


def test_calls_go_to_the_current_stream(s24):
    from paper_2404_01847_amd import binding
    side = torch.cuda.Stream()
    assert binding._stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert binding._stream() == side.cuda_stream != torch.cuda.default_stream().cuda_stream


# ------------------------------------------------------------------ GELU in the epilogues
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
# the 128 x 128, the 256 x 128 and the 256 x 256 tile, ragged in the tokens
@pytest.mark.parametrize("p,q,tile", [(8136, 64, (2, 2)), (8136, 2112, (4, 2)), (16390, 2112, (4, 4))])
def test_gelu_of_every_16_bit_value_in_the_epilogues(s24, dtype, p, q, tile):
    """H and dZ have the bits of the activation kernels for each of the 65536 values that Z can hold."""
    td, r = torch_dtype(dtype), 1024
    new = lambda: torch.empty((p, r), dtype=td, device="cuda")
    bits = lambda x: x.view(torch.int16)
    W = torch.zeros((r, q), dtype=td, device="cuda")
    W[torch.arange(r), torch.arange(r) % 4] = 1.0             # Z[n][m] = X[n][m % 4]
    v, vt = (torch.empty((a // 64, b, 32), dtype=td, device="cuda") for a, b in ((q, r), (r, q)))
    m, mt = (torch.empty((a // 64, b, 4), dtype=torch.int16, device="cuda") for a, b in ((q, r), (r, q)))
    s24.compress(W, None, v, m, vt, mt)
    g = torch.Generator(device="cuda").manual_seed(5)
    dY = torch.randn((p, q), generator=g, device="cuda").to(td)
    seen = torch.zeros(65536, dtype=torch.bool, device="cuda")
    for first in range(0, 65536, 4 * p):
        every = (first + torch.arange(4 * p, device="cuda")) % 65536
        X = torch.zeros((p, q), dtype=td, device="cuda")
        X[:, :4] = every.to(torch.int16).view(td).view(p, 4)
        Z, H, two = new(), new(), new()
        assert tiles_run(lambda: s24.spmm_fwd_act(X, v, m, None, Z, H, s24.ACT_GELU_ERF)) == [tile]
        s24.act_fwd(Z, two, s24.ACT_GELU_ERF)
        assert torch.equal(bits(H), bits(two))
        seen[bits(Z).flatten().long() & 0xFFFF] = True
        Z = every.to(torch.int16).view(td).view(p, 4).repeat(1, r // 4).contiguous()
        dH, dZ = new(), new()
        assert tiles_run(lambda: s24.spmm_bwd_dx_act(dY, v, m, Z, dZ, s24.ACT_GELU_ERF)) == [tile]
        s24.spmm_bwd_dx(dY, v, m, dH)
        s24.act_bwd(dH, Z, two, s24.ACT_GELU_ERF)
        assert torch.equal(bits(dZ), bits(two))
    value = torch.arange(65536, device="cuda").to(torch.int16).view(td).float()
    normal = value.abs() >= (2.0 ** -126 if dtype == "bf16" else 2.0 ** -14)
    assert bool(seen[value.isfinite() & normal].all())        # the forward met every normal value


@pytest.mark.parametrize("p,q,tile", [(8136, 64, (2, 2)), (8136, 2112, (4, 2)), (16390, 2112, (4, 4))])
def test_gelu_of_zeros_and_large_values_in_the_epilogues(s24, p, q, tile):
    """Zeros and every finite bf16 value from 16 on, of both signs, among values between: the bits of the activation kernels."""
    r = 1024
    new = lambda: torch.empty((p, r), dtype=torch.bfloat16, device="cuda")
    bits = lambda x: x.view(torch.int16)
    W = torch.zeros((r, q), dtype=torch.bfloat16, device="cuda")
    W[torch.arange(r), torch.arange(r) % 4] = 1.0             # Z[n][m] = X[n][m % 4]
    v, vt = (torch.empty((a // 64, b, 32), dtype=torch.bfloat16, device="cuda") for a, b in ((q, r), (r, q)))
    m, mt = (torch.empty((a // 64, b, 4), dtype=torch.int16, device="cuda") for a, b in ((q, r), (r, q)))
    s24.compress(W, None, v, m, vt, mt)
    g = torch.Generator(device="cuda").manual_seed(6)
    dY = torch.randn((p, q), generator=g, device="cuda").bfloat16()
    n = torch.arange(4 * p, device="cuda")
    pick, sign = torch.randint(0, 3, n.shape, generator=g, device="cuda"), n % 2 * 0x8000
    large = 0x4180 + n // 2 % 0x3E00                          # 16 ... the largest finite value
    between = torch.randint(0x3880, 0x4180, n.shape, generator=g, device="cuda")    # 2^-14 ... 16
    every = torch.where(pick == 0, large, torch.where(pick == 1, between, 0)) + sign
    every[:2 * 0x3E00] = (large + sign)[:2 * 0x3E00]
    every[-4 * 512:] = (n % 2 * 0x8000)[-4 * 512:]            # and whole tiles of zeros
    val = every.to(torch.int16).view(torch.bfloat16).view(p, 4)
    X = torch.zeros((p, q), dtype=torch.bfloat16, device="cuda")
    X[:, :4] = val
    Z, H, dH, dZ, two = new(), new(), new(), new(), new()
    assert tiles_run(lambda: s24.spmm_fwd_act(X, v, m, None, Z, H, s24.ACT_GELU_ERF)) == [tile]
    assert torch.equal(Z, val.repeat(1, r // 4))
    s24.act_fwd(Z, two, s24.ACT_GELU_ERF)
    assert torch.equal(bits(H), bits(two))
    Z = val.repeat(1, r // 4).contiguous()                    # with the zeros' signs
    assert tiles_run(lambda: s24.spmm_bwd_dx_act(dY, v, m, Z, dZ, s24.ACT_GELU_ERF)) == [tile]
    s24.spmm_bwd_dx(dY, v, m, dH)
    s24.act_bwd(dH, Z, two, s24.ACT_GELU_ERF)
    assert torch.equal(bits(dZ), bits(two))


# ------------------------------------------------------------------ several weights in one mask / compress launch
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
# 3, 150, 766, 1628 and 4105 tiles of 32 x 32 blocks: the lines lie at 256 and 1024.  Weights of whole tiles, with an edge both ways and of a
# single chunk
@pytest.mark.parametrize("shapes", [[(64, 64), (128, 192)], [(1088, 832), (64, 3072), (832, 1088)], [(4096, 1024), (2112, 3520), (64, 64), (64, 4160)],
                                    [(2112, 3520), (4160, 4032), (64, 4160), (1088, 832)], [(8192, 8192), (1088, 64)]])
def test_several_weights_in_one_compress_pass(s24, dtype, shapes):
    td = torch_dtype(dtype)
    g = torch.Generator(device="cuda").manual_seed(7)
    Ws = [torch.randn((r, 2 * q), generator=g, device="cuda").to(td)[:, :q] if k == 1 else torch.randn((r, q), generator=g, device="cuda").to(td)
          for k, (r, q) in enumerate(shapes)]                 # the second one is a window of a wider matrix

    def buffers():
        new = lambda shape, t: torch.full(shape, 3, dtype=t, device="cuda")
        return [(new((q // 64, r, 32), td), new((q // 64, r, 4), torch.int16), new((r // 64, q, 32), td), new((r // 64, q, 4), torch.int16),
                 new((r // 4, q // 4), torch.int16)) for r, q in shapes]

    one, all_, given = buffers(), buffers(), buffers()
    for W, (v, m, vt, mt, mask) in zip(Ws, one):
        s24.transposable_mask(W, mask)                        # checked against the oracle elsewhere
        s24.compress(W, mask, v, m, vt, mt)
    assert mask_tiles_run(lambda: s24.compress_batch([(W, None, *b) for W, b in zip(Ws, all_)])) == [_mask_tile(dtype, "fused", shapes)]
    assert mask_tiles_run(lambda: s24.compress_batch([(W, o[4], *b[:4], None) for W, o, b in zip(Ws, one, given)])) == [_mask_tile(dtype, "given", shapes)]
    bits = lambda x: x.view(torch.int32 if x.dtype == torch.float32 else torch.int16)
    for W, (r, q), a, b, c in zip(Ws, shapes, one, all_, given):
        assert all(torch.equal(bits(x), bits(y)) for x, y in zip(a, b))
        assert all(torch.equal(bits(x), bits(y)) for x, y in zip(a[:4], c[:4]))
        # and the operands hold what the mask keeps, in order: the definition, spelled out
        keep = torch.stack([(a[4].to(torch.int32) >> t) & 1 for t in range(16)], -1).view(r // 4, q // 4, 4, 4).bool()
        keep = keep.permute(0, 2, 1, 3).reshape(r, q)
        for dense, k, v, m in ((W, keep, a[0], a[1]), (W.t(), keep.t(), a[2], a[3])):
            rows, cols = dense.shape
            kept = dense.contiguous()[k.contiguous()].view(rows, cols // 64, 32).transpose(0, 1).contiguous()
            assert torch.equal(bits(v), bits(kept))
            at = torch.arange(cols, device="cuda").expand(rows, cols)[k.contiguous()].view(rows, cols // 64, 4, 8).to(torch.int64) % 4
            word = (at << (2 * torch.arange(8, device="cuda"))).sum(-1).transpose(0, 1)
            assert torch.equal(m.to(torch.int64) & 0xFFFF, word)


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("spread", [0, 14])
def test_search_alone_of_large_weights(s24, dtype, spread):
    """2070 tiles of 32 x 32 blocks: bf16 scores in integers and queues the blocks that these cannot hold (one in forty, or with
    a spread of binades nearly all); the masks are those of the fused search, whose scores are fp64."""
    r, q, td = 5888, 5760, torch_dtype(dtype)
    g = torch.Generator(device="cuda").manual_seed(11)
    W = torch.randn((r, q), generator=g, device="cuda") * 2.0 ** (-spread * torch.rand((r, q), generator=g, device="cuda")).floor()
    W = W.to(td)
    new = lambda *shape, t=td: torch.empty(shape, dtype=t, device="cuda")
    alone, fused = new(r // 4, q // 4, t=torch.int16), new(r // 4, q // 4, t=torch.int16)
    s24.transposable_mask(W, alone)
    s24.compress(W, None, new(q // 64, r, 32), new(q // 64, r, 4, t=torch.int16), new(r // 64, q, 32), new(r // 64, q, 4, t=torch.int16), mask_out=fused)
    assert torch.equal(alone, fused)


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("spread", [0, 3, 60])
def test_pruned_gradients_of_any_magnitude(s24, dtype, spread):
    """Groups whose sums lie on either side of what the short form of the draw takes (2^-100 to 2^100, and zero), subnormals and sums
    that overflow among them, zeros as ReLU leaves them, elements that the sum absorbs: bit for bit as the oracle."""
    p, r = 320, 208
    rng = np.random.default_rng(130 + spread)
    lo, hi = (-24, 15) if dtype == "f16" else (-149, 127) if dtype == "f32" else (-133, 127)
    e = np.repeat(rng.integers(lo, hi + 1, (p // 4, r)), 4, axis=0) - rng.integers(0, spread + 1, (p, r))
    e[:, :8] = np.repeat(np.repeat(rng.integers(-103, -97, (p // 4, 4)), 4, axis=0), 2, axis=1)      # around the limits themselves
    e[:, 4:8] = -e[:, 4:8]
    x = np.ldexp(rng.choice([-1.0, 1.0], (p, r)) * (1 + rng.random((p, r)) * (rng.random((p, r)) < 0.8)), np.clip(e, lo, hi))
    x[rng.random((p, r)) < 0.3] = 0.0
    x = np.clip(x, -65504.0, 65504.0) if dtype == "f16" else np.clip(x, -3.3e38, 3.3e38)
    x = x.astype(np.float32)
    dY = x if dtype == "f32" else x.astype(np.float16) if dtype == "f16" else si.f32_to_bf16_bits(torch.from_numpy(x))
    vals = torch.zeros((p // 64, r, 32), dtype=torch_dtype(dtype), device="cuda")
    meta = torch.zeros((p // 64, r, 4), dtype=torch.int16, device="cuda")
    s24.mvue24(dev_bf16(dY), 41, vals, meta)
    want_v, want_m = oracle.pack(*oracle.mvue24(dY, 41))
    assert np.array_equal(host_bits(meta).astype(np.uint16), want_m.astype(np.uint16))
    word = np.uint32 if dtype == "f32" else np.uint16
    assert np.array_equal(host_bits(vals).view(word), want_v.view(word))


def test_short_reciprocal_of_every_float_that_it_takes(s24):
    """2^-100 to 2^100, both ends among them: the bits of the division."""
    first, last = ((127 + e) << 23 for e in (-100, 100))
    different = torch.zeros(1, dtype=torch.int64, device="cuda")
    s24.probe_reciprocal(first, last - first + 1, different)
    assert int(different) == 0
    s24.probe_reciprocal(1, 1 << 23, different)               # subnormals and the smallest normal value are not for it: seen to differ
    assert int(different) > 0


# ------------------------------------------------------------------ fp32 weight gradients with several batches in flight
# 32-tiles in at most a workgroup per compute unit (192 of them), in one to two (512) and in more (1088), and 64-tiles (768): one, two or four
# batches of eight token pairs in flight
@pytest.mark.parametrize("rq", [(176, 1008), (1024, 512), (1072, 1008), (2048, 1536)])
# per slice: no batch and a rest, one, three, four, five and seven with a rest, eight, nine, ten and eleven with a rest
@pytest.mark.parametrize("p", [15, 127, 128, 129, 400, 512, 513, 647, 1031, 1024, 1216, 1290, 1500])
def test_f32_weight_gradient_batches(s24, rq, p):
    (r, q), g = rq, torch.Generator(device="cuda").manual_seed(p)
    dY, X = (torch.randn((p, n), generator=g, device="cuda") for n in (r, q))
    dW = torch.full((r, q), 5.0, device="cuda")
    s24.dense_dw(dY, X, dW)
    ref = dY.double().t() @ X.double()
    # eight slices and their sum: an error of sqrt(p) roundings of 2^-24 at most, as a chain of p / 8 has
    assert float((dW.double() - ref).norm() / ref.norm()) < 2.0 ** -24 * p ** 0.5


# ------------------------------------------------------------------ weight gradients on the 256 x 128 tile
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
# 144 such tiles in all; whole chunks and remainders; edges ragged along both axes; and 288 small ones, the cheaper up to
# about 1200 tokens
@pytest.mark.parametrize("case", [(2048, 0.0), (2003, 1.0), (1804, 0.0), (1100, 0.0)])
def test_medium_tile_weight_gradients(s24, dtype, case):
    p, beta = case
    lam, d, f = 2e-4, 752, 3056
    shapes = [(d, f), (f, d)]
    dY = [si.random_matrix(90 + i, (p, r), 1e-2, dtype) for i, (r, q) in enumerate(shapes)]
    X = [si.random_matrix(92 + i, (p, q), 1.0, dtype) for i, (r, q) in enumerate(shapes)]
    W = [si.random_matrix(94 + i, sh, 0.02, dtype) for i, sh in enumerate(shapes)]
    dW0 = [si.random_matrix(96 + i, sh, 1e-3, "f32") for i, sh in enumerate(shapes)]
    masks = [oracle.transposable_mask(w) for w in W]
    got = [dev(w).clone() for w in dW0]
    probs = [(dev_bf16(dY[i]), dev_bf16(X[i]), got[i], dev_bf16(W[i]), dev(masks[i]), lam) for i in range(2)]
    assert tiles_run(lambda: s24.dense_dw_batch(probs, beta=beta)) == [(4, 2, 32) if p > 1200 else (2, 2, 32)]
    plain = [dev(w).clone() for w in dW0]
    s24.dense_dw_batch([(dev_bf16(dY[i]), dev_bf16(X[i]), plain[i], None, None, 0.0) for i in range(2)], beta=beta)
    for i, (r, q) in enumerate(shapes):
        rows = np.unique(np.concatenate([[0, 63, 64, 127, 128, 255, 256, r - 1], np.random.default_rng(i).integers(0, r, 40)]))
        ref = si.to_f32(dY[i])[:, rows].astype(np.float64).T @ si.to_f32(X[i]).astype(np.float64) + beta * dW0[i][rows].astype(np.float64)
        assert_close(host_f64(plain[i])[rows], ref, tol_for(dtype), f"dense_dw_batch {case} {i}")
        two = plain[i].clone()
        s24.masked_decay_grad(two, dev_bf16(W[i]), dev(masks[i]), lam)     # the decay's bits are the separate kernel's
        assert torch.equal(got[i].view(torch.int32), two.view(torch.int32))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
# no more tiles of 192 x 128 than compute units (192 and 248); whole chunks and remainders of one and of 31 tokens; ragged both ways
@pytest.mark.parametrize("p,d,f,beta", [(3264, 752, 3056, 0.0), (3201, 752, 3056, 1.0), (3231, 960, 3056, 0.0)])
def test_weight_gradients_on_the_192_row_tile(s24, dtype, p, d, f, beta):
    td = torch_dtype(dtype)
    g = torch.Generator(device="cuda").manual_seed(p)
    rnd = lambda sh, std: (torch.randn(sh, generator=g, device="cuda") * std).to(td)
    probs = []
    for r, q in [(d, f), (f, d)]:
        W, mask = rnd((r, q), 0.02), torch.empty((r // 4, q // 4), dtype=torch.int16, device="cuda")
        s24.transposable_mask(W, mask)
        probs.append((rnd((p, r), 1e-2), rnd((p, q), 1.0), torch.full((r, q), 1e-3, device="cuda"), W, mask, 2e-4))
    assert tiles_run(lambda: s24.dense_dw_batch(probs, beta=beta)) == [(3, 2, 32)]
    for dY, X, dW, W, mask, lam in probs:
        alone = torch.full_like(dW, 1e-3)      # other tiles, which are compared with the definition elsewhere: the same bits
        s24.dense_dw_decay(dY, X, alone, W, mask, lam, beta=beta)
        assert torch.equal(dW.view(torch.int32), alone.view(torch.int32))
        ref = dY.double().t() @ X.double() + beta * 1e-3
        keep = torch.stack([(mask.to(torch.int32) >> t) & 1 for t in range(16)], -1).view(*mask.shape, 4, 4).permute(0, 2, 1, 3).reshape(dW.shape)
        ref += lam * W.double() * (1 - keep)
        assert float((dW.double() - ref).norm() / ref.norm()) < 1e-5   # sums of 3200 products in fp32


# ------------------------------------------------------------------ dense products on the smaller tiles
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
# the 128 x 128 tile and the 256 x 128 one (136 of them), ragged both ways; 2, 4, 6 and 10 chunks of 32 against a ring of four
@pytest.mark.parametrize("pr", [(1, 16), (130, 144), (2050, 2032)])
@pytest.mark.parametrize("q", [64, 128, 192, 320])
def test_dense_product_tiles(s24, dtype, pr, q):
    p, r = pr
    X, W = si.random_matrix(100 + p, (p, q), 1.0, dtype), si.random_matrix(101 + r, (r, q), 0.02, dtype)
    Y = torch.full((p, r), 7.0, dtype=torch_dtype(dtype), device="cuda")
    x, w = dev_bf16(X), dev_bf16(W)
    assert tiles_run(lambda: s24.dense_gemm(x, w, Y)) == [(4, 2) if p == 2050 else (2, 2)]
    rows = np.unique(np.concatenate([[0, p - 1], np.random.default_rng(p).integers(0, p, 40), np.arange(min(p, 260))]))
    ref = si.to_f32(X)[rows].astype(np.float64) @ si.to_f32(W).astype(np.float64).T
    assert_close(host_f64(Y)[rows], ref, tol_for(dtype), f"dense_gemm {pr} {q}")


# ------------------------------------------------------------------ sparse weight gradients by size of the output
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
# 128 x 128, 256 x 128 (136 of them), 256 x 256 tiles (256 of them) and, a column more, 128 x 128 again; ragged both ways; one,
# three and four chunks against a ring of three
@pytest.mark.parametrize("rq", [(144, 272), (2032, 2064), (4080, 4080), (4080, 4112)])
@pytest.mark.parametrize("p,beta", [(64, 0.0), (192, 1.0), (256, 0.0)])
def test_sparse_weight_gradient_tiles(s24, dtype, rq, p, beta):
    (r, q), lam = rq, 2e-4
    dY, X = si.random_matrix(110 + p, (p, r), 1e-2, dtype), si.random_matrix(111 + p, (p, q), 1.0, dtype)
    W, dW0 = si.random_matrix(112 + r, (r, q), 0.02, dtype), si.random_matrix(113 + r, (r, q), 1e-3, "f32")
    mask = oracle.transposable_mask(W)
    vz, mz = oracle.mvue24(dY, 7)
    v, m = oracle.pack(vz, mz)
    plain, decayed = dev(dW0).clone(), dev(dW0).clone()
    vd, md, x = dev_bf16(v), dev(m), dev_bf16(X)
    assert tiles_run(lambda: s24.spmm_dw(vd, md, x, plain, beta=beta)) == [{272: (2, 2), 2064: (4, 2), 4080: (4, 4), 4112: (2, 2)}[q]]
    s24.spmm_dw(dev_bf16(v), dev(m), dev_bf16(X), decayed, beta=beta, W=dev_bf16(W), mask=dev(mask), lam=lam)
    rows = np.unique(np.concatenate([[0, r - 1], np.random.default_rng(r).integers(0, r, 40), np.arange(min(r, 130))]))
    rows = np.resize(rows, (rows.size + 15) // 16 * 16)     # the oracle takes multiples of 16: the first ones again
    ref = oracle.spmm_fwd(np.ascontiguousarray(X.T), np.ascontiguousarray(vz[rows]), np.ascontiguousarray(mz[rows])).T + beta * dW0[rows].astype(np.float64)
    assert_close(host_f64(plain)[rows], ref, tol_for(dtype), f"spmm_dw {rq} {p}")
    two = plain.clone()
    s24.masked_decay_grad(two, dev_bf16(W), dev(mask), lam)
    assert torch.equal(decayed.view(torch.int32), two.view(torch.int32))


# one lane, a vector and a remainder, the four-vector pass and what it leaves, more vectors than 256 workgroups take in one
# pass, and with per-block counts more than they take in eight
@pytest.mark.parametrize("n", [1, 7, 8, 8193, 32768, 40970, 2097152 + 8 * 300 + 5, 4194304 + 21])
def test_mask_flips_by_size(s24, n):
    rng = np.random.default_rng(n)
    a, b = rng.integers(0, 65536, n).astype(np.uint16), rng.integers(0, 65536, n).astype(np.uint16)
    flips, per = torch.full((1,), 9, dtype=torch.int64, device="cuda"), torch.ones(n, dtype=torch.int32, device="cuda")
    s24.mask_flips(dev(a), dev(b), flips, per)
    want = np.unpackbits((a ^ b).view(np.uint8).reshape(n, 2), axis=1).sum(1)
    assert flips.item() == want.sum() and np.array_equal(per.cpu().numpy(), 1 + want.astype(np.int32))
    s24.mask_flips(dev(a), dev(b), flips)
    assert flips.item() == want.sum()


def test_gated_backward_of_few_tokens_and_many_features_keeps_the_plain_products_bits(s24):
    p, f, r = 13, 49152, 64                  # 192 large tiles of one row: the fused epilogue, and a plain product of few tokens
    dY, Wd = si.random_matrix(120, (p, r), 1e-2, "bf16"), si.random_matrix(121, (r, f), 0.02, "bf16")
    vt, mt = oracle.pack(*oracle.compress(Wd, oracle.transposable_mask(Wd))[2:])
    GU = dev_bf16(si.random_matrix(122, (p, 2 * f), 1.0, "bf16"))
    dH, dGU, two = torch.empty((p, f), dtype=torch.bfloat16, device="cuda"), torch.empty_like(GU), torch.empty_like(GU)
    s24.spmm_bwd_dx_glu(dev_bf16(dY), dev_bf16(vt), dev(mt), GU, dGU, s24.GATE_SILU)
    s24.spmm_bwd_dx(dev_bf16(dY), dev_bf16(vt), dev(mt), dH)
    s24.glu_bwd(dH, GU, two, s24.GATE_SILU)
    assert torch.equal(dGU.view(torch.int16), two.view(torch.int16))


def test_backward_of_few_tokens_and_many_features_keeps_the_plain_products_bits(s24):
    # 192 large tiles of one row: the fused gated epilogue takes them, at a token count that the slices are for; ten chunks,
    # so that the slices would sum in another order
    p, f, r = 13, 49152, 640
    dY, Wd = si.random_matrix(120, (p, r), 1e-2, "bf16"), si.random_matrix(121, (r, f), 0.02, "bf16")
    vt, mt = oracle.pack(*oracle.compress(Wd, oracle.transposable_mask(Wd))[2:])
    dY, vt, mt = dev_bf16(dY), dev_bf16(vt), dev(mt)
    GU = dev_bf16(si.random_matrix(122, (p, 2 * f), 1.0, "bf16"))
    dH, dGU, two = torch.empty((p, f), dtype=torch.bfloat16, device="cuda"), torch.empty_like(GU), torch.empty_like(GU)
    s24.spmm_bwd_dx(dY, vt, mt, dH)
    s24.spmm_bwd_dx_glu(dY, vt, mt, GU, dGU, s24.GATE_SILU)
    s24.glu_bwd(dH, GU, two, s24.GATE_SILU)
    assert torch.equal(dGU.view(torch.int16), two.view(torch.int16))
    Z = GU[:, :f].contiguous()
    dZ, two = torch.empty_like(Z), torch.empty_like(Z)
    for act in (s24.ACT_RELU, s24.ACT_GELU_ERF):
        s24.spmm_bwd_dx_act(dY, vt, mt, Z, dZ, act)
        s24.act_bwd(dH, Z, two, act)
        assert torch.equal(dZ.view(torch.int16), two.view(torch.int16))


# ------------------------------------------------------------------ 16-bit weight gradients of ragged token counts
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
# fewer tokens than one 32-token step of the contraction, and two to four steps with a remainder
@pytest.mark.parametrize("p", [1, 31, 33, 48, 63, 70, 100])
def test_weight_gradient_of_a_ragged_token_count_keeps_infinities(s24, dtype, p):
    """Tokens that a ragged chunk holds twice, or holds instead of ones past the last, contribute nothing."""
    r, q = 768, 3072     # alone 144 small tiles, 64 tokens to a stage; as a pair 288 of them, 32 to a stage
    dY, X = dev_bf16(si.random_matrix(160 + p, (p, r), 1e-2, dtype)), dev_bf16(si.random_matrix(161 + p, (p, q), 1.0, dtype))
    dY[dY == 0] = 1.0    # zero times infinity is another case
    at = {5: p - 1, 6: max(p - 20, 0), 7: max(p - 40, 0), 8: 0}
    for col, t in at.items():
        X[t, col] = float("inf")
    single, pair = torch.zeros((r, q), device="cuda"), [torch.zeros((r, q), device="cuda") for _ in range(2)]
    s24.dense_dw(dY, X, single)
    s24.dense_dw_batch([(dY, X, dW, None, None, 0.0) for dW in pair])
    for dW in (single, *pair):
        for col, t in at.items():
            assert torch.equal(dW[:, col], torch.copysign(torch.full((r,), float("inf"), device="cuda"), dY[t].float())), (p, t)
        assert torch.isfinite(dW[:, 9:]).all()


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
# (p, rq, rq of the problem beside it, tiles alone, tiles in the pair): small tiles alone (64 tokens to a stage) against small (32) and medium tiles in the
# pair, with a last stage that holds part of one 32-token step or of both; medium tiles alone and large ones in the pair; and
# an output whose last columns run in small tiles beside large ones, alone one column of large tiles wide, in the pair two
@pytest.mark.parametrize("case", [(p, (768, 3072), (3072, 768), [(2, 2, 64)], [(2, 2, 32)]) for p in (17, 33, 48, 57, 63, 64, 70, 90, 97, 112, 121, 127, 191)] +
                         [(3001, (768, 3072), (3072, 768), [(2, 2, 64)], [(4, 2, 32)])] +
                         [(5537, (1408, 3776), (3776, 1408), [(4, 2, 32)], [(4, 4, 32)])] +
                         [(p, (2048, 8448), (2048, 8448), [(4, 4, 32), (2, 2, 64)], [(4, 4, 32), (2, 2, 64)]) for p in (97, 112, 3001)])
def test_weight_gradients_have_the_same_bits_in_every_tile(s24, dtype, case):
    p, a, b, tiles_alone, tiles_pair = case
    gen = torch.Generator(device="cuda").manual_seed(p)
    rnd = lambda n, std: (torch.randn((p, n), generator=gen, device="cuda") * std).to(torch_dtype(dtype))
    probs = [(rnd(r, 1e-2), rnd(q, 1.0), torch.zeros((r, q), device="cuda"), None, None, 0.0) for r, q in (a, b)]
    assert tiles_run(lambda: s24.dense_dw_batch(probs)) == tiles_pair
    for dY, X, dW, *_ in probs:
        alone = torch.zeros_like(dW)
        assert tiles_run(lambda: s24.dense_dw(dY, X, alone)) == tiles_alone
        assert torch.equal(alone.view(torch.int32), dW.view(torch.int32)), case
        rows = torch.cat([torch.arange(0, dW.shape[0], 61), torch.tensor([dW.shape[0] - 1])])
        ref = host_f64(dY)[:, rows.numpy()].T @ host_f64(X)
        assert_close(host_f64(dW)[rows.numpy()], ref, F32_TOL, f"dense_dw_batch {case}")


# ------------------------------------------------------------------ the last input gradient and the weight gradients in one call
def backward_operands(s24, p, q, r, dtype, seed, f=None):
    """Of a layer q -> r -> q on p tokens (gated: r -> f between): the compressed transpose of its first weight, the gradient there, and the two
    weight gradients."""
    f = f or r
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch_dtype(dtype)
    rnd = lambda *shape: torch.randn(shape, generator=gen, device="cuda").to(dt)
    new = lambda *shape, t=dt: torch.full(shape, 7, dtype=t, device="cuda")
    W1, W2, X, H, dY, dZ = rnd(r, q), rnd(q, f), rnd(p, q), rnd(p, f), rnd(p, q), rnd(p, r)
    masks, ops = [], []
    for W in (W1, W2):
        a, b = W.shape
        o = new(b // 64, a, 32), new(b // 64, a, 4, t=torch.int16), new(a // 64, b, 32), new(a // 64, b, 4, t=torch.int16)
        masks.append(new(a // 4, b // 4, t=torch.int16))
        s24.compress(W, None, *o, mask_out=masks[-1])
        ops.append(o)
    grads = [new(q, f, t=torch.float32), new(r, q, t=torch.float32)]
    problems = lambda decay: [(dY, H, grads[0], W2 if decay else None, masks[1] if decay else None, 1e-3),
                              (dZ, X, grads[1], W1 if decay else None, masks[0] if decay else None, 1e-3)]
    return dZ, ops[0][2], ops[0][3], new(p, q), grads, problems, X


# fp32 (p, q, r): 32-tiles in eight slices with four, one and two batches of tokens in flight; a chain of a few tokens and a contraction of four slices, which
# run in turn; ragged in every direction
BACKWARD = [("f32", s, k and ("f32", k)) for s, k in [((512, 256, 1024), 4), ((100, 128, 512), 1), ((1200, 192, 576), 4), ((1200, 192, 1344), 2), ((7, 64, 512), None),
                                                      ((130, 64, 448), None), ((515, 320, 1088), 1)]]
# 16-bit: slices of four, two and one row blocks; one token, less than a step of 32, a step and a rest, a ring of whole steps, many whole steps and a
# rest of one token
BACKWARD += [("bf16", s, ("slices", k)) for s, k in [((256, 768, 3072), 4), ((200, 512, 1344), 2), ((1, 64, 128), 1), ((128, 128, 448), 1), ((704, 128, 448), 2), ((705, 128, 448), 2)]]
BACKWARD += [("f16", s, ("slices", k)) for s, k in [((100, 512, 1408), 1), ((31, 256, 1024), 1), ((257, 320, 1088), 2)]]

# 16-bit, whole grids (p, q, r, f): tiles of 192 x 128, of 256 x 256 in a part of a round and in two and a strip, of 256 x 128; ragged in every direction
BACKWARD += [("bf16", s, ("grid", *k, 32)) for s, k in [((8192, 768, 3072), (3, 2)), ((2475, 1408, 3776), (4, 4)), ((3001, 2048, 11008, 5504), (4, 4)), ((3083, 576, 4608, 2304), (4, 2))]]
BACKWARD += [("f16", s, ("grid", *k, 32)) for s, k in [((5939, 896, 2368), (3, 2)), ((1795, 640, 4480, 2240), (4, 2))]]


def compare_with_two_calls(s24, dZ, vT, mT, dX, problems, variant):
    """One call in the expected variant against the two that it stands for: the same bits."""
    outputs = [dX, *(pr[2] for pr in problems)]
    kept = [t.clone() for t in outputs]
    assert joint_run(lambda: s24.spmm_bwd_dx_dw(dZ, vT, mT, dX, problems)) == variant
    got = [t.clone() for t in outputs]
    for t, k in zip(outputs, kept):
        t.copy_(k)
    s24.spmm_bwd_dx(dZ, vT, mT, dX)
    tiles = tiles_run(lambda: s24.dense_dw_batch(problems))
    for a, b in zip(got, outputs):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    if variant and variant[0] == "grid":   # priced as the tile that the gradients take by themselves (their strip, if they have one, comes second)
        assert variant[1:] == tiles[0]


@pytest.mark.parametrize("decay", [True, False])
@pytest.mark.parametrize("dtype, pqr, variant", BACKWARD)
def test_input_and_weight_gradients_in_one_call_have_the_bits_of_two(s24, dtype, pqr, variant, decay):
    p, q, r, *f = pqr
    dZ, vT, mT, dX, grads, problems, _ = backward_operands(s24, p, q, r, dtype, p + r, *f)
    compare_with_two_calls(s24, dZ, vT, mT, dX, problems(decay), variant)


# a gradient alone, three and four of them
@pytest.mark.parametrize("dtype, pqr, count, variant", [("f32", (512, 256, 1024), 1, ("f32", 4)), ("f32", (512, 256, 1024), 3, ("f32", 1)), ("f32", (100, 128, 512), 4, ("f32", 1)),
                                                        ("bf16", (256, 768, 3072), 1, ("slices", 4)), ("bf16", (200, 512, 1344), 3, ("slices", 2)), ("f16", (100, 512, 1408), 4, ("slices", 1)),
                                                        ("bf16", (8192, 768, 3072), 1, None), ("bf16", (4097, 768, 2048), 3, ("grid", 3, 2, 32)), ("f16", (4097, 768, 2048), 4, ("grid", 4, 2, 32))])
def test_one_to_four_weight_gradients_beside_an_input_gradient(s24, dtype, pqr, count, variant):
    dZ, vT, mT, dX, grads, problems, _ = backward_operands(s24, *pqr, dtype, 7)
    more = [(*pr[:2], torch.empty_like(pr[2]), *pr[3:]) for pr in problems(True)]
    compare_with_two_calls(s24, dZ, vT, mT, dX, (problems(True) + more)[:count], variant)


@pytest.mark.parametrize("dtype, pqr, odd", [(*c, o) for c in (("f32", (512, 256, 1024)), ("bf16", (256, 768, 3072)), ("bf16", (8192, 768, 3072))) for o in ("decay on one", "an empty one")] +
                         [("f32", (512, 256, 1024), "one gradient twice")])   # 16-bit problems of one grid must not overlap
def test_gradients_that_share_no_grid_run_in_turn(s24, dtype, pqr, odd):
    dZ, vT, mT, dX, grads, problems, X = backward_operands(s24, *pqr, dtype, 9)
    first, second = problems(True)
    if odd == "decay on one":
        second = (*second[:3], None, None, 0.0)
    elif odd == "an empty one":
        second = (dZ, X[:, :0].contiguous(), second[2][:, :0].contiguous(), *second[3:])
    else:
        second = (2 * first[0], *first[1:])
    compare_with_two_calls(s24, dZ, vT, mT, dX, [first, second], None)


@pytest.mark.parametrize("dtype, pqr", [("f32", (512, 256, 1024)), ("bf16", (256, 768, 3072)), ("bf16", (8192, 768, 3072))])
@pytest.mark.parametrize("over", ["X", "H", "dY"])
def test_an_input_gradient_over_an_operand_of_a_weight_gradient_comes_first(s24, dtype, pqr, over):
    """In place of what a weight gradient reads: as the two calls in their order."""
    dZ, vT, mT, dX, grads, problems, X = backward_operands(s24, *pqr, dtype, 5)
    target = {"X": X, "H": problems(True)[0][1].view(-1)[:X.numel()].view(X.shape), "dY": problems(True)[0][0]}[over]
    kept = target.clone()
    s24.spmm_bwd_dx(dZ, vT, mT, target)
    s24.dense_dw_batch(problems(True))
    want = [t.clone() for t in (target, *grads)]
    target.copy_(kept)
    assert joint_run(lambda: s24.spmm_bwd_dx_dw(dZ, vT, mT, target, problems(True))) is None
    for a, b in zip(want, (target, *grads)):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))

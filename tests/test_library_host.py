"""CPU-side checks of the HIP library: it loads without a GPU, exports every
symbol include/s24.h declares, and rejects bad arguments on the host before
anything is launched.  No kernel runs here."""
import ctypes as C
import functools
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    import paper_2404_01847_amd as s24
    if not os.path.exists(s24.lib_path()):
        from paper_2404_01847_amd.build import build
        build(verbose=False)
    return s24.lib()


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "s24.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(s24_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(lib):
    names = declared_symbols()
    assert len(names) >= 13
    for n in names:
        assert hasattr(lib, n), n
    from paper_2404_01847_amd import binding
    assert sorted(binding.EXPORTS) == names


def test_pattern_table_is_the_lexicographic_enumeration(lib, legal_blocks):
    import paper_2404_01847_amd as s24
    assert s24.pattern_table() == legal_blocks


def test_strerror_covers_all_codes(lib):
    import paper_2404_01847_amd as s24
    texts = {s24.strerror(c) for c in range(0, -7, -1)}
    assert len(texts) == 7 and "ok" in texts
    assert "unknown" in s24.strerror(-99)


OK, NULL, SHAPE, DTYPE, ALIGN, UNSUP = 0, -1, -2, -3, -4, -6
P = 0x1000  # a fake, well-aligned device address: validation never dereferences it


def test_mask_argument_errors(lib):
    f = lib.s24_transposable_mask
    assert f(None, 1, 8, 8, 8, P, None, None) == NULL
    assert f(P, 1, 8, 8, 8, None, None, None) == NULL
    assert f(P, 7, 8, 8, 8, P, None, None) == DTYPE
    assert f(P, 1, 6, 8, 8, P, None, None) == SHAPE
    assert f(P, 1, 8, 10, 12, P, None, None) == SHAPE
    assert f(P, 1, -4, 8, 8, P, None, None) == SHAPE
    assert f(P, 1, 8, 8, 4, P, None, None) == SHAPE          # ldw < q
    assert f(P + 2, 1, 8, 8, 8, P, None, None) == ALIGN
    assert f(P, 1, 8, 8, 10, P, None, None) == ALIGN          # row stride not a multiple of 8 bytes
    assert f(P + 8, 0, 8, 8, 8, P, None, None) == ALIGN       # fp32 rows need 16 bytes
    assert f(P, 1, 0, 8, 8, P, None, None) == OK              # empty: nothing to do


def test_compress_batch_argument_errors(lib):
    from paper_2404_01847_amd.binding import _CompressProblem
    good = _CompressProblem(P, None, P, P, P, P, None, 64, 64, 64)

    def f(*problems, count=None, dt=1):
        return lib.s24_compress_batch((_CompressProblem * max(len(problems), 1))(*problems), len(problems) if count is None else count, dt, None)

    changed = lambda **kw: _CompressProblem(*[kw.get(n, getattr(good, n)) for n, _ in _CompressProblem._fields_])
    assert f(count=0) == OK and lib.s24_compress_batch(None, 1, 1, None) == NULL
    assert f(good, count=-1) == SHAPE and f(*[good] * 5) == SHAPE and f(good, dt=7) == DTYPE
    assert f(good, changed(q=72)) == SHAPE and f(good, changed(valsT=None)) == NULL and f(good, changed(vals=P + 8)) == ALIGN
    assert f(good, changed(mask=P)) == UNSUP                   # searched and given masks do not mix
    assert f(changed(r=0, W=None), changed(q=0, mask=P)) == OK   # empty weights are skipped
    import paper_2404_01847_amd as s24
    assert s24.compress_batch([]) is None                      # no weights: nothing to do, as in the C call


def test_compress_argument_errors(lib):
    f = lib.s24_compress
    assert f(P, 1, 64, 64, 64, None, None, P, P, P, None, None) == NULL
    assert f(P, 1, 64, 96, 96, None, P, P, P, P, None, None) == SHAPE    # q not a multiple of 64
    assert f(P, 1, 16, 64, 64, None, P, P, P, P, None, None) == SHAPE    # r not a multiple of 64
    assert f(P, 1, 64, 64, 64, None, P + 4, P, P, P, None, None) == ALIGN
    assert f(P, 1, 0, 64, 64, None, P, P, P, P, None, None) == OK


def test_gemm_argument_errors(lib):
    assert lib.s24_spmm_fwd(P, P, P, P, 4, 96, 16, 1, None) == SHAPE          # q % 64
    assert lib.s24_spmm_fwd(P, P, P, P, 4, 64, 24, 1, None) == SHAPE          # r % 16
    assert lib.s24_spmm_fwd(P, P, None, P, 4, 64, 16, 1, None) == NULL
    assert lib.s24_spmm_fwd(P, P, P, P + 2, 4, 64, 16, 1, None) == ALIGN
    assert lib.s24_spmm_fwd(P, P, P, P, 4, 64, 16, 3, None) == DTYPE
    assert lib.s24_spmm_fwd(P, P, P, P, 0, 64, 16, 1, None) == OK
    assert lib.s24_spmm_fwd_swiglu(P, P, P, P, P, 4, 96, 16, 1, None) == SHAPE      # q % 64
    assert lib.s24_spmm_fwd_swiglu(P, P, P, P, P, 4, 64, 24, 1, None) == SHAPE      # f % 16
    assert lib.s24_spmm_fwd_swiglu(P, P, P, P, None, 4, 64, 16, 1, None) == NULL
    assert lib.s24_spmm_fwd_swiglu(P, P, P, P, P, 0, 64, 16, 1, None) == OK
    assert lib.s24_spmm_bwd_dx_swiglu(P, P, P, P, P, 4, 16, 96, 1, None) == SHAPE   # r % 64
    assert lib.s24_spmm_bwd_dx_swiglu(P, P, P, None, P, 4, 16, 64, 1, None) == NULL
    assert lib.s24_spmm_bwd_dx_swiglu(P, P, P, P, P, 4, 16, 64, 1, None) == UNSUP   # too few tiles for the fused kernel
    assert lib.s24_spmm_bwd_dx_swiglu(P, P, P, P, P, 4, 16, 64, 0, None) == UNSUP   # fp32
    assert lib.s24_spmm_bwd_dx(P, P, P, P, 4, 16, 96, 0.0, 1, None) == SHAPE  # r % 64
    assert lib.s24_spmm_bwd_dx(P, P, P, P, 4, 16, 64, 0.5, 1, None) == UNSUP  # beta must be 0 or 1
    assert lib.s24_dense_dw(P, P, P, 4, 24, 16, 0.0, 1, None) == SHAPE
    assert lib.s24_dense_dw(P, P, P, 4, 16, 16, 2.0, 1, None) == UNSUP
    assert lib.s24_dense_dw(P, None, P, 4, 16, 16, 0.0, 1, None) == NULL
    assert lib.s24_dense_dw_decay(P, P, P, P, 1, P, 1e-4, 4, 24, 16, 0.0, 1, None) == SHAPE
    assert lib.s24_dense_dw_decay(P, P, P, None, 1, P, 1e-4, 4, 16, 16, 0.0, 1, None) == NULL
    assert lib.s24_dense_dw_decay(P, P, P, P, 7, P, 1e-4, 4, 16, 16, 0.0, 1, None) == DTYPE
    assert lib.s24_dense_dw_decay(P, P, P, P, 1, P + 2, 1e-4, 4, 16, 16, 0.0, 1, None) == ALIGN
    assert lib.s24_dense_dw_decay(P, P, P, P, 1, P, 1e-4, 4, 16, 0, 0.0, 1, None) == OK
    assert lib.s24_dense_gemm(P, P, P, 4, 32, 16, 1, None) == SHAPE
    assert lib.s24_dense_gemm(P, P, P, 0, 64, 16, 1, None) == OK
    # feature extents at or beyond 2^23 (32-bit byte offsets inside a tile) and token counts at or beyond 2^31
    big = 1 << 23
    assert lib.s24_spmm_fwd(P, P, P, P, 4, big, 16, 1, None) == SHAPE
    assert lib.s24_spmm_fwd(P, P, P, P, 4, 64, big, 1, None) == SHAPE
    assert lib.s24_spmm_bwd_dx(P, P, P, P, 4, big, 64, 0.0, 1, None) == SHAPE
    assert lib.s24_dense_dw(P, P, P, 4, big, 16, 0.0, 1, None) == SHAPE
    assert lib.s24_dense_gemm(P, P, P, 1 << 31, 64, 16, 1, None) == SHAPE
    # the compressed operands' alignment is what the kernels' 16- and 8-byte stores need
    assert lib.s24_compress(P, 1, 64, 64, 64, None, P + 8, P, P, P, None, None) == ALIGN
    assert lib.s24_compress(P, 1, 64, 64, 64, None, P, P + 2, P, P, None, None) == ALIGN
    assert lib.s24_compress(P, 1, 64, 64, 64, None, P, P, P, P + 4, None, None) == ALIGN


def test_probe_argument_errors(lib):
    assert lib.s24_probe_matrix_rate(0, -1, 8, P, None) == SHAPE
    assert lib.s24_probe_matrix_rate(1, 4, 8, None, None) == NULL
    assert lib.s24_probe_matrix_rate(0, 0, 8, None, None) == OK
    assert lib.s24_probe_copy(P, P, 24, None) == SHAPE
    assert lib.s24_probe_copy(P, None, 32, None) == NULL
    assert lib.s24_probe_copy(P + 4, P, 32, None) == ALIGN
    assert lib.s24_probe_copy(None, None, 0, None) == OK
    assert lib.s24_probe_reciprocal(1, -1, P, None) == SHAPE and lib.s24_probe_reciprocal(1, 1 << 32, P, None) == SHAPE
    assert lib.s24_probe_reciprocal(1, 5, None, None) == NULL and lib.s24_probe_reciprocal(1, 5, P + 4, None) == ALIGN
    assert lib.s24_probe_reciprocal(0, 0, None, None) == OK


def test_mvue_argument_errors(lib):
    assert lib.s24_mvue24(P, 1, 96, 16, 16, 1, P, P, None) == SHAPE            # p % 64
    assert lib.s24_mvue24(P, 1, 64, 16, 8, 1, P, P, None) == SHAPE             # ld < r
    assert lib.s24_mvue24(P, 4, 64, 16, 16, 1, P, P, None) == DTYPE
    assert lib.s24_mvue24(P, 1, 64, 16, 16, 1, None, P, None) == NULL
    assert lib.s24_mvue24(P, 1, 64, 16, 16, 1, P + 8, P, None) == ALIGN
    assert lib.s24_mvue24(P, 1, 0, 16, 16, 1, None, None, None) == OK
    assert lib.s24_spmm_dw(P, P, P, P, None, 1, None, 0.0, 96, 16, 16, 0.0, 1, None) == SHAPE
    assert lib.s24_spmm_dw(P, P, P, P, None, 1, None, 0.0, 64, 16, 16, 0.5, 1, None) == UNSUP
    assert lib.s24_spmm_dw(P, None, P, P, None, 1, None, 0.0, 64, 16, 16, 0.0, 1, None) == NULL
    assert lib.s24_spmm_dw(P, P, P, P, P, 1, None, 1e-4, 64, 16, 16, 0.0, 1, None) == NULL    # decay without a mask
    assert lib.s24_spmm_dw(P, P, P, P, None, 1, None, 0.0, 64, 16, 0, 0.0, 1, None) == OK


def test_monitor_argument_errors(lib):
    assert lib.s24_mask_flips(P, P, -1, None, P, None) == SHAPE
    assert lib.s24_mask_flips(P, P, 16, None, None, None) == NULL
    assert lib.s24_mask_flips(P, P, 16, None, P + 4, None) == ALIGN
    assert lib.s24_l1_norm_gap(P, 1, 6, 8, 8, P, None) == SHAPE
    assert lib.s24_l1_norm_gap(P, 9, 8, 8, 8, P, None) == DTYPE
    assert lib.s24_l1_norm_gap(P, 1, 8, 8, 8, None, None) == NULL
    assert lib.s24_l1_norm_gap(P, 1, 0, 8, 8, None, None) == OK


def test_elementwise_argument_errors(lib):
    assert lib.s24_masked_decay_grad(P, P, 1, None, 1e-4, 16, 16, None) == NULL
    assert lib.s24_masked_decay_grad(P, P, 1, P, 1e-4, 16, 24, None) == SHAPE
    assert lib.s24_masked_decay_grad(P + 4, P, 1, P, 1e-4, 16, 16, None) == ALIGN
    assert lib.s24_masked_decay_grad(P, P, 5, P, 1e-4, 16, 16, None) == DTYPE
    assert lib.s24_swiglu_fwd(P, P, P, 4, 12, 16, 1, None) == SHAPE
    assert lib.s24_swiglu_fwd(P, P, P, 4, 16, 8, 1, None) == SHAPE            # ld < f
    assert lib.s24_swiglu_fwd(P, None, P, 4, 16, 16, 1, None) == NULL
    assert lib.s24_swiglu_bwd(P, P, P, P, None, 4, 16, 16, 1, None) == NULL
    assert lib.s24_swiglu_bwd(P, P, P, P, P + 8, 4, 16, 16, 1, None) == ALIGN
    assert lib.s24_act_fwd(P, P, 12, 0, 1, None) == SHAPE
    assert lib.s24_act_fwd(P, P, 16, 9, 1, None) == DTYPE
    assert lib.s24_act_bwd(P, P, None, 16, 0, 1, None) == NULL
    assert lib.s24_act_fwd(P, P, 0, 0, 1, None) == OK


def test_gated_family_argument_errors(lib):
    R, Cm = 0, 1
    # s24_glu_fwd(Z, lz, ldz, H, lh, ldh, p, f, gate, dt, stream)
    assert lib.s24_glu_fwd(P, R, 32, P, R, 16, 4, 12, 1, 2, None) == SHAPE             # f % 8
    assert lib.s24_glu_fwd(P, R, 24, P, R, 16, 4, 16, 1, 2, None) == SHAPE             # ldz < 2f
    assert lib.s24_glu_fwd(P, Cm, 8, P, R, 16, 4, 16, 1, 2, None) == SHAPE             # column-major needs p % 8
    assert lib.s24_glu_fwd(P, Cm, 4, P, Cm, 8, 8, 16, 1, 2, None) == SHAPE             # ldz < p
    assert lib.s24_glu_fwd(P, 2, 32, P, R, 16, 4, 16, 1, 2, None) == DTYPE             # layout enum
    assert lib.s24_glu_fwd(P, R, 32, P, R, 16, 4, 16, 5, 2, None) == DTYPE             # gate enum
    assert lib.s24_glu_fwd(P, R, 32, P, R, 16, 4, 16, 1, 3, None) == DTYPE
    assert lib.s24_glu_fwd(None, R, 32, P, R, 16, 4, 16, 1, 2, None) == NULL
    assert lib.s24_glu_fwd(P + 8, R, 32, P, R, 16, 4, 16, 1, 2, None) == ALIGN
    assert lib.s24_glu_fwd(None, R, 32, None, R, 16, 0, 16, 1, 2, None) == OK
    # s24_glu_bwd(dH, lh, ldh, Z, lz, ldz, dZ, p, f, gate, dt, stream)
    assert lib.s24_glu_bwd(P, R, 16, P, R, 32, None, 4, 16, 0, 1, None) == NULL
    assert lib.s24_glu_bwd(P, R, 8, P, R, 32, P, 4, 16, 0, 1, None) == SHAPE           # ldh < f
    assert lib.s24_glu_bwd(P, Cm, 8, P, R, 32, P, 4, 16, 0, 1, None) == SHAPE          # mixed layouts need p % 8
    assert lib.s24_glu_bwd(P, R, 16, P, R, 32, P + 2, 4, 16, 0, 1, None) == ALIGN
    # s24_bias_grad(dZ, layout, ld, p, n, db, beta, dt, stream)
    assert lib.s24_bias_grad(P, R, 16, 4, 12, P, 0.0, 1, None) == SHAPE                # n % 8
    assert lib.s24_bias_grad(P, R, 8, 4, 16, P, 0.0, 1, None) == SHAPE                 # ld < n
    assert lib.s24_bias_grad(P, Cm, 8, 4, 16, P, 0.0, 1, None) == SHAPE                # column-major needs p % 8
    assert lib.s24_bias_grad(P, R, 16, 4, 16, P, 0.5, 1, None) == UNSUP
    assert lib.s24_bias_grad(P, R, 16, 4, 16, None, 0.0, 1, None) == NULL
    assert lib.s24_bias_grad(P, R, 16, 4, 16, P + 2, 0.0, 1, None) == ALIGN
    assert lib.s24_bias_grad(P, R, 16, 4, 16, P, 0.0, 8, None) == DTYPE
    assert lib.s24_bias_grad(None, R, 16, 4, 0, None, 0.0, 1, None) == OK
    # s24_spmm_fwd_bias(X, vals, meta, bias, Y, p, q, r, dt, stream)
    assert lib.s24_spmm_fwd_bias(P, P, P, P, P, 4, 96, 16, 2, None) == SHAPE
    assert lib.s24_spmm_fwd_bias(P, P, P, P + 4, P, 4, 64, 16, 2, None) == ALIGN       # bias 8-byte aligned
    assert lib.s24_spmm_fwd_bias(P, P, None, None, P, 4, 64, 16, 2, None) == NULL
    assert lib.s24_spmm_fwd_bias(P, P, P, None, P, 0, 64, 16, 2, None) == OK
    # s24_spmm_fwd_glu(X, vals, meta, bias, GU, H, p, q, f, gate, dt, stream)
    assert lib.s24_spmm_fwd_glu(P, P, P, None, P, P, 4, 64, 24, 1, 2, None) == SHAPE   # f % 16
    assert lib.s24_spmm_fwd_glu(P, P, P, None, P, P, 4, 64, 16, 3, 2, None) == DTYPE   # gate
    assert lib.s24_spmm_fwd_glu(P, P, P, None, P, None, 4, 64, 16, 1, 2, None) == NULL
    assert lib.s24_spmm_fwd_glu(P, P, P, None, P, P, 0, 64, 16, 1, 2, None) == OK
    # s24_spmm_bwd_dx_glu(dY, valsT, metaT, GU, dGU, p, f, r, gate, dt, stream)
    assert lib.s24_spmm_bwd_dx_glu(P, P, P, P, P, 4, 16, 96, 1, 2, None) == SHAPE
    assert lib.s24_spmm_bwd_dx_glu(P, P, P, P, P, 4, 16, 64, 7, 2, None) == DTYPE
    assert lib.s24_spmm_bwd_dx_glu(P, P, P, P, P, 4, 16, 64, 1, 2, None) == UNSUP      # too few tiles
    assert lib.s24_spmm_bwd_dx_glu(P, P, P, P, P, 4, 16, 64, 1, 0, None) == UNSUP      # fp32
    # s24_spmm_fwd_act(X, vals, meta, bias, Z, H, p, q, r, act, dt, stream)
    assert lib.s24_spmm_fwd_act(P, P, P, None, P, P, 4, 96, 16, 1, 1, None) == SHAPE
    assert lib.s24_spmm_fwd_act(P, P, P, None, P, P, 4, 64, 16, 4, 1, None) == DTYPE   # activation enum
    assert lib.s24_spmm_fwd_act(P, P, P, None, P, None, 4, 64, 16, 1, 1, None) == NULL
    assert lib.s24_spmm_fwd_act(P, P, P, None, P, P, 0, 64, 16, 1, 1, None) == OK
    # s24_spmm_bwd_dx_act(dY, valsT, metaT, Z, dZ, p, f, r, act, dt, stream)
    assert lib.s24_spmm_bwd_dx_act(P, P, P, P, P, 4, 16, 96, 1, 1, None) == SHAPE
    assert lib.s24_spmm_bwd_dx_act(P, P, P, None, P, 4, 16, 64, 1, 1, None) == NULL
    assert lib.s24_spmm_bwd_dx_act(P, P, P, P, P, 4, 16, 64, 1, 0, None) == UNSUP     # fp32: the two-call route
    # s24_dense_dw_batch(problems, count, beta, dt, stream): a host array of problem records
    import ctypes
    from paper_2404_01847_amd.binding import _DwProblem
    good = _DwProblem(P, P, P, None, None, 4, 16, 16, 0.0)
    arr = (_DwProblem * 2)(good, good)
    ptr = ctypes.cast(arr, ctypes.c_void_p)
    assert lib.s24_dense_dw_batch(ptr, 5, 0.0, 1, None) == SHAPE                     # at most four problems
    assert lib.s24_dense_dw_batch(ptr, 2, 0.5, 1, None) == UNSUP
    assert lib.s24_dense_dw_batch(ptr, 2, 0.0, 9, None) == DTYPE
    assert lib.s24_dense_dw_batch(None, 2, 0.0, 1, None) == NULL
    assert lib.s24_dense_dw_batch(None, 0, 0.0, 1, None) == OK
    arr[1] = _DwProblem(P, P, P, None, None, 4, 24, 16, 0.0)
    assert lib.s24_dense_dw_batch(ptr, 2, 0.0, 1, None) == SHAPE                     # the second problem's q
    arr[1] = _DwProblem(P, None, P, None, None, 4, 16, 16, 0.0)
    assert lib.s24_dense_dw_batch(ptr, 2, 0.0, 1, None) == NULL
    arr[1] = _DwProblem(P, P, P, P, None, 4, 16, 16, 1e-4)
    assert lib.s24_dense_dw_batch(ptr, 2, 0.0, 1, None) == NULL                      # decay without a mask
    arr[0] = _DwProblem(P, P, P, None, None, 4, 16, 0, 0.0)
    arr[1] = _DwProblem(None, None, None, None, None, 4, 0, 16, 0.0)
    assert lib.s24_dense_dw_batch(ptr, 2, 0.0, 1, None) == OK                        # empty outputs: nothing to do
    # s24_spmm_bwd_dx_dw(dY, valsT, metaT, dX, p, q, r, problems, count, dt, stream): all of both parts before the first launch
    def both(pr=(good, good), dY=P, vT=P, mT=P, dX=P, p=4, q=16, r=64, count=None, dt=1):
        host = (_DwProblem * max(len(pr), 1))(*pr)
        return lib.s24_spmm_bwd_dx_dw(dY, vT, mT, dX, p, q, r, ctypes.cast(host, ctypes.c_void_p) if pr else None, len(pr) if count is None else count, dt, None)
    assert both(r=96) == SHAPE and both(r=0) == SHAPE and both(q=24) == SHAPE and both(p=-1) == SHAPE
    assert both(dt=9) == DTYPE and both(dY=None) == NULL and both(vT=None) == NULL and both(dX=None) == NULL and both(dX=P + 8) == ALIGN
    assert both(mT=None) == NULL and both(mT=P + 2) == ALIGN
    assert both(count=5) == SHAPE and both(count=-1) == SHAPE and both(pr=(), count=2) == NULL
    for pr, status in (((P, P, P, None, None, 4, 24, 16, 0.0), SHAPE), ((P, None, P, None, None, 4, 16, 16, 0.0), NULL), ((P, P, P + 4, None, None, 4, 16, 16, 0.0), ALIGN),
                       ((P, P, P, P, None, 4, 16, 16, 1e-4), NULL), ((P, P, P, P, P + 2, 4, 16, 16, 1e-4), ALIGN)):
        bad = _DwProblem(*pr)
        assert both((bad,)) == status and both((good, bad)) == status and both((good, good, good, bad)) == status
        assert both((bad,), p=0) == status and both((bad,), q=0) == status      # nothing to do for the other part
    empty = _DwProblem(None, None, None, None, None, 4, 0, 16, 0.0)
    for nothing in (dict(p=0), dict(q=0)):
        assert both((), **nothing) == OK and both((empty, empty), **nothing) == OK and both((empty,), dY=None, vT=None, mT=None, dX=None, **nothing) == OK
    # binary16 is a valid dtype everywhere a dtype is taken
    assert lib.s24_transposable_mask(P, 2, 6, 8, 8, P, None, None) == SHAPE
    assert lib.s24_spmm_fwd(P, P, P, P, 0, 64, 16, 2, None) == OK
    assert lib.s24_mvue24(P, 2, 0, 16, 16, 1, None, None, None) == OK


@pytest.fixture(scope="module")
def plain_headers(tmp_path_factory):
    """The headers of csrc/ that hold no HIP, behind C symbols."""
    d = tmp_path_factory.mktemp("headers")
    (d / "headers.cpp").write_text("""
#include "s24_overlap.h"
#include "s24_split.h"
extern "C" int dw_overlap(const void *p, int n, int esize) { return s24_dw_problems_overlap((const s24_dw_problem *)p, n, esize); }
extern "C" int dx_meets(const void *dY, const void *vT, const void *mT, const void *dX, int p, int q, int r, const void *pr, int n, int esize)
{
    return s24_dx_meets_dw(dY, vT, mT, dX, p, q, r, (const s24_dw_problem *)pr, n, esize);
}
extern "C" int token_pairs(int t) { return s24_token_pairs(t); }
extern "C" int slice_begin(int n, int s, int slices) { return s24_slice_begin(n, s, slices); }
""")
    so = str(d / "headers.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2404_01847_amd", "csrc"), str(d / "headers.cpp"), "-o", so], check=True)
    return C.CDLL(so)


# up to the largest token count that the entry points take; eight slices, as the weight gradients have
@pytest.mark.parametrize("tokens", [1, 2, 15, 16, 17, 4097, 2 ** 29 - 1, 2 ** 29, 2 ** 29 + 1, 2 ** 30 + 7, 2 ** 31 - 2, 2 ** 31 - 1])
def test_slices_of_the_tokens_cover_each_pair_once(plain_headers, tokens):
    pairs = plain_headers.token_pairs(tokens)
    assert pairs == -(-tokens // 2)
    bounds = [plain_headers.slice_begin(pairs, s, 8) for s in range(9)]
    assert bounds == [pairs * s // 8 for s in range(9)]
    assert bounds[0] == 0 and bounds[8] == pairs and 2 * (pairs - 1) < tokens


def test_overlapping_weight_gradients_are_found(plain_headers):
    from paper_2404_01847_amd.binding import _DwProblem
    step = 0x100000                          # distinct buffers, each larger than any used below
    def problem(k, p=64, q=32, r=48, **other):
        d = dict(dY=(8 * k + 1) * step, X=(8 * k + 2) * step, dW=(8 * k + 3) * step, W=(8 * k + 4) * step, mask=(8 * k + 5) * step)
        d.update(other)
        return _DwProblem(d["dY"], d["X"], d["dW"], d["W"], d["mask"], p, q, r, 1e-4)
    def overlap(*problems):
        return bool(plain_headers.dw_overlap((_DwProblem * len(problems))(*problems), len(problems), 4))
    a = problem(0)
    grad, cells = 3 * step, 48 * 32
    assert not overlap(a) and not overlap(a, problem(1), problem(2), problem(3))
    for name, size in (("dW", 4 * cells), ("X", 64 * 32 * 4), ("dY", 64 * 48 * 4), ("W", 4 * cells), ("mask", cells // 8)):
        for at, hit in ((grad, True), (grad + 4 * cells - 16, True), (grad + 4 * cells, False), (grad - size + 16, True), (grad - size, False)):
            assert overlap(a, problem(1, **{name: at})) == hit, (name, at)
            assert overlap(problem(1, **{name: at}), problem(2), a) == hit, (name, at)
    assert not overlap(a, problem(1, W=None, mask=grad))            # no decay: the mask is not read
    assert not overlap(a, problem(1, r=0, dW=grad, X=grad))         # an empty output
    assert not overlap(a, problem(1, p=0, X=grad, dY=grad)) and overlap(a, problem(1, p=0, dW=grad))


def test_input_gradient_that_meets_a_weight_gradient_is_found(plain_headers):
    from paper_2404_01847_amd.binding import _DwProblem
    step = 0x100000
    p, q, r, es = 64, 32, 64, 2
    at = dict(dY=1, vT=2, mT=3, dX=4, X=5, dW=6, W=7, mask=8)
    size = dict(dY=p * r * es, vT=r * q // 2 * es, mT=r * q // 8, dX=p * q * es, X=p * q * es, dW=r * q * 4, W=r * q * es, mask=r * q // 8)
    def meets(decay=True, r_dw=r, **moved):
        b = {k: C.c_void_p(moved.get(k, v * step)) for k, v in at.items()}
        pr = (_DwProblem * 1)(_DwProblem(b["dY"], b["X"], b["dW"], b["W"] if decay else None, b["mask"], p, q, r_dw, 1e-4))
        return bool(plain_headers.dx_meets(b["dY"], b["vT"], b["mT"], b["dX"], p, q, r, pr, 1, es))
    assert not meets()                           # dY is read by both
    for written, others in (("dX", ("dY", "X", "dW", "W", "mask")), ("dW", ("dY", "vT", "mT", "dX"))):
        for o in others:
            for to, hit in ((at[o] * step, True), (at[o] * step + size[o] - 16, True), (at[o] * step + size[o], False), (at[o] * step - size[written] + 16, True),
                            (at[o] * step - size[written], False)):
                assert meets(**{written: to}) == hit, (written, o)
    assert not meets(decay=False, dX=at["W"] * step) and not meets(r_dw=0, dX=at["dW"] * step)


@pytest.mark.parametrize("call, odd", [("dense_dw_batch", k) for k in ((1, 0), (0, 1), (1, 1), (0, 3), (1, 3))] +
                         [("spmm_bwd_dx_dw", k) for k in ((0, 0), (1, 0), (0, 1), (1, 3))])
@pytest.mark.parametrize("dt, other", [("float32", "bfloat16"), ("bfloat16", "float16"), ("float16", "float32")])
def test_batched_weight_gradients_refuse_mixed_dtypes(monkeypatch, call, odd, dt, other):
    """One dtype speaks for all operands of a call: with another one among them the kernels would read past its end."""
    import torch
    from paper_2404_01847_amd import binding
    monkeypatch.setattr(binding, "lib", lambda: pytest.fail("the library was called"))
    dt, other = getattr(torch, dt), getattr(torch, other)
    p, q, r = 4, 16, 64
    new = lambda *shape, t=dt: torch.zeros(shape, dtype=t)
    problems = [[new(p, r), new(p, q), new(r, q, t=torch.float32), new(r, q), new(r // 4, q // 4, t=torch.int16), 0.5] for _ in range(2)]
    which, operand = odd
    problems[which][operand] = problems[which][operand].to(other)
    with pytest.raises(ValueError, match="share one dtype"):
        if call == "dense_dw_batch":
            binding.dense_dw_batch(problems)
        else:
            binding.spmm_bwd_dx_dw(new(p, r), new(1, q, 32), new(1, q, 4, t=torch.int16), new(p, q), problems)


def test_binding_refuses_to_run_without_library(monkeypatch, tmp_path):
    from paper_2404_01847_amd import binding
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_LIB_PATH", str(tmp_path / "libs24.so"))
    with pytest.raises(FileNotFoundError):
        binding.lib()


def _device_code(path):
    """The gfx950 code objects of the library's offload bundles (one per source file)."""
    data, out, at = open(path, "rb").read(), [], 0
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    while (at := data.find(magic, at)) >= 0:
        count = int.from_bytes(data[at + 24:at + 32], "little")
        pos = at + 32
        for _ in range(count):
            offset, size, idlen = (int.from_bytes(data[pos + 8 * k:pos + 8 * k + 8], "little") for k in range(3))
            name = data[pos + 24:pos + 24 + idlen]
            if b"gfx950" in name:
                out.append(data[at + offset:at + offset + size])
            pos += 24 + idlen
        at += 24
    return out


@functools.lru_cache(maxsize=None)
def _registers(operand):
    m = re.fullmatch(r"([av])(\d+)|([av])\[(\d+):(\d+)\]", operand)
    if not m:
        return frozenset()
    if m.group(1):
        return frozenset({(m.group(1), int(m.group(2)))})
    return frozenset((m.group(3), k) for k in range(int(m.group(4)), int(m.group(5)) + 1))


ASM_MATRIX_OPS = ("v_mfma_f32_16x16x32", "v_smfmac_f32_16x16x64")
OPERAND_GAP, RESULT_GAP = 2, 18   # wait states from a vector write to a matrix instruction, and from one to its result's use


def _functions(listing):
    """llvm-objdump's listing -> {symbol: [(address, op, operands, branch target or None)]}"""
    out, base = {}, 0
    for line in listing.splitlines():
        head = re.match(r"([0-9a-f]+) <(.*)>:$", line)
        if head:
            base, code = int(head.group(1), 16), out.setdefault(head.group(2), [])
        elif line.startswith("\t") and "//" in line:
            text, _, note = line.partition("//")
            op, _, rest = text.strip().partition(" ")
            target = re.search(r"<[^>]*?(?:\+0x([0-9a-f]+))?>$", note.strip()) if "branch" in op else None
            code.append((int(note.split(":")[0], 16), op, rest, target and base + int(target.group(1) or "0", 16)))
    return out


def _asm_hazards(code):
    """Places of one function where an operand of a matrix instruction written as asm may have been written by a vector
    instruction within OPERAND_GAP wait states, or where anything but a matrix instruction adding to the same accumulator may
    touch a result within RESULT_GAP, on any path.  An instruction counts as one wait state, s_nop as what it says."""
    step = []   # (wait states, kind, registers read or written, registers written)
    for _, op, rest, _ in code:
        args = [a.strip() for a in rest.split(",")] if rest else []
        regs = [_registers(a.split(" ")[0]) for a in args]
        every = set().union(*regs)
        if op == "s_nop":
            step.append((int(args[0], 0) + 1, "wait", every, set()))
        elif op.startswith(ASM_MATRIX_OPS):
            step.append((1, "asm", set().union(*regs[:4]), regs[0]))
        elif op.startswith(("v_mfma", "v_smfmac")):
            step.append((1, "matrix", every, regs[0]))
        elif op.startswith("v_swap"):
            step.append((1, "vector", every, every))
        elif op.startswith("v_"):
            step.append((1, "vector", every, regs[0] if regs else set()))
        else:
            step.append((1, "other", every, set()))
    at = {c[0]: k for k, c in enumerate(code)}
    assert not any(c[1].startswith(("s_setpc", "s_swappc", "s_call", "s_cbranch_g")) for c in code)
    starts = sorted({0} | {at[c[3]] for c in code if c[3] is not None} |
                    {k + 1 for k, c in enumerate(code) if ("branch" in c[1] or c[1] == "s_endpgm") and k + 1 < len(code)})
    ends = dict(zip(starts, starts[1:] + [len(code)]))
    entry, found, todo = {0: ({}, {})}, set(), [0]   # block -> (register -> wait states left until usable as operand, as result)
    while todo:
        block = todo.pop()
        ready, done = (dict(s) for s in entry[block])   # -> wait state at which it is usable
        clock = 0
        for k in range(block, ends[block]):
            wait, kind, regs, wrote = step[k]
            if kind == "asm":
                found.update((k, r, "operand") for r in regs if ready.get(r, 0) > clock)
                found.update((k, r, "result") for r in regs - wrote if done.get(r, 0) > clock)
            elif kind != "matrix":
                found.update((k, r, "result") for r in regs if done.get(r, 0) > clock)
            clock += wait
            if kind == "asm":
                done.update((r, clock + RESULT_GAP) for r in wrote)
            elif kind == "vector":
                ready.update((r, clock + OPERAND_GAP) for r in wrote)
        left = tuple({r: t - clock for r, t in s.items() if t > clock} for s in (ready, done))
        _, op, _, target = code[ends[block] - 1]
        follow = [] if target is None else [at[target]]
        if op not in ("s_branch", "s_endpgm") and ends[block] < len(code):
            follow.append(ends[block])
        for nxt in follow:   # the worst of the paths that meet
            old = entry.get(nxt)
            new = left if old is None else tuple({r: max(o.get(r, 0), n.get(r, 0)) for r in {**o, **n}} for o, n in zip(old, left))
            if new != old:
                entry[nxt] = new
                todo.append(nxt)
    return sorted((code[k][0], code[k][1], code[k][2], r, what) for k, r, what in found)


def _listing(*lines):
    """Lines "op operands" of a function at address 0, four bytes each; "-> n" is a branch to line n."""
    out = ["0000000000000000 <f>:"]
    for k, line in enumerate(lines):
        line, _, to = line.partition(" -> ")
        out.append(f"\t{line} // {4 * k:012X}: 00000000" + (f" <f+0x{4 * int(to):x}>" if to else ""))
    return "\n".join(out)


def test_hazard_check_follows_every_path_and_operand():
    dense, sparse = "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]", "v_smfmac_f32_16x16x64_f16 v[8:11], v[0:3], v[16:23], v30 abid:1"
    hazards = lambda *lines: [(a // 4, r, what) for a, _, _, r, what in _asm_hazards(_functions(_listing(*lines))["f"])]
    drain = ("s_nop 15", "s_nop 1")
    assert hazards("v_mov_b32_e32 v0, v50", "s_nop 1", dense, dense, *drain, "v_accvgpr_read_b32 v9, a3", "s_endpgm") == []
    assert hazards("v_mov_b32_e32 v0, v50", "s_nop 0", dense, "s_endpgm") == [(2, ("v", 0), "operand")]
    assert hazards("v_perm_b32 v30, v1, v2, v3", "s_nop 0", sparse, "s_endpgm") == [(2, ("v", 30), "operand")]
    assert hazards("v_mov_b32_e32 v9, 0", "s_nop 0", sparse, "s_endpgm") == [(2, ("v", 9), "operand")]      # the accumulator
    assert hazards("v_accvgpr_write_b32 a2, v9", dense, "s_endpgm") == [(1, ("a", 2), "operand")]
    assert hazards(dense, "s_nop 15", "s_nop 0", "ds_write_b32 v9, a1", "s_endpgm") == [(3, ("a", 1), "result")]
    assert hazards(sparse, dense.replace("v[0:3]", "v[8:11]"), "s_endpgm") == [(1, ("v", k), "result") for k in range(8, 12)]
    # around a loop: the last instruction of the body is just ahead of the first
    assert hazards("s_mov_b32 s0, 0", sparse, "s_nop 7", "v_mov_b32_e32 v17, 0", "s_cbranch_scc1 65532 -> 1", "s_endpgm") == [(1, ("v", 17), "operand")]
    # out of it: the fall-through waits, the jump does not
    assert hazards("s_cbranch_scc0 5 -> 6", sparse, "s_cbranch_scc1 2 -> 5", *drain, "v_mov_b32_e32 v60, v8", "s_endpgm") == [(5, ("v", 8), "result")]
    # nothing follows a jump but its target
    assert hazards(sparse, "s_branch 1 -> 3", "v_mov_b32_e32 v60, v8", *drain, "v_mov_b32_e32 v60, v8", "s_endpgm") == []


def test_matrix_instructions_written_as_asm_keep_their_distances(lib, tmp_path):
    """The compiler pads no hazards around the 16-wide matrix instructions in inline asm; the built library has none."""
    import paper_2404_01847_amd as s24
    objdump = "/opt/rocm/llvm/bin/llvm-objdump"
    if not os.path.exists(objdump):
        assert not os.path.exists("/opt/rocm/bin/hipcc"), "a compiler without its disassembler: the hazards go unchecked"
        pytest.skip("no llvm-objdump")
    found = 0
    for k, code in enumerate(_device_code(s24.lib_path())):
        if b"dense_tn_dma_kernel" not in code:
            continue
        obj = tmp_path / f"{k}.co"
        obj.write_bytes(code)
        text = subprocess.run([objdump, "-d", "--mcpu=gfx950", "--no-show-raw-insn", str(obj)], capture_output=True, text=True, check=True).stdout
        for name, code in _functions(text).items():
            matrix = sum(c[1].startswith(ASM_MATRIX_OPS) for c in code)
            found += matrix
            if matrix:
                assert _asm_hazards(code) == [], name
    assert found > 1000


def test_short_kernels_take_few_arguments(lib, tmp_path):
    """A launch pays on the host for each argument, and a step of a few hundred tokens waits for the host."""
    import paper_2404_01847_amd as s24
    readelf = "/opt/rocm/llvm/bin/llvm-readelf"
    if not os.path.exists(readelf):
        assert not os.path.exists("/opt/rocm/bin/hipcc"), "a compiler without its readelf: the arguments go uncounted"
        pytest.skip("no llvm-readelf")
    counted = {"spmm_slice_kernel": 0, "f32_nt_kernel": 0, "dx_dw_kernel": 0, "f32_nt_tn_kernel": 0}
    for k, code in enumerate(_device_code(s24.lib_path())):
        obj = tmp_path / f"{k}.co"
        obj.write_bytes(code)
        notes = subprocess.run([readelf, "--notes", str(obj)], capture_output=True, text=True, check=True).stdout
        for kernel in re.split(r"^  - ", notes, flags=re.M):   # one entry of amdhsa.kernels each
            name = re.search(r"^    \.name: +(\S+)", kernel, flags=re.M)
            for short in counted:
                if name and short in name[1]:
                    counted[short] += 1
                    assert len(re.findall(r"\.value_kind: +(?!hidden)", kernel)) <= 5, name[1]
    assert all(counted.values()), counted

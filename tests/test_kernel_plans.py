"""The shapes of the GPU tests reach the kernel instantiations that those tests are there for (the planners run on the host)."""
import os

import pytest

import kernel_plans as K
import test_gpu_forward_stream as fwd
import test_gpu_gemm_f32_tiles as f32


@pytest.fixture(scope="module")
def lib():
    import paper_1409_5705_amd as m
    if not os.path.exists(m.binding.LIB_PATH):
        from paper_1409_5705_amd.build import build_library
        build_library()
    return m.lib()


@pytest.mark.parametrize("copy,shapes", [(False, [(4, 2), (2, 2), (1, 2)]), (True, [(4, 2), (2, 4), (1, 2)])])
def test_stream_forward_shapes(lib, copy, shapes):
    got = {K.forward(lib, B, J, D, copy) for J, D, B in fwd.SHAPES}
    reached = {(mt, ntl, split > 1) for mt, ntl, split in got if mt}
    assert reached == {(mt, ntl, split) for mt, ntl in shapes for split in (False, True)}


def test_apply_shapes(lib):
    import test_gpu_gemm_f32x3 as x3
    plans = [K.gemm_f32(lib, "apply", N, J, D) for J, D, N in f32.APPLY_SHAPES + x3.FP32_SHAPES]
    assert {p[::2] for p in plans if p} == {(t, direct) for t in K.TILES for direct in (False, True)}


@pytest.mark.parametrize("kind", ["projections", "shrink", "residual"])
def test_sparse_code_shapes(lib, kind):
    plans = [p for p in (K.gemm_f32(lib, kind, B, J, D) for J, D, B in f32.SC_SHAPES + [(1001, 301, 99), (64, 4, 3)]) if p]
    assert {(t, direct) for t, _, direct in plans} == {(t, direct) for t in K.TILES for direct in (False, True)}
    assert len({t for t, split, _ in plans if split > 1}) >= 2


def test_three_term_shapes(lib):
    import test_gpu_gemm_f32x3 as x3
    plans = [K.gemm_f32x3(lib, "apply", N, J, D) for J, D, N in x3.APPLY_SHAPES]
    assert all(plans) and all(K.gemm_f32x3(lib, "apply", N, J, D) for J, D, N in [(1003, 2047, 300), (1001, 2049, 333)]), list(zip(x3.APPLY_SHAPES, plans))
    assert {(t, split > 1) for t, split in plans} == {(t, s) for t in K.X3_TILES for s in (False, True)}
    assert all(K.gemm_f32x3(lib, "apply", k, m, n) for m, n, k in x3.NOT_FINITE_APPLY)
    reached = [K.gemm_f32x3(lib, "logits", B, J, D) for B, J, D in x3.NOT_FINITE_LOGITS]
    assert all(reached) and {p[0] for p in reached} == set(K.X3_TILES) and {p[1] > 1 for p in reached} == {False, True}, reached
    assert {K.gemm_f32(lib, "apply", N, J, D)[::2] for J, D, N in x3.FP32_SHAPES} == {("128x64", True), ("128x64", False)}


@pytest.mark.parametrize("kind", ["projections", "shrink", "residual"])
def test_three_term_shapes_of_contiguous_operands(lib, kind):
    import test_gpu_gemm_f32x3 as x3
    plans = [K.gemm_f32x3(lib, kind, B, J, D) for J, D, B in (x3.LOGITS_SHAPES if kind == "projections" else x3.SC_SHAPES)]
    assert {(p[0], p[1] > 1) for p in plans if p} == {(t, s) for t in K.X3_TILES for s in (False, True)}


def test_shapes_whose_row_kernels_add_up_the_splits(lib):
    import test_gpu_split_sums as s

    for kind, shapes in (("logits", s.MLR_SHAPES), ("projections", s.DML_SHAPES)):
        assert all(K.split(lib, kind, *shape) > 1 for shape in shapes[:-1])
        assert K.split(lib, kind, *shapes[-1]) == 1


def test_shapes_of_the_forward_on_rows(lib):
    from test_gpu_forward_rows import SHAPES
    plans = [K.forward(lib, *s, copy) for s in SHAPES for copy in (False, True)]
    assert all(mt > 0 for mt, _, _ in plans), list(zip([s for s in SHAPES for _ in "ab"], plans))
    assert {mt for mt, _, _ in plans} == {1, 2, 4} and {split > 1 for _, _, split in plans} == {False, True}


def test_adding_up_elsewhere_is_cheaper(lib):
    """A k-split whose parts the row kernel adds up pays no launch for their sum: the same contraction is split at fewer products
    where it is a projection than where it is a shrink step, and never estimated slower."""
    for B, J in ((400, 300), (410, 292), (663, 60), (512, 1024)):
        first = {kind: next(D for D in range(256, 40000, 32) if K.split(lib, kind, B, J, D) > 1) for kind in ("projections", "shrink")}
        assert first["projections"] < first["shrink"], (B, J, first)
        assert all(K.estimate(lib, "projections", B, J, D) <= K.estimate(lib, "shrink", B, J, D) for D in range(32, 10000, 500))

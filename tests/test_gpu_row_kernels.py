"""The row-wise kernels at the edges of what they keep in registers: row lengths around every change of kernel, rows with
and without 16-byte alignment, one and two launches per power iteration.  Tolerances are those of the fp32 parity tests."""
import numpy as np
import pytest

import sfb_synth as S
from parity import TOL_F32, mlr_u_check, rel_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sfb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_5705_amd as m
    m.lib()
    return m


@pytest.fixture(scope="module")
def ctx(sfb):
    c = sfb.Context(0)
    yield c
    c.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("J", [1, 255, 256, 257, 260, 1023, 1024, 1025, 1028, 4095, 4096, 4097, 4100, 8191, 8192, 8193, 8196, 16384, 16385])
def test_softmax_row_lengths(ctx, sfb, oracle, J):
    print("softmax", J, flush=True)
    D, B = 20, 9
    W0 = S.normal_matrix(J, D, 0.3, seed=36)
    X, y = S.mlr_batch(J, D, B, seed=36)
    U, V = torch.empty((B, J), device="cuda:0"), torch.empty((B, D), device="cuda:0")
    ctx.sfb_compute_sf(sfb.SFB_MLR, dev(W0), dev(X), Y=dev(y), U=U, V=V)
    Uo, Vo = oracle.mlr_sf(W0, X, y)
    assert np.array_equal(host(V), X)
    if J > 1:                                    # (one class: its probability is 1 whatever the sample, the factor 0)
        mlr_u_check(host(U), Uo, y, TOL_F32)


@pytest.mark.parametrize("J,B", [(J, 9) for J in (1, 256, 257, 512, 513, 1024, 1025, 4096, 4097)] +
                         [(J, 515) for J in (256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096)])   # more than two samples a CU
def test_sdca_row_lengths(ctx, J, B):
    from oracle import sdca as O
    print("sdca", J, B, flush=True)
    D, lam, N, beta = 72, 1e-3, 5000, 0.5
    W0 = S.normal_matrix(J, D, 0.1, seed=31)
    X, y = S.mlr_batch(J, D, B, seed=31)
    X[3] = 0.0                                   # a zero sample
    P0 = S.sdca_dual_points(J, y, seed=31)
    P, dU = dev(P0), torch.empty((B, J), device="cuda:0")
    ctx.sfb_sdca_mlr_sf(dev(W0), dev(X), P, lam, N, beta, dU)
    rows = np.arange(B) if B < 10 else np.array([0, 3, 255, 256, 511, 514])      # (samples do not see each other)
    dUo, Po = O.sdca_mlr_sf(W0, P0[rows], X[rows], lam, N, beta)
    if J > 1:                                    # (one class: its probability is 1 whatever the sample, the factor 0)
        assert rel_err(host(dU)[rows], dUo) <= TOL_F32
    assert rel_err(host(P)[rows], Po) <= TOL_F32


@pytest.mark.parametrize("J,D,B", [
    (128, 64, 32), (130, 63, 40), (17, 1, 3), (16, 5, 20),                       # one chunk, few columns
    (1000, 300, 100), (1000, 301, 100), (333, 257, 64), (520, 1024, 70),         # partials added by every workgroup
    (1000, 300, 10), (1001, 1023, 40), (900, 1025, 33), (4096, 127, 130),        # not: no room, too many, rows too long
])
def test_power_iteration(ctx, sfb, oracle, J, D, B):
    """One ISTA iteration: the codes are soft(x W^T / L, lambda / L), so they show L."""
    print("power", J, D, B, flush=True)
    W0 = S.sc_dictionary(J, D, seed=32)
    X = S.sc_batch(D, B, seed=32)
    for iters in (1, 2, 9):
        U, V = torch.empty((B, J), device="cuda:0"), torch.empty((B, D), device="cuda:0")
        ctx.sfb_compute_sf(sfb.SFB_SC, dev(W0), dev(X), U=U, V=V, lam=0.1, ista_iters=1, power_iters=iters)
        Uo, Vo, _ = oracle.sc_sf(W0, X, lam=0.1, ista_iters=1, power_iters=iters)
        assert rel_err(host(U), Uo) <= TOL_F32 and rel_err(host(V), Vo) <= TOL_F32


@pytest.mark.parametrize("J,D", [(5, 1), (7, 64), (6, 255), (9, 1023), (10, 1024), (3, 1025), (1, 4)])
def test_prox_row_lengths(ctx, sfb, oracle, J, D):
    W0 = S.normal_matrix(J, D, 1.5 / np.sqrt(D), seed=33)
    W0[0] *= 0.1
    W0[J // 2] = 0.0 if J > 2 else W0[J // 2]
    for mode_g, mode_o in ((sfb.SFB_PROX_PROJECT, oracle.PROX_PROJECT), (sfb.SFB_PROX_NORMALIZE, oracle.PROX_NORMALIZE)):
        W = dev(W0)
        ctx.sfb_prox_rows(W, mode_g)
        assert rel_err(host(W), oracle.prox_rows(W0, mode_o)) <= TOL_F32


@pytest.mark.parametrize("K,D", [(1, 3), (255, 37), (1024, 64), (1025, 66)])
def test_dml_row_lengths(ctx, sfb, oracle, K, D):
    B = 21
    W0 = S.normal_matrix(K, D, 0.02 / np.sqrt(K * D), seed=34)    # (every distance far below the margin: no rounding decides)
    X, Y, sim = S.dml_batch(D, B, seed=34)
    U, V = torch.empty((B, K), device="cuda:0"), torch.empty((B, D), device="cuda:0")
    n = torch.full((1,), 77, dtype=torch.int32, device="cuda:0")
    ctx.sfb_compute_sf(sfb.SFB_DML, dev(W0), dev(X), Y=dev(Y), sim=dev(sim), U=U, V=V, n_active=n)
    Uo, Vo, no = oracle.dml_sf(W0, X, Y, sim)
    assert int(host(n)[0]) == no
    assert rel_err(host(U), Uo) <= TOL_F32 and rel_err(host(V), Vo) <= TOL_F32

"""The 64-wide step factorisation against LAPACK and the oracle, at the edges
of its blocks, tiles and of the size where the tiled factorisation takes over.

Tolerances: the factor within 10x the difference of the oracle's and LAPACK's
factors of the same matrix (1e-13 at least); L W = I through the solves, that
is Eq. (1) within 1e-9 of the oracle."""
import numpy as np
import pytest
import scipy.linalg

import synthetic

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    import paper_2008_07437_amd as m
    m._lib._load()
    return m


def _dev(a):
    import torch
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def _sites(orc, n, seed):
    x, y = synthetic.jittered_grid(n, seed)
    p = orc.morton_order(x, y)
    return x[p], y[p]


# one and two rows past and before a 64-block, a tile, the last tile's padding
@pytest.mark.parametrize("n,nb", [(1, 128), (31, 128), (32, 128), (33, 128), (63, 128), (64, 128),
                                  (65, 256), (95, 256), (97, 256), (255, 512), (257, 512),
                                  (383, 768), (385, 768), (513, 1024), (700, 1024)])
def test_factor_block_edges(lib, orc, n, nb):
    print("factor n=%d nb=%d" % (n, nb), flush=True)
    th = (1.4, 0.6, 0.1, 0.7, 1.1, -0.4)
    x, y = _sites(orc, n, 3)
    A = lib.cov_generate(_dev(x), _dev(y), th, {"nb": nb})
    assert lib.potrf_tiled(A) == 0
    got = A.to_dense().cpu().numpy()
    S = orc.cov_dense(x, y, th)
    low, info = orc.potrf(S)
    assert info == 0
    floor = np.max(np.abs(low - scipy.linalg.cholesky(S, lower=True)))
    assert np.max(np.abs(got - low)) <= max(10 * floor, 1e-13)
    z = orc.simulate_z(x, y, th, synthetic.normal_eps(2 * n, 3))
    ref = orc.loglik(x, y, z, th)
    res, F = lib.loglik(_dev(x), _dev(y), _dev(z), th, {"nb": nb}, keep=True)
    for key in ("loglik", "logdet", "quad"):
        assert abs(res[key][0] - ref[key]) <= 1e-9 * max(abs(ref[key]), 1.0), key
    w = F.w(n).cpu().numpy()  # W and W^T through both solves
    np.testing.assert_allclose(S @ w, z, rtol=0, atol=1e-9 * np.max(np.abs(z)))


# around 6,144 rows at every larger tile size: 64-wide steps throughout (tile
# steps, from 8,194 rows on, are in test_gpu_tiled.py)
@pytest.mark.parametrize("n,nb", [(3071, 128), (3072, 256), (3073, 512), (3100, 768), (3600, 1024)])
def test_tiled_and_tail(lib, n, nb):
    print("tiled n=%d nb=%d" % (n, nb), flush=True)
    import torch
    th = synthetic.THETA_REF
    x, y = synthetic.jittered_grid(n, 4)
    A = lib.cov_generate(_dev(x), _dev(y), th, {"nb": nb})
    S = A.to_dense()
    S = S + torch.tril(S, -1).T
    assert lib.potrf_tiled(A) == 0
    low = A.to_dense()
    ref = torch.linalg.cholesky(S)
    cpu = torch.as_tensor(scipy.linalg.cholesky(S.cpu().numpy(), lower=True)).cuda()
    floor = float((ref - cpu).abs().max())
    assert float((low - cpu).abs().max()) <= max(10 * floor, 1e-13)


# block counts at the edges of the groups of four panels and of their shares,
# tiles of two, four and eight blocks, the band of the tiles kept (0: all) and
# both sides of the largest matrix that is factored in steps throughout
@pytest.mark.parametrize("n,nb,band", [(127, 128, 0), (129, 128, 0), (161, 128, 0), (289, 256, 0),
                                       (352, 256, 0), (545, 128, 0), (1056, 512, 0),
                                       (4095, 128, 0), (4097, 512, 0), (545, 128, 2),
                                       (600, 128, 3), (700, 256, 2)])
def test_grouped_updates(lib, n, nb, band):
    print("grouped n=%d nb=%d band=%d" % (n, nb, band), flush=True)
    import torch
    # a short range and sites in rows: the banded matrix stays positive definite
    th = (1.0, 1.0, 0.03, 0.5, 1.0, 0.5)
    x, y = synthetic.jittered_grid(n, 4)
    opts = {"nb": nb, "precision": lib.MVG_DST, "band_tiles": band} if band else {"nb": nb}
    A = lib.cov_generate(_dev(x), _dev(y), th, opts)
    S = A.to_dense()
    S = S + torch.tril(S, -1).T
    assert lib.potrf_tiled(A) == 0
    low = A.to_dense()
    cpu = torch.as_tensor(scipy.linalg.cholesky(S.cpu().numpy(), lower=True)).cuda()
    floor = float((torch.linalg.cholesky(S) - cpu).abs().max())
    assert float((low - cpu).abs().max()) <= max(10 * floor, 1e-13)


# a duplicated site: the failing pivot in the first, a middle and the last block
@pytest.mark.parametrize("at", [1, 17, 40, 200, 299])
def test_first_failing_pivot(lib, orc, at):
    print("duplicate at %d" % at, flush=True)
    x, y = _sites(orc, 300, 6)
    x[at], y[at] = x[at - 1], y[at - 1]
    z = np.ones(600)
    ref = orc.loglik(x, y, z, synthetic.THETA_REF)
    got = lib.loglik(_dev(x), _dev(y), _dev(z), synthetic.THETA_REF, {"nb": 128})
    assert ref["info"] > 0 and got["status"][0] == ref["info"]
    assert got["loglik"][0] == -np.inf


def test_batched_block_edges(lib, orc):
    """Tasks of one block to sixteen, at the edges of the blocks, in one batch;
    the no-allocation form (groups of tasks) gives the same bits."""
    sizes = [1, 2, 31, 32, 33, 63, 64, 65, 96, 97, 255, 256, 257, 480, 511, 512]
    tasks, ref = [], []
    for i, n in enumerate(sizes):
        th = synthetic.jittered_thetas(1, 40 + i)[0]
        x, y = _sites(orc, n, 50 + i)
        z = orc.simulate_z(x, y, th, synthetic.normal_eps(2 * n, 50 + i))
        tasks.append((_dev(x), _dev(y), _dev(z), th))
        ref.append(orc.loglik(x, y, z, th))
    got = lib.loglik_many(tasks)
    for i, r in enumerate(ref):
        for key in ("loglik", "logdet", "quad"):
            assert abs(got[key][i] - r[key]) <= 1e-9 * max(abs(r[key]), 1.0), (sizes[i], key)
    again = lib.loglik_many_noalloc(tasks * 8)
    for key in ("loglik", "logdet", "quad", "status"):
        assert np.array_equal(again[key], np.tile(got[key], 8)), key


# prediction errors on both sides of the switch to transposed right-hand sides,
# with odd numbers of targets and one to several tiles
@pytest.mark.parametrize("n,m,nb", [(40, 79, 128), (40, 80, 128), (150, 128, 128), (150, 65, 256),
                                    (300, 129, 128), (700, 200, 512), (600, 97, 768)])
def test_prediction_errors(lib, orc, n, m, nb):
    print("prediction errors n=%d m=%d nb=%d" % (n, m, nb), flush=True)
    th = synthetic.THETA_REF
    x, y = _sites(orc, n, 8)
    z = orc.simulate_z(x, y, th, synthetic.normal_eps(2 * n, 8))
    x0, y0 = synthetic.uniform_targets(m, 8)
    ref, ref_mse = orc.cokrige(x, y, z, th, x0, y0, with_mse=True)
    _, F = lib.loglik(_dev(x), _dev(y), _dev(z), th, {"nb": nb}, keep=True)
    zhat, mse = lib.cokrige_predict(F, _dev(x0), _dev(y0), with_mse=True)
    np.testing.assert_allclose(zhat.cpu().numpy(), ref, rtol=0, atol=1e-10)
    np.testing.assert_allclose(mse.cpu().numpy(), ref_mse, rtol=1e-8, atol=1e-12)


@pytest.mark.parametrize("n,nb", [(1, 128), (33, 128), (200, 128), (300, 256), (600, 512), (1100, 1024)])
def test_factor_times_vector(lib, n, nb):
    """Z = L eps against the dense product of the same factor; 1e-13 of the
    row's largest partial sum (at most 2n roundings of 1e-16)."""
    print("L eps n=%d nb=%d" % (n, nb), flush=True)
    x, y = synthetic.jittered_grid(n, 2)
    A = lib.cov_generate(_dev(x), _dev(y), synthetic.THETA_REF, {"nb": nb})
    assert lib.potrf_tiled(A) == 0
    eps = synthetic.normal_eps(2 * n, 2)
    low = A.to_dense().cpu().numpy()
    got = lib.mvg_trmv(A, _dev(eps)).cpu().numpy()
    assert np.all(np.abs(got - low @ eps) <= 1e-13 * (np.abs(low) @ np.abs(eps)))

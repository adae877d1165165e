"""What a prediction may depend on: the factor and its own target, not how many
targets share the call."""
import numpy as np
import pytest

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


def _factor(lib, orc, n, nb, th):
    x, y = synthetic.jittered_grid(n, 8)
    p = orc.morton_order(x, y)
    x, y, z = x[p], y[p], synthetic.normal_eps(2 * n, 8)
    _, F = lib.loglik(_dev(x), _dev(y), _dev(z), th, {"nb": nb}, keep=True)
    return x, y, F, F.w(n).cpu().numpy()


# locations at the edges of a partial sum (256 of them) and past 64 sums, every
# form of the covariance (closed orders, the quadrature below 128 locations, the
# polynomials), and targets from one to several times what a workgroup takes
@pytest.mark.parametrize("n,nb,nu", [(1, 128, (0.5, 1.0)), (100, 128, (0.7, 1.1)), (255, 128, (0.5, 1.5)),
                                     (256, 256, (0.5, 1.0)), (257, 256, (0.7, 1.1)), (1000, 256, (0.5, 1.0)),
                                     (5000, 512, (0.5, 1.0)), (16400, 1024, (0.5, 1.0))])
def test_alone_equals_in_a_map(lib, orc, n, nb, nu):
    print("alone = in a map: n=%d" % n, flush=True)
    th = (1.2, 0.8, 0.1, nu[0], nu[1], 0.4)
    x, y, F, w = _factor(lib, orc, n, nb, th)
    m = 3001
    x0, y0 = (_dev(v) for v in synthetic.uniform_targets(m, 8))
    got = lib.cokrige_predict(F, x0, y0).cpu().numpy()
    for lo, hi in ((0, 1), (1, 2), (m - 1, m), (7, 24), (100, 133), (500, 1600)):
        part = lib.cokrige_predict(F, x0[lo:hi].contiguous(), y0[lo:hi].contiguous()).cpu().numpy()
        assert np.array_equal(part, got[lo:hi]), (lo, hi)
    at = np.array([0, 15, 16, 17, 1500, m - 1])
    c0 = orc.cross_cov_targets(x, y, x0.cpu().numpy()[at], y0.cpu().numpy()[at], th)
    # 2n products, each and their sums rounded: 2n + 8 roundings of 2^-53, and
    # covariances within 1e-13 relative
    for k, t in enumerate(at):
        for j in range(2):
            terms = c0[:, 2 * k + j] * w
            tol = (1e-13 + (2 * n + 8) * 2.0 ** -53) * np.abs(terms).sum()
            assert abs(got[t, j] - terms.sum()) <= tol, (t, j)


# the errors' three solves: one target, 2 to 79, 80 and more
@pytest.mark.parametrize("n,nb", [(40, 128), (300, 128), (1000, 256), (1500, 512), (1100, 1024)])
def test_errors_alone_equal_in_a_map(lib, orc, n, nb):
    print("errors alone = in a map: n=%d nb=%d" % (n, nb), flush=True)
    _, _, F, _ = _factor(lib, orc, n, nb, synthetic.THETA_REF)
    x0, y0 = (_dev(v) for v in synthetic.uniform_targets(700, 8))

    def call(lo, hi):
        return lib.cokrige_predict(F, x0[lo:hi].contiguous(), y0[lo:hi].contiguous(), with_mse=True)[1].cpu().numpy()
    got = call(0, 700)
    for lo, hi in ((0, 80), (63, 191), (100, 301), (619, 700)):
        assert np.array_equal(call(lo, hi), got[lo:hi]), (lo, hi)
    few = call(0, 79)
    for lo, hi in ((0, 2), (3, 20), (30, 64)):
        assert np.array_equal(call(lo, hi), few[lo:hi]), (lo, hi)
    # the solves agree to the tolerance of the errors against the oracle
    np.testing.assert_allclose(few, got[:79], rtol=1e-8, atol=1e-12)
    np.testing.assert_allclose(call(5, 6), got[5:6], rtol=1e-8, atol=1e-12)

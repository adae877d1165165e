"""Device memory that a call holds beside its inputs, outputs and matrices: the
high-water mark of the device's memory pool, from which the library allocates."""
import ctypes

import pytest

import synthetic

pytestmark = pytest.mark.gpu

USED_CURRENT, USED_HIGH = 7, 8  # hipMemPoolAttr


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
    return torch.as_tensor(a).cuda()


def _held(f):
    """The most that f held at once (bytes), beyond what was held before."""
    import torch
    with open("/proc/self/maps") as maps:
        hip = ctypes.CDLL(next(s.split()[-1] for s in maps if "libamdhip64" in s))
    pool, v = ctypes.c_void_p(), ctypes.c_uint64(0)
    assert hip.hipDeviceGetDefaultMemPool(ctypes.byref(pool), torch.cuda.current_device()) == 0
    torch.cuda.synchronize()
    # (a larger freed block taken again would count in full)
    assert hip.hipMemPoolTrimTo(pool, ctypes.c_size_t(0)) == 0
    assert hip.hipMemPoolSetAttribute(pool, USED_HIGH, ctypes.byref(v)) == 0
    assert hip.hipMemPoolGetAttribute(pool, USED_CURRENT, ctypes.byref(v)) == 0
    before = v.value
    f()
    torch.cuda.synchronize()
    assert hip.hipMemPoolGetAttribute(pool, USED_HIGH, ctypes.byref(v)) == 0
    return v.value - before


# 2, 31 and 47 chunks of 1,024 columns: one pass and two
@pytest.mark.parametrize("n,nb", [(1000, 512), (15800, 1024), (24000, 512)])
def test_factor_times_vector(lib, n, nb):
    """L eps holds at most 33 padded vectors, whatever the number of tiles, and
    is the product of the dense factor's rows (1e-13 of their largest sums)."""
    import torch
    print("workspace of L eps, n=%d" % n, flush=True)
    x, y = synthetic.jittered_grid(n, 1)
    A = lib.cov_generate(_dev(x), _dev(y), synthetic.THETA_REF, {"nb": nb})
    assert lib.potrf_tiled(A) == 0
    eps = _dev(synthetic.normal_eps(2 * n, 1))
    out = []
    held = _held(lambda: out.append(lib.mvg_trmv(A, eps)))
    assert 0 < held <= 33 * 8 * nb * A.shape()["ntiles"]
    low = A.to_dense()
    want = (low @ eps[:, None])[:, 0]
    low.abs_()
    assert bool(torch.all((out[0] - want).abs() <= 1e-13 * (low @ eps.abs()[:, None])[:, 0]))


# the server admits a request by mvg_footprint: what a batch of small likelihoods
# holds may not be more than its tasks' footprints (at any tile size) together
@pytest.mark.parametrize("sizes", [[20] * 1023 + [512], [512] + [1] * 1100, [32, 33, 64, 65, 128, 300] * 20,
                                   [512] * 64])
def test_batch_within_footprints(lib, sizes):
    print("workspace of a batch, n = %d .. %d" % (min(sizes), max(sizes)), flush=True)
    data = {}
    for n in set(sizes):
        x, y = synthetic.jittered_grid(n, 1)
        data[n] = (_dev(x), _dev(y), _dev(synthetic.normal_eps(2 * n, 1)), (1.0, 1.0, 0.1, 0.7, 1.0, 0.5))
    got = []
    held = _held(lambda: got.append(lib.loglik_many([data[n] for n in sizes])))
    assert 0 < held <= sum(lib.mvg_footprint(n, {"nb": 128}) for n in sizes)
    # the same bits as one by one, wherever a task's workspace lies
    for n in set(sizes):
        alone = lib.loglik_many([data[n]])
        at = [i for i, s in enumerate(sizes) if s == n]
        for key in ("loglik", "logdet", "quad", "status"):
            assert (got[0][key][at] == alone[key][0]).all(), (n, key)

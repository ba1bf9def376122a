"""nuts_potential_grad on the caller's row-major data against the same
evaluation on laid-out data: ragged row counts, every column shape, pointers
aligned to one element only, host and device arguments, refused labels.

Both take the same fp64 sums in another order over N rows: U is a sum of
positive terms (1e-13 relative), grad U within 1e-13 of the summed terms'
magnitude.
"""
import numpy as np
import pytest

import workloads
from tests.gpu_common import grad_tol, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sampler():
    import paper_1912_11554_amd as nuts
    return nuts.Sampler(0)


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("N,D", [(1, 1), (127, 8), (129, 9), (2049, 12), (4100, 16), (31, 17), (4097, 25), (20001, 55),
                                 (65, 64), (1111, 65), (515, 128), (2051, 129), (77, 256), (1003, 257), (3001, 320)])
def test_matches_laid_out_data(sampler, dt, N, D):
    import torch

    X, y, w = workloads.make_logistic(N, D, w_scale=0.5, key=[80, N * 1000 + D], dtype=dt)
    say("oneshot", N, D, dt)
    d = sampler.data(X, y)
    U_ref, g_ref = d.potential_grad(w[None], prior_scale=1.7)
    # rows that start one element into an allocation
    flat = torch.zeros(N * D + 1, dtype=torch.float64 if dt == "f64" else torch.float32, device="cuda")
    flat[1:] = torch.from_numpy(X.reshape(-1)).cuda()
    yflat = torch.zeros(N + 3, dtype=torch.uint8, device="cuda")
    yflat[3:] = torch.from_numpy(y).cuda()
    for Xa, ya in ((X, y), (flat[1:].view(N, D), yflat[3:])):
        U, g = sampler.potential_grad(Xa, ya, w, prior_scale=1.7)
        assert abs(U - U_ref[0]) <= 1e-13 * abs(U_ref[0])
        assert (np.abs(g - g_ref[0]) <= grad_tol(X, w, g_ref[0], 1.7, 1e-13)).all()


def test_device_position_and_outputs(sampler):
    import torch

    import paper_1912_11554_amd as nuts

    N, D = 700, 13
    X, y, w = workloads.make_logistic(N, D, w_scale=0.5, key=[81, N])
    U_ref, g_ref = sampler.potential_grad(X, y, w)
    t = [torch.from_numpy(a).cuda() for a in (X, y, w)]
    U = torch.zeros(1, dtype=torch.float64, device="cuda")
    g = torch.zeros(D, dtype=torch.float64, device="cuda")
    say("oneshot device pointers")
    rc = sampler._L.nuts_potential_grad(sampler._h, t[0].data_ptr(), t[1].data_ptr(), N, D, nuts.NUTS_F64, 1.0,
                                        t[2].data_ptr(), U.data_ptr(), g.data_ptr())
    assert rc == nuts.NUTS_OK
    assert float(U[0]) == U_ref and (g.cpu().numpy() == g_ref).all()


@pytest.mark.parametrize("at", [0, 500, 999])
def test_bad_label_is_refused(sampler, at):
    import paper_1912_11554_amd as nuts

    X, y, w = workloads.make_logistic(1000, 5, w_scale=0.5, key=[82, 1])
    ref = sampler.potential_grad(X, y, w)
    bad = y.copy()
    bad[at] = 2
    say("oneshot bad label", at)
    with pytest.raises(nuts.NutsError) as e:
        sampler.potential_grad(X, bad, w)
    assert e.value.code == nuts.NUTS_EINVAL and "other than 0 or 1" in str(e.value)
    again = sampler.potential_grad(X, y, w)  # the next call is not affected
    assert again[0] == ref[0] and (again[1] == ref[1]).all()

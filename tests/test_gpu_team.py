"""GPU parity of chains that share the device on the grid path: data sets held
in LDS as 64-row tiles on one group or several a chain (D <= 64), several
chains a launch, data of their own, and the streaming kernels beside them.

Bars as in test_gpu_sampler.py: decisions bit-exact, positions and energies
within 1e-9 for fp64 data; for fp32 data positions within 1e-6 and the
acceptance statistic, a mean of exponentials of energy differences, within the
no-cancellation bound 3e-8 N of the fp32 row losses.
"""
import numpy as np
import pytest

import workloads
from tests.gpu_common import compare_chain, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sampler():
    import paper_1912_11554_amd as nuts
    return nuts.Sampler(0)


def _check(orc, X, y, r, chains, key, per_chain=False, **kw):
    f32 = X.dtype == np.float32
    N = X.shape[-2]
    for c in chains:
        Xc, yc = (X[c], y[c]) if per_chain else (X, y)
        ref = orc.nuts(Xc.astype(np.float64), yc, seed=key, chain=c, **kw)
        compare_chain(r["samples"][c], r["stats"][c], ref, atol=1e-6 if f32 else 1e-9,
                      accept_atol=max(1e-6, 3e-8 * N) if f32 else None)


# rows around a tile, around the tiles of one round of a group's seven workers
# and around the most that run on a lone group; columns on either side of every
# tile shape
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("N,D", [(1, 1), (63, 4), (64, 5), (65, 8), (448, 9), (449, 12), (2240, 4), (2241, 13),
                                 (1000, 16), (1537, 17), (700, 24), (513, 25), (900, 32), (321, 33), (640, 48),
                                 (257, 49), (1111, 64)])
def test_tiles(sampler, orc, N, D, dtype):
    X, y, _ = workloads.make_logistic(N, D, w_scale=0.8 / np.sqrt(D), key=[70, 1000 * N + D], dtype=dtype)
    kw = dict(step_size=0.5 / np.sqrt(0.2 * N + 1), max_tree_depth=6, num_warmup=1, num_samples=6)
    say("team tiles", N, D, dtype)
    r = sampler.sample(X, y, num_chains=3, seed=21, path=2, **kw)
    _check(orc, X, y, r, range(3), 21, **kw)


@pytest.mark.parametrize("C,N,D", [(5, 700, 3), (40, 130, 11), (70, 900, 20), (300, 260, 30)])
def test_chains_with_their_own_data(sampler, orc, C, N, D):
    sets = [workloads.make_logistic(N, D, w_scale=0.8 / np.sqrt(D), key=[71, 1000 * N + c]) for c in range(C)]
    X, y = np.stack([s[0] for s in sets]), np.stack([s[1] for s in sets])
    kw = dict(step_size=0.5 / np.sqrt(0.2 * N + 1), max_tree_depth=6, num_warmup=0, num_samples=5)
    say("team per-chain data", C, N, D)
    r = sampler.sample(X, y, num_chains=C, seed=22, per_chain=True, **kw)
    _check(orc, X, y, r, sorted({0, 1, C // 2, C - 2, C - 1}), 22, per_chain=True, **kw)


def test_wide_data_of_their_own_is_refused(sampler):
    import paper_1912_11554_amd as nuts
    sets = [workloads.make_logistic(20, 65, w_scale=0.1, key=[75, c]) for c in range(3)]
    X, y = np.stack([s[0] for s in sets]), np.stack([s[1] for s in sets])
    say("wide per-chain data")
    for path in (nuts.NUTS_PATH_AUTO, nuts.NUTS_PATH_WAVE, nuts.NUTS_PATH_GRID, nuts.NUTS_PATH_BATCH):
        with pytest.raises(nuts.NutsError) as e:
            sampler.sample(X, y, step_size=0.1, num_chains=3, num_warmup=0, num_samples=1, max_tree_depth=2,
                           per_chain=True, path=path)
        assert e.value.code == nuts.NUTS_EUNSUPPORTED


# launches of fewer chains than the call has: shared rows that need several
# groups a chain; and wide rows, which stream, side by side
@pytest.mark.parametrize("C,N,D", [(12, 20000, 25), (150, 3000, 10), (9, 1500, 100), (130, 4000, 70),
                                   (257, 2000, 130)])
def test_chains_over_several_launches(sampler, orc, C, N, D):
    X, y, _ = workloads.make_logistic(N, D, w_scale=0.8 / np.sqrt(D), key=[72, 1000 * N + D])
    kw = dict(step_size=0.5 / np.sqrt(0.2 * N + 1), max_tree_depth=5, num_warmup=0, num_samples=4)
    say("team launches", C, N, D)
    r = sampler.sample(X, y, num_chains=C, seed=23, **kw)
    _check(orc, X, y, r, sorted({0, C // 2 - 1, C // 2, C - 1}), 23, **kw)
    assert r["grad_evals"] == int(r["stats"]["num_steps"].sum()) + C


# wide rows beyond the caches: chains that share the device take no longer than
# the same chains one after another (a lone chain's step reads all the rows at
# the memory's rate; 130 at once on one group each took 1.15 times as long)
def test_many_wide_chains_no_slower_than_in_turn(sampler):
    import torch
    N, D, C = 500000, 200, 130
    g = torch.Generator(device="cuda").manual_seed(1)
    X = torch.randn(N, D, generator=g, device="cuda", dtype=torch.float64)
    y = (torch.rand(N, generator=g, device="cuda") < 0.5).to(torch.uint8)
    say("wide chains in turn", N, D, C)
    d = sampler.data(X, y)
    del X
    us = {}
    for c in (1, 1, C):  # (the first call loads the kernel)
        r = d.sample(step_size=1e-7, max_tree_depth=3, num_warmup=0, num_samples=4, num_chains=c, seed=1,
                     time_kernel=True)
        us[c] = 1e3 * r["kernel_ms"] / r["grad_evals"]
    d.free()
    assert us[C] < us[1], us


@pytest.mark.parametrize("extra", [dict(uturn_generalized=True), dict(subtree_merge=True),
                                   dict(adapt_step_size=True)])
@pytest.mark.parametrize("N,D", [(500, 6), (3000, 21)])
def test_optional_features(sampler, orc, N, D, extra):
    X, y, _ = workloads.make_logistic(N, D, w_scale=0.8 / np.sqrt(D), key=[73, 1000 * N + D])
    kw = dict(step_size=0.5 / np.sqrt(0.2 * N + 1), max_tree_depth=6, num_warmup=8, num_samples=6, **extra)
    say("team features", N, D, extra)
    r = sampler.sample(X, y, num_chains=2, seed=24, **kw)
    _check(orc, X, y, r, range(2), 24, **kw)


# one chain whose rows no longer fit in the device's LDS: the streaming kernels
# of the narrow shapes
@pytest.mark.parametrize("N,D", [(1250000, 4), (500000, 11), (300000, 20)])
def test_narrow_rows_that_stream(sampler, orc, N, D):
    X, y, _ = workloads.make_logistic(N, D, w_scale=0.8 / np.sqrt(D), key=[74, D])
    kw = dict(step_size=0.5 / np.sqrt(0.2 * N + 1), max_tree_depth=4, num_warmup=0, num_samples=2)
    say("grid stream", N, D)
    r = sampler.sample(X, y, seed=25, **kw)
    # energies are sums over N rows: the acceptance statistic within 1e-12 |H|
    ref = orc.nuts(X, y, seed=25, chain=0, **kw)
    compare_chain(r["samples"][0], r["stats"][0], ref, accept_atol=1e-12 * N)

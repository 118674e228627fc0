"""Sets that one block propagates (up to 3072 rows): steps and paces_expmv
against the same run with the launches of larger sets, which event timing
(profile level 1) always takes.  The arithmetic of a row is the same, so
amplitudes per basis state, sets, counts, K and spectral bounds agree bit for
bit; norm, energy, populations and a(t) are sums in another order, within
4 n u of their terms' sum (n <= 3072 rows, u = 2^-53: 1.4e-12 of at most 1,
or of the spectrum's width for the energy).  The sizes cross the block's
limit while the set grows, so that a step outgrows it in place and from
scratch."""
import numpy as np
import pytest

import paper_2603_07341_amd as P
from tests.gpu_helpers import sort_rows
import workloads as WL

pytestmark = pytest.mark.gpu

SUM_TOL = 4 * 3072 * 2.0 ** -53


@pytest.mark.parametrize("name,over,steps", [
    ("ring4", {}, 60),                                     # 1 row to 2500
    ("ring4", dict(precision=32), 30),
    ("ring16", dict(eps_sigma=0.05, eps_seed=3, k=2, k_init=2), 24),
    ("ring16", dict(precision=32, k=2, k_init=2), 24),     # holes, two words
    ("sq6x6", dict(precision=64, max_states=0), 5),        # 2D, six columns
    ("sq6x6", dict(extent=[3, 3, 1], precision=64, max_states=2000, n_modes=2,
                   cutoff=[5, 3], omega=[1.0, 0.3], g=[1.0, 0.4]), 12),
    ("cube4", dict(extent=[3, 3, 3], n_modes=1, cutoff=[5], omega=[1.0],
                   g=[1.0], precision=64, max_states=3000), 14),
])
def test_steps_equal_the_spread_launches(name, over, steps):
    cfg = dict(WL.CONFIGS[name], **over)
    p, run, init = WL.model_params(cfg), WL.run_params(cfg), WL.initial_state(cfg)
    a, b = (P.Sim(P.Model(p), run, *init) for _ in range(2))
    b.profile(True)
    a.step(steps)
    b.step(steps)
    ka, aa = sort_rows(*a.state())
    kb, ab = sort_rows(*b.state())
    assert np.array_equal(ka, kb)
    assert np.array_equal(aa, ab)
    ra, rb = a.series(), b.series()
    exact = [0, 7, 8, 9, 10, 11]  # t, n_S, n_M, K, E_min, E_max
    assert np.array_equal(ra[:, exact], rb[:, exact])
    width = (rb[:, 11] - rb[:, 10])[:, None]
    assert np.all(np.abs(ra[:, 2:3] - rb[:, 2:3]) <= SUM_TOL * width)
    rest = [1, 3, 4, 5] + list(range(12, ra.shape[1]))
    assert np.all(np.abs(ra[:, rest] - rb[:, rest]) <= SUM_TOL)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 1024, 1025, 2049, 3071,
                               3072, 3073])
def test_expmv_about_the_limit(n):
    import torch
    cfg = dict(WL.CONFIGS["ring16"])
    m = P.Model(WL.model_params(cfg))
    exc, occ, coef = WL.phonon_ball_state(cfg, 3)
    rng = np.random.default_rng(n)
    on = np.sort(rng.permutation(len(exc))[:n])
    keys = m.pack(exc[on], occ[on])
    amps = coef.view(np.complex128)[on]
    out = m.expmv(torch.from_numpy(keys.view(np.int64)).cuda(),
                  torch.from_numpy(amps.copy()).cuda(), cfg["dt"]).cpu().numpy()
    # a sim on exactly this set (theta 0, k 0) with the spread launches
    s = P.Sim(m, dict(WL.run_params(cfg), theta=0.0, k=0, k_init=0),
              *WL.initial_state(cfg))
    s.set_state(keys, amps)
    s.profile(True)
    s.step(1)
    k, a = sort_rows(*s.state())
    order = np.lexsort(keys.T[::-1])
    assert np.array_equal(k, keys[order])
    assert np.array_equal(a, out[order])


@pytest.mark.parametrize("over,steps", [
    (dict(extent=[65, 1, 1], cutoff=[2], k=1, k_init=1), 10),
    (dict(extent=[100, 1, 1], cutoff=[2], k=1, k_init=2), 8),
    (dict(extent=[300, 1, 1], cutoff=[1], k=1, k_init=1, init="local",
          precision=32), 20),
])
def test_small_sets_on_more_sites_than_a_wave(over, steps):
    # the record's populations come from several waves; each must land in
    # its own step's record
    test_steps_equal_the_spread_launches("ring16", over, steps)

"""paces_expmv builds the columns of a given set from one lookup per pair of
slots; a sim on exactly this set (theta 0, k 0) looks every slot up.  The
arithmetic of a row is the same, so the amplitudes agree bit for bit.  The
sets are random parts of a grown one, so that neighbours are missing in both
directions: one row, the edges of a block and of the one-block limit, and all
rows; one to three dimensions, one to four modes, one to ten key words.  A key
held by the first and the last row is refused."""
import numpy as np
import pytest

import paper_2603_07341_amd as P
from tests.gpu_helpers import sort_rows
import workloads as WL

pytestmark = pytest.mark.gpu

SHAPES = {
    "ring16": ("ring16", {}),
    "open4": ("ring4", dict(periodic=[0, 0, 0])),
    "sq6x6": ("sq6x6", dict(max_states=0)),
    "cube4": ("cube4", dict(max_states=0)),
    "line-4-modes": ("ring4", dict(n_modes=4, cutoff=[3, 2, 4, 1],
                                   omega=[1.0, 0.7, 0.4, 1.3],
                                   g=[0.6, 0.5, 0.4, 0.3])),
}


@pytest.fixture(scope="module", params=list(SHAPES))
def grown(request):
    name, over = SHAPES[request.param]
    cfg = dict(WL.CONFIGS[name], precision=64, n_real=1, **over)
    run = dict(WL.run_params(cfg), max_states=0, theta=1e-6, k=2, k_init=3)
    m = P.Model(WL.model_params(cfg))
    s = P.Sim(m, run, *WL.initial_state(cfg))
    for _ in range(40):
        s.step(1)
        if s.size() > 5000:
            break
    return cfg, run, m, s.state()[0]


@pytest.mark.parametrize("n", [1, 255, 257, 3073, 10 ** 9])
def test_columns_of_a_given_set(grown, n):
    import torch
    cfg, run, m, all_keys = grown
    rng = np.random.default_rng(n)
    n = min(n, len(all_keys))
    keys = np.ascontiguousarray(all_keys[rng.permutation(len(all_keys))[:n]])
    amps = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    amps /= np.linalg.norm(amps)
    kd = torch.from_numpy(keys.view(np.int64)).cuda()
    pd = torch.from_numpy(amps).cuda()
    out = m.expmv(kd, pd, cfg["dt"]).cpu().numpy()
    s = P.Sim(m, dict(run, theta=0.0, k=0, k_init=0), *WL.initial_state(cfg))
    s.set_state(keys, amps)
    s.profile(True)
    s.step(1)
    k, a = sort_rows(*s.state())
    order = np.lexsort(keys.T[::-1])
    assert np.array_equal(k, keys[order])
    assert np.array_equal(a, out[order])
    if n > 1:
        kd[n - 1] = kd[0]
        with pytest.raises(P.PacesError) as e:
            m.expmv(kd, pd, cfg["dt"])
        assert e.value.status == 1


@pytest.mark.parametrize("dt", [-0.01, -0.2, -2.5])
@pytest.mark.parametrize("n", [2500, 20000])
def test_backwards_in_time(n, dt):
    # H is real, so exp(+i H t) phi is the conjugate of exp(-i H t) conj(phi):
    # the same operations with the imaginary parts negated, hence bit for bit
    import torch
    cfg = dict(WL.CONFIGS["ring16"])
    m = P.Model(WL.model_params(cfg))
    exc, occ, _ = WL.phonon_ball_state(cfg, 4)
    rng = np.random.default_rng(n)
    on = np.sort(rng.permutation(len(exc))[:n])
    kd = torch.from_numpy(m.pack(exc[on], occ[on]).view(np.int64)).cuda()
    amps = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    phi = torch.from_numpy(amps / np.linalg.norm(amps)).cuda()
    back = m.expmv(kd, phi, dt)
    ref = m.expmv(kd, phi.conj().resolve_conj(), -dt)
    assert torch.equal(back, ref.conj().resolve_conj())
    # and it undoes the step forward (128 u |.|_inf per application)
    there = m.expmv(kd, back, -dt)
    bound = 2 * 128 * 2.0 ** -53 * float(phi.abs().max())
    assert float((there - phi).abs().max()) <= bound * max(1.0, abs(dt) * 40)

"""The cut of one realization to its heaviest rows, decided on the GPU: sets
given through paces_set_state with weights made for the edges of the radix
select, truncated to a fixed size (q_nom, k = 0, so the new set is the
selection itself), against a sort by (weight descending, splitmix64 hash of
the key, key).  Selections must agree exactly: no tolerance."""
import numpy as np
import pytest

import paper_2603_07341_amd as P
import workloads as WL

pytestmark = pytest.mark.gpu

M64 = np.uint64(0xFFFFFFFFFFFFFFFF)


def mix(x):
    with np.errstate(over="ignore"):
        z = x + np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))


def heaviest(keys, amps, q):
    h = np.zeros(len(keys), dtype=np.uint64)
    for w in range(keys.shape[1]):
        h = mix(h ^ keys[:, w])
    wt = amps.real * amps.real + amps.imag * amps.imag
    order = np.lexsort(tuple(keys.T[::-1]) + (h, -wt))
    return keys[np.sort(order[:q])]


def weights(kind, n, rng):
    if kind == "spread":      # heavy tail, all distinct
        return 10.0 ** (-14 * rng.random(n))
    if kind == "close":       # one exponent, mantissas that differ late
        return 1.0 + np.arange(n)[rng.permutation(n)] * 2.0 ** -40
    if kind == "orbits":      # groups of sixteen equal amplitudes
        return np.repeat(10.0 ** (-9 * rng.random(-(-n // 16))), 16)[:n]
    if kind == "equal":       # more ties than the device orders
        return np.full(n, 0.25)
    w = 10.0 ** (-9 * rng.random(n))
    w[rng.random(n) < 0.6] = 0.0   # "zeros": most rows without amplitude
    return w


@pytest.mark.parametrize("name", ["ring16", "cube4"])
@pytest.mark.parametrize("kind", ["spread", "close", "orbits", "equal", "zeros"])
@pytest.mark.parametrize("n,q", [(2, 1), (300, 299), (4000, 1), (5000, 3001),
                                 (5000, 5000), (60000, 31237)])
def test_cut_keeps_the_heaviest(name, kind, n, q):
    cfg = dict(WL.CONFIGS[name], precision=64)
    m = P.Model(WL.model_params(cfg))
    rng = np.random.default_rng(n + q)
    N, V = WL.n_sites(cfg), cfg["n_modes"]
    occ = rng.integers(0, 4, (2 * n, N * V)).astype(np.uint16)
    exc = rng.integers(0, N, 2 * n).astype(np.int32)
    keys = np.unique(m.pack(exc, occ), axis=0)
    keys = keys[rng.permutation(len(keys))[:n]]
    assert len(keys) == n
    amps = (weights(kind, n, rng) + 0j)
    run = dict(WL.run_params(cfg), max_states=0, q_nom=q, theta=0.0, k=0,
               k_init=0)
    s = P.Sim(m, run, *WL.initial_state(cfg))
    s.set_state(keys, amps)
    s.step(1)
    got = s.get_set(P.SET_M)
    want = heaviest(keys, amps, q)
    sort = lambda a: a[np.lexsort(a.T[::-1])]  # noqa: E731
    assert np.array_equal(sort(got), sort(want))
    assert np.array_equal(sort(s.get_set(P.SET_S)), sort(want))

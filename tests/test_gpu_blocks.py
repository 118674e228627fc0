"""Freed device blocks that the library keeps for later allocations: calls
from several threads on their own streams, sims made and freed in between,
and sets of changing size give what single calls on fresh memory give, bit
for bit (amplitudes do not depend on row order or memory)."""
import threading

import numpy as np
import pytest

import paper_2603_07341_amd as P
from tests.gpu_helpers import sort_rows
import workloads as WL

pytestmark = pytest.mark.gpu


def inputs(m, cfg, n_max):
    import torch
    exc, occ, coef = WL.phonon_ball_state(cfg, n_max)
    keys = torch.from_numpy(m.pack(exc, occ).view(np.int64)).cuda()
    return keys, torch.from_numpy(coef.view(np.complex128).copy()).cuda()


@pytest.mark.parametrize("threads", [1, 4])
def test_expmv_and_sims_reuse_blocks(threads):
    import torch
    cfg = dict(WL.CONFIGS["ring16"])
    run, init = WL.run_params(cfg), WL.initial_state(cfg)
    m = P.Model(WL.model_params(cfg))
    sets = [inputs(m, cfg, n) for n in (1, 2, 3)]
    ref = [m.expmv(k, p, 0.01).cpu().numpy() for k, p in sets]
    s = P.Sim(m, run, *init)
    s.step(4)
    ref_state = sort_rows(*s.state())
    s.close()
    bad = []

    def work(which):
        try:
            st = torch.cuda.Stream()
            with torch.cuda.stream(st):
                for i in range(6):
                    q = (i + which) % len(sets)
                    out = m.expmv(*sets[q], 0.01, stream=st)
                    st.synchronize()
                    if not np.array_equal(out.cpu().numpy(), ref[q]):
                        bad.append(("expmv", which, i))
                    sim = P.Sim(m, run, *init, stream=st)
                    sim.step(4, stream=st)
                    k, a = sort_rows(*sim.state(stream=st))
                    sim.close()
                    if not (np.array_equal(k, ref_state[0]) and
                            np.array_equal(a, ref_state[1])):
                        bad.append(("sim", which, i))
        except Exception as e:  # reported by the main thread
            bad.append(repr(e))

    ts = [threading.Thread(target=work, args=(w,)) for w in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad, bad[:3]

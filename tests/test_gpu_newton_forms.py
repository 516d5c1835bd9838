"""The Newton solver on both sides of its dispatch: an env whose joint sides and contact slots fit the 64 lanes
of a wavefront (2 J + S <= 64) is solved by one, a larger one by the whole workgroup."""
import numpy as np
import pytest

import oracle
import scenes
from helpers import TOL_1, rel_err4

pytestmark = pytest.mark.gpu


def _scene(links, n, terrain, share):
    # a chain that lies on the ground: 3 slots per link; 12 links fill 60 lanes, 13 would need 65
    rob = scenes.make_chain(n_links=links, seg_len=0.2, direction=(1.0, 0.0, 0.0), top=(0.0, 0.0, 0.02), lo=-0.4, hi=0.4, world_anchor=True)
    ter = scenes.make_heightfield(seed=3) if terrain == "field" else scenes.make_plane()
    sc = scenes.make_scene(rob, ter, n, params=scenes.SimParams(solver=1, krylov_iters=8, warm_start=share))
    return sc


@pytest.mark.parametrize("share", [0.0, 0.8])
@pytest.mark.parametrize("terrain", ["plane", "field"])
@pytest.mark.parametrize("links", [1, 12, 13, 16])
def test_newton_step_at_the_edge_of_a_wavefront(links, terrain, share):
    """One step from a moving state against the oracle (a cut-off iterate may take another branch in an
    env: the bulk within the state tolerance of one step, nothing beyond 1e-2), and the same bits however
    many envs share a workgroup."""
    import paper_1810_05762_amd as P
    n = 13
    sc = _scene(links, n, terrain, share)
    dt = float(np.float32(1.0 / 60.0))
    outs = []
    for epb in (1, 2, 4, 8, 5) if links <= 12 else (1, 2, 4, 3):   # (a larger env's slots need more threads)
        sim = P.Sim(sc)
        sim.set_envs_per_block(epb)
        sim.reset(5)
        for s in range(12):
            sim.step(scenes.actions_for_step(2, s, n, sc.robot.n_dofs), dt, 4, 3)
        start = sim.get_state()
        sim.set_state(start)
        sim.record_contacts(True)
        sim.step(scenes.actions_for_step(2, 12, n, sc.robot.n_dofs), dt, 4, 3)
        outs.append((start.cpu().numpy(), sim.get_state().cpu().numpy()))
        touching = sim.get_contacts()["active"].sum()
        sim.check(); sim.close()
    for o in outs[1:]:
        assert np.array_equal(o[0], outs[0][0]) and np.array_equal(o[1], outs[0][1])
    assert touching > 0
    ref = oracle.OracleSim(sc, threads=4)
    ref.set_state(outs[0][0].astype(np.float64))
    ref.step(scenes.actions_for_step(2, 12, n, sc.robot.n_dofs), dt, 4, 3)
    e = rel_err4(outs[0][1].astype(np.float64), ref.get_state()).max(1)
    print(links, terrain, share, np.median(e), e.max())
    assert np.median(e) <= TOL_1 and e.max() <= 1e-2

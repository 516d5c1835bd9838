"""Lanes per joint at their edges: one, two or four lanes relax a joint, by the number of envs in a workgroup, and the
lanes behind the last joint repeat its work.  Chains whose joints fill a wavefront exactly, leave most of one over
or hang from the world, against the oracle, and the same bits whatever the number of lanes."""
import numpy as np
import pytest

import oracle
import scenes
from helpers import TOL_1, folded_chains, rel_err4

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("links,anchored", [(1, True), (5, True), (14, False), (16, True)])
@pytest.mark.parametrize("extra", [{}, {"warm_start": 0.8}, {"self_collide": 1}], ids=["plain", "warm", "pairs"])
def test_joint_lanes_at_the_edges_of_wavefronts(links, anchored, extra):
    import paper_1810_05762_amd as P
    n = 19
    rob = scenes.make_chain(n_links=links, seg_len=0.15, direction=(1.0, 0.0, 0.0), top=(0.0, 0.0, 0.12), world_anchor=anchored)
    sc = scenes.make_scene(rob, scenes.make_plane(), n, params=scenes.SimParams(**extra))
    dt, sub, its = float(np.float32(1.0 / 60.0)), 4, 16
    act = [scenes.actions_for_step(5, s, n, max(rob.n_dofs, 1))[:, :rob.n_dofs] for s in range(9)]
    outs = []
    for epb in (1, 2, 3, 4, 8, 16):
        if 2 * epb * rob.n_joints > 448:      # (more than a workgroup takes)
            continue
        sim = P.Sim(sc)
        sim.set_envs_per_block(epb)
        sim.reset(11)
        for s in range(8):
            sim.step(act[s], dt, sub, its)
        start = sim.get_state()
        sim.set_state(start)                  # (both sides begin without kept impulses)
        sim.set_step_count(8)
        sim.step(act[8], dt, sub, its)
        outs.append([start.cpu().numpy(), sim.get_state().cpu().numpy()] + [x.cpu().numpy() for x in sim.get_obs()])
        sim.check(); sim.close()
    ref = oracle.OracleSim(sc, threads=4)
    ref.set_state(outs[0][0].astype(np.float64))
    ref.step(act[8], dt, sub, its)
    # one step in single precision: the bound of the other one-step comparisons with the oracle
    assert rel_err4(outs[0][1].astype(np.float64), ref.get_state()).max() <= TOL_1
    for o in outs[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(o, outs[0]))


@pytest.mark.parametrize("links", [12, 14])
@pytest.mark.parametrize("warm", [0.0, 0.8])
def test_one_lane_per_joint_reads_the_velocity_of_the_world_as_zero(links, warm):
    """Chains that hang from the world and are folded up: the candidate pairs of the search lie where the first sweep
    reads the world's velocity, and with 12 and 14 joints of 16 envs some wavefronts of joints clear none of it."""
    import paper_1810_05762_amd as P
    n = 32
    rob = scenes.make_chain(n_links=links, seg_len=0.15, direction=(1.0, 0.0, 0.0), top=(0.0, 0.0, 0.4))
    sc = scenes.make_scene(rob, scenes.make_plane(), n, params=scenes.SimParams(self_collide=1, warm_start=warm))
    start = folded_chains(rob, n).astype(np.float32)
    act = scenes.actions_for_step(5, 0, n, rob.n_dofs)
    dt, sub, its = float(np.float32(1.0 / 60.0)), 4, 16
    outs = []
    for epb in (2, 8, 16):
        sim = P.Sim(sc)
        sim.set_envs_per_block(epb)
        sim.record_contacts(True)
        sim.set_state(start)
        sim.step(act, dt, sub, its)
        pairs, dropped = sim.get_pair_contacts()
        assert len(pairs) >= n and dropped == 0
        outs.append([sim.get_state().cpu().numpy()] + [x.cpu().numpy() for x in sim.get_obs()])
        sim.check(); sim.close()
    ref = oracle.OracleSim(sc, threads=4)
    ref.set_state(start.astype(np.float64))
    ref.step(act, dt, sub, its)
    assert rel_err4(outs[0][0].astype(np.float64), ref.get_state()).max() <= TOL_1
    for o in outs[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(o, outs[0]))

"""The reset places a robot's joints a level of its tree at a time: state against the oracle's recipe, which
goes through the joints in order, for deep, flat and looped robots, with masks and ragged last workgroups."""
import numpy as np
import pytest

import oracle
import scenes
from scenes.robots import _Builder

pytestmark = pytest.mark.gpu


def _robots():
    chain = scenes.make_chain(n_links=14, seg_len=0.1, top=(0.0, 0.0, 3.0))
    bld = _Builder("loop")      # body 2 is the child of two joints: no tree, joint after joint
    for k, x in enumerate((0.0, 0.4, 0.8)):
        bld.body(f"b{k}", 0.05, 0.3, 0, (x, 0.0, 1.0), mass=1.0)
    for pa, pb, x in ((0, 1, 0.2), (1, 2, 0.6), (0, 2, 0.5)):
        bld.joint(pa, pb, (x, 0.0, 1.0), [((0.0, 1.0, 0.0), -1.0, 1.0)], 1.0)
    return {"chain14": chain, "loop": bld.build(root_body=0, feet=(), term_height=-1e9, alive_bonus=0.0),
            "star": scenes.make_star(), "single": scenes.make_single(), "ant": scenes.make_ant(), "humanoid": scenes.make_humanoid()}


@pytest.mark.parametrize("epb", [1, 4, 5, 16])
@pytest.mark.parametrize("name", ["chain14", "loop", "star", "single", "ant", "humanoid"])
def test_reset_of_every_kind_of_tree_matches_the_oracle(name, epb):
    """A pose is at most 14 rotations from the root: 16 x 2^-22 (sums of a few rounded products of order 1
    each, velocities of order 2) is 4e-6."""
    import paper_1810_05762_amd as P
    n = 2 * epb + 1
    sc = scenes.make_scene(_robots()[name], scenes.make_plane(), n, params=scenes.SimParams(warm_start=0.8 if epb == 4 else 0.0))
    sim, ref = P.Sim(sc), oracle.OracleSim(sc)
    sim.set_envs_per_block(epb)
    sim.reset(7); ref.reset(7)
    np.testing.assert_allclose(sim.get_state().cpu().numpy(), ref.get_state(), atol=4e-6)
    for s in range(3):
        sim.step(scenes.actions_for_step(3, s, n, max(sc.robot.n_dofs, 1))[:, :sc.robot.n_dofs], 1.0 / 60.0, 4, 4)
    before = sim.get_state().cpu().numpy()
    mask = np.zeros(n, np.uint8); mask[[0, n - 1]] = 1
    sim.reset(8, mask); ref.reset(8, mask)
    after = sim.get_state().cpu().numpy()
    np.testing.assert_allclose(after[mask == 1], ref.get_state()[mask == 1], atol=4e-6)
    assert np.array_equal(after[mask == 0], before[mask == 0])
    # the observation, reward and done flag of every env are those of the state it now has
    ref.set_state(after.astype(np.float64)); ref.set_step_count(0)
    np.testing.assert_allclose(sim.get_obs()[0].cpu().numpy()[mask == 1], ref.get_obs()[0][mask == 1], atol=1e-4)
    sim.check(); sim.close()


@pytest.mark.parametrize("share", [0.0, 0.8])
@pytest.mark.parametrize("name", ["chain14", "loop", "star", "single", "humanoid"])
def test_reset_of_many_workgroups_gives_the_bits_of_one_launch(name, share):
    """More than six rounds of workgroups (1536) are reset by a kernel of their own ahead of the step kernel's
    launch, fewer inside it: the same state, observation, reward, done flag, step counter and kept impulses."""
    import paper_1810_05762_amd as P
    n = 1537
    rob = _robots()[name]
    rob.term_height = -1e9
    sc = scenes.make_scene(rob, scenes.make_plane(), n, params=scenes.SimParams(warm_start=share, max_episode_steps=4))
    mask = np.zeros(n, np.uint8); mask[[0, 5, 64, n - 1]] = 1
    ref = oracle.OracleSim(sc)
    ref.reset(7)
    outs = []
    for epb in (1, 2, 5):
        sim, got = P.Sim(sc), []
        sim.set_envs_per_block(epb)
        sim.reset(7)
        got += [sim.get_state().cpu().numpy()] + [x.cpu().numpy() for x in sim.get_obs()]
        np.testing.assert_allclose(got[0], ref.get_state(), atol=4e-6)
        for s in range(3):
            sim.step(scenes.actions_for_step(3, s, n, max(rob.n_dofs, 1))[:, :rob.n_dofs], 1.0 / 60.0, 2, 4)
        sim.reset(8, mask)
        got += [sim.get_state().cpu().numpy()] + [x.cpu().numpy() for x in sim.get_obs()]
        sim.step(None, 1.0 / 60.0, 2, 4)          # the fourth step of the envs that were not reset: their episode is over
        got += [sim.get_state().cpu().numpy()] + [x.cpu().numpy() for x in sim.get_obs()]
        assert np.array_equal(got[-1] != 0, mask == 0)
        sim.check(); sim.close()
        outs.append(got)
    for o in outs[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(o, outs[0]))

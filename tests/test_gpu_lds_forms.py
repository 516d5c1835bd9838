"""Workgroups that take nearly all of LDS: small robots with as many envs as fit, where the terrain search's lists
have little or no room of their own."""
import numpy as np
import pytest

import scenes
from scenes.robots import _Builder

pytestmark = pytest.mark.gpu


def _robot(kind):
    if kind == "sphere":
        return scenes.make_single(radius=0.1, pos=(0.0, 0.0, 0.1))
    if kind == "capsule":
        return scenes.make_single(radius=0.1, seg_len=0.3, pos=(0.0, 0.0, 0.1))
    if kind == "two spheres":
        return scenes.make_loose([(0.1, 0.0, 0, (0.0, 0.0, 0.1), 1.0), (0.1, 0.0, 0, (0.19, 0.0, 0.1), 1.0)])
    if kind == "two links":
        return scenes.make_chain(n_links=2, seg_len=0.3, direction=(1.0, 0.0, 0.0), top=(0.0, 0.0, 0.03), world_anchor=False)
    bld = _Builder("hinged sphere")
    bld.joint(-1, bld.body("ball", 0.1, 0.0, 0, (0.0, 0.0, 0.08), mass=1.0), (0.0, 0.1, 0.08), [((0.0, 1.0, 0.0), -1.0, 1.0)], 1.0)
    return bld.build(root_body=0, feet=(), term_height=-1e9, alive_bonus=0.0)


@pytest.mark.parametrize("kind,field,collide,epb", [("sphere", False, 0, 441), ("capsule", False, 0, 370), ("two links", False, 0, 205),
                                                    ("sphere", True, 0, 45), ("hinged sphere", True, 0, 44), ("two spheres", True, 1, 40),
                                                    ("sphere", True, 0, 17)])
def test_step_of_the_largest_workgroups_equals_that_of_single_envs(kind, field, collide, epb):
    """The same bits as one env per workgroup: the forms of a family share their arithmetic, and full lists
    only send a slot to the direct search."""
    import paper_1810_05762_amd as P
    n = 2 * epb + 1
    ter = scenes.make_heightfield(seed=5, nx=64, ny=64) if field else scenes.make_plane()
    sc = scenes.make_scene(_robot(kind), ter, n, params=scenes.SimParams(self_collide=collide))
    outs = []
    for E in (1, epb):
        sim = P.Sim(sc)
        sim.set_envs_per_block(E)
        assert sim.launch_info()["lds_bytes"] <= 160 * 1024 - 256
        sim.reset(3)
        for s in range(6):
            sim.step(scenes.actions_for_step(1, s, n, max(sc.robot.n_dofs, 1))[:, :sc.robot.n_dofs], 1.0 / 60.0, 4, 8)
        sim.record_contacts(True)
        sim.step(None, 1.0 / 60.0, 4, 8)
        rec = sim.get_contacts()
        assert rec["active"].sum() > 0
        outs.append((sim.get_state().cpu().numpy(), rec.tobytes()))
        sim.check(); sim.close()
    assert np.isfinite(outs[0][0]).all()
    assert np.array_equal(outs[0][0], outs[1][0]) and outs[0][1] == outs[1][1]


@pytest.mark.parametrize("links,collide,warm,epb", [(4, 1, 0.0, 30), (5, 0, 0.8, 28)])
def test_a_workgroup_beyond_the_last_bytes_of_lds_is_refused(links, collide, warm, epb):
    """The tables of these chains end within the last 256 bytes of the 160 KiB, which the kernel itself uses;
    one env less runs."""
    import paper_1810_05762_amd as P
    rob = scenes.make_chain(n_links=links)
    sc = scenes.make_scene(rob, scenes.make_heightfield(seed=3, nx=64, ny=64), 50, params=scenes.SimParams(self_collide=collide, warm_start=warm))
    sim = P.Sim(sc)
    with pytest.raises(P.SimError):
        sim.set_envs_per_block(epb)
    sim.set_envs_per_block(epb - 1)
    sim.reset(3)
    sim.step(scenes.actions_for_step(1, 0, 50, rob.n_dofs), 1.0 / 60.0, 2, 4)
    assert np.isfinite(sim.get_state().cpu().numpy()).all()
    sim.check(); sim.close()

"""Workgroups that take nearly all of LDS."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("links,warm,epb", [(4, 0.0, 30), (8, 0.8, 21)])
def test_a_workgroup_beyond_the_last_bytes_of_lds_is_refused(links, warm, epb):
    """The tables of these chains end within the last 256 bytes of the 160 KiB, which the kernel itself uses;
    one env less runs."""
    import paper_1810_05762_amd as P
    rob = scenes.make_chain(n_links=links)
    sc = scenes.make_scene(rob, scenes.make_heightfield(seed=3, nx=64, ny=64), 50, params=scenes.SimParams(self_collide=1, warm_start=warm))
    sim = P.Sim(sc)
    with pytest.raises(P.SimError):
        sim.set_envs_per_block(epb)
    sim.set_envs_per_block(epb - 1)
    sim.reset(3)
    sim.step(scenes.actions_for_step(1, 0, 50, rob.n_dofs), 1.0 / 60.0, 2, 4)
    assert np.isfinite(sim.get_state().cpu().numpy()).all()
    sim.check(); sim.close()

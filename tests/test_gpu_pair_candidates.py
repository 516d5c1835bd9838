"""The search for capsule-capsule candidates over its whole range: more body pairs than a thread keeps, more
agent pairs than threads, odd and even body counts, and agents whose origins lie far from zero."""
import numpy as np
import pytest

import oracle
import scenes
from test_gpu_pairs import assert_same_pair_sets

pytestmark = pytest.mark.gpu


def _scene(bodies, group, n, spread, seed):
    rng = np.random.default_rng(seed)
    rob = scenes.make_loose([(0.05, 0.2 if k % 3 else 0.0, k % 3, (0.3 * k, 0.0, 5.0), 1.0) for k in range(bodies)])
    sc = scenes.make_scene(rob, scenes.make_plane(), n, params=scenes.SimParams(gravity=(0.0, 0.0, 0.0), self_collide=1, group_size=group))
    sc.env_origins = np.repeat(rng.uniform(-2000.0, 2000.0, (n // group, 3)) * np.array([1.0, 1.0, 0.0]), group, axis=0)
    sc.env_origins[:, :2] += rng.uniform(-spread, spread, (n, 2))
    sc.env_origins = sc.env_origins.astype(np.float32).astype(np.float64)
    st = np.repeat(scenes.rest_state(rob), n, axis=0)
    st[:, :, 0:3] = np.array([0.0, 0.0, 5.0]) + rng.uniform(-spread, spread, (n, bodies, 3))
    q = rng.normal(size=(n, bodies, 4))
    st[:, :, 3:7] = q / np.linalg.norm(q, axis=2, keepdims=True)
    return sc, st.astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("bodies,group,epb,n", [(14, 1, 32, 64), (14, 1, 5, 12), (16, 1, 1, 4), (16, 1, 16, 48), (4, 16, 128, 256), (1, 16, 256, 256),
                                                (16, 1, 2, 6), (16, 1, 4, 12), (16, 2, 2, 6), (16, 4, 4, 8), (16, 16, 16, 48), (13, 4, 4, 20), (3, 3, 12, 30), (2, 8, 8, 40)])
def test_candidates_of_every_split_equal_the_oracles_contacts(bodies, group, epb, n):
    """The set of contacts after one substep is the oracle's, in workgroups that hold them all."""
    import paper_1810_05762_amd as P
    h = float(np.float32(1.0 / 240.0))
    for spread in (0.2, 0.3, 0.45, 0.7, 1.0, 1.5, 2.2, 3.3, 5.0):      # the densest that a workgroup holds
        sc, st = _scene(bodies, group, n, spread, seed=bodies + epb)
        ref = oracle.OracleSim(sc, threads=4)
        ref.set_state(st); ref.step(None, h, 1, 2)
        po = ref.get_pair_contacts(cap=65536)
        if np.bincount(po["env_a"] // epb, minlength=1).max(initial=0) <= P.binding.SIM_PAIR_CAP - 8:
            break
    assert len(po) > 0
    sim = P.Sim(sc)
    sim.set_envs_per_block(epb)
    sim.set_state(st)
    sim.record_contacts(True)
    sim.step(None, h, 1, 2)
    pg, dropped = sim.get_pair_contacts()
    print(bodies, group, epb, n, spread, len(po))
    assert dropped == 0
    assert_same_pair_sets(pg, po)
    sim.check(); sim.close()

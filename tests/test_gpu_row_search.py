"""The search by rows of cells against the stand-alone generation (one thread per slot over its whole box): rows
cut in pieces, spheres, small and ragged fields, borders."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("epb", [1, 4, 5, 16])
@pytest.mark.parametrize("cell,n,radius,seg", [(0.1, 14, 0.05, 0.3), (0.03, 33, 0.05, 0.3),
                                               (0.02, 40, 0.04, 0.0), (0.4, 2, 0.1, 0.5), (0.1, 29, 0.3, 1.2)])
def test_fused_search_records_what_the_whole_box_gives(cell, n, radius, seg, epb):
    """Byte for byte: both keep the lexicographic minimum of (distance, feature) in one operation order."""
    import paper_1810_05762_amd as P
    rng = np.random.default_rng(n)
    terrain = scenes.make_flat_heightfield(nx=n, ny=n + 1, cell=cell)
    terrain.heights = rng.uniform(0, 1.5 * cell, (n + 1, n)).astype(np.float32)
    rob = scenes.make_single(radius=radius, seg_len=seg, axis=1, pos=(0, 0, 0))
    N = 301
    sc = scenes.make_scene(rob, terrain, N, params=scenes.SimParams(contact_margin=0.02))
    sc.env_origins = rng.uniform(-0.2, 0.2, (N, 3)).astype(np.float32).astype(np.float64)
    st = np.zeros((N, 1, 13))
    st[:, 0, 0:2] = rng.uniform(-0.3, 0.3 + n * cell, (N, 2))
    st[:, 0, 2] = rng.uniform(-radius, 2.0 * radius + 0.5 * seg, N)
    q = rng.normal(size=(N, 4))
    st[:, 0, 3:7] = q / np.linalg.norm(q, axis=1, keepdims=True)
    sim = P.Sim(sc)
    sim.set_envs_per_block(epb)
    sim.set_state(st.astype(np.float32).astype(np.float64))
    sim.record_contacts(True)
    before = sim.generate_contacts()
    sim.step(None, 1e-4, 1, 1)
    rec = sim.get_contacts()
    assert rec["active"].sum() > 10
    assert rec.tobytes() == before.tobytes()
    sim.check(); sim.close()

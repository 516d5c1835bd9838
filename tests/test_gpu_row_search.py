"""The search by rows of cells against the stand-alone generation (one thread per slot over its whole box, from
global memory): rows cut in pieces, boxes and lists too large for the rows, spheres, small and ragged fields, borders
of the field and of the copy that an env keeps of it."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("epb", [1, 4, 5, 16])
@pytest.mark.parametrize("cell,n,radius,seg", [(0.1, 14, 0.05, 0.3), (0.03, 33, 0.05, 0.3), (0.012, 61, 0.05, 0.3), (0.006, 90, 0.05, 0.3),
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


@pytest.mark.parametrize("epb", [1, 4, 5, 16])
@pytest.mark.parametrize("cell,n", [(0.1, 64), (0.03, 80)])
def test_bodies_beside_the_copy_of_the_field(cell, n, epb):
    """The copy reaches 14 cells from the root (1.4 m here at most): the links of a 1.8 m chain that lies on the
    ground in any direction are inside it, across each of its four edges and outside.  Byte for byte, as above."""
    import paper_1810_05762_amd as P
    rng = np.random.default_rng(n)
    terrain = scenes.make_flat_heightfield(nx=n, ny=n + 1, cell=cell)
    terrain.heights = rng.uniform(0, 1.5 * cell, (n + 1, n)).astype(np.float32)
    links, seg, radius = 6, 0.3, 0.05
    rob = scenes.make_chain(n_links=links, seg_len=seg, radius=radius, direction=(1.0, 0.0, 0.0), top=(0.0, 0.0, 0.0), world_anchor=False)
    N = 301
    sc = scenes.make_scene(rob, terrain, N, params=scenes.SimParams(contact_margin=0.02))
    sc.env_origins = rng.uniform(-0.2, 0.2, (N, 3)).astype(np.float32).astype(np.float64)
    yaw, pitch = rng.uniform(-np.pi, np.pi, N), rng.uniform(-0.1, 0.1, N)
    cy, sy, cp, sp = np.cos(0.5 * yaw), np.sin(0.5 * yaw), np.cos(0.5 * pitch), np.sin(0.5 * pitch)
    q = np.stack((cy * cp, -sy * sp, cy * sp, sy * cp), 1)       # yaw about z after pitch about y
    along = np.stack((np.cos(yaw) * np.cos(pitch), np.sin(yaw) * np.cos(pitch), -np.sin(pitch)), 1)
    root = np.stack((rng.uniform(0.0, n * cell, N), rng.uniform(0.0, n * cell, N), rng.uniform(0.0, 3.0 * radius, N)), 1)
    st = np.zeros((N, links, 13))
    st[:, :, 0:3] = root[:, None] + along[:, None] * (seg * np.arange(links))[None, :, None]
    st[:, :, 3:7] = q[:, None]
    sim = P.Sim(sc)
    sim.set_envs_per_block(epb)
    sim.set_state(st.astype(np.float32).astype(np.float64))
    sim.record_contacts(True)
    before = sim.generate_contacts()
    sim.step(None, 1e-4, 1, 1)
    rec = sim.get_contacts()
    assert rec["active"].sum() > 100
    assert rec.tobytes() == before.tobytes()
    sim.check(); sim.close()

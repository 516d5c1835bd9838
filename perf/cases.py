"""The work that users of the simulator have it do, as cases that can be timed and compared.

A case names a robot, a ground, a number of environments, the stepping parameters and a `mode`,
the loop around the step that a program of that kind runs:

  step      one `step_obs` with the next actions of a ring: the inner loop of training a policy
  episodes  `reset` of the environments whose episode has ended, then `step_obs`
  plan      `set_state` to one snapshot, a few steps, `get_state`: candidate rollouts of a planner
  crowd     `step_obs` of colliding agents in one scene, `regroup` before every tenth step

Starting states are robots on the ground (half of them upright, half fallen, joints anywhere within
their limits, moving slowly), drawn from the seed with torch on the GPU, so the first pass already
meets contacts; the passes after it go on from there, as a training run does (`plan` starts over).
"""
import math

import numpy as np
import torch

import paper_1810_05762_amd as sim355
import scenes

DT = 1.0 / 60.0
RING = 8            # action tensors a pass takes in turn
PLAN_STEPS = 3
REGROUP_EVERY = 10
REGROUP_CELL, REGROUP_REACH = 2.4, 1.2   # metres; roots of two touching humanoids are at most about 1.2 m apart


def _case(robot, terrain, envs, substeps, iterations, mode="step", warm=0.0, newton=False, height_map=False,
          self_collide=False, group=1, task=False, state=False):
    return {"robot": robot, "terrain": terrain, "envs": envs, "substeps": substeps, "iterations": iterations,
            "mode": mode, "warm": warm, "newton": newton, "height_map": height_map, "self_collide": self_collide,
            "group": group, "task": task, "state": state}


def listed():
    return [
        # a handful of robots: debugging a reward, evaluating a policy; a step is all latency
        dict(_case("ant", "plane", 16, 2, 8), name="ant16_plane"),
        # a sampling planner: 64 candidate action sequences from one snapshot
        dict(_case("humanoid", "heightfield", 64, 4, 20, mode="plan", state=True), name="plan64_heightfield"),
        # the usual reinforcement-learning batch on flat ground, episodes ending all the time
        dict(_case("ant", "plane", 1024, 4, 16, mode="episodes"), name="ant1024_episodes"),
        # the same batch of humanoids, full body state read back for a privileged critic
        dict(_case("humanoid", "plane", 1024, 4, 20, state=True), name="humanoid1024_plane"),
        # a batch that is no power of two (what is left of a machine shared with a learner)
        dict(_case("humanoid", "heightfield", 1500, 4, 20), name="humanoid1500_heightfield"),
        # the paper's own solver at the batch size its cost allows
        dict(_case("humanoid", "heightfield", 1024, 4, 3, newton=True, state=True), name="newton1024_heightfield"),
        # agents in one shared scene that bump into each other, groups chosen again as they move
        dict(_case("humanoid", "plane", 1000, 4, 20, mode="crowd", self_collide=True, group=16), name="crowd1000_plane"),
        # the headline workload: uneven terrain, one full workgroup on every compute unit
        dict(_case("humanoid", "heightfield", 4096, 4, 20), name="humanoid4096_heightfield"),
        # the same with half the sweeps and the rows warm-started
        dict(_case("humanoid", "heightfield", 4096, 4, 10, warm=0.8), name="warm4096_heightfield"),
        # everything the flagrun tasks use: collisions within and between agents, height map, pushes, targets, auto-reset
        dict(_case("humanoid", "heightfield", 4096, 4, 20, height_map=True, self_collide=True, group=4, task=True),
             name="flagrun4096_heightfield"),
        # many simultaneous contacts at small substeps
        dict(_case("humanoid", "heightfield", 8192, 8, 32), name="humanoid8192_fine_substeps"),
        # as many environments as a large-batch method takes: throughput alone counts
        dict(_case("humanoid", "heightfield", 65536, 4, 20), name="humanoid65536_heightfield"),
    ]


def draw(rng):
    def envs(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    robot = rng.choice(("ant", "humanoid", "humanoid"))
    terrain = rng.choice(("plane", "heightfield", "heightfield"))
    substeps, iterations = rng.choice(((2, 8), (4, 16), (4, 20), (4, 20), (8, 32)))
    kind = rng.choice(("step", "step", "step", "step", "episodes", "plan", "warm", "newton", "flagrun", "crowd"))
    if kind == "step":
        return _case(robot, terrain, envs(1, 20000), substeps, iterations, height_map=rng.random() < 0.2,
                     state=rng.random() < 0.3)
    if kind == "episodes":
        return _case(robot, terrain, envs(64, 16384), substeps, iterations, mode="episodes")
    if kind == "plan":
        return _case(robot, terrain, envs(8, 2048), 4, iterations, mode="plan", state=True)
    if kind == "warm":
        return _case(robot, terrain, envs(16, 8192), substeps, max(8, iterations // 2), warm=0.8)
    if kind == "newton":
        return _case(robot, terrain, envs(16, 4096), 4, rng.choice((2, 3)), newton=True, warm=rng.choice((0.0, 0.8)))
    if kind == "flagrun":
        group = rng.choice((1, 2, 4, 8))
        return _case(robot, terrain, group * envs(8, 8192 // group), 4, 20, height_map=True, self_collide=True,
                     group=group, task=True)
    return _case(robot, "plane", envs(100, 6000), 4, 20, mode="crowd", self_collide=True, group=rng.choice((4, 16)))


# ---- starting states

def _origins(case, terrain, rng):
    """World position of every environment's origin, [N][3], on the ground."""
    n, group = case["envs"], case["group"]
    if case["mode"] == "crowd":
        return scenes.crowd_origins(n, 0.3, int(rng.integers(1 << 30)))
    o = np.zeros((n, 3))
    k, slot = np.divmod(np.arange(n), group)
    side = int(math.ceil(math.sqrt(group)))
    if terrain.kind == scenes.PLANE:
        per_row = int(math.ceil(math.sqrt(k[-1] + 1)))
        step = 5.0 if group == 1 else 50.0
        o[:, 0], o[:, 1] = (k % per_row) * step, (k // per_row) * step
    else:
        ex, ey = terrain.extent
        o[:, 0] = rng.uniform(4.0, ex - 4.0, k[-1] + 1)[k]
        o[:, 1] = rng.uniform(4.0, ey - 4.0, k[-1] + 1)[k]
    o[:, 0] += (slot % side - 0.5 * (side - 1)) * 1.5
    o[:, 1] += (slot // side - 0.5 * (side - 1)) * 1.5
    if terrain.kind == scenes.HEIGHTFIELD:
        i = np.clip((o[:, 0] / terrain.cell).astype(int), 0, terrain.nx - 1)
        j = np.clip((o[:, 1] / terrain.cell).astype(int), 0, terrain.ny - 1)
        o[:, 2] = terrain.heights[j, i]
    return o.astype(np.float32).astype(np.float64)


def _qmul(a, b):
    aw, ax, ay, az = a.unbind(-1)
    bw, bx, by, bz = b.unbind(-1)
    return torch.stack((aw * bw - ax * bx - ay * by - az * bz, aw * bx + ax * bw + ay * bz - az * by,
                        aw * by - ax * bz + ay * bw + az * bx, aw * bz + ax * by - ay * bx + az * bw), -1)


def _qrot(q, v):
    u = q[..., 1:]
    v = v.expand_as(u)
    t = torch.linalg.cross(u, v) + q[..., :1] * v
    return v + 2.0 * torch.linalg.cross(u, t)


def _states(robot, terrain, origins, gen, dev):
    """[N][B][13]: assembled robots on the ground, every other one upright."""
    n = origins.shape[0]

    def t(a):
        return torch.as_tensor(np.asarray(a), dtype=torch.float64, device=dev)

    def uniform(*shape):
        return torch.rand(*shape, generator=gen, device=dev, dtype=torch.float64)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device=dev, dtype=torch.float64)

    base = normal(n, 4)
    upright = (torch.arange(n, device=dev) % 2 == 0)[:, None]
    base = torch.where(upright, t([1.0, 0.0, 0.0, 0.0]) + 0.05 * base, base)
    x, q = [None] * robot.n_bodies, [None] * robot.n_bodies
    q[0] = base / base.norm(dim=1, keepdim=True)
    x[0] = torch.zeros(n, 3, dtype=torch.float64, device=dev)
    for j in range(robot.n_joints):
        a, b = int(robot.j_parent[j]), int(robot.j_child[j])
        lo, hi = t(robot.j_lo[j]), t(robot.j_hi[j])
        ang = torch.where(t(robot.j_mode[j]) == scenes.HINGE, lo + (hi - lo) * uniform(n, 3), lo * 0.0)
        phi = torch.where(upright, 0.3, 1.0) * (ang @ t(robot.j_axes[j]))
        half = 0.5 * phi.norm(dim=1, keepdim=True)
        dq = torch.cat((half.cos(), 0.5 * phi * torch.sinc(half / math.pi)), 1)
        q[b] = _qmul(q[a], dq)
        x[b] = x[a] + _qrot(q[a], t(robot.j_anchor[j] - robot.rest_pos[a])) - _qrot(q[b], t(robot.j_anchor[j] - robot.rest_pos[b]))
    x, q = torch.stack(x, 1), torch.stack(q, 1)
    # the lowest end sphere ends up 4 cm inside to 2 cm above the highest ground next to it
    axis = torch.zeros(robot.n_bodies, 3, dtype=torch.float64, device=dev)
    axis[torch.arange(robot.n_bodies), torch.as_tensor(robot.axis, device=dev).long()] = t(robot.half_len)
    arm = _qrot(q, axis)
    ends = torch.cat((x - arm, x + arm), 1)
    org = t(origins)
    ground = torch.zeros(n, 2 * robot.n_bodies, dtype=torch.float64, device=dev)
    if terrain.kind == scenes.HEIGHTFIELD:
        h = t(terrain.heights)
        i = ((ends[..., 0] + org[:, None, 0]) / terrain.cell).long().clamp(0, terrain.nx - 2)
        k = ((ends[..., 1] + org[:, None, 1]) / terrain.cell).long().clamp(0, terrain.ny - 2)
        ground = torch.stack((h[k, i], h[k, i + 1], h[k + 1, i], h[k + 1, i + 1])).amax(0) - org[:, None, 2]
    gap = (ends[..., 2] - t(robot.radius).repeat(2) - ground).amin(1)
    x[..., 2] += (uniform(n) * 0.06 - 0.04 - gap)[:, None]
    # one slow motion of the whole figure
    v, w = 0.5 * normal(n, 1, 3), 1.0 * normal(n, 1, 3)
    vel = v + torch.linalg.cross(w.expand_as(x), x - x[:, :1])
    return torch.cat((x, q, vel, w.expand_as(x)), 2).float().contiguous()


def prepare(case, seed):
    dev = torch.device("cuda:0")
    rng = np.random.default_rng([int(seed), 17])
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    robot = scenes.make_ant() if case["robot"] == "ant" else scenes.make_humanoid()
    terrain = scenes.make_plane() if case["terrain"] == "plane" else scenes.make_heightfield(seed=int(seed) % 1000)
    params = scenes.SimParams(height_map=int(case["height_map"]), self_collide=int(case["self_collide"]),
                              group_size=case["group"], warm_start=case["warm"], solver=int(case["newton"]))
    n = case["envs"]
    scene = scenes.Scene(robot=robot, terrain=terrain, num_envs=n, env_origins=_origins(case, terrain, rng), params=params)
    sim = sim355.Sim(scene, device=dev)
    snapshot = _states(robot, terrain, scene.env_origins, gen, dev)
    sim.set_state(snapshot)
    if case["task"]:
        sim.set_task(scenes.TaskParams(seed=int(seed)))
    actions = [2.0 * torch.rand(n, sim.act_dim, generator=gen, device=dev) - 1.0 for _ in range(RING)]
    return {"sim": sim, "mode": case["mode"], "snapshot": snapshot, "actions": actions, "pass": 0, "seed": int(seed),
            "step": (DT, case["substeps"], case["iterations"]), "state": case["state"],
            "done": torch.zeros(n, dtype=torch.uint8, device=dev)}


def run(s):
    sim, k = s["sim"], s["pass"]
    s["pass"] = k + 1
    if s["mode"] == "plan":
        sim.set_state(s["snapshot"])
        for i in range(PLAN_STEPS):
            out = sim.step_obs(s["actions"][i], *s["step"])
        return (*out, sim.get_state())
    if s["mode"] == "episodes":
        sim.reset(s["seed"] + k, mask=s["done"])
    elif s["mode"] == "crowd" and k % REGROUP_EVERY == 0:
        sim.regroup(REGROUP_CELL, REGROUP_REACH)
    out = sim.step_obs(s["actions"][k % RING], *s["step"])
    s["done"] = out[2]
    return (*out, sim.get_state()) if s["state"] else out


# ---- what a pass cannot do without

def work(case):
    """Body state in and out, actions in, observation, reward and done flag out (and the kept
    impulses, and the state read back); the arithmetic of the step's algorithm with the contacts a
    robot of that kind has on average."""
    robot = scenes.make_ant() if case["robot"] == "ant" else scenes.make_humanoid()
    hf = case["terrain"] == "heightfield"
    n, bodies, joints, dofs = case["envs"], robot.n_bodies, robot.n_joints, robot.n_dofs
    slots = robot.n_slots(hf)
    active = 1.4 if case["robot"] == "ant" else (3.3 if hf else 2.3)
    steps = PLAN_STEPS if case["mode"] == "plan" else 1
    words = steps * (2 * 13 * bodies + dofs + robot.obs_dim + (165 if case["height_map"] else 0) + 1.25)
    if case["state"]:
        words += 2 * 13 * bodies
    if case["mode"] == "plan":
        words += 2 * 13 * bodies
    if case["warm"]:
        words += 2 * (6 * joints + 3 * slots)
    blocks = 2.0 * joints + active
    # set-up per substep: joint rows 420, contact rows 150, forces and integration 240 a body, reach test 30 a slot,
    # fine search 2000 for every slot near the ground
    setup = joints * 420.0 + active * 150.0 + bodies * 240.0 + slots * 30.0 + (active * 2000.0 if hf else 0.0)
    if case["newton"]:
        apply_ = joints * 162.0 + active * 80.0 + 12.0 * blocks
        krylov = 8
        solve = case["iterations"] * ((krylov + 2) * apply_ + (6 * joints + 3 * active) * (14.0 * krylov + 20.0)) + apply_
    else:
        solve = case["iterations"] * (joints * 156.0 + active * 95.0 + 6.0 * blocks + 6.0 * bodies)
    if case["self_collide"]:
        setup += len(robot.collide_pairs) * 12.0 + (case["group"] - 1) * 12.0
    return {"bytes": n * words * 4.0, "flops": steps * n * case["substeps"] * (setup + solve)}


def tolerance(case):
    """Measured against the same steps in double precision (three seeds, up to 1024 environments, first and second
    pass): observations and states within 5e-6 (3.4e-5 with the Newton solver, whose cut-off iterates are more
    sensitive), rewards within 1.4e-4, which is one joint of one robot counted on the other side of its limit.
    A foot flag that falls on the other side of its threshold is 1 in an observation of root mean square 7 to 13,
    an Euler angle that does so at +-pi is 2 pi."""
    return {"rel": 1e-3 if case["newton"] else 6e-4, "max": 0.9, "differ": 1e-3}

"""The work that programs give this library, as cases that can be timed and compared.

A case is a dict of plain values; `prepare` makes from it what a program holds before the call (an Env or a Server with
its buffers), `run` makes one pass through the public entry points, and `work` says how many bytes a pass cannot do
without.  The kinds of pass:

  step     one Env.step of every env into the next slot of a rollout buffer (a policy in the loop: the common use)
  rollout  one Env.rollout of T steps with the actions given up front (random-policy collection, replay)
  render   one Env.render of the current state (evaluation frames)
  serve    one step request of every client of a Server, submitted together and collected together

Tasks: "maze" (seeded maze, goal sprite), "keydoor" (seeded maze with door, key, goal and decor), "rooms" (an ASCII map
with doors and keys), "mixed" (per-env shapes).  Episode clocks are staggered, so that episodes end and reset throughout,
as they do in a long run.
"""
import math

import numpy as np
import torch

from paper_2605_19926_amd import jx

DTYPES = {"u8": (0, torch.uint8, 1), "bf16": (1, torch.bfloat16, 2), "f32": (2, torch.float32, 4)}
LAYOUTS = {"nhwc": 0, "nchw": 1}
PI16 = math.pi / 16

# Five rooms joined by locked and unlocked doors, three keys, spawn and goal candidates, coloured walls.
ROOMS = [
    "################",
    "#S....1..#....G#",
    "#.....1..#.....#",
    "#..r.....R..y..#",
    "#.....1..#.....#",
    '##"#######\\#####',
    "#......#.......#",
    "#.2222.#..S....#",
    "#.2..2.B.......#",
    "#.2222.#...b...#",
    "#......#.......#",
    "####Y#######.###",
    "#..............#",
    "#.S.....33...G.#",
    "#..............#",
    "################",
]

BASE = {"kind": "step", "task": "maze", "n": 256, "side": 16, "h": 64, "w": 64, "actions": 6, "cap": 512,
        "dtype": "u8", "layout": "nhwc", "prev": False, "shade": 0, "T": 1, "mode": "", "form": 0, "waves": 0, "groups": 1}
STEP_SLOTS = 16  # rollout-buffer slots of the step kind


def _case(name=None, **kw):
    c = dict(BASE, **kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # a first program, an evaluation loop: few small envs, one call at a time, so latency is what counts
        _case("step-16", n=16, side=8, actions=4, cap=256),
        # a learner with a few hundred envs that takes its network's input format and the previous action
        _case("step-256-f32", n=256, task="rooms", dtype="f32", layout="nchw", prev=True),
        # the headline batch with a policy in the loop, default mapping
        _case("step-4096", n=4096),
        # large mazes with key, door and decor at the Atari frame size; 8 of the 8192 envs reset in each step
        _case("step-keydoor-8192", n=8192, task="keydoor", side=32, h=84, w=84, cap=1024),
        # a learner in bfloat16 on an ASCII map
        _case("step-rooms-2048-bf16", n=2048, task="rooms", dtype="bf16", prev=True),
        # random-policy collection: the headline rollout, 128 steps in one launch
        _case("rollout-4096", kind="rollout", n=4096, T=128, mode="fused", waves=8),
        # the same into a learner's float32 buffer
        _case("rollout-rooms-2048-f32", kind="rollout", task="rooms", n=2048, T=128, mode="fused", waves=4, dtype="f32",
              layout="nchw", prev=True),
        # uneven shapes in one persistent launch: the largest batch
        _case("rollout-mixed-16384", kind="rollout", task="mixed", n=16384, side=64, h=128, w=128, cap=1024, T=32,
              mode="fused", form=1, waves=4, groups=2),
        # captured per-step launches, the default rollout mode
        _case("rollout-graph-1024", kind="rollout", n=1024, side=25, T=64, mode="graph", shade=8),
        # evaluation frames at the largest size, long rays between pillars
        _case("render-500-128px", kind="render", n=500, side=64, h=128, w=128, cap=256),
        # remote clients: results come back to host memory
        _case("serve-host-24", kind="serve", n=24, most=48, device=False),
        # clients whose consumer is on the same GPU: results stay in device rings
        _case("serve-rings-96", kind="serve", n=96, most=512, device=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 5 + ["rollout"] * 3 + ["render", "serve"])
    if kind == "serve":
        return _case(kind="serve", n=rng.randint(3, 90), most=_log_int(rng, 4, 500), device=rng.random() < 0.5)
    task = rng.choice(["maze", "maze", "keydoor", "rooms"])
    dtype = rng.choice(["u8", "u8", "u8", "bf16", "f32"])
    c = _case(kind=kind, task=task, side=16 if task == "rooms" else _log_int(rng, 8, 64), actions=rng.choice([4, 6, 6]),
              cap=rng.randint(200, 1024), dtype=dtype, layout=rng.choice(["nhwc", "nhwc", "nchw"]),
              shade=rng.choice([0, 0, 0, 8]))
    if rng.random() < 0.5:
        c["h"] = c["w"] = rng.choice([32, 64, 64, 84, 128])
    else:
        c["h"], c["w"] = 2 * rng.randint(16, 64), 4 * rng.randint(8, 32)
    c["prev"] = kind != "render" and dtype != "u8"
    if kind == "rollout":
        c["T"] = _log_int(rng, 5, 128)
        c["mode"] = rng.choice(["fused", "fused", "graph"])
        c["waves"] = rng.choice([4, 8])
        if c["mode"] == "fused" and dtype == "u8" and rng.random() < 0.3:
            c["form"], c["waves"], c["groups"] = 1, 4, 2
    n = _log_int(rng, 12, 8192)
    frame = c["h"] * c["w"] * 3 * DTYPES[dtype][2]
    n = min(n, int(180e6 // frame) if kind != "rollout" else int(5e9 // (frame * c["T"])), int(8e6 // c["side"] ** 2))
    c["n"] = max(1, n)
    return c


# ---- what a program holds before the call ------------------------------------
def _cfg(task, side, h, w, actions=6, cap=512, dtype="u8", layout="nhwc", shade=0, loop=0.1):
    keydoor = task == "keydoor"
    return {"side": side, "n_colors": 8, "loop_frac": 0.0 if keydoor or task == "rooms" else loop, "key_door": int(keydoor),
            "goal_sprite": 1, "max_decor": 2 if keydoor else 0, "obs_h": h, "obs_w": w, "fov_deg": 60.0,
            "n_actions": actions, "episode_cap": cap, "move": 0.1, "turn": PI16, "pickup_radius": 0.3, "r_goal": 1.0,
            "r_key": 0.5, "shade_levels": shade, "shade_dist": 8.0,
            "ascii_map": "\n".join(ROOMS) if task == "rooms" else None, "obs_layout": LAYOUTS[layout],
            "obs_dtype": DTYPES[dtype][0]}


def _cfg_of(case):
    return _cfg(case["task"], case["side"], case["h"], case["w"], case["actions"], case["cap"], case["dtype"], case["layout"],
                case["shade"], 1.0 if case["kind"] == "render" else 0.1)


def _mixed(case):
    """Configurations and each env's index: map side, frame size and task vary from env to env."""
    sides = [s for s in (8, 16, 32, 64) if s <= case["side"]]
    sizes = [s for s in (32, 64, 128) if s <= case["h"]]
    cfgs = [_cfg(t, s, p, p, case["actions"], case["cap"] if t == "keydoor" else case["cap"] // 2)
            for s in sides for p in sizes for t in ("maze", "keydoor")]
    return cfgs, np.random.default_rng(case["n"]).integers(0, len(cfgs), case["n"]).astype(np.int32)


def _seeds(seed, n, first=0):
    return (np.uint64(seed % 2**31) << np.uint64(32)) + np.arange(first, first + n, dtype=np.uint64)


def _actions(case, seed, steps):
    return np.random.default_rng([seed, 1]).integers(0, case["actions"], (steps, case["n"]), dtype=np.uint8)


def _clients(case):
    """(envs, side, frame size) of each client: log-uniform batch sizes, any side from 8 to 64, 64 or 84 pixels."""
    k = np.arange(case["n"])
    u = (k * 0.6180339887) % 1.0
    envs = np.clip(np.floor(np.exp(u * math.log(case["most"] + 1))), 1, case["most"]).astype(int)
    return list(zip(envs.tolist(), (8 + k * 37 % 57).tolist(), np.where(k % 2, 84, 64).tolist()))


def _prepare_serve(case, seed):
    srv = jx.Server(hbm_budget=512 << 20, n_streams=4)
    rng = np.random.default_rng([seed, 1])
    sizes = _clients(case)
    envs = sum(n for n, _, _ in sizes)
    total = sum(n * p * p * 3 for n, _, p in sizes)
    if case["device"]:
        slots = 2
        obs = torch.zeros(slots * total, dtype=torch.uint8, device="cuda")
        rew = torch.zeros(slots * envs, device="cuda")
        done = torch.zeros(slots * envs, dtype=torch.uint8, device="cuda")
    else:
        slots = 1
        obs, rew, done = np.zeros(total, np.uint8), np.zeros(envs, np.float32), np.zeros(envs, np.uint8)
    clients, o, e = [], 0, 0
    for j, (n, side, p) in enumerate(sizes):
        cfg = _cfg("keydoor" if j % 3 == 0 else "maze", side, p, p)
        fb = n * p * p * 3
        bufs = (obs[slots * o:slots * (o + fb)], rew[slots * e:slots * (e + n)], done[slots * e:slots * (e + n)])
        if case["device"]:
            cid, _ = srv.open_dev(_seeds(seed, n, e), cfg, *bufs, slots=slots)
        else:
            cid, _ = srv.open(_seeds(seed, n, e), cfg)
        clients.append((cid, rng.integers(0, 6, (32, n), dtype=np.uint8), None if case["device"] else bufs))
        o, e = o + fb, e + n
    while srv.stats()["clients_pending"]:
        pass
    return {"case": case, "srv": srv, "clients": clients, "out": (obs, rew, done), "k": 0}


def prepare(case, seed):
    if case["kind"] == "serve":
        return _prepare_serve(case, seed)
    n, kind = case["n"], case["kind"]
    cfgs, index = _mixed(case) if case["task"] == "mixed" else ([_cfg_of(case)], None)
    env = jx.Env(_seeds(seed, n), cfgs, index)
    env.reset()
    cap = np.array([c["episode_cap"] for c in cfgs])
    env.set_state({"t": (np.arange(n) % (cap[0] if index is None else cap[index])).astype(np.uint32)})
    if case["waves"]:
        env.set_launch(form=case["form"], waves_per_group=case["waves"], groups_per_cu=case["groups"])
    _, dtype, size = DTYPES[case["dtype"]]
    slots = {"step": STEP_SLOTS, "rollout": case["T"], "render": 1}[kind]
    state = {"case": case, "env": env, "k": 0,
             "obs": torch.empty((slots, env.obs_bytes // size), dtype=dtype, device=env.dev)}
    if kind != "render":
        steps = 64 if kind == "step" else case["T"]
        state["actions"] = torch.from_numpy(_actions(case, seed, steps)).to(env.dev)
        state["rew"] = torch.empty((slots, n), device=env.dev)
        state["done"] = torch.empty((slots, n), dtype=torch.uint8, device=env.dev)
        state["prev"] = torch.empty((slots, n), dtype=torch.uint8, device=env.dev) if case["prev"] else None
    return state


# ---- one pass ------------------------------------------------------------------
def run(state):
    case, k = state["case"], state["k"]
    state["k"] = k + 1
    if case["kind"] == "step":
        s = k % STEP_SLOTS
        obs, rew, done = state["obs"][s], state["rew"][s], state["done"][s]
        prev = state["prev"][s] if case["prev"] else None
        state["env"].step(state["actions"][k % 64], obs, rew, done, prev)
        return obs, rew, done, prev
    if case["kind"] == "rollout":
        env = state["env"]
        env.rollout(state["actions"], state["obs"], state["rew"], state["done"], case["T"], obs_stride=env.obs_bytes,
                    graph=case["mode"] == "graph", fused=case["mode"] == "fused", prev=state["prev"])
        return state["obs"], state["rew"], state["done"], state["prev"]
    if case["kind"] == "render":
        state["env"].render(state["obs"][0])
        return state["obs"][0]
    srv = state["srv"]
    tickets = [srv.submit(cid, acts[k % 32]) for cid, acts, _ in state["clients"]]
    for (cid, _, out), ticket in zip(state["clients"], tickets):
        srv.wait(cid, ticket, out=out)
    return state["out"]


def _state_bytes(side):
    # map; pose, clocks, tiles, decor, flags and seed read; the same without map and seed written
    return side * side + 58 + 43


def work(case):
    """Frames, actions, rewards and dones of the pass once, each env's state and map once."""
    if case["kind"] == "serve":
        return {"bytes": sum(n * (p * p * 3 + 6 + _state_bytes(side)) for n, side, p in _clients(case)), "flops": 0}
    T = case["T"]
    io = 0 if case["kind"] == "render" else 6 + int(case["prev"])
    if case["task"] == "mixed":
        cfgs, index = _mixed(case)
        each = [T * (c["obs_h"] * c["obs_w"] * 3 + io) + _state_bytes(c["side"]) for c in cfgs]
        return {"bytes": int(np.array(each)[index].sum()), "flops": 0}
    frame = case["h"] * case["w"] * 3 * DTYPES[case["dtype"]][2]
    return {"bytes": case["n"] * (T * (frame + io) + _state_bytes(case["side"])), "flops": 0}


# ---- the same in 64 bits, for the ASCII map -----------------------------------
PALETTE = [(180, 40, 40), (40, 160, 40), (40, 60, 180), (190, 170, 40), (150, 40, 170), (40, 160, 170), (200, 110, 30),
           (150, 150, 150)]
NUMBERED = PALETTE + [(230, 230, 230)]                                        # walls '1' to '9'
DOORS = {"R": (120, 0, 0), "B": (0, 30, 130), "Y": (140, 120, 0), '"': (70, 110, 230), "\\": (230, 200, 60)}
SPRITES = [(255, 40, 40), (40, 110, 255), (255, 200, 40), (255, 230, 0)]      # red, blue, yellow key; goal
CEILING, GROUND = (50, 50, 60), (90, 80, 70)
TWO_PI = float(np.float32(2 * math.pi))


class _Rooms:
    """Episodes on ROOMS in float64: the rules of include/jx.h for ASCII maps, over all envs at once."""

    def __init__(self, case, seed):
        self.case, n = case, case["n"]
        self.dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
        N = self.N = len(ROOMS)
        tiles = "".join(ROOMS)
        self.spawns = [i for i, c in enumerate(tiles) if c == "S"]
        self.goals = [i for i, c in enumerate(tiles) if c == "G"]
        self.keys = [tiles.index(c) for c in "rby"]
        doors = [i for i, c in enumerate(tiles) if c in DOORS]
        wall = [c == "#" or c.isdigit() for c in tiles]
        colour = [NUMBERED[int(c) - 1] if c.isdigit() else DOORS.get(c, PALETTE[i % 8]) for i, c in enumerate(tiles)]
        self.wall = torch.tensor(wall, device=self.dev)
        self.colour = torch.tensor(colour, dtype=torch.int64, device=self.dev)
        self.bit = torch.tensor([1 << doors.index(i) if i in doors else 0 for i in range(N * N)], device=self.dev)
        self.bumps = torch.tensor([c in '"\\' for c in tiles], device=self.dev)
        self.opened_by = [sum(1 << doors.index(i) for i in doors if tiles[i] == c) for c in "RBY"]
        self.seeds = _seeds(seed, n)
        self.ep = np.zeros(n, np.uint64)
        self.x, self.y, self.th = (torch.zeros(n, dtype=torch.float64, device=self.dev) for _ in range(3))
        self.goal, self.open, self.taken = (torch.zeros(n, dtype=torch.int64, device=self.dev) for _ in range(3))
        self.reset(np.ones(n, bool))
        self.t = torch.arange(n, device=self.dev) % case["cap"]

    def reset(self, which):
        """The first draws of each episode's SplitMix64 stream: spawn, heading, goal."""
        def follow(s):
            s = s + np.uint64(0x9E3779B97F4A7C15)
            z = (s ^ (s >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
            z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
            return s, z ^ (z >> np.uint64(31))

        def pick(z, ids):
            return np.array(ids)[((z >> np.uint64(32)) * np.uint64(len(ids)) >> np.uint64(32)).astype(int)]

        s = self.seeds[which] ^ follow(self.ep[which] + np.uint64(1))[1]
        s, z = follow(s)
        spawn = pick(z, self.spawns)
        s, z = follow(s)
        heading = (z >> np.uint64(40)).astype(np.float64) * (TWO_PI * 2.0**-24)
        s, z = follow(s)
        at = torch.from_numpy(np.flatnonzero(which)).to(self.dev)
        self.x[at] = torch.from_numpy(spawn % self.N + 0.5).to(self.dev)
        self.y[at] = torch.from_numpy(spawn // self.N + 0.5).to(self.dev)
        self.th[at] = torch.from_numpy(heading.astype(np.float32).astype(np.float64)).to(self.dev)
        self.goal[at] = torch.from_numpy(pick(z, self.goals)).to(self.dev)
        self.open[at] = self.taken[at] = 0

    def blocked(self, ids, doors):
        return self.wall[ids] | ((self.bit[ids] != 0) & (self.bit[ids] & doors == 0))

    def step(self, a):
        c, N = self.case, self.N
        turn, move = float(np.float32(PI16)), float(np.float32(0.1))
        fwd, side = (a == 0).double() - (a == 1).double(), torch.zeros_like(self.x)
        if c["actions"] == 6:
            side, a = (a == 3).double() - (a == 2).double(), a - 2
        cs, sn = self.th.cos(), self.th.sin()
        self.th = self.th + turn * ((a == 3).double() - (a == 2).double())
        self.th = torch.where(self.th < 0, self.th + TWO_PI, torch.where(self.th >= TWO_PI, self.th - TWO_PI, self.th))
        for axis, d in (("x", move * (fwd * cs - side * sn)), ("y", move * (fwd * sn + side * cs))):
            to = getattr(self, axis) + d
            ids = (self.y.floor() * N + to.floor() if axis == "x" else to.floor() * N + self.x.floor()).long()
            stop = self.blocked(ids, self.open)
            setattr(self, axis, torch.where(stop, getattr(self, axis), to))
            self.open |= torch.where(stop & self.bumps[ids], self.bit[ids], 0)
        reward = torch.zeros_like(self.x)
        for k, key in enumerate(self.keys):
            near = (self.x - (key % N + 0.5)) ** 2 + (self.y - (key // N + 0.5)) ** 2 < float(np.float32(0.3)) ** 2
            near &= self.taken >> k & 1 == 0
            self.taken |= near.long() << k
            self.open |= torch.where(near, self.opened_by[k], 0)
            reward += 0.5 * near
        there = (self.y.floor() * N + self.x.floor()).long() == self.goal
        reward += there
        self.t += 1
        done = there | (self.t >= c["cap"])
        ended = done.cpu().numpy()
        if ended.any():
            self.ep[ended] += np.uint64(1)
            self.reset(ended)
            self.t = torch.where(done, 0, self.t)
        return reward

    def frames(self):
        c, N = self.case, self.N
        H, W = c["h"], c["w"]
        tan = math.tan(math.radians(60.0) / 2)
        cs, sn = self.th.cos()[:, None], self.th.sin()[:, None]
        off = (2 * torch.arange(W, device=self.dev, dtype=torch.float64) + 1 - W) / W * tan
        rx, ry = cs - off * sn, sn + off * cs
        x, y = self.x[:, None].expand_as(rx), self.y[:, None].expand_as(rx)
        fx, fy = x.floor(), y.floor()
        ids = (fy * N + fx).long()
        dx, dy = (1 / rx).abs(), (1 / ry).abs()
        tx = torch.where(rx > 0, fx + 1 - x, x - fx) * dx
        ty = torch.where(ry > 0, fy + 1 - y, y - fy) * dy
        depth, face, going = torch.zeros_like(rx), torch.zeros_like(ids), torch.ones_like(ids, dtype=torch.bool)
        while going.any():
            over_x = tx < ty
            depth = torch.where(going, torch.where(over_x, tx, ty), depth)
            face = torch.where(going, (~over_x).long(), face)
            ids = torch.where(going, ids + torch.where(over_x, rx.sign(), N * ry.sign()).long(), ids)
            tx, ty = torch.where(over_x, tx + dx, tx), torch.where(over_x, ty, ty + dy)
            going = going & ~self.blocked(ids, self.open[:, None])
        wall = self.colour[ids] >> face[..., None]
        if c["shade"]:
            level = (depth * c["shade"] / 8.0).floor().clamp(max=c["shade"] - 1).long()
            wall = wall * (c["shade"] - level)[..., None] // c["shade"]
        rows = (H / (2 * depth) - 0.5).ceil().clamp(0, H // 2)
        best = torch.full_like(rx, math.inf)
        tall, sprite = torch.zeros_like(rx), torch.zeros_like(wall)
        col = torch.arange(W, device=self.dev) + 0.5
        for k in range(4):
            at = self.goal if k == 3 else torch.full_like(self.goal, self.keys[k])
            ddx, ddy = at[:, None] % N + 0.5 - self.x[:, None], at[:, None] // N + 0.5 - self.y[:, None]
            z, u = ddx * cs + ddy * sn, ddy * cs - ddx * sn
            seen = (z > 0.05) & ((col - W / 2 * (1 + u / (tan * z))).abs() < W / 8 / (tan * z)) & (z < depth) & (z <= best)
            if k < 3:
                seen &= (self.taken[:, None] >> k & 1) == 0
            best = torch.where(seen, z, best)
            tall = torch.where(seen, (H / 4 / z - 0.5).ceil().clamp(0, H // 2), tall)
            sprite = torch.where(seen[..., None], torch.tensor(SPRITES[k], device=self.dev), sprite)
        out = torch.empty((c["n"], H, W, 3), dtype=torch.int64, device=self.dev)
        for r in range(H):
            i = H // 2 - 1 - r if r < H // 2 else r - H // 2
            back = torch.tensor(CEILING if r < H // 2 else GROUND, device=self.dev)
            out[:, r] = torch.where((i < tall)[..., None], sprite, torch.where((i < rows)[..., None], wall, back))
        return out


def exact(case, seed):
    """Normalised frames and rewards in float64 on the ASCII map.  Elsewhere the episodes come from generated mazes and
    breadth-first searches, which take minutes this way, and byte frames are whole numbers: those have no value here."""
    if case["task"] != "rooms" or case["kind"] == "render":
        return None
    T, n = case["T"], case["n"]
    if n * T * case["w"] > 40e6:
        return None
    rooms = _Rooms(case, seed)
    a = torch.from_numpy(_actions(case, seed, 64 if case["kind"] == "step" else T)).to(rooms.dev).long()
    floats = case["dtype"] != "u8"
    frames = torch.empty((T, n * case["h"] * case["w"] * 3), dtype=torch.float64, device=rooms.dev) if floats else None
    rewards = torch.empty((T, n), dtype=torch.float64, device=rooms.dev)
    for t in range(T):
        rewards[t] = rooms.step(a[t])
        if floats:
            f = rooms.frames()
            frames[t] = (f.permute(0, 3, 1, 2) if case["layout"] == "nchw" else f).reshape(-1).double() / 255
    if case["kind"] == "step":
        return (frames[0] if floats else None), rewards[0], None, None
    return frames, rewards, None, None

"""GPU: episode resets against the oracle where the row masks and searches can go
wrong: map sides around 8, 16, 32 and 64 (bit-string offsets, mask width), maps
whose structure is not a maze's (loaded through the state image), and ASCII maps
with and without candidates.  Every field of a reset is an integer or an exact
function of one, so the comparison is exact."""
import numpy as np
import pytest

import tests.gpu_util as U
import oracle as orc
import workloads as W

pytestmark = pytest.mark.gpu

KINDS = {
    "maze": dict(loop_frac=0.1, goal_sprite=1),
    "tree": dict(loop_frac=0.0, key_door=1, max_decor=2),
    "loops": dict(loop_frac=0.5, key_door=1, max_decor=2),
}


def _interior(kind, side, rng):
    """A map that no generator makes: border walls around random tiles, an open
    hall, one winding corridor, or a single floor tile."""
    g = np.ones((side, side), np.uint8)
    if kind == "random":
        g[1:-1, 1:-1] = rng.random((side - 2, side - 2)) < 0.35
    elif kind == "rooms":  # on a maze's lattice, but with dead-end separators and cut-off parts
        g[1:-1, 1:-1] = rng.random((side - 2, side - 2)) < 0.25
        g[::2, ::2] = 1
    elif kind == "hall":
        g[1:-1, 1:-1] = 0
    elif kind == "corridor":  # a snake: the longest shortest paths
        g[1:-1:2, 1:-1] = 0
        for k, y in enumerate(range(2, side - 2, 2)):
            g[y, side - 2 if k % 2 == 0 else 1] = 0
    else:
        g[side // 2, side // 2] = 0
    if (g == 0).sum() == 0:
        g[1, 1] = 0
    return g


def _check_next_episode(cfg, n, maps=None):
    """Steps every env over its time limit and compares the new episode."""
    import torch
    from paper_2605_19926_amd import jx
    seeds = W.seeds(31, n)
    env = jx.Env(seeds, cfg)
    env.reset()
    N, lay = cfg["side"], env.state_layout()
    image = env.get_state_bytes()
    at = lay["maps"][0] + jx.unpack_state(image, lay)["map_offset"].astype(np.int64)
    grids = [orc.layout(cfg, int(s)) for s in seeds]
    if maps is not None:
        grids = maps
        for i in range(n):
            image[at[i]:at[i] + N * N] = maps[i].reshape(-1)
    env.set_state({"t": np.full(n, cfg["episode_cap"] - 1, np.uint32), "episode": np.arange(n, dtype=np.uint32)}, image)
    obs = env.new_obs()
    # an out-of-range action: nothing moves, the clock runs out
    env.step(torch.full((n,), 250, dtype=torch.uint8, device=env.dev), obs)
    S = env.get_state()
    oc = orc.make_cfg(cfg)
    for i in range(n):
        want = orc.reset(grids[i], oc, int(seeds[i]), i + 1).as_dict()
        errs = U.compare_reset_state(U.gpu_state_dict(S, i), want)
        assert not errs, f"side {N} env {i}: {errs}"
    assert int(env.done.sum()) == n
    env.close()


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("side", [5, 6, 8, 15, 16, 17, 31, 32, 33, 47, 63, 64])
def test_maze_resets(side, kind):
    _check_next_episode(W.env_cfg(side=side, obs_h=32, obs_w=32, episode_cap=64, **KINDS[kind]), 12)


@pytest.mark.parametrize("kind", ["random", "rooms", "hall", "corridor", "single"])
@pytest.mark.parametrize("side", [5, 16, 31, 32, 33, 34, 47, 63, 64])
def test_resets_on_loaded_maps(side, kind):
    rng = np.random.default_rng(side)
    cfg = W.env_cfg(side=side, obs_h=32, obs_w=32, episode_cap=64, key_door=1, max_decor=2)
    _check_next_episode(cfg, 16, [_interior(kind, side, rng) for _ in range(16)])


@pytest.mark.parametrize("text,side", [(W.MAP16, 16), (W.MAP16, 33), (W.MAP16.replace("G", "."), 16),
                                       (W.MAP16.replace("G", ".").replace("S", " "), 64), (W.ROOM64, 64)])
def test_ascii_resets(text, side):
    _check_next_episode(W.env_cfg(side=side, obs_h=32, obs_w=32, episode_cap=64, ascii_map=text, goal_sprite=1), 12)

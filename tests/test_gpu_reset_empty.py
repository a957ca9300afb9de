"""GPU: the reset of an env whose loaded map has no floor tile.  No draw can place
the agent then: it stands off the map, at (-0.5, -0.5), without a goal, door, key
or decor, and every later action is refused by the map's edge."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side,kw", [(8, dict(key_door=1, max_decor=2)), (20, dict(key_door=1, max_decor=2)),
                                     (40, dict(key_door=1)), (64, {}), (16, dict(ascii_map=W.MAP16))])
def test_reset_on_a_map_without_floor(side, kw):
    import torch
    from paper_2605_19926_amd import jx
    n = 6
    cfg = W.env_cfg(side=side, obs_h=32, obs_w=32, episode_cap=64, goal_sprite=1, **kw)
    env = jx.Env(W.seeds(37, n), cfg)
    env.reset()
    lay, image = env.state_layout(), env.get_state_bytes()
    at = lay["maps"][0] + jx.unpack_state(image, lay)["map_offset"].astype(np.int64)
    for o in at:
        image[o:o + side * side] = 1
    env.set_state({"t": np.full(n, cfg["episode_cap"] - 1, np.uint32)}, image)
    obs = env.new_obs()
    env.step(torch.full((n,), 250, dtype=torch.uint8, device=env.dev), obs)   # out of range: the clock runs out
    for _ in range(2):
        S = env.get_state()
        assert (S["x"] == -0.5).all() and (S["y"] == -0.5).all(), (S["x"], S["y"])
        for name in ("goal", "door", "key"):
            assert (S[name] == -1).all(), name
        assert (S["n_decor"] == 0).all() and (S["episode"] == 1).all()
        env.step(torch.zeros(n, dtype=torch.uint8, device=env.dev), obs)
    env.close()

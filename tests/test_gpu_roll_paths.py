"""GPU: the kernels that fused rollouts and steps choose among by batch, frame and
waves per env, at the edges of their ranges: workgroup slots without an env, rows
of more than one wave's 64 columns (two casting waves, resets in both), column
groups that leave lanes idle, every frame format.  Each is compared bit for bit
with one-wave single steps, which the oracle tests cover."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

ROOMS = dict(side=16, ascii_map=W.MAP16, goal_sprite=1)
TREE = dict(side=20, key_door=1, goal_sprite=1, max_decor=2)
MAZE64 = dict(side=64, loop_frac=0.3, goal_sprite=1)


def _run(cfg, n, T, launch, fused):
    """Frames, rewards, dones, previous actions and state after T steps."""
    import torch
    from paper_2605_19926_amd import jx
    env = jx.Env(W.seeds(41, n), cfg)
    env.reset()
    env.set_state({"t": (np.arange(n) % cfg["episode_cap"]).astype(np.uint32)})
    if launch:
        env.set_launch(**launch)
    a = torch.from_numpy(W.actions(41, T, n, cfg["n_actions"] + 1)).to(env.dev)  # out-of-range ones among them
    obs = torch.zeros(T * env.obs_bytes, dtype=torch.uint8, device=env.dev)
    rew, done, prev = (torch.zeros((T, n), dtype=d, device=env.dev) for d in (torch.float32, torch.uint8, torch.uint8))
    if fused:
        env.rollout(a, obs, rew, done, T, obs_stride=env.obs_bytes, graph=False, fused=True, prev=prev)
    else:
        for t in range(T):
            env.step(a[t], obs[t * env.obs_bytes:(t + 1) * env.obs_bytes], rew[t], done[t], prev[t])
    torch.cuda.synchronize()
    state = env.get_state_bytes()
    env.close()
    return obs, rew, done, prev, state


def _same(x, y):
    import torch
    return all(bool(np.array_equal(p, q)) if isinstance(p, np.ndarray) else torch.equal(p, q) for p, q in zip(x, y))


ONE = dict(waves_per_group=1, waves_per_env=1)
SHAPES = [(TREE, 64, 64), (TREE, 84, 84), (TREE, 30, 44), (ROOMS, 128, 128), (ROOMS, 66, 68), (MAZE64, 128, 100),
          (MAZE64, 2, 4)]


@pytest.mark.parametrize("wpe", [2, 4])
@pytest.mark.parametrize("base,h,w", SHAPES)
def test_several_waves_per_env(base, h, w, wpe):
    cfg = W.env_cfg(obs_h=h, obs_w=w, episode_cap=9, **base)
    for n in (1, 7):
        want = _run(cfg, n, 14, ONE, False)
        for fused in (False, True):
            got = _run(cfg, n, 14, dict(waves_per_group=4, waves_per_env=wpe), fused)
            assert _same(got, want), f"n {n} fused {fused}"


@pytest.mark.parametrize("layout,dtype", [(0, 1), (0, 2), (1, 0), (1, 1), (1, 2)])
def test_several_waves_per_env_formats(layout, dtype):
    cfg = W.env_cfg(obs_h=34, obs_w=72, episode_cap=9, obs_layout=layout, obs_dtype=dtype, **ROOMS)
    want = _run(cfg, 5, 12, ONE, False)
    for wpe in (2, 4):
        for fused in (False, True):
            assert _same(_run(cfg, 5, 12, dict(waves_per_group=4, waves_per_env=wpe), fused), want), (wpe, fused)


@pytest.mark.parametrize("n,wpb", [(2048, 8), (2049, 8), (3072, 4), (3073, 4), (3073, 1), (4100, 2)])
def test_dense_rollouts_of_small_frames(n, wpb):
    """Around the batch from which small frames take the kernel of 4 waves per SIMD."""
    cfg = W.env_cfg(obs_h=32, obs_w=32, episode_cap=5, **TREE)
    want = _run(cfg, n, 7, ONE, False)
    assert _same(_run(cfg, n, 7, dict(waves_per_group=wpb), True), want)


@pytest.mark.parametrize("n,h,w,fmt", [(512, 64, 64, (0, 0)), (513, 64, 64, (0, 0)), (1536, 64, 64, (0, 0)),
                                       (1537, 64, 64, (0, 0)), (768, 72, 80, (0, 0)), (1025, 84, 84, (0, 0)),
                                       (769, 64, 64, (1, 1)), (30, 128, 128, (1, 2))])
def test_mapping_left_to_the_library(n, h, w, fmt):
    """Around the batches and frames from which an env gets more than one wave."""
    cfg = W.env_cfg(obs_h=h, obs_w=w, episode_cap=6, obs_layout=fmt[0], obs_dtype=fmt[1], **TREE)
    want = _run(cfg, n, 8, dict(form=2, waves_per_group=1, groups_per_cu=2) if fmt == (0, 0) else
                dict(waves_per_group=4, waves_per_env=2), False)
    for launch in (None, dict(waves_per_group=8)):
        for fused in (False, True):
            assert _same(_run(cfg, n, 8, launch, fused), want), (launch, fused)


@pytest.mark.parametrize("n,T", [(40, 1), (40, 2), (8193, 3), (8193, 4)])
def test_rollout_left_to_the_library(n, T):
    """Around the steps and envs from which a rollout is one launch: two calls in a
    row against the same steps one by one, with the frames of every step in one slot."""
    import torch
    from paper_2605_19926_amd import jx
    cfg = W.env_cfg(obs_h=64, obs_w=44, episode_cap=3, side=9)
    got = []
    for graph in (True, False):
        env = jx.Env(W.seeds(43, n), cfg)
        env.reset()
        a = torch.from_numpy(W.actions(43, T, n, 6)).to(env.dev)
        obs = env.new_obs()
        rew, done = torch.zeros((T, n), device=env.dev), torch.zeros((T, n), dtype=torch.uint8, device=env.dev)
        for _ in range(2):
            env.rollout(a, obs, rew, done, T, obs_stride=0, graph=graph)
        torch.cuda.synchronize()
        got.append((obs, rew, done, env.get_state_bytes()))
        env.close()
    assert _same(*got)


@pytest.mark.parametrize("w", [64, 68, 84, 88, 128])
def test_float32_rows_around_the_wave(w):
    """NHWC float32 rows of one wave, and of more in one pass or two."""
    cfg = W.env_cfg(obs_h=18, obs_w=w, episode_cap=9, obs_dtype=2, **TREE)
    byte = W.env_cfg(obs_h=18, obs_w=w, episode_cap=9, **TREE)
    want = _run(byte, 6, 11, ONE, False)
    frames = (want[0].cpu().numpy().astype(np.float32) / np.float32(255)).view(np.uint8)
    for launch in (ONE, dict(waves_per_group=4, waves_per_env=2), dict(waves_per_group=4, waves_per_env=4)):
        for fused in (False, True):
            got = _run(cfg, 6, 11, launch, fused)
            assert np.array_equal(got[0].cpu().numpy(), frames) and _same(got[1:4], want[1:4]), (launch, fused)


@pytest.mark.parametrize("layout,dtype", [(0, 0), (1, 0), (0, 1), (0, 2)])
@pytest.mark.parametrize("n,side", [(3072, 16), (3073, 16), (4097, 32)])
def test_rollouts_of_two_waves_per_simd(n, side, layout, dtype):
    """Around the batch from which groups of 4 waves hold back the CU's third group."""
    cfg = W.env_cfg(side=side, obs_h=54, obs_w=52, episode_cap=5, obs_layout=layout, obs_dtype=dtype, goal_sprite=1)
    want = _run(cfg, n, 6, ONE, False)
    assert _same(_run(cfg, n, 6, dict(waves_per_group=4), True), want)

"""GPU: kernels that the library takes only under a mapping of its own choice or only
launch by launch, each compared bit for bit with per-step launches of one wave per
env (groups of one wave), which the oracle tests cover: the persistent and the
pipelined per-step kernels on ASCII maps, the fused kernel of one wave per env in
every frame format, and what runs after the autotuner."""
import numpy as np
import pytest

import workloads as W
from tests.test_gpu_roll_paths import ONE, ROOMS, TREE, _run, _same

pytestmark = pytest.mark.gpu

FORMATS = [(layout, dtype) for layout in (0, 1) for dtype in (0, 1, 2)]


def _env(cfgs, n, index=None):
    from paper_2605_19926_amd import jx
    env = jx.Env(W.seeds(53, n), cfgs, index)
    env.reset()
    return env


def _steps(env, acts, launch, how):
    """Frames, rewards, dones and state after the steps; how: step, rollout (launch by
    launch), graph or fused."""
    import torch
    T, n, ob = acts.shape[0], env.n, env.obs_bytes
    if launch:
        env.set_launch(**launch)
    obs = torch.zeros(T * ob, dtype=torch.uint8, device=env.dev)
    rew = torch.zeros((T, n), device=env.dev)
    done = torch.zeros((T, n), dtype=torch.uint8, device=env.dev)
    if how == "step":
        for t in range(T):
            env.step(acts[t], obs[t * ob:(t + 1) * ob], rew[t], done[t])
    else:
        env.rollout(acts, obs, rew, done, T, obs_stride=ob, graph=how == "graph", fused=how == "fused")
    torch.cuda.synchronize()
    return obs, rew, done, env.get_state_bytes()


def test_per_step_forms_on_ascii_maps():
    """ASCII maps beside a generated maze: doors open and keys are taken on the way."""
    import torch
    cfgs = [W.ASCII["cfg"], W.ASCII_TINY["cfg"], dict(W.ASCII_TINY["cfg"], n_actions=6),
            W.env_cfg(side=16, loop_frac=0.1, goal_sprite=1, episode_cap=60)]
    n, T = 520, 90
    env = _env(cfgs, n, (np.arange(n) * 7 % 4).astype(np.int32))
    snap = env.get_state_bytes()
    acts = torch.from_numpy(W.actions(53, T, n, 6)).to(env.dev)
    want = _steps(env, acts, ONE, "step")
    assert float(want[1].max()) >= 0.5
    for launch in ([dict(form=1, waves_per_group=w, groups_per_cu=g, store_mode=s) for w, g, s in
                    ((1, 8, 0), (2, 4, 0), (4, 1, 1), (8, 1, 0))] +
                   [dict(form=2, waves_per_group=p, groups_per_cu=g, store_mode=s) for p, g, s in
                    ((1, 2, 0), (2, 2, 1), (4, 1, 0))]):
        for how in ("step", "rollout"):
            env.set_state_bytes(snap)
            assert _same(_steps(env, acts, launch, how), want), (launch, how)
    env.close()


@pytest.mark.parametrize("base", [dict(ROOMS), dict(TREE)])
def test_shaded_rollouts(base):
    """Distance shading in the fused kernels against single steps."""
    import torch
    env = _env(W.env_cfg(obs_h=64, obs_w=64, episode_cap=40, shade_levels=6, shade_dist=9.0, **base), 96)
    snap = env.get_state_bytes()
    acts = torch.from_numpy(W.actions(31, 50, 96, 6)).to(env.dev)
    want = _steps(env, acts, ONE, "step")
    for launch in (ONE, dict(waves_per_group=8), dict(form=1, waves_per_group=4, groups_per_cu=2)):
        for how in ("fused", "graph"):
            env.set_state_bytes(snap)
            assert _same(_steps(env, acts, launch, how), want), (launch, how)
    env.close()


@pytest.mark.parametrize("n,px", [(2048, 64), (300, 128)])
def test_steps_and_rollouts_after_tuning(n, px):
    import torch
    env = _env(W.env_cfg(obs_h=px, obs_w=px, episode_cap=9, goal_sprite=1, side=16, loop_frac=0.1), n)
    snap = env.get_state_bytes()
    acts = torch.from_numpy(W.actions(59, 8, n, 6)).to(env.dev)
    want = _steps(env, acts, ONE, "step")
    env.set_state_bytes(snap)
    env.autotune(acts, 4, env.new_obs())
    for how in ("step", "rollout", "graph", "fused"):
        env.set_state_bytes(snap)
        assert _same(_steps(env, acts, None, how), want), how
    env.close()


@pytest.mark.parametrize("base", [dict(ROOMS), dict(TREE)])
@pytest.mark.parametrize("layout,dtype", FORMATS)
def test_one_wave_rollouts_in_every_format(layout, dtype, base):
    for h, w in ((34, 72), (64, 64), (18, 128)):
        cfg = W.env_cfg(obs_h=h, obs_w=w, episode_cap=9, obs_layout=layout, obs_dtype=dtype, **base)
        want = _run(cfg, 9, 12, ONE, False)
        for store in (0, 1):
            assert _same(_run(cfg, 9, 12, dict(ONE, store_mode=store), True), want), (h, w, store)


@pytest.mark.parametrize("base", [dict(ROOMS), dict(TREE)])
@pytest.mark.parametrize("layout,dtype", FORMATS)
def test_full_chip_rollouts_in_every_format(layout, dtype, base):
    """From 6 envs per CU the library runs one wave per env."""
    cfg = W.env_cfg(obs_h=34, obs_w=36, episode_cap=5, obs_layout=layout, obs_dtype=dtype, **base)
    for n in (1537, 2050):
        assert _same(_run(cfg, n, 4, None, True), _run(cfg, n, 4, ONE, False)), n


@pytest.mark.parametrize("base", [dict(ROOMS), dict(TREE), dict(side=40, loop_frac=0.2, goal_sprite=1)])
@pytest.mark.parametrize("layout,dtype", [f for f in FORMATS if f[1]])
def test_large_frames_under_two_waves(layout, dtype, base):
    """Frames around the size from which the casting wave writes a third, up to an env
    per CU: odd numbers of row-pair blocks, idle lanes, a last block for one wave only."""
    for n, h, w in ((5, 84, 84), (3, 128, 128), (2, 62, 112), (2, 126, 72), (256, 90, 76), (257, 90, 76)):
        cfg = W.env_cfg(obs_h=h, obs_w=w, episode_cap=4, obs_layout=layout, obs_dtype=dtype, **base)
        T = 9 if n < 200 else 3
        want = _run(cfg, n, T, ONE, False)
        assert _same(_run(cfg, n, T, dict(waves_per_group=4, waves_per_env=2), True), want), (n, h, w)


@pytest.mark.parametrize("layout,dtype", FORMATS)
@pytest.mark.parametrize("n", [768, 769])
def test_wide_rows_under_four_waves(layout, dtype, n):
    """Around the batch from which one wave of four casts the wide rows of float frames."""
    cfg = W.env_cfg(obs_h=10, obs_w=72, episode_cap=4, obs_layout=layout, obs_dtype=dtype, **TREE)
    want = _run(cfg, n, 6, ONE, False)
    assert _same(_run(cfg, n, 6, dict(waves_per_group=4, waves_per_env=4), True), want)

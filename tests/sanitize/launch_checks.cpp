// The launch mappings that the context hands to the kernels, on the CPU: the
// library's host code over fake_hip.h, whose launches are recorded.
#include "fake_hip.h"

#include <unistd.h>

#include "../../paper_2605_19926_amd/csrc/jx_abi.cpp"

namespace {

struct Ctx {
  jx_ctx* c = nullptr;
  std::vector<uint8_t> ws, obs;
  std::vector<uint8_t> act, done;
  std::vector<float> rew;
  int n;
  jx_env_cfg cfg{};
  Ctx(int n_envs, int px, int T = 8, int layout = 0, int dtype = 0) : n(n_envs) {
    cfg.side = 8;
    cfg.obs_layout = layout;
    cfg.obs_dtype = dtype;
    cfg.n_colors = 8;
    cfg.goal_sprite = 1;
    cfg.obs_h = cfg.obs_w = px;
    cfg.fov_deg = 60.f;
    cfg.n_actions = 6;
    cfg.episode_cap = 64;
    cfg.move = 0.1f;
    cfg.turn = 0.2f;
    cfg.pickup_radius = 0.3f;
    cfg.r_goal = 1.f;
    const size_t bytes = jx_workspace_bytes(n, &cfg, 1, nullptr);
    ws.resize(bytes + 256);
    uint8_t* base = ws.data() + (256 - ((uintptr_t)ws.data() & 255)) % 256;
    std::vector<uint64_t> seeds(n);
    for (int i = 0; i < n; ++i) seeds[i] = (uint64_t)i;
    CHECK(jx_create(&c, 0, nullptr, base, bytes) == JX_OK, "create: %s", jx_last_error());
    CHECK(jx_reset(c, n, seeds.data(), &cfg, 1, nullptr, nullptr) == JX_OK, "reset: %s", jx_last_error());
    act.resize((size_t)T * n);
    done.resize((size_t)T * n);
    rew.resize((size_t)T * n);
    obs.resize((size_t)jx_obs_bytes(c) + 64);
  }
  ~Ctx() { jx_destroy(c); }
  uint8_t* frames() { return obs.data() + (64 - ((uintptr_t)obs.data() & 63)) % 64; }
  void set(int form, int wpg, int gpc, int store, int wpe) {
    const jx_launch l{form, wpg, gpc, store, wpe};
    CHECK(jx_set_launch(c, &l) == JX_OK, "set_launch: %s", jx_last_error());
  }
  fake::Launch step() {
    CHECK(jx_step(c, act.data(), frames(), rew.data(), done.data(), nullptr) == JX_OK, "step: %s", jx_last_error());
    return fake::launches.back();
  }
  fake::Launch render() {
    CHECK(jx_render(c, frames(), nullptr) == JX_OK, "render: %s", jx_last_error());
    return fake::launches.back();
  }
  fake::Launch rollout(int flags, int T = 8) {
    CHECK(jx_rollout(c, T, act.data(), frames(), 0, rew.data(), done.data(), nullptr, flags) == JX_OK, "rollout: %s",
          jx_last_error());
    return fake::launches.back();
  }
};

// One wave per env is what a group of one wave gives; larger groups and a mapping
// left to the library take more on a batch that leaves the chip idle.
void check_waves_per_env() {
  for (int n : {1, 128, 512, 700}) {
    Ctx x(n, 128);
    const int fused = n <= 512 ? 4 : 2;
    CHECK(x.step().waves_per_env == 4, "left to the library: step n %d", n);
    CHECK(x.rollout(JX_ROLLOUT_FUSED).waves_per_env == fused, "left to the library: fused n %d", n);
    for (int wpg : {1, 2, 4, 8}) {
      x.set(0, wpg, 1, 0, 1);
      CHECK(x.step().waves_per_env == (wpg >= 4 ? 4 : 1), "groups of %d: step n %d", wpg, n);
      CHECK(x.rollout(JX_ROLLOUT_FUSED).waves_per_env == std::min(wpg, fused), "groups of %d: fused n %d", wpg, n);
      CHECK(x.rollout(JX_ROLLOUT_GRAPH).waves_per_env == std::min(wpg, fused), "groups of %d: graph n %d", wpg, n);
      for (int wpe : {2, 4})
        if (wpe <= wpg) {
          x.set(0, wpg, 1, 0, wpe);
          CHECK(x.step().waves_per_env == wpe && x.rollout(JX_ROLLOUT_FUSED).waves_per_env == wpe, "asked for %d", wpe);
        }
    }
    jx_render(x.c, nullptr, nullptr);
    CHECK(fake::launches.back().waves_per_env == 1, "a render without frames n %d", n);
  }
  Ctx big(2048, 128);
  CHECK(big.step().waves_per_env == 1 && big.rollout(JX_ROLLOUT_FUSED).waves_per_env == 1, "a full chip");
  Ctx small(256, 64);  // 12 KB frames
  CHECK(small.step().waves_per_env == 1, "small frames");
}

// A render shares envs where the batch leaves the chip idle, whatever is asked of steps.
void check_renders() {
  for (int n : {100, 768, 1024, 1025, 4096})
    for (int px : {16, 64, 84, 128}) {
      if (n == 4096 && px == 128) continue;
      Ctx x(n, px, 1);
      const int idle = px > 64 ? (n <= 1024 ? 4 : 1) : 1;
      CHECK(x.render().waves_per_env == idle, "left to the library: n %d, %d px", n, px);
      for (int wpg : {2, 4, 8})
        for (int wpe : {1, 2, 4}) {
          if (wpe > wpg) continue;
          x.set(0, wpg, 1, 0, wpe);
          CHECK(x.render().waves_per_env == (wpg >= 4 ? idle : 1), "groups of %d, %d asked for: n %d, %d px", wpg, wpe, n, px);
          if (wpe > 1) CHECK(x.step().waves_per_env == wpe, "a step takes the %d asked for", wpe);
        }
    }
}

// What jx_get_launch returns is what a step runs, and setting it changes no step.
void check_reported_mapping() {
  for (int n : {16, 700, 4096})
    for (int px : {16, 128}) {
      if (n == 4096 && px == 128) continue;
      Ctx x(n, px);
      const fake::Launch before = x.step();
      jx_launch l{};
      CHECK(jx_get_launch(x.c, &l) == JX_OK, "get_launch");
      CHECK(l.form == before.cfg.form && l.waves_per_group == before.cfg.waves_per_group &&
                l.store_mode == before.cfg.store_mode && l.waves_per_env == before.cfg.waves_per_env,
            "n %d: reports groups of %d, runs %d", n, l.waves_per_group, before.cfg.waves_per_group);
      x.set(1, 2, 4, 1, 1);
      CHECK(jx_set_launch(x.c, &l) == JX_OK, "restored");
      const fake::Launch after = x.step();
      CHECK(after.cfg.form == before.cfg.form && after.cfg.waves_per_group == before.cfg.waves_per_group &&
                after.cfg.store_mode == before.cfg.store_mode && after.waves_per_env == before.waves_per_env,
            "n %d: a restored mapping runs groups of %d, before %d", n, after.cfg.waves_per_group,
            before.cfg.waves_per_group);
      jx_launch again{};
      jx_get_launch(x.c, &again);
      CHECK(std::memcmp(&again, &l, sizeof l) == 0, "n %d: reported again", n);
    }
  Ctx x(64, 16);
  for (int form : {0, 1, 2}) {
    x.set(form, 2, 3, 1, form == 0 ? 2 : 1);
    jx_launch l{};
    jx_get_launch(x.c, &l);
    CHECK(l.form == form && l.waves_per_group == 2 && l.groups_per_cu == 3 && l.store_mode == 1 &&
              l.waves_per_env == (form == 0 ? 2 : 1), "a mapping that was set, form %d", form);
  }
}

// The graph flag takes one launch, but for a single step and a few steps of very many
// envs with larger byte frames.
void check_graph_flag() {
  for (int layout : {0, 1})
    for (int dtype : {0, 1, 2})
      for (int px : {16, 64})
        for (int n : {8192, 8193}) {
          if (px * px * (dtype + 1) > 64 * 64 && n == 8192) continue;
          Ctx x(n, px, 4, layout, dtype);
          for (int T : {1, 2, 3, 4}) {
            const size_t first = fake::launches.size();
            x.rollout(JX_ROLLOUT_GRAPH, T);
            const bool steps = T == 1 || (T < 4 && n > 8192 && dtype == 0 && px == 64);
            const size_t made = fake::launches.size() - first;
            CHECK(made == (steps ? (size_t)T : 1u) && fake::launches.back().kind == (steps ? "batch" : "fused"),
                  "layout %d, type %d, %d px, n %d, T %d: %zu launches", layout, dtype, px, n, T, made);
          }
        }
}

// The tuner's pick drives per-step launches; fused rollouts, which it does not
// time, keep the library's own mapping until a caller sets the pick.
int g_timed = 0, g_want = 0;
double scripted_ms() { return g_timed++ / 2 == g_want ? 0.5 : 1.0; }  // each candidate is timed twice

bool same_cfg(const LaunchCfg& a, const LaunchCfg& b) { return std::memcmp(&a, &b, sizeof a) == 0; }

void check_tuned_mapping() {
  const std::string cache = "/tmp/jx_launch_checks_" + std::to_string(getpid()) + ".txt";
  fake::elapsed_ms = scripted_ms;
  for (int want = 0; want < 48; ++want) {
    std::remove(cache.c_str());
    Ctx x(4096, 16);
    const LaunchCfg fused = x.rollout(JX_ROLLOUT_FUSED).cfg, graph = x.rollout(JX_ROLLOUT_GRAPH).cfg;
    g_timed = 0;
    g_want = want;
    jx_launch pick{}, again{};
    CHECK(jx_autotune(x.c, x.act.data(), 8, x.frames(), cache.c_str(), &pick) == JX_OK, "tune: %s", jx_last_error());
    for (int cached = 0; cached < 2; ++cached) {
      const LaunchCfg step = x.step().cfg;
      CHECK(step.form == pick.form && step.waves_per_group == pick.waves_per_group && step.store_mode == pick.store_mode &&
                step.waves_per_env == pick.waves_per_env, "candidate %d: the step's mapping", want);
      CHECK(same_cfg(x.rollout(JX_ROLLOUT_FUSED).cfg, fused), "candidate %d: fused rollout", want);
      CHECK(same_cfg(x.rollout(JX_ROLLOUT_GRAPH).cfg, graph), "candidate %d: graph rollout", want);
      if (cached == 0) CHECK(jx_autotune(x.c, x.act.data(), 8, x.frames(), cache.c_str(), &again) == JX_OK, "cached");
    }
    CHECK(std::memcmp(&pick, &again, sizeof pick) == 0, "candidate %d: the cached pick", want);
    jx_set_launch(x.c, &pick);
    const LaunchCfg set = x.rollout(JX_ROLLOUT_FUSED).cfg;
    CHECK(pick.form == 2 || (set.form == pick.form && set.waves_per_group == pick.waves_per_group &&
                             set.store_mode == pick.store_mode), "candidate %d: a pick that was set", want);
  }
  std::remove(cache.c_str());
}

// Every candidate is named by the waves per env that it runs, and timed once.
void check_tuner_candidates() {
  fake::elapsed_ms = scripted_ms;
  for (int n : {128, 1024, 2048})  // 4 waves where 1 is asked for, up to 4 envs per CU
    for (int want = 0; want < 44; ++want) {
      if (n != 128 && want % 9) continue;
      Ctx x(n, n == 2048 ? 16 : 128, 1);
      const size_t first = fake::launches.size();
      g_timed = 0;
      g_want = want;
      jx_launch pick{};
      CHECK(jx_autotune(x.c, x.act.data(), 1, x.frames(), nullptr, &pick) == JX_OK, "tune: %s", jx_last_error());
      std::vector<std::string> seen;
      for (size_t k = first; k < fake::launches.size(); k += 2) {
        const fake::Launch& l = fake::launches[k];
        CHECK(l.cfg.form != 0 || l.cfg.waves_per_env == l.waves_per_env, "n %d: groups of %d are named %d, run %d", n,
              l.cfg.waves_per_group, l.cfg.waves_per_env, l.waves_per_env);
        char key[64];
        std::snprintf(key, sizeof key, "%d/%d/%d/%d/%d", l.cfg.form, l.cfg.waves_per_group, l.cfg.groups_per_cu,
                      l.cfg.store_mode, l.waves_per_env);
        CHECK(std::find(seen.begin(), seen.end(), key) == seen.end(), "n %d: %s is timed twice", n, key);
        seen.push_back(key);
      }
      CHECK(seen.size() == (n == 2048 ? 48u : 46u), "n %d: %zu candidates", n, seen.size());
      const fake::Launch s = x.step();
      CHECK(pick.form != 0 || s.waves_per_env == pick.waves_per_env, "n %d: picked %d waves per env, runs %d", n,
            pick.waves_per_env, s.waves_per_env);
    }
}

}  // namespace

int main() {
  check_waves_per_env();
  check_renders();
  check_reported_mapping();
  check_graph_flag();
  check_tuned_mapping();
  check_tuner_candidates();
  std::printf("launch checks: %d failures\n", fake::fails);
  return fake::fails != 0;
}

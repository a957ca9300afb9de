// The serving loop's host side on the CPU: the real server over fake_hip.h, whose
// launches run nothing and end when the check says so.
#define FAKE_THREADS
#include "fake_hip.h"
#include "jx_common.h"

extern "C" const char* jx_last_error(void) { return jx::g_last_error.c_str(); }  // (jx_abi.cpp's)

#include "../../paper_2605_19926_amd/csrc/jx_server.cpp"

namespace {

constexpr int kPx = 64;

jx_env_cfg config() {
  jx_env_cfg c{};
  c.side = 8;
  c.n_colors = 8;
  c.goal_sprite = 1;
  c.obs_h = c.obs_w = kPx;
  c.fov_deg = 60.f;
  c.n_actions = 6;
  c.episode_cap = 64;
  c.move = 0.1f;
  c.turn = 0.2f;
  c.pickup_radius = 0.3f;
  c.r_goal = 1.f;
  return c;
}

struct Srv {
  jx_server* s = nullptr;
  explicit Srv(size_t budget, int mode = JX_SERVE_COALESCE, int streams = 2) {
    CHECK(jx_server_create(&s, 0, budget, streams, mode, 0) == JX_OK, "create: %s", jx_last_error());
  }
  ~Srv() { jx_server_destroy(s); }
  // large_map: 4 KB of map and 48 B of frame per env, so that the budget is spent on state
  int open(int n, jx_status want = JX_OK, bool large_map = false) {
    std::vector<uint64_t> seeds(n, 7);
    jx_env_cfg c = config();
    if (large_map) {
      c.side = 64;
      c.obs_h = c.obs_w = 4;
    }
    int32_t id = -1;
    const jx_status st = jx_server_open(s, n, seeds.data(), &c, &id);
    CHECK(st == want, "open of %d: %d, %s", n, st, jx_last_error());
    return id;
  }
  uint64_t submit(int id, int n) {
    std::vector<uint8_t> a(n, 1);
    uint64_t t = 0;
    CHECK(jx_server_submit(s, id, a.data(), &t) == JX_OK, "submit: %s", jx_last_error());
    return t;
  }
  jx_status wait(uint64_t t, double timeout) { return jx_server_wait(s, t, timeout, nullptr, nullptr, nullptr, nullptr); }
  template <typename F>
  auto locked(F&& f) {
    std::lock_guard<std::mutex> g(s->mu);
    return f();
  }
  // true once f() (under the lock) holds; false after 5 s
  template <typename F>
  bool soon(F&& f) {
    for (int i = 0; i < 5000; ++i) {
      if (locked(f)) return true;
      std::this_thread::sleep_for(std::chrono::milliseconds(1));
    }
    return false;
  }
};

// A wait polls, then sleeps: it ends at its time limit, on either side of the
// poll's length, and with the request.
void check_wait_timeouts() {
  Srv v(64 << 20);
  const int id = v.open(4);
  fake::events_done = false;
  const uint64_t t = v.submit(id, 4);
  CHECK(v.wait(t, 0.0) == JX_EBUSY, "poll");
  for (double limit : {1e-6, 50e-6, 100e-6, 101e-6, 2e-3, 50e-3}) {
    const double began = now_s();
    CHECK(v.wait(t, limit) == JX_EBUSY, "limit %g", limit);
    const double took = now_s() - began;
    CHECK(took >= limit && took < limit + 2.0, "a wait of %g s took %g", limit, took);
  }
  std::thread later([&] {
    std::this_thread::sleep_for(std::chrono::milliseconds(20));
    fake::events_done = true;
  });
  double latency = 0;
  CHECK(jx_server_wait(v.s, t, -1.0, nullptr, nullptr, nullptr, &latency) == JX_OK, "wait without limit");
  CHECK(latency >= 0.02 && latency < 5.0, "latency %g", latency);
  later.join();
  CHECK(v.wait(t, 0.0) == JX_EINVAL, "collected twice");
  // finished before the wait begins
  const uint64_t u = v.submit(id, 4);
  CHECK(v.soon([&] { return v.s->requests[u]->status.load() == 2; }), "finished");
  CHECK(v.wait(u, 0.0) == JX_OK, "poll of a finished request");
}

// A scheduler that found no room for a launch's results goes on when a collected
// request gives its room back, and only then.
void check_full_arena() {
  const int n = 64;  // 786 KB of frames a step
  for (int mode : {JX_SERVE_COALESCE, JX_SERVE_PLAIN}) {
    Srv v(size_t(n) * kPx * kPx * 3 * 3 / 2, mode);
    const int id = v.open(n);
    uint64_t a = v.submit(id, n);
    CHECK(v.soon([&] { return v.s->requests[a]->status.load() == 2; }), "the first request runs");
    for (int k = 0; k < 20; ++k) {
      const uint64_t b = v.submit(id, n);
      CHECK(v.soon([&] { return v.s->starved; }), "mode %d: the second waits for room", mode);
      CHECK(v.wait(b, 2e-3) == JX_EBUSY, "mode %d: no room yet", mode);
      CHECK(v.wait(a, 0.0) == JX_OK, "mode %d: the first is collected", mode);
      CHECK(v.soon([&] { return v.s->requests[b]->status.load() == 2; }), "mode %d: the second runs then", mode);
      a = b;
    }
    CHECK(v.wait(a, 5.0) == JX_OK, "the last");
  }
}

// Closed clients are released once their requests have run, whichever comes first,
// and nothing is left to look for.
void check_closing() {
  Srv v(64 << 20);
  for (int k = 0; k < 20; ++k) {
    const int id = v.open(3), other = v.open(5);
    const uint64_t t = v.submit(id, 3), u = v.submit(id, 3);
    CHECK(jx_server_close(v.s, id) == JX_OK, "close");
    const jx_status twice = jx_server_close(v.s, id);  // still running, or gone already
    CHECK(twice == JX_OK || twice == JX_EINVAL, "close twice: %d", twice);
    CHECK(jx_server_close(v.s, other) == JX_OK, "close of an idle client");
    CHECK(v.wait(t, 5.0) == JX_OK && v.wait(u, 5.0) == JX_OK, "results stay collectable");
    CHECK(v.soon([&] { return v.s->clients.empty(); }), "released");
    CHECK(v.locked([&] { return v.s->closing == 0 && v.s->arena.used() == 0; }), "%d clients still counted", v.s->closing);
  }
  // a client that never was admitted leaves at once
  Srv w(512 << 10);
  const int a = w.open(80, JX_OK, true), b = w.open(90, JX_EBUSY, true);
  CHECK(jx_server_close(w.s, b) == JX_OK, "close of a queued client");
  CHECK(w.locked([&] { return w.s->closing == 0 && w.s->clients.size() == 1; }), "queued client");
  CHECK(jx_server_close(w.s, a) == JX_OK && w.soon([&] { return w.s->clients.empty() && w.s->closing == 0; }), "the other");
}

// A client closed before its admission fails is not looked for afterwards.
void check_closing_failed_admission() {
  for (int again = 0; again < 2; ++again) {
    Srv v(512 << 10);
    const int a = v.open(80, JX_OK, true), b = v.open(90, JX_EBUSY, true);
    const uint64_t t = v.submit(b, 90);
    if (!again) CHECK(jx_server_close(v.s, b) == JX_OK, "close while queued");
    fake::fail_uploads = 1;
    CHECK(jx_server_close(v.s, a) == JX_OK, "room for the queued client");
    CHECK(v.wait(t, 5.0) == JX_EDEVICE, "its request fails with the admission");
    if (again) jx_server_close(v.s, b);  // closed after the failure
    CHECK(v.soon([&] { return v.s->closing == 0; }), "%d clients still counted, closed %s its admission failed",
          v.s->closing, again ? "after" : "before");
    fake::fail_uploads = 0;
  }
}

}  // namespace

int main() {
  check_wait_timeouts();
  check_full_arena();
  check_closing();
  check_closing_failed_admission();
  std::printf("server checks: %d failures\n", fake::fails);
  return fake::fails != 0;
}

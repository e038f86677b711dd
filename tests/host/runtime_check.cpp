// The library's host side against a stand-in for the HIP runtime (no GPU),
// built and run by tests/test_host_library.py: runtime_check <scenario>.
#include <sys/wait.h>
#include <unistd.h>

#include <chrono>
#include <functional>
#include <string>
#include <thread>
#include <vector>

#include "fake_hip.hpp"
#include "icr.h"

static int failures = 0;
#define CHECK(c, ...)                                                        \
  do {                                                                       \
    if (!(c)) {                                                              \
      ++failures;                                                            \
      std::printf("line %d: %s: ", __LINE__, #c);                            \
      std::printf(__VA_ARGS__);                                              \
      std::printf("\n");                                                     \
    }                                                                        \
  } while (0)

// A box of n^3 nodes, six tetrahedra to a cell, its top layer clamped.
struct Grid {
  int n;
  std::vector<double> nodes, E, nu;
  std::vector<int32_t> tets;
  std::vector<uint8_t> fixed;
  explicit Grid(int n_) : n(n_) {
    for (int k = 0; k < n; ++k)
      for (int j = 0; j < n; ++j)
        for (int i = 0; i < n; ++i) {
          nodes.insert(nodes.end(), {0.01 * i, 0.01 * j, 0.01 * k});
          fixed.push_back(k == n - 1);
        }
    static const int path[6][2] = {{1, 2}, {1, 4}, {2, 1}, {2, 4}, {4, 1}, {4, 2}};
    for (int k = 0; k + 1 < n; ++k)
      for (int j = 0; j + 1 < n; ++j)
        for (int i = 0; i + 1 < n; ++i)
          for (auto &p : path) {
            const int c[4] = {0, p[0], p[0] + p[1], 7};
            for (int q : c) tets.push_back(i + (q & 1) + n * (j + (q >> 1 & 1) + n * (k + (q >> 2))));
          }
    E.assign(tets.size() / 4, 5e3);
    nu.assign(E.size(), 0.4);
  }
  int count() const { return n * n * n; }
  icr_scene *scene(bool factor = true) const {
    icr_scene *s = nullptr;
    const double g[3] = {0, 0, -9.81};
    CHECK(icr_create(&s, nullptr) == ICR_OK, "create");
    CHECK(icr_assemble(s, nodes.data(), count(), tets.data(), (int)E.size(), E.data(), nu.data(), 1e3, 0.1, 0.1, 0.01,
                       g, fixed.data()) == ICR_OK, "%s", icr_last_error(s));
    if (factor) CHECK(icr_factor(s) == ICR_OK, "%s", icr_last_error(s));
    return s;
  }
};

// A call that has to grow the scene's buffers and cannot, at every one of its
// allocations in turn, then the smaller call from before: that one has to
// allocate again and must not touch what was given back.
static void regrow(const char *name, const std::function<void(icr_scene *)> &setup,
                   const std::function<icr_status(icr_scene *)> &small, const std::function<icr_status(icr_scene *)> &large) {
  const Grid grid(8);
  long at = 0;
  for (;; ++at) {
    icr_scene *s = grid.scene();
    setup(s);
    const icr_status st0 = small(s);
    CHECK(st0 == ICR_OK || st0 == ICR_WARN_NOT_CONVERGED, "%s: %s", name, icr_last_error(s));
    fake::fail_in = at;
    const icr_status st = large(s);
    const bool failed = fake::fail_in == 0 && st != ICR_OK && st != ICR_WARN_NOT_CONVERGED;
    fake::fail_in = -1;
    if (failed) {
      CHECK(st == ICR_E_OOM, "%s, allocation %ld: status %d", name, at, st);
      icr_release_idle();
      const long before = fake::mallocs;
      const icr_status again = small(s);
      CHECK(again == st0, "%s, allocation %ld: %s", name, at, icr_last_error(s));
      CHECK(fake::mallocs > before, "%s, allocation %ld: the smaller call kept the released buffers", name, at);
      CHECK(fake::stale == 0, "%s, allocation %ld: released memory used", name, at);
      fake::stale = 0;
    }
    icr_destroy(s);
    icr_release_idle();
    if (!failed) break;
  }
  CHECK(at > 0, "%s: no allocation", name);   // some of them are served by blocks just released
  CHECK(fake::bytes == 0, "%s: %zu bytes left", name, fake::bytes);
}

// device arrays of the caller
template <class T>
static T *device(const std::vector<T> &v) {
  void *p = nullptr;
  if (hipMalloc(&p, v.size() * sizeof(T)) != hipSuccess) std::abort();
  std::memcpy(p, v.data(), v.size() * sizeof(T));
  return static_cast<T *>(p);
}

static void scenario_regrow() {
  const auto none = [](icr_scene *) {};
  std::vector<int32_t> free_nodes(300);
  for (int i = 0; i < 300; ++i) free_nodes[i] = i;
  int32_t *ids = device(free_nodes);
  std::vector<int32_t> m_ids(4 * 300, -1);
  std::vector<double> m_w(4 * 300, 1.0);
  for (int i = 0; i < 300; ++i) m_ids[4 * i] = i;
  int32_t *mi = device(m_ids);
  double *mw = device(m_w), *out = device(std::vector<double>(900 * 900)), *vec = device(std::vector<double>(3600));
  int8_t *status = device(std::vector<int8_t>(600));
  const size_t mine = fake::bytes;
  fake::bytes = 0;
  regrow("W_H", none, [&](icr_scene *s) { return icr_build_WH(s, 20, ids, nullptr, out); },
         [&](icr_scene *s) { return icr_build_WH(s, 40, ids, nullptr, out); });
  // (the nodes' own buffers are large enough from the start)
  regrow("mapped W_H", [&](icr_scene *s) { CHECK(icr_build_WH(s, 60, ids, nullptr, out) == ICR_OK, "W_H"); },
         [&](icr_scene *s) { return icr_build_WH(s, 20, mi, mw, out); },
         [&](icr_scene *s) { return icr_build_WH(s, 40, mi, mw, out); });
  auto solve = [&](int n) {
    return [=](icr_scene *s) {
      int32_t sweeps = 0;
      return icr_solve_contacts(s, n, out, vec, vec, 0.01, vec, status, 2, 1e300, 8, &sweeps, nullptr);
    };
  };
  regrow("contact solve", none, solve(20), solve(600));
  icr_obstacle obs{};
  obs.normal[2] = 1.0;
  auto step = [&](int n, int precision) {
    return [=](icr_scene *s) {
      icr_step_opts o{};
      o.n_contacts = n;
      o.n_newton = 2;
      o.max_sweeps = 2;
      o.j_inner = 8;
      o.tol = 1e300;
      o.precision = precision;
      return icr_step(s, &obs, &o, nullptr);
    };
  };
  const std::vector<double> mu(300, 0.5);
  auto candidates = [&](icr_scene *s) { CHECK(icr_set_candidates(s, 250, free_nodes.data(), mu.data()) == ICR_OK, "set"); };
  auto reserved = [&](icr_scene *s) {
    candidates(s);
    CHECK(icr_reserve(s, 200, ICR_FP64) == ICR_OK, "reserve");
  };
  regrow("step", candidates, step(20, ICR_FP64), step(40, ICR_FP64));
  regrow("mixed step", candidates, step(20, ICR_FP32_IR), step(40, ICR_FP32_IR));
  regrow("step with pairs",
         [&](icr_scene *s) {
           reserved(s);
           std::vector<int32_t> pi(4 * 10, -1);
           std::vector<double> pw(4 * 10, 0.0), pn(3 * 10, 0.0);
           for (int i = 0; i < 10; ++i) pi[4 * i] = 280 + i, pw[4 * i] = 1.0, pn[3 * i + 2] = 1.0;
           CHECK(icr_set_pairs(s, 10, pi.data(), pw.data(), pn.data(), mu.data()) == ICR_OK, "%s", icr_last_error(s));
         },
         step(20, ICR_FP64), step(40, ICR_FP64));
  fake::bytes += mine;
  // a list of pairs or candidates that could not be stored is not there
  const Grid grid(8);
  icr_scene *s = grid.scene();
  reserved(s);
  for (long at = 0; at < 2; ++at) {
    fake::fail_in = at;
    CHECK(icr_set_candidates(s, 20, free_nodes.data() + 100, mu.data()) == ICR_E_OOM, "allocation %ld", at);
    fake::fail_in = -1;
    CHECK(step(250, ICR_FP64)(s) == ICR_OK, "the former candidates are gone: %s", icr_last_error(s));
  }
  std::vector<int32_t> pi(4 * 10, -1);
  std::vector<double> pw(4 * 10, 0.0), pn(3 * 10, 0.0);
  for (int i = 0; i < 10; ++i) pi[4 * i] = 280 + i, pw[4 * i] = 1.0, pn[3 * i + 2] = 1.0;
  for (long at = 0;; ++at) {
    icr_release_idle();
    fake::fail_in = at;
    const icr_status st = icr_set_pairs(s, 10, pi.data(), pw.data(), pn.data(), mu.data());
    fake::fail_in = -1;
    if (st == ICR_OK) {
      CHECK(at > 0, "no allocation");
      break;
    }
    CHECK(st == ICR_E_OOM, "allocation %ld", at);
    CHECK(step(5, ICR_FP64)(s) == ICR_OK, "pairs that could not be stored are in force: %s", icr_last_error(s));
  }
  // results of a step whose buffers are gone
  fake::fail_in = 3;
  CHECK(icr_reserve(s, 400, ICR_FP64) == ICR_E_OOM, "reserve");
  fake::fail_in = -1;
  CHECK(icr_get_step_results(s, nullptr, nullptr, vec, nullptr, nullptr, nullptr, nullptr, nullptr) == ICR_E_STATE,
        "results from released buffers");
  icr_destroy(s);
}

// Memory that is kept for the next scene: closing one, or growing its buffers,
// waits for the device first, as freeing the memory would.
static void scenario_close() {
  const Grid grid(8);
  for (bool moved : {false, true}) {
    icr_scene *s = grid.scene();
    if (moved) CHECK(icr_set_stream(s, (void *)0x30) == ICR_OK, "stream");
    const size_t held = fake::bytes;
    long frees = fake::frees;
    CHECK(icr_reserve(s, 20, ICR_FP64) == ICR_OK && icr_reserve(s, 40, ICR_FP64) == ICR_OK, "%s", icr_last_error(s));
    CHECK(fake::frees > frees, "no wait before the buffers of 20 contacts were handed on");
    frees = fake::frees;
    icr_destroy(s);
    CHECK(fake::frees > frees, "no wait before the scene's memory was handed on");
    CHECK(fake::bytes >= held, "nothing kept of %zu bytes", held);
    const size_t kept = fake::bytes;
    s = grid.scene();
    CHECK(fake::bytes == kept, "%zu bytes, then %zu with a scene of the same size", kept, fake::bytes);
    icr_destroy(s);
    icr_release_idle();
    CHECK(fake::bytes == 0, "%zu bytes left", fake::bytes);
  }
}

// Memory that no scene takes is freed ten seconds later, without a call of the
// library, also when others are closed and opened meanwhile.
static void scenario_idle_time() {
  using namespace std::chrono;
  const Grid small(5), large(8);
  auto held = [] {
    std::lock_guard<std::mutex> l(fake::mtx);
    return fake::bytes;
  };
  icr_scene *s = large.scene();
  const auto t0 = steady_clock::now();
  icr_destroy(s);
  const size_t big = held();
  CHECK(big > 0, "nothing kept");
  std::this_thread::sleep_until(t0 + seconds(5));
  icr_scene *live = small.scene();
  s = small.scene();
  icr_destroy(s);
  CHECK(held() >= big, "freed before its time");
  std::this_thread::sleep_until(t0 + milliseconds(12000));
  CHECK(held() < big, "%zu of %zu bytes still there", held(), big);
  // a forked child has no such thread, and ends without waiting for it, also
  // while the parent's is inside a free
  fake::slow_frees = 1;
  std::this_thread::sleep_until(t0 + milliseconds(15500));
  const pid_t child = fork();
  if (child == 0) {
    alarm(5);   // ends the child if it waits
    std::exit(0);
  }
  int end = 0;
  CHECK(child > 0 && waitpid(child, &end, 0) == child && WIFEXITED(end) && WEXITSTATUS(end) == 0, "child ended with %d", end);
  std::this_thread::sleep_until(t0 + milliseconds(19000));
  icr_factor_info info{};
  CHECK(icr_get_factor_info(live, &info) == ICR_OK, "info");
  CHECK(held() < (size_t)info.device_bytes + (2u << 20), "%zu bytes beside a scene of %lld", held(),
        (long long)info.device_bytes);
  icr_destroy(live);
  icr_release_idle();
  CHECK(held() == 0, "%zu bytes left", held());
  // the process ends with idle memory: no call of the runtime after its end
  // (its clean-up was registered before the library's first release: see main)
  icr_destroy(large.scene());
}

int main(int argc, char **argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  std::atexit([] {   // as the runtime's clean-up
    fake::ended = true;
    std::this_thread::sleep_for(std::chrono::milliseconds(200));
    if (fake::late) std::_Exit(3);
  });
  if (what == "regrow")
    scenario_regrow();
  else if (what == "close")
    scenario_close();
  else if (what == "idle_time")
    scenario_idle_time();
  else
    return 2;
  CHECK(fake::stale == 0, "%ld", fake::stale);
  std::printf(failures ? "%d failures\n" : "ok\n", failures);
  return failures != 0;
}

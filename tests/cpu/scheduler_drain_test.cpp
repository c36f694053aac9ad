// The scheduler's failure path on the CPU: whatever ends a tick, the executor
// has waited for what it enqueued before any job, plan or group goes.
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "scheduler.h"

using namespace muster;

static int g_failed = 0;
#define CHECK(c)                                                    \
  do {                                                              \
    if (!(c)) {                                                     \
      std::printf("  FAILED %s:%d: %s\n", __FILE__, __LINE__, #c);  \
      ++g_failed;                                                   \
    }                                                               \
  } while (0)

static double fake_clock() {
  static double t = 0.0;
  return t += 0.001;
}

enum Fail { NONE, STEP, SYNC, BEGIN, FINISH };

struct Fake;
struct FakeJob : JobHandle {
  Fake* ex = nullptr;
  int level = 0;
  ~FakeJob() override;
};

struct Fake : Executor {
  Fail fail = NONE;
  int fail_at = 0;        // the call of that kind that throws
  muster_status st = MUSTER_E_NOMEM;
  int calls = 0;
  bool in_flight = false;  // work enqueued and not waited for
  int released_in_flight = 0, drains = 0;
  bool poisoned = false;
  void maybe(Fail f) {
    if (fail == f && calls++ == fail_at) throw Error{st, "fake"};
  }
  uint64_t footprint(const muster_job&) override { return 1; }
  uint64_t budget() override { return 0; }
  bool fits(uint64_t) override { return true; }
  std::unique_ptr<JobHandle> admit(const muster_job&) override {
    auto h = std::make_unique<FakeJob>();
    h->ex = this;
    return h;
  }
  void step(const GroupKey&, const std::vector<JobHandle*>&,
            const std::vector<std::pair<uint64_t, int>>&) override {
    maybe(STEP);
    in_flight = true;
  }
  void forget_groups_except(const std::vector<GroupKey>&) override {
    if (in_flight) ++released_in_flight;
  }
  void sync(const std::vector<JobHandle*>&) override {
    maybe(SYNC);
    in_flight = false;
  }
  int level(JobHandle& h) override { return static_cast<FakeJob&>(h).level; }
  bool nonfinite(JobHandle&) override { return false; }
  void begin_level(JobHandle& h, int level) override {
    in_flight = true;
    maybe(BEGIN);
    static_cast<FakeJob&>(h).level = level;
    in_flight = false;
  }
  void finish(JobHandle&, double, muster_report*) override {
    in_flight = true;
    maybe(FINISH);
    in_flight = false;
  }
  uint64_t held_bytes(JobHandle&) override { return 1; }
  void on_device_error() override { poisoned = true; }
  void drain() noexcept {
    ++drains;
    in_flight = false;
  }
};

FakeJob::~FakeJob() {
  if (ex->in_flight) ++ex->released_in_flight;
}

static muster_job job(int window, int levels) {
  muster_job j;
  std::memset(&j, 0, sizeof j);
  j.N = 2;
  for (int d = 0; d < 3; ++d) j.dims[d] = 8;
  j.params.levels = levels;
  for (int l = 0; l < levels; ++l) j.params.iters[l] = 1;
  j.params.window = window;
  j.params.metric = MUSTER_METRIC_SILNCC;
  j.params.K = 5;
  return j;
}

// Two groups (windows 3 and 5); the given call of the given kind throws.
static void run(const char* what, Fail f, int at, muster_status st) {
  std::printf("%s\n", what);
  Fake ex;
  ex.fail = f;
  ex.fail_at = at;
  ex.st = st;
  Scheduler s(ex, 8, fake_clock);
  const uint64_t a = s.submit(job(3, 2)), b = s.submit(job(5, 2));
  for (int k = 0; k < 4; ++k) s.tick();
  CHECK(s.poll(a) == 3 && s.poll(b) == 3);
  CHECK(ex.drains >= 1);
  CHECK(ex.released_in_flight == 0);
  CHECK(ex.poisoned == (st == MUSTER_E_DEVICE));
  muster_report r{};
  std::string err;
  CHECK(s.wait(a, &r, &err) == st && err == "fake");
  CHECK(s.wait(b, &r, &err) == st);
}

int main() {
  run("the second group's step", STEP, 1, MUSTER_E_NOMEM);
  run("the second group's step, device error", STEP, 1, MUSTER_E_DEVICE);
  run("the wait after the steps", SYNC, 0, MUSTER_E_DEVICE);
  run("a change of level", BEGIN, 1, MUSTER_E_NOMEM);
  run("the outputs", FINISH, 0, MUSTER_E_NOMEM);
  {
    std::printf("a stopped server\n");
    Fake ex;
    Scheduler s(ex, 8, fake_clock);
    s.submit(job(3, 2));
    s.tick();
    ex.in_flight = true;
    s.stop();
    s.shutdown();
    CHECK(ex.released_in_flight == 0);
  }
  if (g_failed) {
    std::printf("%d checks failed\n", g_failed);
    return 1;
  }
  std::printf("all passed\n");
  return 0;
}

// Checks of the C ABI's host code on the CPU (tests/test_native_api.py builds and runs them): which
// launches and copies the library issues, with which addresses, over a HIP runtime of the check's
// own (fake_hip.h).  Kernels do nothing; what the host reads back -- residuals, states of the
// iterations -- is what the check says.  The structures have nodes and no elements: K has no blocks.
#include "fake_hip.h"

#include "hipsso.h"
#include "sso_internal.h"

#include <new>

using namespace sso;

// Host memory that may run short: requests of at least this many bytes are refused (0: none).  The
// library's own go this way too.
static std::atomic<size_t> refuse_from{0};
void* operator new(size_t n) {
  const size_t from = refuse_from;
  if (from && n >= from) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

static int failures = 0;
#define CHECK(c)                                                       \
  do {                                                                 \
    if (!(c)) {                                                        \
      std::printf("FAIL %s:%d: %s\n", __FILE__, __LINE__, #c);         \
      ++failures;                                                      \
    }                                                                  \
  } while (0)

static bool is(const std::string& name, const char* kernel) {
  return name.find(kernel) != std::string::npos;
}
static int launches(const char* kernel) {
  int n = 0;
  for (const auto& k : fake::state().launches)
    if (is(k.first, kernel)) n += k.second;
  return n;
}

// What the GPU would do, as far as the host sees it.
struct Script {
  std::vector<double> rr;      // ||r||^2 of the true residuals in turn, ||b||^2 being 1; then 0
  size_t next = 0;
  bool singular = false;       // factorisations find a pivot that is too small
  double residual() { return next < rr.size() ? rr[next++] : 0.0; }
} script;

static void finish_state(PcgState* st) {
  st->it = 5;
  st->done = 1;
  st->status = SSO_OK;
}

static void kernel(const fake::Launch& l) {
  if (is(l.name, "k_direct_clear") || is(l.name, "k_front_")) {
    const DirectArgs* probs = l.arg<const DirectArgs*>(1);
    const int n = !probs ? 1 : is(l.name, "k_direct_clear") ? l.arg<int>(2) : (int)l.grid.y;
    for (int i = 0; i < n; ++i) {
      const DirectArgs a = probs ? probs[i] : l.arg<DirectArgs>(0);
      bool ok = fake::valid(a.flag, sizeof *a.flag, l.stream, "the direct solver's flag");
      if (is(l.name, "k_front_")) {
        for (const void* p : {(const void*)a.fronts, (const void*)a.nodes, (const void*)a.items,
                              (const void*)a.fact, (const void*)a.K})
          ok = fake::valid(p, 8, l.stream, l.name.c_str()) && ok;
        if (is(l.name, "forward") || is(l.name, "backward"))
          for (const void* p : {(const void*)a.rhs, (const void*)a.sol, (const void*)a.b})
            ok = fake::valid(p, 8, l.stream, l.name.c_str()) && ok;
      }
      if (ok) *a.flag = is(l.name, "k_front_first") && script.singular ? 1u : is(l.name, "clear") ? 0u : *a.flag;
    }
  } else if (is(l.name, "k_finish_many")) {
    const ResidualJob* jobs = l.arg<const ResidualJob*>(0);
    double* out = l.arg<double*>(1);
    for (unsigned i = 0; i < l.grid.x; ++i) {
      out[3 * i] = script.residual();
      out[3 * i + 1] = 1.0;
      out[3 * i + 2] = *jobs[i].flag ? 1.0 : 0.0;
    }
  } else if (is(l.name, "k_finish") && l.arg<int>(2) == 2) {
    double* out = l.arg<double*>(3);
    out[0] = script.residual();
    out[1] = 1.0;
    if (const unsigned* w = l.arg<const unsigned*>(4)) out[2] = *w;
    if (const unsigned* w = l.arg<const unsigned*>(5)) out[3] = *w;
  } else if (is(l.name, "k_pcg_init")) {
    const PcgDesc<double>* d = l.arg<const PcgDesc<double>*>(0);
    if (fake::valid(d, sizeof *d, l.stream, "descriptor")) {
      for (const void* p : {(const void*)d->K, (const void*)d->Dinv, (const void*)d->b,
                            (const void*)d->x, (const void*)d->r, (const void*)d->z,
                            (const void*)d->p[0], (const void*)d->p[1], (const void*)d->Ap})
        fake::valid(p, 4, l.stream, "operand of an iteration");
      *d->st = PcgState();
    }
  } else if (is(l.name, "k_scalar_rows")) {
    for (int i = 7; i < 10; ++i) fake::valid(l.arg<const void*>(i), 4, l.stream, "scalar view");
  } else if (is(l.name, "k_update_single")) {
    finish_state(l.arg<PcgState*>(7));
  } else if (is(l.name, "k_pcg_wg")) {
    const PcgDesc<double>* d = l.arg<const PcgDesc<double>*>(0);
    for (unsigned i = 0; i < l.grid.x; ++i)
      if (fake::valid(d[i].st, sizeof(PcgState), l.stream, "state")) finish_state(d[i].st);
  } else if (is(l.name, "k_gather_states")) {
    PcgState* const* st = l.arg<PcgState* const*>(0);
    PcgState* out = l.arg<PcgState*>(2);
    for (int i = 0; i < l.arg<int>(1); ++i)
      if (fake::valid(st[i], sizeof(PcgState), l.stream, "state")) {
        finish_state(st[i]);
        out[i] = *st[i];
      }
  }
}

// Device arrays of the check.
template <class T>
static T* device(int64_t n) {
  T* p = nullptr;
  hipMallocFromPoolAsync(reinterpret_cast<void**>(&p), sizeof(T) * (size_t)n,
                         reinterpret_cast<hipMemPool_t>((size_t)fake::state().device + 1), nullptr);
  return p;
}

struct Structure {
  int n;
  sso_mesh m{};
  double *load, *grad, *u;
  explicit Structure(int nodes, bool prescribed = false) : n(nodes) {
    m.n_nodes = n;
    m.xyz = device<double>(3 * n);
    m.fixed = device<uint8_t>(6 * n);
    m.f_nodal = device<double>(6 * n);
    if (prescribed) m.u_prescribed = device<double>(6 * n);
    load = device<double>(6 * n);
    grad = device<double>(3 * n);
    u = device<double>(6 * n);
  }
};

static sso_options options(int solver = SSO_SOLVER_AUTO, int precision = SSO_PREC_FP64) {
  sso_options o{};
  o.precision = precision;
  o.rtol = 1e-8;
  o.max_it = 1000;
  o.refine_steps = 20;
  o.solver = solver;
  return o;
}

static sso_problem* create(const Structure& s, const sso_options& o, hipStream_t stream = nullptr) {
  sso_problem* p = nullptr;
  // memory anew, and so zeroed: the pattern that no kernel builds is then one without blocks
  CHECK(sso_pool_trim(fake::state().device, 0) == SSO_OK);
  CHECK(sso_problem_create(&s.m, &o, stream, &p) == SSO_OK && p);
  return p;
}

static void begin_check() {
  script = Script();
  fake::state().launches.clear();
  fake::state().fail = nullptr;
  fake::state().busy.clear();
  fake::state().limit.clear();
  fake::state().device = 0;
}

// ---- the checks ----------------------------------------------------------------------------

// A begun solve that ends before any launch took it has displacements of 0 and no factor: what
// follows it solves by PCG, and never with arrays that were not allocated.
static void ended_before_a_launch() {
  for (int precision : {SSO_PREC_FP64, SSO_PREC_MIXED})
    for (int nodes : {20, 400})
      for (bool prescribed : {false, true})
        for (bool listed : {false, true}) {
          begin_check();
          Structure s(nodes, prescribed);
          sso_problem* p = create(s, options(SSO_SOLVER_AUTO, precision));
          CHECK(sso_solve_begin(p) == SSO_OK);
          if (listed) {        // in a call that asks for no iterations
            sso_batch* b = nullptr;
            int32_t done = 1;
            CHECK(sso_batch_create(nullptr, &b) == SSO_OK);
            CHECK(sso_batch_iterate(b, &p, 1, 0, &done) == SSO_OK && done == 0);
            sso_batch_destroy(b);
          }
          sso_stats st;
          CHECK(sso_solve_end(p, s.u, &st) == SSO_ENOTCONV);
          CHECK(sso_adjoint(p, SSO_OBJ_LINEAR, s.load, s.grad, nullptr, nullptr, &st) == SSO_OK);
          CHECK(sso_adjoint(p, SSO_OBJ_USER, s.load, s.grad, nullptr, nullptr, &st) == SSO_OK);
          CHECK(sso_adjoint(p, SSO_OBJ_COMPLIANCE, nullptr, s.grad, nullptr, nullptr, &st) == SSO_OK);
          double out[3];
          CHECK(sso_size_objective(p, 1.0, 1.0, 0.1, out, s.grad, nullptr, &st) == SSO_OK);
          int64_t before = 0, after = 0;
          CHECK(sso_problem_bytes(p, &before) == SSO_OK);
          const int taken = fake::state().allocations[0];
          CHECK(sso_size_objective_noalloc(p, 1.0, 1.0, 0.1, out, s.grad, nullptr, &st) == SSO_OK);
          CHECK(sso_problem_bytes(p, &after) == SSO_OK && after == before &&
                taken == fake::state().allocations[0]);
          CHECK(launches("k_front_") == 0);
          // and a solve of its own is direct as ever
          CHECK(sso_solve(p, s.u, &st) == SSO_OK && st.solver == SSO_SOLVER_AUTO);
          CHECK(launches("k_front_first") > 0);
          sso_problem_destroy(p);
        }
}

// A begun mixed-precision solve runs the recurrences that its options name, whatever the problem ran
// before.
static void mixed_recurrences_named_anew() {
  for (int second : {SSO_SOLVER_STANDARD, SSO_SOLVER_FUSED}) {
    begin_check();
    Structure s(400);
    sso_options o = options(SSO_SOLVER_FUSED, SSO_PREC_MIXED);
    o.max_it = 8;
    o.refine_steps = 1;
    sso_problem* p = create(s, o);
    script.rr = {1.0, 1.0};            // of x = 0, and of the outer step's direction
    CHECK(sso_solve(p, s.u, nullptr) == SSO_ENOTCONV);
    o.solver = second;
    CHECK(sso_set_options(p, &o) == SSO_OK);
    script = Script();
    script.rr = {1.0, 1.0};
    CHECK(sso_solve_begin(p) == SSO_OK);
    sso_batch* b = nullptr;
    int32_t done = 0;
    CHECK(sso_batch_create(nullptr, &b) == SSO_OK);
    CHECK(sso_batch_iterate(b, &p, 1, 4, &done) == SSO_OK && done == 1);
    sso_stats st;
    CHECK(sso_solve_end(p, s.u, &st) == SSO_ENOTCONV && st.solver == second);
    sso_batch_destroy(b);
    sso_problem_destroy(p);
  }
}

// One call with iterations enough brings a begun solve to its end, whatever it takes: a plan still in
// the making, refinement, a factorisation that fails.
static void one_call_ends_a_solve() {
  struct {
    std::vector<double> rr;    // after each step
    bool singular;
    int substitutions;         // forward sweeps of the lowest level
    int solver;
  } cases[] = {
      {{1e-18}, false, 1, SSO_SOLVER_AUTO},                     // met at once
      {{1e-10, 1e-18}, false, 2, SSO_SOLVER_AUTO},              // one refinement
      {{1e-4, 1e-8, 1e-12, 1e-15, 1e-18}, false, 5, SSO_SOLVER_AUTO},
      {{1e-10, 0.9e-10, 0.9e-10, 0.0}, false, 2, SSO_SOLVER_AUTO},   // stuck: PCG corrects
      {{1.0}, true, 1, SSO_SOLVER_STANDARD},                    // a pivot too small: PCG
  };
  for (int precision : {SSO_PREC_FP64, SSO_PREC_MIXED})
    for (int nodes : {400, 20000})         // the larger plan is not there when the call is made
      for (const auto& c : cases) {
        begin_check();
        Structure s(nodes);
        sso_problem* p = create(s, options(SSO_SOLVER_AUTO, precision));
        script.rr = c.rr;
        script.singular = c.singular;
        CHECK(sso_solve_begin(p) == SSO_OK);
        sso_batch* b = nullptr;
        CHECK(sso_batch_create(nullptr, &b) == SSO_OK);
        int32_t done = 0;
        CHECK(sso_batch_iterate(b, &p, 1, 1000, &done) == SSO_OK && done == 1);
        CHECK(launches("k_front_first") > 0);
        sso_stats st;
        CHECK(sso_solve_end(p, s.u, &st) == SSO_OK && st.solver == c.solver);
        CHECK(launches("k_correct_many") == c.substitutions - 1);
        sso_batch_destroy(b);
        sso_problem_destroy(p);
      }
}

// A call gives each problem the iterations asked for and no more: one is one step.
static void iterations_are_steps() {
  begin_check();
  Structure s(400);
  sso_problem* p = create(s, options());
  script.rr = {1e-4, 1e-8, 1e-12, 1e-18};
  CHECK(sso_solve_begin(p) == SSO_OK);
  sso_batch* b = nullptr;
  CHECK(sso_batch_create(nullptr, &b) == SSO_OK);
  int32_t done = 1;
  for (int k = 0; k < 2; ++k) {
    CHECK(sso_batch_iterate(b, &p, 1, 1, &done) == SSO_OK && done == 0);
    CHECK(launches("k_correct_many") == k);
  }
  CHECK(sso_batch_iterate(b, &p, 1, 2, &done) == SSO_OK && done == 1);
  CHECK(launches("k_correct_many") == 3);
  CHECK(sso_batch_iterate(b, &p, 1, 2, &done) == SSO_OK && done == 1);
  CHECK(launches("k_correct_many") == 3);
  CHECK(sso_solve_end(p, s.u, nullptr) == SSO_OK);
  sso_batch_destroy(b);
  sso_problem_destroy(p);
}

// Several problems: those whose plans are there are launched at once, the others follow within the
// call; problems that iterate by PCG are in the first launch.
static void a_call_with_several() {
  begin_check();
  Structure large(30000), small(300), other(300);
  sso_options o = options();
  sso_problem* ps[3] = {create(large, o), create(small, o), nullptr};
  o.solver = SSO_SOLVER_STANDARD;
  ps[2] = create(other, o);
  for (sso_problem* p : ps) CHECK(sso_solve_begin(p) == SSO_OK);
  int32_t ready[3] = {2, 2, 2}, done[3] = {0, 0, 0};
  for (int i = 0; i < 3; ++i)
    CHECK(sso_solve_ready(ps[i], &ready[i]) == SSO_OK && (ready[i] == 0 || ready[i] == 1));
  CHECK(ready[2] == 1);
  sso_batch* b = nullptr;
  CHECK(sso_batch_create(nullptr, &b) == SSO_OK);
  CHECK(sso_batch_iterate(b, ps, 3, 1000, done) == SSO_OK && done[0] && done[1] && done[2]);
  for (int i = 0; i < 3; ++i) {
    sso_stats st;
    CHECK(sso_solve_ready(ps[i], &ready[i]) == SSO_OK && ready[i] == 1);
    CHECK(sso_solve_end(ps[i], nullptr, &st) == SSO_OK);
    CHECK(st.solver == (i == 2 ? SSO_SOLVER_STANDARD : SSO_SOLVER_AUTO));
    CHECK(sso_solve_ready(ps[i], &ready[i]) == SSO_EINVAL);      // no longer begun
  }
  CHECK(sso_solve_ready(nullptr, ready) == SSO_EINVAL);
  sso_batch_destroy(b);
  for (sso_problem* p : ps) sso_problem_destroy(p);
}

// An allocation that fails in a call leaves nothing that the next call takes for complete.
static void allocations_that_fail() {
  const std::vector<std::function<int(sso_problem*, const Structure&)>> calls = {
      [](sso_problem* p, const Structure& s) { return sso_solve(p, s.u, nullptr); },
      [](sso_problem* p, const Structure& s) {
        double out[3];
        const int st = sso_solve(p, s.u, nullptr);
        return st != SSO_OK ? st : sso_size_objective(p, 1.0, 1.0, 0.1, out, s.grad, nullptr, nullptr);
      },
      [](sso_problem* p, const Structure& s) {
        const int st = sso_solve(p, s.u, nullptr);
        return st != SSO_OK ? st : sso_adjoint(p, SSO_OBJ_LINEAR, s.load, s.grad, nullptr, nullptr, nullptr);
      },
      [](sso_problem* p, const Structure&) {
        const int32_t *a, *b, *c, *d;
        int64_t e, f;
        return sso_pattern(p, &a, &b, &c, &d, &e, &f);
      },
      [](sso_problem* p, const Structure& s) {
        sso_batch* b = nullptr;
        int32_t done = 0;
        int st = sso_batch_create(nullptr, &b);
        for (int again = 0; again < 3; ++again) {     // the same launch tables, again after a failure
          st = sso_solve_begin(p);
          while (st == SSO_OK && !done) st = sso_batch_iterate(b, &p, 1, 8, &done);
          if (st == SSO_OK) break;
        }
        sso_batch_destroy(b);
        return st != SSO_OK ? st : sso_solve_end(p, s.u, nullptr);
      },
  };
  for (size_t c = 0; c < calls.size(); ++c)
    for (int solver = SSO_SOLVER_AUTO; solver <= SSO_SOLVER_WG; ++solver)
      for (int precision : {SSO_PREC_FP64, SSO_PREC_MIXED}) {
        if (solver == SSO_SOLVER_WG && precision == SSO_PREC_MIXED) continue;
        for (int k = 0, failed = 1; failed && k < 200; ++k) {
          begin_check();
          Structure s(solver == SSO_SOLVER_WG ? 130 : 24000);   // buffers of their own
          sso_options o = options(SSO_SOLVER_STANDARD), named = options(solver, precision);
          o.max_it = named.max_it = 8;
          sso_problem* p = create(s, o);
          CHECK(sso_set_options(p, &named) == SSO_OK);   // what it needs is allocated by the call
          int n = 0;
          script.rr.assign(40, 1.0);       // far from met: inner solves and corrections run
          fake::state().fail = [&](const char* what) {
            return std::strcmp(what, "copy") && n++ >= k ? hipErrorOutOfMemory : hipSuccess;
          };
          const int st = calls[c](p, s);
          fake::state().fail = nullptr;
          failed = n > k;
          if (!failed) CHECK(st == SSO_OK || st == SSO_ENOTCONV);
          script = Script();
          script.rr.assign(40, 1.0);
          CHECK(calls[c](p, s) != SSO_EHIP);
          sso_problem_destroy(p);
          if (fake::state().faults) {
            std::printf("call %zu solver %d precision %d allocation %d\n", c, solver, precision, k);
            return;
          }
        }
      }
}

// A launch that fails at any of its calls leaves nothing running, and the problems where a later
// call takes them to their end; a correction is never added again.
static void launches_that_fail() {
  for (int steps : {1, 2}) {            // the failing launch factors, or refines
    for (int k = 0, failed = 1; failed && k < 500; ++k) {
      begin_check();
      Structure s(400), t(300), w(100);
      sso_options o = options();
      sso_problem* ps[3] = {create(s, o), nullptr, nullptr};
      o.solver = SSO_SOLVER_STANDARD;
      ps[1] = create(t, o);
      o.solver = SSO_SOLVER_WG;
      ps[2] = create(w, o);
      int32_t done[3] = {0, 0, 0}, ready = 0;
      for (sso_problem* p : ps) CHECK(sso_solve_begin(p) == SSO_OK);
      while (!ready) CHECK(sso_solve_ready(ps[0], &ready) == SSO_OK);
      script.rr.assign(20, 1e-10);
      sso_batch* b = nullptr;
      CHECK(sso_batch_create(nullptr, &b) == SSO_OK);
      if (steps == 2) CHECK(sso_batch_iterate(b, ps, 1, 1, done) == SSO_OK && !done[0]);
      int calls = 0;
      fake::state().busy.clear();
      fake::state().fail = [&](const char*) { return calls++ >= k ? hipErrorOutOfMemory : hipSuccess; };
      int st = sso_batch_launch(b, ps, 3, 1);
      fake::state().fail = nullptr;
      failed = calls > k;
      if (failed && st != SSO_OK) {
        for (const auto& q : fake::state().busy) CHECK(!q.second);
      } else {
        CHECK(st == SSO_OK);            // or it did without: PCG in place of the direct solver
        CHECK(sso_batch_wait(b, ps, 3, done) == SSO_OK);
      }
      const int added = launches("k_correct_many"), factored = launches("k_front_first");
      script = Script();                // the next residual is met
      CHECK(sso_batch_iterate(b, ps, 3, 1000, done) == SSO_OK && done[0] && done[1] && done[2]);
      // a correction that may have been added is not added again: x is solved for anew
      if (failed && st != SSO_OK && steps == 2 && added > 0)
        CHECK(launches("k_front_first") > factored && launches("k_correct_many") == added);
      for (sso_problem* p : ps) CHECK(sso_solve_end(p, nullptr, nullptr) == SSO_OK);
      sso_batch_destroy(b);
      for (sso_problem* p : ps) sso_problem_destroy(p);
      if (!failed) CHECK(k > 5);
    }
  }
}

// The null stream is the current device's: a problem that ends while another device is current is
// waited for on its own, and its memory goes to no other device's problems.
static void ended_on_another_device() {
  begin_check();
  auto& hip = fake::state();
  for (int pass = 0; pass < 2; ++pass)
    for (int device : {1, 0}) {
      hip.device = device;
      Structure s(20000);
      sso_options o = options(pass ? SSO_SOLVER_STANDARD : SSO_SOLVER_AUTO);
      sso_problem* p = nullptr;          // from the memory that earlier problems left, zeroed
      for (const auto& m : hip.device_memory) std::memset(m.first, 0, m.second.bytes);
      CHECK(sso_problem_create(&s.m, &o, nullptr, &p) == SSO_OK);
      hip.device = 1 - device;
      hip.waited.clear();
      sso_problem_destroy(p);
      CHECK(hip.device == 1 - device);
      CHECK(!hip.waited.empty());
      for (int d : hip.waited) CHECK(d == device);
    }
  hip.device = 0;
}

// Host memory that is too short for the elimination's plan leaves the problem to PCG.
static void no_host_memory_for_a_plan() {
  for (bool late : {false, true})        // the solver named at first, so that the solve plans
    for (int begun : {0, 1}) {
      begin_check();
      Structure s(60000);
      sso_options o = options(late ? SSO_SOLVER_STANDARD : SSO_SOLVER_AUTO);
      CHECK(sso_pool_trim(0, 0) == SSO_OK);
      refuse_from = 200000;              // the pattern's row pointers are 240 kB
      sso_problem* p = nullptr;
      CHECK(sso_problem_create(&s.m, &o, nullptr, &p) == SSO_OK && p);
      o.solver = SSO_SOLVER_AUTO;
      CHECK(sso_set_options(p, &o) == SSO_OK);
      sso_stats st{};
      if (begun) {
        sso_batch* b = nullptr;
        int32_t done = 0;
        CHECK(sso_solve_begin(p) == SSO_OK);
        CHECK(sso_batch_create(nullptr, &b) == SSO_OK);
        CHECK(sso_batch_iterate(b, &p, 1, 8, &done) == SSO_OK && done);
        sso_batch_destroy(b);
        CHECK(sso_solve_end(p, s.u, &st) == SSO_OK);
      } else {
        CHECK(sso_solve(p, s.u, &st) == SSO_OK);
      }
      CHECK(st.solver == SSO_SOLVER_STANDARD && launches("k_front_") == 0);
      refuse_from = 0;
      sso_problem_destroy(p);
    }
}

// The direct solver's arrays leave an eighth of the device's memory to those who come later: problems
// that are created and kept go on by PCG from there, and their own later calls find memory.
static void memory_left_for_others() {
  begin_check();
  CHECK(sso_pool_trim(0, 0) == SSO_OK);
  Structure s(20000);
  size_t left = 0, total = 0;
  fake::state().limit[0] = (size_t)640 << 20;
  std::vector<sso_problem*> ps;
  int direct = 0;
  for (int k = 0; k < 12; ++k) {
    sso_stats st{};
    sso_problem* p = create(s, options());
    if (!p) break;
    ps.push_back(p);
    CHECK(sso_solve(p, s.u, &st) == SSO_OK);
    direct += st.solver == SSO_SOLVER_AUTO;
    hipMemGetInfo(&left, &total);
    if (st.solver == SSO_SOLVER_AUTO) CHECK(left >= total / 8);
    double out[3];
    CHECK(sso_size_objective(p, 1.0, 1.0, 0.1, out, s.grad, nullptr, nullptr) == SSO_OK);
  }
  CHECK(ps.size() == 12 && direct >= 1 && direct < 12);
  for (sso_problem* p : ps) sso_problem_destroy(p);
  // memory that ended problems left counts as free
  sso_stats st{};
  sso_problem* p = nullptr;
  for (const auto& m : fake::state().device_memory) std::memset(m.first, 0, m.second.bytes);
  sso_options o = options();
  CHECK(sso_problem_create(&s.m, &o, nullptr, &p) == SSO_OK);
  CHECK(sso_solve(p, s.u, &st) == SSO_OK && st.solver == SSO_SOLVER_AUTO);
  sso_problem_destroy(p);
}

int main(int argc, char** argv) {
  fake::state().kernel = kernel;
  const std::map<std::string, void (*)()> checks = {
      {"ended_before_a_launch", ended_before_a_launch},
      {"ended_on_another_device", ended_on_another_device},
      {"mixed_recurrences_named_anew", mixed_recurrences_named_anew},
      {"one_call_ends_a_solve", one_call_ends_a_solve},
      {"iterations_are_steps", iterations_are_steps},
      {"a_call_with_several", a_call_with_several},
      {"allocations_that_fail", allocations_that_fail},
      {"launches_that_fail", launches_that_fail},
      {"memory_left_for_others", memory_left_for_others},
      {"no_host_memory_for_a_plan", no_host_memory_for_a_plan},
  };
  for (const auto& c : checks)
    if (argc < 2 || c.first == argv[1]) c.second();
  CHECK(argc < 2 || checks.count(argv[1]));
  CHECK(fake::state().faults == 0);
  std::printf("%s (%d failures)\n", failures ? "failed" : "ok", failures);
  std::fflush(stdout);
  std::_Exit(failures ? 1 : 0);
}

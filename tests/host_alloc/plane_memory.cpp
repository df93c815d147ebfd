// The plane pass's own memory (reordered Green's tables, half spectra) is optional: whatever
// a plan can run without it on a device, it runs on that device with it.  For every kind of call,
// precision and boundary condition, the bytes that a plan made without the pass holds after the
// call are the limit (and limits up to what the whole plan holds): the whole plan must then
// succeed too, hold no more than the limit, and give back what it holds.  Below the limit the call
// fails and may be repeated; nothing leaks.  Calls that never take the pass (FP64 PCG) allocate
// nothing for it beyond the plan's tables, and a server of FP64 solves nothing at all.  Exit
// status 0 = pass.
#include <cstdio>
#include <functional>
#include <vector>

#include "fake_hip.h"
#include "gps.h"

namespace gps {
gps_status compact_plan_create(int nx, int ny, int nz, double h, int bc, gps_plan** out);
gps_status compact_plan_footprint(int nx, int ny, int nz, int bc, int precision, int maxit,
                                  int nonlinear_pb, int refine, size_t* tables, size_t* buffers,
                                  size_t* transient);
gps_status batch_open(gps_plan* pl, int nslots, int check_neutral);
}  // namespace gps

static int failures = 0, checks = 0;
#define EXPECT(cond, ...)                                            \
  do {                                                               \
    ++checks;                                                        \
    if (!(cond)) {                                                   \
      std::fprintf(stderr, "FAILED %s:%d: %s: ", __FILE__, __LINE__, #cond); \
      std::fprintf(stderr, __VA_ARGS__);                             \
      std::fprintf(stderr, "\n");                                    \
      ++failures;                                                    \
    }                                                                \
  } while (0)

constexpr int N = 16;
static std::vector<double> rho(N* N* N, 0.0), eps(N* N* N, 1.0), phi(N* N* N);

using Call = std::function<gps_status(gps_plan*)>;
struct Kind {
  const char* name;
  int precision;
  bool plane;                  // runs as x, plane, x where the device has room
  int refine;
  Call call;
};

static gps_plan* make(int bc, const Kind& k, bool compact) {
  gps_plan* p = nullptr;
  const gps_status st = compact ? gps::compact_plan_create(N, N, N, 0.5, bc, &p)
                                : gps_plan_create(N, N, N, 0.5, bc, &p);
  EXPECT(st == GPS_OK, "create %d", st);
  gps_options o;
  gps_plan_get_options(p, &o);
  o.precision = k.precision;
  o.maxit = 20;
  o.refine_every = k.refine;
  EXPECT(gps_plan_set_options(p, &o) == GPS_OK, "options");
  return p;
}

static void run(int bc, const Kind& k) {
  fake::limit = ~size_t(0);
  gps_plan* p = make(bc, k, true);
  EXPECT(k.call(p) == GPS_OK, "%s bc %d: compact", k.name, bc);
  EXPECT(gps_plan_device_bytes(p) == fake::used, "%s bc %d: bytes", k.name, bc);
  const size_t least = fake::used;
  gps_plan_destroy(p);
  EXPECT(fake::used == 0, "%s bc %d: leak", k.name, bc);

  p = make(bc, k, false);
  fake::launches.clear();
  EXPECT(k.call(p) == GPS_OK, "%s bc %d: whole", k.name, bc);
  EXPECT((fake::count("k_plane") > fake::count("k_plane_table")) == k.plane, "%s bc %d: route",
         k.name, bc);
  EXPECT(gps_plan_device_bytes(p) == fake::used, "%s bc %d: bytes", k.name, bc);
  const size_t most = fake::used;
  EXPECT(most > least, "%s bc %d: whole plan's bytes", k.name, bc);
  if (k.precision == GPS_PREC_FP64 && !k.plane) {
    gps_plan* bare = nullptr;
    gps_plan* full = nullptr;
    gps::compact_plan_create(N, N, N, 0.5, bc, &bare);
    gps_plan_create(N, N, N, 0.5, bc, &full);
    const size_t tables = gps_plan_device_bytes(full) - gps_plan_device_bytes(bare);
    gps_plan_destroy(bare);
    gps_plan_destroy(full);
    EXPECT(most - least == tables, "%s bc %d: %zu bytes beside the tables", k.name, bc,
           most - least - tables);
  }
  gps_plan_destroy(p);

  for (int i = 0; i <= 8; ++i) {
    const size_t limit = least + (most - least) * i / 8;
    fake::limit = ~size_t(0);                    // (the plan's transient may exceed the limit)
    p = make(bc, k, false);
    fake::limit = limit;
    for (int j = 0; j < 2; ++j) {
      fake::launches.clear();
      EXPECT(k.call(p) == GPS_OK, "%s bc %d: limit %d of 8, call %d", k.name, bc, i, j);
      EXPECT(fake::used <= limit, "%s bc %d: %zu bytes above %zu", k.name, bc, fake::used, limit);
      EXPECT(gps_plan_device_bytes(p) == fake::used, "%s bc %d: bytes", k.name, bc);
      gps_plan_release_buffers(p);
    }
    gps_plan_destroy(p);
    EXPECT(fake::used == 0, "%s bc %d: leak", k.name, bc);
  }

  // below what the call needs: an error, twice, then as a fresh plan without the pass
  for (int i = 1; i <= 40; ++i) {
    fake::limit = ~size_t(0);
    p = make(bc, k, false);
    gps_plan* bare = make(bc, k, true);
    const size_t tables = gps_plan_device_bytes(bare);
    gps_plan_destroy(bare);
    fake::limit = tables + (least - tables) * i / 41;
    for (int j = 0; j < 2; ++j)
      EXPECT(k.call(p) == GPS_E_NOMEM, "%s bc %d: %d of 41, call %d", k.name, bc, i, j);
    EXPECT(gps_plan_device_bytes(p) == fake::used, "%s bc %d: bytes after an error", k.name, bc);
    fake::limit = ~size_t(0);
    EXPECT(k.call(p) == GPS_OK, "%s bc %d: %d of 41, then room", k.name, bc, i);
    EXPECT(fake::used == least, "%s bc %d: %d of 41: %zu bytes, not %zu", k.name, bc, i, fake::used,
           least);
    gps_plan_destroy(p);
    EXPECT(fake::used == 0, "%s bc %d: leak", k.name, bc);
  }
}

// A timed pass reports the bytes of the kernel that ran: the plane pass's where the solve
// takes it, else (refinement, a timed y pass, a plan without it) those of the three passes.
static void timed(int refine) {
  fake::limit = ~size_t(0);
  const Kind k{"timed", GPS_PREC_MIXED, true, refine, nullptr};
  for (int kind : {GPS_K_XFWD, GPS_K_YFWD, GPS_K_ZCONV, GPS_K_YINV, GPS_K_XINV}) {
    double bytes[2];
    bool planes[2];
    for (int compact = 0; compact < 2; ++compact) {
      gps_plan* p = make(GPS_BC_FREE, k, compact);
      EXPECT(gps_plan_set_timing(p, kind) == GPS_OK, "timing");
      fake::launches.clear();
      EXPECT(gps_solve_generalized(p, rho.data(), eps.data(), phi.data(), 1e-6) == GPS_OK, "timed");
      planes[compact] = fake::count("k_plane") > fake::count("k_plane_table");
      EXPECT(gps_plan_timing(p, nullptr, nullptr, &bytes[compact]) == GPS_OK, "timing");
      gps_plan_destroy(p);
    }
    const bool y = kind == GPS_K_YFWD || kind == GPS_K_YINV;
    EXPECT(!planes[1] && planes[0] == (!refine && !y), "kind %d, refine %d: route", kind, refine);
    const bool differs = planes[0] && (kind == GPS_K_ZCONV || kind == GPS_K_XINV);
    EXPECT((bytes[0] != bytes[1]) == differs && bytes[1] > 0.0, "kind %d, refine %d: bytes %g, %g",
           kind, refine, bytes[0], bytes[1]);
  }
}

// A solve that starts from the previous iterate may need no iteration at all, so few are
// queued before its first poll (every state that is read here says done): half a chunk, two
// chunks without an iterate to start from.
static void warm() {
  fake::limit = ~size_t(0);
  const Kind k{"warm", GPS_PREC_FP64, false, 0, nullptr};
  gps_plan* p = make(GPS_BC_FREE, k, false);
  gps_options o;
  gps_plan_get_options(p, &o);
  o.warm_start = 1;
  EXPECT(gps_plan_set_options(p, &o) == GPS_OK, "options");
  EXPECT(gps_plan_set_timing(p, GPS_K_YFWD) == GPS_OK, "timing");
  for (int call = 0; call < 3; ++call) {
    fake::launches.clear();
    EXPECT(gps_solve_generalized(p, rho.data(), eps.data(), phi.data(), 1e-6) == GPS_OK, "warm");
    const int queued = fake::count("k_fxfwdIdLi8ELi4ELi6ELi3E");   // XF_SOLVE_REF at length 32
    const int expect = call == 0 ? 2 * o.check_every : o.check_every / 2;
    EXPECT(queued == expect, "call %d: %d iterations before the first poll", call, queued);
  }
  gps_plan_destroy(p);
}

// A plan is made within the bytes that one without the pass needs at the most, and allocates
// nothing after it has freed its transient (the next plan then finds both blocks again).
static void create(int bc) {
  gps_plan* p = nullptr;
  fake::limit = ~size_t(0);
  fake::peak = 0;
  EXPECT(gps::compact_plan_create(N, N, N, 0.5, bc, &p) == GPS_OK, "bc %d", bc);
  gps_plan_destroy(p);
  const size_t least = fake::peak;
  fake::peak = 0;
  fake::frees = fake::late = 0;
  EXPECT(gps_plan_create(N, N, N, 0.5, bc, &p) == GPS_OK, "bc %d", bc);
  EXPECT(fake::late == 0, "bc %d: %d allocations after a free", bc, fake::late);
  gps_plan_destroy(p);
  const size_t most = fake::peak;
  EXPECT(most > least, "bc %d", bc);
  for (int i = 0; i <= 16; ++i) {
    fake::limit = least + (most - least) * i / 16;
    EXPECT(gps_plan_create(N, N, N, 0.5, bc, &p) == GPS_OK, "bc %d: limit %d of 16", bc, i);
    gps_plan_destroy(p);
    EXPECT(fake::used == 0, "bc %d: leak", bc);
    fake::limit = least * (i + 1) / 18;
    EXPECT(gps_plan_create(N, N, N, 0.5, bc, &p) == GPS_E_NOMEM, "bc %d: %d of 18", bc, i);
    EXPECT(p == nullptr && fake::used == 0, "bc %d: leak", bc);
  }
}

// An FP64 server whose budget holds two plans without the pass keeps both.
static void serve_fp64(int bc) {
  fake::limit = ~size_t(0);
  const int sizes[2] = {16, 18}, slots = 2;
  size_t budget = 0, transient = 0;
  for (int n : sizes) {
    size_t t = 0, b = 0, tr = 0;
    gps::compact_plan_footprint(n, n, n, bc, GPS_PREC_FP64, 20, 0, 0, &t, &b, &tr);
    budget += t + slots * b;
    transient = tr;                  // the second plan's: while it is made the first is resident
  }
  budget += transient;
  gps_server_options o{};
  o.budget_bytes = budget;
  o.max_active = 1;
  o.precision = GPS_PREC_FP64;
  o.fd_order = 16;
  o.maxit = 20;
  o.batch_slots = slots;
  gps_server* srv = nullptr;
  EXPECT(gps_server_create(&o, &srv) == GPS_OK, "server");
  std::vector<double> f(18 * 18 * 18, 0.0), e(f.size(), 1.0), u(f.size());
  for (int i = 0; i < 4; ++i) {
    const int n = sizes[i % 2];
    gps_request q{};
    q.nx = q.ny = q.nz = n;
    q.h = 0.5;
    q.bc = bc;
    q.rho = f.data();
    q.eps = e.data();
    q.phi = u.data();
    q.tol = 1e-6;
    long long t = 0;
    gps_result res{};
    EXPECT(gps_server_submit(srv, &q, &t) == GPS_OK, "submit bc %d, %d", bc, i);
    EXPECT(gps_server_wait(srv, t, &res) == GPS_OK && res.status == GPS_OK, "bc %d, %d", bc, i);
    EXPECT(res.plan_reused == (i >= 2), "bc %d: request %d made a plan again", bc, i);
  }
  gps_server_stats st{};
  gps_server_get_stats(srv, &st);
  EXPECT(st.plans_evicted == 0 && st.buffers_released == 0, "bc %d: %d evicted, %d released", bc,
         st.plans_evicted, st.buffers_released);
  EXPECT(st.bytes_peak <= budget, "bc %d: peak", bc);
  gps_server_destroy(srv);
  EXPECT(fake::used == 0, "bc %d: leak", bc);
}

int main() {
  const Call solve = [](gps_plan* p) {
    return gps_solve_generalized(p, rho.data(), eps.data(), phi.data(), 1e-6);
  };
  const Call vacuum = [](gps_plan* p) { return gps_solve_vacuum(p, rho.data(), phi.data()); };
  const Call sc = [](gps_plan* p) {
    return gps_solve_sc(p, rho.data(), eps.data(), phi.data(), 1e-6, GPS_METHOD_SC, 0.6);
  };
  const Call batch = [](gps_plan* p) { return gps::batch_open(p, 3, 0); };
  // a solve and then the polarization charge: the scratch field comes last
  const Call both = [](gps_plan* p) {
    const gps_status st = gps_solve_generalized(p, rho.data(), eps.data(), phi.data(), 1e-6);
    return st != GPS_OK ? st
                        : gps_polarization_charge(p, rho.data(), eps.data(), phi.data(), phi.data());
  };
  const Kind kinds[] = {
      {"solve mixed", GPS_PREC_MIXED, true, 0, solve},
      {"solve fp64", GPS_PREC_FP64, false, 0, solve},
      {"refined mixed", GPS_PREC_MIXED, false, 5, solve},
      {"vacuum mixed", GPS_PREC_MIXED, true, 0, vacuum},
      {"vacuum fp64", GPS_PREC_FP64, true, 0, vacuum},
      {"sc mixed", GPS_PREC_MIXED, true, 0, sc},
      {"sc fp64", GPS_PREC_FP64, true, 0, sc},
      {"batch mixed", GPS_PREC_MIXED, true, 0, batch},
      {"batch fp64", GPS_PREC_FP64, false, 0, batch},
      {"solve and polarization mixed", GPS_PREC_MIXED, true, 0, both},
  };
  for (int bc : {GPS_BC_FREE, GPS_BC_SURFACE, GPS_BC_PERIODIC, GPS_BC_WIRE})
    for (const Kind& k : kinds) {
      const bool periodic = bc == GPS_BC_PERIODIC;
      if (periodic && (k.refine > 0 || std::strncmp(k.name, "sc", 2) == 0)) continue;
      run(bc, k);
    }
  warm();
  timed(0);
  timed(5);
  for (int bc : {GPS_BC_FREE, GPS_BC_SURFACE, GPS_BC_PERIODIC, GPS_BC_WIRE}) {
    create(bc);
    serve_fp64(bc);
    size_t t0 = 0, b0 = 0, t1 = 0, b1 = 0;
    gps_plan_footprint(N, N, N, bc, GPS_PREC_FP64, 20, 0, 0, &t0, &b0, nullptr);
    gps::compact_plan_footprint(N, N, N, bc, GPS_PREC_FP64, 20, 0, 0, &t1, &b1, nullptr);
    EXPECT(b0 == b1 && t0 > t1, "bc %d: FP64 footprint", bc);
  }
  std::printf("plane memory: %d checks, %d failures\n", checks, failures);
  return failures == 0 ? 0 : 1;
}

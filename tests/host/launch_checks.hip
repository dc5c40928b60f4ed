// Launches of libuot without a GPU: the library's host code linked against
// the recording HIP runtime below, which runs no kernel.
//   launch_checks lines    solves, half-steps and objectives over lengths of lines
//   launch_checks planes   solves over the planes that one block may hold
//   launch_checks barycenters   ... over the rows of several fields that it may hold
//   launch_checks instances     solves of 1-D grids and planes at every segment length
// print the largest dynamic LDS that each kernel was launched with;
//   launch_checks routes   the pass kernels of solves on either side of the rules
//   launch_checks slices   the tap slices of lines
//   launch_checks failing   a launch that fails is reported by its own call and
//                           leaves no error behind
// Built host-only (tests/test_line_launches_cpu.py).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "uot.h"

// ---------------------------------------------------------------------------
// the recording runtime
// ---------------------------------------------------------------------------
namespace {
struct Seen {
  size_t lds = 0;
  std::string shape;
  dim3 grid;               // of its last launch
};
std::map<const void*, Seen> g_seen;
std::string g_shape;          // what the driver is running
long g_launches = 0;          // launches so far
long g_fail_at = -1;          // the launch that fails
hipError_t g_last = hipSuccess;
dim3 g_grid, g_block;
size_t g_lds;
char g_handle[64];            // every stream, event and graph
}  // namespace

extern "C" {
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t) {
  g_grid = g;
  g_block = b;
  g_lds = lds;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = g_grid;
  *b = g_block;
  *lds = g_lds;
  *s = nullptr;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void**, size_t lds, hipStream_t) {
  Seen& s = g_seen[f];
  s.grid = grid;
  if (lds > s.lds || s.shape.empty()) {
    s.lds = lds;
    s.shape = g_shape;
  }
  if (g_launches++ == g_fail_at) return g_last = hipErrorInvalidConfiguration;
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "recorded error"; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = g_handle; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 4; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)g_handle; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { *g = (hipGraph_t)g_handle; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *e = (hipGraphExec_t)g_handle;
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)g_handle; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
// (what comes back from the device is zero but for its first word, the stop flag of a control block)
hipError_t hipMemcpy(void* d, const void*, size_t n, hipMemcpyKind k) {
  if (k == hipMemcpyDeviceToHost) {
    std::memset(d, 0, n);
    if (n >= 4) static_cast<char*>(d)[0] = 1;
  }
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
}

// ---------------------------------------------------------------------------
// the driver
// ---------------------------------------------------------------------------
static int failures = 0;
#define EXPECT(cond)                                                                                              \
  do {                                                                                                            \
    if (!(cond)) {                                                                                                \
      std::fprintf(stderr, "FAILED %s:%d: %s (%s; %s)\n", __FILE__, __LINE__, #cond, uot_last_error(), g_shape.c_str()); \
      ++failures;                                                                                                 \
    }                                                                                                             \
  } while (0)

static void* const kDev = reinterpret_cast<void*>(0x10000);   // never dereferenced on the host
static uot_ctx* ctx;

static uot_geom grid(int dim, int64_t a, int64_t b, int64_t c) {
  uot_geom g;
  std::memset(&g, 0, sizeof(g));
  g.kind = UOT_GEOM_GRID;
  g.dim = dim;
  const int64_t n[3] = {a, b, c};
  for (int k = 0; k < dim; ++k) {
    g.n[k] = n[k];
    g.h[k] = 1.0 / 64;
  }
  return g;
}
static uot_problem problem(int dtype, const uot_geom& g) {
  uot_problem pb;
  std::memset(&pb, 0, sizeof(pb));
  pb.dtype = dtype;
  pb.geom = g;
  pb.p = pb.q = pb.dx = pb.dy = kDev;
  pb.F1.kind = pb.F2.kind = UOT_DIV_KL;
  pb.F1.lambda = pb.F2.lambda = 0.1;
  return pb;
}
// c = h^2 log2(e) / eps of those grids
static uot_params params(double c) {
  uot_params pr;
  std::memset(&pr, 0, sizeof(pr));
  pr.eps = 1.4426950408889634 / (64.0 * 64.0 * c);
  pr.max_iter = 1;
  pr.check_every = 2;
  return pr;
}
static void note(const char* what, int dtype, const uot_geom& g, int nb, double c) {
  char s[160];
  std::snprintf(s, sizeof(s), "%s f%d %lldx%lldx%lld fields %d c %g", what, dtype == UOT_F32 ? 32 : 64, (long long)g.n[0],
                (long long)g.n[1], (long long)g.n[2], nb, c);
  g_shape = s;
}
static void solve(int dtype, const uot_geom& g, int nb, double c) {
  note("solve", dtype, g, nb, c);
  uot_problem pb = problem(dtype, g);
  uot_params pr = params(c);
  uot_result res;
  size_t n = 0;
  if (nb == 1) {
    EXPECT(uot_workspace_size(&pb, &n) == UOT_OK);
    EXPECT(uot_solve(ctx, &pb, &pr, kDev, kDev, kDev, n, &res) == UOT_OK);
  } else {
    EXPECT(uot_fields_workspace_size(&pb, nb, &n) == UOT_OK);
    EXPECT(uot_solve_fields(ctx, &pb, nb, &pr, kDev, kDev, kDev, n, &res) == UOT_OK);
  }
}
static void barycenter(int dtype, const uot_geom& g, int nb, double c, int kind = UOT_DIV_KL, double alpha2 = 0.0) {
  note(kind == UOT_DIV_KL ? "barycentre KL" : kind == UOT_DIV_TV ? "barycentre TV" : "barycentre RG", dtype, g, nb, c);
  static const std::vector<double> alpha(64, 1.0);
  uot_bary_problem bp;
  std::memset(&bp, 0, sizeof(bp));
  bp.dtype = dtype;
  bp.n = nb;
  bp.geom = g;
  bp.p = bp.dx = bp.dy = kDev;
  bp.alpha = alpha.data();
  bp.F1.kind = bp.F2.kind = UOT_DIV_KL;
  bp.F1.lambda = bp.F2.lambda = 0.1;
  bp.F2.kind = kind;
  bp.F2.alpha = alpha2;
  bp.F2.beta = 1.3;
  uot_params pr = params(c);
  uot_result res;
  size_t n = 0;
  EXPECT(uot_bary_workspace_size(&bp, &n) == UOT_OK);
  EXPECT(uot_barycenter(ctx, &bp, &pr, kDev, kDev, kDev, kDev, n, &res) == UOT_OK);
}
static void one_pass(int dtype, const uot_geom& g, double c) {
  note("half-step and objective", dtype, g, 1, c);
  uot_problem pb = problem(dtype, g);
  const double eps = params(c).eps;
  size_t n = 0;
  double r = 0;
  uot_objective_values o;
  EXPECT(uot_workspace_size(&pb, &n) == UOT_OK);
  EXPECT(uot_half_step(ctx, &pb, eps, 0, kDev, kDev, kDev, &r, kDev, n) == UOT_OK);
  EXPECT(uot_objective(ctx, &pb, eps, kDev, kDev, nullptr, nullptr, &o, kDev, n) == UOT_OK);
}

// the kernels of a host-only build: what a launch names, and the kernel's symbol
struct OffloadEntry {
  uint64_t reserved;
  uint16_t version, kind;
  uint32_t flags;
  const void* address;
  const char* name;
  uint64_t size, data;
  void* aux;
};
extern "C" {
extern const OffloadEntry __start_llvm_offload_entries[], __stop_llvm_offload_entries[];
}

// what the shapes below were launched with
static void print_lds() {
  for (const OffloadEntry* e = __start_llvm_offload_entries; e != __stop_llvm_offload_entries; ++e) {
    const auto s = g_seen.find(e->address);
    if (s != g_seen.end()) std::printf("%s %zu %s\n", e->name, s->second.lds, s->second.shape.c_str());
  }
}

// the longest segments, and shorter ones
static const double kC[] = {0.01, 0.3};

// lines along either axis, few and many
static void lines() {
  for (int dt : {UOT_F32, UOT_F64})
    for (double c : kC)
      for (int64_t n = 1; n <= 4096; n += n < 1100 ? 1 : 7) {
        for (int64_t m : {3, 600}) {
          solve(dt, grid(2, n, m, 0), 1, c);
          solve(dt, grid(2, m, n, 0), 1, c);
        }
        solve(dt, grid(1, n, 0, 0), 1, c);
        one_pass(dt, grid(1, n, 0, 0), c);
        one_pass(dt, grid(2, 3, n, 0), c);
        one_pass(dt, grid(3, n, 5, 2), c);
      }
}

// planes of up to 4096 cells and somewhat more, one per block, few blocks and many
static void planes() {
  for (int dt : {UOT_F32, UOT_F64})
    for (double c : kC)
      for (int64_t a = 1; a <= 4096; ++a)
        for (int64_t b = 1; a * b <= 4200 && b <= 4096; ++b) {
          solve(dt, grid(3, 2, a, b), 1, c);
          if (a * b <= 1024) solve(dt, grid(3, 2, a, b), 200, c);
        }
}

// 1-D grids and planes under every segment length
static void instances() {
  for (int dt : {UOT_F32, UOT_F64})
    for (double c : {0.01, 0.1, 0.3, 0.7, 1.5, 3.0}) {
      for (int64_t n = 1; n <= 800; ++n) solve(dt, grid(1, n, 0, 0), 1, c);
      for (int64_t a = 1; a <= 256; ++a)
        for (int64_t b = 1; a * b <= 4096 && b <= 256; ++b)
          for (int m : {2, 400}) solve(dt, grid(3, m, a, b), 1, c);
    }
}

// barycentres, a row of every field in one block
static void barycenters() {
  for (int dt : {UOT_F32, UOT_F64})
    for (double c : kC)
      for (int nb = 1; nb <= 64; ++nb)
        for (int64_t n = 1; nb * n <= 4200 && n <= 4096; ++n) {
          barycenter(dt, grid(2, 3, n, 0), nb, c);
          if (nb * n <= 1024) barycenter(dt, grid(2, 400, n, 0), nb, c);
        }
}

// every launch of a call fails in turn
template <typename F> static void each_launch_fails(const char* what, F&& call) {
  g_shape = what;
  g_launches = 0;
  g_fail_at = -1;
  EXPECT(call() == UOT_OK && hipGetLastError() == hipSuccess);
  const long n = g_launches;
  EXPECT(n > 0);
  for (long k = 0; k < n; ++k) {
    g_shape = std::string(what) + ", launch " + std::to_string(k) + " of " + std::to_string(n);
    g_launches = 0;
    g_fail_at = k;
    EXPECT(call() == UOT_E_HIP);
    EXPECT(hipGetLastError() == hipSuccess);
    g_fail_at = -1;
    EXPECT(call() == UOT_OK);   // the context still works
  }
}

static void failing() {
  const uot_geom shapes[] = {grid(1, 100, 0, 0), grid(1, 3000, 0, 0), grid(2, 40, 50, 0), grid(3, 6, 20, 30)};
  uot_result res;
  for (int dt : {UOT_F32, UOT_F64})
    for (const uot_geom& g : shapes)
      for (int graph : {0, 1}) {
        uot_problem pb = problem(dt, g);
        uot_params pr = params(0.01);
        pr.use_graph = graph;
        size_t n = 0;
        EXPECT(uot_workspace_size(&pb, &n) == UOT_OK);
        each_launch_fails("solve", [&] { return uot_solve(ctx, &pb, &pr, kDev, kDev, kDev, n, &res); });
        each_launch_fails("asynchronous solve", [&] {
          const int rc = uot_solve_async(ctx, &pb, &pr, kDev, kDev, kDev, n);
          return rc ? rc : uot_sync_result(ctx, &res);
        });
      }
}

// the pass kernels a call launches
template <typename Call> static void route(Call&& call) {
  g_seen.clear();
  call();
  std::printf("route %s:", g_shape.c_str());
  for (const OffloadEntry* e = __start_llvm_offload_entries; e != __stop_llvm_offload_entries; ++e)
    if (g_seen.count(e->address) && (std::strstr(e->name, "k_line") || std::strstr(e->name, "k_plane") || std::strstr(e->name, "k_grid") ||
                                      std::strstr(e->name, "k_gtab")))
      std::printf(" %s", e->name);
  std::printf("\n");
}
static void routes() {
  for (int dt : {UOT_F32, UOT_F64})
    for (const uot_geom& g : {grid(2, 8, 512, 0), grid(2, 8, 2048, 0), grid(2, 200, 2048, 0), grid(2, 2048, 8, 0), grid(2, 8, 2050, 0),
                              grid(2, 2050, 8, 0), grid(3, 8, 32, 32), grid(3, 8, 64, 64), grid(3, 8, 16, 256), grid(3, 8, 80, 80),
                              grid(3, 30, 80, 80)})
      route([&] { solve(dt, g, 1, 0.01); });
  for (int dt : {UOT_F32, UOT_F64})
    for (int n : {40, 500, 1000})
      route([&] { solve(dt, grid(1, n, 0, 0), 1, 0.01); });
  for (int dt : {UOT_F32, UOT_F64})
    for (int n : {40, 500, 1000}) {
      const uot_geom g = grid(1, n, 0, 0);
      uot_problem pb = problem(dt, g);
      const double eps = params(0.01).eps;
      size_t wsb = 0;
      double r = 0, ms[3];
      int nk = 0;
      EXPECT(uot_workspace_size(&pb, &wsb) == UOT_OK);
      note("half-step", dt, g, 1, 0.01);
      route([&] { EXPECT(uot_half_step(ctx, &pb, eps, 0, kDev, kDev, kDev, &r, kDev, wsb) == UOT_OK); });
      note("timed", dt, g, 1, 0.01);
      route([&] { EXPECT(uot_time_half_step(ctx, &pb, eps, kDev, 1, ms, &nk, kDev, wsb, 0) == UOT_OK && nk == 1); });
    }
  const int bary[][3] = {{2, 64, 64}, {8, 50, 50}, {10, 80, 80}, {10, 81, 81}, {10, 150, 150}, {12, 48, 48}, {16, 64, 64},
                         {20, 50, 50}, {24, 20, 40}, {24, 96, 96}, {30, 64, 64}, {33, 40, 60}, {60, 32, 32}};
  for (int dt : {UOT_F32, UOT_F64})
    for (const auto& b : bary) {
      const uot_geom g = grid(2, b[1], b[2], 0);
      route([&] { barycenter(dt, g, b[0], 0.01, UOT_DIV_TV); });
      if (b[0] == 12 || b[0] == 24) {
        route([&] { barycenter(dt, g, b[0], 0.01, UOT_DIV_KL); });
        route([&] { barycenter(dt, g, b[0], 0.01, UOT_DIV_RG); });
      }
    }
}

static void flow(int dtype, const uot_geom& g, int species) {
  note("flow", dtype, g, species, 0.01);
  uot_flow_problem fp;
  std::memset(&fp, 0, sizeof(fp));
  fp.dtype = dtype;
  fp.kind = UOT_FLOW_GROWTH;
  fp.species = species;
  fp.geom = g;
  fp.p0 = fp.q = fp.dx = kDev;
  fp.tau = 0.01;
  fp.alpha = 1.0;
  uot_params pr = params(0.01);
  size_t n = 0;
  EXPECT(uot_flow_workspace_size(&fp, &n) == UOT_OK);
  EXPECT(uot_flow(ctx, &fp, &pr, 1, kDev, kDev, kDev, n, nullptr) == UOT_OK);
}

// the tap slices of lines under the WF cost, of solves of several fields and flows of several species
static void slices() {
  for (int dt : {UOT_F32, UOT_F64})
    for (int nb : {1, 2, 3, 5})
      for (int n : {700, 1500, 2000, 2500, 3000, 4000, 4096})
        for (double cut : {0.3, 4.0}) {
          uot_geom g = grid(1, n, 0, 0);
          g.cost = UOT_COST_WF;
          g.cut = cut * n / 64;
          for (bool flows : {false, true}) {
            g_seen.clear();
            if (flows) flow(dt, g, nb);
            else solve(dt, g, nb, 0.01);
            for (const OffloadEntry* e = __start_llvm_offload_entries; e != __stop_llvm_offload_entries; ++e)
              if (g_seen.count(e->address) && std::strstr(e->name, "k_grid_contig"))
                std::printf("%s f%d fields %d cells %d cut %g: %u\n", flows ? "flow" : "slices", dt == UOT_F32 ? 32 : 64,
                            nb, n, cut, g_seen[e->address].grid.z);
          }
        }
}

int main(int argc, char** argv) {
  if (argc < 2 || uot_create(&ctx, nullptr) != UOT_OK) return 2;
  const std::string what = argv[1];
  if (what == "lines") lines();
  if (what == "planes") planes();
  if (what == "barycenters") barycenters();
  if (what == "instances") instances();
  if (what == "failing") failing();
  else if (what == "slices") slices();
  else if (what == "routes") routes();
  else print_lds();
  uot_destroy(ctx);
  if (failures) {
    std::fprintf(stderr, "%d launch check(s) failed\n", failures);
    return 1;
  }
  std::printf("launch checks passed\n");
  return 0;
}

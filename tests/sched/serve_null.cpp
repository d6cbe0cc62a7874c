// The HIP backend of the serving loop (serve.hip, compiled for the host) on a
// null device: the runtime calls and the kernel launches below do nothing but
// keep the runtime's per-thread record of the last error.  Checks whose fault
// an error is: a copy that fails for one request leaves the others running, a
// launch of the tick that fails ends all of them.  Prints "ok <name>" and exits
// 0, or prints the failed check and exits 1.
#include <condition_variable>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>

#include "ctx.h"
#include "dist_internal.h"
#include "ray_kernels.h"
#include "serve.h"

using namespace dist;

#define CHECK(c)                                                              \
  do {                                                                        \
    if (!(c)) {                                                               \
      std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c);    \
      std::exit(1);                                                           \
    }                                                                         \
  } while (0)

// ---- the runtime ------------------------------------------------------------
static thread_local hipError_t t_last = hipSuccess;
static const float* g_bad_src = nullptr;       // copies from here fail
static bool g_fail_march = false;              // the next march launch fails
static std::mutex g_mu;
static std::condition_variable g_cv;
static int g_ticks = 0, g_open = 0;            // ticks begun; ticks that may go on

static hipError_t fail(hipError_t e) { return t_last = e; }

extern "C" {
hipError_t hipGetLastError() {
  const hipError_t e = t_last;
  t_last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "null device"; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void* src, size_t, hipMemcpyKind, hipStream_t) {
  return src == g_bad_src ? fail(hipErrorInvalidValue) : hipSuccess;
}
}

// ---- the context ------------------------------------------------------------
int dist_set_error(int code, const char*, ...) { return code; }
int ctx_alloc(dist_ctx*, void** p, size_t n) { *p = std::malloc(n); return *p ? DIST_OK : DIST_EHIP; }
void ctx_free(dist_ctx*, void* p, size_t) { std::free(p); }
int slots_per_image(int hw, int) { return 2 * hw; }
void fold_into(const dist_ctx*, const float*, int, float*, float*, hipStream_t) {}

namespace dist {
int validate_params_ext(const dist_trace_params*, int, int) { return DIST_OK; }
int validate_camera_ext(const dist_camera&, const dist_trace_params*) { return DIST_OK; }
void fill_desc_ext(ImgDesc&, const dist_camera&, const dist_trace_params*, int, int, int) {}
int mlp_granule(int) { return 32; }
int adj_tile_rows(int) { return 64; }
int adjoint_waves() { return 8; }
int mlp_row_groups(int, int) { return 1; }
size_t adj_mask_words(int, const NetDev&) { return 64; }
void launch_adam(float*, float*, float*, const float*, int, float, float, float, float, int, hipStream_t) {}
void launch_eval(int, const EvalArgs&, int, hipStream_t) {}
void launch_adjoint(int, const AdjArgs&, int, hipStream_t) {}
void launch_advance(const RayPool&, const ImgDesc*, int*, int*, const AdvEntry*, const int*, int, hipStream_t) {}
void launch_normals(const RayPool&, const ImgDesc*, const int*, const int*, int, const float*, float, float*, float4*,
                    hipStream_t) {}
void launch_samples(const RayPool&, const ImgDesc*, const int*, const int*, int, int, int, int, const SeedIn&, int*,
                    int*, int*, int*, int*, int*, float4*, int*, hipStream_t, int, const SplitList*, int4*) {}
void launch_fill_i32(int*, int, int, hipStream_t) {}
void launch_fill_u64(unsigned long long*, int, hipStream_t) {}
void launch_finalize(const RayPool&, const ImgDesc*, const int*, int, int, const FinalizeOut&, hipStream_t) {}
void launch_gz_reduce(float*, int, int, int, const int*, const int*, int, int, int, const float*, int, int,
                      const float*, int, float*, hipStream_t, int, int) {}
void launch_render_loss(const float*, const float*, const float*, const float*, const float*, const float*, int, int,
                        float, float, float, float*, float*, float*, float*, hipStream_t) {}
void launch_sum_ordered(const float*, int, float*, hipStream_t) {}
// a tick waits here until the scenario lets it go on
void launch_tick_begin(const TickIo&, int*, int, hipStream_t) {
  std::unique_lock<std::mutex> lk(g_mu);
  ++g_ticks;
  g_cv.notify_all();
  g_cv.wait(lk, [] { return g_open >= g_ticks; });
}
void launch_march_pool(const MarchArgs&, int, hipStream_t) {
  std::lock_guard<std::mutex> lk(g_mu);
  if (g_fail_march) (void)fail(hipErrorLaunchFailure);
  g_fail_march = false;
}
void launch_tick_end(const TickIo&, hipStream_t) {}   // no ray is active: an image ends after its last split
}  // namespace dist

static void wait_tick(int n) {
  std::unique_lock<std::mutex> lk(g_mu);
  g_cv.wait(lk, [&] { return g_ticks >= n; });
}
static void open_ticks(int n) {
  std::lock_guard<std::mutex> lk(g_mu);
  g_open = n;
  g_cv.notify_all();
}

static dist_ctx* make_ctx() {
  dist_ctx* c = new dist_ctx();
  c->n_cu = 4;
  c->nl = 3;
  c->L = 4;
  c->kmax = 128;
  c->out_dims = {128, 128, 1};
  c->wpad = {128, 128, 0};
  c->budget = (size_t)256 << 20;
  return c;
}

static uint64_t submit(dist_ctx* c, const float* z) {
  dist_camera cam{};
  cam.H = cam.W = 8;
  dist_request r{};
  r.kind = DIST_REQ_RENDER;
  r.n_views = 1;
  r.cams = &cam;
  r.z = z;
  r.prm.max_steps = 20;
  r.prm.c2f_levels = 2;            // three ticks: the splits, then the full-resolution rays
  r.prm.k_samples = 1;
  r.prm.precision = DIST_BF16;
  uint64_t t = 0;
  CHECK(dist_submit(c, &r, &t) == DIST_OK);
  return t;
}

static int status_of(dist_ctx* c, uint64_t t) {
  dist_result r{};
  CHECK(dist_poll(c, t, &r, -1) == DIST_OK);
  return r.status;
}

int main(int argc, char** argv) {
  const std::string s = argc > 1 ? argv[1] : "";
  const float z[4] = {}, bad[4] = {};
  dist_ctx* c = make_ctx();
  const uint64_t a = submit(c, z);
  wait_tick(1);                     // a runs
  if (s == "copy") {
    g_bad_src = bad;
    const uint64_t b = submit(c, bad);
    open_ticks(1 << 30);
    CHECK(status_of(c, a) == DIST_OK);
    (void)status_of(c, b);
    CHECK(status_of(c, submit(c, z)) == DIST_OK);
  } else if (s == "launch") {
    {
      std::lock_guard<std::mutex> lk(g_mu);
      g_fail_march = true;
    }
    open_ticks(1 << 30);
    CHECK(status_of(c, a) == DIST_EHIP);
    CHECK(status_of(c, submit(c, z)) == DIST_OK);
  } else {
    return 2;
  }
  serve_shutdown(c);
  delete c;
  std::printf("ok %s\n", s.c_str());
  return 0;
}

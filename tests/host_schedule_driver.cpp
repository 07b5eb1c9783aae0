// Runs the 2-D host side (csrc/dugks_host.cpp) on the CPU with stand-ins for the
// kernels and the HIP calls that record what dugks_step enqueues: which buffer a
// launch reads, at which step, how many steps it takes, and what is captured.
// tests/test_host_schedule.py builds and runs it.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <vector>

#include "dugks.h"
#include "dugks_internal.h"
#include <hip/hip_runtime.h>

struct Op {
  const dugks::InstDev* inst;
  int buf, count, rows;
  long long step;
  const long long* base;
};
struct Graph { std::vector<Op> ops; };
static Graph* capture = nullptr;
static int captures = 0, launches = 0, fails = 0;
static bool caller_captures = false;
static const void* where = nullptr;   // the buffer that holds the state
static long long at = 0;       // its step

static void fail(const char* what, long long a, long long b) {
  fprintf(stderr, "%s: %lld, expected %lld (step %lld)\n", what, a, b, at);
  ++fails;
}
static void run(const Op& o) {
  const long long step = o.base ? o.step + o.base[0] : o.step;
  if (o.inst->buf[o.buf] != where) fail("buffer read", (long long)o.inst->buf[o.buf], (long long)where);
  if (step != at) fail("step index", step, at);
  where = o.inst->buf[o.buf ^ 1];
  at += o.count;
  ++launches;
}
static int enqueue(const dugks::StepArgs& a, const dugks::Launch& l, int count, int measure) {
  if (measure) return 0;   // takes no step
  const Op o{a.insts, a.parity, count, l.rows_per_wave, a.step, a.step_base};
  if (capture) capture->ops.push_back(o);
  else run(o);
  return 0;
}

namespace dugks {
int launch_step_fused(const StepArgs& a, const Launch& l, void*, int measure) { return enqueue(a, l, 1, measure); }
int launch_step2(const StepArgs& a, const Launch& l, void*) { return enqueue(a, l, 2, 0); }
int launch_step_plain(const StepArgs& a, int, int, void*) { return enqueue(a, Launch{}, 1, 0); }
int launch_set_base(const InstDev* insts, InstDev* replay, int n, int buf, long long* base, long long step, void*) {
  base[0] = step;
  for (int i = 0; i < n; ++i)
    for (int b = 0; b < 2; ++b) replay[i].buf[b] = insts[i].buf[b ^ buf];
  return 0;
}
int launch_init_eq(const InstDev*, const InstDev& in, const double*, int parity, void*) {
  where = in.buf[parity];
  at = 0;
  return 0;
}
int launch_set_f_pass(const InstDev*, const InstDev&, const double*, int, int, int, void*) { return 0; }
int launch_get_phi(const InstDev*, const InstDev&, double*, int, long long, void*) { return 0; }
int launch_get_f(const InstDev*, const InstDev&, double*, int, long long, void*) { return 0; }
int launch_reduce_widths(const InstDev*, const InstDev&, const double*, int, long long, const double*, double*, double*, void*) { return 0; }
int reduce_partials() { return 1; }
int launch_norms_noalloc(const InstDev*, const InstDev&, const double*, int, long long, const double*, double*, void*) { return 0; }
int launch_fill_u32(unsigned* p, unsigned v, long long n, void*) {
  for (long long i = 0; i < n; ++i) p[i] = v;
  return 0;
}
float neq_scale_host(int, float) { return 1.0f; }
}  // namespace dugks

extern "C" {
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { capture = new Graph; ++captures; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { *g = (hipGraph_t)capture; capture = nullptr; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t*, char*, size_t) { *e = (hipGraphExec_t)g; return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) { delete (Graph*)g; return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
  for (const Op& o : ((Graph*)e)->ops) run(o);
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = caller_captures ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = malloc(n); return hipSuccess; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = malloc(n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)8; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t* d) { *d = 0; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)8; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)8; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*) { memset(a, 0, sizeof(*a)); return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return ""; }
}

struct Ctx {
  dugks_ctx* h = nullptr;
  std::vector<double> phi, g;
  void* ws = nullptr;
  Ctx(int storage, int bcx, int bcy, bool source, int nx = 70, int ny = 20) : phi((size_t)nx * ny, 1.0), g((size_t)nx * ny, 0.0) {
    std::vector<double> xf(nx + 1), yf(ny + 1);
    for (int i = 0; i <= nx; ++i) xf[i] = i;
    for (int i = 0; i <= ny; ++i) yf[i] = i;
    dugks_params p;
    memset(&p, 0, sizeof(p));
    p.abi_version = DUGKS_ABI_VERSION;
    p.storage = storage;
    p.bc[0] = p.bc[1] = bcx;
    p.bc[2] = p.bc[3] = bcy;
    p.kernel = DUGKS_KERNEL_FUSED;
    p.c = 1.0;
    p.cfl = 0.5;
    p.alpha = 1e-2;
    must(dugks_create(&h, nx, ny, xf.data(), yf.data(), 9, &p));
    if (source) must(dugks_set_source(h, g.data(), 0.0));
    const size_t n = dugks_workspace_bytes(h);
    ws = aligned_alloc(256, (n + 255) / 256 * 256);
    must(dugks_bind(h, ws, n, nullptr));
    must(dugks_set_phi(h, phi.data(), 1));
    captures = 0;
  }
  ~Ctx() { dugks_destroy(h); free(ws); }
  void must(int rc) { if (rc) { fprintf(stderr, "rc %d: %s\n", rc, dugks_last_error(h)); ++fails; } }
  int step(int n) {   // launches of the run
    const int before = launches;
    must(dugks_step(h, n));
    return launches - before;
  }
};

// Runs of every length from every phase: a chain of launches, each reading what
// the one before wrote; two steps a launch wherever a run has two steps left;
// graphs where a run holds four steps from a step divisible by 4 (and a short one
// need not split a pair for them), captured at most once for each length.
static void runs() {
  for (int storage = DUGKS_F64; storage <= DUGKS_BF16NEQ; ++storage)
    for (int kind = 0; kind < 3; ++kind) {   // periodic; Dirichlet data is not needed for mirror walls; a source
      const bool neq = storage == DUGKS_F16NEQ || storage == DUGKS_BF16NEQ;
      if (neq && kind == 2) continue;
      const int bc = kind == 1 ? DUGKS_BC_MIRROR : DUGKS_BC_PERIODIC;
      Ctx c(storage, bc, bc, kind == 2);
      const bool pairs = !neq && kind != 2;
      long long done = 0;
      unsigned seed = 1;
      for (int k = 0; k < 400; ++k) {
        const int n = k < 60 ? k % 10 : (int)((seed = seed * 1103515245u + 12345u) >> 16) % 80;
        dugks_info a, b;
        dugks_get_info(c.h, &a);
        const int l = c.step(n);
        dugks_get_info(c.h, &b);
        const int lead = (int)((4 - done % 4) % 4);
        const bool splits = pairs && lead % 2 == 1 && n % 2 == 0 && n < lead + 64;   // a pair, for a graph
        const int in_graphs = n >= lead + 4 && !splits ? (n - lead) / 4 * 4 : 0;
        if (b.graph_steps - a.graph_steps != in_graphs) fail("steps in graphs", b.graph_steps - a.graph_steps, in_graphs);
        const int rest = in_graphs ? n - lead - in_graphs : n;
        const int want = !pairs ? n : in_graphs / 2 + (rest + 1) / 2 + (in_graphs ? (lead + 1) / 2 : 0);
        if (l != want) fail("launches", l, want);
        done += n;
        if (at != done) fail("steps", at, done);
      }
      if (captures > 2) fail("captures", captures, 2);
    }
}

// under the caller's capture: one step a launch, none from the library's graphs
static void captured() {
  Ctx c(DUGKS_F64, DUGKS_BC_PERIODIC, DUGKS_BC_PERIODIC, false);
  c.step(3);
  caller_captures = true;
  for (int n : {2, 4, 33}) {
    const int l = c.step(n);
    if (l != n) fail("captured launches", l, n);
  }
  caller_captures = false;
  if (captures) fail("captures", captures, 0);
}

// a caller's rows a wave are taken as given, beside walls too: one item for each
// strip of 62 columns and chunk of so many rows
static void chosen() {
  for (int bc : {DUGKS_BC_PERIODIC, DUGKS_BC_MIRROR})
    for (int storage = DUGKS_F64; storage <= DUGKS_BF16NEQ; ++storage) {
      const int nx = 130, ny = 41;
      Ctx c(storage, bc, bc, false, nx, ny);
      for (int rows : {1, 3, 8, 41, 100}) {
        c.must(dugks_set_launch(c.h, rows, 1, DUGKS_SCHED_GRID, 1));
        dugks_info i;
        dugks_get_info(c.h, &i);
        const long long want = (long long)((nx + 61) / 62) * ((ny + rows - 1) / rows);
        if (i.work_items != want) fail("work items", i.work_items, want);
      }
    }
}

int main() {
  runs();
  captured();
  chosen();
  if (!fails) puts("ok");
  return fails ? 1 : 0;
}

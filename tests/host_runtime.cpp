// The library's host code (snn_api.cpp) over a stand-in for the HIP runtime: device memory is host memory, a stream is a queue
// whose operations run when something waits for them (the latest moment a GPU may take), allocations and copies can be refused,
// kernels are replaced by what a check needs of them.  One program, a check per name on the command line (tests/test_host_runtime.py).
#define __align__(x) __attribute__((aligned(x)))
#define HIP_SYMBOL(x) (&x)
#include "snn_api.cpp"

#include <atomic>
#include <chrono>
#include <functional>
#include <map>
#include <mutex>
#include <thread>

// ---- the runtime --------------------------------------------------------------------------------
struct ihipStream_t {
  std::vector<std::function<void()>> q;
  size_t done = 0;
  void drain(size_t upto) { while (done < upto) q[done++](); }
};
struct ihipEvent_t { ihipStream_t *s = nullptr; size_t at = 0; };
static std::mutex g_mem_mutex;
static std::map<void *, size_t> g_mem;      // device allocations
static size_t g_largest = ~(size_t)0;       // larger ones are refused
static int g_mallocs = 0, g_refused = 0;
static int g_copies_left = -1;              // asynchronous copies until one fails (-1: none does)
static void put(hipStream_t s, std::function<void()> f) { if (s) s->q.push_back(f); else f(); }

#define HIP(name, ...) extern "C" hipError_t name(__VA_ARGS__)
static hipError_t device_alloc(void **p, size_t n) {
  std::lock_guard<std::mutex> hold(g_mem_mutex);
  if (n > g_largest) { ++g_refused; return hipErrorOutOfMemory; }
  ++g_mallocs;
  *p = std::calloc(1, n ? n : 1);
  g_mem[*p] = n;
  return hipSuccess;
}
HIP(hipMalloc, void **p, size_t n) { return device_alloc(p, n); }
HIP(hipExtMallocWithFlags, void **p, size_t n, unsigned) { return device_alloc(p, n); }
HIP(hipFree, void *p) {
  std::lock_guard<std::mutex> hold(g_mem_mutex);
  if (p) g_mem.erase(p);
  return hipSuccess; // (kept: a queued operation may still name it)
}
HIP(hipHostMalloc, void **p, size_t n, unsigned) { *p = std::calloc(1, n); return hipSuccess; }
HIP(hipHostFree, void *p) { std::free(p); return hipSuccess; }
HIP(hipPointerGetAttributes, hipPointerAttribute_t *a, const void *p) {
  std::lock_guard<std::mutex> hold(g_mem_mutex);
  auto it = g_mem.upper_bound(const_cast<void *>(p));
  const bool dev = it != g_mem.begin() && (--it, static_cast<const char *>(p) < static_cast<const char *>(it->first) + it->second);
  a->type = dev ? hipMemoryTypeDevice : hipMemoryTypeHost;
  return hipSuccess;
}
HIP(hipMemcpyAsync, void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st) {
  if (g_copies_left == 0) return hipErrorUnknown;
  if (g_copies_left > 0) --g_copies_left;
  put(st, [=] { std::memcpy(d, s, n); });
  return hipSuccess;
}
HIP(hipMemcpy2DAsync, void *, size_t, const void *, size_t, size_t, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
HIP(hipMemcpy, void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
HIP(hipMemset, void *d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
HIP(hipMemsetAsync, void *d, int v, size_t n, hipStream_t st) { put(st, [=] { std::memset(d, v, n); }); return hipSuccess; }
HIP(hipMemGetInfo, size_t *f, size_t *t) { *f = *t = (size_t)288 << 30; return hipSuccess; }
HIP(hipStreamCreateWithFlags, hipStream_t *s, unsigned) { *s = new ihipStream_t(); return hipSuccess; }
HIP(hipStreamDestroy, hipStream_t) { return hipSuccess; }
HIP(hipStreamSynchronize, hipStream_t s) { if (s) s->drain(s->q.size()); return hipSuccess; }
HIP(hipDeviceSynchronize) { return hipSuccess; }
HIP(hipEventCreate, hipEvent_t *e) { *e = new ihipEvent_t(); return hipSuccess; }
HIP(hipEventCreateWithFlags, hipEvent_t *e, unsigned) { *e = new ihipEvent_t(); return hipSuccess; }
HIP(hipEventDestroy, hipEvent_t) { return hipSuccess; }
HIP(hipEventRecord, hipEvent_t e, hipStream_t s) { e->s = s; e->at = s ? s->q.size() : 0; return hipSuccess; }
HIP(hipStreamWaitEvent, hipStream_t s, hipEvent_t e, unsigned) {
  ihipStream_t *from = e->s;
  const size_t at = e->at;
  if (from && from != s) put(s, [=] { from->drain(at); });
  return hipSuccess;
}
HIP(hipEventElapsedTime, float *ms, hipEvent_t, hipEvent_t) { *ms = 0.0f; return hipSuccess; }
HIP(hipStreamBeginCapture, hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; } // (the checks run with SNN_GRAPH=0)
HIP(hipStreamEndCapture, hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }
HIP(hipGraphInstantiate, hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipErrorNotSupported; }
HIP(hipGraphLaunch, hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
HIP(hipGraphDestroy, hipGraph_t) { return hipSuccess; }
HIP(hipGraphExecDestroy, hipGraphExec_t) { return hipSuccess; }
HIP(hipGetDeviceCount, int *n) { *n = 1; return hipSuccess; }
HIP(hipSetDevice, int) { return hipSuccess; }
HIP(hipGetLastError) { return hipSuccess; }
HIP(hipGetSymbolAddress, void **p, const void *s) { *p = const_cast<void *>(s); return hipSuccess; }
extern "C" const char *hipGetErrorString(hipError_t) { return "refused"; }

// ---- the kernels --------------------------------------------------------------------------------
static double g_rate = 0.0;                              // what launch_count_spikes finds
static std::function<void(const NetDev &, const WsArgs *)> g_forward; // what a forward pass does on the GPU
hipError_t launch_pack_inputs(const uint8_t *in, uint64_t *mask, int T, int B, int n_in, int Wd, hipStream_t s) {
  put(s, [=] { // row 0 of mask is step 0
    for (size_t r = 0; r < (size_t)T * B; ++r)
      for (int w = 0; w < Wd; ++w) {
        uint64_t v = 0;
        for (int k = 64 * w; k < n_in && k < 64 * w + 64; ++k) v |= (uint64_t)(in[r * n_in + k] != 0) << (k & 63);
        mask[((size_t)B + r) * Wd + w] = v;
      }
  });
  return hipSuccess;
}
hipError_t launch_forward(const NetDev &net, const int *bounds, int n_tiles, float *, const StoreSpec &, double *, int, float *,
                          hipStream_t s, const SpanHook *, const FwdCallbacks *cb, const WsArgs *ws) {
  for (int k = 0; k < n_tiles && cb && cb->tile_inputs; ++k) {
    const hipError_t e = cb->tile_inputs(cb->ctx, bounds[k], bounds[k + 1]);
    if (e != hipSuccess) return e;
  }
  const NetDev *n = &net;
  if (g_forward) put(s, [=] { g_forward(*n, ws); });
  return hipSuccess;
}
hipError_t launch_count_spikes(const CountJobs &jobs, hipStream_t s) {
  for (int k = 0; k < jobs.count; ++k) {
    const CountJob j = jobs.j[k];
    put(s, [=] { *j.count += (unsigned long long)(g_rate * 64.0 * (double)j.n_words); });
  }
  return hipSuccess;
}
hipError_t launch_fill_zero(void *p, size_t n, hipStream_t s) { put(s, [=] { std::memset(p, 0, n); }); return hipSuccess; }
hipError_t launch_fill_zero_jobs(ZeroJobs jobs, hipStream_t s) {
  for (int k = 0; k < jobs.count; ++k) launch_fill_zero(jobs.j[k].p, jobs.j[k].bytes, s);
  return hipSuccess;
}
hipError_t launch_recompute(const NetDev &, int, int, const float *, float *, int, size_t, int, float *, hipStream_t) { return hipSuccess; }
hipError_t launch_recompute_currents(const NetDev &, int, int, float *, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t launch_recompute_scan(const NetDev &, int, int, const float *, float *, int, size_t, int, float *, hipStream_t, const float *,
                                 int) { return hipSuccess; }
hipError_t launch_loss(const double *, const int32_t *, int, int, int, float *, float *, float *, hipStream_t) { return hipSuccess; }
hipError_t launch_adjoint_head(const NetDev &, int, int, int, float *, const float *, float *, int, float *, hipStream_t,
                               const SpanHook *) { return hipSuccess; }
hipError_t launch_up_product(const NetDev &, int, int, int, int, const float *, float *, hipStream_t, const SpanHook *) { return hipSuccess; }
hipError_t launch_adjoint_jobs(const NetDev &, const AdjJobs &, float *, const WsArgs &, hipStream_t, const SpanHook *) { return hipSuccess; }
int ws_max_resident_groups(int) { return 256; }
int ws_max_resident_groups_mfma(int) { return 256; }
int ws_max_resident_groups_mfma8(int) { return 256; }
void adjoint_prepare(const NetDev &, const WsArgs &) {}
hipError_t launch_dw(const uint64_t *, int, int, int, const float *, size_t, int, int, int, int, int, int, int, double *, hipStream_t, int) {
  return hipSuccess;
}
static DwBatch g_dw; // the last one
hipError_t launch_dw_mfma(DwBatch b, int, hipStream_t) { g_dw = b; return hipSuccess; }
hipError_t launch_dw_tile(DwBatch b, int, hipStream_t) { g_dw = b; return hipSuccess; }
bool bwd_stage_fusable(const NetDev &, int) { return false; }
int bwd_pre_placement(const NetDev &) { return 0; }
hipError_t launch_bwd_stage(const NetDev &, const AdjJobs &, float *, DwBatch, DuJob, const float *, PreJobs, hipStream_t, const SpanHook *) {
  return hipSuccess;
}
hipError_t launch_bwd_inter(const NetDev &, InterJobs, hipStream_t, const SpanHook *) { return hipSuccess; }
hipError_t launch_transpose(const float *, float *, int, int, hipStream_t) { return hipSuccess; }
static unsigned long long g_mask[3]; // synapses, groups by column, of the fullest slice
static int g_column_counts = 0, g_column_fills = 0;
hipError_t launch_csr_count(const uint8_t *, int, uint32_t *, unsigned long long *out, bool columns, hipStream_t s) {
  g_column_counts += columns;
  put(s, [=] { out[0] = g_mask[0]; out[1] = 0; if (columns) { out[2] = g_mask[1]; out[3] = g_mask[2]; } });
  return hipSuccess;
}
hipError_t launch_csr_fill(const uint8_t *, const float *, int, uint32_t, uint32_t *, uint16_t *, float *, uint64_t *, bool columns, hipStream_t) {
  g_column_fills += columns;
  return hipSuccess;
}
hipError_t launch_finish_grads(FinishJobs, hipStream_t) { return hipSuccess; }
hipError_t launch_finish_grad_csr(const double *, const uint32_t *, const uint16_t *, int, float *, hipStream_t) { return hipSuccess; }
hipError_t launch_unpack_spikes(const uint64_t *, int, int, int, int, uint8_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_copy(const void *, void *, size_t, hipStream_t) { return hipSuccess; }
bool snn_kernel_shape_ok(const NetDev &, char *, size_t) { return true; }
unsigned currents_choice(const NetDev &, int) { return 0; }
static const size_t LIST_ENTRIES = (size_t)1 << 20;
size_t currents_lists_entries(const NetDev &n) { return n.N[0] > 256 ? LIST_ENTRIES : 0; }

// ---- the checks ---------------------------------------------------------------------------------
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); std::exit(1); } } while (0)
struct Net {
  snn_config cfg{};
  snn_ctx *c = nullptr;
  std::vector<uint8_t> x;
  std::vector<int32_t> y;
  Net(int width, int T, int B, int n_in = 64, hipStream_t stream = nullptr) {
    cfg.n_in = n_in; cfg.n_layers = 1; cfg.n_hidden[0] = width; cfg.n_out = 8; cfg.T = T; cfg.batch = B;
    cfg.alpha = cfg.beta_out = 0.9f; cfg.theta = 1.0f; cfg.surr_beta = 10.0f; cfg.stream = stream;
    if (snn_init(&cfg, &c) != SNN_OK) { std::printf("snn_init: %s\n", snn_last_error(c)); std::exit(1); }
    fill(0);
  }
  void fill(int k) { // batch number k
    x.assign((size_t)cfg.T * cfg.batch * cfg.n_in, (uint8_t)(k & 1));
    y.assign((size_t)cfg.batch, k % cfg.n_out);
  }
  snn_status bind() { return snn_bind_inputs(c, x.data(), y.data(), cfg.T); }
  snn_status forward() { return snn_forward(c, x.data(), y.data(), cfg.T, nullptr); }
  bool holds(int k) const { // the inputs and labels of batch k are the bound ones
    for (size_t i = (size_t)cfg.batch; i < (size_t)(cfg.T + 1) * cfg.batch; ++i)
      if (c->net.mask[0][i] != (k & 1 ? ~0ull : 0ull)) return false;
    for (int b = 0; b < cfg.batch; ++b)
      if (c->labels[b] != k % cfg.n_out) return false;
    return true;
  }
  ~Net() { snn_destroy(c); }
};

// Spike trains in host memory that work on the caller's own stream still writes when the library is called
static void caller_stream() {
  for (int entry = 0; entry < 2; ++entry) {
    hipStream_t mine;
    hipStreamCreateWithFlags(&mine, 0);
    Net n(64, 20, 4, 64, mine);
    std::vector<uint8_t> later(n.x.size(), 1);
    n.y.assign(n.y.size(), 1);
    hipMemcpyAsync(n.x.data(), later.data(), later.size(), hipMemcpyDeviceToHost, mine);
    CHECK((entry ? n.forward() : n.bind()) == SNN_OK);
    CHECK(n.holds(1));
  }
}

// No room for the staging buffers: the batch that was bound stays, whole
static void no_room_for_staging() {
  for (int entry = 0; entry < 2; ++entry) {
    Net n(64, 20, 4);
    void *x = nullptr;
    hipMalloc(&x, n.x.size());
    CHECK(snn_bind_inputs(n.c, (uint8_t *)x, n.y.data(), n.cfg.T) == SNN_OK); // batch 0, from device memory
    n.fill(1);
    g_largest = (size_t)1 << 20;
    CHECK((entry ? n.forward() : n.bind()) != SNN_OK);
    g_largest = ~(size_t)0;
    hipStreamSynchronize(n.c->stream);
    CHECK(n.c->T_bound == n.cfg.T && n.holds(0));
    CHECK(snn_bptt(n.c, SNN_STANDARD, 0, 0, 0, nullptr) == SNN_OK);
    CHECK((entry ? n.forward() : n.bind()) == SNN_OK && n.holds(1));
  }
}

// A copy that fails leaves labels of one batch and spike trains of another: nothing is bound then
static void copy_fails() {
  for (int entry = 0; entry < 2; ++entry) {
    Net n(64, 20, 4);
    CHECK(n.bind() == SNN_OK);
    n.fill(1);
    g_copies_left = 1; // the labels arrive
    CHECK((entry ? n.forward() : n.bind()) == SNN_E_HIP);
    g_copies_left = -1;
    CHECK(snn_bptt(n.c, SNN_STANDARD, 0, 0, 0, nullptr) == SNN_E_STATE);
    CHECK(n.bind() == SNN_OK && n.holds(1) && snn_bptt(n.c, SNN_STANDARD, 0, 0, 0, nullptr) == SNN_OK);
  }
}

// A chip-wide kernel that gave up waiting: the call says so, and the next one starts afresh
static void time_out_is_reported() {
  Net n(512, 20, 4);
  CHECK(n.bind() == SNN_OK);
  std::vector<float> v((size_t)n.cfg.T * n.cfg.batch * 512);
  const auto give_up = [](const NetDev &, const WsArgs *ws) { *ws->err = 1u; };
  for (int entry = 0; entry < 3; ++entry) {
    const auto call = [&] {
      return entry == 0 ? n.forward() : entry == 1 ? snn_debug_states(n.c, v.data()) : snn_bptt(n.c, SNN_STANDARD, 0, 0, 0, nullptr);
    };
    g_forward = give_up;
    CHECK(call() == SNN_E_HIP);
    g_forward = nullptr;
    CHECK(call() == SNN_OK);
  }
}

// Two contexts whose kernels wait between workgroups, from two threads on one GPU: never at the same time.  One whose kernels wait
// for nobody runs beside them.
static void turns() {
  static std::atomic<int> inside{0}, overlaps{0}, narrow_runs{0};
  static std::atomic<bool> alone{true};
  g_forward = [](const NetDev &n, const WsArgs *) {
    if (n.N[0] <= 256) { ++narrow_runs; return; }
    if (++inside > 1) ++overlaps;
    for (int i = 0; i < 400 && !alone && narrow_runs == 0; ++i) std::this_thread::sleep_for(std::chrono::milliseconds(5));
    std::this_thread::sleep_for(std::chrono::milliseconds(3));
    --inside;
  };
  Net a(512, 20, 4), b(1100, 20, 4), narrow(64, 20, 4);
  const auto work = [](Net &n, bool noalloc) {
    std::vector<float> v((size_t)n.cfg.T * n.cfg.batch * n.c->net.SN);
    void *x, *y;
    hipMalloc(&x, n.x.size());
    hipMalloc(&y, n.y.size() * 4);
    for (int k = 0; k < 4; ++k) {
      CHECK(n.forward() == SNN_OK);
      CHECK(snn_bptt(n.c, SNN_CHUNK, 0, 5, 0, nullptr) == SNN_OK);
      CHECK(snn_debug_states(n.c, v.data()) == SNN_OK);
      if (noalloc) CHECK(snn_forward_noalloc(n.c, (uint8_t *)x, (int32_t *)y, n.cfg.T, nullptr) == SNN_OK);
    }
  };
  std::thread ta(work, std::ref(a), true), tb(work, std::ref(b), false);
  ta.join();
  tb.join();
  CHECK(overlaps == 0);
  alone = false; // the wide pass goes on until the narrow one has run
  std::thread tw([&] { CHECK(a.forward() == SNN_OK); });
  while (inside == 0) std::this_thread::yield();
  const auto t0 = std::chrono::steady_clock::now();
  CHECK(narrow.forward() == SNN_OK);
  CHECK(std::chrono::steady_clock::now() - t0 < std::chrono::seconds(1));
  tw.join();
  g_forward = nullptr;
}

// Contexts that come and go on several threads: no uncached block belongs to two of them
static void blocks() {
  static std::mutex m;
  static std::map<void *, int> owner;
  std::vector<std::thread> ts;
  for (int k = 0; k < 4; ++k)
    ts.emplace_back([] {
      for (int i = 0; i < 400; ++i) {
        Net n(257, 1, 1);
        std::unique_lock<std::mutex> hold(m);
        CHECK(n.c->ws.bar && ++owner[n.c->ws.bar] == 1);
        hold.unlock();
        std::this_thread::yield();
        hold.lock();
        --owner[n.c->ws.bar];
      }
    });
  for (auto &t : ts) t.join();
}

// A context's first training step allocates its state storage and its workspace, each once; where the device has no room for the
// lists of active neurons behind the workspace, that is found out once
static void workspace() {
  {
    Net n(512, 40, 4);
    CHECK(n.bind() == SNN_OK);
    const int before = g_mallocs;
    CHECK(snn_bptt(n.c, SNN_CHUNK, 0, 5, 0, nullptr) == SNN_OK);
    CHECK(n.c->net.lists && g_mallocs == before + 2);
    CHECK(snn_bptt(n.c, SNN_CHUNK, 0, 5, 0, nullptr) == SNN_OK && n.forward() == SNN_OK);
    CHECK(n.c->net.lists && g_mallocs == before + 2);
  }
  for (int entry = 0; entry < 2; ++entry) {
    Net n(512, 40, 4);
    CHECK(n.forward() == SNN_OK); // (a workspace that has to grow)
    snn_stats st{};
    const size_t least = snn_bytes_required(&n.cfg, SNN_STANDARD, 40, 0, 0);
    CHECK(snn_bptt(n.c, SNN_STANDARD, 0, 0, least, &st) == SNN_OK);
    CHECK(!n.c->net.lists && (size_t)(st.bytes_states + st.bytes_spikes + st.bytes_workspace) == least);
  }
  Net n(512, 40, 4);
  CHECK(n.bind() == SNN_OK);
  g_largest = LIST_ENTRIES * sizeof(uint16_t);
  const int refused = g_refused;
  CHECK(snn_bptt(n.c, SNN_CHUNK, 0, 5, 0, nullptr) == SNN_OK);
  CHECK(!n.c->net.lists && g_refused == refused + 1);
  const int before = g_mallocs;
  CHECK(snn_bptt(n.c, SNN_CHUNK, 0, 5, 0, nullptr) == SNN_OK);
  CHECK(snn_bptt(n.c, SNN_STANDARD, 0, 0, 0, nullptr) == SNN_OK);
  CHECK(!n.c->net.lists && g_refused == refused + 1);
  CHECK(g_mallocs <= before + 1); // (the state storage of the other strategy)
  g_largest = ~(size_t)0;
}

// Which kernel takes the weight gradients never follows the memory that is free: where there is no room for its workspace it walks
// shorter ranges of steps
static size_t device_bytes() {
  size_t sum = 0;
  for (const auto &m : g_mem) sum += m.second;
  return sum;
}
static void split_room() {
  const auto by_split = [](const Net &n) {
    CHECK(g_dw.count == 3 && g_dw.split_steps >= 1 && g_dw.split_steps <= SNN_BWD_TILE);
    for (int i = 0; i < 3; ++i) CHECK(g_dw.d[i].split && g_dw.d[i].scale && g_dw.d[i].octets);
  };
  for (size_t room : {~(size_t)0, (size_t)150 << 20, (size_t)75 << 20}) {
    g_largest = room;
    Net n(2048, 300, 64);
    CHECK(n.bind() == SNN_OK);
    for (int k = 0; k < 2; ++k) {
      const int refused = g_refused;
      CHECK(snn_bptt(n.c, SNN_CHUNK, 0, 5, 0, nullptr) == SNN_OK);
      by_split(n);
      CHECK(k == 0 || g_refused == refused);
    }
    CHECK(g_dw.split_steps == n.c->dw_steps);
    CHECK((room == ~(size_t)0) == (n.c->dw_steps == SNN_BWD_TILE));
  }
  g_largest = ~(size_t)0;
}

// That workspace is one of training steps, inside their budget but for SNN_DW_STEPS_LEAST steps
static void split_workspace() {
  size_t evaluation[3]; // (the first context of that size leaves its uncached block to the next)
  for (int k = 0; k < 3; ++k) {
    k == 1 ? setenv("SNN_DW", "mfma", 1) : unsetenv("SNN_DW");
    const size_t before = device_bytes();
    Net n(2048, 300, 64);
    CHECK(n.bind() == SNN_OK && n.forward() == SNN_OK);
    evaluation[k] = device_bytes() - before;
  }
  CHECK(evaluation[1] == evaluation[2]);
  for (int strategy : {SNN_STANDARD, SNN_CHUNK, SNN_DOUBLE, SNN_HIER})
    for (int F : {5, 100, 200})
      for (double more : {1.0, 1.02, 1.3, 3.0, 0.0}) {
        const int C = strategy == SNN_HIER ? 2 : 200;
        Net n(2048, 300, 64);
        CHECK(n.bind() == SNN_OK);
        const size_t least = snn_bytes_required(&n.cfg, (snn_strategy)strategy, 300, C, F), budget = (size_t)(more * (double)least);
        const size_t before = device_bytes();
        snn_stats st{};
        CHECK(snn_bptt(n.c, (snn_strategy)strategy, C, F, budget, &st) == SNN_OK);
        const size_t counted = (size_t)(st.bytes_states + st.bytes_spikes + st.bytes_workspace), spikes = (size_t)st.bytes_spikes; // (held since snn_init)
        CHECK(!budget || counted <= budget);
        CHECK(more != 1.0 || counted == least);
        CHECK(device_bytes() - before <= counted - spikes + dw_bytes(n.c->net, SNN_DW_STEPS_LEAST) + 512);
        CHECK(g_dw.split_steps >= SNN_DW_STEPS_LEAST && (more > 0.0 || g_dw.split_steps == SNN_BWD_TILE));
        // whatever the plan, the parts lie inside one of the two allocations and do not meet
        std::vector<std::pair<const unsigned char *, const unsigned char *>> parts;
        const size_t octets = (size_t)n.c->dw_steps * dw_split_octets(64);
        for (int l = 0; l < 2; ++l) {
          const size_t cols = l ? 8 : 2048;
          const auto add = [&](const void *p, size_t bytes) { parts.push_back({(const unsigned char *)p, (const unsigned char *)p + bytes}); };
          add(n.c->dw.split[l], octets * 48 * cols);
          add(n.c->dw.scale[l] - SNN_DW_SPECIAL, (SNN_DW_SPECIAL + octets / 4 * cols) * 4);
          for (int i = l; i < 3; i += 2) add(n.c->dw.octets[i], octets * 64 * n.c->net.Wd[i ? 1 : 0]);
        }
        std::sort(parts.begin(), parts.end());
        for (size_t i = 1; i < parts.size(); ++i) CHECK(parts[i - 1].second <= parts[i].first);
        const bool own = n.c->dw_ws && parts[0].first == n.c->dw_ws;
        const unsigned char *const base = own ? n.c->dw_ws : (const unsigned char *)n.c->dubuf;
        CHECK(parts[0].first >= base + (own ? 0 : adjoint_work_bytes(n.c->net, F > n.cfg.T ? n.cfg.T : F)) && parts.back().second <= base + g_mem[(void *)base]);
      }
}

// A launch of the sequential forward part by column has places for its spikes whatever the width: for the longest tile of every layer
static void column_places() {
  for (int N : {2897, 2900, 3000, 4095, 4096, 8100, 8192})
    for (int B : {1, 8, 9, 16, 20, 32}) {
      Net n(N, 2, B, 1);
      const size_t state = ((size_t)B * N * 4 + 255) & ~(size_t)255, slices = (N + 63) / 64, waves = B <= 8 ? 1 : B <= 16 ? 2 : 4;
      CHECK(g_mem[n.c->cur_state] >= state + SNN_FWD_TILE * slices * waves * 128);
      CHECK(n.c->ws.xl_col >= SNN_FWD_TILE * slices * waves * 128 && n.c->ws.xl_col % 128 == 0);
      CHECK(g_mem[n.c->cur_state] >= state + n.c->ws.xl_col && g_mem[n.c->cur_state] >= state + (size_t)n.c->ws.xg_stride * 4);
    }
}

// The form by column of a masked matrix is kept where its kernel can run, the mask suits it and the device has the room; handing weights over
// does not fail for it
static void column_form() {
  const auto kept = [](int N, int B, double density, double groups_per_slice, size_t room = ~(size_t)0) {
    Net n(N, 2, B, 1);
    g_mask[0] = (unsigned long long)(density * N * N);
    g_mask[1] = (unsigned long long)(groups_per_slice * ((N + 63) / 64));
    g_mask[2] = (unsigned long long)groups_per_slice;
    std::vector<float> w((size_t)N * N);
    std::vector<uint8_t> mask((size_t)N * N, 1);
    g_largest = room;
    int fills[2];
    for (int k = 0; k < 2; ++k) { // handed over once more
      g_column_fills = 0;
      CHECK(snn_set_weights(n.c, SNN_W_REC, 0, w.data(), mask.data()) == SNN_OK);
      fills[k] = g_column_fills;
    }
    g_largest = ~(size_t)0;
    CHECK(n.c->csr_pk[0] && n.c->csr_nnz[0] == g_mask[0] && fills[0] == fills[1] && fills[0] == (n.c->csr_ell[0] > 0));
    CHECK(n.c->csr_longest[0] == (n.c->csr_ell[0] ? 8 * g_mask[2] : 0));
    return n.c->csr_ell[0] > 0;
  };
  const int N = 4096;
  CHECK(kept(N, 32, 0.1, 58) && kept(N, 1, 0.01, 8) && kept(2897, 16, 0.3, 115) && kept(8192, 8, 0.002, 4));
  g_column_counts = 0;
  CHECK(!kept(2800, 32, 0.1, 40) && !kept(N, 33, 0.1, 58) && !kept(8700, 8, 0.002, 5) && g_column_counts == 0);
  CHECK(!kept(N, 32, 0.5, 260) && !kept(N, 32, 0.1, 512)); // the dense-stored walk is ahead; a full column in every slice
  setenv("SNN_NO_WS", "1", 1);
  g_column_counts = 0;
  CHECK(!kept(N, 32, 0.1, 58) && g_column_counts == 0);
  unsetenv("SNN_NO_WS");
  CHECK(!kept(N, 32, 0.2, 115, (size_t)(0.2 * N * N) * 8 + (1 << 20))); // room for the packed rows alone
}

// The activity that the kernels of the currents are chosen by is that of the last call, whatever the call and the batch size, and
// stays while the new one is near it (a recorded step holds the choice)
static void rates() {
  for (int B : {4, 80})
    for (int entry = 0; entry < 3; ++entry) {
      Net n(512, 20, B);
      const auto call = [&] {
        if (entry == 0) return n.forward();
        CHECK(n.bind() == SNN_OK);
        snn_stats st{};
        return snn_bptt(n.c, SNN_CHUNK, 0, 5, 0, entry == 1 ? nullptr : &st);
      };
      const auto known = [&](double r) { return std::fabs(n.c->net.rate[0] - r) < 1e-3 && std::fabs(n.c->net.rate[1] - r) < 1e-3; };
      CHECK(n.c->net.rate[0] < 0.0f && n.c->net.rate[1] < 0.0f);
      g_rate = 0.45;
      CHECK(call() == SNN_OK && n.c->net.lists && known(0.45));
      g_rate = 0.40; // within a quarter
      CHECK(call() == SNN_OK && known(0.45));
      g_rate = 0.05;
      CHECK(call() == SNN_OK && known(0.05));
      g_rate = 0.0;
      CHECK(call() == SNN_OK && known(0.01));
    }
}

int main(int argc, char **argv) {
  setenv("SNN_GRAPH", "0", 1);
  const std::map<std::string, void (*)()> checks{{"caller_stream", caller_stream}, {"no_room_for_staging", no_room_for_staging}, {"copy_fails", copy_fails},
                                              {"time_out_is_reported", time_out_is_reported},
                                              {"turns", turns}, {"blocks", blocks}, {"workspace", workspace},
                                              {"rates", rates}, {"split_room", split_room}, {"split_workspace", split_workspace}, {"column_places", column_places}, {"column_form", column_form}};
  const auto it = checks.find(argc > 1 ? argv[1] : "");
  if (it == checks.end()) return 2;
  it->second();
  return 0;
}

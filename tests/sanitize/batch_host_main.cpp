// Batched decoding's host side where queued work fails, answers late or never answers, without a GPU: the runtime is
// compiled for the host only, and the HIP calls it makes are defined here.  "Device" memory is host memory, and the three
// kernels whose results the host waits for or keeps a mirror of do what they do on the device: the push of the slots'
// state, the selection of a prompt's token (into the ring) and that of a step (one word a slot).
//
//   hipcc -x hip -O0 -g -std=c++17 --cuda-host-only -no-hip-rt -fuse-cuid=none [host sanitizers] tests/sanitize/batch_host_main.cpp
#include "../../paper_2604_23467_amd/csrc/ll_runtime.hip"

#include <cstdio>
#include <cstdlib>
#include <thread>

namespace fake {

enum When { AT_ONCE, LATE, IN_SYNC, NEVER };     // when a selection's tokens reach pinned memory
When when = AT_ONCE;
int token = 7;                                   // what it selects
const void* bad_launch = nullptr;                // the launch of this kernel reports an error, once
const void* sync_fails_behind = nullptr;         // the first wait behind the launch of this kernel reports an error
bool seen = false;
int syncs = 0;
hipError_t last = hipSuccess;
int* pending = nullptr;                          // words that the queued work is still to write
int npending = 0;
std::thread late;

void deliver() {
  for (int i = 0; i < npending; ++i) *(volatile int*)(pending + i) = token;
  npending = 0;
}
void select(int* words, int count) {
  pending = words;
  npending = count;
  if (when == AT_ONCE) deliver();
  if (when == LATE) {
    late = std::thread([] { std::this_thread::sleep_for(std::chrono::milliseconds(3)); deliver(); });
  }
}
void reset() {
  if (late.joinable()) late.join();
  when = AT_ONCE; token = 7; bad_launch = sync_fails_behind = nullptr; seen = false; last = hipSuccess; npending = 0;
}
template <typename F> const void* id(F* f) { return reinterpret_cast<const void*>(f); }

}  // namespace fake

// (the compiler refers to the device code by this name and does not let C++ define it)
__asm__(".data\n.globl __hip_fatbin\n__hip_fatbin: .zero 64\n.text\n");

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h = nullptr; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, dim3*, dim3*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

static dim3 g_grid, g_block;
static size_t g_lds;
static hipStream_t g_stream;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  g_grid = grid; g_block = block; g_lds = lds; g_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
  *grid = g_grid; *block = g_block; *lds = g_lds; *s = g_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t) {
  auto arg = [&](int i, auto like) { return *static_cast<decltype(like)*>(args[i]); };
  if (f == fake::bad_launch) {
    fake::bad_launch = nullptr;
    return fake::last = hipErrorLaunchFailure;
  }
  if (f == fake::sync_fails_behind) fake::seen = true;
  if (f == fake::id(&bt_push_kernel)) {
    const int *h_state = arg(0, (const int*)nullptr), *h_table = arg(2, (const int*)nullptr);
    int *state = arg(1, (int*)nullptr), *table = arg(3, (int*)nullptr);
    const int stride = arg(4, 0), first = arg(5, 0);
    memcpy(state, h_state, sizeof(BatchState));
    if (arg(6, (const DevState*)nullptr)) reinterpret_cast<BatchState*>(state)->next_token[first] = fake::token;
    memcpy(table + (size_t)first * stride, h_table + (size_t)first * stride, (size_t)grid.x * stride * 4);
  }
  if (g && f == fake::id(&sample_kernel<1>)) fake::select(g->host_ring, 1);
  if (g && f == fake::id(&bt_select_kernel<1>)) fake::select(g->batch->h_out, grid.x);
  return hipSuccess;
}
hipError_t hipGetLastError(void) { const hipError_t e = fake::last; fake::last = hipSuccess; return e; }
hipError_t hipStreamSynchronize(hipStream_t) {
  ++fake::syncs;
  if (fake::late.joinable()) fake::late.join();
  if (fake::when == fake::IN_SYNC) fake::deliver();
  if (fake::seen) {
    fake::sync_fails_behind = nullptr;
    fake::seen = false;
    return hipErrorLaunchFailure;
  }
  return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) { return hipStreamSynchronize(nullptr); }
const char* hipGetErrorString(hipError_t) { return "made up"; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  alignas(256) static char scratch[LL_STATIC_SCRATCH_BYTES];
  *p = scratch;
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(1, n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemset(void* d, int v, size_t n) { memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { return hipMemset(d, v, n); }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
// (the instance launches kernel by kernel, so that graphs and events are not reached)
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t*) { return hipErrorNotSupported; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float*, hipEvent_t, hipEvent_t) { return hipErrorNotSupported; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 1; return hipSuccess; }
}

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "check failed: %s (line %d): %s\n", #c, __LINE__, ll_last_error()); return 1; } } while (0)

// Everything that is kept of a batch's sequences, on the host and on the device
struct Books {
  std::vector<int> free_pages, table, device_table;
  std::vector<std::vector<int>> pages;
  BatchState state, device_state;
  explicit Books(const Batch* B)
      : free_pages(B->free_pages), table(B->h_table, B->h_table + BT_MAX_BATCH * B->L.pt_stride),
        device_table(B->at<int>(B->L.page_table), B->at<int>(B->L.page_table) + BT_MAX_BATCH * B->L.pt_stride),
        pages(B->pages), state(*B->h_state), device_state(*B->at<BatchState>(B->L.state)) {}
  bool operator==(const Books& o) const {
    return free_pages == o.free_pages && table == o.table && device_table == o.device_table && pages == o.pages &&
           !memcmp(&state, &o.state, sizeof state) && !memcmp(&device_state, &o.device_state, sizeof state);
  }
};

int joins_that_fail(Batch* B) {
  const int32_t prompt[20] = {1, 2, 3};
  int32_t first = -5;
  struct { const char* what; const void *bad_launch, *bad_sync; fake::When when; int token; } cases[] = {
      {"slot table not sent", fake::id(&bt_push_kernel), nullptr, fake::AT_ONCE, 7},
      {"rows not moved", fake::id(&bt_scatter_kernel), nullptr, fake::AT_ONCE, 7},
      {"work ends without its token", nullptr, nullptr, fake::NEVER, 7},
      {"the wait for a late token fails", nullptr, fake::id(&bt_scatter_kernel), fake::NEVER, 7},
      {"the wait behind the token fails", nullptr, fake::id(&bt_scatter_kernel), fake::AT_ONCE, 7},
      {"the token says that the prompt's kernels failed", nullptr, nullptr, fake::AT_ONCE, -1}};
  for (const auto& c : cases) {
    const Books before(B);
    fake::bad_launch = c.bad_launch; fake::sync_fails_behind = c.bad_sync; fake::when = c.when; fake::token = c.token;
    const int32_t rc = ll_batch_add(prompt, 20, &first);
    fake::reset();
    std::printf("%s: %d %s\n", c.what, rc, ll_last_error());
    CHECK(rc < 0 && first == -5);
    CHECK(Books(B) == before);
  }
  return 0;
}

int main() {
  const ll_config c{1, 128, 2, 64, 136, 64, 64, 10000.f, 1e-5f, LL_FLAG_EAGER};
  const size_t bytes = ll_workspace_bytes(&c);
  void* ws = std::aligned_alloc(256, bytes);
  memset(ws, 0, bytes);
  ll_layer_weights lw{ws, ws, ws, ws, ws, ws, ws, ws, ws};       // never read here
  const ll_weights w{ws, &lw, ws, ws};
  CHECK(ll_init(&c, &w, ws, bytes, nullptr) == LL_OK);
  const size_t pool_bytes = ll_batch_pool_bytes(8, 8);           // seven pages of eight positions
  void* pool = std::aligned_alloc(256, pool_bytes);
  memset(pool, 0, pool_bytes);
  CHECK(ll_batch_open(4, 8, 8, pool, pool_bytes) == LL_OK);
  Batch* B = g->batch;
  const int32_t prompt[64] = {1, 2, 3};
  int32_t first = -5, out[4];

  // a join that fails leaves nothing behind, in an empty batch and beside a sequence
  if (joins_that_fail(B)) return 1;
  CHECK(ll_batch_step(out) == LL_E_STATE);                       // nobody is in the batch
  CHECK(ll_batch_add(prompt, 55, &first) == 0 && first == 7);    // all seven pages are there
  CHECK(ll_batch_remove(0) == LL_OK);
  CHECK(ll_batch_add(prompt, 14, &first) == 0 && ll_batch_add(prompt, 3, &first) == 1 && ll_batch_remove(0) == LL_OK);
  if (joins_that_fail(B)) return 1;

  // a step's tokens: there at once, late, only once the stream has been waited for
  for (fake::When when : {fake::AT_ONCE, fake::LATE, fake::IN_SYNC}) {
    const Books before(B);
    fake::reset();
    fake::when = when;
    fake::token = 20 + when;
    fake::syncs = 0;
    const auto t0 = std::chrono::steady_clock::now();
    CHECK(ll_batch_step(out) == LL_OK);
    const auto took = std::chrono::steady_clock::now() - t0;
    CHECK(out[1] == 20 + when && B->h_state->pos[1] == before.state.pos[1] + 1 && B->h_state->next_token[1] == 20 + when);
    CHECK(fake::syncs == (when == fake::IN_SYNC) && (when != fake::IN_SYNC || took > std::chrono::milliseconds(kPollMs)));
  }
  // never: the step is reported, and the lists are those from before it, also where it was to take a page
  while (B->h_state->pos[1] % 8) { fake::reset(); CHECK(ll_batch_step(out) == LL_OK); }
  for (const void* bad : {(const void*)nullptr, fake::id(&bt_select_kernel<1>)}) {
    const Books before(B);
    fake::reset();
    fake::when = fake::NEVER;
    fake::sync_fails_behind = bad;
    CHECK(ll_batch_step(out) == LL_E_HIP && Books(B) == before);
  }
  fake::reset();
  CHECK(ll_batch_step(out) == LL_OK && B->pages[1].size() == 2);

  CHECK(ll_shutdown() == LL_OK);
  std::free(pool);
  std::free(ws);
  std::printf("sanitizer run ok\n");
  return 0;
}

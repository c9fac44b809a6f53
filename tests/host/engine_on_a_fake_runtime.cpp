// The engine's host code on a stand-in for the HIP runtime: memory is host memory, streams run in order at once, graphs
// record and replay, and kernel launches are noted by name.  Of the kernels only what the tests look at happens: the
// kernel that begins a step applies the page-table changes, and the words that the host waits for are written.  A runtime call can be made to
// fail, device memory to be scarce, and the words to be missing.  Linked with the library's own objects instead of the HIP runtime; built and run by tests/test_host_device.py.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

#include <chrono>
#include <functional>
#include <map>
#include <string>
#include <vector>

#include "../../include/pl.h"
#include "../../paper_2509_19128_amd/csrc/pl_common.h"

#define CHECK(cond)                                                                                   \
  do {                                                                                                \
    if (!(cond)) {                                                                                    \
      fprintf(stderr, "check failed at line %d: %s (%s)\n", __LINE__, #cond, pl_last_error());        \
      exit(1);                                                                                        \
    }                                                                                                 \
  } while (0)

// ---- the runtime ---------------------------------------------------------------------------------------
namespace {
struct Launch {
  std::string kernel;
  dim3 grid;
  pl::StepBegin begin;
  pl::AttnParams attn;
  int cap;   // records of the work list that the kernel that begins a step writes
  pl::SampleParams sample;
  const uint64_t *mark_at;   // of the kernel that ends a pass
  uint64_t *end_word;
};
std::map<const void *, std::string> names;
std::map<void *, size_t> device_memory;
size_t device_used = 0, device_high = 0, device_limit = ~(size_t)0;
int host_allocations = 0, fail_event_record = 0;   // fail_event_record: the how-manieth hipEventRecord from now fails
bool capturing = false, copying = true;   // copying: copies and fills happen
std::vector<Launch> done, captured;
dim3 call_grid, call_block;
int products = 0;   // launches whose buffers were looked at
int clock_khz = 100000;
uint64_t device_clock = 0, step_ticks = 0;   // step_ticks: what passes from the beginning of a step or pass to its end
bool words_come = true;                      // the kernels' words reach the host
bool words_late = false;                     // and do so when somebody synchronises
std::vector<std::function<void()>> late;

// A device that is behind: nothing enqueued has run until an event behind it (or its stream) is waited for, so the host memory that
// copies read must stay as it is.
struct Copy { const char *from; size_t bytes; int at; };
std::vector<Copy> on_their_way;
std::map<hipEvent_t, int> recorded;
bool behind = false;
int enqueued = 0, finished = 0, waits = 0, synchronised = 0, copied_behind = 0;   // copied_behind: synchronisations before the last hipMemcpy
size_t table_bytes = 0;   // copies of the page table, whose rows in use stay the same, are not looked at

void finish(int upto) {
  if (upto > finished) finished = upto;
  size_t k = 0;
  for (const Copy &c : on_their_way)
    if (c.at > finished) on_their_way[k++] = c;
  on_their_way.resize(k);
}

// The buffers of a product and of the kernels that take its slices lie in one allocation each.
void buffers_fit(const std::string &kernel, void **args) {
  auto number = [&](int i) { return (int64_t) * (const int *)args[i]; };
  auto fits = [&](int i, int64_t bytes) {
    const char *p = *(const char *const *)args[i];
    auto in = device_memory.upper_bound((void *)p);
    CHECK(in != device_memory.begin());
    --in;
    const int64_t room = (const char *)in->first + in->second - p;
    if (bytes <= room) return;
    fprintf(stderr, "%s: %lld bytes into %lld\n", kernel.c_str(), (long long)bytes, (long long)room);
    CHECK(!"a buffer holds what a kernel reads or writes");
  };
  std::vector<int> t;   // numbers among the template's arguments
  const size_t at = kernel.find("_kernelI");
  for (size_t i = at; at != std::string::npos && kernel[i] && kernel.compare(i, 2, "EE"); ++i)
    if (kernel[i] == 'L') t.push_back(atoi(kernel.c_str() + i + 2));
  auto is = [&](const char *name) { return kernel.find(name) != std::string::npos; };
  if (is("gemm_gu_")) {   // x, w, mid, slices, M, N, K, n_main, ...
    const int64_t M = number(4), N = number(5), K = number(6), rem = N - number(7), slices = number(is("joint") ? 9 : 8);
    fits(0, 2 * M * K); fits(1, 2 * N * K); fits(2, M * N); fits(3, 4 * slices * M * rem);
  } else if (is("gemm_")) {   // x, w, y, M, N, K, ksteps, ...
    const int64_t M = number(3), N = number(4), K = number(5), per = number(6) * 64;
    const bool fold = is("fold"), plain = is("gemm_kernel");
    const int64_t slices = fold ? 1 : (K + per - 1) / per, ld = plain ? number(10) : N;
    fits(0, 2 * M * K); fits(1, 2 * N * K);
    fits(2, !fold && t[is("rounds") ? 0 : 4] == 1 ? M * N : 4 * slices * M * ld);
  } else if (is("swiglu_reduce")) {
    fits(0, 4 * number(1) * number(2) * number(3));
  } else if (is("resid_rmsnorm")) {
    const int64_t row = number(5) * number(6);
    fits(0, 4 * row); fits(1, 4 * number(2) * row); fits(4, 2 * row);
  } else if (is("rope_append")) {
    const int64_t n = number(8), hd = number(11);
    fits(0, 4 * number(1) * n * (number(9) + 2 * number(10)) * hd); fits(6, 2 * n * number(9) * hd);
  } else {
    return;
  }
  ++products;
}

void run(const Launch &l) {
  done.push_back(l);
  if (l.kernel.find("step_begin_kernel") != std::string::npos && l.begin.updates && l.attn.work)
    for (int i = 0; i < l.begin.updates[0]; ++i) l.begin.page_table[l.begin.updates[2 + 2 * i]] = l.begin.updates[3 + 2 * i];
  auto word = [](uint64_t *at, uint64_t value) {
    if (words_come && words_late) late.push_back([=] { *at = value; });
    else if (words_come) *at = value;
  };
  auto pass_word = [](uint64_t mark) { return mark << pl::PASS_CLOCK_BITS | (device_clock & pl::PASS_CLOCK); };
  if (l.kernel.find("step_begin_kernel") != std::string::npos) {
    if (l.begin.time) word(l.begin.time, l.begin.mark_at ? pass_word(l.begin.mark) : device_clock);
    if (l.begin.mark_at) *l.begin.mark_at = l.begin.mark;
    device_clock += step_ticks;
  }
  if (l.end_word) word(l.end_word, pass_word(*l.mark_at));
  for (int r = 0; l.sample.results && r < l.sample.n; ++r) {
    word(&l.sample.results[r].time, device_clock);
    word(&l.sample.results[r].token_logprob, 5);
  }
}
}  // namespace

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *m; return &m; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { names[host] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) { call_grid = grid; call_block = block; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *s) {
  *grid = call_grid; *block = call_block; *shared = 0; *s = nullptr;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3, void **args, size_t, hipStream_t) {
  Launch l{names[f], grid, {}, {}, 0, {}, nullptr, nullptr};
  buffers_fit(l.kernel, args);
  if (l.kernel.find("step_begin_kernel") != std::string::npos) {
    l.begin = *(const pl::StepBegin *)args[0];
    l.attn = *(const pl::AttnParams *)args[1];
    l.cap = *(const int *)args[2];
  } else if (l.kernel.find("attn_") != std::string::npos) {
    l.attn = *(const pl::AttnParams *)args[0];
  } else if (l.kernel.find("sample_") != std::string::npos) {
    l.sample = *(const pl::SampleParams *)args[0];
  } else if (l.kernel.find("pass_end_kernel") != std::string::npos) {
    l.mark_at = *(const uint64_t *const *)args[0];
    l.end_word = *(uint64_t *const *)args[1];
  }
  if (capturing) captured.push_back(l); else run(l);
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) {
  *p = nullptr;
  if (device_used + n > device_limit) return hipErrorOutOfMemory;
  *p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);   // pages that nothing touches take no memory
  device_memory[*p] = n;
  device_used += n;
  if (device_used > device_high) device_high = device_used;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  if (!p) return hipSuccess;
  CHECK(device_memory.count(p));
  device_used -= device_memory[p];
  munmap(p, device_memory[p]);
  device_memory.erase(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = calloc(1, n); ++host_allocations; return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); --host_allocations; return hipSuccess; }
hipError_t hipMemGetInfo(size_t *f, size_t *t) { *f = device_limit - device_used; *t = device_limit; return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
  copied_behind = synchronised;
  if (copying) memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  CHECK(!capturing);
  if (copying) memcpy(d, s, n);
  if (behind && n != table_bytes) {
    for (const Copy &c : on_their_way) CHECK((const char *)s + n <= c.from || c.from + c.bytes <= (const char *)s);
    on_their_way.push_back(Copy{(const char *)s, n, ++enqueued});
  }
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { CHECK(!capturing); if (copying) memset(d, v, n); return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) { CHECK(a == hipDeviceAttributeWallClockRate); *v = clock_khz; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "made to fail"; }
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorNotFound; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free((void *)s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) {
  finish(enqueued);
  ++synchronised;
  for (auto &w : late) w();
  late.clear();
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { recorded.erase(e); free((void *)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  recorded[e] = enqueued;
  return fail_event_record && --fail_event_record == 0 ? hipErrorUnknown : hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) { return behind && recorded[e] > finished ? hipErrorNotReady : hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { finish(recorded[e]); ++waits; return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { capturing = true; captured.clear(); return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { capturing = false; *g = (hipGraph_t) new std::vector<Launch>(captured); return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t) {
  *x = (hipGraphExec_t) new std::vector<Launch>(*(std::vector<Launch> *)g);
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t) {
  for (const Launch &l : *(std::vector<Launch> *)x) run(l);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete (std::vector<Launch> *)g; return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { delete (std::vector<Launch> *)x; return hipSuccess; }
}

// ---- the tests -----------------------------------------------------------------------------------------
namespace {
pl_model_cfg shape(int kv_heads, int batch, int context, int64_t pool_tokens) {
  pl_model_cfg c{};
  c.n_layers = 2; c.d_model = 256; c.n_q_heads = 8; c.n_kv_heads = kv_heads; c.head_dim = 32; c.d_ffn = 256; c.vocab = 512;
  c.rope_theta = 1e4f; c.rms_eps = 1e-6f; c.max_batch = batch; c.max_context = context; c.kv_pool_tokens = pool_tokens;
  c.kv_page_tokens = 32; c.n_weight_buffers = 1; c.seed = 7; c.device = 0;
  return c;
}
pl_engine *engine(const pl_model_cfg &c) {
  pl_engine *e = nullptr;
  CHECK(pl_create(&c, &e) == PL_OK);
  std::vector<char> blob(pl_weight_nbytes(e));
  CHECK(pl_load_weights(e, blob.data(), blob.size()) == PL_OK);
  return e;
}
const Launch &last(const char *kernel) {
  for (size_t i = done.size(); i-- > 0;)
    if (done[i].kernel.find(kernel) != std::string::npos) return done[i];
  CHECK(!"launched");
  abort();
}

// A step that takes new pages and then ends early must not leave the device's page table without them.
void early_return() {
  for (int at = 1; at <= 2; ++at) {   // the first event of the step (before its launch) and the second (behind it)
    pl_engine *e = engine(shape(2, 2, 128, 512));
    std::vector<int32_t> prompt(20, 3);
    for (int i = 0; i < 2; ++i) CHECK(pl_add_sequence(e, i, prompt.data(), 20, 60, 1.f, nullptr) == PL_OK);
    pl_step_out out{};
    for (int i = 0; i < 32; ++i) CHECK(pl_decode_step(e, nullptr, &out) == PL_OK);
    fail_event_record = at;
    CHECK(pl_decode_step(e, nullptr, &out) == PL_E_HIP);
    CHECK(pl_decode_step(e, nullptr, &out) == PL_OK);
    const int32_t *table = last("step_begin_kernel").begin.page_table;   // pages are handed out in ascending order
    CHECK(table[0] == 0 && table[4] == 1);
    CHECK(table[1] == 2 && table[5] == 3);
    pl_destroy(e);
  }
}

// A step whose results do not come is an error, however its end was waited for, and leaves its sequences as they were; a pass
// whose words do not come (they carry its time alone) has read its prompt all the same.
void missing_words() {
  pl_engine *e = engine(shape(2, 2, 256, 512));
  std::vector<int32_t> prompt(20, 3);
  int32_t slot = -1, read = 0, token = -1, position = -1;
  CHECK(pl_add_sequence(e, 1, prompt.data(), 20, 200, 1.f, &slot) == PL_OK);
  words_come = false;
  CHECK(pl_prefill(e, slot, &read) == PL_OK && read == 19);
  pl_step_out out{};
  out.token = &token;
  out.position = &position;
  for (int i = 0; i < 70; ++i) {
    const bool profiled = i % 5 == 3;
    CHECK(pl_debug_set_profile(e, profiled ? 2 : 0) == PL_OK);
    pl_stats before{}, after{};
    words_come = false;
    CHECK(pl_get_stats(e, &before) == PL_OK && pl_decode_step(e, nullptr, &out) == PL_E_HIP && pl_get_stats(e, &after) == PL_OK);
    CHECK(after.steps == before.steps && after.tokens_emitted == before.tokens_emitted && before.steps == (uint64_t)i);
    words_come = true;
    CHECK(pl_decode_step(e, nullptr, &out) == PL_OK && out.n == 1 && token == 5 && position == 19 + i);
  }
  pl_destroy(e);
}

// Passes that a caller waits for end by a synchronisation of their stream every so often, however many background passes lie between them.
void passes_synchronise() {
  for (int background = 0; background <= 40; ++background) {
    pl_engine *e = engine(shape(2, 2, 128, 256));
    std::vector<int32_t> prompt(20, 3);
    int32_t slot = -1;
    auto read = [&](bool wait) {
      CHECK(pl_add_sequence(e, 1, prompt.data(), 20, 4, 1.f, &slot) == PL_OK);
      CHECK((wait ? pl_prefill(e, slot, nullptr) : pl_prefill_async(e, slot, nullptr)) == PL_OK && pl_retire_sequence(e, slot) == PL_OK);
    };
    synchronised = 0;
    int passes = 0, most = 0;   // most: passes from one synchronisation to the next that a pass in between could have brought
    for (int i = 0, before = 0; i < 100; ++i) {
      for (int b = 0; b < background; ++b) read(false);
      read(true);
      passes += background + 1;
      if (synchronised != before) { before = synchronised; passes = 0; }
      most = passes > most ? passes : most;
    }
    CHECK(most < 32);
    pl_destroy(e);
  }
}

// Steps and passes like one that took longer than polling lasts are not polled for: the caller's core is free meanwhile.
void long_waits() {
  pl_engine *e = engine(shape(2, 4, 1024, 4096));
  std::vector<int32_t> prompt(901, 3);
  int32_t slot = -1;
  auto host_ms = [](auto f) {
    const auto t0 = std::chrono::steady_clock::now();
    f();
    return std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  };
  auto pass = [&](int rows) {
    CHECK(pl_add_sequence(e, 1, prompt.data(), rows + 1, 4, 1.f, &slot) == PL_OK && pl_prefill(e, slot, nullptr) == PL_OK && pl_retire_sequence(e, slot) == PL_OK);
  };
  pl_step_out out{};
  words_late = true;
  step_ticks = 1000000;   // 10 ms
  pass(500);
  CHECK(host_ms([&] { for (int i = 0; i < 30; ++i) pass(500 + i); }) < 100);   // (polling would take 4 ms each)
  CHECK(pl_add_sequence(e, 2, prompt.data(), 20, 900, 1.f, &slot) == PL_OK && pl_decode_step(e, nullptr, &out) == PL_OK && pl_decode_step(e, nullptr, &out) == PL_OK);
  CHECK(out.step_ms == 10.f);
  CHECK(host_ms([&] { for (int i = 0; i < 28; ++i) CHECK(pl_decode_step(e, nullptr, &out) == PL_OK); }) < 100);
  // but shorter ones are, also shorter passes than the long one, and no synchronisation ends them
  words_late = false;
  step_ticks = 1000;
  synchronised = 0;
  CHECK(pl_decode_step(e, nullptr, &out) == PL_OK && out.step_ms < 1 && synchronised == 1);
  for (int i = 0; i < 50; ++i) CHECK(pl_decode_step(e, nullptr, &out) == PL_OK);
  pass(100);
  for (int i = 0; i < 20; ++i) pass(900);
  CHECK(synchronised <= 1 + 2 + 1);
  pl_destroy(e);
}

// One measure of a step's GPU time, whatever its end was waited for by: from its first kernel to its last result, by the device's own clock.  (The
// stand-in's events measure nothing.)
void step_time() {
  clock_khz = 25000;
  pl_engine *e = engine(shape(2, 2, 256, 512));
  step_ticks = 50000;
  std::vector<int32_t> prompt(20, 3);
  CHECK(pl_add_sequence(e, 1, prompt.data(), 20, 200, 1.f, nullptr) == PL_OK && pl_prefill(e, 0, nullptr) == PL_OK);
  pl_step_out out{};
  for (int i = 0; i < 100; ++i) CHECK(pl_debug_set_profile(e, i % 7 == 6 ? 1 + i % 2 : 0) == PL_OK && pl_decode_step(e, nullptr, &out) == PL_OK && out.step_ms == 2.f);
  pl_stats st{};
  CHECK(pl_get_stats(e, &st) == PL_OK && st.gpu_ms_total == 200. && st.prefill_ms == 2.);
  pl_destroy(e);
  clock_khz = 0;
  pl_engine *none = nullptr;
  const pl_model_cfg c = shape(2, 2, 256, 512);
  CHECK(pl_create(&c, &none) == PL_E_HIP);
}

// Logits are copied by a stream that waits for no other: behind a synchronisation of theirs, which a step that was polled for has not had.
void logits_behind_their_stream() {
  pl_engine *e = engine(shape(2, 2, 256, 512));
  std::vector<int32_t> prompt(2, 3);
  std::vector<float> logits(2 * 512);
  CHECK(pl_add_sequence(e, 1, prompt.data(), 2, 200, 1.f, nullptr) == PL_OK);
  pl_step_out out{};
  for (int i = 0; i < 40; ++i) {
    CHECK(pl_decode_step(e, nullptr, &out) == PL_OK);
    const int before = synchronised;
    CHECK(pl_debug_get_logits(e, logits.data(), 2 * 512) == PL_OK && copied_behind > before);
  }
  pl_destroy(e);
}

// A step takes the same attention route whether it is replayed from a graph or launched kernel by kernel.
void same_route() {
  for (int n = 60; n <= 128; ++n) {
    bool rotates[2];
    for (int graphs = 0; graphs < 2; ++graphs) {
      pl_engine *e = engine(shape(8, 128, 256, 128 * 256));
      CHECK(pl_debug_set_graphs(e, graphs) == PL_OK);
      std::vector<int32_t> prompt(20, 3);
      for (int i = 0; i < n; ++i) CHECK(pl_add_sequence(e, i, prompt.data(), 20, 60, 1.f, nullptr) == PL_OK);
      pl_step_out out{};
      CHECK(pl_decode_step(e, nullptr, &out) == PL_OK);
      rotates[graphs] = !last("attn_decode_kernel").attn.q;
      pl_destroy(e);
    }
    CHECK(rotates[0] == rotates[1]);
  }
}

// The records that a step or a pass of few rows may write end where the list ends, whatever a graph rounds its grid up to,
// and the attention reads no further.
void list_capacity() {
  for (int kv_heads : {1, 2, 3, 4, 8})
    for (int head_dim : {32, 64, 128})
      for (int context : {128, 256, 1024})
        for (int graphs = 0; graphs < 2; ++graphs) {
          pl_model_cfg c = shape(kv_heads, 4, context, 4 * context);
          c.n_q_heads = kv_heads * 8;
          c.head_dim = head_dim;
          pl_engine *e = engine(c);
          CHECK(pl_debug_set_graphs(e, graphs) == PL_OK);
          pl_step_out out{};
          std::vector<int32_t> prompt(context - 8, 3);
          for (int rows : {1, 2, 7, 31, 32, 33, 63, 64, 65, 85, 100, 119, 128, 129, 200, 247}) {
            if (rows >= context - 8) break;
            done.clear();
            int32_t slot = -1;
            CHECK(pl_add_sequence(e, 1, prompt.data(), rows + 1, 4, 1.f, &slot) == PL_OK);
            CHECK(pl_prefill(e, slot, nullptr) == PL_OK && pl_decode_step(e, nullptr, &out) == PL_OK);
            CHECK(pl_retire_sequence(e, slot) == PL_OK);
            for (const Launch &l : done) {
              if (!l.attn.work) continue;
              const int64_t records = (l.attn.tickets - l.attn.work) / 8;   // the tickets follow the list
              if (l.kernel.find("step_begin_kernel") != std::string::npos) CHECK(l.cap <= records);
              if (l.kernel.find("attn_decode_kernel") != std::string::npos) CHECK((int64_t)l.grid.x <= records * l.attn.Hkv);
            }
          }
          pl_destroy(e);
        }
}

// The buffers of the prompt passes give way where memory is tight, whatever does not fit beside them: an engine whose pool is
// one page is created down to well below what it takes with room, also where the pool takes what is left (pool_tokens 0).
void scarce_memory() {
  pl_model_cfg c = shape(2, 64, 256, 32);
  c.vocab = 8192;
  device_high = 0;
  pl_destroy(engine(c));
  const size_t needed = device_high, reserve = (size_t)6 << 30, less = (size_t)2 << 20;
  for (int64_t pool_tokens : {32, 0}) {
    c.kv_pool_tokens = pool_tokens;
    for (size_t missing = 0; missing < less; missing += (size_t)64 << 10) {
      device_limit = needed - missing + (pool_tokens ? 0 : reserve);
      pl_engine *e = nullptr;
      CHECK(pl_create(&c, &e) == PL_OK);
      pl_destroy(e);
    }
    device_limit = needed / 2 + (pool_tokens ? 0 : reserve);
    pl_engine *e = nullptr;
    CHECK(pl_create(&c, &e) == PL_E_NOMEM && device_memory.empty());
    device_limit = ~(size_t)0;
  }
}

// Rows of a pass: a whole prompt of up to 4096, half of that where the buffers do not fit or would take pages from a pool that takes what
// is left; the metadata of a pass lies as close as its rows allow.
void pass_rows() {
  const size_t reserve = (size_t)6 << 30, mib = (size_t)1 << 20;
  pl_model_cfg c = shape(2, 2, 4096, 8192);
  device_high = 0;
  pl_destroy(engine(c));
  const size_t needed = device_high;
  for (int what = 0; what < 3; ++what) {   // room; a byte too little; a pool that would be half of what its slots can use
    c.kv_pool_tokens = what == 2 ? 0 : 8192;
    device_limit = what == 0 ? needed : what == 1 ? needed - 1 : reserve + needed - 2 * mib;
    pl_engine *e = engine(c);
    std::vector<int32_t> prompt(4001, 3);
    int32_t slot = -1, read = 0;
    CHECK(pl_add_sequence(e, 1, prompt.data(), 4001, 4, 1.f, &slot) == PL_OK && pl_prefill(e, slot, &read) == PL_OK && read == 4000);
    pl_stats st{};
    CHECK(pl_get_stats(e, &st) == PL_OK && st.prefill_passes == (what == 0 ? 1u : 2u) && st.kv_pages_total == 256);
    const Launch &l = last("step_begin_kernel");
    const int rows = what == 0 ? 4000 : 4000 - 2048;
    CHECK(l.begin.src.row_slot - (const int32_t *)l.begin.src.seq_id == 2 * ((rows + 63) / 64 * 64));   // (ids of eight bytes)
    // beside decode steps, whose kernels would wait for a long pass's, no more than 768 rows
    CHECK(pl_add_sequence(e, 2, prompt.data(), 4001, 4, 1.f, &slot) == PL_OK && pl_prefill_async(e, slot, &read) == PL_OK && read == 4000);
    const uint64_t before = st.prefill_passes;
    CHECK(pl_get_stats(e, &st) == PL_OK && st.prefill_passes - before == 6 && last("step_begin_kernel").attn.n_seq == 4000 - 5 * 768);
    pl_destroy(e);
    device_limit = ~(size_t)0;
  }
}

// Every launch of a pass, whatever its row count, finds its operands and its slices in the buffers (the runtime above looks): shapes whose
// long product comes in slices from a row count on that is no multiple of a tile's rows, for engines of few and many slots, and the
// shapes of common decoders; with room, and with the rows that are left where memory is tight.
void pass_buffers() {
  struct { int d, q, kv, f, batch, context; } shapes[] = {{3584, 28, 4, 9728, 96, 1024}, {3584, 28, 4, 9728, 128, 1024}, {3584, 28, 4, 9728, 1, 640},
    {3328, 26, 2, 8448, 1, 640}, {1536, 12, 2, 8960, 64, 4224}, {3584, 28, 4, 18944, 256, 2100}, {5120, 40, 8, 27648, 128, 1300}, {1024, 8, 2, 8192, 130, 700},
    {2048, 16, 8, 10240, 16, 1500}, {4096, 32, 8, 14336, 200, 1100}, {8192, 64, 8, 28672, 512, 900}};
  for (const auto &m : shapes)
    for (int tight = 0; tight < 2; ++tight) {
      pl_model_cfg c = shape(m.kv, m.batch, m.context, m.context + 31);
      c.d_model = m.d; c.n_q_heads = m.q; c.head_dim = 128; c.d_ffn = m.f;
      copying = false;   // (weights of gigabytes)
      if (tight) device_limit = device_high - 1;
      device_high = 0;
      pl_engine *e = nullptr;
      CHECK(pl_create(&c, &e) == PL_OK);
      const int64_t bytes = pl_weight_nbytes(e);
      void *blob = mmap(nullptr, bytes, PROT_READ, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
      CHECK(pl_load_weights(e, blob, bytes) == PL_OK && pl_debug_set_graphs(e, 0) == PL_OK);
      munmap(blob, bytes);
      copying = true;
      std::vector<int32_t> prompt(m.context, 3);
      for (int rows = 2; rows < m.context; ++rows) {
        done.clear();
        int32_t slot = -1, read = 0;
        CHECK(pl_add_sequence(e, 1, prompt.data(), rows + 1, 1, 1.f, &slot) == PL_OK);
        CHECK(pl_prefill(e, slot, &read) == PL_OK && read == rows);
        CHECK(pl_retire_sequence(e, slot) == PL_OK);
      }
      pl_destroy(e);
      device_limit = ~(size_t)0;
    }
  CHECK(products > 100000);

  // and a call whose slices do not fit is refused
  const pl::GemmSplit down = pl::gemm_pick_split(64, 1536, 8960, 0), gu = pl::gemm_pick_split(256, 37888, 3584, 1);
  CHECK(pl::gemm_pass_slices(557, 1536, 8960, down) == down.splits && down.splits > 1 && gu.rem_splits > 1);
  float *ws = (float *)&done;   // (not null)
  done.clear();
  CHECK(pl::launch_gemm_pass(nullptr, nullptr, ws, (int64_t)down.splits * 557 * 1536 - 1, 557, 1536, 8960, 0, down, nullptr) == -1);
  CHECK(pl::launch_gemm_pass(nullptr, nullptr, ws, 2000 * 1536 - 1, 2000, 1536, 1536, 0, pl::GemmSplit{1, 1536, 1}, nullptr) == -1);
  CHECK(done.empty());

  // A SwiGLU product with a remainder takes slices of it only where it writes them, at up to 128 rows: more rows are launched without room for any, fewer are not.
  void *x = nullptr, *w = nullptr, *y = nullptr;
  CHECK(hipMalloc(&x, 2 * 512 * 3584) == hipSuccess && hipMalloc(&w, 2ll * 37888 * 3584) == hipSuccess && hipMalloc(&y, 512ll * 37888) == hipSuccess);
  auto bf16 = [](void *p) { return (const bf16_t *)p; };
  for (int rows : {129, 200, 256}) CHECK(pl::launch_gemm(bf16(x), bf16(w), y, nullptr, rows, 37888, 3584, 1, gu, false, nullptr) == 0);
  for (int rows : {257, 300, 512}) CHECK(pl::launch_gemm_pass(bf16(x), bf16(w), y, 0, rows, 37888, 3584, 1, gu, nullptr) == 0);
  CHECK(done.size() >= 6);
  done.clear();
  CHECK(pl::launch_gemm(bf16(x), bf16(w), y, nullptr, 128, 37888, 3584, 1, gu, false, nullptr) == -1 && done.empty());
  for (void *p : {x, w, y}) CHECK(hipFree(p) == hipSuccess);
}

// Background reading does not wait for the device while the host images of its passes fit the pinned memory, and no image is overwritten
// before its copy has run, whatever passes (long, short, of one prompt or of many) come one behind the other.
void pass_images() {
  for (int graphs = 0; graphs < 2; ++graphs) {
    pl_model_cfg c = shape(2, 128, 31744, 128 * 256 + 4 * 31744);
    pl_engine *e = engine(c);
    CHECK(pl_debug_set_graphs(e, graphs) == PL_OK);
    table_bytes = (size_t)c.max_batch * ((c.max_context + c.kv_page_tokens - 1) / c.kv_page_tokens) * 4;
    std::vector<int32_t> prompt(c.max_context, 3);
    behind = true;
    waits = 0;
    int32_t slot = -1, blocking = -1;
    CHECK(pl_add_sequence(e, 1, prompt.data(), 30001, 4, 1.f, &slot) == PL_OK && pl_prefill_async(e, slot, nullptr) == PL_OK && waits == 0);
    CHECK(pl_add_sequence(e, 2, prompt.data(), 31001, 4, 1.f, &slot) == PL_OK && pl_prefill_async(e, slot, nullptr) == PL_OK && waits > 0);
    for (int i = 0; i < 100; ++i) {
      CHECK(pl_add_sequence(e, 10 + i, prompt.data(), 2 + i * 2, 4, 1.f, &slot) == PL_OK && pl_prefill_async(e, slot, nullptr) == PL_OK);
      if (i % 40 == 20) CHECK(pl_add_sequence(e, 200 + i, prompt.data(), 9001, 4, 1.f, &blocking) == PL_OK && pl_prefill(e, blocking, nullptr) == PL_OK);
    }
    pl_step_out out{};
    CHECK(pl_decode_step(e, nullptr, &out) == PL_OK && out.n > 0);
    for (int i = 0; i < 30; ++i) {   // nothing on its way, then a little: no wait
      CHECK(pl_retire_sequence(e, slot) == PL_OK && (waits = 0) == 0);
      CHECK(pl_add_sequence(e, 300 + i, prompt.data(), 1000, 4, 1.f, &slot) == PL_OK && pl_prefill_async(e, slot, nullptr) == PL_OK && waits == 0);
    }
    pl_destroy(e);
    behind = false;
    on_their_way.clear();
  }
}

// One rule says whether a pass's product comes in slices, at every row count: where it is clear which way is faster (us at 513 to
// 640 rows, folded / in slices: 3584 x 9728, 13 slices, 57-71 / 88-94; 1536 x 8960, 9 slices, 39-41 / 37; 4096 x 11008, 4 slices, 557 rows, 85 / 72), it says so.
void slices_rule() {
  auto slices = [](int M, int N, int K, int rows) { const pl::GemmSplit ks = pl::gemm_pick_split(M, N, K, 0); CHECK(ks.splits > 1); return pl::gemm_pass_slices(rows, N, K, ks); };
  for (int rows = 500; rows <= 700; ++rows) {
    CHECK(slices(96, 3584, 9728, rows) == 1 && slices(1, 3328, 8448, rows > 512 ? rows : 513) == 1 && slices(130, 1024, 8192, rows) == 1);
    CHECK(slices(64, 1536, 8960, rows) > 1 && slices(64, 4096, 11008, rows < 560 ? rows : 560) > 1 && slices(512, 8192, 28672, rows < 512 ? rows : 512) > 1);
  }
}

// Operands of 2 GiB are refused whichever kernel the sizes call for: offsets into them have 31 bits.
void operand_limits() {
  const int K = 1 << 21;
  float nothing = 0;
  for (int rows : {512, 600, 1024, 4096}) {
    for (int N : {64, 256, 480})
      for (int splits : {1, 2, 64, 65, 128, 129, 256, 400, 8192})
        for (int mode : {0, 1}) {
          done.clear();
          if (mode == 0 || splits == 1) CHECK(pl_gemm_bf16(&nothing, &nothing, &nothing, rows, N, K, mode, splits, nullptr) == PL_E_INVAL);
          const pl::GemmSplit ks{splits, N, 1};
          CHECK(pl::launch_gemm(nullptr, nullptr, nullptr, &nothing, rows, N, K, mode, ks, false, nullptr) == -1);
          CHECK(pl::launch_gemm_folded(nullptr, nullptr, nullptr, rows, N, K, mode, ks, nullptr) == -1);
          CHECK(pl::launch_gemm_pass(nullptr, nullptr, nullptr, (int64_t)1 << 40, rows, N, K, mode, ks, nullptr) == -1);
          CHECK(done.empty());
        }
  }
  // and an engine whose rows are long enough to come near that reads its prompts in passes of fewer rows
  for (int f : {262144, 524288, 1048576}) {
    pl_model_cfg c = shape(2, 2, 4096, 8192);
    c.d_ffn = f;
    copying = false;
    pl_engine *e = nullptr;
    CHECK(pl_create(&c, &e) == PL_OK);
    const int64_t bytes = pl_weight_nbytes(e);
    void *blob = mmap(nullptr, bytes, PROT_READ, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    CHECK(pl_load_weights(e, blob, bytes) == PL_OK);
    munmap(blob, bytes);
    copying = true;
    std::vector<int32_t> prompt(4096, 3);
    int32_t slot = -1, read = 0;
    CHECK(pl_add_sequence(e, 1, prompt.data(), 4096, 1, 1.f, &slot) == PL_OK && pl_prefill(e, slot, &read) == PL_OK && read == 4095);
    pl_destroy(e);
  }
}
}  // namespace

int main(int, char **argv) {
  const std::string test = argv[1];
  if (test == "early_return") early_return();
  else if (test == "missing_words") missing_words();
  else if (test == "passes_synchronise") passes_synchronise();
  else if (test == "long_waits") long_waits();
  else if (test == "step_time") step_time();
  else if (test == "logits_behind_their_stream") logits_behind_their_stream();
  else if (test == "same_route") same_route();
  else if (test == "list_capacity") list_capacity();
  else if (test == "scarce_memory") scarce_memory();
  else if (test == "pass_rows") pass_rows();
  else if (test == "pass_buffers") pass_buffers();
  else if (test == "pass_images") pass_images();
  else if (test == "slices_rule") slices_rule();
  else if (test == "operand_limits") operand_limits();
  else return 2;
  CHECK(device_memory.empty() && host_allocations == 0);
  puts("ok");
  return 0;
}

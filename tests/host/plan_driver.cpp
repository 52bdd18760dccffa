// The library's host code (mivit_api.cpp, mivit_noalloc.hip) over a HIP runtime
// and kernel launchers that only keep count: device memory is host memory, a launch
// records what was launched.  Each scenario prints "name value" lines that
// tests/test_plan_host.py compares.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "../../include/mivit.h"
#include "../../paper_2011_13579_amd/csrc/mivit_device.h"

namespace {
int64_t n_malloc, n_copied, in_use;
int64_t memory = INT64_MAX;  // of the device
std::map<void*, size_t> blocks;
std::string launches;  // forward launches since the last reset
int64_t tb_end;        // last traceback launch: end of its table, from the items
float now;             // ms; each forward launch takes what `cost` says
std::map<std::string, float> cost;
}  // namespace

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  ++n_malloc;
  *p = nullptr;
  if (in_use + (int64_t)n > memory) return hipErrorOutOfMemory;
  *p = std::malloc(n ? n : 1);
  blocks[*p] = n;
  in_use += (int64_t)n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  auto it = blocks.find(p);
  if (it == blocks.end()) {
    std::printf("hipFree of memory that was not allocated\n");
    std::abort();
  }
  in_use -= (int64_t)it->second;
  blocks.erase(it);
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  n_copied += (int64_t)n;
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = nullptr, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorUnknown; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorUnknown; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return hipErrorUnknown;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorUnknown; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = (hipEvent_t) new float(0), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return delete (float*)e, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { return *(float*)e = now, hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
  return *ms = *(float*)b - *(float*)a, hipSuccess;
}
// the table kernel of mivit_noalloc.hip: nothing is launched
hipError_t hipGetSymbolAddress(void** p, const void*) { return *p = (void*)256, hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) {
  return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*,
                           void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
}

// (the host-only build of mivit_noalloc.hip has no device code to register)
extern "C" const char __hip_fatbin[8] = {};

namespace mivit {
static hipError_t launched(const std::string& what) {
  launches += (launches.empty() ? "" : " ") + what;
  now += cost.count(what) ? cost[what] : 1.0f;
  return hipSuccess;
}
hipError_t launch_fwd(int radix, int, int, const DevCode*, const Item*, int, const void*, uint64_t*,
                      void*, int32_t*, int32_t*, hipStream_t) {
  return launched("generic" + std::to_string(radix));
}
hipError_t launch_grad(const DevCode*, const GradFrame*, int, int, const uint32_t*, const float*,
                       float*, hipStream_t) {
  return hipSuccess;
}
hipError_t launch_quant(const float*, int8_t*, int64_t, float, hipStream_t) { return hipSuccess; }
hipError_t launch_fwd_rot(int, int, int, int, const DevCode*, const Item*, const int2*, int,
                          const void*, uint64_t*, void*, int32_t*, int32_t*, int32_t*, int,
                          hipStream_t) {
  return launched("rot");
}
hipError_t launch_fwd_wide(int, int, int, int wpf, bool packed, const DevCode*, const Item*,
                           const SplitUnit*, int, const void*, uint64_t*, void*, int32_t*,
                           int32_t*, WideBound*, int64_t*, const SplitUnit*, int, int64_t*,
                           SplitUnit*, int32_t*, hipStream_t) {
  return launched((packed ? "wpk" : "wide") + std::to_string(wpf));
}
hipError_t launch_fwd_r4p(int, const DevCode*, const Item*, const SplitUnit*, int, const int8_t*,
                          uint64_t*, int64_t*, int32_t*, int32_t*, int32_t*, int, R4Bound*,
                          int64_t*, const SplitUnit*, int, int64_t*, hipStream_t) {
  return launched("r4p");
}
hipError_t launch_fwd_r4q(const DevCode*, const Item*, const SplitUnit*, int, const int8_t*,
                          uint64_t*, int64_t*, int32_t*, int32_t*, int32_t*, int, R4Bound*,
                          int64_t*, const SplitUnit*, int, int64_t*, hipStream_t) {
  return launched("r4q");
}
hipError_t launch_fwd_r4_mfma(const MfmaGroups&, const DevCode*, const Item*, int, const int8_t*,
                              uint64_t*, int64_t*, int32_t*, int32_t*, hipStream_t) {
  return launched("mfma");
}
hipError_t launch_tb_seg(int, const DevCode*, const Item*, int, const uint64_t*, const int32_t*,
                         uint32_t*, int, hipStream_t) {
  return hipSuccess;
}
hipError_t launch_tb_r4p(int, const Item* items, const int2* table, int n, const uint64_t*,
                         const int32_t*, uint32_t*, int, hipStream_t) {
  tb_end = (int64_t)((const char*)(table + n) - (const char*)items);
  return hipSuccess;
}
hipError_t launch_zero_i32(int32_t*, int, hipStream_t) { return hipSuccess; }
hipError_t launch_fill_random(void*, int64_t, int, uint32_t, hipStream_t) { return hipSuccess; }
bool mfma_groups(int, int, const uint32_t*, MfmaGroups*) { return false; }
}  // namespace mivit

namespace {

mivit_code code(int K, std::vector<uint32_t> gens) {
  mivit_code c;
  std::memset(&c, 0, sizeof c);
  c.K = K;
  c.beta = (int32_t)gens.size();
  for (size_t b = 0; b < gens.size(); ++b) c.gen[b] = gens[b];
  return c;
}
const mivit_code kK5 = code(5, {023, 035}), kK7 = code(7, {0133, 0171}),
                 kK8 = code(8, {0247, 0371}), kK9 = code(9, {0557, 0663, 0711}),
                 kK9r4 = code(9, {0463, 0535, 0733, 0745});

mivit_opts opts(int dtype, int radix) {
  mivit_opts o;
  std::memset(&o, 0, sizeof o);
  o.dtype = dtype;
  o.radix = radix;
  return o;
}

std::vector<mivit_frame> frames(const mivit_code& c, int n, int stages) {
  std::vector<mivit_frame> f((size_t)n);
  for (int k = 0; k < n; ++k) {
    std::memset(&f[k], 0, sizeof f[k]);
    f[k].llr_offset = (int64_t)k * stages * c.beta;
    f[k].bit_offset = (int64_t)k * ((stages + 31) / 32) * 32;
    f[k].n_stages = f[k].n_out = stages;
    f[k].flags = MIVIT_START_KNOWN;
  }
  return f;
}

// Allocations of, and bytes copied by, the creation of a plan over n frames.
void tables(const char* name, const mivit_code& c, int dtype, int radix, int n, int stages) {
  const mivit_opts o = opts(dtype, radix);
  const std::vector<mivit_frame> f = frames(c, n, stages);
  const int64_t before = in_use;
  n_malloc = n_copied = 0;
  mivit_plan* p = nullptr;
  const mivit_status s = mivit_plan_create(&p, &c, 1, f.data(), n, &o);
  std::printf("tables.%s.status %d\n", name, (int)s);
  std::printf("tables.%s.allocations %lld\n", name, (long long)n_malloc);
  std::printf("tables.%s.copied %lld\n", name, (long long)n_copied);
  if (p) mivit_plan_destroy(p);
  std::printf("tables.%s.left %lld\n", name, (long long)(in_use - before));
}

// A plan that leaves the radix open, over frames of four lengths (which share
// no packed lane group: twice radix 2's survivors), on a device whose memory
// holds only the latter.
void open_radix_memory(const char* name, const mivit_code& c) {
  const mivit_opts o = opts(MIVIT_I8, 0);
  std::vector<mivit_frame> f = frames(c, 4, 400000);
  for (int k = 0; k < 4; ++k) f[k].n_stages -= 1000 * k, f[k].n_out -= 1000 * k;
  const int64_t before = in_use, stages = 4 * 400000;
  memory = before + stages * (1 << (c.K - 1)) / 8 * 3 / 2;
  mivit_plan* p = nullptr;
  const mivit_status s = mivit_plan_create(&p, &c, 1, f.data(), 4, &o);
  memory = INT64_MAX;
  launches.clear();
  uint32_t word = 0;
  if (p) mivit_decode(p, &word, &word, nullptr, nullptr, nullptr);
  std::printf("open_radix_memory.%s %d %s\n", name, (int)s, launches.c_str());
  if (p) mivit_plan_destroy(p);
  std::printf("open_radix_memory.%s.left %lld\n", name, (long long)(in_use - before));
}

// What the tuner keeps for four short frames where `fastest` runs fastest.
void tuned(const char* name, const mivit_code& c, int dtype, const char* fastest) {
  mivit_opts o = opts(dtype, 0);
  o.flags = MIVIT_PLAN_AUTOTUNE;
  const std::vector<mivit_frame> f = frames(c, 4, 300);
  cost.clear();
  cost[fastest] = 0.5f;
  mivit_plan* p = nullptr;
  const mivit_status s = mivit_plan_create(&p, &c, 1, f.data(), 4, &o);
  launches.clear();
  uint32_t word = 0;
  if (p) mivit_decode(p, &word, &word, nullptr, nullptr, nullptr);
  std::printf("tuned.%s %d %s\n", name, (int)s, launches.c_str());
  if (p) mivit_plan_destroy(p);
  cost.clear();
}

void described(const char* name, const mivit_code& c, int dtype, int variant, int n) {
  mivit_opts o = opts(dtype, 0);
  o.variant = variant;
  const std::vector<mivit_frame> f = frames(c, n, 300);
  mivit_plan* p = nullptr;
  char text[512] = "";
  if (mivit_plan_create(&p, &c, 1, f.data(), n, &o) == MIVIT_OK)
    mivit_plan_describe(p, text, sizeof text);
  launches.clear();
  uint32_t word = 0;
  if (p) mivit_decode(p, &word, &word, nullptr, nullptr, nullptr);
  std::printf("described.%s %s: %s\n", name, launches.c_str(), text);
  if (p) mivit_plan_destroy(p);
}

// The allocation-free call's limit: 64 MiB of items, wavefront entries, frame
// pairs, end states and survivors, whatever else it keeps.
int64_t noalloc_bytes(const mivit_code& c, int dtype, int64_t F, int S) {
  const bool packed = dtype == MIVIT_I8 && c.beta == 2 && (c.K == 5 || c.K == 7);
  const int64_t fpw = packed ? 2 * (64 >> (c.K - 1)) : c.K <= 7 ? 64 >> (c.K - 1) : 1;
  const int64_t waves = (F + fpw - 1) / fpw, pairs = packed ? (F + 1) / 2 : 0;
  auto up = [](int64_t x) { return (x + 255) / 256 * 256; };
  int64_t o = up((int64_t)sizeof(mivit::DevCode));
  o = up(o + F * (int64_t)sizeof(mivit::Item));
  o = up(o + waves * (int64_t)(packed || c.K > 7 ? sizeof(mivit::SplitUnit) : sizeof(int2)));
  o = up(o + pairs * (int64_t)sizeof(int2));
  o = up(o + F * 4);
  const int64_t ws = packed ? mivit::surv_words_r4p(c.K, S) : mivit::surv_words_blocks32(c.K, S);
  return o + ((packed ? pairs : F) * ws + mivit::kSurvSlackWords) * 8;
}

mivit_status uniform(bool noalloc, const mivit_code& c, int dtype, int F, int n) {
  uint32_t word = 0;
  launches.clear();
  return noalloc ? mivit_decode_uniform_noalloc(&word, dtype, &c, F, n, 1, &word, nullptr, nullptr)
                 : mivit_decode_uniform(&word, dtype, &c, F, n, 1, &word, nullptr, nullptr);
}

void noalloc_limit(const char* name, const mivit_code& c, int dtype) {
  int refused = 0, accepted = 0;
  int64_t room = 0;  // most bytes from the items to the traceback table's end
  for (int n : {1, 20, 33, 100, 1000, 2048, 20000}) {
    const int S = n + c.K - 1;
    int lo = 0, hi = 1 << 22;  // the largest batch within the limit
    while (hi - lo > 1) {
      const int mid = lo + (hi - lo) / 2;
      (noalloc_bytes(c, dtype, mid, S) <= 64 << 20 ? lo : hi) = mid;
    }
    refused += uniform(true, c, dtype, lo, n) != MIVIT_OK;
    if (tb_end > room) room = tb_end;
    accepted += uniform(true, c, dtype, lo + 1, n) != MIVIT_ENOMEM;
  }
  std::printf("noalloc_limit.%s %d %d\n", name, refused, accepted);
  std::printf("noalloc_room.%s %lld\n", name, (long long)room);
}

void same_kernel(const char* name, const mivit_code& c, int dtype, int F, int n) {
  const mivit_status a = uniform(false, c, dtype, F, n);
  const std::string plan = launches;
  const mivit_status b = uniform(true, c, dtype, F, n);
  std::printf("same_kernel.%s %d%d %s %s\n", name, (int)a, (int)b, plan.c_str(), launches.c_str());
}

}  // namespace

int main() {
  tables("k7_split", kK7, MIVIT_I8, 4, 128, 2176);
  tables("k7_open", kK7, MIVIT_I8, 0, 512, 4000);
  tables("k7_float", kK7, MIVIT_F32, 0, 512, 4000);
  tables("k9_split", kK9, MIVIT_I8, 0, 512, 4000);
  tables("k9_rate_quarter", kK9r4, MIVIT_I8, 0, 512, 4000);
  open_radix_memory("k7", kK7);
  open_radix_memory("k5", kK5);
  for (const char* w : {"wide1", "wide2", "wide4", "generic2"})
    tuned((std::string("k9_f32.") + w).c_str(), kK9, MIVIT_F32, w);
  for (const char* w : {"wide1", "wide2", "generic2"})
    tuned((std::string("k8_f32.") + w).c_str(), kK8, MIVIT_F32, w);
  for (const char* w : {"wide1", "wide4"})
    tuned((std::string("k9_f16.") + w).c_str(), kK9, MIVIT_F16, w);
  for (const char* w : {"wide1", "wide2"})
    tuned((std::string("k8_f16.") + w).c_str(), kK8, MIVIT_F16, w);
  described("k9_few", kK9, MIVIT_F32, 0, 4);
  described("k9_many", kK9, MIVIT_F32, 0, 4096);
  described("k9_v6", kK9, MIVIT_F32, 6, 4);
  described("k9_v7", kK9, MIVIT_F32, 7, 4);
  described("k8_few", kK8, MIVIT_F32, 0, 4);
  described("k8_f16", kK8, MIVIT_F16, 0, 4096);
  noalloc_limit("k3_f32", code(3, {7, 5}), MIVIT_F32);
  noalloc_limit("k4_i8", code(4, {015, 017}), MIVIT_I8);
  noalloc_limit("k5_i8", kK5, MIVIT_I8);
  noalloc_limit("k7_i8", kK7, MIVIT_I8);
  noalloc_limit("k7_f16", kK7, MIVIT_F16);
  noalloc_limit("k8_i8", kK8, MIVIT_I8);
  noalloc_limit("k9_f32", kK9, MIVIT_F32);
  noalloc_limit("k9r4_i8", kK9r4, MIVIT_I8);
  same_kernel("k7_short", kK7, MIVIT_I8, 1, 500);
  same_kernel("k7_long", kK7, MIVIT_I8, 1, 600);
  same_kernel("k7_few", kK7, MIVIT_I8, 1024, 40);
  same_kernel("k7_many", kK7, MIVIT_I8, 1100, 40);
  same_kernel("k5_long", kK5, MIVIT_I8, 1, 600);
  same_kernel("k5_many", kK5, MIVIT_I8, 4200, 40);
  same_kernel("k9_i8", kK9, MIVIT_I8, 3, 200);
  same_kernel("k9_f32", kK9, MIVIT_F32, 3, 200);
  same_kernel("k8_f32_many", kK8, MIVIT_F32, 3000, 50);
  std::printf("done 1\n");
  return 0;
}

// The library's host code (mivit_api.cpp) over a HIP runtime and kernel
// launchers that only keep count: device memory is host memory, a launch
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
}

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
hipError_t launch_tb_r4p(int, const Item*, const int2*, int, const uint64_t*, const int32_t*,
                         uint32_t*, int, hipStream_t) {
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
  std::printf("done 1\n");
  return 0;
}

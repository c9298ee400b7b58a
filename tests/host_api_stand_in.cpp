// The host side of the library (csrc/qoda_api.hip) compiled for the CPU over stand-ins for the HIP runtime and for the kernel
// launches, so that a test without a GPU can see which launches a call makes, let one of them fail, and capture and replay
// them.  "Device" memory is host memory, filled with a pattern when it is allocated.  Launches are recorded by name; the only
// effects they model are those on statistics: the norm pass adds to the fit's, its consumer moves it away; under bucket scope the
// quantize pass adds to the sums of its nodes, the clearing launches (the last kernel of the pass among them) clear theirs; held tiles
// leave a mark in their nodes' rows of the exchange area.
#include "../paper_2505_14371_amd/csrc/qoda_api.hip"
#include "../paper_2505_14371_amd/csrc/qoda_choices.h"

#include <cstdlib>
#include <functional>

namespace {
std::string g_log;
int g_fail_at = -1;           // launches until one fails; -1: none
bool g_capturing = false;
long long g_allocated = 0;
int g_hist_runs = 0;          // workgroups a node of the last norm pass with a histogram
int g_stale = 0;              // rows of the exchange area that a pass with held tiles found in use
std::vector<std::function<void()>> g_graph;

hipError_t record(const std::string &name, std::function<void()> effect = nullptr) {
  if (g_fail_at == 0) { g_fail_at = -1; return hipErrorLaunchFailure; }
  if (g_fail_at > 0) --g_fail_at;
  g_log += name + "\n";
  if (g_capturing) { if (effect) g_graph.push_back(effect); }
  else if (effect) effect();
  return hipSuccess;
}
}  // namespace

extern "C" {
void stand_in_reset() { g_log.clear(); g_fail_at = -1; }
const char *stand_in_log() { return g_log.c_str(); }
void stand_in_fail_at(int n) { g_fail_at = n; }
void stand_in_capture(int on) { g_capturing = on != 0; if (on) g_graph.clear(); }
int stand_in_hist_runs() { return g_hist_runs; }
int stand_in_stale() { return g_stale; }
int stand_in_alt_blocks(int G, int K, int bucket, int bits) { return alt_blocks(G, K, bucket != 0, bits); }
int stand_in_decode_blocks(int G, int K, int mode, int bucket, int bits) { return decode_blocks(G, K, mode, bucket != 0, bits); }
int stand_in_quantize_bins(long long n, int prev, int bits) { return quantize_bins(n, prev != 0, bits); }
long long stand_in_allocated() { return g_allocated; }   // bytes, of all allocations so far
void stand_in_replay() { for (auto &f : g_graph) f(); }

hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) {
  *p = std::malloc(n);
  if (!*p) return hipErrorOutOfMemory;
  std::memset(*p, 0xCD, n);
  g_allocated += (long long)n;
  return hipSuccess;
}
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemset(void *p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *s) { *p = const_cast<void *>(s); return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st) {
  *st = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { *e = reinterpret_cast<hipEvent_t>(std::malloc(1)); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { std::free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { *t = 1.0f; return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stand-in failure"; }
}

namespace qoda {

static void move_histograms(const Dev &a) {   // what the consumer of the histogram does with it
  const size_t n = (size_t)a.K * a.L * kHistBins;
  std::memcpy(a.hist_last, a.hist, n * sizeof(unsigned int));
  std::memset(a.hist, 0, n * sizeof(unsigned int));
}

hipError_t launch_zero_u32(unsigned int *p, size_t n, hipStream_t) { return record("zero", [=] { std::memset(p, 0, 4 * n); }); }
hipError_t launch_sumsq(const Dev &a, bool with_hist, hipStream_t) {
  if (!with_hist) return record("norms");
  g_hist_runs = a.GS;
  return record("norms+hist", [=] { for (size_t i = 0; i < (size_t)a.K * a.L; ++i) a.hist[i * kHistBins + 1] += 1; });
}
hipError_t launch_norm_finalize(const Dev &, hipStream_t) { return record("norm_finalize"); }
hipError_t launch_norm_vector(const Dev &, hipStream_t) { return record("norm_vector"); }
static void clear_sums(unsigned int *hist, size_t pairs) {
  for (size_t i = 0; i < pairs; ++i) std::memset(hist + i * kHistBins, 0, kGridPoints * sizeof(unsigned long long));
}
hipError_t launch_quantize(const Dev &a, unsigned int, hipStream_t) {
  if (a.scope != kScopeBucket) return record("quantize");
  return record("quantize_b:" + std::to_string(a.GS), [=] {
    for (size_t i = (size_t)a.node0 * a.L; i < (size_t)(a.node0 + a.nnodes) * a.L; ++i)
      for (int j : {0, kGridPoints - 1}) reinterpret_cast<unsigned long long *>(a.hist + i * kHistBins)[j] += 1;
  });
}
hipError_t launch_quantize_small(const Dev &a, unsigned int, hipStream_t) {
  return record("quantize_small", [=] { for (size_t i = 0; i < a.nnodes * exch_row(a.G); ++i) g_stale += a.exch[i] != 0; });
}
hipError_t launch_quantize_held(const Dev &a, unsigned int, hipStream_t) {
  return record("quantize_held:" + std::to_string(a.NT), [=] {
    for (int k = a.node0 - a.row0; k < a.node0 - a.row0 + a.nnodes; ++k) g_stale += a.exch[k * exch_row(a.G)]++ != 0;
  });
}
hipError_t launch_delta_finalize(const Dev &a, hipStream_t) {
  return record("delta", [=] { if (a.clear_exch) std::memset(a.exch, 0, 8 * a.nnodes * exch_row(a.G)); if (a.hist_old) clear_sums(a.hist_old, (size_t)a.K * a.L); });
}
hipError_t launch_step_scalars(const Dev &, hipStream_t) { return record("step_scalars"); }
hipError_t launch_decode(const Dev &, int mode, unsigned int, hipStream_t) { return record("decode:" + std::to_string(mode)); }
hipError_t launch_alt_scalars(const Dev &, hipStream_t) { return record("alt_scalars"); }
hipError_t launch_alt_finalize(const Dev &, hipStream_t) { return record("alt_finalize"); }
hipError_t launch_index_hist(const Dev &a, unsigned int, hipStream_t) { return record("index_hist:" + std::to_string(a.GS)); }
hipError_t launch_bucket_max(const Dev &a, hipStream_t) { return record("bucket_max:" + std::to_string(a.GS)); }
hipError_t launch_bucket_hist(const Dev &a, hipStream_t) { return record("bucket_hist:" + std::to_string(a.GS)); }
hipError_t launch_fit_pool_b(const Dev &, hipStream_t) { return record("fit_pool_b"); }
hipError_t launch_fit_typemax(const Dev &, hipStream_t) { return record("fit_typemax"); }
hipError_t launch_fit_pool(const Dev &a, hipStream_t) { return record("fit_pool", [=] { move_histograms(a); }); }
hipError_t launch_fit_dp(const Dev &a, int source, hipStream_t) {
  if (source == kFitLayers) return record("fit_dp:layers", [=] { move_histograms(a); });
  return record(source == kFitBuckets ? "fit_dp:buckets" : "fit_dp:pooled");
}
hipError_t launch_zero_stats(unsigned int *h, double *, size_t n, hipStream_t) { return record("zero_stats", [=] { clear_sums(h, n); }); }
hipError_t launch_copy(const void *, void *, size_t, hipStream_t) { return record("copy"); }
hipError_t launch_stream(const void *, void *, size_t, int, void *, hipStream_t) { return record("stream"); }
hipError_t launch_build_tables(const Dev &, int, hipStream_t) { return record("build_tables"); }
// small uploads through kernel arguments: done, not recorded
hipError_t launch_stage_words(void *dst, const void *src, size_t n, hipStream_t) { std::memcpy(dst, src, 4 * n); return hipSuccess; }
hipError_t launch_stage_pointers(void **dst, const void *const *src, size_t n, hipStream_t) {
  std::memcpy(dst, src, n * sizeof(void *));
  return hipSuccess;
}
hipError_t launch_stage_node(void **dst, const void *const *src, size_t n, const void *msg, const void *prev, hipStream_t) {
  std::memcpy(dst, src, n * sizeof(void *));
  dst[n] = const_cast<void *>(msg);
  dst[n + 1] = const_cast<void *>(prev);
  return hipSuccess;
}

}  // namespace qoda

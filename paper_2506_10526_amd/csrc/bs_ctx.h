// Internal context and plan objects behind the opaque handles of bs.h.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <map>
#include <memory>
#include <string>
#include <vector>

#include "../../include/bs.h"
#include "bs_plan.h"
#include "fft_lds.h"

struct DevBuf {
  void* p = nullptr;
  size_t bytes = 0;
  std::vector<unsigned char> mirror;   // bytes last uploaded into p from the host (tables only)
  bool in_graph = false;               // a captured graph copies a table into p on every replay
};

struct CountCache {
  std::vector<int32_t> tri;       // triangle list the counts were made for
  int64_t* d_counts = nullptr;    // device int64 per triangle
  std::vector<int64_t> h_counts;  // host copy
  double dev = 0.0;               // max |count - rint(count)| when the counts were made
  double bound = 0.0;             // certified bound on that distance (bsplan::count_error_bound)
};

struct Est3;

struct bs_ctx {
  int device = 0;
  hipStream_t stream = nullptr;
  std::string err;
  std::map<std::string, DevBuf> ws;      // grow-only workspace slots
  std::map<int, void*> tw32, tw64;        // twiddle tables exp(-2 pi i m / L), by L
  std::map<long long, void*> dftw;       // eta-synthesis twiddle words, by M
  std::map<uint64_t, CountCache> counts;  // geometry-keyed count caches
  bool timing = false;
  hipEvent_t ev[8] = {};
  double last_ms[4] = {0, 0, 0, 0};
  bool have_timing = false;
  double last_count_dev = 0.0;
  double last_count_bound = 0.0;   // error bound that certified the rounding of the last counts
  int last_grid_M = 0;   // delay-axis grid of the last 3D contraction
  double last_flops_vox = 0.0, last_vox = 0.0;   // algorithmic MFMA flops per voxel, voxels (MFMA synthesis path)
  std::map<std::string, int> tuned;       // autotuned launch parameters, by shape key
  // bumped whenever a workspace of the 3D estimate (ctx_plan3_ws) is reallocated or uploaded to again
  uint64_t est3_ws_gen = 0;
  // last prepared 3D estimate, reused while its key and est3_ws_gen still match
  std::shared_ptr<Est3> est3;
  std::vector<std::unique_ptr<std::vector<unsigned char>>> graph_tables;   // host copies read by captured uploads
  std::string est3_key;
  uint64_t est3_gen = 0;
};

struct bs_bins {
  bs_ctx* ctx = nullptr;
  bsplan::Plan P;
  int8_t* d_lut = nullptr;
};

// Device address of the allocation-free entry points' scratch array on `device` (current), looked
// up once per device (bs_noalloc.cpp).
int noalloc_scratch_init(int device);

// ---- helpers implemented in bs_api.cpp ----
// Certified bound on |x - T| of the FP64 ring counts of triangles `tri` ([n][3] bins) whose
// triple sum has a longest chain of `depth` roundings (bsplan::count_error_bound).
double ring_count_bound(const bsplan::Plan& P, const std::vector<int>& tri, double depth);
int ctx_fail(bs_ctx* c, int code, const std::string& msg);
void* ctx_ws(bs_ctx* c, const char* name, size_t bytes);       // grow-only; NULL on failure
const void* ctx_twiddle(bs_ctx* c, int L, bool fp64);          // NULL on failure
// The workspaces that a prepared bs_estimate_3d points to: those of its tag, PLAN3_TAG.  Other calls' workspaces
// may change between two estimates without a new plan.
constexpr const char* PLAN3_TAG = "c3";
inline bool ctx_plan3_ws(const std::string& name) { return name.compare(0, 2, PLAN3_TAG) == 0; }
// Host table -> named device workspace.  A table equal to what the workspace already holds is not
// copied again: a copy from pageable memory would hold the host until the stream reaches it, so
// repeated calls could no longer be queued ahead of the running kernels.  Under stream capture the copy is
// recorded, not made, and made again on every replay: it reads a host copy that the context keeps, and the
// workspace's contents are not known from then on, so every later call copies.
inline bool capturing(hipStream_t s) {   // the null stream cannot be captured
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  return s && hipStreamIsCapturing(s, &st) == hipSuccess && st != hipStreamCaptureStatusNone;
}
template <typename X>
inline X* upload(bs_ctx* c, const std::string& name, const std::vector<X>& v, int& rc) {
  X* d = (X*)ctx_ws(c, name.c_str(), std::max<size_t>(v.size() * sizeof(X), 16));
  if (!d) { rc = ctx_fail(c, BS_ENOMEM, "workspace " + name); return nullptr; }
  DevBuf& wb = c->ws[name];
  const size_t nb = v.size() * sizeof(X);
  const unsigned char* hv = (const unsigned char*)v.data();
  const bool cap = nb > 0 && capturing(c->stream);
  if (nb > 0 && (cap || wb.in_graph || !(wb.mirror.size() == nb && std::memcmp(wb.mirror.data(), hv, nb) == 0))) {
    const void* src = v.data();
    if (cap) {
      c->graph_tables.push_back(std::make_unique<std::vector<unsigned char>>(hv, hv + nb));
      src = c->graph_tables.back()->data();
      wb.in_graph = true;
    }
    wb.mirror.clear();
    if (hipMemcpyAsync(d, src, nb, hipMemcpyHostToDevice, c->stream) != hipSuccess) {
      rc = ctx_fail(c, BS_EHIP, "upload " + name);
      return nullptr;
    }
    if (!wb.in_graph) wb.mirror.assign(hv, hv + nb);
    if (ctx_plan3_ws(name)) ++c->est3_ws_gen;
  }
  rc = BS_OK;
  return d;
}
FftPlan make_fft_plan(int L);
// true when every pass of `p` over nl lines fits the in-place LDS FFT with `threads` threads and
// at most bmax butterflies per thread (bmax / 2 in radix-8 passes)
bool fft_ip_fits(const FftPlan& p, int nl, int threads, int bmax);
bool fft_len_ok(int L);
struct MabsFieldArgs;
int ring_fields_prepare(bs_ctx* c, const bs_bins* b, const bs_weights* w, bool fp64, bool count_mode,
                        bool ignore_chan, const int* d_bins, void* out, long long bin_stride, MabsFieldArgs& a);
void ring_fields_launch(MabsFieldArgs a, bool fp64, int nblocks, int nch, hipStream_t s);

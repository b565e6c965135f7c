// C ABI: 3D bispectrum (delay transform along frequency, |k| shells) and its fields.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <array>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "bs_ctx.h"
#include "bs_kernels.h"
#include "bs_est3.h"

#define HIPCHK(ctx, call)                                                                         \
  do {                                                                                            \
    hipError_t e_ = (call);                                                                       \
    if (e_ != hipSuccess)                                                                         \
      return ctx_fail(ctx, BS_EHIP, std::string(#call) + ": " + hipGetErrorString(e_));          \
  } while (0)

#define LAUNCHCHK(ctx, what)                                                                      \
  do {                                                                                            \
    hipError_t e_ = hipGetLastError();                                                            \
    if (e_ != hipSuccess) return ctx_fail(ctx, BS_EHIP, std::string(what) + ": " + hipGetErrorString(e_)); \
  } while (0)

void build_plan3(const bsplan::Plan& P, const std::vector<int>& blocks, bool fp64, Plan3& p) {
  const int n = P.n, nub = 2 * P.vmax + 1;
  const long long n2 = (long long)n * n;
  p.blocks = blocks;
  p.hj.clear(); p.offT.clear(); p.offG.clear();
  p.wv.clear(); p.wu.clear(); p.we.clear();
  p.totT = p.totG = 0;
  p.H = 0;
  p.NLe = fp64 ? 8 : 16;
  if (P.nc >= 1024) p.NLe = fp64 ? 4 : 8;
  p.NLd = (P.nc > 512) ? 4 : (fp64 ? 8 : 16);   // long delay axes: small blocks, several per CU
  bool iv_ok = P.kind == BS_SHELL_K && P.smax < 65536;
  for (size_t j = 0; j < blocks.size(); ++j) {
    int h = std::max(0, P.eta_hi[blocks[j]]);
    p.hj.push_back(h);
    p.H = std::max(p.H, h);
    p.offT.push_back(p.totT);
    p.offG.push_back(p.totG);
    p.totT += (long long)(h + 1) * nub * n;
    p.totG += (long long)(h + 1) * n2;
    for (int e = 0; e <= h; ++e) {
      // the shell's cells at |eta| = e as one range [lo, hi] of s, if they are one
      int lo = -1, hi = -2;
      for (int sv = 1; sv <= P.smax; ++sv)
        if (P.lut[(size_t)e * (P.smax + 1) + sv] == blocks[j]) { if (lo < 0) lo = sv; hi = sv; }
      for (int sv = std::max(lo, 1); sv <= hi && iv_ok; ++sv)
        iv_ok = P.lut[(size_t)e * (P.smax + 1) + sv] == blocks[j];
      if (lo < 0) { lo = 1; hi = 0; }   // empty
      iv_ok = iv_ok && hi < 65536;
      const int pad = iv_ok ? (lo | (hi << 16)) : 0;
      for (int q0 = 0; q0 < nub; q0 += p.NLv) p.wv.push_back({(int)j, e, q0, pad});
    }
    for (int xv = 0; xv < n; ++xv)
      for (int e0 = 0; e0 <= h; e0 += p.NLu) p.wu.push_back({(int)j, e0, xv, 0});
    for (long long l0 = 0; l0 < n2; l0 += p.NLe) p.we.push_back({(int)j, 0, (int)l0, 0});
  }
  p.shell_iv = iv_ok;
}

namespace {

// Twiddle table of the eta synthesis x(t) = sum_q a_q (Re G_q cos(2 pi q t / M) - Im G_q sin(2 pi q t / M)):
// entry m holds (cos, sin) of 2 pi m / M in FP32.  Cached per M.
const void* ctx_dft_twiddle(bs_ctx* c, int M) {
  auto it = c->dftw.find(M);
  if (it != c->dftw.end()) return it->second;
  std::vector<float> h(2 * (size_t)M);
  const long double tp = 2.0L * 3.14159265358979323846264338327950288L;
  for (int m = 0; m < M; ++m) {
    const long double ang = tp * (long double)m / (long double)M;
    h[2 * m] = (float)cosl(ang);
    h[2 * m + 1] = (float)sinl(ang);
  }
  void* d = nullptr;
  if (hipMalloc(&d, h.size() * 4) != hipSuccess) { (void)hipGetLastError(); return nullptr; }
  if (hipMemcpy(d, h.data(), h.size() * 4, hipMemcpyHostToDevice) != hipSuccess) { (void)hipFree(d); return nullptr; }
  c->dftw[M] = d;
  return d;
}

// M: length of the eta pass (nc, or a shorter grid that closes the same triangles)
int fields3_prepare(bs_ctx* c, const bs_bins* b, bool fp64, bool indicator, const Plan3& p, const std::string& t,
                    int M, Fields3Dev& fd) {
  const auto& P = b->P;
  const int n = P.n, nc = P.nc, nh = P.nh, nub = 2 * P.vmax + 1, nvb = P.vmax + 1;
  const size_t cz = fp64 ? 16 : 8;
  int rc = BS_OK;
  fd.fp64 = fp64;
  fd.indicator = indicator;
  Shell3Geom& g = fd.g;
  g.n = n; g.nh = nh; g.nc = nc; g.vmax = P.vmax; g.nub = nub; g.nvb = nvb;
  g.H = p.H; g.smax = P.smax; g.S1 = P.smax + 1;
  g.lut = b->d_lut;
  g.uvm = nullptr;
  fd.tw_nc = ctx_twiddle(c, nc, fp64);
  fd.tw_n = ctx_twiddle(c, n, fp64);
  fd.M = M;
  fd.tw_M = ctx_twiddle(c, M, fp64);
  if (!fd.tw_nc || !fd.tw_n || !fd.tw_M) return ctx_fail(c, BS_ENOMEM, "twiddle tables");
  fd.D = nullptr;
  if (!indicator) {
    fd.D = ctx_ws(c, (t + "_D").c_str(), (size_t)(2 * p.H + 1) * nub * nvb * cz);
    if (!fd.D) return ctx_fail(c, BS_ENOMEM, "workspace (delay)");
  }
  fd.Tm = ctx_ws(c, (t + "_T").c_str(), (size_t)p.totT * cz);
  fd.Gm = ctx_ws(c, (t + "_G").c_str(), (size_t)p.totG * cz);
  if (!fd.Tm || !fd.Gm) return ctx_fail(c, BS_ENOMEM, "workspace (3D passes)");
  fd.d_shell = upload(c, t + "_shell", p.blocks, rc); if (rc) return rc;
  fd.d_hj = upload(c, t + "_hj", p.hj, rc); if (rc) return rc;
  fd.d_offT = upload(c, t + "_offT", p.offT, rc); if (rc) return rc;
  fd.d_offG = upload(c, t + "_offG", p.offG, rc); if (rc) return rc;
  fd.d_wv = upload(c, t + "_wv", p.wv, rc); if (rc) return rc;
  fd.d_wu = upload(c, t + "_wu", p.wu, rc); if (rc) return rc;
  fd.d_we = upload(c, t + "_we", p.we, rc); if (rc) return rc;
  return BS_OK;
}

// Launches the field pipeline prepared in `fd` (no allocation, copy or synchronisation).
// With F != NULL the eta pass writes the real fields F ([block][fd.M n^2]); with F == NULL the
// pipeline stops after the u pass and the caller consumes the line-major spectra fd.Gm.
int fields3_enqueue(bs_ctx* c, const void* vis, const bs_weights* w, const Plan3& p, Fields3Dev& fd, void* F) {
  const int n = fd.g.n, nc = fd.g.nc;
  const size_t cz = fd.fp64 ? 16 : 8;
  Shell3Geom g = fd.g;
  g.uvm = w ? w->uv_mask : nullptr;
  // the delay, v and u passes transform in place (one LDS buffer, twice the resident blocks)
  // whenever their FFT plans fit, the FP64 eta pass at lengths with a compile-time transform;
  // BS_3D_FFT_TWO_BUFFERS (tests) keeps the two-buffer forms
  const bool two = getenv("BS_3D_FFT_TWO_BUFFERS") != nullptr;
  if (!fd.indicator) {
    Delay3Args d{};
    d.g = g; d.vis = vis; d.chw = w ? w->chan_w : nullptr; d.out = fd.D; d.tw = fd.tw_nc;
    d.plan = make_fft_plan(nc); d.NL = p.NLd;
    // smallest radices first: the first pass writes with a lane stride of R elements, and the small
    // radices spread those writes over the LDS banks better (any order gives the same DFT)
    if (!getenv("BS_3D_RADIX_DESC")) std::reverse(d.plan.rad, d.plan.rad + d.plan.nr);
    d.ip = two ? 0 : fft_ip_fits(d.plan, p.NLd, 256, 2) ? 2 : fft_ip_fits(d.plan, p.NLd, 256, 4) ? 4 : 0;
    size_t lds = ((d.ip ? 1 : 2) * (size_t)p.NLd * (nc + 1) + nc) * cz;
    if (fd.fp64) launch_delay3_f64(d, c->stream, lds); else launch_delay3_f32(d, c->stream, lds);
    LAUNCHCHK(c, "delay transform");
  }
  Pass3Args a{};
  a.g = g; a.shell_of_block = fd.d_shell; a.hj = fd.d_hj;
  // v pass
  a.work = fd.d_wv; a.off_in = nullptr; a.off_out = fd.d_offT; a.in = fd.D; a.out = fd.Tm; a.tw = fd.tw_n;
  a.plan = make_fft_plan(n); a.NL = p.NLv; a.indicator = fd.indicator ? 1 : 0;
  if (!getenv("BS_3D_RADIX_DESC")) std::reverse(a.plan.rad, a.plan.rad + a.plan.nr);   // as for the delay pass
  a.shell_iv = p.shell_iv && !getenv("BS_3D_SHELL_TABLE") ? 1 : 0;
  a.ip = two ? 0 : fft_ip_fits(a.plan, p.NLv, 256, 2) ? 2 : fft_ip_fits(a.plan, p.NLv, 256, 4) ? 4 : 0;
  launch_vpass3(a, (int)p.wv.size(), fd.fp64, c->stream, ((a.ip ? 1 : 2) * (size_t)p.NLv * (n + 1) + n) * cz);
  LAUNCHCHK(c, "v pass");
  // u pass
  a.work = fd.d_wu; a.off_in = fd.d_offT; a.off_out = fd.d_offG; a.in = fd.Tm; a.out = fd.Gm; a.NL = p.NLu;
  a.gs = fd.Gs; a.off_gs = fd.d_offGs; a.scale = fd.gscale;
  a.ip = two ? 0 : fft_ip_fits(a.plan, p.NLu, 256, 2) ? 2 : fft_ip_fits(a.plan, p.NLu, 256, 4) ? 4 : 0;
  launch_upass3(a, (int)p.wu.size(), fd.fp64, c->stream, ((a.ip ? 1 : 2) * (size_t)p.NLu * (n + 1) + n) * cz);
  LAUNCHCHK(c, "u pass");
  a.gs = nullptr; a.off_gs = nullptr; a.ip = two ? 0 : 1; a.shell_iv = 0;
  if (!F) return BS_OK;
  // eta pass (C2R), output length M
  const int M = fd.M;
  a.work = fd.d_we; a.off_in = fd.d_offG; a.off_out = nullptr; a.in = fd.Gm; a.out = F;
  a.tw = fd.tw_M; a.plan = make_fft_plan(M / 2); a.NL = p.NLe; a.M = M;
  if (fd.fp64) std::reverse(a.plan.rad, a.plan.rad + a.plan.nr);   // smallest radices first, as above
  a.scale = 1.0 / ((double)M * (double)n * (double)n);
  a.fstride = (long long)M * n * n;
  launch_etapass3(a, (int)p.we.size(), fd.fp64, c->stream, 2 * (size_t)p.NLe * (M / 2 + 1) * cz);
  LAUNCHCHK(c, "eta pass");
  return BS_OK;
}

// Both steps at once (fields output, count pass).
int run_fields3(bs_ctx* c, const bs_bins* b, const void* vis, const bs_weights* w, bool fp64, bool indicator,
                const Plan3& p, int M, void* F, const std::string& tag) {
  if (b->P.nc % 2) return ctx_fail(c, BS_EUNSUPPORTED, "3D fields need an even number of channels");
  Fields3Dev fd;
  int rc = fields3_prepare(c, b, fp64, indicator, p, tag, M, fd);
  if (rc) return rc;
  return fields3_enqueue(c, vis, w, p, fd, F);
}

int check_3d_inputs(bs_ctx* c, const bs_bins* b, const bs_weights* w) {
  if (b->P.kind != BS_SHELL_K) return ctx_fail(c, BS_EINVAL, "3D estimator needs BS_SHELL_K bins");
  if (w && w->ng) return ctx_fail(c, BS_EUNSUPPORTED, "3D estimator needs separable weights (uv_mask, chan_w)");
  if (!fft_len_ok(b->P.nc) || (b->P.nc % 2)) return ctx_fail(c, BS_EUNSUPPORTED, "nc must be even and 2^a 3^b");
  return BS_OK;
}

uint64_t hash_bytes3(uint64_t h, const void* p, size_t n) {
  const unsigned char* q = (const unsigned char*)p;
  for (size_t i = 0; i < n; ++i) { h ^= q[i]; h *= 1099511628211ULL; }
  return h;
}

}  // namespace

int filter_fields_3d(bs_ctx* c, const bs_bins* b, const void* vis, const bs_weights* w, int32_t precision,
                     void* fields, double* count_fields) {
  int rc = check_3d_inputs(c, b, w);
  if (rc) return rc;
  const auto& P = b->P;
  const bool fp64 = precision == BS_FP64;
  const long long fst = (long long)P.nc * P.n * P.n;
  std::vector<int> blocks;
  for (int j = 0; j < P.nbins; ++j) if (P.modes[j] > 0) blocks.push_back(j);
  // fields of empty shells are zero; non-empty ones are written block by block
  for (int pass = 0; pass < 2; ++pass) {
    void* out = pass == 0 ? fields : (void*)count_fields;
    if (!out) continue;
    bool f64 = pass == 1 ? true : fp64;
    size_t esz = f64 ? 8 : 4;
    HIPCHK(c, hipMemsetAsync(out, 0, (size_t)P.nbins * fst * esz, c->stream));
    if (pass == 0 && !vis) return ctx_fail(c, BS_EINVAL, "vis is NULL");
    for (int j : blocks) {
      Plan3 p;
      build_plan3(P, std::vector<int>{j}, f64, p);
      void* dst = (char*)out + (size_t)j * fst * esz;
      rc = run_fields3(c, b, vis, w, f64, pass == 1, p, P.nc, dst, pass == 0 ? "ff3" : "ff3c");
      if (rc) return rc;
    }
  }
  return BS_OK;
}

int est3_prepare(bs_ctx* c, const bs_bins* b, const bs_weights* w, int32_t precision, const std::string& tag,
                 Est3& e) {
  int rc = check_3d_inputs(c, b, w);
  if (rc) return rc;
  if (precision < 0 || precision > 2) return ctx_fail(c, BS_EINVAL, "bad precision");
  const auto& P = b->P;
  e.tag = tag;
  e.precision = precision;
  e.fp64 = precision == BS_FP64;
  e.ntri = (int)(P.tri.size() / 3);
  if (e.ntri == 0) return BS_OK;
  const int ntri = e.ntri;
  // ---- blocks, pairs, triangle -> (pair, column) ----
  std::map<int, int> blk;
  for (int x : P.tri) blk.emplace(x, 0);
  e.blocks.clear();
  for (auto& kv : blk) { kv.second = (int)e.blocks.size(); e.blocks.push_back(kv.first); }
  if ((int)e.blocks.size() > kMaxFields) return ctx_fail(c, BS_EUNSUPPORTED, "more than 32 shells in use");
  // The contraction forms one product row F_a F_b per shell pair and sums it against every shell
  // c, so a triangle can be served by any of its three pairs (the triple product is symmetric).
  // Pairs are chosen greedily (most still-unserved triangles first, ties to the smaller pair) to
  // cover all triangles with few rows: each row costs one product per voxel.
  std::vector<std::array<int, 3>> tb(ntri);
  for (int t = 0; t < ntri; ++t)
    for (int q = 0; q < 3; ++q) tb[t][q] = blk[P.tri[3 * t + q]];
  auto pkey = [](int x, int y) { return x < y ? std::make_pair(x, y) : std::make_pair(y, x); };
  std::vector<int> pairs, tpair(ntri, -1), tcol(ntri, -1);
  int left = ntri;
  while (left > 0) {
    std::map<std::pair<int, int>, int> gain;
    for (int t = 0; t < ntri; ++t) {
      if (tpair[t] >= 0) continue;
      std::set<std::pair<int, int>> seen;   // a triangle counts once per pair
      for (int q = 0; q < 3; ++q) {
        auto k = pkey(tb[t][q], tb[t][(q + 1) % 3]);
        if (seen.insert(k).second) ++gain[k];
      }
    }
    auto best = gain.begin();
    for (auto it = gain.begin(); it != gain.end(); ++it)
      if (it->second > best->second) best = it;
    const int pi = (int)(pairs.size() / 2);
    const int pa = best->first.first, pb = best->first.second;
    pairs.push_back(pa); pairs.push_back(pb);
    for (int t = 0; t < ntri; ++t) {
      if (tpair[t] >= 0) continue;
      for (int q = 0; q < 3; ++q) {
        if (pkey(tb[t][q], tb[t][(q + 1) % 3]) == best->first) {
          tpair[t] = pi;
          tcol[t] = tb[t][(q + 2) % 3];
          --left;
          break;
        }
      }
    }
  }
  e.npairs = (int)(pairs.size() / 2);
  if (e.npairs > kMaxPairs) return ctx_fail(c, BS_EUNSUPPORTED, "more than 112 shell pairs in use");
  // Column choice and row order.  A triangle goes to one of its chosen pairs whose third shell is
  // below 16 (the first field column tile) when it has one; the pairs that still serve a triangle
  // with a third shell of 16 or more come first, so the MFMA contraction needs the second column
  // tile only for the leading ceil(n_high / 16) pair row tiles.
  {
    std::map<std::pair<int, int>, int> pidx;
    for (int i = 0; i < e.npairs; ++i) pidx[pkey(pairs[2 * i], pairs[2 * i + 1])] = i;
    for (int t = 0; t < ntri; ++t) {
      int best = -1, bcol = -1;
      for (int q = 0; q < 3; ++q) {
        auto it = pidx.find(pkey(tb[t][q], tb[t][(q + 1) % 3]));
        if (it == pidx.end()) continue;
        const int col = tb[t][(q + 2) % 3];
        if (best < 0 || (bcol >= 16 && col < 16)) { best = it->second; bcol = col; }
      }
      tpair[t] = best;
      tcol[t] = bcol;
    }
    std::vector<char> high(e.npairs, 0);
    for (int t = 0; t < ntri; ++t) high[tpair[t]] |= tcol[t] >= 16;
    std::vector<int> order;
    for (int pass = 0; pass < 2; ++pass)
      for (int i = 0; i < e.npairs; ++i)
        if ((bool)high[i] == (pass == 0)) order.push_back(i);
    std::vector<int> where(e.npairs), np2;
    for (int i = 0; i < e.npairs; ++i) { where[order[i]] = i; np2.push_back(pairs[2 * order[i]]); np2.push_back(pairs[2 * order[i] + 1]); }
    for (int t = 0; t < ntri; ++t) tpair[t] = where[tpair[t]];
    pairs.swap(np2);
    int nhigh = 0;
    for (char h : high) nhigh += h;
    e.nhigh = nhigh;
    e.ct1_tiles = (nhigh + 15) / 16;
  }
  e.nvox = (long long)P.nc * P.n * P.n;
  e.d_pairs = upload(c, tag + "_pairs", pairs, rc); if (rc) return rc;
  e.d_tp = upload(c, tag + "_tpair", tpair, rc); if (rc) return rc;
  e.d_tc = upload(c, tag + "_tcol", tcol, rc); if (rc) return rc;
  e.nblk = std::min<long long>(2048, (e.nvox + 127) / 128);
  e.chunk = ((e.nvox + e.nblk - 1) / e.nblk + 127) / 128 * 128;
  e.nblk = (e.nvox + e.chunk - 1) / e.chunk;
  // FP64 fields (counts and FP64 data) on the shortest delay grid that closes the same triangles and has a
  // compile-time transform: with true closure (3 H < nc) any M > 3 H does, and the sums are rescaled
  // by (M / nc)^2.  At 768 channels and H = 104 it halves the fields (M = 384).
  e.M64 = P.nc;
  if (P.true_closure && !getenv("BS_3D_FULLGRID"))
    for (int m : {96, 128, 192, 256, 384, 512, 768})
      if (m > 3 * P.eta_max && m < P.nc) { e.M64 = m; break; }
  e.vox64 = (long long)e.M64 * P.n * P.n;
  // Up to two blocks a CU of three 128-voxel slabs or more, beyond them blocks of a dozen slabs, at most 1024 (two
  // resident a CU, two rounds).  us of the FP64 contraction, least slabs of 3 / 6 / 12 / 24: 16^2 x 32 9.8 / 13 / 21 /
  // 43, 48^2 x 96 23 / 22 / 27 / 45, 48^2 x 192 31 / 34 / 35 / 45, 48^2 x 768 162 / 157 / 150 / 182.
  e.nblk64 = std::max<long long>(1, std::max(std::min<long long>(512, e.vox64 / (3 * 128)),
                                             std::min<long long>(1024, e.vox64 / (12 * 128))));
  e.chunk64 = ((e.vox64 + e.nblk64 - 1) / e.nblk64 + 127) / 128 * 128;
  e.nblk64 = (e.vox64 + e.chunk64 - 1) / e.chunk64;
  // partial sums: one slot per contraction block, or per wave of the MFMA synthesis kernel (8 x 256)
  e.partial = (double*)ctx_ws(c, (tag + "_partial").c_str(), (size_t)std::max<long long>(e.nblk, 2048) * 112 * 32 * 8);
  e.reduced = (double*)ctx_ws(c, (tag + "_reduced").c_str(), (size_t)112 * 32 * 8);
  if (!e.partial || !e.reduced) return ctx_fail(c, BS_ENOMEM, "workspace (partials)");
  e.rho3 = 1.0;
  if (w && w->chan_w) {
    std::vector<float> hw(P.nc);
    HIPCHK(c, hipMemcpyAsync(hw.data(), w->chan_w, P.nc * sizeof(float), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    double s = 0;
    for (float x : hw) s += (double)x * x * x;
    e.rho3 = s / P.nc;
  }
  // ---- counts (FP64, cached per geometry and uv support) ----
  uint64_t key = P.hash ^ 0x3d3d3d3d3d3d3d3dULL;
  if (w && w->uv_mask) {
    std::vector<uint8_t> hm((size_t)P.n * P.nh);
    HIPCHK(c, hipMemcpyAsync(hm.data(), w->uv_mask, hm.size(), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    key = hash_bytes3(key, hm.data(), hm.size());
  }
  auto it = c->counts.find(key);
  if (it == c->counts.end()) {
    // Certification of the rounding: the FP64 count fields come from C2C passes along v and u
    // and a C2R pass along eta (three rounded normalisations); the contraction's longest chain
    // of roundings is one run of MFMA steps, the flushes of the runs of a wave's quarter of the block's
    // chunk, the four waves of the block, and the two stages of the fixed-order partial sums.  Runs of
    // kCon64Flush voxels are the fastest; where only shorter ones certify the counts (64 or 32 voxels on
    // blocks of few slabs: 128^2 x 324: depth 206 / 152 / 140), those are taken.
    const double eps_field = bsplan::field_error_units(2 * bsplan::fft_stage_units(P.n) + bsplan::fft_stage_units(e.M64) + 2, 3);
    int flush = kCon64Flush;
    double bound = 0.0;
    for (int run : {kCon64Flush, 64, 32}) {
      const double depth = (double)run + (double)((e.chunk64 / 4 + run - 1) / run) + 3.0 + (double)kReduceGroup +
                           (double)((e.nblk64 + kReduceGroup - 1) / kReduceGroup);
      double most = 0.0;
      for (int t = 0; t < ntri; ++t)
        most = std::max(most, bsplan::count_error_bound((double)P.modes[P.tri[3 * t]], (double)P.modes[P.tri[3 * t + 1]],
                                                        (double)P.modes[P.tri[3 * t + 2]], eps_field, depth));
      if (run == kCon64Flush || most < bound) { bound = most; flush = run; }
      if (bound < 0.5) break;
    }
    c->last_count_bound = bound;
    if (!(bound < 0.5))
      return ctx_fail(c, BS_ECOUNT, "3D triangle counts cannot be certified at this size (FP64 error bound " +
                                        std::to_string(bound) + " >= 1/2)");
    Plan3 pc;
    build_plan3(P, e.blocks, true, pc);
    void* F64 = ctx_ws(c, "c3_F64", (size_t)e.blocks.size() * e.vox64 * 8);
    if (!F64) return ctx_fail(c, BS_ENOMEM, "workspace (count fields)");
    rc = run_fields3(c, b, nullptr, w, true, true, pc, e.M64, F64, "c3c");
    if (rc) return rc;
    Con3Args ca{};
    ca.F = F64; ca.vox = e.vox64; ca.nbu = (int)e.blocks.size(); ca.pairs = e.d_pairs; ca.npairs = e.npairs;
    ca.chunk = e.chunk64; ca.partial = e.partial; ca.ct1 = e.ct1_tiles; ca.flush = flush;
    launch_contract64(ca, (int)e.nblk64, c->stream);
    LAUNCHCHK(c, "count contraction");
    double* Ssum = (double*)ctx_ws(c, "c3_Ssum", (size_t)ntri * 8 + 16);
    unsigned long long* bad = (unsigned long long*)ctx_ws(c, "count_dev", 256);
    if (!Ssum || !bad) return ctx_fail(c, BS_ENOMEM, "workspace (count sums)");
    Fin3Args f{};
    f.partial = e.partial; f.nparts = (int)e.nblk64; f.nent = (e.npairs + 15) / 16 * 16 * 32; f.tri_pair = e.d_tp; f.tri_col = e.d_tc; f.ntri = ntri;
    f.T3D = nullptr; f.Ssum = Ssum; f.sfac = (double)e.vox64 * (double)e.vox64;
    launch_fin3(f, e.reduced, c->stream);
    LAUNCHCHK(c, "count finalize");
    CountCache cc;
    if (hipMalloc(&cc.d_counts, (size_t)ntri * 8) != hipSuccess) { (void)hipGetLastError(); return ctx_fail(c, BS_ENOMEM, "count cache"); }
    HIPCHK(c, hipMemsetAsync(bad, 0, 8, c->stream));
    launch_round_counts(Ssum, ntri, cc.d_counts, bad, c->stream);
    LAUNCHCHK(c, "count rounding");
    double dev = 0.0;
    HIPCHK(c, hipMemcpyAsync(&dev, bad, 8, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    c->last_count_dev = dev;
    if (!(dev <= bound)) {
      (void)hipFree(cc.d_counts);
      return ctx_fail(c, BS_ECOUNT, "3D triangle count off an integer by " + std::to_string(dev) + ", beyond its error bound " +
                                        std::to_string(bound));
    }
    cc.dev = dev;
    cc.bound = bound;
    cc.tri.assign(P.tri.begin(), P.tri.end());
    it = c->counts.emplace(key, std::move(cc)).first;
  }
  e.d_counts = it->second.d_counts;
  e.count_dev = it->second.dev;
  e.count_bound = it->second.bound;
  // ---- data fields and contraction ----
  build_plan3(P, e.blocks, e.fp64, e.pd);
  // Delay-axis grid of the fused path.  With true closure (3 H < nc) any grid M > 3 H closes the
  // same triangles as the nc grid, so the smallest FFT-friendly multiple of 128 above 3 H is used
  // and the sums are rescaled by (M / nc)^2 (sum over M n^2 voxels of fields normalised by
  // 1 / (M n^2) versus nc n^2).
  int M = P.nc;
  if (P.true_closure && !getenv("BS_3D_FULLGRID")) {
    for (int m = 128; m < P.nc; m += 128)
      if (m > 3 * P.eta_max && fft_len_ok(m) && P.nc % 2 == 0) { M = m; break; }
  }
  e.fused = !e.fp64 && (M % 128 == 0) && !getenv("BS_3D_UNFUSED");
  if (!e.fused) M = e.fp64 ? e.M64 : P.nc;
  e.M = M;
  e.sfac = ((double)M / P.nc) * ((double)M / P.nc);
  rc = fields3_prepare(c, b, e.fp64, false, e.pd, tag + "d", e.fp64 ? e.M64 : P.nc, e.fd);
  if (rc) return rc;
  if (e.fused) {
    const long long nlines = (long long)P.n * P.n;
    e.fblocks = (int)std::min<long long>(nlines, 512);
    Fused3Args& fa = e.fa;
    fa = Fused3Args{};
    fa.G = e.fd.Gm; fa.offG = e.fd.d_offG; fa.hj = e.fd.d_hj; fa.nbu = (int)e.blocks.size(); fa.nlines = nlines;
    fa.M = M;
    fa.plan = make_fft_plan(M / 2);
    fa.tw = ctx_twiddle(c, M, false);
    if (!fa.tw) return ctx_fail(c, BS_ENOMEM, "twiddle table");
    fa.scale = 1.0 / ((double)M * (double)P.n * (double)P.n);
    fa.pairs = e.d_pairs; fa.npairs = e.npairs;
    fa.lines_per_block = (nlines + e.fblocks - 1) / e.fblocks;
    // leading blocks whose delay support is narrow are summed directly in the kernel
    fa.nlow = 0;
    while (fa.nlow < fa.nbu && e.pd.hj[fa.nlow] <= FUSED_DIRECT_H && !getenv("BS_3D_ALLFFT")) ++fa.nlow;
    fa.partial = e.partial;
    const size_t ld = (size_t)M / 2 + (size_t)M / 32 + 2;   // the kernel's padded FFT line
    int stage_len = 0;
    for (int h : e.pd.hj) stage_len += h + 1;
    if (stage_len > 512) return ctx_fail(c, BS_EUNSUPPORTED, "fused 3D contraction: more than 512 delay modes per line");
    // FFT buffers, twiddles, two spectrum stages, pair table, prefix and slot tables
    size_t lds = 2 * fa.nbu * ld * 8 + (size_t)M * 8 + 2 * 512 * 8 + (224 + 33 + 512) * 4;
    lds = std::max<size_t>(lds, 112 * 32 * 8);
    if (lds > 160 * 1024) return ctx_fail(c, BS_EUNSUPPORTED, "fused 3D contraction does not fit in LDS");
    e.lds = lds;
    // split-BF16: eta synthesis on MFMA over line groups of 16 x_u (fragments written by the u pass)
    std::vector<int> Sj, kb{0};
    int Smax = 0;
    for (int h : e.pd.hj) { Sj.push_back((h + 16) / 16); kb.push_back(kb.back() + Sj.back()); Smax = std::max(Smax, Sj.back()); }
    // fragment stage (+ a zero hi / lo pair), twiddles, synthesis schedule and every wave's field
    // rows (+ one zero row each)
    const size_t dlds = (size_t)(2 * kb.back() + 2) * 1024 + (size_t)M * 8 + (size_t)DFT_MAX_STEPS * DFT_SCHED * 4 +
                        (size_t)DFT_WAVES * (DFT_MAX_FIELDS + 1) * DFT_LDQ * 4;
    e.dft = e.precision == BS_SPLIT_BF16 && P.n % 16 == 0 && fa.nbu <= DFT_MAX_FIELDS && Smax <= DFT_MAX_STEPS &&
            dlds <= 160 * 1024 && (e.pd.NLu == 16 || e.pd.NLu == 8) && (M / 16) % DFT_WAVES == 0 &&
            nlines / 16 * kb.back() * 2048 < 0x80000000ll &&   // byte offsets into the fragment array
            !getenv("BS_3D_FFT");
    if (e.dft) {
      const long long ngroups = nlines / 16;
      std::vector<long long> offGs;
      long long tot = 0;
      for (int sj : Sj) { offGs.push_back(tot); tot += ngroups * sj * 128; }
      e.fd.Gs = ctx_ws(c, (tag + "_Gs").c_str(), (size_t)tot * 16);
      if (!e.fd.Gs) return ctx_fail(c, BS_ENOMEM, "workspace (spectrum fragments)");
      e.fd.d_offGs = upload(c, tag + "_offGs", offGs, rc); if (rc) return rc;
      // copy table, per stage fragment f = 2 kb[j] + s2: offset of group 0 (16-byte units), per-group
      // stride, and H_j - 16 (s2 / 2) (the lanes whose first mode 4 (lane / 16) lies above it copy nothing)
      std::vector<int> ctab;
      for (int j = 0; j < fa.nbu; ++j)
        for (int s2 = 0; s2 < 2 * Sj[j]; ++s2)
          ctab.insert(ctab.end(), {(int)(offGs[j] + 64 * s2), (int)(128 * Sj[j]), e.pd.hj[j] - 16 * (s2 >> 1), 0});
      e.fd.d_ctab = upload(c, tag + "_ctab", ctab, rc); if (rc) return rc;
      e.fd.gscale = fa.scale;
      Dft3Args& da = e.da;
      da = Dft3Args{};
      da.Gs = e.fd.Gs;
      da.ctab = e.fd.d_ctab;
      for (int j = 0; j < fa.nbu; ++j) { da.offGs[j] = offGs[j]; da.Sj[j] = Sj[j]; da.Hj[j] = e.pd.hj[j]; }
      for (int j = 0; j <= fa.nbu; ++j) da.kb[j] = kb[j];
      da.nbu = fa.nbu; da.n = P.n; da.M = M; da.Smax = Smax;
      da.W = ctx_dft_twiddle(c, M);
      if (!da.W) return ctx_fail(c, BS_ENOMEM, "eta twiddle fragments");
      da.pairs = e.d_pairs; da.npairs = e.npairs; da.ct1_tiles = e.ct1_tiles;
      da.ngroups = (int)ngroups;
      // BS_3D_DFT_BLOCKS / BS_3D_DFT_FLUSH (tests): fewer blocks and shorter flush intervals put
      // several line groups and flushes on every wave of a small cube
      const char* eb = getenv("BS_3D_DFT_BLOCKS");
      const char* ef = getenv("BS_3D_DFT_FLUSH");
      da.flush_vox = ef ? std::max(256, atoi(ef)) : 8192;
      e.dblocks = (int)std::min<long long>(ngroups, eb ? std::max(1, atoi(eb)) : 256);
      da.groups_per_block = (int)((ngroups + e.dblocks - 1) / e.dblocks);
      e.dblocks = (int)((ngroups + da.groups_per_block - 1) / da.groups_per_block);
      da.partial = e.partial;
      e.dlds = dlds;
    }
  } else {
    e.F = ctx_ws(c, (tag + "_F").c_str(), (size_t)e.blocks.size() * (e.fp64 ? e.vox64 * 8 : e.nvox * 4));
    if (!e.F) return ctx_fail(c, BS_ENOMEM, "workspace (fields)");
  }
  return BS_OK;
}

// Launches one estimate of the prepared plan on `vis` (no allocation, copy or synchronisation,
// so it may be captured into a graph).
int est3_enqueue(bs_ctx* c, const bs_bins* b, const void* vis, const bs_weights* w, Est3& e, double norm, double* B,
                 int64_t* N_tri, double* N_eff, const float* rho3_w) {
  if (e.ntri == 0) return BS_OK;
  int rc;
  int nparts = (int)(e.fp64 ? e.nblk64 : e.nblk);
  if (e.fused) {
    rc = fields3_enqueue(c, vis, w, e.pd, e.fd, nullptr);
    if (rc) return rc;
    if (c->timing) { (void)hipEventRecord(c->ev[5], c->stream); (void)hipEventRecord(c->ev[2], c->stream); }
    if (e.dft) {
      launch_dft3(e.da, e.dblocks, e.dlds, c->stream);
      LAUNCHCHK(c, "eta synthesis and contraction");
      nparts = e.dblocks;   // one summed slot per block (the first of its waves' slots)
    } else {
      launch_fused3(e.fa, e.precision == BS_FP32 ? 1 : 2, e.fblocks, e.lds, c->stream);
      LAUNCHCHK(c, "fused contraction");
      nparts = e.fblocks;
    }
  } else {
    rc = fields3_enqueue(c, vis, w, e.pd, e.fd, e.F);
    if (rc) return rc;
    if (c->timing) { (void)hipEventRecord(c->ev[5], c->stream); (void)hipEventRecord(c->ev[2], c->stream); }
    Con3Args ca{};
    ca.F = e.F; ca.vox = e.fp64 ? e.vox64 : e.nvox; ca.nbu = (int)e.blocks.size(); ca.pairs = e.d_pairs; ca.npairs = e.npairs;
    ca.chunk = e.fp64 ? e.chunk64 : e.chunk; ca.partial = e.partial; ca.ct1 = e.ct1_tiles; ca.flush = kCon64Flush;
    if (e.fp64) launch_contract64(ca, (int)e.nblk64, c->stream);
    else launch_contract3(ca, e.precision == BS_FP32 ? 1 : 2, (int)e.nblk, c->stream);
    LAUNCHCHK(c, "contraction");
  }
  if (c->timing) (void)hipEventRecord(c->ev[3], c->stream);
  Fin3Args f{};
  f.partial = e.partial; f.nparts = nparts; f.tri_pair = e.d_tp; f.tri_col = e.d_tc; f.ntri = e.ntri;
  if (e.fused && e.dft) f.pstride = DFT_WAVES;
  if (e.fp64 || (e.fused && e.dft)) f.nent = (e.npairs + 15) / 16 * 16 * 32;
  f.T3D = e.d_counts; f.rho3 = e.rho3; f.rho3_w = rho3_w; f.nc = b->P.nc; f.nvox = (double)e.nvox; f.norm = norm; f.sfac = e.sfac;
  f.B = B; f.N = N_tri; f.Neff = N_eff;
  launch_fin3(f, e.reduced, c->stream);
  LAUNCHCHK(c, "finalize");
  return BS_OK;
}

extern "C" int bs_estimate_3d(bs_ctx* c, const bs_bins* b, const void* vis, const bs_weights* w, int32_t precision,
                              double norm, double* B, int64_t* N_tri, double* N_eff) {
  if (!c || !b || !b->d_lut) return ctx_fail(c, BS_EINVAL, "bs_estimate_3d: NULL context or host-only bins");
  if (hipSetDevice(c->device) != hipSuccess) return ctx_fail(c, BS_EHIP, "hipSetDevice");
  int rc = check_3d_inputs(c, b, w);
  if (rc) return rc;
  if (!vis || !B || !N_tri) return ctx_fail(c, BS_EINVAL, "vis, B and N_tri must be non-NULL");
  if (precision < 0 || precision > 2) return ctx_fail(c, BS_EINVAL, "bad precision");
  if (c->timing) { (void)hipEventRecord(c->ev[0], c->stream); (void)hipEventRecord(c->ev[4], c->stream); }
  // Calls reuse the last prepared estimate (pair cover, work lists, uploaded tables: 1.3 ms of host work
  // on the 256^2 x 768 cube) as long as the bins, the uv mask's contents, precision and path switches
  // are the same and none of its workspaces has changed since.  The channel weights do not enter it: the kernels
  // read them, rho3 included.
  const bs_weights wm{nullptr, w ? w->uv_mask : nullptr, nullptr};
  uint64_t mask = 0;
  if (wm.uv_mask) {
    std::vector<uint8_t> hm((size_t)b->P.n * b->P.nh);
    HIPCHK(c, hipMemcpyAsync(hm.data(), wm.uv_mask, hm.size(), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    mask = hash_bytes3(b->P.hash, hm.data(), hm.size());
  }
  std::string key = std::to_string((uintptr_t)b) + ":" + std::to_string((uintptr_t)b->d_lut) + ":" +
                    std::to_string(b->P.hash) + ":" + std::to_string(precision) + (wm.uv_mask ? ":m" : ":") + std::to_string(mask);
  for (const char* k : {"BS_3D_FULLGRID", "BS_3D_UNFUSED", "BS_3D_ALLFFT", "BS_3D_FFT", "BS_3D_DFT_BLOCKS",
                        "BS_3D_DFT_FLUSH", "BS_FORCE_ENOMEM"}) {
    const char* v = getenv(k);
    key += std::string(":") + (v ? v : "-");
  }
  std::shared_ptr<Est3> held;
  if (c->est3 && c->est3_key == key && c->est3_gen == c->est3_ws_gen) {
    held = c->est3;
  } else {
    held = std::make_shared<Est3>();
    rc = est3_prepare(c, b, &wm, precision, PLAN3_TAG, *held);
    if (rc) return rc;
    // a replay of a captured call that planned anew copies that call's tables into the workspaces, so the
    // contents of the tables are unknown from then on and every call plans anew
    bool in_graph = false;
    for (const auto& kv : c->ws) in_graph = in_graph || (kv.second.in_graph && ctx_plan3_ws(kv.first));
    c->est3 = in_graph ? nullptr : held;
    c->est3_key = key;
    c->est3_gen = c->est3_ws_gen;
  }
  Est3& e = *held;
  if (e.ntri == 0) return BS_OK;
  c->last_count_dev = e.count_dev;
  c->last_count_bound = e.count_bound;
  rc = est3_enqueue(c, b, vis, w, e, norm, B, N_tri, N_eff, w ? w->chan_w : nullptr);
  if (rc) return rc;
  c->last_grid_M = e.M;
  c->last_flops_vox = 0.0;
  c->last_vox = 0.0;
  if (e.dft) {
    double modes = 0.0;
    for (int h : e.pd.hj) modes += h + 1;
    // synthesis: 3 bf16 products x 2 flops x 2 real modes per Hermitian mode; contraction: every
    // pair against the first 16 fields, the pairs serving a third shell of 16+ against all fields
    const double F = (double)e.blocks.size();
    c->last_flops_vox = 12.0 * modes + 6.0 * (e.npairs * std::min(F, 16.0) + e.nhigh * std::max(F - 16.0, 0.0));
    c->last_vox = (double)e.M * b->P.n * b->P.n;
  }
  if (c->timing) { (void)hipEventRecord(c->ev[1], c->stream); c->have_timing = true; }
  return BS_OK;
}

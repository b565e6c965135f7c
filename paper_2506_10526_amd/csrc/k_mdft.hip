// Eq. (dft): the 2D DFT that takes the ergodically collapsed MABS over the channel separations
// (dnu1, dnu2) = (n, m) channels to the cylindrical 3D bispectrum at (k_par1 a, k_par2 b).
// The sum runs over n, m in the half-open range [-L/2, L/2) (one period: the printed limits
// would count the end separation twice), i.e. a length-L DFT of the window laid out by residue,
// so each axis is one FP64 LDS FFT.  The input is real, hence the output is Hermitian: the pass
// along n keeps the half spectrum a < H = L/2 + 1 and the pass along m writes row L - a as the
// mirror of row a, so that the output leaves in whole contiguous rows.
#include <hip/hip_runtime.h>

#include "bs_kernels.h"

namespace {

using C = Cx<double>;
constexpr int MDFT_THREADS = 512;   // largest block; the host picks 256 or 512
constexpr int MDFT_M_THREADS = 256; // pass m of a compile-time length
constexpr int MDFT_NB = 8;          // loads in flight per thread

// array index of separation d in [-h, h]: non-circular collapse at d + L - 1, circular at d mod L
__device__ __forceinline__ int sep_index(const MdftArgs& a, int d) { return a.circ ? (d < 0 ? d + a.L : d) : d + a.L - 1; }

// LDS line stride: r mod 16 elements
constexpr __host__ __device__ int mdft_ld(int L, int r) { return L + (16 + r - L % 16) % 16; }

__device__ __forceinline__ double nan0(double v) { return v == v ? v : 0.0; }

// Window entry at residues (r, c): separations n = r and m = c below L - h, else r - L and c - L,
// so that n, m run over [-h, L - 1 - h], one period with each separation once.
__device__ __forceinline__ double window_at(const MdftArgs& a, const double* __restrict__ Bt, int r, int c) {
  const int lim = a.L - 1 - a.h;
  const int rm = sep_index(a, r <= lim ? r : r - a.L), cm = sep_index(a, c <= lim ? c : c - a.L);
  return nan0(Bt[(long long)rm * a.S + cm]);
}

// Both passes loop over work groups (triangle, block of lines) so that each block copies the
// twiddle table into LDS once.  Blocks take groups in a strided order: the groups in flight at any
// time are neighbours, which keeps the HBM accesses of the whole grid on a narrow band of pages.
//
// Pass n deals each XCD one contiguous eighth of the groups, in that order: a group's rows are runs of 64
// bytes that start anywhere in a line, and the neighbour that holds the rest of the line meets it in the same
// L2 (dealt to the XCDs in turn, the pass fetched 2.9 times its input).
//
// Pass n: W = 2 CB window columns (residues) c0 .. c0 + W - 1 per group, columns 2q and 2q + 1 packed
// into complex line q (z = x0 + i x1), transformed along n; the half spectra a < H of both columns
// go to Y[t][a][c] (runs of W contiguous entries per a).
// LC: the length at compile time (four column pairs, 512 threads, all of a thread's loads in flight at once), 0:
// any.  Bound: HBM (8 bytes in, 8 out per window entry).  133 x 768^2: 500 us with the run-time transform
// and groups dealt to the XCDs in turn, now 356 (3.7 TB/s).  Blocks of 256
// threads or two column pairs, a prefetch of the next group and slices of triangles whose half spectra
// stay in the 256 MB cache between the passes were all slower.
template <int BM, int LC>
__global__ __launch_bounds__(MDFT_THREADS) void k_mdft_n(MdftArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int L = LC ? LC : a.L, H = L / 2 + 1, CB = LC ? 4 : a.nl, lg = LC ? 3 : a.lgnl + 1;
  const int ld = LC ? mdft_ld(LC, 4) : a.ld, TH = LC ? MDFT_THREADS : (int)blockDim.x;
  constexpr int NB = LC ? (8 * LC + MDFT_THREADS - 1) / MDFT_THREADS : MDFT_NB;
  const int W = 2 * CB;
  C* A = reinterpret_cast<C*>(smem);
  C* tw = A + CB * ld;
  double* Ad = reinterpret_cast<double*>(A);
  const C* __restrict__ twg = static_cast<const C*>(a.tw);
  for (int i = threadIdx.x; i < L; i += TH) tw[i] = twg[i];
  const int gx = (L + W - 1) / W;
  const int total = W * L;
  int g0 = blockIdx.x, step = gridDim.x, ge = a.nt * gx;
  if constexpr (LC) {   // gridDim.x is a multiple of 8 (fewer groups than that leave blocks without work)
    const int per = (ge + 7) / 8, x0 = (int)(blockIdx.x & 7) * per;
    g0 = x0 + (int)(blockIdx.x >> 3);
    step = gridDim.x >> 3;
    ge = x0 + per < ge ? x0 + per : ge;
  }
  for (int g = g0; g < ge; g += step) {
    const int t = g / gx;
    const int c0 = (g - t * gx) * W;
    const double* __restrict__ Bt = a.B + (long long)t * a.S * a.S;
    // consecutive threads take consecutive columns of one row (W * 8 contiguous bytes); the first
    // chunk is loaded by every thread before the barrier that frees the previous group's lines
    auto load = [&](int base, double* v) {
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const int i = base + u * TH;
        const int c = c0 + (i & (W - 1));
        v[u] = i < total && c < L ? window_at(a, Bt, i >> lg, c) : 0.0;
      }
    };
    auto store = [&](int base, const double* v) {
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const int i = base + u * TH;
        const int k = i & (W - 1);
        if (i < total) Ad[2 * ((k >> 1) * ld + (i >> lg)) + (k & 1)] = v[u];
      }
    };
    double v[NB];
    load(threadIdx.x, v);
    __syncthreads();
    store(threadIdx.x, v);
    if constexpr (!LC) for (int base = threadIdx.x + NB * TH; base < total; base += NB * TH) {
      load(base, v);
      store(base, v);
    }
    __syncthreads();
    if constexpr (LC) lds_fft_ct<-1, double, LC, 4, MDFT_THREADS, mdft_ld(LC, 4)>(A, 4, tw, 1);
    else lds_fft_ip<-1, double, BM>(A, a.plan, CB, tw, 1, ld);
    // z = x0 + i x1 transformed: X0[a] = (Z[a] + conj Z[-a]) / 2, X1[a] = (Z[a] - conj Z[-a]) / (2i)
    C* __restrict__ Y = static_cast<C*>(a.X) + (long long)t * H * L;
    for (int i = threadIdx.x; i < W * H; i += TH) {
      const int k = i & (W - 1), e = i >> lg;
      const int c = c0 + k;
      if (c >= L) continue;
      const C* line = A + (k >> 1) * ld;
      const C z = line[e];
      const C zm = cconj(line[e ? L - e : 0]);
      C y;
      if (k & 1) {
        const C d = csub(z, zm);
        y = cmk(0.5 * d.y, -0.5 * d.x);
      } else {
        y = cscale(cadd(z, zm), 0.5);
      }
      Y[(long long)e * L + c] = y;
    }
  }
}

// Pass m: NL rows a < H of Y per group, transformed along m, scaled; row a of the output and its
// Hermitian mirror, row L - a, are written whole.  LC: as in pass n (two rows, 256 threads).  Bound: HBM (16
// bytes in, 32 out per half-spectrum entry); 133 x 768^2: 376 us before, now 339, 5.6 TB/s; shorter lengths were
// bound by the index arithmetic of the run-time transform (133 x 192^2: 21 us less).
template <int BM, int LC>
__global__ __launch_bounds__(MDFT_THREADS) void k_mdft_m(MdftArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  C* tw = reinterpret_cast<C*>(smem);
  C* A = tw + (LC ? LC : a.L);
  const int L = LC ? LC : a.L, H = L / 2 + 1, NL = LC ? 2 : a.nl, TH = LC ? MDFT_M_THREADS : (int)blockDim.x;
  constexpr int NB = LC ? (2 * LC + MDFT_M_THREADS - 1) / MDFT_M_THREADS : MDFT_NB;
  const C* __restrict__ twg = static_cast<const C*>(a.tw);
  for (int i = threadIdx.x; i < L; i += TH) tw[i] = twg[i];
  const float rL = 1.0f / (float)L;
  const int gx = (H + NL - 1) / NL;
  const int total = NL * L;
  const double sc = a.scale;
  for (int g = blockIdx.x; g < a.nt * gx; g += gridDim.x) {
    const int t = g / gx;
    const int e0 = (g - t * gx) * NL;
    const C* __restrict__ Y = static_cast<const C*>(a.X) + (long long)t * H * L;
    auto load = [&](int base, C* v) {
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const int i = base + u * TH;
        int p, c;
        if constexpr (LC) { p = i / LC; c = i % LC; } else fdivmod(i, L, rL, p, c);
        v[u] = i < total && e0 + p < H ? Y[(long long)(e0 + p) * L + c] : cmk(0.0, 0.0);
      }
    };
    auto store = [&](int base, const C* v) {
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const int i = base + u * TH;
        if (i < total) A[i] = v[u];
      }
    };
    C v[NB];
    load(threadIdx.x, v);
    __syncthreads();
    store(threadIdx.x, v);
    for (int base = threadIdx.x + NB * TH; base < total; base += NB * TH) {
      load(base, v);
      store(base, v);
    }
    __syncthreads();
    if constexpr (LC) lds_fft_ct<-1, double, LC, 2, MDFT_M_THREADS, LC>(A, 2, tw, 1);
    else lds_fft_ip<-1, double, BM>(A, a.plan, NL, tw, 1, L);
    C* __restrict__ out = static_cast<C*>(a.out) + (long long)t * L * L;
    for (int i = threadIdx.x; i < total; i += TH) {
      int p, b;
      if constexpr (LC) { p = i / LC; b = i % LC; } else fdivmod(i, L, rL, p, b);
      const int e = e0 + p;
      if (e >= H) continue;
      const C val = cscale(A[i], sc);
      out[(long long)e * L + b] = val;
      // real input: out(-a, -b) = conj out(a, b) fills the rows a >= H
      if (e >= 1 && L - e >= H) out[(long long)(L - e) * L + (b ? L - b : 0)] = cconj(val);
    }
  }
}

void launch_mdft(void (*k)(MdftArgs), int grid, size_t lds, const MdftArgs& a, hipStream_t s) {
  (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(k, dim3(grid), dim3(a.threads), lds, s, a);
}

// Compile-time lengths: 2^a, 3 2^a and 9 2^a from 64 to 1024 (the band sizes in use and their averages over 2, 4
// and 8 channels).  Run-time transform against this one at 133 (74) triangles, us: 96 45 / 21, 192 87 / 43,
// 384 265 / 181, 768 844 / 678, 1024 1190 / 875.
template <int LC>
void pick(const MdftArgs& a, void (**n)(MdftArgs), void (**m)(MdftArgs)) {
  if (a.L != LC || !fft_ct_plan(a.plan, LC)) return;
  *n = k_mdft_n<2, LC>;
  *m = k_mdft_m<2, LC>;
}
bool pick_any(const MdftArgs& a, void (**n)(MdftArgs), void (**m)(MdftArgs)) {
  *n = *m = nullptr;
  pick<64>(a, n, m);
  pick<96>(a, n, m);
  pick<128>(a, n, m);
  pick<144>(a, n, m);
  pick<192>(a, n, m);
  pick<256>(a, n, m);
  pick<288>(a, n, m);
  pick<384>(a, n, m);
  pick<512>(a, n, m);
  pick<576>(a, n, m);
  pick<768>(a, n, m);
  pick<1024>(a, n, m);
  return *n;
}

}  // namespace

void launch_mdft_n(const MdftArgs& a, size_t lds, hipStream_t s) {
  const int groups = a.nt * ((a.L + 2 * a.nl - 1) / (2 * a.nl));
  const int grid = a.grid < groups ? a.grid : groups;
  void (*n)(MdftArgs), (*m)(MdftArgs);
  // two blocks a CU, so that the groups in flight of an XCD are neighbours (768: 686 us a call, 704 with eight)
  if (a.nl == 4 && a.threads == MDFT_THREADS && a.ld == mdft_ld(a.L, 4) && pick_any(a, &n, &m))
    launch_mdft(n, ((grid < 512 ? grid : 512) + 7) / 8 * 8, lds, a, s);
  else launch_mdft(a.bm == 2 ? k_mdft_n<2, 0> : k_mdft_n<4, 0>, grid, lds, a, s);
}

void launch_mdft_m(const MdftArgs& a, size_t lds, hipStream_t s) {
  const int groups = a.nt * ((a.H + a.nl - 1) / a.nl);
  const int grid = a.grid < groups ? a.grid : groups;
  void (*n)(MdftArgs), (*m)(MdftArgs);
  // a block a group: with no tail of a strided loop, and the dispatcher's order (768: 15 us less than 4096 blocks)
  if (a.nl == 2 && a.threads == MDFT_M_THREADS && pick_any(a, &n, &m)) launch_mdft(m, groups < 1 << 22 ? groups : 1 << 22, lds, a, s);
  else launch_mdft(a.bm == 2 ? k_mdft_m<2, 0> : k_mdft_m<4, 0>, grid, lds, a, s);
}

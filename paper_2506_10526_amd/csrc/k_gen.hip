// Seeded synthetic cubes on the GPU and the Monte Carlo accumulators.
//
// A realization is the quadratic non-Gaussian field of the validation set-up (Sec. 4, Eq. mb1)
// built from counter-based white noise:
//   white(i), i = (z n + x) n + y: Philox4x64-10 (Salmon et al. 2011) with key (seed, realization)
//     and counter (i / 4, 0, 0, 0); the four 64-bit outputs give 24-bit uniforms
//     u_j = ((x_j >> 40) + 1/2) 2^-24 and two Box-Muller pairs for voxels 4c .. 4c+3;
//   g = irfftn(rfftn(white) sqrt(A P(k))), P = (k^2)^(index/2), P(0) = 0, A = sigma^2 N / sum P;
//   delta = g + f (g^2 - mean g^2);  V[z] = rfft2(delta[z]) w(z)   (complex64 [nc][n][n/2+1]).
//
// Passes (every one an LDS-staged Stockham transform of a group of lines):
//   rows_white : white noise generated in registers, two real rows packed as one complex row,
//                forward FFT along y, split into the two half spectra               -> W
//   axis<0>    : forward C2C along x                                                 (W in place)
//   axis<2>    : forward C2C along z, times sqrt(A P(k)), inverse C2C along z        (W in place)
//   axis<1>    : inverse C2C along x                                                 (W in place)
//   rows_mid   : two half spectra packed as one complex row, inverse FFT along y -> g, sum g^2; in the same
//                block g + f (g^2 - sigma^2), forward FFT along y, split              (W in place)
//   mean       : mean g^2 (fixed-order reduction)
//   axis<3>    : forward C2C along x, the sample mean's share -f (mean g^2 - sigma^2) n^2 of the one cell q = 0
//                of each channel, times w(z)                                          (W in place)
// W is the caller's output cube; g never leaves LDS (writing it out to subtract the sample mean before the
// transform took two more passes over the cube).  Bound: HBM, 2.2 GB at 256^2 x 768 (each pass reads and
// writes W), except rows_white, which is bound by Philox's 64-bit products.  256^2 x 768: 1544 us
// with eight passes, run-time FFT plans and 120 us of sum P, now 950 (white 161, x 128 each, z 211, mid 190,
// sum P 23).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "bs_gen.h"
#include "fft_lds.h"

namespace {

typedef Cx<float> C;

// ---------------------------------------------------------------- Philox4x64-10
struct U4 {
  unsigned long long v[4];
};

__device__ __forceinline__ U4 philox4x64_10(unsigned long long c0, unsigned long long k0, unsigned long long k1) {
  const unsigned long long M0 = 0xD2E7470EE14C6C93ULL, M1 = 0xCA5A826395121157ULL;
  const unsigned long long W0 = 0x9E3779B97F4A7C15ULL, W1 = 0xBB67AE8584CAA73BULL;
  unsigned long long x0 = c0, x1 = 0, x2 = 0, x3 = 0;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) { k0 += W0; k1 += W1; }
    // one 64 x 64 -> 128 product each (high and low halves from the same partial products)
    const unsigned __int128 p0 = (unsigned __int128)x0 * M0, p1 = (unsigned __int128)x2 * M1;
    x0 = (unsigned long long)(p1 >> 64) ^ x1 ^ k0;
    x1 = (unsigned long long)p1;
    x2 = (unsigned long long)(p0 >> 64) ^ x3 ^ k1;
    x3 = (unsigned long long)p0;
  }
  U4 o;
  o.v[0] = x0; o.v[1] = x1; o.v[2] = x2; o.v[3] = x3;
  return o;
}

__device__ __forceinline__ float u24(unsigned long long x) {
  return ((float)(unsigned)(x >> 40) + 0.5f) * 5.9604644775390625e-8f;  // 2^-24
}

// Four standard normals of voxels 4c .. 4c+3.
__device__ __forceinline__ void normals4(unsigned long long c, unsigned long long seed, unsigned long long real,
                                         float* z) {
  U4 x = philox4x64_10(c, seed, real);
  const float r01 = sqrtf(-2.0f * logf(u24(x.v[0])));
  const float r23 = sqrtf(-2.0f * logf(u24(x.v[2])));
  float s, co;
  sincospif(2.0f * u24(x.v[1]), &s, &co);
  z[0] = r01 * co;
  z[1] = r01 * s;
  sincospif(2.0f * u24(x.v[3]), &s, &co);
  z[2] = r23 * co;
  z[3] = r23 * s;
}

__device__ __forceinline__ int signed_idx(int i, int m) { return i < (m + 1) / 2 ? i : i - m; }

// sqrt(A P(k)) for k^2 (float); P(0) = 0.
__device__ __forceinline__ float spec_amp(float k2, float sqrtA, float e4, int m2) {
  if (k2 <= 0.f) return 0.f;
  return m2 ? sqrtA / sqrtf(k2) : sqrtA * powf(k2, e4);
}

// ---------------------------------------------------------------- sum of P over the full grid
// P depends on |q| alone, so block z (|q_z| = z <= nc / 2) sums the quadrant q_x, q_y >= 0 with the number
// of grid points each cell stands for.
__device__ __forceinline__ double mult_of(int q, int m) { return q == 0 || 2 * q == m ? 1.0 : 2.0; }
__global__ __launch_bounds__(256) void k_gen_psum(GenArgs a) {
  const int z = blockIdx.x, h = a.n / 2 + 1;
  const double kz = a.cz * (double)z;
  double s = 0.0;
  for (int t = threadIdx.x; t < h * h; t += 256) {
    const int x = t / h, y = t - x * h;
    const double kx = a.cxy * (double)x, ky = a.cxy * (double)y;
    const double k2 = kz * kz + kx * kx + ky * ky;
    if (k2 > 0.0) s += mult_of(x, a.n) * mult_of(y, a.n) * (a.m2 ? 1.0 / k2 : pow(k2, 0.5 * a.index));
  }
  __shared__ double red[256];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) a.part[z] = mult_of(z, a.nc) * red[0];
}

// sqrtA = sqrt(sigma^2 N / sum P), the nc / 2 + 1 partials summed in a fixed order.
__global__ __launch_bounds__(256) void k_gen_amp(GenArgs a) {
  __shared__ double red[256];
  double s = 0.0;
  for (int z = threadIdx.x; z <= a.nc / 2; z += 256) s += a.part[z];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  s = red[0];
  const double nvox = (double)a.nc * a.n * a.n;
  a.stat[0] = s > 0.0 ? sqrt(a.sigma * a.sigma * nvox / s) : 0.0;
}

// ---------------------------------------------------------------- rows along y
// Block: NL row pairs (rows 2p, 2p+1, p = blockIdx.x NL + l), packed as one complex row each.
// L: n when lds_fft_ct transforms the rows (16 pairs a block), else 0; IP: in-place FFT bound
// (butterflies per thread) of the run-time plan, 0 = two buffers.
constexpr int GEN_ROWS = 16;
// (Twiddles from the global table: staged in LDS the row passes ran 5 % slower, fewer blocks a CU.)
template <int SIGN, int IP, int L>
__device__ __forceinline__ C* gen_row_fft(const GenArgs& a, C* A, C* B, int nl) {
  const C* tw = (const C*)a.tw_n;
  if constexpr (L > 0) { lds_fft_ct<SIGN, float, L, GEN_ROWS, 256, L + 1>(A, nl, tw, 1); return A; }
  else if constexpr (IP > 0) { lds_fft_ip<SIGN, float, IP>(A, a.pn, nl, tw, 1, a.n + 1); return A; }
  else return lds_fft<SIGN, float>(A, B, a.pn, nl, tw, 1, a.n + 1);
}

// the two real rows' half spectra from Z = X0 + i X1
template <int L>
__device__ __forceinline__ void gen_row_split(const GenArgs& a, const C* R, long long p0, int nl) {
  const int n = L ? L : a.n, nh = n / 2 + 1, ld = n + 1;
  for (int t = threadIdx.x; t < nl * nh; t += 256) {
    const int l = t / nh, k = t - l * nh;
    const C zk = R[l * ld + k];
    const C zm = R[l * ld + (k ? n - k : 0)];
    C x0, x1;
    x0.x = 0.5f * (zk.x + zm.x);
    x0.y = 0.5f * (zk.y - zm.y);
    x1.x = 0.5f * (zk.y + zm.y);
    x1.y = -0.5f * (zk.x - zm.x);
    const long long row = 2 * (p0 + l);
    a.W[row * nh + k] = x0;
    a.W[(row + 1) * nh + k] = x1;
  }
}

template <int IP, int L>
__global__ __launch_bounds__(256) void k_gen_rows_white(GenArgs a) {
  extern __shared__ unsigned char smem[];
  const int n = L ? L : a.n, ld = n + 1, NL = L ? GEN_ROWS : a.NL;
  C* bufA = (C*)smem;
  C* bufB = bufA + (size_t)NL * ld;
  const long long npairs = (long long)a.nc * n / 2;
  const long long p0 = (long long)blockIdx.x * NL;
  const int nl = (int)((npairs - p0) < NL ? (npairs - p0) : NL);
  const unsigned long long seed = a.state[0], real = a.state[1];
  const int chunks = n / 4;
  for (int t = threadIdx.x; t < nl * chunks; t += 256) {
    const int l = t / chunks, ch = t - l * chunks;
    const long long row = 2 * (p0 + l);
    float z0[4], z1[4];
    normals4((unsigned long long)((row * n) / 4 + ch), seed, real, z0);
    normals4((unsigned long long)(((row + 1) * n) / 4 + ch), seed, real, z1);
#pragma unroll
    for (int q = 0; q < 4; ++q) bufA[l * ld + 4 * ch + q] = C{z0[q], z1[q]};
  }
  __syncthreads();
  gen_row_split<L>(a, gen_row_fft<-1, IP, L>(a, bufA, bufB, nl), p0, nl);
}

// Inverse along y of two half spectra at once, per-block partial sums of g^2, then the quadratic field
// about sigma^2 and forward along y again.
template <int IP, int L>
__global__ __launch_bounds__(256) void k_gen_rows_mid(GenArgs a) {
  extern __shared__ unsigned char smem[];
  const int n = L ? L : a.n, nh = n / 2 + 1, ld = n + 1, NL = L ? GEN_ROWS : a.NL;
  C* bufA = (C*)smem;
  C* bufB = bufA + (size_t)NL * ld;
  const long long npairs = (long long)a.nc * n / 2;
  const long long p0 = (long long)blockIdx.x * NL;
  const int nl = (int)((npairs - p0) < NL ? (npairs - p0) : NL);
  // k and n - k from one pair of entries (self-conjugate terms are real); eight in flight
  for (int t0 = threadIdx.x; t0 < nl * nh; t0 += 8 * 256) {
    C x0[8], x1[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int t = t0 + 256 * u, l = t / nh, k = t - l * nh;
      if (t < nl * nh) {
        const C* row = a.W + 2 * (p0 + l) * nh + k;
        x0[u] = row[0];
        x1[u] = row[nh];
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int t = t0 + 256 * u, l = t / nh, k = t - l * nh;
      if (t >= nl * nh) break;
      if (k == 0 || 2 * k == n) { x0[u].y = 0.f; x1[u].y = 0.f; }
      C* line = bufA + l * ld;
      line[k] = C{x0[u].x - x1[u].y, x0[u].y + x1[u].x};
      if (k > 0 && 2 * k < n) line[n - k] = C{x0[u].x + x1[u].y, x1[u].x - x0[u].y};
    }
  }
  __syncthreads();
  C* R = gen_row_fft<1, IP, L>(a, bufA, bufB, nl);
  const float sc = (float)(1.0 / ((double)a.nc * n * n));
  const float f = (float)a.fng, m = (float)(a.sigma * a.sigma);
  double s2 = 0.0;
  for (int t = threadIdx.x; t < nl * n; t += 256) {
    const int l = t / n, y = t - l * n;
    const C z = R[l * ld + y];
    const float g0 = z.x * sc, g1 = z.y * sc;
    s2 += (double)g0 * g0 + (double)g1 * g1;
    R[l * ld + y] = C{g0 + f * (g0 * g0 - m), g1 + f * (g1 * g1 - m)};
  }
  __shared__ double red[256];
  red[threadIdx.x] = s2;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) a.part[blockIdx.x] = red[0];
  gen_row_split<L>(a, gen_row_fft<-1, IP, L>(a, R, R == bufA ? bufB : bufA, nl), p0, nl);
}

// stat[1] = mean g^2 over the nparts block sums (fixed order).
__global__ __launch_bounds__(256) void k_gen_mean(GenArgs a, int nparts) {
  __shared__ double red[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < nparts; i += 256) s += a.part[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) a.stat[1] = red[0] / ((double)a.nc * a.n * a.n);
}

// ---------------------------------------------------------------- C2C along a strided axis
// Lines: the W elements (o, l, b) with l the transform index; o in [0, outer), b in [0, inner),
// address (o L + l) inner + b.  A block takes NL consecutive lines of the flattened (o, b) order,
// so consecutive lines are consecutive addresses.
// OP 0: forward; 1: inverse; 2: forward, times sqrt(A P), inverse (z axis, outer = 1);
// 3: forward, cell q = 0 corrected for the sample mean, times w(o) (x axis, o = z).
// IP > 0: in-place FFT with at most IP butterflies per thread (one line buffer), else two buffers.
// CT > 0: L when lds_fft_ct transforms gen_lines(CT) lines a block.  Neighbouring blocks, whose pieces of
// NL elements share cache lines, run on one XCD.
constexpr int gen_lines(int L, bool z) {
  int nl = 16;
  while (z && nl > 1 && nl * (L + 2) * 8 > 32 * 1024) nl /= 2;
  return nl;
}
__device__ __forceinline__ int gen_xcd_block(int id, int nb) {
  const int q = nb >> 3, r = nb & 7, x = id & 7, j = id >> 3;
  return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + j;
}
struct GenLine {
  long long base;
  float p, q;
};
template <int OP, int IP, int CT>
__global__ __launch_bounds__(256) void k_gen_axis(GenArgs a, int L_, int outer, int inner, int NL_) {
  extern __shared__ unsigned char smem[];
  const int L = CT ? CT : L_, NL = CT ? gen_lines(CT, OP == 2) : NL_;
  const int ld = L + 1;
  C* bufA = (C*)smem;
  C* bufB = bufA + (size_t)NL * ld;
  // per line: address, and what its elements need beside it (2: k_x and k_y; 3: weight, mean correction)
  GenLine* ln = (GenLine*)(bufA + (size_t)NL * ld * (IP > 0 ? 1 : 2));
  // the x passes keep their table in LDS (137 -> 128 us at 256^2 x 768); the z pass reads the global one
  // (its blocks' LDS bounds how many a CU holds: 214 -> 245 us with the table in it)
  const C* tw = (const C*)(L == a.n ? a.tw_n : a.tw_nc);
  if constexpr (OP != 2) {
    C* twl = (C*)(ln + NL);
    for (int i = threadIdx.x; i < L; i += 256) twl[i] = tw[i];
    tw = twl;
  }
  const long long nlines = (long long)outer * inner;
  const long long g0 = (long long)gen_xcd_block(blockIdx.x, gridDim.x) * NL;
  const int nl = (int)((nlines - g0) < NL ? (nlines - g0) : NL);
  if ((int)threadIdx.x < nl) {
    const long long gl = g0 + threadIdx.x;
    const long long o = gl / inner, b = gl - o * inner;
    GenLine q;
    q.base = o * (long long)L * inner + b;
    q.p = q.q = 0.f;
    if (OP == 2) {   // outer == 1: line = x nh + y
      const int x = (int)(gl / a.nh), y = (int)(gl - (long long)x * a.nh);
      q.p = (float)(a.cxy * signed_idx(x, a.n));
      q.q = (float)(a.cxy * y);
    } else if (OP == 3) {
      q.p = a.chw ? a.chw[o] : 1.f;
      // delta was formed about sigma^2 instead of the sample mean: the difference is a constant, so it
      // is the one cell q = 0 of the channel that changes
      if (b == 0) q.q = (float)(a.fng * (a.stat[1] - (double)(float)(a.sigma * a.sigma)) * a.n * a.n);
    }
    ln[threadIdx.x] = q;
  }
  __syncthreads();
  // eight loads in flight per thread before their LDS stores
  for (int t0 = threadIdx.x; t0 < L * NL; t0 += 8 * 256) {
    C v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int t = t0 + u * 256, l = t / NL, bl = t - l * NL;
      if (t < L * NL && bl < nl) v[u] = a.W[ln[bl].base + (long long)l * inner];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int t = t0 + u * 256, l = t / NL, bl = t - l * NL;
      if (t < L * NL && bl < nl) bufA[(size_t)bl * ld + l] = v[u];
    }
  }
  __syncthreads();
  const FftPlan& pl = (L == a.n) ? a.pn : a.pnc;
  C* R = bufA;
  if constexpr (CT > 0) {
    lds_fft_ct<OP == 1 ? 1 : -1, float, CT, gen_lines(CT, OP == 2), 256, CT + 1>(bufA, nl, tw, 1);
  } else if constexpr (IP > 0) {
    if (OP == 1) lds_fft_ip<1, float, IP>(bufA, pl, nl, tw, 1, ld);
    else lds_fft_ip<-1, float, IP>(bufA, pl, nl, tw, 1, ld);
  } else if (OP == 1) {
    R = lds_fft<1, float>(bufA, bufB, pl, nl, tw, 1, ld);
  } else {
    R = lds_fft<-1, float>(bufA, bufB, pl, nl, tw, 1, ld);
  }
  if (OP == 2) {
    const float sqrtA = (float)a.stat[0];
    const float e4 = (float)(0.25 * a.index);
    for (int t = threadIdx.x; t < L * nl; t += 256) {
      const int bl = t / L, l = t - bl * L;
      const float kz = (float)(a.cz * signed_idx(l, a.nc)), kx = ln[bl].p, ky = ln[bl].q;
      const float s = spec_amp(kz * kz + kx * kx + ky * ky, sqrtA, e4, a.m2);
      R[(size_t)bl * ld + l] = cscale(R[(size_t)bl * ld + l], s);
    }
    __syncthreads();
    if constexpr (CT > 0) {
      lds_fft_ct<1, float, CT, gen_lines(CT, true), 256, CT + 1>(R, nl, tw, 1);
    } else if constexpr (IP > 0) {
      lds_fft_ip<1, float, IP>(R, pl, nl, tw, 1, ld);
    } else {
      C* other = (R == bufA) ? bufB : bufA;
      R = lds_fft<1, float>(R, other, pl, nl, tw, 1, ld);
    }
  }
  for (int t = threadIdx.x; t < L * NL; t += 256) {
    const int l = t / NL, bl = t - l * NL;
    if (bl < nl) {
      C v = R[(size_t)bl * ld + l];
      if (OP == 3) {
        if (l == 0) v.x -= ln[bl].q;
        v = cscale(v, ln[bl].p);
      }
      a.W[ln[bl].base + (long long)l * inner] = v;
    }
  }
}

// ---------------------------------------------------------------- Monte Carlo accumulators
// Welford update of the per-triangle mean and M2 with one realization's B (NaN entries skipped),
// then the realization counter of the generator state advances by one.
__global__ __launch_bounds__(256) void k_mc_accumulate(const double* __restrict__ B, int ntri,
                                                      long long* __restrict__ cnt, double* __restrict__ mean,
                                                      double* __restrict__ m2, unsigned long long* state) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t < ntri) {
    const double b = B[t];
    if (b == b) {
      const long long k = cnt[t] + 1;
      const double d = b - mean[t];
      const double mu = mean[t] + d / (double)k;
      m2[t] += d * (b - mu);
      mean[t] = mu;
      cnt[t] = k;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) state[1] += 1ULL;
}

__global__ void k_mc_zero(long long* cnt, double* mean, double* m2, int ntri) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t < ntri) { cnt[t] = 0; mean[t] = 0.0; m2[t] = 0.0; }
}

__global__ void k_gen_set_state(unsigned long long* state, unsigned long long seed, unsigned long long real) {
  if (threadIdx.x == 0 && blockIdx.x == 0) { state[0] = seed; state[1] = real; }
}

template <typename K>
void set_lds(K k, size_t lds) {
  (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

}  // namespace

// ---------------------------------------------------------------- launchers
void launch_gen_amp(const GenArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_gen_psum, dim3(a.nc / 2 + 1), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_gen_amp, dim3(1), dim3(256), 0, s, a);
}

void launch_gen_set_state(unsigned long long* state, unsigned long long seed, unsigned long long real, hipStream_t s) {
  hipLaunchKernelGGL(k_gen_set_state, dim3(1), dim3(64), 0, s, state, seed, real);
}

template <int OP, int IP, int CT>
static void launch_axis_t(const GenArgs& a, int nb, size_t lds, hipStream_t s, int L, int outer, int inner, int NL) {
  set_lds(k_gen_axis<OP, IP, CT>, lds);
  hipLaunchKernelGGL((k_gen_axis<OP, IP, CT>), dim3(nb), dim3(256), lds, s, a, L, outer, inner, NL);
}
// compile-time transforms: uv grids of 48 to 256, bands of 96 2^k and 128 2^k channels
template <int OP>
static void launch_axis(const GenArgs& a, int ip, int nb, size_t lds, hipStream_t s, int L, int outer, int inner, int NL) {
  const FftPlan& pl = OP == 2 ? a.pnc : a.pn;
  const int ct = ip > 0 && fft_ct_plan(pl, L) && NL == gen_lines(L, OP == 2) ? L : 0;
  if constexpr (OP == 2) {
    if (ct == 96) return launch_axis_t<OP, 2, 96>(a, nb, lds, s, L, outer, inner, NL);
    if (ct == 192) return launch_axis_t<OP, 2, 192>(a, nb, lds, s, L, outer, inner, NL);
    if (ct == 384) return launch_axis_t<OP, 2, 384>(a, nb, lds, s, L, outer, inner, NL);
    if (ct == 512) return launch_axis_t<OP, 2, 512>(a, nb, lds, s, L, outer, inner, NL);
    if (ct == 576) return launch_axis_t<OP, 2, 576>(a, nb, lds, s, L, outer, inner, NL);
    if (ct == 768) return launch_axis_t<OP, 2, 768>(a, nb, lds, s, L, outer, inner, NL);
  }
  if constexpr (OP != 2) {
    if (ct == 48) return launch_axis_t<OP, 2, 48>(a, nb, lds, s, L, outer, inner, NL);
    if (ct == 64) return launch_axis_t<OP, 2, 64>(a, nb, lds, s, L, outer, inner, NL);
    if (ct == 96) return launch_axis_t<OP, 2, 96>(a, nb, lds, s, L, outer, inner, NL);
    if (ct == 192) return launch_axis_t<OP, 2, 192>(a, nb, lds, s, L, outer, inner, NL);
  }
  if (ct == 128) return launch_axis_t<OP, 2, 128>(a, nb, lds, s, L, outer, inner, NL);
  if (ct == 256) return launch_axis_t<OP, 2, 256>(a, nb, lds, s, L, outer, inner, NL);
  if (ip == 2) launch_axis_t<OP, 2, 0>(a, nb, lds, s, L, outer, inner, NL);
  else if (ip == 4) launch_axis_t<OP, 4, 0>(a, nb, lds, s, L, outer, inner, NL);
  else launch_axis_t<OP, 0, 0>(a, nb, lds, s, L, outer, inner, NL);
}

int gen_row_blocks(const GenArgs& a) {
  const long long npairs = (long long)a.nc * a.n / 2;
  return (int)((npairs + a.NL - 1) / a.NL);
}

template <int IP, int L>
static void launch_rows_t(const GenArgs& a, bool mid, int rb, size_t lds, hipStream_t s) {
  if (mid) { set_lds(k_gen_rows_mid<IP, L>, lds); hipLaunchKernelGGL((k_gen_rows_mid<IP, L>), dim3(rb), dim3(256), lds, s, a); }
  else { set_lds(k_gen_rows_white<IP, L>, lds); hipLaunchKernelGGL((k_gen_rows_white<IP, L>), dim3(rb), dim3(256), lds, s, a); }
}
static void launch_rows(const GenArgs& a, bool mid, int rb, size_t lds, hipStream_t s) {
  switch (a.ipx > 0 && fft_ct_plan(a.pn, a.n) && a.NL == GEN_ROWS ? a.n : 0) {
    case 48: return launch_rows_t<2, 48>(a, mid, rb, lds, s);
    case 64: return launch_rows_t<2, 64>(a, mid, rb, lds, s);
    case 96: return launch_rows_t<2, 96>(a, mid, rb, lds, s);
    case 128: return launch_rows_t<2, 128>(a, mid, rb, lds, s);
    case 192: return launch_rows_t<2, 192>(a, mid, rb, lds, s);
    case 256: return launch_rows_t<2, 256>(a, mid, rb, lds, s);
  }
  if (a.ipx == 2) launch_rows_t<2, 0>(a, mid, rb, lds, s);
  else if (a.ipx == 4) launch_rows_t<4, 0>(a, mid, rb, lds, s);
  else launch_rows_t<0, 0>(a, mid, rb, lds, s);
}

void launch_gen_cube(const GenArgs& a, hipStream_t s) {
  // the rows use the plan and line count of the x passes (a.NL == a.NLx), hence a.ipx
  const size_t lds_rows = (a.ipx ? 1 : 2) * (size_t)a.NL * (a.n + 1) * sizeof(C);
  const int rb = gen_row_blocks(a);
  // axis passes: x (L = n, outer = nc, inner = nh), z (L = nc, outer = 1, inner = n nh)
  const int NLx = a.NLx, NLz = a.NLz;
  const size_t lds_x = ((a.ipx ? 1 : 2) * (size_t)NLx * (a.n + 1) + a.n) * sizeof(C) + (size_t)NLx * sizeof(GenLine);
  const size_t lds_z = (a.ipz ? 1 : 2) * (size_t)NLz * (a.nc + 1) * sizeof(C) + (size_t)NLz * sizeof(GenLine);
  const long long lx = (long long)a.nc * a.nh, lz = (long long)a.n * a.nh;
  const int bx = (int)((lx + NLx - 1) / NLx), bz = (int)((lz + NLz - 1) / NLz);
  launch_rows(a, false, rb, lds_rows, s);
  launch_axis<0>(a, a.ipx, bx, lds_x, s, a.n, a.nc, a.nh, NLx);
  launch_axis<2>(a, a.ipz, bz, lds_z, s, a.nc, 1, a.n * a.nh, NLz);
  launch_axis<1>(a, a.ipx, bx, lds_x, s, a.n, a.nc, a.nh, NLx);
  launch_rows(a, true, rb, lds_rows, s);
  hipLaunchKernelGGL(k_gen_mean, dim3(1), dim3(256), 0, s, a, rb);
  launch_axis<3>(a, a.ipx, bx, lds_x, s, a.n, a.nc, a.nh, NLx);
}

void launch_mc_accumulate(const double* B, int ntri, long long* cnt, double* mean, double* m2,
                          unsigned long long* state, hipStream_t s) {
  hipLaunchKernelGGL(k_mc_accumulate, dim3((ntri + 255) / 256), dim3(256), 0, s, B, ntri, cnt, mean, m2, state);
}

void launch_mc_zero(long long* cnt, double* mean, double* m2, int ntri, hipStream_t s) {
  if (ntri > 0) hipLaunchKernelGGL(k_mc_zero, dim3((ntri + 255) / 256), dim3(256), 0, s, cnt, mean, m2, ntri);
}

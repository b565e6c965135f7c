// Eq. (vg): every visibility goes to the grid point nearest its baseline, q = rint(U / du) per
// axis, with the flag factor F; the grid is the half plane q_v >= 0 (a point with q_v < 0 stands
// for (-q_u, -q_v), the visibility conjugated; a point on the line q_v = 0, which the half plane
// stores whole, also enters at (-q_u, 0) conjugated), and chan_avg consecutive channels are gridded
// together.  A thread sums the channel group of each of its visibilities in registers and adds it to
// the FP64 cell sums and the integer counts with atomics (through LDS for the crowded cells around
// the origin); the cell sums are then written in the output precision.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "bs_kernels.h"

namespace {

constexpr int GRID_THREADS = 1024;

__global__ void k_grid_zero(GridArgs a) {
  const long long cells = (long long)a.nco * a.n * (a.n / 2 + 1);
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < cells; i += (long long)gridDim.x * blockDim.x) {
    a.acc[2 * i] = 0.0;
    a.acc[2 * i + 1] = 0.0;
    a.cnt[i] = 0;
  }
}

// A baseline's grid point, decided once a call: q = rint(U / du) per axis in FP64, reversed where q_v < 0.
// Code: 0 = off the grid, else 1 | reversed << 1 | q_v << 2 | (q_u + 2048) << 13.
__global__ __launch_bounds__(256) void k_grid_code(GridArgs a) {
  const double half = (double)(a.n / 2);
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < a.nvis; i += gridDim.x * 256LL) {
    double qu = rint(a.uv[2 * i] / a.du), qv = rint(a.uv[2 * i + 1] / a.du);
    const bool neg = qv < 0.0;
    if (neg) {
      qu = -qu;
      qv = -qv;
    }
    const bool in = fabs(qu) < half && fabs(qv) < half;
    a.code[i] = in ? 1u | (neg ? 2u : 0u) | (unsigned)(int)qv << 2 | (unsigned)((int)qu + 2048) << 13 : 0u;
  }
}

__device__ __forceinline__ void cell_add(const GridArgs& a, long long o, long long cell, double re, double im, int c) {
  const long long plane = (long long)a.n * (a.n / 2 + 1);
  double* d = a.acc + 2 * (o * plane + cell);
  unsafeAtomicAdd(d, re);
  unsafeAtomicAdd(d + 1, im);
  atomicAdd(a.cnt + o * plane + cell, c);
}
// acc / cnt index of hot cell h in one plane, -1 beyond a small grid
__device__ __forceinline__ int hot_cell(const GridArgs& a, int h) {
  const int iu = h / a.hot - (a.hot - 1), iv = h - (h / a.hot) * a.hot;
  if (iu <= -a.n / 2 || iu >= a.n / 2 || iv >= a.n / 2) return -1;
  return (iu < 0 ? iu + a.n : iu) * (a.n / 2 + 1) + iv;
}

// Short baselines crowd into the cells around the origin (number density ~ 1 / U^2), so the cells |q_u| <
// a.hot, q_v < a.hot are summed in LDS and the others take global atomics.  blockIdx.y: output channel o
// (all its input channels: a visibility's group is summed in registers first); blockIdx.x: the
// baselines i of share blockIdx.x of gridDim.x.  A thread takes four consecutive baselines (VEC: with
// 16-byte loads), and every channel's visibilities and flags are loaded before any is used, four
// channels at a time: the loads of flagged samples are wasted, but no load waits for a flag.
// Bound: HBM (9 bytes a sample) and the far cells' atomics.  hot = 64 fills a CU's LDS (8128 cells) and holds
// nine tenths of log-uniform baselines; with one share a channel its sums are stored for good.  262,144 baselines x
// 768 channels, 4:1, flags: 1560 us with 32 x 63 LDS cells, a division per channel group and loads that
// waited for flags, now 695.
template <bool VEC, bool PHASE>
__global__ __launch_bounds__(GRID_THREADS) void k_grid_scatter(GridArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char grid_sh[];
  const int hot = a.hot, nhot = grid_nhot(hot);
  double* hre = (double*)grid_sh;
  double* him = hre + nhot;
  int* hc = (int*)(him + nhot);
  const int nh = a.n / 2 + 1;
  const long long o = blockIdx.y;
  for (int h = threadIdx.x; h < nhot; h += GRID_THREADS) {
    hre[h] = 0.0;
    him[h] = 0.0;
    hc[h] = 0;
  }
  __syncthreads();
  const long long vb = (long long)blockIdx.x * a.share, ve = vb + a.share < a.nvis ? vb + a.share : a.nvis;
  const float2* __restrict__ vis = reinterpret_cast<const float2*>(a.vis);
  for (long long i0 = vb + 4 * threadIdx.x; i0 < ve; i0 += 4 * GRID_THREADS) {
    unsigned code[4];
    double re[4], im[4];
    int c[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      code[q] = i0 + q < ve ? a.code[i0 + q] : 0u;
      re[q] = im[q] = 0.0;
      c[q] = 0;
    }
    if constexpr (PHASE) {   // exp(i k_o . delta), delta the offset from the grid point
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (!code[q]) continue;
        const double U = a.uv[2 * (i0 + q)], V = a.uv[2 * (i0 + q) + 1];
        double sn, cs;
        sincos(a.knode[2 * o] * (U - a.du * rint(U / a.du)) + a.knode[2 * o + 1] * (V - a.du * rint(V / a.du)), &sn, &cs);
        re[q] = cs;
        im[q] = sn;
        c[q] = 1;
      }
    } else {
      for (int k0 = 0; k0 < a.chan_avg; k0 += 4) {
        float2 v[4][4];
        unsigned f[4][4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (k0 + k < a.chan_avg) {
            const long long j = (o * a.chan_avg + k0 + k) * a.nvis + i0;
            if constexpr (VEC) {   // nvis % 4 == 0: the four are in or out together
              const float4 x = *reinterpret_cast<const float4*>(vis + j), y = *reinterpret_cast<const float4*>(vis + j + 2);
              v[k][0] = make_float2(x.x, x.y);
              v[k][1] = make_float2(x.z, x.w);
              v[k][2] = make_float2(y.x, y.y);
              v[k][3] = make_float2(y.z, y.w);
              const unsigned w = a.flags ? *reinterpret_cast<const unsigned*>(a.flags + j) : 0u;
#pragma unroll
              for (int q = 0; q < 4; ++q) f[k][q] = w >> (8 * q) & 255u;
            } else {
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const bool in = i0 + q < ve;
                v[k][q] = in ? vis[j + q] : make_float2(0.f, 0.f);
                f[k][q] = in && a.flags ? a.flags[j + q] : 0u;
              }
            }
          }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (k0 + k < a.chan_avg) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
              if (!f[k][q]) {
                re[q] += (double)v[k][q].x;
                im[q] += (double)v[k][q].y;
                ++c[q];
              }
          }
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (!code[q] || !c[q]) continue;
      const int iu = (int)(code[q] >> 13) - 2048, iv = (int)(code[q] >> 2 & 2047u);
      const double vi = code[q] & 2u ? -im[q] : im[q];
      if (iu > -hot && iu < hot && iv < hot) {
        const int h = (iu + hot - 1) * hot + iv;
        atomicAdd(&hre[h], re[q]);
        atomicAdd(&him[h], vi);
        atomicAdd(&hc[h], c[q]);
        if (iv == 0) {   // the mirror baseline on the stored line q_v = 0: (-q_u, 0), conjugated
          const int hm = (-iu + hot - 1) * hot;
          atomicAdd(&hre[hm], re[q]);
          atomicAdd(&him[hm], -vi);
          atomicAdd(&hc[hm], c[q]);
        }
      } else {
        cell_add(a, o, (long long)(iu < 0 ? iu + a.n : iu) * nh + iv, re[q], vi, c[q]);
        if (iv == 0) cell_add(a, o, (long long)(iu > 0 ? a.n - iu : -iu) * nh, re[q], -vi, c[q]);
      }
    }
  }
  __syncthreads();
  // the only share: the cells' sums (no other path writes them: a far baseline's mirror on the line q_v = 0 is
  // far too); else this share's partials, stored whole and added over the shares in order
  const long long base = (o * gridDim.x + blockIdx.x) * nhot, plane = o * a.n * nh;
  for (int h = threadIdx.x; h < nhot; h += GRID_THREADS) {
    if (gridDim.x == 1) {
      const int cell = hot_cell(a, h);
      if (cell < 0) continue;
      *(double2*)&a.acc[2 * (plane + cell)] = make_double2(hre[h], him[h]);
      a.cnt[plane + cell] = hc[h];
    } else {
      *(double2*)&a.hot_v[2 * (base + h)] = make_double2(hre[h], him[h]);
      a.hot_c[base + h] = hc[h];
    }
  }
}

// The LDS cells' partials added over the shares in order, one plain store per cell and output channel.
__global__ __launch_bounds__(256) void k_grid_hot(GridArgs a, int shares) {
  const int h = blockIdx.x * 256 + threadIdx.x, nhot = grid_nhot(a.hot);
  const long long o = blockIdx.y;
  if (h >= nhot) return;
  const int cell = hot_cell(a, h);
  if (cell < 0) return;
  double re = 0.0, im = 0.0;
  int c = 0;
  for (int b = 0; b < shares; ++b) {
    const long long k = (o * shares + b) * nhot + h;
    re += a.hot_v[2 * k];
    im += a.hot_v[2 * k + 1];
    c += a.hot_c[k];
  }
  const long long at = o * a.n * (a.n / 2 + 1) + cell;
  a.acc[2 * at] = re;
  a.acc[2 * at + 1] = im;
  a.cnt[at] = c;
}

template <typename T>
__global__ void k_grid_fin(GridArgs a, T* __restrict__ out, int32_t* __restrict__ ng) {
  const long long cells = (long long)a.nco * a.n * (a.n / 2 + 1);
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < cells; i += (long long)gridDim.x * blockDim.x) {
    out[2 * i] = (T)__hip_atomic_load(a.acc + 2 * i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    out[2 * i + 1] = (T)__hip_atomic_load(a.acc + 2 * i + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    ng[i] = __hip_atomic_load(a.cnt + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

}  // namespace

void launch_grid_zero(const GridArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_grid_zero, dim3(1024), dim3(256), 0, s, a);
}

void launch_grid_scatter(const GridArgs& a, hipStream_t s) {
  const long long cb = (a.nvis + 255) / 256;
  hipLaunchKernelGGL(k_grid_code, dim3((unsigned)(cb < 2048 ? cb : 2048)), dim3(256), 0, s, a);
  const unsigned shares = (unsigned)grid_shares(a);
  const size_t lds = (size_t)grid_nhot(a.hot) * 20;
  const bool vec = a.nvis % 4 == 0 && (uintptr_t)a.vis % 16 == 0 && (uintptr_t)a.flags % 4 == 0;
  void (*k)(GridArgs) = a.knode ? k_grid_scatter<false, true> : vec ? k_grid_scatter<true, false> : k_grid_scatter<false, false>;
  (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  for (int o0 = 0; o0 < a.nco; o0 += 65535) {   // grid.y limit
    GridArgs b = a;
    const int no = a.nco - o0 < 65535 ? a.nco - o0 : 65535;
    b.acc += 2 * (long long)o0 * a.n * (a.n / 2 + 1);
    b.cnt += (long long)o0 * a.n * (a.n / 2 + 1);
    if (a.knode) b.knode += 2 * o0;
    b.vis += 2 * (long long)o0 * a.chan_avg * a.nvis;
    if (a.flags) b.flags += (long long)o0 * a.chan_avg * a.nvis;
    b.hot_v += 2 * (long long)o0 * shares * grid_nhot(a.hot);
    b.hot_c += (long long)o0 * shares * grid_nhot(a.hot);
    hipLaunchKernelGGL(k, dim3(shares, no), dim3(GRID_THREADS), lds, s, b);
    if (shares > 1)
      hipLaunchKernelGGL(k_grid_hot, dim3((grid_nhot(a.hot) + 255) / 256, no), dim3(256), 0, s, b, (int)shares);
  }
}

void launch_grid_fin(const GridArgs& a, bool fp64, void* out, int32_t* ng, hipStream_t s) {
  if (fp64) hipLaunchKernelGGL(k_grid_fin<double>, dim3(1024), dim3(256), 0, s, a, static_cast<double*>(out), ng);
  else hipLaunchKernelGGL(k_grid_fin<float>, dim3(1024), dim3(256), 0, s, a, static_cast<float*>(out), ng);
}

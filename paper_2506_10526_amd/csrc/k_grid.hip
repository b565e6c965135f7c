// Eq. (vg): every visibility goes to the grid point nearest its baseline, q = rint(U / du) per
// axis, with the flag factor F; the grid is the half plane q_v >= 0 (a point with q_v < 0 stands
// for (-q_u, -q_v), the visibility conjugated; a point on the line q_v = 0, which the half plane
// stores whole, also enters at (-q_u, 0) conjugated), and chan_avg consecutive channels are gridded
// together.  A thread sums the channel group of each of its visibilities in registers; the sums of the
// crowded cells around the origin are formed in LDS, the far baselines' group sums staged by cell (or added
// with atomics), and the cell sums written in the output precision.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "bs_kernels.h"

namespace {

constexpr int GRID_THREADS = 1024;

// Whether acc and cnt hold a cell at all when every far baseline off the line q_v = 0 is staged: an LDS cell
// (stored whole) or one of that line (atomics); the others are not cleared, written or read.
__device__ __forceinline__ bool cell_held(const GridArgs& a, int iu, int iv) {
  const int u = iu < a.n / 2 ? iu : a.n - iu;   // |q_u|
  return iv == 0 || (u < a.hot && iv < a.hot && u < a.n / 2 && iv < a.n / 2);
}
__global__ void k_grid_zero(GridArgs a) {
  const int nh = a.n / 2 + 1, plane = a.n * nh;
  const long long i0 = blockIdx.x * (long long)blockDim.x + threadIdx.x, step = (long long)gridDim.x * blockDim.x;
  const long long cells = (long long)a.nco * (a.all_staged ? a.n : plane);
  for (long long i = i0; i < cells; i += step) {
    const long long at = a.all_staged ? i * nh : i;
    *(double2*)&a.acc[2 * at] = make_double2(0.0, 0.0);
    a.cnt[at] = 0;
  }
  if (a.cap > 0)
    for (long long i = i0; i < plane + 2; i += step) a.fcnt[i] = 0;   // two totals after the cells
}

// A baseline's place, decided once a call: its grid point is q = rint(U / du) per axis in FP64, reversed where
// q_v < 0.  Code: kind | reversed << 2 | (q_v = 0) << 3 | payload << 4, kind
//   0 off the grid;  1 LDS cell (payload its index);  2 staged (payload the slot);  3 global atomics (payload
//   the cell)
// A far baseline on the line q_v = 0, which enters two cells, is not staged.  Slots are handed out in baseline
// order, a block's far baselines in one run; fcell and frank keep a slot's cell and its rank there for the
// cells' lists.  STAGE takes four baselines a thread, so that a block's atomic on the total hands out 1024; a
// short list without staging takes one a thread, its FP64 divisions the only thing that takes time.
template <bool STAGE>
__global__ __launch_bounds__(256) void k_grid_code(GridArgs a) {
  constexpr int NB = STAGE ? 4 : 1;
  __shared__ unsigned wsum[4], wbase;
  const double half = (double)(a.n / 2);
  const int nh = a.n / 2 + 1, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (long long b0 = blockIdx.x * 256LL * NB; b0 < a.nvis; b0 += gridDim.x * 256LL * NB) {
    const long long i0 = b0 + NB * threadIdx.x;
    unsigned code[NB], cell[NB], far = 0u;
    bool stage[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      code[q] = cell[q] = 0u;
      stage[q] = false;
      if (i0 + q >= a.nvis) continue;
      double qu = rint(a.uv[2 * (i0 + q)] / a.du), qv = rint(a.uv[2 * (i0 + q) + 1] / a.du);
      const bool neg = qv < 0.0;
      if (neg) {
        qu = -qu;
        qv = -qv;
      }
      if (!(fabs(qu) < half && fabs(qv) < half)) continue;
      const int iu = (int)qu, iv = (int)qv;
      if (iu > -a.hot && iu < a.hot && iv < a.hot) {
        code[q] = 1u | (unsigned)((iu + a.hot - 1) * a.hot + iv) << 4;
      } else {
        cell[q] = (unsigned)((iu < 0 ? iu + a.n : iu) * nh + iv);
        code[q] = 3u | cell[q] << 4;
        stage[q] = STAGE && iv > 0;
        far += stage[q];
      }
      code[q] |= (neg ? 4u : 0u) | (iv == 0 ? 8u : 0u);
    }
    if constexpr (STAGE) {
      unsigned inc = far;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const unsigned x = __shfl_up(inc, o);
        if (lane >= o) inc += x;
      }
      if (lane == 63) wsum[w] = inc;
      __syncthreads();
      if (threadIdx.x == 0) {
        const unsigned tot = wsum[0] + wsum[1] + wsum[2] + wsum[3];
        wbase = tot ? atomicAdd(a.fcnt + a.n * nh, tot) : 0u;
      }
      __syncthreads();
      unsigned slot = wbase + inc - far;
      for (int k = 0; k < w; ++k) slot += wsum[k];
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        if (!stage[q]) continue;
        if (slot < (unsigned)a.cap) {   // past the staging space: atomics
          a.fcell[slot] = cell[q];
          a.frank[slot] = atomicAdd(a.fcnt + cell[q], 1u);
          code[q] = 2u | (code[q] & 4u) | slot << 4;
        }
        ++slot;
      }
      __syncthreads();   // wsum and wbase are written again
    }
#pragma unroll
    for (int q = 0; q < NB; ++q)
      if (i0 + q < a.nvis) a.code[i0 + q] = code[q];
  }
}
// the far cells' runs in the list of slots, in no particular order of cells (four cells a thread and one atomic
// a block: all of them meet on one address; 4096^2, an atomic a wave, 174 us)
__global__ __launch_bounds__(256) void k_grid_off(GridArgs a) {
  __shared__ unsigned wsum[4], base;
  const int plane = a.n * (a.n / 2 + 1), lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i0 = 4 * (blockIdx.x * 256 + threadIdx.x);
  unsigned k[4], sum = 0u;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    k[q] = i0 + q < plane ? a.fcnt[i0 + q] : 0u;
    sum += k[q];
  }
  unsigned inc = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned x = __shfl_up(inc, o);
    if (lane >= o) inc += x;
  }
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned tot = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    base = tot ? atomicAdd(a.fcnt + plane + 1, tot) : 0u;
  }
  __syncthreads();
  unsigned at = base + inc - sum;
  for (int v = 0; v < w; ++v) at += wsum[v];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (i0 + q < plane) a.foff[i0 + q] = at;
    at += k[q];
  }
}
__global__ __launch_bounds__(256) void k_grid_list(GridArgs a) {
  const unsigned tot = a.fcnt[a.n * (a.n / 2 + 1)], m = tot < (unsigned)a.cap ? tot : (unsigned)a.cap;
  for (unsigned s = blockIdx.x * 256 + threadIdx.x; s < m; s += gridDim.x * 256) a.flist[a.foff[a.fcell[s]] + a.frank[s]] = s;
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
// a.hot, q_v < a.hot are summed in LDS.  A far baseline's group sum goes to its slot of a staging array, in
// baseline order, so that neighbouring threads fill whole lines; k_grid_fin gathers a cell's slots.  (Slots
// in cell order cost 200 us more in scattered 16-byte stores: 24 blocks' staging planes share an L2; float64
// atomics on the far cells ran at 27 G a second, 65 us per percent of the samples.)
// blockIdx.y: output channel o (all its input channels: a visibility's group is summed in registers
// first); blockIdx.x: the baselines i of share blockIdx.x of gridDim.x.  A thread takes four consecutive
// baselines (VEC: with 16-byte loads), and every channel's visibilities and flags are loaded before any is
// used, four channels at a time: the loads of flagged samples are wasted, but no load waits for a flag.
// Bound: HBM (9 bytes a sample).  hot = 64 fills a CU's LDS (8128 cells) and holds nine tenths of
// log-uniform baselines; with one share a channel its sums are stored for good.  262,144 baselines x 768
// channels, 4:1, flags: 1560 us with 32 x 63 LDS cells, a division per channel group, loads that waited for
// flags and atomics for the far cells; 695 with the atomics alone left, now 453: 4.3 TB/s.
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
      const unsigned kind = code[q] & 3u, at = code[q] >> 4;
      const double vi = code[q] & 4u ? -im[q] : im[q];
      if (kind == 2u) {   // every slot is written, a wholly flagged baseline's with zeros
        const long long p = o * a.cap + at;
        *(double2*)&a.stage_v[2 * p] = make_double2(re[q], vi);
        a.stage_c[p] = c[q];
      } else if (!kind || !c[q]) {
        continue;
      } else if (kind == 1u) {
        atomicAdd(&hre[at], re[q]);
        atomicAdd(&him[at], vi);
        atomicAdd(&hc[at], c[q]);
        if (code[q] & 8u) {   // q_v = 0: the mirror baseline on the stored line, (-q_u, 0), conjugated
          const int hm = 2 * (hot - 1) * hot - (int)at;
          atomicAdd(&hre[hm], re[q]);
          atomicAdd(&him[hm], -vi);
          atomicAdd(&hc[hm], c[q]);
        }
      } else {
        cell_add(a, o, at, re[q], vi, c[q]);
        if (code[q] & 8u) cell_add(a, o, at ? a.n * nh - (int)at : 0, re[q], -vi, c[q]);
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

// The LDS cells' partials added over the shares, one plain store per cell and output channel.  A block takes 32
// cells; eight groups of threads sum interleaved shares, four loads in flight, then the groups in order (a
// thread a cell over all shares waited for each in turn: 1 channel, 262,144 baselines, 256^2 65 us a call, now 34).
__global__ __launch_bounds__(256) void k_grid_hot(GridArgs a, int shares) {
  __shared__ double sr[8][32], si[8][32];
  __shared__ int sc[8][32];
  const int l = threadIdx.x & 31, q = threadIdx.x >> 5, h = blockIdx.x * 32 + l, nhot = grid_nhot(a.hot);
  const long long o = blockIdx.y;
  double re = 0.0, im = 0.0;
  int c = 0;
  if (h < nhot)
#pragma unroll 4
    for (int b = q; b < shares; b += 8) {
      const long long k = (o * shares + b) * nhot + h;
      const double2 v = *(const double2*)&a.hot_v[2 * k];
      re += v.x;
      im += v.y;
      c += a.hot_c[k];
    }
  sr[q][l] = re;
  si[q][l] = im;
  sc[q][l] = c;
  __syncthreads();
  if (q || h >= nhot) return;
  const int cell = hot_cell(a, h);
  if (cell < 0) return;
  for (int k = 1; k < 8; ++k) {
    re += sr[k][l];
    im += si[k][l];
    c += sc[k][l];
  }
  const long long at = o * a.n * (a.n / 2 + 1) + cell;
  *(double2*)&a.acc[2 * at] = make_double2(re, im);
  a.cnt[at] = c;
}

// The cell sums in the output precision.
template <typename T>
__global__ void k_grid_out(GridArgs a, T* __restrict__ out, int32_t* __restrict__ ng) {
  const long long cells = (long long)a.nco * a.n * (a.n / 2 + 1);
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < cells; i += (long long)gridDim.x * blockDim.x) {
    const double2 v = *(const double2*)&a.acc[2 * i];
    out[2 * i] = (T)v.x;
    out[2 * i + 1] = (T)v.y;
    ng[i] = a.cnt[i];
  }
}
// The same with the far cells' staged group sums gathered first.  Blocks are dealt to the eight XCDs in turn;
// block b works on a channel o with o mod 8 = b mod 8, so that the gathers of a channel meet its staging
// plane in one L2; the channels past a multiple of eight are spread over all of them (4 channels of 2048^2 on
// four XCDs: 220 us a call, now 93).  192 channels of 256^2, 262,144 baselines: 98 us (105 reading every cell
// of acc, which k_grid_zero then had to clear: 21 us, now 5).
template <typename T>
__global__ __launch_bounds__(256) void k_grid_fin(GridArgs a, T* __restrict__ out, int32_t* __restrict__ ng, int nx) {
  const int plane = a.n * (a.n / 2 + 1);
  int y = blockIdx.x / nx;
  if (y < a.nco / 8 * 8) y = (blockIdx.x >> 3) / nx * 8 + (blockIdx.x & 7);
  const long long o = y;
  const int i = (y < a.nco / 8 * 8 ? (blockIdx.x >> 3) % nx : blockIdx.x % nx) * 256 + threadIdx.x;
  if (o >= a.nco || i >= plane) return;
  const long long at = o * plane + i;
  const int nh = a.n / 2 + 1, iu = i / nh;
  double2 v = make_double2(0.0, 0.0);
  int c = 0;
  if (!a.all_staged || cell_held(a, iu, i - iu * nh)) {
    v = *(const double2*)&a.acc[2 * at];
    c = a.cnt[at];
  }
  const unsigned k = a.fcnt[i];
  const unsigned* run = a.flist + a.foff[i];
  for (unsigned s = 0; s < k; ++s) {
    const long long p = o * a.cap + run[s];
    const double2 t = *(const double2*)&a.stage_v[2 * p];
    v.x += t.x;
    v.y += t.y;
    c += a.stage_c[p];
  }
  out[2 * at] = (T)v.x;
  out[2 * at + 1] = (T)v.y;
  ng[at] = c;
}

}  // namespace

void launch_grid_zero(const GridArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_grid_zero, dim3(1024), dim3(256), 0, s, a);
}

void launch_grid_scatter(const GridArgs& a, hipStream_t s) {
  if (a.cap > 0) {
    const long long cb = (a.nvis + 1023) / 1024, lb = (a.cap + 255) / 256;
    hipLaunchKernelGGL(k_grid_code<true>, dim3((unsigned)std::min(cb, 2048LL)), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_grid_off, dim3((a.n * (a.n / 2 + 1) + 1023) / 1024), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_grid_list, dim3((unsigned)std::min(lb, 1024LL)), dim3(256), 0, s, a);
  } else {
    hipLaunchKernelGGL(k_grid_code<false>, dim3((unsigned)std::min((a.nvis + 255) / 256, 2048LL)), dim3(256), 0, s, a);
  }
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
    b.stage_v += 2 * (long long)o0 * a.cap;
    b.stage_c += (long long)o0 * a.cap;
    hipLaunchKernelGGL(k, dim3(shares, no), dim3(GRID_THREADS), lds, s, b);
    if (shares > 1)
      hipLaunchKernelGGL(k_grid_hot, dim3((grid_nhot(a.hot) + 31) / 32, no), dim3(256), 0, s, b, (int)shares);
  }
}

void launch_grid_fin(const GridArgs& a, bool fp64, void* out, int32_t* ng, hipStream_t s) {
  if (a.cap == 0) {
    if (fp64) hipLaunchKernelGGL(k_grid_out<double>, dim3(1024), dim3(256), 0, s, a, static_cast<double*>(out), ng);
    else hipLaunchKernelGGL(k_grid_out<float>, dim3(1024), dim3(256), 0, s, a, static_cast<float*>(out), ng);
    return;
  }
  const int nx = (a.n * (a.n / 2 + 1) + 255) / 256, o8 = (a.nco + 7) / 8;
  // channels in slices whose blocks fit a grid
  const int per = std::max(1, std::min(o8, (1 << 20) / nx)) * 8;
  const size_t plane = (size_t)a.n * (a.n / 2 + 1);
  for (int o0 = 0; o0 < a.nco; o0 += per) {
    GridArgs b = a;
    b.nco = std::min(per, a.nco - o0);
    b.acc += 2 * o0 * plane;
    b.cnt += o0 * plane;
    b.stage_v += 2 * (long long)o0 * a.cap;
    b.stage_c += (long long)o0 * a.cap;
    const dim3 g((unsigned)((long long)nx * b.nco));
    if (fp64) hipLaunchKernelGGL(k_grid_fin<double>, g, dim3(256), 0, s, b, static_cast<double*>(out) + 2 * o0 * plane, ng + o0 * plane, nx);
    else hipLaunchKernelGGL(k_grid_fin<float>, g, dim3(256), 0, s, b, static_cast<float*>(out) + 2 * o0 * plane, ng + o0 * plane, nx);
  }
}

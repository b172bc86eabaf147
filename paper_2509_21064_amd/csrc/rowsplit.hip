// Sparse QUBO, few restarts, x too large for LDS or too few restarts to fill
// the chip: a workgroup takes one restart and a share of the rows.
//
// The row-parallel kernel (spmm.hip) gathers x_j of all restarts of a row from
// L2 and is bound by the lines it takes: for n = 5 * 10^4, d = 100, B = 10 five
// million gathers of 40 bytes are 830 MB of 128-byte lines an iteration, 45 us
// at the 18 TB/s the L2s deliver.  Here a workgroup loads its restart's x into
// LDS, a range of columns at a time, and gathers from there; what the L2s then
// serve are the entries (4 bytes each, once per restart: 205 MB) and x once per
// workgroup (51 MB).  A row's entries are in column order and its accumulators
// stay in registers from range to range, so every sum has the row-parallel
// kernel's order and bits.
//
// Entries: slices of 64 rows, a lane per row, a workgroup's rows ordered by their
// number of entries in each range so that a wave's rows are equally long; per
// slice and range groups of four entries a lane (16 bytes, coalesced).  An entry is the
// column's offset in the range (low half) and the weight as float16 (high half,
// exact up to 2048); padding has weight 0.  The rounded sum is held in float32,
// exact below 2^24.
//
// Measured at that size: 21 us a launch (row-parallel 45), of which the gathers
// take the LDS about 12 (25,400 of 44,000 cycles); four groups of entries in flight (left to itself the
// compiler loads a group and waits for it: 31 us; eight in flight: 23), the next
// range's x loaded during the gathers, and the sums put back into row order
// through LDS for the update (row by row in slice order it took 6 us more).
#include <algorithm>

#include "common.h"

namespace pdbo {

constexpr int kSplitThreads = 1024, kSplitWaves = kSplitThreads / 64;
typedef uint32_t su32x4 __attribute__((ext_vector_type(4)));
typedef float sf32x4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float sf32x4a __attribute__((ext_vector_type(4)));
constexpr int kSplitAhead = 4;
constexpr int kSplitLoads = 10;  // 16-byte loads of a thread for a range of 40,960 columns

// R: slices per wave.  MODE as launch_spmm's 0 and 1.
template <int R, int GK, int MODE>
__global__ void __launch_bounds__(kSplitThreads) csr_split(SpmmDev D, int parity) {
  extern __shared__ __attribute__((aligned(16))) float xs[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = D.n, B = D.B, nseg = D.grid;
  // workgroup w runs on XCD w % 8: neighbours in `id` share a segment's entries
  // and an XCD's L2
  const int per = (nseg * B + 7) / 8, id = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
  if (id >= nseg * B) return;
  const int seg = id / B, b = id % B;
  const float* __restrict__ X = D.X[parity] + (size_t)b * n;
  float* __restrict__ Xn = D.X[parity ^ 1] + (size_t)b * n;
  float* __restrict__ Y = D.Y + (size_t)b * n;
  const int row0 = seg * D.srows, rows = min(D.srows, n - row0), ns = D.srows / 64;
  float acc[R], accr[R];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = accr[r] = 0.f;
  // a range of x goes through registers: the next one's loads are in flight
  // while this one's gathers run
  sf32x4 v[kSplitLoads];
  auto fetch = [&](int h) {
    const int base = h * D.srange, cnt = min(D.srange, n - base);
#pragma unroll
    for (int u = 0; u < kSplitLoads; ++u) {
      const int i = 4 * (tid + u * kSplitThreads);
      if (i + 4 <= cnt) {
        v[u] = *(const sf32x4*)(X + base + i);
      } else if (i < cnt) {
#pragma unroll
        for (int q = 0; q < 4; ++q) v[u][q] = X[base + min(i + q, cnt - 1)];
      }
    }
  };
  fetch(0);
  for (int h = 0; h < D.sranges; ++h) {
    const int cnt = min(D.srange, n - h * D.srange);
    if (h) __syncthreads();  // the last range's gathers are done
#pragma unroll
    for (int u = 0; u < kSplitLoads; ++u) {
      const int i = 4 * (tid + u * kSplitThreads);
      if (i < cnt) *(sf32x4a*)(xs + i) = v[u];  // up to srange, a multiple of 4
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int s = r * kSplitWaves + wid;
      int2 m = D.smeta[((size_t)seg * ns + min(s, ns - 1)) * D.sranges + h];
      if (s >= ns) m.y = 0;  // no slice; the wave still fetches its share of x
      const su32x4* p = (const su32x4*)D.sent + (size_t)m.x * 64 + lane;
      float a = acc[r], ar = accr[r];
      // kSplitAhead groups in flight (as many past the end are allocated)
      su32x4 e[kSplitAhead];
#pragma unroll
      for (int u = 0; u < kSplitAhead; ++u) e[u] = p[(size_t)u * 64];
      if (r == 0 && h + 1 < D.sranges) fetch(h + 1);  // behind these: loads return in order
      __builtin_amdgcn_sched_barrier(0);
      auto group = [&](su32x4 g) {
        float x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = xs[g[u] & 0xffffu];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float w = (float)__builtin_bit_cast(_Float16, (uint16_t)(g[u] >> 16));
          a = fmaf(w, x[u], a);
          ar = fmaf(w, x[u] > 0.5f ? 1.f : 0.f, ar);
        }
      };
      int k = 0;
      for (; k + kSplitAhead <= m.y; k += kSplitAhead) {
        p += kSplitAhead * 64;
#pragma unroll
        for (int u = 0; u < kSplitAhead; ++u) {
          group(e[u]);
          e[u] = p[(size_t)u * 64];
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int u = 0; u < kSplitAhead; ++u)
        if (k + u < m.y) group(e[u]);
      acc[r] = a;
      accr[r] = ar;
    }
  }
  // the sums back into the order of the rows, so that the state is read and
  // written in whole lines
  __syncthreads();
  float2* sums = (float2*)xs;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int s = r * kSplitWaves + wid;
    if (s >= ns) continue;
    const int q = D.srow[row0 + s * 64 + lane];
    if (q >= 0) sums[q] = make_float2(acc[r], accr[r]);
  }
  __syncthreads();
  const int win = (MODE == 0 && D.win) ? *D.win : -1;
  GdaP gp = D.gp;
  gp.gkind = GK;
  long long S = 0, C = 0;
  for (int q = tid; q < rows; q += kSplitThreads) {
    const int i = row0 + q;
    const float x = X[i];
    const float2 g = sums[q];
    if (x > 0.5f) {
      S += (long long)g.y;
      C += D.cp[i];
    }
    if constexpr (MODE == 0) {
      float xn, yn;
      gda_update(x, Y[i], fmaf(D.kos, g.x, D.cps[i]), gp, xn, yn);
      if (b == win) D.best_x[i] = (uint8_t)(Xn[i] > 0.5f);  // about to be overwritten
      Xn[i] = xn;
      Y[i] = yn;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    S += __shfl_xor(S, o);
    C += __shfl_xor(C, o);
  }
  __syncthreads();  // the sums are read
  long long* red = (long long*)xs;
  if (lane == 0) {
    red[wid] = S;
    red[kSplitWaves + wid] = C;
  }
  __syncthreads();
  if (tid < 2) {
    long long t = 0;
    for (int w = 0; w < kSplitWaves; ++w) t += red[tid * kSplitWaves + w];
    D.part[((size_t)tid * D.W + b) * nseg + seg] = t;  // one slice, W = B
  }
}

template <int GK, int MODE>
static hipError_t launch_split_r(const SpmmDev& d, int parity, hipStream_t s) {
  const int r = (d.srows / 64 + kSplitWaves - 1) / kSplitWaves;
  auto kern = r <= 1 ? csr_split<1, GK, MODE>
              : r <= 2 ? csr_split<2, GK, MODE> : r <= 4 ? csr_split<4, GK, MODE> : csr_split<8, GK, MODE>;
  if (r > 8 || d.srange > 4 * kSplitLoads * kSplitThreads) return hipErrorInvalidValue;
  const size_t lds = std::max({(size_t)d.srange * 4, (size_t)d.srows * 8, (size_t)2 * kSplitWaves * 8});
  hipError_t e = allow_lds((const void*)kern, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((d.grid * d.B + 7) / 8 * 8), dim3(kSplitThreads), lds, s, d, parity);
  return hipGetLastError();
}

hipError_t launch_csr_split(const SpmmDev& d, int mode, int parity, hipStream_t s) {
  if (mode == 1) return launch_split_r<0, 1>(d, parity, s);
  switch (d.gp.gkind) {
    case 0: return launch_split_r<0, 0>(d, parity, s);
    case 1: return launch_split_r<1, 0>(d, parity, s);
    default: return launch_split_r<2, 0>(d, parity, s);
  }
}

}  // namespace pdbo

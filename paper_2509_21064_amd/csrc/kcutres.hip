// Max-k-Cut with one workgroup of sixteen waves per restart for a whole call:
// the probabilities X of all nodes in LDS (updated in place between two
// barriers), the logits Z and the duals y in registers.
//
// The layout is that of the resident CSR kernel (resident.hip): position p =
// tid + 1024 j holds node order[p] (by decreasing degree), a slice of 64
// positions is its full groups of four entries and at most one group of those
// left over, an entry is one word, {index of the first of the K words of X_j |
// float16 weight << 16}; groups are streamed from L2, the next one on its way
// while one is summed.  X of a node takes K words, one more when that makes
// their number odd (K = 6, 8; K = 2 and 4 are read as one 8- or 16-byte word).
//
// The row-parallel kernels it takes over from spent 39 us an iteration at
// n = 10,000, k = 3, B = 100 (20,000 edges): 26 in the row kernel, which moves
// the whole state through memory and takes an argmax of every neighbour, and 12
// in the best of B.  Here the rounded assignment's objective is kept by
// differences: nodes whose category changed are put on a list in LDS and their
// edges recounted (an edge between two changed nodes at the lower position),
// from a byte per node with its category before and after.
//
// The sums run in the row-parallel kernels' order and the incumbent and the
// trace are rebuilt from the restarts' own improvements (resident_merge_kernel),
// so a run is bit for bit theirs.
#include <climits>

#include "common.h"

namespace pdbo {

typedef uint32_t ku32x4 __attribute__((ext_vector_type(4)));
#define PDBO_AS1 __attribute__((address_space(1)))
#define PDBO_AS3 __attribute__((address_space(3)))
#define PDBO_AS4 __attribute__((address_space(4)))

constexpr int kKrThreads = 1024;
constexpr int kKrWaves = kKrThreads / 64;
constexpr int kKrQueue = 1024;                // changed nodes of one iteration kept in LDS
constexpr int kKrRows = 16;                   // positions per thread, at most
constexpr int kKrRegs = 32;                   // logits per thread, at most
constexpr size_t kKrSmall = kKrQueue * 2 + 4 * 8 + kKrWaves * 8 + 16;
constexpr size_t kKrLds = 160 * 1024;

__host__ __device__ constexpr int kr_stride(int k) { return k == 6 ? 7 : k == 8 ? 9 : k; }

// positions, in whole rows of 32
__host__ __device__ inline int kr_rows32(int n) { return (n + 31) / 32 * 32; }

// Copies of X in LDS (as many as fit, at most four: they spread a gather over
// the banks as in resident.hip), 0: the instance does not fit.
int kcutres_copies(int n, int k) {
  const int R = (n + kKrThreads - 1) / kKrThreads, np = kr_rows32(n);
  if (R > kKrRows || R * k > kKrRegs) return 0;
  const int64_t words = (int64_t)np * kr_stride(k);
  for (int c = 4; c >= 1; c /= 2)
    if ((size_t)c * words * 4 + np + kKrSmall <= kKrLds && c * words <= 65536) return c;
  return 0;
}

// first word of position p in copy c: positions are permuted within rows of 32
__host__ __device__ inline int kr_word(int c, int p, int np, int stride) {
  const int q = c == 0 ? p : p ^ ((((p >> 5) * (2 * c + 9) + 7 * c) ^ (p >> 8)) & 31);
  return (c * np + q) * stride;
}

int kcutres_word(int n, int k, int c, int p) { return kr_word(c, p, kr_rows32(n), kr_stride(k)); }

template <int K>
__device__ __forceinline__ void kr_read(uint32_t word, float (&x)[K]) {
  if constexpr (K == 2) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    const f2 v = *(const PDBO_AS3 f2*)(size_t)(word << 2);
    x[0] = v.x;
    x[1] = v.y;
  } else if constexpr (K == 4) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const f4 v = *(const PDBO_AS3 f4*)(size_t)(word << 2);
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = v[u];
  } else {
#pragma unroll
    for (int u = 0; u < K; ++u) x[u] = *((const PDBO_AS3 float*)(size_t)(word << 2) + u);
  }
}

template <int K, int GK>
__global__ void __launch_bounds__(kKrThreads) kcut_resident(KcutDev D, int nsteps, int nc) {
  constexpr int ST = kr_stride(K);
  // dynamic LDS only, so that X starts at address 0
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.x, n = D.n, np = kr_rows32(n);
  float* X = (float*)lds;
  long long* dacc = (long long*)(lds + (size_t)nc * np * ST * 4);
  int64_t* red = (int64_t*)(dacc + 4);
  int* qn = (int*)(red + kKrWaves);
  uint16_t* queue = (uint16_t*)(qn + 4);
  uint8_t* cat = (uint8_t*)(queue + kKrQueue);  // category | the one before the last update << 4
  const int R = (n + kKrThreads - 1) / kKrThreads;
  const PDBO_AS1 uint32_t* ent = (const PDBO_AS1 uint32_t*)D.rent;
  const PDBO_AS4 int* slices = (const PDBO_AS4 int*)D.rslice;
  // slice {first word, full groups << 1 | a group is left over}, {0, 0} past the last
  auto slice = [&](int j) {
    const int s = j * kKrWaves + wid;
    if (s >= (n + 63) / 64) return make_int2(0, 0);
    return make_int2(__builtin_amdgcn_readfirstlane(slices[2 * s]),
                     __builtin_amdgcn_readfirstlane(slices[2 * s + 1]));
  };
  auto load = [&](int2 sl, int g) { return *(const PDBO_AS1 ku32x4*)(ent + sl.x + 256 * g + 4 * lane); };
  auto put = [&](int p, const float(&x)[K]) {
    for (int c = 0; c < nc; ++c) {
      float* w = X + kr_word(c, p, np, ST);
#pragma unroll
      for (int u = 0; u < K; ++u) w[u] = x[u];
    }
  };
  // vectors read at the uniform index of a loop (an unrolled loop would leave
  // the instruction cache)
  typedef float vec32 __attribute__((ext_vector_type(32)));
  typedef float vec16 __attribute__((ext_vector_type(16)));
  vec32 zr = {};
  vec16 yr = {};
  uint64_t rnow = 0, rbefore = 0, rbest = 0;  // categories of the thread's positions, four bits each
#pragma unroll 1
  for (int j = 0; j < R; ++j) {
    const int p = tid + j * kKrThreads;
    const int v = D.order[min(p, n - 1)];
    float z[K], x[K];
#pragma unroll
    for (int u = 0; u < K; ++u) {
      z[u] = D.Z[((size_t)b * n + v) * K + u];
      zr[j * K + u] = z[u];
    }
    yr[j] = D.Y[(size_t)b * n + v];
    softmax_k<K>(z, x);
    const int c = argmax_k<K>(x);
    rnow |= (uint64_t)c << (4 * j);
    if (p < n) {
      put(p, x);
      cat[p] = (uint8_t)(c | c << 4);
    }
  }
  if (tid < 4) {
    dacc[tid] = 0;
    qn[tid] = 0;
  }
  const int64_t t0 = *D.t_dev;
  int64_t bF = D.rbestF[b], bT = D.rbestT[b];
  int ntr = 0;
  __syncthreads();

  // position of an entry's word
  auto node = [&](uint32_t word) {
    const int q = (int)word / ST;  // ST is a constant
    int p = q;
    for (int c = 1; c < nc; ++c)
      if (q >= c * np) p = kr_word(c, q - c * np, np, 1) - c * np;
    return p;
  };
  auto weight = [&](uint32_t e) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(e >> 16)); };

  // weight of the edges inside the parts, from scratch
  auto count_all = [&]() -> int64_t {
    int64_t S = 0;
#pragma unroll 1
    for (int j = 0; j < R; ++j) {
      const int2 sl = slice(j);
      const int ng = (sl.y >> 1) + (sl.y & 1), own = (int)(rnow >> (4 * j)) & 15;
      const bool ok = tid + j * kKrThreads < n;
#pragma unroll 1
      for (int g = 0; g < ng; ++g) {
        const ku32x4 e = load(sl, g);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (ok && (cat[node(e[u] & 0xffffu)] & 15) == own) S += (int)weight(e[u]);
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) S += __shfl_xor(S, o);
    if (lane == 0) red[wid] = S;
    __syncthreads();
    const int64_t F = row16_sum_i64(red[lane & 15]) / 2;
    __syncthreads();
    return F;
  };
  // 8 lanes to each changed node, over its edges
  auto count_changes = [&](int cnt) {
    long long d = 0;
    for (int q = tid >> 3; q < cnt; q += kKrThreads / 8) {
      const int p = queue[q], s = p >> 6, own = cat[p];
      const int ng = (slices[2 * s + 1] >> 1) + (slices[2 * s + 1] & 1);
      const PDBO_AS1 uint32_t* e0 = ent + slices[2 * s] + 4 * (p & 63);
      for (int r = tid & 7; r < 4 * ng; r += 8) {
        const uint32_t e = e0[256 * (r >> 2) + (r & 3)];
        const int w = (int)weight(e), o = node(e & 0xffffu), c = cat[o];
        if ((c & 15) != c >> 4 && o < p) continue;  // counted there
        d += ((own & 15) == (c & 15) ? w : 0) - (own >> 4 == c >> 4 ? w : 0);
      }
    }
    return d;
  };

  int64_t F = count_all();  // of the last evaluated iterate
  bool improved = false;
  auto offer = [&](int64_t t, uint64_t r) {
    if (F >= bF) return;
    bF = F;
    bT = t;
    if (tid == 0) {
      const uint64_t ts = wall_clock();
      D.rtr[(size_t)b * kResTrace + ntr] = TraceRec{t, F, (int64_t)b, ts};
    }
    ++ntr;
    rbest = r;
    improved = true;
  };
  // as the row-parallel kernels: the state a call starts from is offered when
  // its count is >= 1 (it may have been set)
  if (t0 >= 1) offer(t0, rnow);

  for (int s = 0;; ++s) {
    // X^{t0+s} is in LDS.  The differences of the iterate before it are
    // complete; then those of this one, read in the next iteration.
    const long long dprev = dacc[(s + 3) & 3];
    F += dprev;
    // (a call's first iterate is offered whatever its difference: the state
    // before it was not)
    if (dprev || s == 2) offer(t0 + s - 1, rbefore);
    const int cnt = qn[s & 1];
    if (cnt > kKrQueue) {
      const int64_t Fs = count_all();
      if (tid == 0) dacc[s & 3] = Fs - F;
    } else if (cnt > 0) {
      const long long d = count_changes(cnt);
      if (d) atomicAdd((unsigned long long*)&dacc[s & 3], (unsigned long long)d);
    }
    if (s == nsteps) break;
    int2 sl = slice(0);
    ku32x4 cur = load(sl, 0);
#pragma unroll 1
    for (int j = 0; j < R; ++j) {
      const int2 nx = j + 1 < R ? slice(j + 1) : make_int2(0, 0);
      const int nf = sl.y >> 1, ng = nf + (sl.y & 1);
      float acc[K], xi[K];
#pragma unroll
      for (int u = 0; u < K; ++u) acc[u] = 0.f;
      kr_read<K>((uint32_t)(min(tid + j * kKrThreads, n - 1) * ST), xi);
#pragma unroll 1
      for (int g = 0; g < ng; ++g) {
        const ku32x4 e = cur;
        cur = g + 1 < ng ? load(sl, g + 1) : load(nx, 0);
        float v[4][K];
#pragma unroll
        for (int m = 0; m < 4; ++m) kr_read<K>(e[m] & 0xffffu, v[m]);
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
          for (int u = 0; u < K; ++u) acc[u] = fmaf(weight(e[m]), v[m][u], acc[u]);
      }
      if (ng == 0) cur = load(nx, 0);
      // X is at most 1 or, where a node's logits have overflowed, NaN in all its
      // words.  Padding entries gather other rows' words: a wave that meets a NaN
      // sums again without them.
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(acc[0] != acc[0]) != 0, 0)) {
#pragma unroll
        for (int u = 0; u < K; ++u) acc[u] = 0.f;
#pragma unroll 1
        for (int g = 0; g < ng; ++g) {
          const ku32x4 e = load(sl, g);
#pragma unroll 1
          for (int m = 0; m < 4; ++m) {
            float v[K];
            kr_read<K>(e[m] & 0xffffu, v);
#pragma unroll
            for (int u = 0; u < K; ++u)
              acc[u] = e[m] >> 16 ? fmaf(weight(e[m]), v[u], acc[u]) : acc[u];
          }
        }
      }
      sl = nx;
      const float y = yr[j];
      float gr[K], m = 0.f;
#pragma unroll
      for (int u = 0; u < K; ++u) {
        gr[u] = fmaf(D.tos, acc[u], y * kg_deriv<GK>(xi[u]));
        m = fmaf(xi[u], gr[u], m);
      }
#pragma unroll
      for (int u = 0; u < K; ++u) {
        float z = zr[j * K + u];
        z = fmaf(-D.gp.alpha, xi[u] * (gr[u] - m), z);
        zr[j * K + u] = z;
      }
      yr[j] = fmaf(D.gp.beta, kg_value<GK, K>(xi), y);
    }
    __syncthreads();  // every gather of X^{t0+s} is done
    rbefore = rnow;
    rnow = 0;
#pragma unroll 1
    for (int j = 0; j < R; ++j) {
      const int p = tid + j * kKrThreads;
      float z[K], x[K];
#pragma unroll
      for (int u = 0; u < K; ++u) z[u] = zr[j * K + u];
      softmax_k<K>(z, x);
      const int c = argmax_k<K>(x), old = (int)(rbefore >> (4 * j)) & 15;
      rnow |= (uint64_t)c << (4 * j);
      if (p < n) {
        put(p, x);
        cat[p] = (uint8_t)(c | old << 4);
        if (c != old) {
          const int q = atomicAdd(&qn[(s + 1) & 1], 1);
          if (q < kKrQueue) queue[q] = (uint16_t)p;
        }
      }
    }
    if (tid == 0) {
      dacc[(s + 1) & 3] = 0;  // last read in iteration s - 2
      qn[s & 1] = 0;          // read above; next appended to in iteration s + 1
    }
    __syncthreads();
  }
  __syncthreads();
  const long long dlast = dacc[nsteps & 3];
  F += dlast;
  if (dlast || nsteps == 1) offer(t0 + nsteps, rnow);

#pragma unroll 1
  for (int j = 0; j < R; ++j) {
    const int p = tid + j * kKrThreads;
    if (p >= n) continue;
    const int v = D.order[p];
#pragma unroll
    for (int u = 0; u < K; ++u) D.Z[((size_t)b * n + v) * K + u] = zr[j * K + u];
    D.Y[(size_t)b * n + v] = yr[j];
    if (improved) D.best_xr[(size_t)b * n + v] = (uint8_t)((rbest >> (4 * j)) & 15);
  }
  if (tid == 0) {
    D.rbestF[b] = bF;
    D.rbestT[b] = bT;
    D.Flast[b] = F;
    D.rtl[b] = ntr;
  }
}

template <int K>
static hipError_t launch_kr(const KcutDev& d, int nsteps, hipStream_t s) {
  auto kern = d.gp.gkind == 0 ? kcut_resident<K, 0> : kcut_resident<K, 1>;
  const int nc = kcutres_copies(d.n, K), np = kr_rows32(d.n);
  const size_t lds = (size_t)nc * np * kr_stride(K) * 4 + np + kKrSmall;
  hipError_t e = allow_lds((const void*)kern, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(d.B), dim3(kKrThreads), lds, s, d, nsteps, nc);
  return hipGetLastError();
}

// A launch's records fit kResTrace.  Restarts beyond the first kKrTogether wait
// for a CU within a launch, so launches are then short and the times of
// improvements tell when they were made to within one (n = 10^4, k = 3, B = 300:
// 8 ms; 64 iterations a launch cost n = 1000, B = 1024 15%: 10.2 -> 11.7 us an
// iteration).
constexpr int kKrTogether = 256, kKrSteps = 256;

hipError_t launch_kcut_resident(const KcutDev& d, int nsteps, hipStream_t s) {
  const int most = d.B > kKrTogether ? kKrSteps : kResTrace - 1;
  for (int done = 0; done < nsteps;) {
    const int k = nsteps - done < most ? nsteps - done : most;
    hipError_t e = hipErrorInvalidValue;
    switch (d.k) {
      case 2: e = launch_kr<2>(d, k, s); break;
      case 3: e = launch_kr<3>(d, k, s); break;
      case 4: e = launch_kr<4>(d, k, s); break;
      case 5: e = launch_kr<5>(d, k, s); break;
      case 6: e = launch_kr<6>(d, k, s); break;
      case 7: e = launch_kr<7>(d, k, s); break;
      case 8: e = launch_kr<8>(d, k, s); break;
    }
    if (e != hipSuccess) return e;
    e = launch_resident_merge(d.rtr, d.rtl, d.B, d.n, d.best_xr, d.inc, d.best_x, d.trace, d.trace_len,
                              d.trace_cap, d.t_dev, k, s);
    if (e != hipSuccess) return e;
    done += k;
  }
  return hipSuccess;
}

// Z (restart-major) from z0 (restart-major float64), or drawn by the library's
// generator with coordinate index i k + c; Y = y0
__global__ void kcut_resident_init_kernel(const double* __restrict__ z0, KcutDev D, float y0,
                                          uint64_t seed) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t nk = (size_t)D.n * D.k;
  if (idx >= nk * D.B) return;
  D.Z[idx] = z0 ? (float)z0[idx] : philox_start(seed, (uint32_t)(idx / nk), (uint32_t)(idx % nk));
  if (idx < (size_t)D.B * D.n) D.Y[idx] = y0;
}

hipError_t launch_kcut_resident_init(const double* z0, const KcutDev& d, float y0, uint64_t seed,
                                     hipStream_t s) {
  const size_t tot = (size_t)d.B * d.n * d.k;
  hipLaunchKernelGGL(kcut_resident_init_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, z0,
                     d, y0, seed);
  return hipGetLastError();
}

}  // namespace pdbo

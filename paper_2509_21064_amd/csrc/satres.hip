// Max-k-SAT over positions, k = 2..5: the restart-resident kernel, the adjoint
// of the Lagrangian and its value, on literals instead of variables.
//
// LDS holds for every variable both factors its literals contribute, x (a
// negated literal) and 1 - x (a plain one), as adjacent words, so a literal's
// factor is one gather: its code is the index of a word.  Position p = tid +
// 1024 j holds variable order[p] (by decreasing number of occurrences).  The
// occurrences of a slice of 64 positions are stored in groups of four per lane:
// K planes of 8 bytes per lane (a wave reads 512 contiguous bytes), the codes
// of the o-th other literal for the four occurrences, o < K - 1, and their
// weights as float16, signed by the position's own literal (exact for weights
// up to 2048).  A slice is its full groups and, when a list has entries left
// over, one group of up to three; the counts are uniform over the wave, padding
// entries have weight 0.
//
// What bounds it: LDS cycles of the gathers (k - 1 per occurrence), L2 bytes of
// the lists (2 k per occurrence) and VALU issue.  The kernel it took over from
// kept x alone: 22 VALU instructions per 3-SAT occurrence (decode, sign,
// conversion, and the count of unsatisfied clauses at their owner) and four
// logarithms per variable, 9000 per wave and iteration at n = 20,000,
// m = 84,000 (counters: VALU busy 94% of the cycles); for k > 3 its lists were
// not interleaved.  Here an occurrence takes 4 (k = 3), and
// - the count is kept by differences: a variable whose rounding changed is put
//   on a list in LDS, and the waves then take its occurrences, 16 lanes to a
//   variable; a clause with several changed variables is counted at the one of
//   lowest position (an x whose rounding has just changed is stored with its
//   sign bit set);
// - the table is kept in up to four copies, permuted against each other within
//   rows of 32 words, when they fit, and each code names the copy whose bank is
//   the emptiest in its gather (a wave's gather takes as many cycles as the
//   fullest bank has addresses, for each half of the wave).
#include <climits>

#include "common.h"

namespace pdbo {

typedef uint32_t su32x2 __attribute__((ext_vector_type(2)));
#define PDBO_AS1 __attribute__((address_space(1)))
#define PDBO_AS3 __attribute__((address_space(3)))
#define PDBO_AS4 __attribute__((address_space(4)))

constexpr int kSrThreads = 1024;
constexpr int kSrWaves = kSrThreads / 64;
constexpr int kSrQueue = 768;  // changed variables of one iteration kept in LDS
// list, differences, partial sums and counters behind the table
constexpr size_t kSrSmall = kSrQueue * 2 + 4 * 8 + kSrWaves * 8 + 16;
constexpr size_t kSrLds = 160 * 1024;

// words of one copy of the table: whole rows of 32
static int sr_words(int n) { return (2 * n + 31) / 32 * 32; }

int satres_copies(int n, int k) {
  if (k < 2 || k > 5) return 0;
  const int w = sr_words(n);
  for (int c = 4; c >= 1; c /= 2)
    if ((size_t)c * w * 4 + kSrSmall <= kSrLds && c * w <= 65536) return c;
  return 0;
}

// Word of a literal (2 p + plain) in copy c: pairs stay adjacent (one 8-byte
// store of a lane), rows of 32 words are permuted by an XOR of the pair's index.
__host__ __device__ inline int sr_word(int c, int w) {
  return c == 0 ? w : w ^ (((((w >> 5) * (2 * c + 5) + 5 * c) ^ (w >> 9)) & 15) << 1);
}

int satres_word(int n, int c, int w) { return c * sr_words(n) + sr_word(c, w); }

// MARKS: the sign bits of the table's x mark changed roundings and are dropped
// (sat_resident, whose x lies in [0, 1]); otherwise a factor is taken as it is,
// negative for an x outside the box.
template <bool MARKS>
__device__ __forceinline__ float sr_lit(uint32_t idx) {
  const float v = *(const PDBO_AS3 float*)(size_t)(idx << 2);
  return MARKS ? fabsf(v) : v;
}

template <int K> struct SrGroup { su32x2 c[K - 1], w; };

template <int K>
__device__ __forceinline__ SrGroup<K> sr_load(const PDBO_AS1 uint32_t* p) {
  SrGroup<K> g;
#pragma unroll
  for (int o = 0; o < K - 1; ++o) g.c[o] = *(const PDBO_AS1 su32x2*)(p + 128 * o);
  g.w = *(const PDBO_AS1 su32x2*)(p + 128 * (K - 1));
  return g;
}

__device__ __forceinline__ uint32_t sr_half(su32x2 v, int u) {
  return u & 1 ? v[u >> 1] >> 16 : v[u >> 1] & 0xffffu;
}
__device__ __forceinline__ float sr_weight(su32x2 v, int u) {
  return (float)__builtin_bit_cast(_Float16, (uint16_t)sr_half(v, u));
}

// N occurrences of a group: the product of the other literals' factors times
// the signed weight.  3-SAT adds the four of a full group to four sums and
// those left over to the first; the other k have one sum, in order (the orders
// of the kernels in maxsat.hip).  Without MARKS the factors may be anything, NaN
// and infinities included, and what a padding entry (weight bits all zero; a
// clause of weight zero has the sign bit set) gathered is left out.
template <int K, int N, bool MARKS>
__device__ __forceinline__ void sr_terms(const SrGroup<K>& g, float (&s)[4]) {
  float f[N][K - 1];
#pragma unroll
  for (int u = 0; u < N; ++u)
#pragma unroll
    for (int o = 0; o < K - 1; ++o) f[u][o] = sr_lit<MARKS>(sr_half(g.c[o], u));
#pragma unroll
  for (int u = 0; u < N; ++u) {
    float prod = f[u][0];
#pragma unroll
    for (int o = 1; o < K - 1; ++o) prod *= f[u][o];
    if constexpr (!MARKS) prod = sr_half(g.w, u) != 0u ? prod : 0.f;
    float& a = s[K == 3 && N == 4 ? u : 0];
    a = fmaf(sr_weight(g.w, u), prod, a);
  }
}

// Adjoint sums of the wave's slices j = 0..: next() moves cur on to the next
// group, across slices, so that its entries are on their way while the gathers
// of the present one run.
template <int K, bool MARKS>
struct SrWalk {
  const PDBO_AS1 uint32_t* ent;
  const PDBO_AS4 int* slices;  // {first word, full groups << 1 | a group is left over}
  int wid, lane2, nslices;
  SrGroup<K> cur;
  // (loaded where it is used, the wave's number being opaque: kept over the
  // iterations the slices would take more scalar registers than there are)
  __device__ __forceinline__ int2 slice(int j) const {
    int w = wid;
    asm volatile("" : "+s"(w));
    const int s = j * kSrWaves + w;
    if (s >= nslices) return make_int2(0, 0);
    return make_int2(__builtin_amdgcn_readfirstlane(slices[2 * s]),
                     __builtin_amdgcn_readfirstlane(slices[2 * s + 1]));
  }
  __device__ __forceinline__ const PDBO_AS1 uint32_t* at(int2 sl, int g) const {
    return ent + sl.x + g * (128 * K) + lane2;
  }
  __device__ __forceinline__ void start() { cur = sr_load<K>(at(slice(0), 0)); }
  // the sum of slice j (sl); nx: the slice after it
  __device__ __forceinline__ float sum(int2 sl, int2 nx) {
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    const int nf = sl.y >> 1, ng = nf + (sl.y & 1);
    for (int g = 0; g < nf; ++g) {
      const SrGroup<K> c = cur;
      cur = sr_load<K>(g + 1 < ng ? at(sl, g + 1) : at(nx, 0));
      sr_terms<K, 4, MARKS>(c, s);
    }
    if (sl.y & 1) {
      const SrGroup<K> c = cur;
      cur = sr_load<K>(at(nx, 0));
      sr_terms<K, 3, MARKS>(c, s);
    }
    return K == 3 ? (s[0] + s[1]) + (s[2] + s[3]) : s[0];
  }
};

// g and g' of the entropy at the same x, with two logarithms: a term of g is 0
// where its argument is not positive, and g' is constant where its clip moves x
// (lo, hi: its values there; lo for a NaN too).  Same values as g_value and
// g_deriv, for every x; with BOX for x in [0, 1], where g is 0 at both ends.
struct GEnds {
  float lo, hi;
};
template <int GK>
__device__ __forceinline__ GEnds g_ends() {
  return GK == 0 ? GEnds{0.f, 0.f} : GEnds{g_deriv(0.f, 1), g_deriv(1.f, 1)};
}
template <int GK, bool BOX>
__device__ __forceinline__ void g_both(float x, GEnds e, float& gv, float& gd) {
  if constexpr (GK == 0) {
    gv = g_value(x, 0);
    gd = g_deriv(x, 0);
  } else {
#pragma clang fp contract(off)  // g is the sum of two rounded products
    if constexpr (BOX) {
      const bool in = x > 0.f && x < 1.f;
      const float xi = in ? x : 0.5f;
      const float l0 = logf(xi), l1 = logf(1.f - xi);
      const float a = xi * l0, c = (1.f - xi) * l1;
      gv = in ? a + c : 0.f;
      gd = x < kEntropyEps ? e.lo : x > 1.f - kEntropyEps ? e.hi : l0 - l1;
    } else {
      const bool p0 = x > 0.f, p1 = x < 1.f;
      const float x0 = p0 ? x : 1.f, x1 = p1 ? 1.f - x : 1.f;
      const float l0 = logf(x0), l1 = logf(x1);
      const float a = p0 ? x0 * l0 : 0.f, c = p1 ? x1 * l1 : 0.f;
      gv = a + c;
      gd = !(x >= kEntropyEps) ? e.lo : x > 1.f - kEntropyEps ? e.hi : l0 - l1;
    }
  }
}

// Per-position values of a thread in registers.  Up to eight they are an array
// and the loops over them are unrolled; for more the code of an unrolled
// iteration (55 KB at 20) leaves the instruction cache, so they are a vector
// read at the loop's uniform index, and the loops stay loops.
template <int R> struct SrRegs {
  static constexpr bool roll = false;
  float v[R];
};
template <> struct SrRegs<20> {
  static constexpr bool roll = true;
  typedef float vec __attribute__((ext_vector_type(32)));
  vec v;
};

// R: positions per thread (at most); nc: copies of the table.
template <int K, int R, int GK>
__global__ void __launch_bounds__(kSrThreads)
    sat_resident(SatDev D, int64_t t0, int nsteps, int words, int nc) {
  // dynamic LDS only, so that the table starts at address 0
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  float* tab = (float*)lds;
  long long* dacc = (long long*)(lds + (size_t)nc * words * 4);
  int64_t* red = (int64_t*)(dacc + 4);
  int* qn = (int*)(red + kSrWaves);
  uint16_t* queue = (uint16_t*)(qn + 4);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.x, n = D.n;
  auto put = [&](int p, float xs, float one_minus) {
    const float2 v = make_float2(xs, one_minus);
    *(float2*)(tab + 2 * p) = v;
    for (int c = 1; c < nc; ++c) *(float2*)(tab + c * words + sr_word(c, 2 * p)) = v;
  };
  constexpr int UN = SrRegs<R>::roll ? 1 : R;  // unrolling of the loops over j
  // x and y move between variable order in global memory and positions through
  // LDS, several loads of a thread in flight
  SrRegs<R> yr = {}, xn = {};
  const size_t row = (size_t)b * D.ld;
#pragma unroll 4
  for (int i = tid; i < n; i += kSrThreads) tab[D.pos[i]] = D.Y[row + i];
  __syncthreads();
#pragma unroll UN
  for (int j = 0; j < R; ++j) yr.v[j] = tab[min(tid + j * kSrThreads, n - 1)];
  __syncthreads();
#pragma unroll 4
  for (int i = tid; i < n; i += kSrThreads) {
    const float x = fabsf(D.X[row + i]);  // the sign bit is ours
    put(D.pos[i], x, 1.f - x);
  }
  if (tid < 4) {
    dacc[tid] = 0;
    qn[tid] = 0;
  }
  int64_t bF = D.rbestF[b], bT = D.rbestT[b];
  uint64_t bTs = D.rbestTs[b];
  const float ios = D.ios;
  const GEnds ends = g_ends<GK>();
  GdaP gp = D.gp;
  gp.gkind = GK;
  __syncthreads();

  // weight of the clauses all of whose literals are false, from scratch
  auto count_all = [&]() -> int64_t {
    int64_t S = 0;
#pragma unroll 4
    for (int j = tid; j < D.m; j += kSrThreads) {
      bool sat = false;
#pragma unroll
      for (int l = 0; l < K; ++l) {
        const uint32_t code = D.plit[(size_t)l * D.m + j];
        const float x = fabsf(tab[code & ~1u]);  // plain literals are the odd words
        sat = sat || (x > 0.5f) == ((code & 1u) != 0u);
      }
      if (!sat) S += D.w[j];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) S += __shfl_xor(S, o);
    if (lane == 0) red[wid] = S;
    __syncthreads();
    const int64_t F = row16_sum_i64(red[lane & 15]);
    __syncthreads();
    return F;
  };
  int64_t F = count_all();  // of the last evaluated iterate

  // roundings of the thread's positions, bit j: of the iterate in the table, of
  // the one before it and of the best one of this call (written at its end: the
  // incumbent improves at almost every early iteration, and its bytes go to
  // scattered addresses)
  uint32_t rnow = 0, rbefore = 0, rbest = 0;
#pragma unroll UN
  for (int j = 0; j < R; ++j) {
    const int p = tid + j * kSrThreads;
    if (p < n && tab[2 * p] > 0.5f) rnow |= 1u << j;
  }
  // the iterate of iteration t, of roundings r, has objective F
  bool improved = false;
  auto offer = [&](int64_t t, uint32_t r) {
    if (F >= bF) return;
    bF = F;
    bT = t;
    if (tid == 0) bTs = wall_clock();
    rbest = r;
    improved = true;
  };

  SrWalk<K, true> walk{(const PDBO_AS1 uint32_t*)D.pent, (const PDBO_AS4 int*)D.pslice, wid, 2 * lane,
                       (n + 63) / 64, {}};
  // 16 lanes to each changed variable, over its occurrences
  auto count_changes = [&](int cnt) {
    long long d = 0;
    for (int q = tid >> 4; q < cnt; q += kSrThreads / 16) {
      const int p = queue[q];
      const bool own = fabsf(tab[2 * p]) > 0.5f;  // after the change
      const int s = p >> 6;
      const int base = walk.slices[2 * s], nf = walk.slices[2 * s + 1] >> 1;
      const int len = D.pinc_ptr[p + 1] - D.pinc_ptr[p], full = len & ~3;
      for (int r = tid & 15; r < len; r += 16) {
        const int g = r < full ? r >> 2 : nf, u = r < full ? r & 3 : r - full;
        const PDBO_AS1 uint16_t* e =
            (const PDBO_AS1 uint16_t*)(walk.ent + base + g * (128 * K) + 2 * (p & 63)) + u;
        bool now = true, was = true, mine = true;
#pragma unroll
        for (int o = 0; o < K - 1; ++o) {
          const uint32_t code = e[256 * o];
          // the literal's position: codes of copies are permuted within rows
          uint32_t c = code, w = code;
          for (int k = 1; k < nc; ++k)
            if (code >= (uint32_t)(k * words)) c = code - k * words, w = sr_word(k, c);
          const float v = tab[w & ~1u];
          const bool r1 = fabsf(v) > 0.5f, ch = __float_as_uint(v) >> 31 != 0u;
          const bool plain = w & 1u;  // false where the rounding is 0
          now = now && r1 != plain;
          was = was && (r1 != ch) != plain;
          mine = mine && !(ch && (int)(w >> 1) < p);
        }
        const float wt = (float)__builtin_bit_cast(_Float16, (uint16_t)e[256 * (K - 1)]);
        // the own literal, negated where the weight is positive, is false
        // after the change when own == negated, and before it otherwise
        const bool false_now = own == (wt > 0.f);
        if (mine && (false_now ? now : was)) d += false_now ? (int)fabsf(wt) : -(int)fabsf(wt);
      }
    }
    return d;
  };

  for (int s = 0;; ++s) {
    // x^{t0+s} is in the table.  The differences of the iterate before it are
    // complete; then those of this one, read in the next iteration.
    const long long dprev = dacc[(s + 3) & 3];
    F += dprev;
    // (a call's first iterate is offered whatever its difference: the state
    // before it was not)
    if (dprev || s == 2) offer(t0 + s - 1, rbefore);
    const int cnt = qn[s & 1];
    if (cnt > kSrQueue) {
      const int64_t Fs = count_all();
      if (tid == 0) dacc[s & 3] = Fs - F;
    } else if (cnt > 0) {
      const long long d = count_changes(cnt);
      if (d) atomicAdd((unsigned long long*)&dacc[s & 3], (unsigned long long)d);
    }
    if (s == nsteps) break;
    uint32_t ch = 0;  // bit j: the update changes the rounding of position j
    int tv = tid;  // opaque, so that no address is kept over the iterations
    asm volatile("" : "+v"(tv));
    walk.start();
    int2 sl = walk.slice(0);
#pragma unroll UN
    for (int j = 0; j < R; ++j) {
      if (wid * 64 + j * kSrThreads >= n) break;  // none of the wave's
      const int2 nx = j + 1 < R ? walk.slice(j + 1) : make_int2(0, 0);
      const float grad = walk.sum(sl, nx) * ios;
      sl = nx;
      const int p = tv + j * kSrThreads;
      const float x = fabsf(tab[2 * min(p, n - 1)]);  // lanes past n: unused
      float gv, gd;
      g_both<GK, true>(x, ends, gv, gd);
      // one coordinate of Alg. 1, as gda_update
      const float y = yr.v[j], dL = fmaf(y, gd, grad);
      float a = fminf(fmaxf(fmaf(-gp.alpha, dL, x), 0.f), 1.f);
      if (__builtin_amdgcn_ballot_w64(!(y > 0.f))) {
        const bool pert = (fabsf(x - 0.5f) <= gp.delta) && (fabsf(dL) <= 2.f * gp.delta) && (y <= 0.f);
        if (pert) a = x <= 0.5f ? 0.5f - gp.delta : 0.5f + gp.delta;
      }
      yr.v[j] = fmaf(gp.beta, gv, y);
      xn.v[j] = a;
      ch |= (a > 0.5f) != (((rnow >> j) & 1u) != 0u) && p < n ? 1u << j : 0u;
    }
    __syncthreads();  // every gather of x^{t0+s} is done
    asm volatile("" : "+v"(tv));
#pragma unroll UN
    for (int j = 0; j < R; ++j) {
      const int p = tv + j * kSrThreads;
      if (p < n) put(p, (ch >> j) & 1u ? -xn.v[j] : xn.v[j], 1.f - xn.v[j]);
    }
    if (tid == 0) {
      dacc[(s + 1) & 3] = 0;  // last read in iteration s - 2
      qn[s & 1] = 0;          // read above; next appended to in iteration s + 1
    }
    rbefore = rnow;
    rnow ^= ch;
    while (ch) {
      const int j = __builtin_ctz(ch);
      ch &= ch - 1u;
      const int q = atomicAdd(&qn[(s + 1) & 1], 1);
      if (q < kSrQueue) queue[q] = (uint16_t)(tv + j * kSrThreads);
    }
    __syncthreads();
  }
  __syncthreads();
  const long long dlast = dacc[nsteps & 3];
  F += dlast;
  if (dlast || nsteps == 1) offer(t0 + nsteps, rnow);

#pragma unroll 4
  for (int i = tid; i < n; i += kSrThreads) D.X[row + i] = fabsf(tab[2 * D.pos[i]]);
  __syncthreads();
#pragma unroll UN
  for (int j = 0; j < R; ++j) {
    const int p = tid + j * kSrThreads;
    if (p < n) *(float2*)(tab + 2 * p) = make_float2(yr.v[j], (rbest >> j) & 1u ? 1.f : 0.f);
  }
  __syncthreads();
#pragma unroll 4
  for (int i = tid; i < n; i += kSrThreads) {
    const float2 v = *(const float2*)(tab + 2 * D.pos[i]);
    D.Y[row + i] = v.x;
    if (improved) D.best_xr[(size_t)b * n + i] = (uint8_t)(v.y != 0.f);
  }
  if (tid == 0) {
    D.rbestF[b] = bF;
    D.rbestT[b] = bT;
    D.rbestTs[b] = bTs;
    D.Flast[b] = F;
  }
}

template <int K, int R, int GK>
static hipError_t launch_sr_k(const SatDev& d, int64_t t0, int nsteps, hipStream_t s) {
  auto kern = sat_resident<K, R, GK>;
  const int words = sr_words(d.n), nc = satres_copies(d.n, K);
  const size_t lds = (size_t)nc * words * 4 + kSrSmall;
  hipError_t e = allow_lds((const void*)kern, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(d.B), dim3(kSrThreads), lds, s, d, t0, nsteps, words, nc);
  return hipGetLastError();
}

template <int K, int GK>
static hipError_t launch_sr_r(const SatDev& d, int64_t t0, int nsteps, hipStream_t s) {
  const int r = (d.n + kSrThreads - 1) / kSrThreads;
  if (r <= 1) return launch_sr_k<K, 1, GK>(d, t0, nsteps, s);
  if (r <= 2) return launch_sr_k<K, 2, GK>(d, t0, nsteps, s);
  if (r <= 4) return launch_sr_k<K, 4, GK>(d, t0, nsteps, s);
  if (r <= 8) return launch_sr_k<K, 8, GK>(d, t0, nsteps, s);
  if (r <= 20) return launch_sr_k<K, 20, GK>(d, t0, nsteps, s);
  return hipErrorInvalidValue;
}

template <int GK>
static hipError_t launch_sr(const SatDev& d, int64_t t0, int nsteps, hipStream_t s) {
  switch (d.k) {
    case 2: return launch_sr_r<2, GK>(d, t0, nsteps, s);
    case 3: return launch_sr_r<3, GK>(d, t0, nsteps, s);
    case 4: return launch_sr_r<4, GK>(d, t0, nsteps, s);
    case 5: return launch_sr_r<5, GK>(d, t0, nsteps, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_sat_resident(const SatDev& d, int64_t t0, int nsteps, hipStream_t s) {
  return d.gp.gkind == 0 ? launch_sr<0>(d, t0, nsteps, s) : launch_sr<1>(d, t0, nsteps, s);
}

// ---- adjoint at given points: gradient (MODE 0) or Lagrangian backward (MODE 1)
//
// The sums are formed by position and handed over through LDS, so that x, y and
// the results move through global memory in variable order, contiguously.
template <int K, int R, int MODE, int GK>
__global__ void __launch_bounds__(kSrThreads)
    sat_adjoint_res(SatDev D, const float* __restrict__ X, int ldx, const float* __restrict__ Yv,
                    const float* __restrict__ dL, float* __restrict__ dx, float* __restrict__ dy,
                    int ldo, int words, int nc) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  float* tab = (float*)lds;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.x, n = D.n;
  const float* xb = X + (size_t)b * ldx;
  SrWalk<K, false> walk{(const PDBO_AS1 uint32_t*)D.pent, (const PDBO_AS4 int*)D.pslice, wid, 2 * lane,
                        (n + 63) / 64, {}};
  walk.start();
  for (int i = tid; i < n; i += kSrThreads) {
    const int p = D.pos[i];
    const float2 v = make_float2(xb[i], 1.f - xb[i]);
    for (int c = 0; c < nc; ++c) *(float2*)(tab + c * words + sr_word(c, 2 * p)) = v;
  }
  __syncthreads();
  float g[R];
  int2 sl = walk.slice(0);
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int2 nx = j + 1 < R ? walk.slice(j + 1) : make_int2(0, 0);
    g[j] = walk.sum(sl, nx) * D.ios;
    sl = nx;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int p = tid + j * kSrThreads;
    if (p < n) tab[D.order[p]] = g[j];
  }
  __syncthreads();
  const float scale = MODE == 1 ? dL[b] : 1.f;
  const GEnds ends = g_ends<GK>();
  for (int i = tid; i < n; i += kSrThreads) {
    if (MODE == 0) {
      dx[(size_t)b * ldo + i] = tab[i];
    } else {
      float gv, gd;
      g_both<GK, false>(xb[i], ends, gv, gd);
      dx[(size_t)b * ldo + i] = scale * fmaf(Yv[(size_t)b * ldx + i], gd, tab[i]);
      dy[(size_t)b * ldo + i] = scale * gv;
    }
  }
}

template <int K, int MODE, int GK>
static hipError_t launch_sra_k(const SatDev& d, const float* X, int ldx, const float* Y,
                               const float* dL, float* dx, float* dy, int ldo, int nb, hipStream_t s) {
  const int words = sr_words(d.n), nc = satres_copies(d.n, K);
  const size_t lds = (size_t)nc * words * 4;
  const int r = (d.n + kSrThreads - 1) / kSrThreads;
  auto kern = r <= 4 ? sat_adjoint_res<K, 4, MODE, GK>
                     : r <= 8 ? sat_adjoint_res<K, 8, MODE, GK> : sat_adjoint_res<K, 20, MODE, GK>;
  hipError_t e = allow_lds((const void*)kern, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(nb), dim3(kSrThreads), lds, s, d, X, ldx, Y, dL, dx, dy, ldo, words, nc);
  return hipGetLastError();
}

template <int K>
static hipError_t launch_sra(int mode, const SatDev& d, const float* X, int ldx, const float* Y,
                             const float* dL, float* dx, float* dy, int ldo, int nb, hipStream_t s) {
  if (mode == 0) return launch_sra_k<K, 0, 0>(d, X, ldx, Y, dL, dx, dy, ldo, nb, s);
  return d.gp.gkind == 0 ? launch_sra_k<K, 1, 0>(d, X, ldx, Y, dL, dx, dy, ldo, nb, s)
                         : launch_sra_k<K, 1, 1>(d, X, ldx, Y, dL, dx, dy, ldo, nb, s);
}

hipError_t launch_satres_adjoint(int mode, const SatDev& d, const float* X, int ldx, const float* Y,
                                 const float* dL, float* dx, float* dy, int ldo, int nb,
                                 hipStream_t s) {
  switch (d.k) {
    case 2: return launch_sra<2>(mode, d, X, ldx, Y, dL, dx, dy, ldo, nb, s);
    case 3: return launch_sra<3>(mode, d, X, ldx, Y, dL, dx, dy, ldo, nb, s);
    case 4: return launch_sra<4>(mode, d, X, ldx, Y, dL, dx, dy, ldo, nb, s);
    case 5: return launch_sra<5>(mode, d, X, ldx, Y, dL, dx, dy, ldo, nb, s);
    default: return hipErrorInvalidValue;
  }
}

// ---- Lagrangian value, clause-major: one workgroup per restart -------------
//
// Four clauses of a thread have their codes and weights, then their factors, in
// flight together; the sum runs over them in order.
template <int K, int GK>
__global__ void __launch_bounds__(kSrThreads)
    sat_fwd_res(SatDev D, const float* __restrict__ x, const float* __restrict__ y,
                float* __restrict__ L) {
  constexpr int U = 4;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  float* tab = (float*)lds;
  __shared__ double red[kSrWaves];
  const int b = blockIdx.x, tid = threadIdx.x, n = D.n, m = D.m;
  const float* xb = x + (size_t)b * n;
  const float* yb = y + (size_t)b * n;
  for (int i = tid; i < n; i += kSrThreads) {
    const float v = xb[i];
    *(float2*)(tab + 2 * D.pos[i]) = make_float2(v, 1.f - v);
  }
  __syncthreads();
  double acc = 0.0;
  for (int j0 = tid; j0 < m; j0 += U * kSrThreads) {
    uint32_t code[U][K];
    int w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = min(j0 + u * kSrThreads, m - 1);
      w[u] = D.w[j];
#pragma unroll
      for (int l = 0; l < K; ++l) code[u][l] = D.plit[(size_t)l * m + j];
    }
    float prod[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float f[K];
#pragma unroll
      for (int l = 0; l < K; ++l) f[l] = tab[code[u][l]];
      prod[u] = f[0];
#pragma unroll
      for (int l = 1; l < K; ++l) prod[u] *= f[l];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (j0 + u * kSrThreads < m) acc += (double)w[u] * (double)prod[u] * (double)D.ios;
  }
  const GEnds ends = g_ends<GK>();
  for (int i = tid; i < n; i += kSrThreads) {
    float gv, gd;
    g_both<GK, false>(xb[i], ends, gv, gd);
    acc += (double)yb[i] * (double)gv;
  }
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if ((tid & 63) == 0) red[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) {
    double tot = 0.0;
    for (int w = 0; w < kSrWaves; ++w) tot += red[w];
    L[b] = (float)tot;
  }
}

template <int K>
static hipError_t launch_srf(const SatDev& d, const float* x, const float* y, int nb, float* L,
                             hipStream_t s) {
  const size_t lds = (size_t)sr_words(d.n) * 4;
  auto kern = d.gp.gkind == 0 ? sat_fwd_res<K, 0> : sat_fwd_res<K, 1>;
  hipError_t e = allow_lds((const void*)kern, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(nb), dim3(kSrThreads), lds, s, d, x, y, L);
  return hipGetLastError();
}

hipError_t launch_satres_fwd(const SatDev& d, const float* x, const float* y, int nb, float* L,
                             hipStream_t s) {
  switch (d.k) {
    case 2: return launch_srf<2>(d, x, y, nb, L, s);
    case 3: return launch_srf<3>(d, x, y, nb, L, s);
    case 4: return launch_srf<4>(d, x, y, nb, L, s);
    case 5: return launch_srf<5>(d, x, y, nb, L, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace pdbo

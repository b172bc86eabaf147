// Restart-resident CSR kernel over positions: one workgroup of sixteen waves
// per restart for a whole call, x in LDS (double-buffered), y and c'/s in
// registers, one barrier per iteration.
//
// Position p = tid + 1024 j holds row order[p] (rows by decreasing degree), and
// the entries name positions, so a slice of 64 consecutive positions is one
// wave's rows of one j and its lists have nearly the same length.  A slice is
// its full groups (four entries per lane, 16 bytes that one ds_read_b128 or
// dwordx4 of the wave fetches for 256 entries) and, when a row has entries left
// over, one group of up to three; the counts are uniform over the wave.  The
// padding entries have weight 0 (0 * x added to a sum that starts at +0 leaves
// every bit of it).  An entry is one word: the byte offset of x_j in the low
// half, the weight as float16 (exact for |weight| <= 2048) in the high half,
// read in place by a mixed-precision FMA.
//
// What bounds it: VALU issue, and LDS cycles of the gathers.  The kernel it
// took over from (csr_persistent's interleaved, double-buffered variant) issued
// 227 VALU instructions per wave and iteration on n = 2000, 12,000 entries
// (counters: VALU busy 87% of the cycles): eight per entry (decode, conversion,
// rounding, objective) and about sixty in the reductions of the objective.
// - The entries above take two, and the first groups of every row stay in
//   registers over the iterations, decoded.
// - The objective of round(x) is kept by differences: with r the rounding and D
//   the coordinates whose rounding changed (d_i = +-1),
//     2 (F(r') - F(r)) = sum_{i in D} d_i (kappa sum_j Ahat_ij (r'_j + r_j) + 2 c'_i),
//   an identity in integers; the lanes owning the coordinates of D add their
//   terms with one LDS atomic each.  An x_j whose rounding has just changed is
//   stored with its sign bit set (x >= 0; the gathers take |x|, a free operand
//   modifier), so r_j needs no second copy.  On n = 2000 (Max-Cut, 6000 edges)
//   an iteration changes 26 coordinates of a restart on average before t = 50,
//   3 up to t = 400, 0.2 after 1000.  The sum of an iteration's differences is
//   read one iteration later, behind the barrier that is there anyway.
// - A gather of 64 lanes takes as many cycles as the fullest of the 32 banks
//   has addresses, for each half of the wave (measured with fixed patterns):
//   about 3.6 + 3.6 at random addresses.  x is therefore kept in two copies
//   whose rows of 32 words are permuted against each other, and the host names
//   for each entry the copy whose bank is the emptier one (n = 2000: 1.20 to
//   1.03 us an iteration; four copies: 1.03).
#include <climits>

#include "common.h"

namespace pdbo {

typedef uint32_t ru32x4 __attribute__((ext_vector_type(4)));

constexpr int kResThreads = 1024;
constexpr int kResWaves = kResThreads / 64;
constexpr size_t kResSmall = 4 * 8 + kResWaves * 8;  // differences and partial sums
constexpr size_t kResLds = 160 * 1024;

// entries in LDS, or in global memory (a pointer of that address space, so that
// the loads are not flat, which would also wait for the LDS counter)
#define PDBO_AS1 __attribute__((address_space(1)))
#define PDBO_AS3 __attribute__((address_space(3)))
#define PDBO_AS4 __attribute__((address_space(4)))
__device__ __forceinline__ ru32x4 ld4(const uint32_t* p) { return *(const ru32x4*)p; }
__device__ __forceinline__ ru32x4 ld4(const PDBO_AS1 uint32_t* p) {
  return *(const PDBO_AS1 ru32x4*)p;
}

__device__ __forceinline__ float ent_w(uint32_t e) {
  return (float)__builtin_bit_cast(_Float16, (uint16_t)(e >> 16));
}

// x_j of entry e, with its sign bit, from the iterate whose copies start at LDS
// byte address XB
template <uint32_t XB>
__device__ __forceinline__ float ent_x(uint32_t e) {
  return *((const PDBO_AS3 float*)(size_t)(e & 0xffffu) + XB / 4);
}

// One full group of a row's gradient sum.  SEQ: one accumulator in entry order
// (the order of the row-parallel path); otherwise the first and third entry
// into one, the others into a second (the order of csr_persistent).
template <bool SEQ, uint32_t XB>
__device__ __forceinline__ void res_group(ru32x4 e, float& a0, float& a1) {
  const float x0 = fabsf(ent_x<XB>(e.x)), x1 = fabsf(ent_x<XB>(e.y));
  const float x2 = fabsf(ent_x<XB>(e.z)), x3 = fabsf(ent_x<XB>(e.w));
  a0 = fmaf(ent_w(e.x), x0, a0);
  if constexpr (SEQ) {
    a0 = fmaf(ent_w(e.y), x1, a0);
    a0 = fmaf(ent_w(e.z), x2, a0);
    a0 = fmaf(ent_w(e.w), x3, a0);
  } else {
    a1 = fmaf(ent_w(e.y), x1, a1);
    a0 = fmaf(ent_w(e.z), x2, a0);
    a1 = fmaf(ent_w(e.w), x3, a1);
  }
}

// sum over a row's ng groups of weight times r'_j (BOTH: r'_j + r_j), exact in
// float32: the host has bounded twice the row's absolute sum below 2^24
template <bool BOTH, uint32_t XB, typename EP>
__device__ __forceinline__ float res_rounded(EP ent, int ng) {
  float a = 0.f;
#pragma unroll 1
  for (int k = 0; k < ng; ++k, ent += 256) {
    const ru32x4 e = ld4(ent);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float v = ent_x<XB>(e[u]);
      const bool r1 = fabsf(v) > 0.5f;
      float r = r1 ? 1.f : 0.f;
      if constexpr (BOTH) r += (r1 != (__float_as_uint(v) >> 31 != 0u)) ? 1.f : 0.f;
      a = fmaf(ent_w(e[u]), r, a);
    }
  }
  return a;
}

template <bool V> struct res_bool { static constexpr bool value = V; };
template <uint32_t V> struct res_u32 { static constexpr uint32_t value = V; };

// Per R (positions per thread): copies of x (as many as a 16-bit offset and the
// LDS hold), full groups of a row in registers, and whether its left-over group
// is (128 registers per thread).
template <int R> constexpr int res_copies() { return R <= 8 ? 2 : 1; }
template <int R> constexpr int res_full() { return R == 1 ? 3 : R == 2 ? 2 : R == 4 ? 1 : 0; }
template <int R> constexpr bool res_rest() { return R <= 4; }

// Word of position p in copy c: its row of 32 words (one per bank) is permuted
// by an XOR that depends on the copy and the row, so that a store of a wave
// still meets every bank once.
__host__ __device__ inline int res_word(int c, int p) {
  return c == 0 ? p : p ^ ((((p >> 5) * (2 * c + 9) + 7 * c) ^ (p >> 8)) & 31);
}

// LDSE: the entries are staged in LDS (else what the registers do not hold is
// streamed from L2, each read a contiguous block of the wave).
template <int R, bool SEQ, int GK, bool LDSE>
__global__ void __launch_bounds__(kResThreads) csr_resident(CsrDev D, int64_t t00, int nsteps) {
  constexpr int NP = R * kResThreads;               // positions, padded
  constexpr int NC = res_copies<R>();
  constexpr uint32_t XB = NC * NP * sizeof(float);   // bytes of the copies of an iterate
  constexpr int GC = res_full<R>();
  constexpr bool TC = res_rest<R>();
  static_assert(XB <= 65536, "16-bit byte offsets");
  // dynamic LDS only, so that it starts at address 0: the copies of x^t and of
  // x^{t+1}, the entries (LDSE), the differences and the waves' partial sums
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.x, n = D.n;
  uint32_t* entl = (uint32_t*)(lds + 2 * XB);
  long long* dacc = (long long*)(lds + 2 * XB + (LDSE ? (size_t)D.nrent * 4 : 0));
  int32_t(*red)[2] = (int32_t(*)[2])(dacc + 4);
  int32_t* cpl = (int32_t*)(red + kResWaves);  // c' by position (R <= 4)
  if constexpr (R <= 4)
    for (int q = tid; q < NP; q += kResThreads) cpl[q] = D.rcp[q];
  auto cp_of = [&](int j) {
    const int p = tid + j * kResThreads;
    if constexpr (R <= 4) return cpl[p];
    else return D.rcp[p];
  };
  if constexpr (LDSE) {
    const ru32x4* src = (const ru32x4*)D.rent;
    const int nw4 = (int)(D.nrent / 4);  // whole 16-byte words
    for (int q = tid; q < nw4; q += kResThreads) ((ru32x4*)entl)[q] = src[q];
  }
  const PDBO_AS1 uint32_t* entg = (const PDBO_AS1 uint32_t*)D.rent;
  // slice {first word, full groups << 1 | a group is left over} of the wave's
  // positions j: in scalar registers, or (R > 4: there are not enough) loaded
  // again where they are used, w being opaque
  auto load_slice = [&](int j, int w) {
    const PDBO_AS4 int* v = (const PDBO_AS4 int*)((const PDBO_AS4 int2*)D.rslice + j * kResWaves + w);
    return make_int2(v[0], v[1]);
  };
  int2 slk[R <= 4 ? R : 1];
  if constexpr (R <= 4)
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int2 v = load_slice(j, wid);
      slk[j] = make_int2(__builtin_amdgcn_readfirstlane(v.x), __builtin_amdgcn_readfirstlane(v.y));
    }
  auto slice_of = [&](int j) {
    if constexpr (R <= 4) return slk[j];
    int w = wid;
    asm volatile("" : "+s"(w));
    return load_slice(j, w);
  };
  // word of the thread's position j in copy c
  auto word = [&](int c, int j) { return c * NP + res_word(c, tid + j * kResThreads); };
  float xr[R], yr[R], cps[R];
  ru32x4 ec[R][GC > 0 ? GC : 1];  // full groups, zero past the last
  uint32_t et[R][3];              // left-over entries, likewise
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int p = tid + j * kResThreads;
    xr[j] = yr[j] = cps[j] = 0.f;  // positions past n stay at 0
    if (p < n) {
      const int i = D.order[p];
      xr[j] = fabsf(D.X[(size_t)b * D.ld + i]);  // the sign bit is ours
      yr[j] = D.Y[(size_t)b * D.ld + i];
      cps[j] = D.cps[i];
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) ((float*)lds)[word(c, j)] = xr[j];
    const int2 sl = slice_of(j);
    const PDBO_AS1 uint32_t* e = entg + sl.x + 4 * lane;
#pragma unroll
    for (int g = 0; g < GC; ++g) ec[j][g] = g < sl.y >> 1 ? ld4(e + 256 * g) : ru32x4{0, 0, 0, 0};
    if constexpr (TC) {
      const ru32x4 t = sl.y & 1 ? ld4(e + 256 * (sl.y >> 1)) : ru32x4{0, 0, 0, 0};
      et[j][0] = t.x;
      et[j][1] = t.y;
      et[j][2] = t.z;
    }
  }
  if (tid < 4) dacc[tid] = 0;
  const int64_t t0 = D.t_dev ? *D.t_dev : t00;
  int64_t bF2 = D.rbestF[b], bT = D.rbestT[b];
  bF2 = bF2 == LLONG_MAX ? bF2 : 2 * bF2;  // twice the objectives throughout
  uint64_t bTs = D.rbestTs[b];
  int ntr = 0;
  const float kos = D.kos;
  GdaP gp = D.gp;
  gp.gkind = GK;  // a constant: only this kind's g and g' are computed
  __syncthreads();

  uint64_t wfl = 0;  // the last update changed some rounding of the wave's
  int64_t F2;        // twice the objective of the last evaluated iterate

  // The loops below run in few iterations: over j not unrolled, the thread's
  // own x read back from LDS (xb: a res_u32, 0 or XB).
  auto own = [&](auto xb, int j) {
    return *(const PDBO_AS3 float*)(size_t)(decltype(xb)::value + 4u * (uint32_t)(tid + j * kResThreads));
  };
  // The iterate of iteration t has objective F2 / 2.  Its rounding is that of x
  // at xb, or (before) that of x before the changes the sign bits mark.
  auto offer = [&](int64_t t, auto xb, auto before) {
    if (F2 >= bF2) return;
    bF2 = F2;
    bT = t;
    if (tid == 0) {
      bTs = wall_clock();
      if (D.rtr) D.rtr[(size_t)b * kResTrace + ntr] = TraceRec{t, F2 / 2, (int64_t)b, bTs};
    }
    ++ntr;
    uint8_t* dst = D.best_xr + (size_t)b * n;
#pragma unroll 1
    for (int j = 0; j < R; ++j) {
      const int p = tid + j * kResThreads;
      const float v = own(xb, j);
      const bool r = fabsf(v) > 0.5f;
      if (p < n) dst[D.order[p]] = (uint8_t)(decltype(before)::value ? r != (__float_as_uint(v) >> 31 != 0u) : r);
    }
  };
  auto row_rounded = [&](int j, auto xb, auto both) {
    const int2 sl = load_slice(j, wid);
    const int ng = (sl.y >> 1) + (sl.y & 1);
    if constexpr (LDSE)
      return res_rounded<decltype(both)::value, decltype(xb)::value>((const uint32_t*)entl + sl.x + 4 * lane, ng);
    else
      return res_rounded<decltype(both)::value, decltype(xb)::value>(entg + sl.x + 4 * lane, ng);
  };

  {  // the starting state's objective, from scratch
    constexpr res_u32<0> xb{};
    int S = 0, C = 0;
#pragma unroll 1
    for (int j = 0; j < R; ++j) {
      const int cp = cp_of(j);
      const float r = row_rounded(j, xb, res_bool<false>{});
      if (own(xb, j) > 0.5f) {
        S += (int)r;
        C += cp;
      }
    }
    S = wave_sum_i32(S);
    C = wave_sum_i32(C);
    if (lane == 0) {
      red[wid][0] = S;
      red[wid][1] = C;
    }
    __syncthreads();
    S = lane < kResWaves ? red[lane][0] : 0;
    C = lane < kResWaves ? red[lane][1] : 0;
    F2 = (int64_t)D.kappa * wave_sum_i32(S) + 2 * (int64_t)wave_sum_i32(C);
    // the row-parallel path, whose contexts SEQ serves, also offers the state a
    // call starts from when its count is >= 1 (it may have been set)
    if (SEQ && t0 >= 1) offer(t0, xb, res_bool<false>{});
  }

  // Iteration s, x^{t0+s} at xb (s odd: XB): true after the last iterate.
  auto iteration = [&](auto xbv, int s) -> bool {
    constexpr uint32_t xb = decltype(xbv)::value, xo = XB - xb;
    // differences of this iterate from the one before, read in the next
    // iteration; then the sum of the previous iterate's
    if (wfl) {
      long long d2 = 0;
#pragma unroll 1
      for (int j = 0; j < R; ++j) {
        const float v = own(xbv, j);
        const bool ch = __float_as_uint(v) >> 31 != 0u;
        if (!__builtin_amdgcn_ballot_w64(ch)) continue;
        const int cp = cp_of(j);
        const float r = row_rounded(j, xbv, res_bool<true>{});
        const long long d = (long long)D.kappa * (int)r + 2 * (long long)cp;
        if (ch) d2 += fabsf(v) > 0.5f ? d : -d;
      }
      if (d2) atomicAdd((unsigned long long*)&dacc[s & 3], (unsigned long long)d2);
    }
    const long long dprev = dacc[(s + 3) & 3];
    // the slot of iteration s + 1, last read in iteration s - 2
    if (tid == 0) dacc[(s + 1) & 3] = 0;
    // (a call's first iterate is offered whatever its difference: the state
    // before it was not)
    auto previous = [&]() {
      if (dprev || s == 2) {
        F2 += dprev;
        offer(t0 + s - 1, xbv, res_bool<true>{});
      }
    };
    if (s == nsteps) {
      previous();
      __syncthreads();
      const long long dlast = dacc[nsteps & 3];
      F2 += dlast;
      if (dlast || nsteps == 1) offer(t0 + nsteps, xbv, res_bool<false>{});
      return true;
    }
    wfl = 0;
    // rows whose gathers are in flight together: with entries in registers one
    // at a time is faster (n = 2000: 0.93 against 1.03 us an iteration; the
    // update of one overlaps the gathers of other waves), with all of them
    // streamed two (n = 8000: 4.2 against 4.3 us)
    constexpr int JP = TC ? 1 : 2;
#pragma unroll
    for (int j0 = 0; j0 < R; j0 += JP) {
      float a0[JP], a1[JP], xt[JP][3];
#pragma unroll
      for (int u = 0; u < JP; ++u) {
        a0[u] = a1[u] = 0.f;
        if constexpr (TC)
#pragma unroll
          for (int v = 0; v < 3; ++v) xt[u][v] = fabsf(ent_x<xb>(et[j0 + u][v]));
      }
      int2 sl[JP];
      int most = 0;
#pragma unroll
      for (int u = 0; u < JP; ++u) {
        sl[u] = slice_of(j0 + u);
        most = max(most, sl[u].y >> 1);
      }
#pragma unroll
      for (int g = 0; g < GC; ++g) {
        if (g >= most) break;
#pragma unroll
        for (int u = 0; u < JP; ++u) res_group<SEQ, xb>(ec[j0 + u][g], a0[u], a1[u]);
      }
#pragma unroll
      for (int u = 0; u < JP; ++u) {
        const int nf = sl[u].y >> 1, ng = TC ? nf : nf + (sl[u].y & 1);
        if (ng > GC) {  // the next group's entries are on their way while one is summed
          const int off = sl[u].x + 4 * lane;
          auto load = [&](int g) {
            if constexpr (LDSE) return ld4((const uint32_t*)entl + off + 256 * g);
            else return ld4(entg + off + 256 * g);
          };
          ru32x4 e = load(GC);
#pragma unroll 1
          for (int g = GC; g < nf; ++g) {
            const ru32x4 en = load(min(g + 1, ng - 1));
            res_group<SEQ, xb>(e, a0[u], a1[u]);
            e = en;
          }
          if (!TC && ng > nf) {
#pragma unroll
            for (int v = 0; v < 3; ++v) a0[u] = fmaf(ent_w(e[v]), fabsf(ent_x<xb>(e[v])), a0[u]);
          }
        }
        if constexpr (TC)
#pragma unroll
          for (int v = 0; v < 3; ++v) a0[u] = fmaf(ent_w(et[j0 + u][v]), xt[u][v], a0[u]);
      }
#pragma unroll
      for (int u = 0; u < JP; ++u) {
        const int j = j0 + u;
        float a, c;
        gda_update_wave(xr[j], yr[j], fmaf(SEQ ? a0[u] : a0[u] + a1[u], kos, cps[j]), gp, a, c);
        const bool ch = (a > 0.5f) != (xr[j] > 0.5f);
        wfl |= __builtin_amdgcn_ballot_w64(ch);
        xr[j] = a;
        yr[j] = c;
        const float xs = ch ? -a : a;
#pragma unroll
        for (int cc = 0; cc < NC; ++cc) ((float*)(lds + xo))[word(cc, j)] = xs;
      }
    }
    previous();  // here, not where dprev is read: the gathers do not wait for it
    __syncthreads();
    return false;
  };
  for (int s = 0;; s += 2) {
    if (iteration(res_u32<0>{}, s)) break;
    if (iteration(res_u32<XB>{}, s + 1)) break;
  }

#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int p = tid + j * kResThreads;
    if (p < n) {
      const int i = D.order[p];
      D.X[(size_t)b * D.ld + i] = xr[j];
      D.Y[(size_t)b * D.ld + i] = yr[j];
    }
  }
  if (tid == 0) {
    D.rbestF[b] = bF2 == LLONG_MAX ? bF2 : bF2 / 2;
    D.rbestT[b] = bT;
    D.rbestTs[b] = bTs;
    D.Flast[b] = F2 / 2;
    if (D.rtr) D.rtl[b] = ntr;
  }
}

// positions per thread: the compiled counts
int csr_resident_rows(int n) {
  const int r = (n + kResThreads - 1) / kResThreads;
  return r <= 1 ? 1 : r <= 2 ? 2 : r <= 4 ? 4 : r <= 8 ? 8 : r <= 16 ? 16 : 0;
}

int csr_resident_copies(int n) {
  switch (csr_resident_rows(n)) {
    case 1: return res_copies<1>();
    case 2: return res_copies<2>();
    case 4: return res_copies<4>();
    case 8: return res_copies<8>();
    default: return res_copies<16>();
  }
}

int csr_resident_word(int n, int c, int p) {
  return c * csr_resident_rows(n) * kResThreads + res_word(c, p);
}

static size_t csr_resident_lds(int n, int64_t nrent, bool ents) {
  return 2 * (size_t)csr_resident_copies(n) * csr_resident_rows(n) * kResThreads * 4 +
         (ents ? (size_t)nrent * 4 : 0) + kResSmall +
         (csr_resident_rows(n) <= 4 ? (size_t)csr_resident_rows(n) * kResThreads * 4 : 0);
}

bool csr_resident_staged(int n, int64_t nrent) { return csr_resident_lds(n, nrent, true) <= kResLds; }

template <int R, bool SEQ, int GK, bool LDSE>
static hipError_t launch_res_k(const CsrDev& d, int64_t t0, int nsteps, hipStream_t s) {
  auto kern = csr_resident<R, SEQ, GK, LDSE>;
  const size_t lds = csr_resident_lds(d.n, d.nrent, LDSE);
  hipError_t e = allow_lds((const void*)kern, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(d.B), dim3(kResThreads), lds, s, d, t0, nsteps);
  return hipGetLastError();
}

template <int R, int GK>
static hipError_t launch_res_r(const CsrDev& d, int64_t t0, int nsteps, hipStream_t s) {
  const bool in_lds = csr_resident_staged(d.n, d.nrent);
  if (d.seq)
    return in_lds ? launch_res_k<R, true, GK, true>(d, t0, nsteps, s)
                  : launch_res_k<R, true, GK, false>(d, t0, nsteps, s);
  return in_lds ? launch_res_k<R, false, GK, true>(d, t0, nsteps, s)
                : launch_res_k<R, false, GK, false>(d, t0, nsteps, s);
}

template <int GK>
static hipError_t launch_res(const CsrDev& d, int64_t t0, int nsteps, hipStream_t s) {
  switch (csr_resident_rows(d.n)) {
    case 1: return launch_res_r<1, GK>(d, t0, nsteps, s);
    case 2: return launch_res_r<2, GK>(d, t0, nsteps, s);
    case 4: return launch_res_r<4, GK>(d, t0, nsteps, s);
    case 8: return launch_res_r<8, GK>(d, t0, nsteps, s);
    case 16: return launch_res_r<16, GK>(d, t0, nsteps, s);
    default: return hipErrorInvalidValue;
  }
}

// ---- incumbent and trace of a call, from the restarts' own improvements ----
//
// A global improvement at iteration t is an improvement of its restart too, so
// the records the restarts kept (at most one per restart and iteration of the
// launch) hold them all: at each iteration the least (F, b) of its records is
// an improvement when F is below the incumbent and every earlier iteration's.
// The restarts run free of each other, so the time of an improvement is the
// latest of those up to its iteration: the incumbent of iteration t is known
// when every improvement up to t has been made, and times increase with t.
constexpr int kMergeThreads = 1024;

__global__ void __launch_bounds__(kMergeThreads)
    resident_merge_kernel(const TraceRec* __restrict__ rtr, const int32_t* __restrict__ rtl, int B,
                          int n, const uint8_t* __restrict__ best_xr, Incumbent* inc,
                          uint8_t* best_x, TraceRec* trace, int32_t* trace_len, int trace_cap,
                          int64_t* t_dev, int nsteps) {
  constexpr int NW = kMergeThreads / 64;
  // slot u: iteration t0 + u; slot 0 is the state the call started from
  __shared__ long long sF[kResTrace];
  __shared__ int sb[kResTrace];
  __shared__ int spos[kResTrace];
  __shared__ unsigned long long sts[kResTrace];  // times of the improvements, 0 elsewhere
  __shared__ long long wmin[NW];
  __shared__ int wcnt[NW];
  __shared__ int last;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int64_t t0 = *t_dev;
  const int64_t F0 = inc->F;
  const int len0 = *trace_len;
  for (int u = tid; u < kResTrace; u += kMergeThreads) {
    sF[u] = LLONG_MAX;
    sb[u] = INT_MAX;
    sts[u] = 0;
  }
  if (tid == 0) last = -1;
  __syncthreads();
  auto records = [&](auto f) {  // every record, by the waves
    for (int b = wid; b < B; b += NW) {
      const int m = rtl[b];
      for (int r = lane; r < m; r += 64) {
        const TraceRec q = rtr[(size_t)b * kResTrace + r];
        f(q, b, (int)(q.t - t0));
      }
    }
  };
  records([&](const TraceRec& q, int, int u) { atomicMin(&sF[u], (long long)q.F); });
  __syncthreads();
  records([&](const TraceRec& q, int b, int u) {
    if (q.F == sF[u]) atomicMin(&sb[u], b);
  });
  __syncthreads();
  // exclusive running minimum over the slots, one slot per thread
  static_assert(kResTrace == kMergeThreads, "one slot per thread");
  const int64_t F = sF[tid];
  int64_t m = F;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t v = __shfl_up(m, o);
    if (lane >= o && v < m) m = v;
  }
  if (lane == 63) wmin[wid] = m;
  __syncthreads();
  int64_t before = __shfl_up(m, 1);
  if (lane == 0) before = LLONG_MAX;
  for (int w = 0; w < wid; ++w) before = before < wmin[w] ? before : wmin[w];
  const bool imp = F < before && F < F0;
  const uint64_t bal = __ballot(imp);
  if (lane == 0) wcnt[wid] = __popcll(bal);
  __syncthreads();
  int pos = __popcll(bal & ((uint64_t(1) << lane) - 1));
  for (int w = 0; w < wid; ++w) pos += wcnt[w];
  spos[tid] = imp ? pos : -1;
  if (imp) atomicMax(&last, tid);
  __syncthreads();
  const int lu = last;
  records([&](const TraceRec& q, int b, int u) {
    if (spos[u] >= 0 && b == sb[u] && q.F == sF[u]) sts[u] = q.ts;
  });
  __syncthreads();
  // inclusive running maximum of the times
  uint64_t ts = sts[tid];
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t v = __shfl_up(ts, o);
    if (lane >= o && v > ts) ts = v;
  }
  if (lane == 63) wmin[wid] = (long long)ts;
  __syncthreads();
  for (int w = 0; w < wid; ++w) ts = ts > (uint64_t)wmin[w] ? ts : (uint64_t)wmin[w];
  if (imp) {
    const TraceRec q{t0 + tid, F, (int64_t)sb[tid], ts};
    const int at = len0 + pos;
    if (at < trace_cap) {
      trace[at] = q;
      if (tid == lu || at == trace_cap - 1) *trace_len = at + 1;
    } else if (tid == lu) {
      *trace_len = trace_cap;
    }
    if (tid == lu) *inc = Incumbent{q.F, q.t, q.b, q.ts};
  }
  if (lu >= 0) {
    // the winner's last improvement is its least objective, which is the
    // incumbent's: its kept vector is the incumbent's
    const uint8_t* src = best_xr + (size_t)sb[lu] * n;
    for (int i = tid; i < n; i += kMergeThreads) best_x[i] = src[i];
  }
  __syncthreads();
  if (tid == 0) *t_dev = t0 + nsteps;
}

hipError_t launch_resident_merge(const TraceRec* rtr, const int32_t* rtl, int B, int n,
                                 const uint8_t* best_xr, Incumbent* inc, uint8_t* best_x,
                                 TraceRec* trace, int32_t* trace_len, int trace_cap, int64_t* t_dev,
                                 int nsteps, hipStream_t s) {
  hipLaunchKernelGGL(resident_merge_kernel, dim3(1), dim3(kMergeThreads), 0, s, rtr, rtl, B, n, best_xr,
                     inc, best_x, trace, trace_len, trace_cap, t_dev, nsteps);
  return hipGetLastError();
}

hipError_t launch_csr_resident(const CsrDev& d, int64_t t0, int nsteps, hipStream_t s) {
  // a launch has at most one record per iteration (the starting state's among
  // them) and restart: calls are cut so that these fit
  for (int done = 0; done < nsteps;) {
    const int k = d.rtr ? (nsteps - done < kResTrace - 1 ? nsteps - done : kResTrace - 1) : nsteps - done;
    hipError_t e = d.gp.gkind == 0 ? launch_res<0>(d, t0 + done, k, s) : launch_res<1>(d, t0 + done, k, s);
    if (e != hipSuccess) return e;
    if (d.rtr) {
      e = launch_resident_merge(d.rtr, d.rtl, d.B, d.n, d.best_xr, d.inc, d.best_x, d.trace, d.trace_len,
                                d.trace_cap, d.t_dev, k, s);
      if (e != hipSuccess) return e;
    }
    done += k;
  }
  return hipSuccess;
}

}  // namespace pdbo

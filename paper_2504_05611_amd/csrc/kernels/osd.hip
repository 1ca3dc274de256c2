// OSD-0 (order-0 ordered-statistics decoding) and OSD-CS for the shots BP did
// not converge on: the elimination kernels and their launchers.  The decoder's
// BP side (decode.hip) hands over the FP32 posteriors of those shots through a
// device queue; see decode.hip for the whole pipeline.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>

#include "../host/device.h"
#include "../host/timing.h"
#include "decoder.h"

namespace tmcs {
namespace dec {



// Posteriors each thread has in flight in the selection passes: 8 in the
// windowed variant (hundreds of thousands of columns; 20-25 % faster there),
// 1 in the prefix variant (at most 16384 columns: the registers cost it a
// workgroup per SIMD, 50 % slower on BB [[144,12,12]] teleport).
template <bool WIN>
constexpr int sel_unroll() { return WIN ? 8 : 1; }

// Coherent (L2) 32-bit load: rowmap entries are updated with atomics and by
// other waves of the workgroup within one shot.
__device__ __forceinline__ int32_t ld_l2(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Inclusive prefix sum over the 64 lanes of a wave.
__device__ __forceinline__ int wave_incl_scan(int x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  return x;
}

__device__ __forceinline__ uint32_t order_key(float x) {
  if (x == 0.0f) x = 0.0f;   // -0 and +0 compare equal
  const uint32_t b = __float_as_uint(x);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Wave-uniform broadcast of lane `src`'s 64-bit value (src must be wave-uniform).
__device__ __forceinline__ uint64_t bcast64(uint64_t x, int src) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, src);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), src);
  return ((uint64_t)hi << 32) | lo;
}

// Bitonic sort of npad = (threads) * KPT 64-bit keys, ascending.  Thread t
// holds elements t*KPT .. t*KPT+KPT-1 in registers; partners within a thread are
// compared in registers, partners within a wave via lane shuffles, and only the
// strides that cross waves go through LDS (`keys`), which also receives the low
// 32 bits (the column indices) of the sorted keys.
template <int KPT>
__device__ __forceinline__ void bitonic_sort_regs(uint64_t (&x)[KPT], uint64_t* keys, int npad) {
  const int tid = threadIdx.x;
  for (int k = 2; k <= npad; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      if (j < KPT) {
#pragma unroll
        for (int jj = KPT / 2; jj >= 1; jj >>= 1) {
          if (jj != j) continue;
#pragma unroll
          for (int r = 0; r < KPT; ++r) {
            if (r & jj) continue;
            const int e = tid * KPT + r;
            const bool up = (e & k) == 0;
            const uint64_t a0 = x[r], a1 = x[r | jj];
            const bool sw = (a0 > a1) == up;
            x[r] = sw ? a1 : a0;
            x[r | jj] = sw ? a0 : a1;
          }
        }
      } else if (j < KPT * 64) {
        const int tj = j / KPT;                       // partner lane distance
        const bool lower = (tid & tj) == 0;
#pragma unroll
        for (int r = 0; r < KPT; ++r) {
          const int e = tid * KPT + r;
          const bool up = (e & k) == 0;
          const uint64_t y = __shfl_xor(x[r], tj, 64);
          // the lower element of the pair keeps the minimum when sorting up
          const bool take_min = lower == up;
          x[r] = take_min ? (x[r] < y ? x[r] : y) : (x[r] > y ? x[r] : y);
        }
      } else {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < KPT; ++r) keys[tid * KPT + r] = x[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < KPT; ++r) {
          const int e = tid * KPT + r;
          const bool up = (e & k) == 0;
          const uint64_t y = keys[e ^ j];
          const bool take_min = ((e & j) == 0) == up;
          x[r] = take_min ? (x[r] < y ? x[r] : y) : (x[r] > y ? x[r] : y);
        }
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < KPT; ++r) {
    ((uint32_t*)keys)[tid * KPT + r] = (uint32_t)x[r];
  }
  __syncthreads();
}

// The (L_v, v) order of every job's columns, for the dense variants with 256
// threads: row job of `out` gets the column indices.  In place of the posteriors
// (out = llr) where nothing reads them afterwards.
//
// A kernel of its own: up to 16384 8-byte keys take 128 KB of LDS, which the
// elimination then held for its whole length, one workgroup per compute unit and
// mostly one wave of its four at work, and the keys' registers (252, with spills)
// allowed no second one either.  OSD-CS of order 7 on 8192 shots of the BB
// [[144,12,12]] memory experiment (1822 jobs): 36.0 ms with the sort inside, 17.5
// without it and 1.8 here (16 waves sort a job, not 4).
template <int KPT, int NT>
__global__ void __launch_bounds__(NT) k_osd_sort(const float* llr, int32_t* out, int n, const int32_t* jobs,
                                                 const int32_t* counters, int cnt_total) {
  extern __shared__ __align__(8) unsigned char sm[];
  uint64_t* keys = (uint64_t*)sm;                                  // [NT * KPT]
  const int tid = threadIdx.x, total = counters[cnt_total];
  for (int jn = (int)blockIdx.x; jn < total; jn += (int)gridDim.x) {
    const int64_t row = (int64_t)(jobs ? jobs[jn] : jn) * n;
    uint64_t x[KPT];
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
      const int i = r * NT + tid;
      x[r] = i < n ? (((uint64_t)order_key(llr[row + i]) << 32) | (uint32_t)i) : ~0ull;
    }
    bitonic_sort_regs<KPT>(x, keys, NT * KPT);
    for (int i = tid; i < n; i += NT) out[row + i] = ((const int32_t*)keys)[i];
    __syncthreads();
  }
}

// Bit p of a register-resident bit vector (p < 64 * MW).
template <int MW, int W>
__device__ __forceinline__ uint64_t bit_of(const uint64_t (&v)[W], int p) {
  uint64_t pw = 0ull;
#pragma unroll
  for (int w = 0; w < MW; ++w)
    if ((p >> 6) == w) pw = v[w];
  return (pw >> (p & 63)) & 1ull;
}

// W = words per basis vector: MW syndrome words then RW combination words.
//
// The basis is kept fully reduced: basis vector i has a 1 at its pivot row p_i
// and 0 at every other pivot row.  A candidate column h is then reduced by
// XORing exactly the basis vectors whose pivot rows lie in supp(h) (at most the
// column degree).  New basis vectors are created up to 63 at a time by one wave,
// made fully reduced among themselves, and the older vectors are then reduced
// against them.
//
// The syndrome rides along in lane 63 of the wave that is creating them, so it is
// reduced by each new vector like a candidate, at no cost, and OSD-0 stops at the
// very column that completes the span.  Few columns are needed (median / largest
// of 40 shots: BB [[144,12,12]] teleportation 27 / 169, memory at p = 2e-3 37 /
// 112, weight-6 Pauli string 10 / 34); looking only after every 256 candidates
// built 116 vectors a shot on the teleportation circuit, 2.2 us each with the
// reductions that follow, where the chain of pivots is all there is to do.
// Milliseconds before and after: 11.0 and 3.0 there (32768 shots, 36 % in OSD),
// 1.7 and 0.33 on the Pauli string, 2.2 and 0.92 on the memory.
// Combination words that no column has reached yet are zero and left out in the
// variants that stop early (those that run to full rank lose more by the branch
// per word: 51 instead of 36 ms of OSD-CS on 8192 shots of that circuit).
// BL: the basis lives in LDS (after the sort keys) instead of HBM.
// NT: threads per workgroup (64: one wave decodes a shot on its own).
//
// WIN (DEMs beyond the dense limits): the scan that ends at the early stop only
// ever looks at a prefix of the sorted order, and those columns touch few rows.
// The shot therefore works on a window: the npad - 1 smallest keys at most
// (radix selection, then a sort), cut where the rows they touch would exceed
// win_rows, with those rows renumbered 0, 1, ... in order of first touch.  Kept
// columns are zero outside the window's rows, so independence tests, the early
// stop and the solution are exactly those of the full OSD-0 whenever s is
// spanned inside the window.  Otherwise (window too small) the shot keeps BP's
// hard decision and is flagged (flags bit 3, stats osd_incomplete).
//
// PFX (DEMs within the dense limits but wider than npad): the same selection
// gives the npad - 1 smallest keys, and the elimination runs on that prefix of
// the order with H's own rows.  If s is spanned there, the result is the full
// OSD-0's; otherwise the job goes to a retry list, which the full-sort variant
// then decodes, so every shot gets the exact OSD-0 correction.
//
// MULTI (windowed variant only): one launch serves the OSD queues of several
// decode items; job g of a counter shared by the launch belongs to item i with
// pref[i] <= g < pref[i + 1] (prefix sums of the items' queue lengths), and the
// workgroup switches to that item's arguments, basis and row table.  Every
// item's window has the same shape (npad = WIN_KEYS, 64 MW local rows), so the
// LDS layout does not change.
template <int MW, int RW, int KPT, bool BL, int NT, bool WIN = false, bool PFX = false, bool MULTI = false>
// (dense, 256 threads: three workgroups per compute unit where the vectors leave the registers for it)
__global__ void __launch_bounds__(NT, !BL && !WIN && !PFX && MW <= 15 ? 3 : 1) k_osd(OSDArgs a, OSDMulti mu) {
  constexpr int W = MW + RW;
  static_assert(!(WIN && BL), "the window variant keeps its basis in HBM");
  static_assert(!(WIN && PFX), "one front end per variant");
  static_assert(!MULTI || WIN, "multi-item launches use the windowed variant");
  constexpr bool SORTED = !BL && !WIN && !PFX;                     // the order comes from k_osd_sort
  extern __shared__ __align__(8) unsigned char sm[];
  // local capacity: rank and rows of the problem the elimination sees
  const int cap_r = WIN ? 64 * MW : a.rank;
  const int cap_m = WIN ? 64 * MW : a.m;
  uint64_t* keys = (uint64_t*)sm;                                  // [npad] (BL, WIN: u32 column indices; SORTED: none)
  uint64_t* lbasis = BL ? (uint64_t*)((uint32_t*)sm + a.npad) : keys + a.npad;   // BL: [rank][W]
  // [rank] pivot row of basis i
  int32_t* pivot = (int32_t*)(BL ? lbasis + (size_t)a.rank * W : SORTED ? keys : keys + a.npad);
  int32_t* kept = pivot + cap_r;                                   // [rank] column of basis i
  int32_t* prow = kept + cap_r;                                    // [m] basis index of a pivot row, or -1
  // (an offset from sm, not an integer cast, so that the compiler keeps LDS addressing)
  const size_t acc_off = ((size_t)((unsigned char*)(prow + cap_m) - sm) + 7) & ~(size_t)7;
  // [W] s + the basis vectors taken into it: zero on every pivot row.  Its syndrome
  // part is zero iff s lies in the span of the kept columns, and its combination
  // part then names the kept columns whose sum is s.
  uint64_t* acc = (uint64_t*)(sm + acc_off);
  uint32_t* tk = (uint32_t*)(acc + W);                             // OSD-CS: [npad / 32] kept sorted positions
  // WIN: after the sort, keys holds npad u32 column indices followed by npad
  // per-position counts (then exclusive offsets) of newly touched rows
  int32_t* pcnt = (int32_t*)keys + a.npad;
  __shared__ int s_job, s_r, s_done, s_inc, s_inst;
  __shared__ int s_pref[MAX_MULTI_OSD + 1];
  __shared__ uint64_t s_red;
  __shared__ unsigned long long s_best;     // OSD-CS: (order key of the soft weight, candidate rank)
  __shared__ int s_tpos[64], s_nt, s_f1, s_f2;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  uint64_t* B = BL ? lbasis : a.basis + (int64_t)blockIdx.x * cap_r * W;
  int32_t* fpos = WIN ? a.rowmap + (int64_t)blockIdx.x * 2 * a.m : nullptr;   // [m] first window position
  int32_t* lmap = WIN ? fpos + a.m : nullptr;                                  // [m] local row index
  int cur = -1;                                                                // MULTI: current item
  // A workgroup's first job is its own number; the others come from the counter.
  // (A counter gives out about 85 values a microsecond: thousands of workgroups
  // asking for a first job took 50 us of every launch, most of them for none.)
  int total = 0;                                                               // MULTI: thread 0's
  if constexpr (MULTI) {
    if (tid == 0) {
      s_pref[0] = 0;
      for (int i = 0; i < mu.n; ++i) s_pref[i + 1] = s_pref[i] + mu.tab[i].counters[mu.tab[i].cnt_total];
      total = s_pref[mu.n];
    }
  } else {
    total = a.counters[a.cnt_total];
    if ((int)blockIdx.x >= total) return;
  }
  bool first_job = true;
  auto next_job = [&]() -> int {                                               // thread 0
    if (first_job) return (int)blockIdx.x;
    if (total <= (int)gridDim.x) return total;
    return (int)gridDim.x + atomicAdd(MULTI ? mu.next : &a.counters[a.cnt_next], 1);
  };
  while (true) {
    if (tid == 0) {
      if constexpr (MULTI) {
        const int g = next_job();
        int i = 0;
        while (i < mu.n && g >= s_pref[i + 1]) ++i;
        s_inst = i;
        s_job = i < mu.n ? g - s_pref[i] : 0;
      } else {
        s_job = next_job();
      }
      first_job = false;
    }
    __syncthreads();
    const int jn = s_job;
    if constexpr (MULTI) {
      const int inst = s_inst;
      __syncthreads();
      if (inst >= mu.n) break;
      if (inst != cur) {                     // uniform: the workgroup moves to the next item
        cur = inst;
        a = mu.tab[inst];
        B = a.basis + (int64_t)blockIdx.x * cap_r * W;
        fpos = a.rowmap + (int64_t)blockIdx.x * 2 * a.m;
        lmap = fpos + a.m;
      }
    } else {
      __syncthreads();
      if (jn >= total) break;
    }
    const int job = a.jobs ? a.jobs[jn] : jn;
    const int64_t ls = a.osd_queue[job];
    const int64_t shot = a.shot0 + ls;
    const float* L = a.osd_llr + (int64_t)job * a.n;
    int n_loc = a.n, rank_loc = a.rank, n0 = a.n;
    if (tid == 0) { s_r = 0; s_done = 0; s_inc = 0; }
    if (tid < W) acc[tid] = !WIN && tid < a.mw ? a.synd[ls * a.mw + tid] : 0ull;
    __syncthreads();
    const int32_t* order = SORTED ? a.sorted + (int64_t)job * a.n : nullptr;
    if constexpr (!WIN && !PFX) {
      // 1. sort columns by (L_v, v)
      for (int r = tid; r < a.m; r += NT) prow[r] = -1;
      if (a.order > 0)
        for (int i = tid; i < (a.npad >> 5); i += NT) tk[i] = 0u;
      if constexpr (!SORTED) {
        uint64_t x[KPT];
#pragma unroll
        for (int r = 0; r < KPT; ++r) {
          const int i = tid * KPT + r;
          x[r] = i < a.n ? (((uint64_t)order_key(L[i]) << 32) | (uint32_t)i) : ~0ull;
        }
        bitonic_sort_regs<KPT>(x, keys, a.npad);
      }
      __syncthreads();
    } else {
      __shared__ int s_hist[256];
      __shared__ int s_wsum[NT / 64];
      __shared__ int s_sel, s_want, s_in, s_cnt, s_cut, s_total;
      if (tid == 0) s_cnt = 0;
      __syncthreads();
      // 1a. the window: every key below the npad-th smallest 32-bit order key, so
      // at most npad - 1 columns, and all of them when n < npad
      constexpr int SEL_UNROLL = sel_unroll<WIN>();
      // f(key, v) for every column, SEL_UNROLL posteriors per thread in flight
      // (unconditional loads: the last index is clamped and masked out afterwards)
      auto each = [&](auto f) {
        for (int v0 = tid; v0 < a.n; v0 += NT * SEL_UNROLL) {
          uint32_t k[SEL_UNROLL];
#pragma unroll
          for (int i = 0; i < SEL_UNROLL; ++i) {
            const int v = v0 + i * NT;
            k[i] = order_key(L[v < a.n ? v : a.n - 1]);
          }
#pragma unroll
          for (int i = 0; i < SEL_UNROLL; ++i)
            if (v0 + i * NT < a.n) f(k[i], v0 + i * NT);
        }
      };
      // the (npad - 1)-th (from 0) of the keys that `walk` goes over: radix selection, 8 bits per pass
      auto select8 = [&](auto walk) -> uint32_t {
        uint32_t pre = 0u;
        int want = a.npad - 1;
        for (int pass = 0; pass < 4; ++pass) {
          const int sh = 24 - 8 * pass;
          const uint32_t hmask = pass == 0 ? 0u : (0xFFFFFFFFu << (sh + 8));
          for (int i = tid; i < 256; i += NT) s_hist[i] = 0;
          __syncthreads();
          walk([&](uint32_t k, int) {
            if ((k & hmask) == (pre & hmask)) atomicAdd(&s_hist[(k >> sh) & 255u], 1);
          });
          __syncthreads();
          if (wave == 0) {
            int c[4], t = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) { c[q] = s_hist[lane * 4 + q]; t += c[q]; }
            const int incl = wave_incl_scan(t);
            int e = incl - t;
            if (e <= want && want < incl) {
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                if (e <= want && want < e + c[q]) { s_sel = lane * 4 + q; s_want = want - e; }
                e += c[q];
              }
            }
          }
          __syncthreads();
          pre |= (uint32_t)s_sel << sh;
          want = s_want;
          __syncthreads();
        }
        return pre;
      };
      uint32_t kstar = 0xFFFFFFFFu;
      bool listed = false;             // the window's keys are in place
      const bool all = a.n < a.npad;
      if constexpr (!WIN) {
        if (!all) kstar = select8(each);
      } else if (!all) {
        // A histogram of the upper 11 bits (a quarter of an octave per bin) tells a
        // bin with the wanted key; if the keys up to that bin's end fit in the LDS
        // from `keys` to `acc`, they are gathered and the exact key is found there.
        // Otherwise the bin is divided by the next 11 bits, and by the last 10.
        // Two to four passes over the posteriors (four where the cut falls among many
        // equal ones), where 8 bits at a time take four and a fifth to gather.  They run at the memory's rate (0.4 MB
        // a shot): on the d = 21 CNOT, 4096 shots, 3.85 before and 3.18 ms now, and its
        // retries 2.62 and 2.24 ms.  The prefix variants' posteriors come from L2,
        // and what the list adds cost BB [[144,12,12]] teleportation 7 %.
        static_assert(NT == 256 && KPT >= 4, "eight bins per thread, in the place of the keys");
        constexpr int LIST = 2 * KPT;  // gathered keys per thread
        const int cap = min((int)(acc_off / 8), NT * LIST);
        int32_t* hist = (int32_t*)keys;
        uint32_t pre = 0u;
        int want = a.npad - 1, below = 0, sh = 32;
        bool fits = false;
        do {
          const int d = sh > 11 ? 11 : sh;
          const uint32_t hmask = sh == 32 ? 0u : 0xFFFFFFFFu << sh;
          sh -= d;
          for (int i = tid; i < 2048; i += NT) hist[i] = 0;
          __syncthreads();
          each([&](uint32_t k, int) {
            if ((k & hmask) == pre) atomicAdd(&hist[(k >> sh) & ((1u << d) - 1)], 1);
          });
          __syncthreads();
          int c[8], t = 0;
#pragma unroll
          for (int q = 0; q < 8; ++q) { c[q] = hist[tid * 8 + q]; t += c[q]; }
          const int incl = wave_incl_scan(t);
          if (lane == 63) s_wsum[wave] = incl;
          __syncthreads();
          int e = incl - t;
          for (int q = 0; q < wave; ++q) e += s_wsum[q];
          if (e <= want && want < e + t) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
              if (e <= want && want < e + c[q]) { s_sel = tid * 8 + q; s_want = want - e; s_in = c[q]; }
              e += c[q];
            }
          }
          __syncthreads();
          pre |= (uint32_t)s_sel << sh;
          below += want - s_want;
          want = s_want;
          fits = below + s_in <= cap;
          __syncthreads();
        } while (sh > 0 && !fits);
        if (fits) {
          const uint32_t last = pre | (uint32_t)((1ull << sh) - 1ull);
          each([&](uint32_t k, int v) {
            if (k <= last) keys[atomicAdd(&s_cnt, 1)] = ((uint64_t)k << 32) | (uint32_t)v;
          });
          __syncthreads();
          const int got = s_cnt;
          kstar = select8([&](auto f) {
            for (int i = tid; i < got; i += NT) f((uint32_t)(keys[i] >> 32), i);
          });
          uint64_t x[LIST];
#pragma unroll
          for (int r = 0; r < LIST; ++r) x[r] = tid + r * NT < got ? keys[tid + r * NT] : ~0ull;
          if (tid == 0) s_cnt = 0;
          __syncthreads();
#pragma unroll
          for (int r = 0; r < LIST; ++r)
            if ((uint32_t)(x[r] >> 32) < kstar) keys[atomicAdd(&s_cnt, 1)] = x[r];
          listed = true;
        } else {
          kstar = pre;
        }
      }
      // 1b. gather and sort the window's keys
      if (!listed)
        each([&](uint32_t k, int v) {
          if (all || k < kstar) keys[atomicAdd(&s_cnt, 1)] = ((uint64_t)k << 32) | (uint32_t)v;
        });
      __syncthreads();
      n0 = s_cnt;
      uint64_t x[KPT];
#pragma unroll
      for (int r = 0; r < KPT; ++r) {
        const int i = tid * KPT + r;
        x[r] = i < n0 ? keys[i] : ~0ull;
      }
      bitonic_sort_regs<KPT>(x, keys, a.npad);
      const uint32_t* col32 = (const uint32_t*)keys;
      if constexpr (PFX) {
        // the prefix of the order, on H's rows
        n_loc = n0;
        for (int r = tid; r < a.m; r += NT) prow[r] = -1;
        __syncthreads();
      } else {
      // 1c. first window position touching each row
      for (int j = tid; j < n0; j += NT) {
        const int col = (int)col32[j];
        for (int32_t k = a.col_ptr[col]; k < a.col_ptr[col + 1]; ++k) atomicMin(&fpos[a.csc_row[k]], j);
      }
      if (tid == 0) s_cut = n0;
      __syncthreads();
      // 1d. rows first touched at each position, exclusive offsets, and the cut:
      // the first position whose new rows would exceed win_rows
      int cnt[KPT], tsum = 0;
#pragma unroll
      for (int r = 0; r < KPT; ++r) {
        const int j = tid * KPT + r;
        cnt[r] = 0;
        if (j < n0) {
          const int col = (int)col32[j];
          for (int32_t k = a.col_ptr[col]; k < a.col_ptr[col + 1]; ++k) cnt[r] += ld_l2(&fpos[a.csc_row[k]]) == j;
        }
        tsum += cnt[r];
      }
      const int wincl = wave_incl_scan(tsum);
      if (lane == 63) s_wsum[wave] = wincl;
      __syncthreads();
      int off = wincl - tsum;
      for (int q = 0; q < wave; ++q) off += s_wsum[q];
      if (tid == NT - 1) s_total = off + tsum;
#pragma unroll
      for (int r = 0; r < KPT; ++r) {
        const int j = tid * KPT + r;
        if (j < n0) {
          pcnt[j] = off;
          if (off + cnt[r] > a.win_rows) atomicMin(&s_cut, j);
        }
        off += cnt[r];
      }
      __syncthreads();
      n_loc = s_cut;
      rank_loc = n_loc < n0 ? pcnt[n_loc] : s_total;      // rows of the window = bound on its rank
      // 1e. local row numbers, in order of first touch
      for (int j = tid; j < n_loc; j += NT) {
        const int col = (int)col32[j];
        int t = pcnt[j];
        for (int32_t k = a.col_ptr[col]; k < a.col_ptr[col + 1]; ++k) {
          const int r = a.csc_row[k];
          if (ld_l2(&fpos[r]) == j) __hip_atomic_store(&lmap[r], t++, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
      for (int r = tid; r < rank_loc; r += NT) prow[r] = -1;
      __syncthreads();
      // 1f. the syndrome in local rows; a detection event outside the window
      // cannot be spanned by it
      for (int wd = tid; wd < a.mw; wd += NT) {
        uint64_t x = a.synd[ls * a.mw + wd];
        for (; x; x &= x - 1) {
          const int r = wd * 64 + (__ffsll((unsigned long long)x) - 1);
          if (ld_l2(&fpos[r]) >= n_loc) s_inc = 1;
          else {
            const int lr = ld_l2(&lmap[r]);
            atomicXor((unsigned long long*)&acc[lr >> 6], (unsigned long long)(1ull << (lr & 63)));
          }
        }
      }
      __syncthreads();
      }
    }
    // WIN, PFX: every column of H is in the window, so the result is the full OSD-0's
    const bool whole = !(WIN || PFX) || n_loc == a.n;
    const bool skip = WIN && !whole && s_inc;
    // rows of the elimination: H's, or the window's local numbers
    auto row_of = [&](int32_t k) -> int {
      const int r = a.csc_row[k];
      if constexpr (WIN) return ld_l2(&lmap[r]);
      else return r;
    };
    // 2. information set, 63 sorted candidates per wave and pass
    constexpr bool EARLY = WIN || PFX;
    const bool early = EARLY || a.order == 0;
    for (int base = 0; base < (skip ? 0 : n_loc); base += 63 * (NT / 64)) {
      const int r_start = s_r;
      __syncthreads();           // every wave has read s_r before wave 0 advances it
      if (r_start >= rank_loc || s_done) break;
      const int idx = base + 63 * wave + lane;
      const int col = lane < 63 && idx < n_loc ? (SORTED ? order[idx] : ((const int32_t*)keys)[idx]) : -1;
      uint64_t v[W];
#pragma unroll
      for (int w = 0; w < W; ++w) v[w] = 0ull;
      if (col >= 0) {
        const int32_t k0 = a.col_ptr[col], k1 = a.col_ptr[col + 1];
        for (int32_t k = k0; k < k1; ++k) {
          const int r = row_of(k);
#pragma unroll
          for (int w = 0; w < MW; ++w)
            if ((r >> 6) == w) v[w] ^= 1ull << (r & 63);
        }
        // phase 1: the basis vectors pivoted on rows of h
        for (int32_t k = k0; k < k1; ++k) {
          const int i = prow[row_of(k)];
          if (i >= 0) {
            const uint64_t* b = B + (int64_t)i * W;
#pragma unroll
            for (int w = 0; w < W; ++w) v[w] ^= b[w];
          }
        }
      }
      __syncthreads();           // phase 1 everywhere before any wave publishes new pivots
      int r_done = r_start;
      for (int q = 0; q < NT / 64; ++q) {
        if (wave == q) {
          // phase 2: in-order pass over this wave's candidates whose syndrome
          // part is still nonzero (zero ones depend on earlier columns)
          if (lane == 63) {
#pragma unroll
            for (int w = 0; w < W; ++w) v[w] = acc[w];
          }
          int r = r_done;
          int mine = -1;      // pivot row of the basis vector this lane became
          auto nonzero = [&]() -> uint64_t {
            uint64_t o = 0ull;
#pragma unroll
            for (int w = 0; w < MW; ++w) o |= v[w];
            return __ballot(o != 0ull);
          };
          constexpr uint64_t SYND = 1ull << 63;
          uint64_t nz = nonzero(), live = nz & ~SYND;
          while (live && r < rank_loc && (!early || (nz & SYND))) {
            const int j = __ffsll((unsigned long long)live) - 1;
            uint64_t b[MW];
#pragma unroll
            for (int w = 0; w < MW; ++w) b[w] = bcast64(v[w], j);
            int p = -1;
#pragma unroll
            for (int w = 0; w < MW; ++w)
              if (p < 0 && b[w]) p = w * 64 + (__ffsll((unsigned long long)b[w]) - 1);
            if (lane == j) {
              mine = p;
              pivot[r] = p;
              kept[r] = col;
              prow[p] = r;
              if (!WIN && !PFX && a.order > 0) atomicOr(&tk[idx >> 5], 1u << (idx & 31));
            }
            const uint64_t mask = (lane > j) ? 0ull - bit_of<MW, W>(v, p) : 0ull;
#pragma unroll
            for (int w = 0; w < MW; ++w) v[w] ^= b[w] & mask;
#pragma unroll
            for (int w = 0; w < RW; ++w) {
              if (EARLY && 64 * w > r) break;
              const uint64_t own = w == (r >> 6) ? 1ull << (r & 63) : 0ull;    // the column itself
              if (lane == j) v[MW + w] ^= own;
              v[MW + w] ^= bcast64(v[MW + w], j) & mask;
            }
            ++r;
            nz = nonzero();
            live = nz & ~SYND & (~1ull << j);
          }
          const bool done = early && !(nz & SYND);
          if (lane == 63) {
#pragma unroll
            for (int w = 0; w < W; ++w) acc[w] = v[w];
            s_r = r;
            if (done) s_done = 1;
          }
          if (!done) {
            // make the new vectors fully reduced among themselves (latest first)
            uint64_t piv_lanes = __ballot(mine >= 0);
            while (piv_lanes) {
              const int j = 63 - __clzll((long long)piv_lanes);
              piv_lanes &= ~(1ull << j);
              const int pj = __builtin_amdgcn_readlane(mine, j);
              const uint64_t mask = (mine >= 0 && lane < j) ? 0ull - bit_of<MW, W>(v, pj) : 0ull;
#pragma unroll
              for (int w = 0; w < MW; ++w) v[w] ^= bcast64(v[w], j) & mask;
#pragma unroll
              for (int w = 0; w < RW; ++w) {
                if (EARLY && 64 * w >= r) break;
                v[MW + w] ^= bcast64(v[MW + w], j) & mask;
              }
            }
            if (mine >= 0) {
              const int i = prow[mine];
#pragma unroll
              for (int w = 0; w < W; ++w) B[(int64_t)i * W + w] = v[w];
            }
          }
        }
        __syncthreads();
        // Stop as soon as s lies in the span of the kept columns.  Columns of the
        // full information set are independent, so s has exactly one
        // representation over them; the one found here (zero on the columns not
        // yet kept) is it, and the rest of the scan could only add zeros.
        if (s_done) break;       // (uniform; the loop over base ends there too)
        const int r_new = s_r;
        if (r_new > r_done) {
          // older basis vectors: clear their bits at the new pivots
          for (int i = tid; i < r_done; i += NT) {
            uint64_t bi[W];
#pragma unroll
            for (int w = 0; w < W; ++w) bi[w] = B[(int64_t)i * W + w];
            bool changed = false;
            for (int j = r_done; j < r_new; ++j) {
              if (bit_of<MW, W>(bi, pivot[j])) {
                const uint64_t* bj = B + (int64_t)j * W;
#pragma unroll
                for (int w = 0; w < W; ++w) bi[w] ^= bj[w];
                changed = true;
              }
            }
            if (changed) {
#pragma unroll
              for (int w = 0; w < W; ++w) B[(int64_t)i * W + w] = bi[w];
            }
          }
          // candidates of later waves: reduce against the new vectors
          if (wave > q) {
            uint64_t m[W];
#pragma unroll
            for (int w = 0; w < W; ++w) m[w] = 0ull;
            for (int j = r_done; j < r_new; ++j) {
              const uint64_t msk = 0ull - bit_of<MW, W>(v, pivot[j]);
              const uint64_t* bj = B + (int64_t)j * W;
#pragma unroll
              for (int w = 0; w < W; ++w) m[w] ^= bj[w] & msk;
            }
#pragma unroll
            for (int w = 0; w < W; ++w) v[w] ^= m[w];
          }
        }
        r_done = r_new;
        __syncthreads();
      }
    }
    // 3. the solution is in acc
    __syncthreads();
    const int r = s_r;
    int left = skip ? 1 : 0;
    for (int w = tid; w < MW; w += NT) left |= acc[w] != 0ull;
    const int unspanned = __syncthreads_or(left);
    // WIN: a window that does not span s says nothing about H unless it is all of H
    const bool incomplete = unspanned && !whole;
    const int not_in_span = unspanned && whole;
    // the row table of a windowed shot is left all-sentinel for the next one
    auto reset_rows = [&]() {
      if constexpr (WIN) {
        const uint32_t* col32 = (const uint32_t*)keys;
        for (int j = tid; j < n0; j += NT) {
          const int col = (int)col32[j];
          for (int32_t k = a.col_ptr[col]; k < a.col_ptr[col + 1]; ++k)
            __hip_atomic_store(&fpos[a.csc_row[k]], WIN_NONE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    };
    if ((PFX || (WIN && a.retry)) && incomplete) {
      // PFX: the full sort decides this one; WIN with a retry list (the smaller
      // first window): the full window does
      if (tid == 0) a.retry[atomicAdd(&a.counters[a.cnt_retry], 1)] = job;
      reset_rows();
      __syncthreads();
      continue;
    }
    if constexpr (!WIN && !PFX) {
      if (tid == 0) { s_f1 = -1; s_f2 = -1; }
      if (a.order > 0 && !not_in_span) {
        // OSD-CS: T = sorted positions not kept; candidates e_T of weight one over
        // T and of weight two over T's first `order` positions.  The soft weight of
        // a candidate sums L over e_S + rep(e_T) (kept columns in order of
        // selection) and then over e_T; the lightest wins, ties to the earlier.
        auto col_at = [&](int p) -> int {
          return SORTED ? order[p] : ((const int32_t*)keys)[p];
        };
        auto weight = [&](int c1, int c2) -> float {
          uint64_t x[RW];
#pragma unroll
          for (int w = 0; w < RW; ++w) x[w] = acc[MW + w];
          for (int q = 0; q < 2; ++q) {
            const int cc = q ? c2 : c1;
            if (cc < 0) continue;
            for (int32_t k = a.col_ptr[cc]; k < a.col_ptr[cc + 1]; ++k) {
              const int pi = prow[a.csc_row[k]];
              if (pi >= 0) {
                const uint64_t* bp = B + (int64_t)pi * W + MW;
#pragma unroll
                for (int w = 0; w < RW; ++w) x[w] ^= bp[w];
              }
            }
          }
          float c = 0.0f;
#pragma unroll
          for (int w = 0; w < RW; ++w)
            for (uint64_t y = x[w]; y; y &= y - 1) c = __fadd_rn(c, L[kept[w * 64 + (__ffsll((unsigned long long)y) - 1)]]);
          if (c1 >= 0) c = __fadd_rn(c, L[c1]);
          if (c2 >= 0) c = __fadd_rn(c, L[c2]);
          return c;
        };
        auto pair_of = [](int q, int nt, int* pa, int* pb) {
          int a0 = 0;
          while (q >= nt - 1 - a0) { q -= nt - 1 - a0; ++a0; }
          *pa = a0;
          *pb = a0 + 1 + q;
        };
        if (tid == 0) {
          int cnt = 0;
          for (int p = 0; p < n_loc && cnt < a.order; ++p)
            if (!((tk[p >> 5] >> (p & 31)) & 1u)) s_tpos[cnt++] = p;
          s_nt = cnt;
          s_best = ((unsigned long long)order_key(weight(-1, -1)) << 32);   // OSD-0 itself, rank 0
        }
        __syncthreads();
        unsigned long long best = ~0ull;
        for (int p = tid; p < n_loc; p += NT) {
          if ((tk[p >> 5] >> (p & 31)) & 1u) continue;
          const unsigned long long key = ((unsigned long long)order_key(weight(col_at(p), -1)) << 32) | (uint32_t)(1 + p);
          best = key < best ? key : best;
        }
        const int nt = s_nt, npairs = nt * (nt - 1) / 2;
        for (int q = tid; q < npairs; q += NT) {
          int ia, ib;
          pair_of(q, nt, &ia, &ib);
          const unsigned long long key = ((unsigned long long)order_key(weight(col_at(s_tpos[ia]), col_at(s_tpos[ib]))) << 32)
                                         | (uint32_t)(1 + a.npad + q);
          best = key < best ? key : best;
        }
        atomicMin(&s_best, best);
        __syncthreads();
        if (tid == 0) {
          const uint32_t rk = (uint32_t)(s_best & 0xFFFFFFFFu);
          int c1 = -1, c2 = -1;
          if (rk >= 1 && rk <= (uint32_t)a.npad) {
            c1 = col_at((int)rk - 1);
          } else if (rk > (uint32_t)a.npad) {
            int ia, ib;
            pair_of((int)rk - 1 - a.npad, nt, &ia, &ib);
            c1 = col_at(s_tpos[ia]);
            c2 = col_at(s_tpos[ib]);
          }
          for (int q = 0; q < 2; ++q) {
            const int cc = q ? c2 : c1;
            if (cc < 0) continue;
            for (int32_t k = a.col_ptr[cc]; k < a.col_ptr[cc + 1]; ++k) {
              const int pi = prow[a.csc_row[k]];
              if (pi >= 0)
                for (int w = 0; w < RW; ++w) acc[MW + w] ^= B[(int64_t)pi * W + MW + w];
            }
          }
          s_f1 = c1;
          s_f2 = c2;
        }
        __syncthreads();
      }
    }
    uint64_t pm[MAX_OW] = {0ull, 0ull, 0ull, 0ull};
    auto flip = [&](int col) {
      for (int w = 0; w < a.ow; ++w) pm[w] ^= a.obs_mask[(int64_t)w * a.n + col];
    };
    if (incomplete) {
      // BP's hard decision stands
      for (int v = tid; v < a.n; v += NT) {
        const bool e = L[v] < 0.0f;
        if (e) flip(v);
        if (a.ehat) a.ehat[shot * a.n + v] = e ? 1 : 0;
      }
    } else {
      if (a.ehat)
        for (int v = tid; v < a.n; v += NT) a.ehat[shot * a.n + v] = 0;
      __syncthreads();
      for (int i = tid; i < r; i += NT) {
        if ((acc[MW + (i >> 6)] >> (i & 63)) & 1ull) {
          const int col = kept[i];
          flip(col);
          if (a.ehat) a.ehat[shot * a.n + col] = 1;
        }
      }
      if constexpr (!WIN && !PFX) {
        // OSD-CS: the flipped columns outside the information set
        if (tid == 0)
          for (int q = 0; q < 2; ++q) {
            const int cc = q ? s_f2 : s_f1;
            if (cc < 0) continue;
            flip(cc);
            if (a.ehat) a.ehat[shot * a.n + cc] = 1;
          }
      }
    }
    for (int w = 0; w < a.ow; ++w) pm[w] = block_xor_u64(pm[w], &s_red);
    if (tid == 0) {
      for (int w = 0; w < a.ow; ++w) write_pred(a.pred, a.stride, a.nobs, shot, pm[w], w);
      if (a.flags) a.flags[shot] = (uint8_t)(2 | (not_in_span ? 4 : 0) | (incomplete ? 8 : 0));
      if (a.stats && not_in_span) atomicAdd((unsigned long long*)&a.stats->not_in_span, 1ull);
      if (a.stats && incomplete) atomicAdd((unsigned long long*)&a.stats->osd_incomplete, 1ull);
      if (a.stats && a.jobs) atomicAdd((unsigned long long*)&a.stats->osd_prefix_retry, 1ull);
    }
    reset_rows();
    __syncthreads();
  }
}

// The grid that is resident at once (at most `grid`): a workgroup keeps taking
// jobs until there are none, so one that has to wait for a place only starts its
// first job when the others are done.
int resident_grid(const void* kernel, int threads, size_t lds, int grid) {
  static std::mutex mu;
  static std::map<std::tuple<int, const void*, size_t>, int> known;
  int dev = 0;
  hipGetDevice(&dev);
  std::lock_guard<std::mutex> lock(mu);
  auto it = known.find({dev, kernel, lds});
  if (it == known.end()) {
    int cus = 0, per_cu = 0;
    hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, lds) != hipSuccess || per_cu < 1) {
      (void)hipGetLastError();
      per_cu = 1 << 10;
    }
    it = known.emplace(std::make_tuple(dev, kernel, lds), std::max(1, cus) * per_cu).first;
  }
  return std::max(1, std::min(grid, it->second));
}

template <int MW, int RW, int KPT, bool BL, bool PFX = false>
tmcs_status launch_osd(const OSDArgs& a, int grid, size_t lds, hipStream_t s) {
  constexpr int NT = BL ? 64 : OSD_THREADS;
  auto k = k_osd<MW, RW, KPT, BL, NT, false, PFX>;
  if (lds > 64 * 1024 && hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return fail(TMCS_EUNSUPPORTED, "OSD workspace does not fit in LDS");
  // the full-sort pass over jobs a prefix left open is timed on its own
  grid = resident_grid((const void*)k, NT, lds, grid);
  TMCS_LAUNCH(a.jobs ? "k_osd_retry" : "k_osd", k, dim3(grid), dim3(NT), lds, s, a, OSDMulti{nullptr, 0, nullptr});
  return hip_check(hipGetLastError(), "k_osd launch");
}

// prefix pass: PFX_KEYS_WAVE (one wave) or PFX_KEYS_WG (256 threads) keys, 4 per thread
template <int MW>
tmcs_status launch_osd_pfx(bool bl, const OSDArgs& a, int grid, size_t lds, hipStream_t s) {
  // (one wave: at most PFX_KEYS_WAVE - 1 pivots, so PFX_KEYS_WAVE / 64 words of combination part)
  return bl ? launch_osd<MW, PFX_KEYS_WAVE / 64, PFX_KEYS_WAVE / 64, true, true>(a, grid, lds, s)
            : launch_osd<MW, MW, PFX_KEYS_WG / OSD_THREADS, false, true>(a, grid, lds, s);
}

tmcs_status dispatch_osd_pfx(int mw, bool bl, const OSDArgs& a, int grid, size_t lds, hipStream_t s) {
  if (bl) {
    if (mw <= 1) return launch_osd_pfx<1>(true, a, grid, lds, s);
    if (mw <= 2) return launch_osd_pfx<2>(true, a, grid, lds, s);
    if (mw <= 4) return launch_osd_pfx<4>(true, a, grid, lds, s);
    if (mw <= 5) return launch_osd_pfx<5>(true, a, grid, lds, s);
    if (mw <= 8) return launch_osd_pfx<8>(true, a, grid, lds, s);
    return fail(TMCS_EUNSUPPORTED, "OSD basis in LDS: too many detectors");
  }
  if (mw <= 1) return launch_osd_pfx<1>(false, a, grid, lds, s);
  if (mw <= 2) return launch_osd_pfx<2>(false, a, grid, lds, s);
  if (mw <= 4) return launch_osd_pfx<4>(false, a, grid, lds, s);
  if (mw <= 5) return launch_osd_pfx<5>(false, a, grid, lds, s);
  if (mw <= 8) return launch_osd_pfx<8>(false, a, grid, lds, s);
  if (mw <= 12) return launch_osd_pfx<12>(false, a, grid, lds, s);
  if (mw <= 15) return launch_osd_pfx<15>(false, a, grid, lds, s);
  if (mw <= 18) return launch_osd_pfx<18>(false, a, grid, lds, s);
  if (mw <= 24) return launch_osd_pfx<24>(false, a, grid, lds, s);
  if (mw <= 32) return launch_osd_pfx<32>(false, a, grid, lds, s);
  return fail(TMCS_EUNSUPPORTED, "OSD supports at most 2048 detectors in this build");
}

template <int KPT, int NT>
tmcs_status launch_sort(const OSDArgs& a, int grid, hipStream_t s) {
  auto k = k_osd_sort<KPT, NT>;
  const size_t lds = (size_t)KPT * NT * 8;
  if (lds > 64 * 1024 && hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return fail(TMCS_EUNSUPPORTED, "OSD sort does not fit in LDS");
  grid = resident_grid((const void*)k, NT, lds, grid);
  TMCS_LAUNCH("k_osd_sort", k, dim3(grid), dim3(NT), lds, s, a.osd_llr, a.sorted, a.n, a.jobs, a.counters, a.cnt_total);
  return hip_check(hipGetLastError(), "k_osd_sort launch");
}

tmcs_status dispatch_sort(const OSDArgs& a, hipStream_t s) {
  const int grid = 1 << 14;                          // (cut to what is resident)
  switch (a.npad) {
    case 256: return launch_sort<1, 256>(a, grid, s);
    case 512: return launch_sort<2, 256>(a, grid, s);
    case 1024: return launch_sort<4, 256>(a, grid, s);
    case 2048: return launch_sort<2, 1024>(a, grid, s);
    case 4096: return launch_sort<4, 1024>(a, grid, s);
    case 8192: return launch_sort<8, 1024>(a, grid, s);
    case 16384: return launch_sort<16, 1024>(a, grid, s);
    default: return fail(TMCS_EUNSUPPORTED, "OSD sort size");
  }
}

// basis in LDS, one wave per shot: small DEMs only (m <= 512, sort length <= 4096)
template <int MW>
tmcs_status dispatch_kpt_lds(int kpt, const OSDArgs& a, int grid, size_t lds, hipStream_t s) {
  switch (kpt) {
    case 4: return launch_osd<MW, MW, 4, true>(a, grid, lds, s);
    case 8: return launch_osd<MW, MW, 8, true>(a, grid, lds, s);
    case 16: return launch_osd<MW, MW, 16, true>(a, grid, lds, s);
    case 32: return launch_osd<MW, MW, 32, true>(a, grid, lds, s);
    case 64: return launch_osd<MW, MW, 64, true>(a, grid, lds, s);
    default: return fail(TMCS_EUNSUPPORTED, "OSD sort size");
  }
}

bool osd_lds_basis_ok(int mw, int npad) { return mw <= 8 && npad <= 4096; }

// Windowed OSD-0 with 64 MW local rows.  A smaller window (WIN_SMALL_MW or
// WIN_MID_MW) runs first and hands the shots it cannot settle to a.retry; the full one
// (WIN_MW) decodes those (a.jobs = the retry list), timed as k_osd_retry.
template <int MW, bool MULTI>
tmcs_status launch_osd_win_t(const OSDArgs& a, const OSDMulti& mu, int grid, size_t lds, hipStream_t s) {
  auto k = k_osd<MW, MW, WIN_KEYS / OSD_THREADS, false, OSD_THREADS, true, false, MULTI>;
  if (lds > 64 * 1024 && hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return fail(TMCS_EUNSUPPORTED, "OSD workspace does not fit in LDS");
  grid = resident_grid((const void*)k, OSD_THREADS, lds, grid);
  TMCS_LAUNCH(a.jobs ? "k_osd_retry" : "k_osd", k, dim3(grid), dim3(OSD_THREADS), lds, s, a, mu);
  return hip_check(hipGetLastError(), "k_osd launch");
}

tmcs_status launch_osd_win(const OSDArgs& a, int grid, size_t lds, hipStream_t s, int mw) {
  const OSDMulti none{nullptr, 0, nullptr};
  if (mw == WIN_SMALL_MW) return launch_osd_win_t<WIN_SMALL_MW, false>(a, none, grid, lds, s);
  if (mw == WIN_MID_MW) return launch_osd_win_t<WIN_MID_MW, false>(a, none, grid, lds, s);
  if (mw == WIN_MW) return launch_osd_win_t<WIN_MW, false>(a, none, grid, lds, s);
  return fail(TMCS_EINVAL, "windowed OSD: unsupported window size");
}

tmcs_status launch_osd_win_multi(const OSDArgs& first, const OSDMulti& mu, int grid, size_t lds, hipStream_t s,
                                 int mw) {
  if (mu.n < 1 || mu.n > MAX_MULTI_OSD) return fail(TMCS_EINVAL, "multi-item OSD: 1..16 items");
  if (first.npad != WIN_KEYS) return fail(TMCS_EINVAL, "multi-item OSD: windowed items only");
  // the first item's arguments set the LDS layout, which every windowed item shares
  if (mw == WIN_SMALL_MW) return launch_osd_win_t<WIN_SMALL_MW, true>(first, mu, grid, lds, s);
  if (mw == WIN_MID_MW) return launch_osd_win_t<WIN_MID_MW, true>(first, mu, grid, lds, s);
  if (mw == WIN_MW) return launch_osd_win_t<WIN_MW, true>(first, mu, grid, lds, s);
  return fail(TMCS_EINVAL, "windowed OSD: unsupported window size");
}

tmcs_status dispatch_osd(int mw, int kpt, bool bl, const OSDArgs& a, int grid, size_t lds, hipStream_t s) {
  if (bl) {
    if (mw <= 1) return dispatch_kpt_lds<1>(kpt, a, grid, lds, s);
    if (mw <= 2) return dispatch_kpt_lds<2>(kpt, a, grid, lds, s);
    if (mw <= 4) return dispatch_kpt_lds<4>(kpt, a, grid, lds, s);
    if (mw <= 5) return dispatch_kpt_lds<5>(kpt, a, grid, lds, s);
    if (mw <= 8) return dispatch_kpt_lds<8>(kpt, a, grid, lds, s);
    return fail(TMCS_EUNSUPPORTED, "OSD basis in LDS: too many detectors");
  }
  const tmcs_status st = dispatch_sort(a, s);
  if (st != TMCS_OK) return st;
  if (mw <= 1) return launch_osd<1, 1, 1, false>(a, grid, lds, s);
  if (mw <= 2) return launch_osd<2, 2, 1, false>(a, grid, lds, s);
  if (mw <= 4) return launch_osd<4, 4, 1, false>(a, grid, lds, s);
  if (mw <= 5) return launch_osd<5, 5, 1, false>(a, grid, lds, s);
  if (mw <= 8) return launch_osd<8, 8, 1, false>(a, grid, lds, s);
  if (mw <= 12) return launch_osd<12, 12, 1, false>(a, grid, lds, s);
  if (mw <= 15) return launch_osd<15, 15, 1, false>(a, grid, lds, s);
  if (mw <= 18) return launch_osd<18, 18, 1, false>(a, grid, lds, s);
  if (mw <= 24) return launch_osd<24, 24, 1, false>(a, grid, lds, s);
  if (mw <= 32) return launch_osd<32, 32, 1, false>(a, grid, lds, s);
  return fail(TMCS_EUNSUPPORTED, "OSD supports at most 2048 detectors in this build");
}

}  // namespace dec
}  // namespace tmcs

// Min-sum BP for large graph-like DEMs (surface codes): one pass over the checks
// per iteration, a shot's state streamed through a ring of tiles in LDS.
//
// What bounds it: VALU issue (about 21 instructions per edge step, all of it: no
// column pass; 26 per edge and iteration counted, which fill 75 % of the issue slots
// over the launch of d = 11 to 29 at two p).  Nearly every mechanism of a surface
// code touches two detectors, and they are near each other in detector order (time,
// then place).  So a check's lane can rebuild L_v of an edge from its own state and
// that of the one other check c' of the column, L_v = lambda_v + the two messages
// in ascending check order, and never needs an L array: state is 12 bytes per check,
// read and written once per iteration in whole lines.
//
// Checks are cut, in detector order, into tiles of P (one check per lane), each
// tile sorted so that the 64 checks of a wave (a chunk) have the same number of
// edges of each kind.  While tile i is computed, tiles i - h .. i + h are in the
// LDS ring (h: the most tiles between the two checks of an inline column), tile
// i + h + 1 is on its way from device memory, and the new state of tile i goes to
// the other of the team's two state buffers.  Records name the neighbour by its
// fixed ring address.  One barrier per tile.
//
// A chunk's steps, the same in its 64 lanes:
//   K0 inline edges whose own check is the column's first: L = (lambda + own) + other,
//   K1 inline edges whose own check is the second:         L = (lambda + other) + own,
//   KL edges of the other columns (three or more checks, checks too far apart, or
//      a lambda beyond the table), whose L_v a short pass computed before the tiles.
// A column of one check is inline with c' = a part whose messages are -0.  No-op
// edges read lambda (or L) = +inf, which changes nothing.
// Record of an inline step: ring place * 4 << 16 | lambda index * 4 << 8 |
// position of the edge in c'; of another step: place of its L * 4 << 16.
//
// Measured against the two-pass kernel with its state in device memory (k_bp_dev,
// which reads 16 bytes of check state and 4 of L per edge at scattered places),
// ms: 4096 shots of the d = 21 non-local CNOT at p = 1e-3 42.6 -> 13.3, d = 15 at
// p = 1e-4 and 1e-3 in one launch 13.8 -> 4.5.  The vector instructions of a
// d = 21 iteration (21 per step, chunks padded to 84,000) are 40 us of a CU's
// issue slots at 2.2 GHz; an iteration takes 45.
//
// State as in bp_team.h; position j is the step at which the edge comes.  Every
// sum has the definition's order and nothing is contracted, so results are
// bit-identical to it.  Signs are taken from the sign bit and the second minimum
// is the median of (n1, n2, |q|): without infinities L and q are never -0 or NaN
// (the launcher's caller bounds the magnitudes).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <type_traits>
#include <vector>

#include "../host/device.h"
#include "../host/timing.h"
#include "bp_stream.h"
#include "bp_team.h"

namespace tmcs {
namespace dec {

namespace {

constexpr int PAD_ROWS = 4;                 // rows of records read past the end
using ArgsPtr = const TMCS_CONST_AS StreamArgs*;

typedef float v3f __attribute__((ext_vector_type(3)));
struct Part {
  float n1, n2;
  uint32_t w;
};
__device__ __forceinline__ Part ld_part(const unsigned char* base, uint32_t byte) {
  typedef v3f v3f_a4 __attribute__((aligned(4)));
  const v3f x = *(const TMCS_GLOBAL_AS v3f_a4*)(base + byte);
  return Part{x.x, x.y, __float_as_uint(x.z)};
}
__device__ __forceinline__ void st_part(unsigned char* base, uint32_t byte, const Part& s) {
  typedef v3f v3f_a4 __attribute__((aligned(4)));
  v3f x;
  x.x = s.n1;
  x.y = s.n2;
  x.z = __uint_as_float(s.w);
  *(TMCS_GLOBAL_AS v3f_a4*)(base + byte) = x;
}
// message of edge `jr & 31` of a check
__device__ __forceinline__ float message(const Part& s, uint32_t jr) {
  return with_sign(((s.w ^ jr) & W_POS) == 0u ? s.n2 : s.n1, s.w << (jr & 31u));
}

// Dynamic LDS.  The ring first, as three planes of CAP words (n1, n2, word), so
// that a record's 16-bit byte address reaches all three with offsets that are
// part of the instruction; the rest at fixed places after it.
struct Shared {
  int job, flag, pos, inst;
  int unsat[2];
  int pref[MAX_MULTI + 1];
  uint32_t hist[TMCS_BP_HIST_BINS];                // (thread 0)
  unsigned long long pm[MAX_OW];
  unsigned long long cnt[4];                       // nontrivial, converged, osd, iterations (thread 0)
};
static_assert(sizeof(Shared) <= STREAM_LDS_SHARED, "LDS layout");

template <int CAP, bool MULTI>
__global__ void __launch_bounds__(1024, 8) k_bp_stream(StreamArgs, StreamMulti mu) {
  extern __shared__ __align__(16) unsigned char sm[];
  constexpr uint32_t PLANE = CAP * 4, LAM = 3 * PLANE, SHARED = LAM + STREAM_LAMS * 4, LCOL = SHARED + STREAM_LDS_SHARED;
  Shared& sh = *(Shared*)(sm + SHARED);
  const int tid = threadIdx.x, P = blockDim.x, NW = P >> 6;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  ArgsPtr a = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  unsigned char* buf0 = nullptr;                   // the team's two state buffers, [NT P + 1] parts (the last: messages of -0)
  uint32_t bufsz = 0;
  auto ring_part = [&](uint32_t byte) -> Part {
    const unsigned char* p = sm + byte;
    return Part{*(const float*)p, *(const float*)(p + PLANE), *(const uint32_t*)(p + 2 * PLANE)};
  };
  auto ring_put = [&](uint32_t byte, const Part& s) {
    unsigned char* p = sm + byte;
    *(float*)p = s.n1;
    *(float*)(p + PLANE) = s.n2;
    *(uint32_t*)(p + 2 * PLANE) = s.w;
  };
  auto bind = [&]() {
    const uint32_t NS = (uint32_t)(a->NT * P);
    bufsz = (uint32_t)a->buf;
    buf0 = a->state + (int64_t)blockIdx.x * 2 * bufsz;
    for (int i = tid; i < STREAM_LAMS; i += P) *(float*)(sm + LAM + i * 4) = gload(a->lamtab + i);
    if (tid == 0) {
      ring_put((CAP - 1) * 4, Part{0.0f, 0.0f, W_SIGNS | W_POS});
      *(float*)(sm + LCOL + (uint32_t)a->NL * 4) = __builtin_inff();
    }
    if (tid < 2) st_part(buf0, (uint32_t)tid * bufsz + NS * 12, Part{0.0f, 0.0f, W_SIGNS | W_POS});
    __syncthreads();
  };
  int32_t total = 0;                               // MULTI: thread 0's
  int cur = -1;                                    // MULTI: item the team works on
  if constexpr (!MULTI) {
    total = a->queue ? a->counters[0] : (int32_t)a->nshots;
    if ((int)blockIdx.x >= total) return;
    bind();
  } else if (tid == 0) {
    sh.pref[0] = 0;
    for (int i = 0; i < mu.n; ++i)
      sh.pref[i + 1] = sh.pref[i] + (mu.tab[i].queue ? mu.tab[i].counters[0] : (int32_t)mu.tab[i].nshots);
    total = sh.pref[mu.n];
  }
  for (int i = tid; i < TMCS_BP_HIST_BINS; i += P) sh.hist[i] = 0u;
  if (tid < 4) sh.cnt[tid] = 0ull;
  auto flush = [&]() {
    __syncthreads();
    // (as many copies of the statistics as spare the teams waiting on each other's adds)
    tmcs_decode_stats* stats = reread(a)->stats;
    if (stats) {
      stats += blockIdx.x % STAT_SHARDS;
      for (int i = tid; i < TMCS_BP_HIST_BINS; i += P)
        if (sh.hist[i]) atomicAdd((unsigned long long*)&stats->bp_iter_hist[i], (unsigned long long)sh.hist[i]);
      if (tid == 0) {
        if (sh.cnt[0]) atomicAdd((unsigned long long*)&stats->nontrivial, sh.cnt[0]);
        if (sh.cnt[1]) atomicAdd((unsigned long long*)&stats->converged, sh.cnt[1]);
        if (sh.cnt[2]) atomicAdd((unsigned long long*)&stats->osd, sh.cnt[2]);
        if (sh.cnt[3]) atomicAdd((unsigned long long*)&stats->bp_iters, sh.cnt[3]);
      }
    }
    __syncthreads();
    for (int i = tid; i < TMCS_BP_HIST_BINS; i += P) sh.hist[i] = 0u;
    if (tid < 4) sh.cnt[tid] = 0ull;
    __syncthreads();
  };
  // a team's first job is its own number, the others come from a counter, one at
  // a time (a shot takes far longer than an atomic)
  int ticket = (int)blockIdx.x;
  while (true) {
    if (tid == 0) {
      if constexpr (MULTI) {
        int i = 0;
        while (i < mu.n && ticket >= sh.pref[i + 1]) ++i;
        sh.inst = i;
        sh.job = i < mu.n ? ticket - sh.pref[i] : 0;
      } else {
        sh.job = ticket;
      }
      sh.flag = 0;
      sh.unsat[0] = 0;
      sh.unsat[1] = 0;
      for (int w = 0; w < MAX_OW; ++w) sh.pm[w] = 0ull;
    }
    __syncthreads();
    if constexpr (MULTI) {
      const int inst = __builtin_amdgcn_readfirstlane(sh.inst);
      if (inst != cur) {                           // uniform: the team moves to the next item
        if (cur >= 0) flush();
        if (inst >= mu.n) break;
        cur = inst;
        a = (ArgsPtr)(uintptr_t)(mu.tab + inst);
        bind();
      }
    }
    const int job = __builtin_amdgcn_readfirstlane(sh.job);
    if (!MULTI && job >= total) break;
    const int T = a->T, NT = a->NT;
    const float alpha = a->alpha;
    int ls = job;                                  // shot of the pass
    // state of iteration 1 into the first buffer
    {
      const ArgsPtr c = reread(a);
      if (c->queue) ls = __builtin_amdgcn_readfirstlane(gload(c->queue + job));
      const int mw = c->mw;
      const uint64_t* sy = c->synd + (int64_t)ls * mw;
      int fl = 0;
#pragma unroll 2
      for (int i = 0; i < NT; ++i) {
        const int slot = i * P + tid;
        const int4 s0 = gload(c->pinit + slot);
        const int sb = s0.w < 0 ? 0 : (int)((gload(sy + (s0.w >> 6)) >> (s0.w & 63)) & 1ull);
        fl |= sb;
        st_part(buf0, (uint32_t)slot * 12, Part{__fmul_rn(alpha, __int_as_float(s0.x)), __fmul_rn(alpha, __int_as_float(s0.y)),
                                                (uint32_t)s0.z ^ (sb ? (W_SIGNS | W_SC) : 0u)});
      }
      // a detection event on a check without edges: never satisfied
      if (c->lone)
        for (int w = tid; w < mw; w += P)
          if (gload(sy + w) & gload(c->lone + w)) fl |= 3;
      if (fl) atomicOr(&sh.flag, fl);
    }
    if (tid == 0) ticket = total > (int)gridDim.x ? (int)gridDim.x + atomicAdd(MULTI ? mu.next : &a->counters[1], 1) : total;
    __syncthreads();
    const int f0 = __builtin_amdgcn_readfirstlane(sh.flag);
    int itr = 0;
    bool conv = true;
    unsigned char* st = buf0;                      // state of iteration t
    if (f0 & 1) {
      conv = false;
      unsigned char* nst = buf0 + bufsz;           // state of iteration t + 1
      for (int t = 1;; ++t) {
        const int h = a->h, R = a->R;
        // L^t of the columns that are not inline
        {
          const int NL = a->NL, K = a->KL;
          const uint32_t* const lrec = a->lrec;
          for (int i = tid; i < NL; i += P) {
            float acc = gload(a->lamL + i);
#pragma unroll 4
            for (int k = 0; k < K; ++k) {
              const uint32_t r = gload(lrec + (size_t)k * NL + i);
              acc = __fadd_rn(acc, message(ld_part(st, (r >> 5) * 12), r));
            }
            *(float*)(sm + LCOL + (uint32_t)i * 4) = acc;
          }
        }
        // the first tiles into the ring
        {
          const int first = min(h + 1, NT);
          for (int i = 0; i < first; ++i) ring_put((uint32_t)(i * P + tid) * 4, ld_part(st, (uint32_t)(i * P + tid) * 12));
        }
        __syncthreads();
        int unsat = (f0 >> 1) & 1;
        auto sweep = [&](auto UPD) {
          constexpr bool update = decltype(UPD)::value;
          const uint32_t* rp = a->rec + (size_t)(((const TMCS_CONST_AS int32_t*)(uintptr_t)a->row0)[wave]) * 64;
          const TMCS_CONST_AS int32_t* const desc = (const TMCS_CONST_AS int32_t*)(uintptr_t)a->desc;
          const uint32_t lane4 = (uint32_t)lane * 4;
          uint32_t r0 = at_byte(rp, lane4), r1 = at_byte(rp + 64, lane4);   // records are read two steps ahead
          const uint32_t tile4 = (uint32_t)P * 4, ring4 = (uint32_t)(R * P) * 4;
          uint32_t own = 0u, put = (uint32_t)(h + 1) * tile4;   // ring places of tiles i and i + h + 1
          uint32_t out = (uint32_t)tid * 12, fetch = (uint32_t)((h + 1) * P + tid) * 12;   // their places in the buffers
          int dk = desc[wave];
          for (int i = 0; i < NT; ++i) {
            const int dnext = desc[(i + 1) * NW + wave];
            const bool more = i + h + 1 < NT;
            Part in{0.0f, 0.0f, 0u};
            if (more) in = ld_part(st, fetch);
            const Part o = ring_part(own + (uint32_t)tid * 4);
            const uint32_t ago = o.w & W_POS;
            float n1 = BP_BIG, n2 = BP_BIG;
            uint32_t lt = 0u, nb = 0u, hx = 0u;     // lt: steps that brought a new minimum, the last in bit 0
            const int K0 = dk & 255, K01 = K0 + ((dk >> 8) & 255), K = K01 + ((dk >> 16) & 255);
            auto own_msg = [&](int j) -> float { return with_sign(ago == (uint32_t)j ? o.n2 : o.n1, o.w << j); };
            auto take = [&](float Lv, float mo) {
              hx ^= __float_as_uint(Lv);
              if constexpr (update) {
                const float qv = __fsub_rn(Lv, mo);
                const float aq = fabsf(qv);
                // (a difference of floats is negative exactly when the first is smaller)
                lt = __builtin_amdgcn_alignbit(lt, __float_as_uint(__fsub_rn(aq, n1)), 31);
                n2 = __builtin_amdgcn_fmed3f(n1, n2, aq);
                n1 = __builtin_amdgcn_fmed3f(n1, aq, -__builtin_inff());   // (min, without a canonicalising move)
                nb = __builtin_amdgcn_alignbit(nb, __float_as_uint(qv), 31);
              }
            };
            // steps j .. end - 1, two at a time: a record's register is refilled after use
            int j = 0;
            auto run = [&](int end, auto&& step) {
              for (; j + 1 < end; j += 2) {
                step(j, r0);
                r0 = at_byte(rp + 128, lane4);
                step(j + 1, r1);
                r1 = at_byte(rp + 192, lane4);
                rp += 128;
              }
              if (j < end) {
                step(j, r0);
                r0 = r1;
                r1 = at_byte(rp + 128, lane4);
                rp += 64;
                ++j;
              }
            };
            auto lam_of = [&](uint32_t r) -> float { return *(const float*)(sm + LAM + ((r >> 8) & 0xFFu)); };
            run(K0, [&](int j, uint32_t r) {
              const float lam = lam_of(r), mt = message(ring_part(r >> 16), r), mo = own_msg(j);
              take(__fadd_rn(__fadd_rn(lam, mo), mt), mo);
            });
            run(K01, [&](int j, uint32_t r) {
              const float lam = lam_of(r), mt = message(ring_part(r >> 16), r), mo = own_msg(j);
              take(__fadd_rn(__fadd_rn(lam, mt), mo), mo);
            });
            run(K, [&](int j, uint32_t r) { take(*(const float*)(sm + LCOL + (r >> 16)), own_msg(j)); });
            const uint32_t sc = o.w & W_SC;
            unsat |= (int)((hx >> 31) ^ (sc >> 5));
            if constexpr (update) {
              nb = K > 0 ? nb << (32 - K) : 0u;
              const uint32_t ag = lt ? (uint32_t)(K - __ffs(lt)) : W_POS;
              // message sign of edge j = s_c + parity + sgn q_j (mod 2)
              const uint32_t flip = ((uint32_t)__popc(nb) & 1u) != (sc >> 5) ? W_SIGNS : 0u;
              st_part(nst, out, Part{__fmul_rn(alpha, n1), __fmul_rn(alpha, n2), ((nb ^ flip) & W_SIGNS) | sc | ag});
            }
            if (more) ring_put(put + (uint32_t)tid * 4, in);
            own = own + tile4 == ring4 ? 0u : own + tile4;
            put = put + tile4 == ring4 ? 0u : put + tile4;
            out += (uint32_t)P * 12;
            fetch += (uint32_t)P * 12;
            dk = dnext;
            if (i + 1 < NT) __syncthreads();
          }
        };
        if (t < T) sweep(std::true_type{});
        else sweep(std::false_type{});
        if (__ballot(unsat != 0) != 0ull && lane == 0) sh.unsat[t & 1] = 1;   // (every writer stores 1)
        if (tid == 0) sh.unsat[(t + 1) & 1] = 0;            // read by every lane before the last barriers
        __syncthreads();
        if (!__builtin_amdgcn_readfirstlane(sh.unsat[t & 1])) { itr = t; conv = true; break; }
        if (t >= T) { itr = T; break; }
        unsigned char* const x = st;
        st = nst;
        nst = x;
      }
    }
    // finalise: prediction from the hard decision, or hand the posteriors to OSD;
    // L is rebuilt from the state of the last iteration (still in its buffer)
    const ArgsPtr c = reread(a);
    if (tid == 0) sh.pos = (!conv && c->use_osd) ? atomicAdd(&c->counters[2], 1) : -1;
    __syncthreads();
    const int pos = __builtin_amdgcn_readfirstlane(sh.pos);
    const int64_t shot = c->shot0 + ls;
    const int n = c->n;
    auto llr_at = [&](int v) -> float {
      const float lam = gload(c->lam + v);
      if (!(f0 & 1)) return lam;                   // (no BP run: the priors)
      const int2 r = gload((const int2*)c->vrec + v);
      if (r.x == -1) return *(const float*)(sm + LCOL + (uint32_t)r.y * 4);
      const Part s0 = ld_part(st, ((uint32_t)r.x >> 5) * 12), s1 = ld_part(st, ((uint32_t)r.y >> 5) * 12);
      return __fadd_rn(__fadd_rn(lam, message(s0, (uint32_t)r.x)), message(s1, (uint32_t)r.y));
    };
    if (pos >= 0 || c->llr || c->ehat) {
#pragma unroll 2
      for (int v = tid; v < n; v += P) {
        const float Lv = llr_at(v);
        if (pos >= 0) c->osd_llr[(int64_t)pos * n + v] = Lv;
        if (c->llr) c->llr[shot * n + v] = Lv;
        if (c->ehat && pos < 0) c->ehat[shot * n + v] = Lv < 0.0f ? 1 : 0;
      }
    }
    if (pos < 0 && (f0 & 1)) {
      for (int i = tid; i < c->noc; i += P)
        if (llr_at(gload(c->ocol + i)) < 0.0f)
          for (int w = 0; w < c->ow; ++w) {
            const uint64_t m = gload(c->omask + (int64_t)w * c->noc + i);
            if (m) atomicXor(&sh.pm[w], (unsigned long long)m);
          }
    }
    __syncthreads();
    if (tid == 0) {
      if (pos < 0)
        for (int w = 0; w < c->ow; ++w)
          write_pred(c->pred, c->stride, c->nobs, shot, (f0 & 1) ? sh.pm[w] ^ c->pm_iso[w] : c->pm_lam[w], w);
      else c->osd_queue[pos] = ls;
      if (c->iters) c->iters[shot] = itr;
      if (c->flags) c->flags[shot] = (uint8_t)((conv ? 1 : 0) | (pos >= 0 ? 2 : 0));
      sh.cnt[0] += (itr > 0 || !conv) ? 1 : 0;
      sh.cnt[1] += conv ? 1 : 0;
      sh.cnt[2] += pos >= 0 ? 1 : 0;
      sh.cnt[3] += (unsigned long long)itr;
      sh.hist[itr < TMCS_BP_HIST_BINS - 1 ? itr : TMCS_BP_HIST_BINS - 1] += 1u;
    }
  }
  if constexpr (!MULTI) flush();
}

}  // namespace

// ------------------------------------------------------------------ host
tmcs_status build_stream_sched(const Dem& D, int P, StreamSched* out) {
  const tmcs_status no = TMCS_EUNSUPPORTED;   // (not an error of the call: no message)
  StreamSched s;
  s.P = P;
  const int NW = P / 64;
  s.NT = (D.rows + P - 1) / P;
  if (D.rows == 0 || (int64_t)s.NT * P >= (1 << 26)) return no;
  auto deg = [&](int v) { return D.col_ptr[v + 1] - D.col_ptr[v]; };
  // lambda values of the inline columns, the most frequent ones in the table
  std::vector<float> lam(D.cols), lamtab;
  std::vector<int32_t> lam_idx(std::max(D.cols, 1), 0);
  {
    std::map<float, std::pair<int64_t, int>> found;          // value: columns, table index
    for (int v = 0; v < D.cols; ++v) {
      lam[v] = (float)std::log((1.0 - D.priors[v]) / D.priors[v]);
      if (deg(v) > 0) ++found[lam[v]].first;
    }
    std::vector<std::pair<int64_t, float>> order;
    for (auto& f : found) order.push_back({-f.second.first, f.first});
    std::sort(order.begin(), order.end());
    for (auto& f : found) f.second.second = -1;
    for (size_t i = 0; i < order.size() && i + 1 < (size_t)STREAM_LAMS; ++i) {
      found[order[i].second].second = (int)i;
      lamtab.push_back(order[i].second);
    }
    for (int v = 0; v < D.cols; ++v) lam_idx[v] = deg(v) > 0 ? found[lam[v]].second : -1;
  }
  // tiles between the two checks of a column; columns beyond the ring go through memory
  auto span = [&](int v) { return D.row_idx[D.col_ptr[v + 1] - 1] / P - D.row_idx[D.col_ptr[v]] / P; };
  for (int v = 0; v < D.cols; ++v)
    if (deg(v) == 2) s.h = std::max(s.h, (int32_t)span(v));
  s.h = std::max(1, s.h);
  if (s.h > 1 && (2 * s.h + 2) * P >= STREAM_CAP_MAX) s.h = std::max(1, ((STREAM_CAP_MAX - 1) / P - 2) / 2);
  s.R = 2 * s.h + 2;
  // (the last place of a plane holds the part whose messages are -0)
  s.cap = s.R * P < STREAM_CAP_MIN ? STREAM_CAP_MIN : STREAM_CAP_MAX;
  if (s.R * P >= s.cap) return no;
  std::vector<int32_t> lplace(std::max(D.cols, 1), -1);
  for (int v = 0; v < D.cols; ++v)
    if (deg(v) > 2 || (deg(v) == 2 && span(v) > s.h) || (deg(v) > 0 && lam_idx[v] < 0)) {
      lplace[v] = s.NL++;
      s.KL = std::max(s.KL, (int32_t)deg(v));
    }
  // every LDS address of a record has 16 bits
  if (s.NL >= 16384) return no;
  lamtab.resize(STREAM_LAMS, INFINITY);
  // edges of every check by kind
  std::vector<std::vector<int32_t>> kind[3];
  for (auto& k : kind) k.resize(D.rows);
  for (int c = 0; c < D.rows; ++c)
    for (int32_t e = D.row_ptr[c]; e < D.row_ptr[c + 1]; ++e) {
      const int v = D.col_idx[e];
      const int k = lplace[v] >= 0 ? 2 : D.row_idx[D.col_ptr[v]] == c ? 0 : 1;
      kind[k][c].push_back(e);
    }
  // tiles in detector order, each sorted by its checks' numbers of edges of each kind
  std::vector<int32_t> check((size_t)s.NT * P, -1), slot_of(D.rows);
  for (int i = 0; i < s.NT; ++i) {
    std::vector<int> items;
    for (int c = i * P; c < std::min(D.rows, (i + 1) * P); ++c) items.push_back(c);
    auto key = [&](int c) {
      const int a = (int)kind[0][c].size(), b = (int)kind[1][c].size(), l = (int)kind[2][c].size();
      return ((l * 2 + (a > b)) * 64 + std::min(a, b)) * 128 + a + b;
    };
    std::stable_sort(items.begin(), items.end(), [&](int x, int y) { return key(x) < key(y); });
    for (size_t j = 0; j < items.size(); ++j) {
      check[(size_t)i * P + j] = items[j];
      slot_of[items[j]] = (int32_t)((size_t)i * P + j);
    }
  }
  std::vector<int32_t> desc((size_t)(s.NT + 1) * NW, 0), pos(std::max<int64_t>(D.edges, 1), 0), row0(NW, 0);
  for (int i = 0; i < s.NT; ++i)
    for (int w = 0; w < NW; ++w) {
      size_t K[3] = {0, 0, 0};
      for (int j = 0; j < 64; ++j) {
        const int c = check[(size_t)i * P + w * 64 + j];
        for (int k = 0; c >= 0 && k < 3; ++k) K[k] = std::max(K[k], kind[k][c].size());
      }
      if (K[0] + K[1] + K[2] > (size_t)PART_MAX_DEG) return no;
      desc[(size_t)i * NW + w] = (int32_t)(K[0] | K[1] << 8 | K[2] << 16);
      for (int j = 0; j < 64; ++j) {
        const int c = check[(size_t)i * P + w * 64 + j];
        if (c < 0) continue;
        size_t base = 0;
        for (int k = 0; k < 3; base += K[k], ++k)
          for (size_t x = 0; x < kind[k][c].size(); ++x) pos[kind[k][c][x]] = (int32_t)(base + x);
      }
    }
  // records: wave after wave, tile after tile
  const uint32_t PAD_IN = (uint32_t)(STREAM_LAMS - 1) * 4 << 8, PAD_L = (uint32_t)s.NL * 4 << 16, NONE = (uint32_t)(s.cap - 1) * 4;
  std::vector<uint32_t> rec;
  for (int w = 0; w < NW; ++w) {
    row0[w] = (int32_t)(rec.size() / 64);
    for (int i = 0; i < s.NT; ++i) {
      const int32_t dk = desc[(size_t)i * NW + w];
      for (int k = 0; k < 3; ++k)
        for (int x = 0; x < ((dk >> (8 * k)) & 255); ++x)
          for (int j = 0; j < 64; ++j) {
            const int c = check[(size_t)i * P + w * 64 + j];
            // (no-op edge: a neighbour inside the ring, here the lane's own check, and lambda = +inf)
            uint32_t r = k < 2 ? PAD_IN | (uint32_t)((i % s.R) * P + w * 64 + j) * 4 << 16 : PAD_L;
            if (c >= 0 && x < (int)kind[k][c].size()) {
              const int32_t e = kind[k][c][x];
              const int v = D.col_idx[e];
              if (k == 2) {
                r = (uint32_t)lplace[v] * 4 << 16;
              } else {
                uint32_t addr = NONE, p = 0;       // degree 1: messages of -0
                if (deg(v) == 2) {
                  const int32_t q = D.row_idx[D.col_ptr[v]] == c ? D.col_ptr[v] + 1 : D.col_ptr[v];
                  const int32_t sl = slot_of[D.row_idx[q]];
                  addr = (uint32_t)((sl / P % s.R) * P + sl % P) * 4;
                  p = (uint32_t)pos[D.csc_edge[q]];
                }
                r = addr << 16 | (uint32_t)lam_idx[v] * 4 << 8 | p;
              }
            }
            rec.push_back(r);
          }
    }
  }
  rec.resize(rec.size() + (size_t)PAD_ROWS * 64, 0u);
  // iteration 1 (q = lambda) by slot
  std::vector<int4> pinit((size_t)s.NT * P);
  for (size_t i = 0; i < pinit.size(); ++i) {
    const int c = check[i];
    float n1 = BP_BIG, n2 = BP_BIG;
    uint32_t word = W_POS;
    if (c >= 0) {
      int par = 0;
      for (int32_t e = D.row_ptr[c]; e < D.row_ptr[c + 1]; ++e) {
        const float q = lam[D.col_idx[e]], aq = std::fabs(q);
        if (aq < n1) { n2 = n1; n1 = aq; word = (uint32_t)pos[e]; }
        else if (aq < n2) { n2 = aq; }
        par ^= q < 0.0f ? 1 : 0;
      }
      for (int32_t e = D.row_ptr[c]; e < D.row_ptr[c + 1]; ++e)
        word |= (uint32_t)(par ^ (lam[D.col_idx[e]] < 0.0f ? 1 : 0)) << (31 - pos[e]);
    }
    pinit[i] = make_int4(0, 0, (int32_t)word, c);
    std::memcpy(&pinit[i].x, &n1, 4);
    std::memcpy(&pinit[i].y, &n2, 4);
  }
  // a column's messages: slot << 5 | position; the slot past the last has messages of -0
  const uint32_t NOMSG = (uint32_t)(s.NT * P) << 5;
  auto msg = [&](int32_t q) { return (uint32_t)slot_of[D.row_idx[q]] << 5 | (uint32_t)pos[D.csc_edge[q]]; };
  std::vector<uint32_t> lrec((size_t)s.KL * s.NL, NOMSG);
  std::vector<float> lamL(s.NL);
  std::vector<uint2> vrec(std::max(D.cols, 1), make_uint2(NOMSG, NOMSG));
  for (int v = 0; v < D.cols; ++v) {
    const int32_t q = D.col_ptr[v];
    if (lplace[v] >= 0) {
      lamL[lplace[v]] = lam[v];
      for (int k = 0; k < deg(v); ++k) lrec[(size_t)k * s.NL + lplace[v]] = msg(q + k);
      vrec[v] = make_uint2(~0u, (uint32_t)lplace[v]);
    } else {
      if (deg(v) > 0) vrec[v].x = msg(q);
      if (deg(v) > 1) vrec[v].y = msg(q + 1);
    }
  }
  // columns that flip an observable (those without edges are counted apart)
  std::vector<int32_t> ocol;
  for (int v = 0; v < D.cols; ++v) {
    bool any = false;
    for (int w = 0; w < D.obs_words; ++w) any = any || D.obs_mask[(size_t)v * D.obs_words + w];
    if (any && deg(v) > 0) ocol.push_back(v);
  }
  s.noc = (int32_t)ocol.size();
  std::vector<uint64_t> omask((size_t)D.obs_words * ocol.size());
  for (size_t i = 0; i < ocol.size(); ++i)
    for (int w = 0; w < D.obs_words; ++w) omask[(size_t)w * ocol.size() + i] = D.obs_mask[(size_t)ocol[i] * D.obs_words + w];
  Uploader up("BP schedule");
  tmcs_status st;
  if ((st = up(&s.rec, rec)) != TMCS_OK || (st = up(&s.desc, desc)) != TMCS_OK ||
      (st = up(&s.row0, row0)) != TMCS_OK || (st = up(&s.pinit, pinit)) != TMCS_OK ||
      (st = up(&s.lamtab, lamtab)) != TMCS_OK || (st = up(&s.lrec, lrec)) != TMCS_OK ||
      (st = up(&s.lamL, lamL)) != TMCS_OK || (st = up(&s.vrec, vrec)) != TMCS_OK ||
      (st = up(&s.ocol, ocol)) != TMCS_OK || (st = up(&s.omask, omask)) != TMCS_OK) {
    free_stream_sched(&s);
    return st;
  }
  *out = s;
  return TMCS_OK;
}

void free_stream_sched(StreamSched* s) {
  (void)hipFree(s->rec); (void)hipFree(s->desc); (void)hipFree(s->row0); (void)hipFree(s->pinit); (void)hipFree(s->lamtab);
  (void)hipFree(s->lrec); (void)hipFree(s->lamL); (void)hipFree(s->vrec); (void)hipFree(s->ocol); (void)hipFree(s->omask);
  *s = StreamSched();
}

namespace {
template <int CAP, bool MULTI>
tmcs_status launch(const StreamArgs& a, const StreamMulti& mu, int grid, int P, size_t lds, hipStream_t stream) {
  auto k = k_bp_stream<CAP, MULTI>;
  if (lds > 64 * 1024 && hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return fail(TMCS_EUNSUPPORTED, "BP ring does not fit in LDS");
  TMCS_LAUNCH("k_bp_stream", k, dim3((unsigned)grid), dim3((unsigned)P), lds, stream, a, mu);
  return hip_check(hipGetLastError(), "k_bp_stream launch");
}
}  // namespace

tmcs_status launch_bp_stream(const StreamArgs& a, const StreamMulti& mu, int cap, int grid, int P, size_t lds,
                             hipStream_t stream) {
  if (P < 64 || P > 1024 || P % 64 || grid < 1) return fail(TMCS_EINVAL, "BP launch shape");
  if (cap == STREAM_CAP_MIN)
    return mu.n > 0 ? launch<STREAM_CAP_MIN, true>(a, mu, grid, P, lds, stream)
                    : launch<STREAM_CAP_MIN, false>(a, mu, grid, P, lds, stream);
  return mu.n > 0 ? launch<STREAM_CAP_MAX, true>(a, mu, grid, P, lds, stream)
                  : launch<STREAM_CAP_MAX, false>(a, mu, grid, P, lds, stream);
}

}  // namespace dec
}  // namespace tmcs

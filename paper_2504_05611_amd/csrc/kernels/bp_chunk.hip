// Min-sum BP with a shot's whole state in LDS: one workgroup (a team of P lanes)
// decodes one shot at a time, two passes per iteration.
//
// What bounds it: VALU issue, with LDS close behind (a random 4- or 12-byte read
// per edge and pass).  So the layout is chosen to leave as few instructions per
// edge as possible: everything that only steers a loop is the same in the 64
// lanes of a wave and lives in scalar registers.
//
// Checks are cut into parts of at most PART_MAX_DEG edges, f = 1, 2, 4, ... equal
// parts to a check, in f neighbouring lanes.  64 parts with the same f and nearly
// the same number of edges form a chunk, one part per lane; 64 columns of nearly
// the same degree form a column chunk.  A chunk takes as many steps as its largest
// part or column; the others get no-op edges there.  Chunks go to the waves of
// the team by longest processing time, and a wave walks its chunks as a few runs
// (chunks of one width), whose lengths it reads from a table in LDS.
//
// State: per part {n1, n2, word}, 12 bytes.  n1, n2: the two smallest |q| of the
// whole check, already times alpha (times 1 with per-edge weights).  word: the
// sign of the message to edge j in bit 31 - j, s_c in bit 5, and in bits 0..4
// the part's edge that holds the minimum (31: another part's, or none).  So edge
// j's message is (j == word & 31 ? n2 : n1) with bit 31 of word << j on its sign.
// Ties need no rule: if two edges share the minimum, n1 = n2.
//
// Column pass: L_v = lambda_v + messages in ascending check order, one record per
// edge: {part address << 12 | j}.  No-op edges read a part whose messages are -0.
// Check pass: q = L_v - message, its minima and signs, and H [L < 0] = s; one
// 16-bit column address per edge, in any order of the part's edges (32 bits when
// the columns need it).  No-op edges read L = +inf, which changes nothing.
// A split check's parts merge their minima and parities with DPP exchanges.
//
// Measured against lists of one edge per lane with per-lane flags and (checks of
// more than 30 edges) a sign byte per edge, ms: 10^6 shots of the d = 5 non-local
// CNOT 10.7 -> 5.5, 65,536 of BB [[144,12,12]] memory 33.2 -> 16.9, 32,768 of its
// teleportation 72.7 -> 19.6 (8192 with learned weights 49.9 -> 9.2), 1021 of the
// d = 11 CNOT 0.58 -> 0.44.  About 13 vector instructions per edge step in the check
// pass and 8 in the column pass (57 together before); with no-op edges, chunk ends
// and a shot's start and end the counters give 41 per edge and iteration at d = 5
// (2.4 iterations a shot) and 30 on BB [[144,12,12]] memory (11.5).  Vector
// instructions fill 93 and 100 % of their issue slots there, LDS (with bank
// conflicts) 39 and 52 % of its cycles.
//
// Sums run in ascending check order and nothing is contracted, so results are
// bit-identical to the FP32 definition in decode.hip.
//
// EXACT (per-edge weights, or scalings and iterations that could reach infinity):
// comparisons as written in the definition, so that a NaN is neither negative nor
// a minimum, and the weight multiplies at use.  Otherwise signs are taken from
// the sign bit and the second minimum is the median of (n1, n2, |q|): L and q are
// never -0 there (a sum of floats is -0 only if every term is), nor NaN.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <utility>
#include <vector>

#include "../host/device.h"
#include "../host/timing.h"
#include "bp_chunk.h"
#include "bp_team.h"

namespace tmcs {
namespace dec {

namespace {

constexpr int R_PART = 12;                   // column-pass record: part address << R_PART | j
constexpr int HDR = 8;                      // table words per wave before the runs
constexpr int USUAL_RUNS = 8;               // runs of a wave in both passes together, typically

// Value of the lane whose index differs in bit `step`, for values that agree
// within groups of `step` lanes (1, 2: swaps; 4, 8: mirrors of 8 and 16 lanes).
template <typename T>
__device__ __forceinline__ T part_xchg(T x, int step) {
  const int v = __builtin_bit_cast(int, x);
  int r;
  if (step == 1) r = __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);
  else if (step == 2) r = __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true);
  else if (step == 4) r = __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true);
  else if (step == 8) r = __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, true);
  else r = __shfl_xor(v, step, 64);
  return __builtin_bit_cast(T, r);
}

using ArgsPtr = const TMCS_CONST_AS ChunkArgs*;

template <bool EXACT, bool MULTI, bool WIDE>
__global__ void __launch_bounds__(1024, 8) k_bp_chunk(ChunkArgs, ChunkMulti mu) {
  extern __shared__ __align__(16) unsigned char sm[];
  __shared__ int s_job, s_flag, s_pos, s_inst;
  __shared__ int s_unsat[2];
  __shared__ int s_pref[MAX_MULTI + 1];
  __shared__ unsigned long long s_pm[MAX_OW];
  __shared__ unsigned long long s_cnt[4];          // nontrivial, converged, osd, iterations (thread 0)
  __shared__ uint32_t s_hist[TMCS_BP_HIST_BINS];   // (thread 0)
  const int tid = threadIdx.x, P = blockDim.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  ArgsPtr a = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  unsigned char* const st = sm;                    // [Ms + 1] parts of 12 bytes (slot Ms: messages of -0)
  unsigned char* Lb = nullptr;                     // [Ns + 1] L by column slot (slot Ns: +inf)
  int32_t* tab = nullptr;                          // [ntab] runs
  auto part = [&](uint32_t byte, float* n1, float* n2, uint32_t* w) {
    const float* p = (const float*)(st + byte);
    *n1 = p[0];
    *n2 = p[1];
    *w = __float_as_uint(p[2]);
  };
  auto ld_L = [&](uint32_t byte) -> float { return *(const float*)(Lb + byte); };
  auto bind = [&]() {
    const int Ms = a->Ms, Ns = a->Ns, ntab = a->ntab;
    Lb = st + ((((uint32_t)Ms + 1) * 12 + 15) & ~15u);
    tab = (int32_t*)(Lb + ((uint32_t)Ns + 1) * 4);
    for (int i = tid; i < ntab; i += P) tab[i] = gload(a->tab + i);
    if (tid == 0) {
      float* z = (float*)(st + (uint32_t)Ms * 12);
      z[0] = 0.0f;
      z[1] = 0.0f;
      z[2] = __uint_as_float(W_SIGNS | W_POS);
      *(float*)(Lb + (uint32_t)Ns * 4) = __builtin_inff();
    }
    __syncthreads();
  };
  int32_t total = 0;                               // MULTI: thread 0's
  int cur = -1;                                    // MULTI: item the team works on
  if constexpr (!MULTI) {
    total = a->queue ? a->counters[0] : (int32_t)a->nshots;
    if ((int)blockIdx.x >= total) return;
    bind();
  } else if (tid == 0) {
    s_pref[0] = 0;
    for (int i = 0; i < mu.n; ++i)
      s_pref[i + 1] = s_pref[i] + (mu.tab[i].queue ? mu.tab[i].counters[0] : (int32_t)mu.tab[i].nshots);
    total = s_pref[mu.n];
  }
  for (int i = tid; i < TMCS_BP_HIST_BINS; i += P) s_hist[i] = 0u;
  if (tid < 4) s_cnt[tid] = 0ull;
  auto flush = [&]() {
    __syncthreads();
    // (as many copies of the statistics as spare the teams waiting on each other's adds)
    tmcs_decode_stats* stats = reread(a)->stats;
    if (stats) {
      stats += blockIdx.x % STAT_SHARDS;
      for (int i = tid; i < TMCS_BP_HIST_BINS; i += P)
        if (s_hist[i]) atomicAdd((unsigned long long*)&stats->bp_iter_hist[i], (unsigned long long)s_hist[i]);
      if (tid == 0) {
        if (s_cnt[0]) atomicAdd((unsigned long long*)&stats->nontrivial, s_cnt[0]);
        if (s_cnt[1]) atomicAdd((unsigned long long*)&stats->converged, s_cnt[1]);
        if (s_cnt[2]) atomicAdd((unsigned long long*)&stats->osd, s_cnt[2]);
        if (s_cnt[3]) atomicAdd((unsigned long long*)&stats->bp_iters, s_cnt[3]);
      }
    }
    __syncthreads();
    for (int i = tid; i < TMCS_BP_HIST_BINS; i += P) s_hist[i] = 0u;
    if (tid < 4) s_cnt[tid] = 0ull;
    __syncthreads();
  };
  // A team's first job is its own number; thread 0 takes the others from a
  // counter, several at a time: a counter gives out about 85 values a
  // microsecond, fewer than the teams of a small DEM finish shots (d = 5: 5.7
  // instead of 10.7 ms per 10^6 shots), and as many teams as there are shots
  // never ask for one.  Batches grow with the number of teams (small DEMs, short
  // shots); with few teams they stay at one shot, so that the launch ends evenly.
  int ticket = (int)blockIdx.x, left = 0;
  const int batch = max(1, (int)gridDim.x / 1024);
  auto take = [&]() {
    if (left == 0) {
      ticket = total > (int)gridDim.x ? (int)gridDim.x + atomicAdd(MULTI ? mu.next : &a->counters[1], batch) : total;
      left = batch;
    } else {
      ++ticket;
    }
    --left;
  };
  while (true) {
    if (tid == 0) {
      if constexpr (MULTI) {
        int i = 0;
        while (i < mu.n && ticket >= s_pref[i + 1]) ++i;
        s_inst = i;
        s_job = i < mu.n ? ticket - s_pref[i] : 0;
      } else {
        s_job = ticket;
      }
      s_flag = 0;
      s_unsat[0] = 0;
      s_unsat[1] = 0;
      for (int w = 0; w < MAX_OW; ++w) s_pm[w] = 0ull;
    }
    __syncthreads();
    if constexpr (MULTI) {
      const int inst = __builtin_amdgcn_readfirstlane(s_inst);
      if (inst != cur) {                           // uniform: the team moves to the next item
        if (cur >= 0) flush();
        if (inst >= mu.n) break;
        cur = inst;
        a = (ArgsPtr)(uintptr_t)(mu.tab + inst);
        bind();
      }
    }
    const int job = __builtin_amdgcn_readfirstlane(s_job);
    if (!MULTI && job >= total) break;
    const int T = a->T;
    const bool use_w = EXACT && a->wv != nullptr;
    const float alpha = use_w ? 1.0f : a->alpha;
    int ls = job;                                  // shot of the pass
    // state of iteration 1
    {
      const ArgsPtr c = reread(a);
      if (c->queue) ls = __builtin_amdgcn_readfirstlane(gload(c->queue + job));
      const int mw = c->mw;
      const uint64_t* sy = c->synd + (int64_t)ls * mw;
      int fl = 0;
      for (int i = tid; i < c->Ms; i += P) {
        const int4 s0 = gload(c->pinit + i);
        const int sb = s0.w < 0 ? 0 : (int)((gload(sy + (s0.w >> 6)) >> (s0.w & 63)) & 1ull);
        fl |= sb;
        float* p = (float*)(st + (uint32_t)i * 12);
        const float m1 = __int_as_float(s0.x), m2 = __int_as_float(s0.y);
        p[0] = use_w ? m1 : __fmul_rn(alpha, m1);
        p[1] = use_w ? m2 : __fmul_rn(alpha, m2);
        p[2] = __uint_as_float((uint32_t)s0.z ^ (sb ? (W_SIGNS | W_SC) : 0u));
      }
      // a detection event on a check without edges: never satisfied
      if (c->lone)
        for (int w = tid; w < mw; w += P)
          if (gload(sy + w) & gload(c->lone + w)) fl |= 3;
      if (fl) atomicOr(&s_flag, fl);
    }
    if (tid == 0) take();
    __syncthreads();
    const int f0 = __builtin_amdgcn_readfirstlane(s_flag);
    int itr = 0;
    bool conv = true;
    // message of edge j (the low five bits of jr) of a part
    auto message = [&](float n1, float n2, uint32_t w, uint32_t jr, float wt) -> float {
      float mag = ((w ^ jr) & W_POS) == 0u ? n2 : n1;
      if (EXACT && use_w) mag = __fmul_rn(wt, mag);
      return with_sign(mag, w << (jr & 31u));
    };
    if (f0 & 1) {
      conv = false;
      const int32_t* hd = tab + wave * HDR;
      for (int t = 1;; ++t) {
        // column pass: L^t from the state of iteration t
        {
          const int vrow0 = __builtin_amdgcn_readfirstlane(hd[0]);
          uint32_t slot4 = (uint32_t)(__builtin_amdgcn_readfirstlane(hd[1]) + lane) * 4;
          const int vruns = __builtin_amdgcn_readfirstlane(hd[2]), vrun0 = __builtin_amdgcn_readfirstlane(hd[3]);
          const uint32_t* const rp = a->vrec + (size_t)vrow0 * 64;
          const float* const wp = use_w ? a->wv + (int64_t)(t - 1) * a->wv_stride + (size_t)vrow0 * 64 : nullptr;
          const float* const lamp = a->lamp;
          uint32_t at = (uint32_t)lane * 4;        // byte of the lane's next record
          // chunks of K edges per column, K known: the next chunk's records are in flight
          auto fixed = [&](auto KC, int cnt) {
            constexpr int K = decltype(KC)::value;
            uint32_t r[K];
            float wt[K];
#pragma unroll
            for (int u = 0; u < K; ++u) {
              r[u] = at_byte(rp, at + u * 256);
              wt[u] = EXACT && use_w ? at_byte(wp, at + u * 256) : 0.0f;
            }
            float acc = at_byte(lamp, slot4);
            for (int i = 0; i < cnt; ++i) {
              float n1[K], n2[K];
              uint32_t w[K], rn[K];
              float wn[K];
#pragma unroll
              for (int u = 0; u < K; ++u) part(r[u] >> R_PART, &n1[u], &n2[u], &w[u]);
              at += K * 256;
#pragma unroll
              for (int u = 0; u < K; ++u) {
                rn[u] = at_byte(rp, at + u * 256);
                wn[u] = EXACT && use_w ? at_byte(wp, at + u * 256) : 0.0f;
              }
              const float nlam = at_byte(lamp, slot4 + 256);
#pragma unroll
              for (int u = 0; u < K; ++u) acc = __fadd_rn(acc, message(n1[u], n2[u], w[u], r[u], wt[u]));
              *(float*)(Lb + slot4) = acc;
              acc = nlam;
              slot4 += 256;
#pragma unroll
              for (int u = 0; u < K; ++u) {
                r[u] = rn[u];
                wt[u] = wn[u];
              }
            }
          };
          for (int q = 0; q < vruns; ++q) {
            const int K = __builtin_amdgcn_readfirstlane(tab[vrun0 + 2 * q]);
            const int cnt = __builtin_amdgcn_readfirstlane(tab[vrun0 + 2 * q + 1]);
            switch (K) {
              case 1: fixed(std::integral_constant<int, 1>{}, cnt); break;
              case 2: fixed(std::integral_constant<int, 2>{}, cnt); break;
              case 3: fixed(std::integral_constant<int, 3>{}, cnt); break;
              case 4: fixed(std::integral_constant<int, 4>{}, cnt); break;
              default:
                for (int i = 0; i < cnt; ++i) {
                  float acc = at_byte(lamp, slot4);
#pragma unroll 2
                  for (int u = 0; u < K; ++u) {
                    const uint32_t r = at_byte(rp, at);
                    const float wt = EXACT && use_w ? at_byte(wp, at) : 0.0f;
                    at += 256;
                    float n1, n2;
                    uint32_t w;
                    part(r >> R_PART, &n1, &n2, &w);
                    acc = __fadd_rn(acc, message(n1, n2, w, r, wt));
                  }
                  *(float*)(Lb + slot4) = acc;
                  slot4 += 256;
                }
            }
          }
        }
        __syncthreads();
        // check pass: H [L^t < 0] = s ?  and, if t < T, the state of iteration t + 1
        int unsat = (f0 >> 1) & 1;
        auto check_pass = [&](auto UPD) {
          constexpr bool update = decltype(UPD)::value;
          const int crow0 = __builtin_amdgcn_readfirstlane(hd[4]);
          uint32_t slot12 = (uint32_t)(__builtin_amdgcn_readfirstlane(hd[5]) + lane) * 12;
          const int cruns = __builtin_amdgcn_readfirstlane(hd[6]), crun0 = __builtin_amdgcn_readfirstlane(hd[7]);
          const uint32_t* const rp = a->crec + (size_t)crow0 * (WIDE ? 64 : 32);
          const float* const wp = use_w ? a->wc + (int64_t)(t - 1) * a->wc_stride + (size_t)crow0 * 64 : nullptr;
          // two steps per round: their L values were read one round ahead, their
          // records two (chunks follow each other in the stream)
          uint32_t at = (uint32_t)lane * 4, wat = (uint32_t)lane * 4;
          uint32_t ra = at_byte(rp, at), rb = WIDE ? at_byte(rp, at + 256) : 0u;
          float La = ld_L(WIDE ? ra : (ra & 0xFFFFu)), Ln = ld_L(WIDE ? rb : (ra >> 16));
          at += WIDE ? 512 : 256;
          ra = at_byte(rp, at);
          if (WIDE) rb = at_byte(rp, at + 256);
          for (int q = 0; q < cruns; ++q) {
            const int K = __builtin_amdgcn_readfirstlane(tab[crun0 + 2 * q]);
            const int cf = __builtin_amdgcn_readfirstlane(tab[crun0 + 2 * q + 1]);
            const int cnt = cf & 0xFFFF, f = cf >> 16;
            for (int i = 0; i < cnt; ++i) {
              float n1o, n2o;
              uint32_t wo;
              part(slot12, &n1o, &n2o, &wo);
              const uint32_t ago = wo & W_POS;
              float n1 = BP_BIG, n2 = BP_BIG;
              uint32_t lt = 0u, nb = 0u, hx = 0u;    // lt: steps that brought a new minimum, the last in bit 0
              auto step = [&](int j, float Lv, float wt) {
                if constexpr (EXACT) hx ^= Lv < 0.0f ? 0x80000000u : 0u;
                else hx ^= __float_as_uint(Lv);
                if constexpr (update) {
                  float mag = ago == (uint32_t)j ? n2o : n1o;
                  if (EXACT && use_w) mag = __fmul_rn(wt, mag);
                  const float qv = __fsub_rn(Lv, with_sign(mag, wo << j));
                  const float aq = fabsf(qv);
                  if constexpr (EXACT) {
                    const bool lt1 = aq < n1;
                    n2 = lt1 ? n1 : (aq < n2 ? aq : n2);
                    n1 = lt1 ? aq : n1;
                    lt = (lt << 1) | (lt1 ? 1u : 0u);
                    nb = (nb << 1) | (qv < 0.0f ? 1u : 0u);
                  } else {
                    // (a difference of floats is negative exactly when the first is smaller)
                    lt = __builtin_amdgcn_alignbit(lt, __float_as_uint(__fsub_rn(aq, n1)), 31);
                    n2 = __builtin_amdgcn_fmed3f(n1, n2, aq);
                    n1 = __builtin_amdgcn_fmed3f(n1, aq, -__builtin_inff());   // (min, without a canonicalising move)
                    nb = __builtin_amdgcn_alignbit(nb, __float_as_uint(qv), 31);
                  }
                }
              };
#pragma unroll 2
              for (int j = 0; j < K; j += 2) {
                const float L0 = La, L1 = Ln;
                float w0 = 0.0f, w1 = 0.0f;
                if (EXACT && update && use_w) {
                  w0 = at_byte(wp, wat);
                  w1 = at_byte(wp, wat + 256);
                  wat += 512;
                }
                La = ld_L(WIDE ? ra : (ra & 0xFFFFu));
                Ln = ld_L(WIDE ? rb : (ra >> 16));
                at += WIDE ? 512 : 256;
                ra = at_byte(rp, at);
                if (WIDE) rb = at_byte(rp, at + 256);
                step(j, L0, w0);
                step(j + 1, L1, w1);
              }
              uint32_t par = 0u;
              float m1 = n1, m2 = n2;
              if constexpr (update) {
                nb <<= 32 - K;
                par = (uint32_t)__popc(nb) << 31;
              }
              // parts of one check: minima and parities of the whole
              for (int s = 1; s < f; s <<= 1) {
                hx ^= part_xchg(hx, s);
                if constexpr (update) {
                  par ^= part_xchg(par, s);
                  const float o1 = part_xchg(m1, s), o2 = part_xchg(m2, s);
                  m2 = fminf(fmaxf(m1, o1), fminf(m2, o2));
                  m1 = fminf(m1, o1);
                }
              }
              const uint32_t sc = wo & W_SC;
              unsat |= (int)((hx >> 31) ^ (sc >> 5));
              if constexpr (update) {
                // (lt = 0, or a minimum that is another part's: none here)
                const uint32_t ag = lt && n1 == m1 ? (uint32_t)(K - __ffs(lt)) : W_POS;
                // message sign of edge j = s_c + parity + sgn q_j (mod 2)
                const uint32_t flip = (par >> 31) != (sc >> 5) ? W_SIGNS : 0u;
                float* p = (float*)(st + slot12);
                p[0] = use_w ? m1 : __fmul_rn(alpha, m1);
                p[1] = use_w ? m2 : __fmul_rn(alpha, m2);
                p[2] = __uint_as_float(((nb ^ flip) & W_SIGNS) | sc | ag);
              }
              slot12 += 768;
            }
          }
        };
        if (t < T) check_pass(std::true_type{});
        else check_pass(std::false_type{});
        if (__ballot(unsat != 0) != 0ull && lane == 0) s_unsat[t & 1] = 1;   // (every writer stores 1)
        if (tid == 0) s_unsat[(t + 1) & 1] = 0;            // read by every lane before the last barrier
        __syncthreads();
        if (!__builtin_amdgcn_readfirstlane(s_unsat[t & 1])) { itr = t; conv = true; break; }
        if (t >= T) { itr = T; break; }
      }
    }
    // finalise: prediction from the hard decision, or hand the posteriors to OSD
    const ArgsPtr c = reread(a);
    if (tid == 0) s_pos = (!conv && c->use_osd) ? atomicAdd(&c->counters[2], 1) : -1;
    __syncthreads();
    const int pos = __builtin_amdgcn_readfirstlane(s_pos);
    const int64_t shot = c->shot0 + ls;
    const int n = c->n;
    if (pos >= 0 || c->llr || c->ehat)
      for (int v = tid; v < n; v += P) {
        const int vm = gload(c->vmap + v);
        const float Lv = (vm >= 0 && (f0 & 1)) ? ld_L((uint32_t)vm * 4) : gload(c->lam + v);   // (no BP run: the priors)
        if (pos >= 0) c->osd_llr[(int64_t)pos * n + v] = Lv;
        if (c->llr) c->llr[shot * n + v] = Lv;
        if (c->ehat && pos < 0) c->ehat[shot * n + v] = Lv < 0.0f ? 1 : 0;
      }
    if (pos < 0 && (f0 & 1)) {
      for (int w = 0; w < c->ow; ++w) {
        uint64_t pm = 0ull;
        for (int i = tid; i < c->noc; i += P)
          if (ld_L((uint32_t)gload(c->oslot + i) * 4) < 0.0f) pm ^= gload(c->omask + (int64_t)w * c->noc + i);
        if (pm) atomicXor(&s_pm[w], (unsigned long long)pm);
      }
    }
    __syncthreads();
    if (tid == 0) {
      if (pos < 0)
        for (int w = 0; w < c->ow; ++w)
          write_pred(c->pred, c->stride, c->nobs, shot, (f0 & 1) ? s_pm[w] ^ c->pm_iso[w] : c->pm_lam[w], w);
      else c->osd_queue[pos] = ls;
      if (c->iters) c->iters[shot] = itr;
      if (c->flags) c->flags[shot] = (uint8_t)((conv ? 1 : 0) | (pos >= 0 ? 2 : 0));
      s_cnt[0] += (itr > 0 || !conv) ? 1 : 0;
      s_cnt[1] += conv ? 1 : 0;
      s_cnt[2] += pos >= 0 ? 1 : 0;
      s_cnt[3] += (unsigned long long)itr;
      s_hist[itr < TMCS_BP_HIST_BINS - 1 ? itr : TMCS_BP_HIST_BINS - 1] += 1u;
    }
  }
  if constexpr (!MULTI) flush();
}

// (a grid has at most 65535 rows of blocks, and there may be more iterations)
__global__ void __launch_bounds__(256) k_chunk_weights(const float* __restrict__ w, int64_t E, int T,
                                                       const int32_t* __restrict__ vedge, int64_t nv,
                                                       const int32_t* __restrict__ cedge, int64_t nc,
                                                       float* __restrict__ wv, float* __restrict__ wc) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int t = blockIdx.y; t < T; t += gridDim.y) {
    if (i < nv) {
      const int32_t e = vedge[i];
      wv[t * nv + i] = e < 0 ? 0.0f : w[t * E + e];
    } else if (i < nv + nc) {
      const int32_t e = cedge[i - nv];
      wc[t * nc + (i - nv)] = e < 0 ? 0.0f : w[t * E + e];
    }
  }
}

// ------------------------------------------------------------------ host
struct Chunk {
  int K = 0, f = 1;
  std::vector<int> item;   // [64] check part (c * 64 + part index is not needed: parts of a check are neighbours) or column; -1: empty
};

// Instructions of a chunk (the check pass measured about 12 per edge and 30 per chunk; the column pass 8 and 6).
long chunk_cost_c(const Chunk& c) {
  int s = 0;
  while ((1 << s) < c.f) ++s;
  return 30 + 12l * c.K + 9l * s;
}
long chunk_cost_v(const Chunk& c) { return 6 + 8l * c.K; }

// Chunks to NW waves, longest first; a wave's chunks end up in runs of one width.
template <typename Cost>
long assign_chunks(std::vector<Chunk>& ch, int NW, Cost cost, std::vector<std::vector<int>>* waves) {
  std::vector<int> order(ch.size());
  for (size_t i = 0; i < order.size(); ++i) order[i] = (int)i;
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return cost(ch[x]) > cost(ch[y]); });
  waves->assign(NW, {});
  std::vector<long> load(NW, 0);
  for (int i : order) {
    const int w = (int)(std::min_element(load.begin(), load.end()) - load.begin());
    (*waves)[w].push_back(i);
    load[w] += cost(ch[i]);
  }
  return *std::max_element(load.begin(), load.end());   // (no chunks: 0)
}

std::vector<Chunk> column_chunks(const Dem& D) {
  std::vector<int> items;
  auto deg = [&](int v) { return D.col_ptr[v + 1] - D.col_ptr[v]; };
  for (int v = 0; v < D.cols; ++v)
    if (deg(v) > 0) items.push_back(v);
  std::stable_sort(items.begin(), items.end(), [&](int x, int y) { return deg(x) < deg(y); });
  std::vector<Chunk> out;
  for (size_t i = 0; i < items.size(); i += 64) {
    Chunk c;
    c.item.assign(64, -1);
    for (size_t j = 0; j < 64 && i + j < items.size(); ++j) {
      c.item[j] = items[i + j];
      c.K = std::max(c.K, (int)deg(items[i + j]));
    }
    out.push_back(c);
  }
  return out;
}

// Parts of at most `most` edges; f parts of a check in lanes f i .. f i + f - 1.
bool check_chunks(const Dem& D, int most, std::vector<Chunk>* out) {
  out->clear();
  auto deg = [&](int c) { return D.row_ptr[c + 1] - D.row_ptr[c]; };
  std::vector<std::vector<int>> by_f(7);
  for (int c = 0; c < D.rows; ++c) {
    if (deg(c) == 0) continue;
    int s = 0;
    while (((deg(c) + (1 << s) - 1) >> s) > most) ++s;
    if (s > 6) return false;
    by_f[s].push_back(c);
  }
  for (int s = 0; s <= 6; ++s) {
    auto& items = by_f[s];
    auto size = [&](int c) { return (deg(c) + (1 << s) - 1) >> s; };
    std::stable_sort(items.begin(), items.end(), [&](int x, int y) { return size(x) < size(y); });
    const size_t per = 64u >> s;
    for (size_t i = 0; i < items.size(); i += per) {
      Chunk c;
      c.f = 1 << s;
      c.item.assign(64, -1);
      for (size_t j = 0; j < per && i + j < items.size(); ++j) {
        for (int k = 0; k < c.f; ++k) c.item[j * c.f + k] = items[i + j];
        c.K = std::max(c.K, size(items[i + j]));
      }
      c.K = (c.K + 1) & ~1;                        // two steps per record
      out->push_back(c);
    }
  }
  return true;
}

// Runs of one width that a wave walks: {K, chunks | f << 16 (check pass)}.
std::vector<std::pair<int32_t, int32_t>> wave_runs(const std::vector<int>& list, const std::vector<Chunk>& ch, bool check_pass) {
  std::vector<std::pair<int32_t, int32_t>> runs;
  for (size_t i = 0; i < list.size();) {
    size_t k = i;
    while (k < list.size() && k - i < 0xFFFF && ch[list[k]].K == ch[list[i]].K && ch[list[k]].f == ch[list[i]].f) ++k;
    runs.push_back({ch[list[i]].K, (int32_t)(k - i) | (check_pass ? ch[list[i]].f << 16 : 0)});
    i = k;
  }
  return runs;
}

// The chunks of a team of NW waves, which wave takes which, and its LDS bytes.
struct ChunkPlan {
  std::vector<Chunk> cc, vc;
  std::vector<std::vector<int>> cw, vw;
  size_t lds = 0;
};

size_t plan_lds(const ChunkPlan& p, int NW) {
  ChunkSched s;
  s.Ms = (int32_t)p.cc.size() * 64;
  s.Ns = (int32_t)p.vc.size() * 64;
  s.ntab = NW * HDR;
  for (const auto& w : p.cw) s.ntab += 2 * (int32_t)wave_runs(w, p.cc, true).size();
  for (const auto& w : p.vw) s.ntab += 2 * (int32_t)wave_runs(w, p.vc, false).size();
  return s.lds();
}

// The plan whose check chunks take the team the fewest instructions, of those
// that fit in one compute unit's LDS; false if none does.
bool plan_chunks(const Dem& D, int NW, ChunkPlan* out) {
  ChunkPlan p;
  p.vc = column_chunks(D);
  assign_chunks(p.vc, NW, chunk_cost_v, &p.vw);
  long best_cost = -1;
  for (int most : {PART_MAX_DEG, 20, 16, 12, 10, 8}) {
    if (!check_chunks(D, most, &p.cc)) continue;
    const long cost = assign_chunks(p.cc, NW, chunk_cost_c, &p.cw);
    p.lds = plan_lds(p, NW);
    // (a smaller part size also takes more state: at equal cost the larger one stays)
    if (p.lds + CHUNK_LDS_STATIC > 160 * 1024 || (best_cost >= 0 && cost >= best_cost)) continue;
    best_cost = cost;
    *out = p;
  }
  return best_cost >= 0;
}

}  // namespace

bool chunk_fits(const Dem& D, int P, size_t* lds, size_t* usual) {
  ChunkPlan p;
  if (!plan_chunks(D, P / 64, &p)) return false;
  ChunkSched s;
  s.Ms = (int32_t)p.cc.size() * 64;
  s.Ns = (int32_t)p.vc.size() * 64;
  s.ntab = P / 64 * (HDR + 2 * USUAL_RUNS);
  *lds = p.lds;
  *usual = s.lds();
  return true;
}

tmcs_status build_chunk_sched(const Dem& D, int P, ChunkSched* out) {
  const int NW = P / 64;
  ChunkSched s;
  s.P = P;
  std::vector<float> lam(D.cols);
  for (int v = 0; v < D.cols; ++v) lam[v] = (float)std::log((1.0 - D.priors[v]) / D.priors[v]);
  ChunkPlan plan;
  if (!plan_chunks(D, NW, &plan)) return TMCS_EUNSUPPORTED;   // (not an error of the call: no message)
  const auto &cc = plan.cc, &vc = plan.vc;
  const auto &cw = plan.cw, &vw = plan.vw;
  s.Ms = (int32_t)cc.size() * 64;
  s.Ns = (int32_t)vc.size() * 64;
  s.wide = (size_t)s.Ns * 4 > 0xFFFFu;
  // slots in the order of the waves' lists; a check's part and the edge's place in it
  std::vector<int32_t> part_slot((size_t)std::max<int64_t>(D.edges, 1), 0), part_pos(part_slot), vmap(std::max(D.cols, 1), -1);
  std::vector<int4> pinit((size_t)s.Ms);
  std::vector<int32_t> tab((size_t)NW * HDR, 0);
  int32_t slot = 0;
  for (int w = 0; w < NW; ++w)
    for (int i : vw[w]) {
      for (int j = 0; j < 64; ++j)
        if (vc[i].item[j] >= 0) vmap[vc[i].item[j]] = slot + j;
      slot += 64;
    }
  std::vector<float> lamp((size_t)s.Ns + 64, 0.0f);
  for (int v = 0; v < D.cols; ++v)
    if (vmap[v] >= 0) lamp[vmap[v]] = lam[v];
  // check streams
  std::vector<uint32_t> crec, vrec;
  std::vector<int32_t> cedge, vedge;
  const uint32_t PADL = (uint32_t)s.Ns * 4;
  slot = 0;
  for (int w = 0; w < NW; ++w) {
    tab[w * HDR + 4] = (int32_t)(cedge.size() / 64);
    tab[w * HDR + 5] = slot;
    for (int i : cw[w]) {
      const Chunk& c = cc[i];
      std::vector<uint32_t> addr((size_t)c.K * 64, PADL);
      std::vector<int32_t> edge((size_t)c.K * 64, -1);
      for (int j = 0; j < 64; ++j) {
        const int chk = c.item[j];
        int4 r = make_int4(0, 0, (int32_t)W_POS, chk);
        float n1 = BP_BIG, n2 = BP_BIG;
        if (chk >= 0) {
          const int32_t e0 = D.row_ptr[chk], e1 = D.row_ptr[chk + 1], part = j % c.f;
          const int size = (e1 - e0 + c.f - 1) / c.f;
          const int32_t p0 = std::min(e1, e0 + part * size), p1 = std::min(e1, p0 + size);
          int32_t arg = -1;
          int par = 0;
          for (int32_t e = e0; e < e1; ++e) {
            const float q = lam[D.col_idx[e]], aq = std::fabs(q);
            if (aq < n1) { n2 = n1; n1 = aq; arg = e; }
            else if (aq < n2) { n2 = aq; }
            par ^= q < 0.0f ? 1 : 0;
          }
          uint32_t word = arg >= p0 && arg < p1 ? (uint32_t)(arg - p0) : W_POS;
          for (int32_t e = p0; e < p1; ++e) {
            const int k = e - p0;
            part_slot[e] = slot + j;
            part_pos[e] = k;
            addr[(size_t)k * 64 + j] = (uint32_t)vmap[D.col_idx[e]] * 4;
            edge[(size_t)k * 64 + j] = e;
            word |= (uint32_t)(par ^ (lam[D.col_idx[e]] < 0.0f ? 1 : 0)) << (31 - k);
          }
          r.z = (int32_t)word;
        }
        std::memcpy(&r.x, &n1, 4);
        std::memcpy(&r.y, &n2, 4);
        pinit[(size_t)slot + j] = r;
      }
      if (s.wide) {
        crec.insert(crec.end(), addr.begin(), addr.end());
      } else {
        for (int k = 0; k < c.K; k += 2)
          for (int j = 0; j < 64; ++j) crec.push_back(addr[(size_t)k * 64 + j] | addr[(size_t)(k + 1) * 64 + j] << 16);
      }
      cedge.insert(cedge.end(), edge.begin(), edge.end());
      slot += 64;
    }
  }
  // column streams
  const uint32_t PADC = ((uint32_t)s.Ms * 12) << R_PART;
  slot = 0;
  for (int w = 0; w < NW; ++w) {
    tab[w * HDR + 0] = (int32_t)(vedge.size() / 64);
    tab[w * HDR + 1] = slot;
    for (int i : vw[w]) {
      const Chunk& c = vc[i];
      for (int k = 0; k < c.K; ++k)
        for (int j = 0; j < 64; ++j) {
          const int v = c.item[j];
          if (v >= 0 && D.col_ptr[v] + k < D.col_ptr[v + 1]) {
            const int32_t e = D.csc_edge[D.col_ptr[v] + k];
            vrec.push_back(((uint32_t)part_slot[e] * 12) << R_PART | (uint32_t)part_pos[e]);
            vedge.push_back(e);
          } else {
            vrec.push_back(PADC);
            vedge.push_back(-1);
          }
        }
      slot += 64;
    }
  }
  s.vrows = (int32_t)(vedge.size() / 64);
  s.crows = (int32_t)(cedge.size() / 64);
  for (int i = 0; i < CHUNK_PAD_ROWS * 64; ++i) {
    vrec.push_back(PADC);
    crec.push_back(0u);
  }
  // runs
  for (int w = 0; w < NW; ++w)
    for (int pass = 0; pass < 2; ++pass) {
      const auto& list = pass ? cw[w] : vw[w];
      const auto& ch = pass ? cc : vc;
      tab[w * HDR + (pass ? 7 : 3)] = (int32_t)tab.size();
      const auto runs = wave_runs(list, ch, pass == 1);
      for (const auto& r : runs) {
        tab.push_back(r.first);
        tab.push_back(r.second);
      }
      tab[w * HDR + (pass ? 6 : 2)] = (int32_t)runs.size();
    }
  s.ntab = (int32_t)tab.size();
  // columns that flip an observable
  std::vector<int32_t> oslot;
  std::vector<int> oc;
  for (int v = 0; v < D.cols; ++v) {
    bool any = false;
    for (int w = 0; w < D.obs_words; ++w) any = any || D.obs_mask[(size_t)v * D.obs_words + w];
    if (any && vmap[v] >= 0) { oc.push_back(v); oslot.push_back(vmap[v]); }
  }
  s.noc = (int32_t)oc.size();
  std::vector<uint64_t> omask((size_t)D.obs_words * oc.size());
  for (size_t i = 0; i < oc.size(); ++i)
    for (int w = 0; w < D.obs_words; ++w) omask[(size_t)w * oc.size() + i] = D.obs_mask[(size_t)oc[i] * D.obs_words + w];
  Uploader up("BP schedule");
  tmcs_status st;
  if ((st = up(&s.vrec, vrec)) != TMCS_OK || (st = up(&s.crec, crec)) != TMCS_OK ||
      (st = up(&s.tab, tab)) != TMCS_OK || (st = up(&s.lamp, lamp)) != TMCS_OK ||
      (st = up(&s.pinit, pinit)) != TMCS_OK || (st = up(&s.vmap, vmap)) != TMCS_OK ||
      (st = up(&s.oslot, oslot)) != TMCS_OK || (st = up(&s.omask, omask)) != TMCS_OK ||
      (st = up(&s.vedge, vedge)) != TMCS_OK || (st = up(&s.cedge, cedge)) != TMCS_OK) {
    free_chunk_sched(&s);
    return st;
  }
  *out = s;
  return TMCS_OK;
}

void free_chunk_sched(ChunkSched* s) {
  (void)hipFree(s->vrec); (void)hipFree(s->crec); (void)hipFree(s->tab); (void)hipFree(s->lamp); (void)hipFree(s->pinit); (void)hipFree(s->vmap);
  (void)hipFree(s->oslot); (void)hipFree(s->omask); (void)hipFree(s->vedge); (void)hipFree(s->cedge);
  *s = ChunkSched();
}

tmcs_status launch_chunk_weights(const ChunkSched& s, const float* w, int T, int64_t E, float* wv, float* wc,
                                 hipStream_t stream) {
  const int64_t nv = (int64_t)s.vrows * 64, nc = (int64_t)s.crows * 64;
  if (nv + nc == 0 || T < 1) return TMCS_OK;
  TMCS_LAUNCH("k_chunk_weights", k_chunk_weights, dim3((unsigned)((nv + nc + 255) / 256), (unsigned)std::min(T, 65535)), dim3(256), 0, stream,
              w, E, T, s.vedge, nv, s.cedge, nc, wv, wc);
  return hip_check(hipGetLastError(), "k_chunk_weights launch");
}

namespace {
template <bool EXACT, bool MULTI, bool WIDE>
tmcs_status launch(const ChunkArgs& a, const ChunkMulti& mu, int grid, int P, size_t lds, hipStream_t stream) {
  auto k = k_bp_chunk<EXACT, MULTI, WIDE>;
  if (lds > 64 * 1024 && hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return fail(TMCS_EUNSUPPORTED, "BP state does not fit in LDS");
  TMCS_LAUNCH("k_bp", k, dim3((unsigned)grid), dim3((unsigned)P), lds, stream, a, mu);
  return hip_check(hipGetLastError(), "k_bp_chunk launch");
}
}  // namespace

tmcs_status launch_bp_chunk(const ChunkArgs& a, const ChunkMulti& mu, bool exact, bool wide, int grid, int P, size_t lds,
                            hipStream_t stream) {
  if (P < 64 || P > 1024 || P % 64 || grid < 1) return fail(TMCS_EINVAL, "BP launch shape");
  if (mu.n > 0) {
    if (exact) return wide ? launch<true, true, true>(a, mu, grid, P, lds, stream) : launch<true, true, false>(a, mu, grid, P, lds, stream);
    return wide ? launch<false, true, true>(a, mu, grid, P, lds, stream) : launch<false, true, false>(a, mu, grid, P, lds, stream);
  }
  if (exact) return wide ? launch<true, false, true>(a, mu, grid, P, lds, stream) : launch<true, false, false>(a, mu, grid, P, lds, stream);
  return wide ? launch<false, false, true>(a, mu, grid, P, lds, stream) : launch<false, false, false>(a, mu, grid, P, lds, stream);
}

}  // namespace dec
}  // namespace tmcs

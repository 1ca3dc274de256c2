// Weighted (neural) min-sum BP for training per-edge, per-iteration weights.
//
// Forward (T flooding iterations, no early stop):
//   m_t(c,v) = w_t(c,v) * sigma_t(c,v) * mu_t(c,v),  sigma = (-1)^{s_c} prod_{v'!=v} sgn q_{t-1},
//   mu = min_{v'!=v} |q_{t-1}| (1e30 if empty);  L_t = lambda + sum_c m_t;  q_t = L_t - m_t.
// It writes L_t for every t and, per iteration, the compressed check state
// (min1, min2, argmin edge, second argmin edge, sign parity, syndrome bit, one
// sign bit of q_{t-1} per edge).  The per-edge messages are not stored: the
// backward pass rebuilds them from that state.
//
// Backward, given G_t = dLoss/dL_t (reverse mode through the unrolled forward;
// the gradient of a min goes to the lowest-index edge attaining it, signs and
// the 1e30 of an empty minimum carry none):
//   gL_t(v) = G_t(v) + sum_c gq_t(v->c);  gm_t = gL_t(v) - gq_t(v->c);
//   dLoss/dw_t(c,v) = gm_t sigma_t mu_t;
//   gq_{t-1} at the argmin edge of each message += gm_t w_t sigma_t sgn(q_{t-1}).
// gq_t is nonzero only on each check's argmin and second-argmin edge, so it is
// carried as two numbers per check.
//
// A shot's working state lives in LDS, or (GS, when it exceeds the 160 KB of a
// compute unit, as for the surface-code CNOT at d >= 15) in a slab of device
// memory per workgroup with the same layout.
//
// Checks are walked by groups of f neighbouring lanes (f a power of two, at most
// GROUP_STEPS edges to a lane), so a check of 161 edges takes as long as one of
// 35 and edge arrays are read in runs; the lanes' minima (ties to the lower edge)
// and sums meet by lane exchanges.
//
// What bounds both passes: latency of the graph's arrays (L2) and of LDS in the
// dependent chain of a check or column.  So a lane has the loads of several edges
// in flight (GROUP_STEPS, COL_STEPS; columns sorted by degree, their records and
// weights laid out step by step).  512 shots of the BB [[144,12,12]] teleportation,
// T = 20, ms: forward 4.7 with a thread per check, 2.9 with groups, 1.8 with loads
// in flight; backward 25.5, 2.4 (rows, below), 1.9.
//
// The backward pass writes every shot's dLoss/dw as rows [shot][T][E], which a
// second kernel sums over the shots.  Added straight into dLoss/dw, one atomic
// per shot, iteration and edge, the same numbers took 25.5 ms for 512 shots of
// the BB [[144,12,12]] teleportation (454 million atomics, 18 a nanosecond);
// the rows cost 1.8 GB each way, their sum 0.34 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "../host/device.h"
#include "../host/scratch.h"
#include "../host/timing.h"

namespace tmcs {

namespace {

constexpr float WBP_BIG = 1e30f;
constexpr int GROUP_STEPS = 6;                // most edges of a check that one lane walks
constexpr int COL_STEPS = 4;                  // edges of a column in flight per lane
constexpr size_t ROWS_MAX = (size_t)4 << 30;  // bytes of dLoss/dw rows in flight: more shots go in several rounds

struct WbpDevice {
  int device = -1;
  int32_t *row_ptr = nullptr, *col_idx = nullptr, *col_ptr = nullptr, *csc_row = nullptr, *csc_edge = nullptr;
  float* lam = nullptr;
  uint64_t* synd = nullptr;
  size_t cap_synd = 0;
  unsigned char* gstate = nullptr;   // GS: [grid][slab] per-workgroup state
  size_t cap_gstate = 0;
  int32_t* gchk = nullptr;           // [ngroups][64] check of each lane (-1: none)
  int32_t* gf = nullptr;             // [ngroups] lanes per check
  int32_t ngroups = 0;
  int32_t* vcol = nullptr;           // [nvchunks][64] columns by degree (-1: none)
  int32_t* vrow = nullptr;           // [nvchunks + 1] first row of each chunk's edges
  int2* vce = nullptr;               // [vrows][64] check and CSR edge of a column's k-th edge (edge -1: none)
  int32_t nvchunks = 0, vrows = 0;
  float* wcol = nullptr;             // [T][vrows][64] weights in that order
  size_t cap_wcol = 0;
  float* rows = nullptr;             // [shots of a round][T][E] dLoss/dw by shot
  size_t cap_rows = 0;
  size_t most_rows = ROWS_MAX / 4;   // floats of rows worth asking for (less once the device had no room)
  std::mutex mu;                     // held while a call sizes the scratch and enqueues its kernels
  hipEvent_t last = nullptr;         // after the last kernel that used the scratch
};

bool g_force_gs = false;             // keep the state in device memory even when it fits in LDS

// Per-iteration record in the workspace.
struct Layout {
  int64_t state;    // bytes of [m] float4-like {n1, n2, nag, a2}
  int64_t flags;    // bytes of [m] u8 (bit0 sign parity, bit1 syndrome), padded to 4
  int64_t signs;    // bytes of [nwords] u32
  int64_t iter;     // bytes per iteration
  int64_t shot;     // bytes per shot (T iterations)
};

Layout layout(const Dem& d, int T) {
  Layout L;
  const int64_t nwords = (d.edges + 31) / 32;
  L.state = (int64_t)d.rows * 16;
  L.flags = ((int64_t)d.rows + 3) / 4 * 4;
  L.signs = nwords * 4;
  L.iter = L.state + L.flags + L.signs;
  L.shot = L.iter * T;
  return L;
}

struct WbpArgs {
  const int32_t* row_ptr;
  const int32_t* col_idx;
  const int32_t* col_ptr;
  const int32_t* csc_row;
  const int32_t* csc_edge;
  const float* lam;
  const uint64_t* synd;      // [n_shots][mw]
  int32_t mw;
  int32_t m, n, T;
  int64_t E;
  int64_t nshots;            // shots of the call
  int64_t shot0, shot1;      // the shots of this launch
  const float* w;            // [T][E]
  float* llr;                // [T][n_shots][n]  (forward output)
  const float* gllr;         // [T][n_shots][n]  (backward input)
  float* rows;               // [shots][T][E]    (backward output)
  float* gw;                 // [T][E]           (the same without rows: added to)
  const int32_t* gchk;       // [ngroups][64]
  const int32_t* gf;         // [ngroups]
  int32_t ngroups;
  const int32_t* vcol;       // [nvchunks][64]
  const int32_t* vrow;       // [nvchunks + 1]
  const int2* vce;           // [vrows][64]
  const float* wcol;         // [T][vrows][64] (forward, COL)
  int32_t nvchunks, vrows;
  unsigned char* ws;         // workspace
  Layout lay;
  unsigned char* gstate;     // GS: per-workgroup slabs
  int64_t slab;              // GS: bytes per slab
};

// 32-bit load from L2 (GS: the sign words are updated with atomics)
__device__ __forceinline__ uint32_t ld_sign(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// (value, edge) pairs in order of value, then edge
__device__ __forceinline__ bool before(float x, int32_t ex, float y, int32_t ey) { return x < y || (x == y && ex < ey); }

// COL: weights laid out by column record (a.wcol), else read from a.w by edge.
template <bool GS, bool COL>
__global__ void __launch_bounds__(1024) k_wbp_forward(WbpArgs a) {
  extern __shared__ __align__(8) unsigned char sm[];
  unsigned char* base = GS ? a.gstate + (int64_t)blockIdx.x * a.slab : sm;
  const int tid = threadIdx.x, NT = blockDim.x;
  const int lane = tid & 63, wave = tid >> 6, NW = NT >> 6;
  const int m = a.m, n = a.n;
  const int64_t nwords = (a.E + 31) / 32;
  auto sbit = [&](const uint32_t* es, int64_t e) -> int {
    return (int)(((GS ? ld_sign(&es[e >> 5]) : es[e >> 5]) >> (e & 31)) & 1u);
  };
  float* Lf = (float*)base;                              // [n]
  float* n1s = Lf + n;                                   // [m]
  float* n2s = n1s + m;                                  // [m]
  int32_t* ags = (int32_t*)(n2s + m);                    // [m]
  uint32_t* es = (uint32_t*)(ags + m);                   // [nwords]
  uint8_t* cf = (uint8_t*)(es + nwords);                 // [m]
  for (int64_t shot = blockIdx.x; shot < a.nshots; shot += gridDim.x) {
    const uint64_t* sy = a.synd + shot * a.mw;
    for (int c = tid; c < m; c += NT) {
      cf[c] = (uint8_t)(((sy[c >> 6] >> (c & 63)) & 1ull) << 1);
      n1s[c] = 0.0f;
      n2s[c] = 0.0f;
      ags[c] = -1;
    }
    for (int v = tid; v < n; v += NT) Lf[v] = a.lam[v];
    for (int64_t i = tid; i < nwords; i += NT) es[i] = 0u;
    __syncthreads();
    for (int t = 1; t <= a.T; ++t) {
      unsigned char* rec = a.ws + shot * a.lay.shot + (int64_t)(t - 1) * a.lay.iter;
      int4* st = (int4*)rec;
      uint8_t* fl_out = rec + a.lay.state;
      uint32_t* sg_out = (uint32_t*)(rec + a.lay.state + a.lay.flags);
      const float* wold = t == 1 ? nullptr : a.w + (int64_t)(t - 2) * a.E;   // (t = 1: q = lambda)
      // check pass: q_{t-1} = L_{t-1} - m_{t-1}; new (min1, min2, argmin, 2nd argmin, parity)
      for (int g = wave; g < a.ngroups; g += NW) {
        const int c = a.gchk[g * 64 + lane], f = a.gf[g], sub = lane & (f - 1);
        const int cc = c < 0 ? 0 : c;
        const int32_t r0 = a.row_ptr[cc] + sub, r1 = c < 0 ? 0 : a.row_ptr[cc + 1];
        const float m1 = n1s[cc], m2 = n2s[cc];
        const int32_t ag = ags[cc];
        const uint8_t fl = cf[cc];
        const int sc = (fl >> 1) & 1, sp = fl & 1;
        constexpr int32_t NONE = 0x7FFFFFFF;
        float n1 = WBP_BIG, n2 = WBP_BIG;
        int32_t nag = NONE, a2 = NONE;
        int npar = 0;
        for (int32_t e0 = r0; e0 < r1; e0 += GROUP_STEPS * f) {
          int32_t col[GROUP_STEPS];
          float wo[GROUP_STEPS];
#pragma unroll
          for (int u = 0; u < GROUP_STEPS; ++u) {              // (past the end: the last edge again, unused)
            const int32_t e = min(e0 + u * f, r1 - 1);
            col[u] = a.col_idx[e];
            wo[u] = wold ? wold[e] : 1.0f;
          }
#pragma unroll
          for (int u = 0; u < GROUP_STEPS; ++u) {
            const int32_t e = e0 + u * f;
            if (e >= r1) break;
            const float Lv = Lf[col[u]];
            const int se = sbit(es, e);
            const float mag = __fmul_rn(wo[u], e == ag ? m2 : m1);
            const float mo = (sc ^ sp ^ se) ? -mag : mag;
            const float q = __fsub_rn(Lv, mo);
            const float aq = fabsf(q);
            const int ng = q < 0.0f ? 1 : 0;
            if (aq < n1) { n2 = n1; a2 = nag; n1 = aq; nag = e; }
            else if (aq < n2) { n2 = aq; a2 = e; }
            npar ^= ng;
            if (ng != se) atomicXor(&es[e >> 5], 1u << (e & 31));
          }
        }
        for (int s = 1; s < f; s <<= 1) {
          const float o1 = __shfl_xor(n1, s, 64), o2 = __shfl_xor(n2, s, 64);
          const int32_t og = __shfl_xor(nag, s, 64), ob = __shfl_xor(a2, s, 64);
          npar ^= __shfl_xor(npar, s, 64);
          // the two first of the four in order
          const bool mine = before(n1, nag, o1, og);
          const float x = mine ? o1 : n1, y = mine ? n2 : o2;          // the other's first, the winner's second
          const int32_t ex = mine ? og : nag, ey = mine ? a2 : ob;
          n1 = mine ? n1 : o1;
          nag = mine ? nag : og;
          const bool bx = before(x, ex, y, ey);
          n2 = bx ? x : y;
          a2 = bx ? ex : ey;
        }
        if (c >= 0 && sub == 0) {
          nag = nag == NONE ? -1 : nag;
          a2 = a2 == NONE ? -1 : a2;
          n1s[c] = n1;
          n2s[c] = n2;
          ags[c] = nag;
          cf[c] = (uint8_t)((sc << 1) | npar);
          st[c] = make_int4(__float_as_int(n1), __float_as_int(n2), nag, a2);
          fl_out[c] = (uint8_t)((sc << 1) | npar);
        }
      }
      __syncthreads();
      for (int64_t i = tid; i < nwords; i += NT) sg_out[i] = GS ? ld_sign(&es[i]) : es[i];
      // variable pass: L_t = lambda + sum_c m_t (checks ascending), a column to a
      // lane, COL_STEPS edges' records and weights in flight
      const float* wt = COL ? a.wcol + (int64_t)(t - 1) * a.vrows * 64 : a.w + (int64_t)(t - 1) * a.E;
      for (int g = wave; g < a.nvchunks; g += NW) {
        const int v = a.vcol[g * 64 + lane];
        const int row = a.vrow[g], K = a.vrow[g + 1] - row;
        float acc = v >= 0 ? a.lam[v] : 0.0f;
        for (int k0 = 0; k0 < K; k0 += COL_STEPS) {
          int2 r[COL_STEPS];
          float ww[COL_STEPS];
#pragma unroll
          for (int u = 0; u < COL_STEPS; ++u) {
            const int64_t at = (int64_t)(row + min(k0 + u, K - 1)) * 64 + lane;
            r[u] = a.vce[at];
            ww[u] = COL ? wt[at] : wt[max(r[u].y, 0)];
          }
#pragma unroll
          for (int u = 0; u < COL_STEPS; ++u) {
            if (k0 + u >= K) break;
            const int c = r[u].x, e = r[u].y;                  // (e < 0: the column has fewer edges)
            if (e < 0) continue;
            const uint8_t fl = cf[c];
            const int se = sbit(es, e);
            const float mag = __fmul_rn(ww[u], e == ags[c] ? n2s[c] : n1s[c]);
            const int neg = ((fl >> 1) ^ fl ^ se) & 1;
            acc = __fadd_rn(acc, neg ? -mag : mag);
          }
        }
        if (v >= 0) Lf[v] = acc;
      }
      __syncthreads();
      float* Lout = a.llr + ((int64_t)(t - 1) * a.nshots + shot) * n;
      for (int v = tid; v < n; v += NT) Lout[v] = Lf[v];       // (next written after the next check pass's barrier)
    }
    __syncthreads();
  }
}

// ROWS: dLoss/dw by shot into a.rows, else added to a.gw.
template <bool GS, bool ROWS>
__global__ void __launch_bounds__(1024) k_wbp_backward(WbpArgs a) {
  extern __shared__ __align__(8) unsigned char sm[];
  unsigned char* base = GS ? a.gstate + (int64_t)blockIdx.x * a.slab : sm;
  const int tid = threadIdx.x, NT = blockDim.x;
  const int lane = tid & 63, wave = tid >> 6, NW = NT >> 6;
  const int m = a.m, n = a.n;
  float* gL = (float*)base;                              // [n]
  float* g1n = gL + n;                                   // [m] gradient routed to argmin (next iteration)
  float* g2n = g1n + m;                                  // [m] ... to the second argmin
  for (int64_t shot = a.shot0 + blockIdx.x; shot < a.shot1; shot += gridDim.x) {
    const int4* stn = nullptr;                           // the next iteration's check states
    for (int t = a.T; t >= 1; --t) {
      const unsigned char* rec = a.ws + shot * a.lay.shot + (int64_t)(t - 1) * a.lay.iter;
      const int4* st = (const int4*)rec;
      const uint8_t* fl_in = rec + a.lay.state;
      const uint32_t* sg = (const uint32_t*)(rec + a.lay.state + a.lay.flags);
      const float* G = a.gllr + ((int64_t)(t - 1) * a.nshots + shot) * n;
      const float* w = a.w + (int64_t)(t - 1) * a.E;
      float* row = ROWS ? a.rows + ((shot - a.shot0) * a.T + (t - 1)) * a.E : a.gw + (int64_t)(t - 1) * a.E;
      // gL_t(v) = G_t(v) + sum_c gq_t(v->c): two edges of each check, the next
      // iteration's argmins, carry any
      if constexpr (GS) {
        for (int v = tid; v < n; v += NT) {
          float acc = G[v];
          if (stn)
            for (int32_t k = a.col_ptr[v]; k < a.col_ptr[v + 1]; ++k) {
              const int32_t c = a.csc_row[k], e = a.csc_edge[k];
              const int4 s = stn[c];
              if (e == s.z) acc += g1n[c];
              else if (e == s.w) acc += g2n[c];
            }
          gL[v] = acc;
        }
      } else {
        for (int v = tid; v < n; v += NT) gL[v] = G[v];
        __syncthreads();
        if (stn)
          for (int c = tid; c < m; c += NT) {
            const int4 s = stn[c];
            if (s.z >= 0) atomicAdd(&gL[a.col_idx[s.z]], g1n[c]);
            if (s.w >= 0) atomicAdd(&gL[a.col_idx[s.w]], g2n[c]);
          }
      }
      __syncthreads();
      // per check: dLoss/dw_t and the gradient reaching q_{t-1}
      for (int g = wave; g < a.ngroups; g += NW) {
        const int c = a.gchk[g * 64 + lane], f = a.gf[g], sub = lane & (f - 1);
        const int cc = c < 0 ? 0 : c;
        const int32_t r0 = a.row_ptr[cc] + sub, r1 = c < 0 ? 0 : a.row_ptr[cc + 1];
        const int4 s = st[cc];
        const float n1 = __int_as_float(s.x), n2 = __int_as_float(s.y);
        const int32_t nag = s.z, a2 = s.w;
        int32_t agn = -2, a2n = -2;
        float g1 = 0.0f, g2 = 0.0f;
        if (stn) {
          const int4 sn = stn[cc];
          agn = sn.z;
          a2n = sn.w;
          g1 = g1n[cc];
          g2 = g2n[cc];
        }
        const uint8_t fl = fl_in[cc];
        const int sc = (fl >> 1) & 1, sp = fl & 1;
        float acc1 = 0.0f, acc2 = 0.0f;
        for (int32_t e0 = r0; e0 < r1; e0 += GROUP_STEPS * f) {
          int32_t col[GROUP_STEPS];
          float we[GROUP_STEPS];
          uint32_t sw[GROUP_STEPS];
#pragma unroll
          for (int u = 0; u < GROUP_STEPS; ++u) {              // (past the end: the last edge again, unused)
            const int32_t e = min(e0 + u * f, r1 - 1);
            col[u] = a.col_idx[e];
            we[u] = w[e];
            sw[u] = sg[e >> 5];
          }
#pragma unroll
          for (int u = 0; u < GROUP_STEPS; ++u) {
            const int32_t e = e0 + u * f;
            if (e >= r1) break;
            const float gq = e == agn ? g1 : (e == a2n ? g2 : 0.0f);
            const float gm = gL[col[u]] - gq;
            const int se = (int)((sw[u] >> (e & 31)) & 1u);
            const float sigma = (sc ^ sp ^ se) ? -1.0f : 1.0f;
            const float mu = e == nag ? n2 : n1;
            const bool on = mu < WBP_BIG * 0.5f;           // (an empty minimum carries no gradient)
            if constexpr (ROWS) row[e] = on ? gm * sigma * mu : 0.0f;
            else if (on) atomicAdd(&row[e], gm * sigma * mu);
            const float ce = on ? gm * we[u] * sigma : 0.0f;
            if (e == nag) acc2 += ce; else acc1 += ce;
          }
        }
        for (int x = 1; x < f; x <<= 1) {
          acc1 += __shfl_xor(acc1, x, 64);
          acc2 += __shfl_xor(acc2, x, 64);
        }
        if (c >= 0 && sub == 0) {
          float o1 = 0.0f, o2 = 0.0f;
          if (nag >= 0) o1 = ((sg[nag >> 5] >> (nag & 31)) & 1u) ? -acc1 : acc1;
          if (a2 >= 0) o2 = ((sg[a2 >> 5] >> (a2 & 31)) & 1u) ? -acc2 : acc2;
          g1n[c] = o1;
          g2n[c] = o2;
        }
      }
      stn = st;
      __syncthreads();
    }
  }
}

// Weights in the order of the forward pass's column records (a grid has at most
// 65535 rows of blocks, and there may be more iterations).
__global__ void __launch_bounds__(256) k_wbp_weights(const float* __restrict__ w, int64_t E, int T, const int2* __restrict__ vce,
                                                     int64_t n, float* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int32_t e = vce[i].y;
  for (int64_t t = blockIdx.y; t < T; t += gridDim.y) out[t * n + i] = e < 0 ? 0.0f : w[t * E + e];
}

// gw[i] += sum over shots of rows[shot][i]; blockIdx.y takes every gridDim.y-th
// run of SUM_RUN shots (runs, then the runs' sums: a few hundred terms never meet
// one accumulator).  The addition is atomic whatever the grid: the gradient is the
// caller's, and calls on other streams or DEM handles may be adding to it.
constexpr int SUM_RUN = 8;
__global__ void __launch_bounds__(256) k_wbp_sum(const float* __restrict__ rows, int64_t TE, int64_t nshots,
                                                 float* gw) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= TE) return;
  float tot = 0.0f;
  for (int64_t s0 = (int64_t)blockIdx.y * SUM_RUN; s0 < nshots; s0 += (int64_t)gridDim.y * SUM_RUN) {
    float x[SUM_RUN];
#pragma unroll
    for (int k = 0; k < SUM_RUN; ++k) x[k] = s0 + k < nshots ? rows[(s0 + k) * TE + i] : 0.0f;
    tot += ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
  }
  atomicAdd(&gw[i], tot);
}

__global__ void k_wbp_transpose(const uint64_t* __restrict__ det, int32_t m, int64_t stride, int64_t nshots,
                                int32_t mw, uint64_t* __restrict__ synd) {
  __shared__ uint64_t tile[64];
  const int lane = threadIdx.x;
  const int64_t w = blockIdx.x;
  const int rt = blockIdx.y;
  const int row = rt * 64 + lane;
  tile[lane] = row < m ? det[(int64_t)row * stride + w] : 0ull;
  __syncthreads();
  uint64_t out = 0ull;
  for (int i = 0; i < 64; ++i) out |= ((tile[i] >> lane) & 1ull) << i;
  const int64_t s = w * 64 + lane;
  if (s < nshots) synd[s * mw + rt] = out;
}

template <typename T>
tmcs_status upload(T** dst, const std::vector<T>& v) {
  const size_t bytes = std::max<size_t>(v.size(), 1) * sizeof(T);
  if (hipMalloc((void**)dst, bytes) != hipSuccess) return fail(TMCS_ENOMEM, "hipMalloc failed (wbp)");
  if (!v.empty() && hipMemcpy(*dst, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice) != hipSuccess)
    return fail(TMCS_EDEVICE, "hipMemcpy failed (wbp)");
  return TMCS_OK;
}

// The training kernels keep their own device copy of the graph (separate
// from the decoder's) in a static map keyed by the DEM handle.
struct Registry {
  std::mutex mu;
  std::vector<std::pair<const Dem*, WbpDevice*>> items;
};
Registry g_reg;

tmcs_status ensure(const Dem& D, WbpDevice** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return fail(TMCS_EDEVICE, "no HIP device");
  std::lock_guard<std::mutex> lock(g_reg.mu);
  for (auto& it : g_reg.items)
    if (it.first == &D && it.second->device == dev) { *out = it.second; return TMCS_OK; }
  WbpDevice* d = new WbpDevice();
  d->device = dev;
  std::vector<float> lam(D.cols);
  for (int j = 0; j < D.cols; ++j) lam[j] = (float)std::log((1.0 - D.priors[j]) / D.priors[j]);
  std::vector<int32_t> csc_row(D.row_idx.begin(), D.row_idx.end());
  tmcs_status st;
  if ((st = upload(&d->row_ptr, D.row_ptr)) != TMCS_OK || (st = upload(&d->col_idx, D.col_idx)) != TMCS_OK ||
      (st = upload(&d->col_ptr, D.col_ptr)) != TMCS_OK || (st = upload(&d->csc_row, csc_row)) != TMCS_OK ||
      (st = upload(&d->csc_edge, D.csc_edge)) != TMCS_OK || (st = upload(&d->lam, lam)) != TMCS_OK)
    return st;
  // groups: checks with edges by lanes per check, then size
  std::vector<std::vector<int>> by_f(7);
  for (int c = 0; c < D.rows; ++c) {
    const int deg = D.row_ptr[c + 1] - D.row_ptr[c];
    int s = 0;
    while (s < 6 && ((deg + (1 << s) - 1) >> s) > GROUP_STEPS) ++s;
    by_f[s].push_back(c);                              // (checks without edges too: their state is written)
  }
  std::vector<int32_t> gchk, gf;
  for (int s = 0; s <= 6; ++s) {
    auto& items = by_f[s];
    std::stable_sort(items.begin(), items.end(), [&](int x, int y) {
      return D.row_ptr[x + 1] - D.row_ptr[x] < D.row_ptr[y + 1] - D.row_ptr[y];
    });
    const size_t per = 64u >> s;
    for (size_t i = 0; i < items.size(); i += per) {
      gf.push_back(1 << s);
      for (int l = 0; l < 64; ++l) {
        const size_t k = i + (size_t)(l >> s);
        gchk.push_back(k < items.size() ? items[k] : -1);
      }
    }
  }
  d->ngroups = (int32_t)gf.size();
  // columns by degree, 64 to a chunk
  std::vector<int> order(D.cols);
  for (int v = 0; v < D.cols; ++v) order[v] = v;
  auto cdeg = [&](int v) { return D.col_ptr[v + 1] - D.col_ptr[v]; };
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return cdeg(x) < cdeg(y); });
  std::vector<int32_t> vcol, vrow(1, 0);
  std::vector<int2> vce;
  for (size_t i = 0; i < order.size(); i += 64) {
    int K = 0;
    for (size_t j = i; j < std::min(order.size(), i + 64); ++j) K = std::max(K, (int)cdeg(order[j]));
    for (size_t j = i; j < i + 64; ++j) vcol.push_back(j < order.size() ? order[j] : -1);
    for (int k = 0; k < K; ++k)
      for (size_t j = i; j < i + 64; ++j) {
        const bool has = j < order.size() && k < cdeg(order[j]);
        const int32_t q = has ? D.col_ptr[order[j]] + k : 0;
        vce.push_back(has ? make_int2(D.row_idx[q], D.csc_edge[q]) : make_int2(0, -1));
      }
    vrow.push_back(vrow.back() + K);
  }
  d->nvchunks = (int32_t)(vcol.size() / 64);
  d->vrows = vrow.back();
  if ((st = upload(&d->gchk, gchk)) != TMCS_OK || (st = upload(&d->gf, gf)) != TMCS_OK ||
      (st = upload(&d->vcol, vcol)) != TMCS_OK || (st = upload(&d->vrow, vrow)) != TMCS_OK ||
      (st = upload(&d->vce, vce)) != TMCS_OK ||
      (st = hip_check(hipEventCreateWithFlags(&d->last, hipEventDisableTiming | hipEventDisableSystemFence), "hipEventCreate")) != TMCS_OK)
    return st;
  g_reg.items.push_back({&D, d});
  *out = d;
  return TMCS_OK;
}

// A call's turn at the handle's scratch (syndromes, laid-out weights, gradient
// rows, slabs).  Calls may come from several threads and on several streams: each
// one's kernels wait for those of the call before it, which costs an event per
// call (2.6 us; with a system-scope fence, which only other devices and the host
// need, 3.5).  A call that is being captured takes no turn, since its kernels run at
// every replay, whatever else then does; it uses neither the laid-out weights nor
// the rows (COL, ROWS), so replays only share what a forward pass always shared,
// its syndromes (512 shots of the BB [[144,12,12]] teleportation, T = 20, ms: forward
// 2.07 instead of 1.80, backward 4.35 instead of 2.20).
struct Turn {
  WbpDevice* d;
  hipStream_t stream;
  std::lock_guard<std::mutex> lock;
  bool captured;
  tmcs_status st = TMCS_OK;
  Turn(WbpDevice* d, hipStream_t stream) : d(d), stream(stream), lock(d->mu), captured(stream_capturing(stream)) {
    if (!captured) st = hip_check(hipStreamWaitEvent(stream, d->last, 0), "wait for the last call on this DEM");
  }
  // Also after an error: kernels of the call may be on their way.
  ~Turn() {
    if (!captured) (void)hipEventRecord(d->last, stream);
  }
};

// Device copy and arguments; the forward pass also needs the syndromes by shot.
tmcs_status prepare(const Dem& D, int T, const uint64_t* det, uint64_t n_shots, WbpDevice* d, WbpArgs* a,
                    hipStream_t stream, bool forward) {
  const int mw = std::max((D.rows + 63) / 64, 1);
  if (forward) {
    const size_t need = (size_t)n_shots * mw;
    if (d->cap_synd < need) {
      hipFree(d->synd);
      d->synd = nullptr;
      d->cap_synd = 0;
      if (hipMalloc((void**)&d->synd, need * sizeof(uint64_t)) != hipSuccess) return fail(TMCS_ENOMEM, "hipMalloc (wbp syndromes)");
      d->cap_synd = need;
    }
    const int64_t stride = (int64_t)((n_shots + 63) / 64);
    TMCS_LAUNCH("k_wbp_transpose", k_wbp_transpose, dim3((unsigned)stride, (unsigned)mw), dim3(64), 0, stream, det,
                D.rows, stride, (int64_t)n_shots, mw, d->synd);
  }
  WbpArgs& A = *a;
  A.row_ptr = d->row_ptr; A.col_idx = d->col_idx; A.col_ptr = d->col_ptr; A.csc_row = d->csc_row;
  A.csc_edge = d->csc_edge; A.lam = d->lam; A.synd = d->synd; A.mw = mw;
  A.gchk = d->gchk; A.gf = d->gf; A.ngroups = d->ngroups;
  A.vcol = d->vcol; A.vrow = d->vrow; A.vce = d->vce; A.nvchunks = d->nvchunks; A.vrows = d->vrows;
  A.m = D.rows; A.n = D.cols; A.T = T; A.E = D.edges; A.nshots = (int64_t)n_shots;
  A.shot0 = 0; A.shot1 = (int64_t)n_shots;
  A.lay = layout(D, T);
  return TMCS_OK;
}

// per-workgroup device-memory slabs of `bytes` each for the GS variants
tmcs_status slabs(WbpDevice* d, int grid, size_t bytes, WbpArgs* a) {
  const size_t slab = (bytes + 255) & ~(size_t)255;
  const size_t need = slab * (size_t)grid;
  if (d->cap_gstate < need) {
    hipFree(d->gstate);
    d->gstate = nullptr;
    d->cap_gstate = 0;
    if (hipMalloc((void**)&d->gstate, need) != hipSuccess) return fail(TMCS_ENOMEM, "hipMalloc (wbp state)");
    d->cap_gstate = need;
  }
  a->gstate = d->gstate;
  a->slab = (int64_t)slab;
  return TMCS_OK;
}

// Threads of a workgroup: enough that a pass over the edges is a few dozen steps,
// and every CU full where its LDS holds only one or two workgroups.
int threads_for(const Dem& D) {
  const int64_t t = (D.edges / 32 + 63) / 64 * 64;
  return (int)std::min<int64_t>(1024, std::max<int64_t>(64, t));
}

int grid_for(uint64_t n_shots, int threads) {
  int dev = 0, cus = 0;
  hipGetDevice(&dev);
  hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  return (int)std::max<int64_t>(1, std::min<int64_t>((int64_t)n_shots, (int64_t)std::max(cus, 1) * (2048 / threads)));
}

}  // namespace

void wbp_set_global_state(bool on) { g_force_gs = on; }

size_t wbp_workspace_bytes(const Dem& d, int T, uint64_t n_shots) {
  return (size_t)layout(d, T).shot * (size_t)n_shots;
}

tmcs_status wbp_forward_run(const Dem& D, const float* w, int T, const uint64_t* det, uint64_t n_shots, float* llr,
                            void* ws, size_t ws_bytes, hipStream_t stream) {
  if (n_shots == 0) return TMCS_OK;
  if (!det || !llr || !ws) return fail(TMCS_EINVAL, "null buffer");
  if (ws_bytes < wbp_workspace_bytes(D, T, n_shots)) return fail(TMCS_EINVAL, "workspace too small");
  WbpDevice* d = nullptr;
  WbpArgs a{};
  tmcs_status st = ensure(D, &d);
  if (st != TMCS_OK) return st;
  const Turn turn(d, stream);
  if ((st = turn.st) != TMCS_OK || (st = prepare(D, T, det, n_shots, d, &a, stream, true)) != TMCS_OK) return st;
  a.w = w; a.llr = llr; a.ws = (unsigned char*)ws;
  const int64_t nwc = (int64_t)T * d->vrows * 64;
  bool col = !turn.captured;
  if (col && d->cap_wcol < (size_t)nwc) {
    hipFree(d->wcol);
    d->wcol = nullptr;
    d->cap_wcol = 0;
    col = hipMalloc((void**)&d->wcol, (size_t)nwc * sizeof(float)) == hipSuccess;   // (no room: by edge)
    if (col) d->cap_wcol = (size_t)nwc;
    else { (void)hipGetLastError(); d->wcol = nullptr; }
  }
  a.wcol = d->wcol;
  if (col && nwc)
    TMCS_LAUNCH("k_wbp_weights", k_wbp_weights, dim3((unsigned)((d->vrows * 64 + 255) / 256), (unsigned)std::min(T, 65535)), dim3(256), 0, stream,
                w, D.edges, T, d->vce, (int64_t)d->vrows * 64, d->wcol);
  const int64_t nwords = (D.edges + 31) / 32;
  const size_t lds = (size_t)D.cols * 4 + (size_t)D.rows * 13 + (size_t)nwords * 4 + 16;
  const int threads = threads_for(D);
  const int grid = grid_for(n_shots, threads);
  if (g_force_gs || lds > 160 * 1024) {
    if ((st = slabs(d, grid, lds, &a)) != TMCS_OK) return st;
    auto k = col ? k_wbp_forward<true, true> : k_wbp_forward<true, false>;
    TMCS_LAUNCH("k_wbp_forward", k, dim3(grid), dim3(threads), 0, stream, a);
    return hip_check(hipGetLastError(), "k_wbp_forward launch");
  }
  auto k = col ? k_wbp_forward<false, true> : k_wbp_forward<false, false>;
  if (lds > 64 * 1024 && hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return fail(TMCS_EUNSUPPORTED, "weighted BP state does not fit in LDS");
  TMCS_LAUNCH("k_wbp_forward", k, dim3(grid), dim3(threads), lds, stream, a);
  return hip_check(hipGetLastError(), "k_wbp_forward launch");
}

tmcs_status wbp_backward_run(const Dem& D, const float* w, int T, const uint64_t* det, uint64_t n_shots,
                             const float* gllr, float* gw, const void* ws, size_t ws_bytes, hipStream_t stream) {
  if (n_shots == 0) return TMCS_OK;
  if (!det || !ws) return fail(TMCS_EINVAL, "null buffer");
  if (ws_bytes < wbp_workspace_bytes(D, T, n_shots)) return fail(TMCS_EINVAL, "workspace too small");
  WbpDevice* d = nullptr;
  WbpArgs a{};
  tmcs_status st = ensure(D, &d);
  if (st != TMCS_OK) return st;
  const int64_t TE = (int64_t)T * D.edges;
  if (TE == 0) return TMCS_OK;
  const Turn turn(d, stream);
  if ((st = turn.st) != TMCS_OK || (st = prepare(D, T, det, n_shots, d, &a, stream, false)) != TMCS_OK) return st;
  a.w = w; a.gllr = gllr; a.gw = gw; a.ws = (unsigned char*)ws;
  // rounds of shots whose rows fit ROWS_MAX, or what the device has left; no rows at
  // all where not even one shot's do
  int64_t round = turn.captured ? 0 : std::min<int64_t>((int64_t)n_shots, (int64_t)(d->most_rows / (size_t)TE));
  if (round > 0 && d->cap_rows < (size_t)(round * TE)) {
    hipFree(d->rows);
    d->rows = nullptr;
    d->cap_rows = 0;
    const size_t got = alloc_most((size_t)round, 1, [&](size_t shots) {
      if (hipMalloc((void**)&d->rows, shots * (size_t)TE * sizeof(float)) == hipSuccess) return true;
      (void)hipGetLastError();
      d->rows = nullptr;
      return false;
    });
    if (got < (size_t)round) d->most_rows = got * (size_t)TE;
    round = (int64_t)got;
    d->cap_rows = got * (size_t)TE;
  }
  const bool rows = round > 0;
  if (!rows) round = (int64_t)n_shots;
  a.rows = d->rows;
  const size_t lds = (size_t)D.cols * 4 + (size_t)D.rows * 8 + 16;
  const int threads = threads_for(D);
  const int grid = grid_for((uint64_t)round, threads);
  const bool gs = g_force_gs || lds > 160 * 1024;
  if (gs && (st = slabs(d, grid, lds, &a)) != TMCS_OK) return st;
  auto k = gs ? (rows ? k_wbp_backward<true, true> : k_wbp_backward<true, false>)
              : (rows ? k_wbp_backward<false, true> : k_wbp_backward<false, false>);
  if (!gs && lds > 64 * 1024 &&
      hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return fail(TMCS_EUNSUPPORTED, "weighted BP state does not fit in LDS");
  for (int64_t s0 = 0; s0 < (int64_t)n_shots; s0 += round) {
    a.shot0 = s0;
    a.shot1 = std::min<int64_t>((int64_t)n_shots, s0 + round);
    TMCS_LAUNCH("k_wbp_backward", k, dim3(grid), dim3(threads), gs ? 0 : lds, stream, a);
    if ((st = hip_check(hipGetLastError(), "k_wbp_backward launch")) != TMCS_OK) return st;
    if (!rows) continue;
    // small graphs: the shots are split too, so that the sum fills the GPU
    const int64_t bx = (TE + 255) / 256, runs = (a.shot1 - s0 + SUM_RUN - 1) / SUM_RUN;
    const int64_t by = std::max<int64_t>(1, std::min<int64_t>(runs, 2048 / std::max<int64_t>(bx, 1)));
    TMCS_LAUNCH("k_wbp_sum", k_wbp_sum, dim3((unsigned)bx, (unsigned)by), dim3(256), 0, stream, d->rows, TE, a.shot1 - s0, gw);
    if ((st = hip_check(hipGetLastError(), "k_wbp_sum launch")) != TMCS_OK) return st;
  }
  return TMCS_OK;
}

void wbp_release(const Dem& D) {
  std::lock_guard<std::mutex> lock(g_reg.mu);
  for (size_t i = 0; i < g_reg.items.size(); ++i) {
    if (g_reg.items[i].first != &D) continue;
    WbpDevice* d = g_reg.items[i].second;
    hipFree(d->row_ptr); hipFree(d->col_idx); hipFree(d->col_ptr); hipFree(d->csc_row); hipFree(d->csc_edge);
    hipFree(d->lam); hipFree(d->synd); hipFree(d->gstate); hipFree(d->gchk); hipFree(d->gf); hipFree(d->rows);
    hipFree(d->vcol); hipFree(d->vrow); hipFree(d->vce); hipFree(d->wcol);
    if (d->last) (void)hipEventDestroy(d->last);
    delete d;
    g_reg.items.erase(g_reg.items.begin() + i);
    --i;
  }
}

}  // namespace tmcs

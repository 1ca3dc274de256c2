// BP with the per-shot state in LDS (bp_chunk.hip): schedule, kernel arguments
// and launcher, used by the decoder's host side (decode.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "../host/internal.h"
#include "decoder.h"

namespace tmcs {
namespace dec {

// Device schedule of one DEM for teams of P lanes.
struct ChunkSched {
  int P = 0;
  bool wide = false;             // column addresses beyond 16 bits: one 32-bit check record per step
  int32_t Ms = 0, Ns = 0;        // check-part slots, column slots (multiples of 64)
  int32_t ntab = 0;              // words of tab
  int32_t vrows = 0, crows = 0;  // steps of all waves: rows of 64 weights per iteration
  int32_t noc = 0;               // columns that flip an observable
  uint32_t* vrec = nullptr;      // column-pass records
  uint32_t* crec = nullptr;      // check-pass records
  int32_t* tab = nullptr;        // per wave: where its streams and slots start, its runs
  float* lamp = nullptr;         // lambda_v by column slot
  int4* pinit = nullptr;         // {n1, n2, word, check} of iteration 1 by check-part slot
  int32_t* vmap = nullptr;       // [n] column -> slot (-1: a column without edges)
  int32_t* oslot = nullptr;      // [noc] slots of the columns that flip an observable
  uint64_t* omask = nullptr;     // [ow][noc] their masks
  int32_t* vedge = nullptr;      // [vrows][64] CSR edge of each column-pass step (-1: none)
  int32_t* cedge = nullptr;      // [crows][64] the same for the check pass
  size_t lds() const { return lds_state() + ((size_t)Ns + 1) * 4 + (size_t)ntab * 4; }
  size_t lds_state() const { return (((size_t)Ms + 1) * 12 + 15) & ~(size_t)15; }
};

struct ChunkArgs {
  const uint32_t* vrec;
  const uint32_t* crec;
  const int32_t* tab;
  const float* lamp;
  const int4* pinit;
  const int32_t* vmap;
  const int32_t* oslot;
  const uint64_t* omask;
  int32_t Ms, Ns, ntab, noc;
  int32_t n, ow, mw, T;
  float alpha;
  const float* wv;           // nullable [T][vrows][64]: weights by column-pass step
  const float* wc;           // [T][crows][64]: the same by check-pass step
  int64_t wv_stride, wc_stride;
  const float* lam;
  const uint64_t* synd;      // [chunk shots][mw] shot-major syndrome words
  const uint64_t* lone;      // nullable [mw]: checks without edges
  int64_t stride;            // words per row of pred
  int64_t shot0, nshots;
  const int32_t* queue;      // nullable: identity
  int32_t* counters;
  int32_t* osd_queue;
  float* osd_llr;            // [chunk][n]
  uint64_t* pred;            // [k][stride]
  tmcs_decode_stats* stats;  // [STAT_SHARDS]
  uint8_t* ehat;
  float* llr;
  int32_t* iters;
  uint8_t* flags;
  int32_t use_osd, nobs;
  uint64_t pm_lam[MAX_OW];   // observables flipped by the hard decision of lambda (a shot with s = 0)
  uint64_t pm_iso[MAX_OW];   // observables of the columns without edges whose lambda < 0
};

struct ChunkMulti {
  const ChunkArgs* tab;      // device [n]: the items' arguments
  int32_t n;
  int32_t* next;             // device job counter shared by the launch (zeroed before it)
};

// Rows of records (and weights) that prefetches read past the end of a stream.
constexpr int CHUNK_PAD_ROWS = 8;
// LDS bytes beyond the dynamic part (counters, histogram, job state).
constexpr size_t CHUNK_LDS_STATIC = 1024;

// Whether a team of P lanes on this DEM fits in a compute unit's LDS.  The run
// tables grow with the waves, so a DEM may fit for a few and not for sixteen.
// *lds: the team's bytes; *usual: the same with tables of the usual length, which
// is what the number of teams is chosen by before their size is known.
bool chunk_fits(const Dem& D, int P, size_t* lds, size_t* usual);
// TMCS_EUNSUPPORTED, without a message, where it does not fit.
tmcs_status build_chunk_sched(const Dem& D, int P, ChunkSched* out);
void free_chunk_sched(ChunkSched* s);
// Lays out CSR-ordered weights w [T][E] by schedule step into wv and wc.
tmcs_status launch_chunk_weights(const ChunkSched& s, const float* w, int T, int64_t E, float* wv, float* wc,
                                 hipStream_t stream);
// exact: messages by comparisons that also order NaN and infinities as the
// definition does (per-edge weights, extreme alpha).  mu.n > 0: a multi launch.
tmcs_status launch_bp_chunk(const ChunkArgs& a, const ChunkMulti& mu, bool exact, bool wide, int grid, int P, size_t lds,
                            hipStream_t stream);

}  // namespace dec
}  // namespace tmcs

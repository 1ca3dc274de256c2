// BP that streams a shot's state through LDS (bp_stream.hip): schedule, kernel
// arguments and launcher, used by the decoder's host side (decode.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "../host/internal.h"
#include "decoder.h"

namespace tmcs {
namespace dec {

constexpr int STREAM_LAMS = 64;             // entries of the lambda table (the last: +inf)
constexpr int STREAM_CAP_MIN = 2048, STREAM_CAP_MAX = 4096 + 64;   // checks the ring holds (one place is taken)
constexpr size_t STREAM_LDS_SHARED = 512;   // job state, counters, histogram

// Device schedule of one DEM for teams of P lanes (tiles of P checks).
struct StreamSched {
  int P = 0;
  int32_t NT = 0;                // tiles
  int32_t h = 0, R = 0;          // tiles a column may span to either side, tiles of the ring (2 h + 2)
  int32_t NL = 0, KL = 0;        // columns through memory and their largest degree
  int32_t cap = 0;               // ring capacity
  int32_t noc = 0;               // columns that flip an observable
  uint32_t* rec = nullptr;       // per wave: records of its chunks, tile after tile
  int32_t* desc = nullptr;       // [NT + 1][waves] steps of each kind
  int32_t* row0 = nullptr;       // [waves] first row of each wave's records
  int4* pinit = nullptr;         // [NT P] {n1, n2, word, check} of iteration 1 by slot
  float* lamtab = nullptr;       // [STREAM_LAMS]
  uint32_t* lrec = nullptr;      // [KL][NL] slot << 5 | position
  float* lamL = nullptr;         // [NL]
  uint2* vrec = nullptr;         // [n] the column's one or two messages, or {~0, its place among the NL}
  int32_t* ocol = nullptr;       // [noc] columns that flip an observable
  uint64_t* omask = nullptr;     // [ow][noc] their masks
  size_t lds() const { return (size_t)cap * 12 + STREAM_LAMS * 4 + STREAM_LDS_SHARED + ((size_t)NL + 1) * 4; }
  size_t buf_bytes() const { return ((size_t)NT * P * 12 + 12 + 255) & ~(size_t)255; }
  size_t team_bytes() const { return 2 * buf_bytes(); }
};

struct StreamArgs {
  const uint32_t* rec;
  const int32_t* desc;
  const int32_t* row0;
  const int4* pinit;
  const float* lamtab;
  const uint32_t* lrec;
  const float* lamL;
  const uint2* vrec;
  const int32_t* ocol;
  const uint64_t* omask;
  int32_t NT, h, R, NL, KL, noc;
  int32_t n, ow, mw, T;
  float alpha;
  unsigned char* state;      // [grid][2][buf]
  int64_t buf;               // bytes of one buffer
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

struct StreamMulti {
  const StreamArgs* tab;     // device [n]: the items' arguments
  int32_t n;
  int32_t* next;             // device job counter shared by the launch (zeroed before it)
};

// Builds the schedule; TMCS_EUNSUPPORTED where the DEM is not of this kind.
tmcs_status build_stream_sched(const Dem& D, int P, StreamSched* out);
void free_stream_sched(StreamSched* s);
// mu.n > 0: a multi launch.
tmcs_status launch_bp_stream(const StreamArgs& a, const StreamMulti& mu, int cap, int grid, int P, size_t lds, hipStream_t stream);

}  // namespace dec
}  // namespace tmcs

// Device tables of the matching kernels (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/ds3.h"

namespace ds3 {

struct MatchConst {
  int max_iters;
  float lambda0, lambda_min, step_tol, ang_tol, range_tol;
  int radius;
  double q_min;
};

// One decoded direction: queries (another view's points in the reference camera) against a reference.
struct MatchDir {
  int64_t ref_off;  // pixel offset of the reference in the ray-image buffer
  int64_t qry_off;  // pixel offset of the queries in their arena
  int64_t out_off;  // offset of the per-query idx in the temporary idx buffer
  int32_t Hr, Wr, Hq, Wq;
};

// One side of the mutual check: pixels of `self`, forward matches into `other` and back.
struct MutualDir {
  int64_t fwd_off, bwd_off;  // offsets in the temporary idx buffer (self->other, other->self)
  int64_t out_off;           // offset of the final idx / valid outputs (write_out only)
  const float* conf_self;    // confidences of self (pixel 0), written by the ray-image pass
  const float* conf_other;   // confidences of other (pixel 0)
  int32_t H_self, W_self, H_other, W_other;
  int32_t count_slot;        // 2 edge (pixels of i) or 2 edge + 1 (pixels of j)
  int32_t write_out;         // 1 for the j side of an edge
  int64_t part_off;          // first per-tile count of this side in the count partials
};

// Blocks are dealt to 8 bins (block b -> bin b mod 8, which the dispatcher places on XCD b mod 8). The entries' items
// are laid end to end, and bin x takes the run [x * per_bin, (x + 1) * per_bin) of them: the bins are even for any sizes,
// and what shares data is kept on one XCD by the order of the entries.
struct ItemMap {
  const int32_t* prefix;  // per entry: its first item; [n] = total
  int n, total, per_bin;
};

// One or two directions whose tables are kernel arguments.
struct MatchOne {
  const float* rays;
  const float* range;
  const void* qry;
  int32_t* idx;
  float* p;        // may be NULL
  int32_t* iters;  // may be NULL
  int32_t Hr, Wr, Hq, Wq;
};
struct MatchFew {
  MatchOne d[2];
  unsigned blocks0;  // blocks of d[0], filled by the launcher
};

struct MutualPair {
  MutualDir d[2];
  int tiles0;
};

// A side's partial counts and pixels.
struct NuSide {
  int64_t first;
  int64_t npx;
  int32_t n_parts;
  int32_t pad;
};

inline bool match_big(int H, int W) { return int64_t(H) * W > (int64_t(1) << 24); }

int launch_raymap(const void* arena, int64_t n0, const void* arena1, int64_t n1, ds3_dtype dt, float* rays, float* range,
                  float* conf, hipStream_t s);
int launch_match_few(MatchFew F, int n_dirs, ds3_dtype dt, const MatchConst& P, hipStream_t s);
// LM step counting of the batched launch: per-block sums spread over kStepStripes counters, 128 B apart.
constexpr int kStepStripes = 256;
constexpr int kStripeStride = 32;
// step_stripes may be NULL (no counting); it must start at zero.
// Query tiles of the batched matching: kMatchTile x kMatchTile pixels.
constexpr int kMatchTile = 16;
constexpr int kStripRows = 4;  // a wave's 16x4 queries
constexpr int kMatchStrips = kMatchTile / kStripRows;
inline int32_t match_strips(int H, int W) {
  return int32_t(kMatchStrips * ((H + kMatchTile - 1) / kMatchTile) * ((W + kMatchTile - 1) / kMatchTile));
}
// Strips per block of a call with this many: one while the card's 8192 waves are not filled twice over, up to eight (the
// lookup of a block's direction is then spread over two tiles).
inline int match_per(int64_t strips) { return int(strips < 32768 ? 1 : strips < 131072 ? strips / 16384 : 8); }
// per: strips per block; big: some reference has match_big pixels.
int launch_match_batched(const float* rays, const float* range, const void* cross, ds3_dtype dt, bool big,
                         const MatchDir* dirs, const ItemMap& map, int per, const MatchConst& P, int32_t* idx_tmp,
                         unsigned* step_stripes, hipStream_t s);
int launch_sum_stripes(const unsigned* step_stripes, unsigned long long* out, hipStream_t s);
// per: runs of kMutualPx pixels per block.
int launch_mutual(const MutualDir* md, const ItemMap& map, int per, const MatchConst& P, const int32_t* idx_tmp,
                  int32_t* idx_final, uint8_t* valid, unsigned* part, hipStream_t s);
int launch_mutual_pair(const MutualPair& M, int tiles, const MatchConst& P, const int32_t* idx_tmp, int32_t* idx_final,
                       uint8_t* valid, unsigned* part, hipStream_t s);
// The mutual check goes by runs of this many pixels (four per thread of a block).
constexpr int kMutualPx = 1024;
inline int32_t mutual_runs(int H, int W) { return int32_t((int64_t(H) * W + kMutualPx - 1) / kMutualPx); }
// Runs per block of a call with this many in all: one while the card's 2048 blocks are not filled twice over.
inline int mutual_per(int64_t runs) { return int(runs < 8192 ? 1 : runs < 32768 ? runs / 4096 : 8); }

// nu and admission from the per-tile partials; sides[2 e] = pixels of i, sides[2 e + 1] = pixels of j.
int launch_nu(const unsigned* part, const NuSide* sides, int n_edges, double nu_min, float* nu, int32_t* admit,
              hipStream_t s);
int launch_nu_pair(const unsigned* part, const NuSide& i, const NuSide& j, double nu_min, float* nu, int32_t* admit,
                   hipStream_t s);

}  // namespace ds3

// Host-side launch interface of the general (CSR / any dense) row passes.
#pragma once

#include "aa_common.hpp"
#include "aa_dense.hpp"

namespace aa {

// What leaves a block of a gradient pass for a column without a slot in its LDS table: records of two
// words (column, term) when one vector is updated, of three (column, term for w, term for phi) when both
// are.  The first kRecords* of a block stay in its LDS and go to the bins at the end.  Those that find no room
// there, or their bin full ("late" ones), are written out as they come and in the end sorted by bin, in pieces of at most
// kSort* (what LDS holds), and go to the bins, too, if the block's share of those has room for all of its records; those of
// other blocks, and what finds no room there, stay in their piece.  The first pieces of all blocks lie side by side,
// then the second ones.
constexpr int kRecordsTwoVec = 5120, kRecordsTwoVecDense = 2048, kRecordsOneVec = 4096;
constexpr int kSortOneVec = 16384, kSortTwoVec = 12288;

// Columns from `head` on are dealt to nb bins (a power of two, 0: no binning) in groups of
// 2^group_log2: group g = (col - head) >> group_log2 goes to bin (g + kBinTurn (g / nb)) % nb, where it is group
// g / nb; a bin spans `cols` columns in all.  (Every deal of nb groups starts kBinTurn bins further: without that
// the frequent columns of fields padded to 1024 or 512 columns all lay in one bin or two.  Whole step over 65,536
// rows of 80 such fields 113 and 94 us, now 72; 1000 columns a field 71.)  A group is 16
// columns (one 64-byte line of a model vector) when there are many columns, so that the
// owners read and write the model in whole lines; with fewer columns that traffic is small
// beside the records', and groups of 4 spread a run of frequent neighbouring columns (the
// head of a vocabulary, say) over four times as many bins -- the bin with the most records
// sets the update kernel's time.
// A bin has room for `segments` segments of `seg_cap` records -- block b of the pass takes segment b % segments -- all bins
// for `share` records a block, and a block for `pieces` pieces of `piece` late ones (multiples of four).  A block reserves its places in
// a bin with an atomic, and 256 blocks that add to one address wait for each other.  The owner's waves read a segment
// each.  Epoch of four pools of 65,536 rows over 2^20 columns, one segment / eight: 228 / 220 us; update over 23,000
// sentence pairs 21.9 / 19.9 us a pass.
struct BinPlan {
  int32_t nb, nb_log2, cols, segments, seg_cap, share, piece, pieces, group_log2;
};
constexpr int kMaxBins = 256, kBinSegments = 8;
constexpr int kBinTurn = 157;  // (odd, and near 0.618 of 256: few deals are multiples of few bins)
constexpr int kBinGroupLog2 = 4, kBinFineGroupLog2 = 2;
constexpr int64_t kBinFineColsMax = 1 << 18;  // groups of 4 up to this many binned columns
constexpr int kBinColsMax = 8192;  // LDS floats of a bin's owner in the update kernel
// The workspace has room for 48 records of 16 bytes a candidate, at least 65,536 and at most 2^27 (2 GiB).
constexpr size_t kRecordBytes = 16, kLateRecordBytes = 14;
inline size_t general_record_capacity(int32_t count_max) {
  const size_t want = 48 * (size_t)(count_max > 0 ? count_max : 0);
  return want < 65536 ? 65536 : (want > ((size_t)1 << 27) ? ((size_t)1 << 27) : want);
}
// Bytes of it for the runs, a word for each bin, piece and block: two a record are enough for few candidates (64 bytes a
// candidate where a block has 16 rows), from 2913 on all pieces of all blocks are fewer: at most one for kSortTwoVec
// records of 12 bytes and one more a block.
inline size_t general_run_bytes(int32_t count_max) {
  const size_t cap = general_record_capacity(count_max), few = (kRecordBytes - kLateRecordBytes) * cap;
  const size_t pieces = kRecordBytes * cap / (12 * (size_t)kSortTwoVec) + 256, need = (pieces * 256 * 4 + 255) & ~(size_t)255;
  return few < need ? few : need;
}
// floats of the per-block sums of the first columns; a pass uses 256 * head * nvec of them, the records begin behind those
inline size_t general_part_floats(int32_t d) {
  const size_t per_block = 2 * (size_t)d < 16384 ? 2 * (size_t)d : 16384;
  return 256 * per_block;
}
// Bytes for the records of a pass (with 10.5 MB of the sums' and the runs' 17 at most: less than 2^31).
inline int64_t general_record_bytes(int32_t d, int32_t head, int nvec, int32_t count_max) {
  return (int64_t)(general_record_capacity(count_max) * kRecordBytes - general_run_bytes(count_max) +
                   (general_part_floats(d) - 256 * (size_t)head * nvec) * sizeof(float));
}
// Of 14 bytes a record -- 84 records a candidate of a pass over one vector, 56 over two -- the bins take one and a quarter
// times what the blocks' LDS holds, but at most seven eighths (late room is a block's own: with smaller bins the blocks that
// finish last would find all of them full); the rest is late room, for late records and those that find their bin full, and
// what finds none there goes to the accumulators.  (Late records pass through it: 200,000 rows of 75 uniform columns 166 us,
// with a quarter of all room in the bins, and less late room, 211.)  What the runs and the first columns' sums leave
// free is the bins', too: about 11 records a candidate (7) and a million.
inline BinPlan general_bin_plan(int32_t d, int32_t head, int nvec, int32_t count_max, int32_t nblk) {
  BinPlan p{0, 0, 0, 0, 0, 0, 0, 0, kBinGroupLog2};
  const int gl = (int64_t)d - head <= kBinFineColsMax ? kBinFineGroupLog2 : kBinGroupLog2;
  const int64_t group = (int64_t)1 << gl;
  const int64_t groups = ((int64_t)d - head + group - 1) / group;
  if (groups <= 0 || nvec < 1) return p;
  int nb = 1, lg = 0;
  while (nb * 2 <= kMaxBins && nb * 2 <= groups) {
    nb *= 2;
    ++lg;
  }
  const int64_t cols = group * ((groups + nb - 1) / nb);
  if (cols * nvec > kBinColsMax) return p;  // too many columns for the owners' LDS: atomics instead
  p.nb = nb;
  p.nb_log2 = lg;
  p.group_log2 = gl;
  p.cols = (int32_t)cols;
  const int rec = nvec == 2 ? 12 : 8;
  const int64_t all = general_record_capacity(count_max) * kLateRecordBytes / rec;
  const int64_t in_lds = (int64_t)nblk * (nvec == 2 ? kRecordsTwoVec : kRecordsOneVec);
  int64_t binned = in_lds + in_lds / 4 > 49152 ? in_lds + in_lds / 4 : 49152;
  // (segments where all that the blocks hold fits them one and a quarter times: with less room the blocks that finish last
  // would find their segment full)
  p.segments = nblk >= 8 * kBinSegments && binned <= all / 8 * 7 ? kBinSegments : 1;
  if (binned > all / 8 * 7) binned = all / 8 * 7;
  const int64_t late = all - binned, spare = general_record_bytes(d, head, nvec, count_max) / rec - all;
  binned += spare < late ? spare : late;
  p.seg_cap = (int32_t)(binned / ((int64_t)nb * p.segments)) & ~3;
  p.share = nb * p.segments * p.seg_cap / nblk;
  const int32_t each = (int32_t)(late / nblk), most = nvec == 2 ? kSortTwoVec : kSortOneVec;
  p.pieces = (each + most - 1) / most;
  p.piece = p.pieces > 0 ? (each / p.pieces) & ~3 : 0;
  return p;
}

// The header's flags of the bins of which the pieces still have records: the table ahead of the blocks' counts (a pointer
// of its own among the arguments costs k_rows_grad for hard thresholds, at 128 registers, two of them in memory).
__host__ __device__ inline int32_t *left_marks(int32_t *blk_late) { return blk_late - kMaxBins; }

struct GenArgs {
  // features
  const float *x;
  int64_t ld;
  int32_t d;
  const int64_t *rowptr;
  const int32_t *col;
  const float *val;
  const float *y;
  const int32_t *rows;
  int32_t count_max;
  const int32_t *m_dev;
  const float *w;
  const float *phi;
  const float *bias;
  const float *T;
  float gamma, one_minus_gamma;
  DrawKey key;
  int32_t do_keep;
  float *logit;
  float *prob;
  uint8_t *flags;
  float *loss_out;
  const float *loss_in;
  // (w[c], phi[c]) side by side for the columns past `head`, indexed by column: one gather
  // brings both values of a column that is not in LDS (written before the pass; element 0 is always
  // readable; NULL unless the pass updates both vectors)
  const float2 *wp;
  // atomic accumulators (zeroed before the pass); with bins, acc_used[bin] (zeroed too) is set
  // by whoever adds to a column of that bin
  double *acc_w;     // [d]
  double *acc_p;     // [d]
  int32_t *acc_used; // [kMaxBins]
  // per-block kept count and bias-gradient sum of a gradient pass (plain stores)
  int32_t *blk_cnt;  // [blocks of the pass]
  float *blk_gb;     // [blocks of the pass]
  // per-block sums of the first `head` columns: part[(block * nvec + vec) * head + column],
  // written whole by every block of a gradient pass (no clearing needed)
  float *part;
  int32_t head;
  // entries of the other columns leave a block as records (see BinPlan): recs[(bin * segments + segment) * seg_cap + i],
  // with the count in bin_fill[segment * kMaxBins + bin] (zeroed before the pass); behind the bins the late ones of block and piece p,
  // [(p * blocks + block) * piece + i], with a bin's run (start | count << 16) in
  // runs[(bin * pieces + p) * blocks + block] and the block's count in blk_late; left_marks(blk_late)[bin] (zeroed
  // before the pass) is set by whoever leaves some of the bin there
  int32_t *recs;
  int32_t *runs;
  unsigned *bin_fill;
  int32_t *blk_late;
  BinPlan plan;
  // optional device-side update counter (step size lr / sqrt(t)): block 0 of a gradient pass
  // copies it to *t_snap, which the update kernel reads (the counter itself changes there)
  const int32_t *t_upd;
  int32_t *t_snap;
};

// Columns whose gradient sums leave a block as plain stores instead of atomics, for a pass
// that updates nvec vectors over d columns; blocks of a gradient pass at most.
int32_t general_head_columns(int32_t d, int nvec, bool csr);
// Whether the update kernel can leave the workspace ready for the next pass (see ApplyArgs).
bool general_keeps_ready(int32_t d, int nvec, bool csr);
constexpr int kGeneralGradBlocks = 256;
// floats ahead of the accumulators: 16 scalars, tables of kMaxBins words: a flag per bin (left_marks), the blocks' counts of
// late records, another flag per bin (acc_used), the fill counts of the bins' segments (an even count in all: the
// accumulators behind it are doubles)
constexpr int kGeneralHeader = 16 + (3 + kBinSegments) * kMaxBins;
// floats the header and the two accumulators of d doubles take
inline size_t general_clear_floats(int32_t d) { return kGeneralHeader + 4 * (size_t)d; }

struct ApplyArgs {
  int32_t d;
  double *acc_w;
  double *acc_p;
  int32_t *acc_used;  // [bin] 0: the pass added nothing to the accumulators of the bin's columns
  // Leave the workspace as the next pass of the same call needs it, so that no preparing
  // launch has to run in between (bins only): every bin owner clears its fill count, its flags
  // and whatever it read from the accumulators, and with two updated vectors writes the new
  // (w[c], phi[c]) pairs of its columns.
  int32_t keep_ready;
  float2 *wp_out;     // pairs, indexed by column (NULL: none)
  const int32_t *blk_cnt;  // per-block kept counts and bias-gradient sums of the pass
  const float *blk_gb;
  const int32_t *m_dev;
  int32_t m_max;
  float *w;
  float *phi;
  float *bias;
  const float *part;  // per-block sums of the first `head` columns (see GenArgs)
  int32_t head, nvec, nblk_pass;
  const int32_t *recs;  // records of the other columns (see GenArgs)
  const int32_t *runs;
  unsigned *bin_fill;
  int32_t *blk_late;
  BinPlan plan;
  float lambda, lr, lr_a, l2_a;
  int32_t *t_upd;          // optional update counter: the Boss step size is lr / sqrt(updates so far)
  const int32_t *t_snap;   // its value before this step (written by the pass kernel)
  int32_t *kept_hist;
  const uint8_t *flags;
  int32_t P;
  const int32_t *idx;
  int32_t *kept_pos;
  int32_t *kept_ids;
  const float *loss_pool;
  float *loss;
  int32_t *kept_count;
};

int32_t general_pass_blocks(int32_t count, bool csr, int mode);
hipError_t launch_general_pass(const GenArgs &a, int mode, bool csr, int32_t nblk,
                               hipStream_t stream, hipEvent_t started = nullptr,
                               hipEvent_t stopped = nullptr);
hipError_t launch_zero_f32(float *p, size_t count, hipStream_t stream);
// Zeroes p[0, count) and writes wp[c] = (w[c], phi[c]) for head <= c < d (one launch).
hipError_t launch_prepare_general(float *p, size_t count, const float *w, const float *phi,
                                  float2 *wp, int32_t head, int32_t d, hipStream_t stream);
hipError_t launch_general_apply(const ApplyArgs &a, hipStream_t stream);

}  // namespace aa

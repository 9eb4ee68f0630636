// General row passes: CSR rows, and dense rows no other pass takes (fewer than 4
// or more than 8192 floats).  A group of GL lanes walks the
// stored entries of a row; phi and w are read through the caches (they are the
// only reused data; a gradient pass keeps their first entries in LDS); a second
// kernel folds the gradient sums into the model.
// Device-wide fp32 atomics are what such a pass must avoid on MI355X: about 20 G/s
// on scattered addresses, and adds to one address run one after the other, about
// 13 ns each, while bag-of-words data puts most entries on a few hot columns.  So:
//  * the first columns (frequency-ranked column ids, the usual layout of such data,
//    put the hot ones there) have a slot each in an LDS table of the block and leave
//    it as plain stores into a per-block array that the second kernel sums;
//  * any other column may claim one of a few thousand hashed LDS slots, first come
//    first served (a hot column outside the first ones -- a bias-like feature at the
//    end, the head of a second vocabulary -- comes early and keeps its slot);
//  * entries that find their slots taken, and in the end the hashed slots, become records
//    that are sorted by column bin: the block that owns a bin in the second kernel sums its
//    records in LDS.  A block's first records stay in LDS until it is done and go to the
//    bins' arrays (one integer atomic per block and bin reserves the space); the others
//    are written out as they come, those that find their bin full join them, and they are
//    sorted in pieces at the end;
//  * only what does not fit (records beyond a block's room, or more columns than the
//    bins can cover) is added to dense accumulators in HBM.
#include <type_traits>

#include "aa_compact.hpp"
#include "aa_general.hpp"

namespace aa {

namespace {

typedef float f4v __attribute__((ext_vector_type(4), aligned(4)));  // (any float address)
typedef int i4v __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned u2v __attribute__((ext_vector_type(2)));
typedef unsigned u3v __attribute__((ext_vector_type(3)));

// v moved by a DPP control.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

// Sum over aligned groups of WIDTH lanes, halves first.  For 16 lanes by rotations inside the row,
// no trip through LDS: after each addition the values repeat with half the period, so rotating
// by 8, 4, 2 and 1 adds the same pairs as exchanging with lane ^ 8, ^ 4, ^ 2 and ^ 1.
template <int WIDTH>
__device__ __forceinline__ float gsum(float v) {
  if (WIDTH == 16) {
    v = dpp_add<0x128>(v);  // row_ror:8
    v = dpp_add<0x124>(v);
    v = dpp_add<0x122>(v);
    return dpp_add<0x121>(v);
  }
#pragma unroll
  for (int off = WIDTH / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

// Per-block LDS: kDirect* slots for columns 0..kDirect*-1 (one sum per updated vector) and as
// many entries of the model vectors themselves, kHashed* slots with a column tag each, and a
// block's first kRecords* records.  About 150 KB: one block of 16 waves per compute unit.
// The sums are doubles: on MI355X `ds_add_f32` retires about one lane every three cycles,
// `ds_add_f64` three lanes a cycle (measured, scattered addresses), and the sums come out
// closer to exact.
constexpr int kDirectTwoVec = 3072, kHashedTwoVec = 1024;
constexpr int kDirectTwoVecDense = 4096, kHashedTwoVecDense = 1024;
constexpr int kDirectOneVec = 8192, kHashedOneVec = 2048;
constexpr int kGradThreads = 1024, kPoolThreads = 256;
constexpr int kClaimRows = 16;  // rows per wave from which a column of every row that lost its slot would show

__device__ __forceinline__ int bin_of(int c, int head, const BinPlan &p) {
  const int g = (c - head) >> p.group_log2;
  return (g + (int)__umul24((unsigned)g >> p.nb_log2, kBinTurn)) & (p.nb - 1);
}

// The set of two hashed slots a column may have.  A run of H neighbouring columns past the table fills the sets evenly;
// columns a power of two apart go to different sets, and which of them meet depends on the block.  (With
// c ^ c >> 11 the frequent columns of fields padded to 512 columns met in every block, four to a set: whole step over
// 65,536 rows of 80 such fields 245 us, now 72; fields of 1000 columns 68 and 70.)
template <int H>
__device__ __forceinline__ int hashed_set(int c, int factor) {
  constexpr int kLog2 = H == 2048 ? 10 : 9;
  static_assert(H == 2 << kLog2, "slots");
  return (int)((((unsigned)c << 5) + __umul24((unsigned)c >> kLog2, (unsigned)factor)) >> 5) & (H / 2 - 1);
}

// Adds one entry's terms to the dense accumulators in HBM (the path of last resort).  They
// are doubles like every other sum of entries: which entries end up here depends on timing,
// so their sum must not round before it meets the rest of the column's total.
template <bool SVM, bool ASSIST>
__device__ __forceinline__ void add_global(const GenArgs &a, int c, double ta, double tb) {
  // tells the owner of the column's bin to read its columns' accumulators at all (an entry
  // that goes this way must not make every owner read every accumulator)
  if (a.plan.nb > 0) a.acc_used[bin_of(c, a.head, a.plan)] = 1;
  if (SVM && ta != 0.0) unsafeAtomicAdd(a.acc_w + c, ta);
  if (ASSIST) {
    const double t = SVM ? tb : ta;
    if (t != 0.0) unsafeAtomicAdd(a.acc_p + c, t);
  }
}

// A gradient pass.  A group of GL lanes walks a row's entries twice: for the dot products, and with the
// row's coefficients for the sums.  One block of 16 waves per compute unit (LDS); nothing in the row loop
// makes the waves of a block wait for each other.
// What bounds it: on short rows over a wide vocabulary the instructions per entry (walk, LDS sums,
// records), on long sparse rows the gathers of columns that are not in LDS.  The records used to meet in
// an LDS buffer that the block looked at, and emptied, together every eight rows of a wave:
// 55 % of the wave cycles were waits.  Now those that the buffer has no room for go to memory as they
// come, and the block sorts all of them by bin once, at the end.
// The loop's code had about 96 vector instructions an entry, and a pass over 456,000 sentence pairs (25.8 M entries) issued
// 47.6 M for all it does, 58 % of its issue cycles.  Lane sets in scalar registers, one sum's address instead of two branches, no
// division a record, row extents clipped once a round and record stores without a branch leave 62, and 41.8 M, 55 %, with the
// waves waiting 38 instead of 50 % of their cycles: the update over 460,000 pairs 170.4 -> 157.1 us, an epoch of four
// pools of 65,536 rows over 2^20 columns 233.3 -> 228.3 (all of it together: which part gave how much was not measured).
// NEAR: every column is in the table; no tags, records and gathers.  Whole updates without / so, rows of 56 entries, one
// vector over 8000 columns: 1000 rows 14.9 / 11.7 us, 20,000 20.2 / 16.6, 300,000 49.4 / 35.2; both over 3000: 20,000 20.1 / 17.0,
// 300,000 57.2 / 46.9.
template <int GL, int MODE, bool CSR, bool NEAR>
__global__ __launch_bounds__(kGradThreads) void k_rows_grad(const GenArgs a) {
  static_assert(CSR || !NEAR, "dense rows choose turn by turn");
  constexpr bool POOL = (MODE & kPool) != 0;
  constexpr bool SVM = (MODE & kSvm) != 0;
  constexpr bool ASSIST = (MODE & kAssist) != 0;
  constexpr bool HARD = (MODE & kHard) != 0;  // keep by the row's own loss, no Assistant
  constexpr bool NEED_PHI = (POOL && !HARD) || ASSIST;
  constexpr int G = kWave / GL, kWaves = kGradThreads / kWave;
  constexpr int NVEC = (SVM ? 1 : 0) + (ASSIST ? 1 : 0);
  constexpr bool TWO = NVEC == 2;
  constexpr int D = TWO ? (CSR ? kDirectTwoVec : kDirectTwoVecDense) : kDirectOneVec;  // slots 0..D-1: column = slot
  constexpr int H = TWO ? (CSR ? kHashedTwoVec : kHashedTwoVecDense) : kHashedOneVec;  // hashed slots, two to a set
  constexpr int RW = TWO ? 3 : 2, C = TWO ? kSortTwoVec : kSortOneVec;
  constexpr int R = TWO ? (CSR ? kRecordsTwoVec : kRecordsTwoVecDense) : kRecordsOneVec;  // records held in LDS
  // LDS: the sums (slots, then hashed slots; per vector), the first D entries of the model, the hashed
  // slots' columns, the first records; at the end the same memory holds a piece of records being sorted
  constexpr int kSumBytes = 8 * NVEC * (D + H), kModelBytes = 4 * NVEC * D, kTagBytes = 4 * H;
  constexpr int kHeldBytes = 4 * RW * R, kSortBytes = 4 * RW * C;
  constexpr int kTableBytes = kSumBytes + kModelBytes + kTagBytes + kHeldBytes;
  __shared__ __attribute__((aligned(16))) char s_mem[kTableBytes > kSortBytes ? kTableBytes : kSortBytes];
  __shared__ __attribute__((aligned(16))) int s_hist[kMaxBins], s_base[kMaxBins];
  __shared__ int s_nrec[1], s_more, s_next;
  __shared__ int s_cnt[kWaves];
  __shared__ float s_gb[kWaves];
  int *const s_tag = reinterpret_cast<int *>(s_mem);  // (in front: an access's own offset has 16 bits)
  double *const s_sum = reinterpret_cast<double *>(s_mem + kTagBytes);  // [vector][D + H]
  float *const s_model = reinterpret_cast<float *>(s_mem + kTagBytes + kSumBytes);  // one vector: [D]; two: pairs
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int *const s_held = reinterpret_cast<int *>(s_mem + kSumBytes + kModelBytes + kTagBytes);
  const bool binned = a.plan.nb > 0;
  const int factor = (int)((0x9E3779B1u * (2 * blockIdx.x + 1)) >> 8 | 1u);  // (odd, 24 bits)
  const int grp = lane / GL, sub = lane % GL;

  int total = a.count_max;
  if (!POOL && a.m_dev) total = min(max(*a.m_dev, 0), a.count_max);
  const int nwaves = gridDim.x * kWaves, gwave = blockIdx.x * kWaves + wave;
  const int per = total / nwaves, rem = total % nwaves;
  const int lo = gwave * per + min(gwave, rem);
  const int hi = lo + per + (gwave < rem ? 1 : 0);

  // One row per lane, 64 rows per round: extent, label, draw, incoming loss.
  struct RowInfo {
    long long e0;
    int len;
    float y, u, lin;
  };
  auto row_id = [&](int round) {
    const int j_l = lo + round * kWave + lane;
    return j_l < hi && a.rows ? a.rows[j_l] : j_l;
  };
  auto load_rows = [&](int round, int row_l) {
    RowInfo r{0, 0, 0.f, 2.f, 0.f};
    const int j_l = lo + round * kWave + lane;
    if (j_l < hi) {
      if (CSR) {
        r.e0 = a.rowptr[row_l];
        r.len = (int)(a.rowptr[row_l + 1] - r.e0);
      } else {
        r.e0 = (long long)row_l * a.ld;
        r.len = a.d;
      }
      if (SVM) r.y = a.y[row_l];
      if (POOL && a.do_keep) r.u = keep_uniform(a.key, (uint32_t)j_l);
      if (ASSIST && !SVM) r.lin = a.loss_in[j_l];
    }
    return r;
  };
  RowInfo first_rows;
  {  // (the model's loads go out together, and the first rows' behind them)
    float mw[D / kGradThreads], mp[D / kGradThreads];
#pragma unroll
    for (int i = 0; i < D / kGradThreads; ++i) {
      const int k = min((int)threadIdx.x + i * kGradThreads, a.d - 1);
      if (SVM) mw[i] = a.w[k];
      if (ASSIST) mp[i] = a.phi[k];
    }
    int id = row_id(0);
    __builtin_amdgcn_sched_barrier(0);
    // (no more than the model has columns for: one vector of 3000, 8192 rows of 56 entries 15.4 -> 14.4 us)
    const int used = NEAR || a.d <= D ? a.d : D + H;
#pragma unroll
    for (int v = 0; v < NVEC; ++v)
      for (int k = threadIdx.x; k < used; k += kGradThreads) s_sum[v * (D + H) + k] = 0.0;
    for (int k = threadIdx.x; !NEAR && a.d > D && k < H; k += kGradThreads) s_tag[k] = -1;
    if (threadIdx.x == 0) s_nrec[0] = s_more = s_next = 0;
    __builtin_amdgcn_sched_barrier(0);
    first_rows = load_rows(0, id);
#pragma unroll
    for (int i = 0; i < D / kGradThreads; ++i) {
      const int k = threadIdx.x + i * kGradThreads;
      if (SVM) s_model[TWO ? 2 * k : k] = mw[i];
      if (ASSIST) s_model[TWO ? 2 * k + 1 : k] = mp[i];
    }
  }
  __syncthreads();
  if (a.t_upd && blockIdx.x == 0 && threadIdx.x == 0) *a.t_snap = *a.t_upd;

  const float b = (NEED_PHI && a.bias) ? *a.bias : 0.f;
  const float T = (ASSIST || HARD) ? *a.T : 0.f;
  float gb = 0.f;
  int kept = 0;
  const int held = binned ? R : 0, cap = held + (binned ? a.plan.pieces * a.plan.piece : 0);
  int32_t *const late = a.recs + (size_t)a.plan.nb * a.plan.segments * a.plan.seg_cap * RW;  // records that LDS has no room for
  auto piece_at = [&](int piece) { return late + ((size_t)piece * gridDim.x + blockIdx.x) * a.plan.piece * RW; };
  // Late records are stored through a buffer resource: a lane without one gives an offset out of range, and the store
  // needs no branch.  Loads and stores share one counter here: behind a store under a condition the wait for the next
  // unit's entries, requested before it, would be a wait for its acknowledgement, too.
  constexpr int kNone = (int)0x80000000;  // out of every resource's range
  const __amdgpu_buffer_rsrc_t r_late = __builtin_amdgcn_make_buffer_rsrc(late, 0, binned ? kNone : 0, 0x00020000);
  // the piece that the wave's last records went to: places from piece_lo to piece_hi, byte offset of place 0
  const int piece_len = a.plan.piece;
  int piece_lo = held, piece_hi = held, piece_off = 0;
  auto piece_of_place = [&](int place) { return (int)((unsigned)(place - held) / (unsigned)piece_len); };
  auto offset_of = [&](int piece) {
    return (int)((((unsigned)piece * gridDim.x + blockIdx.x - (unsigned)piece) * (unsigned)piece_len - (unsigned)held) * (4u * RW));
  };
  // Places for N records a lane, those of the lanes in want[k]; all lanes take part.  A block's first `held` records stay
  // in LDS until the end, the others go to where they will be sorted: off[k] is what their store is given.
  // (Lane sets are masks in scalar registers throughout: as booleans that cross a branch they are a vector register
  // and three instructions each.)
  auto place_records = [&](auto n_const, const uint64_t *want, const int *c, const float *ta, const float *tb, int *off)
                           __attribute__((always_inline)) {
    constexpr int N = decltype(n_const)::value;
    int count = 0;
#pragma unroll
    for (int k = 0; k < N; ++k) count += __popcll(want[k]);
#pragma unroll
    for (int k = 0; k < N; ++k) off[k] = kNone;
    if (count == 0) return;
    int first = 0;
    {
      int at = 0;
      asm volatile("" : "+v"(at));  // (one lane adds: nothing to combine)
      if (lane == 0) first = atomicAdd(s_nrec + at, count);
    }
    first = __builtin_amdgcn_readfirstlane(first);
    int pos[N];
#pragma unroll
    for (int k = 0, next = first; k < N; ++k) {
      pos[k] = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(want[k] >> 32),
                                              __builtin_amdgcn_mbcnt_lo((uint32_t)want[k], (uint32_t)next));
      next += __popcll(want[k]);
    }
    if (first >= piece_hi && first < cap) {  // (on to the piece that `first` lies in)
      const int piece = piece_of_place(first);
      piece_lo = held + piece * piece_len;
      piece_hi = min(piece_lo + piece_len, cap);
      piece_off = offset_of(piece);
    }
    if (first >= piece_lo && first + count <= piece_hi) {
#pragma unroll
      for (int k = 0; k < N; ++k) {
        const int o = pos[k] * (4 * RW) + piece_off;
        off[k] = __builtin_amdgcn_inverse_ballot_w64(want[k]) ? o : kNone;
      }
      return;
    }
    if (first + count <= held) {
#pragma unroll
      for (int k = 0; k < N; ++k) {
        if (__builtin_amdgcn_inverse_ballot_w64(want[k])) {
          s_held[pos[k] * RW] = c[k];
          s_held[pos[k] * RW + 1] = __float_as_int(ta[k]);
          if (TWO) s_held[pos[k] * RW + RW - 1] = __float_as_int(tb[k]);
        }
      }
      return;
    }
    // on both sides of a boundary, or beyond the block's room
    // (a lane's records lie in one piece or in it and the next: with several, one is longer than 64 N)
    static_assert(kSortTwoVec / 2 > 8 * kWave && kSortOneVec / 2 > 8 * kWave, "at most one boundary");
    const int piece = first < cap && max(first, held) < cap && cap > held ? piece_of_place(max(first, held)) : 0;
    const int ends = held + (piece + 1) * piece_len, off_here = offset_of(piece), off_next = offset_of(piece + 1);
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const bool mine = __builtin_amdgcn_inverse_ballot_w64(want[k]);
      if (mine && pos[k] < held) {
        s_held[pos[k] * RW] = c[k];
        s_held[pos[k] * RW + 1] = __float_as_int(ta[k]);
        if (TWO) s_held[pos[k] * RW + RW - 1] = __float_as_int(tb[k]);
      }
      if (mine && pos[k] >= held && pos[k] < cap) off[k] = pos[k] * (4 * RW) + (pos[k] < ends ? off_here : off_next);
    }
    if (first + count > cap) {
      // (one copy of what adds to the accumulators: copies behind every entry cost hundreds of scalar registers
      // parked in vector ones)
#pragma unroll 1
      for (int k = 0; k < N; ++k) {
        int ck = c[0];
        float tak = ta[0], tbk = tb[0];
        bool out = __builtin_amdgcn_inverse_ballot_w64(want[0]) && pos[0] >= cap;
#pragma unroll
        for (int i = 1; i < N; ++i) {
          ck = i == k ? c[i] : ck;
          tak = i == k ? ta[i] : tak;
          tbk = i == k ? tb[i] : tbk;
          out = i == k ? __builtin_amdgcn_inverse_ballot_w64(want[i]) && pos[i] >= cap : out;
        }
        if (out) add_global<SVM, ASSIST>(a, ck, tak, tbk);
      }
    }
  };
  auto store_records = [&](auto n_const, const int *c, const float *ta, const float *tb, const int *off)
                           __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < decltype(n_const)::value; ++k) {
      if constexpr (TWO)
        __builtin_amdgcn_raw_buffer_store_b96(u3v{(unsigned)c[k], __float_as_uint(ta[k]), __float_as_uint(tb[k])}, r_late,
                                              off[k], 0, 0);
      else
        __builtin_amdgcn_raw_buffer_store_b64(u2v{(unsigned)c[k], __float_as_uint(ta[k])}, r_late, off[k], 0, 0);
    }
  };
  auto append = [&](auto n_const, const uint64_t *want, const int *c, const float *ta, const float *tb)
                    __attribute__((always_inline)) {
    int off[decltype(n_const)::value];
    place_records(n_const, want, c, ta, tb, off);
    store_records(n_const, c, ta, tb, off);
  };

  // Entries are read through buffer resources: a lane with nothing to read gives an offset past the
  // resource's range, for which the hardware returns zero without a memory access.  No load of the row loop
  // sits behind a branch then, and the next unit's entries stay in flight while this one's gathers are waited for
  // (with exec-masked loads every wait was for everything in flight).
  constexpr long long kSpan = 0x7fffffffll / 4;  // entries within reach of a 32-bit byte offset
  const __amdgpu_buffer_rsrc_t r_col = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int32_t *>(CSR ? a.col : nullptr), 0, CSR ? kNone : 0, 0x00020000);
  // (the model past the table, where a 32-bit offset reaches all of it)
  constexpr int kColBytes = TWO ? 8 : 4;
  const bool reach = a.d <= (int)(0x7fffffffu / kColBytes);
  const void *const far_src = TWO ? (const void *)a.wp : (const void *)(ASSIST ? a.phi : a.w);
  const __amdgpu_buffer_rsrc_t r_far = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(far_src), 0,
                                                                       CSR && reach ? a.d * kColBytes : 0, 0x00020000);
  const __amdgpu_buffer_rsrc_t r_val = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float *>(CSR && a.val ? a.val : a.T), 0, CSR && a.val ? kNone : 0, 0x00020000);
  const int rows_max = per + (rem > 0 ? 1 : 0);
  const int rounds = (rows_max + kWave - 1) / kWave;
  for (int round = 0; round < rounds; ++round) {
    const int base = lo + round * kWave;
    const int cnt = max(0, min(kWave, hi - base));
    const RowInfo ri = round == 0 ? first_rows : load_rows(round, row_id(round));
    long long e0_l = ri.e0;
    int len_l = ri.len, src_l = lane;
    float y_l = ri.y, u_l = ri.u, lin_l = ri.lin;
    constexpr int kPiece = 4 * GL;  // entries of a row that its lanes read with one load
    // A unit, the work of a lane group at a time, is a row of up to two pieces and whatever follows (the first M
    // places), or two rows of one piece, which then share the chain of round trips (1,000,000 sentence pairs:
    // pass 151 us with a row at a time, 138 with two).
    int M = cnt;
    if constexpr (CSR) {
      const bool whole = lane < cnt && (len_l > kPiece || (len_l > 0 && (e0_l + len_l < 4 || e0_l + len_l > kSpan)));
      const unsigned long long m_whole = __ballot(whole), mine = whole ? m_whole : ~m_whole;
      M = __popcll(m_whole);
      const int first_short = M;
      // (few rows leave lane groups idle in pairs, and a unit without a second piece costs half: one update over 5000
      // sentence pairs 18.6 us paired, 17.8 not)
      if (cnt <= G) M = cnt;
      const int to = 4 * ((whole ? 0 : first_short) + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mine >> 32),
                                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)mine, 0u)));
      auto put = [&](int v) { return __builtin_amdgcn_ds_permute(to, v); };
      const int e_lo = put((int)(uint32_t)e0_l), e_hi = put((int)(e0_l >> 32));
      e0_l = ((long long)e_hi << 32) | (uint32_t)e_lo;
      len_l = put(len_l);
      src_l = put(lane);
      if (SVM) y_l = __int_as_float(put(__float_as_int(y_l)));
      if (POOL) u_l = __int_as_float(put(__float_as_int(u_l)));
      if (ASSIST && !SVM) lin_l = __int_as_float(put(__float_as_int(lin_l)));
    }
    const int units = M + (cnt - M + 1) / 2;  // (lanes without a row have the last places)
    const int iters = (units + G - 1) / G;
    // The unit's two pieces, four neighbouring entries a lane and piece.  The piece that ends with
    // a row shares entries with the one before it, so that every load is a whole one inside the
    // row; entries k < skip belong there.  A row that ends before the matrix's fourth entry has nothing
    // to share with: it is left to the walk one by one, and so is one past the reach of a 32-bit offset.
    struct Pieces {
      i4v c[2];
      f4v x[2];
      int skip[2];  // (4 and more: nothing here)
      int at;       // place of the row whose scalars this lane works out: even lanes slot 0, odd ones slot 1
    };
    auto quick_len = [&](long long e0, int len) { return e0 + len >= 4 && e0 + len <= kSpan ? min(len, 2 * kPiece) : 0; };
    const int quick_l = CSR ? quick_len(e0_l, len_l) : 0, first_l = (int)e0_l;
    const bool rest = !CSR || __ballot(len_l > quick_l) != 0ull;  // (anything in the wave's rows past the pieces)
    auto request = [&](int it, Pieces &p) __attribute__((always_inline)) {
      const int unit = it * G + grp;
      const bool pair = unit >= M;
      const int at0 = pair ? 2 * unit - M : unit, at1 = pair ? at0 + 1 : at0;
      p.at = (sub & 1) ? at1 : at0;
      int off[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int at = q == 0 ? at0 : at1;
        const int e0 = __builtin_amdgcn_ds_bpermute(4 * at, first_l);
        const int len_any = __builtin_amdgcn_ds_bpermute(4 * at, quick_l);
        const int len = at < cnt ? len_any : 0, last = len - 4;
        const int e = q == 1 && !pair ? 4 * sub + kPiece : 4 * sub;
        off[q] = e < len ? (e0 + min(e, last)) * 4 : kNone;
        p.skip[q] = e - last;
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        p.c[q] = __builtin_bit_cast(i4v, __builtin_amdgcn_raw_buffer_load_b128(r_col, off[q], 0, 0));
        p.x[q] = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(r_val, off[q], 0, 0));
      }
    };
    Pieces ahead;
    if (CSR && iters > 0) request(0, ahead);
    if (CSR && !NEAR && round == 0 && per >= kClaimRows) {
      // A column that every row has must find a hashed slot: the columns of the block's first row get theirs
      // before the waves race for them (left to the race, the two length columns of the translation batches lost it
      // in one block of ten, whose entries then met in one bin: update kernel 21 -> 134 us).
      if (wave == 0 && grp == 0) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int c = ahead.c[k / 4][k % 4];
          if (k % 4 >= ahead.skip[k / 4] && (k < 4 || M > 0) && c >= D) {
            int *const tags = s_tag + 2 * hashed_set<H>(c, factor);
            const int old = atomicCAS(tags, -1, c);
            if (old != -1 && old != c) atomicCAS(tags + 1, -1, c);
          }
        }
      }
      __syncthreads();
    }
    if constexpr (CSR && !NEAR) {  // (as many stores behind the first request as behind the others, see r_late)
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        int none = kNone;
        asm volatile("" : "+v"(none));  // (not one for all)
        store_records(std::integral_constant<int, 1>{}, &lane, &b, &b, &none);
      }
    }
    for (int it = 0; it < iters; ++it) {
      // The waves of a SIMD are served in the order of their age, and the block waits for the youngest: a wave in an
      // earlier quarter of its rows goes first.  (460,000 sentence pairs: the waves' rows ended 64 to 107 us after the
      // launch, now 78 to 103, pass 128.1 -> 125.7 us; 300,000 over 8000 columns 46.0 -> 42.9; pools of 65,536 rows over
      // 2^20 columns 41.3 -> 39.8.  Limits at 1/2, 1/4, 1/8 or 1/3, 1/9, 1/27 of the rows left: 0.5 to 2 us more; the
      // priorities by age alone: nothing.)
      {
        const int first = it * G, left = hi - base - (first < M ? first : 2 * first - M), rows = hi - lo;
        if (left * 4 > rows * 3)
          __builtin_amdgcn_s_setprio(3);
        else if (left * 2 > rows)
          __builtin_amdgcn_s_setprio(2);
        else if (left * 4 > rows)
          __builtin_amdgcn_s_setprio(1);
        else
          __builtin_amdgcn_s_setprio(0);
      }
      const int unit = it * G + grp;
      const bool pair = unit >= M;
      // Row scalars are worked out by the lanes of a row: even lanes have the row in slot 0, odd ones slot 1.
      const int at = CSR ? ahead.at : unit;
      const bool live = at < cnt, teller = live && (sub == 0 || (sub == 1 && pair));
      auto of_row = [&](int v) { return __builtin_amdgcn_ds_bpermute(4 * at, v); };
      const int j = base + (CSR ? of_row(src_l) : at);
      const float u = POOL ? __int_as_float(of_row(__float_as_int(u_l))) : 0.f;
      const float yy = SVM ? __int_as_float(of_row(__float_as_int(y_l))) : 0.f;
      const float lin = ASSIST && !SVM ? __int_as_float(of_row(__float_as_int(lin_l))) : 0.f;
      // what is left of a row of its own after the first two pieces
      long long e0 = 0;
      int len = 0, slow = 0;
      if (rest) {
        e0 = ((long long)of_row((int)(e0_l >> 32)) << 32) | (uint32_t)of_row((int)(uint32_t)e0_l);
        const int len_any = of_row(len_l);
        len = live && !pair ? len_any : 0;
        slow = CSR ? quick_len(e0, len) : 0;
      }
      float dp[2] = {0.f, 0.f}, dw[2] = {0.f, 0.f};
      // Shares of the dot products.  The columns that are not in LDS are gathered without a
      // branch (an entry with nothing to fetch asks for nothing), so that the gathers leave together.
      // Column -1: no entry.
      auto gather = [&](auto n_const, const int *c, float2 *far, bool all_near) __attribute__((always_inline)) {
        constexpr int N = decltype(n_const)::value;
#pragma unroll
        for (int k = 0; k < N; ++k) far[k] = make_float2(0.f, 0.f);
        if (all_near) return;  // (no such columns: a round trip less)
        if (CSR && reach) {
#pragma unroll
          for (int k = 0; k < N; ++k) {
            const int off = c[k] >= D ? c[k] * kColBytes : kNone;
            if (TWO) {
              const u2v v = __builtin_bit_cast(u2v, __builtin_amdgcn_raw_buffer_load_b64(r_far, off, 0, 0));
              far[k] = make_float2(__uint_as_float(v.x), __uint_as_float(v.y));  // both values with one gather
            } else {
              far[k].x = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r_far, off, 0, 0));
            }
          }
          return;
        }
#pragma unroll
        for (int k = 0; k < N; ++k) {
          const int cf = c[k] >= D ? c[k] : 0;
          if (TWO)
            far[k] = a.wp[cf];
          else
            far[k].x = (ASSIST ? a.phi : a.w)[cf];
        }
      };
      auto dot_entries = [&](auto n_const, const int *c, const float *xv, const float2 *far,
                             int q) __attribute__((always_inline)) {
        constexpr int N = decltype(n_const)::value;
        // (the entries that are in LDS are read together, and ahead of the chain of additions: left to the compiler each
        // is read and waited for behind a branch of its own, inside the chain.  An epoch over 2^20 columns, about 100 entries a
        // row, 41.9 -> 40.8 us a pass, 20,000 rows over 200,000 25.3 -> 24.7; not for dense rows, where all columns of a turn
        // are on one side: step over 16,384 of 9000 709 us, with this 773)
        auto in_lds = [&](int k) __attribute__((always_inline)) {
          const int cn = NEAR ? max(c[k], 0) : min(max(c[k], 0), D - 1);
          return TWO ? reinterpret_cast<const float2 *>(s_model)[cn] : make_float2(s_model[cn], 0.f);
        };
        float2 near[N];
        if constexpr (CSR) {
#pragma unroll
          for (int k = 0; k < N; ++k) near[k] = in_lds(k);
#pragma unroll
          for (int k = 0; k < N; ++k) {
            asm volatile("" : "+v"(near[k].x));
            if (TWO) asm volatile("" : "+v"(near[k].y));
          }
        }
#pragma unroll
        for (int k = 0; k < N; ++k) {
          if constexpr (!CSR) near[k] = in_lds(k);
          const bool in = c[k] >= 0;
          const float mw = !NEAR && c[k] >= D ? far[k].x : near[k].x;
          const float mp = TWO ? (!NEAR && c[k] >= D ? far[k].y : near[k].y) : mw;
          if (SVM) dw[q] = in ? __fmaf_rn(mw, xv[k], dw[q]) : dw[q];
          if (NEED_PHI) dp[q] = in ? __fmaf_rn(mp, xv[k], dp[q]) : dp[q];
        }
      };
      int c_unit[8];
      float x_unit[8];
      bool second = false;  // anything in slot 1
      if constexpr (CSR) {
        Pieces cur = ahead;
        asm volatile("" : "+v"(cur.c[0]), "+v"(cur.c[1]), "+v"(cur.x[0]), "+v"(cur.x[1]));  // (waited for here)
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          c_unit[k] = k % 4 >= cur.skip[k / 4] ? cur.c[k / 4][k % 4] : -1;
          x_unit[k] = cur.x[k / 4][k % 4];
        }
        float2 far[8];
        gather(std::integral_constant<int, 8>{}, c_unit, far, NEAR);
        __builtin_amdgcn_sched_barrier(0);
        request(it + 1, ahead);  // (past the last unit: no accesses)
        __builtin_amdgcn_sched_barrier(0);
        if (!a.val) {
#pragma unroll
          for (int k = 0; k < 8; ++k) x_unit[k] = 1.f;
        }
        dot_entries(std::integral_constant<int, 4>{}, c_unit, x_unit, far, 0);
        dp[1] = pair ? 0.f : dp[0];  // (one row: its sums go on, in the order of the scoring kernels)
        dw[1] = pair ? 0.f : dw[0];
        second = __ballot(cur.skip[1] < 4) != 0ull;
        if (second) dot_entries(std::integral_constant<int, 4>{}, c_unit + 4, x_unit + 4, far + 4, 1);
      }
      constexpr int kRest = CSR && TWO ? 4 : 8;  // (eight: more registers than there are)
      auto walk = [&](int eb, bool all_near) __attribute__((always_inline)) {
        int c[kRest];
        float xv[kRest];
        float2 far[kRest];
        if constexpr (CSR) {  // four neighbours a lane here too
          i4v cq[kRest / 4] = {};
          f4v xq[kRest / 4] = {};
          if (e0 + len >= 4) {
#pragma unroll
            for (int q = 0; q < kRest / 4; ++q) {
              const int first = min(eb + q * kPiece, len - 4);
              if (eb + q * kPiece < len) {
                cq[q] = *reinterpret_cast<const i4v *>(a.col + e0 + first);
                if (a.val) xq[q] = *reinterpret_cast<const f4v *>(a.val + e0 + first);
              }
            }
          } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              if (k < 4 - len) continue;
              cq[0][k] = a.col[e0 + len - 4 + k];
              if (a.val) xq[0][k] = a.val[e0 + len - 4 + k];
            }
          }
#pragma unroll
          for (int k = 0; k < kRest; ++k) {
            c[k] = k % 4 >= eb + k / 4 * kPiece - (len - 4) ? cq[k / 4][k % 4] : -1;
            xv[k] = a.val ? xq[k / 4][k % 4] : 1.f;
          }
        } else {
#pragma unroll
          for (int k = 0; k < kRest; ++k) {
            const int e = eb + k * GL;
            c[k] = e < len ? e : -1;
            xv[k] = e < len ? a.x[e0 + e] : 0.f;
          }
        }
        gather(std::integral_constant<int, kRest>{}, c, far, all_near);
        dot_entries(std::integral_constant<int, kRest>{}, c, xv, far, CSR ? 1 : 0);
      };
      if constexpr (CSR) {
        if (rest)
          for (int eb = slow + 4 * sub; eb < len; eb += kRest * GL) walk(eb, NEAR);
      } else {  // (first the columns that are in LDS)
        static_assert(CSR || D % (kRest * GL) == 0, "no turn on both sides");
        int eb = sub;
        for (; eb < min(len, D); eb += kRest * GL) walk(eb, true);
        for (; eb < len; eb += kRest * GL) walk(eb, false);
      }
      // the sums of this lane's slot
      auto own = [&](float v0, float v1) __attribute__((always_inline)) {
        if (!CSR) return gsum<GL>(v0);
        v0 = gsum<GL>(v0);
        v1 = gsum<GL>(v1);
        asm volatile("" : "+v"(v0), "+v"(v1));  // (both there: a choice, not a branch)
        return pair && !(sub & 1) ? v0 : v1;
      };
      float g = 0.f;
      bool keep = live;
      if (NEED_PHI) {
        const float s = own(dp[0], dp[1]) + b;
        g = sigmoidf_(s);
        if (POOL) {
          if (a.do_keep) keep = live && keep_decision(u, g, a.gamma, a.one_minus_gamma);
          if (teller) {
            if (a.logit) a.logit[j] = s;
            if (a.prob) a.prob[j] = g;
            if (a.flags) a.flags[j] = keep ? 1 : 0;
          }
        }
      }
      float loss = lin, cw_own = 0.f, resid_own = 0.f;
      if (SVM) {
        const float marg = yy * own(dw[0], dw[1]);
        loss = fmaxf(0.f, 1.f - marg);
        if (HARD) {  // shrinking by the objective value itself
          keep = live && loss > T;
          if (teller && a.flags) a.flags[j] = keep ? 1 : 0;
        }
        if (teller && (HARD || keep) && a.loss_out) a.loss_out[j] = loss;
        cw_own = (keep && marg < 1.f) ? yy : 0.f;
      }
      if (ASSIST) {
        const float z = loss > T ? 1.f : 0.f;
        resid_own = keep ? g - z : 0.f;
        if (teller) gb += resid_own;
      }
      if (teller && keep) kept += 1;
      // the coefficients of both slots' rows, in every lane (quad_perm 0,0,2,2 and 1,1,3,3)
      const float cw[2] = {dpp_move<0xA0>(cw_own), dpp_move<0xF5>(cw_own)};
      const float resid[2] = {dpp_move<0xA0>(resid_own), dpp_move<0xF5>(resid_own)};
      // Second walk.  A column's sum is its slot's, or that of the hashed slot that holds it; an entry that
      // finds neither leaves as a record.  N entries of a lane together (column -1: none): their tag reads
      // are in flight at once.
      const bool has_w[2] = {SVM && cw[0] != 0.f, SVM && cw[1] != 0.f};
      const bool has_p[2] = {ASSIST && resid[0] != 0.f, ASSIST && resid[1] != 0.f};
      const uint64_t contrib[2] = {__ballot(has_w[0] || has_p[0]), __ballot(has_w[1] || has_p[1])};
      auto add_at = [&](int q, int at, float ta, float tb) __attribute__((always_inline)) {  // (at: byte offset)
        double *const to = reinterpret_cast<double *>(reinterpret_cast<char *>(s_sum) + at);
        if (!TWO || has_w[q]) unsafeAtomicAdd(to, (double)ta);
        if (TWO && has_p[q]) unsafeAtomicAdd(to + (D + H), (double)tb);
      };
      auto scatter = [&](auto n_const, const int *c, const float *xv, int slot, bool all_near, uint64_t *miss, float *ta,
                         float *tb) __attribute__((always_inline)) {
        constexpr int N = decltype(n_const)::value;
#pragma unroll
        for (int k = 0; k < N; ++k) {
          const int q = slot + k / 4;
          ta[k] = SVM ? (has_w[q] ? cw[q] * xv[k] : 0.f) : resid[q] * xv[k];
          tb[k] = TWO ? (has_p[q] ? resid[q] * xv[k] : 0.f) : 0.f;
          miss[k] = 0;
        }
        if (all_near) {  // (every column has its slot)
#pragma unroll
          for (int k = 0; k < N; ++k)
            if (__builtin_amdgcn_inverse_ballot_w64(contrib[slot + k / 4] & __ballot(c[k] >= 0)))
              add_at(slot + k / 4, 8 * c[k], ta[k], tb[k]);
          return;
        }
        int2 tag[N];
        int set[N];  // byte offset of the set's tags
#pragma unroll
        for (int k = 0; k < N; ++k) {
          set[k] = 8 * hashed_set<H>(c[k], factor);
          tag[k] = *reinterpret_cast<const int2 *>(reinterpret_cast<const char *>(s_tag) + set[k]);
        }
        uint64_t far[N], first_is[N], second_is[N], claim = 0;
#pragma unroll
        for (int k = 0; k < N; ++k) {
          far[k] = contrib[slot + k / 4] & __ballot(c[k] >= D);
          first_is[k] = __ballot(tag[k].x == c[k]);
          second_is[k] = __ballot(tag[k].y == c[k]);
          claim |= far[k] & ~(first_is[k] | second_is[k]) & __ballot(tag[k].y == -1);  // (the second of a set is taken last)
        }
        if (claim != 0ull) {  // (rare after the first rows)
#pragma unroll
          for (int k = 0; k < N; ++k) {
            if (__builtin_amdgcn_inverse_ballot_w64(far[k] & ~(first_is[k] | second_is[k]))) {
              // (a tag changes once, from -1 to its column)
              int *const tags = reinterpret_cast<int *>(reinterpret_cast<char *>(s_tag) + set[k]);
              if (tag[k].x == -1) {
                const int old = atomicCAS(tags, -1, c[k]);
                tag[k].x = old == -1 ? c[k] : old;
              }
              if (tag[k].x != c[k] && tag[k].y == -1) {
                const int old = atomicCAS(tags + 1, -1, c[k]);
                tag[k].y = old == -1 ? c[k] : old;
              }
            }
            first_is[k] = __ballot(tag[k].x == c[k]);
            second_is[k] = __ballot(tag[k].y == c[k]);
          }
        }
#pragma unroll
        for (int k = 0; k < N; ++k) {
          int in_set = 2 * set[k] + 8 * D + (__builtin_amdgcn_inverse_ballot_w64(second_is[k]) ? 8 : 0);
          asm volatile("" : "+v"(in_set));  // (one address, one addition: not a branch for either)
          const int at = c[k] >= D ? in_set : 8 * c[k];
          const uint64_t near = contrib[slot + k / 4] & __ballot((unsigned)c[k] < (unsigned)D);
          const uint64_t has = first_is[k] | second_is[k];
          miss[k] = far[k] & ~has;
          if (__builtin_amdgcn_inverse_ballot_w64(near | (far[k] & has))) add_at(slot + k / 4, at, ta[k], tb[k]);
        }
      };
      if constexpr (CSR) {
        // (two vectors: eight at once are more registers than there are; one vector, four at once: update over 460,000
        // sentence pairs 171 us, with eight 168, over 1000 rows of 56 entries 20.3 and 21.1)
        uint64_t miss[8];
        float ta[8], tb[8];
        if constexpr (!TWO) {
          int off[8] = {kNone, kNone, kNone, kNone, kNone, kNone, kNone, kNone};
          if (second) {
            scatter(std::integral_constant<int, 8>{}, c_unit, x_unit, 0, NEAR, miss, ta, tb);
            if (!NEAR) place_records(std::integral_constant<int, 8>{}, miss, c_unit, ta, tb, off);
          } else {
            scatter(std::integral_constant<int, 4>{}, c_unit, x_unit, 0, NEAR, miss, ta, tb);
            if (!NEAR) place_records(std::integral_constant<int, 4>{}, miss, c_unit, ta, tb, off);
#pragma unroll
            for (int k = 4; k < 8; ++k) ta[k] = tb[k] = 0.f;
          }
          if (!NEAR) store_records(std::integral_constant<int, 8>{}, c_unit, ta, tb, off);
        } else {
          int off[4];
          scatter(std::integral_constant<int, 4>{}, c_unit, x_unit, 0, NEAR, miss, ta, tb);
          if (!NEAR) {
            place_records(std::integral_constant<int, 4>{}, miss, c_unit, ta, tb, off);
            store_records(std::integral_constant<int, 4>{}, c_unit, ta, tb, off);
          }
#pragma unroll
          for (int k = 0; k < 4; ++k) off[k] = kNone;
          if (second) {
            scatter(std::integral_constant<int, 4>{}, c_unit + 4, x_unit + 4, 1, NEAR, miss, ta, tb);
            if (!NEAR) place_records(std::integral_constant<int, 4>{}, miss, c_unit + 4, ta, tb, off);
          }
          if (!NEAR) store_records(std::integral_constant<int, 4>{}, c_unit + 4, ta, tb, off);
        }
      }
      // entries beyond; the wave's groups step together
      if (rest) {
        int steps_len = has_w[0] || has_p[0] ? len - slow : 0;
#pragma unroll
        for (int off = GL; off < kWave; off <<= 1) steps_len = max(steps_len, __shfl_xor(steps_len, off, kWave));
        steps_len = __builtin_amdgcn_readfirstlane(steps_len);  // (what follows is the wave's then: scalar counts)
        auto walk_again = [&](int eb, bool all_near) __attribute__((always_inline)) {
          const int e = slow + eb + sub;
          int c = -1;
          float xv = 0.f, ta, tb;
          uint64_t miss;
          if ((has_w[0] || has_p[0]) && e < len) {
            c = CSR ? a.col[e0 + e] : e;
            xv = CSR ? (a.val ? a.val[e0 + e] : 1.f) : a.x[e0 + e];
          }
          scatter(std::integral_constant<int, 1>{}, &c, &xv, 0, all_near, &miss, &ta, &tb);
          if (!all_near) append(std::integral_constant<int, 1>{}, &miss, &c, &ta, &tb);
        };
        if constexpr (CSR) {
          for (int eb = 0; eb < steps_len; eb += GL) walk_again(eb, NEAR);
        } else {
          int eb = 0;
          for (; eb < min(steps_len, D); eb += GL) walk_again(eb, true);
          for (; eb < steps_len; eb += GL) walk_again(eb, false);
        }
      }
    }
  }

  // kept count and bias-gradient sum of the block: wave sums, then wave order (one store per
  // block; thousands of waves adding to one address would run one after the other)
  int kw = kept;
  float gbw = gb;
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) {
    kw += __shfl_xor(kw, off, kWave);
    gbw += __shfl_xor(gbw, off, kWave);
  }
  if (lane == 0) {
    s_cnt[wave] = kw;
    s_gb[wave] = gbw;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int kb = 0;
    float gbb = 0.f;
    for (int i = 0; i < kWaves; ++i) {
      kb += s_cnt[i];
      gbb += s_gb[i];
    }
    a.blk_cnt[blockIdx.x] = kb;
    a.blk_gb[blockIdx.x] = gbb;
  }
  // The hashed slots.  Which columns won one depends on the order in which the waves arrived, so a
  // slot's sum must leave the block without rounding: as up to three records, floats that add up
  // to the double exactly (24 bits each; the sums are multiples of the smallest float).
  static_assert(H % kGradThreads == 0, "whole turns of the block");
  for (int turn = 0; !NEAR && a.d > D && turn < H / kGradThreads; ++turn) {
    const int k = turn * kGradThreads + threadIdx.x;
    int c = s_tag[k];
    double va = s_sum[D + k], vb = TWO ? s_sum[(D + H) + D + k] : 0.0;
    if (c >= 0 && !(fabs(va) <= 3e38 && fabs(vb) <= 3e38)) {  // (no float for it, or no number)
      add_global<SVM, ASSIST>(a, c, va, vb);
      c = -1;
    }
    uint64_t want[3];
    int cols[3];
    float ta[3], tb[3];
#pragma unroll
    for (int part = 0; part < 3; ++part) {
      ta[part] = (float)va;
      tb[part] = (float)vb;
      va -= (double)ta[part];
      vb -= (double)tb[part];
      cols[part] = c;
      want[part] = __ballot(c >= 0 && (ta[part] != 0.f || tb[part] != 0.f));
    }
    append(std::integral_constant<int, 3>{}, want, cols, ta, tb);
  }
  // the first columns: this block's sums, zeros included
  float *const mine = a.part + (size_t)blockIdx.x * NVEC * a.head;
  for (int k = threadIdx.x; k < a.head; k += kGradThreads) {
    mine[k] = (float)s_sum[k];
    if (TWO) mine[a.head + k] = (float)s_sum[(D + H) + k];
  }
  if (NEAR || !binned) return;
  __syncthreads();
  // The records in LDS go to the bins, a run per bin (one integer atomic per block and bin reserves the space); one
  // that finds its bin full joins the late ones.
  const int n = min(s_nrec[0], cap);
  const int segment = blockIdx.x & (a.plan.segments - 1);
  int beyond = max(n - held, 0);
  {
    const int m = min(n, held);
    constexpr int kPer = R / kGradThreads;
    static_assert(R % kGradThreads == 0, "whole turns of the block");
    if (threadIdx.x < kMaxBins) s_hist[threadIdx.x] = 0;
    __syncthreads();
    int rank[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int i = threadIdx.x + q * kGradThreads;
      rank[q] = i < m ? atomicAdd(s_hist + bin_of(s_held[i * RW], D, a.plan), 1) : 0;
    }
    __syncthreads();
    if ((int)threadIdx.x < a.plan.nb) {
      const int h = s_hist[threadIdx.x];
      const int base = h > 0 ? (int)atomicAdd(a.bin_fill + segment * kMaxBins + threadIdx.x, (unsigned)h) : 0;
      s_base[threadIdx.x] = base;
      const int over = min(base + h - a.plan.seg_cap, h);
      if (over > 0) atomicAdd(&s_more, over);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int i = threadIdx.x + q * kGradThreads;
      if (i >= m) continue;
      int r[RW];
#pragma unroll
      for (int w = 0; w < RW; ++w) r[w] = s_held[i * RW + w];
      const int bin = bin_of(r[0], D, a.plan), pos = s_base[bin] + rank[q];
      if (pos < a.plan.seg_cap) {
        int32_t *const dst = a.recs + (((size_t)bin * a.plan.segments + segment) * a.plan.seg_cap + pos) * RW;
#pragma unroll
        for (int w = 0; w < RW; ++w) dst[w] = r[w];
      } else {
        const int place = beyond + atomicAdd(&s_next, 1);
        if (place < cap - held) {
          const int piece = (int)((unsigned)place / (unsigned)a.plan.piece);
          int32_t *const dst = piece_at(piece) + (place - piece * a.plan.piece) * RW;
#pragma unroll
          for (int w = 0; w < RW; ++w) dst[w] = r[w];
        } else {
          add_global<SVM, ASSIST>(a, r[0], __int_as_float(r[1]), TWO ? __int_as_float(r[RW - 1]) : 0.f);
        }
      }
    }
    beyond = min(beyond + s_more, cap - held);
  }
  // The others, a piece (at most C) at a time, sorted by bin (a counting sort by way of LDS) and on to the bins like
  // those above, if the block's share of the bins has room for all of its records.  What stays goes back to where it was,
  // and its owner finds it as one run (start, count) of the piece.  (Nothing on to the bins / all that finds room / so: update
  // kernel over 460,000 sentence pairs, whose 5.4 M records were 512 runs of 41 a bin strewn over 60 MB, 27.5 / 14.2 / 13.9
  // us and this pass 126.3 / 129.6 / 129.1; whole update over as many rows of 60 uniform columns 333 / 347 / 335, of 82 480 / 702 /
  // 482.  The next piece's loads ahead of the stores: no gain; two bins' places with one atomic: 129.0, but 0.2 us
  // more over small pools.)
  if (threadIdx.x == 0) a.blk_late[blockIdx.x] = beyond;
  const bool binnable = min(n, held) + beyond <= a.plan.share;
  int *const s_rec = reinterpret_cast<int *>(s_mem);
  constexpr int kPer = C / kGradThreads;
  for (int piece = 0; piece * a.plan.piece < beyond; ++piece) {
    int32_t *const src = piece_at(piece);
    const int m = min(a.plan.piece, beyond - piece * a.plan.piece);
    __syncthreads();  // (everybody is done with what the memory held before)
    if (threadIdx.x < kMaxBins) s_hist[threadIdx.x] = 0;
    int r[kPer][RW], rank[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      if (q * kGradThreads >= m) break;  // (the same for the whole block)
      const int i = min((int)threadIdx.x + q * kGradThreads, m - 1);
#pragma unroll
      for (int w = 0; w < RW; ++w) r[q][w] = src[(size_t)i * RW + w];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      if (q * kGradThreads >= m) break;
      rank[q] = 0;
      if ((int)threadIdx.x + q * kGradThreads < m) rank[q] = atomicAdd(s_hist + bin_of(r[q][0], D, a.plan), 1);
    }
    __syncthreads();
    const bool owns = (int)threadIdx.x < a.plan.nb;
    const int h = owns ? s_hist[threadIdx.x] : 0;
    int to = a.plan.seg_cap;  // (used after the records have moved in LDS: the round trip is under way meanwhile)
    if (binnable && h > 0) to = (int)atomicAdd(a.bin_fill + segment * kMaxBins + threadIdx.x, (unsigned)h);
    if (wave == 0) {  // four bins a lane
      static_assert(kMaxBins == 4 * kWave, "one wave scans the bins");
      const int4 n4 = reinterpret_cast<const int4 *>(s_hist)[lane];
      const int mine = n4.x + n4.y + n4.z + n4.w;
      int before = mine;
#pragma unroll
      for (int off = 1; off < kWave; off <<= 1) {
        const int v = __shfl_up(before, off, kWave);
        if (lane >= off) before += v;
      }
      before -= mine;
      reinterpret_cast<int4 *>(s_base)[lane] = make_int4(before, before + n4.x, before + n4.x + n4.y, before + n4.x + n4.y + n4.z);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      if (q * kGradThreads >= m) break;
      if ((int)threadIdx.x + q * kGradThreads < m) {
        const int pos = s_base[bin_of(r[q][0], D, a.plan)] + rank[q];
#pragma unroll
        for (int w = 0; w < RW; ++w) s_rec[pos * RW + w] = r[q][w];
      }
    }
    __syncthreads();
    if (owns) {
      const int start = s_base[threadIdx.x], fit = min(max(a.plan.seg_cap - to, 0), h);
      if (fit < h) left_marks(a.blk_late)[threadIdx.x] = 1;
      a.runs[((size_t)threadIdx.x * a.plan.pieces + piece) * gridDim.x + blockIdx.x] = (start + fit) | ((h - fit) << 16);
      s_hist[threadIdx.x] = to - start;  // (place in the bin less place in the piece)
    }
    if (!binnable) {  // whole 128-bit words (a piece is a multiple of four records)
      for (int i = threadIdx.x; 4 * i < m * RW; i += kGradThreads)
        reinterpret_cast<int4 *>(src)[i] = reinterpret_cast<const int4 *>(s_rec)[i];
      continue;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < m; i += kGradThreads) {
      int r[RW];
#pragma unroll
      for (int w = 0; w < RW; ++w) r[w] = s_rec[i * RW + w];
      const int bin = bin_of(r[0], D, a.plan), pos = i + s_hist[bin];
      int32_t *const dst =
          pos < a.plan.seg_cap ? a.recs + (((size_t)bin * a.plan.segments + segment) * a.plan.seg_cap + pos) * RW : src + i * RW;
#pragma unroll
      for (int w = 0; w < RW; ++w) dst[w] = r[w];
    }
  }
}

// The scoring pass: the stored entries of a row by GL lanes, phi through the caches.
template <int GL, bool CSR>
__global__ __launch_bounds__(kPoolThreads) void k_rows_general(const GenArgs a) {
  constexpr int G = kWave / GL, kUnroll = 8;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int grp = lane / GL, sub = lane % GL;
  const int total = a.count_max;
  const int nwaves = gridDim.x * nw, gwave = blockIdx.x * nw + wave;
  const int per = total / nwaves, rem = total % nwaves;
  const int lo = gwave * per + min(gwave, rem);
  const int hi = lo + per + (gwave < rem ? 1 : 0);
  const float b = a.bias ? *a.bias : 0.f;
  for (int base = lo; base < hi; base += kWave) {
    const int cnt = min(kWave, hi - base);
    // one row per lane, 64 rows per round: extent, draw
    long long e0_l = 0;
    int len_l = 0;
    float u_l = 2.f;
    if (lane < cnt) {
      const int j_l = base + lane;
      const int row_l = a.rows ? a.rows[j_l] : j_l;
      if (CSR) {
        e0_l = a.rowptr[row_l];
        len_l = (int)(a.rowptr[row_l + 1] - e0_l);
      } else {
        e0_l = (long long)row_l * a.ld;
        len_l = a.d;
      }
      if (a.do_keep) u_l = keep_uniform(a.key, (uint32_t)j_l);
    }
    const int iters = (cnt + G - 1) / G;
    for (int it = 0; it < iters; ++it) {
      const int li = it * G + grp;
      const bool live = li < cnt;
      const int j = base + li;
      const long long e0 = __shfl(e0_l, li, kWave);
      const int len_any = __shfl(len_l, li, kWave);  // every lane takes part in the shuffle
      const int len = live ? len_any : 0;
      const float u = __shfl(u_l, li, kWave);
      float dp = 0.f;
      if constexpr (CSR) {
        // four neighbouring entries a lane: one load per array for 4 GL entries.  The piece that ends
        // with the row shares entries with the one before it, so that every load is a whole one inside
        // the row (entries k < skip belong there); rows that end before the matrix's fourth
        // entry have nothing to share with and are read one by one.
        for (int e = 4 * sub; e < len; e += 8 * GL) {
          i4v c[2] = {};
          f4v xv[2] = {};
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int first = min(e + q * 4 * GL, len - 4);
            if (e + q * 4 * GL < len && e0 + len >= 4) {
              c[q] = *reinterpret_cast<const i4v *>(a.col + e0 + first);
              if (a.val) xv[q] = *reinterpret_cast<const f4v *>(a.val + e0 + first);
            }
          }
          if (e0 + len < 4) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              if (k < 4 - len) continue;
              c[0][k] = a.col[e0 + len - 4 + k];
              xv[0][k] = a.val ? a.val[e0 + len - 4 + k] : 0.f;
            }
          }
          float m[2][4];
#pragma unroll
          for (int q = 0; q < 2; ++q) {
#pragma unroll
            for (int k = 0; k < 4; ++k) m[q][k] = a.phi[k >= e + q * 4 * GL - (len - 4) ? c[q][k] : 0];
          }
#pragma unroll
          for (int q = 0; q < 2; ++q) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const float added = __fmaf_rn(m[q][k], a.val ? xv[q][k] : 1.f, dp);
              dp = k >= e + q * 4 * GL - (len - 4) ? added : dp;
            }
          }
        }
      } else {
        for (int e = sub; e < len; e += GL * kUnroll) {
          float xv[kUnroll];
#pragma unroll
          for (int u = 0; u < kUnroll; ++u) xv[u] = e + u * GL < len ? a.x[e0 + e + u * GL] : 0.f;
#pragma unroll
          for (int u = 0; u < kUnroll; ++u) dp = __fmaf_rn(a.phi[e + u * GL < len ? e + u * GL : 0], xv[u], dp);
        }
      }
      dp = gsum<GL>(dp);
      const float s = dp + b;
      const float g = sigmoidf_(s);
      const bool keep = live && (!a.do_keep || keep_decision(u, g, a.gamma, a.one_minus_gamma));
      if (sub == 0 && live) {
        if (a.logit) a.logit[j] = s;
        if (a.prob) a.prob[j] = g;
        if (a.flags) a.flags[j] = keep ? 1 : 0;
      }
    }
  }
}

// p is 16-byte aligned: 128-bit stores, then the few floats left over.
__global__ __launch_bounds__(256) void k_zero_f32(float *p, size_t count) {
  const size_t n4 = count / 4, tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  float4 *p4 = reinterpret_cast<float4 *>(p);
  for (size_t i = tid; i < n4; i += stride) p4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  if (tid < count - 4 * n4) p[4 * n4 + tid] = 0.f;
}

// Scoring pass over CSR rows with the first kScoreTableCols entries of phi in LDS: one block of
// 16 waves per compute unit loads them once and then walks its rows; only columns past the
// table are gathered through the caches.  The gathers of k_rows_general go through the vector L1, which
// serves a lane or so a cycle, and from a few thousand columns on miss it.  Same outputs and the same
// order of additions per row as k_rows_general<16, true>, so the two give the same bits.
// What bounds it: the vector memory path.  1,000,000 rows of 56 entries over 64,002 columns (448 MB),
// per launch: 163 us with a 32-bit load per entry (16 loads and 8 gathers a step, a sigmoid per row and
// group), 155 with one 128-bit load per array and half slot and the sigmoids of 64 rows at a time, 151 with
// the requests going on across rounds.  With non-temporal loads it is 128, but the rows are then gone from
// the memory-side cache and the copy of the kept rows that follows takes 126 instead of 97.  With all of the
// table's loads in flight together 137; 300,000 rows over 64,002 columns 57.9 -> 44.9, 30,000 over 40,002 20.1 -> 11.6.
constexpr int kScoreTableCols = 39936;  // 156 KB of the 160 KB
constexpr int kScoreTableThreads = 1024;
// Taken for pools of at least kScoreTableMinRows rows over more than kScoreTableMinCols columns, and
// for kScoreTableManyRows rows over fewer, when the table holds at least half of phi.  Scoring calls alone, values,
// k_rows_general / this.  Rows of 30 to 82 entries, columns Zipf-like: 24,576 rows over 40,002 5.2 / 9.5, 32,768 over 64,002
// 6.2 / 9.9, 49,152 8.8 / 10.2, 65,536 11.3 / 11.0, 98,304 17.8 / 14.0; over 8002 49,152 8.2 / 9.5, 65,536 10.2 / 10.1,
// 98,304 15.8 / 13.0.  Columns uniform: 32,768 over 40,002 9.6 / 9.6, 49,152 13.3 / 9.7; over 8002 49,152 9.0 / 9.5,
// 98,304 18.8 / 13.0.  Rows of 4 to 20 entries: 65,536 7.4 / 9.5, 98,304 10.7 / 9.5; of 150 to 250: 32,768 over 40,002
// 17.0 / 18.2, 49,152 23.9 / 19.9, over 2002 49,152 17.4 / 20.0, 65,536 21.2 / 23.7, 98,304 31.9 / 29.6.
// On 65,536 rows of about 100 entries over 2^20 Zipf-distributed columns, where a quarter of the entries lie
// past the table, k_rows_general stays ahead (34 us against 48).
constexpr int kScoreTableMinCols = 16384, kScoreTableMinRows = 49152, kScoreTableManyRows = 98304;
constexpr int kScoreTableMaxCols = 2 * kScoreTableCols;

// No load of the main loop sits behind a branch (a lane with nothing to read asks for an
// offset outside its buffer resource, which costs no memory access and reads as zero), so the
// waits the compiler places count the loads in flight exactly and never drain them: the
// entries of the row groups one and two steps ahead and the cold-column gathers of the next
// group stay outstanding while the current group is added up, and the row extents arrive a
// round (64 rows) ahead, the row ids two rounds.  Rows longer than one chunk (128 entries)
// are skipped in the loop and walked afterwards, a lane group each.
template <bool VAL>
__global__ __launch_bounds__(kScoreTableThreads) void k_score_table(const GenArgs a) {
  constexpr int GL = 16, G = kWave / GL, kUnroll = 8, kChunk = GL * kUnroll;
  __shared__ __attribute__((aligned(16))) float s_phi[kScoreTableCols];
  __shared__ float s_row[kScoreTableThreads / kWave][kWave];  // sums of a wave's round
  const int D = min(kScoreTableCols, a.d);
  const int lane = threadIdx.x & 63, nw = kScoreTableThreads >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = lane / GL, sub = lane % GL;
  const int total = a.count_max;
  const int nwaves = gridDim.x * nw, gwave = blockIdx.x * nw + wave;
  const int per = total / nwaves, rem = total % nwaves;
  const int lo = gwave * per + min(gwave, rem);
  const int hi = lo + per + (gwave < rem ? 1 : 0);
  const float b = a.bias ? *a.bias : 0.f;
  // an address that is always readable, for lanes with nothing to load
  const int *const nowhere = reinterpret_cast<const int *>(a.rowptr);

  // Entries and cold columns are read through buffer resources: a lane with nothing to read
  // gives an offset past the resource's range, for which the hardware returns zero without a
  // memory access -- no stand-in addresses.  Offsets are 32 bits: rows whose entries
  // lie beyond kSpan bytes of the arrays take the walk after the loop.
  constexpr int kNone = (int)0x80000000;         // out of every resource's range
  constexpr long long kSpan = 0x7fffffffll / 4;  // entries within reach of a 32-bit byte offset
  const __amdgpu_buffer_rsrc_t r_col = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int32_t *>(a.col), 0, kNone, 0x00020000);
  const __amdgpu_buffer_rsrc_t r_val = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float *>(VAL ? a.val : a.phi), 0, kNone, 0x00020000);
  const __amdgpu_buffer_rsrc_t r_phi = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float *>(a.phi), 0, a.d * 4, 0x00020000);
  struct Slot {  // two half chunks per lane group
    i4v c[2];
    f4v x[2];
    float far[kUnroll];
    int skip[2];
  };
  // Half h of a slot: entries [e, e + kHalfChunk) of the row that starts at entry e0 and has len
  // entries, four neighbours a lane.  The piece that ends with the row shares entries with the one
  // before it, so that every load is a whole one inside the row; entries k < skip belong there.
  constexpr int kHalfChunk = GL * 4;
  static_assert(kUnroll == 8, "two pieces of four");
  auto request_half = [&](int e0, int len, int e, int h, Slot &t) __attribute__((always_inline)) {
    const int first = e + 4 * sub, last = len - 4;
    t.skip[h] = first - last;
    const int off = first < len ? (e0 + min(first, last)) * 4 : kNone;
    t.c[h] = __builtin_bit_cast(i4v, __builtin_amdgcn_raw_buffer_load_b128(r_col, off, 0, 0));
    if (VAL) t.x[h] = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(r_val, off, 0, 0));
  };
  auto gather = [&](Slot &t) __attribute__((always_inline)) {  // columns past the table
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int c = t.c[u / 4][u % 4];
      t.far[u] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(r_phi, c >= D ? c * 4 : kNone, 0, 0));
    }
  };
  auto dot_half = [&](const Slot &t, int h, float dp) __attribute__((always_inline)) {
    float near[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) near[k] = s_phi[min(t.c[h][k], D - 1)];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float m = t.c[h][k] >= D ? t.far[4 * h + k] : near[k];
      const float added = VAL ? __fmaf_rn(m, t.x[h][k], dp) : dp + m;
      dp = k >= t.skip[h] ? added : dp;
    }
    return dp;
  };
  auto emit = [&](int j, float dp, float u) __attribute__((always_inline)) {
    const float s = dp + b;
    const float g = sigmoidf_(s);
    if (a.logit) a.logit[j] = s;
    if (a.prob) a.prob[j] = g;
    if (a.flags)
      a.flags[j] = (!a.do_keep || keep_decision(u, g, a.gamma, a.one_minus_gamma)) ? 1 : 0;
  };

  // raw loads of the row id of pool position j and of the extent of a row
  auto row_id = [&](int j) __attribute__((always_inline)) {
    return *((j < hi && a.rows) ? a.rows + j : nowhere);
  };
  struct Extent {
    int64_t lo, hi;
  };
  auto extent = [&](int j, int raw_id) __attribute__((always_inline)) {
    const int row = j < hi ? (a.rows ? raw_id : j) : 0;
    Extent e;
    e.lo = a.rowptr[row];
    e.hi = a.rowptr[row + 1];
    return e;
  };
  // The table: all of a thread's pieces in flight together, between the loads of the first rows' ids and extents.
  // (A word at a time in a loop, and the ids behind it, a launch took at least 19 us.)
  const int id_first = row_id(lo + lane), id_next = row_id(lo + kWave + lane);
  const float last_phi = a.phi[min((D & ~3) + lane, a.d - 1)];  // (a column of the model's last few)
  constexpr int kTurns = (kScoreTableCols / 4 + kScoreTableThreads - 1) / kScoreTableThreads;
  f4v phi_in[kTurns];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < kTurns; ++q) {
    const int k = 4 * ((int)threadIdx.x + q * kScoreTableThreads);
    phi_in[q] = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(r_phi, k * 4, 0, 0));
  }
  __builtin_amdgcn_sched_barrier(0);
  const Extent first_rows = extent(lo + lane, id_first);
  Extent cur = first_rows;
  Extent next = extent(lo + kWave + lane, id_next);
  int id_after = row_id(lo + 2 * kWave + lane);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < kTurns; ++q) {
    const int k = 4 * ((int)threadIdx.x + q * kScoreTableThreads);
    if (k + 4 <= D) *reinterpret_cast<float4 *>(s_phi + k) = make_float4(phi_in[q].x, phi_in[q].y, phi_in[q].z, phi_in[q].w);
  }
  if (threadIdx.x < (D & 3)) s_phi[(D & ~3) + threadIdx.x] = last_phi;
  __syncthreads();
  bool any_longer = false;

  // A step gives every group of 16 lanes two half slots of 64 entries: both chunks of one row of
  // 65 to 128 entries, or the only chunks of two rows of up to 64.  Per round the wave's 64 rows
  // are put in that order -- the M longer rows, then the S shorter ones, each class in pool order --
  // with one ds_permute per value.  Unit u of a round (group u % 4 of step u / 4) is sorted row u and,
  // from M on, sorted row u + SH beside it (SH = half of S): neighbouring groups read neighbouring rows.
  constexpr int kAhead = 3;  // steps in flight
  struct Round {
    int base;               // its first pool position
    int M, SH, rows, steps; // (at least kAhead steps, so that requests are one round ahead at most)
    unsigned long long here;  // rows that take part
    int e0, len, src;       // of sorted row `lane`: first entry, entries, place in pool order
  };
  // (the next 64 rows' extents are in `cur`; those of the round after and the row ids of the one
  // after that go out here, loads that wait for nothing)
  auto make_round = [&](int base) __attribute__((always_inline)) {
    Round r;
    r.base = base;
    const bool valid = base + lane < hi;
    int len_cur = valid ? (int)(cur.hi - cur.lo) : 0;
    // (out of reach, or no four entries up to the row's end: a row for the walk after the loop)
    if (cur.hi > kSpan || (len_cur > 0 && cur.hi < 4)) len_cur = kChunk + 1;
    any_longer = any_longer || (valid && len_cur > kChunk);
    const bool two = valid && len_cur > kHalfChunk && len_cur <= kChunk;
    const bool one = valid && len_cur <= kHalfChunk;
    const unsigned long long m_two = __ballot(two), m_one = __ballot(one);
    const int S = __popcll(m_one);
    r.M = __popcll(m_two);
    r.SH = (S + 1) / 2;
    r.rows = r.M + S;
    r.steps = max(kAhead, (r.M + r.SH + G - 1) / G);
    r.here = m_two | m_one;
    auto rank_in = [&](unsigned long long mask) __attribute__((always_inline)) {
      return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                            __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
    };
    const int dest = two ? rank_in(m_two) : one ? r.M + rank_in(m_one) : r.rows + rank_in(~r.here);
    r.e0 = __builtin_amdgcn_ds_permute(dest * 4, (int)cur.lo);
    r.len = __builtin_amdgcn_ds_permute(dest * 4, len_cur);
    r.src = __builtin_amdgcn_ds_permute(dest * 4, lane);
    cur = next;
    next = extent(base + 2 * kWave + lane, id_after);
    id_after = row_id(base + 3 * kWave + lane);
    return r;
  };
  // sorted rows of this lane's group in step `it` (-1: none); *same: both halves are one row's
  auto halves = [&](const Round &r, int it, int *rowA, int *rowB, bool *same) __attribute__((always_inline)) {
    const int u = it * G + grp;
    *same = u < r.M;
    *rowA = u < r.M + r.SH ? u : -1;
    *rowB = *same ? u : (u < r.M + r.SH && u + r.SH < r.rows ? u + r.SH : -1);
  };
  auto request_step = [&](const Round &r, int it, Slot &s) __attribute__((always_inline)) {
    int rowA, rowB;
    bool same;
    halves(r, it, &rowA, &rowB, &same);
    const int e0A = __shfl(r.e0, max(rowA, 0), kWave), lenA = __shfl(r.len, max(rowA, 0), kWave);
    const int e0B = __shfl(r.e0, max(rowB, 0), kWave), lenB = __shfl(r.len, max(rowB, 0), kWave);
    request_half(e0A, rowA >= 0 ? lenA : 0, 0, 0, s);
    request_half(e0B, rowB >= 0 ? lenB : 0, same ? kHalfChunk : 0, 1, s);
  };

  Slot t[kAhead];
  if (lo < hi) {
    // `ask` is the round whose entries are being requested, `use` the one whose rows are added up,
    // kAhead steps behind: the requests go on across the end of a round.
    __builtin_amdgcn_s_setprio(3);
    Round ask = make_round(lo);
    Round use = ask;
    int asked = 0, used = 0;
#pragma unroll
    for (int p = 0; p < kAhead; ++p) request_step(ask, asked++, t[p]);
    gather(t[0]);
    bool more = true;
#pragma unroll 1
    while (more) {
#pragma unroll
      for (int p = 0; p < kAhead; ++p) {
        gather(t[(p + 1) % kAhead]);  // the next step: its entries were requested two steps ago
        int rowA, rowB;
        bool same;
        halves(use, used, &rowA, &rowB, &same);
        float dpA = dot_half(t[p], 0, 0.f);
        float dpB = dot_half(t[p], 1, same ? dpA : 0.f);  // (one row: its sum goes on)
        if (asked == ask.steps && ask.base + kWave < hi) {
          ask = make_round(ask.base + kWave);
          asked = 0;
        }
        request_step(ask, asked, t[p]);  // (past the last round: nothing)
        ++asked;
        dpA = gsum<GL>(dpA);
        dpB = gsum<GL>(dpB);
        const int atA = __shfl(use.src, max(rowA, 0), kWave), atB = __shfl(use.src, max(rowB, 0), kWave);
        if (sub == 0 && rowA >= 0 && !same) s_row[wave][atA] = dpA;
        if (sub == 0 && rowB >= 0) s_row[wave][atB] = dpB;
        if (++used == use.steps) {
          // the round's rows, one a lane: what follows from the sums costs as much for 64 rows as for
          // four, and the stores are whole lines
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          const int j = use.base + lane;
          const float u = a.do_keep ? keep_uniform(a.key, (uint32_t)j) : 2.f;
          if ((use.here >> lane) & 1ull) emit(j, s_row[wave][lane], u);
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          more = use.base + kWave < hi;
          if (!more) break;
          // (a wave that is behind goes first, as in k_rows_grad: 137.3 -> 136.4 us, 1,000,000 rows of 56 ones over
          // 16,002 columns 68.2 -> 66.2, 300,000 23.8 -> 22.2)
          const int left = hi - use.base - kWave, mine = hi - lo;
          if (left * 4 > mine * 3)
            __builtin_amdgcn_s_setprio(3);
          else if (left * 2 > mine)
            __builtin_amdgcn_s_setprio(2);
          else if (left * 4 > mine)
            __builtin_amdgcn_s_setprio(1);
          else
            __builtin_amdgcn_s_setprio(0);
          use = ask;
          used = 0;
        }
      }
    }
  }
  if (__ballot(any_longer) == 0ull) return;
  // Rows of more than one chunk or out of reach: a row a lane group, chunk after chunk in the order above, with
  // 64-bit addresses; the requests go on across the ends of rows here too.  100,000 rows of 200 entries, one row of a
  // wave at a time and entry by entry / so / k_rows_general: over 512 columns 132 / 30.7 / 29.6 us, over 2000
  // 134 / 31.1 / 31.5, over 10,000 136 / 33.0 / 40.3, over 50,000 165 / 39.9 / 145.
  for (int base = lo; base < hi; base += kWave) {
    const int j_l = base + lane;
    const Extent e_l = base == lo ? first_rows : extent(j_l, row_id(j_l));
    const int len_l = j_l < hi ? (int)(e_l.hi - e_l.lo) : 0;
    const bool early = len_l > 0 && e_l.hi < 4;  // (ends before the matrix's fourth entry: one by one)
    const bool mine = !early && (len_l > kChunk || (j_l < hi && e_l.hi > kSpan));
    const unsigned long long m_mine = __ballot(mine);
    if (__ballot(mine || early) == 0ull) continue;
    if (early) {
      float dp = 0.f;
      for (int k = 0; k < len_l; ++k) {
        const int c = a.col[e_l.lo + k];
        const float m = c < D ? s_phi[c] : a.phi[c];
        dp = VAL ? __fmaf_rn(m, a.val[e_l.lo + k], dp) : dp + m;
      }
      s_row[wave][lane] = dp;
    }
    const int n = __popcll(m_mine);
    if (n > 0) {
      const unsigned long long m_same = mine ? m_mine : ~m_mine;
      const int to = 4 * ((mine ? 0 : n) + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m_same >> 32),
                                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)m_same, 0u)));
      const int lo_s = __builtin_amdgcn_ds_permute(to, (int)(uint32_t)e_l.lo);
      const int hi_s = __builtin_amdgcn_ds_permute(to, (int)(e_l.lo >> 32));
      const int len_s = __builtin_amdgcn_ds_permute(to, len_l), src_s = __builtin_amdgcn_ds_permute(to, lane);
      // a group's next chunk: sorted row and first entry
      int at = grp, e = 0;
      // (what: twice the chunk's row, plus one for the row's last; -1 past the last row.  A lane with nothing
      // to read gets the matrix's first entries -- there are four: some row here ends behind them.)
      auto request_chunk = [&](Slot &s, int *what) __attribute__((always_inline)) {
        const int from = min(at, kWave - 1);
        const long long e0 = ((long long)__shfl(hi_s, from, kWave) << 32) | (uint32_t)__shfl(lo_s, from, kWave);
        const int len_any = __shfl(len_s, from, kWave), len = at < n ? len_any : 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int first = e + h * kHalfChunk + 4 * sub, last = len - 4;
          const long long off = first < len ? e0 + min(first, last) : 0;
          s.skip[h] = first - last;
          s.c[h] = *reinterpret_cast<const i4v *>(a.col + off);
          if (VAL) s.x[h] = *reinterpret_cast<const f4v *>(a.val + off);
        }
        const bool ends = e + kChunk >= len;
        *what = at < n ? 2 * at + (ends ? 1 : 0) : -1;
        at = at < n && ends ? at + G : at;
        e = ends ? 0 : e + kChunk;
      };
      int what[kAhead];
#pragma unroll
      for (int p = 0; p < kAhead; ++p) request_chunk(t[p], &what[p]);
      gather(t[0]);
      float dp = 0.f;
#pragma unroll 1
      while (__ballot(what[0] >= 0) != 0ull) {
#pragma unroll
        for (int p = 0; p < kAhead; ++p) {
          gather(t[(p + 1) % kAhead]);
          dp = dot_half(t[p], 0, dp);
          dp = dot_half(t[p], 1, dp);
          const int done = what[p];
          request_chunk(t[p], &what[p]);
          const float sum = gsum<GL>(dp);
          const int place = __shfl(src_s, max(done, 0) >> 1, kWave);
          const bool ends = done >= 0 && (done & 1);
          if (ends && sub == 0) s_row[wave][place] = sum;
          dp = ends ? 0.f : dp;
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (mine || early) emit(j_l, s_row[wave][lane], a.do_keep ? keep_uniform(a.key, (uint32_t)j_l) : 2.f);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
}

// What a pass that updates both vectors needs beforehand, in one launch: the accumulators and
// the header cleared, and the two model vectors side by side for the columns past the LDS table.
__global__ __launch_bounds__(256) void k_prepare_general(float *p, size_t count, const float *w,
                                                         const float *phi, float2 *wp, int head,
                                                         int d) {
  const size_t n4 = count / 4, tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  float4 *p4 = reinterpret_cast<float4 *>(p);
  for (size_t i = tid; i < n4; i += stride) p4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  if (tid < count - 4 * n4) p[4 * n4 + tid] = 0.f;
  for (size_t c = head + tid; c < (size_t)d; c += stride) wp[c] = make_float2(w[c], phi[c]);
}

// Folds the gradient sums into the model.  Blocks [0, nh): 32 of the first `head` columns each,
// 16 threads per column adding the per-block sums of the pass in a fixed order; blocks after
// them: the other columns -- one block per bin, which adds the bin's records up in LDS (plus
// whatever overflowed into the dense accumulators), or with no bins a strided share of the
// accumulators; then one block per compaction tile.  Every block adds up the per-block kept
// counts of the pass for itself.
// Eight waves: a bin's owner waits for records, then for its LDS sums, then for its columns, and has a
// compute unit to itself -- more waves keep more of that in flight, until their barriers and
// the shares of the blocks with little to do cost more.  Sparse epoch (d = 2^20, pools of 65,536),
// per step, 4 / 8 / 16 waves: 73.4 / 68.2 / 69.6 us; pools of 8000 35.0 / 31.3 / 34.0.
constexpr int kApplyWaves = 8, kApplyThreads = kApplyWaves * kWave;
constexpr int kHeadCols = kApplyThreads / 16;

// The update of one column from its gradient sums (m == 0: the model stays).
struct Fold {
  const ApplyArgs &a;
  int m;
  float inv_m, shrink, scale;
  __device__ Fold(const ApplyArgs &args, int m_) : a(args), m(m_), inv_m(m_ > 0 ? 1.f / (float)m_ : 0.f) {
    // step size: constant, or lr / sqrt(number of updates made, this one included)
    float lr = args.lr;
    if (args.t_upd && m_ > 0) lr = args.lr / sqrtf((float)(*args.t_snap + 1));
    shrink = 1.f - lr * args.lambda;
    scale = lr * inv_m;
  }
  // w_old, ph: the column's current values, loaded by the caller
  __device__ __forceinline__ void loaded(int k, float gw, float gp, float w_old, float ph) const {
    if (m <= 0) return;
    const float wn = __fmaf_rn(scale, gw, shrink * w_old);
    const float pn = ph - a.lr_a * __fmaf_rn(a.l2_a, ph, gp * inv_m);
    if (a.w) a.w[k] = wn;
    if (a.phi) a.phi[k] = pn;
    if (a.wp_out) a.wp_out[k] = make_float2(wn, pn);  // (both vectors are updated then)
  }
  __device__ __forceinline__ void column(int k, float gw, float gp) const {
    loaded(k, gw, gp, a.w ? a.w[k] : 0.f, a.phi ? a.phi[k] : 0.f);
  }
  // four columns from k on (the same arithmetic per column), as 128-bit stores
  __device__ __forceinline__ void loaded4(int k, f4v gw, f4v gp, f4v w_old, f4v ph) const {
    if (m <= 0) return;
    f4v wn, pn;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      wn[i] = __fmaf_rn(scale, gw[i], shrink * w_old[i]);
      pn[i] = ph[i] - a.lr_a * __fmaf_rn(a.l2_a, ph[i], gp[i] * inv_m);
    }
    if (a.w) *reinterpret_cast<f4v *>(a.w + k) = wn;
    if (a.phi) *reinterpret_cast<f4v *>(a.phi + k) = pn;
    if (a.wp_out) {  // (both vectors are updated then)
      const f4v lo = {wn[0], pn[0], wn[1], pn[1]}, hi = {wn[2], pn[2], wn[3], pn[3]};
      f4v *const dst = reinterpret_cast<f4v *>(a.wp_out + k);
      dst[0] = lo;
      dst[1] = hi;
    }
  }
};

// Kept count of the pass (and the sum of its bias gradients): one per-block value per thread of
// the first four waves.
static_assert(kGeneralGradBlocks == 4 * kWave && kApplyWaves >= 4, "pass_totals adds up four waves' counts");
__device__ __forceinline__ int pass_totals(const ApplyArgs &a, int cnt, float gbs, int *s_m,
                                           float *s_g, float *gb_out) {
  const int t = threadIdx.x;
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) {
    cnt += __shfl_xor(cnt, off, kWave);
    gbs += __shfl_xor(gbs, off, kWave);
  }
  if ((t & 63) == 0) {
    s_m[t >> 6] = cnt;
    s_g[t >> 6] = gbs;
  }
  __syncthreads();
  *gb_out = (s_g[0] + s_g[1]) + (s_g[2] + s_g[3]);
  const int m_pass = s_m[0] + s_m[1] + s_m[2] + s_m[3];
  return a.m_dev ? min(max(*a.m_dev, 0), a.m_max) : m_pass;
}

__device__ __forceinline__ int bin_local(int col, const ApplyArgs &a) {
  const int rel = col - a.head, gl = a.plan.group_log2;
  return (((rel >> gl) >> a.plan.nb_log2) << gl) | (rel & ((1 << gl) - 1));
}

__device__ __forceinline__ int bin_column(int k, int bin, const ApplyArgs &a) {
  const int gl = a.plan.group_log2;
  const int turn = k >> gl, g = (turn << a.plan.nb_log2) | ((bin - turn * kBinTurn) & (a.plan.nb - 1));
  return a.head + ((g << gl) | (k & ((1 << gl) - 1)));
}

// The late records of a bin that it had no room for: a run in every sorted piece of every block.
// Sixteen lanes read a run, four runs of a lane group in flight together, two records a lane of each.  What a run has
// beyond four times the average (of 64 runs, and beyond kShortRun) the whole block reads, run after run: a frequent
// column that found no slot in one block makes one run of thousands, which sixteen lanes walked alone (256 rows of
// 60 entries in one bin, 65,280 rows of two anywhere: update 184 -> 63 us).
template <int RW, class Add>
__device__ __forceinline__ void late_records(const ApplyArgs &a, int bin, int n_mine, int *s_run, int *s_limit,
                                             unsigned long long *s_long, int pieces, Add add) {
  constexpr int kGroups = kApplyThreads / 16, kRuns = 4, kShortRun = 128;
  const int tid = threadIdx.x, grp = tid / 16, sub = tid % 16, nblk = a.nblk_pass;
  const int32_t *const runs = a.runs + (size_t)bin * a.plan.pieces * nblk;
  const int32_t *const late = a.recs + (size_t)a.plan.nb * a.plan.segments * a.plan.seg_cap * RW;
  for (int piece = 0; piece < pieces; ++piece) {
    __syncthreads();
    if (tid < kGeneralGradBlocks) {
      const int run = piece * a.plan.piece < n_mine ? runs[(size_t)piece * nblk + tid] : 0;
      s_run[tid] = run;
      int sum = run >> 16;
#pragma unroll
      for (int off = kWave / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off, kWave);
      const int limit = max(kShortRun, sum / (kWave / 4));
      const unsigned long long is_long = __ballot((run >> 16) > limit);
      if ((tid & 63) == 0) {
        s_limit[tid >> 6] = limit;
        s_long[tid >> 6] = is_long;
      }
    }
    __syncthreads();
    auto run_at = [&](int blk) {
      return late + (((size_t)piece * nblk + min(blk, nblk - 1)) * a.plan.piece + (s_run[blk] & 0xffff)) * RW;
    };
    for (int b0 = grp; b0 < nblk; b0 += kRuns * kGroups) {
      int cnt[kRuns], longest = 0;
      const int32_t *at[kRuns];
#pragma unroll
      for (int i = 0; i < kRuns; ++i) {
        const int blk = min(b0 + i * kGroups, kGeneralGradBlocks - 1);
        cnt[i] = min(s_run[blk] >> 16, s_limit[blk / kWave]);
        if (b0 + i * kGroups >= nblk) cnt[i] = 0;
        longest = max(longest, cnt[i]);
        at[i] = cnt[i] > 0 ? run_at(blk) : late;
      }
      // (Every load is unconditional: a load under a condition makes the compiler wait for all loads in flight
      // where the paths join.  An index past the end is clamped and the value then not used.)
      for (int j = sub; j - sub < longest; j += 32) {
        int r[2 * kRuns][RW];
#pragma unroll
        for (int i = 0; i < 2 * kRuns; ++i) {
          const int k = max(min(j + 16 * (i & 1), cnt[i / 2] - 1), 0);
#pragma unroll
          for (int w = 0; w < RW; ++w) r[i][w] = at[i / 2][k * RW + w];
        }
#pragma unroll
        for (int i = 0; i < 2 * kRuns; ++i)
          if (j + 16 * (i & 1) < cnt[i / 2]) add(r[i]);
      }
    }
    for (int w = 0; w < kGeneralGradBlocks / kWave; ++w) {
      for (unsigned long long m = s_long[w]; m != 0ull; m &= m - 1) {
        const int blk = w * kWave + __ffsll((long long)m) - 1, cnt = s_run[blk] >> 16;
        const int32_t *const run = run_at(blk);
        constexpr int kTurns = 4;
        for (int j = s_limit[w] + tid; j - tid < cnt; j += kTurns * kApplyThreads) {
          int r[kTurns][RW];
#pragma unroll
          for (int i = 0; i < kTurns; ++i) {
            const int k = min(j + i * kApplyThreads, cnt - 1);
#pragma unroll
            for (int v = 0; v < RW; ++v) r[i][v] = run[k * RW + v];
          }
#pragma unroll
          for (int i = 0; i < kTurns; ++i)
            if (j + i * kApplyThreads < cnt) add(r[i]);
        }
      }
    }
  }
}

// The block that owns a bin.  Everything it needs from memory (the first records and columns
// per thread, in registers) is requested before anything is used: one round trip, not five.
template <int RW>
__device__ __forceinline__ void apply_bin(const ApplyArgs &a, int bin, double *s_bin, int *s_m,
                                          float *s_g, int *s_run, int *s_late,
                                          unsigned long long *s_long) {
  // per thread: kRec records of the first batch, which is requested before the bin's fill count
  // is known (1024 records a bin; with 4096, small pools read megabytes of stale ones); kCol runs
  // of four columns (a bin's columns come in groups of at least four neighbours) --
  // 4 * kCol * kApplyThreads covers any bin of a pass that updates two vectors, and half of the
  // largest bin of one that updates one
  constexpr int kRec = 2, kCol = 2;
  const int tid = threadIdx.x, cols = a.plan.cols, cap = a.plan.seg_cap;
  const int cnt = tid < a.nblk_pass ? a.blk_cnt[tid] : 0;
  const int n_mine = tid < a.nblk_pass ? a.blk_late[tid] : 0;
  // a segment a wave, or one for all
  static_assert(kBinSegments == kApplyWaves, "a segment a wave");
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), segment = a.plan.segments == 1 ? 0 : wave;
  const int first = a.plan.segments == 1 ? tid : tid & 63, turn = a.plan.segments == 1 ? kApplyThreads : kWave;
  const int n = (int)min(a.bin_fill[segment * kMaxBins + bin], (unsigned)cap);
  const int left = left_marks(a.blk_late)[bin];
  const int acc_used = a.acc_used[bin];
  const int32_t *const rec = a.recs + ((size_t)bin * a.plan.segments + segment) * cap * RW;
  int r0[kRec][RW];
  const int batch = kRec * turn;
  // (Every load below is unconditional: a load under a condition makes the compiler wait for
  // all loads in flight where the paths join, and the requests would go out one at a time.
  // An index past the end is clamped to the last record, whose value is then not used.)
  auto load_batch = [&](int (*__restrict__ r)[RW], int base, int last) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kRec; ++u)
#pragma unroll
      for (int w = 0; w < RW; ++w) r[u][w] = rec[(size_t)min(base + first + u * turn, last) * RW + w];
  };
  load_batch(r0, 0, cap - 1);  // past the fill count: stale, in bounds, not used
  int col[kCol];   // first column of the run, -1: none, or not all four exist (the model's end)
  f4v wo[kCol], po[kCol];
  const float *const w_src = a.w ? a.w : a.phi, *const p_src = a.phi ? a.phi : a.w;
#pragma unroll
  for (int u = 0; u < kCol; ++u) {
    const int k = 4 * (tid + u * kApplyThreads);
    int c = bin_column(k, bin, a);
    if (k >= cols || c + 4 > a.d) c = -1;
    col[u] = c;
    const int c_safe = c >= 0 ? c : a.d - 4;  // (bins exist: so do more than four columns)
    wo[u] = *reinterpret_cast<const f4v *>(w_src + c_safe);
    po[u] = *reinterpret_cast<const f4v *>(p_src + c_safe);
  }
  // A bin of few columns keeps several copies of its sums, one per lane residue, so that the
  // lanes of a wave that meet on a hot column add to different addresses (an odd stride puts
  // the copies of a column into different LDS banks).
  const int span = a.nvec * cols + 1;
  int copies = 1;
  while (copies < 16 && 2 * copies * span <= kBinColsMax) copies *= 2;
  double *const s_mine = s_bin + (tid & (copies - 1)) * span;
  for (int k = tid; k < copies * span; k += kApplyThreads) s_bin[k] = 0.0;
  if (tid < kGeneralGradBlocks) {
    int most = n_mine;
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) most = max(most, __shfl_xor(most, off, kWave));
    if ((tid & 63) == 0) s_late[tid >> 6] = most;
  }
  float gb_unused;
  const int m = pass_totals(a, cnt, 0.f, s_m, s_g, &gb_unused);  // barrier: the sums are zero
  const Fold fold(a, m);
  auto add = [&](const int *r) __attribute__((always_inline)) {
    const int k = bin_local(r[0], a);
    const float ta = __int_as_float(r[1]), tb = __int_as_float(r[RW - 1]);
    if (ta != 0.f) unsafeAtomicAdd(s_mine + k, (double)ta);
    if (RW == 3 && tb != 0.f) unsafeAtomicAdd(s_mine + cols + k, (double)tb);
  };
  // The records past the first batch: N neighbouring ones a load, kWide loads a lane, the next ones in flight while
  // these are added up.  (Bins of 21,000: that is what a block's waves need in flight to read them at the rate of memory.)
  constexpr int N = RW == 2 ? 2 : 1, kWide = 4;
  const __amdgpu_buffer_rsrc_t r_bin =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(rec), 0, ((n + 1) & ~1) * (4 * RW), 0x00020000);
  struct Wide {
    int r[kWide][N][RW];
  };
  auto load_wide = [&](int base, Wide &b) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kWide; ++u) {
      const int off = (base + N * (first + u * turn)) * (4 * RW);
      if constexpr (N == 2) {
        const i4v v = __builtin_bit_cast(i4v, __builtin_amdgcn_raw_buffer_load_b128(r_bin, off, 0, 0));
#pragma unroll
        for (int w = 0; w < 4; ++w) b.r[u][w / 2][w % 2] = v[w];
      } else {
        const u3v v = __builtin_bit_cast(u3v, __builtin_amdgcn_raw_buffer_load_b96(r_bin, off, 0, 0));
#pragma unroll
        for (int w = 0; w < RW; ++w) b.r[u][0][w] = (int)v[w];
      }
    }
  };
  auto add_wide = [&](int base, const Wide &b) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kWide; ++u)
#pragma unroll
      for (int k = 0; k < N; ++k)
        if (base + N * (first + u * turn) + k < n) add(b.r[u][k]);
  };
  const int wide = kWide * N * turn;
  Wide b0, b1;
  load_wide(batch, b0);
#pragma unroll
  for (int u = 0; u < kRec; ++u)
    if (first + u * turn < n) add(r0[u]);
  for (int base = batch; base < n; base += 2 * wide) {
    load_wide(base + wide, b1);
    add_wide(base, b0);
    load_wide(base + 2 * wide, b0);
    add_wide(base + wide, b1);
  }
  const int most = max(max(s_late[0], s_late[1]), max(s_late[2], s_late[3]));
  if (most > 0 && left != 0) late_records<RW>(a, bin, n_mine, s_run, s_late, s_long, (most + a.plan.piece - 1) / a.plan.piece, add);
  __syncthreads();
  auto sum_of = [&](int k) {  // over the copies, in order
    double v = 0.0;
    for (int c = 0; c < copies; ++c) v += s_bin[c * span + k];
    return v;
  };
  // (the dense accumulators hold something only if an entry found no room in LDS or in a bin);
  // a column's total is rounded to fp32 once, after everything has been added in doubles
  auto acc_w_of = [&](int c) { return (acc_used && a.w) ? a.acc_w[c] : 0.0; };
  auto acc_p_of = [&](int c) { return (acc_used && a.phi) ? a.acc_p[c] : 0.0; };
  // The runs held in registers, in three sweeps -- sums out of LDS, then (rarely) the
  // accumulators, then nothing but stores: a load between two stores would make every store
  // wait for the one before it to be acknowledged.
  double ga[kCol][4], gp[kCol][4];
#pragma unroll
  for (int u = 0; u < kCol; ++u) {
    if (4 * u * kApplyThreads >= cols) break;  // (no thread has a run this far out)
    const int k = min(4 * (tid + u * kApplyThreads), cols - 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double va = sum_of(k + i), vb = a.nvec == 2 ? sum_of(cols + k + i) : va;
      ga[u][i] = a.w ? va : 0.0;
      gp[u][i] = vb;
    }
  }
  if (acc_used) {
    double *const w_acc = a.w ? a.acc_w : a.acc_p, *const p_acc = a.phi ? a.acc_p : a.acc_w;
    double xa[kCol][4], xp[kCol][4];
#pragma unroll
    for (int u = 0; u < kCol; ++u) {
      const int c_safe = col[u] >= 0 ? col[u] : a.d - 4;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        xa[u][i] = w_acc[c_safe + i];
        xp[u][i] = p_acc[c_safe + i];
      }
    }
#pragma unroll
    for (int u = 0; u < kCol; ++u) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ga[u][i] += a.w ? xa[u][i] : 0.0;
        gp[u][i] += a.phi ? xp[u][i] : 0.0;
      }
    }
    if (a.keep_ready) {  // what was read is cleared for the next pass (this bin's columns only)
#pragma unroll
      for (int u = 0; u < kCol; ++u) {
        if (col[u] < 0) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          w_acc[col[u] + i] = 0.0;
          p_acc[col[u] + i] = 0.0;
        }
      }
    }
  }
#pragma unroll
  for (int u = 0; u < kCol; ++u) {
    if (4 * u * kApplyThreads >= cols) break;
    if (col[u] < 0) continue;
    f4v fa, fp;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      fa[i] = (float)ga[u][i];
      fp[i] = (float)gp[u][i];
    }
    fold.loaded4(col[u], fa, fp, wo[u], po[u]);
  }
  // what is left: runs past the registers' reach, and the model's last columns where fewer
  // than four exist
  for (int k = tid; k < cols; k += kApplyThreads) {
    const int c = bin_column(k, bin, a);
    if (c >= a.d || (k < 4 * kCol * kApplyThreads && (c & ~3) + 4 <= a.d)) continue;
    const double va = sum_of(k), vb = a.nvec == 2 ? sum_of(cols + k) : va;
    fold.column(c, (float)(acc_w_of(c) + (a.w ? va : 0.0)), (float)(acc_p_of(c) + vb));
    if (acc_used && a.keep_ready) {
      if (a.w) a.acc_w[c] = 0.0;
      if (a.phi) a.acc_p[c] = 0.0;
    }
  }
  if (a.keep_ready && tid < kBinSegments) {  // (read at the top; the next pass counts from zero)
    a.bin_fill[tid * kMaxBins + bin] = 0u;
    if (tid == 0) a.acc_used[bin] = left_marks(a.blk_late)[bin] = 0;
  }
}

__global__ __launch_bounds__(kApplyThreads) void k_apply_general(const ApplyArgs a, int nh, int nrest) {
  __shared__ int s_int[40];
  __shared__ float s_part[2][16][kHeadCols];
  __shared__ int s_m[kApplyWaves];
  __shared__ float s_g[kApplyWaves];
  __shared__ double s_bin[kBinColsMax + 1];  // (+1: the odd stride of a single copy)
  __shared__ int s_run[kGeneralGradBlocks], s_late[kGeneralGradBlocks / kWave];
  __shared__ unsigned long long s_long[kGeneralGradBlocks / kWave];
  // roles by block number: the other columns first (the bin owners have the longest way to
  // go), then the first columns, then the compaction tiles
  const int bid = (int)blockIdx.x, hb = bid - nrest;
  if (bid >= nh + nrest) {
    CompactArgs c;
    c.flags = a.flags;
    c.P = a.P;
    c.idx = a.idx;
    c.kept_pos = a.kept_pos;
    c.kept_ids = a.kept_ids;
    c.loss_pool = a.loss_pool;
    c.loss = a.loss;
    c.kept_count = a.kept_count;
    c.tile_off = nullptr;
    tile_compact<kApplyWaves>(c, bid - nh - nrest, s_int);
    return;
  }
  if (bid < nrest && a.plan.nb > 0) {  // nrest == nb
    // Blocks go to the eight XCDs in turn: neighbouring bins, whose columns and records share cache lines, are owned on
    // one XCD.  (In order: the updates of four pools of 65,536 rows over 2^20 columns 64.7 us, so 59.1; three
    // pools of 20,000 rows over 200,000 34.2 and 27.7, of 3000 over 40,000 21.3 and 20.1.)
    const int bin = (nrest & 7) != 0 ? bid : (bid & 7) * (nrest >> 3) + (bid >> 3);
    if (a.nvec == 2)
      apply_bin<3>(a, bin, s_bin, s_m, s_g, s_run, s_late, s_long);
    else
      apply_bin<2>(a, bin, s_bin, s_m, s_g, s_run, s_late, s_long);
    return;
  }
  const int t = threadIdx.x;
  const int cnt = t < a.nblk_pass ? a.blk_cnt[t] : 0;
  const float gbs = (t < a.nblk_pass && a.phi && a.bias) ? a.blk_gb[t] : 0.f;
  if (hb >= 0) {
    const int cl = t % kHeadCols, q = t / kHeadCols;
    const int k = hb * kHeadCols + cl;
    float sw = 0.f, sp = 0.f;
    // (loads without conditions, so that they are all in flight together; with one updated
    // vector both pointers name the same sums and one of the two results is dropped)
    const int k_safe = min(k, a.head - 1);
    {  // (all zeros when nothing was kept)
      const size_t stride = (size_t)a.nvec * a.head;
      const float *pw = a.part + k_safe, *pp = a.part + (a.w ? a.head : 0) + k_safe;
#pragma unroll 8
      for (int b = q; b < a.nblk_pass; b += 16) {
        sw += pw[b * stride];
        sp += pp[b * stride];
      }
    }
    if (!a.w || k >= a.head) sw = 0.f;
    if (!a.phi || k >= a.head) sp = 0.f;
    // (the accumulators take entries of the other columns only)
    float gw = 0.f, gp = 0.f;
    const float wo = (a.w ? a.w : a.phi)[k_safe], po = (a.phi ? a.phi : a.w)[k_safe];
    s_part[0][q][cl] = sw;
    s_part[1][q][cl] = sp;
    float gb_pass;
    const int m = pass_totals(a, cnt, gbs, s_m, s_g, &gb_pass);  // barrier
    const Fold fold(a, m);
    if (hb == 0 && t == 0 && a.kept_hist) *a.kept_hist = m;
    if (hb == 0 && t == 0 && a.t_upd && m > 0) *a.t_upd = *a.t_snap + 1;
    if (q == 0 && k < a.head) {
      for (int i = 0; i < 16; ++i) {
        gw += s_part[0][i][cl];
        gp += s_part[1][i][cl];
      }
      fold.loaded(k, gw, gp, wo, po);
    }
    if (hb == 0 && t == 0 && a.phi && a.bias && m > 0) *a.bias = *a.bias - a.lr_a * (gb_pass * fold.inv_m);
  } else {
    float gb_pass;
    const int m = pass_totals(a, cnt, gbs, s_m, s_g, &gb_pass);
    const Fold fold(a, m);
    for (int k = a.head + bid * blockDim.x + t; k < a.d; k += nrest * blockDim.x)
      fold.column(k, a.w ? (float)a.acc_w[k] : 0.f, a.phi ? (float)a.acc_p[k] : 0.f);
  }
}

// A model that fits a gradient pass's table takes kernels without tags, records and gathers.
template <int GL, bool CSR, int MODE>
void launch_grad(const GenArgs &a, int nblk, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  constexpr bool TWO = (MODE & kSvm) != 0 && (MODE & kAssist) != 0;
  if constexpr (CSR) {
    if (a.d <= (TWO ? kDirectTwoVec : kDirectOneVec)) {
      launch_stamped((k_rows_grad<GL, MODE, true, true>), dim3(nblk), dim3(kGradThreads), st, e0, e1, a);
      return;
    }
  }
  launch_stamped((k_rows_grad<GL, MODE, CSR, false>), dim3(nblk), dim3(kGradThreads), st, e0, e1, a);
}

template <int GL, bool CSR>
hipError_t launch_gl(const GenArgs &a, int mode, int nblk, hipStream_t st, hipEvent_t e0,
                     hipEvent_t e1) {
  switch (mode) {
    case kPool:
      launch_stamped((k_rows_general<GL, CSR>), dim3(nblk), dim3(kPoolThreads), st, e0, e1, a);
      break;
    case kSvm:
      launch_grad<GL, CSR, kSvm>(a, nblk, st, e0, e1);
      break;
    case kAssist:
      launch_grad<GL, CSR, kAssist>(a, nblk, st, e0, e1);
      break;
    case kSvm | kAssist:
      launch_grad<GL, CSR, kSvm | kAssist>(a, nblk, st, e0, e1);
      break;
    case kPool | kSvm | kAssist:
      launch_grad<GL, CSR, kPool | kSvm | kAssist>(a, nblk, st, e0, e1);
      break;
    case kPool | kSvm | kHard:
      launch_grad<GL, CSR, kPool | kSvm | kHard>(a, nblk, st, e0, e1);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

int32_t general_pass_blocks(int32_t count, bool csr, int mode) {
  // Gradient passes flush a private LDS table per block, so they take few, fat blocks (one
  // per compute unit); the scoring pass has no such cost and takes many thin ones.
  const bool grad = (mode & (kSvm | kAssist)) != 0;
  const int waves = (grad ? kGradThreads : kPoolThreads) / kWave;
  const int rows_per_block = waves * (csr ? 4 : 1);
  const int cap = grad ? kGeneralGradBlocks : 256 * 16;
  int64_t want = ((int64_t)count + rows_per_block - 1) / rows_per_block;
  if (want > cap) want = cap;
  if (want < 1) want = 1;
  return (int32_t)want;
}

hipError_t launch_general_pass(const GenArgs &a, int mode, bool csr, int32_t nblk,
                               hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  if (csr && mode == kPool && a.d <= kScoreTableMaxCols &&
      a.count_max >= (a.d > kScoreTableMinCols ? kScoreTableMinRows : kScoreTableManyRows)) {
    if (a.val)
      launch_stamped(k_score_table<true>, dim3(kGeneralGradBlocks), dim3(kScoreTableThreads), st, e0, e1, a);
    else
      launch_stamped(k_score_table<false>, dim3(kGeneralGradBlocks), dim3(kScoreTableThreads), st, e0, e1, a);
    return hipGetLastError();
  }
  if (csr) return launch_gl<16, true>(a, mode, nblk, st, e0, e1);
  return launch_gl<64, false>(a, mode, nblk, st, e0, e1);
}

hipError_t launch_prepare_general(float *p, size_t count, const float *w, const float *phi,
                                  float2 *wp, int32_t head, int32_t d, hipStream_t st) {
  if ((reinterpret_cast<uintptr_t>(p) & 15) != 0 || (reinterpret_cast<uintptr_t>(wp) & 7) != 0)
    return hipErrorInvalidValue;
  const size_t work = count / 4 > (size_t)d ? count / 4 : (size_t)d;
  size_t blocks = (work + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_prepare_general, dim3((unsigned)blocks), dim3(256), 0, st, p, count, w, phi,
                     wp, head, d);
  return hipGetLastError();
}

hipError_t launch_zero_f32(float *p, size_t count, hipStream_t st) {
  if (count == 0) return hipSuccess;
  if ((reinterpret_cast<uintptr_t>(p) & 15) != 0) return hipErrorInvalidValue;
  size_t blocks = (count / 4 + 255) / 256;
  if (blocks > 2048) blocks = 2048;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_zero_f32, dim3((unsigned)blocks), dim3(256), 0, st, p, count);
  return hipGetLastError();
}

bool general_keeps_ready(int32_t d, int nvec, bool csr) {
  return general_bin_plan(d, general_head_columns(d, nvec, csr), nvec, 1, 1).nb > 0;
}

int32_t general_head_columns(int32_t d, int nvec, bool csr) {
  const int direct = nvec == 2 ? (csr ? kDirectTwoVec : kDirectTwoVecDense) : kDirectOneVec;
  return d < direct ? d : direct;
}

hipError_t launch_general_apply(const ApplyArgs &a, hipStream_t st) {
  const int nh = (a.head + kHeadCols - 1) / kHeadCols;
  int nrest = (a.d - a.head + 1023) / 1024;
  if (nrest > 1024) nrest = 1024;
  if (nrest < 0) nrest = 0;
  if (a.plan.nb > 0) nrest = a.plan.nb;
  if (nh + nrest < 1) nrest = 1;
  hipLaunchKernelGGL(k_apply_general, dim3(nh + nrest + (a.flags ? compact_tiles(a.P) : 0)), dim3(kApplyThreads),
                     0, st, a, nh, nrest);
  return hipGetLastError();
}

}  // namespace aa

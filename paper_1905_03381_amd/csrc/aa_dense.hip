// Dense row passes for gfx950.
//
// One wave64 (or an aligned group of LPR lanes for short rows) owns a feature
// row: each lane loads VPL 128-bit pieces, so a wave-wide load instruction
// covers 1 KiB of contiguous row.  A wave owns a contiguous chunk of the pool,
// so row ids, labels and the Philox draws are produced 64 at a time, one per
// lane, and broadcast per row.  All loads of up to RIF rows are issued before
// the first is consumed (at the dense configuration a wave's whole share of the
// pool is in flight at once); phi and w are staged in LDS once per block; dot
// products are folded with DPP row operations and lane reads (no LDS traffic);
// the gradient sums of the kept rows accumulate per lane in registers and are
// combined per block in LDS in a fixed order.
#include "aa_batching.hpp"
#include "aa_compact.hpp"
#include "aa_dense.hpp"

#include <type_traits>

// Feature rows are read once per step: non-temporal loads keep them from displacing the
// model vectors and block partials in L2.
#ifndef AA_ROW_LOAD
#define AA_ROW_LOAD(p) __builtin_nontemporal_load(p)
#endif

namespace aa {

namespace {

__device__ __forceinline__ int wave_sum_int(int v) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

// Phase time stamps of measurement builds (compiled out otherwise).
#ifdef AA_PHASE_TRACE
#define AA_STAMP(k) (t_stamp[k] = (unsigned long long)wall_clock64())
#else
#define AA_STAMP(k) ((void)0)
#endif

// Per-lane sums of one wave into its own LDS slot (row groups folded first).
// Slot layout: red[(wave * NVEC + vec) * ROW4 + column].
template <int LPR, int VPL>
__device__ __forceinline__ void wave_slot_store(f4 (&acc)[VPL], f4 *slot, int lane) {
  if (LPR < kWave) {
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
      acc[v].x = fold_groups<LPR>(acc[v].x);
      acc[v].y = fold_groups<LPR>(acc[v].y);
      acc[v].z = fold_groups<LPR>(acc[v].z);
      acc[v].w = fold_groups<LPR>(acc[v].w);
    }
  }
  if (lane < LPR) {
#pragma unroll
    for (int v = 0; v < VPL; ++v) slot[v * LPR + lane] = acc[v];
  }
}

template <int LPR, int VPL, int MODE, int NW, int RIF>
__global__ __launch_bounds__(NW * 64)
    __attribute__((amdgpu_waves_per_eu((MODE & 3) ? 4 : 1, (MODE & 3) ? 4 : 8))) void k_rows_pass(const PassArgs a) {
  constexpr bool POOL = (MODE & kPool) != 0;
  constexpr bool SVM = (MODE & kSvm) != 0;
  constexpr bool ASSIST = (MODE & kAssist) != 0;
  constexpr bool HARD = (MODE & kHard) != 0;  // keep by the row's own loss, no Assistant
  constexpr bool GRAD = SVM || ASSIST;
  constexpr bool NEED_PHI = (POOL && !HARD) || ASSIST;
  constexpr int G = kWave / LPR;  // rows per wave iteration
  constexpr int ROW4 = LPR * VPL;
  constexpr int NVEC = (SVM ? 1 : 0) + (ASSIST ? 1 : 0);
  constexpr int NT = NW * 64;
  constexpr int STG = (ROW4 + NT - 1) / NT;  // staged 128-bit pieces per thread and vector

  __shared__ int s_int[20];
  __shared__ float s_flt[20];
  __shared__ int s_carry[NW];
  __shared__ f4 s_w[SVM ? ROW4 : 1];
  __shared__ f4 s_phi[NEED_PHI ? ROW4 : 1];
  __shared__ f4 s_red[GRAD ? NW * NVEC * ROW4 : 1];  // one slot per wave and vector

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int grp = lane / LPR, sub = lane % LPR;
  const f4 zero4 = {0.f, 0.f, 0.f, 0.f};

  int total = a.count_max;
  if (!POOL && a.m_dev) total = min(max(*a.m_dev, 0), a.count_max);

  // balanced contiguous chunk of rows for this wave
  const int nwaves = gridDim.x * NW, gwave = blockIdx.x * NW + wave;
  const int per = total / nwaves, rem = total % nwaves;
  const int lo = gwave * per + min(gwave, rem);
  const int hi = lo + per + (gwave < rem ? 1 : 0);

  // ---- start-up, ordered so that the row loads leave as early as possible:
  // row ids of the first 64 rows, model vectors into registers, first rows,
  // labels and draws, then the model vectors into LDS behind one barrier.
  int base = lo;
  int cnt = min(kWave, hi - base);  // rows of the current group of up to 64 (<= 0: none)
  int row_l = 0;
  if (lane < cnt) row_l = a.rows ? a.rows[base + lane] : base + lane;

  f4 st_w[STG], st_p[STG];
#pragma unroll
  for (int q = 0; q < STG; ++q) {
    const int c = q * NT + threadIdx.x;
    st_w[q] = (SVM && c < a.d4) ? reinterpret_cast<const f4 *>(a.w)[c] : zero4;
    st_p[q] = (NEED_PHI && c < a.d4) ? reinterpret_cast<const f4 *>(a.phi)[c] : zero4;
  }
  const float b = (NEED_PHI && a.bias) ? *a.bias : 0.f;
  const float T = (ASSIST || HARD) ? *a.T : 0.f;

  f4 x[RIF][VPL];
  // Every load of the next RIF rows, before any is used.  When the row fills the lane layout
  // (d4 == ROW4) the loads are unconditional: a slot past the end of the group re-reads the
  // group's last row (a cache hit) and is never consumed, so the loads carry no branches.
  const bool full = a.d4 == ROW4;
  // (The two cases are two loops, not one loop with a case inside: the compiler would share
  // code between them, and with it the waits that the conditional loads need.)
  auto issue_rows = [&](int it0) {
    if (full) {
#pragma unroll
      for (int r = 0; r < RIF; ++r) {
        const int li = (it0 + r) * G + grp;
        const int row = __shfl(row_l, min(li, cnt - 1), kWave);
        const f4 *xr = reinterpret_cast<const f4 *>(a.x + (int64_t)row * a.ld);
#pragma unroll
        for (int v = 0; v < VPL; ++v) x[r][v] = AA_ROW_LOAD(xr + v * LPR + sub);
      }
    } else {
#pragma unroll
      for (int r = 0; r < RIF; ++r) {
        const int li = (it0 + r) * G + grp;
        const int row = __shfl(row_l, li & 63, kWave);
        const f4 *xr = reinterpret_cast<const f4 *>(a.x + (int64_t)row * a.ld);
#pragma unroll
        for (int v = 0; v < VPL; ++v) {
          const int c = v * LPR + sub;
          x[r][v] = (li < cnt && c < a.d4) ? AA_ROW_LOAD(xr + c) : zero4;
        }
      }
    }
  };
  float y_l = 0.f, u_l = 2.f, lin_l = 0.f;
  auto lane_inputs = [&]() {  // one row per lane: label, draw, incoming loss
    y_l = 0.f;
    u_l = 2.f;
    lin_l = 0.f;
    if (lane < cnt) {
      if (SVM) y_l = a.y[row_l];
      if (POOL && a.do_keep) u_l = keep_uniform(a.key, (uint32_t)(base + lane));
      if (ASSIST && !SVM) lin_l = a.loss_in[base + lane];
    }
  };
  if (cnt > 0) {
    issue_rows(0);
    lane_inputs();
  }
  // Carried compaction of the previous pool: its loads leave behind the first rows, the
  // count of the flags before this block's 64 positions rides on the start-up barrier,
  // and the last wave places the survivors while the rows are still arriving.
  const bool carry = POOL && GRAD && a.prev.flags != nullptr && (int)blockIdx.x * kWave < a.prev.P;
  int carry_cnt = 0, carry_id = 0;
  uint8_t carry_flag = 0;
  float carry_loss = 0.f;
  if (POOL && GRAD && carry) {
    const int j0 = blockIdx.x * kWave;
    const uint4 *p16 = reinterpret_cast<const uint4 *>(a.prev.flags);
    for (int q = threadIdx.x; q < (j0 >> 4); q += NT) {
      const uint4 v = p16[q];
      carry_cnt += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);  // bytes are 0 or 1
    }
    if (wave == NW - 1 && j0 + lane < a.prev.P) {
      carry_flag = a.prev.flags[j0 + lane];
      carry_id = a.prev.idx ? a.prev.idx[j0 + lane] : j0 + lane;
      if (a.prev.loss) carry_loss = a.prev.loss_pool[j0 + lane];
    }
  }
#pragma unroll
  for (int q = 0; q < STG; ++q) {
    const int c = q * NT + threadIdx.x;
    if (c < ROW4) {
      if (SVM) s_w[c] = st_w[q];
      if (NEED_PHI) s_phi[c] = st_p[q];
    }
  }
  if (POOL && GRAD && carry) {
    carry_cnt = wave_sum_int(carry_cnt);
    if (lane == 0) s_carry[wave] = carry_cnt;
  }
  __syncthreads();
  if (POOL && GRAD && carry && wave == NW - 1) {
    int before = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) before += s_carry[i];
    const unsigned long long mask = __ballot(carry_flag != 0);
    if (carry_flag != 0) {
      const int pos = before + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
      if (a.prev.kept_pos) a.prev.kept_pos[pos] = blockIdx.x * kWave + lane;
      if (a.prev.kept_ids) a.prev.kept_ids[pos] = carry_id;
      if (a.prev.loss) a.prev.loss[pos] = carry_loss;
    }
    if (lane == 0 && a.prev.kept_count && (int)(blockIdx.x + 1) * kWave >= a.prev.P)
      *a.prev.kept_count = before + __popcll(mask);
  }

  f4 gw[VPL], gp[VPL];
#pragma unroll
  for (int v = 0; v < VPL; ++v) {
    gw[v] = zero4;
    gp[v] = zero4;
  }
  float gb = 0.f;
  int kept = 0;
  int it0 = 0;

  while (cnt > 0) {
    const int iters = (cnt + G - 1) / G;
#pragma unroll
    for (int r = 0; r < RIF; ++r) {
      const int it = it0 + r;
      if (it >= iters) break;
      const int li = it * G + grp;
      const bool live = li < cnt;
      const int j = base + li;
      float g = 0.f;
      bool keep = live;
      if (NEED_PHI) {
        float dp = 0.f;
#pragma unroll
        for (int v = 0; v < VPL; ++v) dp = dot4(x[r][v], s_phi[v * LPR + sub], dp);
        dp = row_group_sum<LPR>(dp, lane);
        const float s = dp + b;
        g = sigmoidf_(s);
        if (POOL) {
          const float u = __shfl(u_l, li & 63, kWave);
          if (a.do_keep) keep = live && keep_decision(u, g, a.gamma, a.one_minus_gamma);
          if (sub == 0 && live) {
            if (a.logit) a.logit[j] = s;
            if (a.prob) a.prob[j] = g;
            if (a.flags) a.flags[j] = keep ? 1 : 0;
          }
        }
      }
      if (GRAD) {
        const float yy = SVM ? __shfl(y_l, li & 63, kWave) : 0.f;
        const float lin = (ASSIST && !SVM) ? __shfl(lin_l, li & 63, kWave) : 0.f;
        float loss = lin;
        if (SVM) {
          float dw = 0.f;
#pragma unroll
          for (int v = 0; v < VPL; ++v) dw = dot4(x[r][v], s_w[v * LPR + sub], dw);
          dw = row_group_sum<LPR>(dw, lane);
          const float marg = yy * dw;
          loss = fmaxf(0.f, 1.f - marg);
          if (HARD) {  // shrinking by the objective value itself
            keep = live && loss > T;
            if (sub == 0 && live && a.flags) a.flags[j] = keep ? 1 : 0;
          }
          if (sub == 0 && (HARD ? live : keep) && a.loss_out) a.loss_out[j] = loss;
          const float cw = (keep && marg < 1.f) ? yy : 0.f;  // -d hinge / d margin, times y
#pragma unroll
          for (int v = 0; v < VPL; ++v) gw[v] = axpy4(cw, x[r][v], gw[v]);
        }
        if (ASSIST) {
          const float z = loss > T ? 1.f : 0.f;       // label: Boss loss above the threshold
          const float resid = keep ? g - z : 0.f;     // d cross-entropy / d logit
#pragma unroll
          for (int v = 0; v < VPL; ++v) gp[v] = axpy4(resid, x[r][v], gp[v]);
          if (sub == 0) gb += resid;
        }
        if (sub == 0 && keep) kept += 1;
      }
    }
    // next rows: the same group of 64, or the next group
    it0 += RIF;
    if (it0 >= iters) {
      it0 = 0;
      base += kWave;
      cnt = min(kWave, hi - base);
      if (cnt > 0) {
        row_l = lane < cnt ? (a.rows ? a.rows[base + lane] : base + lane) : 0;
        issue_rows(0);
        lane_inputs();
      }
    } else {
      issue_rows(it0);
    }
  }

  if (GRAD) {
    // Block reduction behind a single barrier: every wave drops its sums into its own LDS
    // slot as soon as its rows are done, then one thread per 128-bit column adds the
    // slots in wave order and stores the block's partial vectors.
    f4 *slot = s_red + wave * NVEC * ROW4;
    if (SVM) wave_slot_store<LPR, VPL>(gw, slot, lane);
    if (ASSIST) wave_slot_store<LPR, VPL>(gp, slot + (SVM ? ROW4 : 0), lane);
    const int kw = wave_sum_int(kept);
    const float gbw = group_sum<kWave>(gb);
    if (lane == 0) {
      s_int[wave] = kw;
      s_flt[wave] = gbw;
    }
    __syncthreads();
    f4 *part = reinterpret_cast<f4 *>(a.partial) + (size_t)blockIdx.x * NVEC * ROW4;
    for (int c = threadIdx.x; c < NVEC * ROW4; c += NT) {
      f4 t = s_red[c];
#pragma unroll
      for (int q = 1; q < NW; ++q) t += s_red[q * NVEC * ROW4 + c];
      part[c] = t;
    }
    if (threadIdx.x == 0) {
      int ks = 0;
      float gs = 0.f;
      for (int i = 0; i < NW; ++i) {
        ks += s_int[i];
        gs += s_flt[i];
      }
      a.blk_cnt[blockIdx.x] = ks;
      a.blk_gb[blockIdx.x] = gs;
    }
  }
  if (GRAD && a.t_upd && blockIdx.x == 0 && threadIdx.x == 0) *a.t_snap = *a.t_upd;
}

// A small batch of rows already chosen (at most kRankSelectMax): one row per lane group, no loop.
// Nothing but round trips bounds it: the row count, then the ids and losses, then the rows.  Each
// is requested for all it depends on at once and without a condition; the model goes straight to
// the registers of the lanes that use it (no barrier in front of the rows).
//
// kAssist alone can take its labels against the running threshold AFTER this batch (med_init):
// every block finds the batch's two middle losses for itself while its rows are on their way.
// sorted[k] is the largest loss with at most k losses below it, so a loss only has to count the
// smaller ones: two instructions per pair, half of the pairs per thread for up to 256 losses.
// Measured on 256 rows of 512 floats: k_rows_pass 12.6 us, this 6.1 us.
template <int LPR, int VPL, int MODE, int NW>
__global__ __launch_bounds__(NW * 64) void k_rows_once(const PassArgs a) {
  constexpr bool SVM = (MODE & kSvm) != 0;
  constexpr bool ASSIST = (MODE & kAssist) != 0;
  constexpr int G = kWave / LPR;  // rows per wave
  constexpr int ROW4 = LPR * VPL;
  constexpr int NVEC = (SVM ? 1 : 0) + (ASSIST ? 1 : 0);
  constexpr int NT = NW * 64;
  constexpr bool MEDIAN = ASSIST && !SVM;
  static_assert(NT >= kRankSelectMax, "a loss per thread");

  __shared__ int s_int[NW];
  __shared__ float s_flt[NW];
  __shared__ f4 s_red[NW * NVEC * ROW4];  // one slot per wave and vector
  __shared__ __attribute__((aligned(16))) float s_med[MEDIAN ? kRankSelectMax : 1];
  __shared__ int s_below[MEDIAN ? kRankSelectMax : 1];
  __shared__ int s_key[MEDIAN ? 2 * NW : 1];
  __shared__ int s_nan[MEDIAN ? NW : 1];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int grp = lane / LPR, sub = lane % LPR;
  const f4 zero4 = {0.f, 0.f, 0.f, 0.f};

  const int m_given = *a.m_dev;
  const float *const model = SVM ? a.w : a.phi;
  f4 mw[SVM ? VPL : 1], mp[ASSIST ? VPL : 1];
#pragma unroll
  for (int v = 0; v < VPL; ++v) {  // (columns past the row are cleared below, with the row's)
    const int c = min(v * LPR + sub, a.d4 - 1);
    if (SVM) mw[v] = reinterpret_cast<const f4 *>(a.w)[c];
    if (ASSIST) mp[v] = reinterpret_cast<const f4 *>(a.phi)[c];
  }
  float b = ASSIST ? *(a.bias ? a.bias : a.phi) : 0.f;
  if (!a.bias) b = 0.f;
  float T = ASSIST ? *a.T : 0.f;
  const bool median = MEDIAN && a.med_init != nullptr;
  const int med_init_old = *(median ? a.med_init : a.m_dev);
  if (a.t_upd && blockIdx.x == 0 && tid == 0) *a.t_snap = *a.t_upd;

  const int total = min(max(m_given, 0), a.count_max);
  if (total == 0) return;  // (an empty batch updates nothing: no sum of this pass is used)
  const int last = total - 1;
  const int pos = (blockIdx.x * NW + wave) * G + grp;
  const bool keep = pos <= last;
  const int at = min(pos, last);  // (a group past the end re-reads the last row and drops it)
  int row = a.rows ? a.rows[at] : at;
  float lin = MEDIAN ? a.loss_in[at] : 0.f;
  const int mine = min(tid, last);
  float x_loss = MEDIAN ? (median ? a.loss_in : model)[median ? mine : 0] : 0.f;
  arrived(row);
  const float yy = SVM ? a.y[row] : 0.f;
  const f4 *xr = reinterpret_cast<const f4 *>(a.x + (int64_t)row * a.ld);
  f4 x[VPL];
#pragma unroll
  for (int v = 0; v < VPL; ++v) x[v] = AA_ROW_LOAD(xr + min(v * LPR + sub, a.d4 - 1));

  if (median) {
    // (ids and losses were requested before the rows: no wait here is a wait for the rows)
    const int per = total <= kRankSelectMax / 2 ? kRankSelectMax / 2 : kRankSelectMax;
    const int i = tid & (per - 1), part = tid / per, parts = min(NT / per, 2);
    if (tid < kRankSelectMax) s_med[tid] = tid < total ? x_loss : __builtin_inff();
    const unsigned long long nan = __ballot(x_loss != x_loss);
    if (lane == 0) s_nan[wave] = nan != 0ull;
    __syncthreads();
    int has_nan = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) has_nan |= s_nan[q];
    const float v_mine = s_med[i];
    const int n4 = (total + 3) / 4, share = (n4 + parts - 1) / parts;
    int below = 0;
    if (part < parts && i < total) {
      const int end = min(n4, (part + 1) * share);
#pragma unroll 4
      for (int q = part * share; q < end; ++q) {  // 128-bit LDS broadcasts
        const f4 v = *reinterpret_cast<const f4 *>(s_med + 4 * q);
        below += v.x < v_mine ? 1 : 0;
        below += v.y < v_mine ? 1 : 0;
        below += v.z < v_mine ? 1 : 0;
        below += v.w < v_mine ? 1 : 0;
      }
    }
    if (parts == 2) {
      if (part == 1 && i < total) s_below[i] = below;
      __syncthreads();
      if (part == 0 && i < total) below += s_below[i];
    }
    // the largest losses with at most (total - 1) / 2 and total / 2 losses below them, as
    // integers in the order of the floats
    const int bits = __float_as_int(v_mine), key = bits ^ ((bits >> 31) & 0x7fffffff);
    const bool cand = part == 0 && i < total;
    int k_lo = cand && below <= (total - 1) / 2 ? key : (int)0x80000000;
    int k_hi = cand && below <= total / 2 ? key : (int)0x80000000;
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
      k_lo = max(k_lo, __shfl_xor(k_lo, off, kWave));
      k_hi = max(k_hi, __shfl_xor(k_hi, off, kWave));
    }
    if (lane == 0) {
      s_key[wave] = k_lo;
      s_key[NW + wave] = k_hi;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      k_lo = max(k_lo, s_key[q]);
      k_hi = max(k_hi, s_key[NW + q]);
    }
    const float lo_mid = __int_as_float(k_lo ^ ((k_lo >> 31) & 0x7fffffff));
    const float hi_mid = __int_as_float(k_hi ^ ((k_hi >> 31) & 0x7fffffff));
    if (has_nan)
      T = __builtin_nanf("");  // a NaN loss has no rank: the threshold becomes NaN, visibly
    else
      T = running_threshold(lo_mid, hi_mid, total, med_init_old, T, a.med_momentum);
    if (blockIdx.x == 0 && tid == 0) *a.T_next = T;
  }

  if (a.d4 != ROW4) {
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
      if (v * LPR + sub < a.d4) continue;
      x[v] = zero4;
      if (SVM) mw[v] = zero4;
      if (ASSIST) mp[v] = zero4;
    }
  }
  float g = 0.f, loss = lin, cw = 0.f, resid = 0.f;
  if (ASSIST) {
    float dp = 0.f;
#pragma unroll
    for (int v = 0; v < VPL; ++v) dp = dot4(x[v], mp[v], dp);
    g = sigmoidf_(row_group_sum<LPR>(dp, lane) + b);
  }
  if (SVM) {
    float dw = 0.f;
#pragma unroll
    for (int v = 0; v < VPL; ++v) dw = dot4(x[v], mw[v], dw);
    const float marg = yy * row_group_sum<LPR>(dw, lane);
    loss = fmaxf(0.f, 1.f - marg);
    cw = marg < 1.f ? yy : 0.f;  // -d hinge / d margin, times y
    if (sub == 0 && keep && a.loss_out) a.loss_out[pos] = loss;
  }
  if (ASSIST) resid = keep ? g - (loss > T ? 1.f : 0.f) : 0.f;  // label: Boss loss above the threshold
  f4 *slot = s_red + wave * NVEC * ROW4;
  f4 acc[VPL];
  if (SVM) {
#pragma unroll
    for (int v = 0; v < VPL; ++v) acc[v] = keep ? axpy4(cw, x[v], zero4) : zero4;
    wave_slot_store<LPR, VPL>(acc, slot, lane);
  }
  if (ASSIST) {
#pragma unroll
    for (int v = 0; v < VPL; ++v) acc[v] = keep ? axpy4(resid, x[v], zero4) : zero4;
    wave_slot_store<LPR, VPL>(acc, slot + (SVM ? ROW4 : 0), lane);
  }
  const int kw = wave_sum_int(sub == 0 && keep ? 1 : 0);
  const float gbw = group_sum<kWave>(sub == 0 ? resid : 0.f);
  if (lane == 0) {
    s_int[wave] = kw;
    s_flt[wave] = gbw;
  }
  __syncthreads();
  f4 *part = reinterpret_cast<f4 *>(a.partial) + (size_t)blockIdx.x * NVEC * ROW4;
  for (int c = tid; c < NVEC * ROW4; c += NT) {
    f4 t = s_red[c];
#pragma unroll
    for (int q = 1; q < NW; ++q) t += s_red[q * NVEC * ROW4 + c];
    part[c] = t;
  }
  if (tid == 0) {
    int ks = 0;
    float gs = 0.f;
    for (int i = 0; i < NW; ++i) {
      ks += s_int[i];
      gs += s_flt[i];
    }
    a.blk_cnt[blockIdx.x] = ks;
    a.blk_gb[blockIdx.x] = gs;
  }
}

// The gradient passes over rows of more than 128 floats: the whole-step pool pass (score, keep, both
// gradient sums; or the hard-threshold variant) and the Boss / Assistant passes over rows already
// chosen.  FULL: the row fills the 64-lane layout exactly (d == 256 VPL); otherwise a piece past
// the end of the row re-reads its last piece and is masked, so the loads stay unconditional.  A
// wave requests RIF rows at once and
// nothing sits between those requests and their use that the memory pipeline would have to
// finish first: every small load that does not depend on the row ids (model vectors,
// scalars, the flags of the carried compaction) is requested before the ids are waited for,
// the labels right behind the ids, the rows last; the per-row outputs (logit, probability,
// keep flag, loss) are collected one per lane and stored once per group of 64 rows, so no
// store is pending while rows arrive.  Loads return in request order, so row r of a batch
// is consumed as soon as it is there while rows r+1.. are still on their way.
// Without gradient sums (MODE == kPool) it is the generator's half of k_boss_and_draw.
// ANY: rows of any width (at least four floats), stride and address: read in pieces that start at
// any float, the last one ending with the row, and summed in doubles, and a coefficient of zero adds
// nothing whatever the row holds, as in the general kernels.
enum StepRows : int { kFullRows, kPartRows, kAnyRows };

typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));  // (any float address)
typedef uint32_t u4u __attribute__((ext_vector_type(4), aligned(4)));

template <int VPL, int MODE, int NW, int ROWS = kFullRows>
struct StepLds {
  using Acc = std::conditional_t<ROWS == kAnyRows, f64x4, f4>;
  static constexpr bool kGrad = (MODE & (kSvm | kAssist)) != 0;
  static constexpr bool kPhi = ((MODE & kPool) && !(MODE & kHard)) || (MODE & kAssist);
  static constexpr int kVec = ((MODE & kSvm) ? 1 : 0) + ((MODE & kAssist) ? 1 : 0);
  int n[NW];
  float g[NW];
  int carry[NW];
  __attribute__((aligned(16))) f4 w[(MODE & kSvm) ? kWave * VPL : 1];
  f4 phi[kPhi ? kWave * VPL : 1];
  Acc red[kGrad ? NW * kVec * kWave * VPL : 1];  // one slot per wave and vector
};

template <int VPL, int MODE, int ROWS, int NW, int RIF>
__device__ __forceinline__ void step_rows(const PassArgs &a, int bid, int nblk, StepLds<VPL, MODE, NW, ROWS> &lds) {
  constexpr bool FULL = ROWS == kFullRows, ANY = ROWS == kAnyRows;
  using Acc = typename StepLds<VPL, MODE, NW, ROWS>::Acc;
  constexpr bool POOL = (MODE & kPool) != 0;
  constexpr bool SVM = (MODE & kSvm) != 0;
  constexpr bool ASSIST = (MODE & kAssist) != 0;
  constexpr bool HARD = (MODE & kHard) != 0;  // keep by the row's own loss, no Assistant
  constexpr bool GRAD = SVM || ASSIST;
  constexpr bool NEED_PHI = (POOL && !HARD) || ASSIST;
  constexpr int ROW4 = kWave * VPL;
  constexpr int NVEC = (SVM ? 1 : 0) + (ASSIST ? 1 : 0);
  constexpr int NT = NW * 64;
  constexpr int STG = (ROW4 + NT - 1) / NT;
  const float *const model = SVM ? a.w : a.phi;  // (always there)

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const f4 zero4 = {0.f, 0.f, 0.f, 0.f};
#ifdef AA_PHASE_TRACE
  unsigned long long t_stamp[kTraceStamps] = {};
#endif
  AA_STAMP(0);  // entry

  // balanced contiguous chunk of pool positions (or of the rows given) for this wave
  int total = a.count_max;
  if (!POOL) total = min(max(*a.m_dev, 0), a.count_max);
  const int nwaves = nblk * NW, gwave = bid * NW + wave;
  const int per = total / nwaves, rem = total % nwaves;
  const int lo = gwave * per + min(gwave, rem);
  const int hi = lo + per + (gwave < rem ? 1 : 0);

  int base = lo;
  int cnt = min(kWave, hi - base);  // rows of the current group of up to 64 (<= 0: none)

  // ---- Requests that depend on nothing, all unconditional: a load under a condition would
  // make every later wait for an older load a wait for everything (the pending counts of the
  // two paths are merged pessimistically), so absent inputs read a stand-in address (the
  // first 16 bytes of a model vector: it holds four floats at least, at any float address with ANY)
  // and indices are clamped; what was read for nothing is dropped by a select.
  const int32_t *stand_in = reinterpret_cast<const int32_t *>(model);
  const int in_group = min(lane, max(cnt, 1) - 1);
  const bool listed = a.rows != nullptr && cnt > 0;
  int row_l = (listed ? a.rows : stand_in)[listed ? base + in_group : 0];
  if (!a.rows) row_l = base + in_group;
  float lin_l = 0.f;  // Boss losses that come with the rows
  if (ASSIST && !SVM) lin_l = (cnt > 0 ? a.loss_in : model)[cnt > 0 ? base + in_group : 0];

  const bool carry = POOL && GRAD && a.prev.flags != nullptr && bid * kWave < a.prev.P;
  const int cj0 = bid * kWave;     // this block places positions [cj0, cj0 + 64)
  const int n16 = carry ? (cj0 >> 4) : 0;  // 16-byte pieces of flags before them
  const u4u *p16 = n16 > 0 ? reinterpret_cast<const u4u *>(a.prev.flags)
                           : reinterpret_cast<const u4u *>(model);
  u4u carry_v = p16[min((int)threadIdx.x, max(n16, 1) - 1)];
  const int cpos = carry ? min(cj0 + lane, a.prev.P - 1) : 0;
  uint8_t carry_flag = (carry ? a.prev.flags : reinterpret_cast<const uint8_t *>(model))[cpos];
  int carry_id = ((carry && a.prev.idx) ? a.prev.idx : stand_in)[a.prev.idx ? cpos : 0];
  float carry_loss = ((carry && a.prev.loss) ? a.prev.loss_pool : model)[a.prev.loss ? cpos : 0];
  // 128-bit piece c of a row or model vector (ANY: the last one from d - 4 on)
  auto piece_of = [&](const float *v, int c) __attribute__((always_inline)) {
    if (ANY) return (f4)*reinterpret_cast<const f4u *>(v + min(4 * c, a.d - 4));
    return reinterpret_cast<const f4 *>(v)[c];
  };
  f4 st_w[STG], st_p[STG];
#pragma unroll
  for (int q = 0; q < STG; ++q) {
    const int c = min(q * NT + (int)threadIdx.x, FULL ? ROW4 - 1 : a.d4 - 1);
    if (SVM) st_w[q] = piece_of(a.w, c);
    if (NEED_PHI) st_p[q] = piece_of(a.phi, c);
  }
  float b = (NEED_PHI && a.bias ? a.bias : model)[0];
  if (!(NEED_PHI && a.bias)) b = 0.f;
  float T = (ASSIST || HARD) ? *a.T : 0.f;

  // Everything above is there after one memory round trip.  It is all consumed here, before
  // the rows are requested: the model vectors go to LDS, the carried flags are counted, and
  // values only needed later are pinned (arrived()) so that no wait for them can end up
  // behind the row requests, where it would be a wait for the rows.
  arrived(row_l);
  arrived(carry_id);
  arrived(carry_loss);
  arrived(b);
  arrived(T);
  if (ASSIST && !SVM) arrived(lin_l);
  AA_STAMP(1);  // ids, model, scalars, carried flags are there
  int carry_cnt = 0;
  if ((int)threadIdx.x < n16)
    carry_cnt = __popc(carry_v.x) + __popc(carry_v.y) + __popc(carry_v.z) + __popc(carry_v.w);
  if (!carry || cj0 + lane >= a.prev.P || wave != NW - 1) carry_flag = 0;
  if (carry && !a.prev.idx) carry_id = cj0 + lane;
  const unsigned long long carry_mask = __ballot(carry_flag != 0);
  for (int q = threadIdx.x + NT; q < n16; q += NT) {  // previous pools above 16 NT positions
    const u4u v = p16[q];
    carry_cnt += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
  }
#pragma unroll
  for (int q = 0; q < STG; ++q) {
    const int c = q * NT + threadIdx.x;
    if (ANY) {  // (what the last piece shares with the one before it is zero in the row, and has to be here)
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        if (SVM && a.d - 4 + i < 4 * c) st_w[q][i] = 0.f;
        if (NEED_PHI && a.d - 4 + i < 4 * c) st_p[q][i] = 0.f;
      }
    }
    if (c < ROW4) {  // (columns past the row: any finite value would do, the row is zero there)
      if (SVM) lds.w[c] = FULL || c < a.d4 ? st_w[q] : zero4;
      if (NEED_PHI) lds.phi[c] = FULL || c < a.d4 ? st_p[q] : zero4;
    }
  }
  if (carry) {
    carry_cnt = wave_sum_int(carry_cnt);
    if (lane == 0) lds.carry[wave] = carry_cnt;
  }

  // ---- requests that need the ids: the labels, then the rows; nothing is requested after
  // them until they are consumed
  f4 x[RIF][VPL];
  auto issue_rows = [&](int it0) {
#pragma unroll
    for (int r = 0; r < RIF; ++r) {
      // a slot past the end of the group re-reads the group's last row and is never consumed
      const int li = min(it0 + r, cnt - 1);
      const int row = __builtin_amdgcn_readlane(row_l, li);
      const float *xr = a.x + (int64_t)row * a.ld;
#pragma unroll
      for (int v = 0; v < VPL; ++v) {
        const int c = FULL ? v * kWave + lane : min(v * kWave + lane, a.d4 - 1);
        if (ANY)
          x[r][v] = AA_ROW_LOAD(reinterpret_cast<const f4u *>(xr + min(4 * c, a.d - 4)));
        else
          x[r][v] = AA_ROW_LOAD(reinterpret_cast<const f4 *>(xr) + c);
      }
    }
  };
  // The barrier that publishes the model vectors comes before the row requests: the memory
  // pipeline accepts a compute unit's requests only as fast as earlier ones complete, so a
  // barrier behind them would hold every wave until the last wave's requests were accepted.
  __syncthreads();
  AA_STAMP(2);  // past the start-up barrier
  float y_l = 0.f, u_l = 2.f;
  if (cnt > 0) {
    if (SVM) y_l = a.y[row_l];
    issue_rows(0);
    if (POOL && !HARD) u_l = keep_uniform(a.key, (uint32_t)(base + in_group));
  }
  AA_STAMP(3);  // rows requested, draws made
  if (carry && wave == NW - 1) {
    int before = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) before += lds.carry[i];
    const unsigned long long mask = carry_mask;
    if (carry_flag != 0) {
      const int pos = before + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
      if (a.prev.kept_pos) a.prev.kept_pos[pos] = cj0 + lane;
      if (a.prev.kept_ids) a.prev.kept_ids[pos] = carry_id;
      if (a.prev.loss) a.prev.loss[pos] = carry_loss;
    }
    if (lane == 0 && a.prev.kept_count && cj0 + kWave >= a.prev.P)
      *a.prev.kept_count = before + __popcll(mask);
  }

  // ANY: a coefficient of zero adds no zero times infinity.  With hard thresholds, where it is every rejected
  // row's, the row is replaced by zeros; kept rows are passed over by a branch.  (The other way round steps
  // on 200,000 rows of 31 floats took 44.5 us instead of 39.3 and 64.2 instead of 62.5.)
  auto added = [&](float coef, const f4 &row) __attribute__((always_inline)) {
    return !(ANY && HARD) || coef != 0.f ? row : zero4;
  };
  Acc gw[VPL], gp[VPL];
#pragma unroll
  for (int v = 0; v < VPL; ++v) {
    gw[v] = Acc{0, 0, 0, 0};
    gp[v] = Acc{0, 0, 0, 0};
  }
  float gb = 0.f;
  int kept = 0;

  while (cnt > 0) {
    // outputs of the group, one row per lane, stored after its last batch
    float o_logit = 0.f, o_prob = 0.f, o_loss = 0.f;
    int o_keep = 0;
    for (int it0 = 0; it0 < cnt; it0 += RIF) {
#pragma unroll
      for (int r = 0; r < RIF; ++r) {
        const int li = it0 + r;        // wave-uniform
        const bool live = li < cnt;
        const int src = li & 63;
        float g = 0.f, s = 0.f, loss = 0.f;
        bool keep = live;
        if (!FULL) {  // (the layouts double in width: only the second half can lie past the row)
#pragma unroll
          for (int v = VPL / 2; v < VPL; ++v) {
            const int c = v * kWave + lane;
            if (c >= a.d4) x[r][v] = zero4;
            if (ANY) {  // (what the last piece shares with the one before it counts there)
#pragma unroll
              for (int i = 0; i < 3; ++i)
                if (a.d - 4 + i < 4 * c) x[r][v][i] = 0.f;
            }
          }
        }
        if (NEED_PHI) {
          float dp = 0.f;
#pragma unroll
          for (int v = 0; v < VPL; ++v) dp = dot4(x[r][v], lds.phi[v * kWave + lane], dp);
          dp = row_group_sum<kWave>(dp, lane);
          s = dp + b;
          g = sigmoidf_(s);
          if (POOL) keep = live && keep_decision(lane_read(u_l, src), g, a.gamma, a.one_minus_gamma);
        }
        const float yy = SVM ? lane_read(y_l, src) : 0.f;
        if (GRAD && (HARD ? live || ANY : keep)) {
          if (SVM) {
            float dw = 0.f;
#pragma unroll
            for (int v = 0; v < VPL; ++v) dw = dot4(x[r][v], lds.w[v * kWave + lane], dw);
            dw = row_group_sum<kWave>(dw, lane);
            const float marg = yy * dw;
            loss = fmaxf(0.f, 1.f - marg);
            if (HARD) keep = live && loss > T;  // shrinking by the objective value itself
            const float cw = (keep && marg < 1.f) ? yy : 0.f;  // -d hinge / d margin, times y
            if (!ANY || HARD || cw != 0.f) {
#pragma unroll
              for (int v = 0; v < VPL; ++v) gw[v] = axpy4(cw, added(cw, x[r][v]), gw[v]);
            }
          } else {
            loss = lane_read(lin_l, src);
          }
          if (ASSIST) {
            const float z = loss > T ? 1.f : 0.f;    // label: Boss loss above the threshold
            const float resid = g - z;               // d cross-entropy / d logit (kept rows only)
            if (!ANY || resid != 0.f) {
#pragma unroll
              for (int v = 0; v < VPL; ++v) gp[v] = axpy4(resid, x[r][v], gp[v]);
            }
            gb += resid;
          }
          if (keep) kept += 1;
        }
        if (lane == li) {
          o_logit = s;
          o_prob = g;
          o_loss = loss;
          o_keep = keep ? 1 : 0;
        }
#ifdef AA_PHASE_TRACE
        if (t_stamp[4] == 0) AA_STAMP(4);  // first row arrived and used
#endif
      }
      if (it0 + RIF < cnt) issue_rows(it0 + RIF);
    }
    if (lane < cnt) {
      const int j = base + lane;
      if (POOL && !HARD && a.logit) a.logit[j] = o_logit;
      if (POOL && !HARD && a.prob) a.prob[j] = o_prob;
      if (POOL && a.flags) a.flags[j] = (uint8_t)o_keep;
      if (SVM && (HARD || o_keep) && a.loss_out) a.loss_out[j] = o_loss;
    }
    base += kWave;
    cnt = min(kWave, hi - base);
    if (cnt > 0) {
      const int in_next = min(lane, cnt - 1);
      row_l = a.rows ? a.rows[base + in_next] : base + in_next;
      if (SVM) y_l = a.y[row_l];
      if (ASSIST && !SVM) lin_l = a.loss_in[base + in_next];
      issue_rows(0);
      if (POOL && !HARD) u_l = keep_uniform(a.key, (uint32_t)(base + in_next));
    }
  }

  AA_STAMP(5);  // all rows of this wave consumed
  // Block reduction behind a single barrier: every wave drops its sums into its own LDS
  // slot, then one thread per 128-bit column adds the slots in wave order and stores the
  // block's partial vectors.
  if (GRAD) {
    Acc *slot = lds.red + wave * NVEC * ROW4;
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
      if (SVM) slot[v * kWave + lane] = gw[v];
      if (ASSIST) slot[(SVM ? ROW4 : 0) + v * kWave + lane] = gp[v];
    }
    if (lane == 0) {
      lds.n[wave] = kept;
      lds.g[wave] = gb;
    }
    __syncthreads();
    AA_STAMP(6);  // past the reduction barrier
    f4 *part = reinterpret_cast<f4 *>(a.partial) + (size_t)bid * NVEC * ROW4;
    for (int c = threadIdx.x; c < NVEC * ROW4; c += NT) {
      Acc t = lds.red[c];
#pragma unroll
      for (int q = 1; q < NW; ++q) t += lds.red[q * NVEC * ROW4 + c];
      if constexpr (ANY) {  // (partials as wide as the row, rounded up: see PassArgs::d_pad)
        float *out = a.partial + ((size_t)bid * NVEC + c / ROW4) * a.d_pad;
        const int k0 = 4 * (c % ROW4), first = min(k0, a.d - 4);
        if (k0 >= a.d) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (first + i >= k0) out[first + i] = (float)t[i];
      } else {
        part[c] = t;
      }
    }
    if (threadIdx.x == 0) {
      int ks = 0;
      float gs = 0.f;
      for (int i = 0; i < NW; ++i) {
        ks += lds.n[i];
        gs += lds.g[i];
      }
      a.blk_cnt[bid] = ks;
      a.blk_gb[bid] = gs;
    }
  }
  if (GRAD && a.t_upd && bid == 0 && threadIdx.x == 0) *a.t_snap = *a.t_upd;
#ifdef AA_PHASE_TRACE
  AA_STAMP(7);  // partials stored
  if (POOL && GRAD && a.trace && lane == 0) {
    unsigned long long *tr = a.trace + ((size_t)bid * NW + wave) * kTraceStamps;
    for (int k = 0; k < kTraceStamps; ++k) tr[k] = t_stamp[k];
  }
#endif
}

template <int VPL, int MODE, int ROWS, int NW, int RIF>
__global__ __launch_bounds__(NW * 64)
    __attribute__((amdgpu_waves_per_eu(NW / 4, NW / 4))) void k_step_pass(const PassArgs a) {
  __shared__ StepLds<VPL, MODE, NW, ROWS> lds;
  step_rows<VPL, MODE, ROWS, NW, RIF>(a, blockIdx.x, gridDim.x, lds);
}

// One launch for the two halves of a pipeline tick that do not depend on each other: the Boss and
// Assistant pass over the rows of one batch, and the scoring and keep draws of a later pool with
// the Assistant as it stands.  Blocks take turns between the two, so a compute unit works on one of each
// and the memory system sees a launch of both sizes; as two launches on two streams they cost
// the host two more launches, two event records and two waits per tick.  Per tick at d = 1024,
// pools of 16,384, two batches in the queue: 37 us as two, 27 us so (this kernel 20.8 us for
// 106 MB).
template <int VPL, int ROWS, int RIF>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_boss_and_draw(
    const PassArgs boss, const PassArgs gen, int nb_boss, int nb_gen) {
  __shared__ union {
    StepLds<VPL, kSvm | kAssist, 8, ROWS> boss;
    StepLds<VPL, kPool, 8, ROWS> gen;
  } lds;
  const int both = 2 * min(nb_boss, nb_gen), i = blockIdx.x;
  const bool draws = i < both ? (i & 1) != 0 : nb_gen > nb_boss;
  const int bid = i < both ? i >> 1 : i - (both >> 1);
  if (draws)
    step_rows<VPL, kPool, ROWS, 8, RIF>(gen, bid, nb_gen, lds.gen);
  else
    step_rows<VPL, kSvm | kAssist, ROWS, 8, RIF>(boss, bid, nb_boss, lds.boss);
}

#ifndef AA_FIN_COLS4
#define AA_FIN_COLS4 8
#endif
constexpr int kFinCols4 = AA_FIN_COLS4;        // 128-bit columns reduced by one finalize block
constexpr int kFinGroups = 256 / kFinCols4;    // partial groups per column (256 threads)

// Sum the block partials in a fixed order and apply the SGD updates; extra blocks compact
// the keep flags of a pool pass, one tile each.  A reduce block owns kFinCols4 128-bit
// columns of one gradient vector: thread (group g, column c) adds the partials of blocks
// g, g + kFinGroups, ... in that order, the groups of a wave are folded with a fixed
// butterfly, the four wave sums are added in wave order.  One memory round trip (every
// load is requested before any is used) and one barrier.
// TAIL64: the sums of the columns from a.f64_from on are doubles; a block's columns are all of one kind.
template <bool TAIL64>
__global__ __launch_bounds__(256) void k_finalize(const FinalizeArgs a) {
  __shared__ f4 s_acc[4][kFinCols4];
  __shared__ f64x4 s_acc64[TAIL64 ? 4 : 1][kFinCols4];
  __shared__ int s_int[40];
  __shared__ float s_flt[8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row4 = a.d_pad / 4;
  const int per_vec = row4 / kFinCols4;  // reduce blocks per gradient vector
  const int nred = per_vec * a.nvec;

  if ((int)blockIdx.x >= nred) {
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
    tile_compact(c, (int)blockIdx.x - nred, s_int);
    return;
  }

  // vector 0 is the Boss gradient when w is updated, the Assistant's otherwise
  const int vec = blockIdx.x / per_vec;
  const bool boss = a.w != nullptr && vec == 0;
  float *model = boss ? a.w : a.phi;
  const bool bias_block = !boss && (int)blockIdx.x % per_vec == 0 && a.phi && a.bias;
  const int c4 = tid % kFinCols4, pg = tid / kFinCols4;
  const int col4 = ((int)blockIdx.x % per_vec) * kFinCols4 + c4;
  const int k0 = col4 * 4;

  // Every first load is requested before any is used and none sits under a condition (absent
  // inputs read a stand-in address, indices are clamped, what was read for nothing is
  // dropped): the block pays one memory round trip for counts, scalars, model slice and
  // its first eight partials per thread.
  const int nb = a.nblk;
  const int32_t *ints = a.blk_cnt;                       // always present: the stand-in address
  const int ci = min(tid, nb - 1);
  int cnt_part = a.blk_cnt[ci];
  float gb_part = a.blk_gb[ci];
  const int m_given = *(a.m_dev ? a.m_dev : ints);
  int t_old = *(a.t_upd ? a.t_snap : ints);
  float b_new = *(bias_block ? a.bias : a.blk_gb);       // the bias before this update
  const float t_next = *(a.T_next ? a.T_next : a.blk_gb);
  float old[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) old[i] = model[min(k0 + i, a.d - 1)];
  const f4 zero = {0.f, 0.f, 0.f, 0.f};
  f4 acc = zero;
  const f4 *p = reinterpret_cast<const f4 *>(a.partial + (size_t)vec * a.part_row) + col4;
  const size_t stride = (size_t)a.nvec * a.part_row / 4;
  const bool tail = TAIL64 && k0 >= a.f64_from;          // (the same in the whole block)
  f64x4 acc64 = {0., 0., 0., 0.};
  if (tail) {
    const f64x4 *p64 = reinterpret_cast<const f64x4 *>(a.partial + (size_t)vec * a.part_row + a.f64_from) +
                       (k0 - a.f64_from) / 4;
    for (int base = pg; base < nb; base += 8 * kFinGroups) {
      f64x4 v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = p64[(size_t)min(base + j * kFinGroups, nb - 1) * (stride / 2)];
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (base + j * kFinGroups < nb) acc64 += v[j];
    }
  } else {
    for (int base = pg; base < nb; base += 8 * kFinGroups) {
      f4 v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = p[(size_t)min(base + j * kFinGroups, nb - 1) * stride];
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (base + j * kFinGroups < nb) acc += v[j];     // block order within the group
    }
  }
  if (a.m_dev || tid >= nb) cnt_part = 0;
  if (!bias_block || tid >= nb) gb_part = 0.f;
  if (!a.t_upd) t_old = 0;
  if (pg != 0) old[0] = old[1] = old[2] = old[3] = 0.f;
  for (int i = tid + blockDim.x; i < nb; i += blockDim.x) {  // more than 256 partials
    if (!a.m_dev) cnt_part += a.blk_cnt[i];
    if (bias_block) gb_part += a.blk_gb[i];
  }

  // fold the groups of this wave (lanes that share a column), then the four waves
  if (!tail) {
#pragma unroll
    for (int off = kFinCols4; off < kWave; off <<= 1) {
      acc.x += __shfl_xor(acc.x, off, kWave);
      acc.y += __shfl_xor(acc.y, off, kWave);
      acc.z += __shfl_xor(acc.z, off, kWave);
      acc.w += __shfl_xor(acc.w, off, kWave);
    }
    if (lane < kFinCols4) s_acc[wave][lane] = acc;
  } else {
#pragma unroll
    for (int off = kFinCols4; off < kWave; off <<= 1) {
#pragma unroll
      for (int i = 0; i < 4; ++i) acc64[i] += __shfl_xor(acc64[i], off, kWave);
    }
    if (lane < kFinCols4) s_acc64[TAIL64 ? wave : 0][lane] = acc64;
  }
  cnt_part = wave_sum_int(cnt_part);
  gb_part = group_sum<kWave>(gb_part);
  if (lane == 0) {
    s_int[wave] = cnt_part;
    s_flt[wave] = gb_part;
  }
  __syncthreads();
  const int m = a.m_dev ? min(max(m_given, 0), a.m_max) : (s_int[0] + s_int[1]) + (s_int[2] + s_int[3]);

  // step size: constant, or lr / sqrt(number of updates made so far)
  const int t_new = t_old + (m > 0 ? 1 : 0);
  float lr = a.lr;
  if (a.t_upd && m > 0) lr = a.lr / sqrtf((float)t_new);

  float now[4] = {old[0], old[1], old[2], old[3]};
  const bool bias_thread = bias_block && tid == 0;
  if (m > 0) {
    const float inv_m = 1.f / (float)m;
    if (pg == 0) {
      const f4 g = (s_acc[0][c4] + s_acc[1][c4]) + (s_acc[2][c4] + s_acc[3][c4]);
      float gv[4] = {g.x, g.y, g.z, g.w};
      if constexpr (TAIL64) {
        const f64x4 g64 = (s_acc64[0][c4] + s_acc64[1][c4]) + (s_acc64[2][c4] + s_acc64[3][c4]);
#pragma unroll
        for (int i = 0; i < 4; ++i) gv[i] = tail ? (float)g64[i] : gv[i];
      }
      if (boss) {
        const float shrink = 1.f - lr * a.lambda;
        const float scale = lr * inv_m;
#pragma unroll
        for (int i = 0; i < 4; ++i) now[i] = __fmaf_rn(scale, gv[i], shrink * old[i]);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          now[i] = old[i] - a.lr_a * __fmaf_rn(a.l2_a, old[i], gv[i] * inv_m);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (k0 + i < a.d) model[k0 + i] = now[i];
    }
    if (bias_thread) {
      // bias gradient: per-wave sums of the block partials, added in wave order
      const float gb = (s_flt[0] + s_flt[1]) + (s_flt[2] + s_flt[3]);
      b_new = b_new - a.lr_a * (gb * inv_m);
      *a.bias = b_new;
    }
  }
  if (blockIdx.x == 0 && tid == 0 && a.kept_hist) *a.kept_hist = m;
  if (blockIdx.x == 0 && tid == 0 && a.T_next && m > 0) {
    *a.T_out = t_next;
    *a.T_init = 1;
  }
  if (blockIdx.x == 0 && tid == 0 && a.t_upd) *a.t_upd = t_new;
}

int g_num_cu = 0;

int num_cu() {
  if (g_num_cu == 0) {
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
      g_num_cu = prop.multiProcessorCount;
    if (g_num_cu <= 0) g_num_cu = 256;
  }
  return g_num_cu;
}

struct Shape {
  int lpr, vpl;
};

Shape pick_shape(int32_t d) {
  const int d4 = (d + 3) / 4;
  if (d4 <= 16) return {16, 1};
  if (d4 <= 32) return {32, 1};
  if (d4 <= 64) return {64, 1};
  if (d4 <= 128) return {64, 2};
  if (d4 <= 256) return {64, 4};
  return {64, 8};
}

// The gradient passes take k_step_pass on every 64-lane layout.
bool step_pass_ok(const Shape &s, int mode) { return (mode & (kSvm | kAssist)) != 0 && s.lpr == kWave; }

// Waves per block and rows requested at once per wave of k_step_pass; one block per compute unit.
// A batch costs the same whether its slots hold rows or not, and two blocks per compute unit
// twice the partial sums: with 8 rows at once in two blocks of 8 waves, pools of 8192 rows of
// 512 floats took 18.5 us per step (16.3 with hard thresholds), with 4 in one block 10.8 (10.3).
// Per step at d = 512, P = 4096: 2 rows at once 9.3 us, 4 9.8; P = 16,384: 13.8, 13.7; at
// d = 256, P = 40,000 17.5, 15.7.  Rows of 1 KB or less leave a wave idle soonest: from 16,384
// of them on 16 waves (P = 60,000 21.2 us against 23.1, 200,000 48.5 against 55.5; below it
// 8 waves are level or ahead, 9.6 against 10.6 at 8192).
struct StepShape {
  int nw, rif;
};

StepShape step_shape(int vpl, int32_t count) {
  if (vpl == 1 && count > 16384) return {16, 4};
  if (vpl <= 2) return {8, count <= 4096 ? 2 : 4};
  return {8, 2};
}

// The passes over rows of up to 128 floats (several rows per wave) that keep gradient sums: up to
// 8192 rows, two at once per lane group in one block per compute unit; beyond that eight in
// two.  Whole step at d = 128: P = 600 9.2 -> 8.9 us, 8192 11.7 -> 10.1 (hard thresholds 10.3 ->
// 8.8); with two at once and P = 60,000 24.5 us instead of 19.8.
constexpr int32_t kNarrowFewRows = 8192;

// Waves per block.
int waves_per_block(const Shape &s, int32_t count, int mode) {
  const bool grad = (mode & (kSvm | kAssist)) != 0;
  if (!grad) return 4;
  return step_pass_ok(s, mode) ? step_shape(s.vpl, count).nw : 8;
}

template <int LPR, int VPL, int NW, int RIF>
hipError_t launch_grad(const PassArgs &a, int mode, int nblk, hipStream_t st, hipEvent_t e0,
                       hipEvent_t e1) {
  const dim3 grid(nblk), block(NW * 64);
  switch (mode) {
    case kSvm:
      launch_stamped((k_rows_pass<LPR, VPL, kSvm, NW, RIF>), grid, block, st, e0, e1, a);
      break;
    case kAssist:
      launch_stamped((k_rows_pass<LPR, VPL, kAssist, NW, RIF>), grid, block, st, e0, e1, a);
      break;
    case kSvm | kAssist:
      launch_stamped((k_rows_pass<LPR, VPL, kSvm | kAssist, NW, RIF>), grid, block, st, e0, e1, a);
      break;
    case kPool | kSvm | kAssist:
      launch_stamped((k_rows_pass<LPR, VPL, kPool | kSvm | kAssist, NW, RIF>), grid, block, st, e0, e1, a);
      break;
    case kPool | kSvm | kHard:
      launch_stamped((k_rows_pass<LPR, VPL, kPool | kSvm | kHard, NW, RIF>), grid, block, st, e0, e1, a);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int LPR, int VPL, int NW>
hipError_t launch_once(const PassArgs &a, int mode, int nblk, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  const dim3 grid(nblk), block(NW * 64);
  if (mode == kSvm)
    launch_stamped((k_rows_once<LPR, VPL, kSvm, NW>), grid, block, st, e0, e1, a);
  else if (mode == kAssist)
    launch_stamped((k_rows_once<LPR, VPL, kAssist, NW>), grid, block, st, e0, e1, a);
  else
    launch_stamped((k_rows_once<LPR, VPL, kSvm | kAssist, NW>), grid, block, st, e0, e1, a);
  return hipGetLastError();
}

template <int VPL, int ROWS, int NW, int RIF>
hipError_t launch_step_mode(const PassArgs &a, int mode, int nblk, hipStream_t st, hipEvent_t e0,
                            hipEvent_t e1) {
  const dim3 grid(nblk), block(NW * 64);
  switch (mode) {
    case kPool:
      if constexpr (ROWS == kAnyRows) {  // (the others have a scoring pass of their own)
        launch_stamped((k_step_pass<VPL, kPool, ROWS, NW, RIF>), grid, block, st, e0, e1, a);
        break;
      }
      return hipErrorInvalidValue;
    case kSvm:
      launch_stamped((k_step_pass<VPL, kSvm, ROWS, NW, RIF>), grid, block, st, e0, e1, a);
      break;
    case kAssist:
      launch_stamped((k_step_pass<VPL, kAssist, ROWS, NW, RIF>), grid, block, st, e0, e1, a);
      break;
    case kSvm | kAssist:
      launch_stamped((k_step_pass<VPL, kSvm | kAssist, ROWS, NW, RIF>), grid, block, st, e0, e1, a);
      break;
    case kPool | kSvm | kAssist:
      launch_stamped((k_step_pass<VPL, kPool | kSvm | kAssist, ROWS, NW, RIF>), grid, block, st, e0, e1, a);
      break;
    case kPool | kSvm | kHard:
      launch_stamped((k_step_pass<VPL, kPool | kSvm | kHard, ROWS, NW, RIF>), grid, block, st, e0, e1, a);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Rows that fill the layout have kernels without masks: with those of the others d = 256, 40,000 rows took
// 17.2 us per step instead of 16.8, d = 512, 16,384 13.1 / 12.4, d = 1024, 16,384 16.9 / 16.1 (262,144 the
// same), d = 2048, 8192 17.9 / 17.1.
template <int VPL, int NW, int RIF>
hipError_t launch_step(const PassArgs &a, int mode, int nblk, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  return a.d4 == kWave * VPL ? launch_step_mode<VPL, kFullRows, NW, RIF>(a, mode, nblk, st, e0, e1)
                             : launch_step_mode<VPL, kPartRows, NW, RIF>(a, mode, nblk, st, e0, e1);
}

template <int LPR, int VPL, int RIF>
hipError_t launch_pool(const PassArgs &a, int nblk, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  launch_stamped((k_rows_pass<LPR, VPL, kPool, 4, RIF>), dim3(nblk), dim3(256), st, e0, e1, a);
  return hipGetLastError();
}

}  // namespace

bool dense_fast_ok(const aa_features *F) {
  return F->layout == AA_DENSE && F->d % 4 == 0 && F->d <= kFastDenseMaxD && F->ld % 4 == 0 &&
         (reinterpret_cast<uintptr_t>(F->x) & 15) == 0;
}

int32_t dense_d_pad(int32_t d) {
  const Shape s = pick_shape(d);
  return s.lpr * s.vpl * 4;
}

int32_t dense_pass_blocks(int32_t d, int32_t count, int mode) {
  const Shape s = pick_shape(d);
  const int nw = waves_per_block(s, count, mode);
  const int rows_per_block = nw * (kWave / s.lpr);
  const bool grad = (mode & (kSvm | kAssist)) != 0;
  int64_t want = ((int64_t)count + rows_per_block - 1) / rows_per_block;
  // a small batch of chosen rows: a lane group for each row, however few compute units there are
  if (grad && !(mode & kPool) && count <= kRankSelectMax) return want < 1 ? 1 : (int32_t)want;
  // one block per compute unit, two for many narrow rows; the scoring pass has no sums to leave
  const bool one_per_cu = step_pass_ok(s, mode) || count <= kNarrowFewRows;
  const int64_t cap = (int64_t)num_cu() * (!grad ? 8 : one_per_cu ? 1 : 2);
  if (want > cap) want = cap;
  if (want > kMaxBlocks) want = kMaxBlocks;
  if (want < 1) want = 1;
  return (int32_t)want;
}

hipError_t launch_dense_pass(const PassArgs &a, int mode, int32_t d, int32_t nblk,
                             hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  const Shape s = pick_shape(d);
  if (mode == kPool) {
    if (s.lpr == 16) return launch_pool<16, 1, 4>(a, nblk, st, e0, e1);
    if (s.lpr == 32) return launch_pool<32, 1, 4>(a, nblk, st, e0, e1);
    switch (s.vpl) {
      case 1: return launch_pool<64, 1, 4>(a, nblk, st, e0, e1);
      case 2: return launch_pool<64, 2, 4>(a, nblk, st, e0, e1);
      case 4: return launch_pool<64, 4, 2>(a, nblk, st, e0, e1);
      default: return launch_pool<64, 8, 2>(a, nblk, st, e0, e1);
    }
  }
  // rows already chosen, a lane group for each: the pass without a loop
  if (!(mode & kPool) && a.count_max <= kRankSelectMax) {
    if ((int64_t)nblk * waves_per_block(s, a.count_max, mode) * (kWave / s.lpr) < a.count_max) return hipErrorInvalidValue;
    if (s.lpr == 16) return launch_once<16, 1, 8>(a, mode, nblk, st, e0, e1);
    if (s.lpr == 32) return launch_once<32, 1, 8>(a, mode, nblk, st, e0, e1);
    switch (s.vpl) {
      case 1: return launch_once<64, 1, 8>(a, mode, nblk, st, e0, e1);
      case 2: return launch_once<64, 2, 8>(a, mode, nblk, st, e0, e1);
      case 4: return launch_once<64, 4, 8>(a, mode, nblk, st, e0, e1);
      default: return launch_once<64, 8, 8>(a, mode, nblk, st, e0, e1);
    }
  }
  if (a.med_init) return hipErrorInvalidValue;  // (only the pass above finds a batch's median)
  if (step_pass_ok(s, mode)) {
    const StepShape p = step_shape(s.vpl, a.count_max);
    switch (s.vpl) {
      case 1:
        if (p.nw == 16) return launch_step<1, 16, 4>(a, mode, nblk, st, e0, e1);
        if (p.rif == 2) return launch_step<1, 8, 2>(a, mode, nblk, st, e0, e1);
        return launch_step<1, 8, 4>(a, mode, nblk, st, e0, e1);
      case 2:
        if (p.rif == 2) return launch_step<2, 8, 2>(a, mode, nblk, st, e0, e1);
        return launch_step<2, 8, 4>(a, mode, nblk, st, e0, e1);
      case 4: return launch_step<4, 8, 2>(a, mode, nblk, st, e0, e1);
      // (two rows of 8 KB in flight per wave: with four the hard-threshold variant does not fit
      // its registers -- the compiler then parks every arriving row in scratch, one load at a
      // time, 67 us per step instead of 30 -- and the other is 4 % slower at the register limit)
      default: return launch_step<8, 8, 2>(a, mode, nblk, st, e0, e1);
    }
  }
  const bool few = a.count_max <= kNarrowFewRows;
  if (s.lpr == 16 && few) return launch_grad<16, 1, 8, 2>(a, mode, nblk, st, e0, e1);
  if (s.lpr == 16) return launch_grad<16, 1, 8, 8>(a, mode, nblk, st, e0, e1);
  if (few) return launch_grad<32, 1, 8, 2>(a, mode, nblk, st, e0, e1);
  return launch_grad<32, 1, 8, 8>(a, mode, nblk, st, e0, e1);
}

// Rows of 4 to 1024 floats that are not laid out in 16-byte pieces.  In the general kernel every
// element of theirs was an LDS atomic.  Per step of an epoch at d = 785, pools of 4000: 20.7 us there, 11.2
// here; d = 999, 20,000: 61.5, 22.4; d = 131, 200: 12.7, 8.7.  Single steps of narrow rows, which leave most of a
// wave without a piece: d = 5, 65,536 rows 44.0, 24.3; d = 31, 300 rows 13.4, 8.4, 16,384 19.3, 11.9, 200,000
// 114, 62.6.  Blocks of eight waves with one row each, up to one block per compute unit: 1 to 16
// rows a block are within 7 % from 64 to 4096 rows of 31 to 1023 floats, eight ahead or level.
hipError_t launch_any_rows(const PassArgs &a, int mode, int32_t nblk, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  if (a.d < 4 || a.d > 1024) return hipErrorInvalidValue;
  if (a.d <= 256) return launch_step_mode<1, kAnyRows, 8, 4>(a, mode, nblk, st, e0, e1);
  if (a.d <= 512) return launch_step_mode<2, kAnyRows, 8, 4>(a, mode, nblk, st, e0, e1);
  return launch_step_mode<4, kAnyRows, 8, 2>(a, mode, nblk, st, e0, e1);
}

bool boss_and_draw_ok(int32_t d) {
  const Shape s = pick_shape(d);
  return s.lpr == kWave && s.vpl <= 4;  // (wider: one block's sums fill the LDS of a compute unit)
}

hipError_t launch_boss_and_draw(const PassArgs &boss, const PassArgs &gen, int32_t d, int32_t nb_boss,
                                hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  const Shape s = pick_shape(d);
  if (!boss_and_draw_ok(d) || nb_boss < 1) return hipErrorInvalidValue;
  int nb_gen = (gen.count_max + 15) / 16;  // two rows a wave, up to a block per compute unit
  if (nb_gen > num_cu()) nb_gen = num_cu();
  const dim3 grid(nb_boss + nb_gen), block(512);
  const bool full = boss.d4 == kWave * s.vpl;
  auto go = [&](auto kernel) {
    if (e0 && e1)
      hipExtLaunchKernelGGL(kernel, grid, block, 0, st, e0, e1, 0, boss, gen, (int)nb_boss, nb_gen);
    else
      hipLaunchKernelGGL(kernel, grid, block, 0, st, boss, gen, (int)nb_boss, nb_gen);
    return hipGetLastError();
  };
  switch (s.vpl) {
    case 1: return full ? go(k_boss_and_draw<1, kFullRows, 4>) : go(k_boss_and_draw<1, kPartRows, 4>);
    case 2: return full ? go(k_boss_and_draw<2, kFullRows, 4>) : go(k_boss_and_draw<2, kPartRows, 4>);
    default: return full ? go(k_boss_and_draw<4, kFullRows, 2>) : go(k_boss_and_draw<4, kPartRows, 2>);
  }
}

hipError_t launch_dense_finalize(const FinalizeArgs &a, hipStream_t st) {
  const int nred = a.d_pad / (4 * kFinCols4) * a.nvec;
  const int extra = a.flags ? compact_tiles(a.P) : 0;
  if (a.f64_from < a.d_pad)
    hipLaunchKernelGGL(k_finalize<true>, dim3(nred + extra), dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL(k_finalize<false>, dim3(nred + extra), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace aa

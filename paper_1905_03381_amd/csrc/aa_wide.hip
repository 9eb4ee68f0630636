// Wide dense rows: more columns than a wave can hold sums for in registers (d > 2048), and
// rows of 1025 to 2048 columns with a width, leading dimension or base address that is not a
// multiple of 16 bytes.  A block of 8 waves owns a row, each thread the same columns of every
// row: it keeps those columns of the model and of the gradient sums in registers for the whole
// launch, so a row crosses memory once and no sum needs an atomic or a trip through LDS.
//
// What bounds it: HBM.  Only the dot products cross threads: one value per wave, row and
// vector goes through LDS, one barrier per R rows, while the next R rows are in flight in a
// second set of registers.
#include "aa_wide.hpp"

namespace aa {

namespace {

typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));  // (any float address)

constexpr int kWideWaves = 8, kWideThreads = kWideWaves * kWave;

// Thread t owns the 128-bit pieces t, t + 512, ... of a row.  The last piece of a row whose
// width is not a multiple of four is read from d - 4 on and a piece past the end likewise:
// every load is a whole one, in bounds and without a condition.  Columns such a piece shares
// with the one before are masked to zero, in the rows and in the model.
//
// The gradient sums are doubles (fp64 FMAs run at the fp32 rate here and the pass waits for memory),
// rounded once per block; with two vectors those of the columns from kWideFp32Cols on stay doubles
// until the update kernel has added all blocks up.  That is what the general kernels keep of dense
// rows: the LDS of a block there holds sums of 8192 columns of one vector or 4096 of two, which leave it as
// floats, and everything past them is added in doubles.  (Whole steps with the doubles against all sums
// rounded per block: d = 4137, 4096 rows 22.5 -> 22.9 us, d = 8000 34.7 -> 36.7, 512 rows 16.2 -> 18.7.)
//
// VPT pieces of R rows, twice, are in registers: 4 rows of 17 KB at d = 4137, so that about 130 KB of a
// compute unit's rows are on their way at a time.  Measured: epochs of 4 pools of 4096 rows (the
// general kernels' times in brackets, whose sums go through LDS and sorted records): d = 2052 66 us
// (138), 4093 90 (223), 4137 97 (245), 6145 126 (900), 8000 149 (1475) = 3.5 TB/s of rows; the pass alone
// at d = 4137 19.4 us (53).  Scalars per row -- sigmoid,
// draw, loss -- are worked out for all R rows at once, a row per eight lanes: done row by row in
// every lane they took longer than the dot products (22.0 us).
template <int VPT, int R, int MODE, bool NT = true>
__global__ __launch_bounds__(kWideThreads)
    __attribute__((amdgpu_waves_per_eu(2, 2))) void k_wide_pass(const PassArgs a) {
  constexpr bool POOL = (MODE & kPool) != 0;
  constexpr bool SVM = (MODE & kSvm) != 0;
  constexpr bool ASSIST = (MODE & kAssist) != 0;
  constexpr bool HARD = (MODE & kHard) != 0;  // keep by the row's own loss, no Assistant
  constexpr bool GRAD = SVM || ASSIST;
  constexpr bool NEED_PHI = (POOL && !HARD) || ASSIST;
  constexpr int NVEC = (SVM ? 1 : 0) + (ASSIST ? 1 : 0);
  constexpr int NDOT = (SVM ? 1 : 0) + (NEED_PHI ? 1 : 0);
  constexpr int Q = NDOT * R;  // dot products per batch
  constexpr int kDotW = NEED_PHI ? R : 0;  // the Boss's dots come after the Assistant's
  constexpr int kDotStride = 4 * kWideWaves + 4;
  static_assert(Q <= 16 && 8 * R <= kWave, "a lane of 16 per dot, eight lanes per row");

  __shared__ __attribute__((aligned(16))) float s_dot[2][Q * kDotStride];  // [dot][wave][quarter]

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;

  int total = a.count_max;
  if (!POOL && a.m_dev) total = min(max(*a.m_dev, 0), a.count_max);
  const int per = total / (int)gridDim.x, rem = total % (int)gridDim.x;
  const int lo = blockIdx.x * per + min((int)blockIdx.x, rem);
  const int hi = lo + per + ((int)blockIdx.x < rem ? 1 : 0);

  // the thread's columns: piece v holds columns first[v] .. first[v] + 3
  int first[VPT];
#pragma unroll
  for (int v = 0; v < VPT; ++v) first[v] = min(4 * (v * kWideThreads + (int)threadIdx.x), a.d - 4);
  // only the last piece can be short or absent: which of its columns are the thread's own
  const int c_last = 4 * ((VPT - 1) * kWideThreads + (int)threadIdx.x);
  bool own[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) own[i] = first[VPT - 1] + i >= c_last;

  f4 mw[SVM ? VPT : 1], mp[NEED_PHI ? VPT : 1];
#pragma unroll
  for (int v = 0; v < VPT; ++v) {
    if (SVM) mw[v] = *reinterpret_cast<const f4u *>(a.w + first[v]);
    if (NEED_PHI) mp[v] = *reinterpret_cast<const f4u *>(a.phi + first[v]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {  // (zero on both sides: the row's zero times an infinite entry would be a NaN)
    if (SVM && !own[i]) mw[VPT - 1][i] = 0.f;
    if (NEED_PHI && !own[i]) mp[VPT - 1][i] = 0.f;
  }
  const float b = (NEED_PHI && a.bias) ? *a.bias : 0.f;
  const float T = (ASSIST || HARD) ? *a.T : 0.f;
  if (GRAD && a.t_upd && blockIdx.x == 0 && threadIdx.x == 0) *a.t_snap = *a.t_upd;

  double gw[SVM ? VPT : 1][4], gp[ASSIST ? VPT : 1][4];
#pragma unroll
  for (int v = 0; v < VPT; ++v) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (SVM) gw[v][i] = 0.0;
      if (ASSIST) gp[v][i] = 0.0;
    }
  }
  float gb = 0.f;
  int kept = 0;
  int parity = 0;

  for (int base = lo; base < hi; base += kWave) {
    const int cnt = min(kWave, hi - base);
    // one row per lane (the same 64 rows in every wave): id, label, draw, incoming loss
    const int mine = base + min(lane, cnt - 1);
    const int row_l = a.rows ? a.rows[mine] : mine;
    float y_l = 0.f, u_l = 2.f, lin_l = 0.f;
    if (SVM) y_l = a.y[row_l];
    if (ASSIST && !SVM) lin_l = a.loss_in[mine];
    if (POOL && a.do_keep) u_l = keep_uniform(a.key, (uint32_t)mine);
    float o_logit = 0.f, o_prob = 0.f, o_loss = 0.f;  // outputs of the group, one row per lane
    int o_keep = 0;

    f4u x[2][R][VPT];
    auto issue = [&](int it, f4u (&xb)[R][VPT]) __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        // (a slot past the end of the group re-reads its last row and is not used)
        const int row = __builtin_amdgcn_readlane(row_l, min(it + r, cnt - 1));
        const float *xr = a.x + (int64_t)row * a.ld;
#pragma unroll
        for (int v = 0; v < VPT; ++v)
          if (NT)
            xb[r][v] = __builtin_nontemporal_load(reinterpret_cast<const f4u *>(xr + first[v]));
          else
            xb[r][v] = *reinterpret_cast<const f4u *>(xr + first[v]);
      }
    };
    auto consume = [&](int it, f4u (&xb)[R][VPT]) __attribute__((always_inline)) {
      // dot products: a quarter wave's sums stay in its lanes (dot q in lane q of 16), the
      // quarters and the waves are added behind the barrier
      float dots = 0.f;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        float dp = 0.f, dw = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) xb[r][VPT - 1][i] = own[i] ? xb[r][VPT - 1][i] : 0.f;
#pragma unroll
        for (int v = 0; v < VPT; ++v) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if (NEED_PHI) dp = __fmaf_rn(xb[r][v][i], mp[v][i], dp);
            if (SVM) dw = __fmaf_rn(xb[r][v][i], mw[v][i], dw);
          }
        }
        if (NEED_PHI) {
          dp = row_group_sum<16>(dp, lane);
          dots = (lane & 15) == r ? dp : dots;
        }
        if (SVM) {
          dw = row_group_sum<16>(dw, lane);
          dots = (lane & 15) == kDotW + r ? dw : dots;
        }
      }
      if ((lane & 15) < Q) s_dot[parity][(lane & 15) * kDotStride + wave * 4 + (lane >> 4)] = dots;
      __syncthreads();
      // (the other parity is written next: no second barrier)
      // lanes 8 r .. 8 r + 7 add up row r, one wave's four quarters each, and go on with it
      auto dot_of = [&](int q) __attribute__((always_inline)) {
        const f4 t = *reinterpret_cast<const f4 *>(&s_dot[parity][q * kDotStride + (lane & 7) * 4]);
        float v = (t.x + t.y) + (t.z + t.w);
        v = dpp_add<0xB1>(v);   // quad_perm [1,0,3,2]
        v = dpp_add<0x4E>(v);   // quad_perm [2,3,0,1]
        return dpp_add<0x141>(v);  // row_half_mirror
      };
      const int my = min(lane >> 3, R - 1), li = it + my;
      const bool live = li < cnt && lane < 8 * R;
      const int src = min(li, cnt - 1);
      // (read by every lane: a shuffle among some of them gets zero from the lanes left out)
      const float u = POOL && !HARD ? __shfl(u_l, src, kWave) : 0.f;
      float g = 0.f, s = 0.f, loss = (ASSIST && !SVM) ? __shfl(lin_l, src, kWave) : 0.f;
      bool keep = live;
      if (NEED_PHI) {
        s = dot_of(my) + b;
        g = sigmoidf_(s);
        if (POOL && a.do_keep)
          keep = live && keep_decision(u, g, a.gamma, a.one_minus_gamma);
      }
      float cw = 0.f, resid = 0.f;
      if (SVM) {
        const float yy = __shfl(y_l, src, kWave);
        const float marg = yy * dot_of(kDotW + my);
        loss = fmaxf(0.f, 1.f - marg);
        if (HARD) keep = live && loss > T;      // shrinking by the objective value itself
        cw = (keep && marg < 1.f) ? yy : 0.f;   // -d hinge / d margin, times y
      }
      if (ASSIST && keep) resid = g - (loss > T ? 1.f : 0.f);  // label: Boss loss above the threshold
      if ((lane & 7) == 0) {
        gb += resid;
        kept += keep ? 1 : 0;
      }
      parity ^= 1;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const float c = lane_read(cw, 8 * r), q = lane_read(resid, 8 * r);
        if (SVM && c != 0.f) {
#pragma unroll
          for (int v = 0; v < VPT; ++v) {
#pragma unroll
            for (int i = 0; i < 4; ++i) gw[v][i] = __fma_rn((double)c, (double)xb[r][v][i], gw[v][i]);
          }
        }
        if (ASSIST && q != 0.f) {
#pragma unroll
          for (int v = 0; v < VPT; ++v) {
#pragma unroll
            for (int i = 0; i < 4; ++i) gp[v][i] = __fma_rn((double)q, (double)xb[r][v][i], gp[v][i]);
          }
        }
      }
      if (wave == 0 && (POOL || SVM)) {  // row it + r's outputs: from lane 8 r to lane it + r
        const int from = min(max(lane - it, 0), R - 1) * 8;
        const bool here = lane >= it && lane < it + R;
        const float ts = __shfl(s, from, kWave), tg = __shfl(g, from, kWave);
        const float tl = __shfl(loss, from, kWave);
        const int tk = __shfl(keep ? 1 : 0, from, kWave);
        o_logit = here ? ts : o_logit;
        o_prob = here ? tg : o_prob;
        o_loss = here ? tl : o_loss;
        o_keep = here ? tk : o_keep;
      }
    };

    // The next batch is requested before this one is used, unconditionally (the last batch has a
    // place of its own): a request under a condition would turn every wait into one for all.
    issue(0, x[0]);
    int it = 0;
    for (; it + 2 * R < cnt; it += 2 * R) {
      issue(it + R, x[1]);
      consume(it, x[0]);
      issue(it + 2 * R, x[0]);
      consume(it + R, x[1]);
    }
    if (it + R < cnt) {
      issue(it + R, x[1]);
      consume(it, x[0]);
      consume(it + R, x[1]);
    } else {
      consume(it, x[0]);
    }
    if (wave == 0 && lane < cnt) {
      if (NEED_PHI && POOL && a.logit) a.logit[mine] = o_logit;
      if (NEED_PHI && POOL && a.prob) a.prob[mine] = o_prob;
      if (POOL && a.flags) a.flags[mine] = (uint8_t)o_keep;
      if (SVM && a.loss_out && (HARD || o_keep)) a.loss_out[mine] = o_loss;
    }
  }

  if (GRAD) {
    const int row = a.part_row;
    float *const part = a.partial + (size_t)blockIdx.x * NVEC * row;
#pragma unroll
    for (int v = 0; v < VPT; ++v) {
      constexpr int kPieces = kWideFp32Cols / (4 * kWideThreads);  // pieces of a thread before the doubles
      const int c = 4 * (v * kWideThreads + (int)threadIdx.x);
      auto put = [&](const double (&g)[4], float *to) __attribute__((always_inline)) {
        if (NVEC == 2 && v >= kPieces) {
          double *const out = reinterpret_cast<double *>(to + kWideFp32Cols) - kWideFp32Cols;
          if (c + 4 <= a.d) {
            *reinterpret_cast<f64x4 *>(out + c) = f64x4{g[0], g[1], g[2], g[3]};
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (first[v] + i >= c) out[first[v] + i] = g[i];
          }
        } else if (c + 4 <= a.d) {
          *reinterpret_cast<f4 *>(to + c) = f4{(float)g[0], (float)g[1], (float)g[2], (float)g[3]};
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (first[v] + i >= c) to[first[v] + i] = (float)g[i];
        }
      };
      if (SVM) put(gw[v], part);
      if (ASSIST) put(gp[v], part + (SVM ? row : 0));
    }
    if (wave == 0) {  // (every wave counted the same)
#pragma unroll
      for (int off = kWave / 2; off > 0; off >>= 1) kept += __shfl_xor(kept, off, kWave);
      gb = group_sum<kWave>(gb);
      if (lane == 0) {
        a.blk_cnt[blockIdx.x] = kept;
        a.blk_gb[blockIdx.x] = gb;
      }
    }
  }
}

template <int VPT, int R>
hipError_t launch_vpt(const PassArgs &a, int mode, int nblk, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  const dim3 grid(nblk), block(kWideThreads);
  switch (mode) {
    case kPool:
      if (a.plain_loads)
        launch_stamped((k_wide_pass<VPT, R, kPool, false>), grid, block, st, e0, e1, a);
      else
        launch_stamped((k_wide_pass<VPT, R, kPool>), grid, block, st, e0, e1, a);
      break;
    case kSvm:
      launch_stamped((k_wide_pass<VPT, R, kSvm>), grid, block, st, e0, e1, a);
      break;
    case kAssist:
      launch_stamped((k_wide_pass<VPT, R, kAssist>), grid, block, st, e0, e1, a);
      break;
    case kSvm | kAssist:
      launch_stamped((k_wide_pass<VPT, R, kSvm | kAssist>), grid, block, st, e0, e1, a);
      break;
    case kPool | kSvm | kAssist:
      launch_stamped((k_wide_pass<VPT, R, kPool | kSvm | kAssist>), grid, block, st, e0, e1, a);
      break;
    case kPool | kSvm | kHard:
      launch_stamped((k_wide_pass<VPT, R, kPool | kSvm | kHard>), grid, block, st, e0, e1, a);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

bool wide_rows_ok(const aa_features *F) {
  return F->layout == AA_DENSE && F->d >= kAnyMinD && F->d <= kWideMaxD;
}

int32_t wide_d_pad(int32_t d) { return (d + 31) / 32 * 32; }

int32_t wide_part_row(int32_t d, int nvec) {
  const int32_t pad = wide_d_pad(d);
  return nvec == 2 && pad > kWideFp32Cols ? 2 * pad - kWideFp32Cols : pad;
}

// A block's partial sums are as long as a row per updated vector, written and read again, so few
// rows per block are as much traffic for the sums as for the rows; few blocks leave compute units
// idle.  Four rows a block up to half the compute units, eight beyond that.  Whole steps, one / four /
// eight / sixteen rows a block: d = 2047, 256 rows 10.5 / 8.9 / 8.6 / 10.1 us, 1000 rows 10.8 / 10.6 / 9.6 / 11.2;
// d = 4137 13.9 / 10.6 / 12.4 / 15.8 and 14.6 / 14.3 / 13.7 / 16.4; d = 8000 20.0 / 15.0 / 16.6 / 21.0 and
// 23.1 / 23.2 / 21.9 / 23.8; 4096 rows within 1 %.
// Scoring leaves no sums, but takes the same blocks: with at most 1 / 2 / 4 / 8 of them per compute unit
// 20,000 x 1027 took 17.0 / 19.0 / 24.5 / 32.5 us, 4096 x 4137 10.3 / 13.3 / 16.3 / 13.3, 65,536 x 31
// 12.1 / 14.3 / 16.6 / 21.6: every block fetches the model and fills its pipeline anew.
int32_t wide_pass_blocks(int32_t d, int32_t count) {
  if (d < kWideMinD) {  // a row per wave and block of eight
    const int32_t want = (int32_t)(((int64_t)count + 7) / 8);
    return want < 1 ? 1 : want < kWideBlocks ? want : kWideBlocks;
  }
  const int32_t half = kWideBlocks / 2, four = (int32_t)(((int64_t)count + 3) / 4);
  const int32_t eight = (int32_t)(((int64_t)count + 7) / 8);
  int32_t want = four < half ? four : eight > half ? eight : half;
  if (want > kWideBlocks) want = kWideBlocks;
  return want < 1 ? 1 : want;
}

hipError_t launch_wide_pass(const PassArgs &a, int mode, int32_t nblk, hipStream_t st, hipEvent_t e0,
                            hipEvent_t e1) {
  if (a.d < kAnyMinD || a.d > kWideMaxD) return hipErrorInvalidValue;
  if (a.d < kWideMinD) return launch_any_rows(a, mode, nblk, st, e0, e1);
  switch ((a.d + 4 * kWideThreads - 1) / (4 * kWideThreads)) {
    case 1: return launch_vpt<1, 8>(a, mode, nblk, st, e0, e1);
    case 2: return launch_vpt<2, 4>(a, mode, nblk, st, e0, e1);
    case 3: return launch_vpt<3, 4>(a, mode, nblk, st, e0, e1);
    default: return launch_vpt<4, 1>(a, mode, nblk, st, e0, e1);
  }
}

}  // namespace aa

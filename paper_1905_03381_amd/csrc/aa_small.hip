// Epochs over small pools: one block of 16 waves runs the steps one after the other.
//
// A pool of 256 rows of 128 floats is 128 KB: a step of two launches spends its 9 us on two kernel
// boundaries and on chains of round trips, not on reading.  Here the model stays in LDS, the
// next pool's rows are requested into a second set of registers while this one's are used, and
// nothing waits for another compute unit.  What bounds it then: one compute unit's share of the
// memory system (about 28 bytes per ns) for pools near the limit, the waves' arithmetic below.
#include "aa_small.hpp"

namespace aa {

namespace {

constexpr int kSmallWaves = 16, kSmallTurns = 8;

// lane I of every 16, in all 16
template <int I>
__device__ __forceinline__ float row_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + I, 0xf, 0xf, true));
}

template <int I>
struct Turn {
  static constexpr int value = I;
};

// LPR lanes hold a row (up to 4 LPR floats), a wave takes up to IT (at most kSmallTurns) turns of 64 / LPR rows.
// Per row only the 128-bit products run in all lanes; a turn's two dot products end in one lane
// of every 16 and what follows from them (sigmoid, draw, loss, coefficients) is worked out for
// all rows of the wave at once.
// Per step, two launches / this: 256 rows of 128 floats 9.0 / 4.8 us (hard thresholds 8.0 / 3.1),
// 100 of 64 9.0 / 3.2 (7.8 / 2.0), 20 of 256 9.1 / 2.7 (7.8 / 1.5).  The limit is what the
// registers hold twice, 128 KB of rows; past it a compute unit's reads alone take as long as the
// two launches.
template <int LPR, bool HARD, int IT>
__global__ __launch_bounds__(kSmallWaves * 64)
    __attribute__((amdgpu_waves_per_eu(4, 4))) void k_small_epoch(const SmallEpochArgs a) {
  constexpr int NW = kSmallWaves, G = kWave / LPR, ROW = 4 * LPR;
  constexpr int kRows = NW * IT * G;  // rows a pool has at most
  constexpr int NVEC = HARD ? 1 : 2;
  static_assert(NVEC * ROW <= NW * 64, "a column per thread");
  __shared__ f4 s_model[NVEC][LPR];
  __shared__ f4 s_red[NW][NVEC][LPR];
  __shared__ int s_cnt[NW];
  __shared__ float s_gb[NW];
  __shared__ float s_u[2][HARD ? 1 : kRows];  // draws of this step and the next

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int grp = lane / LPR, sub = lane % LPR;
  const f4 zero4 = {0.f, 0.f, 0.f, 0.f};
  const int piece = min(sub, a.d4 - 1);  // (lanes past the row re-read its last piece and are masked)
  const bool own = sub < a.d4;

  // this thread's column of one of the vectors
  const int vec = tid / ROW, col = tid % ROW;
  const bool column = tid < NVEC * ROW && col < a.d;
  float mine = 0.f;
  if (column) mine = vec == 0 ? a.w[col] : a.phi[col];
  if (tid < NVEC * ROW) reinterpret_cast<float *>(s_model)[tid] = mine;
  // (uniform values are kept in scalar registers: the rows take most of the others)
  auto uniform = [](float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); };
  float b = (!HARD && a.bias) ? uniform(*a.bias) : 0.f;
  const float T = uniform(*a.T);
  int t_now = a.t_upd ? __builtin_amdgcn_readfirstlane(*a.t_upd) : 0;

  auto pool_rows = [&](int t) { return (int)min((int64_t)a.P, a.n_perm - (int64_t)t * a.P); };
  // rows of pool t this wave takes: `per` (fewer at the end) from `lo` on
  struct Share {
    int lo, cnt;
  };
  auto share_of = [&](int t) {
    const int total = pool_rows(t), per = (total + NW - 1) / NW;
    const int lo = min(wave * per, total);
    return Share{lo, min(per, total - lo)};
  };
  // one row per lane; a wave without rows reads the pool's last one
  auto load_ids = [&](int t) {
    t = min(t, a.steps - 1);
    const Share s = share_of(t);
    return a.perm[(int64_t)t * a.P + min(s.lo + min(lane, max(s.cnt, 1) - 1), pool_rows(t) - 1)];
  };

  f4 xa[IT], xb[IT];
  float ya, yb;
  auto request = [&](int t, int id, f4 (&x)[IT], float &y) __attribute__((always_inline)) {
    const int last = max(share_of(min(t, a.steps - 1)).cnt, 1) - 1;
    y = a.y[id];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int row = __shfl(id, min(it * G + grp, last), kWave);
      x[it] = reinterpret_cast<const f4 *>(a.x + (uint64_t)(uint32_t)row * (uint32_t)a.ld)[piece];
    }
  };

  // outputs of the step before, one row per lane: stored behind the wait for this step's rows, so
  // that no wait for rows is a wait for stores just made
  int o_t = -1, o_id = 0, o_pos = -1, o_m = 0;  // (o_pos: -1 where the row was not kept)
  float o_loss = 0.f, o_prob = 0.f;
  auto put = [&]() __attribute__((always_inline)) {
    if (o_t < 0) return;
    const Share sh = share_of(o_t);
    if (lane < sh.cnt) {
      const int j = sh.lo + lane;
      if (!HARD && a.prob) a.prob[j] = o_prob;
      if (a.flags) a.flags[j] = o_pos >= 0 ? 1 : 0;
      if (o_pos >= 0) {
        if (a.kept_pos) a.kept_pos[o_pos] = j;
        if (a.ids) a.ids[o_t * a.ids_stride + o_pos] = o_id;
        if (a.loss) a.loss[o_t * a.loss_stride + o_pos] = o_loss;
      }
    }
    if (tid == 0 && a.kept_hist) a.kept_hist[o_t] = o_m;
  };

  // the draws of pool t, a row per thread: ten rounds of multiplications at a quarter of the
  // rate, so the first waves make them for all (in every wave for its own few rows they were a
  // fifth of a step)
  auto draw = [&](int t) __attribute__((always_inline)) {
    if (HARD || tid >= min(a.P, kRows)) return;
    const uint64_t st = a.step + (uint64_t)t;
    s_u[t & 1][tid] = keep_uniform(DrawKey{a.k0, a.k1, (uint32_t)st, (uint32_t)(st >> 32)}, (uint32_t)tid);
  };

  int id_cur = load_ids(0), id_next = load_ids(1);
  request(0, id_cur, xa, ya);
  draw(0);
  __syncthreads();

  auto step = [&](int t, f4 (&x)[IT], float &y, f4 (&xn)[IT], float &yn) __attribute__((always_inline)) {
    const Share sh = share_of(t);
#pragma unroll
    for (int it = 0; it < IT; ++it) asm volatile("" : "+v"(x[it]));  // the rows are there
    arrived(y);
    arrived(id_next);
    put();
    const int id_after = load_ids(t + 2);
    request(t + 1, id_next, xn, yn);
    const f4 mw = s_model[0][sub], mp = s_model[NVEC - 1][sub];

    // dot products: turn it's in lane it (Assistant) and lane 8 + it (Boss) of every 16
    float v = 0.f;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      if (!own) x[it] = zero4;
      if (!HARD) {
        const float dp = row_group_sum<16>(dot4(x[it], mp, 0.f), lane);
        v = (lane & 15) == it ? dp : v;
      }
      const float dw = row_group_sum<16>(dot4(x[it], mw, 0.f), lane);
      v = (lane & 15) == 8 + it ? dw : v;
    }
    if (LPR >= 32) v += __shfl_xor(v, 16, kWave);
    if (LPR >= 64) v += __shfl_xor(v, 32, kWave);
    const float other = __shfl_xor(v, 8, kWave);
    const float dot_p = (lane & 8) ? other : v, dot_w = (lane & 8) ? v : other;

    // lane `it` (and 8 + it) of every 16 goes on with row it * G + grp
    int me = lane;
    asm volatile("" : "+v"(me));  // (as below)
    const int li = (me & 7) * G + me / LPR;
    const bool live = li < sh.cnt;
    const float yy = __shfl(y, li & 63, kWave);
    float g = 0.f;
    bool keep = live;
    if (!HARD) {
      g = sigmoidf_(dot_p + b);
      keep = live && keep_decision(s_u[t & 1][min(sh.lo + li, kRows - 1)], g, a.gamma, a.one_minus_gamma);
    }
    const float marg = yy * dot_w;
    const float loss = fmaxf(0.f, 1.f - marg);
    if (HARD) keep = live && loss > T;  // shrinking by the objective value itself
    const float cw = (keep && marg < 1.f) ? yy : 0.f;  // -d hinge / d margin, times y
    const float resid = !HARD && keep ? g - (loss > T ? 1.f : 0.f) : 0.f;  // label: Boss loss above T
    const bool once = sub < 8;  // (the lanes that stand for a row)
    const int kept = __popcll(__ballot(keep && once));
    const float gb = HARD ? 0.f : row_group_sum<kWave>(once ? resid : 0.f, lane);

    f4 gw = zero4, gp = zero4;
    // With a wave per row, a rejected row and a turn past the share add nothing at all, as in a single
    // step: zero times an infinite feature would be a NaN.  (Bit i: turn i's row counts.)  Steps of 128
    // rows of 256 floats 4.48 us with every turn added, 4.32 so.  Elsewhere the steps this
    // stands for add every row, and so does it.
    constexpr bool SKIP = LPR == kWave && !HARD;
    const uint32_t counts = SKIP ? (uint32_t)__ballot(keep && once) : ~0u;
    auto turn = [&](auto it) __attribute__((always_inline)) {
      constexpr int i = decltype(it)::value;
      if constexpr (i < IT) {
        if (SKIP && !((counts >> i) & 1u)) return;
        gw = axpy4(row_bcast<i>(cw), x[i], gw);
        if (!HARD) gp = axpy4(row_bcast<i>(resid), x[i], gp);
      }
    };
    turn(Turn<0>{}), turn(Turn<1>{}), turn(Turn<2>{}), turn(Turn<3>{});
    turn(Turn<4>{}), turn(Turn<5>{}), turn(Turn<6>{}), turn(Turn<7>{});
    if (LPR < kWave) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        gw[i] = fold_groups<LPR>(gw[i]);
        if (!HARD) gp[i] = fold_groups<LPR>(gp[i]);
      }
    }
    if (lane < LPR) {
      s_red[wave][0][lane] = gw;
      if (!HARD) s_red[wave][NVEC - 1][lane] = gp;
    }
    if (lane == 0) {
      s_cnt[wave] = kept;
      s_gb[wave] = gb;
    }
    draw(t + 1);  // (here this pool's rows no longer take registers)
    __syncthreads();

    int m = 0, before = 0;
    float gbs = 0.f;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int c = s_cnt[i];
      before += i < wave ? c : 0;
      m += c;
      gbs += s_gb[i];
    }
    m = __builtin_amdgcn_readfirstlane(m);
    before = __builtin_amdgcn_readfirstlane(before);
    gbs = uniform(gbs);
    if (m > 0) {
      const float inv_m = 1.f / (float)m;
      ++t_now;
      const float lr = a.t_upd ? a.lr / sqrtf((float)t_now) : a.lr;
      if (column) {
        const float *red = reinterpret_cast<const float *>(s_red);
        float gsum = 0.f;
#pragma unroll
        for (int i = 0; i < NW; ++i) gsum += red[(i * NVEC + vec) * ROW + col];
        if (vec == 0)
          mine = __fmaf_rn(lr * inv_m, gsum, (1.f - lr * a.lambda) * mine);
        else
          mine = mine - a.lr_a * __fmaf_rn(a.l2_a, mine, gsum * inv_m);
        reinterpret_cast<float *>(s_model)[tid] = mine;
      }
      if (!HARD && a.bias) b = uniform(b - a.lr_a * (gbs * inv_m));
    }
    // row `lane` of the wave: what lane (its turn) of its group worked out
    int here = lane;
    asm volatile("" : "+v"(here));  // (worked out here, not kept in a register across the steps)
    const int from = (here % G) * LPR + ((here / G) & 7);
    const bool row_kept = __shfl(keep ? 1 : 0, from, kWave) != 0 && lane < sh.cnt;
    o_loss = __shfl(loss, from, kWave);
    o_prob = __shfl(g, from, kWave);
    const unsigned long long mask = __ballot(row_kept);
    const int pos = before + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
    o_pos = row_kept ? pos : -1;
    o_t = t;
    o_id = id_cur;
    o_m = m;
    id_cur = id_next;
    id_next = id_after;
    __syncthreads();
  };

  for (int t = 0; t < a.steps; t += 2) {
    step(t, xa, ya, xb, yb);
    if (t + 1 < a.steps) step(t + 1, xb, yb, xa, ya);
  }
  put();
  if (column) {
    if (vec == 0)
      a.w[col] = mine;
    else
      a.phi[col] = mine;
  }
  if (tid == 0) {
    if (!HARD && a.bias) *a.bias = b;
    if (a.t_upd) *a.t_upd = t_now;
  }
}

template <int LPR, bool HARD>
hipError_t launch_turns(const SmallEpochArgs &a, hipStream_t st) {
  const dim3 grid(1), block(kSmallWaves * 64);
  const int per_turn = kSmallWaves * (kWave / LPR);
  if (a.P <= 2 * per_turn)
    hipLaunchKernelGGL((k_small_epoch<LPR, HARD, 2>), grid, block, 0, st, a);
  else if (a.P <= 4 * per_turn)
    hipLaunchKernelGGL((k_small_epoch<LPR, HARD, 4>), grid, block, 0, st, a);
  else
    hipLaunchKernelGGL((k_small_epoch<LPR, HARD, kSmallTurns>), grid, block, 0, st, a);
  return hipGetLastError();
}

template <int LPR>
hipError_t launch_lpr(const SmallEpochArgs &a, bool hard, hipStream_t st) {
  return hard ? launch_turns<LPR, true>(a, st) : launch_turns<LPR, false>(a, st);
}

int lanes_per_row(int32_t d) { return d <= 64 ? 16 : d <= 128 ? 32 : 64; }

}  // namespace

bool small_epoch_ok(int32_t d, int64_t ld, int32_t P) {
  return d <= 256 && ld <= 0x7fffffff && P <= kSmallWaves * kSmallTurns * (kWave / lanes_per_row(d));
}

hipError_t launch_small_epoch(const SmallEpochArgs &a, bool hard, hipStream_t st) {
  if (!small_epoch_ok(a.d, a.ld, a.P) || a.steps < 1 || a.steps > kSmallEpochSteps) return hipErrorInvalidValue;
  switch (lanes_per_row(a.d)) {
    case 16: return launch_lpr<16>(a, hard, st);
    case 32: return launch_lpr<32>(a, hard, st);
    default: return launch_lpr<64>(a, hard, st);
  }
}

}  // namespace aa

// Epochs over small pools: 16 waves run the steps one after the other, in one block or in a team of four.
//
// A pool of 256 rows of 128 floats is 128 KB: a step of two launches spends its 9 us on two kernel
// boundaries and on chains of round trips, not on reading.  Here the model stays in LDS, the
// next pool's rows are requested into a second set of registers while this one's are used, and
// nothing waits for another compute unit.  What bounds it then: one compute unit's share of the
// memory system (about 28 bytes per ns) for pools near the limit, the waves' arithmetic below.
//
// In a team every wave has a SIMD to itself (nearly), and four compute units read: an epoch of 40 pools of 256 x 128
// 192 -> 120 us.  The waves' gradient sums, added up by fours in each block, then go through memory, each in a
// 64-bit word with the step's number beside it, stored and read with relaxed device-scope atomics: a reader takes a word
// whose number is the step's and asks again otherwise, so nothing has to be ordered or counted.  (Four blocks that read
// 256 words of each other: 0.7 to 1.0 us a round; every wave's sums without the additions, four times the words, 3.)
// Every block adds all sums up, in the order of the single block, and updates a model of its own: the same bits.  A word
// has two places, for odd and even steps: a block writes step t + 2's sums when it has read all of step t + 1's, which the
// others wrote after they had read step t's.  Waves of their own do the reading: loads return in order, and a wave with
// the next rows on their way would wait for those first.
// The blocks of a team have to run at once.  k_team_reset clears words and gate ahead of the launch; a block counts
// itself in, the last one opens the gate, and nobody publishes before it is open.  A block that has waited past its
// limit shuts the gate for good; all of them leave then.  So they do if words do not come: the waits behind the gate are
// bounded by the number of requests, which stands still with the waves of a queue that is suspended.  Blocks that have
// got through the last step count themselves, too: the last of four writes the model, and if there are fewer nobody has, and
// the launch behind, which has nothing to do otherwise, does the whole epoch with one block.
#include "aa_small.hpp"

namespace aa {

namespace {

constexpr int kSmallWaves = 16, kSmallTurns = 8;
constexpr int kTeamBlocks = 4, kTeamWaves = kSmallWaves / kTeamBlocks;  // row waves of a block, and as many others
constexpr int kGateWords = 16;  // 64-bit words in front; of 32 bits: blocks that are there, state of the gate, blocks that are through
constexpr int kTeamExtra = 16;  // words behind a block's sums: its waves' kept rows (a byte each), bias gradient, nothing
enum Gate : int { kGateOpen = 1, kGateShut = 2 };
// 100 MHz ticks until the gate opens (some milliseconds, different from call to call)
constexpr long long kGateTicks = 200000;
// pairs of requests for a word once it is, some tenths of a second's (whoever is waited for runs then: this ends a wait that
// could not end otherwise)
constexpr int kWordPolls = 1 << 18;

constexpr size_t team_words(int cols) { return kGateWords + 2 * (size_t)kTeamBlocks * (cols + kTeamExtra); }

__device__ __forceinline__ uint64_t word_of(uint32_t v, int tag) { return ((uint64_t)(uint32_t)tag << 32) | v; }
__device__ __forceinline__ uint64_t load_word(const uint64_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_word(uint64_t *p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int tag_of(uint64_t w) { return (int)(w >> 32); }
__device__ __forceinline__ float value_of(uint64_t w) { return __uint_as_float((uint32_t)w); }
__device__ __forceinline__ int load_gate(const int32_t *state) {
  return __hip_atomic_load(state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void move_gate(int32_t *state, int to) {
  int closed = 0;
  __hip_atomic_compare_exchange_strong(state, &closed, to, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(256) void k_team_reset(uint64_t *words, int count, const int32_t *ends) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x)
    words[i] = i == 0 && *ends == kGateShut ? (uint64_t)kGateShut << 32 : 0;
}

// lane I of every 16, in all 16
template <int I>
__device__ __forceinline__ float row_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + I, 0xf, 0xf, true));
}

template <int I>
struct Turn {
  static constexpr int value = I;
};

// What a wave works out from its rows of a pool.
struct RowSums {
  float g, loss, gb;  // (g and loss: lane i of every 16 (of LPR) for turn i's row, i < 8)
  bool keep;
  int kept;
  f4 gw, gp;          // the sums of this lane's columns, in all lane groups
};

// The rows' part of a step: x: the wave's turns; `own`: the lane holds columns; cnt rows; u_of(i): row i's draw.
template <int LPR, bool HARD, int IT, class Draw>
__device__ __forceinline__ RowSums small_rows(const SmallEpochArgs &a, f4 (&x)[IT], float y, bool own, const f4 &mw,
                                              const f4 &mp, float b, float T, int cnt, Draw u_of) {
  constexpr int G = kWave / LPR;
  const f4 zero4 = {0.f, 0.f, 0.f, 0.f};
  const int lane = threadIdx.x & 63, sub = lane % LPR;
  RowSums out;
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
  asm volatile("" : "+v"(me));  // (worked out here, not kept in a register across the steps)
  const int li = (me & 7) * G + me / LPR;
  const bool live = li < cnt;
  const float yy = __shfl(y, li & 63, kWave);
  out.g = 0.f;
  out.keep = live;
  if (!HARD) {
    out.g = sigmoidf_(dot_p + b);
    const float u = u_of(li);  // (every lane takes part)
    out.keep = live && keep_decision(u, out.g, a.gamma, a.one_minus_gamma);
  }
  const float marg = yy * dot_w;
  out.loss = fmaxf(0.f, 1.f - marg);
  if (HARD) out.keep = live && out.loss > T;  // shrinking by the objective value itself
  const float cw = (out.keep && marg < 1.f) ? yy : 0.f;  // -d hinge / d margin, times y
  const float resid = !HARD && out.keep ? out.g - (out.loss > T ? 1.f : 0.f) : 0.f;  // label: Boss loss above T
  const bool once = sub < 8;  // (the lanes that stand for a row)
  out.kept = __popcll(__ballot(out.keep && once));
  out.gb = HARD ? 0.f : row_group_sum<kWave>(once ? resid : 0.f, lane);

  f4 gw = zero4, gp = zero4;
  // With a wave per row, a rejected row and a turn past the share add nothing at all, as in a single
  // step: zero times an infinite feature would be a NaN.  (Bit i: turn i's row counts.)  Steps of 128
  // rows of 256 floats 4.48 us with every turn added, 4.32 so.  Elsewhere the steps this
  // stands for add every row, and so does it.
  constexpr bool SKIP = LPR == kWave && !HARD;
  const uint32_t counts = SKIP ? (uint32_t)__ballot(out.keep && once) : ~0u;
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
  out.gw = gw;
  out.gp = gp;
  return out;
}

// LPR lanes hold a row (up to 4 LPR floats), a wave takes up to IT (at most kSmallTurns) turns of 64 / LPR rows.
// Per row only the 128-bit products run in all lanes; a turn's two dot products end in one lane
// of every 16 and what follows from them (sigmoid, draw, loss, coefficients) is worked out for
// all rows of the wave at once.
// Per step, two launches / this (a team is faster, see launch_team): 256 rows of 128 floats 9.0 / 4.8 us (hard
// thresholds 8.0 / 3.1), 100 of 64 9.0 / 3.2 (7.8 / 2.0), 20 of 256 9.1 / 2.7 (7.8 / 1.5).  The limit is what the
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

  if (a.words && load_gate(reinterpret_cast<const int32_t *>(a.words) + 2) == kTeamBlocks) return;  // (the team did it)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = lane / LPR, sub = lane % LPR;
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

    const RowSums rs = small_rows<LPR, HARD, IT>(a, x, y, own, mw, mp, b, T, sh.cnt, [&](int li) __attribute__((always_inline)) {
      return s_u[t & 1][min(sh.lo + li, kRows - 1)];
    });
    const bool keep = rs.keep;
    const float loss = rs.loss, g = rs.g, gb = rs.gb;
    const int kept = rs.kept;
    const f4 gw = rs.gw, gp = rs.gp;
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
    float four = 0.f;  // (four waves, then the fours: the order of a team)
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int c = s_cnt[i];
      before += i < wave ? c : 0;
      m += c;
      four = i % kTeamWaves == 0 ? s_gb[i] : four + s_gb[i];
      if (i % kTeamWaves == kTeamWaves - 1) gbs += four;
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
        float gsum = 0.f, four = 0.f;
#pragma unroll
        for (int i = 0; i < NW; ++i) {
          const float r = red[(i * NVEC + vec) * ROW + col];
          four = i % kTeamWaves == 0 ? r : four + r;
          if (i % kTeamWaves == kTeamWaves - 1) gsum += four;
        }
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

// The same in a team: waves 0 to 3 of a block are row waves (of the 16: 4 blockIdx.x + wave), the others read what all
// blocks have published, update the model and hand it over at the second barrier of a step.
// What bounds it, 256 rows of 128 floats, 2.9 us a step: the chain of dot products, coefficients and sums of a wave's eight turns
// (0.9), the words' way to the other blocks and back (1.1), the update (0.3), barriers; meanwhile a row wave stores the
// last step's outputs, requests rows two steps ahead and draws (1.4).
template <int LPR, bool HARD, int IT>
__global__ __launch_bounds__(2 * kTeamWaves * 64)
    __attribute__((amdgpu_waves_per_eu(2, 2))) void k_team_epoch(const SmallEpochArgs a) {
  constexpr int NW = kSmallWaves, G = kWave / LPR, ROW = 4 * LPR, NVEC = HARD ? 1 : 2, COLS = NVEC * ROW;
  constexpr int NT = kTeamWaves * 64, PER = (COLS + NT - 1) / NT;  // readers, columns of a reader
  constexpr int kStride = COLS + kTeamExtra;
  constexpr int kTeamNap = PER == 1 ? 6 : 1;  // between requests for words, in 64 cycles: 0 to 12 within 3 % for one column a reader
  __shared__ f4 s_model[NVEC][LPR], s_red[kTeamWaves][NVEC][LPR];
  __shared__ int s_before[2][kTeamWaves], s_kept[kTeamWaves], s_state, s_through;
  __shared__ float s_b, s_gb[kTeamWaves];
  const int tid = threadIdx.x, lane = tid & 63, in_block = __builtin_amdgcn_readfirstlane(tid >> 6);
  int32_t *const gate = reinterpret_cast<int32_t *>(a.words);
  if (tid < COLS) {
    const int col = tid % ROW;
    reinterpret_cast<float *>(s_model)[tid] = col < a.d ? (tid < ROW ? a.w : a.phi)[col] : 0.f;
  }
  auto pool_rows = [&](int t) { return (int)min((int64_t)a.P, a.n_perm - (int64_t)t * a.P); };

  if (in_block < kTeamWaves) {
    const int wave = blockIdx.x * kTeamWaves + in_block, grp = lane / LPR, sub = lane % LPR;
    const int piece = min(sub, a.d4 - 1);  // (lanes past the row re-read its last piece and are masked)
    const bool own = sub < a.d4;
    const float T = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(*a.T)));
    struct Share {
      int lo, cnt;
    };
    auto share_of = [&](int t) {  // as in k_small_epoch
      const int total = pool_rows(t), per = (total + NW - 1) / NW, lo = min(wave * per, total);
      return Share{lo, min(per, total - lo)};
    };
    auto load_ids = [&](int t) {
      t = min(t, a.steps - 1);
      const Share s = share_of(t);
      return a.perm[(int64_t)t * a.P + min(s.lo + min(lane, max(s.cnt, 1) - 1), pool_rows(t) - 1)];
    };
    auto request = [&](int t, int id, f4 (&x)[IT], float &y) __attribute__((always_inline)) {
      const int last = max(share_of(min(t, a.steps - 1)).cnt, 1) - 1;
      y = a.y[id];
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int row = __shfl(id, min(it * G + grp, last), kWave);
        x[it] = reinterpret_cast<const f4 *>(a.x + (uint64_t)(uint32_t)row * (uint32_t)a.ld)[piece];
      }
    };
    auto draw_of = [&](int t) __attribute__((always_inline)) {  // (a wave has fewer rows than lanes)
      const uint64_t st = a.step + (uint64_t)t;
      const int lo = share_of(min(t, a.steps - 1)).lo;
      return HARD ? 2.f : keep_uniform(DrawKey{a.k0, a.k1, (uint32_t)st, (uint32_t)(st >> 32)}, (uint32_t)(lo + lane));
    };
    // outputs of the step before, one row per lane
    int o_lo = 0, o_cnt = 0, o_id = 0;
    bool o_keep = false;
    float o_loss = 0.f, o_prob = 0.f;
    int32_t *ids = a.ids;
    float *losses = a.loss;
    auto put = [&](int before) __attribute__((always_inline)) {  // (before: kept rows ahead of this wave's, -1: not known)
      const unsigned long long mask = __ballot(o_keep);
      if (lane < o_cnt) {
        const int j = o_lo + lane;
        if (!HARD && a.prob) a.prob[j] = o_prob;
        if (a.flags) a.flags[j] = o_keep ? 1 : 0;
        if (o_keep && before >= 0) {
          const int pos = before + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
          if (a.kept_pos) a.kept_pos[pos] = j;
          if (ids) ids[pos] = o_id;
          if (losses) losses[pos] = o_loss;
        }
      }
    };
    // (rows two steps ahead, in the registers of the pool just done; ids three)
    int id0 = load_ids(0), id1 = load_ids(1), id2 = load_ids(2);
    f4 xa[IT], xb[IT];
    float ya, yb, u = draw_of(0);
    request(0, id0, xa, ya);
    request(1, id1, xb, yb);
    __syncthreads();
    if (s_state != kGateOpen) return;
    auto step = [&](int t, f4 (&x)[IT], float &y) __attribute__((always_inline)) {
      const Share sh = share_of(t);
      const f4 mw = s_model[0][sub], mp = s_model[NVEC - 1][sub];
      const RowSums rs = small_rows<LPR, HARD, IT>(a, x, y, own, mw, mp, s_b, T, sh.cnt, [&](int li) __attribute__((always_inline)) {
        return __shfl(u, li & 63, kWave);
      });
      if (lane < LPR) {
        s_red[in_block][0][lane] = rs.gw;
        if (!HARD) s_red[in_block][NVEC - 1][lane] = rs.gp;
      }
      if (lane == 0) {
        s_kept[in_block] = rs.kept;
        s_gb[in_block] = rs.gb;
      }
      __syncthreads();
      if (t > 0) {
        put(s_before[(t - 1) & 1][in_block]);
        if (ids) ids += a.ids_stride;
        if (losses) losses += a.loss_stride;
      }
      // row `lane` of the wave: what lane (its turn) of its group worked out
      int here = lane;
      asm volatile("" : "+v"(here));
      const int from = (here % G) * LPR + ((here / G) & 7);
      o_keep = __shfl(rs.keep ? 1 : 0, from, kWave) != 0 && lane < sh.cnt;
      o_loss = __shfl(rs.loss, from, kWave);
      o_prob = __shfl(rs.g, from, kWave);
      o_lo = sh.lo;
      o_cnt = sh.cnt;
      o_id = id0;
      request(t + 2, id2, x, y);
      id0 = id1;
      id1 = id2;
      id2 = load_ids(t + 3);
      u = draw_of(t + 1);
      __syncthreads();
    };
    for (int t = 0; t < a.steps; t += 2) {
      step(t, xa, ya);
      if (t + 1 < a.steps) step(t + 1, xb, yb);
    }
    put(s_before[(a.steps - 1) & 1][in_block]);
    __syncthreads();
  } else {
    const int rt = tid - NT;
    const int ends_in = *a.ends;  // (see SmallEpochArgs)
    float b = !HARD && a.bias ? *a.bias : 0.f;
    int t_now = a.t_upd ? *a.t_upd : 0;
    float mine[PER];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int c = min(rt + p * NT, COLS - 1), col = c % ROW;
      mine[p] = col < a.d ? (c < ROW ? a.w : a.phi)[col] : 0.f;
    }
    if (rt == 0) {
      s_b = b;
      s_through = 0;
      if (__hip_atomic_fetch_add(gate, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == kTeamBlocks - 1)
        move_gate(gate + 1, kGateOpen);
      const long long since = wall_clock64(), limit = kGateTicks * (1 + ((since >> 4) & 7));
      int state;
      while ((state = load_gate(gate + 1)) == 0)
        if (wall_clock64() - since > limit) move_gate(gate + 1, kGateShut);
      s_state = state;
    }
    __syncthreads();
    if (s_state != kGateOpen) return;
    // A wait of the block has passed its limit: from the next step on it publishes nothing, waits for nothing and stores no
    // batches, and it does not count itself at the end.
    bool lost = false;
    const int ends = __builtin_amdgcn_readfirstlane(ends_in);
    const int leaves = ends >= 4 && (ends & 3) == (int)blockIdx.x ? (ends >> 2) - 1 : -1;
    for (int t = 0; t < a.steps; ++t) {
      const int tag = t + 1, tag_put = lost ? 0 : tag;  // (a word of number 0 is none)
      uint64_t *const words = a.words + kGateWords + (size_t)(t & 1) * kTeamBlocks * kStride;
      __syncthreads();  // the row waves' sums are in LDS
      {
        uint64_t *const to = words + blockIdx.x * kStride;
        const float *const red = reinterpret_cast<const float *>(s_red);
#pragma unroll
        for (int p = 0; p < PER; ++p) {
          const int c = rt + p * NT;
          if (c >= COLS) break;
          float four = red[c];
#pragma unroll
          for (int i = 1; i < kTeamWaves; ++i) four += red[i * COLS + c];
          store_word(to + c, word_of(__float_as_uint(four), tag_put));
        }
        if (rt < 2) {
          uint32_t kept = 0;
          float four = s_gb[0];
#pragma unroll
          for (int i = 0; i < kTeamWaves; ++i) kept |= (uint32_t)s_kept[i] << (8 * i);
#pragma unroll
          for (int i = 1; i < kTeamWaves; ++i) four += s_gb[i];
          store_word(to + COLS + rt, word_of(rt == 0 ? kept : __float_as_uint(four), tag_put));
        }
      }
      // (what does not depend on them, while they are on their way)
      const float lr = a.t_upd ? a.lr / sqrtf((float)(t_now + 1)) : a.lr;
      float base[PER];
#pragma unroll
      for (int p = 0; p < PER; ++p) base[p] = (1.f - lr * a.lambda) * mine[p];
      // All blocks' kept rows (lane i < 4: block i's) and bias gradients (lane 4 + i), and the sums of this thread's
      // columns.  Two requests are on their way, a little apart: the words come between 0.4 and 1 us after the block's
      // own, and a request takes 0.8.
      struct Words {
        uint64_t v[PER][kTeamBlocks], e;
      } first, second;
      auto request = [&](Words &w) __attribute__((always_inline)) {
        const uint64_t *from = words;  // (worked out anew in every turn)
        asm volatile("" : "+s"(from));
        w.e = load_word(from + (lane & 3) * kStride + COLS + ((lane >> 2) & 1));
#pragma unroll
        for (int p = 0; p < PER; ++p)
#pragma unroll
          for (int i = 0; i < kTeamBlocks; ++i) w.v[p][i] = load_word(from + i * kStride + min(rt + p * NT, COLS - 1));
      };
      auto there = [&](const Words &w) __attribute__((always_inline)) {
        bool ok = tag_of(w.e) == tag;
#pragma unroll
        for (int p = 0; p < PER; ++p)
#pragma unroll
          for (int i = 0; i < kTeamBlocks; ++i) ok = ok && tag_of(w.v[p][i]) == tag;
        return __ballot(!ok) == 0ull;
      };
      __builtin_amdgcn_s_sleep(kTeamNap);
      request(first);
      int polls = lost || t == leaves ? kWordPolls : 0;
      for (;;) {
        __builtin_amdgcn_s_sleep(kTeamNap);
        request(second);
        if (there(first)) break;
        __builtin_amdgcn_s_sleep(kTeamNap);
        request(first);
        if (there(second)) {
          first = second;
          break;
        }
        if (++polls >= kWordPolls) break;
      }
      lost = polls >= kWordPolls;
      int m = 0, before = 0;
      float gbs = 0.f;
      const float ev = value_of(first.e);
#pragma unroll
      for (int i = 0; i < kTeamBlocks; ++i) {
        const uint32_t four = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)first.e, i);
#pragma unroll
        for (int w = 0; w < kTeamWaves; ++w) {
          const int c = (four >> (8 * w)) & 0xff;
          m += c;
          before += i * kTeamWaves + w < (int)blockIdx.x * kTeamWaves + rt ? c : 0;
        }
        gbs += lane_read(ev, 4 + i);
      }
      if (m > 0) {
        const float inv_m = 1.f / (float)m;
        ++t_now;
#pragma unroll
        for (int p = 0; p < PER; ++p) {
          const int c = rt + p * NT;
          if (c >= COLS || c % ROW >= a.d) continue;
          float gsum = 0.f;
#pragma unroll
          for (int i = 0; i < kTeamBlocks; ++i) gsum += value_of(first.v[p][i]);
          if (c < ROW)
            mine[p] = __fmaf_rn(lr * inv_m, gsum, base[p]);
          else
            mine[p] = mine[p] - a.lr_a * __fmaf_rn(a.l2_a, mine[p], gsum * inv_m);
          reinterpret_cast<float *>(s_model)[c] = mine[p];
        }
        if (!HARD && a.bias) b = b - a.lr_a * (gbs * inv_m);
      }
      if (rt < kTeamWaves) s_before[t & 1][rt] = lost ? -1 : before;
      if (lost && lane == 0) s_state = kGateShut;
      if (rt == 0) {
        s_b = b;
        if (blockIdx.x == 0 && a.kept_hist) a.kept_hist[t] = m;
      }
      __syncthreads();
      lost = __builtin_amdgcn_readfirstlane(s_state) != kGateOpen;
    }
    if (rt == 0 && !lost)
      s_through = __hip_atomic_fetch_add(gate + 2, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
    __syncthreads();
    if (s_through == kTeamBlocks) {  // (the others are past their last step: nobody reads the old model any more)
      for (int c = rt; c < COLS; c += NT) {
        const int col = c % ROW;
        if (col < a.d) (c < ROW ? a.w : a.phi)[col] = reinterpret_cast<const float *>(s_model)[c];
      }
      if (rt == 0) {
        if (!HARD && a.bias) *a.bias = b;
        if (a.t_upd) *a.t_upd = t_now;
      }
    }
  }
}

// A team where its exchange costs less than the turns it spares, and over enough steps to make up for its two launches
// more (5 us).  Microseconds a step, one block / team (40 steps, the launches included): two turns a wave, 64 of 128
// 3.04 / 2.40, 100 of 64 3.17 / 2.80, 32 of 256 2.89 / 3.06, with hard thresholds 64 of 128 2.00 / 2.09; four, 128 of 128
// 3.60 / 2.60 (2.28 / 2.06), 64 of 256 3.39 / 3.19 (2.22 / 2.12); eight, 256 of 128 4.82 / 2.96 (3.05 / 2.36), 512 of 64
// 5.16 / 3.33 (3.31 / 2.41), 128 of 256 4.66 / 3.74 (2.99 / 2.30).
template <int LPR, bool HARD, int IT>
hipError_t launch_team(SmallEpochArgs a, hipStream_t st) {
  bool team = false;
  if constexpr (IT > 2 || (!HARD && LPR < kWave)) {
    team = a.words != nullptr && a.steps * IT >= 4 * kSmallTurns;
    if (team) {
      const int count = (int)team_words((HARD ? 1 : 2) * 4 * LPR);
      hipLaunchKernelGGL(k_team_reset, dim3(16), dim3(256), 0, st, a.words, count, a.ends);
      hipLaunchKernelGGL((k_team_epoch<LPR, HARD, IT>), dim3(kTeamBlocks), dim3(2 * kTeamWaves * 64), 0, st, a);
    }
  }
  if (!team) a.words = nullptr;
  hipLaunchKernelGGL((k_small_epoch<LPR, HARD, IT>), dim3(1), dim3(kSmallWaves * 64), 0, st, a);
  return hipGetLastError();
}

template <int LPR, bool HARD>
hipError_t launch_turns(const SmallEpochArgs &a, hipStream_t st) {
  const int per_turn = kSmallWaves * (kWave / LPR);
  if (a.P <= 2 * per_turn) return launch_team<LPR, HARD, 2>(a, st);
  if (a.P <= 4 * per_turn) return launch_team<LPR, HARD, 4>(a, st);
  return launch_team<LPR, HARD, kSmallTurns>(a, st);
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

size_t small_epoch_words_bytes() { return team_words(2 * 4 * kWave) * sizeof(uint64_t); }

hipError_t launch_small_epoch(const SmallEpochArgs &a, bool hard, hipStream_t st) {
  if (!small_epoch_ok(a.d, a.ld, a.P) || a.steps < 1 || a.steps > kSmallEpochSteps) return hipErrorInvalidValue;
  switch (lanes_per_row(a.d)) {
    case 16: return launch_lpr<16>(a, hard, st);
    case 32: return launch_lpr<32>(a, hard, st);
    default: return launch_lpr<64>(a, hard, st);
  }
}

}  // namespace aa

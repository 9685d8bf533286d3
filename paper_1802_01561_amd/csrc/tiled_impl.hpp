// Tiled V-trace kernel, templated on the action count A (instantiated for
// 2 <= A <= 20 by tiled.hip and tiled_a*.hip; A = 9 is DeepMind Lab's set,
// A = 18 the full Atari set).
//
// Work split.  A tile is LANES consecutive lanes (batch entries) for the whole
// unroll; a workgroup walks a tile's time backwards in chunks of L steps (16 by
// default; 8 or 4 for the long-run tile shapes of 32 to 128 lanes; 32 to 256
// for tiles of 8 lanes down to 1, which spread a small batch over the chip), so
// every carry of the reverse recursion stays inside the workgroup.  Within a
// chunk, thread (lane, s) handles step t = t0 + s; the L threads of one lane are
// an aligned segment of a 16-lane DPP row of a wave, or 2 or 4 rows of a wave,
// or 2 or 4 whole waves.  When the batch has a whole
// multiple of the tiles the chip holds workgroups at once, each resident
// workgroup walks an equal share of tiles as one continuous sequence of chunks.
//
// Data path per chunk.
//  1. For each t the chunk's logits are one contiguous run of LANES*A elements
//     (1152 bytes for 16 lanes of fp32 logits with A = 18, nine 128-byte
//     lines; 4608 bytes for 64 lanes).  Threads copy both
//     tensors' runs with 16-byte loads (8- or 4-byte ones where a short run is
//     no multiple of 16 bytes) into LDS.  These whole-line logit loads
//     and the gradient stores are used once, so they carry the non-temporal
//     hint; the [T,B] scalars, whose 64-byte halves neighbouring workgroups
//     share in L2, do not.  The loads of chunk k+1
//     (and its per-step scalars) are issued before chunk k is computed and land
//     in registers, so their latency hides behind the arithmetic.
//  2. Each thread reads its own two rows from LDS: row maxima, exponent sums,
//     the importance ratio (float64, see device_common.hpp), rho and c.
//  3. The recursion v_t - V(x_t) = delta_t + gamma_t c_t (v_{t+1} - V(x_{t+1}))
//     (Remark 1) is an affine map per step.  A suffix scan across the row (DPP
//     row shifts) composes the chunk's maps; applying them to the carry from
//     the later chunk gives every v_t of the chunk at once.
//  4. Advantages, d_values and the gradient row follow.  Gradient rows go
//     through LDS so that the global stores are whole 16-byte vectors along the
//     contiguous [t, b0:b0+LANES, :] runs.
//
// Time rows may start at any element alignment (B * A odd, say): the vectors
// are then unaligned, which gfx950 reads and writes whole.  Where B is not a
// whole number of tiles the last tile moves back over its neighbour's lanes.
// (Copying such rows element by element took 2.4 times as long: T = 100,
// B = 16385, A = 18 254 -> 107 us.)
#pragma once

#include <atomic>
#include <type_traits>

#include "device_common.hpp"
#include "row_stats.hpp"
#include "wave_ops.hpp"

namespace vtrace {
namespace {

constexpr int kL = 16;  // default steps per chunk
constexpr int kFarLanes = 0;  // in place of a tile's lanes: the kernels for rows far apart

// DPP row_shr:(L-1): lane i of a 16-lane row reads lane i-L+1, so the last
// lane of every aligned L-lane segment reads the segment's first (L = 16 is
// kRowShr15).
template <int L>
constexpr int row_shr_to_last() {
  static_assert(L >= 2 && L <= 16, "segment length");
  return 0x110 + (L - 1);
}

// Vectors of 16, 8, 4 or 2 bytes in LDS, and the same at any element alignment
// in global memory: time rows of B * A elements start on a 16-byte boundary
// only for some B, and gfx950 reads and writes unaligned vectors whole.
template <int kBytes>
struct VecOf;
template <>
struct VecOf<16> {
  typedef v4u T;
};
template <>
struct VecOf<8> {
  typedef unsigned int T __attribute__((ext_vector_type(2)));
};
template <>
struct VecOf<4> {
  typedef unsigned int T;
};
template <>
struct VecOf<2> {
  typedef uint16_t T;
};
template <int kBytes, int kAlign>
using GlobalVec __attribute__((aligned(kAlign))) = typename VecOf<kBytes>::T;

constexpr int largest_vector(int bytes) {
  return bytes % 16 == 0 ? 16 : bytes % 8 == 0 ? 8 : bytes % 4 == 0 ? 4 : 2;
}
// LDS rows hold an odd number of vectors: with an even number several steps of
// a lane would read the same banks.
constexpr int odd_pitch(int vectors) { return vectors | 1; }

// L steps per chunk.  L = 16, 8 or 4: the L threads of a lane are one aligned
// segment of a 16-lane DPP row.  L = 32: a lane's threads are two DPP rows of
// a wave, steps 0-15 and 16-31 of the chunk.  L = 64, 128 or 256: one, two or
// four whole waves.
template <int A_, int LANES, typename In, int L>
struct Tile {
  static constexpr int A = A_;
  static constexpr int NT = LANES * L;                         // threads per workgroup
  static constexpr int SEG = LANES * A_;                       // elements per time row
  // Vector sizes: logits, float32 gradients, bfloat16 gradients (a time row's
  // run is a whole number of them).
  static constexpr int IN_VB = largest_vector(SEG * int(sizeof(In)));
  static constexpr int OUT_VB = largest_vector(SEG * 4);
  static constexpr int OUT16_VB = largest_vector(SEG * 2);
  typedef typename VecOf<IN_VB>::T InVec;
  typedef typename VecOf<OUT_VB>::T OutVec;
  static constexpr int IN_ROW = SEG * int(sizeof(In)) / IN_VB;  // vectors per time row, logits
  static constexpr int OUT_ROW = SEG * 4 / OUT_VB;              // vectors per time row, d_logits
  static constexpr int IN_PITCH_V = odd_pitch(IN_ROW);
  static constexpr int OUT_PITCH_V = odd_pitch(OUT_ROW);
  static constexpr int IN_TILE = L * IN_ROW;        // vectors per tensor and chunk
  static constexpr int OUT_TILE = L * OUT_ROW;
  static constexpr int IN_LDS = (L * IN_PITCH_V * IN_VB + 15) / 16 * 16;  // LDS bytes per tensor
  static constexpr int OUT_LDS = (L * OUT_PITCH_V * OUT_VB + 15) / 16 * 16;
  // Suffix-scan stages within a DPP row: log2 L, and 4 from L = 16 on.
  static constexpr int SCAN = L >= 16 ? 4 : L == 8 ? 3 : 2;
  // Short runs per time row share their first and last 128-byte line with the
  // neighbouring tiles: without the non-temporal hint those lines meet in L2
  // (T = 1000, A = 18, 1 lane: B = 2048 289 -> 178 us, B = 64 28.6 -> 24.7; 4
  // lanes, 288-byte runs, B = 2048 135 against 125).
  static constexpr bool kStream = LANES >= 16 || SEG * 4 >= 256;
  static constexpr int LANE_WAVES = L > kWave ? L / kWave : 1;  // waves that share a lane
  static constexpr int NV = (2 * IN_TILE + NT - 1) / NT;  // vectors per thread, both tensors
  static constexpr int NO = (OUT_TILE + NT - 1) / NT;     // gradient vectors per thread
  // LDS: the two logit tiles, and for the gradient kernels a separate
  // staging tile for the gradient rows, so that a chunk needs two barriers
  // (logits staged; gradients staged) instead of four.
  static constexpr int LDS16_TARGETS = 2 * IN_LDS / 16;
  static constexpr int LDS16_GRAD = (2 * IN_LDS + OUT_LDS) / 16;
  static constexpr int IN_PITCH = IN_PITCH_V * IN_VB / int(sizeof(In));  // elements per LDS row
  static constexpr int OUT_PITCH = OUT_PITCH_V * OUT_VB / 4;             // floats per LDS row
  static_assert(NT % kWave == 0 && NT <= 1024, "bad workgroup size");
  static_assert(L == 256 || L == 128 || L == 64 || L == 32 || L == 16 || L == 8 || L == 4, "steps per chunk");
};

// For 32-step chunks (two lanes per wave, each on two DPP rows): x at the
// thread of step `step` (0 or 16) of this thread's lane, i.e. at wave lane
// step or 32 + step.  Two scalar reads per 32-bit half and a select.
template <int kStep>
__device__ __forceinline__ double lane_step_f64(double x, bool upper_lane) {
  const unsigned long long u = __double_as_longlong(x);
  const int lo = static_cast<int>(u & 0xffffffffu), hi = static_cast<int>(u >> 32);
  const int lo0 = __builtin_amdgcn_readlane(lo, kStep), lo1 = __builtin_amdgcn_readlane(lo, 32 + kStep);
  const int hi0 = __builtin_amdgcn_readlane(hi, kStep), hi1 = __builtin_amdgcn_readlane(hi, 32 + kStep);
  const unsigned l = static_cast<unsigned>(upper_lane ? lo1 : lo0), h = static_cast<unsigned>(upper_lane ? hi1 : hi0);
  return __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(h) << 32) | l));
}

// x at thread kLane of the wave, as a wave-uniform value.
template <int kLane>
__device__ __forceinline__ double wave_read_f64(double x) {
  const unsigned long long u = __double_as_longlong(x);
  const unsigned lo = __builtin_amdgcn_readlane(static_cast<int>(u & 0xffffffffu), kLane);
  const unsigned hi = __builtin_amdgcn_readlane(static_cast<int>(u >> 32), kLane);
  return __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo));
}

// L > 64: what each wave leaves for the others of its lane in a chunk.
struct WaveMap {
  double G, D;  // the composite of its steps' maps
  double V;     // V(x) at its first step
};

// Per-thread state carried along the chunk walk.
struct Carry {
  double V, v, A;  // V(x_{t+1}), v_{t+1}, v_{t+1} - V(x_{t+1}) at the later chunk's first step
  double pg, base, ent;
};

// Which variant switches a kernel takes at run time: all of them (kGeneralCall),
// none (kPlainCall: plain V-trace, is_plain_vtrace), only the reward
// transform and the gradient dtype (kPlainRewards: is_plain_vtrace_any_rewards),
// or those two with behaviour log-probabilities in place of behaviour logits,
// so that no behaviour row is read (kPlainLogProbs: is_plain_vtrace_log_probs).
constexpr int kGeneralCall = 0;
constexpr int kPlainCall = 1;
constexpr int kPlainRewards = 2;
constexpr int kPlainLogProbs = 3;

// A lane's loss sums over the threads of its wave (all of them for L <= 64), in
// a fixed order, and with L <= 64 its lane_losses; then the wave's sums to red.
// `counted`: the lane joins the batch's sums (a last tile moved back repeats
// lanes of the tile before it).
template <int LANES, int L>
__device__ __forceinline__ void wave_losses(const StepArgs& a, const Carry& cy, int64_t b, bool counted, double* red) {
  constexpr int kSpan = L < kWave ? L : kWave;
  double pg = cy.pg, base = cy.base, ent = cy.ent;
#pragma unroll
  for (int off = kSpan / 2; off > 0; off >>= 1) {
    pg += __shfl_xor(pg, off, kSpan);
    base += __shfl_xor(base, off, kSpan);
    ent += __shfl_xor(ent, off, kSpan);
  }
  base *= a.baseline_cost;
  ent *= a.entropy_cost;
  if (L <= kWave && threadIdx.x % L == 0 && a.lane_losses) {
    a.lane_losses[3 * b + 0] = static_cast<float>(pg);
    a.lane_losses[3 * b + 1] = static_cast<float>(base);
    a.lane_losses[3 * b + 2] = static_cast<float>(ent);
  }
  if constexpr (L < kWave) {  // the wave's lanes
    if (!counted) pg = base = ent = 0.0;
#pragma unroll
    for (int off = kWave / 2; off >= L; off >>= 1) {
      pg += __shfl_xor(pg, off);
      base += __shfl_xor(base, off);
      ent += __shfl_xor(ent, off);
    }
  }
  const int wv = threadIdx.x / kWave;
  if (threadIdx.x % kWave == 0) {
    red[3 * wv + 0] = pg;
    red[3 * wv + 1] = base;
    red[3 * wv + 2] = ent;
  }
}

// After a barrier: lane_losses of lanes that span several waves, and thread 0
// publishes the workgroup's sums (the waves' in order).
template <int LANES, int L>
__device__ __forceinline__ void workgroup_losses(const StepArgs& a, int64_t b, int64_t b0, int64_t first_counted,
                                                 const double* red) {
  constexpr int kWaves = LANES * L / kWave;
  if constexpr (L > kWave) {
    if (threadIdx.x % L == 0 && a.lane_losses) {
      const int wv = threadIdx.x / kWave;
      for (int c = 0; c < 3; ++c) {
        double x = 0.0;
        for (int i = 0; i < L / kWave; ++i) x += red[3 * (wv + i) + c];
        a.lane_losses[3 * b + c] = static_cast<float>(x);
      }
    }
  }
  if (threadIdx.x == 0) {
    double p[3] = {0.0, 0.0, 0.0};
    for (int i = 0; i < kWaves; ++i) {
      if (L < kWave || b0 + i / (L < kWave ? 1 : L / kWave) >= first_counted)
        for (int c = 0; c < 3; ++c) p[c] += red[3 * i + c];
    }
    publish_losses(a, p[0], p[1], p[2]);
  }
}

// Walks one tile (kMulti false: `tile`, with the carry cy set up by the
// caller), or (kMulti true, L <= 16, whole tiles only) the tiles first_tile + i *
// tile_stride, i < ntiles, one after another as one loop over their chunks, so
// that the prefetch runs across tile boundaries; each lane's loss totals are
// then added to acc[3 * lane], a slot only the lane's step-0 thread touches.
// kFar: L rows of an array lie further apart than 32-bit offsets reach.
template <int A_, int LANES, typename In, int L, bool kGrad, bool kPrecise, bool kMulti, int kPlain, bool kFar>
__device__ __forceinline__ void chunk_walk(const StepArgs& a, v4u* lds, int64_t first_tile,
                                           int64_t tile_stride, int64_t ntiles, Carry& cy,
                                           double* acc, WaveMap* maps, double* red) {
  static_assert(!kMulti || L <= 16, "the multi-tile walk takes lanes within one DPP row");
  using S = Tile<A_, LANES, In, L>;
  constexpr int NT = S::NT;
  typedef typename S::InVec InVec;
  typedef typename S::OutVec OutVec;
  InVec* const lds_in = reinterpret_cast<InVec*>(lds);  // target logits, then behaviour logits
  constexpr int kInLds = S::IN_LDS / S::IN_VB;          // vectors of one tensor
  v4u* const lds_z = lds;
  v4u* const lds_y = lds + S::IN_LDS / 16;
  OutVec* const lds_g = reinterpret_cast<OutVec*>(lds + 2 * S::IN_LDS / 16);  // gradient staging (kGrad)

  const int tid = threadIdx.x;
  const int lane_local = tid / L;
  const int s = tid % L;
  const int wl = tid % kWave;  // the thread's place in its wave
  const int64_t T = a.T, B = a.B;
  const int nchunks = static_cast<int>((T + L - 1) / L);

  // Byte stride of one time row of logits.
  const int64_t in_row = B * A_ * int64_t(sizeof(In));
  // kPlain: the call is plain V-trace (q_s from v_{s+1}, behaviour logits or,
  // for kPlainLogProbs, log-probabilities), so every variant switch below is a
  // compile-time constant; kPlainCall also has rewards as given and float32
  // gradients, while the other plain kernels keep the reward transform and
  // the gradient dtype run-time switches.
  const int correction = kPlain ? kCorrVtrace : a.correction;
  const int q_estimate = kPlain ? 0 : a.q_estimate;
  const int reward_transform = kPlain == kPlainCall ? 0 : a.reward_transform;
  const bool beh_lp = kPlain == kPlainLogProbs || (!kPlain && a.behaviour_log_probs != 0);
  // No-correction and epsilon-correction never look at the behaviour policy.
  const bool no_ratio = correction == kCorrNone || correction == kCorrEpsilon;
  const bool skip_y = beh_lp || no_ratio;
  const bool grad_bf16 = kPlain != kPlainCall && a.grad_bf16 != 0;
  const int64_t gsz = grad_bf16 ? 2 : 4;  // bytes per gradient element
  const int64_t out_row = B * A_ * gsz;
  const float* const lmu_g = static_cast<const float*>(a.behaviour_logits);
  // A tile's first lane.  Where B is not a whole number of tiles the last tile
  // moves back so as to end with the batch (B >= LANES): the lanes it shares
  // with the tile before it are computed and written twice, with the same bits,
  // and counted once in the loss sums.
  auto first_lane = [&](int64_t tile) {
    const int64_t b0 = tile * LANES;
    return kMulti || b0 <= B - LANES ? b0 : B - LANES;
  };

  // Register prefetch: NV vectors covering both tensors, plus this thread's
  // action, reward, discount and value, and at a tile's first chunk its lane's
  // bootstrap value.
  InVec pre[S::NV];
  int32_t p_act = 0;
  float p_r = 0.f, p_g = 0.f, p_V = 0.f, p_Vn = 0.f, p_lmu = 0.f, p_boot = 0.f;

  // Addresses are a wave-uniform base (the chunk's row 0 at the tile's first
  // lane, in scalar registers) plus a per-thread 32-bit offset, the form of the
  // loads' and stores' scalar-base addressing; the launcher checks that L rows
  // of every array fit 32-bit offsets, or takes kFar and 64-bit ones.
  using Off = std::conditional_t<kFar, uint64_t, uint32_t>;
  typedef GlobalVec<S::IN_VB, sizeof(In)> GlobalIn;
  const Off in_row_off = static_cast<Off>(in_row);
  const Off out_row_off = static_cast<Off>(out_row);
  const Off b_off = static_cast<Off>(B);
  auto prefetch = [&](int64_t tile, int k) {
    const int64_t b0 = first_lane(tile);
    const int64_t t0 = T - static_cast<int64_t>(k + 1) * L;
    const int neg = t0 < 0 ? static_cast<int>(-t0) : 0;  // rows before t = 0 reread row `neg`
    const int64_t row0 = t0 * B + b0;                     // may be negative: only rows >= neg are read
    const gptr<const char> zg = offset_bytes(a.target_logits, row0 * A_ * int64_t(sizeof(In)));
    const gptr<const char> yg = offset_bytes(a.behaviour_logits, row0 * A_ * int64_t(sizeof(In)));
    static_for<S::NV>([&](auto I) {
      constexpr int i = decltype(I)::value;
      // Which tensor vector i of every thread belongs to, where that is known
      // at compile time (all but the vector that straddles the two tiles).
      constexpr bool kAllZ = (i + 1) * NT <= S::IN_TILE;
      constexpr bool kAllY = i * NT >= S::IN_TILE;
      constexpr bool kTail = i * NT + NT > 2 * S::IN_TILE;
      const int f = tid + i * NT;
      const bool is_y = kAllY || (!kAllZ && f >= S::IN_TILE);
      if ((!kTail || f < 2 * S::IN_TILE) && !(is_y && skip_y)) {
        const int g = is_y ? f - S::IN_TILE : f;
        int r = g / S::IN_ROW;
        const int c = g % S::IN_ROW;
        r = r < neg ? neg : r;
        const Off off = static_cast<Off>(r) * in_row_off + static_cast<Off>(c * S::IN_VB);
        const auto src = reinterpret_cast<gptr<const GlobalIn>>((is_y ? yg : zg) + off);
        if constexpr (S::kStream)
          pre[i] = __builtin_nontemporal_load(src);
        else
          pre[i] = *src;
      }
    });
    const Off off = static_cast<Off>(s < neg ? neg : s) * b_off + static_cast<Off>(lane_local);
    p_act = offset_elems(a.actions, row0)[off];
    p_r = offset_elems(a.rewards, row0)[off];
    p_g = offset_elems(a.discounts, row0)[off];
    p_V = offset_elems(a.values, row0)[off];
    if constexpr (L > kWave) {  // V(x_{t+1}), which a wave's last thread cannot take from a neighbour
      const int sn = s + 1 < L ? s + 1 : s;
      p_Vn = offset_elems(a.values, row0)[static_cast<Off>(sn < neg ? neg : sn) * b_off +
                                          static_cast<Off>(lane_local)];
    }
    // (Cleared first: a value kept where nothing is loaded would make the
    // compiler wait for the loads just issued.)
    p_lmu = p_boot = 0.f;
    if (beh_lp && !no_ratio) p_lmu = offset_elems(lmu_g, row0)[off];
    if (kMulti && k == 0) p_boot = a.bootstrap_value[b0 + lane_local];
  };

  const double rho_bar = a.rho_bar, c_bar = a.c_bar, lam = a.lambda;
  const float ce = a.entropy_cost;

  int64_t tile = first_tile;  // advanced by the multi-tile walk only
  int k = 0;
  // Chunks to walk: a tile's, or all the tiles' (which may exceed 32 bits).
  using Count = std::conditional_t<kMulti, int64_t, int>;
  const Count total = kMulti ? static_cast<Count>(ntiles * nchunks) : static_cast<Count>(nchunks);
  prefetch(tile, 0);
  // The first chunk is waited for here: with loads outstanding on the loop's
  // entry the compiler waits, in every iteration, for the first of the loads
  // just issued as well (30-task batch 22.8 -> 24.7 us).
  __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
  for (Count it = 0; it < total; ++it) {
    const int64_t b0 = first_lane(tile);
    const int64_t b = b0 + lane_local;
    if constexpr (kMulti) {
      if (k == 0) {
        // A new tile: the carry past its last step is the bootstrap value
        // (v_T = V(x_T), so v_T - V(x_T) = 0).
        cy.V = cy.v = p_boot;
        cy.A = 0.0;
      }
    }
    const int64_t t0 = T - static_cast<int64_t>(k + 1) * L;
    const int64_t t = t0 + s;
    const bool step_ok = t >= 0;
    // [T,B] element (t, b) as the chunk's uniform row 0 plus an offset.
    const int64_t row0 = t0 * B + b0;
    const Off soff = static_cast<Off>(s) * b_off + static_cast<Off>(lane_local);

    // Every thread is past the previous chunk's row reads: the gradient
    // kernels passed their staging barrier after them; the targets-only
    // kernel waits here.
    if constexpr (!kGrad) __syncthreads();
    static_for<S::NV>([&](auto I) {
      constexpr int i = decltype(I)::value;
      const int f = tid + i * NT;
      const bool is_y = f >= S::IN_TILE;
      if ((i * NT + NT <= 2 * S::IN_TILE || f < 2 * S::IN_TILE) && !(is_y && skip_y)) {
        const int g = is_y ? f - S::IN_TILE : f;
        const int r = g / S::IN_ROW, c = g % S::IN_ROW;
        lds_in[(is_y ? kInLds : 0) + r * S::IN_PITCH_V + c] = pre[i];
      }
    });
    int32_t act = p_act;
    float r32 = p_r;
    const float g32 = p_g, V32 = p_V, lmu = p_lmu;
    [[maybe_unused]] const float Vn32 = p_Vn;
    // The next chunk's loads go out before the staging barrier (their
    // registers are free once staged) with float32 logits on the long-run
    // shapes: stress step 0.730 -> 0.714 ms, bf16 gradients 0.682 -> 0.670,
    // targets-only 0.550 -> 0.537.  With bf16 logits (and the raised
    // priority below) only the kernel that reads no behaviour rows gains
    // (0.485-0.491 -> 0.466-0.468 ms, with bf16 gradients 0.453-0.455 ->
    // 0.432-0.433); the others, and the 16-step tiles, measured up to 1%
    // slower and keep them after it.
    constexpr bool kEarlyPrefetch =
        L <= 8 && (std::is_same_v<In, float> || kPlain == kPlainLogProbs);
    // The wave issues those loads at raised priority, so that the other
    // waves' arithmetic on the same SIMD does not delay them: stress step
    // 0.727-0.730 -> 0.714-0.716 ms, 16-step tiles with float32 logits and
    // bf16 logits on the long-run shapes 1-2% faster; bf16 logits on the
    // 16-step tiles measured 1% slower with it and keep normal priority.
    constexpr bool kPrioPrefetch = std::is_same_v<In, float> || L <= 8;
    auto next_prefetch = [&]() {
      if constexpr (kMulti) {
        if (it + 1 < total) {
          const bool next_tile = k + 1 == nchunks;
          prefetch(next_tile ? tile + tile_stride : tile, next_tile ? 0 : k + 1);
        }
      } else {
        if (k + 1 < nchunks) prefetch(tile, k + 1);
      }
    };
    auto issue_prefetch = [&]() {
      if constexpr (kPrioPrefetch) __builtin_amdgcn_s_setprio(2);
      next_prefetch();
      if constexpr (kPrioPrefetch) __builtin_amdgcn_s_setprio(0);
    };
    if constexpr (kEarlyPrefetch) issue_prefetch();
    __syncthreads();
    if constexpr (!kEarlyPrefetch) issue_prefetch();
    r32 = transform_reward(r32, reward_transform);
    if (!step_ok) act = 0;  // rows that do not exist carry a harmless action

    // This thread's rows.
    In* zr = reinterpret_cast<In*>(lds_z) + s * S::IN_PITCH + lane_local * A_;
    const In* yr = reinterpret_cast<const In*>(lds_y) + s * S::IN_PITCH + lane_local * A_;
    const bool act_ok = act >= 0 && act < A_;
    const int act_c = act_ok ? act : 0;
    if (!act_ok) raise_error_flag(a.error_flag);
    // e_j and z_j for the gradient.  The plain loss kernels (every kPlain
    // mode) keep both in registers from the row statistics to the gradient
    // (36 VGPRs that their two waves per SIMD have), which spares each row two
    // LDS round trips; the general kernel, which needs those registers for its
    // switches, takes e_j through this thread's row of the gradient staging tile (free
    // since the previous chunk's stores, which every thread finished before
    // this chunk's logits barrier), where the gradient row later replaces
    // them, and read z_j again from the logit tile.  The targets-only kernels
    // use neither.
    static_assert(!kGrad || kPrecise, "loss kernels form their exponent sums in float64");
    constexpr bool kRowRegs = kGrad && kPlain;
    float e_reg[A_], z_reg[A_];
    float* const lo = kGrad ? reinterpret_cast<float*>(lds_g) + s * S::OUT_PITCH + lane_local * A_ : e_reg;
    float* const e_out = kGrad && !kRowRegs ? lo : e_reg;
    RowStats st = row_stats<A_, kPrecise, kGrad && !kRowRegs>(zr, yr, act_c, act_ok, beh_lp, no_ratio, lmu, e_out,
                                                              kRowRegs ? z_reg : nullptr);
    const StepWeights w = variant_weights(correction, clip_above(st.ratio, rho_bar),
                                          lam * clip_above(st.ratio, c_bar), lam, act_ok);

    const double r = r32, g = g32, V = V32;
    // kSeg: steps of a lane within one DPP row; sr: this thread's place there.
    constexpr int kSeg = L < 16 ? L : 16;
    const int sr = s % kSeg;
    const bool upper_lane = wl >= 32;  // L = 32: the wave's second lane
    double V16 = 0.0;                  // L = 32: V(x) at step 16 of the lane
    if constexpr (L == 32) V16 = lane_step_f64<16>(V, upper_lane);
    // L >= 64: x at the next step of the wave (its last thread takes none).
    [[maybe_unused]] auto wave_next = [&](double x) {
      const double x16 = wave_read_f64<16>(x), x32 = wave_read_f64<32>(x), x48 = wave_read_f64<48>(x);
      double n = dpp_f64<kRowShl1>(x);
      n = wl == 15 ? x16 : n;
      n = wl == 31 ? x32 : n;
      return wl == 47 ? x48 : n;
    };
    double V_next;
    if constexpr (L > kWave)
      V_next = Vn32;
    else if constexpr (L == kWave)
      V_next = wave_next(V);
    else
      V_next = dpp_f64<kRowShl1>(V);
    if (L == 32 && s == 15) V_next = V16;
    if (s == L - 1) V_next = cy.V;
    const double delta = w.rho_v * (r + g * V_next - V);

    // Suffix scan over the lane's segment.  Its last step first absorbs the
    // carry from the later chunk, so that after the scan D holds v_t - V(x_t)
    // on every thread: (G, D) composes the maps of steps s..L-1 applied to
    // that carry.  With 32 steps the scan runs in each DPP row, and the lower
    // row then composes its maps with the upper row's first step.
    double G = g * w.c_v, D = delta;
    if (s == L - 1) D = fma(G, cy.A, D);
    static_for<S::SCAN>([&](auto I) {
      constexpr int off = 1 << decltype(I)::value;
      const double Gn = dpp_f64<0x100 + off>(G);
      const double Dn = dpp_f64<0x100 + off>(D);
      if (sr + off < kSeg) {
        D = fma(G, Dn, D);
        G = G * Gn;
      }
    });
    double D16 = 0.0;  // L = 32: v - V(x) at step 16 of the lane
    if constexpr (L == 32) {
      D16 = lane_step_f64<16>(D, upper_lane);
      if (s < 16) D = fma(G, D16, D);
    }
    // L >= 64: the wave's DPP rows are composed last to first, and the waves of
    // a lane then exchange their composites through LDS (one more barrier);
    // the later waves' composites applied to the carry give what enters this
    // wave.
    double wave_in = 0.0;  // L > 64: v - V(x) at the next wave's first step
    if constexpr (L >= kWave) {
      const double D48 = wave_read_f64<48>(D), G48 = wave_read_f64<48>(G);
      const double G32 = wave_read_f64<32>(G), G16 = wave_read_f64<16>(G);
      const double D32 = fma(G32, D48, wave_read_f64<32>(D));
      const double D16w = fma(G16, D32, wave_read_f64<16>(D));
      const double Dr = wl < 16 ? D16w : wl < 32 ? D32 : D48;
      if (wl < 48) D = fma(G, Dr, D);
      if constexpr (L > kWave) {
        const double Gr2 = G32 * G48, Gr1 = G16 * Gr2;
        const double Gr = wl < 16 ? Gr1 : wl < 32 ? Gr2 : G48;
        if (wl < 48) G *= Gr;
        constexpr int W = S::LANE_WAVES;
        const int w_lane = (tid / kWave) % W;  // this wave's place in its lane
        WaveMap* const lane_maps = maps + lane_local * W;
        if (wl == 0) lane_maps[w_lane] = WaveMap{G, D, V};
        __syncthreads();
        double c = lane_maps[W - 1].D;  // the last wave absorbed the carry
        wave_in = c;
        static_for<W - 1>([&](auto I) {
          constexpr int w2 = W - 2 - decltype(I)::value;
          if (w_lane == w2) {
            wave_in = c;
            D = fma(G, c, D);
          }
          c = fma(lane_maps[w2].G, c, lane_maps[w2].D);
        });
        cy.A = c;
      }
    }
    const double A_t = D;  // v_t - V(x_t)
    const double v_t = V + A_t;
    double v_next;
    if constexpr (L >= kWave)
      v_next = wave_next(v_t);
    else
      v_next = dpp_f64<kRowShl1>(v_t);
    if (L == 32 && s == 15) v_next = V16 + D16;
    if (L > kWave && wl == kWave - 1) v_next = V_next + wave_in;
    if (s == L - 1) v_next = cy.v;
    const double q_next = q_estimate == kQBaseline ? V_next : v_next;
    const double adv = w.rho_pg * (r + g * q_next - V);

    // The segment's first step becomes the carry of the earlier chunk, held by
    // the segment's last thread, the only one that reads it.
    if constexpr (L == 32) {
      cy.A = lane_step_f64<0>(A_t, upper_lane);
      cy.v = lane_step_f64<0>(v_t, upper_lane);
      cy.V = lane_step_f64<0>(V, upper_lane);
    } else if constexpr (L == kWave) {
      cy.A = wave_read_f64<0>(A_t);
      cy.v = wave_read_f64<0>(v_t);
      cy.V = wave_read_f64<0>(V);
    } else if constexpr (L > kWave) {  // cy.A is set above
      cy.V = maps[lane_local * S::LANE_WAVES].V;
      cy.v = cy.V + cy.A;
    } else {
      cy.A = dpp_f64<row_shr_to_last<L>()>(A_t);
      cy.v = dpp_f64<row_shr_to_last<L>()>(v_t);
      cy.V = dpp_f64<row_shr_to_last<L>()>(V);
    }

    auto store_targets = [&]() {
      if (step_ok) {
        if (a.vs) offset_elems(a.vs, row0)[soff] = static_cast<float>(v_t);
        if (a.pg_adv) offset_elems(a.pg_adv, row0)[soff] = static_cast<float>(adv);
      }
    };
    // The loss kernels with chunks of 16 steps or more wait for the next chunk's
    // loads before this chunk's stores (below); the others store as they go.
    constexpr bool kWaitFirst = kGrad && L >= 16;
    if constexpr (!kWaitFirst) store_targets();

    if constexpr (kGrad) {
      // d_logits_j = adv (pi_j - 1[j=a]) + ce pi_j (log pi_j + H), where
      // log pi_j + H = z_j - K.  For j != a this is e_j (alpha + beta z_j).
      const float K = st.mz + st.log_s - st.H;
      // epsilon-correction: the policy-gradient term is -adv log(pi_a + eps),
      // whose gradient is adv pi_a/(pi_a + eps) (pi_j - 1[j=a]).
      const float pa = st.e_a * st.inv_s;
      const bool eps_mode = correction == kCorrEpsilon;
      const float pg_w = eps_mode ? pa / (pa + a.epsilon) : 1.0f;
      const float adv32 = static_cast<float>(adv) * pg_w;
      const float beta = st.inv_s * ce;
      const float alpha = st.inv_s * adv32 - beta * K;
      const float za = st.za;
      const float out_a = -adv32 * st.one_minus_pa + ce * pa * (za - K);
      if (step_ok) {
        const double log_pa = !act_ok ? NAN : eps_mode ? log_prob_plus_eps<kPrecise>(st, a.epsilon) : st.log_pa;
        if constexpr (!kWaitFirst)
          offset_elems(a.d_values, row0)[soff] = static_cast<float>(a.baseline_cost * (V - v_t));
        cy.pg += -adv * log_pa;
        cy.base += 0.5 * A_t * A_t;
        cy.ent += -static_cast<double>(st.H);
      }
      float out[A_];
#pragma unroll
      for (int j = 0; j < A_; ++j) out[j] = e_out[j] * fmaf(beta, kRowRegs ? z_reg[j] : logit_to_float(zr[j]), alpha);
#pragma unroll
      for (int j = 0; j < A_; ++j) lo[j] = out[j];
      lo[act_c] = act_ok ? out_a : NAN;
      // L >= 32 (the shapes of short calls): the workgroup's loss sums are formed
      // and published around the last chunk's gradient barrier, so that their
      // round trip to memory and the gradient stores overlap.
      constexpr bool kEarlyLosses = !kMulti && L >= 32;
      if constexpr (kEarlyLosses) {
        if (k == nchunks - 1) wave_losses<LANES, L>(a, cy, b, b >= tile * LANES, red);
      }
      // The next chunk's loads are waited for here, before this chunk's stores:
      // after them the wait would cover the stores as well, which so have the
      // whole next chunk to complete (T = 100: B = 1021, A = 6 12.5 -> 11.7 us,
      // B = 32, A = 9 7.7 -> 7.4; B = 8192, A = 18 49.2 -> 47.8).  With the 8-step
      // chunks of the stress batch, whose next loads have only just gone out,
      // it cost 7% (702 -> 746 us).
      if constexpr (kWaitFirst) __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
      __syncthreads();
      if constexpr (kEarlyLosses) {
        if (k == nchunks - 1) workgroup_losses<LANES, L>(a, b, b0, tile * LANES, red);
      }
      if constexpr (kWaitFirst) {
        store_targets();
        if (step_ok) offset_elems(a.d_values, row0)[soff] = static_cast<float>(a.baseline_cost * (V - v_t));
      }
      const int neg = t0 < 0 ? static_cast<int>(-t0) : 0;
      const gptr<char> dgr = offset_bytes(a.d_logits, row0 * A_ * gsz);  // the chunk's row 0
      if (!grad_bf16) {
        // The kernel that reads no behaviour rows spends a larger share of
        // each chunk on these stores; issued at raised priority its stress
        // step took 0.528-0.530 -> 0.519-0.522 ms (the default kernel's
        // measured 0.4% slower with it).
        typedef GlobalVec<S::OUT_VB, 4> GlobalOut;
        if constexpr (kPlain == kPlainLogProbs) __builtin_amdgcn_s_setprio(2);
        static_for<S::NO>([&](auto I) {
          constexpr int i = decltype(I)::value;
          const int f = tid + i * NT;
          if (i * NT + NT <= S::OUT_TILE || f < S::OUT_TILE) {
            const int rr = f / S::OUT_ROW, cc = f % S::OUT_ROW;
            if (rr >= neg) {
              const auto dst = reinterpret_cast<gptr<GlobalOut>>(
                  dgr + (static_cast<Off>(rr) * out_row_off + static_cast<Off>(cc * S::OUT_VB)));
              if constexpr (S::kStream)
                __builtin_nontemporal_store(lds_g[rr * S::OUT_PITCH_V + cc], dst);
              else
                *dst = lds_g[rr * S::OUT_PITCH_V + cc];
            }
          }
        });
        if constexpr (kPlain == kPlainLogProbs) __builtin_amdgcn_s_setprio(0);
      } else {
        // bfloat16 rows: each store packs its values from the float32 tile
        // (a 16-byte one two 16-byte LDS vectors).
        typedef GlobalVec<S::OUT16_VB, 2> GlobalOut;
        constexpr int kVals = S::OUT16_VB / 2;  // values per store
        constexpr int kRow = S::SEG / kVals, kTile = L * kRow;
        for (int f = tid; f < kTile; f += NT) {
          const int rr = f / kRow, cc = f % kRow;
          if (rr >= neg) {
            typename VecOf<S::OUT16_VB>::T pk;
            if constexpr (kVals == 8) {
              const v4u* const src = reinterpret_cast<const v4u*>(lds_g + rr * S::OUT_PITCH_V) + 2 * cc;
              const v4u lo = src[0], hi = src[1];
              pk.x = pack_bf16x2(__uint_as_float(lo.x), __uint_as_float(lo.y));
              pk.y = pack_bf16x2(__uint_as_float(lo.z), __uint_as_float(lo.w));
              pk.z = pack_bf16x2(__uint_as_float(hi.x), __uint_as_float(hi.y));
              pk.w = pack_bf16x2(__uint_as_float(hi.z), __uint_as_float(hi.w));
            } else {
              const float* const src = reinterpret_cast<const float*>(lds_g + rr * S::OUT_PITCH_V) + kVals * cc;
              if constexpr (kVals == 4) {
                pk.x = pack_bf16x2(src[0], src[1]);
                pk.y = pack_bf16x2(src[2], src[3]);
              } else if constexpr (kVals == 2) {
                pk = pack_bf16x2(src[0], src[1]);
              } else {
                pk = to_bf16(src[0]);
              }
            }
            const auto dst = reinterpret_cast<gptr<GlobalOut>>(
                dgr + (static_cast<Off>(rr) * out_row_off + static_cast<Off>(cc * S::OUT16_VB)));
            if constexpr (S::kStream)
              __builtin_nontemporal_store(pk, dst);
            else
              *dst = pk;
          }
        }
      }
      if (kMulti && k == nchunks - 1) {
        // The tile's last chunk: this lane's totals over the row (fixed
        // butterfly order), then the workgroup's running sums.
        double lp = cy.pg, lb = cy.base, le = cy.ent;
#pragma unroll
        for (int off = L / 2; off > 0; off >>= 1) {
          lp += __shfl_xor(lp, off, L);
          lb += __shfl_xor(lb, off, L);
          le += __shfl_xor(le, off, L);
        }
        lb *= a.baseline_cost;
        le *= a.entropy_cost;
        if (s == 0) {
          if (a.lane_losses) {
            a.lane_losses[3 * b + 0] = static_cast<float>(lp);
            a.lane_losses[3 * b + 1] = static_cast<float>(lb);
            a.lane_losses[3 * b + 2] = static_cast<float>(le);
          }
          acc[3 * lane_local + 0] += lp;
          acc[3 * lane_local + 1] += lb;
          acc[3 * lane_local + 2] += le;
        }
        cy.pg = cy.base = cy.ent = 0.0;
      }
    }
    if (++k == nchunks && kMulti) {
      k = 0;
      tile += tile_stride;
    }
  }
}

// Tile of a workgroup.  Below 64 lanes a tile's share of a [T,B] time row is
// under 256 bytes and neighbouring tiles share its 128-byte lines, so
// xcd_tile puts workgroups that run side by side on one XCD on neighbouring
// tiles, which then meet in that XCD's L2.  From 64 lanes on nothing is shared
// and tiles go in workgroup order, which measured 1-4% faster for the long-run
// shapes (and the XCD order 1% faster for 16-lane tiles).
template <int LANES>
__device__ __forceinline__ int64_t first_tile_of_workgroup() {
  if constexpr (LANES >= 64) return blockIdx.x;
  return xcd_tile(blockIdx.x, gridDim.x);
}

// kMulti false: one workgroup per tile, tile first_tile_of_workgroup().
//
// kMulti true: the grid is exactly the workgroups the chip holds at once and
// each walks tiles_per_wg whole tiles, first_tile_of_workgroup() + i * gridDim.x.
// When a batch has a whole multiple of that many tiles, this runs it as one
// even generation: one workgroup per tile would instead start a second wave of
// workgroups whenever a slot frees, and leave the chip partly idle at the end.
// The long-run float32 loss kernels of A = 9 use few enough registers for a third
// wave per SIMD, and are held to two: their batches are whole generations of two
// workgroups a CU, which a third slot lets start unevenly (T = 300, B = 32768 227 ->
// 238 us; three fit the kernels of other types and options from the start).
template <int A_, typename In, int L, bool kGrad, int kPlain>
constexpr bool kHoldsTwo = kGrad && L <= 8 && A_ == 9 && std::is_same_v<In, float> &&
                           (kPlain == kPlainCall || kPlain == kPlainRewards);

// The fp64 ratio mode with A > 18 is asked for two waves per SIMD explicitly:
// left to itself the compiler gives A = 19 two registers more than fit.
template <int A_, int LANES, typename In, int L, bool kGrad, bool kPrecise, bool kMulti, int kPlain = kGeneralCall,
          bool kFar = false>
__global__ __launch_bounds__(LANES* L) __attribute__((amdgpu_waves_per_eu(
    (kPrecise && A_ >= 18) ? 2 : 1, kHoldsTwo<A_, In, L, kGrad, kPlain> ? 2 : 8))) void tiled_kernel(
    StepArgs a, int64_t tiles_per_wg) {
  using S = Tile<A_, LANES, In, L>;
  constexpr int NT = S::NT;
  __shared__ v4u lds[kGrad ? S::LDS16_GRAD : S::LDS16_TARGETS];
  __shared__ double red_scratch[3 * (NT / kWave)];
  __shared__ WaveMap maps[L > kWave ? NT / kWave : 1];

  const int lane_local = threadIdx.x / L;
  const int s = threadIdx.x % L;

  if constexpr (kMulti) {
    __shared__ double acc[3 * LANES];  // per-lane loss sums over the workgroup's tiles
    if (s == 0) acc[3 * lane_local + 0] = acc[3 * lane_local + 1] = acc[3 * lane_local + 2] = 0.0;
    Carry cy{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    chunk_walk<A_, LANES, In, L, kGrad, kPrecise, true, kPlain, kFar>(
        a, lds, first_tile_of_workgroup<LANES>(), gridDim.x, tiles_per_wg, cy, acc, maps, red_scratch);
    if constexpr (kGrad) {
      double pg = 0.0, base = 0.0, ent = 0.0;
      if (s == 0) {
        pg = acc[3 * lane_local + 0];
        base = acc[3 * lane_local + 1];
        ent = acc[3 * lane_local + 2];
      }
      finish_losses<NT>(a, pg, base, ent, red_scratch);
    }
  } else {
    const int64_t tile = first_tile_of_workgroup<LANES>();
    // (chunk_walk's first_lane)
    const int64_t b0 = tile * LANES <= a.B - LANES ? tile * LANES : a.B - LANES;
    const int64_t b = b0 + lane_local;
    const double boot = static_cast<double>(a.bootstrap_value[b]);
    Carry cy{boot, boot, 0.0, 0.0, 0.0, 0.0};
    chunk_walk<A_, LANES, In, L, kGrad, kPrecise, false, kPlain, kFar>(a, lds, tile, 0, 1, cy, nullptr, maps,
                                                                       red_scratch);

    if constexpr (kGrad) {
      if constexpr (L >= 32) {
        finish_ticket<NT>(a, red_scratch);
      } else {
        // Per-lane totals over the row (fixed butterfly order), then the workgroup.
        double pg = cy.pg, base = cy.base, ent = cy.ent;
#pragma unroll
        for (int off = L / 2; off > 0; off >>= 1) {
          pg += __shfl_xor(pg, off, L);
          base += __shfl_xor(base, off, L);
          ent += __shfl_xor(ent, off, L);
        }
        base *= a.baseline_cost;
        ent *= a.entropy_cost;
        if (s == 0 && a.lane_losses) {
          a.lane_losses[3 * b + 0] = static_cast<float>(pg);
          a.lane_losses[3 * b + 1] = static_cast<float>(base);
          a.lane_losses[3 * b + 2] = static_cast<float>(ent);
        }
        if (s != 0 || b < tile * LANES) pg = base = ent = 0.0;  // (lanes of the tile before count there)
        finish_losses<NT>(a, pg, base, ent, red_scratch);
      }
    }
  }
}

// Workgroups of the multi-tile kernel that fit on a compute unit at once,
// asked of the runtime once (0 if it cannot say).
template <int A_, int LANES, typename In, int L, bool kGrad>
int multi_workgroups_per_cu() {
  static std::atomic<int> cached{-1};
  int n = cached.load(std::memory_order_relaxed);
  if (n < 0) {
    int blocks = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &blocks, reinterpret_cast<const void*>(tiled_kernel<A_, LANES, In, L, kGrad, false, true>),
            LANES * L, 0) != hipSuccess) {
      (void)hipGetLastError();  // not a launch error: the single-tile kernel runs instead
      blocks = 0;
    }
    n = blocks > 0 ? blocks : 0;
    cached.store(n, std::memory_order_relaxed);
  }
  return n;
}

// Workgroups of the single-tile float32-ratio kernel that fit on a compute
// unit at once, asked of the runtime once (0 if it cannot say).
template <int A_, int LANES, typename In, int L, bool kGrad>
int single_workgroups_per_cu() {
  static std::atomic<int> cached{-1};
  int n = cached.load(std::memory_order_relaxed);
  if (n < 0) {
    int blocks = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &blocks, reinterpret_cast<const void*>(tiled_kernel<A_, LANES, In, L, kGrad, false, false>),
            LANES * L, 0) != hipSuccess) {
      (void)hipGetLastError();
      blocks = 0;
    }
    n = blocks > 0 ? blocks : 0;
    cached.store(n, std::memory_order_relaxed);
  }
  return n;
}

// Compute units of the current device (0 if the runtime cannot say).
int compute_units() {
  constexpr int kMaxDevices = 64;
  static std::atomic<int> cached[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    (void)hipGetLastError();
    return 0;
  }
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n <= 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
      (void)hipGetLastError();
      return 0;
    }
    cached[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

// Launches the kernel; returns its grid size.  The multi-tile kernel runs when
// the batch is a whole number of tiles, two or more of its workgroups fit on a CU, the
// tiles are a whole multiple (at least two) of the resident workgroups, and the
// ratio takes the float32 mode.  Elsewhere one workgroup per tile measured as
// fast or faster: a batch that is not a whole multiple would leave some
// workgroups a tile short, the float64 ratio mode has no registers to spare for
// the longer walk, and with one resident workgroup per CU (the 512-thread
// kernel of bfloat16 logits with A = 18) the multi-tile walk measured 4-10%
// slower.
template <int A_, int LANES, typename In, int L, bool kGrad, bool kPrecise, int kPlain = kGeneralCall>
int64_t launch_kernel(const StepArgs& a, hipStream_t st, int64_t tiles, bool allow_multi) {
  if constexpr (!kPrecise && L <= 16) {
    const int per_cu = allow_multi && a.B % LANES == 0 ? multi_workgroups_per_cu<A_, LANES, In, L, kGrad>() : 0;
    if (per_cu >= 2) {
      const int64_t resident = static_cast<int64_t>(per_cu) * compute_units();
      if (resident > 0 && tiles >= 2 * resident && tiles % resident == 0) {
        hipLaunchKernelGGL((tiled_kernel<A_, LANES, In, L, kGrad, false, true>), dim3(static_cast<unsigned>(resident)),
                           dim3(LANES * L), 0, st, a, tiles / resident);
        return resident;
      }
    }
  }
  hipLaunchKernelGGL((tiled_kernel<A_, LANES, In, L, kGrad, kPrecise, false, kPlain>),
                     dim3(static_cast<unsigned>(tiles)), dim3(LANES * L), 0, st, a, int64_t(1));
  return tiles;
}

// Loss kernels always take the float64 exponent sums; a targets-only call
// takes them when its weights can amplify ratio errors.  kFastOnly: only the
// float32 mode is instantiated (the caller has checked precise_row_sums).
template <int A_, int LANES, typename In, int L, bool kGrad, bool kFastOnly, bool kPlainVariants = false>
int64_t launch_mode(const StepArgs& a, hipStream_t st, int64_t tiles, bool allow_multi) {
  if constexpr (kGrad) {
    if (is_plain_vtrace(a))
      return launch_kernel<A_, LANES, In, L, true, true, kPlainCall>(a, st, tiles, allow_multi);
    if constexpr (kPlainVariants) {
      if (is_plain_vtrace_any_rewards(a))
        return launch_kernel<A_, LANES, In, L, true, true, kPlainRewards>(a, st, tiles, allow_multi);
      if (is_plain_vtrace_log_probs(a))
        return launch_kernel<A_, LANES, In, L, true, true, kPlainLogProbs>(a, st, tiles, allow_multi);
    }
    return launch_kernel<A_, LANES, In, L, true, true>(a, st, tiles, allow_multi);
  } else {
    if constexpr (!kFastOnly) {
      if (precise_row_sums(a, false))
        return launch_kernel<A_, LANES, In, L, false, true>(a, st, tiles, allow_multi);
    }
    return launch_kernel<A_, LANES, In, L, false, false>(a, st, tiles, allow_multi);
  }
}

// The kernel addresses L rows of each array (logits, gradients, [T,B] scalars)
// from a uniform base with 32-bit offsets.
inline bool rows_fit(const StepArgs& a, int L) { return a.B * a.A * 4 < (int64_t(1) << 32) / L; }

// kPlainVariants: loss calls that are plain V-trace but for a reward
// transform, bfloat16 gradients or behaviour log-probabilities take plain
// kernels too (instantiated for the long-run loss shapes only).
template <int A_, int LANES, typename In, int L = kL, bool kFastOnly = false, bool kPlainVariants = false>
hipError_t launch_shape(const StepArgs& a, Mode mode, hipStream_t st, int64_t* nwg, bool allow_multi) {
  if (kFastOnly && precise_row_sums(a, mode == Mode::LossGrad)) return hipErrorInvalidValue;
  if constexpr (kFastOnly) {
    if (mode == Mode::LossGrad) return hipErrorInvalidValue;  // never instantiated
  }
  if (a.B < LANES || !rows_fit(a, L)) return hipErrorInvalidValue;
  const int64_t tiles = (a.B + LANES - 1) / LANES;
  if constexpr (!kFastOnly) {
    if (mode == Mode::LossGrad) {
      *nwg = launch_mode<A_, LANES, In, L, true, false, kPlainVariants>(a, st, tiles, allow_multi);
      return hipGetLastError();
    }
  }
  *nwg = launch_mode<A_, LANES, In, L, false, kFastOnly>(a, st, tiles, allow_multi);
  return hipGetLastError();
}

// Tile shapes with longer contiguous runs per time row (LANES * A elements):
// at T = 1000 the same traffic streams 5-20% faster from 2304- to 9216-byte
// runs than from 1152-byte ones, provided the workgroups keep every CU busy.
template <int LANES_, int L_>
struct Shape {
  static constexpr int LANES = LANES_;
  static constexpr int L = L_;
};
constexpr int kMinWavesPerCu = 8;

// The batch fills the chip once: the tile count is a whole multiple of the CU
// count, every tile's workgroup is resident from the start, and each CU holds
// at least kMinWavesPerCu waves.
template <int A_, typename In, bool kGrad, typename Sh>
bool fills_once(int64_t B, int cus) {
  if (B % Sh::LANES != 0) return false;
  const int64_t tiles = B / Sh::LANES;
  if (tiles % cus != 0) return false;
  const int64_t per_cu = tiles / cus;
  return per_cu <= single_workgroups_per_cu<A_, Sh::LANES, In, Sh::L, kGrad>() &&
         per_cu * (Sh::LANES * Sh::L / kWave) >= kMinWavesPerCu;
}

// The multi-tile walk of this shape runs the batch as even generations.
template <int A_, typename In, bool kGrad, typename Sh>
bool walks_evenly(int64_t B, int cus) {
  if (B % Sh::LANES != 0) return false;
  const int64_t tiles = B / Sh::LANES;
  const int64_t resident = static_cast<int64_t>(multi_workgroups_per_cu<A_, Sh::LANES, In, Sh::L, kGrad>()) * cus;
  return resident >= 2 * static_cast<int64_t>(cus) && tiles >= 2 * resident && tiles % resident == 0;
}

// One workgroup per tile runs the batch as 2 to kMaxGenerations whole
// generations of resident workgroups, each CU holding at least kMinWavesPerCu
// waves.  (Measured up to four generations.)
constexpr int64_t kMaxGenerations = 4;
template <int A_, typename In, bool kGrad, typename Sh>
bool whole_generations(int64_t B, int cus) {
  if (B % Sh::LANES != 0) return false;
  const int64_t tiles = B / Sh::LANES;
  const int per_cu = single_workgroups_per_cu<A_, Sh::LANES, In, Sh::L, kGrad>();
  const int64_t resident = static_cast<int64_t>(per_cu) * cus;
  return per_cu * (Sh::LANES * Sh::L / kWave) >= kMinWavesPerCu && resident > 0 && tiles % resident == 0 &&
         tiles >= 2 * resident && tiles <= kMaxGenerations * resident;
}

enum class ShapeTest { FillsOnce, WalksEvenly, WholeGenerations };

template <int A_, typename In, bool kGrad, typename Sh>
bool shape_fits(ShapeTest test, int64_t B, int cus) {
  switch (test) {
    case ShapeTest::FillsOnce: return fills_once<A_, In, kGrad, Sh>(B, cus);
    case ShapeTest::WalksEvenly: return walks_evenly<A_, In, kGrad, Sh>(B, cus);
    case ShapeTest::WholeGenerations: return whole_generations<A_, In, kGrad, Sh>(B, cus);
  }
  return false;
}

template <int A_, typename In>
bool try_shapes(const StepArgs&, Mode, hipStream_t, int64_t*, bool, hipError_t*, int, ShapeTest) {
  return false;
}
template <int A_, typename In, typename Sh, typename... Rest>
bool try_shapes(const StepArgs& a, Mode mode, hipStream_t st, int64_t* nwg, bool allow_multi, hipError_t* err,
                int cus, ShapeTest test) {
  if (mode == Mode::LossGrad) return false;  // loss calls: launch_long_loss
  if (shape_fits<A_, In, false, Sh>(test, a.B, cus)) {
    *err = launch_shape<A_, Sh::LANES, In, Sh::L, true>(a, mode, st, nwg, allow_multi);
    return true;
  }
  return try_shapes<A_, In, Rest...>(a, mode, st, nwg, allow_multi, err, cus, test);
}

// Launches the first of Shapes (listed longest runs first) whose batch fills
// the chip once, else the first that the multi-tile walk runs as even
// generations (the choice does not depend on allow_multi, which only says
// whether the walk may run), else the first whose single-tile workgroups run
// it as a few whole generations; returns false (launching nothing) when none
// applies or the ratio needs the float64 mode (where the 16-step chunks of the
// default shapes measured as fast or faster).
template <int A_, typename In, typename... Shapes>
bool launch_long(const StepArgs& a, Mode mode, hipStream_t st, int64_t* nwg, bool allow_multi, hipError_t* err) {
  if (precise_row_sums(a, mode == Mode::LossGrad)) return false;
  const int cus = compute_units();
  if (cus <= 0 || !rows_fit(a, 8)) return false;
  return try_shapes<A_, In, Shapes...>(a, mode, st, nwg, allow_multi, err, cus, ShapeTest::FillsOnce) ||
         try_shapes<A_, In, Shapes...>(a, mode, st, nwg, allow_multi, err, cus, ShapeTest::WalksEvenly) ||
         try_shapes<A_, In, Shapes...>(a, mode, st, nwg, allow_multi, err, cus, ShapeTest::WholeGenerations);
}

// Workgroups of the single-tile loss kernel (plain or with variants) that fit
// on a compute unit at once, asked of the runtime once (0 if it cannot say).
template <int A_, int LANES, typename In, int L, int kPlain>
int loss_workgroups_per_cu() {
  static std::atomic<int> cached{-1};
  int n = cached.load(std::memory_order_relaxed);
  if (n < 0) {
    int blocks = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &blocks, reinterpret_cast<const void*>(tiled_kernel<A_, LANES, In, L, true, true, false, kPlain>),
            LANES * L, 0) != hipSuccess) {
      (void)hipGetLastError();
      blocks = 0;
    }
    n = blocks > 0 ? blocks : 0;
    cached.store(n, std::memory_order_relaxed);
  }
  return n;
}

// Loss calls on the long-run shapes: the first of Shapes whose workgroups run
// the batch as 1 to kMaxGenerations whole generations of resident workgroups,
// each CU holding at least kMinWavesPerCu waves; false (launching nothing)
// when none applies.  (The loss kernels fit two workgroups of 256 threads per
// CU, so the multi-tile walk, which needs more, does not serve them.)
template <int A_, typename In>
bool launch_long_loss(const StepArgs&, hipStream_t, int64_t*, hipError_t*, int) {
  return false;
}
template <int A_, typename In, typename Sh, typename... Rest>
bool launch_long_loss(const StepArgs& a, hipStream_t st, int64_t* nwg, hipError_t* err, int cus) {
  if (a.B % Sh::LANES == 0) {
    const int64_t tiles = a.B / Sh::LANES;
    const int fit = is_plain_vtrace(a) ? loss_workgroups_per_cu<A_, Sh::LANES, In, Sh::L, kPlainCall>()
                    : is_plain_vtrace_any_rewards(a)
                        ? loss_workgroups_per_cu<A_, Sh::LANES, In, Sh::L, kPlainRewards>()
                    : is_plain_vtrace_log_probs(a)
                        ? loss_workgroups_per_cu<A_, Sh::LANES, In, Sh::L, kPlainLogProbs>()
                        : loss_workgroups_per_cu<A_, Sh::LANES, In, Sh::L, kGeneralCall>();
    // Whole generations of the workgroups that are resident, or, of kernels that
    // three fit, of two a CU (A = 9: log-probabilities or bfloat16, whose batches of
    // 2^14 to 2^17 lanes took 16-lane tiles otherwise: T = 100, B = 16384, log-
    // probabilities 60 -> 40 us, bfloat16 61 -> 47; B = 131072, T = 20 174 -> 59).
    for (int per_cu = fit; per_cu > 0 && per_cu >= (fit < 2 ? fit : 2); --per_cu) {
      const int64_t resident = static_cast<int64_t>(per_cu) * cus;
      if (per_cu * (Sh::LANES * Sh::L / kWave) >= kMinWavesPerCu && tiles % resident == 0 &&
          tiles <= kMaxGenerations * resident) {
        *err = launch_shape<A_, Sh::LANES, In, Sh::L, false, true>(a, Mode::LossGrad, st, nwg, false);
        return true;
      }
    }
  }
  return launch_long_loss<A_, In, Rest...>(a, st, nwg, err, cus);
}
template <int A_, typename In, typename... Shapes>
bool launch_long_loss(const StepArgs& a, hipStream_t st, int64_t* nwg, hipError_t* err) {
  const int cus = compute_units();
  if (cus <= 0 || !rows_fit(a, 8)) return false;
  return launch_long_loss<A_, In, Shapes...>(a, st, nwg, err, cus);
}

// Batches whose 16 time rows 32-bit offsets do not reach: tiles of 16 lanes by 16
// steps again, in the general kernels alone.  (T = 16, 3914624 lanes, A = 18: loss
// 4.7 ms, 20.8 with one thread per lane; targets 2.2 against 18.7.)
template <int A_, typename In>
hipError_t launch_far(const StepArgs& a, Mode mode, hipStream_t st, int64_t* nwg) {
  constexpr int LANES = 16;
  if (a.B < LANES || a.B >= kTiledMaxLanes) return hipErrorInvalidValue;
  *nwg = (a.B + LANES - 1) / LANES;
  const dim3 grid(static_cast<unsigned>(*nwg)), block(LANES * kL);
  if (mode == Mode::LossGrad)
    hipLaunchKernelGGL((tiled_kernel<A_, LANES, In, kL, true, true, false, kGeneralCall, true>), grid, block, 0, st, a,
                       int64_t(1));
  else if (precise_row_sums(a, false))
    hipLaunchKernelGGL((tiled_kernel<A_, LANES, In, kL, false, true, false, kGeneralCall, true>), grid, block, 0, st, a,
                       int64_t(1));
  else
    hipLaunchKernelGGL((tiled_kernel<A_, LANES, In, kL, false, false, false, kGeneralCall, true>), grid, block, 0, st, a,
                       int64_t(1));
  return hipGetLastError();
}

// Launches tiles of `lanes` lanes, 256 / lanes steps per chunk (kFarLanes: those
// for rows far apart).
template <int A_, typename In>
hipError_t launch_lanes(int lanes, const StepArgs& a, Mode mode, hipStream_t st, int64_t* nwg, bool allow_multi) {
  switch (lanes) {
    case 16: return launch_shape<A_, 16, In, 16>(a, mode, st, nwg, allow_multi);
    case 8: return launch_shape<A_, 8, In, 32>(a, mode, st, nwg, false);
    case 4: return launch_shape<A_, 4, In, 64>(a, mode, st, nwg, false);
    case 2: return launch_shape<A_, 2, In, 128>(a, mode, st, nwg, false);
    case 1: return launch_shape<A_, 1, In, 256>(a, mode, st, nwg, false);
    case kFarLanes: return launch_far<A_, In>(a, mode, st, nwg);
    default: return hipErrorInvalidValue;
  }
}

// Launch for action count A, fp32 or bf16 logits.
template <int A_>
hipError_t launch_any(const StepArgs& a, LogitsType lt, int lanes, Mode mode, hipStream_t st, int64_t* nwg,
                      bool allow_multi) {
  if (lt == LogitsType::F32) return launch_lanes<A_, float>(lanes, a, mode, st, nwg, allow_multi);
  return launch_lanes<A_, uint16_t>(lanes, a, mode, st, nwg, allow_multi);
}

}  // namespace
}  // namespace vtrace

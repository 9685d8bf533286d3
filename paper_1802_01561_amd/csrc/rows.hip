// Row-split V-trace kernel for the action counts beyond the tiled kernel's
// (kTiledMaxActions < A <= kRowsMaxActions): a group of G threads shares one
// step's logit rows.
//
// With many actions a step's two rows are long enough to be read coalesced by
// themselves, and what a single thread cannot hold (2 A logits, A exponentials)
// fits a group's registers: thread i of a group holds K = ceil(A / G)
// neighbouring columns of each row from the loads to the gradient.  A workgroup
// of four waves walks one lane (batch entry) backwards in chunks of L steps,
// kRowsPerGroup rows per group:
//  1. each group forms its rows' maxima and float64 exponent sums (DPP
//     butterflies over the group) and leaves them in LDS;
//  2. after the chunk's one barrier every wave reads them with thread i of the
//     wave on step i, and forms the step's statistics, weights and the reverse
//     recursion (Remark 1) as one affine scan over the wave.  Each of the four
//     waves does this for all L steps, which costs less than a second barrier;
//  3. each group takes its rows' gradient coefficients from that step's thread
//     and writes the gradient from registers.
// The next chunk's rows are loaded before step 2.  LDS is double-buffered, so
// that a wave may start the next chunk while others still read this one's sums.
//
// What bounds it: vector instructions, and for small batches the chain of T / L
// chunks.  Counted at T = 100, B = 4096 (loss call, fp32): 40.5 M wave instructions
// at A = 48 and 35.3 M at A = 22, which keep the vector ALUs busy for more than half
// of 117 and 89 us; per 4 rows of 16 threads 308, of which a column of the two rows
// takes 39 and the rest, three fifths, belongs to the step (the reductions over the
// group, and statistics and scan once per wave, also of the last chunk's steps
// before t = 0).  HBM moves the inputs and outputs alone (78.7 MB written, 80.3
// algorithmic).  Measured (loss call, fp32 logits, against the generic kernel, whose
// single thread per lane reads and writes rows uncoalesced): T = 100, B = 512, A = 48
// 3156 -> 21 us; T = 100, B = 4096, A = 48 3208 -> 117 us (0.08 -> 2.1 TB/s) and A = 22
// 1395 -> 89 us; T = 20, B = 16384, A = 48 658 -> 164 us.  Three waves per SIMD spill nothing
// at K = 2 (116 -> 95 us at A = 22) but do from K = 3 on, where two are faster
// (T = 1000, B = 1024, A = 64: 268 against 350 us).
#include "device_common.hpp"
#include "row_stats.hpp"
#include "wave_ops.hpp"

namespace vtrace {
namespace {

constexpr int kRowsThreads = 256;
constexpr int kRowsPerGroup = 4;
// Workgroups of a launch; larger batches loop over lanes, so that the loss
// ticket, which takes about 10 ns a workgroup, is taken a bounded number of times
// (loss, B = 4096: T = 1, A = 21 59 -> 40 us, T = 100, A = 48 116 -> 108 with 2048
// in place of 4096; targets, which take none, 16 and 59 us with 4096, 16 and 62).
constexpr int64_t kRowsMaxWorkgroups = 4096, kRowsMaxLossWorkgroups = 2048;

// Butterfly moves over the G threads of a group: within a DPP row of 16 by
// quad permutes and mirrors (every thread ends with the same bits: each stage
// adds the same two values in either order), then across rows by xor.
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E, kRowHalfMirror = 0x141, kRowMirror = 0x140;

template <int kCtrl>
__device__ __forceinline__ float dpp_f32(float x) {
  return __uint_as_float(static_cast<unsigned>(
      __builtin_amdgcn_update_dpp(0, static_cast<int>(__float_as_uint(x)), kCtrl, 0xF, 0xF, true)));
}

template <int G, typename T, typename Op>
__device__ __forceinline__ T group_reduce(T x, Op op) {
  auto move = [&](auto C) {
    constexpr int ctrl = decltype(C)::value;
    if constexpr (sizeof(T) == 8)
      return dpp_f64<ctrl>(x);
    else
      return dpp_f32<ctrl>(x);
  };
  x = op(x, move(std::integral_constant<int, kQuadXor1>{}));
  x = op(x, move(std::integral_constant<int, kQuadXor2>{}));
  x = op(x, move(std::integral_constant<int, kRowHalfMirror>{}));
  x = op(x, move(std::integral_constant<int, kRowMirror>{}));
  if constexpr (G == 64) {
    x = op(x, __shfl_xor(x, 16));
    x = op(x, __shfl_xor(x, 32));
  }
  return x;
}

// x at thread kLane of the wave.
template <int kLane>
__device__ __forceinline__ double wave_read_f64(double x) {
  const unsigned long long u = __double_as_longlong(x);
  const unsigned lo = __builtin_amdgcn_readlane(static_cast<int>(u & 0xffffffffu), kLane);
  const unsigned hi = __builtin_amdgcn_readlane(static_cast<int>(u >> 32), kLane);
  return __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo));
}

// A step's row sums, as the groups leave them for the scan.
template <int L>
struct RowSums {
  double sz[L], ed[L], sy[L];
  float mz[L], my[L], za[L], ya[L];
};

// log2 e rounded to 29 bits (4.4e-10 below it, a sixth of the exponential
// polynomial's error): the float64 products of it and a float32 logit are exact, so
// that the fused multiply-add below forms a term's exponent from the exact
// difference z_j - m_z, whatever the size of m_z.
constexpr double kLog2eShort = 0x1.7154765p+0;

// kEps: the epsilon-correction, whose float64 logarithm and exponential of
// every step would cost the other calls' kernel registers.
template <int G, int K, typename In, bool kGrad, bool kEps>
__global__ __launch_bounds__(kRowsThreads, K == 2 ? 3 : 2) void rows_kernel(StepArgs a) {
  constexpr int kGroups = kRowsThreads / G;
  constexpr int R = kRowsPerGroup;
  constexpr int L = R * kGroups;  // steps per chunk: 64 (G = 16) or 16 (G = 64)
  constexpr int kDppRow = 16;
  static_assert(L == 64 || L == 16, "a chunk is one wave's or one DPP row's steps");
  __shared__ RowSums<L> sums[2];
  __shared__ double red_scratch[3 * (kRowsThreads / kWave)];

  const int tid = threadIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int wl = tid % kWave;
  const int s = wl % L;  // this thread's step in the scan (L = 16: the wave's DPP rows repeat it)
  const int gi = tid / G;
  const int i = tid % G;
  const int64_t T = a.T, B = a.B, A = a.A;
  // Columns [c0, c0 + K) of a row.  The last threads of a group start earlier
  // than i K so as to end with the row (A >= K): what they share with their
  // neighbours, columns below i K, joins no sum and is written twice with the
  // same value.
  const int own = i * K;
  const int c0 = own < static_cast<int>(A) - K ? own : static_cast<int>(A) - K;
  const int nchunks = static_cast<int>((T + L - 1) / L);
  const bool beh_lp = a.behaviour_log_probs != 0;
  const int correction = kEps ? kCorrEpsilon : a.correction;
  const bool no_ratio = kEps || correction == kCorrNone || correction == kCorrEpsilon;
  const bool use_y = !beh_lp && !no_ratio;
  const double rho_bar = a.rho_bar, c_bar = a.c_bar, lam = a.lambda;
  const float ce = a.entropy_cost;
  const uint32_t B32 = static_cast<uint32_t>(B), BA32 = static_cast<uint32_t>(B * A);
  // Byte offset of this thread's first column in row sr of a chunk.  (The empty
  // statement keeps the compiler from holding every row's 64-bit address in
  // registers for the whole walk.)
  auto row_offset = [&](int sr, size_t elem_bytes) __attribute__((always_inline)) {
    uint32_t off = (static_cast<uint32_t>(sr) * BA32 + static_cast<uint32_t>(c0)) * static_cast<uint32_t>(elem_bytes);
    asm volatile("" : "+v"(off));
    return off;
  };
  double tot_pg = 0.0, tot_base = 0.0, tot_ent = 0.0;  // wave 0's threads
  int parity = 0;

  for (int64_t b = xcd_tile(blockIdx.x, gridDim.x); b < B; b += gridDim.x) {
    const double boot = a.bootstrap_value[b];
    double cy_V = boot, cy_v = boot, cy_A = 0.0;
    double l_pg = 0.0, l_base = 0.0, l_ent = 0.0;
    bool bad_action = false;

    In pz[R][K], py[R][K];
    int32_t p_act;
    float p_r, p_g, p_V, p_lmu = 0.f;
    // Addresses are a wave-uniform base (the chunk's first row, which may lie
    // before t = 0) plus a 32-bit offset; the launcher checks that L rows fit.
    // Rows before t = 0 reread row 0; nothing of theirs is written or summed.
    auto prefetch = [&](int k) __attribute__((always_inline)) {
      const int64_t t0 = T - static_cast<int64_t>(k + 1) * L;
      const int neg = t0 < 0 ? static_cast<int>(-t0) : 0;
      const int64_t row0 = t0 * B + b;
      const gptr<const char> zg = offset_bytes(a.target_logits, row0 * A * int64_t(sizeof(In)));
      const gptr<const char> yg = offset_bytes(a.behaviour_logits, row0 * A * int64_t(sizeof(In)));
      static_for<R>([&](auto RI) __attribute__((always_inline)) {
        constexpr int r = decltype(RI)::value;
        const int sr = r * kGroups + gi;
        const uint32_t off = row_offset(sr < neg ? neg : sr, sizeof(In));
        const auto zp = reinterpret_cast<gptr<const In>>(zg + off), yp = reinterpret_cast<gptr<const In>>(yg + off);
        static_for<K>([&](auto J) { pz[r][decltype(J)::value] = zp[decltype(J)::value]; });
        if (use_y) static_for<K>([&](auto J) { py[r][decltype(J)::value] = yp[decltype(J)::value]; });
      });
      const uint32_t off = static_cast<uint32_t>(s < neg ? neg : s) * B32;
      p_act = offset_elems(a.actions, row0)[off];
      p_r = offset_elems(a.rewards, row0)[off];
      p_g = offset_elems(a.discounts, row0)[off];
      p_V = offset_elems(a.values, row0)[off];
      if (beh_lp && !no_ratio) p_lmu = offset_elems(static_cast<const float*>(a.behaviour_logits), row0)[off];
    };
    prefetch(0);
    for (int k = 0; k < nchunks; ++k, parity ^= 1) {
      const int64_t t0 = T - static_cast<int64_t>(k + 1) * L;
      const int64_t t = t0 + s;
      const bool step_ok = t >= 0;
      const int64_t row0 = t0 * B + b;
      RowSums<L>& q = sums[parity];
      const int32_t act = step_ok ? p_act : 0;  // rows that do not exist carry a harmless action
      const bool act_ok = act >= 0 && act < A;
      const int act_c = act_ok ? act : 0;
      bad_action = bad_action || !act_ok;
      const float r32 = transform_reward(p_r, a.reward_transform);
      const float g32 = p_g, V32 = p_V, lmu = p_lmu;

      // 1. This group's rows.
      float z[R][K], e[R][K], mzr[R];
      int col_a[R];  // the row's taken action, as a column of this thread (or none)
      static_for<R>([&](auto RI) __attribute__((always_inline)) {
        constexpr int r = decltype(RI)::value;
        if (t0 + (r + 1) * kGroups <= 0) return;  // all of these rows lie before t = 0
        const int sr = r * kGroups + gi;
        col_a[r] = __shfl(act_c, sr) - c0;
        float y[K];
        float mz = logit_to_float(pz[r][0]);
        static_for<K>([&](auto J) {
          constexpr int j = decltype(J)::value;
          z[r][j] = logit_to_float(pz[r][j]);
          mz = __builtin_elementwise_maximum(mz, z[r][j]);
        });
        auto maximum = [](float x, float w) { return __builtin_elementwise_maximum(x, w); };
        auto add = [](double x, double w) { return x + w; };
        mz = group_reduce<G>(mz, maximum);
        mzr[r] = mz;
        const double mzl = static_cast<double>(mz) * kLog2eShort;
        double sz = 0.0, ed = 0.0;
        static_for<K>([&](auto J) {
          constexpr int j = decltype(J)::value;
          const double x = fma(static_cast<double>(z[r][j]), kLog2eShort, -mzl);
          const double ej = exp2_f64_term(x);
          e[r][j] = static_cast<float>(ej);
          const bool mine = c0 + j >= own;
          sz += mine ? ej : 0.0;
          ed += mine ? ej * x : 0.0;
          // Pins the running sums here: the compiler would otherwise keep the
          // terms of several rows live at once.
          asm volatile("" : "+v"(sz), "+v"(ed), "+v"(e[r][j]));
        });
        sz = group_reduce<G>(sz, add);
        ed = group_reduce<G>(ed, add);
        const bool has_a = col_a[r] >= 0 && col_a[r] < K;
        // (The bits or'ed together: a chain of selects becomes an indexed array.)
        unsigned za = 0;
        static_for<K>([&](auto J) {
          constexpr int j = decltype(J)::value;
          za |= col_a[r] == j ? __float_as_uint(z[r][j]) : 0u;
        });
        if (has_a) q.za[sr] = __uint_as_float(za);
        if (use_y) {
          static_for<K>([&](auto J) { y[decltype(J)::value] = logit_to_float(py[r][decltype(J)::value]); });
          float my = y[0];
          static_for<K>([&](auto J) { my = __builtin_elementwise_maximum(my, y[decltype(J)::value]); });
          my = group_reduce<G>(my, maximum);
          const double myl = static_cast<double>(my) * kLog2eShort;
          double sy = 0.0;
          unsigned ya = 0;
          static_for<K>([&](auto J) {
            constexpr int j = decltype(J)::value;
            const double ej = exp2_f64_term(fma(static_cast<double>(y[j]), kLog2eShort, -myl));
            sy += c0 + j >= own ? ej : 0.0;
            ya |= col_a[r] == j ? __float_as_uint(y[j]) : 0u;
            asm volatile("" : "+v"(sy));
          });
          sy = group_reduce<G>(sy, add);
          if (has_a) q.ya[sr] = __uint_as_float(ya);
          if (i == 0) {
            q.my[sr] = my;
            q.sy[sr] = sy;
          }
        }
        if (i == 0) {
          q.mz[sr] = mz;
          q.sz[sr] = sz;
          q.ed[sr] = ed;
        }
        __builtin_amdgcn_sched_barrier(0);  // one row at a time
      });
      if (k + 1 < nchunks) prefetch(k + 1);
      __syncthreads();

      // 2. Thread s of every wave: step t0 + s.
      const float mz = q.mz[s], za = q.za[s];
      RowStats st;
      const double dza = static_cast<double>(za) - static_cast<double>(mz);  // exact
      const double ea = exp2_f64_term(dza * kLog2eShort);
      finish_target_stats(st, mz, dza, q.sz[s], q.ed[s], ea);
      if (no_ratio) {
        st.ratio = 1.0;
      } else if (beh_lp) {
        st.ratio = exp2_f64((st.log_pa - static_cast<double>(lmu)) * kLog2eF64);
      } else {
        const float my = q.my[s];
        const double sy = __builtin_isfinite(my) ? q.sy[s] : NAN;
        const double dya = static_cast<double>(q.ya[s]) - static_cast<double>(my);
        st.ratio = exp2_f64((st.dza - dya) * kLog2eF64) * (sy * st.inv);
      }
      if (!act_ok) st.ratio = NAN;
      const StepWeights w = variant_weights(correction, clip_above(st.ratio, rho_bar),
                                            lam * clip_above(st.ratio, c_bar), lam, act_ok);
      const double r = r32, g = g32, V = V32;
      // A value at the next step: the DPP row's neighbour, and for a row's last
      // thread the next row's first (or the later chunk's carry).
      auto next_step = [&](double x, double carry) {
        double n = dpp_f64<kRowShl1>(x);
        if constexpr (L == 64) {
          const double x16 = wave_read_f64<16>(x), x32 = wave_read_f64<32>(x), x48 = wave_read_f64<48>(x);
          n = s == 15 ? x16 : n;
          n = s == 31 ? x32 : n;
          n = s == 47 ? x48 : n;
        }
        if (s == L - 1) n = carry;
        return n;
      };
      const double V_next = next_step(V, cy_V);
      double Gs = g * w.c_v, D = w.rho_v * (r + g * V_next - V);
      if (s == L - 1) D = fma(Gs, cy_A, D);
      static_for<4>([&](auto I) {
        constexpr int off = 1 << decltype(I)::value;
        const double Gn = dpp_f64<0x100 + off>(Gs);
        const double Dn = dpp_f64<0x100 + off>(D);
        if (s % kDppRow + off < kDppRow) {
          D = fma(Gs, Dn, D);
          Gs = Gs * Gn;
        }
      });
      if constexpr (L == 64) {  // the DPP rows, last to first
        const double D48 = wave_read_f64<48>(D);
        const double D32 = fma(wave_read_f64<32>(Gs), D48, wave_read_f64<32>(D));
        const double D16 = fma(wave_read_f64<16>(Gs), D32, wave_read_f64<16>(D));
        const int row = s / kDppRow;
        const double Dr = row == 2 ? D48 : row == 1 ? D32 : D16;
        if (row < 3) D = fma(Gs, Dr, D);
      }
      const double A_t = D;  // v_t - V(x_t)
      const double v_t = V + A_t;
      const double v_next = next_step(v_t, cy_v);
      const double q_next = a.q_estimate == kQBaseline ? V_next : v_next;
      const double adv = w.rho_pg * (r + g * q_next - V);
      cy_A = wave_read_f64<0>(A_t);
      cy_v = wave_read_f64<0>(v_t);
      cy_V = wave_read_f64<0>(V);

      if (wv == 0 && wl < L && step_ok) {
        const uint32_t off = static_cast<uint32_t>(s) * B32;
        if (a.vs) offset_elems(a.vs, row0)[off] = static_cast<float>(v_t);
        if (a.pg_adv) offset_elems(a.pg_adv, row0)[off] = static_cast<float>(adv);
        if constexpr (kGrad) {
          offset_elems(a.d_values, row0)[off] = static_cast<float>(a.baseline_cost * (V - v_t));
          const double log_pa = !act_ok ? NAN : kEps ? log_prob_plus_eps<true>(st, a.epsilon) : st.log_pa;
          l_pg += -adv * log_pa;
          l_base += 0.5 * A_t * A_t;
          l_ent += -static_cast<double>(st.H);
        }
      }

      // 3. d_logits_j = e_j (alpha + beta (z_j - m_z)) off the taken action; the
      // coefficients come from the row's thread of the scan.  (z_j - m_z and not
      // z_j: a large common offset of a row's logits would show in the float32
      // beta z_j.  Masked logits are held to a size that no entropy cost below 1e8
      // takes out of float32's range; their e_j are 0.)
      // There is one such thread per row, so it forms them in float64 and rounds
      // each once: error of d_logits against float64 at A = 48 2.7e-8, 4.8e-8 with
      // float32 coefficients, in the same time (21 us at T = 100, B = 512).
      if constexpr (kGrad) {
        const float ls_H = st.log_s - st.H;
        const double pa = ea * st.inv, ce64 = ce;
        double adv_w = adv;
        if constexpr (kEps) adv_w = adv * (pa / (pa + static_cast<double>(a.epsilon)));
        const float beta = static_cast<float>(st.inv * ce64);
        const float alpha = static_cast<float>(st.inv * (adv_w - ce64 * ls_H));
        const double taken = ce64 * pa * (dza - ls_H) - adv_w * ((st.sum - ea) * st.inv);
        const float out_a = act_ok ? static_cast<float>(taken) : NAN;
        static_for<R>([&](auto RI) __attribute__((always_inline)) {
          constexpr int r2 = decltype(RI)::value;
          const int sr = r2 * kGroups + gi;
          const float al = __shfl(alpha, sr), be = __shfl(beta, sr), oa = __shfl(out_a, sr);
          if (t0 + sr >= 0) {
            float x[K];
            static_for<K>([&](auto J) {
              constexpr int j = decltype(J)::value;
              x[j] = e[r2][j] * fmaf(be, fmaxf(z[r2][j] - mzr[r2], -1e30f), al);
              if (col_a[r2] == j) x[j] = oa;
            });
            if (a.grad_bf16) {
              const auto o = reinterpret_cast<gptr<uint16_t>>(offset_bytes(a.d_logits, row0 * A * 2) + row_offset(sr, 2));
              static_for<K>([&](auto J) { o[decltype(J)::value] = to_bf16(x[decltype(J)::value]); });
            } else {
              const auto o = reinterpret_cast<gptr<float>>(offset_bytes(a.d_logits, row0 * A * 4) + row_offset(sr, 4));
              static_for<K>([&](auto J) { o[decltype(J)::value] = x[decltype(J)::value]; });
            }
          }
        });
      }
    }
    if (bad_action) raise_error_flag(a.error_flag);
    if constexpr (kGrad) {
      if (wv == 0) {
        l_pg = wave_sum(l_pg);
        l_base = wave_sum(l_base) * a.baseline_cost;
        l_ent = wave_sum(l_ent) * a.entropy_cost;
        if (tid == 0) {
          if (a.lane_losses) {
            a.lane_losses[3 * b + 0] = static_cast<float>(l_pg);
            a.lane_losses[3 * b + 1] = static_cast<float>(l_base);
            a.lane_losses[3 * b + 2] = static_cast<float>(l_ent);
          }
          tot_pg += l_pg;
          tot_base += l_base;
          tot_ent += l_ent;
        }
      }
    }
  }
  if constexpr (kGrad) finish_losses<kRowsThreads>(a, tot_pg, tot_base, tot_ent, red_scratch);
}

template <int G, int K, typename In>
hipError_t launch_rows_shape(const StepArgs& a, Mode mode, hipStream_t st, int64_t* nwg) {
  const int64_t most = mode == Mode::LossGrad ? kRowsMaxLossWorkgroups : kRowsMaxWorkgroups;
  *nwg = a.B < most ? a.B : most;
  const dim3 grid(static_cast<unsigned>(*nwg)), block(kRowsThreads);
  if (mode != Mode::LossGrad)
    hipLaunchKernelGGL((rows_kernel<G, K, In, false, false>), grid, block, 0, st, a);
  else if (a.correction == kCorrEpsilon)
    hipLaunchKernelGGL((rows_kernel<G, K, In, true, true>), grid, block, 0, st, a);
  else
    hipLaunchKernelGGL((rows_kernel<G, K, In, true, false>), grid, block, 0, st, a);
  return hipGetLastError();
}

template <typename In>
hipError_t launch_rows_typed(const StepArgs& a, Mode mode, hipStream_t st, int64_t* nwg) {
  if (a.A <= 32) return launch_rows_shape<16, 2, In>(a, mode, st, nwg);
  if (a.A <= 48) return launch_rows_shape<16, 3, In>(a, mode, st, nwg);
  if (a.A <= 64) return launch_rows_shape<16, 4, In>(a, mode, st, nwg);
  if (a.A <= 128) return launch_rows_shape<64, 2, In>(a, mode, st, nwg);
  if (a.A <= 192) return launch_rows_shape<64, 3, In>(a, mode, st, nwg);
  return launch_rows_shape<64, 4, In>(a, mode, st, nwg);
}

// A workgroup of this kernel takes a lane's chunk whole however short the unroll
// is; one thread per lane takes its A T logits one after another, and from a few
// thousand lanes on fills the chip with them.  That is faster up to the A T below
// (us, row-split / one thread per lane; loss: B = 512, T = 1, A = 21 14 / 16;
// B = 1024, A = 21, T = 1 20 / 16 and T = 2 20 / 28; B = 4096, A = 21, T = 2 40 / 28
// and T = 4 40 / 53, A = 48, T = 1 46 / 35; B = 16384, T = 8, A = 21 104 / 109, T = 2,
// A = 48 127 / 68 and T = 4 128 / 132; B = 60000, T = 1, A = 21 334 / 36, T = 20 450 /
// 432 and A = 48, T = 8 438 / 549, with bfloat16 411 / 312 and 499 / 409.  Targets: B = 1024, T = 1, A = 21 6 / 8; B = 2048
// 10 / 8; B = 4096, T = 2 17 / 15, A = 48, T = 1 19 / 18; B = 16384, A = 21, T = 4 53 /
// 27 and T = 8 54 / 57; B = 60000, A = 48, T = 4 209 / 193 and A = 21, T = 8 192 / 109).
bool one_thread_per_lane(const StepArgs& a, LogitsType lt, Mode mode) {
  if (a.T > 1000) return false;
  const int64_t n = a.A * a.T;
  if (mode != Mode::LossGrad) return a.B >= 2048 && n <= 220 && n * 90 < a.B;
  return a.B >= 1024 && (10 * n * n < (a.B < 8192 ? 11 : 22) * a.B || (lt == LogitsType::BF16 && n * 110 < a.B));
}

}  // namespace

// 64 rows of an array (the longest chunk) must fit the kernel's 32-bit byte
// offsets: 64 B A 4 < 2^32.
bool rows_supported(const StepArgs& a, LogitsType lt, Mode mode) {
  return a.A > kTiledMaxActions && a.A <= kRowsMaxActions && a.B * a.A < (int64_t(1) << 24) &&
         !one_thread_per_lane(a, lt, mode);
}

hipError_t launch_rows(const StepArgs& a, LogitsType lt, Mode mode, hipStream_t st, int64_t* num_workgroups) {
  if (!rows_supported(a, lt, mode)) return hipErrorNotSupported;
  if (lt == LogitsType::F32) return launch_rows_typed<float>(a, mode, st, num_workgroups);
  return launch_rows_typed<uint16_t>(a, mode, st, num_workgroups);
}

}  // namespace vtrace

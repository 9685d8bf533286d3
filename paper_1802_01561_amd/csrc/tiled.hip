// Tiled V-trace kernel: the instantiations for A = 9 and A = 18 and the
// choice of instantiation for every action count (the kernel itself is in
// tiled_impl.hpp).
#include "tiled_impl.hpp"

namespace vtrace {

// Time rows that 32-bit offsets do not reach 16 of: one thread per lane has millions
// of lanes to fill the chip with, and needs no ticket per 16 lanes; tiles win once
// a lane's logits are many (ms, tiles / one thread per lane; rows of 1.05 * 2^26
// elements, loss: A = 18, T = 4 3.9 / 5.4, with bfloat16 logits 3.8 / 3.4, T = 16 4.7 /
// 20.8; A = 9, T = 4 6.4 / 3.5, T = 16 7.7 / 11.8; A = 6, T = 16 10.2 / 11.8; A = 2,
// T = 20 29.6 / 23.8.  Targets: A = 18, T = 4 1.1 / 3.5; A = 6, T = 4 1.45 / 1.47, with
// bfloat16 1.33 / 1.21; A = 9, T = 4 1.13 / 1.13 with bfloat16; A = 2, T = 20 12.9 /
// 10.1).
bool far_tiles_faster(const StepArgs& a, LogitsType lt, Mode mode) {
  const bool f32 = lt == LogitsType::F32;
  if (a.T >= 128) return mode == Mode::LossGrad || a.A >= 4;
  if (mode == Mode::LossGrad) return a.A * a.T >= (f32 ? 72 : 90);
  return a.A >= 4 && a.A * a.T >= (f32 ? 24 : 36);
}

bool tiled_supported(const StepArgs& a, LogitsType lt, Mode mode) {
  return a.A >= 2 && a.A <= kTiledMaxActions &&
         (rows_fit(a, kL) || (a.B < kTiledMaxLanes && far_tiles_faster(a, lt, mode)));
}

// Tiles of 256 threads: `lanes` lanes, 256 / lanes steps per chunk.
constexpr int kTileThreads = 256;

// Steps per chunk of the time-parallel shape: the power of two >= T, 16 to 256.
int one_chunk_steps(int64_t T) {
  int L = 16;
  while (L < T && L < kMaxChunkSteps) L *= 2;
  return L;
}

// Lanes per workgroup, 16 to 1, of the shapes that spread a small batch over
// the chip: fewer lanes and longer chunks make more workgroups and fewer chunks
// one after another, at shorter runs per time row.  The largest tile that gives
// 7/8 of the CUs a workgroup; chunks no longer than the unroll needs.
// Measured (loss call, fp32, calls in a HIP graph, us; 16 / 8 / 4 / 2 / 1 lanes):
//   T = 1000, A = 18: B = 64 197 / 103 / 56 / 35 / 25, B = 512 204 / 110 / 65 /
//   47 / 51, B = 2048 210 / 125 / 127 / 156 / 180;
//   T = 100, A = 6: B = 100 16.5 / 12.1 / 8.9 / 7.6 / 8.3, B = 1021 17.4 / 13.7 /
//   12.5 / 14.6 / 21.8, B = 2048 18.0 / 16.2 / 17.0 / 23.0 / 35.1;
//   T = 20, A = 18: B = 512 11.6 / 9.0 / 9.7 / 11.5 / 15.1.
int tile_lanes(const StepArgs& a, LogitsType lt, Mode mode, int cus, bool one_chunk) {
  const bool loss = mode == Mode::LossGrad, bf16 = lt == LogitsType::BF16;
  int min_lanes = kTileThreads / one_chunk_steps(a.T);
  if (!one_chunk && a.T <= kMaxChunkSteps && min_lanes < 16) min_lanes *= 2;
  auto tiles = [&](int lanes) { return (a.B + lanes - 1) / lanes; };
  int lanes = 16;
  while (lanes > 1 && (lanes > a.B || (lanes > min_lanes && tiles(lanes) * 8 < 7 * static_cast<int64_t>(cus))))
    lanes /= 2;
  // With short rows two chunks of the next larger tile cost no more than one of
  // this on half the CUs (B = 1024, T = 50: A = 6 10.0 against 10.0, A = 9 11.0
  // against 10.4 us; A = 18 13.2 against 12.1; T = 20, 8 to 16 lanes: B = 3000,
  // A = 4 10.5 against 9.9, B = 2048, A = 9 9.8 against 10.5), in loss calls: targets,
  // which take no ticket per workgroup, lose (T = 50, B = 1021, A = 9 4.0 -> 5.0,
  // T = 20, B = 2048, A = 6 3.3 -> 4.6).
  const int next_steps = kTileThreads / (2 * lanes);
  if (loss && lanes < 16 && a.A < (lanes == 8 ? 7 : 16) && a.T <= 2 * next_steps && a.T > next_steps &&
      tiles(2 * lanes) * 2 >= cus)
    lanes *= 2;
  if (lanes < 16 || a.T <= 16 || min_lanes > 8) return lanes;
  // Steps walked, the last chunk's empty ones among them, by 32-step chunks over
  // those by 16-step ones.
  const double waste = static_cast<double>((a.T + 31) / 32 * 32) / static_cast<double>((a.T + 15) / 16 * 16);
  const int64_t n = a.T * a.A;
  if (loss) {
    // One 16-lane workgroup per CU against two of 8 lanes: the second wave per
    // SIMD pays once the walk is long enough for the work of a row, and the later
    // the more of its steps are empty (8 lanes over 16, B = 4096, fp32 / log-
    // probabilities / bf16: T = 125, A = 4 0.94 / 0.92 / 0.89; T = 50, A = 9 1.01 /
    // 1.03 / 0.94 and A = 12 0.94 / 0.98 / 0.91; T = 90, A = 6 0.97 / 0.99 / 0.92;
    // T = 100 (waste 1.14), A = 7 1.01 / 1.03 / 0.96, A = 8 0.96 / 0.97 / 0.90, A = 9
    // 0.98 / 1.01 / 0.93; T = 80 (1.2), A = 9 1.02 / 1.06 / 0.97; T = 48 (1.33), A = 18
    // 1.04 / 1.07 / 1.06; T = 300, A = 6 0.85, A = 18 0.91).
    if (tiles(16) <= cus)
      return static_cast<double>(n) >= (bf16 ? 400.0 : 500.0) * waste * waste * waste * waste ? 8 : 16;
    // A second generation of 16-lane workgroups that would leave half the chip
    // idle runs faster as a third of 8 lanes, in long unrolls of rows too long for
    // three 16-lane workgroups a CU (8 over 16, fp32 / log-probabilities / bf16:
    // T = 500 and 1000, B = 8200 A = 10 to 18 0.88 to 0.93 / 0.88 to 0.96 / 0.86 to 0.93,
    // B = 10000 0.93 to 1.02 / 0.84 to 1.02 / 0.88 to 0.94, B = 12200 0.92 to 1.0 / 0.93
    // to 1.07 / 1.01 to 1.08; T = 300, A = 18, B = 10000 1.01 / 1.1 / 0.97; A = 9 1.05 to
    // 1.2 / 1.0 / 0.91).
    if (tiles(16) > 2 * cus && tiles(16) * 2 <= (bf16 ? 5 : 6) * cus && n >= 6000 && a.A >= (bf16 ? 9 : 10)) return 8;
    return 16;
  }
  // Targets (8 lanes over 16, fp32 / bf16): B = 4096, A = 2 to 6 (bf16: 9), T = 20 to
  // 1000 0.74 to 0.97 / 0.73 to 0.97; A = 15 T = 50 0.92 / 0.90, T = 100 1.03 / 1.01,
  // T = 1000 1.2 / 1.08; B = 32768, A = 2 to 6, T = 50 and 100 0.80 to 0.89 / 0.86 to
  // 0.92, T = 300 1.02 to 1.12; B = 16384, T = 50 1.05 / 1.02.
  const bool short_rows = a.A * (bf16 ? 2 : 4) <= 24;
  if (tiles(16) <= cus) return (short_rows || a.T < 100) && waste <= 1.2 ? 8 : 16;
  return short_rows && a.T <= 128 && waste <= 1.2 && tiles(16) >= 6 * cus ? 8 : 16;
}

// 32 lanes in place of 16 for the 16-step tiles, where both fit.  bf16 A = 18
// (1152-byte rows): once the tiles fill every CU twice (T = 1000: 16384 lanes 593 ->
// 558 us and 32768 lanes 1.23 -> 1.10 ms with 32, 8192 lanes 275 against 297 us),
// and when the whole short batch is one such tile (one workgroup, whose loss sums
// need no cross-workgroup reduction).  fp32 A = 9 (1152-byte rows), where the last
// generation of 32-lane workgroups fills 7/8 of the CUs: loss calls of one chunk, in
// one or two generations (half the tickets; 32 over 16 at T = 1 to 16: B = 7000 0.90
// to 0.95, 8192 0.87 to 0.89, 9000 1.16 to 1.25, 16100 0.90 to 0.95, 20000 1.05 to
// 1.17; T = 20 1.03, 0.97, 1.43, 1.10, 1.34), and targets of long unrolls from two
// on (T = 400: B = 8192 1.05, 15000 to 16380 0.94, 20000 1.31).  bf16 A = 9
// measured slower with 32 lanes at every size.
bool wide_tiles(const StepArgs& a, LogitsType lt, Mode mode, int cus, bool short_batch) {
  if (a.A == 18 && lt == LogitsType::BF16) return a.B >= 64 * static_cast<int64_t>(cus) || (short_batch && a.B == 32);
  if (a.A != 9 || lt != LogitsType::F32) return false;
  const int64_t tiles = (a.B + 31) / 32, generations = (tiles + cus - 1) / cus;
  if ((tiles - (generations - 1) * cus) * 8 < 7 * static_cast<int64_t>(cus)) return false;
  return mode == Mode::LossGrad ? a.T <= 16 && generations <= 2 : a.T >= 100 && generations >= 2;
}

hipError_t launch_tiled(const StepArgs& a, LogitsType lt, Mode mode, hipStream_t st,
                        int64_t* num_workgroups, const TileRule& rule) {
  const int cus = compute_units();
  if (cus <= 0) return hipErrorInvalidDevice;
  int lanes = 16;
  if (rule.time_parallel) {
    lanes = kTileThreads / one_chunk_steps(a.T);
  } else {
    // Batches of A = 9 or 18 that fill the chip in whole generations take the
    // long-run shapes of tiled_long_f32.hip and tiled_long_bf16.hip (32 to 128
    // lanes, chunks of 8 or 4 steps).
    if (rule.shapes && (a.A == 9 || a.A == 18)) {
      hipError_t err = hipSuccess;
      const bool launched = lt == LogitsType::F32
                                ? launch_tiled_long_f32(a, mode, st, num_workgroups, rule.multi, &err)
                                : launch_tiled_long_bf16(a, mode, st, num_workgroups, rule.multi, &err);
      if (launched) return err;
    }
    if (rule.shapes) lanes = tile_lanes(a, lt, mode, cus, rule.one_chunk);
    if (lanes == 16 && rows_fit(a, kL) && wide_tiles(a, lt, mode, cus, a.T <= 16 || !rule.shapes)) {
      if (a.A == 9) return launch_shape<9, 32, float>(a, mode, st, num_workgroups, rule.multi);
      return launch_shape<18, 32, uint16_t>(a, mode, st, num_workgroups, rule.multi);
    }
  }
  // (Such rows are of 2^26 elements or more: more than 16 lanes.)
  if (!rows_fit(a, kL)) lanes = kFarLanes;
  while (lanes != kFarLanes && (lanes > a.B || !rows_fit(a, kTileThreads / lanes)))
    lanes = lanes > a.B ? lanes / 2 : lanes * 2;
  if (a.A == 18) return launch_any<18>(a, lt, lanes, mode, st, num_workgroups, rule.multi);
  if (a.A == 9) return launch_any<9>(a, lt, lanes, mode, st, num_workgroups, rule.multi);
  // The other action counts are instantiated in three more files, which
  // compile in parallel.
  if (a.A >= 2 && a.A <= 8) return launch_tiled_a2_8(a, lt, lanes, mode, st, num_workgroups, rule.multi);
  if (a.A >= 10 && a.A <= 14) return launch_tiled_a10_14(a, lt, lanes, mode, st, num_workgroups, rule.multi);
  if (a.A >= 15 && a.A <= kTiledMaxActions)
    return launch_tiled_a15_20(a, lt, lanes, mode, st, num_workgroups, rule.multi);
  return hipErrorNotSupported;
}

}  // namespace vtrace

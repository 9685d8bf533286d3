// Fused output layer + V-trace: the launch, the workspace and the kernel that
// adds the workgroups' partial sums (the walk itself is in head_impl.hpp).
#include "device_common.hpp"
#include "head.hpp"

namespace vtrace {
namespace {

int head_columns(int64_t A) { return A + 1 > 16 ? 32 : 16; }

// Adds the workgroups' partial sums in a fixed order (float64): d_W, d_bias and
// the loss totals.  Block i covers 32 outputs; each of its 32 half-waves sums the
// workgroups k = half-wave, half-wave + 32, ... (one 128-byte line per step), and
// the 32 sums are added in order.
constexpr int kFinishOutputs = 32;
constexpr int kFinishWaves = 16;
constexpr int kFinishParts = kFinishWaves * kWave / kFinishOutputs;
__global__ __launch_bounds__(kFinishWaves* kWave) void head_finish_kernel(HeadArgs a, int C, int nwg) {
  __shared__ double s_q[kFinishParts][kFinishOutputs];
  const int64_t H = a.H;
  const int A1 = static_cast<int>(a.A) + 1;
  const int64_t n_w = H * A1;
  const int64_t n_out = n_w + A1;
  const int part = threadIdx.x / kFinishOutputs, lane = threadIdx.x % kFinishOutputs;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * kFinishOutputs + lane;
  const size_t stride = static_cast<size_t>(H + 1) * C;
  size_t off = 0;
  if (i < n_w)
    off = static_cast<size_t>(i / A1) * C + static_cast<size_t>(i % A1);
  else if (i < n_out)
    off = static_cast<size_t>(H) * C + static_cast<size_t>(i - n_w);
  double sum = 0.0;
  if (i < n_out) {
    // Unrolled so that several rows' loads are in flight; the additions keep
    // their order.
#pragma unroll 8
    for (int k = part; k < nwg; k += kFinishParts) sum += static_cast<double>(a.grad_partials[k * stride + off]);
  }
  s_q[part][lane] = sum;
  __syncthreads();
  if (part == 0 && i < n_out) {
    double tot = 0.0;
    for (int q = 0; q < kFinishParts; ++q) tot += s_q[q][lane];
    if (i < n_w)
      a.d_weight[i] = static_cast<float>(tot);
    else
      a.d_bias[i - n_w] = static_cast<float>(tot);
  }
  if (blockIdx.x == 0) {
    // Loss totals: each thread adds the workgroups k = thread, thread + 1024,
    // ..., then a fixed-order block reduction.
    __shared__ double s_red[3 * kFinishWaves];
    double p0 = 0.0, p1 = 0.0, p2 = 0.0;
    for (int k = threadIdx.x; k < nwg; k += kFinishWaves * kWave) {
      p0 += a.loss_partials[3 * k + 0];
      p1 += a.loss_partials[3 * k + 1];
      p2 += a.loss_partials[3 * k + 2];
    }
    block_sum3<kFinishWaves * kWave>(p0, p1, p2, s_red);
    if (threadIdx.x == 0) {
      a.losses[0] = static_cast<float>(p0 + p1 + p2);
      a.losses[1] = static_cast<float>(p0);
      a.losses[2] = static_cast<float>(p1);
      a.losses[3] = static_cast<float>(p2);
    }
  }
}

}  // namespace

bool head_hidden_supported(int64_t H) { return H == 64 || H == 128 || H == 256; }

namespace {

// Workgroups of a launch over groups of four lanes, or (split) over lanes.
int64_t head_workgroups(int64_t B, bool split) {
  const int64_t groups = split ? B : (B + kHeadLanes - 1) / kHeadLanes;
  return groups < kHeadMaxWorkgroups ? groups : kHeadMaxWorkgroups;
}

size_t head_loss_bytes(int64_t nwg) {
  const size_t n = 3 * sizeof(double) * static_cast<size_t>(nwg);
  return (n + 255) / 256 * 256;
}

size_t head_bytes(int64_t nwg, int64_t A, int64_t H) {
  return kWsHeaderBytes + head_loss_bytes(nwg) +
         sizeof(float) * static_cast<size_t>(nwg) * static_cast<size_t>(H + 1) * static_cast<size_t>(head_columns(A));
}

// Four consecutive chunks of one lane per workgroup (a workgroup per lane)
// against one chunk of four lanes: while the lanes fit the resident workgroups
// and there is more than one chunk to share.  Measured (H = 256, A = 18, calls in
// a HIP graph, us, four lanes -> one lane): T = 100, B = 32 53 -> 26, B = 200 60 ->
// 33, B = 512 62 -> 45, B = 1024 73 against 74, B = 2048 114 against 130; T = 500,
// B = 200 226 -> 86; T = 20, B = 32 23 -> 18, B = 200 25 -> 24 (H = 128, A = 9,
// B = 512 16 against 19).
bool prefer_split(int64_t T, int64_t B) { return T > 16 && B <= (T > 32 ? 512 : 256); }

}  // namespace

size_t head_workspace_bytes(int64_t B, int64_t A, int64_t H) { return head_bytes(head_workgroups(B, true), A, H); }
size_t head_workspace_least_bytes(int64_t B, int64_t A, int64_t H) {
  return head_bytes(head_workgroups(B, false), A, H);
}

void head_attach_workspace(HeadArgs* a, void* ws, size_t bytes) {
  a->split = prefer_split(a->T, a->B) && bytes >= head_workspace_bytes(a->B, a->A, a->H);
  char* base = static_cast<char*>(ws);
  a->error_flag = reinterpret_cast<unsigned int*>(base + kWsFlagOffset);
  a->loss_partials = reinterpret_cast<double*>(base + kWsHeaderBytes);
  a->grad_partials =
      reinterpret_cast<float*>(base + kWsHeaderBytes + head_loss_bytes(head_workgroups(a->B, a->split)));
}

hipError_t launch_head(const HeadArgs& a, hipStream_t st) {
  const int64_t nwg = head_workgroups(a.B, a.split);
  const unsigned n = static_cast<unsigned>(nwg);
  if (a.H == 64) launch_head_h64(a, st, n);
  else if (a.H == 128) launch_head_h128(a, st, n);
  else if (a.H == 256) launch_head_h256(a, st, n);
  else return hipErrorInvalidValue;
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t n_out = a.H * (a.A + 1) + (a.A + 1);
  const unsigned fb = static_cast<unsigned>((n_out + kFinishOutputs - 1) / kFinishOutputs);
  hipLaunchKernelGGL(head_finish_kernel, dim3(fb), dim3(kFinishWaves * kWave), 0, st, a, head_columns(a.A),
                     static_cast<int>(nwg));
  return hipGetLastError();
}

}  // namespace vtrace

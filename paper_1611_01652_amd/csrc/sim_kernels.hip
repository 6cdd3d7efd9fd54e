// gfx950 kernels around the per-env ones of team_kernels.hip: the controller's
// weight gradient and transposed weights, and the dispatch by team width.
#include <hip/hip_runtime.h>

#include "drivers.h"
#include "sim_internal.h"

namespace sim {

// Weight gradient of the controller as a contraction over env-steps:
//   dW_l[i][k] = sum_n delta_l[n][i] * act_l[n][k],  db_l[i] = sum_n delta_l[n][i]
// (act_1 = s, act_2 = h1, act_3 = h2; delta_1 = d1, delta_2 = d2, delta_3 = du).
// One wave computes one 32x32 output tile of one layer over one chunk of
// env-steps with v_mfma_f32_32x32x2f32 (A = delta rows, B = activations with
// an all-ones column for the bias), and writes the partial tile; the chunks
// are summed in a fixed order by k_wgrad_reduce (no atomics).
typedef float floatx16 __attribute__((ext_vector_type(16)));

__global__ __launch_bounds__(64) void k_wgrad_mfma(const float* __restrict__ tape, int stride, int n_rows, int chunk,
                                                   const WgradTile* __restrict__ tiles, int n_tiles,
                                                   float* __restrict__ partial) {
  const int tile = blockIdx.x, c = blockIdx.y, lane = threadIdx.x;
  const WgradTile T = tiles[tile];
  const int li = lane & 31, lk = lane >> 5;
  const int i = T.i0 + li, j = T.k0 + li;
  const bool ia = i < T.M;
  const bool jb = j < T.K;
  const float one = (j == T.K) ? 1.f : 0.f;
  const int n0 = c * chunk;
  const int n1 = min(n_rows, n0 + chunk);
  floatx16 acc;
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  for (int n = n0; n < n1; n += 2) {
    const int row = n + lk;
    float a = 0.f, b = 0.f;
    if (row < n1) {
      const float* rp = tape + (size_t)row * stride;
      a = ia ? rp[T.a_off + i] : 0.f;
      b = jb ? rp[T.b_off + j] : one;
    }
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
  }
  // D[row][col], col = lane % 32, row = 8 (r / 4) + 4 (lane / 32) + r % 4
  float* out = partial + ((size_t)c * n_tiles + tile) * 1024;
  for (int r = 0; r < 16; ++r) {
    const int row = 8 * (r >> 2) + 4 * lk + (r & 3);
    out[row * 32 + li] = acc[r];
  }
}

__global__ void k_wgrad_reduce(const float* __restrict__ partial, int n_chunks, int n_tiles,
                               const int* __restrict__ map, int n_params, float* __restrict__ g) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n_params) return;
  const int m = map[p];
  float acc = 0.f, comp = 0.f;
  for (int c = 0; c < n_chunks; ++c) kahan_add(&acc, &comp, partial[(size_t)c * n_tiles * 1024 + m]);
  g[p] = acc;
}

hipError_t launch_wgrad(const float* tape, int stride, int n_rows, int chunk, const WgradTile* tiles, int n_tiles,
                        float* partial, const int* map, int n_params, float* g, hipStream_t st) {
  const int n_chunks = (n_rows + chunk - 1) / chunk;
  if (n_chunks > 0) {
    hipLaunchKernelGGL(k_wgrad_mfma, dim3(n_tiles, n_chunks), dim3(64), 0, st, tape, stride, n_rows, chunk, tiles,
                       n_tiles, partial);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_wgrad_reduce, dim3((n_params + 255) / 256), dim3(256), 0, st, partial, n_chunks, n_tiles,
                     map, n_params, g);
  return hipGetLastError();
}

// Transposed controller weights for the forward products: Wt_l[k][n] = W_l[n][k].
__global__ void k_ctrl_transpose(const float* W, float* Wt, int in, int n1, int n2, int no) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  const int s1 = n1 * in, s2 = n2 * n1, s3 = no * n2;
  if (p < s1) {
    const int k = p / n1, n = p - k * n1;           // Wt1[k][n], k < in
    Wt[p] = W[n * in + k];
  } else if (p < s1 + s2) {
    const int q = p - s1, k = q / n2, n = q - k * n2;   // Wt2[k][n], k < n1
    Wt[p] = W[s1 + n1 + n * n1 + k];
  } else if (p < s1 + s2 + s3) {
    const int q = p - s1 - s2, k = q / no, n = q - k * no;   // Wt3[k][n], k < n2
    Wt[p] = W[s1 + n1 + s2 + n2 + n * n2 + k];
  }
}
hipError_t launch_ctrl_transpose(const float* W, float* Wt, int in, int n1, int n2, int no, hipStream_t st) {
  const int n = n1 * in + n2 * n1 + no * n2;
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_ctrl_transpose, dim3((n + 255) / 256), dim3(256), 0, st, W, Wt, in, n1, n2, no);
  return hipGetLastError();
}

__global__ void k_zero_ints(int* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// A lane that waits, for at most `ticks` of the 100 MHz clock, until *flag is
// `value`, and writes what it last saw; and the lane that sets it.  Two streams whose
// kernels do not meet so share a hardware queue.
__global__ void k_wait_flag(const int* flag, int value, int* seen, long long ticks) {
  const long long t0 = wall_clock64();
  int v = 0;
  while (v != value && wall_clock64() - t0 < ticks)
    v = __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  *seen = v;
}
__global__ void k_set_flag(int* flag, int value) {
  __hip_atomic_store(flag, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------------ launchers
hipError_t launch_wait_flag(const int* flag, int value, int* seen, long long ticks, hipStream_t st) {
  hipLaunchKernelGGL(k_wait_flag, dim3(1), dim3(1), 0, st, flag, value, seen, ticks);
  return hipGetLastError();
}
hipError_t launch_set_flag(int* flag, int value, hipStream_t st) {
  hipLaunchKernelGGL(k_set_flag, dim3(1), dim3(1), 0, st, flag, value);
  return hipGetLastError();
}
#define SIM_TEAMS(CALL)                                                                                      \
  switch (team) {                                                                                            \
    case 1: return TeamLaunch<1>::CALL;                                                                      \
    case 2: return TeamLaunch<2>::CALL;                                                                      \
    case 4: return TeamLaunch<4>::CALL;                                                                      \
    case 8: return TeamLaunch<8>::CALL;                                                                      \
    case 16: return TeamLaunch<16>::CALL;                                                                    \
    case 32: return TeamLaunch<32>::CALL;                                                                    \
    case 64: return TeamLaunch<64>::CALL;                                                                    \
    default: return hipErrorInvalidValue;                                                                    \
  }

hipError_t launch_zero(int* p, int n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_zero_ints, dim3((n + 255) / 256), dim3(256), 0, st, p, n);
  return hipGetLastError();
}

hipError_t launch_rollout(const DevModel& M, const TileSet& ts, int team, int grid, size_t lds,
                          const RolloutArgs& a, hipStream_t st) {
  SIM_TEAMS(rollout(M, ts, grid, lds, a, st))
}
hipError_t launch_step(const DevModel& M, const TileSet& ts, int team, int grid, size_t lds, const StepArgs& a,
                       hipStream_t st) {
  SIM_TEAMS(step(M, ts, grid, lds, a, st))
}
hipError_t launch_rollout_grad(const DevModel& M, const TileSet& ts, int team, int grid, size_t lds,
                               const GradArgs& a, hipStream_t st) {
  SIM_TEAMS(grad(M, ts, grid, lds, a, st))
}
hipError_t launch_recompute(const DevModel& M, const TileSet& ts, int team, int grid, size_t lds,
                            const GradArgs& a, hipStream_t st) {
  SIM_TEAMS(recompute(M, ts, grid, lds, a, st))
}
hipError_t launch_rollout_keep(const DevModel& M, const TileSet& ts, int team, int grid, size_t lds,
                               const RolloutArgs& a, hipStream_t st) {
  SIM_TEAMS(rollout_keep(M, ts, grid, lds, a, st))
}

static hipError_t allow_lds_of(int team, int bytes) { SIM_TEAMS(allow_lds(bytes)) }
hipError_t allow_large_lds(int bytes) {
  for (int team = 1; team <= 64; team *= 2) {
    const hipError_t e = allow_lds_of(team, bytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace sim

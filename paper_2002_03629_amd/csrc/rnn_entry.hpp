// Host side of the recurrent-network entry points (included by jacobi_made.hip after its error helpers).
#pragma once

#include "../../include/jacobi_rnn.h"
#include "rnn.hpp"

// rnn_param_grads: up to this many chunks of rows are summed by one workgroup per strip (a chunk takes it ~1.2 us; taking a
// piece and adding the slices in launches of their own, with the gaps to them, takes about 8 us)
constexpr int GRAD_ONE_SLICE = 8;

// LAUNCH(CT) with CT = the number of 32-unit tiles H units take
#define JM_RNN_BY_WIDTH(H, LAUNCH)       \
  switch (((H) + 31) / 32) {             \
    case 1: LAUNCH(1); break;            \
    case 2: LAUNCH(2); break;            \
    case 3: LAUNCH(3); break;            \
    default: LAUNCH(4); break;           \
  }

static int rnn_check_shape(const char* who, int B, int T, int H) {
  if (B < 0 || T < 1 || H < 1) return fail(MADE_ERR_ARG, "%s: B=%d, T=%d, H=%d out of range", who, B, T, H);
  if (H > RNN_MAX_H) return fail(MADE_ERR_ARG, "%s: H=%d, at most %d hidden units are supported", who, H, RNN_MAX_H);
  return MADE_OK;
}

extern "C" int rnn_jacobi_max_steps(int32_t H) {
  if (H < 1 || H > RNN_MAX_H) return 0;
  const int CT = (H + 31) / 32;
  return 32 * RNN_TILES_PER_WAVE * (RNN_WAVES / CT);
}

extern "C" int rnn_forward(const float* W, const float* U, const float* b, const float* x, const float* h0, int32_t B,
                           int32_t T, int32_t H, int32_t I, float* z, float* h, void* stream) {
  TRY(rnn_check_shape("rnn_forward", B, T, H));
  if (I < 1) return fail(MADE_ERR_ARG, "rnn_forward: I=%d must be >= 1", I);
  if (B == 0) return MADE_OK;   // (an empty batch has nothing to point at)
  if (!W || !U || !b || !x || !z || !h) return fail(MADE_ERR_ARG, "rnn_forward: NULL argument");
#define JM_FORWARD(N) hipLaunchKernelGGL((H == 32 * N ? rnn_forward_kernel<N, true> : rnn_forward_kernel<N, false>), dim3(B), dim3(RnnStep<N>::THREADS), 0, \
                                         (hipStream_t)stream, W, U, b, x, h0, z, h, T, H, I)
  JM_RNN_BY_WIDTH(H, JM_FORWARD);
#undef JM_FORWARD
  HIP_TRY(hipGetLastError());
  return MADE_OK;
}

extern "C" int rnn_backward_sequential(const float* W, const float* z, const float* g, int32_t B, int32_t T, int32_t H,
                                       float* d, void* stream) {
  TRY(rnn_check_shape("rnn_backward_sequential", B, T, H));
  if (B == 0) return MADE_OK;
  if (!W || !z || !g || !d) return fail(MADE_ERR_ARG, "rnn_backward_sequential: NULL argument");
#define JM_BACKWARD(N) hipLaunchKernelGGL((H == 32 * N ? rnn_backward_seq_kernel<N, true> : rnn_backward_seq_kernel<N, false>), dim3(B), \
                                          dim3(RnnStep<N>::THREADS), 0, (hipStream_t)stream, W, z, g, d, T, H)
  JM_RNN_BY_WIDTH(H, JM_BACKWARD);
#undef JM_BACKWARD
  HIP_TRY(hipGetLastError());
  return MADE_OK;
}

template <int CT>
static int rnn_launch_jacobi(const RnnJacobiArgs& a, size_t lds, hipStream_t s) {
  static size_t configured = 0;
  if (lds > configured) {
    HIP_TRY(hipFuncSetAttribute((const void*)rnn_jacobi_kernel<CT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    configured = lds;
  }
  hipLaunchKernelGGL(rnn_jacobi_kernel<CT>, dim3(a.B), dim3(RNN_WAVES * 64), lds, s, a);
  HIP_TRY(hipGetLastError());
  return MADE_OK;
}

extern "C" int rnn_backward_jacobi(const float* W, const float* z, const float* g, const float* d_init, int32_t B, int32_t T,
                                   int32_t H, int32_t n_iters, float eps, float* d, int32_t* iters_out,
                                   int32_t* converged_out, void* stream) {
  TRY(rnn_check_shape("rnn_backward_jacobi", B, T, H));
  if (!(eps >= 0.0f)) return fail(MADE_ERR_ARG, "rnn_backward_jacobi: eps must be >= 0");
  if (T > rnn_jacobi_max_steps(H))
    return fail(MADE_ERR_ARG, "rnn_backward_jacobi: T=%d, at most %d steps are supported with H=%d", T, rnn_jacobi_max_steps(H), H);
  if (B == 0) return MADE_OK;
  if (!W || !z || !g || !d) return fail(MADE_ERR_ARG, "rnn_backward_jacobi: NULL argument");
  RnnJacobiArgs a;
  a.W = W;
  a.z = z;
  a.g = g;
  a.d_init = d_init;
  a.d = d;
  a.iters = iters_out;
  a.converged = converged_out;
  a.B = B;
  a.T = T;
  a.H = H;
  a.cap = (n_iters <= 0 || n_iters > T) ? T : n_iters;
  a.eps = eps;
  const int CT = (H + 31) / 32, Tp = round_up(T, 32);
  // (a second copy of X where LDS holds it: every shape but more than 480 steps of up to 32 units)
  const size_t one = (size_t)2 * Tp * (32 * CT + 8) * sizeof(uint16_t);
  a.x_bytes = 2 * one <= 160 * 1024 - 256 ? (int)one : 0;
  const size_t lds = one + a.x_bytes;
  hipStream_t s = (hipStream_t)stream;
  switch (CT) {
    case 1: return rnn_launch_jacobi<1>(a, lds, s);
    case 2: return rnn_launch_jacobi<2>(a, lds, s);
    case 3: return rnn_launch_jacobi<3>(a, lds, s);
    default: return rnn_launch_jacobi<4>(a, lds, s);
  }
}

extern "C" int rnn_param_grads(const float* z, const float* h, const float* x, const float* d, const float* h0, int32_t B,
                               int32_t T, int32_t H, int32_t I, float* dW, float* dU, float* db, void* stream) {
  TRY(rnn_check_shape("rnn_param_grads", B, T, H));
  if (I < 1) return fail(MADE_ERR_ARG, "rnn_param_grads: I=%d must be >= 1", I);
  if (!z || !h || !x || !d || !dW || !dU || !db) return fail(MADE_ERR_ARG, "rnn_param_grads: NULL argument");
  const int CT = (H + 31) / 32;
  const long long rows = (long long)B * T, chunks = (rows + GRAD_ROWS - 1) / GRAD_ROWS;
  // One slice (results stored at once) for up to GRAD_ONE_SLICE chunks, else as many as give every compute unit two
  // workgroups and fit a piece.
  const long long stride = grad_stride(H, I);
  long long slices = chunks <= GRAD_ONE_SLICE ? 1 : std::min<long long>(chunks, 512 / CT);
  slices = std::max<long long>(1, std::min(slices, GRAD_PIECE_FLOATS / stride));
  const long long slice_rows = std::max<long long>(1, (chunks + slices - 1) / slices * GRAD_ROWS);
  slices = std::max<long long>(1, (rows + slice_rows - 1) / slice_rows);
  hipStream_t s = (hipStream_t)stream;
  static std::atomic<unsigned long long> calls{0};
  const unsigned long long key = ++calls;
  if (slices > 1) hipLaunchKernelGGL(rnn_grads_claim_kernel, dim3(1), dim3(1), 0, s, key);
  const dim3 grid(CT, (unsigned)slices, I / GRAD_SLOTS + 1), block(RNN_WAVES * 64);
#define JM_GRADS(N) hipLaunchKernelGGL(rnn_param_grads_kernel<N>, grid, block, 0, s, z, h, x, d, h0, rows, T, H, I, (int)slice_rows, (int)slices, key, dW, dU, db)
  JM_RNN_BY_WIDTH(H, JM_GRADS);
#undef JM_GRADS
  if (slices > 1)
    hipLaunchKernelGGL(rnn_grads_add_kernel, dim3((unsigned)((stride + 255) / 256)), dim3(64 * GRAD_GROUPS), 0, s, key, (int)slices, (int)stride,
                       H * H, H * I, H, dW, dU, db);
  HIP_TRY(hipGetLastError());
  return MADE_OK;
}

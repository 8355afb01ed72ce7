// Output layer of a categorical model with any number of classes (2..256): product, Gumbel-max draw and change
// detection in one kernel; the logits live in LDS only (gfx950 only).
//
// A workgroup owns CAT_ANY_ROWS samples x `pos_per_wg` consecutive positions.  Output row t * C + c is class c of
// position t, so those positions are a run of output rows, covered by at most CAT_ANY_TILES unit tiles of 32 (a tile
// that straddles two workgroups' runs is multiplied by both).  Eight waves take (tile, K part) pairs: a run of n
// tiles is multiplied by 8 / n (rounded down to a power of two) waves per tile, each on an interleaved part of the K
// chunks.  The partial tiles go to LDS, noise and bias are added there, and groups of eight lanes pick the maximum of
// one (sample, position) each.
//
// What bounds it: the weights' way from the memory-side cache, and latency (a wave has two K chunks in flight).  512
// positions of 64 classes, 1024 last-layer units, 100 samples, 17 MB of visible weights and 13 MB of noise a pass:
// before, the logits went to memory (18 us) and were drawn by a second kernel with one workgroup per four draws,
// whose 12800 arrivals at one counter took 114 us; see cat_any_positions for the split.
#pragma once

#include "kernels.hpp"

namespace jm {

constexpr int CAT_ANY_WAVES = 8;
constexpr int CAT_ANY_ROWS = 64;                       // samples per workgroup
constexpr int CAT_ANY_TILES = 9;                       // C = 226..255 not a multiple of 32: one position touches nine tiles
constexpr int CAT_ANY_FULL = 256;                      // output rows of a workgroup's positions, at most
constexpr int CAT_ANY_POS = 32;                        // positions of a workgroup, at most
constexpr int CAT_ANY_PITCH = TILE + 1;

struct CatAnyArgs {
  CatArgs c;             // operands and bookkeeping as for the 256-class kernel
  int C;
  int out_cols;          // D * C
  int pos_per_wg;        // positions per workgroup: <= CAT_ANY_POS, pos_per_wg * C <= CAT_ANY_FULL
  int groups;            // position groups of this launch
};

// One K part of a 32-row weight tile against both sample tiles: chunks c0, c0 + step, ... (CNT of them) requested
// before the first is multiplied.
template <typename T, int CNT>
__device__ __forceinline__ void cat_any_group(const uint4* W, const uint4* A0, const uint4* A1, int c0, int step,
                                              f32x16 (&acc)[2]) {
  uint4 w[CNT][4], a0[CNT][4], a1[CNT][4];
#pragma unroll
  for (int p = 0; p < CNT; ++p) {
    const size_t o = (size_t)(c0 + p * step) * 256;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      w[p][s] = W[o + s * 64];
      a0[p][s] = A0[o + s * 64];
      a1[p][s] = A1[o + s * 64];
    }
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int p = 0; p < CNT; ++p) {
    mfma_chunk<T>(a0[p], w[p], acc[0]);
    mfma_chunk<T>(a1[p], w[p], acc[1]);
  }
}

template <typename T>
__global__ __launch_bounds__(CAT_ANY_WAVES * 64) void categorical_any_kernel(CatAnyArgs p) {
  constexpr int KC = 2 * Elem<T>::EPL;
  const CatArgs& a = p.c;
  // [wave or ninth tile][sample][row of the tile]; logits end up in the slots of K part 0
  __shared__ float part[CAT_ANY_TILES][CAT_ANY_ROWS][CAT_ANY_PITCH];
  __shared__ int sample_s[CAT_ANY_ROWS], changed_s[CAT_ANY_ROWS];
  __shared__ uint8_t x_s[CAT_ANY_ROWS][CAT_ANY_POS];   // the symbols before this pass
  __shared__ int first_s;
  const int n_rows = a.n_rows_ptr ? *a.n_rows_ptr : a.n_rows;
  const int t_first = a.t_first_ptr ? *a.t_first_ptr : 0;
  // the sample tiles that share a run of weights sit on one XCD (workgroup i runs on XCD i % 8); the runs with the
  // longest visible prefixes come first
  const int xcd = blockIdx.x % XCDS, slot = blockIdx.x / XCDS;
  const int pair = slot % a.pair_tiles, group = p.groups - 1 - ((slot / a.pair_tiles) * XCDS + xcd);
  const int row0 = pair * CAT_ANY_ROWS;
  const int tp = a.t_begin + group * p.pos_per_wg;
  const int n_pos = min(p.pos_per_wg, a.t_begin + a.n_pos - tp);
  if (group >= 0 && row0 < n_rows && tp + n_pos > t_first) {   // (uniform per workgroup)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 31, h = lane >> 5;
    const int R0 = tp * p.C, R = n_pos * p.C;                   // output rows [R0, R0 + R)
    const int tile0 = R0 / TILE, n_tiles = (R0 + R - 1) / TILE - tile0 + 1;
    const int lg = n_tiles > 4 ? 3 : n_tiles > 2 ? 2 : n_tiles > 1 ? 1 : 0;
    const int tile_slots = 1 << lg, k_parts = CAT_ANY_WAVES >> lg;   // (n_tiles = 9: wave 0 also takes the ninth)
    // (the list is padded with valid ids to whole pairs of tiles)
    const int n0 = a.rows ? a.rows[row0 + r] : min(row0 + r, a.n_rows - 1);
    const int n1 = a.rows ? a.rows[row0 + 32 + r] : min(row0 + 32 + r, a.n_rows - 1);
    const size_t gsize = (size_t)a.k_chunks * 256;
    const uint4* A0 = (const uint4*)a.A + (size_t)(n0 >> 5) * gsize + h * 32 + (n0 & 31);
    const uint4* A1 = (const uint4*)a.A + (size_t)(n1 >> 5) * gsize + h * 32 + (n1 & 31);
    if (threadIdx.x < 64) {
      sample_s[threadIdx.x] = lane < 32 ? n0 : n1;     // (lane = row of the pair of sample tiles)
      changed_s[threadIdx.x] = 0;
    }
    if (threadIdx.x == 0) first_s = NO_CHANGE;

    // Noise and old symbols, requested before the product so that their way from memory overlaps with it.  Wave w owns
    // samples w, w + 8, ...; a lane owns output rows R0 + lane, + 64, ... of the positions that are re-drawn.
    const int draw_lo = max(a.t_lo - tp, 0) * p.C, draw_hi = min(a.t_hi - tp, n_pos) * p.C;
    constexpr int NS = CAT_ANY_ROWS / CAT_ANY_WAVES, NR = CAT_ANY_FULL / 64;
    float g[NS][NR];
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const int s = wave + i * CAT_ANY_WAVES;
      const int sample = __builtin_amdgcn_readlane(s < 32 ? n0 : n1, s & 31);
      const float* gp = a.noise + (size_t)sample * p.out_cols + R0;
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        g[i][q] = 0.f;
        if (lane + 64 * q >= draw_lo && lane + 64 * q < draw_hi && row0 + s < n_rows) g[i][q] = gp[lane + 64 * q];
      }
    }
    constexpr int NX = CAT_ANY_POS / (CAT_ANY_WAVES * 64 / CAT_ANY_ROWS);
    uint8_t xo[NX];
#pragma unroll
    for (int q = 0; q < NX; ++q) {
      const int s = (q * CAT_ANY_WAVES * 64 + threadIdx.x) / CAT_ANY_POS, tt = threadIdx.x % CAT_ANY_POS;
      const int sample = __shfl(s < 32 ? n0 : n1, s & 31);
      xo[q] = 0;
      if (tt < n_pos && row0 + s < n_rows) xo[q] = a.x[(size_t)sample * a.D + tp + tt];
    }
    __builtin_amdgcn_sched_barrier(0);

    for (int tl = wave & (tile_slots - 1), kp = wave >> lg; tl < n_tiles; tl += tile_slots, kp += k_parts) {
      // (tl >= tile_slots only for the ninth tile, where k_parts = 1; wave 0 multiplies all of it)
      f32x16 acc[2];
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[j][i] = 0.f;
      const int k0 = tl < tile_slots ? kp : 0;
      const int k_end = min(a.tile_kend[tile0 + tl], a.k_cap);
      const int n_chunks = (k_end + KC - 1) / KC;
      const uint4* W = (const uint4*)a.W + (size_t)(tile0 + tl) * gsize + h * 32 + r;
      int c = k0;
      for (; c + k_parts < n_chunks; c += 2 * k_parts) cat_any_group<T, 2>(W, A0, A1, c, k_parts, acc);
      if (c < n_chunks) cat_any_group<T, 1>(W, A0, A1, c, k_parts, acc);
      const int dst = tl < tile_slots ? wave : CAT_ANY_WAVES;
      // acc[j][i]: sample 32 j + 8 (i / 4) + 4 h + i % 4, row r of the tile
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) part[dst][32 * j + 8 * (i >> 2) + 4 * h + (i & 3)][r] = acc[j][i];
    }
#pragma unroll
    for (int q = 0; q < NX; ++q)
      x_s[(q * CAT_ANY_WAVES * 64 + threadIdx.x) / CAT_ANY_POS][threadIdx.x % CAT_ANY_POS] = xo[q];
    __syncthreads();
    // logit + noise, in the slot of K part 0 (an element is read and written by one thread)
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const int rr = lane + 64 * q;
      if (rr < R) {
        const int gr = R0 + rr, tl = gr / TILE - tile0, cc = gr % TILE;
        const int base = tl < tile_slots ? tl : CAT_ANY_WAVES;
        const float b = a.bias[gr];
#pragma unroll
        for (int i = 0; i < NS; ++i) {
          const int s = wave + i * CAT_ANY_WAVES;
          float v = part[base][s][cc];
          for (int k = 1; k < k_parts; ++k) v += part[base + k * tile_slots][s][cc];
          part[base][s][cc] = (v + b) + g[i][q];
        }
      }
    }
    __syncthreads();
    // eight lanes per (sample, position); lowest class on ties
    const int sub = lane & 7;
    for (int it = threadIdx.x >> 3; it < CAT_ANY_ROWS * n_pos; it += CAT_ANY_WAVES * 8) {
      const int s = it & (CAT_ANY_ROWS - 1), tt = it / CAT_ANY_ROWS, t = tp + tt;
      float best = -INFINITY;
      int best_c = 0x7fffffff;
      for (int c = sub; c < p.C; c += 8) {
        const int gr = R0 + tt * p.C + c, tl = gr / TILE - tile0;
        const float v = part[tl < tile_slots ? tl : CAT_ANY_WAVES][s][gr % TILE];
        if (v > best || (v == best && c < best_c)) { best = v; best_c = c; }
      }
#pragma unroll
      for (int off = 4; off > 0; off >>= 1) {
        const float ob = __shfl_xor(best, off);
        const int oc = __shfl_xor(best_c, off);
        if (ob > best || (ob == best && oc < best_c)) { best = ob; best_c = oc; }
      }
      if (sub == 0 && row0 + s < n_rows && t >= a.t_lo && t < a.t_hi) {
        const uint8_t xn = (uint8_t)best_c;
        if (xn != x_s[s][tt]) {
          const int sample = sample_s[s];
          a.x[(size_t)sample * a.D + t] = xn;
          ((T*)a.enc)[frag_offset<T>(sample, t, a.enc_chunks)] = Elem<T>::from_f32(((float)xn - 128.0f) * (1.0f / 128.0f));
          atomicAdd(&changed_s[s], 1);
          atomicMin(&first_s, t);
        }
      }
    }
    __syncthreads();
    // one update per sample, performed before this workgroup reports in (see finish_pass)
    if (threadIdx.x < CAT_ANY_ROWS && changed_s[threadIdx.x] > 0)
      count_changed(&a.changed[(size_t)sample_s[threadIdx.x] * CHG], changed_s[threadIdx.x]);
    if (a.first_changed && threadIdx.x == 0 && first_s != NO_CHANGE) {
      const int old = __hip_atomic_fetch_min(a.first_changed, first_s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("" ::"v"(old));
    }
  }
  if (a.retire.enabled) finish_pass(a.retire, gridDim.x);
}

}  // namespace jm

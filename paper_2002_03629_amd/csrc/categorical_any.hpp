// Output layer of a categorical model with any number of classes (2..256): product, Gumbel-max draw and change
// detection in one kernel; the logits live in LDS only (gfx950 only).
//
// A workgroup owns CAT_ANY_ROWS samples x `pos_per_wg` consecutive positions.  Output row t * C + c is class c of
// position t, so those positions are a run of output rows, covered by at most CAT_ANY_TILES unit tiles of 32 (a tile
// that straddles two workgroups' runs is multiplied by both).  Noise and bias are added to the products in LDS, and groups of
// eight lanes pick the maximum of one (sample, position) each.
//
// A logit is summed as masked_layer_kernel sums it -- NW parts, part p the K chunks p, p + NW, ..., added in the order of p --
// whatever the length of the run: a draw has the same bits in every pass, solver and launch shape, and the same as from
// logits in memory.  Eight waves share the work of a run of n tiles: more than four: a wave takes all parts of a tile; three
// or four: the first five or the last three; two: two parts; one: one.  Waves that start with part 0 add the parts up in
// registers, the others leave theirs in LDS one by one (which is why it is not four and four: 20 patches are too many).
//
// What bounds it: the weights' way from the memory-side cache, and latency (a wave has two K chunks in flight).  512
// positions of 64 classes, 1024 last-layer units, 100 samples, 17 MB of visible weights and 13 MB of noise a pass:
// before, the logits went to memory (18 us) and were drawn by a second kernel with one workgroup per four draws,
// whose 12800 arrivals at one counter took 114 us; see cat_any_positions for the split.
// Taking a logit's parts one by one costs 3 to 8 % of a call against sums split by the length of the run (512 positions of
// 64 classes, 100 samples: 313 -> 329 us; 400 of 128, 64 samples: 280 -> 305; 200 of 200, 100 samples: 204 -> 207), whose bits
// changed with the number of samples still active.
#pragma once

#include "kernels.hpp"

namespace jm {

constexpr int CAT_ANY_WAVES = 8;
static_assert(NW == 8, "the parts of a sum are dealt to eight waves by tile count");
constexpr int CAT_ANY_ROWS = 64;                       // samples per workgroup
constexpr int CAT_ANY_TILES = 9;                       // C = 226..255 not a multiple of 32: one position touches nine tiles
constexpr int CAT_ANY_FULL = 256;                      // output rows of a workgroup's positions, at most
constexpr int CAT_ANY_POS = 32;                        // positions of a workgroup, at most
constexpr int CAT_ANY_PITCH = TILE + 1;
constexpr int CAT_ANY_PATCHES = 16;                    // of 64 x 32 sums in LDS: four tiles and three parts of each, at most

struct CatAnyArgs {
  CatArgs c;             // operands and bookkeeping as for the 256-class kernel
  int C;
  int out_cols;          // D * C
  int pos_per_wg;        // positions per workgroup: <= CAT_ANY_POS, pos_per_wg * C <= CAT_ANY_FULL
  int groups;            // position groups of this launch
};

// Parts [pb, pe) of the sums of a 32-row weight tile and both sample tiles: done(part, sums) for each that has chunks.
// Two chunks are requested before the first is multiplied.
template <typename T, typename F>
__device__ __forceinline__ void cat_any_parts(const uint4* W, const uint4* A0, const uint4* A1, int n_chunks, int pb, int pe, F&& done) {
  constexpr int CNT = 2, J = 2;
  f32x16 acc[J];
#pragma unroll
  for (int j = 0; j < J; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[j][i] = 0.f;
  pe = min(pe, n_chunks);
  for (int p = pb, c = pb; p < pe;) {
    uint4 w[CNT][4], a[J][CNT][4];
    int part[CNT];
    bool last[CNT];
    int at = c;
#pragma unroll
    for (int i = 0; i < CNT; ++i) {
      part[i] = p;
      if (p < pe) at = c;                  // (past the last part: the last chunk once more, unused)
      c += NW;
      last[i] = c >= n_chunks;
      if (last[i]) c = ++p;
      const size_t o = (size_t)at * 256;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        w[i][s] = W[o + s * 64];
#pragma unroll
        for (int j = 0; j < J; ++j) a[j][i][s] = (j ? A1 : A0)[o + s * 64];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < CNT; ++i) {
      if (part[i] < pe) {
#pragma unroll
        for (int j = 0; j < J; ++j) mfma_chunk<T>(a[j][i], w[i], acc[j]);
        if (last[i]) {
          done(part[i], acc);
#pragma unroll
          for (int j = 0; j < J; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;
        }
      }
    }
  }
}

template <typename T>
__global__ __launch_bounds__(CAT_ANY_WAVES * 64) void categorical_any_kernel(CatAnyArgs p) {
  constexpr int KC = 2 * Elem<T>::EPL;
  const CatArgs& a = p.c;
  // [patch][sample][row of the tile]; patch tl = tile tl of the run: the sum from part 0 on, then the logits
  __shared__ float part[CAT_ANY_PATCHES][CAT_ANY_ROWS][CAT_ANY_PITCH];
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
    // waves = 1 << lg tiles x groups of parts; the `rest` parts of a tile that the first group does not have lie in patches
    // of their own, from patch (1 << lg) + tile * rest on  (nine tiles: wave 0 also takes the ninth)
    const int lg = n_tiles > 4 ? 3 : n_tiles > 2 ? 2 : n_tiles > 1 ? 1 : 0;
    const int in_first = lg == 3 ? 8 : lg == 2 ? 5 : 1 << lg, rest = NW - in_first;
    const auto rest_patch = [&](int tl) { return (1 << lg) + tl * rest; };
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

    f32x16 zero;
#pragma unroll
    for (int e = 0; e < 16; ++e) zero[e] = 0.f;
    const int group = wave >> lg, pb = group == 0 ? 0 : lg == 2 ? in_first : group << lg;
    const int pe = group == 0 ? in_first : lg == 2 ? NW : (group + 1) << lg;
    for (int tl = wave & ((1 << lg) - 1); tl < n_tiles; tl += 1 << lg) {
      const int n_chunks = (min(a.tile_kend[tile0 + tl], a.k_cap) + KC - 1) / KC;
      f32x16 tot[2] = {zero, zero};
      const auto store = [&](int patch, const f32x16 (&v)[2]) {   // v[j][e]: sample 32 j + 8 (e / 4) + 4 h + e % 4, row r
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) part[patch][32 * j + 8 * (e >> 2) + 4 * h + (e & 3)][r] = v[j][e];
      };
      cat_any_parts<T>((const uint4*)a.W + (size_t)(tile0 + tl) * gsize + h * 32 + r, A0, A1, n_chunks, pb, pe,
                       [&](int p, const f32x16 (&sums)[2]) {
        if (group) {
          store(rest_patch(tl) + p - in_first, sums);
        } else {
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) tot[j][e] += sums[j][e];
        }
      });
      if (!group) store(tl, tot);
      for (int p = max(pb, n_chunks); group && p < pe; ++p) store(rest_patch(tl) + p - in_first, tot);   // (parts without chunks)
    }
#pragma unroll
    for (int q = 0; q < NX; ++q)
      x_s[(q * CAT_ANY_WAVES * 64 + threadIdx.x) / CAT_ANY_POS][threadIdx.x % CAT_ANY_POS] = xo[q];
    __syncthreads();
    // logit + noise, in the tile's own patch (an element is read and written by one thread)
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const int rr = lane + 64 * q;
      if (rr < R) {
        const int gr = R0 + rr, tl = gr / TILE - tile0, cc = gr % TILE;
        const int base = rest_patch(tl);
        const float b = a.bias[gr];
#pragma unroll
        for (int i = 0; i < NS; ++i) {
          const int s = wave + i * CAT_ANY_WAVES;
          float v = part[tl][s][cc];
          for (int k = 0; k < rest; ++k) v += part[base + k][s][cc];
          part[tl][s][cc] = (v + b) + g[i][q];
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
        const float v = part[tl][s][gr % TILE];
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

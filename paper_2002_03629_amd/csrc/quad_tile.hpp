// Masked layer on 64 x 64 (samples x units) tiles, for batches of a few hundred to a few thousand samples (gfx950 only).
//
// Between the 32 x 32 tiles (latency: the whole K range of a tile in flight at once) and the 128 x 128 ones (throughput:
// operands through an LDS ring) a launch is bound by what the compute units fetch from L2: a 32 x 32 tile takes 128
// bytes of each of its 64 operand rows for every 128 MFMA cycles, 1000 samples of a 2000 x 2000 layer 285 MB of L2
// reads.  Here a workgroup of eight waves owns 2 x 2 MFMA tiles and splits K between its waves: half the L2 traffic, four
// MFMAs per fragment pair, and still no LDS or barrier between the operands and the matrix cores.  A wave requests
// its next chunk (16 KB) ahead of the MFMAs of the one before.  A workgroup fills a compute unit (~200 registers, 128 KB of
// LDS).  The partial sums meet once: two waves finish a quadrant.
//
// A sum is taken in the order of the 32 x 32 kernel (wave w the chunks w, w + NW, ...; the waves' sums added in wave
// order), so that a layer's bits do not depend on which of the two a pass runs on -- that hangs on how many samples the
// host has seen stop.
#pragma once

#include "kernels.hpp"

namespace jm {

constexpr int QUAD = 2 * TILE;           // samples / units per workgroup

template <typename T, int EPI>
__global__ __launch_bounds__(NW * 64) void masked_layer_quad_kernel(LayerArgs a) {
  static_assert(EPI == EPI_RELU || EPI == EPI_BERNOULLI, "epilogues of the 64 x 64 tiles");
  static_assert(NW == 8, "two waves to a quadrant");
  constexpr int KC = 2 * Elem<T>::EPL;
  __shared__ float4 part_s[NW][4][4][64];  // [wave][quadrant][run of four units][lane]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, h = lane >> 5;
  const int n_rows = a.n_rows_ptr ? *a.n_rows_ptr : a.n_rows;
  // An XCD owns unit tiles; the tiles with the longest visible K (units are laid out by degree) are dispatched first.
  const int pairs = (a.n_launch_tiles + 1) / 2;
  const int slot = blockIdx.x / XCDS, order = (slot / a.row_tiles) * XCDS + blockIdx.x % XCDS;   // (row_tiles: of 64)
  const int row0 = (slot % a.row_tiles) * QUAD;
  if (order < pairs && row0 < n_rows) {    // (uniform)
    const int rel0 = 2 * (pairs - 1 - order), tile0 = a.tile_begin + rel0;
    const int last = min(1, a.n_launch_tiles - 1 - rel0);      // (a single tile at the end is multiplied twice)
    int k_end = max(a.tile_kend[tile0], a.tile_kend[tile0 + last]);
    if (k_end > a.k_cap) k_end = a.k_cap;
    const uint4 *Ap[2], *Wp[2];
    const size_t group = (size_t)a.k_chunks * 256;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = row0 + i * TILE + r;
      const int sample = a.a_by_pos ? a.pos_base + min(row, a.n_rows - 1)
                                    : (a.rows ? a.rows[min(row, a.n_rows_pad - 1)] : min(row, a.n_rows - 1));
      Ap[i] = (const uint4*)a.A + (size_t)(sample >> 5) * group + h * 32 + (sample & 31);
      Wp[i] = (const uint4*)a.W + (size_t)(tile0 + min(i, last)) * group + h * 32 + r;
    }
    // What this wave finishes: half of quadrant wave >> 1, sample tile wave >> 2 and unit tile (wave >> 1) & 1.  The weights
    // are the MFMA's row operand, so a lane ends up with one sample and runs of four units col0 + 8 g .. + 3, g < 2.
    const int quad = wave >> 1, unit_tile = quad & 1;
    const int e_row = row0 + (wave >> 2) * TILE + r;
    const bool row_ok = e_row < n_rows, tile_ok = unit_tile <= last;
    const int e_sample = a.rows ? a.rows[min(e_row, a.n_rows_pad - 1)] : min(e_row, a.n_rows - 1);
    const int col0 = (tile0 + min(unit_tile, last)) * TILE + 16 * (wave & 1) + 4 * h;
    float4 bias[2];
#pragma unroll
    for (int g = 0; g < 2; ++g) bias[g] = *(const float4*)(a.bias + col0 + 8 * g);
    // noise and symbols travel while the product runs: 16- and 4-byte pieces where rows are aligned, single ones else
    float u[2][4];
    uint32_t xo[2];
    const int p_lo = a.t_lo, p_hi = min(a.t_hi, a.D);
    if constexpr (EPI == EPI_BERNOULLI) {
      const size_t x_row = (size_t)e_sample * a.D;
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const int col = col0 + 8 * g;
        if (a.io_aligned) {      // (D is a multiple of 16: a run lies wholly inside the row or behind its end)
          const int c = col < a.D ? col : 0;
          const float4 v = *(const float4*)(a.noise + x_row + c);
          u[g][0] = v.x; u[g][1] = v.y; u[g][2] = v.z; u[g][3] = v.w;
          xo[g] = *(const uint32_t*)(a.x + x_row + c);
        } else {
          xo[g] = 0;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const int at = min(col + c, a.D - 1);
            u[g][c] = a.noise[x_row + at];
            xo[g] |= (uint32_t)a.x[x_row + at] << (8 * c);
          }
        }
      }
    }

    f32x16 acc[2][2];            // [sample tile][unit tile]
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    const int n_chunks = (k_end + KC - 1) / KC;
    const int n_mine = n_chunks > wave ? (n_chunks - wave + NW - 1) / NW : 0;   // chunks wave, wave + NW, ...
    struct Chunk { uint4 a[2][4], w[2][4]; };
    auto request = [&](int i, Chunk& c) {
      const size_t at = (size_t)(NW * min(i, n_mine - 1) + wave) * 256;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        c.a[0][s] = Ap[0][at + s * 64];
        c.a[1][s] = Ap[1][at + s * 64];
        c.w[0][s] = Wp[0][at + s * 64];
        c.w[1][s] = Wp[1][at + s * 64];
      }
      __builtin_amdgcn_sched_barrier(0);   // (the scheduler would sink the loads to their first use)
    };
    auto multiply = [&](const Chunk& c) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) mfma_chunk<T>(c.w[j], c.a[i], acc[i][j]);
      __builtin_amdgcn_sched_barrier(0);
    };
    if (n_mine > 0) {
      Chunk c0, c1;
      request(0, c0);
      // (no way out in mid-loop: the accumulators would be copied for it)
      for (int i = 0; i + 1 < n_mine; i += 2) {
        request(i + 1, c1);
        multiply(c0);
        request(i + 2, c0);                // (past the end: the last chunk once more, unused)
        multiply(c1);
      }
      if (n_mine & 1) multiply(c0);
    }

#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x16& s = acc[q >> 1][q & 1];
        part_s[wave][q][g][lane] = make_float4(s[4 * g], s[4 * g + 1], s[4 * g + 2], s[4 * g + 3]);
      }
    __syncthreads();
    float v[8];
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      float4 t = part_s[0][quad][2 * (wave & 1) + g][lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) {
        const float4 s = part_s[w][quad][2 * (wave & 1) + g][lane];
        t.x += s.x; t.y += s.y; t.z += s.z; t.w += s.w;
      }
      v[4 * g] = t.x; v[4 * g + 1] = t.y; v[4 * g + 2] = t.z; v[4 * g + 3] = t.w;
    }
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      v[4 * g] += bias[g].x; v[4 * g + 1] += bias[g].y; v[4 * g + 2] += bias[g].z; v[4 * g + 3] += bias[g].w;
    }
    if constexpr (EPI == EPI_RELU) {
      if (row_ok && tile_ok) {
        T* out = (T*)a.out + frag_row_offset<T>(a.out_by_pos ? a.pos_base + e_row : e_sample, a.out_chunks);
#pragma unroll
        for (int g = 0; g < 2; ++g)
          store_quad<T>(out + frag_col_offset<T>(col0 + 8 * g), fmaxf(v[4 * g], 0.f), fmaxf(v[4 * g + 1], 0.f),
                        fmaxf(v[4 * g + 2], 0.f), fmaxf(v[4 * g + 3], 0.f));
      }
    } else {
      int cnt = 0;
      if (row_ok && tile_ok) {
        const size_t x_row = (size_t)e_sample * a.D, enc_row = frag_row_offset<T>(e_sample, a.enc_chunks);
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          const int col = col0 + 8 * g;
          uint32_t xn = 0, live = 0;       // a byte per position
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            xn |= (u[g][c] < bernoulli_probability(v[4 * g + c]) ? 1u : 0u) << (8 * c);
            live |= (col + c >= p_lo && col + c < p_hi ? 0xffu : 0u) << (8 * c);
          }
          uint32_t d = (xn ^ xo[g]) & live;
          if (d) {                         // an unchanged symbol (and its encoding) is already in place
            if (a.io_aligned && live == 0xffffffffu) {
              *(uint32_t*)(a.x + x_row + col) = xn;
              store_quad<T>((T*)a.enc + (enc_row + frag_col_offset<T>(col)), (float)(xn & 1u), (float)((xn >> 8) & 1u),
                            (float)((xn >> 16) & 1u), (float)(xn >> 24));
            } else {
#pragma unroll
              for (int c = 0; c < 4; ++c)
                if ((d >> (8 * c)) & 0xffu) {
                  const uint32_t s = (xn >> (8 * c)) & 1u;
                  a.x[x_row + col + c] = (uint8_t)s;
                  ((T*)a.enc)[enc_row + frag_col_offset<T>(col + c)] = Elem<T>::from_f32((float)s);
                }
            }
            d |= d >> 4;                   // differing positions: one bit per non-zero byte
            d |= d >> 2;
            d |= d >> 1;
            cnt += __popc(d & 0x01010101u);
          }
        }
      }
      cnt += __shfl_xor(cnt, 32);          // the sample's other lane of this wave
      int old_count = 0;
      if (h == 0 && cnt > 0)
        old_count = __hip_atomic_fetch_add(&a.changed[(size_t)e_sample * CHG], cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("" ::"v"(old_count));   // (performed before this workgroup reports in: see finish_pass)
    }
  }
  if (EPI == EPI_BERNOULLI && a.retire.enabled) finish_pass(a.retire, gridDim.x);
}

}  // namespace jm

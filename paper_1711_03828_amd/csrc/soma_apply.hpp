// soma_apply.hpp -- the binned count updates of a sweep applied and the fields
// computed from the new counts in one pass over the bricks (two bead types).
//
// Between a sweep and the refresh that follows it, the counts would otherwise be
// written by bin_apply_kernel and read again by the field kernel; here a brick's
// counts go from LDS to memory and to the fields in one go.
#pragma once

#include "soma_bins.hpp"
#include "soma_grid.hpp"

namespace soma {

template <bool NT, class T>
__device__ __forceinline__ void store_hint(T *p, T v) {
  if (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// Blocks blk, blk + nblk, ... of the bricks of one grid.  With partials the
// refresh also leaves the sums of the counts (one partial per block, zeros in
// the rest of the n_parts entries that observables read).
// NT grids may have the fields in the blocked copy instead of omega (a.blocked).
// NT: counts and bin entries pass with the non-temporal hint (as in the field
// kernel: grids whose counts outgrow the caches keep their fields there instead).
template <bool COUNT64, bool NT, uint32_t THREADS>
__device__ __forceinline__ void apply_field_bricks(const BinArgs &b, const Grid &g,
                                                   const FieldArgs &a, uint32_t n_bricks,
                                                   uint32_t blk, uint32_t nblk, uint32_t n_parts,
                                                   uint32_t *s_cnt) {
  const uint32_t tid = threadIdx.x;
  const bool stats = a.partials != nullptr;
  FieldSums sums = {};
  for (uint32_t brick = blk; brick < n_bricks; brick += nblk) {
    bin_gather_brick<COUNT64, THREADS, NT>(b, g, a.counts, 1u, brick, s_cnt);
    uint32_t x0, y0, z0;
    brick_origin(b, brick, x0, y0, z0);
    const uint32_t x = x0 + (tid & 15u), y = y0 + ((tid >> 4) & 15u);
    if (x < (uint32_t)g.nx && y < (uint32_t)g.ny) {
#pragma unroll
      for (uint32_t u = 0; u < kBrickCells / THREADS; ++u) {
        const uint32_t z = z0 + ((tid + u * THREADS) >> 8);
        if (z >= (uint32_t)g.nz) break;
        const uint32_t r = z * (uint32_t)g.ny + y, c = r * (uint32_t)g.nx + x;
        const uint32_t i = tid + u * THREADS;
        uint32_t na, nb;
        if (COUNT64) {
          const uint2 v = reinterpret_cast<const uint2 *>(s_cnt)[i];
          store_hint<NT>(reinterpret_cast<unsigned long long *>(a.counts) + c,
                         ((unsigned long long)v.y << 32) | v.x);
          na = v.x;
          nb = v.y;
        } else {
          const uint32_t v = s_cnt[i];
          store_hint<NT>(reinterpret_cast<uint32_t *>(a.counts) + c, v);
          na = v & 0xFFFFu;
          nb = v >> 16;
        }
        float va, vb;
        field_cell(na, nb, a, va, vb);
        const bool off = cell_forbidden(a.forbid, c);
        if (a.ext || a.forbid) field_extras(a, c, off, va, vb);
        if (NT && a.blocked) {
          const uint32_t o = blocked_cell((brick << 11) | i);
          a.blocked[o] = va;
          a.blocked[n_bricks * kBrickCells + o] = vb;
        } else {
          a.omega[c] = va;
          a.omega[a.n_cells + c] = vb;
        }
        if (a.halo) halo_put_rx(a, r, x, va, vb);
        if (stats) field_sum(sums, na, nb, off);
      }
    }
    if (brick + nblk < n_bricks) __syncthreads();   // s_cnt is reused
  }
  if (!stats) return;
  field_partials(a.partials, blk, sums);
  for (uint32_t i = blk + nblk; i < n_parts; i += nblk)
    if (tid == 0u)
      a.partials->sum_a[i] = a.partials->sum_b[i] = a.partials->n1[i] = a.partials->n2[i] =
          a.partials->nab[i] = 0ull;
}

// Large grids (NT) have bricks enough for narrow blocks.
template <bool NT>
constexpr uint32_t kApplyFieldThreads = NT ? kApplyNarrow : kApplyWide;

template <bool COUNT64, bool NT>
__global__ __launch_bounds__(kApplyFieldThreads<NT>) void apply_field_kernel(
    const BinArgs b, const Grid g, const FieldArgs a, uint32_t n_bricks, uint32_t n_parts) {
  extern __shared__ uint32_t s_cnt[];
  advance_counter(a.ctr, a.ctr_by, blockIdx.x);
  apply_field_bricks<COUNT64, NT, kApplyFieldThreads<NT>>(b, g, a, n_bricks, blockIdx.x, gridDim.x, n_parts, s_cnt);
}

}  // namespace soma

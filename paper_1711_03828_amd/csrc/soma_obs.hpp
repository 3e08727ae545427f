// soma_obs.hpp -- FP64 global reductions: chain observables, energies,
// acceptance counters and the count sums of the last field update.
#pragma once

#include "soma_grid.hpp"

namespace soma {

constexpr uint32_t SOMA_FLAG_POSITION_BIT = 1u;  // a position non-finite or |x| >= 2^22

constexpr uint32_t kObsSums = 5u;   // Re^2, Rg^2, b^2, bond energy, field energy

struct Totals {
  unsigned long long accepted[4];   // local, smart MC, learned, bond-Gibbs
  unsigned long long attempted_learned;
  unsigned long long sum_a, sum_b, n1, n2, nab;   // FieldSums
  double re2, rg2, b2, e_bond, e_field, h_nb;
  uint32_t err, pad;
};

struct ObsArgs {
  const float *pos;
  const float *omega;
  uint32_t n_chains, n, n_a;
  uint32_t lpc;      // lanes per chain: ceil(n / kObsBeads)
  double inv_n;      // 1 / n
  double half_k0;
  double inv_nref;
  Grid grid;
  double *partials;   // [kObsSums][plane], the species' blocks from partials[q * plane]
  uint32_t plane;
  uint32_t *err;
  const ArchDev *arch;   // general architecture (types, bonds), or null: linear chain
};

// Sums over the block's four waves, in thread 0.
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double (*s)[NV]) {
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] += __shfl_down(v[j], off, 64);
  const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6;
  if (lane == 0)
#pragma unroll
    for (int j = 0; j < NV; ++j) s[wv][j] = v[j];
  __syncthreads();
  if (threadIdx.x == 0)
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] = ((s[0][j] + s[1][j]) + s[2][j]) + s[3][j];
}

// Per-chain observables, Eqs. (1)-(2) and (13): Re^2 = |r_{N-1} - r_0|^2,
// Rg^2 = (1/N) sum |r_i - r_cm|^2, sum of squared bond lengths, bond energy
// (k0/2) sum b^2 (over the bond list for a general architecture) and field
// energy sum_i omega_t(c_i) / N.  A wave takes the consecutive chains that fill
// its 64 lanes with kObsBeads beads each (a chain on ceil(N / kObsBeads) lanes):
// their positions, one contiguous range, come through LDS in 16-byte loads, and
// a lane's field values are all in flight together.  Rg^2 comes from the vectors
// d_i = r_i - r_0 in FP64 (differences of FP32 positions, a few cells long) as
// (sum |d|^2 - |sum d|^2 / N) / N, in one pass with one sum over the chain's
// lanes.  FP64 sums per lane, one fixed-order block reduction into a partial per
// block.  Bound by its vector instructions (about 85 a bead, 30 of them FP64):
// 262,144 chains of 32 in 35 us (8 beads
// a lane: 51 us at two waves per SIMD; 2 beads: 46 us); one bead per lane, with a second read of the
// positions for Rg^2 and a sum over 32 lanes for every two chains, took 89.6 us.
constexpr uint32_t kObsBeads = 4u;
constexpr uint32_t kObsMaxBlocks = 1024u;   // per species: four waves per SIMD, all resident

template <bool ARCH>
__global__ __launch_bounds__(256) void chain_obs_kernel(const ObsArgs a) {
  __shared__ double s[4][kObsSums];
  __shared__ float s_pos[4][64u * kObsBeads * 3u];
  const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6, per = 64u / a.lpc;
  const uint32_t slot = lane / a.lpc, k = lane - slot * a.lpc;
  const uint32_t i0 = k * kObsBeads;
  const uint32_t waves = gridDim.x * 4u;
  double re2 = 0, rg = 0, b2 = 0, ef = 0;
  bool bad = false;
  for (uint64_t first = (uint64_t)(blockIdx.x * 4u + wv) * per; first < a.n_chains;
       first += (uint64_t)waves * per) {
    const uint32_t here = (uint32_t)min((uint64_t)per, a.n_chains - first);
    const bool live = slot < here;
    {   // the chains' positions, per * n <= 64 * kObsBeads beads
      const float *src = a.pos + first * a.n * 3u;
      const uint32_t words = here * a.n * 3u, quads = words >> 2;
      float *dst = s_pos[wv];
#pragma unroll
      for (uint32_t u = 0; u < kObsBeads * 3u / 4u; ++u) {
        const uint32_t q = lane + 64u * u;
        if (q < quads) *reinterpret_cast<f32x4_halo *>(dst + 4u * q) =
            *reinterpret_cast<const f32x4_halo *>(src + 4u * q);
      }
      const uint32_t t = 4u * quads + lane;
      if (t < words) dst[t] = src[t];
    }
    wave_lds_fence();
    // beads past the end stand at the chain's first bead, where d = 0
    const float *p = s_pos[wv] + (live ? slot : 0u) * a.n * 3u;
    F3 r[kObsBeads];
#pragma unroll
    for (uint32_t u = 0; u < kObsBeads; ++u) {
      const uint32_t i = i0 + u < a.n ? i0 + u : 0u;
      r[u] = F3{p[3 * i], p[3 * i + 1], p[3 * i + 2]};
    }
    const F3 r0 = {p[0], p[1], p[2]};
    const uint32_t ip = i0 > 0u ? i0 - 1u : 0u;   // the bead before the lane's first
    const F3 prev = {p[3 * ip], p[3 * ip + 1], p[3 * ip + 2]};
    const uint32_t ie = a.n - 1u;
    const F3 re = {p[3 * ie], p[3 * ie + 1], p[3 * ie + 2]};
    float w[kObsBeads];
#pragma unroll
    for (uint32_t u = 0; u < kObsBeads; ++u) {
      const uint32_t i = i0 + u < a.n ? i0 + u : 0u;
      const uint32_t t = ARCH ? (uint32_t)a.arch->type[i] : (i >= a.n_a ? 1u : 0u);
      w[u] = a.omega[(size_t)t * a.grid.n_cells + cell_of(a.grid, r[u].x, r[u].y, r[u].z)];
    }
    const double x0 = r0.x, y0 = r0.y, z0 = r0.z;
    double sx = 0, sy = 0, sz = 0, s2 = 0, bc = 0, ec = 0;
    double px = prev.x - x0, py = prev.y - y0, pz = prev.z - z0;
    bool out = false;
#pragma unroll
    for (uint32_t u = 0; u < kObsBeads; ++u) {
      const uint32_t i = i0 + u;
      out |= !(coord_ok(r[u].x) && coord_ok(r[u].y) && coord_ok(r[u].z));
      const double dx = r[u].x - x0, dy = r[u].y - y0, dz = r[u].z - z0;
      sx += dx; sy += dy; sz += dz;
      s2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, s2)));
      if (!ARCH) {
        const double bx = dx - px, by = dy - py, bz = dz - pz;   // exact: = r_i - r_{i-1}
        const double q = fma(bx, bx, fma(by, by, bz * bz));
        bc += i > 0u && i < a.n ? q : 0.0;
        px = dx; py = dy; pz = dz;
      }
      ec += i < a.n ? (double)w[u] : 0.0;
    }
    if (ARCH && live) {   // each bond once, from its lower-numbered end
      for (uint32_t u = 0; u < kObsBeads && i0 + u < a.n; ++u) {
        const uint32_t i = i0 + u;
        const double x = p[3 * i], y = p[3 * i + 1], z = p[3 * i + 2];
        for (uint32_t q = a.arch->nb_start[i]; q < a.arch->nb_start[i + 1]; ++q) {
          const uint32_t j = a.arch->nb[q];
          if (j < i) continue;
          const double bx = x - p[3 * j], by = y - p[3 * j + 1], bz = z - p[3 * j + 2];
          bc += bx * bx + by * by + bz * bz;
        }
      }
    }
    for (uint32_t off = 1u; off < a.lpc; off <<= 1) {   // sums over the chain's lanes, in its first
      const double tx = __shfl_down(sx, off, 64), ty = __shfl_down(sy, off, 64),
                   tz = __shfl_down(sz, off, 64);
      if (k + off < a.lpc) {
        sx += tx;
        sy += ty;
        sz += tz;
      }
    }
    if (live) {
      bad |= out;
      rg += s2;
      b2 += bc;
      ef += ec;
      if (k == 0u) {
        rg -= (sx * sx + sy * sy + sz * sz) * a.inv_n;
        const double ex = re.x - x0, ey = re.y - y0, ez = re.z - z0;
        re2 += ex * ex + ey * ey + ez * ez;
      }
    }
    wave_lds_fence();   // every lane has read before the next chains come in
  }
  if (bad) atomicOr(a.err, SOMA_FLAG_POSITION_BIT);
  double v[kObsSums] = {re2, rg * a.inv_n, b2, a.half_k0 * b2, ef * a.inv_nref};
  block_sum<kObsSums>(v, s);
  if (threadIdx.x == 0)
#pragma unroll
    for (uint32_t q = 0; q < kObsSums; ++q) a.partials[(size_t)q * a.plane + blockIdx.x] = v[q];
}

// Fixed-order reduction of all partials into one Totals record: one block, one
// wave per quantity (five chain sums, H_nb, five count sums, four acceptance
// counters, the learned attempts).  acc_slots holds kAccSlots counters for each
// of local, smart-MC, learned and bond-Gibbs moves; att_slots the attempted
// learned moves.
constexpr uint32_t kTotalsWaves = 16u;

// Sum of an array over the wave, eight loads in flight.
template <class T>
__device__ __forceinline__ T wave_array_sum(const T *p, uint32_t n) {
  T t = 0;
  for (uint32_t i = threadIdx.x & 63u; i < n; i += 512u) {
    T v[8];
#pragma unroll
    for (uint32_t u = 0; u < 8u; ++u) v[u] = p[min(i + 64u * u, n - 1u)];
#pragma unroll
    for (uint32_t u = 0; u < 8u; ++u) t += i + 64u * u < n ? v[u] : T(0);
  }
  for (int off = 32; off > 0; off >>= 1) t += __shfl_down(t, off, 64);
  return t;
}

__global__ __launch_bounds__(64 * kTotalsWaves) void reduce_totals_kernel(
    const double *op, uint32_t n_op, const FieldPartials *fp, uint32_t n_fp,
    const unsigned long long *acc_slots, const unsigned long long *att_slots,
    const uint32_t *err, Totals *out) {
  const uint32_t q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double d = 0.0;
  unsigned long long n = 0;
  if (q <= kObsSums) {
    d = wave_array_sum(q < kObsSums ? op + (size_t)q * n_op : fp->h_nb, q < kObsSums ? n_op : n_fp);
  } else {
    const bool field = q < 11u;
    const unsigned long long *p = q == 6u ? fp->sum_a : q == 7u ? fp->sum_b : q == 8u ? fp->n1
                                  : q == 9u ? fp->n2 : q == 10u ? fp->nab
                                  : q < 15u ? acc_slots + (q - 11u) * kAccSlots : att_slots;
    n = wave_array_sum(p, field ? n_fp : kAccSlots);
  }
  if ((threadIdx.x & 63u) != 0u) return;
  switch (q) {
    case 0: out->re2 = d; break;
    case 1: out->rg2 = d; break;
    case 2: out->b2 = d; break;
    case 3: out->e_bond = d; break;
    case 4: out->e_field = d; break;
    case 5: out->h_nb = d; break;
    case 6: out->sum_a = n; break;
    case 7: out->sum_b = n; break;
    case 8: out->n1 = n; break;
    case 9: out->n2 = n; break;
    case 10: out->nab = n; break;
    case 15:
      out->attempted_learned = n;
      out->err = *err;
      out->pad = 0;
      break;
    default: out->accepted[q - 11u] = n;
  }
}

}  // namespace soma

// soma_arch.hpp -- general molecular architectures: device tables and the SET
// sweep over arbitrary bond graphs.
#pragma once

#include "soma_sweep.hpp"

namespace soma {

constexpr uint32_t kPurposeSetOrder = 8u; // Philox purpose of the shuffled set order

// Sec. 3.1.2, scheme 2, for any architecture: a wave holds A->per_wave
// molecules (consecutive in the launch's chain subset), each on 64/per_wave
// lanes, their positions staged in LDS; every molecule walks its independent
// sets in its own order for this sweep (two sets: set 1 first iff bit 0 of
// word 0 of monomer 0's move draw, as for linear chains; more: a Fisher-Yates
// shuffle from the purpose-8 blocks; set_order = 1: numerical order), the
// members of a set on the molecule's lanes at once.  A move is the LOCAL move
// of the linear kernel, the bond term summed over the monomer's bond list in
// list order, so a linear chain given as an architecture moves bit for bit as
// in mc_sweep_local_kernel.  A monomer of type t sees field plane t and
// counts in half t & 1 of count plane t >> 1 (any number of types).
template <bool COUNT64>
__global__ __launch_bounds__(256) void mc_sweep_arch_kernel(const SweepArgs a_in,
                                                            const ArchDev *__restrict__ A) {
  __shared__ float s_pos[4][3 * kArchMaxN];
  __shared__ uint8_t s_order[4][64][kArchMaxSets];   // per wave and molecule slot
  const SweepArgs a = resolve_sweep(a_in, 0u);
  const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6;
  const uint32_t N = A->n, k = A->n_sets, M = A->per_wave, L = 64u / M;
  const uint32_t mi = lane / L, li = lane - mi * L;
  const uint32_t wave = xcd_remap(blockIdx.x, gridDim.x) * 4u + wv;
  const uint32_t cl0 = wave * M;                       // first molecule of the wave
  const uint32_t n_here = cl0 < a.n_sub ? min(M, a.n_sub - cl0) : 0u;
  const bool mine = mi < n_here;                       // this lane's molecule exists
  const uint32_t cl = cl0 + mi;
  const uint32_t chain = cl * a.sub_k + a.sub_j;
  const uint32_t gchain = a.chain_base + chain;
  float *sp = s_pos[wv] + 3u * N * mi;                 // this lane's molecule in LDS
  float *cp = a.pos + (size_t)(mine ? chain : 0u) * N * 3u;
  uint32_t n_acc = 0;
  if (n_here > 0) {
    for (uint32_t q = li; q < 3u * N; q += L)
      if (mine) sp[q] = cp[q];
    if (mine && li == 0) {
      uint8_t *ord = s_order[wv][mi];
      for (uint32_t s = 0; s < k; ++s) ord[s] = (uint8_t)s;
      if (a.set_order == 0 && k == 2) {
        const Rand4 d = philox(gchain, 0u, a.sweep, a.replica, a.seed_lo, a.seed_hi);
        if (d.x & 1u) { ord[0] = 1; ord[1] = 0; }
      } else if (a.set_order == 0 && k > 2) {
        Rand4 d = {0u, 0u, 0u, 0u};
        for (uint32_t t = k - 1, st = 0; t >= 1; --t, ++st) {
          if ((st & 3u) == 0u)
            d = philox(gchain, (st >> 2) | (kPurposeSetOrder << 16), a.sweep, a.replica, a.seed_lo,
                       a.seed_hi);
          const uint32_t q = st & 3u;
          const uint32_t word = q == 0u ? d.x : (q == 1u ? d.y : (q == 2u ? d.z : d.w));
          const uint32_t j = __umulhi(word, t + 1u);
          const uint8_t tmp = ord[t];
          ord[t] = ord[j];
          ord[j] = tmp;
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    for (uint32_t s = 0; s < k; ++s) {
      const uint32_t set = mine ? s_order[wv][mi][s] : 0u;
      const uint32_t m0 = A->set_start[set], m1 = A->set_start[set + 1];
      // the wave loops as long as any of its molecules has members left
      uint32_t span = mine ? m1 - m0 : 0u;
      for (uint32_t off = 32u; off >= 1u; off >>= 1) span = max(span, (uint32_t)__shfl_xor((int)span, (int)off, 64));
      for (uint32_t base = 0; base < span; base += L) {
        const uint32_t idx = m0 + base + li;
        bool acc = false;
        if (mine && idx < m1) {
          const uint32_t i = A->member[idx];
          const F3 r = {sp[3 * i], sp[3 * i + 1], sp[3 * i + 2]};
          const Rand4 w = philox(gchain, i | (kPurposeMoveA << 16), a.sweep, a.replica, a.seed_lo,
                                 a.seed_hi);
          const F3 t = {fmaf(a.step, uniform11(w.x), r.x), fmaf(a.step, uniform11(w.y), r.y),
                        fmaf(a.step, uniform11(w.z), r.z)};
          const F3 d = t - r;
          F3 qv = {0.f, 0.f, 0.f};
          for (uint32_t b = A->nb_start[i]; b < A->nb_start[i + 1]; ++b) {
            const uint32_t j = A->nb[b];
            const F3 rj = {sp[3 * j], sp[3 * j + 1], sp[3 * j + 2]};
            qv = qv + (2.0f * (r - rj) + d);
          }
          uint32_t x, y, z;
          cell3(a.grid, r.x, r.y, r.z, x, y, z);
          const uint32_t co = cell_index(a.grid, x, y, z);
          const uint32_t cn = cell_index(a.grid, shift_cell(x, r.x, t.x, a.grid.nx),
                                         shift_cell(y, r.y, t.y, a.grid.ny),
                                         shift_cell(z, r.z, t.z, a.grid.nz));
          const uint32_t ty = A->type[i];
          const uint32_t pl = ty * a.grid.n_cells;          // field plane of the type
          const float wo = field_at(a.omega, pl, co);
          const float wn = cn == co ? wo : field_at(a.omega, pl, cn);
          const float d_e = a.half_k0 * (d.x * qv.x + d.y * qv.y + d.z * qv.z) + (wn - wo) * a.inv_nref;
          acc = move_allowed(a, co, cn) && (d_e <= 0.0f || uniform01(w.w) < __expf(-d_e));
          if (acc) {
            sp[3 * i] = t.x;
            sp[3 * i + 1] = t.y;
            sp[3 * i + 2] = t.z;
            if (cn != co) {   // count plane ty >> 1, half ty & 1
              const uint32_t pw = (ty >> 1) * a.grid.n_cells;
              move_count<COUNT64>(a.counts, co + pw, cn + pw, (ty & 1u) != 0u);
            }
          }
        }
        n_acc += (uint32_t)__popcll(__ballot(acc));
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
    for (uint32_t q = li; q < 3u * N; q += L)
      if (mine) cp[q] = sp[q];
  }
  finish_block(a, n_acc);
}

// Sum of bond_term over the monomer's bonds in list order (record rec, positions of
// its molecule at sp), two partners per step.
__device__ __forceinline__ F3 pair_bonds(const float4 *sp, uint4 rec, F3 r, F3 d) {
  const uint32_t n = (rec.x >> 16) & 0x7Fu;
  F3 q = {0.f, 0.f, 0.f};
  uint32_t w = (rec.x >> 24) | (rec.y << 8);   // the next four partners
  uint32_t w1 = __builtin_amdgcn_alignbyte(rec.z, rec.y, 3u), w2 = __builtin_amdgcn_alignbyte(rec.w, rec.z, 3u);
  uint32_t w3 = rec.w >> 24;
#pragma unroll 1
  for (uint32_t b = 0; b < n; b += 2u) {
    const float4 p0 = sp[w & 0xFFu], p1 = sp[(w >> 8) & 0xFFu];
    q = q + bond_term(r, F3{p0.x, p0.y, p0.z}, d);
    const F3 q1 = q + bond_term(r, F3{p1.x, p1.y, p1.z}, d);
    q = sel(b + 1u < n, q1, q);
    w = __builtin_amdgcn_alignbyte(w1, w, 2u);
    w1 = __builtin_amdgcn_alignbyte(w2, w1, 2u);
    w2 = __builtin_amdgcn_alignbyte(w3, w2, 2u);
    w3 >>= 16;
  }
  return q;
}

// The same moves for architectures of at most two independent sets (linear chains,
// stars, combs, even rings; at most 64 members per set and kArchRecBonds bonds per
// monomer), as local_tile: a molecule's lane l holds member l of either set, whose
// draws, cells and field gathers are independent of the other set and go first; the
// two are relabelled by the molecule's set order, and only bond terms and outcomes
// wait for the set before, through LDS.  8.4M monomers in six-armed stars of three
// types on 96^3 cells: 94.5 us, mc_sweep_arch_kernel 165.6; bound by its vector
// instructions (the bond loop runs as long as the hub's list in both passes) and the
// count atomics, which the bins do not shorten here (100.6 us and 12 to apply them).
// per_wave molecules per wave on `lanes` lanes each; inv_lanes = floor(65536 / lanes) + 1.
template <bool COUNT64>
__global__ __launch_bounds__(256) void mc_sweep_pair_kernel(
    const SweepArgs a_in, const ArchDev *__restrict__ A, uint32_t per_wave, uint32_t lanes,
    uint32_t inv_lanes) {
  __shared__ float4 s_pos[4][kArchMaxN];
  const SweepArgs a = resolve_sweep(a_in, 0u);
  const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6;
  const uint32_t mi = (lane * inv_lanes) >> 16, li = lane - mi * lanes;
  const uint32_t cl = (xcd_remap(blockIdx.x, gridDim.x) * 4u + wv) * per_wave + mi;
  const bool mine = mi < per_wave && cl < a.n_sub;   // this lane's molecule exists
  const uint32_t chain = mine ? cl * a.sub_k + a.sub_j : 0u, gchain = a.chain_base + chain;
  const uint4 *rec = reinterpret_cast<const uint4 *>(A->rec[0]) + li;
  const uint4 rec0 = rec[0], rec1 = rec[64];
  const uint32_t i0 = rec0.x & 0xFFu, i1 = rec1.x & 0xFFu;
  float *cp = a.pos + (size_t)chain * a.n * 3u;
  f32x3_bead *p0 = reinterpret_cast<f32x3_bead *>(cp + 3u * i0);
  f32x3_bead *p1 = reinterpret_cast<f32x3_bead *>(cp + 3u * i1);
  const F3 r0 = (F3)*p0, r1 = (F3)*p1;
  const Rand4 w0 = philox(gchain, i0 | (kPurposeMoveA << 16), a.sweep, a.replica, a.seed_lo, a.seed_hi);
  const Rand4 w1 = philox(gchain, i1 | (kPurposeMoveA << 16), a.sweep, a.replica, a.seed_lo, a.seed_hi);
  // monomer 0 is the first member of set 0
  const uint32_t bit = (uint32_t)__builtin_amdgcn_ds_bpermute((int)((lane - li) << 2), (int)(w0.x & 1u));
  const bool odd = a.set_order == 0u && bit != 0u;
  const bool has0 = mine && (rec0.x & 0x800000u) != 0u, has1 = mine && (rec1.x & 0x800000u) != 0u;
  const bool has_a = odd ? has1 : has0, has_b = odd ? has0 : has1;
  const Rand4 wa = odd ? w1 : w0, wb = odd ? w0 : w1;
  const uint4 ka = odd ? rec1 : rec0, kb = odd ? rec0 : rec1;
  float4 *sp = s_pos[wv] + (mine ? mi : 0u) * a.n;
  if (has0) sp[i0] = make_float4(r0.x, r0.y, r0.z, 0.f);
  if (has1) sp[i1] = make_float4(r1.x, r1.y, r1.z, 0.f);
  Trial X, Y;
  X.r = sel(odd, r1, r0);
  Y.r = sel(odd, r0, r1);
  const uint32_t ta = (ka.x >> 8) & 0xFFu, tb = (kb.x >> 8) & 0xFFu;   // types: field planes
  const uint32_t pla = ta * a.grid.n_cells, plb = tb * a.grid.n_cells;
  trial_from(a, pla, X);
  trial_from(a, plb, Y);
  trial_to(a, wa, X);
  trial_to(a, wb, Y);
  trial_gather(a, pla, X, plb, Y);
  const bool ok_a = has_a & move_allowed(a, X.c, X.n), ok_b = has_b & move_allowed(a, Y.c, Y.n);
  wave_lds_fence();
  F3 ra = X.r, rb = Y.r;
  bool acc_a, acc_b;
  {
    const F3 d = X.t - X.r, q = pair_bonds(sp, ka, X.r, d);
    const float d_e = a.half_k0 * (d.x * q.x + d.y * q.y + d.z * q.z) + (X.wn - X.wo) * a.inv_nref;
    acc_a = ok_a & metropolis(d_e, uniform01(wa.w));
    ra = acc_a ? X.t : ra;
    if (acc_a) sp[ka.x & 0xFFu] = make_float4(ra.x, ra.y, ra.z, 0.f);
  }
  wave_lds_fence();
  {
    const F3 d = Y.t - Y.r, q = pair_bonds(sp, kb, Y.r, d);
    const float d_e = a.half_k0 * (d.x * q.x + d.y * q.y + d.z * q.z) + (Y.wn - Y.wo) * a.inv_nref;
    acc_b = ok_b & metropolis(d_e, uniform01(wb.w));
    rb = acc_b ? Y.t : rb;
  }
  const F3 o0 = sel(odd, rb, ra), o1 = sel(odd, ra, rb);
  if (has0) *p0 = f32x3_bead{o0.x, o0.y, o0.z};
  if (has1) *p1 = f32x3_bead{o1.x, o1.y, o1.z};
  // count plane type >> 1, half type & 1
  const uint32_t ca = (ta >> 1) * a.grid.n_cells, cb = (tb >> 1) * a.grid.n_cells;
  if (acc_a & (X.n != X.c)) move_count<COUNT64>(a.counts, X.c + ca, X.n + ca, (ta & 1u) != 0u);
  if (acc_b & (Y.n != Y.c)) move_count<COUNT64>(a.counts, Y.c + cb, Y.n + cb, (tb & 1u) != 0u);
  finish_block(a, (uint32_t)(__popcll(__ballot(acc_a)) + __popcll(__ballot(acc_b))));
}

}  // namespace soma

// soma_bins.hpp -- the occupation histogram (Eq. (4), Sec. 3.1.1) kept current
// through per-brick bins of count updates instead of one memory-side atomic
// per update.
//
// The grid is cut into bricks of 16 x 16 x 8 cells.  A block that moves beads
// to other cells counts its +-1 updates per brick in a small LDS table,
// reserves room in each brick's bin with one atomic per (block, brick) and
// writes the updates there with plain stores (the waves of a persistent grid,
// which run different numbers of tiles, do so wave by wave); a bin that is full takes the
// rest as direct atomics on the counts.  Afterwards `bin_apply_kernel` gives
// every brick one workgroup: the brick's count words go to LDS, the bin's
// updates are added with LDS atomics, and the words go back.  Integer additions are exact and
// order-independent, so the counts are bit-identical to direct atomics (and
// to a recount of the final positions).
//
// An update is 16 bits: bit 15 present, bit 14 minus (-1, else +1), bits
// 11..13 the bead type, bits 0..10 the cell inside the brick
// ((z & 7) * 16 + (y & 15)) * 16 + (x & 15).  A bin entry holds two updates
// (low and high half), typically the -1 at the old cell and the +1 at the new
// cell of one bead; a half with bit 15 clear is empty.
#pragma once

#include "soma_device.hpp"

namespace soma {

constexpr uint32_t kBrickCells = 2048u;      // 16 x 16 x 8
constexpr uint32_t kHistDirect = 0u;         // one atomic per update
constexpr uint32_t kHistBinned = 1u;         // per-brick bins, applied by bin_apply_kernel
constexpr uint32_t kHistAuto = 2u;           // sweep by sweep, whichever is expected to be faster
constexpr uint32_t kUpdPresent = 0x8000u;
constexpr uint32_t kUpdMinus = 0x4000u;

// Every brick has 1 << sub_shift sub-bins; a block (or wave) appends to the one of
// its index, so that those working on one region of the grid at the same time
// (they share its bricks) spread their reservations over different counters
// instead of queueing on one (a returning atomic on one address takes about 100
// ns at the memory side).  16 sub-bins on grids of fewer than kFewBricks bricks,
// whose counters are few; 8 on larger ones, where the entries of a brick then lie
// in fewer lines (134M-bead melt, 13,824 bricks: 40 us less per sweep than with 16;
// a batch of small melts: 323 against 292 us the other way round).  Between 700 and
// 3,000 bricks a cycle takes the same either way within 3%, and there the line is
// that of the recount, which the blocks of bin_apply_kernel decide (kApplyOnlyWide).
constexpr uint32_t kMaxSubShift = 4u, kFewBricks = 2048u;

struct BinArgs {
  uint32_t *bins;        // [n_bricks][1 << sub_shift][cap] entries
  uint32_t *bin_count;   // [n_bricks][1 << sub_shift] entries written (beyond cap: went direct)
  uint32_t cap;          // entries per sub-bin
  uint32_t sub_shift;
  uint32_t nbx, nby, nbz;
};

// Sub-bin of the calling block, and of the calling wave (wpb waves per block).
// Blocks that work on one region are either consecutive (no remapping) or eight
// apart (one XCD's contiguous range); b + floor(b / 8) runs through every residue
// in both cases.  (b mod 16 alone gives an XCD's blocks two of the 16 sub-bins,
// which fill up and send the rest to direct atomics.)
__device__ __forceinline__ uint32_t block_sub_bin(const BinArgs &b) {
  return (blockIdx.x + (blockIdx.x >> 3)) & ((1u << b.sub_shift) - 1u);
}
__device__ __forceinline__ uint32_t wave_sub_bin(const BinArgs &b, uint32_t wpb) {
  return ((blockIdx.x + (blockIdx.x >> 3)) * wpb + (threadIdx.x >> 6)) & ((1u << b.sub_shift) - 1u);
}

// Brick key of cell (x, y, z): brick index << 11 | cell inside the brick.
__device__ __forceinline__ uint32_t brick_key(const BinArgs &b, uint32_t x, uint32_t y,
                                              uint32_t z) {
  const uint32_t brick = __umul24(__umul24(z >> 3, b.nby) + (y >> 4), b.nbx) + (x >> 4);
  return (brick << 11) | ((z & 7u) << 8) | ((y & 15u) << 4) | (x & 15u);
}

// Place of the cell with this brick key in a blocked field plane (n_bricks x 2048
// floats): the key with the cell's bits reordered to z2 z1 y3 y2 x3 x2 z0 y1 y0 x1 x0,
// so that a 128-byte line holds 4 x 4 x 2 cells instead of 32 of one row.
__device__ __forceinline__ uint32_t blocked_cell(uint32_t key) {
  return (key & ~0x1FCu) | ((key & 0x0C0u) << 1) | ((key & 0x00Cu) << 3) | ((key & 0x100u) >> 4) |
         ((key & 0x030u) >> 2);
}

// q = floor(c / d) for c < 2^29: an FP32 estimate, refined once with the
// exact remainder (|error| of the estimate far below 2^23), then fixed by one.
__device__ __forceinline__ uint32_t div_small(uint32_t c, uint32_t d, float inv_d) {
  int q = (int)((float)c * inv_d);
  int r = (int)c - q * (int)d;
  q += (int)floorf((float)r * inv_d);
  r = (int)c - q * (int)d;
  q += r >= (int)d ? 1 : (r < 0 ? -1 : 0);
  return (uint32_t)q;
}

// Brick key of the linear cell c = (z ny + y) nx + x.
__device__ __forceinline__ uint32_t cell_brick_key(const BinArgs &b, const Grid &g, uint32_t c) {
  const uint32_t yz = div_small(c, (uint32_t)g.nx, g.inv_nx);
  const uint32_t x = c - yz * (uint32_t)g.nx;
  const uint32_t z = div_small(yz, (uint32_t)g.ny, g.inv_ny);
  const uint32_t y = yz - z * (uint32_t)g.ny;
  return brick_key(b, x, y, z);
}

// Linear cell index of the cell inside brick `brick` at `local` (slow path only).
__device__ __forceinline__ uint32_t brick_cell(const BinArgs &b, const Grid &g, uint32_t brick,
                                               uint32_t local) {
  const uint32_t bx = brick % b.nbx, rest = brick / b.nbx;
  const uint32_t by = rest % b.nby, bz = rest / b.nby;
  const uint32_t x = bx * 16u + (local & 15u), y = by * 16u + ((local >> 4) & 15u),
                 z = bz * 8u + (local >> 8);
  return (z * (uint32_t)g.ny + y) * (uint32_t)g.nx + x;
}

// One update applied directly to the packed counts (the overflow path).
template <bool COUNT64>
__device__ __forceinline__ void apply_update_direct(void *counts, uint32_t n_cells, uint32_t cell,
                                                    uint32_t upd) {
  const uint32_t t = (upd >> 11) & 7u;
  const bool minus = (upd & kUpdMinus) != 0u;
  const size_t w = (size_t)(t >> 1) * n_cells + cell;
  if (COUNT64) {
    unsigned int *p = reinterpret_cast<unsigned int *>(counts) + 2 * w + (t & 1u);
    atomicAdd(p, minus ? 0xFFFFFFFFu : 1u);
  } else {
    const unsigned int inc = (t & 1u) ? (1u << 16) : 1u;
    atomicAdd(reinterpret_cast<unsigned int *>(counts) + w, minus ? 0u - inc : inc);
  }
}

template <bool COUNT64>
__device__ __forceinline__ void apply_entry_direct(const BinArgs &b, const Grid &g, void *counts,
                                                   uint32_t key, uint32_t entry) {
  const uint32_t brick = key;
  for (int h = 0; h < 2; ++h) {
    const uint32_t upd = (entry >> (16 * h)) & 0xFFFFu;
    if (upd & kUpdPresent)
      apply_update_direct<COUNT64>(counts, g.n_cells, brick_cell(b, g, brick, upd & 2047u), upd);
  }
}

// Table of the bricks that a block's (or a wave's) updates fall in: SLOTS slots
// of {brick, count} in LDS, open addressing with linear probing.
constexpr uint32_t kWaveSlots = 32u, kBlockSlots = 256u;
constexpr uint32_t kTabEmpty = 0xFFFFFFFFu;   // no brick (brick indices are below 2^21)
constexpr uint32_t kNoSlot = 0xFFFFu;

// Slot of `brick` in the table (claimed if new) << 16 | the entry's rank among
// the table's entries for that brick; kNoSlot << 16 if kMaxProbe slots are taken
// by other bricks (chains scattered over more bricks than the table is for).
constexpr uint32_t kMaxProbe = 32u;

template <uint32_t SLOTS>
__device__ __forceinline__ uint32_t tab_insert(uint2 *tab, uint32_t brick) {
  uint32_t h = (__umul24(brick, 0x9E3779u) >> 11) & (SLOTS - 1u);
  uint32_t probe = 0;
#pragma unroll 1
  for (; probe < kMaxProbe; ++probe) {
    const uint32_t old = atomicCAS(&tab[h].x, kTabEmpty, brick);
    if (old == kTabEmpty || old == brick) break;
    h = (h + 1u) & (SLOTS - 1u);
  }
  if (probe == kMaxProbe) return kNoSlot << 16;
  return (h << 16) | atomicAdd(&tab[h].y, 1u);
}

// Stores entry v (brick k, table slot and rank q) at its reserved place, or
// applies it directly if its sub-bin is full or the wave's table was.
template <bool COUNT64>
__device__ __forceinline__ void tab_put(const BinArgs &b, const Grid &g, void *counts,
                                        const uint2 *tab, uint32_t sub, uint32_t k, uint32_t q,
                                        uint32_t v) {
  const uint32_t h = q >> 16;
  const uint32_t pos = h != kNoSlot ? tab[h].y + (q & 0xFFFFu) : 0xFFFFFFFFu;
  if (pos < b.cap) b.bins[(size_t)((k << b.sub_shift) | sub) * b.cap + pos] = v;
  else apply_entry_direct<COUNT64>(b, g, counts, k, v);
}

// Set bits of mask m in the lanes below the calling one.
__device__ __forceinline__ uint32_t mbcnt64(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Up to four entries of each lane (slot s: brick ks, value vs, wanted if bit s of
// `want`), packed into the wave's LDS list (slot 0 of every lane, then slot 1,
// ...): entry lane + 64 p of the list in e[p].  So the steps that follow run once
// per 64 entries with every lane busy, rather than once per slot with the few
// lanes whose bead changed cell.  LDS operations of one wave execute in issue
// order, so the list needs no barrier.
constexpr uint32_t kListSlots = 4u * 64u;

struct BinEntries {
  uint2 e[4];      // {brick, value}
  uint32_t q[4];   // table slot << 16 | rank
  uint32_t n;      // entries of the wave
};

__device__ __forceinline__ BinEntries pack_entries(uint2 *list, uint32_t k0, uint32_t k1, uint32_t k2,
                                                   uint32_t k3, uint32_t v0, uint32_t v1, uint32_t v2,
                                                   uint32_t v3, uint32_t want) {
  const uint32_t lane = __lane_id();
  const uint64_t m0 = __ballot((want & 1u) != 0u), m1 = __ballot((want & 2u) != 0u);
  const uint64_t m2 = __ballot((want & 4u) != 0u), m3 = __ballot((want & 8u) != 0u);
  const uint32_t o1 = (uint32_t)__popcll(m0), o2 = o1 + (uint32_t)__popcll(m1);
  const uint32_t o3 = o2 + (uint32_t)__popcll(m2);
  BinEntries b;
  b.n = o3 + (uint32_t)__popcll(m3);
  if (want & 1u) list[mbcnt64(m0)] = make_uint2(k0, v0);
  if (want & 2u) list[o1 + mbcnt64(m1)] = make_uint2(k1, v1);
  if (want & 4u) list[o2 + mbcnt64(m2)] = make_uint2(k2, v2);
  if (want & 8u) list[o3 + mbcnt64(m3)] = make_uint2(k3, v3);
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (uint32_t p = 0; p < 4u; ++p) {
    b.e[p] = make_uint2(0u, 0u);
    b.q[p] = 0u;
    if (64u * p < b.n && 64u * p + lane < b.n) b.e[p] = list[64u * p + lane];
  }
  return b;
}

template <uint32_t SLOTS>
__device__ __forceinline__ void insert_entries(uint2 *tab, BinEntries &b) {
  const uint32_t lane = __lane_id();
#pragma unroll
  for (uint32_t p = 0; p < 4u; ++p)
    if (64u * p < b.n && 64u * p + lane < b.n) b.q[p] = tab_insert<SLOTS>(tab, b.e[p].x);
}

// One reservation per brick of the table; the slot keeps its base.
__device__ __forceinline__ void reserve_slot(const BinArgs &b, uint2 *slot, uint32_t sub) {
  const uint2 t = *slot;
  if (t.x != kTabEmpty) slot->y = atomicAdd(b.bin_count + ((t.x << b.sub_shift) | sub), t.y);
}

template <bool COUNT64>
__device__ __forceinline__ void put_entries(const BinArgs &b, const Grid &g, void *counts,
                                            const uint2 *tab, uint32_t sub, const BinEntries &n) {
  const uint32_t lane = __lane_id();
#pragma unroll
  for (uint32_t p = 0; p < 4u; ++p)
    if (64u * p < n.n && 64u * p + lane < n.n)
      tab_put<COUNT64>(b, g, counts, tab, sub, n.e[p].x, n.q[p], n.e[p].y);
}

// LDS of the binned count updates of a block of up to WAVES waves.  WAVEWISE:
// tables per wave (persistent grids), else one for the block.
template <uint32_t WAVES, bool WAVEWISE>
struct BinLds {
  uint2 tab[WAVEWISE ? WAVES * kWaveSlots : kBlockSlots];
  uint2 list[WAVES * kListSlots];
};

// Empties the block's table; before the first append, with nothing of an
// earlier one outstanding.  Waves start together here, so the barrier is cheap.
template <uint32_t WAVES, bool WAVEWISE>
__device__ __forceinline__ void bins_begin(BinLds<WAVES, WAVEWISE> &s) {
  if (WAVEWISE) return;
  for (uint32_t i = threadIdx.x; i < kBlockSlots; i += blockDim.x) s.tab[i] = make_uint2(kTabEmpty, 0u);
  __syncthreads();
}

// Appends entries to their bricks' bins: they are counted per brick in the table
// (the rank of an entry is its place among the table's entries for its brick),
// one lane per brick reserves that many places in the brick's sub-bin with one
// atomic, and every entry is stored at reserved base + rank.  Every lane of the
// wave, and of the block unless WAVEWISE, calls this together, once per
// bins_begin.  The 8 waves of a 512-thread block work on neighbouring chains and
// share most of their bricks: with one reservation per (block, brick) instead of
// one per (wave, brick) the binned local sweep of the 134M-bead melt takes 1112 us
// (was 1237), of 8.4M beads on 96^3 cells 58 us (101), of a 16M-bead film, whose
// few bricks make the counters few, 132 us (280).
template <bool COUNT64, uint32_t WAVES, bool WAVEWISE>
__device__ __forceinline__ void bin_append(BinLds<WAVES, WAVEWISE> &s, const BinArgs &b, const Grid &g,
                                           void *counts, uint32_t wpb, uint32_t k0, uint32_t k1,
                                           uint32_t k2, uint32_t k3, uint32_t v0, uint32_t v1,
                                           uint32_t v2, uint32_t v3, uint32_t want) {
  const uint32_t lane = __lane_id(), wv = threadIdx.x >> 6;
  uint2 *list = s.list + wv * kListSlots;
  if (WAVEWISE) {
    uint2 *tab = s.tab + wv * kWaveSlots;
    const uint32_t sub = wave_sub_bin(b, wpb);
    if (lane < kWaveSlots) tab[lane] = make_uint2(kTabEmpty, 0u);
    BinEntries n = pack_entries(list, k0, k1, k2, k3, v0, v1, v2, v3, want);
    insert_entries<kWaveSlots>(tab, n);
    __builtin_amdgcn_wave_barrier();
    if (lane < kWaveSlots) reserve_slot(b, tab + lane, sub);
    __builtin_amdgcn_wave_barrier();
    put_entries<COUNT64>(b, g, counts, tab, sub, n);
    __builtin_amdgcn_wave_barrier();
    return;
  }
  const uint32_t sub = block_sub_bin(b);
  BinEntries n = pack_entries(list, k0, k1, k2, k3, v0, v1, v2, v3, want);
  insert_entries<kBlockSlots>(s.tab, n);
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < kBlockSlots; i += blockDim.x) reserve_slot(b, s.tab + i, sub);
  __syncthreads();
  put_entries<COUNT64>(b, g, counts, s.tab, sub, n);
}

// The count updates of a lane's two beads (bead e moved from the cell with
// brick key from[e] to to[e] if moved[e]; t[e] its type), as bin entries: one
// when both cells lie in one brick, else one per brick.
template <bool COUNT64, uint32_t WAVES, bool WAVEWISE>
__device__ __forceinline__ void bin_moves(BinLds<WAVES, WAVEWISE> &s, const BinArgs &b, const Grid &g,
                                          void *counts, uint32_t wpb, uint32_t from0, uint32_t to0,
                                          uint32_t t0, bool moved0, uint32_t from1, uint32_t to1,
                                          uint32_t t1, bool moved1) {
  const uint32_t hm0 = kUpdPresent | kUpdMinus | (t0 << 11) | (from0 & 2047u);
  const uint32_t hp0 = kUpdPresent | (t0 << 11) | (to0 & 2047u);
  const uint32_t hm1 = kUpdPresent | kUpdMinus | (t1 << 11) | (from1 & 2047u);
  const uint32_t hp1 = kUpdPresent | (t1 << 11) | (to1 & 2047u);
  const bool same0 = (from0 >> 11) == (to0 >> 11), same1 = (from1 >> 11) == (to1 >> 11);
  const uint32_t want = (moved0 ? (same0 ? 1u : 3u) : 0u) | (moved1 ? (same1 ? 4u : 12u) : 0u);
  bin_append<COUNT64>(s, b, g, counts, wpb, from0 >> 11, to0 >> 11, from1 >> 11, to1 >> 11,
                      same0 ? (hm0 | (hp0 << 16)) : hm0, hp0 << 16,
                      same1 ? (hm1 | (hp1 << 16)) : hm1, hp1 << 16, want);
}

// From-scratch histogram through the bins (counts cleared before): species s owns
// the blocks [first[s], first[s + 1]), and lane q of them takes its beads 2q and 2q+1
// (one entry when both lie in one brick), so that a block of 512 consecutive beads
// reserves room once per brick it touches.  Positions are read as three
// 8-byte pairs where `vec2` (8-byte aligned species start).  One launch for all
// species: three of 3.0M, 0.7M and 0.7M beads take 30.4 us, 38.4 in launches of their
// own, and two gaps less.
constexpr uint32_t kHistSpecies = 8u;
struct HistSpecies {
  const float *pos;
  const ArchDev *arch;
  uint64_t n_beads;
  uint32_t n, n_a, vec2, first;
};
struct HistArgs {
  HistSpecies sp[kHistSpecies];   // of n_species used; `first` ascending
  uint32_t n_species;
};

template <bool COUNT64>
__global__ __launch_bounds__(256) void density_hist_binned_kernel(const HistArgs h, Grid g,
                                                                  void *counts, BinArgs b) {
  __shared__ BinLds<4u, false> s_bin;
  bins_begin(s_bin);
  uint32_t sp = 0;
  for (uint32_t k = 1; k < h.n_species; ++k) sp = blockIdx.x >= h.sp[k].first ? k : sp;
  const HistSpecies &S = h.sp[sp];
  const float *pos = S.pos;
  const ArchDev *arch = S.arch;
  const uint64_t n_beads = S.n_beads;
  const uint32_t n = S.n, n_a = S.n_a, vec2 = S.vec2;
  const uint64_t q = (uint64_t)(blockIdx.x - S.first) * blockDim.x + threadIdx.x;
  const uint64_t i0 = 2 * q, i1 = 2 * q + 1;
  const bool has0 = i0 < n_beads, has1 = i1 < n_beads;
  float r[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (has1 && vec2) {
    const float2 *p2 = reinterpret_cast<const float2 *>(pos + 3 * i0);
    const float2 a = p2[0], c = p2[1], d = p2[2];
    r[0] = a.x; r[1] = a.y; r[2] = c.x; r[3] = c.y; r[4] = d.x; r[5] = d.y;
  } else {
    if (has0) { r[0] = pos[3 * i0]; r[1] = pos[3 * i0 + 1]; r[2] = pos[3 * i0 + 2]; }
    if (has1) { r[3] = pos[3 * i1]; r[4] = pos[3 * i1 + 1]; r[5] = pos[3 * i1 + 2]; }
  }
  uint32_t x0, y0, z0, x1, y1, z1;
  cell3(g, r[0], r[1], r[2], x0, y0, z0);
  cell3(g, r[3], r[4], r[5], x1, y1, z1);
  const uint32_t k0 = brick_key(b, x0, y0, z0), k1 = brick_key(b, x1, y1, z1);
  const uint32_t j0 = n_beads <= 0xFFFFFFFFull ? (uint32_t)i0 % n : (uint32_t)(i0 % n);
  const uint32_t j1 = j0 + 1u == n ? 0u : j0 + 1u;
  const uint32_t t0 = bead_type(arch, j0, n_a), t1 = bead_type(arch, j1, n_a);
  const uint32_t h0 = kUpdPresent | (t0 << 11) | (k0 & 2047u);
  const uint32_t h1 = kUpdPresent | (t1 << 11) | (k1 & 2047u);
  const bool same = (k0 >> 11) == (k1 >> 11);
  uint32_t want = 0u;
  if (has0) want |= 1u;
  if (has1) want |= same ? 0u : 2u;
  const uint32_t v0 = (has1 && same) ? (h0 | (h1 << 16)) : h0;
  const uint32_t v1 = h1 << 16;
  // a lane without bead 2q has only bead 2q+1 absent too (n_beads is the end)
  bin_append<COUNT64>(s_bin, b, g, counts, 4u, k0 >> 11, k1 >> 11, 0u, 0u, v0, v1, 0u, 0u, want);
}

// Applies the bins to the counts: one workgroup of THREADS per brick.
// The brick's count words (every plane) are staged in LDS, the bin's updates
// added with LDS atomics, the words written back, and the bin emptied for the
// next sweep.  The sub-bins' fill levels load together with the counts, and
// the entries of two sub-bins are taken as one flat index range, kApplyBatch
// independent loads per thread at a time, so that a block waits on memory a few times
// rather than twice per sub-bin.
// Where the bricks are few and every round trip counts, 512 threads with the fields
// (a film of 450 bricks: 9.9 us, 9.8 with 1024; 131x97x88 cells, 693 bricks: 18.4 and
// 28.5) and 1024 without them, mostly a recount, whose bins are full (420 bricks,
// before the entries were taken pairwise: 15.8 us, 17.0 with 512; now 12.3); 256
// where there are enough bricks to fill the device (13,824: 152 us, 157 with 512;
// whole recounts with 16 sub-bins and 1024 threads against 8 and 256: 432 bricks 35 /
// 45 us, 1,000 60 / 63, 1,440 82 / 83, 2,028 114 / 111, 2,688 147 / 143).
// LDS: planes x 2048 words (u16 pairs) or 2 x planes x 2048 halves (u32 pairs).
constexpr uint32_t kApplyOnlyWide = 1024u, kApplyWide = 512u, kApplyNarrow = 256u;
// Entries that a thread has in flight (narrow blocks have more to take: 134M beads 152
// us with six, 156 with four).
template <uint32_t THREADS>
constexpr uint32_t kApplyBatch = THREADS < kApplyWide ? 6u : 4u;

template <bool COUNT64>
__device__ __forceinline__ void apply_entry_lds(uint32_t *s_cnt, uint32_t planes, uint32_t e) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t upd = (e >> (16 * h)) & 0xFFFFu;
    const uint32_t t = (upd >> 11) & 7u;
    if ((upd & kUpdPresent) && (t >> 1) < planes) {
      const uint32_t i = (t >> 1) * kBrickCells + (upd & 2047u);
      const bool minus = (upd & kUpdMinus) != 0u;
      if (COUNT64) {
        atomicAdd(&s_cnt[i * 2 + (t & 1u)], minus ? 0xFFFFFFFFu : 1u);
      } else {
        const uint32_t inc = (t & 1u) ? (1u << 16) : 1u;
        atomicAdd(&s_cnt[i], minus ? 0u - inc : inc);
      }
    }
  }
}

// Origin of a brick.
__device__ __forceinline__ void brick_origin(const BinArgs &b, uint32_t brick, uint32_t &x0,
                                             uint32_t &y0, uint32_t &z0) {
  const uint32_t bx = brick % b.nbx, rest = brick / b.nbx;
  const uint32_t by = rest % b.nby, bz = rest / b.nby;
  x0 = bx * 16u;
  y0 = by * 16u;
  z0 = bz * 8u;
}

// The brick's counts with its bin's updates added, in LDS (s_cnt), and the bin
// emptied; ends with a barrier.  Cell l = tid + u THREADS of the brick is
// (x0 + (l & 15), y0 + ((l >> 4) & 15), z0 + (l >> 8)).
// NT: counts and entries are read with the non-temporal hint.
template <bool NT, class T>
__device__ __forceinline__ T load_hint(const T *p) {
  return NT ? __builtin_nontemporal_load(p) : *p;
}

template <bool COUNT64, uint32_t THREADS, bool NT = false>
__device__ __forceinline__ void bin_gather_brick(const BinArgs &b, const Grid &g, const void *counts,
                                                 uint32_t planes, uint32_t brick, uint32_t *s_cnt) {
  // Two neighbouring sub-bins to a group of threads (a wave in blocks of 512 with 16
  // sub-bins and of 256 with 8): entry j of the pair lies at j or, in the second one,
  // cap - n0 further.  A flat index over all sub-bins of the brick costs a search per
  // entry: a film's apply and field kernel 11.9 -> 9.5 us, that of 24 melts 17.0 -> 12.0,
  // 1M bond-Gibbs moves on 96^3 cells 10.9 -> 10.3.
  const uint32_t tid = threadIdx.x, n_sub = 1u << b.sub_shift;
  const uint32_t shift = (uint32_t)__builtin_ctz(THREADS) + 1u - b.sub_shift, group = 1u << shift;
  const uint32_t sb = (tid >> shift) * 2u, l = tid & (group - 1u);
  const uint32_t *bin = b.bins + (size_t)((brick << b.sub_shift) | sb) * b.cap;
  const uint2 fill = *reinterpret_cast<const uint2 *>(b.bin_count + ((brick << b.sub_shift) | sb));
  uint32_t x0, y0, z0;
  brick_origin(b, brick, x0, y0, z0);
  const uint32_t x = x0 + (tid & 15u), y = y0 + ((tid >> 4) & 15u);
  constexpr uint32_t kPer = kBrickCells / THREADS;   // cells per thread and plane
  for (uint32_t p = 0; p < planes; ++p) {
    uint2 v[kPer];
#pragma unroll
    for (uint32_t u = 0; u < kPer; ++u) {
      const uint32_t z = z0 + ((tid + u * THREADS) >> 8);
      v[u] = make_uint2(0u, 0u);
      if (x < (uint32_t)g.nx && y < (uint32_t)g.ny && z < (uint32_t)g.nz) {
        const size_t w = (size_t)p * g.n_cells + ((size_t)z * g.ny + y) * g.nx + x;
        if (COUNT64) {
          const unsigned long long q = load_hint<NT>(reinterpret_cast<const unsigned long long *>(counts) + w);
          v[u] = make_uint2((uint32_t)q, (uint32_t)(q >> 32));
        } else {
          v[u].x = load_hint<NT>(reinterpret_cast<const uint32_t *>(counts) + w);
        }
      }
    }
#pragma unroll
    for (uint32_t u = 0; u < kPer; ++u) {
      const uint32_t i = p * kBrickCells + tid + u * THREADS;
      if (COUNT64) reinterpret_cast<uint2 *>(s_cnt)[i] = v[u];
      else s_cnt[i] = v[u].x;
    }
  }
  const uint32_t n0 = min(fill.x, b.cap), n = n0 + min(fill.y, b.cap), skip = b.cap - n0;
  __syncthreads();
  for (uint32_t j0 = l; j0 < n; j0 += kApplyBatch<THREADS> * group) {
    uint32_t e[kApplyBatch<THREADS>];
#pragma unroll
    for (uint32_t u = 0; u < kApplyBatch<THREADS>; ++u) {
      const uint32_t j = min(j0 + u * group, n - 1u);
      e[u] = load_hint<NT>(bin + (j < n0 ? j : j + skip));
    }
#pragma unroll
    for (uint32_t u = 0; u < kApplyBatch<THREADS>; ++u)
      apply_entry_lds<COUNT64>(s_cnt, planes, j0 + u * group < n ? e[u] : 0u);
  }
  __syncthreads();
  if (tid < n_sub) b.bin_count[(brick << b.sub_shift) | tid] = 0u;
}

// The body of one brick's workgroup (s_cnt: the dynamic LDS of the counts).
template <bool COUNT64, uint32_t THREADS>
__device__ __forceinline__ void bin_apply_brick(const BinArgs &b, const Grid &g, void *counts,
                                                uint32_t planes, uint32_t brick, uint32_t *s_cnt) {
  bin_gather_brick<COUNT64, THREADS>(b, g, counts, planes, brick, s_cnt);
  const uint32_t tid = threadIdx.x;
  uint32_t x0, y0, z0;
  brick_origin(b, brick, x0, y0, z0);
  const uint32_t x = x0 + (tid & 15u), y = y0 + ((tid >> 4) & 15u);
  constexpr uint32_t kPer = kBrickCells / THREADS;   // cells per thread and plane
  if (x >= (uint32_t)g.nx || y >= (uint32_t)g.ny) return;
  for (uint32_t p = 0; p < planes; ++p) {
#pragma unroll
    for (uint32_t u = 0; u < kPer; ++u) {
      const uint32_t z = z0 + ((tid + u * THREADS) >> 8);
      if (z < (uint32_t)g.nz) {
        const size_t w = (size_t)p * g.n_cells + ((size_t)z * g.ny + y) * g.nx + x;
        const uint32_t i = p * kBrickCells + tid + u * THREADS;
        if (COUNT64)
          reinterpret_cast<uint2 *>(counts)[w] = reinterpret_cast<const uint2 *>(s_cnt)[i];
        else
          reinterpret_cast<uint32_t *>(counts)[w] = s_cnt[i];
      }
    }
  }
}

template <bool COUNT64, uint32_t THREADS>
__global__ __launch_bounds__(THREADS) void bin_apply_kernel(BinArgs b, Grid g, void *counts,
                                                            uint32_t planes) {
  extern __shared__ uint32_t s_cnt[];
  bin_apply_brick<COUNT64, THREADS>(b, g, counts, planes, blockIdx.x, s_cnt);
}

}  // namespace soma

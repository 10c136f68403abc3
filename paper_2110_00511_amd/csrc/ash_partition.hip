// ash_partition.hip -- batches large enough to be split by key hash first.
//
// What bounds the one-pass kernels on a large batch is one device-scope atomic
// per key: they run at 27 G/s on MI355X whatever the table's size (4 MiB to
// 320 MiB), against 55 G/s for random line reads, 88 G/s for random 16-byte
// stores and about 5 TB/s for streams.  So a large batch is first split into
// bins by the leading bits of the key hash, which costs three streaming
// kernels, and everything that needed atomics then happens per bin in the LDS
// of one block:
//   count    each block takes a contiguous range of positions, drops the
//            copies of a key within 2048 positions in LDS (so a key repeated
//            throughout the batch cannot fill a bin) and counts its remaining
//            keys per bin;
//   scan     per bin, the exclusive prefix of the ranges' counts;
//   scatter  every remaining (key, position) goes to its bin, the ranges' runs
//            in order.
// Nothing is allocated by atomics, and every bin's place is exact, so any
// distribution of keys fits.
#include "ash_device.hpp"
#include "ash_launch.hpp"

#include <algorithm>

namespace ash {

namespace {

constexpr uint32_t kCountThreads = 1024;
constexpr uint32_t kCountItems = kPartTile / kCountThreads;
constexpr int kCountProbes = 3;
constexpr uint32_t kDedupThreads = 1024;
constexpr uint32_t kGroup = 2;  // entries a thread works on together

// An entry of a bin: the key words, then (last word) the position; voxel
// entries hold the number of copies that the entry stands for, less one,
// above the plan's pos_bits.
template <int KD>
constexpr int kEntryWords = SlotWords<KD>::value;

template <int KD>
__device__ __forceinline__ void entry_key(const Slot<kEntryWords<KD>>& e, int32_t (&k)[KD]) {
#pragma unroll
  for (int d = 0; d < KD; ++d) k[d] = (int32_t)e.w[d];
}

template <int KD>
__device__ __forceinline__ Slot<kEntryWords<KD>> load_entry(const uint32_t* __restrict__ entries, uint32_t e) {
  return load_slot<kEntryWords<KD>>(entries + (size_t)e * kEntryWords<KD>);
}

__device__ __forceinline__ uint32_t bin_of(const PartPlan& pl, uint64_t h) {
  return (uint32_t)(((h >> 32) * (uint64_t)pl.nbuckets) >> 32) >> pl.shift;
}

// The range of positions of block b.  Blocks go to the eight XCDs in turn, so
// the blocks of one XCD take neighboring ranges: their runs in a bin adjoin,
// and the lines that two runs share are completed in one L2.
__device__ __forceinline__ uint32_t range_of(const PartPlan& pl, uint32_t b) {
  const uint32_t per = pl.nrange / 8;
  return (b & 7u) * per + (b >> 3);
}

// Inclusive scan over the 64 lanes of a wave.
__device__ __forceinline__ uint32_t wave_incl(uint32_t v) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(v, o, 64);
    if (lane_id() >= (uint32_t)o) v += y;
  }
  return v;
}

// The copies of a voxel's point that one entry can stand for.
__device__ __forceinline__ uint32_t copies_per_entry(const PartPlan& pl) { return 1u << (32u - pl.pos_bits); }

// ---------------------------------------------------------------------------
// Count.  A tile's keys go through an LDS hash table whose entry holds the
// lowest position that has the key so far (a lower one replaces it: the key at
// an entry stays the same).  A key that finds its first kCountProbes entries
// taken by others keeps all its copies: the bins drop the rest, and at half
// load that is one key in about fifteen.  reps: one bit per position, set for the
// positions that go to a bin.  Voxel batches also get each position's link:
// kVoxelWinner + number of copies for a position that goes to a bin, else
// kVoxelLocal + the position it repeats, or kNoSlot for a rejected point.
// Bound by arithmetic (the hash, three divisions for a point) and LDS latency:
// 48 us at 5M points, whose streams alone take 16.  One block of 16 waves per
// CU; the next tile's keys are loaded while the current one is worked on.
template <int KD, typename Src, bool kVoxel>
__global__ __launch_bounds__(kCountThreads) void k_part_count(Src src, PartPlan pl, uint32_t* __restrict__ link,
                                                              uint32_t* __restrict__ zero, uint32_t n_zero,
                                                              Meta* meta) {
  extern __shared__ uint32_t s_hist[];  // nbins
  __shared__ uint32_t s_key[KD][kPartTile];
  __shared__ uint32_t s_tab[2 * kPartTile];
  __shared__ uint32_t s_cnt[kVoxel ? kPartTile : 1];
  constexpr uint32_t kMask = 2 * kPartTile - 1;
  const uint32_t tid = threadIdx.x;
  const uint32_t range = range_of(pl, blockIdx.x);
  const uint32_t begin = min(pl.n, range * pl.per);
  const uint32_t end = min(pl.n, begin + pl.per);
  if (kVoxel) {  // the look-back words and the counters of this call
    for (uint32_t i = blockIdx.x * kCountThreads + tid; i < n_zero; i += gridDim.x * kCountThreads) zero[i] = 0u;
    if (blockIdx.x == 0 && tid < sizeof(Meta) / 4) {
      reinterpret_cast<uint32_t*>(meta)[tid] = tid == offsetof(Meta, epoch) / 4 ? 1u : 0u;
    }
  }
  for (uint32_t b = tid; b < pl.nbins; b += kCountThreads) s_hist[b] = 0u;
  int32_t nk[kCountItems][KD];
  bool nv[kCountItems];
#pragma unroll
  for (uint32_t r = 0; r < kCountItems; ++r) {
    const uint32_t p = begin + r * kCountThreads + tid;
    nv[r] = p < end && src.load(p, nk[r]);
  }
  for (uint32_t t = begin; t < end; t += kPartTile) {
    int32_t k[kCountItems][KD];
    bool valid[kCountItems];
#pragma unroll
    for (uint32_t r = 0; r < kCountItems; ++r) {
      valid[r] = nv[r];
      const uint32_t pos = r * kCountThreads + tid;
#pragma unroll
      for (int d = 0; d < KD; ++d) {
        k[r][d] = nk[r][d];
        s_key[d][pos] = (uint32_t)k[r][d];
      }
      if (kVoxel) s_cnt[pos] = 1u;
      const uint32_t p = t + kPartTile + pos;
      nv[r] = p < end && src.load(p, nk[r]);
    }
#pragma unroll
    for (uint32_t r = 0; r < 2 * kCountItems; ++r) s_tab[r * kCountThreads + tid] = kNoSlot;
    __syncthreads();
    uint32_t at[kCountItems], bin[kCountItems];
    bool open[kCountItems];
#pragma unroll
    for (uint32_t r = 0; r < kCountItems; ++r) {
      const uint64_t h = key_hash<KD>(k[r]);
      bin[r] = bin_of(pl, h);
      at[r] = (uint32_t)(h >> 7) & kMask;
      open[r] = valid[r];
    }
#pragma unroll
    for (int step = 0; step < kCountProbes; ++step) {
      uint32_t o[kCountItems];
#pragma unroll
      for (uint32_t r = 0; r < kCountItems; ++r)
        if (open[r]) o[r] = atomicCAS(&s_tab[at[r]], kNoSlot, r * kCountThreads + tid);
#pragma unroll
      for (uint32_t r = 0; r < kCountItems; ++r) {
        if (!open[r]) continue;
        const uint32_t pos = r * kCountThreads + tid;
        bool eq = o[r] == kNoSlot;
        if (!eq) {
          eq = true;
#pragma unroll
          for (int d = 0; d < KD; ++d) eq = eq && s_key[d][o[r]] == (uint32_t)k[r][d];
          if (eq && pos < o[r]) atomicMin(&s_tab[at[r]], pos);
        }
        if (eq) open[r] = false;
        else at[r] = (at[r] + 1) & kMask;
      }
    }
    __syncthreads();
    uint32_t rep[kCountItems];
#pragma unroll
    for (uint32_t r = 0; r < kCountItems; ++r) {
      const uint32_t pos = r * kCountThreads + tid;
      rep[r] = !valid[r] ? kNoSlot : open[r] ? pos : s_tab[at[r]];
      const bool is_rep = rep[r] == pos;
      const uint64_t bits = __ballot(is_rep);
      const uint32_t p = t + pos;
      if (lane_id() == 0 && p < end) pl.reps[p >> 6] = bits;
      if (kVoxel) {
        if (valid[r] && !is_rep) atomicAdd(&s_cnt[rep[r]], 1u);
      } else if (is_rep) {
        atomicAdd(&s_hist[bin[r]], 1u);
      }
    }
    if (kVoxel) {
      __syncthreads();
      const uint32_t most = copies_per_entry(pl);
#pragma unroll
      for (uint32_t r = 0; r < kCountItems; ++r) {
        const uint32_t pos = r * kCountThreads + tid;
        const uint32_t p = t + pos;
        if (p >= end) continue;
        uint32_t v = kNoSlot;
        if (rep[r] == pos) {
          const uint32_t m = s_cnt[pos];
          v = kVoxelWinner + m;
          atomicAdd(&s_hist[bin[r]], (m + most - 1) / most);
        } else if (valid[r]) {
          v = kVoxelLocal + t + rep[r];
        }
        link[p] = v;
      }
    }
    __syncthreads();
  }
  __syncthreads();
  for (uint32_t b = tid; b < pl.nbins; b += kCountThreads) pl.hist[(size_t)range * pl.nbins + b] = s_hist[b];
}

// ---------------------------------------------------------------------------
// Scan.  hist[range][bin] becomes the exclusive prefix over the ranges, and
// total[bin] their sum.  A block takes 64 bins; its 16 waves hold up to
// kPartRanges / 16 ranges each in registers, so the counts are read once.
__global__ __launch_bounds__(1024) void k_part_scan(PartPlan pl) {
  constexpr uint32_t kRows = kPartRanges / 16;
  __shared__ uint32_t s_sum[16][64];
  const uint32_t lane = lane_id(), w = threadIdx.x >> 6;
  const uint32_t bin = blockIdx.x * 64 + lane;
  uint32_t v[kRows];
  uint32_t sum = 0;
#pragma unroll
  for (uint32_t i = 0; i < kRows; ++i) {
    const uint32_t row = w * kRows + i;
    v[i] = row < pl.nrange && bin < pl.nbins ? pl.hist[(size_t)row * pl.nbins + bin] : 0u;
  }
#pragma unroll
  for (uint32_t i = 0; i < kRows; ++i) sum += v[i];
  s_sum[w][lane] = sum;
  __syncthreads();
  uint32_t before = 0;
  for (uint32_t i = 0; i < w; ++i) before += s_sum[i][lane];
  if (bin >= pl.nbins) return;
#pragma unroll
  for (uint32_t i = 0; i < kRows; ++i) {
    const uint32_t row = w * kRows + i;
    if (row < pl.nrange) pl.hist[(size_t)row * pl.nbins + bin] = before;
    before += v[i];
  }
  if (w == 15) pl.total[bin] = before;
}

// Exclusive scan of v[0 .. n) into LDS s[0 .. n] by a block (n <= kMost); the
// total goes to s[n].
template <uint32_t kThreads, uint32_t kMost>
__device__ __forceinline__ void block_scan_into(const uint32_t* __restrict__ v, uint32_t n, uint32_t* s,
                                                uint32_t* s_wave) {
  constexpr uint32_t kEach = (kMost + kThreads - 1) / kThreads;
  const uint32_t first = threadIdx.x * kEach;
  uint32_t x[kEach];
  uint32_t sum = 0;
#pragma unroll
  for (uint32_t i = 0; i < kEach; ++i) {
    x[i] = first + i < n ? v[first + i] : 0u;
    sum += x[i];
  }
  const uint32_t incl = wave_incl(sum);
  if (lane_id() == 63) s_wave[threadIdx.x >> 6] = incl;
  __syncthreads();
  uint32_t before = incl - sum;
  for (uint32_t w = 0; w < (threadIdx.x >> 6); ++w) before += s_wave[w];
#pragma unroll
  for (uint32_t i = 0; i < kEach; ++i) {
    if (first + i < n) s[first + i] = before;
    before += x[i];
  }
  if (threadIdx.x == kThreads - 1) s[n] = before;
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Scatter.  Every position whose rep bit is set writes its entry at its
// range's cursor of its bin (an LDS atomic; the order within a run does not
// matter).  Bound by the 16-byte stores: 48-50 us at 5M points with about 1000
// bins and 256 ranges, where a line of each run stays open in the L2 until it
// is full; 62 us with 1200 bins and 512 ranges, where none does (that is the
// rate of random stores).
template <int KD, typename Src, bool kVoxel>
__global__ __launch_bounds__(kCountThreads) void k_part_scatter(Src src, PartPlan pl,
                                                                const uint32_t* __restrict__ link) {
  extern __shared__ uint32_t s_cur[];  // nbins + 1
  __shared__ uint32_t s_wave[kCountThreads / 64];
  constexpr int S = kEntryWords<KD>;
  const uint32_t tid = threadIdx.x;
  const uint32_t range = range_of(pl, blockIdx.x);
  const uint32_t begin = min(pl.n, range * pl.per);
  const uint32_t end = min(pl.n, begin + pl.per);
  block_scan_into<kCountThreads, kPartBins>(pl.total, pl.nbins, s_cur, s_wave);
  if (blockIdx.x == 0)
    for (uint32_t b = tid; b <= pl.nbins; b += kCountThreads) pl.base[b] = s_cur[b];
  for (uint32_t b = tid; b < pl.nbins; b += kCountThreads) s_cur[b] += pl.hist[(size_t)range * pl.nbins + b];
  __syncthreads();
  for (uint32_t t = begin; t < end; t += kPartTile) {
    int32_t k[kCountItems][KD];
    uint32_t m[kCountItems];
#pragma unroll
    for (uint32_t r = 0; r < kCountItems; ++r) {
      const uint32_t p = t + r * kCountThreads + tid;
      m[r] = 0;
      if (p >= end) continue;
      const bool is_rep = (pl.reps[p >> 6] >> (p & 63u)) & 1u;
      src.load(p, k[r]);
      if (is_rep) m[r] = kVoxel ? link[p] & ~kVoxelWinner : 1u;
    }
#pragma unroll
    for (uint32_t r = 0; r < kCountItems; ++r) {
      if (m[r] == 0) continue;
      const uint32_t p = t + r * kCountThreads + tid;
      const uint32_t bin = bin_of(pl, key_hash<KD>(k[r]));
      Slot<S> e;
#pragma unroll
      for (int q = 0; q < S; ++q) e.w[q] = 0;
#pragma unroll
      for (int d = 0; d < KD; ++d) e.w[d] = (uint32_t)k[r][d];
      if (kVoxel) {
        const uint32_t most = copies_per_entry(pl);
        for (uint32_t left = m[r]; left > 0;) {
          const uint32_t now = min(left, most);
          e.w[S - 1] = p | ((now - 1u) << pl.pos_bits);
          store_slot<S>(pl.entries + (size_t)atomicAdd(&s_cur[bin], 1u) * S, e);
          left -= now;
        }
      } else {
        e.w[S - 1] = p;
        store_slot<S>(pl.entries + (size_t)atomicAdd(&s_cur[bin], 1u) * S, e);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The distinct keys of a bin in LDS: a hash table of entry numbers, each with
// as many bits of the key's hash above it as fit, so that an entry is compared
// (a read of the bin in L2) only against one that has its key, save for about
// one in 2^tag_bits.
struct BinTable {
  uint32_t* own;
  uint32_t mask;      // entries - 1
  uint32_t num_bits;  // bits of an entry number (all ones is no entry's number)
};

__device__ __forceinline__ BinTable bin_table(uint32_t* lds, uint32_t entries, uint32_t size) {
  return BinTable{lds, entries - 1u, 32u - (uint32_t)__clz((int)(size + 1u))};
}

// Finds the table entries of kGroup bin entries of a thread together (those
// with open[i]; number e[i], entry x[i]), so that their LDS and memory waits
// overlap.  at[i]: the table entry of x[i]'s key, or kNoSlot when the table is
// full of others.  Inserting, the lowest position of a key holds its entry
// in the end, and `lost` is told every bin entry that gives way.
template <int KD, bool kInsert, typename Lost>
__device__ __forceinline__ void bin_place(const BinTable& t, const uint32_t* __restrict__ ent, uint32_t pos_mask,
                                          const uint32_t (&e)[kGroup], const Slot<kEntryWords<KD>> (&x)[kGroup],
                                          bool (&open)[kGroup], uint32_t (&at)[kGroup], const Lost& lost) {
  constexpr int S = kEntryWords<KD>;
  const uint32_t num_mask = (1u << t.num_bits) - 1u;
  uint32_t mine[kGroup], step[kGroup], jump[kGroup];
  bool any = false;
#pragma unroll
  for (uint32_t i = 0; i < kGroup; ++i) {
    int32_t k[KD];
    entry_key<KD>(x[i], k);
    const uint64_t h = key_hash<KD>(k);
    mine[i] = ((uint32_t)(h >> 16) & ~num_mask) | e[i];
    at[i] = (uint32_t)h & t.mask;
    jump[i] = (uint32_t)(h >> 15) | 1u;  // double hashing: a wave waits for its longest probe sequence
    step[i] = 0;
    any = any || open[i];
  }
  while (any) {
    uint32_t o[kGroup];
    bool same[kGroup];
    Slot<S> y[kGroup];
#pragma unroll
    for (uint32_t i = 0; i < kGroup; ++i)
      if (open[i]) o[i] = __hip_atomic_load(&t.own[at[i]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if constexpr (kInsert) {
#pragma unroll
      for (uint32_t i = 0; i < kGroup; ++i)
        if (open[i] && o[i] == kNoSlot) o[i] = atomicCAS(&t.own[at[i]], kNoSlot, mine[i]);
    }
#pragma unroll
    for (uint32_t i = 0; i < kGroup; ++i) {
      if (open[i] && o[i] == kNoSlot) {
        if (!kInsert) at[i] = kNoSlot;
        open[i] = false;
      }
      if (!kInsert && open[i] && o[i] == mine[i]) open[i] = false;
      same[i] = open[i] && ((o[i] ^ mine[i]) & ~num_mask) == 0u;
      if (same[i]) y[i] = load_entry<KD>(ent, o[i] & num_mask);
    }
    any = false;
#pragma unroll
    for (uint32_t i = 0; i < kGroup; ++i) {
      if (!open[i]) continue;
      bool eq = same[i];
      if (eq) {
#pragma unroll
        for (int d = 0; d < KD; ++d) eq = eq && y[i].w[d] == x[i].w[d];
      }
      if (!eq) {
        at[i] = (at[i] + jump[i]) & t.mask;
        if (++step[i] > t.mask) {
          at[i] = kNoSlot;
          open[i] = false;
        }
      } else if (!kInsert) {
        open[i] = false;
      } else {
        const uint32_t p = x[i].w[S - 1] & pos_mask, po = y[i].w[S - 1] & pos_mask;
        if (po <= p) {
          lost(e[i], p);
          open[i] = false;
        } else if (atomicCAS(&t.own[at[i]], o[i], mine[i]) == o[i]) {  // the lower position takes the entry
          lost(o[i] & num_mask, po);
          open[i] = false;
        }  // else another of the same key came in between, at a lower position than po: look again
      }
      any = any || open[i];
    }
  }
}

// Voxelization of one bin: a block finds, for every distinct voxel of the bin,
// its first point and its number of points, and corrects the links: a first
// point's count (where copies came in from other tiles), and every other
// point's first point.  The table has room for twice the mean bin; an entry
// that finds it full (a bin of many times the mean's distinct voxels) is
// settled by a scan over the bin.  Bound by LDS and L2 latency: a wave waits
// for its longest probe sequence, so the table hashes twice (linear probing:
// 324 against 130 us at 5M points), and two blocks of 16 waves share a CU (76
// KB each; one block with twice the bin: 130 against 66 us; bins of 2560 and
// 1900 points gain here what the scatter's shorter runs lose).  A thread works
// on two entries at once: four need 73 registers, or spill at 64 (144 us).
__global__ __launch_bounds__(kDedupThreads, 8) void k_voxel_bins(PartPlan pl, uint32_t table, uint32_t places,
                                                              uint32_t* __restrict__ link) {
  constexpr int KD = 3;
  extern __shared__ uint32_t s_own[];  // table owners, table counts, the first `places` entries' places (16 bits)
  uint32_t* s_cnt = s_own + table;
  uint16_t* s_at = reinterpret_cast<uint16_t*>(s_cnt + table);
  const uint32_t base = pl.base[blockIdx.x];
  const uint32_t size = pl.base[blockIdx.x + 1] - base;
  const uint32_t* __restrict__ ent = pl.entries + (size_t)base * kEntryWords<KD>;
  const uint32_t pos_mask = (1u << pl.pos_bits) - 1u;
  for (uint32_t j = threadIdx.x; j < table / 4; j += kDedupThreads) {
    reinterpret_cast<uint4*>(s_own)[j] = make_uint4(kNoSlot, kNoSlot, kNoSlot, kNoSlot);
    reinterpret_cast<uint4*>(s_cnt)[j] = make_uint4(0u, 0u, 0u, 0u);
  }
  const BinTable t = bin_table(s_own, table, size);
  const auto none = [](uint32_t, uint32_t) {};
  auto group = [&](uint32_t g, uint32_t (&e)[kGroup], Slot<4> (&x)[kGroup], bool (&open)[kGroup]) {
#pragma unroll
    for (uint32_t i = 0; i < kGroup; ++i) {
      e[i] = g + i * kDedupThreads + threadIdx.x;
      open[i] = e[i] < size;
      if (open[i]) x[i] = load_entry<KD>(ent, e[i]);
    }
  };
  __syncthreads();
  for (uint32_t g = 0; g < size; g += kGroup * kDedupThreads) {
    uint32_t e[kGroup], at[kGroup];
    Slot<4> x[kGroup];
    bool open[kGroup], used[kGroup];
    group(g, e, x, open);
#pragma unroll
    for (uint32_t i = 0; i < kGroup; ++i) used[i] = open[i];
    bin_place<KD, true>(t, ent, pos_mask, e, x, open, at, none);
#pragma unroll
    for (uint32_t i = 0; i < kGroup; ++i) {
      if (used[i] && at[i] != kNoSlot) atomicAdd(&s_cnt[at[i]], (x[i].w[3] >> pl.pos_bits) + 1u);
      if (e[i] < places) s_at[e[i]] = (uint16_t)at[i];  // (kNoSlot: 0xFFFF, no entry's place in a table of 2^15)
    }
  }
  __syncthreads();
  for (uint32_t g = 0; g < size; g += kGroup * kDedupThreads) {
    uint32_t e[kGroup], at[kGroup], first[kGroup], count[kGroup];
    Slot<4> x[kGroup];
    bool open[kGroup], used[kGroup];
    group(g, e, x, open);
#pragma unroll
    for (uint32_t i = 0; i < kGroup; ++i) {
      used[i] = open[i];
      open[i] = open[i] && e[i] >= places;
      at[i] = e[i] < places && s_at[e[i]] != 0xFFFFu ? s_at[e[i]] : kNoSlot;
    }
    if (g + kGroup * kDedupThreads > places) {
      uint32_t again[kGroup];
      bin_place<KD, false>(t, ent, pos_mask, e, x, open, again, none);
#pragma unroll
      for (uint32_t i = 0; i < kGroup; ++i)
        if (e[i] >= places) at[i] = again[i];
    }
#pragma unroll
    for (uint32_t i = 0; i < kGroup; ++i) {
      if (!used[i]) continue;
      first[i] = x[i].w[3] & pos_mask;
      count[i] = 0;
      if (at[i] != kNoSlot) {
        count[i] = s_cnt[at[i]];
        const uint32_t o = s_own[at[i]] & ((1u << t.num_bits) - 1u);
        if (o != e[i]) {
          first[i] = ent[(size_t)o * 4 + 3] & pos_mask;
          // another entry of the same point reports
          if (first[i] == (x[i].w[3] & pos_mask)) used[i] = false;
        }
      } else {
        for (uint32_t o = 0; o < size; ++o) {
          const Slot<4> z = load_entry<KD>(ent, o);
          if (z.w[0] != x[i].w[0] || z.w[1] != x[i].w[1] || z.w[2] != x[i].w[2]) continue;
          first[i] = min(first[i], z.w[3] & pos_mask);
          count[i] += (z.w[3] >> pl.pos_bits) + 1u;
        }
      }
    }
#pragma unroll
    for (uint32_t i = 0; i < kGroup; ++i) {
      if (!used[i]) continue;
      const uint32_t p = x[i].w[3] & pos_mask;
      if (first[i] != p) link[p] = first[i];
      else if (count[i] != (x[i].w[3] >> pl.pos_bits) + 1u) link[p] = kVoxelWinner + count[i];
    }
  }
}

// First points are ranked in batch order (the voxel ids) and write their
// voxel's key and count, their own id, and -1 for rejected points.
__global__ __launch_bounds__(kBlock) void k_voxel_number(VoxelKeys src, uint32_t n, const uint32_t* __restrict__ link,
                                                         int32_t* __restrict__ voxel_keys,
                                                         int32_t* __restrict__ counts,
                                                         int32_t* __restrict__ point_voxel, Meta* meta,
                                                         uint64_t* __restrict__ status) {
  __shared__ uint32_t s_prefix;
  __shared__ uint64_t s_scan[kBlock / 64 + 1];
  const uint32_t tile = blockIdx.x;
  const uint32_t base = tile * kScanTile;
  bool win[kScanItems];
  uint32_t v[kScanItems];
  int32_t k[kScanItems][3];
#pragma unroll
  for (int r = 0; r < kScanItems; ++r) {
    const uint32_t p = base + r * kBlock + threadIdx.x;
    v[r] = p < n ? link[p] : 0u;
    win[r] = (v[r] & kVoxelWinner) != 0u && v[r] != kNoSlot;
    if (v[r] == kNoSlot) point_voxel[p] = -1;
    if (win[r]) src.load(p, k[r]);
  }
  uint32_t rank[kScanItems];
  uint32_t total;
  block_rank_rows(win, rank, total, s_scan);
  const uint32_t prefix = block_lookback(status, tile, meta->epoch, total, &meta->status, &s_prefix);
  // the last tile's look-back saw every tile: it records the voxel count
  if (threadIdx.x == 0 && tile == gridDim.x - 1) meta->claims = prefix + total;
#pragma unroll
  for (int r = 0; r < kScanItems; ++r) {
    if (!win[r]) continue;
    const uint32_t id = prefix + rank[r];
    voxel_keys[(size_t)id * 3 + 0] = k[r][0];
    voxel_keys[(size_t)id * 3 + 1] = k[r][1];
    voxel_keys[(size_t)id * 3 + 2] = k[r][2];
    counts[id] = (int32_t)(v[r] & ~kVoxelWinner);
    point_voxel[base + r * kBlock + threadIdx.x] = (int32_t)id;
  }
}

// The other points take their first point's id, through the point of their
// own 2048 that went to the bin where they were dropped in favor of it.
__global__ __launch_bounds__(kBlock) void k_voxel_follow(uint32_t n, const uint32_t* __restrict__ link,
                                                         int32_t* __restrict__ point_voxel) {
  const uint32_t base = blockIdx.x * kScanTile + threadIdx.x;
  uint32_t q[kScanItems];
#pragma unroll
  for (int r = 0; r < kScanItems; ++r) {
    const uint32_t p = base + r * kBlock;
    q[r] = p < n ? link[p] : kNoSlot;
  }
#pragma unroll
  for (int r = 0; r < kScanItems; ++r) {
    if (q[r] & kVoxelWinner) continue;
    if (q[r] & kVoxelLocal) {
      q[r] &= ~kVoxelLocal;
      const uint32_t v = link[q[r]];
      if (!(v & kVoxelWinner)) q[r] = v;
    }
  }
#pragma unroll
  for (int r = 0; r < kScanItems; ++r)
    if (!(q[r] & kVoxelWinner)) point_voxel[base + r * kBlock] = point_voxel[q[r]];
}

inline uint32_t cdiv(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

template <int KD, typename Src, bool kVoxel>
hipError_t partition(const Src& src, const PartPlan& pl, uint32_t* link, uint32_t* zero, uint32_t n_zero, Meta* meta,
                     hipStream_t st) {
  if (pl.n == 0 || pl.nrange == 0 || pl.nrange % 8 != 0 || pl.nrange > kPartRanges || pl.nbins == 0 ||
      pl.nbins > kPartBins || pl.per % kPartTile != 0 || (uint64_t)pl.nrange * pl.per < pl.n)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_part_count<KD, Src, kVoxel>), dim3(pl.nrange), dim3(kCountThreads), pl.nbins * 4, st, src, pl,
                     link, zero, n_zero, meta);
  hipLaunchKernelGGL(k_part_scan, dim3(cdiv(pl.nbins, 64)), dim3(1024), 0, st, pl);
  hipLaunchKernelGGL((k_part_scatter<KD, Src, kVoxel>), dim3(pl.nrange), dim3(kCountThreads), (pl.nbins + 1) * 4, st,
                     src, pl, link);
  return hipGetLastError();
}

}  // namespace

bool part_ranges(PartPlan* pl, uint32_t n) {
  pl->n = n;
  pl->nrange = std::min<uint32_t>(kPartRanges, cdiv(cdiv(n, kPartTile), 8) * 8);
  pl->per = cdiv(cdiv(n, pl->nrange), kPartTile) * kPartTile;
  pl->pos_bits = 1;
  while (pl->pos_bits < 32 && ((uint64_t)1 << pl->pos_bits) < n) ++pl->pos_bits;
  return pl->pos_bits <= 30;
}


hipError_t launch_voxel_partitioned(const PartPlan& pl, const float* pts, float voxel, uint32_t* link,
                                    int32_t* voxel_keys, int32_t* counts, int32_t* point_voxel, Meta* meta,
                                    uint64_t* status, hipStream_t st) {
  const uint32_t tiles = cdiv(pl.n, kScanTile);
  const VoxelKeys src{pts, voxel};
  hipError_t e = partition<3, VoxelKeys, true>(src, pl, link, reinterpret_cast<uint32_t*>(status), tiles * 2, meta, st);
  if (e != hipSuccess) return e;
  constexpr uint32_t table = 8192;  // about half full of a mean bin's voxels at most
  const uint32_t places = table / 4 * 3;
  const uint32_t lds = table * 8 + places * 2;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_voxel_bins), hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_voxel_bins, dim3(pl.nbins), dim3(kDedupThreads), lds, st, pl, table, places, link);
  hipLaunchKernelGGL(k_voxel_number, dim3(tiles), dim3(kBlock), 0, st, src, pl.n, link, voxel_keys, counts,
                     point_voxel, meta, status);
  hipLaunchKernelGGL(k_voxel_follow, dim3(tiles), dim3(kBlock), 0, st, pl.n, link, point_voxel);
  return hipGetLastError();
}

}  // namespace ash

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
//            copies of a key within 4096 positions in LDS (so a key repeated
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
__device__ __forceinline__ Slot<kEntryWords<KD>> load_entry(const uint32_t* entries, uint32_t e) {
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
// Count.  Copies of a key within a tile are dropped as far as one look at an
// LDS hash table finds them; the bins drop the rest.  Two keys that meet at
// one entry in a tile meet at different ones in the next, so that even keys
// that fill the batch come through rarely.  reps: one bit per position, set
// for the positions that go to a bin.  Voxel batches also get each position's link:
// kVoxelWinner + number of copies for a position that goes to a bin, else
// kVoxelLocal + the position it repeats, or kNoSlot for a rejected point.
// 33 to 35 us at 5M points (55 at 10M keys), whose streams alone take 16.  By
// counters no unit is full: VALU 52% busy (35% for keys: the hash, and three
// divisions for a point), LDS 16% (half of it bank conflicts), memory at 2.2
// TB/s, and waves wait 55 to 62% of their time, for LDS and at the barriers
// between a tile's steps.  One block of 16 waves per CU (the LDS holds no
// more); the next tile's keys are loaded while the current one is worked on.
template <int KD, typename Src, bool kVoxel>
__global__ __launch_bounds__(kCountThreads) void k_part_count(Src src, PartPlan pl, uint32_t* __restrict__ link,
                                                              uint32_t* __restrict__ zero, uint32_t n_zero,
                                                              Meta* meta) {
  extern __shared__ uint32_t s_hist[];  // nbins
  __shared__ uint32_t s_key[KD][kPartTile];
  __shared__ uint32_t s_tab[2 * kPartTile];  // (an entry that a tile reads was written in it)
  __shared__ uint32_t s_low[kPartTile];
  __shared__ uint32_t s_cnt[kVoxel ? kPartTile : 1];
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
      s_low[pos] = pos;
      if (kVoxel) s_cnt[pos] = 1u;
      const uint32_t p = t + kPartTile + pos;
      nv[r] = p < end && src.load(p, nk[r]);
    }
    // each key's position to an LDS entry picked by the hash and the tile, the last one written stays;
    // a position whose entry then names another one with its key is a copy
    uint32_t at[kCountItems], bin[kCountItems], rep[kCountItems];
    const uint32_t salt = 2u * (t / kPartTile) + 0x9e3779b1u;
#pragma unroll
    for (uint32_t r = 0; r < kCountItems; ++r) {
      const uint64_t h = key_hash<KD>(k[r]);
      bin[r] = bin_of(pl, h);
      at[r] = ((uint32_t)h * salt) >> (32 - kPartTileLog2 - 1);
      if (valid[r]) s_tab[at[r]] = r * kCountThreads + tid;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < kCountItems; ++r) {
      const uint32_t pos = r * kCountThreads + tid;
      rep[r] = valid[r] ? s_tab[at[r]] : pos;
    }
#pragma unroll
    for (uint32_t r = 0; r < kCountItems; ++r) {
      const uint32_t pos = r * kCountThreads + tid;
      if (rep[r] == pos) continue;
      bool eq = true;
#pragma unroll
      for (int d = 0; d < KD; ++d) eq = eq && s_key[d][rep[r]] == (uint32_t)k[r][d];
      if (!eq) rep[r] = pos;
      else if (pos < s_low[rep[r]]) atomicMin(&s_low[rep[r]], pos);  // the lowest of them stands for all
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < kCountItems; ++r) {
      const uint32_t pos = r * kCountThreads + tid;
      rep[r] = valid[r] ? s_low[rep[r]] : kNoSlot;
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
// Scatter.  Every position whose rep bit is set writes its entry to its bin,
// in its range's run.  A tile's entries are first put in bin order in LDS, so
// that a run's entries of one tile (about 6 with 1400 bins) leave together:
// written one by one they reach memory as 16-byte stores (88 G/s; 149 us at
// 10M keys, against 111).  kItems positions per thread and tile: as many as the
// LDS holds.  Bound by latency like the count, with one block per CU: memory
// moves at 2.8 TB/s, VALU is 17% busy (36% for points), LDS 18%, and waves wait
// two thirds of their time.
template <int KD, typename Src, bool kVoxel, uint32_t kItems>
__global__ __launch_bounds__(kCountThreads) void k_part_scatter(Src src, PartPlan pl,
                                                                const uint32_t* __restrict__ link) {
  constexpr int S = kEntryWords<KD>;
  constexpr uint32_t kTile = kItems * kCountThreads;
  constexpr uint32_t kBinsEach = kPartBins / kCountThreads;
  extern __shared__ uint32_t s_lds[];
  uint32_t* s_word = s_lds;                                               // [KD + 1][kTile]: keys, last words
  uint16_t* s_bin = reinterpret_cast<uint16_t*>(s_word + (KD + 1) * kTile);  // [kTile]
  uint32_t* s_cur = reinterpret_cast<uint32_t*>(s_bin + kTile);           // [nbins + 1]: next entry of the run
  uint32_t* s_cnt = s_cur + pl.nbins + 1;                                 // [nbins]: the tile's entries, then their place
  __shared__ uint32_t s_wave[kCountThreads / 64];
  __shared__ uint32_t s_total;
  const uint32_t tid = threadIdx.x;
  const uint32_t range = range_of(pl, blockIdx.x);
  const uint32_t begin = min(pl.n, range * pl.per);
  const uint32_t end = min(pl.n, begin + pl.per);
  block_scan_into<kCountThreads, kPartBins>(pl.total, pl.nbins, s_cur, s_wave);
  if (blockIdx.x == 0)
    for (uint32_t b = tid; b <= pl.nbins; b += kCountThreads) pl.base[b] = s_cur[b];
  __syncthreads();
  for (uint32_t b = tid; b < pl.nbins; b += kCountThreads) {
    s_cur[b] += pl.hist[(size_t)range * pl.nbins + b];
    s_cnt[b] = 0u;
  }
  const uint32_t most = kVoxel ? copies_per_entry(pl) : 1u;
  int32_t k[kItems][KD];
  uint32_t m[kItems];
  const auto load = [&](uint32_t t) {
#pragma unroll
    for (uint32_t r = 0; r < kItems; ++r) {
      const uint32_t p = t + r * kCountThreads + tid;
      m[r] = 0;
      if (p >= end) continue;
      const bool is_rep = (pl.reps[p >> 6] >> (p & 63u)) & 1u;
      src.load(p, k[r]);
      if (is_rep) m[r] = kVoxel ? link[p] & ~kVoxelWinner : 1u;
    }
  };
  load(begin);
  __syncthreads();
  for (uint32_t t = begin; t < end; t += kTile) {
    uint32_t bin[kItems], rank[kItems];
#pragma unroll
    for (uint32_t r = 0; r < kItems; ++r) {
      if (m[r] == 0) continue;
      bin[r] = bin_of(pl, key_hash<KD>(k[r]));
      rank[r] = atomicAdd(&s_cnt[bin[r]], (m[r] + most - 1u) / most);
    }
    __syncthreads();
    // s_cnt: counts -> places of the bins in the tile's order
    uint32_t cnt[kBinsEach], sum = 0;
#pragma unroll
    for (uint32_t i = 0; i < kBinsEach; ++i) {
      const uint32_t b = tid * kBinsEach + i;
      cnt[i] = b < pl.nbins ? s_cnt[b] : 0u;
      sum += cnt[i];
    }
    const uint32_t incl = wave_incl(sum);
    if (lane_id() == 63) s_wave[tid >> 6] = incl;
    __syncthreads();
    uint32_t place = incl - sum;
    for (uint32_t w = 0; w < (tid >> 6); ++w) place += s_wave[w];
#pragma unroll
    for (uint32_t i = 0; i < kBinsEach; ++i) {
      const uint32_t b = tid * kBinsEach + i;
      if (b < pl.nbins) s_cnt[b] = place;
      place += cnt[i];
    }
    if (tid == kCountThreads - 1) s_total = place;
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < kItems; ++r) {
      uint32_t at = m[r] ? s_cnt[bin[r]] + rank[r] : 0u;
      for (uint32_t left = m[r]; left > 0; ++at) {
        const uint32_t now = min(left, most);
#pragma unroll
        for (int d = 0; d < KD; ++d) s_word[d * kTile + at] = (uint32_t)k[r][d];
        s_word[KD * kTile + at] = (t + r * kCountThreads + tid) | (kVoxel ? (now - 1u) << pl.pos_bits : 0u);
        s_bin[at] = (uint16_t)bin[r];
        left -= now;
      }
    }
    if (t + kTile < end) load(t + kTile);
    __syncthreads();
    const uint32_t total = s_total;
#pragma unroll
    for (uint32_t r = 0; r < kItems; ++r) {
      const uint32_t at = r * kCountThreads + tid;
      if (at >= total) continue;
      const uint32_t b = s_bin[at];
      Slot<S> e;
#pragma unroll
      for (int q = 0; q < S; ++q) e.w[q] = 0;
#pragma unroll
      for (int d = 0; d < KD; ++d) e.w[d] = s_word[d * kTile + at];
      e.w[S - 1] = s_word[KD * kTile + at];
      store_slot<S>(pl.entries + (size_t)(s_cur[b] + at - s_cnt[b]) * S, e);
    }
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < kBinsEach; ++i) {
      const uint32_t b = tid * kBinsEach + i;
      if (b >= pl.nbins) continue;
      s_cur[b] += cnt[i];
      s_cnt[b] = 0u;
    }
    __syncthreads();
  }
}

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
__device__ __forceinline__ void bin_place(const BinTable& t, const uint32_t* ent, uint32_t pos_mask,
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
// settled by a scan over the bin.  Bound by arithmetic and LDS latency (VALU 45%
// busy, LDS 18%, waves wait 55% of their time, memory 2.1 TB/s; at 5 cm links
// written to random places make it 3.8): a wave waits for its longest
// probe sequence, so the table hashes twice (linear probing: 324 against 130 us
// at 5M points), and two blocks of 16 waves share a CU (76 KB each; one block
// with twice the bin: 130 against 66 us; bins of 2560 and 1900 points gain here
// what the scatter's shorter runs lose).  A thread works on two entries at once:
// four need 73 registers, or spill at 64 (144 us).
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
// voxel's key and count, their own id, and -1 for rejected points.  Bound by
// the look-back between tiles, whose words travel through memory (waves wait 76%
// of their time, memory moves at 3.6 TB/s at 5 mm and 1.0 at 5 cm): tiles of
// 4096 points are a quarter as many steps as tiles of 1024 (5M points at 5 mm
// 59 -> 51 us, at 5 cm 41 -> 43; whole calls on 0.7M points and more 0 to 4%
// faster, smaller ones the same).
constexpr uint32_t kNumberThreads = kNumberTile / kScanItems;

__global__ __launch_bounds__(kNumberThreads) void k_voxel_number(VoxelKeys src, uint32_t n, const uint32_t* __restrict__ link,
                                                         int32_t* __restrict__ voxel_keys,
                                                         int32_t* __restrict__ counts,
                                                         int32_t* __restrict__ point_voxel, Meta* meta,
                                                         uint64_t* __restrict__ status) {
  __shared__ uint32_t s_prefix;
  __shared__ uint64_t s_scan[kNumberThreads / 64 + 1];
  const uint32_t tile = blockIdx.x;
  const uint32_t base = tile * kNumberTile;
  bool win[kScanItems];
  uint32_t v[kScanItems];
  int32_t k[kScanItems][3];
#pragma unroll
  for (int r = 0; r < kScanItems; ++r) {
    const uint32_t p = base + r * kNumberThreads + threadIdx.x;
    v[r] = p < n ? link[p] : 0u;
    win[r] = (v[r] & kVoxelWinner) != 0u && v[r] != kNoSlot;
    if (v[r] == kNoSlot) point_voxel[p] = -1;
    if (win[r]) src.load(p, k[r]);
  }
  uint32_t rank[kScanItems];
  uint32_t total;
  block_rank_rows<kNumberThreads>(win, rank, total, s_scan);
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
    point_voxel[base + r * kNumberThreads + threadIdx.x] = (int32_t)id;
  }
}

// The other points take their first point's id, through the point of their
// own 4096 that went to the bin where they were dropped in favor of it.
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

// ---------------------------------------------------------------------------
// Insert by bins.  The new keys of a batch are settled before the table is
// written: bins finds them (an entry that is not one is marked in its
// position's top bit), collect turns their positions into bits and ranks, the
// commit streams over the batch in order, and place puts them into the table,
// bin by bin, with their buffer indices known.  So the table gets one store
// per new key and no atomic, and a batch that overflows leaves it untouched.

// Looks kGroup keys up in the table together (those with open[i]), so that
// their waits overlap: held[i] says whether a committed slot holds k[i].  Each
// sequence is followed to the first EMPTY slot, as in a find.
template <int KD>
__device__ __forceinline__ void table_holds(const TableRef& tb, const int32_t (&k)[kGroup][KD], bool (&open)[kGroup],
                                            bool (&held)[kGroup]) {
  constexpr int S = SlotWords<KD>::value;
  uint32_t s[kGroup];
  bool any = false;
#pragma unroll
  for (uint32_t i = 0; i < kGroup; ++i) {
    held[i] = false;
    s[i] = home_slot(tb, key_hash<KD>(k[i]));
    any = any || open[i];
  }
  constexpr uint32_t kAhead = KD <= 3 ? 4 : 2;  // slots read at a time
  for (uint32_t step = 0; any && step < tb.nslots; step += kAhead) {
    Slot<S> x[kGroup][kAhead];
#pragma unroll
    for (uint32_t i = 0; i < kGroup; ++i) {
      if (!open[i]) continue;
#pragma unroll
      for (uint32_t a = 0; a < kAhead; ++a) {
        const uint32_t at = s[i] + a;
        x[i][a] = load_slot<S>(tb.words + (size_t)(at < tb.nslots ? at : at - tb.nslots) * S);
      }
    }
    any = false;
#pragma unroll
    for (uint32_t i = 0; i < kGroup; ++i) {
      if (!open[i]) continue;
#pragma unroll
      for (uint32_t a = 0; a < kAhead; ++a) {
        if (!open[i]) continue;
        const uint32_t st = x[i][a].w[S - 1];
        if (st == kEmpty) {
          open[i] = false;
        } else if (st < kPending && slot_holds<KD, S>(x[i][a], k[i])) {
          held[i] = true;
          open[i] = false;
        }
      }
      s[i] += kAhead;
      if (s[i] >= tb.nslots) s[i] -= tb.nslots;
      any = any || open[i];
    }
  }
}

// One bin's new keys: the lowest position of each key in the bin, where the
// table does not hold it.  All other entries get kPartLost.  An entry that
// finds the LDS table full is settled by a scan over the bin.  Bound like
// k_voxel_bins by arithmetic (the hash; VALU 50% busy) and LDS latency: 97 us at
// 10M keys, 1.7 TB/s.  A table that holds keys
// costs a lookup per key on top, which makes the general path the faster one;
// a captured insert may be replayed on one all the same.
template <int KD>
__global__ __launch_bounds__(kDedupThreads, 8) void k_insert_bins(PartPlan pl, TableRef tb, uint32_t table,
                                                                  const Meta* meta) {
  constexpr int S = kEntryWords<KD>;
  extern __shared__ uint32_t s_own[];
  const uint32_t base = pl.base[blockIdx.x];
  const uint32_t size = pl.base[blockIdx.x + 1] - base;
  const bool empty = meta->used == 0;  // (a bound on the occupied slots)
  uint32_t* ent = pl.entries + (size_t)base * S;
  for (uint32_t j = threadIdx.x; j < table / 4; j += kDedupThreads)
    reinterpret_cast<uint4*>(s_own)[j] = make_uint4(kNoSlot, kNoSlot, kNoSlot, kNoSlot);
  const BinTable t = bin_table(s_own, table, size);
  const auto lose = [&](uint32_t e, uint32_t p) { ent[(size_t)e * S + S - 1] = p | kPartLost; };
  // the keys' first positions in the batch, against the table
  const auto probe = [&](const uint32_t (&e)[kGroup], const Slot<S> (&x)[kGroup], bool (&open)[kGroup]) {
    int32_t k[kGroup][KD];
    bool held[kGroup];
#pragma unroll
    for (uint32_t i = 0; i < kGroup; ++i) entry_key<KD>(x[i], k[i]);
    table_holds<KD>(tb, k, open, held);
#pragma unroll
    for (uint32_t i = 0; i < kGroup; ++i)
      if (held[i]) lose(e[i], x[i].w[S - 1] & ~kPartLost);
  };
  __syncthreads();
  bool spilled[kGroup];
  uint32_t e[kGroup], at[kGroup];
  Slot<S> x[kGroup];
  bool open[kGroup];
  for (uint32_t g = 0; g < size; g += kGroup * kDedupThreads) {
#pragma unroll
    for (uint32_t i = 0; i < kGroup; ++i) {
      e[i] = g + i * kDedupThreads + threadIdx.x;
      spilled[i] = open[i] = e[i] < size;
      if (open[i]) x[i] = load_entry<KD>(ent, e[i]);
    }
    bin_place<KD, true>(t, ent, ~kPartLost, e, x, open, at, lose);
    bool any = false;
#pragma unroll
    for (uint32_t i = 0; i < kGroup; ++i) {
      spilled[i] = spilled[i] && at[i] == kNoSlot;
      if (!spilled[i]) continue;
      const uint32_t p = x[i].w[S - 1] & ~kPartLost;
      for (uint32_t o = 0; o < size && spilled[i]; ++o) {
        const Slot<S> y = load_entry<KD>(ent, o);
        bool eq = (y.w[S - 1] & ~kPartLost) < p;
#pragma unroll
        for (int d = 0; d < KD; ++d) eq = eq && y.w[d] == x[i].w[d];
        if (eq) {
          lose(e[i], p);
          spilled[i] = false;
        }
      }
      any = any || spilled[i];
    }
    if (any && !empty) probe(e, x, spilled);
  }
  if (empty) return;
  __syncthreads();
  for (uint32_t g = 0; g < table; g += kGroup * kDedupThreads) {
    bool any = false;
#pragma unroll
    for (uint32_t i = 0; i < kGroup; ++i) {
      const uint32_t own = s_own[g + i * kDedupThreads + threadIdx.x];
      open[i] = own != kNoSlot;
      e[i] = own & ((1u << t.num_bits) - 1u);
      if (open[i]) x[i] = load_entry<KD>(ent, e[i]);
      any = any || open[i];
    }
    if (any) probe(e, x, open);
  }
}

// The new keys' positions as bits with ranks within each range: a block reads
// its range's run of every bin and sets bits in LDS, then writes, per 64
// positions, the bits and the number of set bits before them in the range.
// Every entry's rank (with its range above it; kNoSlot for one that is no new
// key) goes to entry_rank, beside the entries, for the kernel that stores the
// bins: there a lookup of the bits by position missed the L2 for most keys.
// Also keeps the counters that the commit changes.  Bound by memory: 53 us at
// 10M keys, 4.4 TB/s (the entries' lines once more, for their last words).
template <int KD>
__global__ __launch_bounds__(1024) void k_part_collect(PartPlan pl, PartRanks pr, const Meta* meta) {
  constexpr int S = kEntryWords<KD>;
  constexpr uint32_t kLanes = 16, kRuns = 1024 / kLanes;  // lanes per run, runs at once
  constexpr uint32_t kRounds = 24;                        // rounds of runs whose first words stay in registers
  extern __shared__ uint32_t s_run[];  // [2][nbins]: first entry and end of each run
  __shared__ uint32_t s_bits[kPartMostPer / 32];
  __shared__ uint32_t s_pre[kPartMostPer / 64];
  __shared__ uint32_t s_wave[16];
  const uint32_t tid = threadIdx.x, lane = tid & (kLanes - 1u), run = tid / kLanes;
  const uint32_t range = range_of(pl, blockIdx.x);
  const uint32_t begin = min(pl.n, range * pl.per);
  const uint32_t end = min(pl.n, begin + pl.per);
  if (blockIdx.x == 0 && tid == 0) {
    pr.state->t = meta->t;
    pr.state->used = meta->used;
    pr.state->permuted = meta->permuted;
    pr.state->spilled = 0;
  }
  const uint32_t* row = pl.hist + (size_t)range * pl.nbins;
  const uint32_t* next = range + 1 < pl.nrange ? row + pl.nbins : pl.total;
  for (uint32_t b = tid; b < pl.nbins; b += 1024) {
    const uint32_t base = pl.base[b];
    s_run[b] = base + row[b];
    s_run[pl.nbins + b] = base + next[b];
  }
  for (uint32_t i = tid; i < kPartMostPer / 32; i += 1024) s_bits[i] = 0u;
  __syncthreads();
  const auto word = [&](uint32_t x) { return pl.entries[(size_t)x * S + S - 1]; };
  const auto set = [&](uint32_t w) {
    if (w & kPartLost) return;
    const uint32_t q = w - begin;
    atomicOr(&s_bits[q >> 5], 1u << (q & 31u));
  };
  const auto rank = [&](uint32_t x, uint32_t w) {
    uint32_t r = kNoSlot;
    if (!(w & kPartLost)) {
      const uint32_t q = w - begin;
      const uint64_t bits = ((uint64_t)s_bits[(q >> 6) * 2 + 1] << 32) | s_bits[(q >> 6) * 2];
      r = (range << 16) | (s_pre[q >> 6] + (uint32_t)__popcll(bits & ((1ull << (q & 63u)) - 1ull)));
    }
    pr.entry_rank[x] = r;
  };
  uint32_t held[kRounds][2];
#pragma unroll
  for (uint32_t u = 0; u < kRounds; ++u) {
    const uint32_t b = u * kRuns + run;
    held[u][0] = held[u][1] = kPartLost;
    if (b >= pl.nbins) continue;
    const uint32_t x = s_run[b] + lane, to = s_run[pl.nbins + b];
    if (x < to) held[u][0] = word(x);
    if (x + kLanes < to) held[u][1] = word(x + kLanes);
  }
#pragma unroll
  for (uint32_t u = 0; u < kRounds; ++u) {
    set(held[u][0]);
    set(held[u][1]);
  }
  for (uint32_t b = run; b < pl.nbins; b += kRuns) {
    const uint32_t skip = b < kRounds * kRuns ? 2 * kLanes : 0u;
    for (uint32_t x = s_run[b] + skip + lane; x < s_run[pl.nbins + b]; x += kLanes) set(word(x));
  }
  __syncthreads();
  uint32_t lo = 0, hi = 0;
  if (tid < kPartMostPer / 64) {
    lo = s_bits[2 * tid];
    hi = s_bits[2 * tid + 1];
  }
  const uint32_t own = __popc(lo) + __popc(hi);
  const uint32_t incl = wave_incl(own);
  if (lane_id() == 63) s_wave[tid >> 6] = incl;
  __syncthreads();
  uint32_t before = incl - own;
  for (uint32_t w = 0; w < (tid >> 6); ++w) before += s_wave[w];
  if (begin + 64 * tid < end) pr.recs[(begin >> 6) + tid] = make_uint4(lo, hi, before, 0u);
  s_pre[tid] = before;
  if (tid == 1023) pr.range_total[range] = before + own;
  __syncthreads();
#pragma unroll
  for (uint32_t u = 0; u < kRounds; ++u) {
    const uint32_t b = u * kRuns + run;
    if (b >= pl.nbins) continue;
    const uint32_t x = s_run[b] + lane, to = s_run[pl.nbins + b];
    if (x < to) rank(x, held[u][0]);
    if (x + kLanes < to) rank(x + kLanes, held[u][1]);
  }
  for (uint32_t b = run; b < pl.nbins; b += kRuns) {
    const uint32_t skip = b < kRounds * kRuns ? 2 * kLanes : 0u;
    for (uint32_t x = s_run[b] + skip + lane; x < s_run[pl.nbins + b]; x += kLanes) rank(x, word(x));
  }
}
static_assert(kPartMostPer / 64 == 1024, "a thread per 64 positions of a range");

// The ranks' bases: new keys before the range of position p, and in all.
// Every thread of a block of kThreads calls it once.
template <uint32_t kThreads>
__device__ __forceinline__ void range_bases(const PartPlan& pl, const PartRanks& pr, uint32_t range, uint32_t* s_two,
                                            uint32_t& before, uint32_t& total) {
  uint32_t a = 0, b = 0;
  for (uint32_t r = threadIdx.x; r < pl.nrange; r += kThreads) {
    const uint32_t v = pr.range_total[r];
    a += r < range ? v : 0u;
    b += v;
  }
  a = wave_sum_u32(a);
  b = wave_sum_u32(b);
  if (lane_id() == 0) {
    s_two[2 * (threadIdx.x >> 6)] = a;
    s_two[2 * (threadIdx.x >> 6) + 1] = b;
  }
  __syncthreads();
  before = 0;
  total = 0;
#pragma unroll
  for (uint32_t w = 0; w < kThreads / 64; ++w) {
    before += s_two[2 * w];
    total += s_two[2 * w + 1];
  }
}

__device__ __forceinline__ uint32_t rank_in(const uint4& rec, uint32_t p) {
  const uint64_t bits = ((uint64_t)rec.y << 32) | rec.x;
  return rec.z + (uint32_t)__popcll(bits & ((1ull << (p & 63u)) - 1ull));
}

// The insert's stream over the batch: new keys take i = h[t + rank], write
// k^B[i] and their rows, every position its index and mask.  Each tile knows
// its ranks from the range's totals, so tiles do not wait for each other.
// The first tile moves t; later kernels read the counters kept by collect.
// Bound by memory: 81 us at 10M new keys with 4-byte rows, 5.1 TB/s.
template <int KD, bool kInline>
__global__ __launch_bounds__(kBlock) void k_part_commit(PartPlan pl, PartRanks pr, TableRef tb,
                                                        const int32_t* __restrict__ keys, int32_t* __restrict__ kB,
                                                        const int32_t* __restrict__ heap, uint32_t cap, ValueSet vs,
                                                        int32_t* __restrict__ out_idx, uint8_t* __restrict__ out_mask,
                                                        Meta* meta, uint32_t* __restrict__ wlist) {
  __shared__ uint2 s_pairs[kInline ? kScanTile : 1];
  __shared__ uint32_t s_two[2 * (kBlock / 64)];
  const uint32_t base = blockIdx.x * kScanTile;
  const uint32_t t0 = pr.state->t;
  uint4 rec[kScanItems];
  int32_t k[kScanItems][KD];
  bool win[kScanItems];
  const BatchKeys<KD> src{keys};
#pragma unroll
  for (int r = 0; r < kScanItems; ++r) {
    const uint32_t p = base + r * kBlock + threadIdx.x;
    rec[r] = p < pl.n ? pr.recs[p >> 6] : make_uint4(0u, 0u, 0u, 0u);
    win[r] = (((p & 32u) ? rec[r].y : rec[r].x) >> (p & 31u)) & 1u;
    if (p < pl.n) src.load(p, k[r]);
  }
  uint32_t before, total;
  range_bases<kBlock>(pl, pr, base / pl.per, s_two, before, total);
  const bool overflow = total > cap - t0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (overflow) {
      meta->result = 0;
      __hip_atomic_fetch_or(&meta->status, kStatusCapacity, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      meta->t = t0 + total;
      raise_used(meta, total);  // a bound: tombstones may be taken
      meta->result = total;
    }
    publish_counts(tb, meta, pl.n);
  }
  const uint32_t first = before + pr.recs[base >> 6].z;  // the tile's first rank
  uint32_t wins = 0;
#pragma unroll
  for (int r = 0; r < kScanItems; ++r) {
    const uint32_t p = base + r * kBlock + threadIdx.x;
    if (p >= pl.n) continue;
    uint32_t i = kNoSlot;
    if (win[r] && !overflow) {
      const uint32_t rank = before + rank_in(rec[r], p);
      i = (uint32_t)heap[t0 + rank];
#pragma unroll
      for (int d = 0; d < KD; ++d) kB[(size_t)i * KD + d] = k[r][d];
      if constexpr (kInline) s_pairs[rank - first] = make_uint2(p, i);
      else if (wlist) wlist[rank] = p;
      ++wins;
    }
    const bool hit = i != kNoSlot;
    if (out_idx) out_idx[p] = hit ? (int32_t)i : -1;
    if (out_mask) out_mask[p] = hit ? 1 : 0;
  }
  if constexpr (kInline) {
    if (vs.n == 0) return;
    wins = wave_sum_u32(wins);
    __syncthreads();  // s_two is read no more
    if (lane_id() == 0) s_two[threadIdx.x >> 6] = wins;
    __syncthreads();
    uint32_t count = 0;
#pragma unroll
    for (uint32_t w = 0; w < kBlock / 64; ++w) count += s_two[w];
    for (int j = 0; j < vs.n; ++j) copy_rows(vs, j, s_pairs, count);
  }
}

// The buffer index of the new key of entry rank r.
struct RankIndex {
  const uint32_t* s_before;  // LDS: ranks before each range
  uint32_t t0;
  bool permuted;             // else h[i] = i from t on
  __device__ __forceinline__ uint32_t of(const int32_t* __restrict__ heap, uint32_t r) const {
    const uint32_t i = t0 + s_before[r >> 16] + (r & 0xFFFFu);
    return permuted ? (uint32_t)heap[i] : i;
  }
};

// The bins' new keys into the table.  A bin's home slots are a part of the
// table of its own: one block marks its slots that are taken in an LDS bitmap
// and gives each new key the first free slot (EMPTY or a tombstone) from its
// home on, as a claim would.  The slots are then written in their order, and
// into an empty table the EMPTY ones with them, as whole lines: random 16-byte
// stores took 161 us for 5M keys in 188 MB and 258 us for 10M in 384 MB.  The
// few keys that reach the end of the part go to the list `spill`, for
// k_place_spilled.  Bound by memory: 114 us for 10M in 384 MB, 5.1 TB/s, the rate
// of a large copy.
template <int KD>
__global__ __launch_bounds__(kDedupThreads) void k_place(PartPlan pl, PartRanks pr, TableRef tb,
                                                         const int32_t* __restrict__ heap, uint32_t cap,
                                                         uint32_t* __restrict__ spill, uint32_t stage) {
  constexpr int S = SlotWords<KD>::value;
  constexpr uint32_t kFree = 0xFFFFu, kStored = 0xFFFEu;  // no entry's key goes here; it is there already
  extern __shared__ uint4 s_lds4[];  // `stage` slots, a bit per slot, nrange + 1 bases, 16 bits per slot
  uint32_t* s_stage = reinterpret_cast<uint32_t*>(s_lds4);
  uint32_t* s_taken = s_stage + stage * S;
  __shared__ uint32_t s_wave[kDedupThreads / 64];
  const uint32_t tid = threadIdx.x;
  const uint32_t lo = (blockIdx.x << pl.shift) * tb.bucket_width;
  const uint32_t whole = tb.bucket_width << pl.shift;
  const uint32_t region = min(tb.nslots - lo, whole);
  const uint32_t words = (whole + 31u) / 32u;
  uint32_t* s_before = s_taken + words;
  uint16_t* s_entry = reinterpret_cast<uint16_t*>(s_before + pl.nrange + 1);
  block_scan_into<kDedupThreads, kPartRanges>(pr.range_total, pl.nrange, s_before, s_wave);
  const uint32_t t0 = pr.state->t;
  if (s_before[pl.nrange] > cap - t0) return;  // the batch overflows: nothing is stored
  const bool empty = pr.state->used == 0;
  const uint32_t base = pl.base[blockIdx.x];
  const uint32_t size = pl.base[blockIdx.x + 1] - base;
  const uint32_t* __restrict__ ent = pl.entries + (size_t)base * S;
  for (uint32_t w = tid; w < words; w += kDedupThreads) {
    const uint32_t first = w * 32u;
    s_taken[w] = first + 32u <= region ? 0u : first >= region ? ~0u : ~0u << (region - first);
  }
  for (uint32_t w = tid; w < (region + 1u) / 2u; w += kDedupThreads) reinterpret_cast<uint32_t*>(s_entry)[w] = ~0u;
  __syncthreads();
  if (!empty) {
    for (uint32_t s = tid; s < region; s += kDedupThreads) {
      const uint32_t st = tb.words[(size_t)(lo + s) * S + S - 1];
      if (st < kTomb) atomicOr(&s_taken[s >> 5], 1u << (s & 31u));
    }
    __syncthreads();
  }
  const RankIndex index{s_before, t0, pr.state->permuted != 0};
  // (four entries of a thread at a time: their loads overlap)
  const uint32_t* __restrict__ rank = pr.entry_rank + base;
  for (uint32_t g = 0; g < size; g += 4 * kDedupThreads) {
    Slot<S> x[4];
    uint32_t r[4];
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
      const uint32_t e = g + i * kDedupThreads + tid;
      r[i] = kNoSlot;
      if (e < size) {
        r[i] = rank[e];
        x[i] = load_entry<KD>(ent, e);
      }
    }
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
      const uint32_t e = g + i * kDedupThreads + tid;
      if (r[i] == kNoSlot) continue;
      int32_t k[KD];
      entry_key<KD>(x[i], k);
      uint32_t at = home_slot(tb, key_hash<KD>(k)) - lo;
      while (at < region) {
        const uint32_t w = at >> 5;
        const uint32_t seen = __hip_atomic_load(&s_taken[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const uint32_t free = ~seen & (~0u << (at & 31u));
        if (free == 0u) {
          at = (w + 1u) << 5;
          continue;
        }
        at = (w << 5) + (uint32_t)__ffs((int)free) - 1u;
        const uint32_t bit = 1u << (at & 31u);
        if (!(atomicOr(&s_taken[w], bit) & bit)) break;
      }
      if (at >= region) {
        spill[atomic_add_u32(&pr.state->spilled, 1u)] = base + e;
        continue;
      }
      const Slot<S> c = committed_slot<KD, S>(k, index.of(heap, r[i]));
      if (e < stage) {
        s_entry[at] = (uint16_t)e;
        store_slot<S>(s_stage + e * S, c);
      } else {  // (the end of a bin larger than the stage)
        s_entry[at] = (uint16_t)kStored;
        store_slot<S>(tb.words + (size_t)(lo + at) * S, c);
      }
    }
  }
  __syncthreads();
  for (uint32_t i = tid; i < region; i += kDedupThreads) {
    const uint32_t e = s_entry[i];
    Slot<S> out;
#pragma unroll
    for (int q = 0; q < S; ++q) out.w[q] = kEmpty;
    if (e < stage) out = load_slot<S>(s_stage + e * S);
    if (e < stage || (empty && e == kFree)) store_slot<S>(tb.words + (size_t)(lo + i) * S, out);
  }
}

// The keys that found no free slot in their part: a CAS on the first free slot
// after it (every slot from their home to there is taken).
template <int KD>
__global__ __launch_bounds__(kBlock) void k_place_spilled(PartPlan pl, PartRanks pr, TableRef tb,
                                                          const int32_t* __restrict__ heap,
                                                          const uint32_t* __restrict__ spill, Meta* meta) {
  constexpr int S = SlotWords<KD>::value;
  __shared__ uint32_t s_before[kPartRanges + 1];
  __shared__ uint32_t s_wave[kBlock / 64];
  const uint32_t n = pr.state->spilled;
  if (blockIdx.x * kBlock >= n) return;
  block_scan_into<kBlock, kPartRanges>(pr.range_total, pl.nrange, s_before, s_wave);
  const RankIndex index{s_before, pr.state->t, pr.state->permuted != 0};
  for (uint32_t q = blockIdx.x * kBlock + threadIdx.x; q < n; q += gridDim.x * kBlock) {
    const Slot<S> x = load_entry<KD>(pl.entries, spill[q]);
    const uint32_t i = index.of(heap, pr.entry_rank[spill[q]]);
    int32_t k[KD];
    entry_key<KD>(x, k);
    const uint64_t desired = ((uint64_t)i << 32) | (uint32_t)k[KD - 1];
    const uint64_t h = key_hash<KD>(k);
    uint64_t s64 = ((uint64_t)bin_of(pl, h) + 1u) * ((uint64_t)tb.bucket_width << pl.shift);
    uint32_t s = s64 >= tb.nslots ? 0u : (uint32_t)s64;
    bool done = false;
    for (uint32_t step = 0; step < tb.nslots && !done; ++step) {
      uint64_t* pair = reinterpret_cast<uint64_t*>(tb.words + (size_t)s * S + S - 2);
      uint64_t seen = __hip_atomic_load(pair, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      while ((uint32_t)(seen >> 32) >= kTomb && !done) {  // EMPTY or a tombstone
        const uint64_t found = cas_pair(reinterpret_cast<uint32_t*>(pair), seen, desired);
        done = found == seen;
        seen = found;
      }
      if (done) {
        const Slot<S> c = committed_slot<KD, S>(k, i);
#pragma unroll
        for (int w = 0; w < S - 2; ++w) tb.words[(size_t)s * S + w] = c.w[w];
      }
      if (++s == tb.nslots) s = 0;
    }
    if (!done) __hip_atomic_fetch_or(&meta->status, kStatusTableFull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

inline uint32_t cdiv(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

constexpr uint32_t kMostLds = 160 * 1024 - 256;  // (the kernels' static LDS is under 256 bytes)

// Lets a kernel be launched with up to kMostLds of dynamic LDS.  The limit
// belongs to the kernel and not to a launch, and several host threads may be
// launching it on batches of different sizes, so it is always set to the same
// value; and before a call's first kernel, so that a failure changes nothing.
template <typename K>
hipError_t allow_lds(K* kernel) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)kMostLds);
}

// LDS of a scatter in tiles of `items` positions per thread.
template <int KD>
uint32_t scatter_lds(const PartPlan& pl, uint32_t items) {
  return items * ((KD + 1) * 4 + 2) * kCountThreads + (2 * pl.nbins + 1) * 4;
}

// Tiles of 8 positions per thread where they fit the LDS beside the bins' counters, else of 4.
template <int KD>
bool wide_tiles(const PartPlan& pl) {
  return KD <= 3 && scatter_lds<KD>(pl, 8) <= kMostLds;
}

template <int KD, typename Src, bool kVoxel>
hipError_t allow_scatter_lds(const PartPlan& pl) {
  return wide_tiles<KD>(pl) ? allow_lds(k_part_scatter<KD, Src, kVoxel, KD <= 3 ? 8 : 4>)
                            : allow_lds(k_part_scatter<KD, Src, kVoxel, 4>);
}

template <int KD, typename Src, bool kVoxel, uint32_t kItems>
hipError_t scatter(const Src& src, const PartPlan& pl, const uint32_t* link, hipStream_t st) {
  hipLaunchKernelGGL((k_part_scatter<KD, Src, kVoxel, kItems>), dim3(pl.nrange), dim3(kCountThreads),
                     scatter_lds<KD>(pl, kItems), st, src, pl, link);
  return hipGetLastError();
}

template <int KD, typename Src, bool kVoxel>
hipError_t partition(const Src& src, const PartPlan& pl, uint32_t* link, uint32_t* zero, uint32_t n_zero, Meta* meta,
                     hipStream_t st) {
  if (pl.n == 0 || pl.nrange == 0 || pl.nrange % 8 != 0 || pl.nrange > kPartRanges || pl.nbins == 0 ||
      pl.nbins > kPartBins || pl.per % kPartTile != 0 || (uint64_t)pl.nrange * pl.per < pl.n)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_part_count<KD, Src, kVoxel>), dim3(pl.nrange), dim3(kCountThreads), pl.nbins * 4, st, src, pl,
                     link, zero, n_zero, meta);
  hipLaunchKernelGGL(k_part_scan, dim3(cdiv(pl.nbins, 64)), dim3(1024), 0, st, pl);
  return wide_tiles<KD>(pl) ? scatter<KD, Src, kVoxel, KD <= 3 ? 8 : 4>(src, pl, link, st)
                            : scatter<KD, Src, kVoxel, 4>(src, pl, link, st);
}

}  // namespace

namespace {

constexpr uint32_t kInsertTable = 16384;  // about half full of a mean bin's keys at most
static_assert(kInsertTable % (kGroup * kDedupThreads) == 0, "whole groups of table entries");

template <int KD>
hipError_t insert_settle(const PartPlan& pl, const PartRanks& pr, const TableRef& tb, const int32_t* keys, Meta* meta,
                         hipStream_t st) {
  hipError_t e = allow_scatter_lds<KD, BatchKeys<KD>, false>(pl);
  if (e == hipSuccess) e = allow_lds(k_place<KD>);
  if (e != hipSuccess) return e;
  e = partition<KD, BatchKeys<KD>, false>(BatchKeys<KD>{keys}, pl, nullptr, nullptr, 0, meta, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_insert_bins<KD>, dim3(pl.nbins), dim3(kDedupThreads), kInsertTable * 4, st, pl, tb,
                     kInsertTable, meta);
  hipLaunchKernelGGL(k_part_collect<KD>, dim3(pl.nrange), dim3(1024), pl.nbins * 8, st, pl, pr, meta);
  return hipGetLastError();
}

template <int KD>
hipError_t insert_store(const PartPlan& pl, const PartRanks& pr, const TableRef& tb, const int32_t* keys, int32_t* kB,
                        const int32_t* heap, uint32_t cap, const ValueSet& vs, int32_t* out_idx, uint8_t* out_mask,
                        Meta* meta, uint32_t* wlist, uint32_t* spill, hipStream_t st) {
  const dim3 tiles(cdiv(pl.n, kScanTile));
  if (wlist)
    hipLaunchKernelGGL((k_part_commit<KD, false>), tiles, dim3(kBlock), 0, st, pl, pr, tb, keys, kB, heap, cap, vs,
                       out_idx, out_mask, meta, wlist);
  else
    hipLaunchKernelGGL((k_part_commit<KD, true>), tiles, dim3(kBlock), 0, st, pl, pr, tb, keys, kB, heap, cap, vs,
                       out_idx, out_mask, meta, wlist);
  const uint32_t region = tb.bucket_width << pl.shift;
  const uint32_t words = (region + 31u) / 32u + pl.nrange + 1 + (region + 1u) / 2u;
  // the stage: what a bin is unlikely to exceed, as far as the LDS goes
  const uint32_t mean = cdiv((uint64_t)pl.n << pl.shift, pl.nbuckets);
  const uint32_t slot = SlotWords<KD>::value * 4;
  const uint32_t stage = std::min((kMostLds - words * 4) / slot, mean + mean / 8 + 64) & ~3u;
  const uint32_t lds = stage * slot + words * 4;
  hipLaunchKernelGGL(k_place<KD>, dim3(pl.nbins), dim3(kDedupThreads), lds, st, pl, pr, tb, heap, cap, spill,
                     stage);
  hipLaunchKernelGGL(k_place_spilled<KD>, dim3(256), dim3(kBlock), 0, st, pl, pr, tb, heap, spill, meta);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_insert_settle(int kd, const PartPlan& pl, const PartRanks& pr, const TableRef& tb,
                                const int32_t* keys, Meta* meta, hipStream_t st) {
  switch (kd) {
    case 1: return insert_settle<1>(pl, pr, tb, keys, meta, st);
    case 2: return insert_settle<2>(pl, pr, tb, keys, meta, st);
    case 3: return insert_settle<3>(pl, pr, tb, keys, meta, st);
    case 4: return insert_settle<4>(pl, pr, tb, keys, meta, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_insert_store(int kd, const PartPlan& pl, const PartRanks& pr, const TableRef& tb,
                               const int32_t* keys, int32_t* kB, const int32_t* heap, uint32_t cap, const ValueSet& vs,
                               int32_t* out_idx, uint8_t* out_mask, Meta* meta, uint32_t* wlist, uint32_t* spill,
                               hipStream_t st) {
  switch (kd) {
    case 1: return insert_store<1>(pl, pr, tb, keys, kB, heap, cap, vs, out_idx, out_mask, meta, wlist, spill, st);
    case 2: return insert_store<2>(pl, pr, tb, keys, kB, heap, cap, vs, out_idx, out_mask, meta, wlist, spill, st);
    case 3: return insert_store<3>(pl, pr, tb, keys, kB, heap, cap, vs, out_idx, out_mask, meta, wlist, spill, st);
    case 4: return insert_store<4>(pl, pr, tb, keys, kB, heap, cap, vs, out_idx, out_mask, meta, wlist, spill, st);
    default: return hipErrorInvalidValue;
  }
}

bool part_buckets(PartPlan* pl, uint32_t nbuckets, uint32_t bucket_width) {
  pl->nbuckets = nbuckets;
  pl->shift = 0;
  const auto bins = [&] { return (uint32_t)(((uint64_t)nbuckets + (1ull << pl->shift) - 1) >> pl->shift); };
  // the largest bins of at most kInsertBinMean positions on average (more than one per CU from 2.6M on)
  const uint64_t most = (uint64_t)kInsertBinMean * nbuckets;
  while (pl->shift < 31 && (uint64_t)pl->n << (pl->shift + 1) <= most) ++pl->shift;
  pl->nbins = bins();
  // a table of few buckets (of a few thousand slots, against at least 2.6M
  // positions) has no bins that small: entries beyond a bin's LDS table are
  // settled by a scan of the bin, quadratic in what does not fit it
  if ((uint64_t)pl->n << pl->shift > most) return false;
  // a bin's part of the table has a bit per slot in LDS
  return pl->nbins <= kPartBins && ((uint64_t)bucket_width << pl->shift) <= kPartMostRegion;
}

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
  const uint32_t tiles = cdiv(pl.n, kScanTile), number = cdiv(pl.n, kNumberTile);
  const VoxelKeys src{pts, voxel};
  hipError_t e = allow_scatter_lds<3, VoxelKeys, true>(pl);
  if (e == hipSuccess) e = allow_lds(k_voxel_bins);
  if (e != hipSuccess) return e;
  e = partition<3, VoxelKeys, true>(src, pl, link, reinterpret_cast<uint32_t*>(status), number * 2,
                                               meta, st);
  if (e != hipSuccess) return e;
  constexpr uint32_t table = 8192;  // about half full of a mean bin's voxels at most
  const uint32_t places = table / 4 * 3;
  const uint32_t lds = table * 8 + places * 2;
  hipLaunchKernelGGL(k_voxel_bins, dim3(pl.nbins), dim3(kDedupThreads), lds, st, pl, table, places, link);
  hipLaunchKernelGGL(k_voxel_number, dim3(number), dim3(kNumberThreads), 0, st, src, pl.n, link, voxel_keys, counts,
                     point_voxel, meta, status);
  hipLaunchKernelGGL(k_voxel_follow, dim3(tiles), dim3(kBlock), 0, st, pl.n, link, point_voxel);
  return hipGetLastError();
}

}  // namespace ash

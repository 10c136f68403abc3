// ash_small.hip -- batches of up to 2048 positions in one block.
//
// A batch this small is all latency: two launches, and in each a chain of
// dependent memory accesses with little else to run meanwhile.  One block of
// 1024 threads holds the whole batch in LDS, so the copies of a key are
// dropped there, the new keys (or the erased ones) are ranked with block
// barriers instead of a look-back, and nothing goes through scratch memory.
// One launch per call, and the table is written only once it is known that the
// batch fits.  Which batches come here, with both sides' times: one_block in
// ash_api.hip.
#include "ash_device.hpp"
#include "ash_launch.hpp"

namespace ash {

namespace {

constexpr uint32_t kThreads = 1024;
constexpr uint32_t kAllWaves = kThreads / 64;

template <int KD, uint32_t kItems>
struct SmallLds {
  uint32_t key[KD][kItems * kThreads];
  uint32_t tab[2 * kItems * kThreads];  // position that holds each key
  int32_t heap[kItems * kThreads];      // h[t ..), the indices this batch may take
  uint32_t count[kItems * kAllWaves];   // flagged positions per 64, then before them
  uint32_t total;
};

// rep[r]: whether this thread's position r * 1024 + threadIdx.x is the first
// of its key (exact: every key finds its entry).
template <int KD, uint32_t kItems>
__device__ __forceinline__ void small_first(SmallLds<KD, kItems>& s, const int32_t (&k)[kItems][KD],
                                            const uint64_t (&h)[kItems], uint32_t n, bool (&rep)[kItems]) {
  constexpr uint32_t kMask = 2 * kItems * kThreads - 1;
#pragma unroll
  for (uint32_t r = 0; r < kItems; ++r)
#pragma unroll
    for (int d = 0; d < KD; ++d) s.key[d][r * kThreads + threadIdx.x] = (uint32_t)k[r][d];
#pragma unroll
  for (uint32_t r = 0; r < 2 * kItems; ++r) s.tab[r * kThreads + threadIdx.x] = kNoSlot;
  __syncthreads();
  uint32_t at[kItems];
#pragma unroll
  for (uint32_t r = 0; r < kItems; ++r) {
    const uint32_t pos = r * kThreads + threadIdx.x;
    at[r] = (uint32_t)(h[r] >> 9) & kMask;
    if (pos >= n) continue;
    while (true) {  // at most half as many keys as entries: ends at a free or matching one
      const uint32_t o = atomicCAS(&s.tab[at[r]], kNoSlot, pos);
      if (o == kNoSlot) break;
      bool eq = true;
#pragma unroll
      for (int d = 0; d < KD; ++d) eq = eq && s.key[d][o] == (uint32_t)k[r][d];
      if (eq) {
        atomicMin(&s.tab[at[r]], pos);  // (the entry's key stays the same)
        break;
      }
      at[r] = (at[r] + 1u) & kMask;
    }
  }
  __syncthreads();
#pragma unroll
  for (uint32_t r = 0; r < kItems; ++r) rep[r] = r * kThreads + threadIdx.x < n && s.tab[at[r]] == r * kThreads + threadIdx.x;
}

// Ranks of the flagged positions in batch order; returns their number.
template <int KD, uint32_t kItems>
__device__ __forceinline__ uint32_t small_ranks(SmallLds<KD, kItems>& s, const bool (&flag)[kItems],
                                                uint32_t (&rank)[kItems]) {
  const uint32_t wave = threadIdx.x >> 6;
  uint64_t bits[kItems];
#pragma unroll
  for (uint32_t r = 0; r < kItems; ++r) {
    bits[r] = __ballot(flag[r]);
    if (lane_id() == 0) s.count[r * kAllWaves + wave] = (uint32_t)__popcll(bits[r]);
  }
  __syncthreads();
  static_assert(kItems * kAllWaves <= 64, "one wave scans the counts");
  if (wave == 0) {
    const uint32_t own = lane_id() < kItems * kAllWaves ? s.count[lane_id()] : 0u;
    uint32_t v = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(v, o, 64);
      if (lane_id() >= (uint32_t)o) v += y;
    }
    if (lane_id() < kItems * kAllWaves) s.count[lane_id()] = v - own;
    if (lane_id() == 63) s.total = v;
  }
  __syncthreads();
#pragma unroll
  for (uint32_t r = 0; r < kItems; ++r)
    rank[r] = s.count[r * kAllWaves + wave] + (uint32_t)__popcll(bits[r] & ((1ull << lane_id()) - 1ull));
  return s.total;
}

// Four slots (64 bytes up to key width 3) of a probe sequence from slot s on.
template <int KD>
struct Ahead {
  static constexpr int S = SlotWords<KD>::value;
  static constexpr uint32_t kSlots = KD <= 3 ? 4 : 2;
  Slot<S> x[kSlots];
  __device__ __forceinline__ void load(const TableRef& tb, uint32_t s) {
#pragma unroll
    for (uint32_t a = 0; a < kSlots; ++a) x[a] = load_slot<S>(tb.words + (size_t)wrap(tb, s + a) * S);
  }
  static __device__ __forceinline__ uint32_t wrap(const TableRef& tb, uint32_t s) {
    return s < tb.nslots ? s : s - tb.nslots;
  }
  // the slots a key may take: EMPTY ones and tombstones
  __device__ __forceinline__ uint32_t free_mask() const {
    uint32_t m = 0;
#pragma unroll
    for (uint32_t a = 0; a < kSlots; ++a) m |= x[a].w[S - 1] >= kTomb ? 1u << a : 0u;
    return m;
  }
};

// What a key's probe sequence holds, up to its first EMPTY slot: the slot and
// state of the committed copy, and the first slots the key may take (those of
// `free` from `from` on; none seen: the table is full).
struct Probe {
  uint32_t slot = kNoSlot, index = kNoSlot;
  uint32_t from = 0, free = 0;
};

template <int KD>
__device__ __forceinline__ Probe small_probe(const TableRef& tb, const int32_t (&k)[KD], uint64_t h) {
  using A = Ahead<KD>;
  Probe f;
  uint32_t s = home_slot(tb, h);
  for (uint32_t step = 0; step < tb.nslots; step += A::kSlots) {
    A a;
    a.load(tb, s);
    if (f.free == 0u) {
      f.from = s;
      f.free = a.free_mask();
    }
#pragma unroll
    for (uint32_t i = 0; i < A::kSlots; ++i) {
      const uint32_t st = a.x[i].w[A::S - 1];
      if (st == kEmpty) return f;
      if (st < kPending && slot_holds<KD, A::S>(a.x[i], k)) {
        f.slot = A::wrap(tb, s + i);
        f.index = st;
        return f;
      }
    }
    s = A::wrap(tb, s + A::kSlots);
  }
  return f;
}

// The slot a new key takes: the first free one of its sequence that no other
// key of the batch has taken.  Only this block writes the table, so the taken
// slots are a set in LDS (tab, all kNoSlot at first) and the slot itself needs
// no atomic: keys whose homes coincide settle in LDS instead of one
// compare-and-swap in memory after another.
template <int KD, uint32_t kItems>
__device__ __forceinline__ uint32_t small_take(SmallLds<KD, kItems>& s, const TableRef& tb, Probe f) {
  using A = Ahead<KD>;
  constexpr uint32_t kMask = 2 * kItems * kThreads - 1;
  for (uint32_t step = 0; step < tb.nslots; step += A::kSlots) {
    while (f.free != 0u) {
      const uint32_t slot = A::wrap(tb, f.from + (uint32_t)__ffs((int)f.free) - 1u);
      f.free &= f.free - 1u;
      uint32_t j = (slot * 0x9e3779b1u) >> 7 & kMask;
      uint32_t o;
      while ((o = atomicCAS(&s.tab[j], kNoSlot, slot)) != kNoSlot && o != slot) j = (j + 1u) & kMask;
      if (o == kNoSlot) return slot;
    }
    f.from = A::wrap(tb, f.from + A::kSlots);
    A a;
    a.load(tb, f.from);
    f.free = a.free_mask();
  }
  return kNoSlot;
}

// An insert or activate of n <= kItems * 1024 positions.
template <int KD, uint32_t kItems, bool kInline>
__global__ __launch_bounds__(kThreads) void k_insert_small(TableRef tb, BatchKeys<KD> src, uint32_t n,
                                                           int32_t* __restrict__ kB, const int32_t* __restrict__ heap,
                                                           uint32_t cap, ValueSet vs, int32_t* __restrict__ out_idx,
                                                           uint8_t* __restrict__ out_mask, Meta* meta,
                                                           uint32_t* __restrict__ wlist) {
  constexpr int S = SlotWords<KD>::value;
  __shared__ SmallLds<KD, kItems> s;
  __shared__ uint2 s_pairs[kInline ? kItems * kThreads : 1];
  const uint32_t tid = threadIdx.x;
  int32_t k[kItems][KD];
  uint64_t h[kItems];
  bool rep[kItems], win[kItems];
  Probe f[kItems];
#pragma unroll
  for (uint32_t r = 0; r < kItems; ++r)
    if (r * kThreads + tid < n) src.load(r * kThreads + tid, k[r]);
  const uint32_t t0 = meta->t;
#pragma unroll
  for (uint32_t r = 0; r < kItems; ++r) {
    const uint32_t pos = r * kThreads + tid;
    if (pos < n && pos < cap - t0) s.heap[pos] = heap[t0 + pos];
    h[r] = key_hash<KD>(k[r]);
  }
  small_first<KD, kItems>(s, k, h, n, rep);
  bool full = false;
#pragma unroll
  for (uint32_t r = 0; r < kItems; ++r) {
    win[r] = false;
    if (!rep[r]) continue;
    f[r] = small_probe<KD>(tb, k[r], h[r]);
    win[r] = f[r].slot == kNoSlot;
    full = full || (win[r] && f[r].free == 0u);
  }
  const bool table_full = __syncthreads_or(full);
#pragma unroll
  for (uint32_t r = 0; r < 2 * kItems; ++r) s.tab[r * kThreads + tid] = kNoSlot;  // (the ranks' barriers follow)
  uint32_t rank[kItems];
  const uint32_t total = small_ranks<KD, kItems>(s, win, rank);
  const bool overflow = table_full || total > cap - t0;
#pragma unroll
  for (uint32_t r = 0; r < kItems; ++r) {
    const uint32_t p = r * kThreads + tid;
    if (p >= n) continue;
    const bool in = win[r] && !overflow;
    uint32_t i = kNoSlot;
    if (in) {
      i = (uint32_t)s.heap[rank[r]];
      const uint32_t at = small_take<KD, kItems>(s, tb, f[r]);  // (fewer live keys than slots: there is one)
      if (at != kNoSlot) store_slot<S>(tb.words + (size_t)at * S, committed_slot<KD, S>(k[r], i));
#pragma unroll
      for (int d = 0; d < KD; ++d) kB[(size_t)i * KD + d] = k[r][d];
      if constexpr (kInline) s_pairs[rank[r]] = make_uint2(p, i);
      else if (wlist) wlist[rank[r]] = p;
    }
    if (out_idx) out_idx[p] = in ? (int32_t)i : -1;
    if (out_mask) out_mask[p] = in ? 1 : 0;
  }
  if constexpr (kInline) {
    if (vs.n > 0 && !overflow) {
      __syncthreads();
      for (int j = 0; j < vs.n; ++j) copy_rows(vs, j, s_pairs, total);
    }
  }
  if (tid == 0) {
    if (overflow) {
      meta->result = 0;
      __hip_atomic_fetch_or(&meta->status, table_full ? kStatusTableFull : kStatusCapacity, __ATOMIC_RELAXED,
                            __HIP_MEMORY_SCOPE_AGENT);
    } else {
      meta->t = t0 + total;
      raise_used(meta, total);  // a bound: tombstones may be taken
      meta->result = total;
    }
    publish_counts(tb, meta, n);
  }
}

// An erase of n <= kItems * 1024 positions.
template <int KD, uint32_t kItems>
__global__ __launch_bounds__(kThreads) void k_erase_small(TableRef tb, BatchKeys<KD> src, uint32_t n,
                                                          int32_t* __restrict__ heap, uint8_t* __restrict__ out_mask,
                                                          Meta* meta) {
  constexpr int S = SlotWords<KD>::value;
  __shared__ SmallLds<KD, kItems> s;
  const uint32_t tid = threadIdx.x;
  int32_t k[kItems][KD];
  uint64_t h[kItems];
  bool rep[kItems], win[kItems];
  Probe f[kItems];
#pragma unroll
  for (uint32_t r = 0; r < kItems; ++r)
    if (r * kThreads + tid < n) src.load(r * kThreads + tid, k[r]);
  const uint32_t t0 = meta->t;
#pragma unroll
  for (uint32_t r = 0; r < kItems; ++r) h[r] = key_hash<KD>(k[r]);
  small_first<KD, kItems>(s, k, h, n, rep);
#pragma unroll
  for (uint32_t r = 0; r < kItems; ++r) {
    if (rep[r]) f[r] = small_probe<KD>(tb, k[r], h[r]);
    win[r] = rep[r] && f[r].slot != kNoSlot;
  }
  uint32_t rank[kItems];
  const uint32_t total = small_ranks<KD, kItems>(s, win, rank);
#pragma unroll
  for (uint32_t r = 0; r < kItems; ++r) {
    const uint32_t p = r * kThreads + tid;
    if (p >= n) continue;
    if (win[r] && rank[r] < t0) {  // erased keys are distinct live ones: always true
      heap[t0 - 1u - rank[r]] = (int32_t)f[r].index;
      tb.words[(size_t)f[r].slot * S + S - 1] = kTomb;
    }
    if (out_mask) out_mask[p] = win[r] ? 1 : 0;
  }
  if (tid == 0) {
    meta->t = t0 - total;
    meta->tombs += total;
    meta->result = total;
    meta->permuted = 1;
    publish_counts(tb, meta);
  }
}

template <int KD, uint32_t kItems>
void insert_items(const TableRef& tb, const int32_t* keys, uint32_t n, int32_t* kB, const int32_t* heap, uint32_t cap,
                  const ValueSet& vs, int32_t* out_idx, uint8_t* out_mask, Meta* meta, uint32_t* wlist,
                  hipStream_t st) {
  if (wlist)
    hipLaunchKernelGGL((k_insert_small<KD, kItems, false>), dim3(1), dim3(kThreads), 0, st, tb, BatchKeys<KD>{keys}, n,
                       kB, heap, cap, vs, out_idx, out_mask, meta, wlist);
  else
    hipLaunchKernelGGL((k_insert_small<KD, kItems, true>), dim3(1), dim3(kThreads), 0, st, tb, BatchKeys<KD>{keys}, n,
                       kB, heap, cap, vs, out_idx, out_mask, meta, wlist);
}

template <int KD>
hipError_t insert_small(const TableRef& tb, const int32_t* keys, uint32_t n, int32_t* kB, const int32_t* heap,
                        uint32_t cap, const ValueSet& vs, int32_t* out_idx, uint8_t* out_mask, Meta* meta,
                        uint32_t* wlist, hipStream_t st) {
  if (n > kSmallBatch) return hipErrorInvalidValue;
  if (n <= kThreads) insert_items<KD, 1>(tb, keys, n, kB, heap, cap, vs, out_idx, out_mask, meta, wlist, st);
  else insert_items<KD, 2>(tb, keys, n, kB, heap, cap, vs, out_idx, out_mask, meta, wlist, st);
  return hipGetLastError();
}

template <int KD>
hipError_t erase_small(const TableRef& tb, const int32_t* keys, uint32_t n, int32_t* heap, uint8_t* out_mask,
                       Meta* meta, hipStream_t st) {
  if (n > kSmallBatch) return hipErrorInvalidValue;
  const BatchKeys<KD> src{keys};
  if (n <= kThreads)
    hipLaunchKernelGGL((k_erase_small<KD, 1>), dim3(1), dim3(kThreads), 0, st, tb, src, n, heap, out_mask, meta);
  else
    hipLaunchKernelGGL((k_erase_small<KD, 2>), dim3(1), dim3(kThreads), 0, st, tb, src, n, heap, out_mask, meta);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_insert_small(int kd, const TableRef& tb, const int32_t* keys, uint32_t n, int32_t* kB,
                               const int32_t* heap, uint32_t cap, const ValueSet& vs, int32_t* out_idx,
                               uint8_t* out_mask, Meta* meta, uint32_t* wlist, hipStream_t st) {
  switch (kd) {
    case 1: return insert_small<1>(tb, keys, n, kB, heap, cap, vs, out_idx, out_mask, meta, wlist, st);
    case 2: return insert_small<2>(tb, keys, n, kB, heap, cap, vs, out_idx, out_mask, meta, wlist, st);
    case 3: return insert_small<3>(tb, keys, n, kB, heap, cap, vs, out_idx, out_mask, meta, wlist, st);
    case 4: return insert_small<4>(tb, keys, n, kB, heap, cap, vs, out_idx, out_mask, meta, wlist, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_erase_small(int kd, const TableRef& tb, const int32_t* keys, uint32_t n, int32_t* heap,
                              uint8_t* out_mask, Meta* meta, hipStream_t st) {
  switch (kd) {
    case 1: return erase_small<1>(tb, keys, n, heap, out_mask, meta, st);
    case 2: return erase_small<2>(tb, keys, n, heap, out_mask, meta, st);
    case 3: return erase_small<3>(tb, keys, n, heap, out_mask, meta, st);
    case 4: return erase_small<4>(tb, keys, n, heap, out_mask, meta, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ash

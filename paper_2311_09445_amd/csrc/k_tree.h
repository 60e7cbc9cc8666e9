// Second half of a priority update: the tree pass (alone, or beside the row gather and the weights).
// Part of per_kernels.hip (included inside namespace per, in the order given there); not a stand-alone header.

// ---------------------------------------------------------------------------------
// priority update: claim (last writer), then one tree pass
// ---------------------------------------------------------------------------------
// Heights 1 .. hb of the tree pass at fixed kernel-argument offsets (slot j = height j + 1).
constexpr int kSubSlots = 13;
struct SubLevels {
  float* ptr[kSubSlots];          // that height of tree 0
  uint32_t stride[kSubSlots];     // floats between trees
  uint32_t n[kSubSlots];          // real nodes of that height
  uint32_t lds_off[kSubSlots];    // where the workgroup keeps its part of that height (floats)
  uint32_t lds_floats;            // total
  uint32_t list_cap;              // height-1 nodes under one workgroup root: entries of the workgroup's node list
  uint32_t hb;
  uint32_t group_batch;           // size of the batch if it claimed through the group entries, else 0
};

// Tree pass.  Workgroup b of tree t owns the subtree under node b of height hb and keeps the
// subtree's nodes of heights 1 .. hb in LDS.
//  0. In one trip it fetches its height-1 nodes, the dirty bits of the leaves below them and the
//     entries of their claim groups.
//  1. Each height-1 node with a claimed leaf (a dirty bit, or the leaf of a group entry written by
//     this batch) is rebuilt by LPS lanes: they read its K leaves and, for the dirty ones only,
//     the stamp entry, whose lower word is the value of the batch element that won that leaf; it
//     replaces the leaf (and is stored), and so does the value of the group entry, which wins
//     against a dirty bit of the same leaf (it is the latest element of its group); the K values
//     are summed pairwise.  Dirty bits and used leaf stamps are cleared at the end.
//  2. Heights 2 .. hb of the subtree are recomputed from LDS and stored.
//  3. Above hb every node counts the arrivals of its children's workgroups; the last one to
//     arrive recomputes it and carries on upwards, so the root is written by whichever
//     workgroup finishes last.  No workgroup ever waits for another.  When there are only a
//     few nodes at height hb this step is skipped (chain == 0): the agent-scope fences it
//     needs cost more than recomputing those heights in the next kernel that reads them.
// Largest hb that tree_pass_height can give a fanout.
template <int LOGK>
constexpr int kMaxPassHeight = LOGK == 1 ? 13 : LOGK == 2 ? 6 : LOGK == 3 ? 4 : LOGK <= 5 ? 3 : 2;

// The batch itself, for a tree pass over a batch that claimed in runs (see claim_runs).
struct BatchRef {
  const uint32_t* idx;   // [T][B]
  const float* prio;
  uint32_t B;
};
struct NoBatch {};
// A small batch that the tree pass claims itself (see gather_batch).
struct SmallBatch {
  ClaimArgs c;
  uint32_t slots;        // of the table of claimed leaves: a power of two, at least twice the batch
};
template <bool RUNS, bool HERE = false>
using BatchParam = typename std::conditional<HERE, SmallBatch, typename std::conditional<RUNS, BatchRef, NoBatch>::type>::type;

// The claim phase of a small batch inside the tree pass: every workgroup reads the whole batch and takes the elements of
// its own subtree into a table in LDS, keyed by leaf, where the latest valid element of a leaf wins by an LDS atomic; the
// leaves' bits go into a word (two for K = 64) per height-1 node.  No stamps and no dirty bits in memory then, and no
// kernel of its own: 512 temporal-difference errors on 100 000 leaves at K = 64, 5.2 us, 6.9 as two kernels.
constexpr uint32_t kHereBatch = 2048;      // largest batch claimed so
constexpr uint32_t kHereSlotBytes = 12;    // of the table of claimed leaves: a key, an element and its value
static uint32_t here_slots(uint32_t B) {   // (at least two per element)
  uint32_t slots = 64;
  while (slots < 2 * B) slots *= 2;
  return slots;
}
// Most elements read over all workgroups (2048 by 1024 of them: 10.5 us, 7.7 as two kernels; 1024: 6.2 and 7.6).
constexpr uint64_t kHereReads = 1u << 20;
struct LeafTable {
  unsigned long long* last;   // element + 1, value bits
  uint32_t* key;              // the leaf, or kNoLeaf
  uint32_t slots;
  static constexpr uint32_t kNoLeaf = 0xFFFFFFFFu;
  __device__ __forceinline__ uint32_t first(uint32_t leaf) const { return (leaf * 0x9E3779B1u) >> (__builtin_clz(slots) + 1u); }
  __device__ __forceinline__ void take(uint32_t leaf, uint32_t j, uint32_t vbits) const {
    uint32_t h = first(leaf);
    for (;;) {   // (the table is at most half full: a free slot comes)
      const uint32_t was = atomicCAS(&key[h], kNoLeaf, leaf);
      if (was == kNoLeaf || was == leaf) break;
      h = (h + 1u) & (slots - 1u);
    }
    atomicMax(&last[h], ((unsigned long long)(j + 1u) << 32) | vbits);
  }
  __device__ __forceinline__ uint32_t value(uint32_t leaf) const {   // of a leaf that has been taken
    uint32_t h = first(leaf);
    while (key[h] != leaf) h = (h + 1u) & (slots - 1u);
    return (uint32_t)last[h];
  }
};

// The work of workgroup b of tree t (b = its subtree's root at height hb).  TRACK_MIN: also renew min1
// (smallest positive leaf) of every rebuilt height-1 node; a compile-time choice, because even as a
// never-taken branch that code cost the pass half a microsecond.
// RUNS: the batch claimed in runs; an entry may stand for several elements, read from the batch.
// HERE: the batch is claimed by this pass itself (see LeafTable).
template <int LOGK, bool TRACK_MIN, bool RUNS = false, bool HERE = false>
__device__ __forceinline__ void tree_job(const Geom& g, const SubLevels& sl, uint32_t t, uint32_t b, uint32_t chain,
                                         BatchParam<RUNS, HERE> batch = BatchParam<RUNS, HERE>{}) {
  constexpr int K = Fan<LOGK>::K;
  constexpr int LPS = Fan<LOGK>::LPS;
  // dynamic LDS: the subtree's nodes, then the list of claimed height-1 nodes (see tree_lds_bytes)
  extern __shared__ __attribute__((aligned(16))) float sub[];   // 16-byte LDS accesses need the alignment
  uint2* s_entry = reinterpret_cast<uint2*>(sub + (sl.lds_floats + 3u) / 4u * 4u);
  uint32_t* s_list = reinterpret_cast<uint32_t*>(s_entry + sl.list_cap);
  uint32_t* s_bits = s_list + sl.list_cap;
  [[maybe_unused]] uint32_t* s_bits_hi = s_bits + sl.list_cap;   // K = 64 only
  [[maybe_unused]] LeafTable table;
  [[maybe_unused]] uint32_t* s_claimed = nullptr;   // HERE: claimed leaves of the subtree's height-1 nodes
  if constexpr (HERE) {
    table.slots = batch.slots;
    const uint32_t words = (sl.lds_floats + 3u) / 4u * 4u + sl.list_cap * (LOGK == 6 ? 5u : 4u);   // (see tree_lds_bytes)
    table.last = reinterpret_cast<unsigned long long*>(sub + (words + 1u) / 2u * 2u);
    table.key = reinterpret_cast<uint32_t*>(table.last + table.slots);
    s_claimed = table.key + table.slots;
  }
  __shared__ uint32_t s_wave[16];
  __shared__ uint32_t s_last;
  const uint32_t hb = sl.hb;
  const unsigned lane = threadIdx.x & 63u;
  const unsigned q = threadIdx.x % LPS;
  const uint32_t grp = threadIdx.x / LPS;
  const uint32_t ngrp = blockDim.x / LPS;

  PER_TRACE_DECL;
  PER_MARK(0);
  PER_MARK_HWID(15);
  // ---- 0. this subtree's height-1 nodes and their dirty flags
  const uint32_t sh1 = (hb - 1) * LOGK;
  const uint32_t n1 = sl.n[0];
  const uint32_t n1_pad = (n1 + K - 1) / K * K;
  const uint32_t lo1 = b << sh1;
  const uint32_t hi1 = min(n1, (b + 1) << sh1);
  float* lvl1 = sl.ptr[0] + (size_t)t * sl.stride[0];
  uint32_t* dirty = g.dirty + (size_t)t * g.dirty_stride;
  float* leaves = g.level[0] + (size_t)t * g.stride[0];
  uint2* owner = reinterpret_cast<uint2*>(g.owner) + (size_t)t * g.owner_stride;   // (value, stamp)
  // the K dirty bits of one height-1 node
  auto node_bits = [&](uint32_t node) -> unsigned long long {
    if constexpr (HERE) {
      const uint32_t i = node - lo1;
      return LOGK == 6 ? ((unsigned long long)s_claimed[2 * i + 1] << 32) | s_claimed[2 * i] : s_claimed[i];
    } else if constexpr (LOGK == 6) {
      const uint2 w = *reinterpret_cast<const uint2*>(dirty + 2 * (size_t)node);
      return ((unsigned long long)w.y << 32) | w.x;
    } else if constexpr (LOGK == 5) {
      return dirty[node];
    } else {
      const uint32_t bit0 = node << LOGK;
      return (dirty[bit0 >> 5] >> (bit0 & 31u)) & ((1u << K) - 1u);
    }
  };
  // the claim group entry of a height-1 node if this batch wrote it for a leaf of that node:
  // (value bits, 0x80000000 | leaf within the node), else y = 0
  uint2* groups = g.nclaim + (size_t)t * g.nclaim_stride;
  // first stamp of this batch, left by its claim phase (a batch that claimed leaf by leaf has no entries)
  const uint32_t floor = !HERE && sl.group_batch ? read_word_with_the_loads(g.sfloor + t) : 0xFFFFFFFFu;
  // (fetched here, decoded there: the comparison would make the wave wait for the entry, and the floor, before it
  // issues the loads that follow)
  auto fetch_entry = [&](uint32_t node) -> uint2 { return groups[LOGK >= 5 ? node : (node << LOGK) >> 5]; };
  auto decode_entry = [&](uint2 e, uint32_t node) -> uint2 {
    bool mine = (e.y >> 6) >= floor;
    if constexpr (RUNS) {   // a run: its length in x, 0xC0000000 | the position of its last element in y (any node of the group may have a part in it)
      const uint32_t n = run_length(e.x);
      if (mine && n > 1) return make_uint2(n, 0xC0000000u | ((e.y >> 6) - floor));
    }
    if constexpr (LOGK < 5) mine = mine && ((e.y & 31u) >> LOGK) == (node & ((32u >> LOGK) - 1u));
    e.y = mine ? 0x80000000u | (e.y & (uint32_t)(K - 1)) : 0u;
    return e;
  };
  // one node per thread and sweep; the first sweep's bits are fetched together with the height-1 nodes
  const uint32_t f_first = lo1 + threadIdx.x;
  unsigned long long bits_first = 0;
  uint2 entry_first = make_uint2(0, 0);
  // HERE: the batch, four elements per lane under way at a time
  [[maybe_unused]] uint32_t el_i[HERE ? 4 : 1];
  [[maybe_unused]] float el_v[HERE ? 4 : 1];
  [[maybe_unused]] uint32_t max_seen = 0;
  [[maybe_unused]] auto fetch_elements = [&](uint32_t first) {
    if constexpr (HERE) {
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) {
        const uint32_t j = first + k * blockDim.x + threadIdx.x;
        const size_t o = (size_t)t * batch.c.B + (j < batch.c.B ? j : 0u);
        el_i[k] = batch.c.idx[o];
        el_v[k] = batch.c.prio[o];
      }
    }
  };
  if constexpr (HERE) {
    fetch_elements(0);
    max_seen = read_max_bits(g, t);
    for (uint32_t i = threadIdx.x; i < table.slots; i += blockDim.x) {
      table.key[i] = LeafTable::kNoLeaf;
      table.last[i] = 0;
    }
    for (uint32_t i = threadIdx.x; i < sl.list_cap * (LOGK == 6 ? 2u : 1u); i += blockDim.x) s_claimed[i] = 0;
  } else if (f_first < hi1) {
    bits_first = node_bits(f_first);
    entry_first = fetch_entry(f_first);
  }
  {
    // slot 0 from memory, the rest zero.  The first four sweeps' loads are issued together (a sweep that
    // waits for its load before the next one starts costs a trip to memory each).
    auto from_memory = [&](uint32_t i) { return (i < sl.lds_off[1] || hb == 1) && lo1 + i < n1_pad; };
    const uint32_t i0 = threadIdx.x, i1 = threadIdx.x + blockDim.x, i2 = i1 + blockDim.x, i3 = i2 + blockDim.x;
    float v0 = 0.0f, v1 = 0.0f, v2 = 0.0f, v3 = 0.0f;
    if (i0 < sl.lds_floats && from_memory(i0)) v0 = lvl1[lo1 + i0];
    if (i1 < sl.lds_floats && from_memory(i1)) v1 = lvl1[lo1 + i1];
    if (i2 < sl.lds_floats && from_memory(i2)) v2 = lvl1[lo1 + i2];
    if (i3 < sl.lds_floats && from_memory(i3)) v3 = lvl1[lo1 + i3];
    if (i0 < sl.lds_floats) sub[i0] = v0;
    if (i1 < sl.lds_floats) sub[i1] = v1;
    if (i2 < sl.lds_floats) sub[i2] = v2;
    if (i3 < sl.lds_floats) sub[i3] = v3;
    for (uint32_t i = threadIdx.x + 4 * blockDim.x; i < sl.lds_floats; i += blockDim.x)
      sub[i] = from_memory(i) ? lvl1[lo1 + i] : 0.0f;
  }
  [[maybe_unused]] uint32_t batch_max = 0, batch_flags = 0;
  if constexpr (HERE) {
    __syncthreads();   // (the table is clear)
    const uint32_t sh = hb * LOGK;
    for (uint32_t first = 0; first < batch.c.B; first += 4 * blockDim.x) {
      if (first) fetch_elements(first);
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) {
        const uint32_t j = first + k * blockDim.x + threadIdx.x, i = el_i[k];
        if (j >= batch.c.B) continue;
        if (!(i < batch.c.size)) {
          if (b == 0) batch_flags |= 1u;   // (of no subtree: reported once)
        } else if ((uint32_t)((unsigned long long)i >> sh) == b) {
          float v = el_v[k];
          if (batch.c.from_td) v = (float)pow(fabs((double)v) + batch.c.td_eps, batch.c.td_alpha);
          if (!valid_priority(v)) {
            batch_flags |= 2u;
          } else {
            table.take(i, j, __float_as_uint(v));
            const uint32_t in = i - (lo1 << LOGK);
            if constexpr (LOGK == 6) atomicOr(&s_claimed[in >> 5], 1u << (in & 31u));
            else atomicOr(&s_claimed[in >> LOGK], 1u << (in & (uint32_t)(K - 1)));
            const uint32_t vb = v > 0.0f ? __float_as_uint(v) : 0u;
            batch_max = vb > batch_max ? vb : batch_max;
          }
        }
      }
    }
    __syncthreads();
    if (f_first < hi1) bits_first = node_bits(f_first);
  }
  // compact the claimed nodes into s_list / s_bits / s_entry: ballot within the wave, wave totals through LDS
  const uint32_t nwaves = blockDim.x >> 6;
  uint32_t nd = 0;
  for (uint32_t f0 = lo1; f0 < hi1; f0 += blockDim.x) {
    const uint32_t f = f0 + threadIdx.x;
    unsigned long long bits = 0;
    uint2 entry = make_uint2(0, 0);
    if (f0 == lo1) {
      bits = bits_first;
      entry = entry_first;
    } else if (f < hi1) {
      bits = node_bits(f);
      if constexpr (!HERE) entry = fetch_entry(f);
    }
    if constexpr (!HERE) entry = decode_entry(entry, f);
    if (!(f < hi1)) entry.y = 0;
    const bool listed = bits != 0 || entry.y != 0;
    const unsigned long long m = __ballot(listed);
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    if (lane == 0) s_wave[threadIdx.x >> 6] = (uint32_t)__popcll(m);
    __syncthreads();
    uint32_t before = nd, total = nd;
    for (uint32_t wv = 0; wv < nwaves; ++wv) {
      const uint32_t c = s_wave[wv];
      if (wv < (threadIdx.x >> 6)) before += c;
      total += c;
    }
    if (listed) {
      s_list[before + rank] = f;
      s_bits[before + rank] = (uint32_t)bits;
      s_entry[before + rank] = entry;
      if constexpr (LOGK == 6) s_bits_hi[before + rank] = (uint32_t)(bits >> 32);
    }
    nd = total;
    __syncthreads();
  }
  PER_MARK(1);

  if (nd > 0) {
    // ---- 1. rebuild the dirty height-1 nodes (list order is irrelevant: nodes are independent).
    // Two nodes per lane group and sweep, the loads of both issued before the first store: a
    // second sweep would otherwise cost a second trip to memory.
    using LeafVec = typename std::conditional<LOGK == 1, float2, float4>::type;
    // RUNS: the lanes of a four that rebuild one node (K >= 16) fetch two of eight elements of its run each and hand them to
    // each other by quad permutes.  (Every lane fetching four for itself: eight loads beside the one of its leaves where
    // there are four now, and a trip to memory for every four elements of a longer run: 2^20 elements on 2^20 leaves
    // 19.2 us at K = 16, 51.2 at K = 64, 17.0 and 42.9 so; on 2^24 at K = 32 34.0 and 33.9.)
    constexpr bool QUADS = RUNS && LPS >= 4;
    constexpr uint32_t RUN_WORDS = QUADS ? 2u : 4u;
    struct Item {
      bool ok;
      uint32_t node, my;
      size_t at;
      LeafVec c;
      uint2 s[RUNS ? 1 : 4];   // (RUNS: of the lane's first dirty leaf; few leaves are)
      uint2 e;
      uint32_t mn;   // (TRACK_MIN only)
      uint32_t ri[RUNS ? RUN_WORDS : 1];   // (RUNS: the first elements of the entry's run; a longer one is read on in finish)
      float rv[RUNS ? RUN_WORDS : 1];
    };
    // A set bit means the leaf was claimed leaf by leaf in this batch: its stamp entry holds the winner's value.
    auto fetch = [&](uint32_t item) -> Item {
      Item it;
      it.ok = item < nd;
      const uint32_t li = it.ok ? item : nd - 1;
      it.node = s_list[li];
      unsigned long long bits = s_bits[li];
      if constexpr (LOGK == 6) bits |= (unsigned long long)s_bits_hi[li] << 32;
      if constexpr (LOGK == 1) {
        it.my = (uint32_t)bits & 3u;
        it.at = (size_t)it.node * 2;
      } else {
        it.my = (uint32_t)(bits >> (4 * q)) & 0xFu;
        it.at = (size_t)it.node * K + 4 * q;
      }
      it.c = *reinterpret_cast<const LeafVec*>(leaves + it.at);
      it.e = s_entry[li];
      if constexpr (RUNS) {
        if (it.e.y >= 0xC0000000u) {
          const size_t e0 = (size_t)t * batch.B + (it.e.y & 0x3FFFFFFFu) + 1u - it.e.x;
#pragma unroll
          for (uint32_t k = 0; k < RUN_WORDS; ++k) {
            const uint32_t el = QUADS ? 4 * k + (threadIdx.x & 3u) : k;
            if (el < it.e.x) {
              it.ri[k] = batch.idx[e0 + el];
              it.rv[k] = batch.prio[e0 + el];
            }
          }
        }
      }
      if constexpr (RUNS) {
        if (it.my) it.s[0] = owner[it.at + (uint32_t)(__ffs((int)it.my) - 1)];
      } else {
#pragma unroll
        for (int k = 0; k < (LOGK == 1 ? 2 : 4); ++k) {
          it.s[k] = make_uint2(0, 0);
          if (it.my & (1u << k)) {
            if constexpr (HERE) it.s[k].x = table.value((uint32_t)it.at + k);
            else it.s[k] = owner[it.at + k];
          }
        }
      }
      return it;
    };
    auto finish = [&](Item& it) {
      float sum;
      auto stamped = [&](uint32_t k) -> float {   // value of dirty leaf k
        if constexpr (RUNS) {
          if (it.my & ((1u << k) - 1u)) return __uint_as_float(owner[it.at + k].x);
          return __uint_as_float(it.s[0].x);
        } else {
          return __uint_as_float(it.s[k].x);
        }
      };
      // the group entry's leaf, if it is one of this lane's
      const uint32_t el = it.e.y & 63u;
      const bool here = it.e.y != 0 && (!RUNS || it.e.y < 0xC0000000u) && (LOGK == 1 || (el >> 2) == q);
      const uint32_t sel = here ? 1u << (el & (LOGK == 1 ? 1u : 3u)) : 0u;
      const float ev = __uint_as_float(it.e.x);
      // the elements of a run, in their order (an element of another node of the group, or of another lane's leaves, is not taken)
      [[maybe_unused]] auto take_run = [&](auto&& set) {
        auto take = [&](uint32_t i, float v) {
          if ((i >> LOGK) != it.node) return;
          const uint32_t l = i & (uint32_t)(K - 1);
          if (LOGK == 1 || (l >> 2) == q) set(LOGK == 1 ? l : l & 3u, v);
        };
        if constexpr (RUNS) {
          const size_t e0 = (size_t)t * batch.B + (it.e.y & 0x3FFFFFFFu) + 1u - it.e.x;
          if constexpr (QUADS) {
            auto four = [&](uint32_t k, uint32_t ei, float ev4) {   // elements k .. k + 3, one in each lane of the four
              if (k >= it.e.x) return;                               // (the same for the lanes of a node)
              const int i = (int)ei, v = __float_as_int(ev4);
              take((uint32_t)quad_lane<0>(i), __int_as_float(quad_lane<0>(v)));
              if (k + 1 < it.e.x) take((uint32_t)quad_lane<1>(i), __int_as_float(quad_lane<1>(v)));
              if (k + 2 < it.e.x) take((uint32_t)quad_lane<2>(i), __int_as_float(quad_lane<2>(v)));
              if (k + 3 < it.e.x) take((uint32_t)quad_lane<3>(i), __int_as_float(quad_lane<3>(v)));
            };
            four(0, it.ri[0], it.rv[0]);
            four(4, it.ri[1], it.rv[1]);
            for (uint32_t k0 = 8; k0 < it.e.x; k0 += 16) {   // (sixteen at a time: fewer are a trip to memory each)
              uint32_t i[4];
              float v[4];
#pragma unroll
              for (uint32_t w = 0; w < 4; ++w) {
                const uint32_t el = k0 + 4 * w + (threadIdx.x & 3u), at = el < it.e.x ? el : it.e.x - 1;
                i[w] = batch.idx[e0 + at];
                v[w] = batch.prio[e0 + at];
              }
#pragma unroll
              for (uint32_t w = 0; w < 4; ++w) four(k0 + 4 * w, i[w], v[w]);
            }
          } else {
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k)
              if (k < it.e.x) take(it.ri[k], it.rv[k]);
            for (uint32_t k0 = 4; k0 < it.e.x; k0 += 4) {   // (four at a time: an element at a time is a trip to memory each)
              uint32_t i[4];
              float v[4];
#pragma unroll
              for (uint32_t k = 0; k < 4; ++k) {
                const uint32_t at = k0 + k < it.e.x ? k0 + k : it.e.x - 1;
                i[k] = batch.idx[e0 + at];
                v[k] = batch.prio[e0 + at];
              }
#pragma unroll
              for (uint32_t k = 0; k < 4; ++k) take(i[k], v[k]);   // (the last element again beyond the end)
            }
          }
        }
      };
      if constexpr (LOGK == 1) {
        if (it.my & 1u) it.c.x = stamped(0);
        if (it.my & 2u) it.c.y = stamped(1);
        if (sel & 1u) it.c.x = ev;
        if (sel & 2u) it.c.y = ev;
        it.my |= sel;
        if constexpr (RUNS) {
          if (it.e.y >= 0xC0000000u) take_run([&](uint32_t l, float v) { if (l) it.c.y = v; else it.c.x = v; it.my |= 1u << l; });
        }
        sum = it.c.x + it.c.y;
        if constexpr (TRACK_MIN) it.mn = min_u32(positive_bits(it.c.x), positive_bits(it.c.y));
      } else {
        if (it.my & 1u) it.c.x = stamped(0);
        if (it.my & 2u) it.c.y = stamped(1);
        if (it.my & 4u) it.c.z = stamped(2);
        if (it.my & 8u) it.c.w = stamped(3);
        if (sel & 1u) it.c.x = ev;
        if (sel & 2u) it.c.y = ev;
        if (sel & 4u) it.c.z = ev;
        if (sel & 8u) it.c.w = ev;
        it.my |= sel;
        if constexpr (RUNS) {
          if (it.e.y >= 0xC0000000u)
            take_run([&](uint32_t l, float v) {
              it.c.x = l == 0 ? v : it.c.x;
              it.c.y = l == 1 ? v : it.c.y;
              it.c.z = l == 2 ? v : it.c.z;
              it.c.w = l == 3 ? v : it.c.w;
              it.my |= 1u << l;
            });
        }
        sum = butterfly_sum<Fan<LOGK>::LOGLPS>((it.c.x + it.c.y) + (it.c.z + it.c.w));
        if constexpr (TRACK_MIN) {
          uint32_t m = min_u32(min_u32(positive_bits(it.c.x), positive_bits(it.c.y)),
                               min_u32(positive_bits(it.c.z), positive_bits(it.c.w)));
          it.mn = butterfly_min<Fan<LOGK>::LOGLPS>(m);
        }
      }
      return sum;
    };
    auto store = [&](const Item& it, float sum) {
      if (it.ok && it.my) *reinterpret_cast<LeafVec*>(leaves + it.at) = it.c;
      if (it.ok && q == 0) {
        // (nontemporal: the scattered 4-byte stores then leave for memory while the pass goes on, instead
        // of all being written back when the kernel ends; measured - 0.15 us per step.  The same for the
        // upper heights, which the next kernel reads first, cost + 1.2 us.)
        __builtin_nontemporal_store(sum, lvl1 + it.node);
        sub[it.node - lo1] = sum;
        if constexpr (TRACK_MIN) g.min1[(size_t)t * g.min1_stride + it.node] = it.mn;
      }
    };
    if constexpr (RUNS && LOGK >= 5) {   // (four nodes: these fanouts have few, large subtrees, and dense batches list most of their nodes)
      for (uint32_t base = 0; base < nd; base += 4 * ngrp) {
        Item i0 = fetch(base + grp), i1 = fetch(base + ngrp + grp), i2 = fetch(base + 2 * ngrp + grp), i3 = fetch(base + 3 * ngrp + grp);
        const float sum0 = finish(i0);
        const float sum1 = finish(i1);
        const float sum2 = finish(i2);
        const float sum3 = finish(i3);
        store(i0, sum0);
        store(i1, sum1);
        store(i2, sum2);
        store(i3, sum3);
      }
    } else {
      for (uint32_t base = 0; base < nd; base += 2 * ngrp) {
        Item i0 = fetch(base + grp);
        if (base + ngrp < nd) {   // uniform over the workgroup
          Item i1 = fetch(base + ngrp + grp);
          PER_MARK(4);
          const float sum0 = finish(i0);
          const float sum1 = finish(i1);
          PER_MARK(5);
          store(i0, sum0);
          store(i1, sum1);
        } else {
          PER_MARK(4);
          const float sum0 = finish(i0);
          PER_MARK(5);
          store(i0, sum0);
        }
      }
    }
    PER_MARK(2);
    // ---- 2. heights 2 .. hb of this subtree, from LDS
    // (unrolled over the slots, so that the per-height facts come out of the kernel arguments at fixed
    // offsets; read through a table in LDS instead, they cost the pass 0.3 us)
    // K = 2: the last six heights (at most 64 nodes below them) are a wave's reduction tree: lane i holds node i,
    // and every step of the butterfly is one more height (left + right; the partner lane adds right + left, the
    // same bits), so those heights cost a lane exchange each instead of a pass over LDS with a barrier.
    [[maybe_unused]] const uint32_t j_wave = LOGK == 1 ? (hb > 7 ? hb - 6 : 1u) : hb;   // first slot the wave computes
#pragma unroll
    for (int j = 1; j < kMaxPassHeight<LOGK>; ++j) {
      if ((uint32_t)j < hb && (LOGK != 1 || (uint32_t)j < j_wave)) {
        __syncthreads();
        const uint32_t sh = (hb - 1 - (uint32_t)j) * LOGK;
        const uint32_t a = b << sh;
        const uint32_t cnt = min(sl.n[j], (b + 1) << sh) - a;   // real nodes of this height in the subtree
        float* par = sl.ptr[j] + (size_t)t * sl.stride[j];
        for (uint32_t base = 0; base < cnt; base += ngrp) {
          const uint32_t e = base + grp;
          const bool ok = e < cnt;
          const float sum = group_sum<LOGK>(sub + sl.lds_off[j - 1] + (size_t)(ok ? e : 0u) * K, q);
          if (ok && q == 0) {
            par[a + e] = sum;
            sub[sl.lds_off[j] + e] = sum;
          }
        }
      }
    }
    if constexpr (LOGK == 1) {
      if (hb > 1) {
        __syncthreads();
        if (threadIdx.x < 64u) {
          const uint32_t children = 1u << (hb - j_wave);   // nodes of slot j_wave - 1 under b (zeros beyond the real ones)
          float v = lane < children ? sub[sl.lds_off[j_wave - 1] + lane] : 0.0f;
          for (uint32_t k = 1; j_wave - 1 + k < hb; ++k) {
            v = v + __shfl_xor(v, 1 << (k - 1));
            const uint32_t js = j_wave - 1 + k;             // the slot (height js + 1) this step has made
            const uint32_t sh = hb - 1 - js;
            const uint32_t a = b << sh;
            const uint32_t cnt = min(sl.n[js], (b + 1) << sh) - a;
            const uint32_t e = lane >> k;
            if ((lane & ((1u << k) - 1u)) == 0 && e < cnt) (sl.ptr[js] + (size_t)t * sl.stride[js])[a + e] = v;
          }
        }
      }
    }
  }

  PER_MARK(3);
  PER_FLUSH();
  // The dirty bits and the stamps of the dirty leaves are cleared again (both arrays are all zero between
  // batches).  Only now: a wait for loaded data also waits for every earlier store of the wave, so
  // stores that nothing depends on go last.
  if constexpr (HERE) {
    raise_max(g, t, batch_max, max_seen);
    if (batch_flags) atomicOr(&g.status[t], batch_flags);
  }
  for (uint32_t i = threadIdx.x; !HERE && i < nd; i += blockDim.x) {
    const uint32_t node = s_list[i];
    unsigned long long bits = s_bits[i];
    if constexpr (LOGK == 6) bits |= (unsigned long long)s_bits_hi[i] << 32;
    if (bits) {
      if constexpr (LOGK == 6) {
        dirty[2 * (size_t)node] = 0;
        dirty[2 * (size_t)node + 1] = 0;
      } else {
        dirty[(node << LOGK) >> 5] = 0;   // for K < 32 the word is shared with neighbours of the same subtree
      }
      while (bits) {   // (few leaves: those that met another leaf of their group, or a batch claiming leaf by leaf)
        owner[(size_t)node * K + (uint32_t)(__ffsll((long long)bits) - 1)] = make_uint2(0, 0);
        bits &= bits - 1;
      }
    }
  }
  // The stamp counter of the group entries: the next batch starts after this one; when that is beyond the
  // turning point, every workgroup clears the entries of its subtree instead and the counter starts over.
  if (!HERE && sl.group_batch) {
    const bool turn = floor + sl.group_batch > kGroupStampTurn;   // (uniform over the launch)
    if (turn) {
      const uint32_t e_lo = LOGK >= 5 ? lo1 : (lo1 << LOGK) >> 5;
      const uint32_t e_hi = LOGK >= 5 ? hi1 : (uint32_t)((((unsigned long long)hi1 << LOGK) + 31u) >> 5);
      for (uint32_t e = e_lo + threadIdx.x; e < e_hi; e += blockDim.x) groups[e] = make_uint2(0, 0);
    }
    if (b == 0 && threadIdx.x == 0) g.sbase[t] = turn ? 1u : floor + sl.group_batch;
  }
  // ---- 3. above the subtree: the last child to arrive recomputes the parent
  if (!chain) return;   // the heights above hb are left to their next reader
  uint32_t node = b;
  for (uint32_t h = hb + 1; h <= g.H; ++h) {
    const uint32_t parent = node >> LOGK;
    const uint32_t nchild = min((uint32_t)K, g.n[h - 1] - parent * K);
    __syncthreads();
    if (threadIdx.x == 0) {
      __threadfence();   // this workgroup's node writes are visible before its arrival is counted
      uint32_t* cnt = g.arrive + (size_t)t * g.arrive_stride + g.arrive_off[h] + parent;
      const uint32_t old = atomicAdd(cnt, 1u);
      const bool last = old == nchild - 1;
      if (last) *cnt = 0;   // ready for the next call
      s_last = last ? 1u : 0u;
      __threadfence();   // and the siblings' writes are visible to the reads below
    }
    __syncthreads();
    if (!s_last) return;
    if (threadIdx.x < 64) {
      const float sum = group_sum<LOGK>(g.level[h - 1] + (size_t)t * g.stride[h - 1] + (size_t)parent * K, lane % LPS);
      if (lane == 0) g.level[h][(size_t)t * g.stride[h] + parent] = sum;
    }
    node = parent;
  }
}

// What a sampling kernel that carried an insertion has left in max_pend (read by the caller when its workgroup
// started) goes into the running maximum; one workgroup per tree does this, after its share of the tree pass.
__device__ __forceinline__ void fold_pending_max(const Geom& g, uint32_t t, uint32_t pend_word) {
  const uint32_t pend = not_before_here(pend_word);
  if (threadIdx.x == 0 && pend) {
    atomicMax(reinterpret_cast<uint32_t*>(&g.max_v[t]), pend);
    g.max_pend[t] = 0u;
  }
}

// Workgroups of at most 512 lanes: two 1024-lane workgroups share a compute unit only while a wave
// stays within an eighth of the SIMD's scalar and vector registers (with one scalar register more the
// second workgroup waits for the first to end and the kernel takes half as long again), and holding
// the compiler to that budget made it spill; 512 lanes run the pass just as fast.
template <int LOGK, bool TRACK_MIN, bool RUNS, bool HERE>
__global__ void __launch_bounds__(512)
k_update_tree(Geom g, SubLevels sl, uint32_t chain, BatchParam<RUNS, HERE> batch) {
  const uint32_t pend = (chain & 2u) && blockIdx.x == 0 ? read_word_with_the_loads(&g.max_pend[blockIdx.y]) : 0u;
  tree_job<LOGK, TRACK_MIN, RUNS, HERE>(g, sl, blockIdx.y, blockIdx.x, chain & 1u, batch);
  if ((chain & 2u) && blockIdx.x == 0) fold_pending_max(g, blockIdx.y, pend);
}

// Second kernel of a fused step whose claim phase rode in the sampling kernel: the tree pass
// (workgroups 0 .. tree_blocks-1) and, beside it, what is left of the sampling call: the
// importance weights and the rows of the sampled indices (JobRanges, offset by tree_blocks).  The
// tree pass is a chain of dependent memory trips and the row traffic fills the gaps; launched with
// workgroups of at most 512 lanes so that the two kinds share the compute units.  Held to 96 scalar
// registers (it needs no scratch memory for that; the row jobs' argument tables would take a few more),
// which the many small trees of a multi-tree buffer gain from (one big tree neither gains nor loses).
// Three such workgroups are resident per compute unit where the machine reserves 16 more scalar
// registers per wave; a cap of 80 makes it four, measured slower: the jobs then slow each other down
// in the memory system by more than the earlier start of the row jobs gives back.
template <int LOGK, bool TRACK_MIN, bool WIDE>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_num_sgpr(96)))
k_tree_finish(Geom g, SubLevels sl, uint32_t chain, uint32_t tree_blocks, FieldTable ft, JobRanges jr, FinishArgs a) {
  // (the lines of the arguments asked for in one batch, through one scalar register: this kernel has none to spare;
  // by the first four waves only: with every wave of a 512-lane workgroup at it, the step of 65 536 samples on 2^24
  // leaves loses 0.3 us where the small workloads gain as much)
  if (threadIdx.x < 256u)
    touch_kernel_arguments_through_one_register<kernarg_lines<Geom, SubLevels, uint32_t, uint32_t, FieldTable, JobRanges, FinishArgs>() < kTouchLines
                                                    ? kernarg_lines<Geom, SubLevels, uint32_t, uint32_t, FieldTable, JobRanges, FinishArgs>() : kTouchLines>();
  const uint32_t t = blockIdx.y;
  if (blockIdx.x < tree_blocks) {
    const uint32_t pend = (chain & 2u) && blockIdx.x == 0 ? read_word_with_the_loads(&g.max_pend[t]) : 0u;
    tree_job<LOGK, TRACK_MIN>(g, sl, t, blockIdx.x, chain & 1u);
    if ((chain & 2u) && blockIdx.x == 0) fold_pending_max(g, t, pend);
    return;
  }
  const uint32_t b = blockIdx.x - tree_blocks;
  PER_TRACE_DECL;
  PER_MARK(0);
  PER_MARK_HWID(15);
  if (b < jr.first[1]) {
    weights_job(g, t, a.B, a.size, a.beta, a.w, a.weight_mode, b, jr.first[1]);
    PER_MARK(3);
    PER_FLUSH();
    return;
  }
  const uint32_t f = job_field(jr, b);
  if (jr.whole_rows) {
    extern __shared__ __attribute__((aligned(16))) uint8_t stage[];
    move_whole_rows(ft, jr, t, a.B, a.idx, g.N, g.status, b - jr.first[2 + f], jr.first[3 + f] - jr.first[2 + f], stage);
  } else if (f < (uint32_t)kMaxFields)
    rows_job<true, WIDE>(ft, f, t, a.B, a.idx, 0, g.N, g.status, b - jr.first[2 + f], jr.first[3 + f] - jr.first[2 + f]);
  PER_MARK(3);
  PER_FLUSH();
}

// Lowest height whose subtrees hold 64 height-1 nodes, or the root of a tree of no more of them; the owners of the
// one-kernel step are never lower.  (A tree of up to 2048 height-1 nodes as one subtree: 512 elements on 100 000 leaves
// at K = 64 took 11.3 us, 3.7 so; a step of 1024 on 30 000 at K = 16, insertion of 16 rows now carried by the sampling,
// 21.5 and 12.3; 64 such trees 40.9 and 32.5.)  Not at K = 2, where the many heights to rebuild cost the sampling as much
// as the pass gains: a step of 64 on 4096 leaves 13.5 us as one subtree, 14.7 as 32.
static uint32_t subtree_height(const Geom& g) {
  if (g.n[1] <= (g.logK == 1 ? 2048u : 64u)) return g.H;
  uint32_t hb = 1;
  while (hb < g.H && (1ull << ((hb - 1) * g.logK)) < 64) ++hb;
  // (higher where that leaves more roots than may be left to the next reader, as long as the pass goes up there: counting
  // the workgroups' arrivals instead takes 0.8 ms on 2^20 leaves at K = 2)
  const uint32_t most = g.logK == 1 ? kMaxPassHeight<1> : g.logK == 2 ? kMaxPassHeight<2> : g.logK == 3 ? kMaxPassHeight<3> : hb;
  while (hb < g.H && hb < most && g.n[hb] > kLazyTopNodes) ++hb;
  return hb;
}

// Height of the workgroup roots of the tree pass.  The pass works through a subtree's claimed nodes a few at a time, a trip
// to memory each, and what lies above is left to the next sampling call, which has the top of the tree in LDS anyway: many
// small subtrees are faster until their roots are too many for every sampling workgroup to rebuild the top from, or for
// the device to hold the workgroups.  subtree_height() gives 1024 nodes to a subtree at K = 32 and 256 at K = 16, which
// leaves trees of few leaves to a handful of workgroups; height 2 gives 32 and 16 (a group entry and a dirty word belong to
// one subtree still).  us per call, subtree_height() and height 2:
//  - K = 32, up to 1024 roots: 512 temporal-difference errors on 30 000 leaves 23.6 and 15.1; a step of 512 there 17.3 and
//    11.7, on 64 such trees 35.8 and 23.0 with 1000 each; 2^20 leaves: `sample` and `update` of 2^18 73.5 and 48.6, 40 000
//    rows inserted 26.3 and 18.5, a step of 64 9.5 and 9.4, the earlier-batch form of 64 10.3 and 10.4.  With 2048
//    roots (2^21 leaves) that form takes 11.1 and 13.2, with 4096 11.1 and 17.0.
//  - K = 16, up to 16 roots, 64 on several trees: a step of 1000 on 4096 leaves 16.1 and 12.5, on 64 trees of 16 384 29.4
//    and 24.6; with more roots nothing is gained (50 000 leaves, 300 samples: 11.5 and 11.6).
//  - no more than 4096 over all trees: 64 trees of 32 768 leaves at K = 16, 300 samples: 17.0 and 20.2; 16 of 2^19 at K =
//    32, 1024 samples: 19.4 and 20.9.
constexpr uint64_t kMostSmallSubtrees = 4096;
static uint32_t tree_pass_height(const Geom& g) {
  const uint32_t hb = subtree_height(g);
  if (hb <= 2 || (g.logK != 4 && g.logK != 5) || g.n[1] <= 64u) return hb;
  const uint32_t most = g.logK == 5 ? 1024u : g.T >= 4 ? 64u : 16u;
  return g.n[2] <= most && (uint64_t)g.n[2] * g.T <= kMostSmallSubtrees ? 2u : hb;
}

// Heights above this one may be left stale by an update (0: never).
uint32_t lazy_top_height(const Geom& g, const Tuning& tn) {
  const uint32_t hb = tree_pass_height(g);
  return tn.lazy_top && hb < g.H && g.n[hb] <= kLazyTopNodes ? hb : 0u;
}

// Dynamic LDS of a tree-pass workgroup: its subtree's nodes (padded to 16 bytes), then per listed
// height-1 node the group entry (8 bytes), the node number and the dirty bits (4 bytes each; 8 for K = 64).
template <int LOGK>
static size_t tree_lds_bytes(const SubLevels& sl) {
  return ((size_t)(sl.lds_floats + 3u) / 4u * 4u + (size_t)sl.list_cap * (LOGK == 6 ? 5u : 4u)) * 4u;
}

// The heights 1 .. hb of a tree-pass workgroup's subtree (hb: tree_pass_height), and where it keeps them in LDS.
template <int LOGK>
static void sub_levels(const Geom& g, uint32_t hb, SubLevels* out) {
  constexpr int K = Fan<LOGK>::K;
  SubLevels sl{};
  sl.hb = hb;
  uint32_t off = 0;
  for (uint32_t h = 1; h <= sl.hb; ++h) {
    const uint32_t j = h - 1;
    sl.ptr[j] = g.level[h];
    sl.stride[j] = g.stride[h];
    sl.n[j] = g.n[h];
    sl.lds_off[j] = off;
    // nodes of this height under one workgroup root, padded to whole child groups
    const uint64_t full = 1ull << ((sl.hb - h) * LOGK);
    const uint64_t padded = h < sl.hb ? ((uint64_t)g.n[h] + K - 1) / K * K : 1;
    off += (uint32_t)(full < padded ? full : padded);
  }
  sl.lds_floats = off;
  sl.list_cap = sl.hb > 1 ? sl.lds_off[1] : 1u;
  *out = sl;
}

// Large batches at K = 32: the pass may take its subtrees of 32 height-1 nodes, one wave each, where tree_pass_height() gives
// them 1024; height 3 is then the work of a kernel behind it, so that the next reader finds what it expects.  A workgroup of 512
// lanes goes through its claimed nodes 256 at a time, a trip to memory or two each, and a tree has few such workgroups.  `sample` and
// `update`, us, subtrees of 1024 and of 32: 1.5 million leaves (46 of the large ones) 2^14 elements 20.9 and 20.6, 2^16
// 29.8 and 25.6, 2^20 190 and 130; 2^22 leaves (128) 2^15 21.9 and 22.6, 2^16 26.4 and 26.0, 2^20 134 and 113; 2^23 (256) 2^17
// 35.0 and 35.9, 2^18 52.7 and 51.5, 2^20 129 and 123; 2^24 (512) 2^18 51.1 and 57.7, 2^20 129 and 132.
// The same beside the rows and weights of a step that updates its own batch: 2^16 on 2^22 leaves 28.4 and 26.1, 2^18 on 2^23 83.3
// and 60.0.  A batch known before (`earlier`) has its claims over with sooner: 2^16 on 2^21 leaves 19.6 and 18.4, on 2^22 17.7 and 18.8.
static bool low_subtrees(const Geom& g, const Tuning& tn, uint32_t B, bool earlier = false) {
  if (g.logK != 5 || tree_pass_height(g) != 3 || lazy_top_height(g, tn) != 3) return false;
  const uint64_t roots = g.n[3], over_trees = roots * g.T;
  return over_trees <= (earlier ? 64u : 128u) ? B >= 512u * roots : over_trees <= (earlier ? 128u : 256u) && B >= 1024u * roots;
}
template <int LOGK>
static hipError_t launch_height_3_k(const Geom& g, const Tuning& tn, hipStream_t s) {
  const uint64_t threads = (uint64_t)g.n[3] * Fan<LOGK>::LPS;
  PER_LAUNCH(KID_RESUM_DENSE, k_resum_dense<LOGK>, dim3((uint32_t)((threads + 63) / 64), g.T), dim3(64), 0, s, g, 3u, 0u, g.n[3]);
  return hipGetLastError();
}

// Sub-level descriptors and workgroup size of the tree pass for the update batch claimed with `c`.
template <int LOGK>
static hipError_t tree_pass_shape(const Geom& g, const Tuning& tn, const ClaimArgs& c, uint32_t hb, SubLevels* out,
                                  uint32_t* tblock_out) {
  const uint32_t B = c.B;
  if (hb > (uint32_t)kSubSlots || hb > (uint32_t)kMaxPassHeight<LOGK>)
    return hipErrorInvalidValue;   // cannot happen for fanouts and capacities accepted at create
  SubLevels sl;
  sub_levels<LOGK>(g, hb, &sl);
  sl.group_batch = c.group_mode ? c.B : 0u;
  // Unless told otherwise: enough lane groups to rebuild in one sweep twice the dirty height-1 nodes a
  // subtree gets on average (never more than it has), so that small batches do not launch idle waves.
  uint32_t tblock = tn.tree_block;
  if (tblock == 0) {
    const uint64_t per_subtree = hb > 1 ? sl.lds_off[1] : 1;
    uint64_t expect = 2 * ((uint64_t)B + g.n[hb] - 1) / g.n[hb];
    if ((uint64_t)g.n[hb] * g.T >= 2048) expect = (expect + 1) / 2;   // many small subtrees (many trees): more workgroups resident instead
    if (expect > per_subtree) expect = per_subtree;
    uint64_t want = expect * Fan<LOGK>::LPS;
    if (hb > 2) {   // the dense heights of the subtree want a lane group per height-2 node
      const uint64_t dense = (uint64_t)(sl.lds_off[2] - sl.lds_off[1]) * Fan<LOGK>::LPS;
      if (dense > want) want = dense;
    }
    tblock = (uint32_t)(want > 1024 ? 1024 : (want + 63) / 64 * 64);
    if (tblock < 64) tblock = 64;
    // A lane per height-1 node of the subtree when the launch stays small (at most eight waves per compute unit
    // of a 256-unit device): the list of claimed nodes is then made in one sweep, and every further sweep would
    // cost a trip to memory of its own (measured on one tree of 2^20 leaves at K = 16:
    // 14.1 -> 13.1 us per step of 32 samples, 14.1 -> 13.6 of 4096).
    const uint64_t one_sweep = per_subtree > 1024 ? 1024 : (per_subtree + 63) / 64 * 64;
    if (one_sweep > tblock && (uint64_t)g.n[hb] * g.T * (one_sweep / 64) <= 4096) tblock = (uint32_t)one_sweep;
    // ... and no more waves than that over the whole launch for a large batch either: workgroups that wait for a
    // second round cost more than the sweeps that smaller ones add (2^22 leaves at K = 16, 65 536 elements: 8.1 us
    // with 512 lanes, 5.6 with 256).
    const uint64_t groups = (uint64_t)g.n[hb] * g.T;
    const uint64_t room = groups >= 4096 ? 1 : 4096 / groups;   // waves per workgroup
    if (tblock > room * 64) tblock = (uint32_t)(room * 64);
  }
  *out = sl;
  *tblock_out = tblock;
  return hipSuccess;
}

template <int LOGK>
static hipError_t launch_tree_k(const Geom& g, const Tuning& tn, const ClaimArgs& c, hipStream_t s) {
  const bool low = low_subtrees(g, tn, c.B);
  SubLevels sl;
  uint32_t tblock;
  hipError_t e = tree_pass_shape<LOGK>(g, tn, c, low ? 2u : tree_pass_height(g), &sl, &tblock);
  if (e != hipSuccess) return e;
  if (tblock > 512) tblock = 512;
  const uint32_t chain = (lazy_top_height(g, tn) ? 0u : 1u) | (c.fold_max ? 2u : 0u);
  const size_t lds = tree_lds_bytes<LOGK>(sl);   // (K = 2: up to 96 KB, above 2^24 leaves)
#define PER_UPDATE_TREE(TM, RN, BATCH)                                                                                     \
  do {                                                                                                                     \
    e = grant_lds<&k_update_tree<LOGK, TM, RN, false>>(tn, lds);                                                           \
    if (e != hipSuccess) return e;                                                                                         \
    PER_LAUNCH(KID_UPDATE_TREE, (k_update_tree<LOGK, TM, RN, false>), dim3(g.n[sl.hb], g.T), dim3(tblock), lds, s, g, sl, chain, BATCH); \
  } while (0)
  const BatchRef batch{c.idx, c.prio, c.B};
  if (c.runs) {
    if (c.track_min) { PER_UPDATE_TREE(true, true, batch); } else { PER_UPDATE_TREE(false, true, batch); }
  } else {
    if (c.track_min) { PER_UPDATE_TREE(true, false, NoBatch{}); } else { PER_UPDATE_TREE(false, false, NoBatch{}); }
  }
#undef PER_UPDATE_TREE
  e = hipGetLastError();
  return e == hipSuccess && low ? launch_height_3_k<LOGK>(g, tn, s) : e;
}

// The height of the subtrees in which a small batch is updated by one kernel, or 0 where two are faster.  Many workgroups of small
// subtrees (tree_pass_height()) are faster than few of large ones (subtree_height()) while the device holds them all at once, which
// their tables of claimed leaves limit; at K = 16 up to 2048 of them.  us per `update` as two kernels, in small subtrees and in large ones:
//  - K = 32: 1024 elements of each of 4 trees of 287 219 leaves, 1124 small subtrees 7.3, 6.9 and 7.0, 1500 7.3, 13.5 and 8.0; 1500 on
//    600 000 leaves, 586 of them 6.3, 9.3 and 6.9, of each of 16 trees of 30 000, 480 of them 8.1, 6.7 and 20.2; 282 of each of 8 of 455 000, 3560 of
//    them 7.7, 8.7 and 6.0.
//  - K = 16: 2048 of each of 4 trees of 16 384, 256 of them 9.5, 5.6 and 6.8; 200 of each of 32, 2048 of them 7.9, 5.5 and 5.7, of each of 64, 4096
//    of them 8.3, 6.3 and 5.8.
// In large ones a workgroup works through what a whole part of the tree gets, four nodes at a time: at K = 32 (1024 nodes) 128 elements on
// the average, 64 on one to three trees (2^20 leaves: 2048 6.8, 10.3 and 6.7; 16 trees of 200 000: 512 of each, 73 a subtree 7.5, 9.0 and 6.8, 2048
// 8.6, 28.5 and 10.1).
static uint32_t update_here_height(const Geom& g, uint32_t B) {
  if (B > kHereBatch) return 0;
  const uint32_t hb = tree_pass_height(g), large = subtree_height(g);
  if (hb < large) {
    const uint64_t table = (uint64_t)here_slots(B) * kHereSlotBytes, held = 256u * (128u * 1024u / table), trees = g.T;
    if (g.n[hb] * trees <= held && (g.logK == 5 || g.n[hb] * trees <= 2048u)) return hb;
    if (g.logK == 5 && B > (trees >= 4u ? 128u : 64u) * (uint64_t)g.n[large]) return 0;
  }
  return (uint64_t)g.n[large] * g.T * B <= kHereReads ? large : 0u;
}

// The update of a small batch as one kernel, in subtrees of height hb.
template <int LOGK>
static hipError_t launch_update_here_k(const Geom& g, const Tuning& tn, ClaimArgs c, uint32_t hb, hipStream_t s) {
  SubLevels sl;
  uint32_t tblock;
  c.group_mode = 0;
  hipError_t e = tree_pass_shape<LOGK>(g, tn, c, hb, &sl, &tblock);
  if (e != hipSuccess) return e;
  const SmallBatch batch{c, here_slots(c.B)};
  uint32_t want = (c.B + 255) / 256 * 64;   // (the batch in one sweep of four elements per lane)
  if (want > tblock && !tn.tree_block) tblock = want;
  if (tblock > 512) tblock = 512;
  const uint32_t chain = lazy_top_height(g, tn) ? 0u : 1u;
  const size_t words = sl.list_cap * (LOGK == 6 ? 2u : 1u);
  const size_t lds = tree_lds_bytes<LOGK>(sl) + 4 + (size_t)batch.slots * kHereSlotBytes + words * 4;
#define PER_UPDATE_HERE(TM)                                                                                               \
  do {                                                                                                                    \
    e = grant_lds<&k_update_tree<LOGK, TM, false, true>>(tn, lds);                                                        \
    if (e != hipSuccess) return e;                                                                                        \
    PER_LAUNCH(KID_UPDATE_TREE, (k_update_tree<LOGK, TM, false, true>), dim3(g.n[sl.hb], g.T), dim3(tblock), lds, s, g, sl, chain, batch); \
  } while (0)
  if (c.track_min) PER_UPDATE_HERE(true); else PER_UPDATE_HERE(false);
#undef PER_UPDATE_HERE
  return hipGetLastError();
}

// The tree pass of the update batch claimed with `c` together with the weights and row jobs in `a` / `rows` (earlier: the batch
// was known before the sampling kernel).
template <int LOGK>
static hipError_t launch_tree_finish_k(const Geom& g, const Tuning& tn, const ClaimArgs& c, const FieldTable* rows,
                                       const FinishArgs& a, bool earlier, hipStream_t s) {
  const bool low = low_subtrees(g, tn, c.B, earlier);
  SubLevels sl;
  uint32_t tblock;
  hipError_t e = tree_pass_shape<LOGK>(g, tn, c, low ? 2u : tree_pass_height(g), &sl, &tblock);
  if (e != hipSuccess) return e;
  if (tblock > 512) tblock = 512;   // half the lanes of a compute unit are left to the other jobs
  FieldTable ft{};
  if (rows) ft = *rows;
  const JobRanges jr = job_ranges(rows ? &ft : nullptr, a.B, tblock, a.w ? a.B : 0u, 0u, g.T, tn.whole_rows);
  const uint32_t tree_blocks = g.n[sl.hb];
  size_t lds = tree_lds_bytes<LOGK>(sl);
  if (lds < whole_rows_lds(jr)) lds = whole_rows_lds(jr);
  const uint32_t chain = (lazy_top_height(g, tn) ? 0u : 1u) | (c.fold_max ? 2u : 0u);
  const dim3 grid(tree_blocks + jr.first[2 + kMaxFields], g.T);
  const bool wide = !jr.whole_rows && any_field_moves_wide(rows ? &ft : nullptr);
#define PER_TREE_FINISH(TM, WD)                                                                                        \
  do {                                                                                                                 \
    e = grant_lds<&k_tree_finish<LOGK, TM, WD>>(tn, lds);                                                              \
    if (e != hipSuccess) return e;                                                                                     \
    PER_LAUNCH(KID_TREE_FINISH, (k_tree_finish<LOGK, TM, WD>), grid, dim3(tblock), lds, s, g, sl, chain, tree_blocks, ft, jr, a); \
  } while (0)
  if (c.track_min) {
    if (wide) { PER_TREE_FINISH(true, true); } else { PER_TREE_FINISH(true, false); }
  } else {
    if (wide) { PER_TREE_FINISH(false, true); } else { PER_TREE_FINISH(false, false); }
  }
#undef PER_TREE_FINISH
  e = hipGetLastError();
  return e == hipSuccess && low ? launch_height_3_k<LOGK>(g, tn, s) : e;
}

// Does a batch of B elements in leaf order claim faster in runs than leaf by leaf?  The atomics of the leaf by leaf form
// cost by the element, wherever they go; in runs the tree pass waits for the elements that it reads back, the longer the
// more of them one workgroup has.  So, from a quarter of an element per group of 32 leaves on (us of `sample` and `update`, leaf by
// leaf and in runs):
//  - from 65 536 elements in all on, if there is one in 56 leaves (at K = 16 below 2^17 elements: in 32; 2^20 leaves: 2^16 elements
//    at K = 16 22.4 and 19.9, at K = 64 26.0 and 23.7, 2^18 at K = 16 53.0 and 28.4; 2^22 leaves: 2^16 at K = 64 23.5 and 24.1, at K = 16
//    21.9 and 22.6, 2^17 31.2 and 27.6, 25.9 and 24.9; 178 351 on 2^23 at K = 16 32.5 and 30.6), or from 196 608 on (2^24 leaves: 2^17 at
//    K = 16 32.5 and 32.4, 2^18 43.7 and 41.5); at K = 16 from 16 384 on with one in 12 leaves (70 000 leaves: 2^14 20.7 and 19.5;
//    300 000: 2^14 17.5 and 17.9, 2^15 20.4 and 18.7);
//  - where the pass has few workgroups of many elements, from 196 608 on: subtrees of 512 or more height-1 nodes (2^22
//    leaves at K = 32: 2^17 elements 28.9 and 28.3, 2^18 45.6 and 33.6; 2^24 at K = 4: 2^18 76 and 77, 2^19 102 and 98), or fewer
//    than 256 subtrees at K = 64, whose runs are the longest (70 000 leaves: 2^17 elements 42.7 and 81, 2^18 51 and 42.6; the
//    line is too low in between: `update` of 200 000 on 200 000 33 and 45); fewer than 256 at K = 32 from 3500 elements each on, where
//    most go leaf by leaf all the same (70 000 leaves, 69 of them: 2^16 26.2 and 34.5, 2^17 34.5 and 53.7, 2^18 42.8 and 40.0; 200 000,
//    `update` alone: 540 000 46 and 53, 800 000 54 and 41);
//  - not with fewer than 32 subtrees of so many nodes (trees of 1025 to 4094 leaves at K = 2, one subtree each; `update` of 8192 elements
//    of each of 16 trees of 4000 26.7 and 46.6), nor from 2048 nodes on (2^24 leaves at K = 2: 2^20 elements 299 and 346).
// Over 110 shapes drawn (every fanout, 2^16 .. 2^24 leaves, 1 .. 16 trees, 2^14 .. 2^20 elements) the chosen form takes 1.2 % longer than
// the better one in the mean, with exponential priorities as with ones of a long tail; leaf by leaf throughout 34 %.
// Sampled batches, that is: those in no order lose up to a tenth by runs (2^14 on 70 000 leaves at K = 16, `update` alone, 10.4 and 11.4).
template <int LOGK>
static bool runs_pay(const Geom& g, uint32_t B) {
  const uint64_t elements = (uint64_t)B * g.T;
  if ((uint64_t)B * 128u < g.N || elements < (LOGK == 4 ? 1u << 14 : 1u << 16)) return false;
  if (elements < 1u << 16) return (uint64_t)B * 12u >= g.N;
  SubLevels sl;
  sub_levels<LOGK>(g, tree_pass_height(g), &sl);
  const uint64_t subtrees = (uint64_t)g.n[sl.hb] * g.T;
  const bool large = sl.list_cap >= 512u;
  if (large && (sl.list_cap >= 2048u || subtrees < 32u)) return false;
  if (large || (LOGK == 6 && subtrees < 256u)) return elements >= 3u << 16;
  if (LOGK == 5 && subtrees < 256u) return elements >= 3500u * subtrees;
  return LOGK < 4 || (uint64_t)B * (LOGK == 4 && elements < 1u << 17 ? 32u : 56u) >= g.N || elements >= 3u << 16;
}

template <int LOGK>
static hipError_t launch_update_k(const Geom& g, const Tuning& tn, ClaimArgs c, hipStream_t s) {
  const uint32_t block = tn.update_block;
  const bool can_run = c.group_mode && !c.from_td && !c.pos, force_runs = can_run && tn.update_runs == 2;
  if (c.group_mode && tn.claim_in_sample && !c.pos && !force_runs)
    if (const uint32_t hb = update_here_height(g, c.B)) return launch_update_here_k<LOGK>(g, tn, c, hb, s);
  c.runs = force_runs || (can_run && tn.update_runs && runs_pay<LOGK>(g, c.B)) ? 1u : 0u;
  if (c.runs) {
    PER_LAUNCH(KID_UPDATE_CLAIM, k_update_claim<true>, dim3((c.B + block - 1) / block, g.T), dim3(block), 0, s, g, c);
  } else {
    PER_LAUNCH(KID_UPDATE_CLAIM, k_update_claim<false>, dim3((c.B + block - 1) / block, g.T), dim3(block), 0, s, g, c);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_tree_k<LOGK>(g, tn, c, s);
}

hipError_t launch_update(const Geom& g, const Tuning& tn, const ClaimArgs& c, hipStream_t s) {
#define CALL(L) launch_update_k<L>(g, tn, c, s)
  PER_DISPATCH_LOGK(g.logK, CALL)
#undef CALL
}

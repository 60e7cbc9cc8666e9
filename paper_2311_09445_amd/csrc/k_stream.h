// A list of steps in one launch on an LDS-resident tree.
// Part of per_kernels.hip (included inside namespace per, in the order given there); not a stand-alone header.

// ---------------------------------------------------------------------------------
// a stream of steps on an LDS-resident tree (small buffers)
// ---------------------------------------------------------------------------------
// The paper keeps the sum tree of its Replay Manager in on-chip memory and lets one kernel, started
// once, work through a stream of requests (Section V-A, "RM on FPGA": buffers of 10K to 100K entries,
// autorun kernels that need no launch per request).  The counterpart here: when a tree
// fits the LDS of one compute unit, one workgroup per tree loads the tree once, runs a whole
// list of steps (insert -> sample -> gather -> update, the order of the separate calls) against
// the LDS copy, and stores the tree back at the end.  Every tree access of a step is then an LDS
// access; only rows, inputs and outputs travel to memory.  Results are those of the separate calls.
//
// A tree whose leaves do not fit beside the rest (MEM: levels in memory) keeps what is above them in LDS and its leaves in
// memory: the paper's 100K-entry buffers at small fanouts are of that size.  per_step and per_insert_step, which come here with one
// step, few groups to read and no further steps to pay for them, also leave the level above the leaves there.  A list of one step that
// updates the batch it draws, or none, stores only the paths of what it has changed (see store_paths).  The workgroup is still the only one
// that touches the tree while the kernel runs, so its own stores, made visible to its other waves by a
// barrier, are all the coherence that takes; every operation then costs a trip or two to memory for the leaf
// groups it reads (sampling: the last level of the walk; insert and update: the groups whose sums change).
// Of narrow trees the copy holds some heights only (see Wide).  Every node is taken for the sum of its children, which
// the host sees to before the launch.
//
// Update inside one workgroup: a valid element raises the leaf (reinterpreted as an integer) to
// a marker above every valid priority pattern, 0x80000001 + its position, by an LDS atomic max; the
// element that finds its own marker afterwards is the last writer and stores its value; then
// every valid element recomputes its ancestors height by height (elements that share a parent
// store the same sum).
// The list of a batch's row pieces (see PieceFields), laid out by the host: worked out by a wave of the kernel, it was what the
// first step waited for (divisions and shares: 1.1 us behind the copy of the tree).
struct PieceList {
  uint8_t* io[kMaxFields];         // as in PieceFields, of tree 0
  uint8_t* base;
  uint64_t base_stride;            // bytes between the payloads of two trees
  uint64_t step_rows;
  uint32_t off[kMaxFields], bytes[kMaxFields], width[kMaxFields], recip[kMaxFields], first[kMaxFields], end[kMaxFields];
  uint32_t items, n;
};
struct StreamKernelArgs {           // one kernel argument, so that its parts sit at known offsets of the segment
  Geom g;
  StreamArgs a;
  PieceList rows, ins;
  uint2 share[16];                  // items of the gather of every row wave
};

// The copy of the tree is held as levels of wide groups.  Every stored height of a narrow tree (K = 2, 4) costs the walk
// and the pass over the ancestors a trip through LDS of its own, whatever its fanout, and a node is nothing but the
// pairwise sum of what lies under it: the copy keeps every fourth height of a K = 2 tree and every second of a K = 4
// one, a level then has sixteen children like the heights of a K = 16 tree, with the same sums in the same order.  The
// heights between two levels are worked out once, when the tree goes back to memory.  (K = 2, 4096 leaves: three levels
// for twelve heights; 50 steps of 64 samples and 4 new rows on it 231 -> 124 us, with what walk_tree and sum_top save.)
template <int LOGK>
struct Wide {
  static constexpr int LOGR = LOGK <= 2 ? 4 : LOGK;   // log2 of a level's children
  static constexpr int R = 1 << LOGR;
  static constexpr int LH = LOGR / LOGK;              // heights a level spans
};
// Height of level v (level V, the root's, may span fewer heights than the others).
template <int LOGK>
__device__ __forceinline__ uint32_t level_height(uint32_t v, uint32_t H) {
  const uint32_t h = v * (uint32_t)Wide<LOGK>::LH;
  return h < H ? h : H;
}

__device__ __forceinline__ uint32_t wave_value(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }   // (the same in all lanes)
__device__ __forceinline__ uint32_t ring_slot(uint32_t cursor, uint32_t j, uint32_t N) {
  const uint32_t s = cursor + j;   // (N <= 2^31, j < N)
  return s >= N ? s - N : s;
}

// Sum of the 4*N children behind g4 in the balanced pairwise order, by a single lane.
template <int N, typename P>
__device__ __forceinline__ float sum_chunks(P grp) {
  if constexpr (N == 1) {
    const Floats4 x = load_floats4(grp);
    return (x.x + x.y) + (x.z + x.w);
  } else {
    return sum_chunks<N / 2>(grp) + sum_chunks<N / 2>(grp + 2 * N);
  }
}

// The tables of heights and levels from the argument segment by vector loads (Geom first), as many entries as there can be, so
// that none waits for another argument first.
__device__ __forceinline__ void fill_stream_tables(uint32_t t, const StreamPlan* plan, LevelTable* tab, uint32_t* off, uint32_t* n) {
  const uint32_t tid = threadIdx.x;
  if (tid <= (uint32_t)kMaxHeight) {
    const Geom* gk = kernarg_at<Geom>(0);
    tab->lvl[tid] = gk->level[tid] + (size_t)t * gk->stride[tid];
    tab->n[tid] = gk->n[tid];
  }
  if (tid >= 64 && tid < 64 + kStreamLevels + 2) off[tid - 64] = plan->off[tid - 64];
  if (tid >= 128 && tid < 128 + kStreamLevels + 1) n[tid - 128] = plan->nodes[tid - 128];
}

// One tree in the LDS of its workgroup.
struct LdsTree {
  float* tree;              // levels in_memory .. V back to back, each padded with zeros to
                            // whole groups and, below the root's children, with one group more: what the nodes beyond the
                            // next level's last have for children
  uint32_t in_memory;       // the lowest levels, so many of them, stay in memory (zero padded to whole groups)
  const uint32_t *off, *n;  // off[v]: where level v starts (floats), off[V + 1]: all floats; n[v]: its real nodes
  uint32_t* max_bits;       // running maximum priority (fp32 bits)
  uint32_t H, V;
};

// Loads every level of tree t into LDS, by lanes 0 .. lanes - 1.  The heights are arrays of their own in memory (zero padded
// to 64 floats) and the levels lie back to back in LDS.  The lowest level is most of it: it goes in 16-byte pieces, eight
// per lane under way at once, and with the first eight the first piece that the lane has of the levels above.  Called by waves that have
// nothing else to do: the first requests of a queue are laid out meanwhile.
template <int LOGK>
__device__ __forceinline__ void lds_tree_load(const LevelTable& tab, const LdsTree& lt, uint32_t lane, uint32_t lanes) {
  constexpr int R = 8;
  typedef GlobalPtr<const float> Source;
  const uint32_t v0 = lt.in_memory, V = lt.V;
  // (all offsets in the lanes of the wave: a piece's level is then found without a trip to LDS per level)
  const uint32_t off_reg = lt.off[min_u32(threadIdx.x & 63u, V + 1u)];
  auto off = [&](uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)off_reg, (int)v); };
  auto above = [&](uint32_t e) {   // the piece at LDS float e, of a level above v0
    uint32_t v = v0 + 1u;
#pragma unroll 1
    for (uint32_t w = v0 + 2u; w <= V; ++w) v += e >= off(w) ? 1u : 0u;   // (the same for the wave: w)
    const uint32_t i = e - lt.off[v];
    Floats4 x = {0.0f, 0.0f, 0.0f, 0.0f};
    if (i < lt.n[v]) x = load_floats4(as_global(static_cast<const float*>(tab.lvl[level_height<LOGK>(v, lt.H)])) + i);
    return x;
  };
  const uint32_t end = off(V + 1), first = off(v0 + 1), n0 = lt.n[v0];
  Floats4 top;
  const uint32_t top_at = first + 4u * (lanes - 1u - lane);   // (the last waves first: the first have their own inputs to ask for)
  Source src = as_global(static_cast<const float*>(tab.lvl[level_height<LOGK>(v0, lt.H)]));
  float* dst = lt.tree + lt.off[v0];
  const uint32_t room = first - lt.off[v0];
  for (uint32_t base = 0; base < room; base += 4u * R * lanes) {
    Floats4 x[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t e = base + 4u * ((uint32_t)k * lanes + lane);
      x[k] = Floats4{0.0f, 0.0f, 0.0f, 0.0f};
      if (e < n0) x[k] = load_floats4(src + e);
    }
    if (base == 0 && top_at < end) top = above(top_at);   // (which level it is of is found while those are on their way)
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t e = base + 4u * ((uint32_t)k * lanes + lane);
      if (e < room) *reinterpret_cast<Floats4*>(dst + e) = x[k];
    }
  }
  if (top_at < end) *reinterpret_cast<Floats4*>(lt.tree + top_at) = top;
  for (uint32_t e = top_at + 4u * lanes; e < end; e += 4u * lanes) *reinterpret_cast<Floats4*>(lt.tree + e) = above(e);
}
// A root that the tree pass has left to its reader while its children are current (trees of three heights whose pass works in
// subtrees of the root's children): it is summed here, from the copy, and stored, since not every step changes the tree.  By one lane,
// 0.3 us; a kernel in front that does it takes 4.5 with its launch, in every replay of a captured step (two steps of 64 samples to a
// graph: on 4096 leaves at K = 16 20.2 us with that kernel, 16.4 so; a queue of a sampling and an update there 18.7 and 14.4).  In builds of
// their own: with a branch for it, lists of 100 steps took 0.4 to 2.3 % longer, a queue of rounds of 512 0.8.  Called by the team's first
// lane, behind the copy; who reads the root first is this lane's wave, or comes by a barrier before.
template <int LOGK>
__device__ __forceinline__ void sum_stale_root(const LevelTable& tab, const LdsTree& lt) {
  static_assert(Wide<LOGK>::LH == 1, "a level is a height");
  const float root = sum_chunks<Wide<LOGK>::R / 4>(static_cast<const float*>(lt.tree) + lt.off[lt.V - 1u]);
  lt.tree[lt.off[lt.V]] = root;
  as_global(tab.lvl[lt.H])[0] = root;
}
// The heights between level v and the next one, from a group of sixteen at level v: a lane per group.  (Nodes beyond a
// height's last are zero, as its padding is.)
template <int LOGK, typename P>
__device__ __forceinline__ void store_between(P grp, uint32_t p, uint32_t h0, const LevelTable& tab, uint32_t H) {
  float x[16];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const Floats4 q = load_floats4(grp + 4 * c);
    x[4 * c] = q.x, x[4 * c + 1] = q.y, x[4 * c + 2] = q.z, x[4 * c + 3] = q.w;
  }
#pragma unroll
  for (int d = 1; d < 4; ++d) {   // x: the sums of blocks of 2^d
#pragma unroll
    for (int i = 0; i < (16 >> d); ++i) x[i] = x[2 * i] + x[2 * i + 1];
    const uint32_t h = h0 + (uint32_t)(d / LOGK);
    if (d % LOGK == 0 && h <= H) {
      GlobalPtr<float> at = as_global(tab.lvl[h]) + (size_t)p * (16 >> d);
#pragma unroll
      for (int i = 0; i < (16 >> d); i += 2) *(GlobalPtr<Floats2>)(at + i) = Floats2{x[i], x[i + 1]};
    }
  }
}
// What the lanes of a wave have found goes into the tree's sticky flags.  Called by whole waves.
__device__ __forceinline__ void report_flags(const Geom& g, uint32_t t, uint32_t flags) {
  if (!__any(flags != 0)) return;
  uint32_t all = 0;
#pragma unroll
  for (uint32_t bit = 1; bit <= 4; bit <<= 1) all |= __any((flags & bit) != 0) ? bit : 0u;
  if ((threadIdx.x & 63u) == 0) atomicOr(&g.status[t], all);
}
// ... and back to memory, with the running maximum.
template <int LOGK>
__device__ __forceinline__ void lds_tree_store(const Geom& g, uint32_t t, const LevelTable& tab, const LdsTree& lt) {
  constexpr uint32_t LH = Wide<LOGK>::LH, R = Wide<LOGK>::R;
  const uint32_t V = lt.V, H = lt.H;
  // (a root less than a whole level above its children is stored by the pass below: the level's sum of it has zeros added)
  const uint32_t end = V * LH == H ? lt.off[V + 1] : lt.off[V];
  const uint32_t v0 = lt.in_memory, n0 = lt.n[v0];
  {   // the lowest level, then those above it
    constexpr int U = 4;
    GlobalPtr<float> dst = as_global(tab.lvl[level_height<LOGK>(v0, H)]);
    const float* src = lt.tree + lt.off[v0];
    for (uint32_t base = 4u * threadIdx.x; base < n0; base += 4u * U * blockDim.x) {
      Floats4 x[U];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const uint32_t e = base + 4u * (uint32_t)k * blockDim.x;
        x[k] = load_floats4(src + (e < n0 ? e : 0u));
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const uint32_t e = base + 4u * (uint32_t)k * blockDim.x;
        if (e < n0) *(GlobalPtr<Floats4>)(dst + e) = x[k];
      }
    }
  }
  for (uint32_t e = lt.off[v0 + 1] + 4u * threadIdx.x, v = v0 + 1u; e < end; e += 4u * blockDim.x) {
    while (v < V && e >= lt.off[v + 1]) ++v;
    const uint32_t i = e - lt.off[v];
    if (i < lt.n[v]) *(GlobalPtr<Floats4>)(as_global(tab.lvl[level_height<LOGK>(v, H)]) + i) = load_floats4(lt.tree + e);
  }
  if constexpr (LH > 1) {
    for (uint32_t w = 0; w < V; ++w) {
      const uint32_t groups = tab.n[level_height<LOGK>(w + 1, H)];
      for (uint32_t p = threadIdx.x; p < groups; p += blockDim.x) {
        if (w == 0 && lt.in_memory) store_between<LOGK>(as_global(static_cast<const float*>(tab.lvl[0])) + (size_t)p * R, p, 0, tab, H);
        else store_between<LOGK>(static_cast<const float*>(lt.tree) + lt.off[w] + (size_t)p * R, p, w * LH, tab, H);
      }
    }
  }
  if (threadIdx.x == 0) g.max_v[t] = __uint_as_float(*lt.max_bits);
}
// Of a list of one step only what it has changed goes back: the leaves of the updated batch (`nodes` in LDS, null: no update)
// and of the insertion, and their ancestors (elements that share one store the same value).  A wave takes 64 elements at one
// level at a time, from the count of what is taken in LDS: waves that have no rows begin as soon as the team has made the tree
// whole (*s_whole), and none waits for the others' results.  (Stored whole, with a barrier in front and behind, a step of 64 samples and 4 rows on
// 4096 leaves at K = 2 spent 1.8 us on it; all of the paths by the team's one wave, 2.0.)
template <int LOGK, int MEM>
__device__ __forceinline__ void store_paths(const LevelTable& tab, const LdsTree& lt, const uint32_t* nodes, uint32_t updated, uint32_t cursor,
                                            uint32_t inserted, uint32_t N, uint32_t* s_taken, const uint32_t* s_whole) {
  constexpr uint32_t LH = Wide<LOGK>::LH, LOGR = Wide<LOGK>::LOGR, R = Wide<LOGK>::R;
  const uint32_t lane = threadIdx.x & 63u, n = nodes ? updated : 0u, elements = n + inserted;
  // (levels in memory have been stored as they were changed; of narrow trees the heights below one of them have not)
  const uint32_t levels = lt.V + 1u - (LH > 1 && MEM ? 1u : (uint32_t)MEM), rounds = (elements + 63u) / 64u;
  for (;;) {
    uint32_t item = 0;
    if (lane == 0) item = atomicAdd(s_taken, 1u);
    item = wave_value(item);
    if (item >= rounds * levels) return;
    uint32_t round = 0;   // (few rounds)
    while (item >= levels) item -= levels, ++round;
    const uint32_t e = round * 64u + lane, v = lt.V - item;   // (the level with the heights between first)
    uint32_t leaf = 0xFFFFFFFFu;
    if (e < n) leaf = nodes[e];
    else if (e < elements) leaf = ring_slot(cursor, e - n, N);
    const bool some = leaf < N;   // (else nothing could be sampled, or no element)
    while (wave_value(*(const volatile uint32_t*)s_whole) == 0u) __builtin_amdgcn_s_sleep(1);   // (the team waits for nobody)
    asm volatile("" ::: "memory");
    const uint32_t node = leaf >> (v * LOGR);
    if constexpr (LH > 1) {   // the heights between level v - 1 and this one: the blocks of two, four, eight children that hold the leaf
      const uint32_t h0 = (v - 1) * LH, child = (leaf >> ((v - 1) * LOGR)) & (R - 1u);
      auto between = [&](auto grp) {
        const Floats4 a = load_floats4(grp + (child & ~7u)), b = load_floats4(grp + (child & ~7u) + 4);
        const bool upper = (child & 4u) != 0;
        const Floats4 x = upper ? b : a;
        const float sa = (a.x + a.y) + (a.z + a.w), sb = (b.x + b.y) + (b.z + b.w);
        constexpr uint32_t d4 = 2 / LOGK;   // heights up to the blocks of four
        if (LOGK == 1 && h0 + 1 <= lt.H) as_global(tab.lvl[h0 + 1])[leaf >> (h0 + 1)] = (child & 2u) ? x.z + x.w : x.x + x.y;
        if (h0 + d4 <= lt.H) as_global(tab.lvl[h0 + d4])[leaf >> ((h0 + d4) * LOGK)] = upper ? sb : sa;
        if (LOGK == 1 && h0 + 3 <= lt.H) as_global(tab.lvl[h0 + 3])[leaf >> (h0 + 3)] = sa + sb;
      };
      if (v && some) {
        if (MEM && v <= (uint32_t)MEM) between(as_global(static_cast<const float*>(tab.lvl[h0])) + (size_t)node * R);
        else between(static_cast<const float*>(lt.tree) + lt.off[v - 1] + (size_t)node * R);
      }
    }
    if (some && v >= (uint32_t)MEM && v * LH <= lt.H) as_global(tab.lvl[v * LH])[node] = lt.tree[lt.off[v] + node];
  }
}

// ---- rows of the stream kernels
// The rows of a batch move in pieces (16 bytes, or the field's access width), 64 pieces of one field at a time by one
// wave: an item.  A wave then works with one access width and one field's constants (with the pieces of all fields
// shared out lane by lane, every lane paid for a chain of selects over the fields, a division, and the loads and
// stores of every width that occurs in its wave).
constexpr uint32_t kInFlight = 6;   // items that a wave which does nothing else has under way at once
constexpr uint32_t kLeastMovers = 6;   // row waves that are left to gather where the others weigh the samples, at least
// How the items of a gather are shared out among the row waves.
enum GatherShares {
  SHARES_NONE,   // (an insertion)
  SHARES_EVEN,   // equally many to every wave, see gather_spans
  SHARES_ANY     // where that works, every wave has a run of at most kInFlight items of one access width (straight code, and all
                 // under way at once), else evenly
};
// Waves that gather in runs where n samples are weighed as well: those that do not weigh, if there are enough.
__host__ __device__ __forceinline__ uint32_t run_waves(uint32_t n, uint32_t rws) {
  const uint32_t weigh = (n + 63u) / 64u;
  return rws >= weigh + kLeastMovers ? rws - weigh : rws;
}
struct PieceFields {               // what the waves ask of one list of fields, in LDS
  uint8_t* io[kMaxFields];         // the caller's array: the rows of this tree (in step 0)
  uint8_t* base;                   // row 0 of this tree's payload
  uint32_t off[kMaxFields];        // where in a stored row the field lies
  uint64_t step_rows;              // rows of the caller's arrays per step
  uint32_t bytes[kMaxFields], width[kMaxFields];
  uint32_t recip[kMaxFields];      // floor(2^32 / pieces per row) + 1
  uint32_t first[kMaxFields], end[kMaxFields];   // its items, all items ordered by width
  uint32_t items, n;               // all items; rows
  uint32_t runs;                   // SHARES_ANY: the length of the runs, 0: shared out evenly
};
__device__ __forceinline__ uint64_t wave_value64(uint64_t x) {
  return (uint64_t)wave_value((uint32_t)(x >> 32)) << 32 | wave_value((uint32_t)x);
}
__device__ __forceinline__ uint8_t* wave_pointer(uint8_t* p) { return reinterpret_cast<uint8_t*>(wave_value64(reinterpret_cast<uint64_t>(p))); }
// The list of a request, by one wave: n rows per tree; field f is `asked` for (where its array is the round says); the `rws`
// row waves share the items out.  share: items of wave i.  (A list of steps has its lists from the host: plan_pieces.)
template <GatherShares SHARES>
__device__ __forceinline__ void fill_piece_fields(const FieldTable* ft, bool asked, uint32_t t, uint32_t n, uint32_t rws, PieceFields* pf,
                                                  uint2* share) {
  const uint32_t lane = threadIdx.x & 63u, f = lane;
  const bool on = f < (uint32_t)kMaxFields && f < ft->n_fields && asked && n;
  const uint32_t E = on ? ft->bytes[f] : 1u, v = on ? ft->vec[f] : 1u, epr = row_elements(E, v);
  const uint32_t w = moves_wide(E, v) ? 16u : v, kind = 4u - (uint32_t)__builtin_ctz(w);   // 0: 16 bytes .. 4: one
  const uint32_t items = on ? (n * epr + 63u) / 64u : 0u;
  // items per width and in front of this field
  uint32_t of_kind[kWidths] = {}, before = 0;
#pragma unroll
  for (uint32_t g = 0; g < (uint32_t)kMaxFields; ++g) {
    const uint32_t its = (uint32_t)__builtin_amdgcn_readlane((int)items, (int)g), kd = (uint32_t)__builtin_amdgcn_readlane((int)kind, (int)g);
#pragma unroll
    for (int c = 0; c < kWidths; ++c) of_kind[c] += kd == (uint32_t)c ? its : 0u;
    before += kd < kind || (kd == kind && g < f) ? its : 0u;
  }
  uint32_t total = 0;
#pragma unroll
  for (int c = 0; c < kWidths; ++c) total += of_kind[c];
  if (f < (uint32_t)kMaxFields) {
    pf->io[f] = on ? reinterpret_cast<uint8_t*>(0) + (uint64_t)t * n * E : nullptr;
    pf->off[f] = on ? (uint32_t)(ft->col[f] - ft->col[0]) : 0u;   // (the fields of a row lie in the order of their numbers)
    pf->bytes[f] = E;
    pf->width[f] = w;
    pf->recip[f] = epr > 1 ? 0xFFFFFFFFu / epr + 1u : 0u;
    pf->first[f] = before;
    pf->end[f] = before + items;
  }
  if (f == 0) {
    pf->base = ft->n_fields ? ft->col[0] + (uint64_t)t * ft->col_stride[0] : nullptr;
    pf->items = total;
    pf->step_rows = 0;
    pf->n = n;
  }
  if constexpr (SHARES == SHARES_NONE) return;
  uint32_t run = 0, waves = rws;
  if constexpr (SHARES == SHARES_ANY) {
    // the shortest runs with which there are waves enough: lane i tries runs of i + 1 (at most 16 * 6 items count here, for which
    // the product with the reciprocal is the quotient)
    waves = run_waves(n, rws);
    const uint32_t len = lane + 1u, recip = (0x10000u + lane) / len;
    uint32_t needed = 0;
#pragma unroll
    for (int c = 0; c < kWidths; ++c) needed += (min_u32(of_kind[c], 1023u) + lane) * recip >> 16;
    const unsigned long long enough = __ballot(needed <= waves && lane < kInFlight);
    run = enough ? 1u + (uint32_t)__builtin_ctzll(enough) : 0u;
    if (f == 0) pf->runs = run;
  }
  if (lane < 16u) {
    uint32_t a = 0, b = 0;
    if (SHARES == SHARES_ANY && run) {
      const uint32_t recip = 0xFFFFu / run + 1u;   // (as above)
      uint32_t start = 0, wave0 = 0;
#pragma unroll
      for (int c = 0; c < kWidths; ++c) {
        const uint32_t takes = (of_kind[c] + run - 1u) * recip >> 16;
        if (lane >= wave0 && lane < wave0 + takes) {
          a = start + (lane - wave0) * run;
          b = a + run < start + of_kind[c] ? a + run : start + of_kind[c];
        }
        start += of_kind[c];
        wave0 += takes;
      }
    } else {
      const uint32_t each = (total + rws - 1) / rws;
      if (lane < rws && lane * each < total) {
        a = lane * each;
        b = a + each < total ? a + each : total;
      }
    }
    share[lane] = make_uint2(a, b);
  }
}
// The same from a list that the host has laid out, by one wave: read when the kernel starts, put into LDS behind the first
// barrier, for which the other waves then need not wait.
struct PieceCopy {
  uint8_t *io, *base;
  uint64_t step_rows;
  uint32_t off, bytes, width, recip, first, end, items, n;
  __device__ __forceinline__ void read(const PieceList* pl, uint32_t t) {
    const uint32_t f = min_u32(threadIdx.x & 63u, (uint32_t)kMaxFields - 1u);
    n = pl->n;
    items = pl->items;
    step_rows = pl->step_rows;
    base = pl->base + (uint64_t)t * pl->base_stride;
    off = pl->off[f];
    bytes = pl->bytes[f];
    width = pl->width[f];
    recip = pl->recip[f];
    first = pl->first[f];
    end = pl->end[f];
    io = pl->io[f];
  }
  __device__ __forceinline__ void put(uint32_t t, PieceFields* pf) const {
    const uint32_t f = threadIdx.x & 63u;
    if (f < (uint32_t)kMaxFields) {
      pf->io[f] = io + (uint64_t)t * n * bytes;
      pf->off[f] = off;
      pf->bytes[f] = bytes;
      pf->width[f] = width;
      pf->recip[f] = recip;
      pf->first[f] = first;
      pf->end[f] = end;
    }
    if (f == 0) {
      pf->base = base;
      pf->items = items;
      pf->step_rows = step_rows;
      pf->n = n;
    }
  }
};
// el / epr, for el < 2^31 (at most 1024 rows of at most 2^20 pieces, and less than a few items beyond them) and recip = floor(2^32 /
// epr) + 1: recip is less than 1 / epr of itself too large, the quotient less than a half, so it comes out right or one too
// large.  (epr = 1: recip = 0, and no branch for it: there is one such quotient per piece.)
__device__ __forceinline__ uint32_t row_of_piece(uint32_t el, uint32_t epr, uint32_t recip) {
  const uint32_t row = __umulhi(el, recip) | (epr == 1 ? el : 0u);
  return row * epr > el ? row - 1u : row;
}
struct RowItem {         // this lane's piece of an item
  uint32_t row;          // row of the batch, 0xFFFFFFFF: no piece
  uint32_t f, w;         // field and access width (the same for the wave; w = 0: no item)
  uint32_t at;           // offset of the piece in the stored row
  uint8_t* io;           // the caller's array (the same for the wave)
  uint32_t out;          // offset of the piece in it
  uint64_t step;         // bytes of that array per step (the same for the wave)
};
// The field of item i < pf.items of a list.
__device__ __forceinline__ uint32_t field_of_item(const PieceFields& pf, uint32_t i) {
  uint32_t f = 0;
#pragma unroll
  for (uint32_t k = 1; k < (uint32_t)kMaxFields; ++k) f = i >= pf.first[k] && i < pf.end[k] ? k : f;
  return wave_value(f);
}
// Item i < pf.items of a list (in step 0).
__device__ __forceinline__ RowItem find_item(const PieceFields& pf, uint32_t i) {
  const uint32_t f = field_of_item(pf, i);
  const uint32_t E = wave_value(pf.bytes[f]), w = wave_value(pf.width[f]), epr = (E + w - 1) / w;
  const uint32_t el = (i - wave_value(pf.first[f])) * 64u + (threadIdx.x & 63u);
  const uint32_t row = row_of_piece(el, epr, wave_value(pf.recip[f]));
  const uint32_t k = el - row * epr, at = k * w + w > E ? E - w : k * w;   // (wide pieces: the last one ends with the field)
  RowItem p;
  p.row = row < wave_value(pf.n) ? row : 0xFFFFFFFFu;
  p.f = f;
  p.w = w;
  p.at = wave_value(pf.off[f]) + at;
  p.io = wave_pointer(pf.io[f]);
  p.out = p.row == 0xFFFFFFFFu ? 0u : row * E + at;   // (at most 1024 rows of at most 1 MiB)
  p.step = wave_value64(pf.step_rows) * E;
  return p;
}
typedef uint32_t Words4 __attribute__((ext_vector_type(4), aligned(4)));   // (16-byte pieces of some fields lie on 4-byte boundaries)
typedef uint32_t Words2 __attribute__((ext_vector_type(2)));
// (One test per width and no else between them: a switch on a value of the wave becomes a dozen branches.  What a narrow
// piece leaves of v stays undefined: setting it would make the wave wait for loads under way.)
__device__ __forceinline__ uint4 load_piece(const uint8_t* p, uint32_t w) {
  GlobalPtr<const uint8_t> src = as_global(p);
  uint4 v;
  if (w == 16u) {
    const Words4 x = *(GlobalPtr<const Words4>)src;
    v = make_uint4(x.x, x.y, x.z, x.w);
  }
  if (w == 8u) {
    const Words2 x = *(GlobalPtr<const Words2>)src;
    v.x = x.x, v.y = x.y;
  }
  if (w == 4u) v.x = *(GlobalPtr<const uint32_t>)src;
  if (w == 2u) v.x = *(GlobalPtr<const uint16_t>)src;
  if (w == 1u) v.x = *(GlobalPtr<const uint8_t>)src;
  return v;
}
__device__ __forceinline__ void store_piece(uint8_t* p, uint32_t w, const uint4& v) {
  GlobalPtr<uint8_t> dst = as_global(p);
  if (w == 16u) {
    const Words4 x = {v.x, v.y, v.z, v.w};
    *(GlobalPtr<Words4>)dst = x;
  }
  if (w == 8u) {
    const Words2 x = {v.x, v.y};
    *(GlobalPtr<Words2>)dst = x;
  }
  if (w == 4u) *(GlobalPtr<uint32_t>)dst = v.x;
  if (w == 2u) *(GlobalPtr<uint16_t>)dst = (uint16_t)v.x;
  if (w == 1u) *(GlobalPtr<uint8_t>)dst = (uint8_t)v.x;
}
// The pieces of a gather that a wave has under way: M items of its share.  Where a piece lies in its row and where it goes
// is known before the rows are; prepared in time, what is left between the batch and its loads is a look at the batch's
// slots.  All loads are on their way before the first store, and all of a wave's items have one access width: the code
// for a width is straight.  (Several waves share a SIMD, and what they issue is what bounds large batches.)
template <int M, bool PACKED = false>
struct GatherItems {
  uint32_t count = 0, w = 0;   // items, their access width
  uint32_t on = 0;             // bit k: this lane has a piece of item k
  // (PACKED: a batch of at most 512 rows, whose number goes into the bits above the 23 of an offset in a stored row, 8 fields of at
  // most 1 MiB.  For the queue, whose waves have no register to spare: what they spill they read back between loads and
  // stores, each time with a wait for all they have under way.  The list of steps, which spills nothing, loses 1 % by it.)
  uint32_t row[M], slot[M], at[PACKED ? 1 : M], out[M];
  const uint8_t* base;         // row 0 of the tree's payload
  uint32_t field[M];
  uint4 v[M];
  // items first .. last - 1 (at most M) of a list, of one access width; MIXED: those of one width that they begin with.  `take`
  // is called with every item's number here and the item
  template <bool MIXED = false, typename F>
  __device__ __forceinline__ void prepare(const PieceFields& pf, uint32_t first, uint32_t last, F&& take) {
    if constexpr (MIXED) {
      if (first < last) {
        const uint32_t width = wave_value(pf.width[field_of_item(pf, first)]);
        uint32_t end = first;
#pragma unroll
        for (uint32_t f = 0; f < (uint32_t)kMaxFields; ++f) end = pf.width[f] == width && pf.end[f] > end ? pf.end[f] : end;
        end = wave_value(end);   // (all items are ordered by width)
        last = last < end ? last : end;
      }
    }
    count = first < last ? (last - first < (uint32_t)M ? last - first : (uint32_t)M) : 0u;
    on = 0;
    base = wave_pointer(pf.base);
#pragma unroll
    for (int k = 0; k < M; ++k) {   // (beyond the last: the first one again, without lanes: no load stands in a branch)
      asm volatile("" ::: "memory");   // (one item after the other: all at once they take more registers than there are)
      if (first + k < last) {
        const RowItem p = find_item(pf, first + k);
        w = p.w;
        on |= p.row != 0xFFFFFFFFu ? 1u << k : 0u;
        row[k] = p.row != 0xFFFFFFFFu ? p.row : 0u;
        out[k] = p.out;
        if constexpr (PACKED) row[k] = row[k] << 23 | p.at;
        else at[k] = p.at;
        field[k] = p.f;
        take(k, p);
      } else {
        row[k] = row[0];
        out[k] = 0;
        if constexpr (!PACKED) at[k] = at[0];
        field[k] = 0;
      }
    }
  }
  template <int C, typename V>
  __device__ __forceinline__ void load_as(uint32_t N, uint32_t row_stride) {
#pragma unroll
    for (int k = 0; k < C; ++k) {
      const V x = *(GlobalPtr<const V>)as_global(base + (uint64_t)(slot[k] < N ? slot[k] : 0u) * row_stride + (PACKED ? row[k] & 0x7FFFFFu : at[PACKED ? 0 : k]));
      if constexpr (sizeof(V) == 16) v[k] = make_uint4(x.x, x.y, x.z, x.w);
      else if constexpr (sizeof(V) == 8) v[k].x = x.x, v[k].y = x.y;
      else v[k].x = x;
    }
  }
  template <int C>
  __device__ __forceinline__ void load_some(const uint32_t* nodes, uint32_t N, uint32_t row_stride) {
#pragma unroll
    for (int k = 0; k < C; ++k) slot[k] = nodes[PACKED ? row[k] >> 23 : row[k]];
    if (w == 16u) load_as<C, Words4>(N, row_stride);
    if (w == 8u) load_as<C, Words2>(N, row_stride);
    if (w == 4u) load_as<C, uint32_t>(N, row_stride);
    if (w == 2u) load_as<C, uint16_t>(N, row_stride);
    if (w == 1u) load_as<C, uint8_t>(N, row_stride);
  }
  // (nodes: the batch's slots)
  __device__ __forceinline__ void load(const uint32_t* nodes, uint32_t N, uint32_t row_stride) {
    if (count == 0) return;
    if (M > 2 && count > 2) load_some<M>(nodes, N, row_stride);
    else load_some<M < 2 ? M : 2>(nodes, N, row_stride);
  }
  template <int C, typename V, typename F>
  __device__ __forceinline__ void store_as(F&& array_of) {
#pragma unroll
    for (int k = 0; k < C; ++k) {
      if ((on >> k) & 1u) {
        GlobalPtr<V> dst = (GlobalPtr<V>)as_global(array_of(k) + out[k]);
        if constexpr (sizeof(V) == 16) *dst = V{v[k].x, v[k].y, v[k].z, v[k].w};
        else if constexpr (sizeof(V) == 8) *dst = V{v[k].x, v[k].y};
        else *dst = (V)v[k].x;
      }
    }
  }
  // (array_of(k): the caller's array for item k; a batch of an empty tree gives zeros and a flag)
  template <typename F>
  __device__ __forceinline__ void store(uint32_t N, uint32_t& flags, F&& array_of) {
    if (count == 0) return;
    if (__builtin_expect(wave_value(slot[0]) >= N, 0)) {
#pragma unroll
      for (int k = 0; k < M; ++k) v[k] = make_uint4(0, 0, 0, 0);
      if (on) flags |= 1u;
    }
    if (M > 2 && count > 2) store_some<M>(array_of);
    else store_some<M < 2 ? M : 2>(array_of);
  }
  template <int C, typename F>
  __device__ __forceinline__ void store_some(F&& array_of) {
    if (w == 16u) store_as<C, Words4>(array_of);
    if (w == 8u) store_as<C, Words2>(array_of);
    if (w == 4u) store_as<C, uint32_t>(array_of);
    if (w == 2u) store_as<C, uint16_t>(array_of);
    if (w == 1u) store_as<C, uint8_t>(array_of);
  }
};
// Items i .. end - 1 of one field of a gather (counted within the field), U at a time: the loads of all, then the stores
// of all.  (nodes: the batch's slots; one beyond the tree gives zeros and a flag)
template <int U, typename V>
__device__ __forceinline__ void gather_span(uint32_t i, uint32_t end, uint32_t n, uint32_t epr, uint32_t recip, uint32_t E, uint32_t row_stride,
                                            const uint8_t* col, uint8_t* io, const uint32_t* nodes, uint32_t N, uint32_t& flags) {
  typedef std::conditional_t<(sizeof(V) < 4), uint32_t, V> Kept;   // (as bytes the compiler packs them and takes them apart again)
#pragma unroll 1
  for (; i < end; i += U) {
    Kept v[U];
    uint32_t slot[U], row[U], at[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {   // (beyond the end: the first piece again, so that no load stands in a branch)
      asm volatile("" ::: "memory");   // (one after the other, as in prepare)
      const uint32_t el = (i + k) * 64u + (threadIdx.x & 63u);
      uint32_t r = row_of_piece(el, epr, recip);
      const bool on = i + k < end && r < n;
      const uint32_t within = on ? (el - r * epr) * (uint32_t)sizeof(V) : 0u;
      r = on ? r : 0u;
      at[k] = within + (uint32_t)sizeof(V) > E ? E - (uint32_t)sizeof(V) : within;   // (wide pieces: the last one ends with the field)
      slot[k] = nodes[r];
      row[k] = on ? r : 0xFFFFFFFFu;
    }
#pragma unroll
    for (int k = 0; k < U; ++k) v[k] = *(GlobalPtr<const V>)as_global(col + (uint64_t)(slot[k] < N ? slot[k] : 0u) * row_stride + at[k]);
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (row[k] != 0xFFFFFFFFu) {
        if (!(slot[k] < N)) {
          v[k] = Kept{};
          flags |= 1u;
        }
        *(GlobalPtr<V>)as_global(io + (row[k] * E + at[k])) = (V)v[k];   // (at most 1024 rows of at most 1 MiB)
      }
  }
}
// Items first .. last - 1 of a list, from beginning to end, a field at a time: what a field asks for is looked up once and the
// code for its access width is straight.  What bounds it is the trip to memory per U items, and what it costs to work out
// the items' places.  Item by item, two at a time, with every lookup anew, a step on 10 000 leaves at K = 16 took 125 us with
// 512 rows of one 165-byte field (1320 items), 15.5 with 512 rows of 165 bytes in five fields, 11.0 with 513 of 41 bytes;
// so it takes 30.7, 8.2 and 6.9.  (U = 8 where the registers allow it: 64 rows' worth of 16-byte pieces for each of eight waves
// is one trip then, 6.6 -> 6.1 us a step on 100 000 leaves; looped and not unrolled over the items: the code a round goes
// through has to stay within the instruction cache.)  array_of(f, io): the caller's array of field f, io: as the list has it.
template <int U, typename F>
__device__ __forceinline__ void gather_spans(const PieceFields& pf, uint32_t first, uint32_t last, const uint32_t* nodes, uint32_t N,
                                            uint32_t row_stride, uint64_t step, uint32_t& flags, F&& array_of) {
  const uint32_t n = wave_value(pf.n);
  const uint8_t* base = wave_pointer(pf.base);
#pragma unroll 1
  while (first < last) {
    const uint32_t f = field_of_item(pf, first);
    const uint32_t E = wave_value(pf.bytes[f]), w = wave_value(pf.width[f]), recip = wave_value(pf.recip[f]), epr = (E + w - 1) / w;
    const uint32_t f0 = wave_value(pf.first[f]), fend = wave_value(pf.end[f]), end = fend < last ? fend : last;
    const uint8_t* col = base + wave_value(pf.off[f]);
    uint8_t* io = array_of(f, wave_pointer(pf.io[f])) + step * (wave_value64(pf.step_rows) * E);
    if (w == 16u) gather_span<U, Words4>(first - f0, end - f0, n, epr, recip, E, row_stride, col, io, nodes, N, flags);
    if (w == 8u) gather_span<U, Words2>(first - f0, end - f0, n, epr, recip, E, row_stride, col, io, nodes, N, flags);
    if (w == 4u) gather_span<U, uint32_t>(first - f0, end - f0, n, epr, recip, E, row_stride, col, io, nodes, N, flags);
    if (w == 2u) gather_span<U, uint16_t>(first - f0, end - f0, n, epr, recip, E, row_stride, col, io, nodes, N, flags);
    if (w == 1u) gather_span<U, uint8_t>(first - f0, end - f0, n, epr, recip, E, row_stride, col, io, nodes, N, flags);
    first = end;
  }
}
// The rows of an insertion at ring slot `cursor`, items first, first + every, ..; row j is left out where bit j of skip is set.
__device__ __forceinline__ void place_row_piece(const RowItem& p, uint8_t* base, uint32_t cursor, uint32_t N, uint32_t row_stride, const uint32_t* skip,
                                                const uint4& v) {
  if (p.row == 0xFFFFFFFFu || (skip && ((skip[p.row >> 5] >> (p.row & 31u)) & 1u))) return;
  store_piece(base + (uint64_t)ring_slot(cursor, p.row, N) * row_stride + p.at, p.w, v);
}
template <typename F>
__device__ __forceinline__ void insert_rows(const PieceFields& pf, uint32_t items, uint32_t first, uint32_t every, uint32_t cursor, uint32_t N,
                                            uint32_t row_stride, uint64_t step, const uint32_t* skip, F&& array_of) {
#pragma unroll 1
  for (uint32_t e = first; e < items; e += every) {
    const RowItem p = find_item(pf, e);
    if (p.row != 0xFFFFFFFFu) place_row_piece(p, wave_pointer(pf.base), cursor, N, row_stride, skip, load_piece(array_of(p) + step * p.step + p.out, p.w));
  }
}
// Waits until this wave's loads have arrived and its stores have been acknowledged.
__device__ __forceinline__ void wait_memory() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// Orders LDS accesses of one wave (which the hardware keeps in order) for the compiler.
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The tree work of one round, as the lanes of the team see it.  MEM: the leaves are in memory.  (A compile-time choice:
// one pointer for both places would make flat accesses, and the wait for one of those is a wait for every load and
// store the wave has under way; a branch at every access costs the registers of both sides.)
constexpr uint32_t kTopNodes = 128;   // a level of at most this many nodes is summed by one wave, with all levels above it
template <int MEM>
struct TreeView {
  float* tree;               // the LDS copy
  float *leaves, *level1;    // MEM: the leaves, the level above them (else they are in the copy, the leaves at offset 0)
  uint32_t off_reg, n_reg;   // lane v of every wave: off[v], real nodes of level v (read from there: an LDS trip less per level)
  uint32_t V, N;
  uint32_t vt;               // the lowest level above the leaves of at most kTopNodes nodes
  uint32_t* s_max;           // running maximum (a team of one wave keeps its own)
  uint32_t* s_arrived;       // team waves that have come to one of its barriers, over all barriers (LDS)
  bool apart;                // there are waves outside the team
  uint32_t team;             // lanes of the team
  uint32_t* s_wild;          // the latest sampling with a uniform outside [0, 1) (0: none)
  const uint32_t* nodes;     // the leaves sampled last (LDS)
  uint32_t met;              // what s_arrived has to reach at the team's next barrier, less a team's waves
  __device__ __forceinline__ uint32_t off(uint32_t v) const { return (uint32_t)__builtin_amdgcn_readlane((int)off_reg, (int)v); }
  __device__ __forceinline__ void set_leaf(uint32_t i, float v) const {
    if constexpr (MEM) as_global(leaves)[i] = v;
    else tree[i] = v;
  }
  __device__ __forceinline__ float leaf(uint32_t i) const {
    if constexpr (MEM) return as_global(leaves)[i];
    else return tree[i];
  }
  __device__ __forceinline__ void set_node(uint32_t v, uint32_t i, float x) const {   // v > 0
    if constexpr (MEM > 1) {
      if (v == 1) {
        as_global(level1)[i] = x;
        return;
      }
    }
    tree[off(v) + i] = x;
  }
  __device__ __forceinline__ uint32_t n(uint32_t v) const { return (uint32_t)__builtin_amdgcn_readlane((int)n_reg, (int)v); }
  // Barrier of the team between phases that hand leaves or sums to other waves of it.  The hardware's barrier would hold
  // the team until the row waves come by; the team's waves count themselves in LDS instead (all of them are resident, and
  // each comes to every barrier, so the wait ends).  Leaves stored to memory are not waited for: the waves of a workgroup
  // share a compute unit, whose memory accesses pass its first-level cache in the order they are issued (which is why a
  // fence of workgroup scope waits for none either).
  __device__ __forceinline__ void sync() {
    if (!apart) {
      lds_barrier();
      return;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if ((threadIdx.x & 63u) == 0) atomicAdd(s_arrived, 1u);
    met += team >> 6;
    while ((int)(wave_value(*(volatile uint32_t*)s_arrived) - met) < 0) {}
    asm volatile("" ::: "memory");
  }
};
// Sum of the children of node `parent` of level v, by a single lane.
template <int LOGK, int MEM>
__device__ __forceinline__ float child_group_sum(const TreeView<MEM>& tv, uint32_t v, uint32_t parent) {
  constexpr int R = Wide<LOGK>::R;
  if constexpr (MEM) {
    if (v == 1) return sum_chunks<R / 4>(as_global(static_cast<const float*>(tv.leaves)) + (size_t)parent * R);
    if (MEM > 1 && v == 2) return sum_chunks<R / 4>(as_global(static_cast<const float*>(tv.level1)) + (size_t)parent * R);
  }
  return sum_chunks<R / 4>(static_cast<const float*>(tv.tree) + tv.off(v - 1) + (size_t)parent * R);
}

// x of the lane whose number differs in bit STEP, where the lanes of a block of 2^STEP all hold the same value (see
// butterfly_move; from sixteen lanes on two halves of a register pair trade rows).
template <int STEP>
__device__ __forceinline__ float add_other_half(float x) {
  if constexpr (STEP <= 3) {
    return x + __int_as_float(butterfly_move<STEP>(__float_as_int(x)));
  } else {
    const unsigned b = __float_as_uint(x);
    auto p = [&] {
      if constexpr (STEP == 4) return __builtin_amdgcn_permlane16_swap(b, b, false, false);
      else return __builtin_amdgcn_permlane32_swap(b, b, false, false);
    }();
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
  }
}
// The sums over blocks of 2, 4, .. 64 lanes of x, the nodes of level vt from node `base` on; those that are nodes of a
// level below the root are stored.  Returns the sum of all.
template <int LOGR, int STEP, int MEM>
__device__ __forceinline__ float sums_above(const TreeView<MEM>& tv, float x, uint32_t base) {
  if constexpr (STEP < 6) {
    x = add_other_half<STEP>(x);
    constexpr uint32_t done = STEP + 1;
    if constexpr (done % LOGR == 0) {
      const uint32_t lane = threadIdx.x & 63u, v = tv.vt + done / LOGR, node = (base + lane) >> done;
      if (v < tv.V && (lane & ((1u << done) - 1u)) == 0 && node < tv.n(v)) tv.tree[tv.off(v) + node] = x;
    }
    return sums_above<LOGR, STEP + 1>(tv, x, base);
  } else {
    return x;
  }
}
// The levels from vt up, recomputed whole by one wave: a lane or two per node of level vt, and above it no trips through
// LDS, only sums of neighbouring lanes (a height of sixteen children was a trip and a chain of 450 cycles, whatever its
// few nodes).  Returns the root.
template <int LOGK, int MEM>
__device__ __forceinline__ float sum_top(const TreeView<MEM>& tv) {
  constexpr int LOGR = Wide<LOGK>::LOGR;
  const uint32_t lane = threadIdx.x & 63u, n = tv.n(tv.vt), at = tv.off(tv.vt);
  const bool two = n > 64u;
  float x = 0.0f, y = 0.0f;
  if (lane < n) x = child_group_sum<LOGK, MEM>(tv, tv.vt, lane);
  if (two && lane + 64u < n) y = child_group_sum<LOGK, MEM>(tv, tv.vt, lane + 64u);
  if (lane < n) tv.tree[at + lane] = x;
  x = sums_above<LOGR, 0>(tv, x, 0u);
  if (two) {
    if (lane + 64u < n) tv.tree[at + 64u + lane] = y;
    x = x + sums_above<LOGR, 0>(tv, y, 64u);
  }
  if (tv.vt < tv.V && lane == 0) tv.tree[tv.off(tv.V)] = x;
  return x;
}

// An update (lane tid < n of the team: leaf i gets v) and then an insertion (lanes with `mine`: row at ring slot `slot`, its
// value or the running maximum), and the ancestors of both in one pass.  Called by the team.
struct UpdateWork {
  bool on, mine, sorted;     // mine: this lane has an element; sorted: the indices are those of the batch sampled last
  bool counted;              // several waves: the running maximum has the elements' values already (see note_update)
  uint32_t n, i, size;       // n: elements (0: no update)
  float v;
  const float* prio;         // sorted, several waves: the values of all elements
  uint32_t batch;            // likewise: the number of that sampling (from 1 on)
};
struct InsertWork {
  bool on, mine, given;      // given: the value is `v`, else the running maximum
  bool whole;                // every row is placed: no deferred ones, no values that may not be valid
  uint32_t n, first, slot;   // first: ring slot of row 0
  float v;
};
// The same as valid_priority(v), in one instruction: plus or minus zero, positive and finite.
__device__ __forceinline__ bool priority_class(float v) { return __builtin_isfpclass(v, 0x20 | 0x40 | 0x80 | 0x100); }
__device__ __forceinline__ bool check_element(const UpdateWork& u, uint32_t& flags) {
  if (!u.mine) return false;
  if (!(u.i < u.size)) flags |= 1u;
  else if (!priority_class(u.v)) flags |= 2u;
  else return true;
  return false;
}

// By a team of one wave.  lane_max: the lanes' share of the running maximum (the greatest of them is it).  Returns the root.
// (Sampled leaves come in order from uniforms in [0, 1): the targets do not decrease then, and the walk keeps their order.
// Elements of one leaf are neighbours and the last of them wins.  One look at the leaves and values says whether that is
// so; where it is not, and for indices that were not sampled, markers decide.  The code of a step that has neither an
// update nor an insertion left out runs without a branch up to the sums: at an instruction every five cycles a branch
// around three of them is no gain.)
template <int LOGK, int MEM>
__device__ __forceinline__ float change_by_wave(TreeView<MEM>& tv, const UpdateWork& u, const InsertWork& ins, float& lane_max,
                                                uint32_t& flags, float total) {
  constexpr int LOGR = Wide<LOGK>::LOGR;
  const uint32_t tid = threadIdx.x;
  const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u.i, 0x130 /* wave_shl:1: from the lane above */, 0xF, 0xF, true);
  const bool last = not_before_here(tid) + 1u >= u.n;   // (worked out here each time: as a mask kept over the steps it costs more, scalar registers are short)
  bool valid = u.mine, won = u.mine && (last || next != u.i);
  const bool plain = u.sorted && __all(!u.mine || (u.i < u.size && priority_class(u.v) && (last || next >= u.i)));
  if (__builtin_expect(!plain, 0)) {   // (out of the way: the code of a round is fetched line by line as it goes)
    valid = check_element(u, flags);
    const uint32_t mark = 0x80000001u + tid;
    if constexpr (MEM) {   // (markers in memory: atomics there, and a read that passes by the first-level cache)
      GlobalPtr<uint32_t> bits = (GlobalPtr<uint32_t>)tv.leaves;
      wait_memory();
      if (valid) __hip_atomic_fetch_max(&bits[u.i], mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      wait_memory();
      won = valid && __hip_atomic_load(&bits[u.i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == mark;
      wait_memory();
    } else {
      uint32_t* bits = reinterpret_cast<uint32_t*>(tv.tree);
      if (valid) atomicMax(&bits[u.i], mark);
      wave_order();
      won = valid && bits[u.i] == mark;
      wave_order();
    }
  }
  if (won) tv.set_leaf(u.i, u.v);
  if (valid && u.v > lane_max) lane_max = u.v;
  wave_order();
  bool placed = ins.mine;
  if (ins.on) {
    float v = ins.v;
    if (ins.given) {
      placed = ins.mine && priority_class(v);
      if (ins.mine && !placed) flags |= 2u;
      if (placed && v > lane_max) lane_max = v;
    } else {
      v = __uint_as_float(wave_max_u32(__float_as_uint(lane_max)));
    }
    if (placed) tv.set_leaf(ins.slot, v);
  }
  // the ancestors (elements that share a parent store the same sum)
  if (u.n + (ins.on ? ins.n : 0u)) {
    const bool together = !ins.on || u.n + ins.n <= 64u;   // (no lane has both)
    if (tv.vt > 1) {
      for (int pass = 0; pass < (together ? 1 : 2); ++pass) {
        const bool act = together ? valid || placed : pass == 0 ? valid : placed;
        const uint32_t leaf = together ? (placed ? ins.slot : u.i) : pass == 0 ? u.i : ins.slot;
        for (uint32_t v = 1; v < tv.vt; ++v) {
          wave_order();
          if (act) {
            const uint32_t parent = leaf >> (v * LOGR);
            tv.set_node(v, parent, child_group_sum<LOGK, MEM>(tv, v, parent));
          }
        }
      }
    }
    wave_order();
    total = sum_top<LOGK, MEM>(tv);
    wave_order();
  }
  return total;
}

// By a team of several waves.
template <int LOGK, int MEM>
__device__ __forceinline__ void change_by_team(TreeView<MEM>& tv, const UpdateWork& u, const InsertWork& ins, uint32_t& flags) {
  constexpr int LOGR = Wide<LOGK>::LOGR;
  const uint32_t tid = threadIdx.x;
  bool valid = false, placed = false;
  if (u.on) {
    valid = check_element(u, flags);
    const uint32_t mark = 0x80000001u + tid;
    bool won = valid, in_order = u.sorted;
    if (in_order) {
      // The last valid element of every run of equal leaves wins (the leaves are in order where no uniform was out of
      // range, else the sampling has left its number in *tv.s_wild).  Within a wave that is read off two masks: where runs
      // begin, and which elements are valid.  A run that reaches the end of its wave may go on in the next one; its last
      // lane then looks at the elements behind it, seldom more than one (their leaves are still in LDS as they were sampled).
      const unsigned lane = tid & 63u;
      const uint32_t wild = *tv.s_wild, behind_wave = (tid | 63u) + 1u;
      const uint32_t next_leaf = behind_wave < u.n ? tv.nodes[behind_wave] : 0xFFFFFFFFu;
      const uint32_t below = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u.i, 0x138 /* wave_shr:1: from the lane below */, 0xF, 0xF, true);
      const unsigned long long begins = __ballot(u.mine && (lane == 0 || below != u.i)), good = __ballot(valid);
      const unsigned long long later = lane == 63u ? 0ull : begins >> (lane + 1u);
      const unsigned run_end = later ? lane + 1u + (unsigned)__builtin_ctzll(later) : 64u;   // first lane behind this lane's run
      const unsigned long long behind = lane == 63u ? 0ull : (good >> (lane + 1u)) & (run_end == 64u && lane == 0 ? ~0ull : (1ull << (run_end - lane - 1u)) - 1ull);
      won = valid && !behind;
      in_order = wave_value(wild) != u.batch;
      if (in_order && won && run_end == 64u && next_leaf == u.i)
        for (uint32_t j = behind_wave; won && j < u.n && tv.nodes[j] == u.i; ++j) won = !priority_class(as_global(u.prio)[j]);
    }
    if (__builtin_expect(!in_order, 0)) {
      if constexpr (MEM) {
        GlobalPtr<uint32_t> bits = (GlobalPtr<uint32_t>)tv.leaves;
        wait_memory();
        tv.sync();
        if (valid) __hip_atomic_fetch_max(&bits[u.i], mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        wait_memory();
        tv.sync();
        won = valid && __hip_atomic_load(&bits[u.i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == mark;
        wait_memory();
        tv.sync();
      } else {
        uint32_t* bits = reinterpret_cast<uint32_t*>(tv.tree);
        if (valid) atomicMax(&bits[u.i], mark);
        tv.sync();
        won = valid && bits[u.i] == mark;
        tv.sync();
      }
    }
    // The insertion comes behind the update.  Where it fills its stretch of the ring whole, the update leaves the leaves
    // there alone, and no barrier of the team is needed between the two.
    const bool leave = ins.on && ins.whole;
    const uint32_t at = u.i >= ins.first ? u.i - ins.first : u.i + (tv.N - ins.first);
    if (won && !(leave && at < ins.n)) tv.set_leaf(u.i, u.v);
    if (!u.counted) {
      const uint32_t m = wave_max_u32(valid && u.v > 0.0f ? __float_as_uint(u.v) : 0u);
      if ((tid & 63u) == 0 && m) atomicMax(tv.s_max, m);
    }
    if (ins.on && !(leave && (u.counted || ins.given))) tv.sync();
  }
  if (ins.on) {
    uint32_t mx = 0;
    if (ins.mine) {
      float v = __uint_as_float(*tv.s_max);
      placed = true;
      if (ins.given) {
        v = ins.v;
        placed = priority_class(v);
        if (!placed) flags |= 2u;
        mx = placed && v > 0.0f ? __float_as_uint(v) : 0u;
      }
      if (placed) tv.set_leaf(ins.slot, v);
    }
    if (ins.given && mx) atomicMax(tv.s_max, mx);
  }
  // the ancestors (elements that share a parent store the same sum)
  if (u.on || ins.on) {
    // A level of no more nodes than there are elements is recomputed whole (fewer lanes than elements).
    const uint32_t elements = (u.on ? u.n : 0u) + (ins.on ? ins.n : 0u);
    for (uint32_t v = 1; v < tv.vt; ++v) {
      tv.sync();
      const uint32_t nodes = tv.n(v);
      if (nodes <= elements) {
        for (uint32_t j = tid; j < nodes; j += tv.team) tv.set_node(v, j, child_group_sum<LOGK, MEM>(tv, v, j));
        continue;
      }
      const uint32_t pu = u.i >> (v * LOGR), pi = ins.slot >> (v * LOGR);
      if (valid) tv.set_node(v, pu, child_group_sum<LOGK, MEM>(tv, v, pu));
      if (placed) tv.set_node(v, pi, child_group_sum<LOGK, MEM>(tv, v, pi));
    }
    tv.sync();
    if (tid < 64u) sum_top<LOGK, MEM>(tv);
  }
}

// The values of the update that comes next raise the running maximum as soon as its elements are known: an insertion
// behind that update finds it raised, without a barrier between the two.  (Only where nothing reads the maximum before the
// update.)  Called by whole waves of a team of several.
__device__ __forceinline__ void note_update(bool mine, uint32_t i, uint32_t size, float v, uint32_t* s_max) {
  const uint32_t m = wave_max_u32(mine && i < size && valid_priority(v) && v > 0.0f ? __float_as_uint(v) : 0u);
  if ((threadIdx.x & 63u) == 0 && m) atomicMax(s_max, m);
}

// Waves of the team with a uniform outside [0, 1) (or -0, which does no harm) leave the number of the sampling.  Lanes without
// a sample hold 0, or a uniform of an earlier one.
__device__ __forceinline__ void note_wild(float u, uint32_t batch, uint32_t* s_wild) {
  if (__builtin_expect(__any(__float_as_uint(u) >= 0x3F800000u), 0)) *s_wild = batch;
}

// One level down: grp points at the children of `node`.
template <int LOGR, typename P>
__device__ __forceinline__ void level_down(P grp, float& r, uint32_t& node, float& val) {
  constexpr int R = 1 << LOGR;
  if constexpr (R <= 16) {
    float c[R];
#pragma unroll
    for (int k = 0; k < R / 4; ++k) {
      const Floats4 x = load_floats4(grp + 4 * k);
      c[4 * k] = x.x, c[4 * k + 1] = x.y, c[4 * k + 2] = x.z, c[4 * k + 3] = x.w;
    }
    turn_down<R>(c, r, node, val);
  } else {   // by the sums of its chunks first; the chosen chunk is read again
    float sums[R / 4];
#pragma unroll
    for (int k = 0; k < R / 4; ++k) {
      const Floats4 x = load_floats4(grp + 4 * k);
      sums[k] = (x.x + x.y) + (x.z + x.w);
    }
    uint32_t chunk = 0;
    turn_down<R / 4>(sums, r, chunk, val);
    const Floats4 x = load_floats4(grp + 4 * chunk);
    const float c[4] = {x.x, x.y, x.z, x.w};
    node = node * (R / 4) + chunk;
    turn_down<4>(c, r, node, val);
  }
}

// Sample i of n (lane i of the team; lanes beyond repeat the last one), uniform u, with seg = total / n: leaf and value,
// 0xFFFFFFFF and 0 where nothing can be sampled.
// A binary step goes right iff the right block is not zero and not r < left block.  That the right block is zero while
// r is not below the left one takes a rounding, or a uniform outside [0, 1): the first walk does not look, and arrives
// at a leaf of zero if it ever should have stayed (a block of sum zero holds nothing else, and nodes beyond a level's
// last have the group of zeros behind its groups for children).  Where that happens to any lane the wave walks again,
// looking.  `call` is called once, behind the few nodes below the root or before the walk's last level (or where there is no
// walk).  (With the right blocks' sums left out, and the sixteen children kept in registers instead of read a second
// time once the chunk of four is known, a level takes two thirds of the 570 cycles it took.)
template <int LOGK, int MEM, bool CALL_LAST, typename F>
__device__ __forceinline__ void walk_tree(const TreeView<MEM>& tv, uint32_t i, uint32_t n, float u, float total, float seg, uint32_t& node,
                                          float& val, F&& call) {
  constexpr int LOGR = Wide<LOGK>::LOGR, R = Wide<LOGK>::R;
  node = 0xFFFFFFFFu;
  val = 0.0f;
  if (!(total > 0.0f)) {
    call();
    return;
  }
  const float r0 = ((float)(i < n ? i : n - 1) + u) * seg;
  float r = r0;
  node = 0;
  uint32_t v = tv.V - 1;
  if (R > 4 && v > 0 && tv.n(v) <= 4u) {   // (few children of the root, the same for all lanes)
    const Floats4 x = load_floats4(static_cast<const float*>(tv.tree) + tv.off(v));
    const float c[4] = {x.x, x.y, x.z, x.w};
    turn_down<4>(c, r, node, val);
    --v;
  }
  if constexpr (!CALL_LAST) call();
  float unused;
  for (; v > (MEM > 1 ? 1u : 0u); --v)
    level_down<LOGR>(static_cast<const float*>(tv.tree) + tv.off(v) + (size_t)min_u32(node, tv.n(v + 1)) * R, r, node, unused);
  bool astray = false;
  if constexpr (MEM > 1) {
    astray = node >= tv.n(2);
    level_down<LOGR>(as_global(static_cast<const float*>(tv.level1)) + (size_t)(astray ? 0u : node) * R, r, node, unused);
  }
  if constexpr (CALL_LAST) call();
  const uint32_t n1 = tv.n(1);
  if constexpr (MEM) {   // (no such group behind the leaves in memory)
    const bool beyond = node >= n1;
    astray = astray || beyond;
    level_down<LOGR>(as_global(static_cast<const float*>(tv.leaves)) + (size_t)(beyond ? 0u : node) * R, r, node, val);
  } else {
    level_down<LOGR>(static_cast<const float*>(tv.tree) + (size_t)min_u32(node, n1) * R, r, node, val);
  }
  if (__builtin_expect(__any(astray || !(val > 0.0f)), 0)) {
    r = r0;
    node = 0;
    for (v = tv.V; v-- > 0;) {
      unsigned child;
      if constexpr (MEM) {
        if (v == 0) descend_looking<LOGR>(as_global(static_cast<const float*>(tv.leaves)) + (size_t)node * R, r, child, val);
        else if (MEM > 1 && v == 1) descend_looking<LOGR>(as_global(static_cast<const float*>(tv.level1)) + (size_t)node * R, r, child, val);
        else descend_looking<LOGR>(static_cast<const float*>(tv.tree) + tv.off(v) + (size_t)node * R, r, child, val);
      } else {
        descend_looking<LOGR>(static_cast<const float*>(tv.tree) + tv.off(v) + (size_t)node * R, r, child, val);
      }
      node = node * R + child;
    }
  }
}
// total / n, the mass a sample stands for.  Where n is a power of two the product with its reciprocal is the same number
// (the scaled total, rounded once either way) without the steps of a division.
__device__ __forceinline__ float mass_per_sample(float total, uint32_t n) {
  const float fn = (float)n;
  return (n & (n - 1u)) == 0u ? total * __uint_as_float(0x7F000000u - __float_as_uint(fn)) : total / fn;
}

// Smallest of the n <= 512 values in LDS (as bits, which order like positive values), by every calling wave for itself.  Called by
// whole waves.
__device__ __forceinline__ uint32_t smallest_value(const float* values, uint32_t n) {
  const uint32_t lane = threadIdx.x & 63u;
  uint32_t m = 0xFFFFFFFFu;
  if (n <= 64u) {
    if (lane < n) m = __float_as_uint(values[lane]);
  } else {
#pragma unroll
    for (uint32_t k = 0; k < 2; ++k) {
      const uint32_t e = 4u * (k * 64u + lane);
      const Floats4 x = load_floats4(values + e);
      const int left = (int)n - (int)e;   // (one number and four constants: e + 1 .. e + 3 were kept over the rounds, spilled)
      if (left > 0) m = min_u32(m, __float_as_uint(x.x));
      if (left > 1) m = min_u32(m, __float_as_uint(x.y));
      if (left > 2) m = min_u32(m, __float_as_uint(x.z));
      if (left > 3) m = min_u32(m, __float_as_uint(x.w));
    }
  }
  return wave_min_u32(m);
}

// Who does the tree work: the first wave, the first few, or every wave, which then moves the rows as well.
// (TEAM_WAVES_SPANS, of a list: where a step's gather is more than its row waves have under way at once.  Only as long as every
// step is fetched ahead: else, with all results waited for in between, every wave at the rows is the faster way, 256 rows of
// 165 bytes in five fields on 10 000 leaves at K = 16 6.0 us a step, 7.7 by the waves that are not the team's.)
enum TeamForm { TEAM_ONE_WAVE, TEAM_WAVES, TEAM_WAVES_SPANS, TEAM_ALL };
static TeamForm team_form(uint32_t samples, uint32_t inserted) {
  const uint32_t most = samples > inserted ? samples : inserted;
  return most <= 64 ? TEAM_ONE_WAVE : most <= 512 ? TEAM_WAVES : TEAM_ALL;
}

// The list of steps.  What bounds it is one chain of instructions and LDS trips from step to step (the tree as one
// step leaves it is what the next samples from), so everything that is not tree work is taken off that chain:
//  - The waves split: the first ones (the team, a lane per sample and per inserted row) do the tree work, the others
//    move the rows and turn values into weights, one step behind, each in a loop of its own.  (As one loop that asks
//    every wave at every turn what it is, the bookkeeping was a quarter of a step.)  Batches of more than 512 leave no
//    waves over; the team then does both in turn.
//  - Inputs are fetched a step ahead.  That is only right where no step reads what a step returns; the host has checked
//    it (StreamArgs::ahead).  Where it does not hold, a step's results are stored and waited for before its update and
//    the inputs of the step behind it are fetched (a build of its own: as a branch it costs the other lists 2 to 5 %, 50
//    steps of 100 samples on 15 000 leaves at K = 8 198 -> 214 us).
//  - The update of step s and the insertion of step s + 1 are adjacent tree changes with nothing read in between: the
//    leaves are written one after the other and the ancestors of both recomputed in one pass.
//  - WAVE: with at most 64 samples and 64 new rows the team is one wave, whose LDS accesses stay in order by
//    themselves: no barriers inside the tree work, two per step in all.  Several team waves meet at barriers of their own
//    (counted in LDS), which do not wait for the row waves.
//  - Barriers wait for LDS only.  A __syncthreads() also waits for every store of the wave to be acknowledged from
//    memory, a microsecond at each phase that writes results or rows.
// The order that memory needs: the stored rows of an insertion are read by the gather of the same step at the earliest
// (its loads are issued behind the barrier that ends the sampling), and overwrite what the gather of the step before has
// read (whose loads are issued in front of the barrier before the insertion's stores); the accesses of a workgroup's waves
// keep that order (see TreeView::sync).
// 100 steps on 10 000 leaves at K = 16 (32 samples, 4 new rows of 41 bytes): 166 us; 1001 us as one phase after the
// other by the whole workgroup with a full barrier between them.
// AHEAD: no step reads what a step returns.  ROOT: the root is not current (see sum_stale_root).
template <int LOGK, TeamForm FORM, int MEM, bool AHEAD, bool ROOT = false>
__global__ void __launch_bounds__(1024)
k_run_steps(StreamKernelArgs ka) {
  constexpr bool WAVE = FORM == TEAM_ONE_WAVE, apart = FORM != TEAM_ALL, SPANS = FORM == TEAM_WAVES_SPANS || FORM == TEAM_ALL;
  const Geom& g = ka.g;
  const StreamArgs& a = ka.a;
  extern __shared__ __attribute__((aligned(16))) float tree[];
  __shared__ LevelTable tab;
  __shared__ uint32_t s_off[kStreamLevels + 2], s_n[kStreamLevels + 1];
  __shared__ uint32_t s_max, s_vmin[2], s_bmin[2], s_wild, s_arrived, s_whole, s_taken;
  __shared__ PieceFields s_rows, s_ins;
  __shared__ uint2 s_share[16];
  const uint32_t t = blockIdx.x;
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint32_t H = g.H, T = g.T, B = a.B, n_ins = a.n_insert, N = g.N;
  const uint32_t V = a.plan.levels;
  fill_stream_tables(t, kernarg_at<StreamPlan>(offsetof(StreamKernelArgs, a) + offsetof(StreamArgs, plan)), &tab, s_off, s_n);
  // (the lists a lane per field, by two waves)
  PieceCopy list;
  uint2 share = make_uint2(0, 0);
  const bool lists = tid >= 384 && tid < 512;
  if (lists) {
    list.read(kernarg_at<PieceList>(tid < 448 ? offsetof(StreamKernelArgs, rows) : offsetof(StreamKernelArgs, ins)), t);
    share = kernarg_at<uint2>(offsetof(StreamKernelArgs, share))[lane & 15u];
  }
  uint32_t max_seen = 0;
  if (tid == 0) {
    max_seen = read_max_bits(g, t);   // (on its way while the tree is asked for)
    s_vmin[0] = s_vmin[1] = s_bmin[0] = s_bmin[1] = kNoMin;
    s_wild = 0;
    s_arrived = 0;
    s_whole = s_taken = 0;
  }
  // lanes of the team, of the rows, of the weights
  const uint32_t wanted = WAVE ? 64u : ((B > n_ins ? B : n_ins) + 63u) / 64u * 64u;
  const uint32_t team = apart ? wanted : 1024u;   // (not apart: every wave comes to the team's barriers)
  const bool in_team = tid < team;
  const uint32_t rn = apart ? 1024u - team : 1024u, rl = apart ? tid - team : tid;
  const uint32_t rw = wave_value(rl >> 6), rws = rn >> 6;   // number of this wave among the row waves, and how many there are
  const uint32_t w0 = apart ? 1024u - (B + 63u) / 64u * 64u : 0u;
  const bool weigher = tid >= w0 && tid - w0 < B;
  __syncthreads();
  if (lists) {
    list.put(t, tid < 448 ? &s_rows : &s_ins);
    if (tid < 400) s_share[lane] = share;
  }
  // inputs of the team: the uniform of the step to sample, value (and index) of the update to apply, inserted priority
  float u_i = 0.0f, u_next = 0.0f, up_v = 0.0f, in_v = 0.0f;
  float beta_i = 0.0f;
  uint32_t up_i = 0;
  const uint32_t j_ins = WAVE ? lane - (64u - n_ins) : tid;   // (WAVE: the last lanes of the wave, so that samples and rows share it)
  const bool inserts = in_team && (!WAVE || lane >= 64u - n_ins) && j_ins < n_ins;
  if (in_team && tid < B) u_i = a.u ? a.u[(size_t)t * B + tid] : counter_uniform(a.rng, tid, t);
  if (inserts && a.ins_prio) in_v = a.ins_prio[(size_t)t * n_ins + j_ins];
  if (!AHEAD || !a.beta) beta_i = a.beta ? a.beta[0] : a.beta_value;
  LdsTree lt;
  lt.tree = tree;
  lt.in_memory = MEM;
  lt.off = s_off;
  lt.n = s_n;
  lt.max_bits = &s_max;
  lt.H = H;
  lt.V = V;
  lds_tree_load<LOGK>(tab, lt, tid, 1024u);
  if (tid == 0) s_max = max_seen;
  uint32_t* nodes = reinterpret_cast<uint32_t*>(tree + s_off[V + 1]);   // [B] sampled leaves of the step
  float* values = reinterpret_cast<float*>(nodes + 512);                // [B] and their values (apart only: B <= 512)
  TreeView<MEM> tv;
  tv.tree = tree;
  tv.leaves = MEM ? tab.lvl[0] : nullptr;
  tv.level1 = MEM > 1 ? tab.lvl[Wide<LOGK>::LH] : nullptr;
  tv.off_reg = s_off[lane <= V + 1 ? lane : V + 1];
  tv.n_reg = s_n[lane <= V ? lane : V];
  tv.V = V;
  tv.N = N;
  tv.vt = 1;
  while (tv.vt < V && tv.n(tv.vt) > kTopNodes) ++tv.vt;
  tv.s_max = &s_max;
  tv.s_arrived = &s_arrived;
  tv.s_wild = &s_wild;
  tv.nodes = nodes;
  tv.apart = apart;
  tv.team = team;
  tv.met = 0;
  __syncthreads();
  if constexpr (ROOT) {
    if (tid == 0) sum_stale_root<LOGK>(tab, lt);
  }
  uint32_t flags = 0;
  float lane_max = __uint_as_float(s_max);   // (WAVE: the lanes' share of it; else s_max counts)

  const bool brief = MEM > 1 || (apart && a.n_steps == 1 && (a.upd_is_sampled || !a.upd_prio));   // (see store_paths; MEM > 1: only launched so)
  auto list_array = [](const RowItem& p) { return p.io; };
  auto work = [&](auto does_tree, auto does_rows) {
    constexpr bool TREE = decltype(does_tree)::value, ROWS = decltype(does_rows)::value;
    const bool gives = a.upd_prio != nullptr, own = a.upd_is_sampled != 0;
    const size_t batch = (size_t)T * B;              // samples of a step, over all trees
    size_t at = (size_t)t * B + tid;                 // this lane's sample in the inputs of step s
    uint32_t cursor = a.cursor, size = a.size, upd_size = 0;
    uint32_t node = 0xFFFFFFFFu;                     // this lane's sample of the step before
    float val = 0.0f;
    float total = tree[s_off[V]];                    // (WAVE: the root as the latest change has left it)
    // this wave's share of the rows, the same in every step: the first item of the insertion, fetched a step ahead, and the
    // items of the gather (SPANS: their numbers; what is kept over the steps for the others takes the registers that the spans
    // have their loads in)
    RowItem ip{};
    ip.row = 0xFFFFFFFFu;
    uint4 iv;
    uint8_t* payload = nullptr;                      // row 0 of this tree
    uint32_t gather_first = 0, gather_last = 0, insert_items = 0;   // items of the insertion
    GatherItems<kInFlight> items;
    uint8_t* io[kInFlight];                          // the caller's arrays for those, in the step before s
    uint64_t io_step[kInFlight];
    if constexpr (ROWS) {
      insert_items = wave_value(s_ins.items);
      payload = wave_pointer(s_ins.base);
      if (rw < insert_items) {
        ip = find_item(s_ins, rw);
        if (ip.row != 0xFFFFFFFFu) iv = load_piece(ip.io + ip.out, ip.w);
      }
      gather_first = wave_value(s_share[rw].x);
      gather_last = wave_value(s_share[rw].y);
      if constexpr (!SPANS)
        items.prepare(s_rows, gather_first, gather_last, [&](int k, const RowItem& p) {
          io[k] = p.io;
          io_step[k] = p.step;
        });
    }
    for (uint32_t s = 0;; ++s) {
      const bool more = s < a.n_steps;
      // ---- rows and weights of the step before
      float w_out = 0.0f, v_out = 0.0f;
      uint32_t n_out = 0;
      if (ROWS && s) {
        if constexpr (SPANS) gather_spans<apart ? 8 : 4>(s_rows, gather_first, gather_last, nodes, N, a.rows_stride, s - 1, flags, [](uint32_t, uint8_t* at) { return at; });
        else items.load(nodes, N, a.rows_stride);
        uint32_t least = 0;
        if (a.out_w && tid >= w0) {   // (whole waves)
          if (a.buffer_norm) least = s_bmin[(s - 1) & 1u];
          else if (TREE) least = s_vmin[(s - 1) & 1u];
          else least = smallest_value(values, B);
        }
        if (weigher) {
          n_out = nodes[tid - w0];
          v_out = TREE ? val : values[tid - w0];
          if (a.out_w) {
            w_out = n_out == 0xFFFFFFFFu ? 0.0f : importance_weight(v_out, __uint_as_float(least), AHEAD && a.beta ? a.beta[s - 1] : beta_i);
          }
        }
      }
      auto store_results = [&]() {   // of the step before
        if (!ROWS || !s) return;
        if constexpr (!SPANS) {
          items.store(N, flags, [&](int k) { return io[k]; });
#pragma unroll
          for (int k = 0; k < kInFlight; ++k) io[k] += io_step[k];
        }
        if (!weigher) return;
        const size_t o = ((size_t)(s - 1) * T + t) * B + (tid - w0);
        a.out_idx[o] = n_out;
        if (a.out_prio) a.out_prio[o] = v_out;
        if (a.out_w) a.out_w[o] = w_out;
      };
      // (One wave of tree work comes late to the next barrier, and soon to the one behind it; several are early at the first
      // and walk longer behind it.)
      constexpr bool stores_first = WAVE || !AHEAD;
      if (stores_first) store_results();
      if (!AHEAD && s) {
        wait_memory();
        lds_barrier();
        if (TREE && tid < B) {
          if (gives) {
            up_v = a.upd_prio[at - batch];
            if (!own) up_i = a.upd_idx[at - batch];
          }
          if (more) u_i = a.u[at];
        }
        if (more) {
          ip.io += ip.step;
          if (ROWS && ip.row != 0xFFFFFFFFu) iv = load_piece(ip.io + ip.out, ip.w);
          if (TREE && inserts && a.ins_prio) in_v = a.ins_prio[((size_t)s * T + t) * n_ins + j_ins];
          beta_i = a.beta[s];
        }
      }
      const bool do_upd = s > 0 && gives, do_ins = more && n_ins > 0;
      const uint32_t first = cursor;
      // (where this step's first piece of the insertion goes, and the next step's: nothing but the store is left to do behind
      // the barrier, which is what the team waits for at the next one)
      uint8_t* place = nullptr;
      uint4 next_iv;
      if (ROWS && do_ins && ip.w) {
        if (AHEAD) ip.io += ip.step;
        if (ip.row != 0xFFFFFFFFu) {
          place = payload + (uint64_t)ring_slot(first, ip.row, N) * a.ins_stride + ip.at;
          if (AHEAD && s + 1 < a.n_steps) next_iv = load_piece(ip.io + ip.out, ip.w);
        }
      }
      // ---- the tree: update of the step before, insertion of this one
      if constexpr (TREE) {
        UpdateWork up;
        up.on = do_upd;
        up.mine = do_upd && tid < B;
        up.sorted = own;
        up.counted = AHEAD;
        up.n = do_upd ? B : 0u;
        up.i = own ? node : up_i;
        up.size = upd_size;
        up.v = up_v;
        up.prio = a.upd_prio + (at - batch - tid);
        up.batch = s;
        InsertWork in;
        in.on = do_ins;
        in.mine = do_ins && inserts;
        in.given = a.ins_prio != nullptr;
        in.whole = !in.given;
        in.n = n_ins;
        in.first = first;
        in.slot = inserts ? ring_slot(first, j_ins, N) : 0u;
        in.v = in_v;
        if constexpr (WAVE) total = change_by_wave<LOGK, MEM>(tv, up, in, lane_max, flags, total);
        else change_by_team<LOGK, MEM>(tv, up, in, flags);
        // inputs of the next round
        if (AHEAD && tid < B) {
          if (more && gives) {
            up_v = a.upd_prio[at];
            if (!own) up_i = a.upd_idx[at];
          }
          if (s + 1 < a.n_steps) u_next = a.u[at + batch];   // (here and not behind the walk: the next wait would be for it)
        }
        if (AHEAD && inserts && s + 1 < a.n_steps && a.ins_prio) in_v = a.ins_prio[((size_t)(s + 1) * T + t) * n_ins + j_ins];
      }
      if (do_ins) {
        cursor = ring_slot(cursor, n_ins, N);
        size = size + n_ins > N ? N : size + n_ins;
      }
      upd_size = size;
      if (!more) {
        if (ROWS && !stores_first) store_results();
        if (TREE && brief) {
          if constexpr (!WAVE) tv.sync();
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          if (tid == 0) *(volatile uint32_t*)&s_whole = 1u;
        }
        break;
      }
      // ---- the rows of the step before have been asked for; the tree is whole.  (A team of one wave has no use for this
      // barrier itself: it passes it as late as the walk allows, where the row waves have long come.)
      const bool late = WAVE && TREE && more && !a.buffer_norm;
      if (!late) lds_barrier();
      if constexpr (ROWS) {
        if (do_ins) {
          if (place) store_piece(place, ip.w, iv);
          if (AHEAD) iv = next_iv;
          if (a.ins_slots)
            for (uint32_t j = rl; j < n_ins; j += rn) a.ins_slots[(size_t)t * n_ins + j] = ring_slot(first, j, N);
          if (rw + rws < insert_items) insert_rows(s_ins, insert_items, rw + rws, rws, first, N, a.ins_stride, s, nullptr, list_array);
        }
        if (!stores_first) store_results();
      }
      if constexpr (ROWS) {
        // (read by the weights of step s - 1, before the barrier)
        if ((TREE || a.buffer_norm) && rl == 0) s_vmin[(s + 1) & 1u] = s_bmin[(s + 1) & 1u] = kNoMin;
        // ---- weights relative to the whole tree: its smallest positive leaf
        if (a.buffer_norm && a.out_w) {
          uint32_t m = kNoMin;
          for (uint32_t e = rl; e < N; e += rn) m = min_u32(m, positive_bits(tv.leaf(e)));
          m = wave_min_u32(m);
          if (lane == 0 && m != kNoMin) atomicMin(&s_bmin[s & 1u], m);
        }
      }
      // ---- sampling
      if constexpr (TREE) {
        if (WAVE || (tid & ~63u) < B) {
          if constexpr (!WAVE) {
            note_wild(u_i, s + 1u, &s_wild);
            total = tree[tv.off(V)];
          }
          walk_tree<LOGK, MEM, true>(tv, tid, B, u_i, total, mass_per_sample(total, B), node, val, [&] {
            if (late) lds_barrier();
          });
          if (node == 0xFFFFFFFFu && tid == 0) flags |= 4u;
          if (ROWS && a.out_w) {
            const uint32_t m = wave_min_u32(tid < B ? __float_as_uint(val) : kNoMin);
            if (lane == 0) atomicMin(&s_vmin[s & 1u], m);
          }
          if (tid < B) {
            nodes[tid] = node;
            if (!ROWS) values[tid] = val;
          }
          if (AHEAD) u_i = u_next;
        }
        if (!WAVE && AHEAD && gives) note_update(tid < B, own ? node : up_i, upd_size, up_v, &s_max);
        at += batch;
      }
      lds_barrier();
    }
  };
  if constexpr (!apart) work(std::true_type{}, std::true_type{});
  else if (in_team) work(std::true_type{}, std::false_type{});
  else work(std::false_type{}, std::true_type{});
  if (WAVE && in_team) {
    const uint32_t m = wave_max_u32(__float_as_uint(lane_max));
    if (tid == 0) s_max = m;
  }
  report_flags(g, t, flags);
  if (brief) {
    if (tid == 0) g.max_v[t] = __uint_as_float(s_max);
    if (a.out_w && tid >= w0) return;   // (the weights are what takes longest)
    store_paths<LOGK, MEM>(tab, lt, a.upd_prio ? nodes : nullptr, B, a.cursor, n_ins, N, &s_taken, &s_whole);
    return;
  }
  __syncthreads();
  lds_tree_store<LOGK>(g, t, tab, lt);
}

// ---------------------------------------------------------------------------------
// a queue of op-coded requests on an LDS-resident tree
// ---------------------------------------------------------------------------------
// The same workgroup-per-tree arrangement, driven by a queue of requests in memory instead of a
// fixed step: each request names its operation (the paper's unified operation code, Section V-A)
// and is decoded when its turn comes.  The queue's length is fixed at launch; the kernel ends after
// its last request.
//
// The requests are taken in rounds of at most one update, then one insertion, then one sampling request: what a step
// of k_run_steps does between two of its samplings, with parts left out where the queue has something else.  A round
// runs as a step does there (see above): tree work and row work in loops of their own, and what a round reads fetched in
// the round before.  One wave decodes: it fetches the requests three rounds ahead (three at a time: a round takes no more) and
// lays out the rounds two ahead, each as one run of words that a wave takes in with two loads, a word per lane; the fields
// of a round are then read from its lanes.  (With every wave at the requests' fields, one LDS trip each, rounds of 64 samples
// on 4096 leaves at K = 16 took 4.0 us where they take 2.0.)  The lists of fields in LDS are made anew only where a request
// asks for other fields or another number of rows than the one before it: making them for every request, and finding
// every wave's items in them, held the round of 512 at 8.5 us, 6.7 without.
// Fetching ahead is only right where a request reads nothing that one just before it writes (an update whose index
// array is the sampled one, say).  The host has checked that (QueueArgs::ahead); where it does not hold, every
// request is a round of its own with an empty one behind it, which brings all results to memory.
// 20 times (insert 16 rows, sample 512, update them) on 30 000 leaves at K = 16: 110 us; 353 us one request after the
// other by the whole workgroup with a full barrier between their phases.  The row waves are at work throughout, and the
// team waits for them at both barriers, a third of the round.
struct QueueKernelArgs {            // one kernel argument (Geom first: see fill_stream_tables)
  Geom g;
  QueueArgs a;
};
constexpr uint32_t kRoundRequests = 3, kRequestWords = sizeof(per_request) / 4;
// A round as words in LDS: its sampling request, the head of its update, its insertion (the count of one it has not is 0), and
// whether the queue goes on up to it.
constexpr uint32_t kRoundSample = 0, kRoundUpdate = kRequestWords, kRoundInsert = 64, kRoundMore = kRoundInsert + kRequestWords;
constexpr uint32_t kRoundWords = kRoundMore + 2, kRoundUpdateWords = kRoundInsert - kRoundUpdate;
static_assert(kRoundWords <= 128 && offsetof(per_request, out_weight) / 4 <= kRoundUpdateWords, "two words per lane, and an update's words among them");
#define PER_REQUEST_WORD(field) (offsetof(per_request, field) / 4)
struct Round {                      // the same, in the lanes of a wave
  uint32_t lo, hi;
  template <uint32_t AT>
  __device__ __forceinline__ uint32_t word() const {
    return (uint32_t)__builtin_amdgcn_readlane((int)(AT < 64 ? lo : hi), (int)(AT & 63u));
  }
  template <uint32_t AT, typename T>
  __device__ __forceinline__ T* pointer() const { return reinterpret_cast<T*>((uint64_t)word<AT + 1>() << 32 | word<AT>()); }
  __device__ __forceinline__ void read(const uint32_t* words) {
    const uint32_t lane = threadIdx.x & 63u;
    lo = words[lane];
    hi = words[64u + lane < kRoundWords ? 64u + lane : 64u];
  }
  __device__ __forceinline__ uint32_t samples() const { return word<kRoundSample + PER_REQUEST_WORD(n)>(); }
  __device__ __forceinline__ uint32_t inserts() const { return word<kRoundInsert + PER_REQUEST_WORD(n)>(); }
  __device__ __forceinline__ uint32_t updates() const { return word<kRoundUpdate + PER_REQUEST_WORD(n)>(); }
  __device__ __forceinline__ bool more() const { return word<kRoundMore>() != 0; }
  // the caller's array of field f, and which fields have one (bit 2f), in the sampling request or the insertion
  template <uint32_t PART>
  __device__ __forceinline__ uint8_t* array(uint32_t f) const {
    static_assert(PART == kRoundSample || PART == kRoundInsert, "");
    const int at = (int)((PART & 63u) + PER_REQUEST_WORD(field) + 2u * f), x = (int)(PART < 64 ? lo : hi);
    return reinterpret_cast<uint8_t*>((uint64_t)(uint32_t)__builtin_amdgcn_readlane(x, at + 1) << 32 | (uint32_t)__builtin_amdgcn_readlane(x, at));
  }
  template <uint32_t PART>
  __device__ __forceinline__ uint32_t asked() const {
    const unsigned long long set = __ballot((PART < 64 ? lo : hi) != 0u);
    return (uint32_t)((set | set >> 1) >> ((PART & 63u) + PER_REQUEST_WORD(field))) & 0x5555u;
  }
};
// Lays out the round that starts with the `left` requests in the lanes of one wave (word w of them in lane w of x or, from 64
// on, of y).  Returns how many it takes.
__device__ __forceinline__ uint32_t lay_out_round(uint32_t x, uint32_t y, uint32_t left, bool single, bool gap, uint32_t* words) {
  const uint32_t lane = threadIdx.x & 63u;
  uint32_t upd = 3, ins = 3, smp = 3, used = 0, stage = 0;   // places of its requests; stage 1: past the update, 2: past the insertion, 3: past the sampling
#pragma unroll
  for (uint32_t k = 0; k < kRoundRequests; ++k) {
    const uint32_t at = k * kRequestWords;
    const uint32_t op = k < left && !gap ? (uint32_t)__builtin_amdgcn_readlane((int)(at < 64 ? x : y), (int)(at & 63u)) : 0u;
    const bool u = op == PER_OP_UPDATE && stage < 1, i = op == PER_OP_INSERT && stage < 2, s = op == PER_OP_SAMPLE && stage < 3;
    if (used == k && (u || i || s) && !(single && k)) {
      if (u) upd = k, stage = 1;
      if (i) ins = k, stage = 2;
      if (s) smp = k, stage = 3;
      used = k + 1;
    }
  }
  if (used == 0 && left && !gap) used = 1;   // (an unknown operation is passed over: the kernel ends whatever the queue holds)
  auto put = [&](uint32_t w, uint32_t value) {
    const uint32_t k = w < kRequestWords ? 0u : w < 2u * kRequestWords ? 1u : 2u;
    const uint32_t part = k == smp ? kRoundSample : k == ins ? kRoundInsert : k == upd ? kRoundUpdate : 0xFFFFFFFFu, j = w - k * kRequestWords;
    if (w < kRoundRequests * kRequestWords && part != 0xFFFFFFFFu && (k != upd || j < kRoundUpdateWords)) words[part + j] = value;
  };
  put(lane, x);
  put(lane + 64u, y);
  if (lane == 0) {
    if (smp == 3) words[kRoundSample + PER_REQUEST_WORD(n)] = 0;
    if (ins == 3) words[kRoundInsert + PER_REQUEST_WORD(n)] = 0;
    if (upd == 3) words[kRoundUpdate + PER_REQUEST_WORD(n)] = 0;
    words[kRoundMore] = left != 0 ? 1u : 0u;
  }
  return used;
}
template <int LOGK, TeamForm FORM, int MEM, bool ROOT = false>
__global__ void __launch_bounds__(1024)
k_run_requests(QueueKernelArgs ka) {
  constexpr bool WAVE = FORM == TEAM_ONE_WAVE, apart = FORM != TEAM_ALL;
  const Geom& g = ka.g;
  const QueueArgs& a = ka.a;
  extern __shared__ __attribute__((aligned(16))) float tree[];
  __shared__ LevelTable tab;
  __shared__ uint32_t s_off[kStreamLevels + 2], s_n[kStreamLevels + 1];
  __shared__ uint32_t s_round[3][kRoundWords];       // round i: s_round[i % 3]
  __shared__ PieceFields s_rows[2], s_ins[2];        // by parity of the round
  __shared__ uint2 s_share[2][16];
  __shared__ uint32_t s_skip[2][32];                 // bit j: row j of the round's insertion is deferred
  __shared__ uint32_t s_max, s_vmin[2], s_bmin[2], s_wild, s_arrived;
  const uint32_t t = blockIdx.x;
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint32_t H = g.H, N = g.N, n_requests = a.n_requests, V = a.plan.levels;
  const FieldTable* fields = kernarg_at<FieldTable>(offsetof(QueueKernelArgs, a) + offsetof(QueueArgs, fields));
  const uint32_t* queue = reinterpret_cast<const uint32_t*>(a.queue);
  const bool single = a.ahead == 0;
  fill_stream_tables(t, kernarg_at<StreamPlan>(offsetof(QueueKernelArgs, a) + offsetof(QueueArgs, plan)), &tab, s_off, s_n);   // (see k_run_steps)
  uint32_t max_seen = 0;
  if (tid == 0) {
    max_seen = read_max_bits(g, t);
    s_vmin[0] = s_vmin[1] = s_bmin[0] = s_bmin[1] = kNoMin;
    s_wild = 0;
    s_arrived = 0;
  }
  if (tid < 64) s_skip[tid >> 5][tid & 31u] = 0;
  // lanes of the team, of the rows (the weights: see k_run_steps)
  const uint32_t team = WAVE ? 64u : apart ? (a.most + 63u) / 64u * 64u : 1024u;
  const bool in_team = tid < team;
  const uint32_t rn = apart ? 1024u - team : 1024u, rl = apart ? tid - team : tid;
  const uint32_t rw = wave_value(rl >> 6), rws = rn >> 6;   // number of this wave among the row waves, and how many there are
  // the decoding wave (one that weighs nothing, as long as there are such): requests of the round to lay out next in its
  // lanes, where they start in the queue
  const bool decodes = !(apart && in_team) && rw == 0;
  uint32_t pos = 0, req_x = 0, req_y = 0, rounds = 0;
  bool gap = false;
  auto fetch = [&] {
    const uint64_t w0 = (uint64_t)(pos < n_requests ? pos : n_requests) * kRequestWords, all = (uint64_t)n_requests * kRequestWords;
    req_x = req_y = 0;
    if (w0 + lane < all) req_x = queue[w0 + lane];
    if (lane + 64u < kRoundRequests * kRequestWords && w0 + lane + 64u < all) req_y = queue[w0 + lane + 64u];
  };
  auto decode = [&] {   // (single: a round with nothing in it behind every request)
    const uint32_t used = lay_out_round(req_x, req_y, pos < n_requests ? n_requests - pos : 0u, single, gap, s_round[rounds % 3u]);
    gap = single && used != 0;
    pos += used;
    ++rounds;
    fetch();
  };
  if (decodes) fetch();
  __syncthreads();
  LdsTree lt;
  lt.tree = tree;
  lt.in_memory = MEM;
  lt.off = s_off;
  lt.n = s_n;
  lt.max_bits = &s_max;
  lt.H = H;
  lt.V = V;
  // The list of one request's fields, by one wave (words: the request's part of its round), with this tree's place in the
  // caller's arrays for an array.  Only where it asks for other fields, or for another number of rows, than the one before
  // it: where the arrays are the waves know from the round.
  auto fill_fields = [&](const uint32_t* words, PieceFields* pf, uint2* share) {
    const uint32_t n = wave_value(words[PER_REQUEST_WORD(n)]);
    bool asked = false;
    if (n && lane < (uint32_t)kMaxFields) {
      const uint32_t* w = words + PER_REQUEST_WORD(field) + 2u * lane;
      asked = (w[0] | w[1]) != 0;
    }
    if (share) fill_piece_fields<apart ? SHARES_ANY : SHARES_EVEN>(fields, asked, t, n, rws, pf, share);
    else fill_piece_fields<SHARES_NONE>(fields, asked, t, n, rws, pf, nullptr);
  };
  // (the first two rounds are laid out, and the fields of the first insertion, beside the others' copy of the tree)
  const uint32_t at_work = apart ? team : 0u;   // first lane of the decoding wave
  if (decodes) {
    decode();
    decode();
    wave_order();
    fill_fields(s_round[0] + kRoundInsert, &s_ins[0], nullptr);
  } else {
    lds_tree_load<LOGK>(tab, lt, tid < at_work ? tid : tid - 64u, 960u);
  }
  if (tid == 0) s_max = max_seen;
  uint32_t* nodes = reinterpret_cast<uint32_t*>(tree + s_off[V + 1]);   // sampled leaves of the round
  float* values = reinterpret_cast<float*>(nodes + 512);                // and their values (apart only: at most 512)
  TreeView<MEM> tv;
  tv.tree = tree;
  tv.leaves = MEM ? tab.lvl[0] : nullptr;
  tv.level1 = MEM > 1 ? tab.lvl[Wide<LOGK>::LH] : nullptr;
  tv.off_reg = s_off[lane <= V + 1 ? lane : V + 1];
  tv.n_reg = s_n[lane <= V ? lane : V];
  tv.V = V;
  tv.N = N;
  tv.vt = 1;
  while (tv.vt < V && tv.n(tv.vt) > kTopNodes) ++tv.vt;
  tv.s_max = &s_max;
  tv.s_arrived = &s_arrived;
  tv.s_wild = &s_wild;
  tv.nodes = nodes;
  tv.apart = apart;
  tv.team = team;
  tv.met = 0;
  const bool lists = !(apart && in_team) && rw == 1;   // (the wave that fills the lists of fields from then on)
  __syncthreads();
  if constexpr (ROOT) {   // (see sum_stale_root)
    if (tid == 0) sum_stale_root<LOGK>(tab, lt);
  }
  uint32_t flags = 0;
  float lane_max = __uint_as_float(s_max);   // (WAVE: the lanes' share of it; else s_max counts)

  auto work = [&](auto does_tree, auto does_rows) {
    constexpr bool TREE = decltype(does_tree)::value, ROWS = decltype(does_rows)::value;
    uint32_t cursor = a.cursor, size = a.size;
    uint32_t node = 0xFFFFFFFFu;             // this lane's sample of the latest sampling request
    float val = 0.0f;
    float total = tree[s_off[V]];            // (WAVE: the root as the latest change has left it)
    uint32_t sampled = 0;                    // sampling requests so far
    Round cur, before, next;                 // this round, the one before it and the one behind it
    cur.read(s_round[0]);
    before = cur;
    uint32_t n_before = 0;                   // samples of the round before
    // what the rounds read: uniform; value and index of the update; inserted priority; rows
    float u_i = 0.0f, u_next = 0.0f, up_v = 0.0f, in_v = 0.0f;
    uint32_t up_i = 0;
    RowItem ip{};
    ip.row = 0xFFFFFFFFu;
    uint4 iv;
    GatherItems<kInFlight, true> items;
    auto list_of = [](uint32_t n, uint32_t asked) { return n ? n << 16 | asked : 0u; };
    // The lists that `items` and `share`, and `ip` and `insert_items`, are of: rows << 16 | fields asked for; and, of the wave
    // that fills them, those in LDS by parity.
    uint32_t sample_list = 0, insert_list = 0, insert_items = 0;
    uint8_t* payload = nullptr;   // row 0 of this tree
    uint32_t in_lds_sample = 0, in_lds_sample_other = 0;   // (this round's and the other one's; of insertions the next round's)
    uint32_t in_lds_insert = 0, in_lds_insert_other = list_of(cur.inserts(), cur.asked<kRoundInsert>());
    uint2 share = make_uint2(0, 0);
    auto inserted_by = [&](uint32_t n) -> uint32_t {   // the row of the insertion that this lane places (>= n: none)
      const uint32_t j = WAVE ? lane - (64u - n) : tid;
      return !WAVE || lane >= 64u - n ? j : 0xFFFFFFFFu;
    };
    // fetches what the tree work of round r reads
    auto fetch_inputs = [&](const Round& r) {
      if (const uint32_t n = r.samples())
        if (tid < n) u_next = as_global(r.pointer<kRoundSample + PER_REQUEST_WORD(u), const float>())[(size_t)t * n + tid];
      if (const uint32_t n = r.updates()) {
        const uint32_t* idx = r.pointer<kRoundUpdate + PER_REQUEST_WORD(idx), const uint32_t>();
        if (tid < n) {
          up_v = as_global(r.pointer<kRoundUpdate + PER_REQUEST_WORD(prio), const float>())[(size_t)t * n + tid];
          if (idx) up_i = as_global(idx)[(size_t)t * n + tid];
        }
      }
      if (const uint32_t n = r.inserts()) {
        const float* prio = r.pointer<kRoundInsert + PER_REQUEST_WORD(prio), const float>();
        const uint32_t j = inserted_by(n);
        if (prio && j < n) in_v = as_global(prio)[(size_t)t * n + j];
      }
    };
    // and its row work: the first item of the insertion (the others come when it is their turn); its deferred rows, those
    // aimed at a protected slot (`at`: the insertion's ring slot; see k_insert_small)
    auto fetch_rows = [&](const Round& r, uint32_t parity, uint32_t at) {
      const uint32_t n = r.inserts();
      if (n == 0) return;
      if (const uint32_t* protect = r.pointer<kRoundInsert + PER_REQUEST_WORD(protect), const uint32_t>()) {
        const uint32_t np = r.word<kRoundInsert + PER_REQUEST_WORD(n_protect)>();
        protect += (size_t)t * np;
        for (uint32_t k = rl; k < np; k += rn) {
          const uint32_t i = as_global(protect)[k];
          if (i < N) {
            const uint32_t p = i >= at ? i - at : i + (N - at);   // position in the ring window
            if (p < n) atomicOr(&s_skip[parity][p >> 5], 1u << (p & 31u));
          }
        }
      }
      const uint32_t list = list_of(n, r.asked<kRoundInsert>());
      if (list != insert_list) {
        insert_list = list;
        insert_items = wave_value(s_ins[parity].items);
        payload = wave_pointer(s_ins[parity].base);
        ip.w = 0;
        ip.row = 0xFFFFFFFFu;
        if (rw < insert_items) ip = find_item(s_ins[parity], rw);
      }
      if (ip.w) {
        const uint8_t* from = r.array<kRoundInsert>(ip.f) + reinterpret_cast<uintptr_t>(ip.io);
        if (ip.row != 0xFFFFFFFFu) iv = load_piece(from + ip.out, ip.w);
      }
    };
    if constexpr (TREE) fetch_inputs(cur);
    if constexpr (ROWS) fetch_rows(cur, 0, cursor);
    u_i = u_next;
    lds_barrier();   // (deferred rows of round 0)

    uint32_t slot = 0;
    for (uint32_t i = 0;; ++i) {
      const uint32_t par = i & 1u, slot_next = slot == 2u ? 0u : slot + 1u;
      const bool more = cur.more();
      const uint32_t n_upd = cur.updates(), n_ins = cur.inserts(), n_smp = cur.samples();
      next.read(s_round[slot_next]);
      // ---- rows and weights of the round before
      const uint32_t w0 = apart ? 1024u - (n_before + 63u) / 64u * 64u : 0u;
      const bool weigher = ROWS && n_before && tid >= w0 && tid - w0 < n_before;
      float w_out = 0.0f, v_out = 0.0f;
      uint32_t n_out = 0;
      if (ROWS && n_before) {
        const uint32_t rest = share.x + items.count;
        if (__builtin_expect(rest < share.y, TREE))
          gather_spans<4>(s_rows[par ^ 1u], rest, share.y, nodes, N, a.fields.row_stride, 0, flags,
                          [&](uint32_t f, uint8_t* io) { return before.array<kRoundSample>(f) + reinterpret_cast<uintptr_t>(io); });
        if constexpr (!TREE) items.load(nodes, N, a.fields.row_stride);
        const bool weigh = before.pointer<kRoundSample + PER_REQUEST_WORD(out_weight), float>() != nullptr;
        uint32_t least = 0;
        if (weigh && tid >= w0) {   // (whole waves)
          if (a.buffer_norm) least = s_bmin[par ^ 1u];
          else if (TREE) least = s_vmin[par ^ 1u];
          else least = smallest_value(values, n_before);
        }
        if (weigher) {
          n_out = nodes[tid - w0];
          v_out = TREE ? val : values[tid - w0];
          if (weigh) w_out = n_out == 0xFFFFFFFFu ? 0.0f : importance_weight(v_out, __uint_as_float(least), __uint_as_float(before.word<kRoundSample + PER_REQUEST_WORD(beta)>()));
        }
      }
      auto store_results = [&] {   // of the round before
        if (!ROWS || !n_before) return;
        if constexpr (!TREE) items.store(N, flags, [&](int k) { return before.array<kRoundSample>(items.field[k]); });
        if (!weigher) return;
        const size_t o = (size_t)t * n_before + (tid - w0);
        float* out_prio = before.pointer<kRoundSample + PER_REQUEST_WORD(out_prio), float>();
        float* out_w = before.pointer<kRoundSample + PER_REQUEST_WORD(out_weight), float>();
        as_global(before.pointer<kRoundSample + PER_REQUEST_WORD(idx), uint32_t>())[o] = n_out;
        if (out_prio) as_global(out_prio)[o] = v_out;
        if (out_w) as_global(out_w)[o] = w_out;
      };
      constexpr bool stores_first = WAVE;
      if (stores_first) store_results();
      // ---- the round behind the next one is laid out; the fields of the next round's insertion and of this round's sample
      if constexpr (ROWS) {
        if (decodes) decode();
        if (lists) {
          const uint32_t ins = list_of(next.inserts(), next.asked<kRoundInsert>()), smp = list_of(n_smp, cur.asked<kRoundSample>());
          if (ins && in_lds_insert != ins) {
            fill_fields(s_round[slot_next] + kRoundInsert, &s_ins[par ^ 1u], nullptr);
            in_lds_insert = ins;
          }
          if (smp && in_lds_sample != smp) {   // (the round before's is the other one)
            fill_fields(s_round[slot] + kRoundSample, &s_rows[par], s_share[par]);
            in_lds_sample = smp;
          }
          const uint32_t other_sample = in_lds_sample_other, other_insert = in_lds_insert_other;
          in_lds_sample_other = in_lds_sample;
          in_lds_insert_other = in_lds_insert;
          in_lds_sample = other_sample;
          in_lds_insert = other_insert;
          if (lane < 32u) s_skip[par ^ 1u][lane] = 0;
        }
      }
      // ---- the tree: update, insertion
      const uint32_t first = cursor;
      uint8_t* place = nullptr;
      if (ROWS && n_ins) {
        if (ip.w && ip.row != 0xFFFFFFFFu && !((s_skip[par][ip.row >> 5] >> (ip.row & 31u)) & 1u))
          place = payload + (uint64_t)ring_slot(first, ip.row, N) * a.fields.row_stride + ip.at;
      }
      if constexpr (TREE) {
        UpdateWork up{};
        up.on = n_upd != 0;
        up.n = n_upd;
        up.mine = tid < n_upd;
        up.sorted = cur.pointer<kRoundUpdate + PER_REQUEST_WORD(idx), uint32_t>() == nullptr;
        up.counted = !single;
        up.i = up.sorted ? node : up_i;
        up.size = size;
        up.v = up_v;
        up.prio = cur.pointer<kRoundUpdate + PER_REQUEST_WORD(prio), const float>() + (size_t)t * n_upd;
        up.batch = sampled;
        InsertWork in{};
        in.on = n_ins != 0;
        if (n_ins) {
          const uint32_t j = inserted_by(n_ins);
          const bool guarded = cur.pointer<kRoundInsert + PER_REQUEST_WORD(protect), const uint32_t>() != nullptr;
          in.n = n_ins;
          in.mine = j < n_ins && !(guarded && ((s_skip[par][(j & 1023u) >> 5] >> (j & 31u)) & 1u));
          in.given = cur.pointer<kRoundInsert + PER_REQUEST_WORD(prio), const float>() != nullptr;
          in.whole = !in.given && !guarded;
          in.first = first;
          in.slot = in.mine ? ring_slot(first, j, N) : 0u;
          in.v = in_v;
        }
        if constexpr (WAVE) total = change_by_wave<LOGK, MEM>(tv, up, in, lane_max, flags, total);
        else change_by_team<LOGK, MEM>(tv, up, in, flags);
        if (!single && more) fetch_inputs(next);
      }
      if (n_ins) {
        cursor = ring_slot(cursor, n_ins, N);
        size = size + n_ins > N ? N : size + n_ins;
      }
      // ---- the rows of the round before have been asked for; the tree is whole (see k_run_steps)
      const bool late = WAVE && TREE && n_smp && !a.buffer_norm && !single;
      if (!late) lds_barrier();
      if constexpr (ROWS) {
        if (n_ins) {
          const bool guarded = cur.pointer<kRoundInsert + PER_REQUEST_WORD(protect), const uint32_t>() != nullptr;
          if (place) store_piece(place, ip.w, iv);
          if (rw + rws < insert_items)
            insert_rows(s_ins[par], insert_items, rw + rws, rws, first, N, a.fields.row_stride, 0, guarded ? s_skip[par] : nullptr,
                        [&](const RowItem& p) { return cur.array<kRoundInsert>(p.f) + reinterpret_cast<uintptr_t>(p.io); });
          if (uint32_t* slots = cur.pointer<kRoundInsert + PER_REQUEST_WORD(idx), uint32_t>()) {
            slots += (size_t)t * n_ins;
            for (uint32_t j = rl; j < n_ins; j += rn)
              as_global(slots)[j] = (s_skip[par][j >> 5] >> (j & 31u)) & 1u ? 0xFFFFFFFFu : ring_slot(first, j, N);
          }
        }
        if (!stores_first) store_results();
      }
      if (!more) break;
      if (single) {   // (what this round has stored is there before the next one's inputs are read)
        wait_memory();
        lds_barrier();
        if constexpr (TREE) fetch_inputs(next);
      }
      if constexpr (ROWS) {
        fetch_rows(next, par ^ 1u, cursor);
        // (read by the weights of the round before, in front of the barrier)
        if ((TREE || a.buffer_norm) && rl == 0) s_vmin[par ^ 1u] = s_bmin[par ^ 1u] = kNoMin;
        if (n_smp) {
          const uint32_t list = list_of(n_smp, cur.asked<kRoundSample>());
          if (list != sample_list) {
            sample_list = list;
            share.x = wave_value(s_share[par][rw].x);
            share.y = wave_value(s_share[par][rw].y);
            if constexpr (!TREE) {
              // (this tree's place in the caller's arrays goes into the offsets of the pieces; where it is too far for those
              // the items are taken like those beyond the first few)
              bool far = false;
              // (a wave's evenly shared items: the first few are kept all the same, but for a team of one wave, whose build
              // has no registers for that)
              const bool none = WAVE && wave_value(s_rows[par].runs) == 0;
              items.template prepare<!WAVE>(s_rows[par], share.x, none ? share.x : share.y, [&](int k, const RowItem& p) {
                far = far || reinterpret_cast<uintptr_t>(p.io) > 0x7FFFFFFFull;
                items.out[k] += (uint32_t)reinterpret_cast<uintptr_t>(p.io);
              });
              if (far) items.count = 0;
            }
          }
          // ---- weights relative to the whole tree: its smallest positive leaf
          if (a.buffer_norm && cur.pointer<kRoundSample + PER_REQUEST_WORD(out_weight), float>()) {
            uint32_t m = kNoMin;
            for (uint32_t e = rl; e < N; e += rn) m = min_u32(m, positive_bits(tv.leaf(e)));
            m = wave_min_u32(m);
            if (lane == 0 && m != kNoMin) atomicMin(&s_bmin[par], m);
          }
        }
      }
      // ---- sampling
      if (n_smp) ++sampled;
      if constexpr (TREE) {
        if (n_smp && (WAVE || (tid & ~63u) < n_smp)) {
          if constexpr (!WAVE) {
            note_wild(u_i, sampled, &s_wild);
            total = tree[tv.off(V)];
          }
          walk_tree<LOGK, MEM, false>(tv, tid, n_smp, u_i, total, mass_per_sample(total, n_smp), node, val, [&] {
            if (late) lds_barrier();
          });
          if (node == 0xFFFFFFFFu && tid == 0) flags |= 4u;
          if (ROWS && cur.pointer<kRoundSample + PER_REQUEST_WORD(out_weight), float>()) {
            const uint32_t m = wave_min_u32(tid < n_smp ? __float_as_uint(val) : kNoMin);
            if (lane == 0) atomicMin(&s_vmin[par], m);
          }
          if (tid < n_smp) {
            nodes[tid] = node;
            if (!ROWS) values[tid] = val;
          }
        }
        u_i = u_next;
        if (!WAVE && !single) {
          if (const uint32_t n = next.updates()) {
            const bool own = next.pointer<kRoundUpdate + PER_REQUEST_WORD(idx), uint32_t>() == nullptr;
            note_update(tid < n, own ? node : up_i, size, up_v, &s_max);
          }
        }
      }
      before = cur;
      n_before = n_smp;
      cur = next;
      slot = slot_next;
      lds_barrier();
    }
  };
  if constexpr (!apart) work(std::true_type{}, std::true_type{});
  else if (in_team) work(std::true_type{}, std::false_type{});
  else work(std::false_type{}, std::true_type{});
  if (WAVE && in_team) {
    const uint32_t m = wave_max_u32(__float_as_uint(lane_max));
    if (tid == 0) s_max = m;
  }
  report_flags(g, t, flags);
  __syncthreads();
  lds_tree_store<LOGK>(g, t, tab, lt);
}

// A list or a queue can work on a tree where its heights (every one padded to whole child groups), or those above the leaves, fit
// beside the step kernel's other LDS data.
constexpr uint32_t kStreamLdsBytes = 156 * 1024, kStreamBatchWords = 1024;   // (the sampled indices and values of a step)
static bool stream_tree_fits(const Geom& g) {
  for (uint32_t skip = 0; skip < 2; ++skip) {
    uint64_t floats = kStreamBatchWords;
    for (uint32_t h = skip; h <= g.H && floats * 4 <= kStreamLdsBytes; ++h)
      floats += h < g.H ? ((uint64_t)g.n[h] + g.K - 1) / g.K * g.K : 4;   // (the root padded to 16 bytes)
    if (floats * 4 <= kStreamLdsBytes && !(skip && g.H < 2)) return true;
  }
  return false;
}
// Levels of the copy (see Wide): the whole tree if that fits, else the levels above the leaves, or above the next one.  Narrow trees take
// less room as levels than as heights, and the groups of zeros behind the levels (512 bytes at most, K = 64) go beyond
// kStreamLdsBytes, so one of the first two fits where stream_tree_fits() says so.
constexpr uint32_t kStreamLdsMost = kStreamLdsBytes + 512;
template <int LOGK>
static StreamPlan plan_stream_levels(const Geom& g, uint32_t most_in_memory) {
  constexpr uint32_t LH = Wide<LOGK>::LH, R = Wide<LOGK>::R;
  StreamPlan p{};
  const uint32_t V = (g.H + LH - 1) / LH;
  if (V > kStreamLevels) return p;
  for (uint32_t skip = 0; skip <= most_in_memory && skip < V; ++skip) {
    uint64_t floats = 0;
    for (uint32_t v = 0; v <= V; ++v) {
      p.off[v] = (uint32_t)floats;
      if (v < skip) continue;
      floats += v < V ? ((uint64_t)g.n[v * LH] + R - 1) / R * R + (v + 1 < V ? R : 0) : 4;
      if (floats * 4 > kStreamLdsMost) break;
    }
    if ((floats + kStreamBatchWords) * 4 > kStreamLdsMost) continue;
    p.off[V + 1] = (uint32_t)floats;
    for (uint32_t v = 0; v <= V; ++v) p.nodes[v] = g.n[v * LH < g.H ? v * LH : g.H];
    p.levels = V;
    p.levels_in_memory = skip;
    p.floats = (uint32_t)floats + kStreamBatchWords;
    return p;
  }
  return p;
}
static StreamPlan plan_stream(const Geom& g, uint32_t most_in_memory) {
  switch (g.logK) {
    case 1: return plan_stream_levels<1>(g, most_in_memory);
    case 2: return plan_stream_levels<2>(g, most_in_memory);
    case 3: return plan_stream_levels<3>(g, most_in_memory);
    case 4: return plan_stream_levels<4>(g, most_in_memory);
    case 5: return plan_stream_levels<5>(g, most_in_memory);
    case 6: return plan_stream_levels<6>(g, most_in_memory);
    default: return StreamPlan{};
  }
}
StreamPlan stream_list_plan(const Geom& g) { return stream_tree_fits(g) ? plan_stream(g, 1) : StreamPlan{}; }
// A step by itself can also leave the level above the leaves in memory: it reads and changes few groups of it, each a trip more.
// (Its tree is on the chip for one step: what counts there is the copy of the tree, not the trips of every step.)
StreamPlan stream_step_plan(const Geom& g) { return plan_stream(g, 2); }

// Waves of the team (where it is not all of them).
static uint32_t team_waves(uint32_t samples, uint32_t inserted) { return ((samples > inserted ? samples : inserted) + 63u) / 64u; }
// Items that n rows are moved in (see fill_piece_fields).
static RowItems row_items(const FieldTable& ft, uint32_t n) {
  RowItems it{};
  for (uint32_t f = 0; f < ft.n_fields; ++f) {
    if (!ft.io[f]) continue;
    const uint32_t w = moves_wide(ft.bytes[f], ft.vec[f]) ? 16u : ft.vec[f];
    const uint64_t items = ((uint64_t)n * row_elements(ft.bytes[f], ft.vec[f]) + 63u) / 64u;
    it.of_width[4 - __builtin_ctz(w)] += items;
    it.all += items;
  }
  return it;
}
// Length of the runs in which a gather of n rows can be shared out among rws row waves (0: it cannot): every wave has at most
// that many items, of one access width, and not more than it can have under way at once.
static uint32_t gather_run(const RowItems& it, uint32_t n, uint32_t rws) {
  for (uint32_t len = 1; len <= kInFlight; ++len) {
    uint64_t needed = 0;
    for (const uint64_t of_this : it.of_width) needed += (of_this + len - 1) / len;
    if (needed <= run_waves(n, rws)) return len;
  }
  return 0;
}
void plan_stream_rows(StreamCall* a) {
  a->gathered = row_items(a->rows, a->B);
  a->placed = row_items(a->ins, a->n_insert);
  const uint32_t team = team_waves(a->B, a->n_insert);
  a->run = team < 16u ? gather_run(a->gathered, a->B, 16u - team) : 0u;
}
// The list of n rows' pieces for the kernel (the items ordered by access width, and those of one width by field).
static void plan_pieces(const FieldTable& ft, const RowItems& it, uint32_t n, uint32_t trees, PieceList* pl) {
  pl->items = (uint32_t)it.all;
  pl->n = n;
  pl->step_rows = (uint64_t)trees * n;
  pl->base = ft.n_fields ? ft.col[0] : nullptr;
  pl->base_stride = ft.n_fields ? ft.col_stride[0] : 0;
  uint32_t at = 0;
  for (uint32_t f = 0; f < (uint32_t)kMaxFields; ++f) pl->bytes[f] = pl->width[f] = 1;
  for (uint32_t w = 16; w; w /= 2) {
    for (uint32_t f = 0; f < ft.n_fields; ++f) {
      const uint32_t E = ft.bytes[f], epr = row_elements(E, ft.vec[f]);
      if (!n || !ft.io[f] || (moves_wide(E, ft.vec[f]) ? 16u : ft.vec[f]) != w) continue;
      pl->io[f] = ft.io[f];
      pl->off[f] = (uint32_t)(ft.col[f] - ft.col[0]);   // (the fields of a row lie in the order of their numbers)
      pl->bytes[f] = E;
      pl->width[f] = w;
      pl->recip[f] = epr > 1 ? 0xFFFFFFFFu / epr + 1u : 0u;
      pl->first[f] = at;
      at += (uint32_t)(((uint64_t)n * epr + 63u) / 64u);
      pl->end[f] = at;
    }
  }
}
// Which of a gather's items every one of the rws row waves has: runs of that length, or (run 0) equally many.
static void plan_shares(const RowItems& it, uint32_t run, uint32_t rws, uint2 (&share)[16]) {
  uint32_t wave = 0;
  if (run) {
    uint32_t start = 0;
    for (const uint64_t of_this : it.of_width) {
      const uint32_t end = start + (uint32_t)of_this;
      for (; start < end; start += run) share[wave++] = make_uint2(start, start + run < end ? start + run : end);
      start = end;
    }
  } else {
    const uint64_t each = (it.all + rws - 1) / rws;
    for (uint64_t first = 0; first < it.all; first += each)
      share[wave++] = make_uint2((uint32_t)first, (uint32_t)(first + each < it.all ? first + each : it.all));
  }
}

// Whether one step (with n_insert new rows, or none) is faster as one launch of the kernel above than as the two or three
// kernels it otherwise takes.  Both sides in hundredths of a microsecond, fitted to measured shapes (every fanout, 300 to 4
// million leaves, 1 to 64 trees, 16 to 512 samples, 0 to 512 new rows of 0 to 1033 bytes in fields of every access width).  On the
// chip: the launch and one step's chain, more with several waves at the tree; the rows, which one compute unit moves, by the
// pieces that every row wave has (in runs each piece is the rest of a trip to memory, evenly shared ones go eight to a trip; a
// new row's pieces one to a trip); the copy of the tree and the trips to levels in memory.  As kernels: two launches, with the
// insertion in the sampling kernel where that can carry it, else three; K = 2 trees are chains of many heights, and so are large
// ones.  (32 samples on 2^20 leaves at K = 16: 12.4 us as kernels, 7.5 on the chip; 64 on each of 64 trees of 2^18: 16.9 and 8.9;
// where it stays away: 256 samples with rows of 165 bytes on 4096 leaves at K = 2, 22 and 71.)
// Where rows are shared evenly, pieces of one byte among them, the two fits are off by up to 15 %, and the chip has to be ahead
// by a tenth, not by 3 % (35 samples with rows of 1033 bytes on each of 64 trees of 1074 leaves at K = 4: 13.2 us as kernels, 15.6 on the
// chip; 63 of 165 bytes on 2416 leaves at K = 64: 9.2 and 10.0).
// Of 580 shapes that the constants were not fitted to (profiles/step_ways.txt) 501 go on the chip, two of them 2.3 and 5.7 % slower
// for it; the way taken is 0.9 % behind the better one on average.  (The kernels are up to 8 us faster at K = 2 and 4 than when the
// constants were fitted, and 5 at K = 32 on few leaves, and still the slower way nearly wherever the fits say so.)
// Batches beyond 256 at K > 2 are left out, though several trees of a few thousand leaves would gain (410 samples on each of 4 trees
// of 27 915 leaves at K = 32: 16.8 and 13.1): of 71 such shapes that the fits would take, three lose 6 to 13 %.
bool step_on_chip_pays(const Geom& g, const Tuning& tn, const StreamCall& a) {
  const uint32_t B = a.B, n_insert = a.n_insert, floats = a.plan.floats, in_memory = a.plan.levels_in_memory;
  if (g.T > 64 || (B > 256 && g.K > 2)) return false;
  uint64_t row = 0;
  for (uint32_t f = 0; f < a.rows.n_fields; ++f) row += a.rows.io[f] ? a.rows.bytes[f] : 0u;
  const uint32_t rws = 16u - team_waves(B, n_insert);
  const uint64_t gathered = a.gathered.all, placed = a.placed.all;
  int64_t here = 520 + (team_form(B, n_insert) == TEAM_ONE_WAVE ? 0 : 138) + (n_insert ? 55 : 0) + (g.T >= 16 ? 71 : 0) + (g.K == 64 ? 37 * B / 64 : 0);
  here += a.run ? 80 * gathered / rws : 136 + 19 * gathered / rws;
  here += (placed > rws ? 81 * (placed - rws) / rws : 0) + floats * 4 / 1024 + (g.K == 2 ? 40 : g.K == 4 ? 20 : 0);
  if (in_memory) {
    here += in_memory == 1 ? 40 + 40 * B / 64 : 100 + 55 * B / 64 + (n_insert ? 25 : 0);
    here += g.K == 2 ? 40 + (in_memory == 1 ? 25 : 60) * B / 64 : g.K == 64 ? 70 + 60 * B / 64 : 0;
  }
  bool has_rows = false;
  for (uint32_t f = 0; f < a.ins.n_fields; ++f) has_rows = has_rows || a.ins.io[f];
  // (asked as for a ring at its start: the way does not change in the one step whose rows go round its end)
  const bool carried = n_insert && sample_can_carry_insert(g, tn, B, has_rows ? &a.ins : nullptr, n_insert, 0);
  int64_t apart = 938 + (!n_insert ? 0 : carried ? 273 : 374 + (g.K <= 4 ? 141 : 0)) + (g.K == 2 ? 106 * (int64_t)g.H - 815 : 0);
  apart += (g.N > 1u << 20 ? 170 : 0) + (g.K == 64 && g.H >= 3 ? 90 : 0) + (g.K == 4 && g.H >= 9 ? 600 : 0);
  apart += (g.K == 4 ? 87 : 0) + (g.K >= 32 ? 55 : 0) + (g.T >= 16 ? 105 : 0) + (int64_t)(176 * g.T * B * row >> 20);
  return here * (a.run ? 103 : 110) < apart * 100;
}

template <int LOGK>
static hipError_t launch_run_steps_k(const Geom& g, const Tuning& tn, const StreamCall& a, hipStream_t s) {
  StreamKernelArgs ka{};
  ka.g = g;
  ka.a = a;
  if (!a.plan.floats) return hipErrorInvalidValue;
  const size_t bytes = (size_t)a.plan.floats * 4;
  // always the largest workgroup, also for small batches: measured faster than a workgroup of the batch's
  // size (the tree copy and the row movers use all lanes)
  TeamForm form = team_form(a.B, a.n_insert);
  if (form != TEAM_ALL && !a.run) form = a.ahead ? TEAM_WAVES_SPANS : TEAM_ALL;
  plan_pieces(a.rows, a.gathered, a.B, g.T, &ka.rows);
  plan_pieces(a.ins, a.placed, a.n_insert, g.T, &ka.ins);
  plan_shares(a.gathered, form == TEAM_ONE_WAVE || form == TEAM_WAVES ? a.run : 0u, form == TEAM_ALL ? 16u : 16u - team_waves(a.B, a.n_insert), ka.share);
  ka.a.rows_stride = a.rows.row_stride;
  ka.a.ins_stride = a.ins.row_stride;
  const uint32_t mem = a.plan.levels_in_memory;
#define PER_RUN(...)                                                                                    \
  do {                                                                                                  \
    hipError_t e = grant_lds<&k_run_steps<LOGK, __VA_ARGS__>>(tn, bytes);                               \
    if (e != hipSuccess) return e;                                                                      \
    PER_LAUNCH(KID_RUN_STEPS, (k_run_steps<LOGK, __VA_ARGS__>), dim3(g.T), dim3(1024), bytes, s, ka);   \
  } while (0)
#define PER_RUN_WHERE(F, A)                                                                             \
  do {                                                                                                  \
    if (mem) PER_RUN(F, 1, A); else PER_RUN(F, 0, A);                                                   \
  } while (0)
#define PER_RUN_WHEN(F)                                                                                 \
  do {                                                                                                  \
    if (a.ahead) PER_RUN_WHERE(F, true); else PER_RUN_WHERE(F, false);                                  \
  } while (0)
  if (a.sum_root) {   // (built for what ensure_sums asks for)
    if (mem || !a.ahead) return hipErrorInvalidValue;
    if constexpr (LOGK == 4 || LOGK == 5) {
      if (form == TEAM_ONE_WAVE) PER_RUN(TEAM_ONE_WAVE, 0, true, true);
      else if (form == TEAM_WAVES) PER_RUN(TEAM_WAVES, 0, true, true);
      else if (form == TEAM_WAVES_SPANS) PER_RUN(TEAM_WAVES_SPANS, 0, true, true);
      else PER_RUN(TEAM_ALL, 0, true, true);
    } else {
      return hipErrorInvalidValue;
    }
  } else if (mem > 1) {   // (built for single steps whose gathers go in runs only)
    if (a.n_steps != 1 || !a.ahead || !a.upd_is_sampled || form > TEAM_WAVES) return hipErrorInvalidValue;
    if (form == TEAM_ONE_WAVE) PER_RUN(TEAM_ONE_WAVE, 2, true); else PER_RUN(TEAM_WAVES, 2, true);
  } else if (form == TEAM_ONE_WAVE) PER_RUN_WHEN(TEAM_ONE_WAVE);
  else if (form == TEAM_WAVES) PER_RUN_WHEN(TEAM_WAVES);
  else if (form == TEAM_WAVES_SPANS) PER_RUN_WHERE(TEAM_WAVES_SPANS, true);
  else PER_RUN_WHEN(TEAM_ALL);
#undef PER_RUN_WHEN
#undef PER_RUN_WHERE
#undef PER_RUN
  return hipGetLastError();
}

hipError_t launch_run_steps(const Geom& g, const Tuning& tn, const StreamCall& a, hipStream_t s) {
#define CALL(L) launch_run_steps_k<L>(g, tn, a, s)
  PER_DISPATCH_LOGK(g.logK, CALL)
#undef CALL
}

template <int LOGK>
static hipError_t launch_run_requests_k(const Geom& g, const Tuning& tn, const QueueArgs& a, bool sum_root, hipStream_t s) {
  QueueKernelArgs ka{};
  ka.g = g;
  ka.a = a;
  if (!a.plan.floats) return hipErrorInvalidValue;
  const size_t bytes = (size_t)a.plan.floats * 4;
  const TeamForm form = team_form(a.most, 0);
  const bool mem = a.plan.levels_in_memory != 0;
#define PER_RUN(...)                                                                                        \
  do {                                                                                                      \
    hipError_t e = grant_lds<&k_run_requests<LOGK, __VA_ARGS__>>(tn, bytes);                                \
    if (e != hipSuccess) return e;                                                                          \
    PER_LAUNCH(KID_RUN_REQUESTS, (k_run_requests<LOGK, __VA_ARGS__>), dim3(g.T), dim3(1024), bytes, s, ka); \
  } while (0)
#define PER_RUN_WHERE(F)                                                                                \
  do {                                                                                                  \
    if (mem) PER_RUN(F, 1); else PER_RUN(F, 0);                                                         \
  } while (0)
  if (sum_root) {
    if (mem) return hipErrorInvalidValue;
    if constexpr (LOGK == 4 || LOGK == 5) {
      if (form == TEAM_ONE_WAVE) PER_RUN(TEAM_ONE_WAVE, 0, true);
      else if (form == TEAM_WAVES) PER_RUN(TEAM_WAVES, 0, true);
      else PER_RUN(TEAM_ALL, 0, true);
    } else {
      return hipErrorInvalidValue;
    }
  } else if (form == TEAM_ONE_WAVE) PER_RUN_WHERE(TEAM_ONE_WAVE);
  else if (form == TEAM_WAVES) PER_RUN_WHERE(TEAM_WAVES);
  else PER_RUN_WHERE(TEAM_ALL);
#undef PER_RUN_WHERE
#undef PER_RUN
  return hipGetLastError();
}

hipError_t launch_run_requests(const Geom& g, const Tuning& tn, const QueueArgs& a, bool sum_root, hipStream_t s) {
#define CALL(L) launch_run_requests_k<L>(g, tn, a, sum_root, s)
  PER_DISPATCH_LOGK(g.logK, CALL)
#undef CALL
}

// A list of steps in one launch on an LDS-resident tree.
// Part of per_kernels.hip (included inside namespace per, in the order given there); not a stand-alone header.

// ---------------------------------------------------------------------------------
// a stream of steps on an LDS-resident tree (small buffers)
// ---------------------------------------------------------------------------------
// The paper keeps the sum tree of its Replay Manager in on-chip memory and lets one kernel, started
// once, work through a stream of requests (Section V-A, "RM on FPGA": buffers of 10K to 100K entries,
// autorun kernels that need no launch per request).  The counterpart here: when all heights of a
// tree fit the LDS of one compute unit, one workgroup per tree loads the tree once, runs a whole
// list of steps (insert -> sample -> gather -> update, the order of the separate calls) against
// the LDS copy, and stores the tree back at the end.  Every tree access of a step is then an LDS
// access; only rows, inputs and outputs travel to memory.  Results are those of the separate calls.
//
// A tree whose leaves do not fit beside the rest (MEM) keeps heights 1 .. H in LDS and its leaves in memory: the
// paper's 100K-entry buffers at small fanouts are of that size.  The workgroup is still the only one that
// touches the tree while the kernel runs, so its own leaf stores, made visible to its other waves by a
// barrier, are all the coherence that takes; every operation then costs a trip or two to memory for the leaf
// groups it reads (sampling: the last level of the walk; insert and update: the groups whose sums change).
//
// Update inside one workgroup: a valid element raises the leaf (reinterpreted as an integer) to
// a marker above every valid priority pattern, 0x80000001 + its position, by an LDS atomic max; the
// element that finds its own marker afterwards is the last writer and stores its value; then
// every valid element recomputes its ancestors height by height (elements that share a parent
// store the same sum).
struct StreamKernelArgs {           // one kernel argument, so that both parts sit at known offsets of the segment
  Geom g;
  StreamArgs a;
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

// One tree in the LDS of its workgroup.
struct LdsTree {
  float* tree;              // levels 0 .. V back to back (level 0 left out when leaves_mem is set), each padded with zeros to
                            // whole groups and, below the root's children, with one group more: what the nodes beyond the
                            // next level's last have for children
  float* leaves_mem;        // null, or the tree's leaves in memory (zero padded to whole groups)
  const uint32_t *off, *n;  // off[v]: where level v starts (floats), off[V + 1]: all floats; n[v]: its real nodes
  uint32_t* max_bits;       // running maximum priority (fp32 bits)
  uint32_t H, V;
};

// Loads every level of tree t into LDS.  The heights are arrays of their own in memory (zero padded to 64 floats) and the
// levels lie back to back in LDS; the copy runs over the LDS floats as one range, four 16-byte pieces per lane in flight
// and all loads of a round before its first store.
template <int LOGK>
__device__ __forceinline__ void lds_tree_load(const LevelTable& tab, const LdsTree& lt) {
  constexpr int R = 4;
  const uint32_t v_first = lt.leaves_mem ? 1u : 0u;
  const uint32_t begin = lt.off[v_first], end = lt.off[lt.V + 1];
  for (uint32_t base = begin; base < end; base += 4u * R * blockDim.x) {
    Floats4 x[R];
    uint32_t v = v_first;   // (the level of this lane's piece: found anew per round, then it only grows)
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t e = base + 4u * ((uint32_t)k * blockDim.x + threadIdx.x);
      if (e < end) {
        while (v < lt.V && e >= lt.off[v + 1]) ++v;
        const uint32_t i = e - lt.off[v];
        x[k] = Floats4{0.0f, 0.0f, 0.0f, 0.0f};
        if (i < lt.n[v]) x[k] = load_floats4(as_global(static_cast<const float*>(tab.lvl[level_height<LOGK>(v, lt.H)])) + i);
      }
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t e = base + 4u * ((uint32_t)k * blockDim.x + threadIdx.x);
      if (e < end) *reinterpret_cast<Floats4*>(lt.tree + e) = x[k];
    }
  }
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
// ... and back to memory, with the running maximum and the flags the lanes have collected.
template <int LOGK>
__device__ __forceinline__ void lds_tree_store(const Geom& g, uint32_t t, const LevelTable& tab, const LdsTree& lt,
                                               uint32_t flags, uint32_t* s_flags) {
  constexpr uint32_t LH = Wide<LOGK>::LH, R = Wide<LOGK>::R;
  const uint32_t V = lt.V, H = lt.H;
  // (a root less than a whole level above its children is stored by the pass below: the level's sum of it has zeros added)
  const uint32_t end = V * LH == H ? lt.off[V + 1] : lt.off[V];
  uint32_t v = lt.leaves_mem ? 1u : 0u;
  for (uint32_t e = lt.off[v] + 4u * threadIdx.x; e < end; e += 4u * blockDim.x) {
    while (v < V && e >= lt.off[v + 1]) ++v;
    const uint32_t i = e - lt.off[v];
    if (i < lt.n[v]) *(GlobalPtr<Floats4>)(as_global(tab.lvl[level_height<LOGK>(v, H)]) + i) = load_floats4(lt.tree + e);
  }
  if constexpr (LH > 1) {
    for (uint32_t w = 0; w < V; ++w) {
      const uint32_t groups = tab.n[level_height<LOGK>(w + 1, H)];
      for (uint32_t p = threadIdx.x; p < groups; p += blockDim.x) {
        if (w == 0 && lt.leaves_mem) store_between<LOGK>(as_global(static_cast<const float*>(lt.leaves_mem)) + (size_t)p * R, p, 0, tab, H);
        else store_between<LOGK>(static_cast<const float*>(lt.tree) + lt.off[w] + (size_t)p * R, p, w * LH, tab, H);
      }
    }
  }
  if (threadIdx.x == 0) g.max_v[t] = __uint_as_float(*lt.max_bits);
  if (flags) atomicOr(s_flags, flags);
  __syncthreads();
  if (threadIdx.x == 0 && *s_flags) atomicOr(&g.status[t], *s_flags);
}

// ---- rows of the stream kernels
// The rows of a batch move in pieces (16 bytes, or the field's access width), 64 pieces of one field at a time by one
// wave: an item.  A wave then works with one access width and one field's constants (with the pieces of all fields
// shared out lane by lane, every lane paid for a chain of selects over the fields, a division, and the loads and
// stores of every width that occurs in its wave).
struct PieceFields {               // what the waves ask of one list of fields, in LDS
  uint8_t* io[kMaxFields];         // the caller's array: the rows of this tree (in step 0)
  uint8_t* col[kMaxFields];        // the field in row 0 of this tree
  uint64_t step[kMaxFields];       // bytes of the caller's array per step
  uint32_t bytes[kMaxFields], vec[kMaxFields];
  uint32_t pieces[kMaxFields];     // pieces of this field
  uint32_t recip[kMaxFields];      // floor(2^32 / pieces per row) + 1
  uint32_t end[kMaxFields];        // items of this field and all before it
  __device__ __forceinline__ uint32_t items() const { return (uint32_t)__builtin_amdgcn_readfirstlane((int)end[kMaxFields - 1]); }
};
// Called by one wave: n rows per tree; field f's array is `io` for tree 0 (null: not asked for), `step` bytes from step to step.
__device__ __forceinline__ void fill_piece_fields(const FieldTable* ft, uint8_t* io, uint32_t t, uint32_t n, uint64_t step_rows,
                                                  PieceFields* pf) {
  const uint32_t f = threadIdx.x & 63u;
  if (f < (uint32_t)kMaxFields) {
    const bool on = f < ft->n_fields && io && n;
    const uint32_t E = on ? ft->bytes[f] : 1u, v = on ? ft->vec[f] : 1u, epr = row_elements(E, v);
    pf->io[f] = on ? io + (uint64_t)t * n * E : nullptr;
    pf->col[f] = ft->col[f] + (uint64_t)t * ft->col_stride[f];
    pf->step[f] = step_rows * E;
    pf->bytes[f] = E;
    pf->vec[f] = v;
    pf->pieces[f] = on ? n * epr : 0u;
    pf->recip[f] = epr > 1 ? 0xFFFFFFFFu / epr + 1u : 0u;
    uint32_t end = on ? (n * epr + 63u) / 64u : 0u;
#pragma unroll
    for (int d = 1; d < kMaxFields; d <<= 1) {
      const uint32_t before = (uint32_t)__shfl_up((int)end, d);
      if (f >= (uint32_t)d) end += before;
    }
    pf->end[f] = end;
  }
}
struct RowItem {        // this lane's piece of an item
  bool on;
  uint32_t f, w, row;   // field and access width (the same for the wave), row of the batch
  uint8_t* stored;      // the piece in row 0 of the tree's payload
  uint8_t* dense;       // the piece in the caller's array (step 0)
};
__device__ __forceinline__ uint32_t wave_value(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }   // (the same in all lanes)
// Item i < pf.items(): fields one after the other.
__device__ __forceinline__ RowItem find_item(const PieceFields& pf, uint32_t i) {
  uint32_t f = 0;
#pragma unroll
  for (uint32_t k = 0; k + 1 < (uint32_t)kMaxFields; ++k) f += i >= pf.end[k] ? 1u : 0u;
  f = wave_value(f);
  const uint32_t E = wave_value(pf.bytes[f]), v = wave_value(pf.vec[f]);
  const uint32_t el = (i - (f ? wave_value(pf.end[f - 1]) : 0u)) * 64u + (threadIdx.x & 63u);
  const bool wide = moves_wide(E, v);
  const uint32_t epr = row_elements(E, v), w = wide ? 16u : v;
  RowItem p;
  p.on = el < pf.pieces[f];
  p.f = f;
  p.w = w;
  // (at most 1024 rows: the reciprocal is exact for less than 2048 pieces per row)
  p.row = epr == 1 ? el : epr < 2048u ? __umulhi(el, wave_value(pf.recip[f])) : el / epr;
  const uint32_t k = el - p.row * epr;
  const uint32_t at = wide && 16u * k + 16u > E ? E - 16u : k * w;
  p.stored = pf.col[f] + at;
  p.dense = pf.io[f] + (uint64_t)p.row * E + at;
  return p;
}
typedef uint32_t Words4 __attribute__((ext_vector_type(4), aligned(4)));   // (16-byte pieces of some fields lie on 4-byte boundaries)
typedef uint32_t Words2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint4 load_piece(const uint8_t* src, uint32_t w) {
  uint4 v;   // (what a narrow piece leaves of it stays undefined: setting it would make the wave wait for loads under way)
  switch (w) {
    case 16: { const Words4 x = *(GlobalPtr<const Words4>)src; v = make_uint4(x.x, x.y, x.z, x.w); } break;
    case 8: { const Words2 x = *(GlobalPtr<const Words2>)src; v.x = x.x; v.y = x.y; } break;
    case 4: v.x = *(GlobalPtr<const uint32_t>)src; break;
    case 2: v.x = *(GlobalPtr<const uint16_t>)src; break;
    default: v.x = *(GlobalPtr<const uint8_t>)src; break;
  }
  return v;
}
__device__ __forceinline__ void store_piece(uint8_t* dst, uint32_t w, const uint4& v) {
  switch (w) {
    case 16: { const Words4 x = {v.x, v.y, v.z, v.w}; *(GlobalPtr<Words4>)dst = x; } break;
    case 8: { const Words2 x = {v.x, v.y}; *(GlobalPtr<Words2>)dst = x; } break;
    case 4: *(GlobalPtr<uint32_t>)dst = v.x; break;
    case 2: *(GlobalPtr<uint16_t>)dst = (uint16_t)v.x; break;
    default: *(GlobalPtr<uint8_t>)dst = (uint8_t)v.x; break;
  }
}
__device__ __forceinline__ uint32_t ring_slot(uint32_t cursor, uint32_t j, uint32_t N) {
  const uint64_t s = (uint64_t)cursor + j;
  return (uint32_t)(s >= N ? s - N : s);
}
// Items i .. end of one field of a gather (nodes: the batch's slots; one beyond the tree gives zeros and a flag), four at a
// time: the loads of all, then the stores of all.
template <typename V>
__device__ __forceinline__ void gather_span(uint32_t i, uint32_t end, uint32_t pieces, uint32_t epr, uint32_t recip, uint32_t E,
                                            uint32_t row_stride, const uint8_t* col, uint8_t* io, const uint32_t* nodes, uint32_t N,
                                            uint32_t& flags) {
  constexpr int U = 4;
#pragma unroll 1
  for (; i < end; i += U) {
    V v[U];
    uint32_t slot[U], el[U], at[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {   // (beyond the end: the first piece again, so that no load stands in a branch)
      el[k] = (i + k) * 64u + (threadIdx.x & 63u);
      if (i + k >= end || el[k] >= pieces) el[k] = 0xFFFFFFFFu;
      const uint32_t e = el[k] == 0xFFFFFFFFu ? 0u : el[k];
      const uint32_t row = epr == 1 ? e : epr < 2048u ? __umulhi(e, recip) : e / epr, within = (e - row * epr) * (uint32_t)sizeof(V);
      at[k] = within + (uint32_t)sizeof(V) > E ? E - (uint32_t)sizeof(V) : within;   // (wide pieces: the last one ends with the field)
      slot[k] = nodes[row];
      el[k] = el[k] == 0xFFFFFFFFu ? el[k] : row;
    }
#pragma unroll
    for (int k = 0; k < U; ++k) v[k] = *(GlobalPtr<const V>)(col + (uint64_t)(slot[k] < N ? slot[k] : 0u) * row_stride + at[k]);
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (el[k] != 0xFFFFFFFFu) {
        if (!(slot[k] < N)) {
          v[k] = V{};
          flags |= 1u;
        }
        *(GlobalPtr<V>)(io + (uint64_t)el[k] * E + at[k]) = v[k];
      }
  }
}
// This wave's share (number `part` of `parts`) of a gather: a run of items, so that it has to do with few fields.  `step`:
// which step's part of the caller's arrays.  (Looped and not unrolled over the items: the code a round goes through has
// to stay within the instruction cache.)
__device__ __forceinline__ void gather_rows(const PieceFields& pf, uint32_t part, uint32_t parts, const uint32_t* nodes, uint32_t N,
                                            uint32_t row_stride, uint64_t step, uint32_t& flags) {
  const uint32_t items = pf.items(), per = (items + parts - 1) / parts;
  uint32_t i = part * per;
  const uint32_t last = i + per < items ? i + per : items;
#pragma unroll 1
  while (i < last) {
    uint32_t f = 0;
#pragma unroll
    for (uint32_t k = 0; k + 1 < (uint32_t)kMaxFields; ++k) f += i >= pf.end[k] ? 1u : 0u;
    f = wave_value(f);
    const uint32_t E = wave_value(pf.bytes[f]), v = wave_value(pf.vec[f]), first = f ? wave_value(pf.end[f - 1]) : 0u;
    const uint32_t fend = wave_value(pf.end[f]), pieces = wave_value(pf.pieces[f]), recip = wave_value(pf.recip[f]);
    const uint32_t end = fend < last ? fend : last, epr = row_elements(E, v);
    const uint8_t* col = pf.col[f];
    uint8_t* io = pf.io[f] + step * pf.step[f];
    switch (moves_wide(E, v) ? 16u : v) {
      case 16: gather_span<Words4>(i - first, end - first, pieces, epr, recip, E, row_stride, col, io, nodes, N, flags); break;
      case 8: gather_span<Words2>(i - first, end - first, pieces, epr, recip, E, row_stride, col, io, nodes, N, flags); break;
      case 4: gather_span<uint32_t>(i - first, end - first, pieces, epr, recip, E, row_stride, col, io, nodes, N, flags); break;
      case 2: gather_span<uint16_t>(i - first, end - first, pieces, epr, recip, E, row_stride, col, io, nodes, N, flags); break;
      default: gather_span<uint8_t>(i - first, end - first, pieces, epr, recip, E, row_stride, col, io, nodes, N, flags); break;
    }
    i = end;
  }
}
// The rows of an insertion at ring slot `cursor`, items first, first + every, ..; row j is left out where bit j of skip is set.
__device__ __forceinline__ void place_row_piece(const RowItem& p, uint32_t cursor, uint32_t N, uint32_t row_stride, const uint32_t* skip,
                                                const uint4& v) {
  if (skip && ((skip[p.row >> 5] >> (p.row & 31u)) & 1u)) return;
  store_piece(p.stored + (uint64_t)ring_slot(cursor, p.row, N) * row_stride, p.w, v);
}
__device__ __forceinline__ void insert_rows(const PieceFields& pf, uint32_t first, uint32_t every, uint32_t cursor, uint32_t N,
                                            uint32_t row_stride, uint64_t step, const uint32_t* skip) {
  const uint32_t items = pf.items();
#pragma unroll 1
  for (uint32_t e = first; e < items; e += every) {
    const RowItem p = find_item(pf, e);
    if (p.on) place_row_piece(p, cursor, N, row_stride, skip, load_piece(p.dense + step * pf.step[p.f], p.w));
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
template <bool MEM>
struct TreeView {
  float* tree;               // the LDS copy
  float* leaves;             // MEM: the leaves (else they are in the copy, level 0 at offset 0)
  uint32_t off_reg, n_reg;   // lane v of every wave: off[v], real nodes of level v (read from there: an LDS trip less per level)
  uint32_t V, N;
  uint32_t vt;               // the lowest level above the leaves of at most kTopNodes nodes
  uint32_t* s_max;           // running maximum (WAVE: the team keeps its own copy)
  uint32_t* s_arrived;       // team waves that have come to one of its barriers, over all barriers (LDS)
  bool apart;                // there are waves outside the team
  uint32_t team;             // lanes of the team
  uint32_t* s_wild;          // the latest sampling with a uniform outside [0, 1) (0: none)
  uint2* s_runs;             // [16] of every team wave: the leaf its elements begin with, what is known of them (see change_tree)
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
  __device__ __forceinline__ uint32_t n(uint32_t v) const { return (uint32_t)__builtin_amdgcn_readlane((int)n_reg, (int)v); }
  // Barrier of the team between phases that hand leaves or sums to other waves of it.  The hardware's barrier would hold
  // the team until the row waves come by; the team's waves count themselves in LDS instead (all of them are resident, and
  // each comes to every barrier, so the wait ends).
  __device__ __forceinline__ void sync() {
    if constexpr (MEM) wait_memory();
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
template <int LOGK, bool MEM>
__device__ __forceinline__ float child_group_sum(const TreeView<MEM>& tv, uint32_t v, uint32_t parent) {
  constexpr int R = Wide<LOGK>::R;
  if constexpr (MEM) {
    if (v == 1) return sum_chunks<R / 4>(as_global(static_cast<const float*>(tv.leaves)) + (size_t)parent * R);
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
template <int LOGR, int STEP, bool MEM>
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
template <int LOGK, bool MEM>
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

// An update of n elements (lane tid < n of the team: leaf ui gets uv) and then an insertion (lanes with `inserts`: row at
// ring slot `slot`, value in_v or the running maximum), and the ancestors of both in one pass.  Called by the team.
struct UpdateWork {
  bool on, mine, sorted;     // sorted: the indices are those of a sampled batch
  uint32_t n, i, size;
  float v;
  uint32_t batch;            // sorted, !WAVE: the number of that sampling (from 1 on)
};
struct InsertWork {
  bool on, mine, given;      // given: the value is `v`, else the running maximum
  uint32_t n, slot;
  float v;
};
// (WAVE: total is the root; else it is read from the copy)
template <int LOGK, bool WAVE, bool MEM>
__device__ __forceinline__ void change_tree(TreeView<MEM>& tv, const UpdateWork& u, const InsertWork& ins, uint32_t& max_bits,
                                            uint32_t& flags, float& total) {
  constexpr int LOGR = Wide<LOGK>::LOGR;
  const uint32_t tid = threadIdx.x;
  bool valid = false, placed = false;
  if (u.on) {
    if (u.mine) {
      if (!(u.i < u.size)) flags |= 1u;
      else if (!valid_priority(u.v)) flags |= 2u;
      else valid = true;
    }
    const uint32_t mx = valid && u.v > 0.0f ? __float_as_uint(u.v) : 0u;
    bool won = valid;
    const uint32_t mark = 0x80000001u + tid;
    // Sampled leaves come in order from uniforms in [0, 1): the targets do not decrease then, and the walk keeps their order.
    // Uniforms outside may return leaves in any order; the markers decide there.  (One wave looks at its leaves; several
    // go by whether a uniform was out of range, in which case the sampling has left its number in *tv.s_wild.)
    bool in_order = u.sorted;
    if (WAVE && in_order) {
      // (elements of one leaf are neighbours, and the last of them wins)
      const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u.i, 0x130 /* wave_shl:1: from the lane above */, 0xF, 0xF, true);
      const bool last = not_before_here(tid) + 1u >= u.n;   // (worked out here each time: as a mask kept over the steps it costs more, scalar registers are short)
      in_order = __all(!u.mine || (valid && (last || next >= u.i)));
      if (in_order) won = valid && (last || next != u.i);
    } else if (!WAVE && in_order) {
      // The last valid element of every run of equal leaves wins.  Within a wave that is read off two masks: where runs
      // begin, and which elements are valid.  A run that reaches the end of its wave may go on in the next ones: each
      // wave leaves the leaf it begins with and whether that first run has a valid element (1) and is all there is (2).
      const unsigned lane = tid & 63u;
      const uint32_t wild = *tv.s_wild;   // (read here, looked at behind the barrier, which hides the trip)
      const uint32_t below = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u.i, 0x138 /* wave_shr:1: from the lane below */, 0xF, 0xF, true);
      const unsigned long long begins = __ballot(u.mine && (lane == 0 || below != u.i)), good = __ballot(valid);
      const unsigned long long later = lane == 63u ? 0ull : begins >> (lane + 1u);
      const unsigned run_end = later ? lane + 1u + (unsigned)__builtin_ctzll(later) : 64u;   // first lane behind this lane's run
      const unsigned long long behind = lane == 63u ? 0ull : (good >> (lane + 1u)) & (run_end == 64u && lane == 0 ? ~0ull : (1ull << (run_end - lane - 1u)) - 1ull);
      const unsigned long long first_run = begins & ~1ull ? (1ull << __builtin_ctzll(begins & ~1ull)) - 1ull : ~0ull;
      if (lane == 0) tv.s_runs[tid >> 6] = make_uint2(u.mine ? u.i : 0xFFFFFFFFu, ((good & first_run) ? 1u : 0u) | ((begins & ~1ull) ? 0u : 2u));
      won = valid && !behind;
      const uint32_t m = wave_max_u32(mx);
      if (lane == 0 && m) atomicMax(tv.s_max, m);
      tv.sync();
      in_order = wave_value(wild) != u.batch;
      if (in_order && won && run_end == 64u)
        for (uint32_t w = (tid >> 6) + 1u; w < (tv.team >> 6); ++w) {
          const uint2 r = tv.s_runs[w];
          if (r.x != u.i) break;
          if (r.y & 1u) won = false;
          if (!(r.y & 2u) || !won) break;
        }
    }
    if (__builtin_expect(!in_order, 0)) {   // (out of the way: the code of a round is fetched line by line as it goes)
      if constexpr (MEM) {   // (markers in memory: atomics there, and a read that passes by the first-level cache)
        GlobalPtr<uint32_t> bits = (GlobalPtr<uint32_t>)tv.leaves;
        if (valid) __hip_atomic_fetch_max(&bits[u.i], mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if constexpr (WAVE) wait_memory(); else tv.sync();
        won = valid && __hip_atomic_load(&bits[u.i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == mark;
        if constexpr (WAVE) wait_memory(); else tv.sync();
      } else {
        uint32_t* bits = reinterpret_cast<uint32_t*>(tv.tree);
        if (valid) atomicMax(&bits[u.i], mark);
        if constexpr (WAVE) wave_order(); else tv.sync();
        won = valid && bits[u.i] == mark;
        if constexpr (WAVE) wave_order(); else tv.sync();
      }
    }
    if (won) tv.set_leaf(u.i, u.v);
    if constexpr (WAVE) {
      const uint32_t m = wave_max_u32(mx);
      max_bits = m > max_bits ? m : max_bits;
      wave_order();
    } else {
      if (!u.sorted && mx) atomicMax(tv.s_max, mx);
      if (ins.on || !u.sorted) tv.sync();   // (the insertion comes behind the update)
    }
  }
  if (ins.on) {
    uint32_t mx = 0;
    if (ins.mine) {
      float v = __uint_as_float(WAVE ? max_bits : *tv.s_max);
      placed = true;
      if (ins.given) {
        v = ins.v;
        placed = valid_priority(v);
        if (!placed) flags |= 2u;
        mx = placed && v > 0.0f ? __float_as_uint(v) : 0u;
      }
      if (placed) tv.set_leaf(ins.slot, v);
    }
    if (ins.given) {
      if constexpr (WAVE) {
        const uint32_t m = wave_max_u32(mx);
        max_bits = m > max_bits ? m : max_bits;
      } else if (mx) {
        atomicMax(tv.s_max, mx);
      }
    }
  }
  // the ancestors (elements that share a parent store the same sum)
  if (u.on || ins.on) {
    if constexpr (WAVE) {
      const bool together = !u.on || !ins.on || u.n + ins.n <= 64u;   // (no lane has both)
      for (int pass = 0; pass < (together ? 1 : 2); ++pass) {
        const bool act = together ? valid || placed : pass == 0 ? valid : placed;
        const uint32_t leaf = together ? (placed ? ins.slot : u.i) : pass == 0 ? u.i : ins.slot;
        for (uint32_t v = 1; v < tv.vt; ++v) {
          wave_order();
          if (act) {
            const uint32_t parent = leaf >> (v * LOGR);
            tv.tree[tv.off(v) + parent] = child_group_sum<LOGK, MEM>(tv, v, parent);
          }
        }
      }
      wave_order();
      total = sum_top<LOGK, MEM>(tv);
      wave_order();
    } else {
      // A level of no more nodes than there are elements is recomputed whole (fewer lanes than elements).
      const uint32_t elements = (u.on ? u.n : 0u) + (ins.on ? ins.n : 0u);
      for (uint32_t v = 1; v < tv.vt; ++v) {
        tv.sync();
        const uint32_t nodes = tv.n(v);
        if (nodes <= elements) {
          for (uint32_t j = tid; j < nodes; j += tv.team) tv.tree[tv.off(v) + j] = child_group_sum<LOGK, MEM>(tv, v, j);
          continue;
        }
        const uint32_t pu = u.i >> (v * LOGR), pi = ins.slot >> (v * LOGR);
        if (valid) tv.tree[tv.off(v) + pu] = child_group_sum<LOGK, MEM>(tv, v, pu);
        if (placed) tv.tree[tv.off(v) + pi] = child_group_sum<LOGK, MEM>(tv, v, pi);
      }
      tv.sync();
      if (tid < 64u) sum_top<LOGK, MEM>(tv);
    }
  }
}

// Waves of the team with a uniform outside [0, 1) (or -0, which does no harm) leave the number of the sampling.  Lanes without
// a sample hold 0, or a uniform of an earlier one.
__device__ __forceinline__ void note_wild(float u, uint32_t batch, uint32_t* s_wild) {
  if (__builtin_expect(__any(__float_as_uint(u) >= 0x3F800000u), 0)) *s_wild = batch;
}

// The binary steps of the walk inside a group held in registers, without a look at the right block: see walk_tree.
// (children: the N children; node: 2 node + 1 for a turn to the right)
template <int N>
__device__ __forceinline__ float first_half_sum(const float (&c)[N]) {   // of c[0 .. N/2), pairwise
  if constexpr (N == 2) {
    return c[0];
  } else {
    float h[N / 2];
#pragma unroll
    for (int i = 0; i < N / 2; ++i) h[i] = c[i];
    if constexpr (N == 4) return h[0] + h[1];
    else {
      float up[N / 4];
#pragma unroll
      for (int i = 0; i < N / 4; ++i) up[i] = h[2 * i] + h[2 * i + 1];
#pragma unroll
      for (int w = N / 8; w >= 1; w /= 2)
#pragma unroll
        for (int i = 0; i < w; ++i) up[i] = up[2 * i] + up[2 * i + 1];
      return up[0];
    }
  }
}
template <int N>
__device__ __forceinline__ void turn_down(const float (&c)[N], float& r, uint32_t& node, float& val) {
  if constexpr (N == 1) {
    val = c[0];
  } else {
    const float L = first_half_sum<N>(c), rest = r - L;
    const bool right = !(r < L);
    r = right ? rest : r;
    node = 2u * node + (right ? 1u : 0u);
    float h[N / 2];
#pragma unroll
    for (int i = 0; i < N / 2; ++i) h[i] = right ? c[N / 2 + i] : c[i];
    turn_down<N / 2>(h, r, node, val);
  }
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
// looking.  (With the right blocks' sums left out, and the sixteen children kept in registers instead of read a second
// time once the chunk of four is known, a level takes two thirds of the 570 cycles it took.)
template <int LOGK, bool MEM>
__device__ __forceinline__ void walk_tree(const TreeView<MEM>& tv, uint32_t i, uint32_t n, float u, float total, float seg, uint32_t& node,
                                          float& val) {
  constexpr int LOGR = Wide<LOGK>::LOGR, R = Wide<LOGK>::R;
  node = 0xFFFFFFFFu;
  val = 0.0f;
  if (!(total > 0.0f)) return;
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
  for (; v > 0; --v) {
    float unused;
    level_down<LOGR>(static_cast<const float*>(tv.tree) + tv.off(v) + (size_t)min_u32(node, tv.n(v + 1)) * R, r, node, unused);
  }
  const uint32_t n1 = tv.n(1);
  bool astray = false;
  if constexpr (MEM) {   // (no such group behind the leaves in memory)
    astray = node >= n1;
    level_down<LOGR>(as_global(static_cast<const float*>(tv.leaves)) + (size_t)(astray ? 0u : node) * R, r, node, val);
  } else {
    level_down<LOGR>(static_cast<const float*>(tv.tree) + (size_t)min_u32(node, n1) * R, r, node, val);
  }
  if (__builtin_expect(__any(astray || !(val > 0.0f)), 0)) {
    r = r0;
    node = 0;
    for (v = tv.V; v-- > 0;) {
      unsigned child;
      if constexpr (MEM) {
        if (v == 0) descend_lane<LOGR>(as_global(static_cast<const float*>(tv.leaves)) + (size_t)node * R, r, child, val);
        else descend_lane<LOGR>(static_cast<const float*>(tv.tree) + tv.off(v) + (size_t)node * R, r, child, val);
      } else {
        descend_lane<LOGR>(static_cast<const float*>(tv.tree) + tv.off(v) + (size_t)node * R, r, child, val);
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

// The list of steps.  What bounds it is one chain of instructions and LDS trips from step to step (the tree as one
// step leaves it is what the next samples from), so everything that is not tree work is taken off that chain:
//  - The waves split: the first ones (the team, a lane per sample and per inserted row) do the tree work, the others
//    move the rows and turn values into weights, one step behind.  Batches of more than 512 leave no waves over; the
//    team then does both in turn.
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
// (its lanes wait for their stores before the barrier that ends the sampling), and overwrite what the gather of the
// step before has read (all of whose loads have arrived at the barrier in front of the insertion's stores).
// 100 steps on 10 000 leaves at K = 16 (32 samples, 4 new rows of 41 bytes): 232 us; 1001 us as one phase after the
// other by the whole workgroup with a full barrier between them.
// AHEAD: no step reads what a step returns.
template <int LOGK, bool WAVE, bool MEM, bool AHEAD>
__global__ void __launch_bounds__(1024)
k_run_steps(StreamKernelArgs ka) {
  const Geom& g = ka.g;
  const StreamArgs& a = ka.a;
  extern __shared__ __attribute__((aligned(16))) float tree[];
  __shared__ LevelTable tab;
  __shared__ uint32_t s_off[kStreamLevels + 2], s_n[kStreamLevels + 1];
  __shared__ uint32_t s_max, s_vmin[2], s_bmin[2], s_wild, s_flags, s_arrived;
  __shared__ uint2 s_runs[16];
  __shared__ PieceFields s_rows, s_ins;
  const uint32_t t = blockIdx.x;
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint32_t H = g.H, T = g.T, B = a.B, n_ins = a.n_insert, N = g.N;
  const uint32_t V = a.levels;
  fill_level_table(H, t, &tab);
  if (tid >= 64 && tid <= 64 + V + 1) {
    s_off[tid - 64] = kernarg_at<StreamArgs>(offsetof(StreamKernelArgs, a))->off[tid - 64];
    if (tid <= 64 + V) s_n[tid - 64] = kernarg_at<Geom>(0)->n[level_height<LOGK>(tid - 64, H)];
  }
  if (tid == 0) {
    s_max = read_max_bits(g, t);
    s_vmin[0] = s_vmin[1] = s_bmin[0] = s_bmin[1] = kNoMin;
    s_wild = 0;
    s_flags = 0;
    s_arrived = 0;
  }
  // lanes of the team, of the rows, of the weights
  const uint32_t wanted = WAVE ? 64u : ((B > n_ins ? B : n_ins) + 63u) / 64u * 64u;
  const bool apart = wanted <= 512u;
  const uint32_t team = apart ? wanted : 1024u;   // (not apart: every wave comes to the team's barriers)
  const bool in_team = tid < team, in_rows = !apart || tid >= team;
  const uint32_t rn = apart ? 1024u - team : 1024u, rl = apart ? tid - team : tid;
  const uint32_t rw = wave_value(rl >> 6), rws = rn >> 6;   // number of this wave among the row waves, and how many there are
  const uint32_t w0 = apart ? 1024u - (B + 63u) / 64u * 64u : 0u;
  const bool weigher = tid >= w0 && tid - w0 < B;
  // (the field tables from the argument segment by vector loads, a lane per field)
  if (tid >= 128 && tid < 256) {
    const bool rows = tid < 192;
    const FieldTable* ft = kernarg_at<FieldTable>(offsetof(StreamKernelArgs, a) + (rows ? offsetof(StreamArgs, rows) : offsetof(StreamArgs, ins)));
    const uint32_t n = rows ? B : n_ins;
    fill_piece_fields(ft, lane < (uint32_t)kMaxFields ? ft->io[lane] : nullptr, t, n, (uint64_t)T * n, rows ? &s_rows : &s_ins);
  }
  __syncthreads();
  const uint32_t insert_items = in_rows ? s_ins.items() : 0u;
  RowItem ip;
  uint4 iv;
  if (rw < insert_items) {   // (the first item of an insertion is fetched a step ahead)
    ip = find_item(s_ins, rw);
    if (ip.on) iv = load_piece(ip.dense, ip.w);
  }
  // inputs of the team: the uniform of the step to sample, value (and index) of the update to apply, inserted priority
  float u_i = 0.0f, u_next = 0.0f, up_v = 0.0f, in_v = 0.0f;
  [[maybe_unused]] float beta_i = 0.0f;
  uint32_t up_i = 0;
  const uint32_t j_ins = WAVE ? lane - (64u - n_ins) : tid;   // (WAVE: the last lanes of the wave, so that samples and rows share it)
  const bool inserts = in_team && (!WAVE || lane >= 64u - n_ins) && j_ins < n_ins;
  if (in_team && tid < B) u_i = a.u[(size_t)t * B + tid];
  if (inserts && a.ins_prio) in_v = a.ins_prio[(size_t)t * n_ins + j_ins];
  if constexpr (!AHEAD) beta_i = a.beta[0];
  __syncthreads();
  LdsTree lt;
  lt.tree = tree;
  lt.leaves_mem = MEM ? tab.lvl[0] : nullptr;
  lt.off = s_off;
  lt.n = s_n;
  lt.max_bits = &s_max;
  lt.H = H;
  lt.V = V;
  lds_tree_load<LOGK>(tab, lt);
  uint32_t* nodes = reinterpret_cast<uint32_t*>(tree + s_off[V + 1]);   // [B] sampled leaves of the step
  float* values = reinterpret_cast<float*>(nodes + 512);                // [B] and their values (apart only: B <= 512)
  TreeView<MEM> tv;
  tv.tree = tree;
  tv.leaves = lt.leaves_mem;
  tv.off_reg = s_off[lane <= V + 1 ? lane : V + 1];
  tv.n_reg = s_n[lane <= V ? lane : V];
  tv.V = V;
  tv.N = N;
  tv.vt = 1;
  while (tv.vt < V && tv.n(tv.vt) > kTopNodes) ++tv.vt;
  tv.s_max = &s_max;
  tv.s_arrived = &s_arrived;
  tv.s_wild = &s_wild;
  tv.s_runs = s_runs;
  tv.apart = apart;
  tv.team = team;
  tv.met = 0;
  uint32_t cursor = a.cursor, size = a.size, upd_size = 0;
  uint32_t flags = 0;
  __syncthreads();
  uint32_t max_bits = s_max;      // (WAVE: the team's copy; else s_max counts)
  uint32_t node = 0xFFFFFFFFu;    // this lane's sample of the step before
  float val = 0.0f;
  float total = tree[s_off[V]];   // (WAVE: the root as the latest change has left it)
  for (uint32_t s = 0;; ++s) {
    const bool more = s < a.n_steps;
    // ---- rows and weights of the step before
    float w_out = 0.0f, v_out = 0.0f;
    uint32_t n_out = 0;
    if (s) {
      if (in_rows) gather_rows(s_rows, rw, rws, nodes, N, a.rows.row_stride, s - 1, flags);
      if (weigher) {
        n_out = nodes[tid - w0];
        v_out = apart ? values[tid - w0] : val;
        if (a.out_w) {
          const uint32_t vmin = s_vmin[(s - 1) & 1u];
          const uint32_t least = a.buffer_norm ? s_bmin[(s - 1) & 1u] : vmin;
          w_out = vmin == kNoMin ? 0.0f : importance_weight(v_out, __uint_as_float(least), AHEAD ? a.beta[s - 1] : beta_i);
        }
      }
    }
    auto store_results = [&]() {   // of the step before
      if (!weigher) return;
      const size_t o = ((size_t)(s - 1) * T + t) * B + (tid - w0);
      a.out_idx[o] = n_out;
      if (a.out_prio) a.out_prio[o] = v_out;
      if (a.out_w) a.out_w[o] = w_out;
    };
    if (!AHEAD && s) {
      store_results();
      wait_memory();
      lds_barrier();
      if (in_team && tid < B) {
        const size_t bo = ((size_t)(s - 1) * T + t) * B + tid;
        if (a.upd_prio) {
          up_v = a.upd_prio[bo];
          if (!a.upd_is_sampled) up_i = a.upd_idx[bo];
        }
        if (more) u_i = a.u[bo + (size_t)T * B];
      }
      if (more) {
        if (rw < insert_items && ip.on) iv = load_piece(ip.dense + (uint64_t)s * s_ins.step[ip.f], ip.w);
        if (inserts && a.ins_prio) in_v = a.ins_prio[((size_t)s * T + t) * n_ins + j_ins];
        if constexpr (!AHEAD) beta_i = a.beta[s];
      }
    }
    // ---- the tree: update of the step before, insertion of this one
    const bool do_upd = s > 0 && a.upd_prio != nullptr, do_ins = more && n_ins > 0;
    if (in_team) {
      const UpdateWork up{do_upd, in_team && tid < B, a.upd_is_sampled != 0, B, a.upd_is_sampled ? node : up_i, upd_size, up_v, s};
      const InsertWork in{do_ins, inserts, a.ins_prio != nullptr, n_ins, inserts ? ring_slot(cursor, j_ins, N) : 0u, in_v};
      change_tree<LOGK, WAVE, MEM>(tv, up, in, max_bits, flags, total);
      // inputs of the next round
      if (AHEAD && in_team && tid < B) {
        const size_t bo = ((size_t)s * T + t) * B + tid;
        if (more && a.upd_prio) {
          up_v = a.upd_prio[bo];
          if (!a.upd_is_sampled) up_i = a.upd_idx[bo];
        }
        if (s + 1 < a.n_steps) u_next = a.u[bo + (size_t)T * B];   // (here and not behind the walk: the next wait would be for it)
      }
    }
    if (do_ins) {
      cursor = ring_slot(cursor, n_ins, N);
      size = size + n_ins > N ? N : size + n_ins;
    }
    upd_size = size;
    // ---- the rows of the step before have been read; the tree is whole
    if (WAVE && MEM && a.buffer_norm) wait_memory();   // (!WAVE: the team has waited for its leaves)
    lds_barrier();
    if (do_ins && in_rows) {
      const uint32_t first = cursor >= n_ins ? cursor - n_ins : cursor + (N - n_ins);
      if (rw < insert_items && ip.on) place_row_piece(ip, first, N, a.ins.row_stride, nullptr, iv);
      insert_rows(s_ins, rw + rws, rws, first, N, a.ins.row_stride, s, nullptr);
      wait_memory();
    }
    if (AHEAD && s) store_results();
    if (!more) break;
    if (AHEAD && s + 1 < a.n_steps && n_ins) {
      if (rw < insert_items && ip.on) iv = load_piece(ip.dense + (uint64_t)(s + 1) * s_ins.step[ip.f], ip.w);
      if (inserts && a.ins_prio) in_v = a.ins_prio[((size_t)(s + 1) * T + t) * n_ins + j_ins];
    }
    if (tid == 0) s_vmin[(s + 1) & 1u] = s_bmin[(s + 1) & 1u] = kNoMin;   // (read by the weights of step s - 1, before the barrier)
    // ---- weights relative to the whole tree: its smallest positive leaf
    if (a.buffer_norm && a.out_w && in_rows) {
      uint32_t m = kNoMin;
      for (uint32_t e = rl; e < N; e += rn) m = min_u32(m, positive_bits(tv.leaf(e)));
      m = wave_min_u32(m);
      if (lane == 0 && m != kNoMin) atomicMin(&s_bmin[s & 1u], m);
    }
    // ---- sampling
    if (in_team && (WAVE || (tid & ~63u) < B)) {
      if constexpr (!WAVE) note_wild(u_i, s + 1u, &s_wild);
      if constexpr (!WAVE) total = tree[tv.off(V)];
      walk_tree<LOGK, MEM>(tv, tid, B, u_i, total, mass_per_sample(total, B), node, val);
      if (node == 0xFFFFFFFFu) {
        if (tid == 0) flags |= 4u;
      } else if (a.out_w) {
        const uint32_t m = wave_min_u32(tid < B ? __float_as_uint(val) : kNoMin);
        if (lane == 0) {
          if constexpr (WAVE) s_vmin[s & 1u] = m;
          else atomicMin(&s_vmin[s & 1u], m);
        }
      }
      if (tid < B) {
        nodes[tid] = node;
        if (apart) values[tid] = val;
      }
      if constexpr (AHEAD) u_i = u_next;
    }
    lds_barrier();
  }
  if (WAVE && tid == 0) s_max = max_bits;
  __syncthreads();
  lds_tree_store<LOGK>(g, t, tab, lt, flags, &s_flags);
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
// runs as a step does there (see above): its tree changes in one pass over the ancestors, rows and weights of the
// sampling request before it beside them, and what it reads fetched in the round before.  The requests themselves come
// in two rounds ahead (three at a time: a round takes no more).
// Fetching ahead is only right where a request reads nothing that one just before it writes (an update whose index
// array is the sampled one, say).  The host has checked that (QueueArgs::ahead); where it does not hold, every
// request is a round of its own with an empty one behind it, which brings all results to memory.
// 20 times (insert 16 rows, sample 512, update them) on 30 000 leaves at K = 16: 188 us; 353 us one request after the
// other by the whole workgroup with a full barrier between their phases.
struct QueueKernelArgs {            // one kernel argument (Geom first: see fill_level_table)
  Geom g;
  QueueArgs a;
};
constexpr uint32_t kRoundRequests = 3, kRequestWords = sizeof(per_request) / 4;
struct QueueRound {                 // what a round takes: places of its requests among the three fetched for it (3: none)
  uint32_t upd, ins, smp, used;
};
// The round that starts with the `left` requests of q (at most three are looked at).
__device__ __forceinline__ QueueRound take_round(const per_request* q, uint32_t left, bool single) {
  QueueRound r{3, 3, 3, 0};
  uint32_t stage = 0;   // 1: past the update, 2: past the insertion, 3: past the sampling
#pragma unroll
  for (uint32_t k = 0; k < kRoundRequests; ++k) {
    const uint32_t op = k < left ? (uint32_t)__builtin_amdgcn_readfirstlane((int)q[k].op) : 0u;
    const bool u = op == PER_OP_UPDATE && stage < 1, i = op == PER_OP_INSERT && stage < 2, s = op == PER_OP_SAMPLE && stage < 3;
    if (r.used == k && (u || i || s) && !(single && k)) {
      if (u) r.upd = k, stage = 1;
      if (i) r.ins = k, stage = 2;
      if (s) r.smp = k, stage = 3;
      r.used = k + 1;
    }
  }
  if (r.used == 0 && left) r.used = 1;   // (an unknown operation is passed over: the kernel ends whatever the queue holds)
  return r;
}
template <int LOGK, bool WAVE, bool MEM>
__global__ void __launch_bounds__(1024)
k_run_requests(QueueKernelArgs ka) {
  const Geom& g = ka.g;
  const QueueArgs& a = ka.a;
  extern __shared__ __attribute__((aligned(16))) float tree[];
  __shared__ LevelTable tab;
  __shared__ uint32_t s_off[kStreamLevels + 2], s_n[kStreamLevels + 1];
  __shared__ per_request s_req[3][kRoundRequests];   // round i: s_req[i % 3]
  __shared__ PieceFields s_rows[2], s_ins[2];        // by parity of the round
  __shared__ uint32_t s_skip[2][32];                 // bit j: row j of the round's insertion is deferred
  __shared__ uint32_t s_max, s_vmin[2], s_bmin[2], s_wild, s_flags, s_arrived;
  __shared__ uint2 s_runs[16];
  const uint32_t t = blockIdx.x;
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint32_t H = g.H, N = g.N, n_requests = a.n_requests;
  const FieldTable* fields = kernarg_at<FieldTable>(offsetof(QueueKernelArgs, a) + offsetof(QueueArgs, fields));
  const uint32_t* queue = reinterpret_cast<const uint32_t*>(a.queue);
  const uint32_t V = a.levels;
  fill_level_table(H, t, &tab);
  if (tid >= 64 && tid <= 64 + V + 1) {
    s_off[tid - 64] = kernarg_at<QueueArgs>(offsetof(QueueKernelArgs, a))->off[tid - 64];
    if (tid <= 64 + V) s_n[tid - 64] = kernarg_at<Geom>(0)->n[level_height<LOGK>(tid - 64, H)];
  }
  if (tid == 0) {
    s_max = read_max_bits(g, t);
    s_vmin[0] = s_vmin[1] = s_bmin[0] = s_bmin[1] = kNoMin;
    s_wild = 0;
    s_flags = 0;
    s_arrived = 0;
  }
  // words of the three requests from `at` on, two per lane of one wave
  const bool fetcher = tid >= 960;
  constexpr uint32_t kFetch = kRoundRequests * kRequestWords;
  static_assert(kFetch <= 128, "two words per lane");
  auto fetch = [&](uint32_t at, uint32_t& x, uint32_t& y) {
    const uint64_t w0 = (uint64_t)at * kRequestWords, all = (uint64_t)n_requests * kRequestWords;
    x = y = 0;
    if (w0 + lane < all) x = queue[w0 + lane];
    if (lane + 64u < kFetch && w0 + lane + 64u < all) y = queue[w0 + lane + 64u];
  };
  auto park = [&](uint32_t slot, uint32_t x, uint32_t y) {
    uint32_t* dst = reinterpret_cast<uint32_t*>(&s_req[slot][0]);
    dst[lane] = x;
    if (lane + 64u < kFetch) dst[lane + 64u] = y;
  };
  if (fetcher) {
    uint32_t x, y;
    fetch(0, x, y);
    park(0, x, y);
  }
  // lanes of the team, of the rows (the weights: see k_run_steps)
  const uint32_t wanted = WAVE ? 64u : (a.most + 63u) / 64u * 64u;
  const bool apart = wanted <= 512u;
  const uint32_t team = apart ? wanted : 1024u;   // (not apart: every wave comes to the team's barriers)
  const bool in_team = tid < team, in_rows = !apart || tid >= team;
  const uint32_t rn = apart ? 1024u - team : 1024u, rl = apart ? tid - team : tid;
  const uint32_t rw = wave_value(rl >> 6), rws = rn >> 6;   // number of this wave among the row waves, and how many there are
  __syncthreads();
  LdsTree lt;
  lt.tree = tree;
  lt.leaves_mem = MEM ? tab.lvl[0] : nullptr;
  lt.off = s_off;
  lt.n = s_n;
  lt.max_bits = &s_max;
  lt.H = H;
  lt.V = V;
  lds_tree_load<LOGK>(tab, lt);
  uint32_t* nodes = reinterpret_cast<uint32_t*>(tree + s_off[V + 1]);   // sampled leaves of the round
  float* values = reinterpret_cast<float*>(nodes + 512);                // and their values (apart only: at most 512)
  TreeView<MEM> tv;
  tv.tree = tree;
  tv.leaves = lt.leaves_mem;
  tv.off_reg = s_off[lane <= V + 1 ? lane : V + 1];
  tv.n_reg = s_n[lane <= V ? lane : V];
  tv.V = V;
  tv.N = N;
  tv.vt = 1;
  while (tv.vt < V && tv.n(tv.vt) > kTopNodes) ++tv.vt;
  tv.s_max = &s_max;
  tv.s_arrived = &s_arrived;
  tv.s_wild = &s_wild;
  tv.s_runs = s_runs;
  tv.apart = apart;
  tv.team = team;
  tv.met = 0;
  uint32_t cursor = a.cursor, size = a.size;
  uint32_t flags = 0;
  uint32_t node = 0xFFFFFFFFu;    // this lane's sample of the latest sampling request
  float val = 0.0f;
  float total = 0.0f;             // (WAVE: the root as the latest change has left it)
  // the round under way, the next one, and where the one after that starts in the queue
  const bool single = a.ahead == 0;
  QueueRound cur = take_round(s_req[0], n_requests, single);
  uint32_t pos = cur.used, pos_cur = 0;
  // what the rounds read: uniform; value and index of the update; inserted priority; rows
  float u_i = 0.0f, u_next = 0.0f, up_v = 0.0f, in_v = 0.0f;
  uint32_t up_i = 0;
  RowItem ip;
  uint4 iv;
  uint32_t sampled = 0;                    // sampling requests so far
  uint32_t sample_n = 0, before_smp = 3;   // the sampling request of the round before: its batch (0: none) and place
  auto inserted_by = [&](const per_request& q) -> uint32_t {   // the row of the insertion that this lane places (>= n: none)
    const uint32_t j = WAVE ? lane - (64u - q.n) : tid;
    return in_team && (!WAVE || lane >= 64u - q.n) ? j : 0xFFFFFFFFu;
  };
  auto fill_fields = [&](const per_request* q, PieceFields* pf) {
    fill_piece_fields(fields, q && lane < (uint32_t)kMaxFields ? static_cast<uint8_t*>(q->field[lane]) : nullptr, t, q ? q->n : 0u, 0, pf);
  };
  // fetches what round r (its requests in q, its insertion at ring slot `at`) reads
  auto fetch_inputs = [&](const QueueRound& r, const per_request* q, uint32_t parity, uint32_t at) {
    if (r.smp < 3) {
      const per_request& w = q[r.smp];
      if (in_team && tid < w.n) u_next = as_global(w.u)[(size_t)t * w.n + tid];
    }
    if (r.upd < 3) {
      const per_request& w = q[r.upd];
      if (in_team && tid < w.n) {
        up_v = as_global(w.prio)[(size_t)t * w.n + tid];
        if (w.idx) up_i = as_global(w.idx)[(size_t)t * w.n + tid];
      }
    }
    if (r.ins < 3) {
      const per_request& w = q[r.ins];
      const uint32_t j = inserted_by(w);
      if (j < w.n && w.prio) in_v = as_global(w.prio)[(size_t)t * w.n + j];
      if (w.protect && in_rows) {   // collision-free insertion: rows aimed at a protected slot are deferred (see k_insert_small)
        const uint32_t* protect = w.protect + (size_t)t * w.n_protect;
        for (uint32_t k = rl; k < w.n_protect; k += rn) {
          const uint32_t i = as_global(protect)[k];
          if (i < N) {
            const uint32_t p = i >= at ? i - at : i + (N - at);   // position in the ring window
            if (p < w.n) atomicOr(&s_skip[parity][p >> 5], 1u << (p & 31u));
          }
        }
      }
      if (in_rows && rw < s_ins[parity].items()) {   // (the first item of the insertion; the others come when it is their turn)
        ip = find_item(s_ins[parity], rw);
        if (ip.on) iv = load_piece(ip.dense, ip.w);
      }
    }
  };
  {   // round 0, and the requests of round 1
    if (tid >= 896 && tid < 960) fill_fields(cur.ins < 3 ? &s_req[0][cur.ins] : nullptr, &s_ins[0]);
    if (fetcher) {
      uint32_t x, y;
      fetch(single ? 0u : pos, x, y);   // (single: round 1 is empty)
      park(1, x, y);
    }
    if (tid < 64) s_skip[tid >> 5][tid & 31u] = 0;
    __syncthreads();
    fetch_inputs(cur, s_req[0], 0, cursor);
    u_i = u_next;
  }
  __syncthreads();
  uint32_t max_bits = s_max;      // (WAVE: the team's copy; else s_max counts)
  total = tree[s_off[V]];

  for (uint32_t i = 0;; ++i) {
    const uint32_t par = i & 1u, slot_cur = i % 3u, slot_next = (i + 1u) % 3u, slot_before = (i + 2u) % 3u;
    const per_request* q = s_req[slot_cur];
    const bool more = pos_cur < n_requests;
    // (single: a round with nothing in it behind every request)
    const bool gap = single && cur.used != 0;
    const QueueRound next = gap ? QueueRound{3, 3, 3, 0} : take_round(s_req[slot_next], n_requests - (pos < n_requests ? pos : n_requests), single);
    // ---- rows and weights of the round before
    const uint32_t w0 = apart ? 1024u - (sample_n + 63u) / 64u * 64u : 0u;
    const bool weigher = sample_n && tid >= w0 && tid - w0 < sample_n;
    float w_out = 0.0f, v_out = 0.0f;
    uint32_t n_out = 0;
    uint32_t* out_idx = nullptr;
    float *out_w = nullptr, *out_prio = nullptr;
    if (sample_n && in_rows) gather_rows(s_rows[par ^ 1u], rw, rws, nodes, N, a.fields.row_stride, 0, flags);
    if (weigher) {
      const per_request& w = s_req[slot_before][before_smp];
      n_out = nodes[tid - w0];
      v_out = apart ? values[tid - w0] : val;
      const size_t o = (size_t)t * sample_n + (tid - w0);
      out_idx = w.idx + o;
      if (w.out_prio) out_prio = w.out_prio + o;
      if (w.out_weight) {
        out_w = w.out_weight + o;
        const uint32_t vmin = s_vmin[par ^ 1u];
        const uint32_t least = a.buffer_norm ? s_bmin[par ^ 1u] : vmin;
        w_out = vmin == kNoMin ? 0.0f : importance_weight(v_out, __uint_as_float(least), w.beta);
      }
    }
    // ---- the requests of the round after the next one are asked for
    const uint32_t pos_after = pos + next.used;
    uint32_t req_x = 0, req_y = 0;
    if (fetcher) fetch(single && next.used ? 0u : pos_after < n_requests ? pos_after : n_requests, req_x, req_y);
    // ---- the tree: update, insertion
    const bool do_upd = cur.upd < 3, do_ins = cur.ins < 3;
    const uint32_t n_ins = do_ins ? wave_value(q[cur.ins].n) : 0u;
    const uint32_t cursor0 = cursor;
    if (in_team) {
      UpdateWork up{};
      up.on = do_upd;
      if (do_upd) {
        const per_request& w = q[cur.upd];
        up.n = wave_value(w.n);
        up.mine = in_team && tid < up.n;
        up.sorted = w.idx == nullptr;
        up.i = w.idx ? up_i : node;
        up.size = size;
        up.v = up_v;
        up.batch = sampled;
      }
      InsertWork in{};
      in.on = do_ins;
      if (do_ins) {
        const uint32_t j = inserted_by(q[cur.ins]);
        in.n = n_ins;
        in.mine = j < n_ins && !((s_skip[par][(j & 1023u) >> 5] >> (j & 31u)) & 1u);
        in.given = q[cur.ins].prio != nullptr;
        in.slot = in.mine ? ring_slot(cursor, j, N) : 0u;
        in.v = in_v;
      }
      change_tree<LOGK, WAVE, MEM>(tv, up, in, max_bits, flags, total);
    }
    if (do_ins) {
      cursor = ring_slot(cursor, n_ins, N);
      size = size + n_ins > N ? N : size + n_ins;
    }
    // ---- tables of the next round's insertion and of this round's sample; the next round's deferred rows, none so far
    if (tid >= 896 && tid < 960) {
      fill_fields(next.ins < 3 ? &s_req[slot_next][next.ins] : nullptr, &s_ins[par ^ 1u]);
      // (s_rows of the round before is still in use: this round's is the other one)
      fill_fields(cur.smp < 3 ? &q[cur.smp] : nullptr, &s_rows[par]);
      if (lane < 32) s_skip[par ^ 1u][lane] = 0;
    }
    // ---- the rows of the round before have been read; the tree is whole
    if (WAVE && MEM) wait_memory();   // (!WAVE: the team has waited for its leaves)
    lds_barrier();
    if (do_ins && in_rows) {
      auto deferred = [&](uint32_t row) -> bool { return ((s_skip[par][row >> 5] >> (row & 31u)) & 1u) != 0; };
      if (rw < s_ins[par].items() && ip.on) place_row_piece(ip, cursor0, N, a.fields.row_stride, s_skip[par], iv);
      insert_rows(s_ins[par], rw + rws, rws, cursor0, N, a.fields.row_stride, 0, s_skip[par]);
      if (q[cur.ins].idx) {
        uint32_t* slots = q[cur.ins].idx + (size_t)t * n_ins;
        for (uint32_t j = rl; j < n_ins; j += rn) as_global(slots)[j] = deferred(j) ? 0xFFFFFFFFu : ring_slot(cursor0, j, N);
      }
      wait_memory();
    }
    if (weigher) {
      *as_global(out_idx) = n_out;
      if (out_prio) *as_global(out_prio) = v_out;
      if (out_w) *as_global(out_w) = w_out;
    }
    if (!more) break;
    if (single) {   // (what this round has stored is there before the next one's inputs are read)
      wait_memory();
      lds_barrier();
    }
    fetch_inputs(next, s_req[slot_next], par ^ 1u, cursor);
    if (tid == 0) s_vmin[par ^ 1u] = s_bmin[par ^ 1u] = kNoMin;   // (read by the weights of the round before, in front of the barrier)
    if (fetcher) park(slot_before, req_x, req_y);                 // (likewise)
    const per_request* smp = cur.smp < 3 ? &q[cur.smp] : nullptr;
    sample_n = smp ? wave_value(smp->n) : 0u;
    before_smp = cur.smp;
    if (smp) {
      ++sampled;
      // ---- weights relative to the whole tree: its smallest positive leaf
      if (a.buffer_norm && smp->out_weight && in_rows) {
        uint32_t m = kNoMin;
        for (uint32_t e = rl; e < N; e += rn) m = min_u32(m, positive_bits(tv.leaf(e)));
        m = wave_min_u32(m);
        if (lane == 0 && m != kNoMin) atomicMin(&s_bmin[par], m);
      }
      // ---- sampling
      if (in_team && (WAVE || (tid & ~63u) < sample_n)) {
        if constexpr (!WAVE) note_wild(u_i, sampled, &s_wild);
        if constexpr (!WAVE) total = tree[tv.off(V)];
        walk_tree<LOGK, MEM>(tv, tid, sample_n, u_i, total, mass_per_sample(total, sample_n), node, val);
        if (node == 0xFFFFFFFFu) {
          if (tid == 0) flags |= 4u;
        } else if (smp->out_weight) {
          const uint32_t m = wave_min_u32(tid < sample_n ? __float_as_uint(val) : kNoMin);
          if (lane == 0) {
            if constexpr (WAVE) s_vmin[par] = m;
            else atomicMin(&s_vmin[par], m);
          }
        }
        if (tid < sample_n) {
          nodes[tid] = node;
          if (apart) values[tid] = val;
        }
      }
    }
    u_i = u_next;
    if (in_rows) wait_memory();   // (the next sampling request may return its results in the same arrays)
    pos_cur = pos;
    pos = pos_after;
    cur = next;
    lds_barrier();
  }
  if (WAVE && tid == 0) s_max = max_bits;
  __syncthreads();
  lds_tree_store<LOGK>(g, t, tab, lt, flags, &s_flags);
}

// A tree can be worked on where its heights (every one padded to whole child groups), or those above the leaves, fit
// beside the step kernel's other LDS data.
constexpr uint32_t kStreamLdsBytes = 156 * 1024, kStreamBatchWords = 1024;   // (the sampled indices and values of a step)
bool stream_tree_fits(const Geom& g) {
  for (uint32_t skip = 0; skip < 2; ++skip) {
    uint64_t floats = kStreamBatchWords;
    for (uint32_t h = skip; h <= g.H && floats * 4 <= kStreamLdsBytes; ++h)
      floats += h < g.H ? ((uint64_t)g.n[h] + g.K - 1) / g.K * g.K : 4;   // (the root padded to 16 bytes)
    if (floats * 4 <= kStreamLdsBytes && !(skip && g.H < 2)) return true;
  }
  return false;
}
// Levels of the copy (see Wide): the whole tree if that fits, else the levels above the leaves.  Narrow trees take less
// room as levels than as heights, and the groups of zeros behind the levels (512 bytes at most, K = 64) go beyond
// kStreamLdsBytes, so one of the two fits where stream_tree_fits() says so.  Returns the LDS floats, the batch's words
// included (0: neither fits).
constexpr uint32_t kStreamLdsMost = kStreamLdsBytes + 512;
template <int LOGK>
static uint32_t plan_stream_levels(const Geom& g, uint32_t* off, uint32_t* levels, uint32_t* leaves_in_memory) {
  constexpr uint32_t LH = Wide<LOGK>::LH, R = Wide<LOGK>::R;
  const uint32_t V = (g.H + LH - 1) / LH;
  if (V > kStreamLevels) return 0u;
  for (uint32_t skip = 0; skip < 2; ++skip) {
    uint64_t floats = 0;
    for (uint32_t v = 0; v <= V; ++v) {
      off[v] = (uint32_t)floats;
      if (v == 0 && skip) continue;
      floats += v < V ? ((uint64_t)g.n[v * LH] + R - 1) / R * R + (v + 1 < V ? R : 0) : 4;
      if (floats * 4 > kStreamLdsMost) break;
    }
    if ((floats + kStreamBatchWords) * 4 > kStreamLdsMost || (skip && V < 2)) continue;
    off[V + 1] = (uint32_t)floats;
    *levels = V;
    *leaves_in_memory = skip;
    return (uint32_t)floats + kStreamBatchWords;
  }
  return 0u;
}

template <int LOGK>
static hipError_t launch_run_steps_k(const Geom& g, const Tuning& tn, StreamArgs a, hipStream_t s) {
  StreamKernelArgs ka{};
  ka.g = g;
  ka.a = a;
  const uint32_t floats = plan_stream_levels<LOGK>(g, ka.a.off, &ka.a.levels, &ka.a.leaves_in_memory);
  if (!floats) return hipErrorInvalidValue;
  const size_t bytes = (size_t)floats * 4;
  // always the largest workgroup, also for small batches: measured faster than a workgroup of the batch's
  // size (the tree copy and the row movers use all lanes)
  const bool wave = a.B <= 64 && a.n_insert <= 64, mem = ka.a.leaves_in_memory != 0;
#define PER_RUN(W, M, A)                                                                                \
  do {                                                                                                  \
    hipError_t e = grant_lds<&k_run_steps<LOGK, W, M, A>>(tn, bytes);                                   \
    if (e != hipSuccess) return e;                                                                      \
    PER_LAUNCH(KID_RUN_STEPS, (k_run_steps<LOGK, W, M, A>), dim3(g.T), dim3(1024), bytes, s, ka);       \
  } while (0)
#define PER_RUN_WHERE(W, A)                                                                             \
  do {                                                                                                  \
    if (mem) PER_RUN(W, true, A); else PER_RUN(W, false, A);                                            \
  } while (0)
  if (wave) {
    if (a.ahead) PER_RUN_WHERE(true, true); else PER_RUN_WHERE(true, false);
  } else {
    if (a.ahead) PER_RUN_WHERE(false, true); else PER_RUN_WHERE(false, false);
  }
#undef PER_RUN_WHERE
#undef PER_RUN
  return hipGetLastError();
}

hipError_t launch_run_steps(const Geom& g, const Tuning& tn, const StreamArgs& a, hipStream_t s) {
#define CALL(L) launch_run_steps_k<L>(g, tn, a, s)
  PER_DISPATCH_LOGK(g.logK, CALL)
#undef CALL
}

template <int LOGK>
static hipError_t launch_run_requests_k(const Geom& g, const Tuning& tn, const QueueArgs& a, hipStream_t s) {
  QueueKernelArgs ka{};
  ka.g = g;
  ka.a = a;
  const uint32_t floats = plan_stream_levels<LOGK>(g, ka.a.off, &ka.a.levels, &ka.a.leaves_in_memory);
  if (!floats) return hipErrorInvalidValue;
  const size_t bytes = (size_t)floats * 4;
  const bool wave = a.most <= 64, mem = ka.a.leaves_in_memory != 0;
#define PER_RUN(W, M)                                                                                   \
  do {                                                                                                  \
    hipError_t e = grant_lds<&k_run_requests<LOGK, W, M>>(tn, bytes);                                   \
    if (e != hipSuccess) return e;                                                                      \
    PER_LAUNCH(KID_RUN_REQUESTS, (k_run_requests<LOGK, W, M>), dim3(g.T), dim3(1024), bytes, s, ka);    \
  } while (0)
  if (wave) {
    if (mem) PER_RUN(true, true); else PER_RUN(true, false);
  } else {
    if (mem) PER_RUN(false, true); else PER_RUN(false, false);
  }
#undef PER_RUN
  return hipGetLastError();
}

hipError_t launch_run_requests(const Geom& g, const Tuning& tn, const QueueArgs& a, hipStream_t s) {
#define CALL(L) launch_run_requests_k<L>(g, tn, a, s)
  PER_DISPATCH_LOGK(g.logK, CALL)
#undef CALL
}

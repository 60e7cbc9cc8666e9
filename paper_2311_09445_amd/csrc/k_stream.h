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

// Sum of the 4*N children behind g4 in the balanced pairwise order, by a single lane.
template <int N>
__device__ __forceinline__ float sum_chunks(const float4* g4) {
  if constexpr (N == 1) {
    const float4 x = g4[0];
    return (x.x + x.y) + (x.z + x.w);
  } else {
    return sum_chunks<N / 2>(g4) + sum_chunks<N / 2>(g4 + N / 2);
  }
}
template <int LOGK>
__device__ __forceinline__ float lane_group_sum(const float* grp) {
  if constexpr (LOGK == 1) {
    const float2 c = *reinterpret_cast<const float2*>(grp);
    return c.x + c.y;
  } else {
    return sum_chunks<(1 << LOGK) / 4>(reinterpret_cast<const float4*>(grp));
  }
}

// Every active lane recomputes the ancestors of its leaf in the LDS tree, one height per barrier.
// (leaves_mem: the leaves in memory, or null when they are part of the LDS copy)
template <int LOGK>
__device__ __forceinline__ void resum_paths_lds(float* tree, const uint32_t* off, uint32_t H, bool active, uint32_t leaf,
                                                const float* leaves_mem) {
  constexpr int K = Fan<LOGK>::K;
  for (uint32_t h = 1; h <= H; ++h) {
    __syncthreads();   // (also makes the leaf stores of the other waves visible: one compute unit, one first-level cache)
    if (active) {
      const uint32_t parent = leaf >> (h * LOGK);
      if (h == 1 && leaves_mem) tree[off[h] + parent] = lane_group_sum<LOGK>(leaves_mem + (size_t)parent * K);
      else tree[off[h] + parent] = lane_group_sum<LOGK>(tree + off[h - 1] + (size_t)parent * K);
    }
  }
}

// One tree in the LDS of its workgroup, and the few words the operations below share.
struct LdsTree {
  float* tree;              // heights 0 .. H back to back, zero padding included (height 0 left out when leaves_mem is set)
  float* leaves_mem;        // null, or the tree's leaves in memory (zero padded to whole groups)
  const uint32_t* off;      // off[h]: where height h starts (floats); off[H + 1]: all floats
  uint32_t* sampled;        // [1024] indices of the latest sampling operation
  uint32_t* max_bits;       // running maximum priority (fp32 bits)
  uint32_t* vmin_bits;      // minimum of the batch being sampled (fp32 bits)
  uint32_t* bmin_bits;      // smallest positive leaf of the tree (fp32 bits), when the weights are relative to it
  uint32_t* skip;           // [32] bit j: row j of the insertion under way is deferred
  uint32_t H, N;
};

// The three operations are called by all 1024 lanes of the workgroup.  Each leaves the tree
// consistent, but its last phase may still be under way in other waves when it returns: the next
// operation starts with a barrier of its own (lds_sample), or the caller places one.

// Insertion of n <= 1024 rows: rows, leaves (given value, or the running maximum on entry), ancestors.
// prio, out_idx and protect point at this tree's part (or are null).
template <int LOGK>
__device__ __forceinline__ void lds_insert(const LdsTree& lt, const FieldTable& rows, uint32_t t, uint64_t dense_row0,
                                           uint32_t n, const float* prio, uint32_t* out_idx, const uint32_t* protect,
                                           uint32_t n_protect, uint32_t& cursor, uint32_t& size, uint32_t& flags) {
  const uint32_t tid = threadIdx.x;
  const uint32_t N = lt.N;
  if (protect) {   // collision-free insertion: rows aimed at a protected slot are deferred (see k_insert_small)
    if (tid < 32) lt.skip[tid] = 0;
    __syncthreads();
    for (uint32_t k = tid; k < n_protect; k += blockDim.x) {
      const uint32_t i = protect[k];
      if (i < N) {
        const uint32_t j = i >= cursor ? i - cursor : i + (N - cursor);   // position in the ring window
        if (j < n) atomicOr(&lt.skip[j >> 5], 1u << (j & 31u));
      }
    }
    __syncthreads();
  }
  (void)move_rows_one_workgroup<false>(rows, t, dense_row0, n, cursor, N, nullptr, protect ? lt.skip : nullptr);
  __syncthreads();   // (also: the tree is loaded, the operation before this one is complete)
  const float max_on_entry = __uint_as_float(*lt.max_bits);
  __syncthreads();
  bool ok = false;
  uint32_t slot = 0;
  if (tid < n) {
    uint64_t sl = (uint64_t)cursor + tid;
    if (sl >= N) sl -= N;
    slot = (uint32_t)sl;
    const bool deferred = protect && ((lt.skip[tid >> 5] >> (tid & 31u)) & 1u);
    if (out_idx) out_idx[tid] = deferred ? 0xFFFFFFFFu : slot;
    if (!deferred) {
      float v = max_on_entry;
      ok = true;
      if (prio) {
        v = prio[tid];
        ok = valid_priority(v);
        if (ok && v > 0.0f) atomicMax(lt.max_bits, __float_as_uint(v));
        if (!ok) flags |= 2u;
      }
      if (ok) (lt.leaves_mem ? lt.leaves_mem : lt.tree + lt.off[0])[slot] = v;
    }
  }
  resum_paths_lds<LOGK>(lt.tree, lt.off, lt.H, ok, slot, lt.leaves_mem);
  const uint64_t end = (uint64_t)cursor + n;
  cursor = (uint32_t)(end >= N ? end - N : end);
  size = size + n > N ? N : size + n;
}

// Priority sampling of B <= 1024 indices with importance weights, and the rows of the sampled
// indices.  u_i: this lane's uniform (lanes >= B: any value).  out_idx (never null), out_w, out_prio
// point at this tree's part.  Returns this lane's index.
template <int LOGK>
__device__ __forceinline__ uint32_t lds_sample(const LdsTree& lt, const FieldTable& rows, uint32_t t, uint64_t dense_row0,
                                               uint32_t B, float u_i, float beta, uint32_t* out_idx, float* out_w,
                                               float* out_prio, bool buffer_norm, uint32_t& flags) {
  constexpr int K = Fan<LOGK>::K;
  const uint32_t tid = threadIdx.x;
  if (tid == 0) {
    *lt.vmin_bits = kNoMin;
    *lt.bmin_bits = kNoMin;
  }
  __syncthreads();
  const float total = lt.tree[lt.off[lt.H]];
  if (buffer_norm && out_w) {   // weights relative to the whole tree: its smallest positive leaf, by a sweep over the LDS copy
    uint32_t m = kNoMin;
    const float* all_leaves = lt.leaves_mem ? lt.leaves_mem : lt.tree + lt.off[0];
    for (uint32_t e = tid; e < lt.N; e += blockDim.x) m = min_u32(m, positive_bits(all_leaves[e]));
    m = wave_min_u32(m);
    if ((tid & 63u) == 0 && m != kNoMin) atomicMin(lt.bmin_bits, m);
  }
  uint32_t node = 0xFFFFFFFFu;
  float val = 0.0f;
  if (total > 0.0f) {
    const uint32_t si = tid < B ? tid : B - 1;
    float r = ((float)si + u_i) * (total / (float)B);
    node = 0;
    val = total;
    for (uint32_t h = lt.H; h-- > 0;) {
      unsigned child;
      if (h == 0 && lt.leaves_mem) descend_lane<LOGK>(lt.leaves_mem + (size_t)node * K, r, child, val);
      else descend_lane<LOGK>(lt.tree + lt.off[h] + (size_t)node * K, r, child, val);
      node = node * K + child;
    }
    if (out_w && tid < B) atomicMin(lt.vmin_bits, __float_as_uint(val));
  } else if (tid == 0) {
    flags |= 4u;
  }
  if (tid < B) {
    lt.sampled[tid] = node;
    out_idx[tid] = node;
    if (out_prio) out_prio[tid] = val;
  }
  __syncthreads();
  // (the weights, a power per sample, are computed while the rows are on their way: every lane that
  // owns a sample also owns a row element of the first sweep, so no wave runs the power twice)
  auto weights = [&]() {
    if (out_w && tid < B)
      out_w[tid] = total > 0.0f ? importance_weight(val, __uint_as_float(buffer_norm ? *lt.bmin_bits : *lt.vmin_bits), beta)
                                : 0.0f;
  };
  if (move_rows_one_workgroup<true>(rows, t, dense_row0, B, 0, lt.N, lt.sampled, nullptr, weights)) flags |= 1u;
  return node;
}

// Priority update of B <= 1024 elements: lane tid < B sets leaf i to v.  Last writer by LDS
// atomics (see the head of this file), then the ancestors.
template <int LOGK>
__device__ __forceinline__ void lds_update(const LdsTree& lt, uint32_t B, uint32_t i, float v, uint32_t size,
                                           uint32_t& flags) {
  const uint32_t tid = threadIdx.x;
  bool valid = false;
  if (tid < B) {
    if (!(i < size)) flags |= 1u;
    else if (!valid_priority(v)) flags |= 2u;
    else valid = true;
  }
  const uint32_t mark = 0x80000001u + tid;
  bool won;
  if (lt.leaves_mem) {   // (the markers go through memory: atomics there, and a read that passes by the first-level cache)
    uint32_t* leaf_bits = reinterpret_cast<uint32_t*>(lt.leaves_mem);
    if (valid) atomicMax(&leaf_bits[i], mark);
    __syncthreads();
    won = valid && __hip_atomic_load(&leaf_bits[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == mark;
    __syncthreads();
    if (won) lt.leaves_mem[i] = v;
  } else {
    uint32_t* leaf_bits = reinterpret_cast<uint32_t*>(lt.tree + lt.off[0]);
    if (valid) atomicMax(&leaf_bits[i], mark);
    __syncthreads();
    won = valid && leaf_bits[i] == mark;
    __syncthreads();
    if (won) lt.tree[lt.off[0] + i] = v;
  }
  if (valid && v > 0.0f) atomicMax(lt.max_bits, __float_as_uint(v));
  resum_paths_lds<LOGK>(lt.tree, lt.off, lt.H, valid, i, lt.leaves_mem);
}

// Loads every height of tree t into LDS (lanes 64 .. 64 + H + 1 have filled s_off, lane 0 the maximum).  The heights
// are arrays of their own in memory and lie back to back in LDS; the copy runs over the LDS floats as one range, eight
// per lane in flight and all loads of a round before its first store, so that a tree of a dozen heights is not a dozen
// trips to memory one after the other.
__device__ __forceinline__ void lds_tree_load(const LevelTable& tab, const LdsTree& lt) {
  constexpr int R = 8;
  const uint32_t h_first = lt.leaves_mem ? 1u : 0u;
  const uint32_t begin = lt.off[h_first], end = lt.off[lt.H + 1];
  for (uint32_t base = begin; base < end; base += (uint32_t)R * blockDim.x) {
    float v[R];
    uint32_t h = h_first;   // (the height of this lane's element: found anew per round, then it only grows)
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t e = base + (uint32_t)k * blockDim.x + threadIdx.x;
      v[k] = 0.0f;
      if (e < end) {
        while (h < lt.H && e >= lt.off[h + 1]) ++h;
        v[k] = tab.lvl[h][e - lt.off[h]];
      }
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t e = base + (uint32_t)k * blockDim.x + threadIdx.x;
      if (e < end) lt.tree[e] = v[k];
    }
  }
}
// ... and back to memory, with the running maximum and the flags the lanes have collected.
__device__ __forceinline__ void lds_tree_store(const Geom& g, uint32_t t, const LevelTable& tab, const LdsTree& lt,
                                               uint32_t flags, uint32_t* s_flags) {
  for (uint32_t h = lt.leaves_mem ? 1u : 0u; h <= lt.H; ++h) {
    float* lvl = tab.lvl[h];
    const float* src = lt.tree + lt.off[h];
    for (uint32_t e = threadIdx.x; e < tab.n[h]; e += blockDim.x) lvl[e] = src[e];
  }
  if (threadIdx.x == 0) g.max_v[t] = __uint_as_float(*lt.max_bits);
  if (flags) atomicOr(s_flags, flags);
  __syncthreads();
  if (threadIdx.x == 0 && *s_flags) atomicOr(&g.status[t], *s_flags);
}

// ---- rows of the stream kernels
// The pieces (16 bytes or the field's access width) in which the rows of a step move are shared out over the lanes
// that carry rows, and which piece a lane has (field, row, place in the row) is the same in every step: it is worked
// out once per launch (a chain of selects over the fields and a division: several hundred cycles for a lone wave).
struct RowPiece {
  uint8_t* stored;    // the piece in row 0 of the tree's payload
  uint8_t* dense;     // the piece in the caller's array, step 0
  uint32_t what;      // row of the step's batch << 8 | field << 5 | bytes moved
  __device__ __forceinline__ uint32_t row() const { return what >> 8; }
  __device__ __forceinline__ uint32_t field() const { return (what >> 5) & 7u; }
  __device__ __forceinline__ uint32_t w() const { return what & 31u; }
};
// What the lanes ask of one list of fields, in LDS (the kernel arguments would take a hundred scalar registers).
struct PieceFields {
  uint8_t* io[kMaxFields];         // the caller's array: the rows of this tree in step 0
  uint8_t* col[kMaxFields];        // the field in row 0 of this tree
  uint64_t step[kMaxFields];       // bytes of the caller's array per step
  uint32_t bytes[kMaxFields], vec[kMaxFields];
  uint32_t end[kMaxFields];        // pieces of this field and all before it
};
// Called by one wave: n rows per tree and step of tree t of T.
__device__ __forceinline__ void fill_piece_fields(const FieldTable* ft, uint32_t t, uint32_t T, uint32_t n, PieceFields* pf) {
  const uint32_t f = threadIdx.x & 63u;
  if (f < (uint32_t)kMaxFields) {
    const bool on = f < ft->n_fields && ft->io[f] && n;
    const uint32_t E = ft->bytes[f];
    pf->io[f] = on ? ft->io[f] + (uint64_t)t * n * E : nullptr;
    pf->col[f] = ft->col[f] + (uint64_t)t * ft->col_stride[f];
    pf->step[f] = (uint64_t)T * n * E;
    pf->bytes[f] = E;
    pf->vec[f] = ft->vec[f];
    uint32_t end = on ? n * row_elements(E, ft->vec[f]) : 0u;
#pragma unroll
    for (int d = 1; d < kMaxFields; d <<= 1) {
      const uint32_t before = (uint32_t)__shfl_up((int)end, d);
      if (f >= (uint32_t)d) end += before;
    }
    pf->end[f] = end;
  }
}
// Piece e < pf.end[last]: fields one after the other, row after row.
__device__ __forceinline__ RowPiece find_piece(const PieceFields& pf, uint32_t e) {
  uint32_t f = 0;
#pragma unroll
  for (uint32_t k = 0; k + 1 < (uint32_t)kMaxFields; ++k) f += e >= pf.end[k] ? 1u : 0u;
  const uint32_t E = pf.bytes[f], v = pf.vec[f], el = e - (f ? pf.end[f - 1] : 0u);
  const bool wide = moves_wide(E, v);
  const uint32_t epr = row_elements(E, v), w = wide ? 16u : v;
  const uint32_t row = el / epr, k = el - row * epr;
  const uint32_t at = wide && 16u * k + 16u > E ? E - 16u : k * w;
  RowPiece p;
  p.stored = pf.col[f] + at;
  p.dense = pf.io[f] + (uint64_t)row * E + at;
  p.what = row << 8 | f << 5 | w;
  return p;
}
typedef uint32_t Words4 __attribute__((ext_vector_type(4), aligned(4)));   // (16-byte pieces of some fields lie on 4-byte boundaries)
typedef uint32_t Words2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint4 load_piece(const uint8_t* src, uint32_t w) {
  uint4 v = make_uint4(0, 0, 0, 0);
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
// Waits until this wave's loads have arrived and its stores have been acknowledged.
__device__ __forceinline__ void wait_memory() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// Orders LDS accesses of one wave (which the hardware keeps in order) for the compiler.
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The list of steps.  What bounds it is one chain of instructions and LDS trips from step to step (the tree as one
// step leaves it is what the next samples from), so everything that is not tree work is taken off that chain:
//  - The waves split: the first ones (the team, a lane per sample and per inserted row) do the tree work, the others
//    move the rows and turn values into weights, one step behind.  Batches of more than 512 leave no waves over; the
//    team then does both in turn.
//  - Inputs are fetched a step ahead.
//  - The update of step s and the insertion of step s + 1 are adjacent tree changes with nothing read in between: the
//    leaves are written one after the other and the ancestors of both recomputed in one pass.
//  - WAVE: with at most 64 samples and 64 new rows the team is one wave, whose LDS accesses stay in order by
//    themselves: no barriers inside the tree work, two per step in all.
//  - Barriers wait for LDS only.  A __syncthreads() also waits for every store of the wave to be acknowledged from
//    memory, a microsecond at each phase that writes results or rows.
// The order that memory needs: the stored rows of an insertion are read by the gather of the same step at the earliest
// (its lanes wait for their stores before the barrier that ends the sampling), and overwrite what the gather of the
// step before has read (all of whose loads have arrived at the barrier in front of the insertion's stores).
// 100 steps on 10 000 leaves at K = 16 (32 samples, 4 new rows of 41 bytes): 282 us; 1001 us as one phase after the
// other by the whole workgroup with a full barrier between them.
template <int LOGK, bool WAVE>
__global__ void __launch_bounds__(1024)
k_run_steps(StreamKernelArgs ka) {
  constexpr int K = Fan<LOGK>::K;
  constexpr int kGather = 4, kInsert = 2;   // pieces a lane holds in registers; a longer list of pieces goes on in a loop
  const Geom& g = ka.g;
  const StreamArgs& a = ka.a;
  extern __shared__ __attribute__((aligned(16))) float tree[];
  __shared__ LevelTable tab;
  __shared__ uint32_t s_off[kMaxHeight + 2];
  __shared__ uint32_t s_max, s_vmin[2], s_bmin[2], s_flags;
  __shared__ PieceFields s_rows, s_ins;
  const uint32_t t = blockIdx.x;
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint32_t H = g.H, T = g.T, B = a.B, n_ins = a.n_insert, N = g.N;
  fill_level_table(H, t, &tab);
  if (tid >= 64 && tid <= 64 + H + 1)
    s_off[tid - 64] = kernarg_at<StreamArgs>(offsetof(StreamKernelArgs, a))->off[tid - 64];
  if (tid == 0) {
    s_max = read_max_bits(g, t);
    s_vmin[0] = s_vmin[1] = s_bmin[0] = s_bmin[1] = kNoMin;
    s_flags = 0;
  }
  // lanes of the team, of the rows, of the weights
  const uint32_t team = WAVE ? 64u : ((B > n_ins ? B : n_ins) + 63u) / 64u * 64u;
  const bool apart = WAVE || team <= 512u;
  const bool in_team = tid < team, in_rows = !apart || tid >= team;
  const uint32_t rn = apart ? 1024u - team : 1024u, rl = apart ? tid - team : tid;
  const uint32_t w0 = apart ? 1024u - (B + 63u) / 64u * 64u : 0u;
  const bool weigher = tid >= w0 && tid - w0 < B;
  // (the field tables from the argument segment by vector loads, a lane per field)
  if (tid >= 128 && tid < 192) fill_piece_fields(kernarg_at<FieldTable>(offsetof(StreamKernelArgs, a) + offsetof(StreamArgs, rows)), t, T, B, &s_rows);
  if (tid >= 192 && tid < 256) fill_piece_fields(kernarg_at<FieldTable>(offsetof(StreamKernelArgs, a) + offsetof(StreamArgs, ins)), t, T, n_ins, &s_ins);
  __syncthreads();
  const uint32_t gather_pieces = s_rows.end[kMaxFields - 1], insert_pieces = s_ins.end[kMaxFields - 1];
  RowPiece gp[kGather], ip[kInsert];
  uint4 gv[kGather], iv[kInsert];
#pragma unroll
  for (int k = 0; k < kGather; ++k)
    if (in_rows && rl + k * rn < gather_pieces) gp[k] = find_piece(s_rows, rl + k * rn);
#pragma unroll
  for (int k = 0; k < kInsert; ++k)
    if (in_rows && rl + k * rn < insert_pieces) {
      ip[k] = find_piece(s_ins, rl + k * rn);
      iv[k] = load_piece(ip[k].dense, ip[k].w());
    }
  // inputs of the team: the uniform of the step to sample, value (and index) of the update to apply, inserted priority
  float u_i = 0.0f, up_v = 0.0f, in_v = 0.0f;
  uint32_t up_i = 0;
  const uint32_t j_ins = WAVE ? lane - (64u - n_ins) : tid;   // (WAVE: the last lanes of the wave, so that samples and rows share it)
  const bool inserts = in_team && (!WAVE || lane >= 64u - n_ins) && j_ins < n_ins;
  if (in_team && tid < B) u_i = a.u[(size_t)t * B + tid];
  if (inserts && a.ins_prio) in_v = a.ins_prio[(size_t)t * n_ins + j_ins];
  __syncthreads();
  LdsTree lt;
  lt.tree = tree;
  lt.leaves_mem = a.leaves_in_memory ? tab.lvl[0] : nullptr;
  lt.off = s_off;
  lt.max_bits = &s_max;
  lt.vmin_bits = lt.bmin_bits = nullptr;
  lt.skip = nullptr;
  lt.sampled = nullptr;
  lt.H = H;
  lt.N = N;
  lds_tree_load(tab, lt);
  uint32_t* nodes = reinterpret_cast<uint32_t*>(tree + s_off[H + 1]);   // [B] sampled leaves of the step
  float* values = reinterpret_cast<float*>(nodes + 512);                // [B] and their values (apart only: B <= 512)
  const bool mem = lt.leaves_mem != nullptr;
  float* leaves = mem ? lt.leaves_mem : tree;                           // (height 0 starts at LDS offset 0)
  const uint32_t off_reg = s_off[lane <= H + 1 ? lane : H + 1];         // offsets from lane registers: an LDS trip less per height
  auto off = [&](uint32_t h) -> uint32_t { return (uint32_t)__builtin_amdgcn_readlane((int)off_reg, (int)h); };
  uint32_t cursor = a.cursor, size = a.size, upd_size = 0;
  uint32_t flags = 0;
  __syncthreads();
  uint32_t max_bits = s_max;      // (WAVE: the team's copy; else s_max counts)
  uint32_t node = 0xFFFFFFFFu;    // this lane's sample of the step before
  float val = 0.0f;
  // barrier between phases of the tree work
  auto sync = [&]() {
    if (mem) wait_memory();
    lds_barrier();
  };
  auto leaf_group_sum = [&](uint32_t h, uint32_t parent) -> float {
    return h == 1 && mem ? lane_group_sum<LOGK>(lt.leaves_mem + (size_t)parent * K)
                         : lane_group_sum<LOGK>(tree + off(h - 1) + (size_t)parent * K);
  };

  for (uint32_t s = 0;; ++s) {
    const bool more = s < a.n_steps;
    // ---- rows and weights of the step before: loads
    float w_out = 0.0f, v_out = 0.0f;
    uint32_t n_out = 0;
    if (s) {
      if (in_rows) {
#pragma unroll
        for (int k = 0; k < kGather; ++k)
          if (rl + k * rn < gather_pieces) {
            const uint32_t slot = nodes[gp[k].row()];
            const bool ok = slot < N;
            if (!ok) flags |= 1u;
            gv[k] = load_piece(gp[k].stored + (uint64_t)(ok ? slot : 0u) * a.rows.row_stride, gp[k].w());
            if (!ok) gv[k] = make_uint4(0, 0, 0, 0);
          }
        for (uint32_t e = rl + kGather * rn; e < gather_pieces; e += rn) {
          const RowPiece p = find_piece(s_rows, e);
          const uint32_t slot = nodes[p.row()];
          const bool ok = slot < N;
          if (!ok) flags |= 1u;
          uint4 v = load_piece(p.stored + (uint64_t)(ok ? slot : 0u) * a.rows.row_stride, p.w());
          if (!ok) v = make_uint4(0, 0, 0, 0);
          store_piece(p.dense + (uint64_t)(s - 1) * s_rows.step[p.field()], p.w(), v);
        }
      }
      if (weigher) {
        n_out = nodes[tid - w0];
        v_out = apart ? values[tid - w0] : val;
        if (a.out_w) {
          const uint32_t vmin = s_vmin[(s - 1) & 1u];
          const uint32_t least = a.buffer_norm ? s_bmin[(s - 1) & 1u] : vmin;
          w_out = vmin == kNoMin ? 0.0f : importance_weight(v_out, __uint_as_float(least), a.beta[s - 1]);
        }
      }
    }
    // ---- the tree: update of the step before, insertion of this one
    const bool do_upd = s > 0 && a.upd_prio != nullptr, do_ins = more && n_ins > 0;
    if (!WAVE || tid < 64u) {
      const uint32_t ui = a.upd_is_sampled ? node : up_i;
      bool valid = false, placed = false;
      uint32_t slot = 0;
      if (do_upd) {
        const bool mine = in_team && tid < B;
        if (mine) {
          if (!(ui < upd_size)) flags |= 1u;
          else if (!valid_priority(up_v)) flags |= 2u;
          else valid = true;
        }
        const uint32_t mx = valid && up_v > 0.0f ? __float_as_uint(up_v) : 0u;
        bool won = valid;
        const uint32_t mark = 0x80000001u + tid;
        uint32_t* bits = reinterpret_cast<uint32_t*>(leaves);
        if (WAVE && a.upd_is_sampled && !__any(mine && !valid)) {
          // (samples come out in leaf order: elements of one leaf are neighbours, and the last of them wins)
          const uint32_t next = (uint32_t)__shfl_down((int)ui, 1);
          won = valid && (tid + 1 >= B || next != ui);
        } else if (mem) {   // (markers in memory: atomics there, and a read that passes by the first-level cache)
          if (valid) atomicMax(&bits[ui], mark);
          if constexpr (WAVE) wait_memory(); else sync();
          won = valid && __hip_atomic_load(&bits[ui], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == mark;
          if constexpr (WAVE) wait_memory(); else sync();
        } else {
          if (valid) atomicMax(&bits[ui], mark);
          if constexpr (WAVE) wave_order(); else sync();
          won = valid && bits[ui] == mark;
          if constexpr (WAVE) wave_order(); else sync();
        }
        if (won) leaves[ui] = up_v;
        if constexpr (WAVE) {
          const uint32_t m = wave_max_u32(mx);
          max_bits = m > max_bits ? m : max_bits;
          wave_order();
        } else {
          if (mx) atomicMax(&s_max, mx);
          sync();
        }
      }
      if (do_ins) {
        uint32_t mx = 0;
        if (inserts) {
          slot = ring_slot(cursor, j_ins, N);
          float v = __uint_as_float(WAVE ? max_bits : s_max);
          placed = true;
          if (a.ins_prio) {
            v = in_v;
            placed = valid_priority(v);
            if (!placed) flags |= 2u;
            mx = placed && v > 0.0f ? __float_as_uint(v) : 0u;
          }
          if (placed) leaves[slot] = v;
        }
        if (a.ins_prio) {
          if constexpr (WAVE) {
            const uint32_t m = wave_max_u32(mx);
            max_bits = m > max_bits ? m : max_bits;
          } else if (mx) {
            atomicMax(&s_max, mx);
          }
        }
      }
      // ancestors of both (elements that share a parent store the same sum)
      if (do_upd || do_ins) {
        if constexpr (WAVE) {
          const bool together = !do_upd || !do_ins || B + n_ins <= 64u;
          for (int pass = 0; pass < (together ? 1 : 2); ++pass) {
            const bool act = together ? valid || placed : pass == 0 ? valid : placed;
            const uint32_t leaf = together ? (placed ? slot : ui) : pass == 0 ? ui : slot;
            for (uint32_t h = 1; h <= H; ++h) {
              wave_order();
              if (act) {
                const uint32_t parent = leaf >> (h * LOGK);
                tree[off(h) + parent] = leaf_group_sum(h, parent);
              }
            }
          }
          wave_order();
        } else {
          for (uint32_t h = 1; h <= H; ++h) {
            sync();
            const uint32_t pu = ui >> (h * LOGK), pi = slot >> (h * LOGK);
            if (valid) tree[off(h) + pu] = leaf_group_sum(h, pu);
            if (placed) tree[off(h) + pi] = leaf_group_sum(h, pi);
          }
        }
      }
      // inputs of the next round
      if (in_team && tid < B) {
        const size_t bo = ((size_t)s * T + t) * B + tid;
        if (more && a.upd_prio) {
          up_v = a.upd_prio[bo];
          if (!a.upd_is_sampled) up_i = a.upd_idx[bo];
        }
      }
    }
    if (do_ins) {
      cursor = ring_slot(cursor, n_ins, N);
      size = size + n_ins > N ? N : size + n_ins;
    }
    upd_size = size;
    // ---- all loads of stored rows have arrived; the tree is whole
    if (in_rows || (mem && (!WAVE || a.buffer_norm))) wait_memory();
    lds_barrier();
    if (do_ins && in_rows) {
      const uint32_t first = cursor >= n_ins ? cursor - n_ins : cursor + (N - n_ins);
#pragma unroll
      for (int k = 0; k < kInsert; ++k)
        if (rl + k * rn < insert_pieces)
          store_piece(ip[k].stored + (uint64_t)ring_slot(first, ip[k].row(), N) * a.ins.row_stride, ip[k].w(), iv[k]);
      for (uint32_t e = rl + kInsert * rn; e < insert_pieces; e += rn) {
        const RowPiece p = find_piece(s_ins, e);
        store_piece(p.stored + (uint64_t)ring_slot(first, p.row(), N) * a.ins.row_stride, p.w(),
                    load_piece(p.dense + (uint64_t)s * s_ins.step[p.field()], p.w()));
      }
      wait_memory();
    }
    if (s) {
      if (in_rows) {
#pragma unroll
        for (int k = 0; k < kGather; ++k)
          if (rl + k * rn < gather_pieces) store_piece(gp[k].dense + (uint64_t)(s - 1) * s_rows.step[gp[k].field()], gp[k].w(), gv[k]);
      }
      if (weigher) {
        const size_t o = ((size_t)(s - 1) * T + t) * B + (tid - w0);
        a.out_idx[o] = n_out;
        if (a.out_prio) a.out_prio[o] = v_out;
        if (a.out_w) a.out_w[o] = w_out;
      }
    }
    if (!more) break;
    if (s + 1 < a.n_steps && n_ins) {
      if (in_rows) {
#pragma unroll
        for (int k = 0; k < kInsert; ++k)
          if (rl + k * rn < insert_pieces) iv[k] = load_piece(ip[k].dense + (uint64_t)(s + 1) * s_ins.step[ip[k].field()], ip[k].w());
      }
      if (inserts && a.ins_prio) in_v = a.ins_prio[((size_t)(s + 1) * T + t) * n_ins + j_ins];
    }
    if (tid == 0) s_vmin[(s + 1) & 1u] = s_bmin[(s + 1) & 1u] = kNoMin;   // (read by the weights of step s - 1, before the barrier)
    // ---- weights relative to the whole tree: its smallest positive leaf
    if (a.buffer_norm && a.out_w && in_rows) {
      uint32_t m = kNoMin;
      for (uint32_t e = rl; e < N; e += rn) m = min_u32(m, positive_bits(leaves[e]));
      m = wave_min_u32(m);
      if (lane == 0 && m != kNoMin) atomicMin(&s_bmin[s & 1u], m);
    }
    // ---- sampling
    if (in_team) {
      const float total = tree[off(H)];
      node = 0xFFFFFFFFu;
      val = 0.0f;
      if (total > 0.0f) {
        const uint32_t si = tid < B ? tid : B - 1;
        float r = ((float)si + u_i) * (total / (float)B);
        node = 0;
        val = total;
        for (uint32_t h = H; h-- > 0;) {
          unsigned child;
          if (h == 0 && mem) descend_lane<LOGK>(lt.leaves_mem + (size_t)node * K, r, child, val);
          else descend_lane<LOGK>(tree + off(h) + (size_t)node * K, r, child, val);
          node = node * K + child;
        }
        if (a.out_w) {
          const uint32_t m = wave_min_u32(tid < B ? __float_as_uint(val) : kNoMin);
          if (lane == 0) {
            if constexpr (WAVE) s_vmin[s & 1u] = m;
            else atomicMin(&s_vmin[s & 1u], m);
          }
        }
      } else if (tid == 0) {
        flags |= 4u;
      }
      if (tid < B) {
        nodes[tid] = node;
        if (apart) values[tid] = val;
      }
      if (tid < B && s + 1 < a.n_steps) u_i = a.u[((size_t)(s + 1) * T + t) * B + tid];
    }
    lds_barrier();
  }
  if (WAVE && tid == 0) s_max = max_bits;
  __syncthreads();
  lds_tree_store(g, t, tab, lt, flags, &s_flags);
}

// ---------------------------------------------------------------------------------
// a queue of op-coded requests on an LDS-resident tree
// ---------------------------------------------------------------------------------
// The same workgroup-per-tree arrangement, driven by a queue of requests in memory instead of a
// fixed step: each request names its operation (the paper's unified operation code, Section V-A)
// and is decoded when its turn comes.  The queue's length is fixed at launch; the kernel ends after
// its last request.
struct QueueKernelArgs {            // one kernel argument (Geom first: see fill_level_table)
  Geom g;
  QueueArgs a;
};

template <int LOGK>
__global__ void __launch_bounds__(1024)
k_run_requests(QueueKernelArgs ka) {
  const Geom& g = ka.g;
  const QueueArgs& a = ka.a;
  extern __shared__ __attribute__((aligned(16))) float tree[];
  __shared__ LevelTable tab;
  __shared__ FieldTable s_ft;        // the buffer's columns with the current request's row arrays
  __shared__ uint32_t s_off[kMaxHeight + 2];
  __shared__ uint32_t s_skip[32];
  __shared__ uint32_t s_max, s_vmin, s_bmin, s_flags;
  const uint32_t t = blockIdx.x;
  const uint32_t tid = threadIdx.x;
  const uint32_t H = g.H;
  fill_level_table(H, t, &tab);
  if (tid >= 64 && tid <= 64 + H + 1)
    s_off[tid - 64] = kernarg_at<QueueArgs>(offsetof(QueueKernelArgs, a))->off[tid - 64];
  if (tid == 0) {
    s_max = read_max_bits(g, t);
    s_flags = 0;
    s_ft = a.fields;
  }
  __syncthreads();
  LdsTree lt;
  lt.tree = tree;
  lt.leaves_mem = a.leaves_in_memory ? tab.lvl[0] : nullptr;
  lt.off = s_off;
  lt.sampled = reinterpret_cast<uint32_t*>(tree + s_off[H + 1]);
  lt.max_bits = &s_max;
  lt.vmin_bits = &s_vmin;
  lt.bmin_bits = &s_bmin;
  lt.skip = s_skip;
  lt.H = H;
  lt.N = g.N;
  lds_tree_load(tab, lt);
  uint32_t cursor = a.cursor, size = a.size;
  uint32_t flags = 0;
  uint32_t last_node = 0xFFFFFFFFu;   // this lane's index from the latest sampling request

  for (uint32_t r = 0; r < a.n_requests; ++r) {
    const per_request& q = a.queue[r];
    const uint32_t n = q.n;
    const size_t to = (size_t)t * n;
    __syncthreads();   // the request before this one is complete (and has finished with s_ft)
    if (tid < (uint32_t)kMaxFields) s_ft.io[tid] = static_cast<uint8_t*>(q.field[tid]);
    __syncthreads();
    if (q.op == PER_OP_INSERT) {
      lds_insert<LOGK>(lt, s_ft, t, to, n, q.prio ? q.prio + to : nullptr, q.idx ? q.idx + to : nullptr,
                       q.protect ? q.protect + (size_t)t * q.n_protect : nullptr, q.n_protect, cursor, size, flags);
    } else if (q.op == PER_OP_SAMPLE) {
      const float u_i = tid < n ? q.u[to + tid] : 0.0f;
      last_node = lds_sample<LOGK>(lt, s_ft, t, to, n, u_i, q.beta, q.idx + to, q.out_weight ? q.out_weight + to : nullptr,
                                   q.out_prio ? q.out_prio + to : nullptr, a.buffer_norm != 0, flags);
    } else if (q.op == PER_OP_UPDATE) {
      float v = 0.0f;
      uint32_t i = last_node;
      if (tid < n) {
        v = q.prio[to + tid];
        if (q.idx) i = q.idx[to + tid];
      }
      lds_update<LOGK>(lt, n, i, v, size, flags);
    }
  }
  __syncthreads();
  lds_tree_store(g, t, tab, lt, flags, &s_flags);
}

// LDS floats of a tree's copy (every height padded to whole child groups), or 0 if it cannot be held beside the step
// kernel's other LDS data.  The whole tree if that fits; else the heights 1 .. H, the leaves staying in memory
// (*leaves_in_memory says which).
constexpr uint32_t kStreamLdsBytes = 156 * 1024;
uint32_t stream_tree_floats(const Geom& g, uint32_t* off, uint32_t* leaves_in_memory) {
  for (uint32_t skip = 0; skip < 2; ++skip) {
    uint64_t floats = 0;
    bool fits = true;
    for (uint32_t h = 0; h <= g.H && fits; ++h) {
      if (off) off[h] = (uint32_t)floats;
      if (h == 0 && skip) continue;
      floats += h < g.H ? ((uint64_t)g.n[h] + g.K - 1) / g.K * g.K : 4;   // (the root padded to 16 bytes)
      fits = floats * 4 <= kStreamLdsBytes;
    }
    if (!fits || (floats + 1024) * 4 > kStreamLdsBytes || (skip && g.H < 2)) continue;
    if (off) off[g.H + 1] = (uint32_t)floats;
    if (leaves_in_memory) *leaves_in_memory = skip;
    return (uint32_t)floats;
  }
  return 0u;
}

template <int LOGK>
static hipError_t launch_run_steps_k(const Geom& g, const Tuning& tn, StreamArgs a, hipStream_t s) {
  StreamKernelArgs ka{};
  ka.g = g;
  ka.a = a;
  const uint32_t floats = stream_tree_floats(g, ka.a.off, &ka.a.leaves_in_memory);
  if (!floats) return hipErrorInvalidValue;
  const size_t bytes = ((size_t)floats + 1024) * 4;   // the tree and the sampled indices of one step
  // always the largest workgroup, also for small batches: measured faster than a workgroup of the batch's
  // size (the tree copy and the row movers use all lanes)
  if (a.B <= 64 && a.n_insert <= 64) {
    hipError_t e = grant_lds<&k_run_steps<LOGK, true>>(tn, bytes);
    if (e != hipSuccess) return e;
    PER_LAUNCH(KID_RUN_STEPS, (k_run_steps<LOGK, true>), dim3(g.T), dim3(1024), bytes, s, ka);
  } else {
    hipError_t e = grant_lds<&k_run_steps<LOGK, false>>(tn, bytes);
    if (e != hipSuccess) return e;
    PER_LAUNCH(KID_RUN_STEPS, (k_run_steps<LOGK, false>), dim3(g.T), dim3(1024), bytes, s, ka);
  }
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
  const uint32_t floats = stream_tree_floats(g, ka.a.off, &ka.a.leaves_in_memory);
  if (!floats) return hipErrorInvalidValue;
  const size_t bytes = ((size_t)floats + 1024) * 4;   // the tree and the indices of the latest sampling request
  hipError_t e = grant_lds<&k_run_requests<LOGK>>(tn, bytes);
  if (e != hipSuccess) return e;
  PER_LAUNCH(KID_RUN_REQUESTS, k_run_requests<LOGK>, dim3(g.T), dim3(1024), bytes, s, ka);
  return hipGetLastError();
}

hipError_t launch_run_requests(const Geom& g, const Tuning& tn, const QueueArgs& a, hipStream_t s) {
#define CALL(L) launch_run_requests_k<L>(g, tn, a, s)
  PER_DISPATCH_LOGK(g.logK, CALL)
#undef CALL
}

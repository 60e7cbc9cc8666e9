// Priority sampling (with the claim phase and the uniforms it can carry), importance weights, and the launcher of the fused sampling calls.
// Part of per_kernels.hip (included inside namespace per, in the order given there); not a stand-alone header.

// ---------------------------------------------------------------------------------
// priority sampling
// ---------------------------------------------------------------------------------
// The topmost heights below the root are copied to LDS (at most kTopSlots of them, highest
// first).  Their descriptors sit at fixed kernel-argument offsets, so the kernel fetches all of
// them with one batch of scalar loads instead of a chain of dependent ones.
constexpr int kTopSlots = 4;
struct TopCopy {
  const float* ptr[kTopSlots];     // that height of tree 0
  uint32_t stride[kTopSlots];      // floats between trees
  uint32_t cnt[kTopSlots];         // floats copied: whole child groups, n[l+1] * K
  uint32_t nreal[kTopSlots];       // real nodes n[l]
  uint32_t nslots;
  const float* root;               // root of tree 0
  uint32_t root_stride;
};

// One lane per sample; grid (ceil(B / block), T).  Dynamic LDS holds the top copy followed by
// one staging area per wave.  Below the copy each level costs one trip to memory: the wave
// fetches its 64 child groups with fully coalesced 16-byte loads (K/4 adjacent lanes per
// group), parks them in LDS rows (see StageRow) and every lane then walks the row of its group.
//
// Uniform of sample i of tree t when the caller supplies none ("uniformly generated random",
// Section II-A): Philox4x32-10 (Salmon et al., SC 2011), ten rounds of two 32x32->64
// multiplications on the counter (i, call low, call high, t) with the key (seed low, seed high)
// bumped by Weyl constants between rounds; first output word, top 24 bits, scaled by 2^-24.
__device__ __forceinline__ float counter_uniform(const RngArgs& rng, uint32_t i, uint32_t t) {
  uint32_t c0 = i, c1 = rng.call_lo, c2 = rng.call_hi, c3 = t;
  uint32_t k0 = rng.seed_lo, k1 = rng.seed_hi;
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    if (round > 0) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
    c0 = hi1 ^ c1 ^ k0;
    c1 = lo1;
    c2 = hi0 ^ c3 ^ k1;
    c3 = lo0;
  }
  return (float)(c0 >> 8) * (1.0f / 16777216.0f);
}

// Chunk (IT*64 + lane) of the wave's 64*C 16-byte chunks, for IT = 0 .. C-1: fetched from the group of the lane that owns
// it and parked in that lane's staging row.  Written as a recursion over IT so that every fetch is issued before the first
// LDS store without the compiler having to promote an array.
template <int LOGK, int IT>
__device__ __forceinline__ void stage_group_per_lane(const float* __restrict__ lvl, uint32_t node, unsigned lane, float* stage) {
  constexpr int K = Fan<LOGK>::K;
  constexpr int C = K / 4;
  constexpr int ROW = K + 4;
  if constexpr (IT < C) {
    const unsigned gch = (unsigned)IT * 64u + lane;
    const uint32_t nd = (uint32_t)__shfl((int)node, (int)(gch / C));
    const float4 x = *reinterpret_cast<const float4*>(lvl + (size_t)nd * K + (gch % C) * 4u);
    stage_group_per_lane<LOGK, IT + 1>(lvl, node, lane, stage);
    *reinterpret_cast<float4*>(stage + (gch / C) * ROW + (gch % C) * 4u) = x;
  }
}

// The same for large batches (the kernel that loops over blocks of samples).  Samples come in leaf order, so lanes that
// stand on one node are neighbours: each distinct group is fetched once, into the row of its rank among the wave's groups,
// and all its lanes walk that row.  (A large batch is bound by what the walk reads and computes per sample, not by the
// tree's bytes: 2^20 samples on 2^24 leaves at K = 32 fetched 128 bytes per sample and height, 400 MB between caches and
// compute units for 60 MB of distinct groups.  Few samples seldom share a group, and the ranks cost the lone wave 0.7 us of
// its chain.)  Beside the K children a row holds the sums of its chunks (4 adjacent children), which the lane that fetches a
// chunk computes once for all lanes of the group, and the number of its node:
//   [K children][K / 4 chunk sums][node] pad
// rows an odd number of 16-byte units apart, so that lanes on different rows read different banks.
// A wave has fewer rows than lanes (ROWS: 5.4 KB at K = 16, 5.6 at 32, 8.1 at 64; at K = 8 all 64 are 3.1) and takes its groups in rounds of as many: a sample in sixteen leaves
// or more, as large batches have it, seldom needs a second round, and the waves wait for memory two thirds of their time
// (counters: 63 % at three waves per SIMD with 64 rows each, 11 KB at K = 32), which more of them fill.  In workgroups of four
// waves, so that no more of them copy the top than before: 2^20 samples on 2^24 leaves 28.2 -> 25.6 us at K = 32 (33 in
// workgroups of two), with the `update` behind them 172 -> 148 at K = 64, 142 -> 138 at K = 16, 166 -> 159 at K = 8.
template <int LOGK, bool FEW = true>
struct StageRow {
  static constexpr int K = 1 << LOGK, C = K / 4;
  static constexpr int UNITS = (K + C + 1 + 3) / 4;
  static constexpr int FLOATS = 4 * (UNITS | 1);
  static constexpr int SUMS = K, NODE = K + C;
  static constexpr int ROWS = !FEW || LOGK <= 3 ? 64 : LOGK == 4 ? 48 : LOGK == 5 ? 32 : 24;   // staged at a time
  static constexpr int FETCHES = (ROWS * C + 63) / 64;                                         // 16-byte loads of a lane for them
};
template <int LOGK>
static uint32_t stage_floats_k(bool few) {   // per wave
  return few ? StageRow<LOGK, true>::ROWS * StageRow<LOGK, true>::FLOATS : StageRow<LOGK, false>::ROWS * StageRow<LOGK, false>::FLOATS;
}
static uint32_t stage_floats(uint32_t logK, bool few) {
  return logK == 3 ? stage_floats_k<3>(few) : logK == 4 ? stage_floats_k<4>(few) : logK == 5 ? stage_floats_k<5>(few) : logK == 6 ? stage_floats_k<6>(few) : 0u;
}
// Few rows: where 64 samples, spread evenly over the leaves, lie in no more groups than seven eighths of them.  (K = 32, `sample` and
// `update`: 2^18 samples on 2^24 leaves 51.9 us with 64 rows, 53.7 with 32; 2^20 samples 141 and 138.  Other fanouts, 64 rows and few,
// groups 0.85 and 0.95 of the rows: K = 16 on 2^24 leaves 77.9 and 72.6, 66.7 and 62.4, on 2^22 31.7 and 31.6, 29.6 and 29.5, but where
// less is staged 1 % the other way, 2^20 leaves at 0.6 22.4 and 22.7; K = 64 on 2^24 83.8 and 64.8, 79.2 and 61.8, on 2^22 31.0 and 30.2,
// 30.3 and 29.2: there the line could lie higher.)
static bool few_rows(const Geom& g, uint32_t B) {
  const double groups = 64.0 * (double)g.N / ((double)B * (double)g.K);
  const int rows = g.logK == 4 ? StageRow<4>::ROWS : g.logK == 5 ? StageRow<5>::ROWS : g.logK == 6 ? StageRow<6>::ROWS : 64;
  return g.logK <= 3 || groups * (1.0 - exp(-64.0 / groups)) <= 0.875 * rows;
}
enum SampleLoop { LOOP_NONE, LOOP_FEW_ROWS, LOOP_ALL_ROWS };   // (see k_sample)
// Chunk (IT*64 + lane) of the wave's `chunks` 16-byte chunks, for IT = 0 .. C-1: first the numbers of all their nodes,
// then every fetch, then the LDS stores.  Written as recursions over IT (not loops over arrays of registers) so that each
// phase is under way as a whole before the next one waits, without the compiler having to promote an array.
template <int C>
struct NodeNumbers {
  uint32_t nd;
  NodeNumbers<C - 1> rest;
};
template <>
struct NodeNumbers<0> {};
template <int LOGK, int IT, int C>
__device__ __forceinline__ void read_nodes(const float* stage, unsigned lane, NodeNumbers<C>& n) {
  using Row = StageRow<LOGK>;
  if constexpr (C > 0) {
    n.nd = __float_as_uint(stage[(size_t)(((unsigned)IT * 64u + lane) / Row::C) * Row::FLOATS + Row::NODE]);
    read_nodes<LOGK, IT + 1>(stage, lane, n.rest);
  }
}
template <int LOGK, int IT, int C>
__device__ __forceinline__ void stage_chunks(const float* __restrict__ lvl, uint32_t chunks, unsigned lane, float* stage, NodeNumbers<C>& n) {
  constexpr int K = Fan<LOGK>::K;
  using Row = StageRow<LOGK>;
  if constexpr (C > 0) {
    if ((uint32_t)IT * 64u < chunks) {   // (the same for the wave)
      const unsigned gch = (unsigned)IT * 64u + lane, c = gch % Row::C;
      const bool mine = gch < chunks;
      const float4 x = *reinterpret_cast<const float4*>(lvl + (size_t)(mine ? n.nd : 0u) * K + c * 4u);
      stage_chunks<LOGK, IT + 1>(lvl, chunks, lane, stage, n.rest);
      if (mine) {
        float* row = stage + (size_t)(gch / Row::C) * Row::FLOATS;
        *reinterpret_cast<float4*>(row + c * 4u) = x;
        row[Row::SUMS + c] = (x.x + x.y) + (x.z + x.w);
      }
    }
  }
}
__device__ __forceinline__ void order_within_wave() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// descend_lane on a staged row: the walk over the chunks from their sums, then the chosen chunk.
template <int LOGK>
__device__ __forceinline__ void descend_row(const float* row, float& r, unsigned& child, float& val) {
  using Row = StageRow<LOGK>;
  float s[Row::C];
  if constexpr (Row::C == 2) {
    const Floats2 x = load_floats2(row + Row::SUMS);
    s[0] = x.x;
    s[1] = x.y;
  } else {
#pragma unroll
    for (int c = 0; c < Row::C; c += 4) {
      const Floats4 x = load_floats4(row + Row::SUMS + c);
      s[c] = x.x;
      s[c + 1] = x.y;
      s[c + 2] = x.z;
      s[c + 3] = x.w;
    }
  }
  const float r0 = r;
  uint32_t at = 0;
  turn_down<Row::C>(s, r, at, val);
  const Floats4 x = load_floats4(row + 4 * at);
  const float c[4] = {x.x, x.y, x.z, x.w};
  turn_down<4>(c, r, at, val);
  child = at;
  if (__builtin_expect(__any(!(val > 0.0f)), 0)) {   // (see descend_lane)
    r = r0;
    descend_chunk<LOGK>(row, s, r, child, val);
  }
}

// One height of the walk: the wave's distinct groups are staged, at most ROWS of them at a time, and every lane walks the row
// of its group.
template <int LOGK, bool FEW>
__device__ __forceinline__ void descend_staged(const float* __restrict__ lvl, uint32_t node, unsigned lane, float* stage, float& r, unsigned& child, float& val) {
  using Row = StageRow<LOGK, FEW>;
  const uint32_t below = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)node, 0x138 /* wave_shr:1: from the lane below */, 0xF, 0xF, true);
  const bool first = lane == 0 || below != node;
  const unsigned long long firsts = __ballot(first);
  const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(firsts >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)firsts, 0u)) + (first ? 1u : 0u) - 1u;
  const uint32_t groups = (uint32_t)__popcll(firsts);
  for (uint32_t base = 0; base < groups; base += Row::ROWS) {   // (one round where samples lie densely)
    const bool mine = rank - base < (uint32_t)Row::ROWS;        // (ranks below base wrap)
    float* row = stage + (size_t)(mine ? rank - base : 0u) * Row::FLOATS;
    if (mine && first) row[Row::NODE] = __uint_as_float(node);
    order_within_wave();
    NodeNumbers<Row::FETCHES> nodes;
    read_nodes<LOGK, 0>(stage, lane, nodes);
    stage_chunks<LOGK, 0>(lvl, min_u32(groups - base, (uint32_t)Row::ROWS) * Row::C, lane, stage, nodes);
    order_within_wave();
    if (mine) descend_row<LOGK>(row, r, child, val);
    order_within_wave();
  }
}

// stale < 0: the tree in memory is whole.  stale >= 0: the last update left the root and the
// `stale` topmost copied heights to this kernel; they are rebuilt here from the highest fresh
// height (which is in the copy), and the first workgroup of each tree stores them back.
//
// The claim phase of a priority update fused into the call can ride along (it touches stamps, dirty
// bits and the running maximum only, none of which sampling reads).  claim_mode 1: the update targets
// exactly the indices sampled here, element by element, so every lane claims its own sample when it has
// it.  claim_mode 2: the update batch lies in other memory; the first claim_blocks workgroups of the
// grid are claim workgroups.  claim_mode 0: no claim here.
//
// RIDE: the kernel carries the insertion that precedes the sampling call (a few rows at ring slots cursor ..).
// Every sampling workgroup works the insertion out for itself: beside the top copy it fetches the child groups
// of all touched nodes of heights 1 .. hp (hp: the height the stale top is rebuilt from) and the new priorities
// of the leaves among them, sums the groups height by height, patches the sums into the top copy and rebuilds
// the top from there; on its way down through memory a lane that comes to a touched group reads the patched
// copy instead.  One more workgroup per tree, the last of the grid, does the same sums and stores them and the
// new leaves, and moves the rows (nothing here reads rows).  Its stores race with the other workgroups' loads
// of the same words, harmlessly: every word it writes is one that every reader replaces by the very value being
// written, so a reader gets the same result from the old word and from the new one.  The running maximum must
// not move while this kernel reads it as the inserted priority, so whatever would raise it here (claim lanes,
// given insert priorities) raises max_pend instead, which the tree pass of the call folds in.
// A single wave's chain of instructions is what a small batch waits for, so the patch is planned on the host
// down to LDS offsets, and the kernel's share is kept short.
struct NoRide { uint32_t none; };
// position of node among the touched nodes of its height (the two ranges back to back)
__device__ __forceinline__ uint32_t plan_pos(const Range2& r, uint32_t node) {
  return node >= r.a0 && node < r.b0 ? node - r.a0 : (r.b0 - r.a0) + (node - r.a1);
}
template <bool RIDE> using RideParam = typename std::conditional<RIDE, InsertRide, NoRide>::type;
__device__ __forceinline__ void ride_rows(const InsertRide& ride, uint32_t t, uint32_t N, uint32_t part, uint32_t parts);   // (k_rows.h)

// LOOP: fewer sampling workgroups than blocks of samples; each takes blocks in turn.
template <int LOGK, bool RIDE, int LOOP>
__global__ void __launch_bounds__(1024)
k_sample(Geom g, TopCopy tc, uint32_t B, uint32_t size, float beta, const float* __restrict__ u,
         uint32_t* __restrict__ out_idx, float* __restrict__ out_prio, float* __restrict__ out_w,
         uint32_t weight_mode, int stale, uint32_t claim_blocks, ClaimArgs c, int claim_mode, RngArgs rng,
         RideParam<RIDE> ride) {
  constexpr int K = Fan<LOGK>::K;
  constexpr int LPS = Fan<LOGK>::LPS;
  constexpr int ROW = LOOP && LOGK >= 3 ? StageRow<LOGK>::FLOATS : K + 4;   // staging row, floats
  constexpr int ROWS = LOOP && LOGK >= 3 ? StageRow<LOGK, LOOP == LOOP_FEW_ROWS>::ROWS : 64;   // of a wave
  using Vec = typename std::conditional<LOGK == 1, float2, float4>::type;
  constexpr int VF = sizeof(Vec) / 4;
  // (lines 1, 3, 6, 7, 10, 11 of the geometry hold what this kernel does not read on trees of few heights: the upper
  // ends of the per-height arrays, the arrival counters, the one-kernel step's words)
  touch_kernel_arguments<kernarg_lines<Geom, TopCopy, uint32_t, uint32_t, float, const float*, uint32_t*, float*, float*, uint32_t,
                                       int, uint32_t, ClaimArgs, int, RngArgs,
                                       typename std::conditional<RIDE, InsertRideHead, NoRide>::type>(),
                         LOGK >= 3 ? 0xCCAu : 0u>();
  extern __shared__ __attribute__((aligned(16))) float lds[];   // 16-byte LDS accesses need the alignment
  __shared__ uint32_t s_min[16];
  __shared__ float s_total;
  const uint32_t t = blockIdx.y;
  const uint32_t H = g.H;
  const unsigned lane = threadIdx.x & 63u;
  const unsigned wave = threadIdx.x >> 6;
  const int nslots = (int)tc.nslots;
  if (blockIdx.x < claim_blocks) {   // claim workgroups come first: their atomics are under way before the descent loads start
    claim_job(g, t, c, blockIdx.x, claim_blocks);
    return;
  }
  uint32_t front = claim_blocks;
  if constexpr (!RIDE) {
    if (weight_mode & kWeightMinHere) {   // then the workgroups of the whole tree's minimum
      const uint32_t parts = weight_mode >> kWeightPartsShift;
      if (blockIdx.x - front < parts) {
        min_job(g, t, blockIdx.x - front, parts);
        return;
      }
      front += parts;
    }
  }
  bool is_mover = false;
  uint32_t movers = 0;
  if constexpr (RIDE) {   // the last workgroups move the rows; the first of them also stores what the insertion changes in the tree
    movers = ride.movers;
    const uint32_t first_mover = gridDim.x - movers;
    if (blockIdx.x > first_mover) {
      ride_rows(ride, t, g.N, blockIdx.x - first_mover, movers);
      return;
    }
    is_mover = blockIdx.x == first_mover;
  }
  const uint32_t bx = blockIdx.x - front;                   // sampling workgroup number
  const uint32_t sample_blocks = gridDim.x - front - movers;
  const bool weights_here = sample_blocks == 1 && (RIDE || !(weight_mode & kWeightMinHere));   // (else the weights job of the kernel behind turns the values into weights)

  PER_TRACE_DECL;
  PER_MARK(0);
  // (a lane's samples: a block of them per round of the sampling workgroups; most launches have a workgroup per block)
  uint32_t s_raw = bx * blockDim.x + threadIdx.x;
  bool active = s_raw < B;
  uint32_t s = active ? s_raw : B - 1;
  size_t o = (size_t)t * B + s;
  // the root, this lane's uniform and the top copy are all fetched in the same trip
  float total = tc.root[(size_t)t * tc.root_stride];
  float u_s = rng.on ? counter_uniform(rng, s, t) : u[o];
  // which buffer of partial batch minima this call fills (stable while this kernel runs: the weights job of
  // the call before has written it), fetched in that same trip
  uint32_t vbuf = 0;
  const bool partial_minima = out_w && !weights_here;
  if (partial_minima) vbuf = read_word_with_the_loads(g.vnext + t);   // (its low bit; taken where it is used, so that nothing waits for the word here)
  // the new priority of this lane's sample and the running maximum, likewise
  float upd_v = 0.0f;
  uint32_t max_seen = 0;
  uint32_t claim_first = 1;
  if (claim_mode == 1) {
    upd_v = c.prio[o];
    max_seen = read_max_bits(g, t);
    claim_first = claim_base(g, t, c.group_mode);
  }

  uint32_t off[kTopSlots + 1];
  off[0] = 0;
#pragma unroll
  for (int i = 0; i < kTopSlots; ++i) off[i + 1] = off[i] + (i < nslots ? tc.cnt[i] : 0u);
  const uint32_t top_floats = off[kTopSlots];
  // the carried insertion's LDS: behind the top copy and the waves' staging rows
  float* rl = lds + top_floats + (LOGK >= 3 ? (size_t)(blockDim.x >> 6) * ROWS * ROW : (size_t)0);
  // Everything it reads is fetched in the trip of the top copy: the loads are issued here, into registers, and
  // parked in LDS once the top copy's own loads are under way (a store to LDS waits for its data).  Lane i takes
  // element i of each height's run of child groups.  A staged leaf that the insertion rewrites is replaced as it
  // is parked (by a valid new priority only).  The plan of all heights comes in one batch of scalar loads and
  // stays in registers: a single wave's chain of instructions and scalar fetches is what a small batch waits for.
  // (plain words, not structures: the compiler keeps structures that lambdas take by reference in memory)
  [[maybe_unused]] uint32_t a1 = 0, c1 = 0, o1 = 0, t1 = 0, a2 = 0, c2 = 0, o2 = 0, t2 = 0, a3 = 0, c3 = 0, o3 = 0, t3 = 0,
                            a4 = 0, c4 = 0, o4 = 0, t4 = 0;   // a: first touched node, c: how many, o: LDS offset, t: top-copy offset
  [[maybe_unused]] float rv1 = 0, rv2 = 0, rv3 = 0, rv4 = 0;
  [[maybe_unused]] float nv1 = -1.0f;   // new priority of this lane's leaf (invalid: the leaf stays)
  static_assert(kRideHeights == 4, "one register per height");
  if constexpr (RIDE) {
    // (first nodes and LDS offsets follow from the lowest height's: fewer words to hold)
    a1 = ride.h[0].a0; c1 = ride.h[0].cnt; t1 = ride.h[0].top_at;
    c2 = ride.h[1].cnt; t2 = ride.h[1].top_at;
    c3 = ride.h[2].cnt; t3 = ride.h[2].top_at;
    c4 = ride.h[3].cnt; t4 = ride.h[3].top_at;
    a2 = a1 >> LOGK; a3 = a2 >> LOGK; a4 = a3 >> LOGK;
    o1 = 0; o2 = c1 * K; o3 = o2 + c2 * K; o4 = o3 + c3 * K;
    if (threadIdx.x < c1 * K) rv1 = g.level[0][(size_t)t * g.stride[0] + (size_t)a1 * K + threadIdx.x];
    if (threadIdx.x < c2 * K) rv2 = g.level[1][(size_t)t * g.stride[1] + (size_t)a2 * K + threadIdx.x];
    if (threadIdx.x < c3 * K) rv3 = g.level[2][(size_t)t * g.stride[2] + (size_t)a3 * K + threadIdx.x];
    if (threadIdx.x < c4 * K) rv4 = g.level[3][(size_t)t * g.stride[3] + (size_t)a4 * K + threadIdx.x];
    const uint32_t j = a1 * K + threadIdx.x - ride.cursor;   // (slots below the cursor wrap to large numbers)
    if (threadIdx.x < c1 * K && j < ride.n) nv1 = ride.prio ? ride.prio[(size_t)t * ride.n + j] : g.max_v[t];
  }
  auto park_ride = [&]() {
    if constexpr (RIDE) {
      if (threadIdx.x < c1 * K) rl[o1 + threadIdx.x] = valid_priority(nv1) ? nv1 : rv1;
      if (threadIdx.x < c2 * K) rl[o2 + threadIdx.x] = rv2;
      if (threadIdx.x < c3 * K) rl[o3 + threadIdx.x] = rv3;
      if (threadIdx.x < c4 * K) rl[o4 + threadIdx.x] = rv4;
    }
  };

  if (nslots > 0) {
    // one flat loop over the vectors of all copied heights (stale ones are skipped)
    uint32_t v_lo = 0;   // off[min(stale, kTopSlots)] / VF, without indexing the array by a run-time value
#pragma unroll
    for (int i = 1; i <= kTopSlots; ++i)
      if (stale >= i) v_lo = off[i] / VF;
    for (uint32_t e = v_lo + threadIdx.x; e < top_floats / VF; e += blockDim.x) {
      const uint32_t f = e * VF;
      const float* src = tc.ptr[0] + (size_t)t * tc.stride[0];
      uint32_t base = 0;
#pragma unroll
      for (int i = 1; i < kTopSlots; ++i) {
        const bool here = i < nslots && f >= off[i];
        src = here ? tc.ptr[i] + (size_t)t * tc.stride[i] : src;
        base = here ? off[i] : base;
      }
      *reinterpret_cast<Vec*>(lds + f) = *reinterpret_cast<const Vec*>(src + (f - base));
    }
    park_ride();
    __syncthreads();
    PER_MARK(1);
    if constexpr (RIDE) {
      PER_MARK(13);
      // the touched nodes height by height: sums of the staged groups, into the groups of the height above,
      // into the top copy where the height is part of it, and (last workgroup) aside for the stores
      const unsigned q = threadIdx.x % LPS;
      const uint32_t grp = threadIdx.x / LPS, ngrp = blockDim.x / LPS;
      // (a, c, o, top: the height's touched nodes; up_a, up_o: those of the height above, if it is patched too)
      auto sum_height = [&](uint32_t a, uint32_t cn, uint32_t o, uint32_t top, bool has_up, uint32_t up_a, uint32_t up_o) {
        for (uint32_t base = 0; base < cn; base += ngrp) {
          const uint32_t at = base + grp;
          const bool ok = at < cn;
          const float sum = group_sum<LOGK>(rl + o + (size_t)(ok ? at : 0u) * K, q);
          if (ok && q == 0) {
            const uint32_t nd = a + at;
            if (is_mover) rl[ride.val_off + (o >> LOGK) + at] = sum;
            if (has_up) rl[up_o + (nd - up_a * K)] = sum;
            if (top != kRideNone) lds[top + nd] = sum;
          }
        }
        __syncthreads();
      };
      const uint32_t hp = ride.hp;
      // One touched node per height (the rows lie under one height-1 node: the usual case of a few rows): one lane
      // group works its way up by itself, each sum patched into the staged group of the height above and read back
      // by the same wave, with no workgroup barrier between the heights.
      const bool chain = c1 == 1 && (hp < 2 || c2 == 1) && (hp < 3 || c3 == 1) && (hp < 4 || c4 == 1);
      if (chain) {
        if (threadIdx.x < (uint32_t)LPS) {
          auto one = [&](uint32_t a, uint32_t o, uint32_t top, bool has_up, uint32_t up_a, uint32_t up_o) {
            const float sum = group_sum<LOGK>(rl + o, q);
            if (q == 0) {
              if (is_mover) rl[ride.val_off + (o >> LOGK)] = sum;
              if (has_up) rl[up_o + (a - up_a * K)] = sum;
              if (top != kRideNone) lds[top + a] = sum;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
          };
          one(a1, o1, t1, hp > 1, a2, o2);
          if (hp > 1) one(a2, o2, t2, hp > 2, a3, o3);
          if (hp > 2) one(a3, o3, t3, hp > 3, a4, o4);
          if (hp > 3) one(a4, o4, t4, false, 0, 0);
        }
        __syncthreads();
      } else {
        sum_height(a1, c1, o1, t1, hp > 1, a2, o2);
        if (hp > 1) sum_height(a2, c2, o2, t2, hp > 2, a3, o3);
        if (hp > 2) sum_height(a3, c3, o3, t3, hp > 3, a4, o4);
        if (hp > 3) sum_height(a4, c4, o4, t4, false, 0, 0);
      }
      if (is_mover) {   // the new leaves, the new sums of heights 1 .. hp, what the running maximum may rise to; the rows
        uint32_t mx = 0;
        bool bad = false;
        float* leaves = g.level[0] + (size_t)t * g.stride[0];
        for (uint32_t j = threadIdx.x; j < ride.n; j += blockDim.x) {
          const uint32_t slot = ride.cursor + j;
          leaves[slot] = rl[o1 + (slot - a1 * K)];   // (the old value again where the new one was invalid)
          if (ride.prio) {
            const float v = ride.prio[(size_t)t * ride.n + j];
            if (!valid_priority(v)) bad = true;
            else if (v > 0.0f) mx = __float_as_uint(v) > mx ? __float_as_uint(v) : mx;
          }
        }
        auto store_height = [&](uint32_t a, uint32_t cn, uint32_t o, int height) {
          float* lvl = g.level[height] + (size_t)t * g.stride[height];
          for (uint32_t at = threadIdx.x; at < cn; at += blockDim.x) lvl[a + at] = rl[ride.val_off + (o >> LOGK) + at];
        };
        store_height(a1, c1, o1, 1);
        if (hp > 1) store_height(a2, c2, o2, 2);
        if (hp > 2) store_height(a3, c3, o3, 3);
        if (hp > 3) store_height(a4, c4, o4, 4);
        if (ride.prio) {
          mx = wave_max_u32(mx);
          if (lane == 0 && mx) atomicMax(&g.max_pend[t], mx);
          if (bad) atomicOr(&g.status[t], 2u);
        }
        PER_MARK(14);
        ride_rows(ride, t, g.N, 0, movers);
        PER_MARK(12);
        PER_FLUSH_TAG(1);
        return;
      }
    }
    PER_MARK(14);
    if (stale >= 0) {   // rebuild slots stale-1 .. 0 and the root, bottom-up
      const unsigned q = threadIdx.x % LPS;
      const uint32_t grp = threadIdx.x / LPS, ngrp = blockDim.x / LPS;
#pragma unroll
      for (int i = kTopSlots - 1; i >= -1; --i) {
        if (i < stale && i + 1 < nslots) {
          const uint32_t nl = i >= 0 ? tc.nreal[i] : 1u;
          const uint32_t cnt = i >= 0 ? tc.cnt[i] : 0u;
          const uint32_t off_l = i >= 0 ? off[i] : 0u;
          for (uint32_t base = 0; base < nl; base += ngrp) {
            const uint32_t j = base + grp;
            const bool real = j < nl;
            const float sum = group_sum<LOGK>(lds + off[i + 1] + (size_t)(real ? j : 0u) * K, q);
            if (q == 0 && real) {
              if (i >= 0) lds[off_l + j] = sum; else s_total = sum;
            }
          }
          for (uint32_t j = nl + threadIdx.x; j < cnt; j += blockDim.x) lds[off_l + j] = 0.0f;   // group padding
          __syncthreads();
        }
      }
      total = s_total;
    }
  }

  // The first workgroup of each tree puts the heights rebuilt above back into memory (also when nothing can be
  // sampled: the host has noted that this kernel makes them current).
  auto store_rebuilt_top = [&]() {
    if (stale >= 0 && bx == 0) {
#pragma unroll
      for (int i = 0; i < kTopSlots; ++i)
        if (i < stale) {
          float* dst = g.level[H - 1 - (uint32_t)i] + (size_t)t * g.stride[H - 1 - (uint32_t)i];
          for (uint32_t j = threadIdx.x; j < tc.nreal[i]; j += blockDim.x) dst[j] = lds[off[i] + j];
        }
      if (threadIdx.x == 0) g.root[(size_t)t * g.root_stride] = total;
    }
  };

  if (!(total > 0.0f)) {   // nothing can be sampled from this tree (uniform over the block)
    store_rebuilt_top();
    for (; s_raw < B; s_raw += sample_blocks * blockDim.x) {
      o = (size_t)t * B + s_raw;
      out_idx[o] = 0xFFFFFFFFu;
      if (out_prio) out_prio[o] = 0.0f;
      if (out_w) out_w[o] = 0.0f;
    }
    // (a fused update of these samples finds no valid index: every element is out of range)
    if (bx == 0 && threadIdx.x == 0) {
      atomicOr(&g.status[t], claim_mode == 1 ? 5u : 4u);
      if (partial_minima) g.vcur[t] = not_before_here(vbuf) & 1u;   // the weights job of this call runs all the same
      if (claim_mode == 1) leave_claim_base(g, t, c.group_mode, true, claim_first);
    }
    return;
  }

  PER_MARK(2);
  const float seg = total / (float)B;
  uint32_t node = 0, least = 0x7F800000u, claim_mx = 0, claim_flags = 0;
  float val = total;
  for (;;) {
  // (the uniform of the next round travels beside this round's walk)
  const uint32_t next_raw = s_raw + sample_blocks * blockDim.x;
  const bool again = LOOP && next_raw - threadIdx.x < B;   // (the same for the workgroup)
  float u_next = 0.0f, upd_next = 0.0f;
  if (again) {
    const uint32_t sn = next_raw < B ? next_raw : B - 1;
    u_next = rng.on ? counter_uniform(rng, sn, t) : u[(size_t)t * B + sn];
    if (claim_mode == 1) upd_next = c.prio[(size_t)t * B + sn];
  }
  const float pos = (float)s + u_s;
  float r = pos * seg;
  node = 0;
  val = total;
#pragma unroll
  for (int i = 0; i < kTopSlots; ++i) {
    if (i < nslots) {
      unsigned child;
      descend_lane<LOGK>(lds + off[i] + (size_t)node * K, r, child, val);
      node = node * K + child;
    }
  }

  PER_MARK(3);
  float* stage = lds + top_floats + (size_t)wave * ROWS * ROW;
  const int l0 = (int)H - 1 - nslots;     // highest height read from memory
  // the pointer of the next level is fetched while the current one is processed
  const float* lvl_next = l0 >= 0 ? g.level[l0] + (size_t)t * g.stride[l0] : nullptr;
  for (int l = l0; l >= 0; --l) {
    const float* lvl = lvl_next;
    if (l > 0) lvl_next = g.level[l - 1] + (size_t)t * g.stride[l - 1];
    unsigned child;
    // (a carried insertion: the group of a touched node is read from the patched copy)
    const float* patched = nullptr;
    if constexpr (RIDE) {
      // touched nodes of height l + 1 (l + 1 <= hp: the copy reaches down to hp)
      const uint32_t pa = l == 0 ? a1 : l == 1 ? a2 : l == 2 ? a3 : a4;
      const uint32_t pc = l == 0 ? c1 : l == 1 ? c2 : l == 2 ? c3 : c4;
      const uint32_t po = l == 0 ? o1 : l == 1 ? o2 : l == 2 ? o3 : o4;
      if (node - pa < pc) patched = rl + po + (size_t)(node - pa) * K;
    }
    if constexpr (LOGK <= 2) {
      if (RIDE && patched) descend_lane<LOGK>(patched, r, child, val);
      else descend_lane<LOGK>(lvl + (size_t)node * K, r, child, val);
    } else if constexpr (LOOP != LOOP_NONE) {
      descend_staged<LOGK, LOOP == LOOP_FEW_ROWS>(lvl, node, lane, stage, r, child, val);
    } else {
      stage_group_per_lane<LOGK, 0>(lvl, node, lane, stage);
      order_within_wave();
      descend_lane<LOGK>(RIDE && patched ? patched : stage + lane * ROW, r, child, val);
      __builtin_amdgcn_wave_barrier();
    }
    node = node * K + child;
    PER_MARK_DYN(4 + (l0 - l));
  }

  if (active) {
    out_idx[o] = node;
    if (out_prio) out_prio[o] = val;
    if (out_w && !weights_here) out_w[o] = val;   // (turned into the weight by the weights job)
    least = min_u32(least, __float_as_uint(val));
  }
  if (!again) break;
  if (claim_mode == 1 && active) claim_element(g, t, size, c.group_mode, claim_first, s, node, upd_v, claim_mx, claim_flags);
  s_raw = next_raw;
  active = s_raw < B;
  s = active ? s_raw : B - 1;
  o = (size_t)t * B + s;
  u_s = u_next;
  upd_v = upd_next;
  }
  // Stores come last on purpose: on this hardware a wait for loaded data also waits for every
  // earlier store of the wave.
  store_rebuilt_top();
  PER_MARK(12);
  PER_FLUSH_TAG(1);
  if (out_w) {
    // Importance weights need the batch minimum of the sampled values.
    const uint32_t m = wave_min_u32(least);
    if (weights_here) {   // the whole batch of this tree is in this block: finish here
      if (lane == 0) s_min[wave] = m;
      __syncthreads();
      uint32_t mm = 0x7F800000u;
      for (uint32_t wv = 0; wv < (blockDim.x >> 6); ++wv) mm = s_min[wv] < mm ? s_min[wv] : mm;
      if (weight_mode & kWeightBufferNorm) mm = buffer_min_bits(g, t, weight_mode);   // (uniform over the launch)
      if (active) out_w[o] = importance_weight(val, __uint_as_float(mm), beta);
    } else {                // partial minima, spread over kVminSlots addresses; the weights job finishes
      vbuf = not_before_here(vbuf) & 1u;
      if (bx == 0 && threadIdx.x == 0) g.vcur[t] = vbuf;   // tells the weights job of this call which buffer it is
      if (lane == 0)
        atomicMin(&g.vmin[((size_t)vbuf * g.T + t) * kVminSlots + ((bx * (blockDim.x >> 6) + wave) % kVminSlots)], m);
    }
  }
  if (claim_mode == 1) {   // element s of the update batch is this lane's own sample
    if (active) claim_element(g, t, size, c.group_mode, claim_first, s, node, upd_v, claim_mx, claim_flags);
    if constexpr (RIDE) {
      claim_mx = wave_max_u32(claim_mx);
      if (lane == 0 && claim_mx > max_seen) atomicMax(&g.max_pend[t], claim_mx);
    } else {
      raise_max(g, t, claim_mx, max_seen);
    }
    if (claim_flags) atomicOr(&g.status[t], claim_flags);
    leave_claim_base(g, t, c.group_mode, bx == 0 && threadIdx.x == 0, claim_first);
  }
}

// Finishes the importance weights of tree t: folds the partial minima that the sampling kernel of this
// call has left in one of the two vmin buffers and turns the sampled values left in w into weights.
// Called by whole workgroups of any size.  Which buffer: vcur, written by that sampling kernel.  The
// first workgroup re-arms the other buffer and makes it the one the next sampling kernel fills (vnext;
// only kernels of later calls read that word).  Nothing of this alternation lives on the host, so a
// captured call can be replayed.  `mode`: see kWeightBufferNorm.
__device__ __forceinline__ void weights_job(const Geom& g, uint32_t t, uint32_t B, uint32_t size, float beta,
                                            float* __restrict__ w, uint32_t mode, uint32_t job_block,
                                            uint32_t job_blocks) {
  __shared__ uint32_t s_wmin[16];
  if (job_block != 0 && job_block * blockDim.x >= B) return;   // nothing to do for this workgroup
  // (both buffers are fetched beside the word that says which one counts: one trip instead of two)
  const uint32_t* part0 = g.vmin + (size_t)t * kVminSlots;
  const uint32_t* part1 = g.vmin + ((size_t)g.T + t) * kVminSlots;
  uint32_t m0 = 0x7F800000u, m1 = 0x7F800000u;
  const uint32_t vword = read_word_with_the_loads(g.vcur + t);
  for (uint32_t j = threadIdx.x; j < kVminSlots; j += blockDim.x) {
    m0 = part0[j] < m0 ? part0[j] : m0;
    m1 = part1[j] < m1 ? part1[j] : m1;
  }
  const uint32_t vbuf = not_before_here(vword) & 1u;
  uint32_t m = wave_min_u32(vbuf ? m1 : m0);
  if ((threadIdx.x & 63u) == 0) s_wmin[threadIdx.x >> 6] = m;
  if (job_block == 0) {
    for (uint32_t j = threadIdx.x; j < kVminSlots; j += blockDim.x)
      g.vmin[((size_t)(vbuf ^ 1u) * g.T + t) * kVminSlots + j] = 0x7F800000u;
    if (threadIdx.x == 0) g.vnext[t] = vbuf ^ 1u;
  }
  __syncthreads();
  uint32_t mm = 0x7F800000u;
  for (uint32_t wv = 0; wv < (blockDim.x >> 6); ++wv) mm = s_wmin[wv] < mm ? s_wmin[wv] : mm;
  // No minimum at all means that nothing could be sampled (the tree's total was zero): weights 0.  (The root
  // itself must not be consulted here: a tree pass running beside this job may already have rewritten it.)
  const bool nothing_sampled = mm == 0x7F800000u;
  if (mode & kWeightBufferNorm) mm = buffer_min_bits(g, t, mode);   // (uniform over the launch)
  for (uint32_t i = job_block * blockDim.x + threadIdx.x; i < B; i += job_blocks * blockDim.x) {
    const size_t o = (size_t)t * B + i;
    w[o] = nothing_sampled ? 0.0f : importance_weight(w[o], __uint_as_float(mm), beta);
  }
}

__global__ void k_weights(Geom g, uint32_t B, uint32_t size, float beta, float* __restrict__ w, uint32_t mode) {
  weights_job(g, blockIdx.y, B, size, beta, w, mode, blockIdx.x, gridDim.x);
}

template <int LOGK>
static hipError_t launch_resum_top_k(const Geom& g, const Tuning& tn, uint32_t hb, hipStream_t s);
static hipError_t launch_finish(const Geom& g, const Tuning& tn, const FieldTable* rows, const FinishArgs& a,
                                hipStream_t s);
template <int LOGK>
static hipError_t launch_tree_k(const Geom& g, const Tuning& tn, const ClaimArgs& c, hipStream_t s);
template <int LOGK>
static hipError_t launch_tree_finish_k(const Geom& g, const Tuning& tn, const ClaimArgs& c, const FieldTable* rows,
                                       const FinishArgs& a, bool earlier, hipStream_t s);

// Waves of a sampling workgroup (carried: what the launch carries of an insertion).  Every workgroup copies the
// top of the tree and, behind an update, rebuilds it from the roots of the tree pass's subtrees.  One wave needs no barriers
// for that and leaves the samples to the most compute units; with more than 256 roots the copy wants more lanes, beyond 1024
// fewer workgroups that make it.  One and two waves (us per step, K = 16): 2^18 leaves, 4096 samples, 4 new rows 13.7 and
// 13.0, 8192 and none 12.6 and 12.1; 2^20 leaves, earlier-batch form of 8192 11.1 and 10.8, 2^22 (1024 roots) 13.3 and
// 13.9; K = 32, 2^22 leaves, 8192: 13.6 and 13.2.  Two and four: 2^20 leaves at K = 8 (2048 roots), earlier-batch form of
// 8192, 13.0 and 12.5.  (Fewer than 48 roots: 0.93 to 1.02 times; K = 8 the same, K = 64 0.97 to 1.01; 131 072 samples on 2^23
// leaves at K = 32 35.3 and 36.0.  About the lines: K = 16, one wave and two, 256 roots, 16 384 samples 14.6 and 15.0, 24 576 16.2 and 16.1; 512
// roots, 2048 samples 12.2 and 11.9, 8192 12.8 both; K = 8, two and four, 1024 roots, 8192 samples 12.2 and 12.6, 2048 roots 13.6 and 13.2.)
// Every workgroup works a carried insertion out for itself, a run of child groups of which must fit its lanes: that is the
// least it may have (up to two waves, up to eight on many trees).  On 64 trees it is better worked out by few workgroups of
// eight waves unless the trees are small (1000 samples, 4 rows each, eight waves and two: 2^18 leaves at K = 16 26.7 and 27.5,
// 4096 27.3 and 26.2; 48 trees of 2^18 18.7 and 18.4, 8 of 4096 17.9 and 13.5).
// The rows of a carried insertion are moved by workgroups of the same size, whole rows each, a sweep of the lanes after the other.
// Where that takes more than four sweeps (rows of many pieces: odd lengths go by bytes) it is the largest size again, two waves on up
// to seven trees, eight on more (4 rows each; one wave and two, 441 samples on 300 000 leaves at K = 16: 319 bytes, five sweeps, 12.6 both,
// 511 14.6 and 12.7, 1033 20.9 and 15.8; two waves and eight, 256 samples on 8 trees of 50 000: 511 bytes, four sweeps, 13.0 and 13.3, 639 13.8 and
// 13.4, 1033 17.6 and 15.0).
struct CarriedRows {
  uint32_t n, pieces;   // rows per tree, elements that one is moved in
  uint32_t movers(uint32_t lanes) const {   // as many as it takes to move every element in one sweep (whole rows each; at most 32)
    const uint64_t all = ((uint64_t)n * pieces + lanes - 1) / lanes;
    const uint32_t most = n < 32u ? n : 32u;
    return all < 1 ? 1u : all < most ? (uint32_t)all : most;
  }
  uint64_t sweeps(uint32_t lanes) const { return ((uint64_t)((n + movers(lanes) - 1) / movers(lanes)) * pieces + lanes - 1) / lanes; }
};
static CarriedRows carried_rows(const FieldTable* ft, uint32_t n) {
  CarriedRows c{n, 0};
  if (ft)
    for (uint32_t f = 0; f < ft->n_fields; ++f)
      if (ft->io[f]) c.pieces += ft->bytes[f] / ft->vec[f];
  return c;
}
static uint32_t sample_waves(const Geom& g, const Tuning& tn, uint32_t B, const CarriedRows& carried) {
  const uint32_t hb = lazy_top_height(g, tn);
  uint32_t waves = 2;
  if (hb && g.n[hb] > 1024u && g.logK == 3) waves = 4;
  if (hb >= 3 && (g.logK == 4 || g.logK == 5) && g.n[hb] > 48u && g.n[hb] <= 256u && (uint64_t)B * g.T <= 16384u) waves = 1;
  if (!carried.n) return waves;
  if (g.T >= 64u && g.N > 8192u) return 8;
  const uint32_t lanes = ((carried.n - 1) / g.K + 2) * g.K, most = g.T >= 8u ? 8u : 2u;
  const uint32_t least = (lanes + 63u) / 64u < most ? (lanes + 63u) / 64u : most;
  if (waves < least) waves = least;
  return waves < most && carried.sweeps(waves * 64u) > 4 ? most : waves;
}
constexpr uint32_t kLoopWaves = 4;   // (of the kernel that loops over blocks with few rows: see StageRow)

// Workgroup size and top copy of a sampling launch for batch B (stale_hb: the height the stale top is rebuilt
// from, or 0).  The copy: at most kTopSlots of the topmost heights (below the root), within the LDS budget, and
// only while a height is small next to what the workgroup's samples would fetch from it one by one.  A launch that carries an
// insertion leaves the leaves out: the walk takes the new ones from the patch, behind the copy.
struct SampleShape {
  TopCopy tc;
  uint32_t waves, wave_bytes, top_bytes;
};
static SampleShape sample_shape(const Geom& g, const Tuning& tn, uint32_t B, uint32_t stale_hb, bool weights_behind, const CarriedRows& carried = {},
                                SampleLoop loop = LOOP_NONE, bool wide = false) {
  constexpr uint32_t kLdsCap = 128 * 1024;
  SampleShape sh{};
  const uint32_t K = g.K;
  sh.wave_bytes = g.logK < 3 ? 0u : (loop ? stage_floats(g.logK, loop == LOOP_FEW_ROWS) : 64u * (K + 4u)) * 4u;   // staging per wave
  // workgroup size: the configured size, or the whole batch in one workgroup when it is small and no kernel comes behind
  // that could finish the weights (where one does, several workgroups are faster from the third wave on: a step of 1024
  // samples on 2^20 leaves at K = 4 takes 20.8 us with one and 16.3 with eight, of 512 at K = 16 12.8 and 11.7);
  // bounded by the LDS the staging rows need (wide, the walk by sixteens: not, since the trees that it serves had no staging rows before)
  uint32_t max_waves = sh.wave_bytes && !wide ? (uint32_t)(kLdsCap / 2 / sh.wave_bytes) : 16u;
  if (max_waves > 16) max_waves = 16;
  if (max_waves < 1) max_waves = 1;
  uint32_t waves = tn.sample_block / 64;
  if (tn.sample_block_auto) waves = loop == LOOP_FEW_ROWS ? kLoopWaves : loop || wide ? 2u : sample_waves(g, tn, B, carried);
  const uint32_t need = (B + 63) / 64;
  if (need <= (weights_behind ? waves : max_waves)) waves = need;
  if (waves > max_waves) waves = max_waves;
  sh.waves = waves;
  const uint32_t block = waves * 64;
  TopCopy& tc = sh.tc;
  uint64_t top = 0;
  for (int l = (int)g.H - 1; l >= (carried.n ? 1 : 0) && tc.nslots < (uint32_t)kTopSlots; --l) {
    const uint64_t cnt = (uint64_t)g.n[l + 1] * K;
    const uint64_t add = cnt * 4;
    if (top + add > tn.lds_budget_bytes || top + add + (uint64_t)waves * sh.wave_bytes > kLdsCap) break;
    const bool needed_for_rebuild = stale_hb && (uint32_t)l >= stale_hb;   // the rebuild of stale heights reads it
    if (cnt > 8ull * block && tn.lds_budget_bytes <= 64 * 1024 && !needed_for_rebuild) break;
    top += add;
    const uint32_t i = tc.nslots++;
    tc.ptr[i] = g.level[l];
    tc.stride[i] = g.stride[l];
    tc.cnt[i] = g.n[l + 1] * K;
    tc.nreal[i] = g.n[l];
  }
  tc.root = g.root;
  tc.root_stride = g.root_stride;
  sh.top_bytes = (uint32_t)top;
  return sh;
}

// A carried insertion: the touched nodes of heights 1 .. hp (two ranges per height, narrowed by K from one height
// to the next) and where their child groups, their new sums and the new leaves sit in LDS.
// Most rows a sampling kernel carries: every workgroup of it sums the touched nodes anew, and beside the kernel of large
// insertions that only pays for few.  The line is drawn by the width of those sums and, for wide ones, by how many trees
// there are (insertion carried and apart, us per step with 165-byte rows):
//  - up to K = 16, 128 rows: a tree of 2^20 leaves at K = 16, 4096 samples: 128 rows 13.8 and 15.3; 64 trees of 2^17: 64 rows
//    26.7 and 28.2, 128 rows 28.1 and 30.0; 64 trees of 2^15 at K = 8, 499 samples: 64 rows 20.1 and 22.0, 256 rows 26.6
//    and 24.2.  K = 32 the same on few trees (16 of 2^17, 1024 samples: 128 rows 19.4 and 21.4), on many 64 rows (64 of
//    2^17: 32 rows 33.4 and 34.9, 64 rows 35.4 and 35.1, 128 rows 38.3 and 36.2);
//  - K = 64: 16 rows, from 512 samples on (64 trees of 2^15, 512 samples: 16 rows 25.2 and 26.0, 32 rows 27.8 and 26.1, 64
//    rows 35.2 and 26.5; 4 of 2^17: 1024 samples 16.8 and 16.9, 64 samples 16.5 and 15.3).
static uint32_t most_rows_carried(const Geom& g, uint32_t B) {
  if (g.logK == 6) return B >= 512u ? 16u : 0u;
  return g.logK == 5 && g.T >= 32u ? 64u : 128u;
}
constexpr uint32_t kRideLdsBytes = 16 * 1024; // most LDS its patch may take
// False when the insertion runs past the ring's end or a run of child groups is longer than the workgroup (`block`
// lanes): the insertion then goes by itself.
static bool plan_ride(const Geom& g, const TopCopy& tc, uint32_t block, uint32_t hp, InsertRide* rd) {
  const uint32_t L = g.logK;
  if ((uint64_t)rd->cursor + rd->n > g.N || hp > (uint32_t)kRideHeights) return false;
  uint32_t a = rd->cursor, b = rd->cursor + rd->n;   // touched nodes [a, b)
  uint32_t floats = 0, vals = 0;
  for (int i = 0; i < kRideHeights; ++i) rd->h[i] = RideHeight{0, 0, 0, kRideNone};
  for (uint32_t h = 1; h <= hp; ++h) {
    a >>= L;
    b = ((b - 1) >> L) + 1;
    RideHeight& P = rd->h[h - 1];
    P.a0 = a;
    P.cnt = b - a;
    P.off = floats;
    if ((uint64_t)P.cnt * g.K > block) return false;
    uint32_t top = 0;   // where the sampling kernel's top copy holds this height
    for (uint32_t i = 0; i < tc.nslots; ++i) {
      if (g.H - 1 - i == h) P.top_at = top;
      top += tc.cnt[i];
    }
    floats += P.cnt * g.K;
    vals += P.cnt;
  }
  rd->hp = hp;
  rd->val_off = floats;
  rd->floats = floats + vals;
  return true;
}

bool sample_can_carry_insert(const Geom& g, const Tuning& tn, uint32_t B, const FieldTable* ft, uint32_t n, uint32_t cursor) {
  const uint32_t hb = lazy_top_height(g, tn);
  if (!hb || hb > (uint32_t)kRideHeights || n == 0 || n > most_rows_carried(g, B) || n > g.N) return false;
  uint64_t bytes = 0;
  if (ft)
    for (uint32_t f = 0; f < ft->n_fields; ++f)
      if (ft->io[f]) bytes += (uint64_t)n * ft->bytes[f];
  if (bytes > 256 * 1024) return false;
  // the top copy must reach down to the height the top is rebuilt from
  const SampleShape sh = sample_shape(g, tn, B, hb, true, carried_rows(ft, n));
  if (sh.tc.nslots == 0 || g.H - sh.tc.nslots > hb) return false;
  // the runs of the patch must fit the workgroup, and the patch its share of the LDS
  InsertRide rd{};
  rd.n = n;
  rd.cursor = cursor;
  return plan_ride(g, sh.tc, sh.waves * 64, hb, &rd) && (uint64_t)rd.floats * 4 <= kRideLdsBytes;
}

// Sampling call with whatever is fused into it.  rows: gather of the sampled rows.  claim: a priority
// update whose claim phase runs where claim_mode says (CLAIM_INLINE / CLAIM_BLOCKS: in the sampling
// kernel, the tree pass then shares the second kernel with the weights and row jobs; CLAIM_FINISH: in
// the second kernel, the tree pass is a third).  ride: an insertion carried by the sampling kernel (the caller
// has checked sample_can_carry_insert and passes the lazily rebuilt height as stale_hb).
template <int TREE, int LOGK>
static hipError_t launch_sample_walk(const Geom& tree, const Geom& g, const Tuning& tn, uint32_t B, uint32_t size, float beta,
                                  const float* u, const RngArgs& rng, uint32_t* out_idx, float* out_w,
                                  float* out_prio, uint32_t weight_mode, uint32_t stale_hb, const FieldTable* rows,
                                  const ClaimArgs* claim, int claim_mode, const InsertRide* ride, hipStream_t s) {
  const CarriedRows carried = ride ? carried_rows(&ride->rows, ride->n) : CarriedRows{};
  SampleShape sh = sample_shape(g, tn, B, stale_hb, rows || claim, carried, LOOP_NONE, TREE != LOGK);
  // No more workgroups than the device holds at once (their staging rows fill its LDS): they take further blocks of
  // samples in turn, with the top of the tree in place and the next uniforms under way, where workgroups of a second
  // round would begin with their arguments and the top of the tree again, two of the five trips to memory of a block.
  // (2^20 samples on 2^24 leaves at K = 32: 59 us with a workgroup per block, 25.6 so, with the rows of descend_staged.)
  const uint64_t units = compute_units(tn.device);
  auto held = [&]() -> uint64_t {   // workgroups the device holds
    uint64_t bytes = (uint64_t)sh.top_bytes + (uint64_t)sh.waves * sh.wave_bytes, by_waves = 32 / sh.waves;
    if (bytes < tn.sample_min_lds) bytes = tn.sample_min_lds;
    const uint64_t by_lds = bytes ? (160 * 1024) / bytes : by_waves, n = by_lds < by_waves ? by_lds : by_waves;
    return (units ? units : 256) * (n < 1 ? 1 : n);
  };
  const SampleLoop loop = ride || (uint64_t)((B + sh.waves * 64 - 1) / (sh.waves * 64)) * g.T <= held() ? LOOP_NONE
                          : few_rows(g, B)                                                              ? LOOP_FEW_ROWS
                                                                                                        : LOOP_ALL_ROWS;
  if (loop) sh = sample_shape(g, tn, B, stale_hb, rows || claim, {}, loop, TREE != LOGK);
  const TopCopy& tc = sh.tc;
  const uint32_t waves = sh.waves;
  const uint32_t block = waves * 64;
  const uint32_t blocks = (B + block - 1) / block;
  uint32_t gx = blocks;
  if (loop) {
    gx = (uint32_t)(held() / g.T < 2 ? 2 : held() / g.T);   // (at least two: one workgroup alone finishes the weights of the block it holds)
    if (gx > blocks) gx = blocks;
    // Where the leaves take up to half the second-level caches (32 MiB), no more workgroups than it takes for all to have as many
    // blocks as the busiest: `sample` and `update` of 2^19 on 3 million leaves at K = 32 87.6 -> 83.5 us, on 2^20 at K = 16
    // 67.2 -> 63.5.  On 2^24 leaves at K = 32 the workgroups without a last block leave more of the memory to the
    // others: 78.2 so, 80.2 with as many blocks each; 286 222 on 7.9 million at K = 16 50.4 and 52.1.
    if ((uint64_t)g.N * g.T * 4u <= 16u << 20 && gx > 2) {
      const uint32_t rounds = (blocks + gx - 1) / gx;
      gx = (blocks + rounds - 1) / rounds;
      if (gx < 2) gx = 2;
    }
  }
  uint32_t parts = 0;
  if (weight_mode & kWeightMinHere) {
    if (ride) return hipErrorInvalidValue;
    parts = min_parts(g, block);
    weight_mode |= parts << kWeightPartsShift;
  }
  size_t bytes = (size_t)sh.top_bytes + (size_t)waves * sh.wave_bytes;
  hipError_t e;
  int stale = -1;
  if (stale_hb) {
    // copied heights above stale_hb are rebuilt in LDS; the copy must reach down to stale_hb
    const int lowest_copied = (int)g.H - (int)tc.nslots;
    if (tc.nslots > 0 && lowest_copied <= (int)stale_hb) {
      stale = (int)g.H - 1 - (int)stale_hb;
    } else {
      if (ride) return hipErrorInvalidValue;
      e = launch_resum_top_k<LOGK>(g, tn, stale_hb, s);
      if (e != hipSuccess) return e;
    }
  }
  if (!claim) claim_mode = CLAIM_NONE;
  InsertRide rd{};
  if (ride) {
    if (stale < 0 || stale_hb != lazy_top_height(g, tn) || claim_mode == CLAIM_BLOCKS) return hipErrorInvalidValue;
    rd = *ride;
    if (!plan_ride(g, tc, block, stale_hb, &rd)) return hipErrorInvalidValue;
    rd.movers = carried.movers(block);
    bytes += (size_t)rd.floats * 4;
  }
  if (bytes < tn.sample_min_lds) bytes = tn.sample_min_lds;   // asking for more LDS than needed spreads workgroups over more CUs
  const bool claim_here = claim_mode == CLAIM_INLINE || claim_mode == CLAIM_BLOCKS;
  uint32_t claim_blocks = 0;
  if (claim_mode == CLAIM_BLOCKS) {
    claim_blocks = (claim->B + block - 1) / block;
    if (claim_blocks > 4096) claim_blocks = 4096;   // the claim job strides
  }
  if (ride) {
    e = grant_lds<&k_sample<LOGK, true, LOOP_NONE>>(tn, bytes);
    if (e != hipSuccess) return e;
    PER_LAUNCH(KID_SAMPLE, (k_sample<LOGK, true, LOOP_NONE>), dim3(gx + claim_blocks + rd.movers, g.T), dim3(block), bytes, s, g, tc, B,
               size, beta, u, out_idx, out_prio, out_w, weight_mode, stale, claim_blocks, claim_here ? *claim : ClaimArgs{},
               claim_here ? claim_mode : (int)CLAIM_NONE, rng, rd);
  } else {
#define PER_SAMPLE(LOOP)                                                                                                       \
  do {                                                                                                                         \
    e = grant_lds<&k_sample<LOGK, false, LOOP>>(tn, bytes);                                                                    \
    if (e != hipSuccess) return e;                                                                                             \
    PER_LAUNCH(KID_SAMPLE, (k_sample<LOGK, false, LOOP>), dim3(gx + claim_blocks + parts, g.T), dim3(block), bytes, s, g, tc, B, size, \
               beta, u, out_idx, out_prio, out_w, weight_mode, stale, claim_blocks, claim_here ? *claim : ClaimArgs{},         \
               claim_here ? claim_mode : (int)CLAIM_NONE, rng, NoRide{});                                                      \
  } while (0)
    if (loop == LOOP_NONE) PER_SAMPLE(LOOP_NONE);
    else if (LOGK <= 3 || loop == LOOP_FEW_ROWS) PER_SAMPLE(LOOP_FEW_ROWS);
    else if constexpr (LOGK > 3) PER_SAMPLE(LOOP_ALL_ROWS);
#undef PER_SAMPLE
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const bool finish_weights = out_w && (gx > 1 || parts);
  if (rows || claim) {   // fused call
    FinishArgs a{};
    a.B = B;
    a.idx = out_idx;
    a.w = finish_weights ? out_w : nullptr;
    a.size = size;
    a.beta = beta;
    a.weight_mode = weight_mode;
    ClaimArgs c2{};
    if (claim) {
      c2 = *claim;
      c2.fold_max = ride ? 1u : 0u;   // the tree pass folds what this kernel has left in max_pend
    }
    if (claim_here) {   // second kernel: tree pass beside the weights and the rows
      if (rows || finish_weights) return launch_tree_finish_k<TREE>(tree, tn, c2, rows, a, claim_mode == CLAIM_BLOCKS, s);
      return launch_tree_k<TREE>(tree, tn, c2, s);
    }
    // second kernel: rows, weights and the claim phase; the tree pass follows
    a.has_claim = claim ? 1u : 0u;
    if (claim) a.claim = c2;
    e = launch_finish(tree, tn, rows, a, s);
    if (e != hipSuccess || !claim) return e;
    return launch_tree_k<TREE>(tree, tn, c2, s);
  }
  if (!finish_weights) return e;
  PER_LAUNCH(KID_WEIGHTS, k_weights, dim3((B + 255) / 256, g.T), dim3(256), 0, s, tree, B, size, beta, out_w, weight_mode);
  return hipGetLastError();
}

// A tree of fanout 2 or 4 as one of fanout 16: every fourth or second height of it.  Where every node is the sum of its children
// a group of sixteen holds the heights in between, the same sums in the same order; the arrays of all heights are a multiple of
// 64 floats apart, zeros beyond the nodes, so its last group is whole.
static Geom of_sixteen(const Geom& g) {
  Geom w = g;
  const uint32_t step = 4u / g.logK;
  w.logK = 4;
  w.K = 16;
  w.H = (g.H + step - 1) / step;
  for (uint32_t h = 0; h <= w.H; ++h) {
    const uint32_t of = h * step < g.H ? h * step : g.H;
    w.n[h] = g.n[of];
    w.stride[h] = g.stride[of];
    w.level[h] = g.level[of];
  }
  return w;
}

// whole_sums: every node is the sum of its children.  A walk in a tree of fanout 2 or 4 then goes by sixteens: a trip to memory and a
// group of its lane in LDS for four (two) heights, where each of them was a trip of its own: 256 samples on 2^20 leaves 9.4 -> 5.9 us
// at K = 2, 4096 7.0 -> 6.4 at K = 4; whole steps, with the faster k_resum_top in front, 512 samples on 607 642 leaves at K = 2 22.9 ->
// 14.5, 2193 on 1 055 898 at K = 4 17.5 -> 15.0; over 90 drawn steps of both fanouts none took longer by more than the runs differ.
// Not where the sampling kernel rebuilds a stale top of such a tree or carries an insertion, nor where it folds the tree's
// minimum (by the real height 1).
// Up to 1024 samples with nothing behind them are one workgroup's, with the weights: 1024 on 131 072 leaves at K = 2 7.1 us by every
// height, 6.0 by sixteens; at K = 4 5.7 and 6.0 from the ninth wave on (512: 4.9 both, of 2^20 leaves 64 4.5 and 4.3).
template <int LOGK>
static hipError_t launch_sample_k(const Geom& g, const Tuning& tn, uint32_t B, uint32_t size, float beta,
                                  const float* u, const RngArgs& rng, uint32_t* out_idx, float* out_w,
                                  float* out_prio, uint32_t weight_mode, uint32_t stale_hb, const FieldTable* rows,
                                  const ClaimArgs* claim, int claim_mode, const InsertRide* ride, bool whole_sums, hipStream_t s) {
  if constexpr (LOGK <= 2) {
    const bool one_workgroup = !rows && !claim && !stale_hb && B > 512u && B <= 1024u;   // of more than eight waves
    bool wide = whole_sums && !ride && !(weight_mode & kWeightMinHere) && g.H * LOGK > 4u && !(LOGK == 2 && one_workgroup);
    if (wide && stale_hb) {
      const SampleShape sh = sample_shape(g, tn, B, stale_hb, rows || claim);
      wide = !sh.tc.nslots || g.H - sh.tc.nslots > stale_hb;
      if (wide) {
        const hipError_t e = launch_resum_top_k<LOGK>(g, tn, stale_hb, s);
        if (e != hipSuccess) return e;
      }
    }
    if (wide)
      return launch_sample_walk<LOGK, 4>(g, of_sixteen(g), tn, B, size, beta, u, rng, out_idx, out_w, out_prio, weight_mode, 0, rows, claim, claim_mode,
                                         nullptr, s);
  }
  return launch_sample_walk<LOGK, LOGK>(g, g, tn, B, size, beta, u, rng, out_idx, out_w, out_prio, weight_mode, stale_hb, rows, claim, claim_mode, ride, s);
}

hipError_t launch_sample(const Geom& g, const Tuning& tn, uint32_t B, uint32_t size, float beta, const float* u,
                         const RngArgs& rng, uint32_t* out_idx, float* out_w, float* out_prio, uint32_t weight_mode,
                         uint32_t stale_hb, const FieldTable* rows, const ClaimArgs* claim, int claim_mode,
                         hipStream_t s, const InsertRide* ride, bool whole_sums) {
#define CALL(L) launch_sample_k<L>(g, tn, B, size, beta, u, rng, out_idx, out_w, out_prio, weight_mode, stale_hb, rows, claim, claim_mode, ride, whole_sums, s)
  PER_DISPATCH_LOGK(g.logK, CALL)
#undef CALL
}

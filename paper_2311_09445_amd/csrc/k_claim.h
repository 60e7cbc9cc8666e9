// First half of a priority update: the claim of leaves by the last writer.
// Part of per_kernels.hip (included inside namespace per, in the order given there); not a stand-alone header.

// ---------------------------------------------------------------------------------
// priority update, first half: claim
// ---------------------------------------------------------------------------------
// Nothing about an update lives on the host (a captured update can be replayed).  The leaf stamps and the
// dirty bits are all zero between update batches: the tree pass that consumes a batch's claims clears
// exactly what the batch has set there (few leaves), so a leaf stamp only orders the elements of one
// batch.  The group entries are not cleared after every batch (that cost 0.5 us of write-back per
// step): their stamps come from a counter in device memory that grows from batch to batch, so an
// entry left by an earlier batch is recognised by its stamp lying below the batch's first.
//
// Leaf by leaf: element j raises the 64-bit stamp of its leaf to (base + j) << 32 | value bits by
// atomic max (base >= 1), and sets the leaf's bit in the dirty mask (one bit per leaf).  The largest j wins
// and carries its value with it.
__device__ __forceinline__ void claim_leaf(const Geom& g, uint32_t t, uint32_t i, uint32_t stamp, uint32_t vbits) {
  atomicMax(reinterpret_cast<unsigned long long*>(g.owner) + (size_t)t * g.owner_stride + i,
            ((unsigned long long)stamp << 32) | vbits);
  atomicOr(&g.dirty[(size_t)t * g.dirty_stride + (i >> 5)], 1u << (i & 31u));
}

// Through group entries: the per-leaf stamps of a large tree live in memory, and a batch spread over
// the tree pays a memory transaction per element to raise them and another to read them back.  A group
// of 32 leaves (64 for K = 64) therefore shares one entry, (stamp << 6 | leaf within the group, value
// bits), in an array small enough to stay in cache.  An element raises its group's entry by a
// returning atomic max.  Only when it meets an element of THIS batch (stamp at or above the batch's
// first) for ANOTHER leaf of the group, the earlier of the two is claimed leaf by leaf instead.
// At the end the entry holds the latest element of the whole group, which is the last writer of
// its leaf; every other leaf's last writer has gone to that leaf's own stamp, where the largest
// stamp wins as before: when it met the entry it either found a later element of another leaf, or
// it was stored and whatever displaced it later (necessarily of another leaf) passed it on.
// Elements for one leaf never need the detour: the later of them dominates the earlier.
// (The stamp has 26 bits here: see kGroupStampTurn.)
__device__ __forceinline__ void claim_in_group(const Geom& g, uint32_t t, uint32_t base, uint32_t j, uint32_t i,
                                               uint32_t vbits) {
  const uint32_t lg = g.logK == 6 ? 6u : 5u;
  const uint32_t slot = i & ((1u << lg) - 1u);
  const uint32_t mine_hi = ((base + j) << 6) | slot;
  const unsigned long long mine = ((unsigned long long)mine_hi << 32) | vbits;
  const unsigned long long old =
      atomicMax(reinterpret_cast<unsigned long long*>(g.nclaim) + (size_t)t * g.nclaim_stride + (i >> lg), mine);
  const uint32_t old_hi = (uint32_t)(old >> 32);
  if ((old_hi >> 6) >= base && (old_hi & 63u) != slot) {
    const bool stays = mine > old;
    const uint32_t out_hi = stays ? old_hi : mine_hi;
    claim_leaf(g, t, (i & ~((1u << lg) - 1u)) | (out_hi & 63u), out_hi >> 6, stays ? (uint32_t)old : vbits);
  }
}

// Dense batches (ClaimArgs::runs: a group gets a quarter of an element or more on the average): consecutive elements of the
// batch for leaves of one group, as a sampled batch has them (it is in leaf order), claim together.  The last of such a
// run raises the group's entry for all of it; the entry then holds the run's length (2 .. 127) with the sign
// bit set, which no valid priority has beside such bits, in place of the value, and the tree pass reads the run's elements
// from the batch.  What is displaced from an entry, or does not get in, goes leaf by leaf as before, element by element if
// it is a run: the lanes of the wave take an element each.  Runs are disjoint pieces of the batch, so the run with the latest
// last element is later than every element of the others.  (One element at a time, 2^20 elements on 2^24 leaves take 1.6
// million atomics of the leaf by leaf form besides 2^20 on the entries: 64 us; the tree pass then picks those leaves' stamps
// up one by one.)
// A wave takes the runs that begin among its 64 elements, to their end among the next 64; only where all of those belong to
// the run do they make one of their own.  So a batch in leaf order whose groups have no more than 64 elements each displaces
// nothing.  (Runs that ended with the wave's elements left the first part of every run on such a border to be displaced, and one
// lane claimed its elements in turn: 2^20 elements on 2^20 leaves 39.4 us at K = 16, 66.2 at K = 64, 8.4 and 9.2 so; on 2^24, 10.5
// both: what its returning atomics take.)
__device__ __forceinline__ uint32_t run_length(uint32_t lo) { return (lo >> 31) && (lo & 0x7FFFFFFFu) >= 2u && (lo & 0x7FFFFFFFu) <= 127u ? lo & 0x7Fu : 1u; }
struct RunElement {
  uint32_t i, vbits, group;
  bool ok;
};
// Element j of the batch, of which i and v are what memory holds (none beyond the batch's end).  What is not valid has a group of
// its own among its 64, so it ends every run.
__device__ __forceinline__ RunElement run_element(const Geom& g, const ClaimArgs& c, uint32_t j, uint32_t i, float v, uint32_t& flags) {
  const bool here = j < c.B, named = here && i < c.size, good = valid_priority(v);
  flags |= here && !named ? 1u : named && !good ? 2u : 0u;
  const bool ok = named && good;
  return RunElement{i, __float_as_uint(v), ok ? i >> (g.logK == 6 ? 6u : 5u) : 0xFFFFFFC0u | (j & 63u), ok};
}
__device__ __forceinline__ unsigned long long group_begins(uint32_t group, uint32_t before, unsigned lane) {   // (before: the group in front of lane 0's)
  const uint32_t below = (uint32_t)__builtin_amdgcn_update_dpp((int)before, (int)group, 0x138 /* wave_shr:1: from the lane below */, 0xF, 0xF, false);
  return __ballot((lane == 0 ? before : below) != group);
}
// Of the elements of a run that stand side by side for one leaf the last dominates the others: a run begins with the last element of its
// first leaf, and one that goes leaf by leaf passes such elements over.  Where most of a run is dominated so its last element claims
// alone, and what dominates before it goes to the leaves' stamps at once: the tree pass would wait for every sixteen elements of the
// run.  (Priorities with a long tail: most of a batch may be for a handful of leaves, whose stamps the elements of displaced runs
// raised one behind the other.  `update` of batches sampled from such priorities, all elements claimed and so: 131 072 on 2^20 leaves at K = 32 51
// and 16.0 us, on 2^21 at K = 64 28.3 and 14.8, 62 033 on 574 707 at K = 16 27.5 and 11.6, 2^18 on 2^22 at K = 8 51 and 17.8, 2^20 on 2^24 at K = 32
// 100 and 38.8.  Batches in no order, whose runs are of one element, pay for what is looked at: 5870 elements of each of 16 trees of 5870
// leaves at K = 4 18.2 us, 17.0 leaf by leaf, 2^18 on 896 794 at K = 8 38.9 both, 2^14 on 70 000 at K = 16 11.4 and 10.4.)
// Most of a run: more than two elements a leaf at K = 32 and 64, where the tree pass has few workgroups, three below.  Dense batches of
// ordinary priorities have 1.3 to 3, and their leaves one by one are as many atomics as before (all as runs, above two and above three: 16 384 of
// each of 64 trees of 8560 leaves at K = 4 28.9, 40.0 and 27.3 us, 326 737 of each of two of 117 667 34.4, 39.0 and 30.5; four elements a
// leaf, 80 000 on 20 000 leaves at K = 8, 36.5, 16.1 and 27.2; 98 000 on 70 000 at K = 32 40.0, 36.1, 40).
// Called by whole waves with their 64 elements, from `first_j` on.  All loads are under way before the first is looked at.
__device__ __forceinline__ void claim_runs(const Geom& g, uint32_t t, const ClaimArgs& c, uint32_t base, uint32_t first_j, uint32_t& mx, uint32_t& flags) {
  const unsigned lane = threadIdx.x & 63u;
  const uint32_t lg = g.logK == 6 ? 6u : 5u;
  const uint32_t* idx = c.idx + (size_t)t * c.B;
  const float* prio = c.prio + (size_t)t * c.B;
  const uint32_t j_mine = first_j + lane, j_next = j_mine + 64u, j_front = first_j ? first_j - 1u : 0u, end = c.B - 1u;
  const uint32_t i_mine = idx[min_u32(j_mine, end)], i_next = idx[min_u32(j_next, end)], i_front = idx[j_front];
  const float v_mine = prio[min_u32(j_mine, end)], v_next = prio[min_u32(j_next, end)], v_front = prio[j_front];
  uint32_t not_here = 0;
  const RunElement mine = run_element(g, c, j_mine, i_mine, v_mine, flags);
  const RunElement next = run_element(g, c, j_next, i_next, v_next, not_here);
  const RunElement before = run_element(g, c, j_front, i_front, v_front, not_here);
  const uint32_t front = first_j ? before.group : 0xFFFFFFFEu;   // (in front of the batch: nothing like any element)
  const uint32_t vb = mine.ok && __uint_as_float(mine.vbits) > 0.0f ? mine.vbits : 0u;
  mx = vb > mx ? vb : mx;
  unsigned long long starts = group_begins(mine.group, front, lane);
  if (!starts) starts = 1;   // (all of one run that began before: a run of its own)
  const unsigned long long next_starts = group_begins(next.group, (uint32_t)__builtin_amdgcn_readlane((int)mine.group, 63), lane);
  const uint32_t beyond = next_starts ? (uint32_t)__builtin_ctzll(next_starts) : 0u;   // elements of the last run among the next 64
  // lanes whose element is for another leaf than the one in front of it (of elements of one run: all of them are valid)
  const unsigned long long leaves = group_begins(mine.i, 0u, lane);
  const unsigned long long next_leaves = group_begins(next.i, (uint32_t)__builtin_amdgcn_readlane((int)mine.i, 63), lane);
  const unsigned long long upto = starts & (~0ull >> (63u - lane));                    // (none: the run began before this wave's elements)
  const bool ends = lane == 63u || ((starts >> (lane + 1u)) & 1u);
  uint32_t i = mine.i, vbits = mine.vbits, j = j_mine, count = 0, of_leaves = 0;
  if (mine.ok && ends && upto) {
    const unsigned start = 63u - (unsigned)__builtin_clzll(upto);
    const unsigned long long later = leaves & (~0ull >> (63u - lane)) & ~(~0ull >> (63u - start));   // leaves that begin behind the run's first
    count = later ? lane - (unsigned)__builtin_ctzll(later) + 2u : 1u;
    of_leaves = 1u + (uint32_t)__popcll(later);
  }
  if (beyond) {
    const uint32_t li = (uint32_t)__builtin_amdgcn_readlane((int)next.i, (int)(beyond - 1u)), lv = (uint32_t)__builtin_amdgcn_readlane((int)next.vbits, (int)(beyond - 1u));
    const unsigned long long later = next_leaves & (~0ull >> (64u - beyond));
    if (lane == 63u && count) {
      i = li;
      vbits = lv;
      j += beyond;
      count = count > 1 ? count + beyond : later ? beyond - (uint32_t)__builtin_ctzll(later) + 1u : 1u;
      of_leaves += (uint32_t)__popcll(later);
    }
  }
  const bool alone = count > 8u + (g.logK <= 4u ? 3u : 2u) * of_leaves;
  if (const unsigned long long split = __ballot(alone)) {   // (a bit per run, at its last lane)
    if (alone) count = 1;
    const unsigned last = lane + (unsigned)__builtin_ctzll(((starts >> 1) | 1ull << 63) >> lane);   // of this lane's run
    const bool to_end = beyond != 0 && (split >> 63);
    if ((split >> last) & 1u && ((lane < last && (leaves >> (lane + 1u)) & 1u) || (lane == 63u && to_end && next_leaves & 1u)))
      claim_leaf(g, t, mine.i, base + j_mine, mine.vbits);
    if (to_end && lane + 1u < beyond && (next_leaves >> (lane + 1u)) & 1u) claim_leaf(g, t, next.i, base + j_next, next.vbits);
  }
  uint32_t out_last = 0, out_n = 0;   // a run that goes leaf by leaf
  if (count) {
    const uint32_t slot = i & ((1u << lg) - 1u);
    const uint32_t mine_hi = ((base + j) << 6) | slot, mine_lo = count > 1 ? 0x80000000u | count : vbits;
    const unsigned long long claim = ((unsigned long long)mine_hi << 32) | mine_lo;
    const unsigned long long old =
        atomicMax(reinterpret_cast<unsigned long long*>(g.nclaim) + (size_t)t * g.nclaim_stride + (i >> lg), claim);
    const uint32_t old_hi = (uint32_t)(old >> 32);
    if ((old_hi >> 6) >= base) {
      const bool stays = claim > old;
      const uint32_t out_hi = stays ? old_hi : mine_hi, out_lo = stays ? (uint32_t)old : mine_lo, n = run_length(out_lo);
      if (n > 1) {
        out_last = (out_hi >> 6) - base;
        out_n = n;
      } else if (!(count == 1 && run_length((uint32_t)old) == 1 && (old_hi & 63u) == slot)) {   // (one leaf: the later of the two dominates)
        claim_leaf(g, t, (i & ~((1u << lg) - 1u)) | (out_hi & 63u), out_hi >> 6, out_lo);
      }
    }
  }
  if (out_n && out_n <= 4u) {   // (short ones, as batches in no order have them: a lane each)
    const uint32_t e0 = out_last + 1u - out_n;
    for (uint32_t e = 0; e < out_n; ++e) claim_leaf(g, t, idx[e0 + e], base + e0 + e, __float_as_uint(prio[e0 + e]));
  }
  for (unsigned long long left = __ballot(out_n > 4u); left; left &= left - 1) {
    const int of = __builtin_ctzll(left);
    const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)out_n, of), e0 = (uint32_t)__builtin_amdgcn_readlane((int)out_last, of) + 1u - n;
    for (uint32_t e = lane; e < n; e += 64u) {
      const uint32_t leaf = idx[e0 + e], above = idx[min_u32(e0 + e + 1u, e0 + n - 1u)];
      const float v = prio[e0 + e];
      if (e + 1u == n || above != leaf) claim_leaf(g, t, leaf, base + e0 + e, __float_as_uint(v));
    }
  }
}

// Does the lane above, which has the next element of the batch, write the same leaf?  Then it is the later writer, and this
// lane need not claim.  (New rows have the largest priority seen so far, so a sampled batch may hold thousands of elements for
// a handful of leaves of one group, side by side, and their atomics on one entry wait for each other: a step of 65 536 with 16 new
// rows on 801 384 leaves at K = 8, priorities spread as a power law, 125 us, 25 so; of 35 774 with 982 new rows on 2^22 at K = 4 226 and
// 31.)  Called by the lanes with a valid element: what a lane that is not among them would hand down is not taken (the
// move leaves kNoElement there, as above the wave's last lane).
__device__ __forceinline__ bool later_writer_above(uint32_t leaf) {
  constexpr uint32_t kNoElement = 0xFFFFFFFFu;
  return (uint32_t)__builtin_amdgcn_update_dpp((int)kNoElement, (int)leaf, 0x130 /* wave_shl:1: from the lane above */, 0xF, 0xF, false) == leaf;
}
// base: the batch's first stamp (group_mode: from the device counter, see claim_base; else 1).
__device__ __forceinline__ void claim_element(const Geom& g, uint32_t t, uint32_t size, uint32_t group_mode,
                                              uint32_t base, uint32_t j, uint32_t i, float v, uint32_t& mx,
                                              uint32_t& flags) {
  if (!(i < size)) flags |= 1u;
  else if (!valid_priority(v)) flags |= 2u;
  else {
    if (later_writer_above(i)) {}
    else if (group_mode) claim_in_group(g, t, base, j, i, __float_as_uint(v));
    else claim_leaf(g, t, i, base + j, __float_as_uint(v));
    const uint32_t vb = v > 0.0f ? __float_as_uint(v) : 0u;
    mx = vb > mx ? vb : mx;
  }
}

// First stamp of the batch being claimed.  Through group entries it is the device counter (stable while the
// claim phase runs: only a tree pass writes it); one lane of the phase (`leader`) leaves it for the
// batch's tree pass.
__device__ __forceinline__ uint32_t claim_base(const Geom& g, uint32_t t, uint32_t group_mode) {
  return group_mode ? read_word_with_the_loads(g.sbase + t) : 1u;
}
// (stores last: the leader's store would otherwise make its wave wait for `base` before it issues its loads)
__device__ __forceinline__ void leave_claim_base(const Geom& g, uint32_t t, uint32_t group_mode, bool leader, uint32_t base) {
  if (group_mode && leader) g.sfloor[t] = base;
}

// Claims elements of the batch, strided over the job's workgroups.  Called by whole workgroups.
// TD: the batch may hold temporal-difference errors to be turned into priorities first (only the
// stand-alone claim kernel carries that code).  RUNS: see claim_runs.
template <bool TD = false, bool RUNS = false>
__device__ __forceinline__ void claim_job(const Geom& g, uint32_t t, const ClaimArgs& c, uint32_t job_block,
                                          uint32_t job_blocks) {
  if (job_block * blockDim.x >= c.B) return;   // nothing to do for this workgroup
  const uint32_t first = claim_base(g, t, c.group_mode);
  const uint32_t max_seen = read_max_bits(g, t);
  uint32_t mx = 0;
  uint32_t flags = 0;
  for (uint32_t base = job_block * blockDim.x; base < c.B; base += job_blocks * blockDim.x) {
    const uint32_t j = base + threadIdx.x;
    if constexpr (RUNS) {
      if (j - (threadIdx.x & 63u) < c.B) claim_runs(g, t, c, first, j - (threadIdx.x & 63u), mx, flags);   // (the same for the wave)
    } else if (j < c.B) {
      float v = c.prio[(size_t)t * c.B + j];
      if constexpr (TD) {
        if (c.from_td)   // priority of a temporal-difference error; a non-finite error stays non-finite and is rejected
          v = (float)pow(fabs((double)v) + c.td_eps, c.td_alpha);
      }
      uint32_t at = j;
      if (c.pos) at = c.pos[(size_t)t * c.B + j];
      const uint32_t i = at < c.B ? c.idx[(size_t)t * c.B + at] : 0xFFFFFFFFu;
      claim_element(g, t, c.size, c.group_mode, first, j, i, v, mx, flags);
    }
  }
  raise_max(g, t, mx, max_seen);
  if (flags) atomicOr(&g.status[t], flags);
  leave_claim_base(g, t, c.group_mode, job_block == 0 && threadIdx.x == 0, first);
}

template <bool RUNS>
__global__ void k_update_claim(Geom g, ClaimArgs c) {
  claim_job<!RUNS, RUNS>(g, blockIdx.y, c, blockIdx.x, gridDim.x);
}

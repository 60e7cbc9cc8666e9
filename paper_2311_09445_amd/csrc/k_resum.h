// Re-summation of node ranges after inserts and of the top heights an update left stale.
// Part of per_kernels.hip (included inside namespace per, in the order given there); not a stand-alone header.

// ---------------------------------------------------------------------------------
// re-summation
// ---------------------------------------------------------------------------------
// Recompute nodes [a, a+count) of height h from their children.  grid (x, T).
template <int LOGK>
__global__ void k_resum_dense(Geom g, uint32_t h, uint32_t a, uint32_t count) {
  constexpr int K = Fan<LOGK>::K;
  constexpr int LPS = Fan<LOGK>::LPS;
  const uint32_t t = blockIdx.y;
  const uint32_t gt = blockIdx.x * blockDim.x + threadIdx.x;
  const uint32_t e = gt / LPS;
  const unsigned q = gt % LPS;
  const bool active = e < count;
  const uint32_t node = a + (active ? e : 0u);
  const float sum = group_sum<LOGK>(g.level[h - 1] + (size_t)t * g.stride[h - 1] + (size_t)node * K, q);
  if (active && q == 0) g.level[h][(size_t)t * g.stride[h] + node] = sum;
}

// One workgroup per tree finishes heights h_start .. H over the node ranges in r (given at
// height h_start and narrowed by K per height).
// The workgroup recomputes the nodes of height h in the two ranges of r from their children.
template <int LOGK>
__device__ __forceinline__ void resum_level(const Geom& g, uint32_t t, uint32_t h, const Range2& r) {
  constexpr int K = Fan<LOGK>::K;
  constexpr int LPS = Fan<LOGK>::LPS;
  const unsigned q = threadIdx.x % LPS;
  const uint32_t grp = threadIdx.x / LPS;
  const uint32_t ngrp = blockDim.x / LPS;
  const float* child = g.level[h - 1] + (size_t)t * g.stride[h - 1];
  float* par = g.level[h] + (size_t)t * g.stride[h];
  for (int part = 0; part < 2; ++part) {
    const uint32_t a = part ? r.a1 : r.a0, b = part ? r.b1 : r.b0;
    for (uint32_t base = a; base < b; base += ngrp) {
      const uint32_t e = base + grp;
      const bool ok = e < b;
      const uint32_t node = ok ? e : a;
      const float sum = group_sum<LOGK>(child + (size_t)node * K, q);
      if (ok && q == 0) par[node] = sum;
    }
  }
}

template <int LOGK>
__global__ void k_resum_tail(Geom g, uint32_t h_start, Range2 r) {
  const uint32_t t = blockIdx.x;
  for (uint32_t h = h_start; h <= g.H; ++h) {
    resum_level<LOGK>(g, t, h, r);
    __syncthreads();
    if (r.b0 > r.a0) { r.a0 >>= LOGK; r.b0 = ((r.b0 - 1) >> LOGK) + 1; }
    if (r.b1 > r.a1) { r.a1 >>= LOGK; r.b1 = ((r.b1 - 1) >> LOGK) + 1; }
  }
}

// A single workgroup handles a height while the groups it must read stay below this many floats.
constexpr uint64_t kTailFloats = 16384;

// Re-sums the heights above `below`, of which the nodes r were rewritten (below = 0: leaf slots).
template <int LOGK>
static hipError_t launch_resum_above_k(const Geom& g, const Tuning& tn, uint32_t below, Range2 r, hipStream_t s) {
  constexpr int K = Fan<LOGK>::K;
  constexpr int LPS = Fan<LOGK>::LPS;
  const uint32_t block = tn.update_block;
  // r holds the rewritten nodes; move to the height above
  uint32_t h = below + 1;
  for (; h <= g.H; ++h) {
    if (r.b0 > r.a0) { r.a0 >>= LOGK; r.b0 = ((r.b0 - 1) >> LOGK) + 1; }
    if (r.b1 > r.a1) { r.a1 >>= LOGK; r.b1 = ((r.b1 - 1) >> LOGK) + 1; }
    const uint64_t nodes = (uint64_t)(r.b0 - r.a0) + (r.b1 - r.a1);
    if (nodes * K <= kTailFloats) break;
    for (int part = 0; part < 2; ++part) {
      const uint32_t a = part ? r.a1 : r.a0, b = part ? r.b1 : r.b0;
      if (b <= a) continue;
      const uint64_t threads = (uint64_t)(b - a) * LPS;
      PER_LAUNCH(KID_RESUM_DENSE, k_resum_dense<LOGK>, dim3((uint32_t)((threads + block - 1) / block), g.T),
                 dim3(block), 0, s, g, h, a, b - a);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  }
  if (h <= g.H) {
    PER_LAUNCH(KID_RESUM_TAIL, k_resum_tail<LOGK>, dim3(g.T), dim3(1024), 0, s, g, h, r);
    return hipGetLastError();
  }
  return hipSuccess;
}

// Every node above height hb, which has at most 4096 (after an update that left them stale).  A lane takes four nodes of
// height hb, the lanes of a wave add up theirs by exchanges, the waves' sums meet in LDS: a binary step after the other, the
// sums of whole children stored on the way: 3.4 us for the 4096 nodes and twelve heights of 2^20 leaves at K = 2, 2.8 at K = 4.  (A
// height after the other from memory, with a barrier behind each: 7.5 and 4.4.)
static_assert(kLazyTopNodes == 4096, "four nodes to a lane, 1024 lanes");
template <int LOGK>
__global__ void __launch_bounds__(1024)
k_resum_top(Geom g, uint32_t hb) {
  __shared__ LevelTable tab;
  __shared__ float s_wave[16];
  const uint32_t t = blockIdx.x, H = g.H, first = 4u * threadIdx.x;
  const unsigned lane = threadIdx.x & 63u;
  fill_level_table(H, t, &tab);
  float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  if (first < g.n[hb]) v = *reinterpret_cast<const float4*>(g.level[hb] + (size_t)t * g.stride[hb] + first);   // (zeros beyond the nodes, to whole 64)
  if (threadIdx.x < 16u) s_wave[threadIdx.x] = 0.0f;
  __syncthreads();
  // the sum of 2^bit nodes of height hb, number `at` of those: a node where that is whole children
  auto node = [&](uint32_t bit, uint32_t at, float sum) {
    if (bit % LOGK) return;
    const uint32_t h = hb + bit / LOGK;
    if (h <= H && at < tab.n[h]) tab.lvl[h][at] = sum;
  };
  const float a = v.x + v.y, b = v.z + v.w;
  node(1, 2 * threadIdx.x, a);
  node(1, 2 * threadIdx.x + 1, b);
  float sum = a + b;
  node(2, threadIdx.x, sum);
  auto pair = [&](uint32_t bit, uint32_t at, unsigned lanes, float other) {
    sum = sum + other;
    if ((lane & (lanes - 1u)) == 0) node(bit, at / lanes, sum);
  };
  pair(3, threadIdx.x, 2, __int_as_float(butterfly_move<0>(__float_as_int(sum))));
  pair(4, threadIdx.x, 4, __int_as_float(butterfly_move<1>(__float_as_int(sum))));
  pair(5, threadIdx.x, 8, __int_as_float(butterfly_move<2>(__float_as_int(sum))));
  pair(6, threadIdx.x, 16, __int_as_float(butterfly_move<3>(__float_as_int(sum))));
  pair(7, threadIdx.x, 32, __shfl_xor(sum, 16));
  pair(8, threadIdx.x, 64, __shfl_xor(sum, 32));
  if (lane == 0) s_wave[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (threadIdx.x >= 16u) return;
  sum = s_wave[lane];
  pair(9, lane, 2, __int_as_float(butterfly_move<0>(__float_as_int(sum))));
  pair(10, lane, 4, __int_as_float(butterfly_move<1>(__float_as_int(sum))));
  pair(11, lane, 8, __int_as_float(butterfly_move<2>(__float_as_int(sum))));
  pair(12, lane, 16, __int_as_float(butterfly_move<3>(__float_as_int(sum))));
  if (lane == 0)
    for (uint32_t h = hb + 12u / LOGK + 1u; h <= H; ++h) tab.lvl[h][0] = sum;   // (one node, all of the above its children)
}

template <int LOGK>
static hipError_t launch_resum_top_k(const Geom& g, const Tuning& tn, uint32_t hb, hipStream_t s) {
  if (hb >= g.H) return hipSuccess;
  const uint32_t lanes = (g.n[hb] + 255u) / 256u * 64u;
  PER_LAUNCH(KID_RESUM_TAIL, k_resum_top<LOGK>, dim3(g.T), dim3(lanes), 0, s, g, hb);
  return hipGetLastError();
}

hipError_t launch_resum_top(const Geom& g, const Tuning& tn, uint32_t hb, hipStream_t s) {
#define CALL(L) launch_resum_top_k<L>(g, tn, hb, s)
  PER_DISPATCH_LOGK(g.logK, CALL)
#undef CALL
}

hipError_t launch_resum_ranges(const Geom& g, const Tuning& tn, Range2 r0, hipStream_t s) {
#define CALL(L) launch_resum_above_k<L>(g, tn, 0, r0, s)
  PER_DISPATCH_LOGK(g.logK, CALL)
#undef CALL
}

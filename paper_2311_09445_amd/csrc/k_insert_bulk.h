// Insertion of many rows: leaves, ancestors and rows in one kernel.
// Part of per_kernels.hip (included inside namespace per, in the order given there); not a stand-alone header.

// ---------------------------------------------------------------------------------
// insertion of many rows
// ---------------------------------------------------------------------------------
// Workgroup b of the first `subtrees` of a tree owns one subtree that the insertion touches (the subtrees of the
// update's tree pass): it writes the new leaves, sums the touched height-1 nodes while it has their leaves in registers,
// and goes up to the subtree's root in LDS.  The workgroups behind them move the rows.  The heights above the subtree
// roots are left to their next reader where an update leaves them too (lazy_top_height), else re-summed by the kernels of
// k_resum.h.  What bounds it is the row traffic when there are rows (2^20 rows of 128 bytes: 49 us, 5.2 TB/s read and
// written), else a chain of two trips to memory and the heights.
// As five kernels (rows, leaves, two or three re-summations) the launches and the trips of each came one after the other:
// 4096 rows of 165 bytes on 2^20 leaves at K = 16: 9.0 us, 4.3 so; 2^20 rows of 128 bytes on 2^24 leaves at K = 32: 68 and 55.
// Rows of an insertion stored whole.  One job per field writes its piece of every row, so the lines of the (contiguous)
// stored rows are written in parts, from workgroups that run at different times.  Here a workgroup takes `R` rows per
// pass: the fields' dense spans of those rows, which are contiguous in the caller's arrays, come in as 16-byte pieces
// (two per lane in flight), are put in their places in LDS, and leave as whole rows, 16 bytes per lane.  Only where every
// field is given (the bytes between fields are written too, as the zeros they are).
// 2^20 rows of five fields (165 bytes, stored 176 apart): 121 us a job per field, 93 so.
constexpr uint32_t kPlaceRows = 64;            // most rows of a pass
constexpr uint32_t kPlaceLds = 16384;          // most staging bytes
constexpr uint64_t kPlaceRowsFrom = 1 << 17;   // rows of a call (all trees) from which this form is taken (65 536 rows: 10.5 us against 9.8)
struct DensePiece {
  uint32_t w[4];
  uint32_t E, at, end, place;                  // bytes per row, first byte in the pass's span, its end, where the field lies in a row
};
__device__ __forceinline__ DensePiece load_dense_piece(const FieldTable& ft, uint32_t rows, uint64_t row0, uint32_t e) {
  const uint8_t* io = nullptr;
  DensePiece p;
  p.E = 1;
  p.place = 0;
  uint32_t first = 0, at = 0;
#pragma unroll
  for (uint32_t f = 0; f < (uint32_t)kMaxFields; ++f) {
    const uint32_t E = f < ft.n_fields ? ft.bytes[f] : 0u, next = first + (rows * E + 15u) / 16u;
    if (e >= first && e < next) {
      io = ft.io[f];
      p.E = E;
      p.place = (uint32_t)(ft.col[f] - ft.col[0]);
      at = e - first;
    }
    first = next;
  }
  p.at = 16u * at;
  p.end = rows * p.E;
  if (p.at + 16u < p.end) p.end = p.at + 16u;
  const uint8_t* src = io + row0 * p.E + p.at;
  if (p.end - p.at == 16u && (reinterpret_cast<uintptr_t>(src) & 3u) == 0) {
    const uint4 x = load_wide(src);
    p.w[0] = x.x;
    p.w[1] = x.y;
    p.w[2] = x.z;
    p.w[3] = x.w;
  } else {
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
      p.w[k] = 0;
#pragma unroll
      for (uint32_t i = 0; i < 4; ++i)
        if (p.at + 4u * k + i < p.end) p.w[k] |= (uint32_t)src[4u * k + i] << (8u * i);
    }
  }
  return p;
}
__device__ __forceinline__ void put_dense_piece(const DensePiece& p, uint32_t RS, uint8_t* stage) {
  uint32_t row = p.at / p.E, off = p.at - row * p.E;
  if ((p.E & 3u) == 0) {
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k)
      if (p.at + 4u * k < p.end) {
        *reinterpret_cast<uint32_t*>(stage + row * RS + p.place + off) = p.w[k];
        off += 4u;
        if (off >= p.E) {
          off = 0;
          ++row;
        }
      }
  } else {
#pragma unroll
    for (uint32_t k = 0; k < 16; ++k)
      if (p.at + k < p.end) {
        stage[row * RS + p.place + off] = (uint8_t)(p.w[k / 4] >> (8u * (k % 4)));
        if (++off >= p.E) {
          off = 0;
          ++row;
        }
      }
  }
}
__device__ __forceinline__ void place_whole_rows(const FieldTable& ft, uint32_t R, uint32_t t, uint32_t n, uint32_t cursor, uint32_t N,
                                                 uint32_t job, uint32_t jobs, uint8_t* stage) {
  const uint32_t RS = ft.row_stride, P = RS / 16u, lane = threadIdx.x, block = blockDim.x;
  uint8_t* base = ft.col[0] + (uint64_t)t * ft.col_stride[0];
  for (uint32_t i = lane; i < R * P; i += block) reinterpret_cast<uint4*>(stage)[i] = make_uint4(0, 0, 0, 0);
  for (uint32_t r0 = job * R; r0 < n; r0 += jobs * R) {
    const uint32_t rows = n - r0 < R ? n - r0 : R;
    uint32_t pieces = 0;
#pragma unroll
    for (uint32_t f = 0; f < (uint32_t)kMaxFields; ++f) pieces += f < ft.n_fields ? (rows * ft.bytes[f] + 15u) / 16u : 0u;
    const uint64_t row0 = (uint64_t)t * n + r0;
    const bool one = lane < pieces, two = lane + block < pieces;
    const DensePiece p0 = load_dense_piece(ft, rows, row0, one ? lane : 0u), p1 = load_dense_piece(ft, rows, row0, two ? lane + block : 0u);
    __syncthreads();   // (the staging bytes are cleared, or the pass before is done with them)
    if (one) put_dense_piece(p0, RS, stage);
    if (two) put_dense_piece(p1, RS, stage);
    for (uint32_t e = lane + 2u * block; e < pieces; e += block) put_dense_piece(load_dense_piece(ft, rows, row0, e), RS, stage);
    __syncthreads();
    for (uint32_t i = lane; i < rows * P; i += block) {
      const uint32_t row = i / P;
      const uint64_t slot = (uint64_t)cursor + r0 + row;
      *reinterpret_cast<uint4*>(base + (slot >= N ? slot - N : slot) * RS + 16u * (i - row * P)) = reinterpret_cast<const uint4*>(stage)[i];
    }
  }
}
// Rows of a pass, or 0 where rows are not stored whole: where a stored row is no longer than a cache line, the parts of a
// line come close enough after each other (2^20 rows of 25 bytes: 33 us a job per field, 72 whole; of 41 bytes 68 and 72).
static uint32_t place_rows(const FieldTable* ft, uint64_t rows) {
  if (!ft || rows < kPlaceRowsFrom || ft->n_fields < 2 || ft->row_stride <= 128) return 0;
  for (uint32_t f = 0; f < ft->n_fields; ++f)
    if (!ft->io[f]) return 0;
  uint32_t R = kPlaceLds / ft->row_stride / 16u * 16u;
  return R > kPlaceRows ? kPlaceRows : R;
}

struct BulkInsert {
  uint32_t n, cursor;
  const float* prio;        // [T][n] or null: the running maximum
  uint32_t* out_idx;        // [T][n] slots written, or null
  uint32_t first_root;      // touched subtree roots: [first_root, first_root + in_first), then from 0 on (the ring wraps)
  uint32_t in_first, subtrees;
  uint32_t track_min;       // also renew min1 of the touched height-1 nodes
  uint32_t whole_rows;      // rows of a pass of place_whole_rows (0: a job per field)
};

template <int LOGK>
__device__ __forceinline__ void insert_job(const Geom& g, const SubLevels& sl, const BulkInsert& a, uint32_t t, uint32_t job) {
  constexpr int K = Fan<LOGK>::K;
  constexpr int LPS = Fan<LOGK>::LPS;
  constexpr int V = LOGK == 1 ? 2 : 4;                // leaves of a node that a lane holds
  using LeafVec = typename std::conditional<LOGK == 1, float2, float4>::type;
  extern __shared__ __attribute__((aligned(16))) float sub[];   // the subtree's nodes of heights 1 .. hb (16-byte LDS accesses need the alignment)
  const uint32_t hb = sl.hb, N = g.N;
  const uint32_t b = job < a.in_first ? a.first_root + job : job - a.in_first;
  const unsigned q = threadIdx.x % LPS;
  const uint32_t grp = threadIdx.x / LPS, ngrp = blockDim.x / LPS;
  const uint32_t lo1 = b << ((hb - 1) * LOGK);
  const uint32_t n1 = sl.n[0], hi1 = min(n1, (b + 1) << ((hb - 1) * LOGK));
  float* lvl1 = sl.ptr[0] + (size_t)t * sl.stride[0];
  float* leaves = g.level[0] + (size_t)t * g.stride[0];
  const float* prio = a.prio ? a.prio + (size_t)t * a.n : nullptr;
  uint32_t* out = a.out_idx ? a.out_idx + (size_t)t * a.n : nullptr;
  const float max_on_entry = prio ? 0.0f : g.max_v[t];
  const uint32_t max_seen = prio ? read_max_bits(g, t) : 0u;
  // row of the insertion that goes to a slot (>= n: none)
  auto row_of = [&](uint32_t slot) -> uint32_t { return slot >= a.cursor ? slot - a.cursor : slot + (N - a.cursor); };
  // Does the insertion touch a leaf of node f?  (its first real slot lies in the ring window, or the window begins in it)
  auto touched = [&](uint32_t f) -> bool { return row_of(f << LOGK) < a.n || (a.cursor >> LOGK) == f; };
  // ---- height 1: the nodes left alone from memory, the others from their leaves
  const uint32_t own = hb > 1 ? sl.lds_off[1] : 1u;
  for (uint32_t i = threadIdx.x; i < sl.lds_floats; i += blockDim.x) {
    const bool node = i < own && lo1 + i < hi1;
    if (node && touched(lo1 + i)) continue;            // (written below)
    sub[i] = node ? lvl1[lo1 + i] : 0.0f;
  }
  uint32_t mx = 0;
  bool bad = false;
  struct Item {
    bool on, all;
    uint32_t f, my, j0;      // my: which of the lane's leaves are written; j0: row of the first, where all are
    LeafVec c;
    float v[V];
  };
  auto fetch = [&](uint32_t f) -> Item {
    Item it;
    it.f = f;
    it.on = f < hi1 && touched(f);
    it.my = 0;
    it.all = true;
    it.c = LeafVec{};
    if (it.on) {
      const uint32_t s0 = (f << LOGK) + (LOGK == 1 ? 0u : 4u * q);
      it.j0 = row_of(s0);
      if (it.j0 < a.n && a.n - it.j0 >= (uint32_t)V && s0 < N && N - s0 >= (uint32_t)V) {   // the usual case: one stretch of rows
        it.my = (1u << V) - 1u;
        if (prio) {
          if constexpr (V == 4) {
            const uint4 w = load_wide(reinterpret_cast<const uint8_t*>(prio + it.j0));
            it.v[0] = __uint_as_float(w.x);
            it.v[1] = __uint_as_float(w.y);
            it.v[2] = __uint_as_float(w.z);
            it.v[3] = __uint_as_float(w.w);
          } else {
            it.v[0] = prio[it.j0];
            it.v[1] = prio[it.j0 + 1];
          }
        }
      } else {
        it.all = false;
#pragma unroll
        for (int k = 0; k < V; ++k) {
          const uint32_t j = s0 + k < N ? row_of(s0 + k) : 0xFFFFFFFFu;
          if (j < a.n) {
            it.my |= 1u << k;
            if (prio) it.v[k] = prio[j];
          }
        }
      }
      if (!it.all || prio) it.c = *reinterpret_cast<const LeafVec*>(leaves + s0);   // (an invalid priority leaves its leaf as it is)
    }
    return it;
  };
  auto finish = [&](Item& it) {
    float c[V];
    if constexpr (LOGK == 1) { c[0] = it.c.x; c[1] = it.c.y; }
    else { c[0] = it.c.x; c[1] = it.c.y; c[2] = it.c.z; c[3] = it.c.w; }
    if (prio) {
#pragma unroll
      for (int k = 0; k < V; ++k) {
        const bool mine = (it.my >> k) & 1u, ok = mine && valid_priority(it.v[k]);
        bad = bad || (mine && !ok);
        c[k] = ok ? it.v[k] : c[k];
        const uint32_t vb = ok && it.v[k] > 0.0f ? __float_as_uint(it.v[k]) : 0u;
        mx = vb > mx ? vb : mx;
      }
    } else {
#pragma unroll
      for (int k = 0; k < V; ++k) c[k] = (it.my >> k) & 1u ? max_on_entry : c[k];
    }
    float sum;
    uint32_t mn = kNoMin;
    const uint32_t s0 = (it.f << LOGK) + (LOGK == 1 ? 0u : 4u * q);
    if constexpr (LOGK == 1) {
      sum = c[0] + c[1];
      if (a.track_min) mn = min_u32(positive_bits(c[0]), positive_bits(c[1]));
      if (it.on && it.my) *reinterpret_cast<float2*>(leaves + s0) = make_float2(c[0], c[1]);
    } else {
      sum = butterfly_sum<Fan<LOGK>::LOGLPS>((c[0] + c[1]) + (c[2] + c[3]));
      if (a.track_min)
        mn = butterfly_min<Fan<LOGK>::LOGLPS>(min_u32(min_u32(positive_bits(c[0]), positive_bits(c[1])), min_u32(positive_bits(c[2]), positive_bits(c[3]))));
      if (it.on && it.my) *reinterpret_cast<float4*>(leaves + s0) = make_float4(c[0], c[1], c[2], c[3]);
    }
    if (it.on && out && it.all && V == 4) {
      store_wide(reinterpret_cast<uint8_t*>(out + it.j0), make_uint4(s0, s0 + 1, s0 + 2, s0 + 3));
    } else if (it.on && out) {
#pragma unroll
      for (int k = 0; k < V; ++k)
        if (it.my & (1u << k)) out[row_of(s0 + k)] = s0 + k;
    }
    if (it.on && q == 0) {
      lvl1[it.f] = sum;
      sub[it.f - lo1] = sum;
      if (a.track_min) g.min1[(size_t)t * g.min1_stride + it.f] = mn;
    }
  };
  // (only the part of the subtree that the window covers is gone through: one or two stretches of nodes)
  const uint32_t w_end = (uint32_t)(((uint64_t)a.cursor + a.n < N ? a.cursor + a.n : N) - 1) >> LOGK;     // last node of the first stretch
  const uint64_t over = (uint64_t)a.cursor + a.n > N ? (uint64_t)a.cursor + a.n - N : 0;                      // slots of the second
  for (int part = 0; part < 2; ++part) {
    if (part == 1 && over == 0) break;
    uint32_t f0 = part ? 0u : a.cursor >> LOGK, f1 = (part ? (uint32_t)((over - 1) >> LOGK) : w_end) + 1;
    if (part && f1 > (a.cursor >> LOGK)) f1 = a.cursor >> LOGK;   // (the node where the window begins and ends is done once)
    if (f0 < lo1) f0 = lo1;
    if (f1 > hi1) f1 = hi1;
    for (uint32_t base = f0; base < f1; base += 2 * ngrp) {
      Item i0 = fetch(base + grp < f1 ? base + grp : 0xFFFFFFFFu);
      if (base + ngrp < f1) {   // (uniform over the workgroup)
        Item i1 = fetch(base + ngrp + grp < f1 ? base + ngrp + grp : 0xFFFFFFFFu);
        finish(i0);
        finish(i1);
      } else {
        finish(i0);
      }
    }
  }
  // ---- heights 2 .. hb of the subtree, from LDS
#pragma unroll
  for (int j = 1; j < kMaxPassHeight<LOGK>; ++j) {
    if ((uint32_t)j < hb) {
      __syncthreads();
      const uint32_t sh = (hb - 1 - (uint32_t)j) * LOGK, first = b << sh;
      const uint32_t cnt = min(sl.n[j], (b + 1) << sh) - first;   // real nodes of this height in the subtree
      float* par = sl.ptr[j] + (size_t)t * sl.stride[j];
      for (uint32_t base = 0; base < cnt; base += ngrp) {
        const uint32_t e = base + grp;
        const bool ok = e < cnt;
        const float sum = group_sum<LOGK>(sub + sl.lds_off[j - 1] + (size_t)(ok ? e : 0u) * K, q);
        if (ok && q == 0) {
          par[first + e] = sum;
          sub[sl.lds_off[j] + e] = sum;
        }
      }
    }
  }
  if (prio) {
    raise_max(g, t, mx, max_seen);
    if (bad) atomicOr(&g.status[t], 2u);
  }
}

template <int LOGK, bool WIDE>
__global__ void __launch_bounds__(1024)
k_insert_bulk(Geom g, SubLevels sl, BulkInsert a, FieldTable ft, JobRanges jr) {
  const uint32_t t = blockIdx.y;
  if (blockIdx.x < a.subtrees) {
    insert_job<LOGK>(g, sl, a, t, blockIdx.x);
    return;
  }
  const uint32_t b = blockIdx.x - a.subtrees, f = job_field(jr, b);
  if (a.whole_rows) {
    extern __shared__ __attribute__((aligned(16))) uint8_t stage[];
    place_whole_rows(ft, a.whole_rows, t, a.n, a.cursor, g.N, b, gridDim.x - a.subtrees, stage);
    return;
  }
  if (f < (uint32_t)kMaxFields)
    rows_job<false, WIDE>(ft, f, t, a.n, nullptr, a.cursor, g.N, g.status, b - jr.first[2 + f], jr.first[3 + f] - jr.first[2 + f]);
}

template <int LOGK>
static hipError_t launch_insert_bulk_k(const Geom& g, const Tuning& tn, const FieldTable* rows, uint32_t n, uint32_t cursor,
                                       const float* prio, uint32_t* out_idx, bool track_min, hipStream_t s) {
  SubLevels sl;
  sub_levels<LOGK>(g, tree_pass_height(g), &sl);
  const uint32_t hb = sl.hb, sh = hb * LOGK;
  BulkInsert a{};
  a.n = n;
  a.cursor = cursor;
  a.prio = prio;
  a.out_idx = out_idx;
  a.track_min = track_min ? 1u : 0u;
  const uint64_t end = (uint64_t)cursor + n;
  const uint32_t roots = g.n[hb], last = (uint32_t)(((end < g.N ? end : g.N) - 1) >> sh);
  a.first_root = cursor >> sh;
  a.in_first = last - a.first_root + 1;
  uint32_t wrapped = end > g.N ? (uint32_t)((end - g.N - 1) >> sh) + 1 : 0;
  if (wrapped > a.first_root) {   // (the ends of the window meet in one subtree: all of them are touched)
    a.first_root = 0;
    a.in_first = roots;
    wrapped = 0;
  }
  a.subtrees = a.in_first + wrapped;
  // a lane group per height-1 node of a subtree, or of what the insertion touches of one
  const uint64_t nodes = hb > 1 ? sl.lds_off[1] : 1, span = ((uint64_t)n >> LOGK) + 2;
  uint64_t block = (nodes < span ? nodes : span) * Fan<LOGK>::LPS;
  block = block > 512 ? 512 : (block + 63) / 64 * 64;
  if (block < 256) block = 256;
  FieldTable ft{};
  if (rows) ft = *rows;
  a.whole_rows = place_rows(rows, (uint64_t)n * g.T);
  const JobRanges jr = job_ranges(rows && !a.whole_rows ? &ft : nullptr, n, (uint32_t)block, 0, 0, g.T);
  const dim3 grid(a.subtrees + (a.whole_rows ? (n + a.whole_rows - 1) / a.whole_rows : jr.first[2 + kMaxFields]), g.T);
  size_t lds = (size_t)sl.lds_floats * 4;
  if (lds < (size_t)a.whole_rows * ft.row_stride) lds = (size_t)a.whole_rows * ft.row_stride;
  if (rows && !a.whole_rows && any_field_moves_wide(&ft)) {
    PER_LAUNCH(KID_INSERT_BULK, (k_insert_bulk<LOGK, true>), grid, dim3((uint32_t)block), lds, s, g, sl, a, ft, jr);
  } else {
    PER_LAUNCH(KID_INSERT_BULK, (k_insert_bulk<LOGK, false>), grid, dim3((uint32_t)block), lds, s, g, sl, a, ft, jr);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || hb >= g.H || lazy_top_height(g, tn)) return e;
  const uint32_t a0 = a.first_root, b0 = a.first_root + a.in_first;
  return launch_resum_above_k<LOGK>(g, tn, hb, Range2{a0, b0, 0, wrapped}, s);
}

hipError_t launch_insert_bulk(const Geom& g, const Tuning& tn, const FieldTable* rows, uint32_t n, uint32_t cursor, const float* prio,
                              uint32_t* out_idx, bool track_min, hipStream_t s) {
#define CALL(L) launch_insert_bulk_k<L>(g, tn, rows, n, cursor, prio, out_idx, track_min, s)
  PER_DISPATCH_LOGK(g.logK, CALL)
#undef CALL
}

// The slots of an insertion by themselves, for calls that return them where they are read from: behind the insertion.
__global__ void __launch_bounds__(256)
k_write_slots(uint32_t n, uint32_t cursor, uint32_t N, uint32_t* __restrict__ out_idx) {
  const uint32_t j = blockIdx.x * 256u + threadIdx.x;
  if (j >= n) return;
  const uint64_t slot = (uint64_t)cursor + j;
  out_idx[(size_t)blockIdx.y * n + j] = (uint32_t)(slot >= N ? slot - N : slot);
}
hipError_t launch_write_slots(const Geom& g, const Tuning& tn, uint32_t n, uint32_t cursor, uint32_t* out_idx, hipStream_t s) {
  PER_LAUNCH(KID_WRITE_SLOTS, k_write_slots, dim3((uint32_t)(((uint64_t)n + 255) / 256), g.T), dim3(256), 0, s, n, cursor, g.N, out_idx);
  return hipGetLastError();
}

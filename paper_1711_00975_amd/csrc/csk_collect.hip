// csk_collect.hip — the candidate pass (Sec. 3.1 item 4: keep the cells whose estimate
// passes a threshold) on gfx950: the Bloom filter of the heavy (row, bucket, sign) items (and the
// exact set of them for the dictionary), built from the counters; the collect kernels, which drop a
// particle whose rows miss the filter and test the rest exactly before inserting its key
// into the candidate set; and their batched forms for many sketches in one set of launches.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "csk_collect_body.h"

namespace csk {

// est(key) >= theta  <=>  at least need = d - floor((d-1)/2) of the d signed row
// estimates are >= theta (Count-Min: all d).  Rows are read until the answer is known.
template <bool TAB_LDS>
__global__ __launch_bounds__(256) void collect_kernel(const float* __restrict__ pos, uint64_t n, Mesh mesh, Tables t,
                                                      const int32_t* __restrict__ M, int32_t theta,
                                                      CandSet cand, uint32_t* err) {
  __shared__ uint32_t tabs_lds[TAB_LDS ? kTabLdsRows * kTableWords : 1];
  const uint32_t* tabs = t.tab;
  if (TAB_LDS) {
    load_tables(tabs_lds, t.tab, t.d);
    __syncthreads();
    tabs = tabs_lds;
  }
  const uint32_t need = t.cm ? t.d : t.d - ((t.d - 1) >> 1);
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    uint64_t key;
    if (!particle_key(pos, i, mesh, key)) {
      atomicOr(err, kErrDomain);
      continue;
    }
    uint32_t pass = 0;
    for (uint32_t r = 0; r < t.d; ++r) {
      if (pass >= need || pass + (t.d - r) < need) break;
      if (row_estimate(tabs + r * kTableWords, M + (uint64_t)r * t.w, t.w, t.cm, key) >= theta) ++pass;
    }
    if (pass >= need) set_insert(cand, key, err);
  }
}

// The candidate pass of a short stream: one particle per thread, every row's counter read at once
// and tested exactly, with no filter to build.  A workgroup's new keys take their places in the list
// with one add to the count: wave by wave those adds, all to one word, took longer than the reads (2.4e5
// particles, 5e4 candidates: 186 us, 26 us so).  That holds back a workgroup's keys, and all of them
// together may hold back a quarter of the slots; a stream that could claim more than there is (n particles
// beside max_cand) lists key by key.
// A key that many particles share claims once per workgroup: of the lanes whose key has the slot of `seen`,
// the first one goes on (2^17 particles of one cell: 0.2 to 1.3 ms with a compare-and-swap each, 20 us so).
template <int MAXD>
__global__ __launch_bounds__(1024) void collect_short_kernel(const float* __restrict__ pos, uint32_t n, Mesh mesh,
                                                            Tables t, const int32_t* __restrict__ M, int32_t theta,
                                                            CandSet cand, uint32_t* err) {
  __shared__ unsigned long long seen[1024];   // a slot per thread
  __shared__ uint32_t found, base, room, some[16];   // some: bit 0 a passing particle of the wave, 1 one outside
  seen[threadIdx.x] = kEmptyKey;
  if (threadIdx.x == 0) found = 0;
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  uint64_t key;
  const bool in = i < n;
  const bool ok = particle_key(pos, in ? i : n - 1, mesh, key) && in;
  const uint32_t need = t.cm ? t.d : t.d - ((t.d - 1) >> 1);
  uint32_t pass = 0;
#pragma unroll
  for (int r = 0; r < MAXD; ++r)
    if ((uint32_t)r < t.d && row_estimate(t.tab + r * kTableWords, M + (uint64_t)r * t.w, t.w, t.cm, key) >= theta) ++pass;
  bool mine = ok && pass >= need;
  const uint32_t of_wave = (__any(mine) ? 1u : 0u) | (__any(in && !ok) ? 2u : 0u);
  if (lane_id() == 0) some[threadIdx.x >> 6] = of_wave;
  __syncthreads();
  uint32_t any = 0;
  for (uint32_t wv = 0; wv < blockDim.x / 64u; ++wv) any |= some[wv];
  if ((any & 2u) && threadIdx.x == 0) atomicOr(err, kErrDomain);   // one a workgroup: all go to one word
  if (!(any & 1u)) return;   // uniform
  if (threadIdx.x == 0) {
    const uint32_t used = set_used(cand);
    room = (uint64_t)used + n <= (uint64_t)cand.max_cand + (cand.slot_mask + 1u) / 4u ? 1u : 2u;
    if (used >= cand.max_cand) room = latched(err, kErrCapacity) ? 3u : 0u;
  }
  if (mine)
    mine = atomicCAS(&seen[(uint32_t)(slot_mix(key) >> 54) & (blockDim.x - 1u)], (unsigned long long)kEmptyKey,
                     (unsigned long long)key) != key;
  __syncthreads();
  if (room == 3u) return;   // uniform: no key can get in, and the error says so
  if (room == 2u) {
    if (mine) set_insert(cand, key, err);
    return;
  }
  const bool is_new = mine && set_claim(cand, key, err, [&]() { return room != 0; }) == kClaimNew;
  const uint32_t at = wave_append(&found, is_new);
  __syncthreads();
  if (threadIdx.x == 0) base = found ? atomicAdd(cand.count, found) : 0u;
  __syncthreads();
  if (is_new) {
    if (base + at < cand.max_cand) cand.list[base + at] = key;
    else atomicOr(err, kErrCapacity);
  }
}

// Items (r, b, sign) with sign * M[r][b] >= theta (Count-Min: M[r][b] >= theta) go into
// the Bloom filter and, when all of them fit, into the exact hot-item set; theta > 0, so
// empty buckets never do.  *hot counts the items.
// Is the signed counter of (r, b, sign) >= theta?  The signed estimate is -M modulo 2^32
// for a negative sign (Count-Min: M itself), exactly as the collect test reads it.
__device__ __forceinline__ void hot_pair(int32_t c, uint32_t cm, int32_t theta, bool valid, bool& hp, bool& hn) {
  hp = valid && c >= theta;
  hn = valid && !cm && ((int32_t)(0u - (uint32_t)c) >= theta);
}

// Loads kFilterVec groups of 4 counters of row r for this thread (16-byte loads when rows
// are 16-byte aligned) before any is tested.
constexpr int kFilterVec = 2;
__device__ __forceinline__ void load_counters(const int32_t* __restrict__ Mr, uint32_t w, uint64_t b0,
                                              int32_t (&c)[kFilterVec][4]) {
  const bool vec = (w & 3u) == 0;
#pragma unroll
  for (int v = 0; v < kFilterVec; ++v) {
    const uint64_t b = b0 + ((uint64_t)v * blockDim.x + threadIdx.x) * 4;
    if (vec && b < w) {
      const int4 q = *(const int4*)(Mr + b);
      c[v][0] = q.x;
      c[v][1] = q.y;
      c[v][2] = q.z;
      c[v][3] = q.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) c[v][e] = (b + e < w) ? Mr[b + e] : 0;
    }
  }
}

// fcols != NULL: the field-probe filter (item fields from the row maps' columns, P prefix
// bits); else the hashed probe of filter_probe().
// Block bx of nbx scans its share of the counters.

// The field-probe filter entries of item (row r, bucket b, sign sg): x = (sg << P) | p for
// every P-bit prefix p of a bucket input h' = h << 1 with umulhi(h', w) = b, i.e.
// h' in [ceil(b 2^32 / w), ceil((b + 1) 2^32 / w) - 1].  For w = 2^P that prefix is b.
__device__ __forceinline__ void field_insert(const uint32_t* __restrict__ cols_r, uint32_t w, uint32_t P, uint32_t b,
                                             uint32_t sg, uint32_t* __restrict__ filter) {
  uint32_t p_lo = b, p_hi = b;
  if ((1u << P) != w) {
    const uint64_t lo = (((uint64_t)b << 32) + w - 1) / w;
    const uint64_t hi = ((((uint64_t)b + 1) << 32) + w - 1) / w - 1;
    p_lo = (uint32_t)(lo >> (32 - P));
    p_hi = (uint32_t)(hi >> (32 - P));
  }
  for (uint32_t p = p_lo; p <= p_hi; ++p) {
    const FilterProbe pr = field_probe(item_field(cols_r, (sg << P) | p));
    atomicOr(&filter[pr.word], pr.mask);
  }
}

__device__ __forceinline__ void hot_insert(uint32_t* table, uint32_t item) {
  uint32_t sl = hot_slot(item);
  for (uint32_t probe = 0; probe < kHotSlots; ++probe) {
    const uint32_t old = atomicCAS(&table[sl], kHotEmpty, item);
    if (old == kHotEmpty || old == item) return;
    sl = (sl + 1) & (kHotSlots - 1);
  }
}

// The most hot items that a filter is used with.
__host__ __device__ __forceinline__ uint32_t filter_most(bool field, uint32_t fspan) {
  return field ? kFieldFilterMaxItems / fspan : kFilterMaxItems;
}

// One scan of the counters builds both the Bloom filter and the exact hot-item set (hot_table, may
// be NULL).  A block gathers the hot items of its counters in LDS and then inserts them with every
// lane busy: item by item where they were found, an insert kept one lane in 64 running through the
// row map's 25 columns.  The first kHotMaxItems items counted go into the set, so that it stays at
// most half full; when there are more, *hot says so and the set is not used.  most: the same for the
// filter.  Bound by the global atomics of the items (64 sketches, 6.6e6 items: about 0.24 ms for one each).
constexpr uint32_t kFilterThreads = 256;
constexpr uint32_t kFilterChunk = kFilterThreads * 4 * kFilterVec;   // counters of one row a block takes at a time
constexpr uint32_t kFilterQueue = 2 * kFilterChunk;

__device__ __forceinline__ void filter_build_body(const int32_t* __restrict__ M, uint32_t d, uint32_t w, uint32_t cm,
                                                  uint32_t bnorm, int32_t theta, const uint32_t* __restrict__ fcols,
                                                  uint32_t P, uint32_t* __restrict__ filter,
                                                  uint32_t* __restrict__ hot, uint32_t* __restrict__ hot_table,
                                                  uint32_t most, uint32_t bx, uint32_t nbx) {
  __shared__ uint64_t queue[kFilterQueue];   // row << 32 | bucket << 1 | sign
  __shared__ uint32_t queued, base;
  __shared__ uint32_t cols[5 * kFieldCols];   // field probes: d <= 5
  const uint32_t per_row = (uint32_t)(((uint64_t)w + kFilterChunk - 1) / kFilterChunk);
  const uint64_t chunks = (uint64_t)d * per_row;
  if (bx >= chunks) return;
  if (threadIdx.x == 0) queued = 0;
  if (fcols)
    for (uint32_t i = threadIdx.x; i < d * kFieldCols; i += kFilterThreads) cols[i] = fcols[i];
  __syncthreads();
  auto drain = [&]() {   // every thread calls it, after a barrier
    const uint32_t nq = queued;
    if (threadIdx.x == 0) base = nq ? atomicAdd(hot, nq) : 0u;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < nq; i += kFilterThreads) {
      const uint64_t it = queue[i];
      const uint32_t r = (uint32_t)(it >> 32), b = (uint32_t)it >> 1, sg = (uint32_t)it & 1u;
      if (base + i >= most) {
        // the filter is not used
      } else if (fcols) {
        field_insert(cols + r * kFieldCols, w, P, b, sg, filter);
      } else {
        const FilterProbe pr = filter_probe(r, b, sg, bnorm);
        atomicOr(&filter[pr.word], pr.mask);
      }
      if (hot_table != nullptr && base + i < kHotMaxItems) hot_insert(hot_table, hot_item(r, b, sg));
    }
    __syncthreads();
    if (threadIdx.x == 0) queued = 0;
    __syncthreads();
  };
  for (uint64_t ch = bx; ch < chunks; ch += nbx) {
    const uint32_t r = (uint32_t)(ch / per_row);
    const uint64_t b0 = (ch % per_row) * (uint64_t)kFilterChunk;
    int32_t c[kFilterVec][4];
    load_counters(M + (uint64_t)r * w, w, b0, c);
#pragma unroll
    for (int v = 0; v < kFilterVec; ++v) {
      const uint64_t b = b0 + ((uint64_t)v * kFilterThreads + threadIdx.x) * 4;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        bool hp, hn;   // never both: theta > 0
        hot_pair(c[v][e], cm, theta, b + e < w, hp, hn);
        if (__any(hp || hn)) {
          const uint32_t at = wave_append(&queued, hp || hn);
          if (hp || hn) queue[at] = (uint64_t)r << 32 | (uint64_t)(b + e) << 1 | (hn ? 1u : 0u);
        }
      }
    }
    __syncthreads();
    if (queued > kFilterQueue - kFilterChunk) drain();   // uniform: read after the barrier
    else __syncthreads();
  }
  drain();
}

__global__ __launch_bounds__(kFilterThreads) void filter_build_kernel(const int32_t* __restrict__ M, uint32_t d,
                                                                      uint32_t w, uint32_t cm, uint32_t bnorm,
                                                                      int32_t theta,
                                                                      const uint32_t* __restrict__ fcols, uint32_t P,
                                                                      uint32_t* __restrict__ filter,
                                                                      uint32_t* __restrict__ hot,
                                                                      uint32_t* __restrict__ hot_table,
                                                                      const uint32_t* __restrict__ gate, uint32_t cap,
                                                                      uint32_t per, uint64_t most, uint32_t most_items) {
  if (gate != nullptr && (uint64_t)min(*gate, cap) * per <= most) return;   // no one will ask the filter
  filter_build_body(M, d, w, cm, bnorm, theta, fcols, P, filter, hot, hot_table, most_items, blockIdx.x, gridDim.x);
}

// Batched forms: blockIdx.y = sketch; a sketch whose call does not use its filter is skipped.
__global__ __launch_bounds__(256) void collect_clear_batch_kernel(const CollectDesc* __restrict__ descs,
                                                                  CollectCall call, uint32_t fw) {
  const uint32_t i = blockIdx.y;
  if (!call.use_filter[i]) return;
  const CollectDesc& c = descs[i];
  const uint64_t total = (uint64_t)fw + 1u;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < total; j += stride) {
    if (j < fw) c.filter[j] = 0u;
    else *c.hot = 0u;
  }
}

__global__ __launch_bounds__(kFilterThreads) void filter_build_batch_kernel(const CollectDesc* __restrict__ descs,
                                                                            CollectCall call, uint32_t field) {
  const uint32_t i = blockIdx.y;
  if (!call.use_filter[i]) return;
  const CollectDesc& c = descs[i];
  filter_build_body(c.M, c.t.d, c.t.w, c.t.cm, c.t.bnorm, call.theta[i], field ? c.t.fcols : nullptr, c.t.fp,
                    c.filter, c.hot, nullptr, filter_most(field, c.t.fspan), blockIdx.x, gridDim.x);
}

// Blocks of a filter build: one per chunk of counters up to 1024 of them, which is what the LDS queues
// let run at once (each adds its hot items to one count).
static uint32_t filter_grid(uint32_t d, uint32_t w) {
  return grid_for((uint64_t)d * (((uint64_t)w + kFilterChunk - 1) / kFilterChunk), 1, 1024);
}

hipError_t launch_filter_build(const Tables& t, const int32_t* M, int32_t theta, uint32_t* filter, uint32_t* hot,
                               uint32_t* hot_table, bool field, hipStream_t s, const uint32_t* gate, uint32_t cap,
                               uint32_t per, uint64_t most) {
  field = field && t.fcols != nullptr;
  FillSpans f{};   // the three clears in one launch
  f.p[0] = filter;
  f.n[0] = field ? kFieldFilterWords : kFilterWords;
  f.p[1] = hot;
  f.n[1] = 1;
  f.p[2] = hot_table;
  f.n[2] = hot_table != nullptr ? kHotSlots : 0;
  f.v[2] = kHotEmpty;
  hipError_t e = launch_fill_spans(f, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(filter_build_kernel, dim3(filter_grid(t.d, t.w)), dim3(kFilterThreads), 0, s, M, t.d, t.w, t.cm,
                     t.bnorm, theta, field ? t.fcols : nullptr, t.fp, filter, hot, hot_table, gate, cap, per, most,
                     filter_most(field, t.fspan));
  return hipGetLastError();
}

static void launch_collect2_d(uint32_t d, uint32_t mode, int hm, dim3 grid, dim3 block, size_t lds, hipStream_t s,
                              const CollectLaunch& c) {
  if (d == 5) launch_collect2_five(mode, hm, grid, block, lds, s, c);
  else if (d < 5) launch_collect2_few(d, mode, hm, grid, block, lds, s, c);
  else launch_collect2_many(d, mode, hm, grid, block, lds, s, c);
}

static size_t collect2_lds_bytes(const Tables& t, bool use_filter, bool field, uint32_t kb) {
  if (t.d != 5) kb = kChars;   // other d hash all six bytes
  if (field) return kb <= 5 ? collect2_lds<true, 5>(4, kFieldFilterWords) : collect2_lds<true, 6>(4, kFieldFilterWords);
  const uint32_t fw = use_filter ? (uint32_t)kFilterWords : 0u;
  return kb <= 5 ? collect2_lds<false, 5>(t.dp, fw) : collect2_lds<false, 6>(t.dp, fw);
}

bool collect_field_form(const Tables& t) {
  return t.d == 5 && t.tabq != nullptr && (t.hash_mode() == kHashPacked || t.hash_mode() == kHashMulHi);
}

bool collect_is_short(uint64_t n, const Tables& t) {
  return t.d <= (uint32_t)kTabLdsRows && n <= kShortStream && n <= (1ull << 19) + t.w / 32u;
}

hipError_t launch_collect_short(const float* pos, uint64_t n, const Mesh& mesh, const Tables& t, const int32_t* M,
                                int32_t theta, const CandSet& cand, uint32_t* err, hipStream_t s) {
  const uint32_t nt = n <= (1u << 16) ? 256u : 1024u;   // few particles: over more CUs
  hipLaunchKernelGGL(collect_short_kernel<kTabLdsRows>, dim3((uint32_t)((n + nt - 1) / nt)), dim3(nt), 0, s, pos,
                     (uint32_t)n, mesh, t, M, theta, cand, err);
  return hipGetLastError();
}

hipError_t launch_collect(const float* pos, uint64_t n, const Mesh& mesh, const Tables& t, const int32_t* M,
                          int32_t theta, const uint32_t* filter, const uint32_t* hot, const CandSet& cand,
                          uint32_t* err, bool field, hipStream_t s) {
  if (t.d <= (uint32_t)kTabLdsRows && mesh.group == 1u) {   // collect2_kernel takes ungrouped keys
    const uint32_t use_filter = (filter != nullptr && hot != nullptr) ? 1u : 0u;
    field = field && use_filter && collect_field_form(t);
    const uint32_t kb = key_bytes_kb(mesh.nch);
    const size_t lds = collect2_lds_bytes(t, use_filter != 0, field, kb);
    const dim3 grid(grid_for((n + kCollectPPT - 1) / kCollectPPT, kCollectThreads, 256)), block(kCollectThreads);
    const CollectDesc cd{mesh, t, M, const_cast<uint32_t*>(filter), const_cast<uint32_t*>(hot),
                         cand, err};
    const CollectLaunch ca{&cd, pos, n, theta, use_filter, field, nullptr, nullptr, nullptr, nullptr, nullptr,
                           kb};
    launch_collect2_d(t.d, mesh.mode, t.hash_mode(), grid, block, lds, s, ca);
  } else {
    hipLaunchKernelGGL(collect_kernel<false>, dim3(grid_for(n, 256, 8192)), dim3(256), 0, s, pos, n, mesh, t, M, theta,
                       cand, err);
  }
  return hipGetLastError();
}

hipError_t launch_collect_batch(const CollectDesc* descs, const CollectDesc* host_descs, uint32_t count,
                                const uint16_t* wg_sketch, const uint32_t* wg_first, const uint32_t* wg_count,
                                uint32_t nwg_total, uint32_t d, uint32_t mesh_mode, int hm, bool field,
                                uint32_t w_max, const CollectCall& call, hipStream_t s) {
  if (count == 0 || nwg_total == 0) return hipSuccess;
  bool any_filter = false;
  size_t lds = 0;
  uint32_t kb = 5;
  for (uint32_t i = 0; i < count; ++i) kb = key_bytes_kb(host_descs[i].mesh.nch) > kb ? key_bytes_kb(host_descs[i].mesh.nch) : kb;
  for (uint32_t i = 0; i < count; ++i) {
    any_filter = any_filter || call.use_filter[i] != 0;
    const size_t b = collect2_lds_bytes(host_descs[i].t, true, field, kb);
    lds = b > lds ? b : lds;
  }
  if (any_filter) {
    const uint32_t fw = field ? kFieldFilterWords : (uint32_t)kFilterWords;
    // the widest sketch decides the grid, so keep it low: the blocks of a narrow one have nothing to do
    const uint32_t most = max(32u, 8192u / count), grid = min(filter_grid(d, w_max), most);
    hipLaunchKernelGGL(collect_clear_batch_kernel, dim3(grid_for((uint64_t)fw + 1, 256, 256), count),
                       dim3(256), 0, s, descs, call, fw);
    hipLaunchKernelGGL(filter_build_batch_kernel, dim3(grid, count), dim3(kFilterThreads), 0, s, descs,
                       call, field ? 1u : 0u);
  }
  const CollectLaunch ca{nullptr, nullptr, 0, 0, 0, field, descs, wg_sketch, wg_first, wg_count, &call, kb};
  launch_collect2_d(d, mesh_mode, hm, dim3(nwg_total), dim3(kCollectThreads), lds, s, ca);
  return hipGetLastError();
}

}  // namespace csk

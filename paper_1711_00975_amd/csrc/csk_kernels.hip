// csk_kernels.hip — gfx950 kernels of the streaming Count-Sketch hot path beside the
// update and the candidate passes, which have files of their own: cell keys, packing, fills, and
// query   (Sec. 2.2 Estimate; Alg. 4 Estimate): lower median of the d signed counters,
// topk    (Sec. 2.2 UpdateHeap; Alg. 1 query): two-stage radix select on
//         (estimate desc, key asc), then an exact rank placement of the k winners.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "csk_kernel_util.h"

namespace csk {

// ------------------------------------------------------------------ keys

__global__ __launch_bounds__(256) void keys_kernel(const float* __restrict__ pos, uint64_t n, Mesh mesh,
                                                   uint64_t* __restrict__ keys) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    uint64_t key;
    keys[i] = particle_key(pos, i, mesh, key) ? key : kEmptyKey;
  }
}

hipError_t launch_keys(const float* pos, uint64_t n, const Mesh& mesh, uint64_t* keys, hipStream_t s) {
  hipLaunchKernelGGL(keys_kernel, dim3(grid_for(n, 256, 8192)), dim3(256), 0, s, pos, n, mesh, keys);
  return hipGetLastError();
}

// Packing: word = qx | qy << 21 | qz << 42 with q = floor(p * 2^21 / L) exactly (the cell
// index of a mesh of 2^21 cells, wrapped), or all ones outside the domain (bit 0 of *err).
__global__ __launch_bounds__(256) void pack_kernel(const float* __restrict__ pos, uint64_t n, Mesh pm,
                                                   uint64_t* __restrict__ out, uint32_t* __restrict__ err) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  bool bad = false;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    int32_t qx, qy, qz;
    const bool ok = (int)cell_index(pos[3 * i], pm, qx) & (int)cell_index(pos[3 * i + 1], pm, qy) &
                    (int)cell_index(pos[3 * i + 2], pm, qz);
    out[i] = ok ? ((uint64_t)(uint32_t)qx | (uint64_t)(uint32_t)qy << kPackBits |
                   (uint64_t)(uint32_t)qz << (2 * kPackBits))
                : kPackedOutside;
    bad |= !ok;
  }
  if (bad) atomicOr(err, 1u);
}

hipError_t launch_pack(const float* pos, uint64_t n, const Mesh& pm, uint64_t* out, uint32_t* err, hipStream_t s) {
  hipLaunchKernelGGL(pack_kernel, dim3(grid_for(n, 256, 8192)), dim3(256), 0, s, pos, n, pm, out, err);
  return hipGetLastError();
}

// ------------------------------------------------------------------ query

// Bound by the random counter reads (d per key, in tables beyond L2; about 5.5e10/s from 320 MiB, 7.3e10/s
// from 20 MiB): the hash tables are staged in LDS, row-interleaved or packed, by few large workgroups
// (3900 small ones staged 30 KiB each), and the counters of all rows of two keys are asked for before any is
// used.  2^20 keys, d = 5: w = 2^20 111 us before, 74 us so; w = 2^24 130 and 101 us.
template <int D, int HM>
__global__ __launch_bounds__(1024) void query_rows_kernel(const uint64_t* __restrict__ keys, uint64_t m, Tables t,
                                                          const int32_t* __restrict__ M, int32_t* __restrict__ est) {
  __shared__ __align__(16) uint32_t ti[kTableWords * HashWords<D, HM>::value];
  stage_tables<HashWords<D, HM>::value>(ti, HM == kHashPacked ? t.tabp : t.tabi, (uint32_t)kChars);
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += 2 * stride) {
    const uint64_t i2 = i + stride;
    const uint64_t key[2] = {keys[i] & 0xFFFFFFFFFFFFull, i2 < m ? keys[i2] & 0xFFFFFFFFFFFFull : 0ull};
    uint32_t c[2][D], ng[2][D];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      uint32_t bk[D];
      rows_bucket_sign_kb<D, HM, kChars>(ti, key[q], t.w, t.wshift, bk, ng[q]);
#pragma unroll
      for (int r = 0; r < D; ++r) c[q][r] = (uint32_t)M[(uint64_t)r * t.w + bk[r]];
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      int32_t v[D];
#pragma unroll
      for (int r = 0; r < D; ++r) v[r] = (int32_t)((ng[q][r] & (t.cm ^ 1u)) ? 0u - c[q][r] : c[q][r]);
      int32_t e;
      if (t.cm) {
        e = v[0];
#pragma unroll
        for (int r = 1; r < D; ++r) e = min(e, v[r]);
      } else {
        e = lower_median<D>(v, D);
      }
      if (q == 0) est[i] = e;
      else if (i2 < m) est[i2] = e;
    }
  }
}

__global__ __launch_bounds__(256) void query_kernel(const uint64_t* __restrict__ keys, uint64_t m, Tables t,
                                                    const int32_t* __restrict__ M, int32_t* __restrict__ est) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride)
    est[i] = estimate_key<32>(t.tab, M, t.d, t.w, t.cm, keys[i] & 0xFFFFFFFFFFFFull);
}

template <int D>
static void launch_query_d(const uint64_t* keys, uint64_t m, const Tables& t, const int32_t* M, int32_t* est,
                           hipStream_t s) {
  const uint32_t nt = m < (1u << 18) ? 256u : 1024u;   // few keys: over more CUs, each reads so many words at a time
  const dim3 grid(grid_for(m, nt, 512)), block(nt);
  const int hm = t.hash_mode();
  if constexpr (D >= 5) {
    if (hm == kHashPacked) {
      hipLaunchKernelGGL((query_rows_kernel<D, kHashPacked>), grid, block, 0, s, keys, m, t, M, est);
      return;
    }
  }
  if (hm == kHashMulHi) hipLaunchKernelGGL((query_rows_kernel<D, kHashMulHi>), grid, block, 0, s, keys, m, t, M, est);
  else hipLaunchKernelGGL((query_rows_kernel<D, kHashShift>), grid, block, 0, s, keys, m, t, M, est);
}

hipError_t launch_query(const uint64_t* keys, uint64_t m, const Tables& t, const int32_t* M, int32_t* est,
                        hipStream_t s) {
  switch (t.d) {
    case 1: launch_query_d<1>(keys, m, t, M, est, s); break;
    case 2: launch_query_d<2>(keys, m, t, M, est, s); break;
    case 3: launch_query_d<3>(keys, m, t, M, est, s); break;
    case 4: launch_query_d<4>(keys, m, t, M, est, s); break;
    case 5: launch_query_d<5>(keys, m, t, M, est, s); break;
    case 6: launch_query_d<6>(keys, m, t, M, est, s); break;
    case 7: launch_query_d<7>(keys, m, t, M, est, s); break;
    case 8: launch_query_d<8>(keys, m, t, M, est, s); break;
    default:
      hipLaunchKernelGGL(query_kernel, dim3(grid_for(m, 256, 8192)), dim3(256), 0, s, keys, m, t, M, est);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------ exact table

// Every key of the router's exact table joins a candidate set.
__global__ __launch_bounds__(256) void table_to_set_kernel(const uint64_t* __restrict__ tk, uint32_t tslots, CandSet cand,
                                                           uint32_t* err) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < tslots; i += gridDim.x * blockDim.x) {
    const uint64_t key = tk[i];
    if (key != kEmptyKey) set_insert(cand, key, err);
  }
}

hipError_t launch_table_to_set(const uint64_t* tk, uint32_t tslots, const CandSet& cand, uint32_t* err, hipStream_t s) {
  hipLaunchKernelGGL(table_to_set_kernel, dim3(grid_for(tslots, 256, 1024)), dim3(256), 0, s, tk, tslots, cand, err);
  return hipGetLastError();
}

// ------------------------------------------------------------------ fills

__global__ void fill_u64_kernel(uint64_t* p, uint64_t n, uint64_t v) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}
__global__ void fill_u32_kernel(uint32_t* p, uint64_t n, uint32_t v) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}
hipError_t launch_fill_u64(uint64_t* p, uint64_t n, uint64_t v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_u64_kernel, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}
hipError_t launch_fill_u32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

// n words of p set to v by the threads i, i + stride, ...: 16 bytes per store between the (fewer
// than four) words before the first 16-byte boundary and those after the last.
__device__ __forceinline__ void fill_span(uint32_t* __restrict__ p, uint64_t n, uint32_t v, uint64_t i, uint64_t stride) {
  using V4 = uint32_t __attribute__((ext_vector_type(4)));
  uint64_t head = ((16u - ((uintptr_t)p & 15u)) & 15u) / 4u;
  head = head < n ? head : n;
  const uint64_t quads = (n - head) / 4, rest = n - head - 4 * quads;
  V4* q = (V4*)(p + head);
  const V4 x = {v, v, v, v};
  for (uint64_t j = i; j < quads; j += stride) q[j] = x;
  if (i < head) p[i] = v;
  if (i < rest) p[head + 4 * quads + i] = v;
}
__global__ __launch_bounds__(256) void fill_spans_kernel(FillSpans f) {
  for (int r = 0; r < kFillSpans; ++r)
    if (f.n[r])
      fill_span(f.p[r], f.n[r], f.v[r], (uint64_t)blockIdx.x * 256 + threadIdx.x, (uint64_t)gridDim.x * 256);
}
__global__ __launch_bounds__(256) void fill_spans_batch_kernel(const ResetSpans* __restrict__ sp) {
  const uint32_t y = blockIdx.y;
  for (int r = 0; r < kFillSpans; ++r)
    if (sp->n[y][r])
      fill_span(sp->p[y][r], sp->n[y][r], sp->v[y][r], (uint64_t)blockIdx.x * 256 + threadIdx.x, (uint64_t)gridDim.x * 256);
}
hipError_t launch_fill_spans_batch(const ResetSpans* spans, uint32_t count, uint64_t max_words, hipStream_t s) {
  if (count == 0 || max_words == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_spans_batch_kernel, dim3(grid_for(max_words, 1024, 1024), count), dim3(256), 0, s, spans);
  return hipGetLastError();
}
hipError_t launch_fill_spans(const FillSpans& f, hipStream_t s) {
  uint64_t total = 0;
  for (int r = 0; r < kFillSpans; ++r) total += f.n[r];
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_spans_kernel, dim3(grid_for(total, 1024, 4096)), dim3(256), 0, s, f);
  return hipGetLastError();
}

// ------------------------------------------------------------------ top-k
//
// Radix select on (estimate desc, key asc) over the candidate list that the inserts keep: three
// digits of the estimate (11 + 11 + 10 bits), four of the key among the ties (12 bits each), one
// launch per digit -- a histogram per block in LDS, summed in device memory, and the block that
// finishes last picks the digit -- then a gather and a rank placement.  A pass is bound by its
// launch and one memory round trip, so the launches are what counts: 9 in place of 28 (compaction
// of the set, a histogram and a pick launch for each of ten 8-bit digits, and five more).  Only as
// many blocks as the candidates need take part; when every tie at the threshold is taken the
// key passes return at once.

constexpr uint32_t kSelThreads = 1024;
constexpr uint32_t kSelItems = 4096;      // candidates per block before another block joins in
constexpr uint32_t kSelGrid = 512;
constexpr uint64_t kOneBlock = 8192;      // candidates at most for the selection in one block
constexpr uint64_t kKeyMax = (1ull << 48) - 1;

__device__ __forceinline__ uint32_t sel_blocks(uint32_t m) {
  const uint32_t b = m / kSelItems + (m % kSelItems ? 1u : 0u);
  return min(max(b, 1u), (uint32_t)gridDim.x);
}

// Exact count of key in the router's table (linear probing from table_slot), or -1.
__device__ __forceinline__ int64_t table_count(const uint64_t* __restrict__ tk, const uint32_t* __restrict__ tc,
                                               uint32_t tmask, uint64_t key) {
  uint32_t sl = table_slot(key, tmask);
  for (uint32_t probe = 0; probe <= tmask; ++probe) {
    const uint64_t k = tk[sl];
    if (k == key) return (int64_t)tc[sl];
    if (k == kEmptyKey) return -1;
    sl = (sl + 1) & tmask;
  }
  return -1;
}

// Is this the last of the `blocks` blocks of a pass to get here?  What the others added to the
// histogram is there when it is: the adds are device-scope atomics, and each wave waits for its
// own before the block counts itself.  (A device-scope fence in every block instead writes back
// the XCD's L2: 350 us a pass for 64 sketches.)  Every thread of the block calls it.
__device__ __forceinline__ bool last_block(SelState* st, uint32_t blocks) {
  __shared__ uint32_t last;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0)
    last = __hip_atomic_fetch_add(&st->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == blocks - 1u ? 1u : 0u;
  __syncthreads();
  return last != 0u;
}

// The bin of a histogram that holds the need-th item: the first whose inclusive count reaches it
// (the last bin, with nothing before it, when none does), the count before it and its own count.
// `global`: the histogram is a pass's, summed by several blocks.  Every thread of the block calls it.
struct SelDigit {
  uint32_t bin, before, here;
};
template <int BITS>
__device__ __forceinline__ SelDigit sel_digit(const uint32_t* hist, bool global, uint32_t need) {
  constexpr uint32_t NB = 1u << BITS, PER = NB / kSelThreads;
  static_assert(PER >= 1 && NB <= kSelBins, "whole bins per thread");
  __shared__ uint32_t wsum[kSelThreads / 64];
  __shared__ SelDigit found;
  const uint32_t tid = threadIdx.x, wave = tid >> 6;
  uint32_t h[PER], sum = 0;
#pragma unroll
  for (uint32_t e = 0; e < PER; ++e) {
    h[e] = global ? __hip_atomic_load(&hist[tid * PER + e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                  : hist[tid * PER + e];
    sum += h[e];
  }
  const uint32_t incl = wave_incl_scan(sum);
  if (lane_id() == 63) wsum[wave] = incl;
  if (tid == 0) found = SelDigit{NB - 1u, 0u, 0u};
  __syncthreads();
  uint32_t cum = incl - sum, total = 0;
  for (uint32_t w = 0; w < kSelThreads / 64; ++w) {
    cum += w < wave ? wsum[w] : 0u;
    total += wsum[w];
  }
  if (need > 0 && need <= total && cum < need && need <= cum + sum) {
    uint32_t e = 0, here = h[0];
#pragma unroll
    for (uint32_t q = 0; q + 1 < PER; ++q)
      if (e == q && cum + h[q] < need) {
        cum += h[q];
        e = q + 1;
        here = h[q + 1];
      }
    found = SelDigit{tid * PER + e, cum, here};
  }
  __syncthreads();
  const SelDigit f = found;
  __syncthreads();   // read before the next call writes it
  return f;
}

// Add the block's histogram to the pass's and, in the last block, pick the digit and move the state
// on (bins are in the order of the selection: estimates descending).  The last block leaves the
// histogram and the block count zero.  FIRST: m and k start the selection.
template <int SHIFT, int BITS, bool KEYS, bool FIRST>
__device__ __forceinline__ void sel_finish_pass(SelState* st, const uint32_t* h, uint32_t m, uint32_t k, uint32_t blocks) {
  constexpr uint32_t NB = 1u << BITS;
  __syncthreads();
  const bool global = blocks > 1;
  if (global) {
    for (uint32_t b = threadIdx.x; b < NB; b += kSelThreads)
      if (h[b]) __hip_atomic_fetch_add(&st->hist[b], h[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!last_block(st, blocks)) return;
  }
  const uint32_t need = FIRST ? min(k, m) : st->k_rem;
  const SelDigit f = sel_digit<BITS>(global ? st->hist : h, global, need);
  if (threadIdx.x == 0) {
    const uint32_t digit = KEYS ? f.bin : NB - 1u - f.bin;
    const uint32_t rem = need - f.before;
    st->k_rem = rem;
    if (!KEYS) {
      st->T = (FIRST ? 0u : st->T) | (digit << SHIFT);
      if (SHIFT == 0) {   // the threshold is known: the key passes are needed when not every tie is taken
        st->ties_all = f.here == rem ? 1u : 0u;
        st->K = f.here == rem ? kKeyMax : 0ull;
      }
    } else {
      st->K |= (uint64_t)digit << SHIFT;
    }
    if (FIRST) {
      st->m = m;
      st->n_sel = 0;
    }
    st->done = 0;
  }
  if (global)
    for (uint32_t b = threadIdx.x; b < NB; b += kSelThreads) st->hist[b] = 0;
}

// First pass of a sketch's top-k: the candidates' estimates from the current counters (with an
// exact table, ov_keys != NULL, a candidate found in it takes its exact count, up to 2^31 - 1) and
// the histogram of their top digit.  The d hash tables (up to 30 KiB) are staged in LDS when there
// are enough candidates to pay for it.
template <int MAXD>
__device__ __forceinline__ void sel_estimate_body(const uint64_t* __restrict__ list, const uint32_t* __restrict__ count,
                                                  uint32_t max_cand, const Tables& t, const int32_t* __restrict__ M,
                                                  uint32_t k, SelState* st, int32_t* __restrict__ ce,
                                                  const uint64_t* __restrict__ ov_keys,
                                                  const uint32_t* __restrict__ ov_counts, uint32_t ov_mask) {
  constexpr bool LDS = MAXD <= kTabLdsRows;
  __shared__ uint32_t tabs_lds[LDS ? kTabLdsRows * kTableWords : 1];
  __shared__ uint32_t h[1 << 11];
  const uint32_t m = min(*count, max_cand), blocks = sel_blocks(m);
  if (blockIdx.x >= blocks) return;
  for (uint32_t b = threadIdx.x; b < (1u << 11); b += kSelThreads) h[b] = 0;
  const bool staged = LDS && m > 8192u;
  if (staged) load_tables(tabs_lds, t.tab, t.d);
  __syncthreads();
  for (uint32_t i = blockIdx.x * kSelThreads + threadIdx.x; i < m; i += blocks * kSelThreads) {
    const uint64_t key = list[i];
    const int64_t exact = ov_keys ? table_count(ov_keys, ov_counts, ov_mask, key) : -1;
    int32_t e;
    if (exact >= 0) e = (int32_t)exact;
    else if (staged) e = estimate_key<MAXD>(tabs_lds, M, t.d, t.w, t.cm, key);
    else e = estimate_key<MAXD>(t.tab, M, t.d, t.w, t.cm, key);
    ce[i] = e;
    atomicAdd(&h[(1u << 11) - 1u - (((uint32_t)e ^ 0x80000000u) >> 21)], 1u);
  }
  sel_finish_pass<21, 11, false, true>(st, h, m, k, blocks);
}

// A pass over given pairs (ck, ce): the histogram of one digit over the current class.
template <int SHIFT, int BITS, bool KEYS, bool FIRST>
__device__ __forceinline__ void sel_pass_body(const uint64_t* __restrict__ ck, const int32_t* __restrict__ ce,
                                              SelState* st, uint32_t k) {
  __shared__ uint32_t h[1 << BITS];
  if (KEYS && st->ties_all) return;
  const uint32_t m = st->m, blocks = sel_blocks(m);
  if (blockIdx.x >= blocks) return;
  const uint32_t T = st->T;
  const uint64_t K = st->K;
  for (uint32_t b = threadIdx.x; b < (1u << BITS); b += kSelThreads) h[b] = 0;
  __syncthreads();
  constexpr uint32_t mask = (1u << BITS) - 1u;
  for (uint64_t i = (uint64_t)blockIdx.x * kSelThreads + threadIdx.x; i < m; i += (uint64_t)blocks * kSelThreads) {
    const uint32_t u = (uint32_t)ce[i] ^ 0x80000000u;
    if constexpr (KEYS) {
      if (u == T) {
        const uint64_t key = ck[i];
        if ((key >> (SHIFT + BITS)) == (K >> (SHIFT + BITS))) atomicAdd(&h[(uint32_t)(key >> SHIFT) & mask], 1u);
      }
    } else {
      bool in = true;
      if constexpr (!FIRST) in = (u >> (SHIFT + BITS)) == (T >> (SHIFT + BITS));
      if (in) atomicAdd(&h[mask - ((u >> SHIFT) & mask)], 1u);
    }
  }
  sel_finish_pass<SHIFT, BITS, KEYS, FIRST>(st, h, m, k, blocks);
}

// Winners: est > T, or est == T and key <= K (T, K from the passes).
__device__ __forceinline__ void sel_gather_body(const uint64_t* __restrict__ ck, const int32_t* __restrict__ ce,
                                                SelState* st, uint32_t k, uint64_t* __restrict__ sk,
                                                int32_t* __restrict__ se) {
  const uint32_t m = st->m, blocks = sel_blocks(m);
  if (blockIdx.x >= blocks || min(k, m) == 0) return;
  const uint32_t T = st->T;
  const uint64_t K = st->K;
  for (uint64_t i0 = (uint64_t)blockIdx.x * kSelThreads; i0 < m; i0 += (uint64_t)blocks * kSelThreads) {
    const uint64_t i = i0 + threadIdx.x;
    bool take = false;
    uint64_t key = 0;
    int32_t e = 0;
    if (i < m) {
      e = ce[i];
      const uint32_t u = (uint32_t)e ^ 0x80000000u;
      take = u >= T;
      if (take) {
        key = ck[i];
        take = u > T || key <= K;
      }
    }
    const uint32_t slot = wave_append(&st->n_sel, take);
    if (take && slot < k) {
      sk[slot] = key;
      se[slot] = e;
    }
  }
}

// Rank of a winner = number of winners ahead of it in (estimate desc, key asc) order; keys are
// distinct, so the ranks are a permutation.  A block places 64 R winners: lane l of each of its 16
// waves compares R of them with the wave's share of every 1024 winners staged in LDS (broadcast
// reads), and the 16 partial counts meet in LDS.  Bound by those n^2 compares, so the usual one is a
// single 64-bit word: the estimate's distance above the smallest winner's (16 bits), then
// 2^48 - 1 - key; winners j come before i when their word is larger.  A staged part with a larger
// distance is compared by (distance, key) in full; one's own larger distance saturates above every
// word of the other parts.  64 sketches of up to 10^4 winners each: 224 us with three compares each, 133 us with one.
// The first block also writes the call's counts: out[0] = min(k, m), out[1] = 1
// (incomplete) when that is below k and the set is partial; *host (pinned, may be NULL) gets m and
// the error latch for a caller that synchronizes.
constexpr uint32_t kRankWide = 4;   // winners per lane when there are many
__device__ __forceinline__ uint64_t rank_word(uint32_t dist, uint64_t k) {
  return dist > 0xFFFFu ? ~0ull : ((uint64_t)dist << 48) | (kKeyMax - k);
}
// The items [i0, i0 + 64 R) at their ranks among n, those below `want` (every thread of the block calls
// it).  T: the smallest item's estimate with its sign flipped.
template <uint32_t R>
__device__ __forceinline__ void rank_block(const uint64_t* __restrict__ sk, const int32_t* __restrict__ se, uint32_t n,
                                           uint32_t T, uint32_t want, uint32_t i0, uint64_t* __restrict__ ok,
                                           int32_t* __restrict__ oe) {
  __shared__ uint64_t tw[kSelThreads];
  __shared__ uint32_t td[kSelThreads];
  __shared__ uint32_t rank[64 * R];
  const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  uint64_t w[R];
  uint32_t cnt[R];
#pragma unroll
  for (uint32_t r = 0; r < R; ++r) {
    const uint32_t i = i0 + 64 * r + lane;
    w[r] = i < n ? rank_word(((uint32_t)se[i] ^ 0x80000000u) - T, sk[i]) : ~0ull;
    cnt[r] = 0;
  }
  if (tid < 64 * R) rank[tid] = 0;
  for (uint32_t j0 = 0; j0 < n; j0 += kSelThreads) {
    __syncthreads();
    const uint32_t j = j0 + tid;
    const uint32_t dist = j < n ? ((uint32_t)se[j] ^ 0x80000000u) - T : 0u;
    const int far = __syncthreads_or(dist > 0xFFFFu);
    tw[tid] = j >= n ? 0ull : far ? kKeyMax - sk[j] : rank_word(dist, sk[j]);   // 0: ahead of nothing
    td[tid] = dist;
    __syncthreads();
    if (n - j0 <= wave * 64u) continue;   // (the barriers above are reached by every thread again)
    if (!far) {
#pragma unroll 4
      for (uint32_t q = wave * 64u; q < wave * 64u + 64u; ++q) {
        const uint64_t x = tw[q];
#pragma unroll
        for (uint32_t r = 0; r < R; ++r) cnt[r] += x > w[r];
      }
    } else {
      uint32_t d[R];
      uint64_t c[R];
#pragma unroll
      for (uint32_t r = 0; r < R; ++r) {
        const uint32_t i = i0 + 64 * r + lane;
        d[r] = i < n ? ((uint32_t)se[i] ^ 0x80000000u) - T : ~0u;
        c[r] = i < n ? kKeyMax - sk[i] : ~0ull;
      }
      for (uint32_t q = wave * 64u; q < wave * 64u + 64u; ++q) {
        const uint64_t x = tw[q];
        const uint32_t e = td[q];
#pragma unroll
        for (uint32_t r = 0; r < R; ++r) cnt[r] += e > d[r] || (e == d[r] && x > c[r]);
      }
    }
  }
#pragma unroll
  for (uint32_t r = 0; r < R; ++r)
    if (cnt[r]) atomicAdd(&rank[64 * r + lane], cnt[r]);
  __syncthreads();
  if (tid < 64 * R && i0 + tid < n && rank[tid] < want) {
    ok[rank[tid]] = sk[i0 + tid];
    oe[rank[tid]] = se[i0 + tid];
  }
  __syncthreads();
}
__device__ __forceinline__ void sel_result(uint32_t m, uint32_t k, const uint32_t* err, uint32_t partial, SelState* st,
                                           uint32_t* out, SelHost* host) {
  const uint32_t bits = *err;
  st->err = bits;
  if (out) {
    out[0] = min(k, m);
    out[1] = (min(k, m) < k && partial) ? 1u : 0u;
  }
  if (host) {
    __hip_atomic_store(&host->m, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&host->err, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}
template <uint32_t R>
__device__ __forceinline__ void sel_rank_body(const uint64_t* __restrict__ sk, const int32_t* __restrict__ se,
                                              SelState* st, uint32_t k, uint64_t* __restrict__ ok,
                                              int32_t* __restrict__ oe, const uint32_t* err, uint32_t partial,
                                              uint32_t* out, SelHost* host) {
  const uint32_t n = min(st->n_sel, k);
  if (blockIdx.x == 0 && threadIdx.x == 0) sel_result(st->m, k, err, partial, st, out, host);
  for (uint32_t i0 = blockIdx.x * 64 * R; i0 < n; i0 += gridDim.x * 64 * R) rank_block<R>(sk, se, n, st->T, n, i0, ok, oe);
}

// The whole selection in one block, for few candidates (any number is right, a large one slow): the
// same passes with their histograms in LDS, then the gather, and the rank placement when k is at
// most kOneRank (else the rank kernel follows).
constexpr uint32_t kOneRank = 1024;
// So few candidates are ranked outright: the square of them takes less than the passes with their barriers
// (the top-100 of a 4093-particle stream: 21.2 us with the passes, 17.6 us so).
constexpr uint32_t kOneDirect = 512;
template <int MAXD>
__global__ __launch_bounds__(kSelThreads) void sel_one_kernel(const uint64_t* __restrict__ list,
                                                              const uint32_t* __restrict__ count, uint32_t max_cand,
                                                              Tables t, const int32_t* __restrict__ M, uint32_t k,
                                                              SelState* st, int32_t* __restrict__ ce,
                                                              uint64_t* __restrict__ sk, int32_t* __restrict__ se,
                                                              uint64_t* __restrict__ ok, int32_t* __restrict__ oe,
                                                              const uint32_t* err, uint32_t partial, uint32_t* out,
                                                              SelHost* host, const uint64_t* __restrict__ ov_keys,
                                                              const uint32_t* __restrict__ ov_counts,
                                                              uint32_t ov_mask) {
  __shared__ uint32_t h[kSelBins];
  __shared__ uint32_t n_sel, lowest;
  const uint32_t tid = threadIdx.x;
  const uint32_t m = min(*count, max_cand);
  const bool direct = m <= kOneDirect && k <= kOneRank;
  if (tid == 0) lowest = ~0u;
  uint32_t need = min(k, m), T = 0;
  uint64_t K = 0;
  auto clear = [&](uint32_t nb) {
    for (uint32_t b = tid; b < nb; b += kSelThreads) h[b] = 0;
    if (tid == 0) n_sel = 0;
    __syncthreads();
  };
  // a thread reads back only the estimates it wrote itself
  clear(1u << 11);
  for (uint32_t i = tid; i < m; i += kSelThreads) {
    const uint64_t key = list[i];
    const int64_t exact = ov_keys ? table_count(ov_keys, ov_counts, ov_mask, key) : -1;
    const int32_t e = exact >= 0 ? (int32_t)exact : estimate_key<MAXD>(t.tab, M, t.d, t.w, t.cm, key);
    ce[i] = e;
    if (direct) atomicMin(&lowest, (uint32_t)e ^ 0x80000000u);
    else atomicAdd(&h[2047u - (((uint32_t)e ^ 0x80000000u) >> 21)], 1u);
  }
  __syncthreads();
  if (direct) {
    if (tid == 0) {
      st->m = m;
      st->n_sel = need;
      sel_result(m, k, err, partial, st, out, host);
    }
    for (uint32_t i0 = 0; i0 < m; i0 += 64 * kRankWide) rank_block<kRankWide>(list, ce, m, lowest, need, i0, ok, oe);
    return;
  }
  SelDigit f = sel_digit<11>(h, false, need);
  T = (2047u - f.bin) << 21;
  need -= f.before;
  clear(1u << 11);
  for (uint32_t i = tid; i < m; i += kSelThreads) {
    const uint32_t u = (uint32_t)ce[i] ^ 0x80000000u;
    if ((u >> 21) == (T >> 21)) atomicAdd(&h[2047u - ((u >> 10) & 2047u)], 1u);
  }
  __syncthreads();
  f = sel_digit<11>(h, false, need);
  T |= (2047u - f.bin) << 10;
  need -= f.before;
  clear(1u << 10);
  for (uint32_t i = tid; i < m; i += kSelThreads) {
    const uint32_t u = (uint32_t)ce[i] ^ 0x80000000u;
    if ((u >> 10) == (T >> 10)) atomicAdd(&h[1023u - (u & 1023u)], 1u);
  }
  __syncthreads();
  f = sel_digit<10>(h, false, need);
  T |= 1023u - f.bin;
  need -= f.before;
  if (f.here == need) {
    K = kKeyMax;
  } else {
#pragma unroll 1
    for (int shift = 36; shift >= 0; shift -= 12) {
      clear(1u << 12);
      for (uint32_t i = tid; i < m; i += kSelThreads) {
        if (((uint32_t)ce[i] ^ 0x80000000u) != T) continue;
        const uint64_t key = list[i];
        if ((key >> (shift + 12)) == (K >> (shift + 12))) atomicAdd(&h[(uint32_t)(key >> shift) & 4095u], 1u);
      }
      __syncthreads();
      f = sel_digit<12>(h, false, need);
      K |= (uint64_t)f.bin << shift;
      need -= f.before;
    }
  }
  clear(0);
  const uint32_t want = min(k, m);
  if (want > 0) {
    for (uint32_t i0 = 0; i0 < m; i0 += kSelThreads) {
      const uint32_t i = i0 + tid;
      bool take = false;
      uint64_t key = 0;
      int32_t e = 0;
      if (i < m) {
        e = ce[i];
        key = list[i];
        const uint32_t u = (uint32_t)e ^ 0x80000000u;
        take = u > T || (u == T && key <= K);
      }
      const uint32_t slot = wave_append(&n_sel, take);
      if (take && slot < k) {
        sk[slot] = key;
        se[slot] = e;
      }
    }
  }
  __syncthreads();
  const uint32_t n = min(n_sel, k);
  if (tid == 0) {
    st->m = m;
    st->n_sel = n;
    st->T = T;   // (the rank kernel's, when it follows)
    sel_result(m, k, err, partial, st, out, host);
  }
  if (k <= kOneRank)
    for (uint32_t i0 = 0; i0 < n; i0 += 64) rank_block<1>(sk, se, n, T, n, i0, ok, oe);
}

// ---- one selection

template <int MAXD>
__global__ __launch_bounds__(kSelThreads) void sel_estimate_kernel(const uint64_t* __restrict__ list,
                                                                   const uint32_t* __restrict__ count,
                                                                   uint32_t max_cand, Tables t,
                                                                   const int32_t* __restrict__ M, uint32_t k,
                                                                   SelState* st, int32_t* __restrict__ ce,
                                                                   const uint64_t* __restrict__ ov_keys,
                                                                   const uint32_t* __restrict__ ov_counts,
                                                                   uint32_t ov_mask) {
  sel_estimate_body<MAXD>(list, count, max_cand, t, M, k, st, ce, ov_keys, ov_counts, ov_mask);
}
template <int SHIFT, int BITS, bool KEYS, bool FIRST>
__global__ __launch_bounds__(kSelThreads) void sel_pass_kernel(const uint64_t* __restrict__ ck,
                                                               const int32_t* __restrict__ ce, SelState* st, uint32_t k) {
  sel_pass_body<SHIFT, BITS, KEYS, FIRST>(ck, ce, st, k);
}
__global__ __launch_bounds__(kSelThreads) void sel_gather_kernel(const uint64_t* __restrict__ ck,
                                                                 const int32_t* __restrict__ ce, SelState* st,
                                                                 uint32_t k, uint64_t* __restrict__ sk,
                                                                 int32_t* __restrict__ se) {
  sel_gather_body(ck, ce, st, k, sk, se);
}
template <uint32_t R>
__global__ __launch_bounds__(kSelThreads) void sel_rank_kernel(const uint64_t* __restrict__ sk,
                                                               const int32_t* __restrict__ se, SelState* st, uint32_t k,
                                                               uint64_t* __restrict__ ok, int32_t* __restrict__ oe,
                                                               const uint32_t* err, uint32_t partial, uint32_t* out,
                                                               SelHost* host) {
  sel_rank_body<R>(sk, se, st, k, ok, oe, err, partial, out, host);
}
// One winner per lane until its blocks fill the card, then four (a quarter of the LDS reads).
static void launch_rank(const uint64_t* sk, const int32_t* se, SelState* st, uint32_t k, uint64_t* ok, int32_t* oe,
                        const uint32_t* err, uint32_t partial, uint32_t* out, SelHost* host, hipStream_t s) {
  if (k <= 16384u)
    hipLaunchKernelGGL((sel_rank_kernel<1>), dim3(grid_for(k, 64, 4096)), dim3(kSelThreads), 0, s, sk, se, st, k, ok, oe,
                       err, partial, out, host);
  else
    hipLaunchKernelGGL((sel_rank_kernel<kRankWide>), dim3(grid_for(k, 64 * kRankWide, 4096)), dim3(kSelThreads), 0, s, sk,
                       se, st, k, ok, oe, err, partial, out, host);
}

// An empty state (a caller's scratch is not cleared) of m pairs: m, or *m_dev clamped to m.
__global__ __launch_bounds__(kSelThreads) void sel_start_kernel(SelState* st, uint32_t m, const uint64_t* m_dev) {
  uint32_t* w = (uint32_t*)st;
  for (uint32_t i = threadIdx.x; i < sizeof(SelState) / 4; i += kSelThreads) w[i] = 0;
  __syncthreads();
  if (threadIdx.x == 0) st->m = m_dev ? (uint32_t)(*m_dev < m ? *m_dev : m) : m;
}

// The passes after the first, the gather and the rank placement.  key_bits: no key has a bit from there up
// (the digits of the tie's key start at 0, so a pass over zero bits can be left out).
static hipError_t select_rest(const uint64_t* ck, const int32_t* ce, uint32_t m_max, uint32_t k, SelState* st,
                              uint64_t* sk, int32_t* se, uint64_t* ok, int32_t* oe, const uint32_t* err,
                              uint32_t partial, uint32_t* out, SelHost* host, uint32_t key_bits, hipStream_t s) {
  const dim3 g(grid_for(m_max, kSelItems, kSelGrid)), b(kSelThreads);
  hipLaunchKernelGGL((sel_pass_kernel<10, 11, false, false>), g, b, 0, s, ck, ce, st, k);
  hipLaunchKernelGGL((sel_pass_kernel<0, 10, false, false>), g, b, 0, s, ck, ce, st, k);
  if (key_bits > 36) hipLaunchKernelGGL((sel_pass_kernel<36, 12, true, false>), g, b, 0, s, ck, ce, st, k);
  hipLaunchKernelGGL((sel_pass_kernel<24, 12, true, false>), g, b, 0, s, ck, ce, st, k);
  hipLaunchKernelGGL((sel_pass_kernel<12, 12, true, false>), g, b, 0, s, ck, ce, st, k);
  hipLaunchKernelGGL((sel_pass_kernel<0, 12, true, false>), g, b, 0, s, ck, ce, st, k);
  hipLaunchKernelGGL(sel_gather_kernel, g, b, 0, s, ck, ce, st, k, sk, se);
  launch_rank(sk, se, st, k, ok, oe, err, partial, out, host, s);
  return hipGetLastError();
}

hipError_t launch_topk(const uint64_t* list, const uint32_t* count, const Tables& t, const int32_t* M,
                       uint32_t max_cand, uint64_t likely, uint32_t k, SelState* st, int32_t* ce, uint64_t* sk, int32_t* se,
                       uint64_t* ok, int32_t* oe, const uint32_t* err, uint32_t partial, uint32_t* out, SelHost* host,
                       uint32_t key_bits, hipStream_t s, const uint64_t* ov_keys, const uint32_t* ov_counts, uint32_t ov_mask) {
  const dim3 g(grid_for(max_cand, kSelItems, kSelGrid)), b(kSelThreads);
  if (likely <= kOneBlock) {
    if (t.d <= (uint32_t)kTabLdsRows)
      hipLaunchKernelGGL((sel_one_kernel<kTabLdsRows>), dim3(1), b, 0, s, list, count, max_cand, t, M, k, st, ce, sk, se,
                         ok, oe, err, partial, out, host, ov_keys, ov_counts, ov_mask);
    else
      hipLaunchKernelGGL((sel_one_kernel<32>), dim3(1), b, 0, s, list, count, max_cand, t, M, k, st, ce, sk, se, ok, oe,
                         err, partial, out, host, ov_keys, ov_counts, ov_mask);
    if (k > kOneRank) launch_rank(sk, se, st, k, ok, oe, err, partial, out, host, s);
    return hipGetLastError();
  }
  if (t.d <= (uint32_t)kTabLdsRows)
    hipLaunchKernelGGL((sel_estimate_kernel<kTabLdsRows>), g, b, 0, s, list, count, max_cand, t, M, k, st, ce, ov_keys,
                       ov_counts, ov_mask);
  else
    hipLaunchKernelGGL((sel_estimate_kernel<32>), g, b, 0, s, list, count, max_cand, t, M, k, st, ce, ov_keys,
                       ov_counts, ov_mask);
  return select_rest(list, ce, max_cand, k, st, sk, se, ok, oe, err, partial, out, host, key_bits, s);
}

static hipError_t select_pairs(const uint64_t* ck, const int32_t* ce, uint32_t m, const uint64_t* m_dev, uint32_t k,
                               SelState* st, uint64_t* sk, int32_t* se, uint64_t* ok, int32_t* oe, const uint32_t* err,
                               hipStream_t s) {
  hipLaunchKernelGGL(sel_start_kernel, dim3(1), dim3(kSelThreads), 0, s, st, m, m_dev);
  hipLaunchKernelGGL((sel_pass_kernel<21, 11, false, true>), dim3(grid_for(m, kSelItems, kSelGrid)), dim3(kSelThreads),
                     0, s, ck, ce, st, k);
  return select_rest(ck, ce, m, k, st, sk, se, ok, oe, err, 0u, nullptr, nullptr, 8 * kChars, s);
}

hipError_t launch_select_pairs_dev(const uint64_t* ck, const int32_t* ce, const uint64_t* m_dev, uint32_t cap,
                                   uint32_t k, SelState* st, uint64_t* sk, int32_t* se, uint64_t* ok,
                                   int32_t* oe, const uint32_t* err, hipStream_t s) {
  return select_pairs(ck, ce, cap, m_dev, k, st, sk, se, ok, oe, err, s);
}

hipError_t launch_select_pairs(const uint64_t* ck, const int32_t* ce, uint32_t m, uint32_t k, SelState* st,
                               uint64_t* sk, int32_t* se, uint64_t* ok, int32_t* oe, const uint32_t* err,
                               hipStream_t s) {
  return select_pairs(ck, ce, m, nullptr, k, st, sk, se, ok, oe, err, s);
}

// ---- the top-k of many sketches at once: block row blockIdx.y serves sketch y of the
// descriptors; per-call k and outputs come by value.

template <int MAXD>
__global__ __launch_bounds__(kSelThreads) void sel_estimate_batch_kernel(const TopkDesc* __restrict__ D, TopkCall call) {
  const TopkDesc& d = D[blockIdx.y];
  sel_estimate_body<MAXD>(d.list, d.count, d.max_cand, d.t, d.M, call.k[blockIdx.y], d.st, d.ce, nullptr, nullptr, 0u);
}
template <int SHIFT, int BITS, bool KEYS>
__global__ __launch_bounds__(kSelThreads) void sel_pass_batch_kernel(const TopkDesc* __restrict__ D, TopkCall call) {
  const TopkDesc& d = D[blockIdx.y];
  sel_pass_body<SHIFT, BITS, KEYS, false>(d.list, d.ce, d.st, call.k[blockIdx.y]);
}
__global__ __launch_bounds__(kSelThreads) void sel_gather_batch_kernel(const TopkDesc* __restrict__ D, TopkCall call) {
  const TopkDesc& d = D[blockIdx.y];
  sel_gather_body(d.list, d.ce, d.st, call.k[blockIdx.y], d.sk, d.se);
}
__global__ __launch_bounds__(kSelThreads) void sel_rank_batch_kernel(const TopkDesc* __restrict__ D, TopkCall call) {
  const uint32_t y = blockIdx.y;
  const TopkDesc& d = D[y];
  sel_rank_body<kRankWide>(d.sk, d.se, d.st, call.k[y], call.keys[y], call.est[y], d.err, call.partial[y], call.out[y], nullptr);
}

hipError_t launch_topk_batch(const TopkDesc* D, uint32_t count, uint32_t d, uint32_t max_cand_max, uint32_t k_max,
                             const TopkCall& call, uint32_t key_bits, hipStream_t s) {
  if (count == 0) return hipSuccess;
  const dim3 g(grid_for(max_cand_max, kSelItems, kSelGrid), count), b(kSelThreads);
  if (d <= (uint32_t)kTabLdsRows)
    hipLaunchKernelGGL((sel_estimate_batch_kernel<kTabLdsRows>), g, b, 0, s, D, call);
  else
    hipLaunchKernelGGL((sel_estimate_batch_kernel<32>), g, b, 0, s, D, call);
  hipLaunchKernelGGL((sel_pass_batch_kernel<10, 11, false>), g, b, 0, s, D, call);
  hipLaunchKernelGGL((sel_pass_batch_kernel<0, 10, false>), g, b, 0, s, D, call);
  if (key_bits > 36) hipLaunchKernelGGL((sel_pass_batch_kernel<36, 12, true>), g, b, 0, s, D, call);
  hipLaunchKernelGGL((sel_pass_batch_kernel<24, 12, true>), g, b, 0, s, D, call);
  hipLaunchKernelGGL((sel_pass_batch_kernel<12, 12, true>), g, b, 0, s, D, call);
  hipLaunchKernelGGL((sel_pass_batch_kernel<0, 12, true>), g, b, 0, s, D, call);
  hipLaunchKernelGGL(sel_gather_batch_kernel, g, b, 0, s, D, call);
  hipLaunchKernelGGL(sel_rank_batch_kernel, dim3(grid_for(k_max, 64 * kRankWide, 1024), count), b, 0, s, D, call);
  return hipGetLastError();
}

}  // namespace csk

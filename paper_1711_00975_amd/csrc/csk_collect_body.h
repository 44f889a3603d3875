// csk_collect_body.h — the collect kernel of the candidate pass (Sec. 3.1 item 4) for sketches of up
// to 8 rows and its batched form, shared by the translation units that compile it for some d each.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "csk_kernel_util.h"

namespace csk {

// One collect launch (or a batch of them): the sketch's descriptor and the per-call stream.
struct CollectLaunch {
  const CollectDesc* c;        // one sketch (kernel argument copy), or NULL for a batch
  const float* pos;
  uint64_t n;
  int32_t theta;
  uint32_t use_filter;
  bool field;
  // batch
  const CollectDesc* descs;
  const uint16_t* wg_sketch;
  const uint32_t* wg_first;
  const uint32_t* wg_count;
  const CollectCall* call;
  uint32_t kb;   // key bytes to look up (d = 5): 5 or 6
};

// The collect kernel of one sketch or a batch for d = 1..4, d = 5 and d = 6..8.
void launch_collect2_few(uint32_t d, uint32_t mode, int hm, dim3 grid, dim3 block, size_t lds, hipStream_t s,
                         const CollectLaunch& c);
void launch_collect2_five(uint32_t mode, int hm, dim3 grid, dim3 block, size_t lds, hipStream_t s, const CollectLaunch& c);
void launch_collect2_many(uint32_t d, uint32_t mode, int hm, dim3 grid, dim3 block, size_t lds, hipStream_t s,
                          const CollectLaunch& c);

namespace collect2 {

// Row-interleaved collect for d <= 8 on an ungrouped mesh.  When a Bloom filter of the hot (row, bucket,
// sign) items is supplied, a particle whose rows pass the filter fewer than `need`
// times cannot have est >= theta (the filter has no false negatives) and is dropped
// without touching the counters; the rest take the exact test.  Each thread loads
// kCollectPPT particles before working on any of them, so that enough position loads
// are in flight to cover HBM latency at one workgroup per CU.
// FP: the field-probe filter (d = 5, w <= 2^24; packed or multiply-high buckets).  Its probe
// tables take the place of the hash tables in LDS and its filter is 2^15 words; the exact
// test of the particles that pass reads the packed or row-interleaved hash tables from
// device memory (all six key bytes).
// Workgroup g of nwg runs the chunks g, g + nwg, ... of the stream.  The sketch's
// arguments are read in place through cp (argument segment or descriptor array).
template <int D, uint32_t MODE, int HM, bool FP, int KB>
__device__ __forceinline__ void collect2_body(const CollectDesc* __restrict__ cp, const float* __restrict__ pos,
                                              uint64_t n, int32_t theta, uint32_t use_filter, uint32_t g,
                                              uint32_t nwg) {
  const CollectDesc& c = *cp;
  const Mesh& mesh = c.mesh;
  const Tables& t = c.t;
  const int32_t* __restrict__ M = c.M;
  const uint32_t* __restrict__ filter = c.filter;
  const uint32_t* __restrict__ hot = c.hot;
  const uint32_t* __restrict__ hot_table = c.hot_table;
  const CandSet& cand = c.cand;
  const uint64_t* set = cand.set;
  const uint32_t slot_mask = cand.slot_mask;
  uint32_t* err = c.err;
  constexpr int DP = FP ? 4 : HashWords<D, HM>::value;
  constexpr int PPT = kCollectPPT;
  constexpr uint32_t FW = FP ? kFieldFilterWords : (uint32_t)kFilterWords;
  static_assert(!FP || (D <= 5 && (HM == kHashPacked || HM == kHashMulHi)),
                "field probes: d <= 5 rows of 25 bits, packed or multiply-high buckets");
  extern __shared__ __align__(16) uint32_t lds3[];
  uint32_t* ti = lds3;
  uint64_t* cache = (uint64_t*)(ti + kTableWords * DP);   // kCollectCache keys
  uint32_t* filt = (uint32_t*)(cache + kCollectCache);
  const uint32_t nhot = use_filter ? *hot : 0xFFFFFFFFu;
  // a hot item takes up to fspan entries of the field-probe filter (1 for w = 2^P)
  const bool uf = use_filter && (FP ? (uint64_t)nhot * t.fspan <= kFieldFilterMaxItems : nhot <= kFilterMaxItems);
  // the exact hot-item set replaces the counter reads when it holds every hot item
  const bool uh = use_filter && hot_table != nullptr && nhot <= kHotMaxItems;
  if (uf) {
    using V4 = uint32_t __attribute__((ext_vector_type(4)));
    static_assert(FW % 4 == 0, "16-byte pieces");
    for (uint32_t i = threadIdx.x; i < FW / 4; i += blockDim.x) ((V4*)filt)[i] = ((const V4*)filter)[i];
  }
  for (uint32_t i = threadIdx.x; i < (uint32_t)kCollectCache; i += blockDim.x) cache[i] = kEmptyKey;
  stage_tables<DP>(ti, FP ? t.tabq : (HM == kHashPacked ? t.tabp : t.tabi), (uint32_t)KB);
  // (bucket, sign) of every row for the exact test: from the staged tables, or (FP) from
  // the packed or row-interleaved tables in device memory over all six key bytes
  auto exact_rows = [&](uint64_t key, uint32_t (&bk)[D], uint32_t (&ng)[D]) {
    if constexpr (FP) rows_bucket_sign_kb<D, HM, kChars>(HM == kHashPacked ? t.tabp : t.tabi, key, t.w, t.wshift, bk, ng);
    else rows_bucket_sign_kb<D, HM, KB>(ti, key, t.w, t.wshift, bk, ng);
  };
  constexpr uint32_t kNeedCS = D - ((D - 1) >> 1);
  const uint32_t need = t.cm ? (uint32_t)D : kNeedCS;
  constexpr uint32_t NT = kCollectThreads;
  const uint64_t chunk = (uint64_t)NT * PPT;
  bool bad = false;
  for (uint64_t first = (uint64_t)g * chunk; first < n; first += (uint64_t)nwg * chunk) {
    const bool full = first + chunk <= n;
    // all PPT position loads are issued before any is used; float records come through a
    // buffer resource over the rest of the stream (loads past it return 0), packed words
    // with a clamped index; particles beyond the stream are masked below
    float px[PPT], py[PPT], pz[PPT];
    uint64_t pw[PPT];
    if constexpr (MODE == kMeshPacked) {
      const uint64_t last = n - 1;
#pragma unroll
      for (int j = 0; j < PPT; ++j) {
        uint64_t i = first + (uint64_t)j * NT + threadIdx.x;
        i = i < last ? i : last;
        pw[j] = __builtin_nontemporal_load((const uint64_t*)pos + i);
      }
    } else {
      const __amdgpu_buffer_rsrc_t span = byte_span(pos + 3 * first, (n - first) * 12);
#pragma unroll
      for (int j = 0; j < PPT; ++j) load_xyz(span, 12u * threadIdx.x, 12u * (uint32_t)j * NT, px[j], py[j], pz[j]);
    }
    // Nearly always every particle of the wave is in [0, L), which needs no wrap and no domain test.
    bool plain = false;
    if constexpr (MODE != kMeshPacked) {
      bool all = full;
#pragma unroll
      for (int j = 0; j < PPT; ++j) all = all && inside_box(px[j], py[j], pz[j], mesh);
      plain = __all(all);
    }
    // keys and the filter verdict of all PPT particles, without branches
    uint64_t keys[PPT];
    uint32_t maybe = 0;
    auto verdict = [&](int j, bool go) {
      if (uf) {
        uint32_t fp = 0;
        if constexpr (FP) {
          uint32_t q[4];
          row_hashes_kb<4, KB>(ti, keys[j], q);
#pragma unroll
          for (int r = 0; r < D; ++r) fp += field_hit(filt, field_bits<kFieldBits>(q, r));
        } else {
          uint32_t bk[D], sg[D];
          rows_bucket_sign_kb<D, HM, KB>(ti, keys[j], t.w, t.wshift, bk, sg);
#pragma unroll
          for (int r = 0; r < D; ++r) {
            const uint32_t ng = sg[r] & (t.cm ^ 1u);
            const FilterProbe pr = filter_probe((uint32_t)r, bk[r], ng, t.bnorm);
            fp += ((filt[pr.word] & pr.mask) == pr.mask) ? 1u : 0u;
          }
        }
        go = go && fp >= need;
      }
      maybe |= (uint32_t)go << j;
    };
    if (plain) {
      if constexpr (MODE != kMeshPacked) {
#pragma unroll
        for (int j = 0; j < PPT; ++j)
          keys[j] = cell_key_of((int32_t)cell_index_inside<MODE>(px[j], mesh), (int32_t)cell_index_inside<MODE>(py[j], mesh),
                                (int32_t)cell_index_inside<MODE>(pz[j], mesh), mesh);
      }
    }
    uint32_t fine = plain ? (1u << PPT) - 1u : 0u;
    if (!plain) {
#pragma unroll
      for (int j = 0; j < PPT; ++j) {
        const bool in = full || (first + (uint64_t)j * NT + threadIdx.x) < n;
        bool ok;
        if constexpr (MODE == kMeshPacked) ok = packed_key<false>(pw[j], mesh, keys[j]);
        else ok = cell_key_m<MODE, false>(px[j], py[j], pz[j], mesh, keys[j]);
        bad |= in && !ok;
        fine |= (uint32_t)(in && ok) << j;
      }
    }
#pragma unroll
    for (int j = 0; j < PPT; ++j) verdict(j, (fine >> j) & 1u);
    // The particles that may pass.  A key seen recently by this workgroup, or already in the
    // set, needs no exact test: heavy cells repeat thousands of times, and the set only ever
    // gains keys.  The first set slot of every candidate is loaded before any is compared,
    // so that the thread waits on one round trip for all its keys rather than one per key.
    auto cache_slot = [](uint64_t key) { return (uint32_t)(key ^ (key >> 21)) & (kCollectCache - 1); };
    uint32_t todo = maybe;
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
      if ((todo >> j) & 1u)
        if (__hip_atomic_load(&cache[cache_slot(keys[j])], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == keys[j])
          todo &= ~(1u << j);
    }
    // the first slot of each key's probe sequence in the set
    uint64_t s0[PPT];
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
      s0[j] = kEmptyKey;
      if ((todo >> j) & 1u) s0[j] = set[(uint32_t)slot_mix(keys[j]) & slot_mask];
    }
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
      if (!((todo >> j) & 1u)) continue;
      bool in = s0[j] == keys[j];
      if (!in && s0[j] != kEmptyKey) in = set_contains(set, slot_mask, keys[j]);   // a longer probe run
      if (in) {
        __hip_atomic_store(&cache[cache_slot(keys[j])], keys[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        todo &= ~(1u << j);
      }
    }
    // Other threads of the workgroup may have inserted a key since the first cache check;
    // looking again before the exact test spares it (one LDS read).
    auto recheck = [&](uint64_t key) {
      return __hip_atomic_load(&cache[cache_slot(key)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == key;
    };
    // The exact test of the rest.  With the hot-item set (2 MiB, resident in L2) the first
    // slot of every row of a group of keys (four for d <= 5, else two) is loaded before any
    // is compared.  Without it the counters are read row by row until the answer is known;
    // in a large table those reads go to HBM, and reading all d rows at once was no faster.
    if (uh) {
      constexpr int GQ = D <= 5 ? 4 : 2;
      static_assert(PPT % GQ == 0, "whole groups of keys");
#pragma unroll
      for (int j0 = 0; j0 < PPT; j0 += GQ) {
        if (!((todo >> j0) & ((1u << GQ) - 1u))) continue;
        uint32_t item[GQ][D], v[GQ][D];
#pragma unroll
        for (int q = 0; q < GQ; ++q) {
          if (!((todo >> (j0 + q)) & 1u)) continue;
          if (recheck(keys[j0 + q])) {
            todo &= ~(1u << (j0 + q));
            continue;
          }
          uint32_t bk[D], ng[D];
          exact_rows(keys[j0 + q], bk, ng);
#pragma unroll
          for (int r = 0; r < D; ++r) {
            item[q][r] = hot_item((uint32_t)r, bk[r], ng[r] & (t.cm ^ 1u));
            v[q][r] = hot_table[hot_slot(item[q][r])];
          }
        }
#pragma unroll
        for (int q = 0; q < GQ; ++q) {
          const int j = j0 + q;
          if (!((todo >> j) & 1u)) continue;
          // row r passes (sign * M >= theta) exactly when its item is in the hot set
          uint32_t pass = 0;
#pragma unroll
          for (int r = 0; r < D; ++r) {
            bool hit = v[q][r] == item[q][r];
            if (!hit && v[q][r] != kHotEmpty) {
              uint32_t sl = (hot_slot(item[q][r]) + 1) & (kHotSlots - 1);
              for (uint32_t probe = 1; probe < kHotSlots; ++probe) {
                const uint32_t x = hot_table[sl];
                if (x == item[q][r]) {
                  hit = true;
                  break;
                }
                if (x == kHotEmpty) break;
                sl = (sl + 1) & (kHotSlots - 1);
              }
            }
            pass += hit ? 1u : 0u;
          }
          if (pass >= need) {
            set_insert(cand, keys[j], err);
            __hip_atomic_store(&cache[cache_slot(keys[j])], keys[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < PPT; ++j) {
        if (!((todo >> j) & 1u) || recheck(keys[j])) continue;
        uint32_t bk[D], ng[D];
        exact_rows(keys[j], bk, ng);
        uint32_t pass = 0;
#pragma unroll
        for (int r = 0; r < D; ++r) {
          if (pass >= need || pass + (uint32_t)(D - r) < need) break;
          const uint32_t c = (uint32_t)M[(uint64_t)r * t.w + bk[r]];
          if ((int32_t)((ng[r] & (t.cm ^ 1u)) ? 0u - c : c) >= theta) ++pass;
        }
        if (pass >= need) {
          set_insert(cand, keys[j], err);
          __hip_atomic_store(&cache[cache_slot(keys[j])], keys[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      }
    }
  }
  if (bad) atomicOr(err, kErrDomain);
}

template <int D, uint32_t MODE, int HM, bool FP, int KB>
__global__ __launch_bounds__(kCollectThreads) void collect2_kernel(CollectDesc c, const float* __restrict__ pos,
                                                                   uint64_t n, int32_t theta, uint32_t use_filter) {
  collect2_body<D, MODE, HM, FP, KB>(&c, pos, n, theta, use_filter, blockIdx.x, gridDim.x);
}

// Many sketches' candidate passes in one launch: workgroup blockIdx.x serves sketch
// wg_sketch[blockIdx.x] as its workgroup blockIdx.x - wg_first[sketch] of wg_count[sketch].
template <int D, uint32_t MODE, int HM, bool FP, int KB>
__global__ __launch_bounds__(kCollectThreads) void collect2_batch_kernel(const CollectDesc* __restrict__ descs,
                                                                         const uint16_t* __restrict__ wg_sketch,
                                                                         const uint32_t* __restrict__ wg_first,
                                                                         const uint32_t* __restrict__ wg_count,
                                                                         CollectCall call) {
  const uint32_t i = wg_sketch[blockIdx.x];
  collect2_body<D, MODE, HM, FP, KB>(descs + i, call.pos[i], call.n[i], call.theta[i], call.use_filter[i],
                                     blockIdx.x - wg_first[i], wg_count[i]);
}

template <int D, uint32_t MM, int HM, bool FP, int KB>
void launch_collect2_kb(dim3 grid, dim3 block, size_t lds, hipStream_t s, const CollectLaunch& c) {
  if (c.c != nullptr)
    hipLaunchKernelGGL((collect2_kernel<D, MM, HM, FP, KB>), grid, block, lds, s, *c.c, c.pos, c.n, c.theta,
                       c.use_filter);
  else
    hipLaunchKernelGGL((collect2_batch_kernel<D, MM, HM, FP, KB>), grid, block, lds, s, c.descs, c.wg_sketch,
                       c.wg_first, c.wg_count, *c.call);
}

// d = 5 hashes exactly the key bytes its mesh needs (5 below 2^40, else 6); other d all six.
template <int D, uint32_t MM, int HM, bool FP = false>
void launch_collect2_one(dim3 grid, dim3 block, size_t lds, hipStream_t s, const CollectLaunch& c) {
  if constexpr (D == 5) {
    if (c.kb == 5) {
      launch_collect2_kb<D, MM, HM, FP, 5>(grid, block, lds, s, c);
      return;
    }
  }
  launch_collect2_kb<D, MM, HM, FP, kChars>(grid, block, lds, s, c);
}

template <int D, uint32_t MM>
void launch_collect2_m(int hm, dim3 grid, dim3 block, size_t lds, hipStream_t s, const CollectLaunch& c) {
  if constexpr (D == 5) {
    if (hm == kHashPacked && c.field) {
      launch_collect2_one<D, MM, kHashPacked, true>(grid, block, lds, s, c);
      return;
    }
    if constexpr (MM != kMeshPacked) {
      if (hm == kHashMulHi && c.field) {
        launch_collect2_one<D, MM, kHashMulHi, true>(grid, block, lds, s, c);
        return;
      }
    }
  }
  if constexpr (D >= 5) {
    if (hm == kHashPacked) {
      launch_collect2_one<D, MM, kHashPacked>(grid, block, lds, s, c);
      return;
    }
  }
  if (hm == kHashMulHi) launch_collect2_one<D, MM, kHashMulHi>(grid, block, lds, s, c);
  else launch_collect2_one<D, MM, kHashShift>(grid, block, lds, s, c);
}

template <int D>
void launch_collect2_dm(uint32_t mode, int hm, dim3 grid, dim3 block, size_t lds, hipStream_t s,
                               const CollectLaunch& c) {
  if (mode == kMeshPacked) launch_collect2_m<D, kMeshPacked>(hm, grid, block, lds, s, c);
  else if (mode == kMeshPow2Ratio) launch_collect2_m<D, kMeshPow2Ratio>(hm, grid, block, lds, s, c);
  else if (mode == kMeshExactRatio) launch_collect2_m<D, kMeshExactRatio>(hm, grid, block, lds, s, c);
  else launch_collect2_m<D, kMeshGeneral>(hm, grid, block, lds, s, c);
}


}  // namespace collect2
}  // namespace csk

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

// LDS of a collect workgroup: the hash (or probe) tables of kb key bytes, dw words an entry, the cache of
// inserted keys, a queue of 64 keys (6 bytes each) per wave, the new keys that are not in the list yet
// (with four control words), and the filter.  With the field-probe filter's 128 KiB the cache and the new
// keys get what is left of the 160 KiB.
constexpr int kCollectCache = 1024;
template <bool FP, int KB>
constexpr uint32_t collect2_cache() {
  return FP ? (KB <= 5 ? 512u : 128u) : (uint32_t)kCollectCache;
}
template <bool FP, int KB>
constexpr uint32_t collect2_fresh() {
  return FP && KB > 5 ? 126u : 254u;
}
template <bool FP, int KB>
constexpr size_t collect2_lds(uint32_t dw, uint32_t filter_words) {
  return (size_t)KB * 1024 * dw + collect2_cache<FP, KB>() * 8ull + (kCollectThreads / 64) * 64 * 6ull +
         collect2_fresh<FP, KB>() * 8ull + 16ull + filter_words * 4ull;
}
static_assert(collect2_lds<true, 6>(4, kFieldFilterWords) <= 160 * 1024 &&
                  collect2_lds<true, 5>(4, kFieldFilterWords) <= 160 * 1024 &&
                  collect2_lds<false, 6>(8, kFilterWords) <= 160 * 1024,
              "one workgroup's LDS");

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
  constexpr uint32_t CE = collect2_cache<FP, KB>();
  constexpr uint32_t kWaves = kCollectThreads / 64u;
  uint32_t* ti = lds3;
  uint64_t* cache = (uint64_t*)(ti + KB * 256 * DP);   // CE keys
  const uint32_t lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t* qlo = (uint32_t*)(cache + CE) + 64u * wave;   // this wave's queue of 64 keys: low words, then high halves
  uint16_t* qhi = (uint16_t*)((uint32_t*)(cache + CE) + 64u * kWaves) + 64u * wave;
  constexpr uint32_t NF = collect2_fresh<FP, KB>();
  uint64_t* fresh = (uint64_t*)((uint32_t*)(cache + CE) + 96u * kWaves);   // NF new keys
  // All workgroups together hold back at most a quarter of the slots: the set stays a table with room.
  const uint32_t hold = min(NF, (slot_mask + 1u) / (4u * nwg));
  // ctl: slots of fresh handed out, the first ones refused (all after are), a key was refused by the set, the
  // set was full before this call (in the end: list base)
  uint32_t* ctl = (uint32_t*)(fresh + NF);
  uint32_t* filt = ctl + 4;
  const uint32_t nhot = use_filter ? *hot : 0xFFFFFFFFu;
  // a hot item takes up to fspan entries of the field-probe filter (1 for w = 2^P)
  const bool uf = use_filter && (FP ? (uint64_t)nhot * t.fspan <= kFieldFilterMaxItems : nhot <= kFilterMaxItems);
  if (uf) {
    using V4 = uint32_t __attribute__((ext_vector_type(4)));
    static_assert(FW % 4 == 0, "16-byte pieces");
    for (uint32_t i = threadIdx.x; i < FW / 4; i += blockDim.x) ((V4*)filt)[i] = ((const V4*)filter)[i];
  }
  for (uint32_t i = threadIdx.x; i < CE; i += blockDim.x) cache[i] = kEmptyKey;
  if (threadIdx.x < 4)
    ctl[threadIdx.x] = threadIdx.x == 1 ? hold : threadIdx.x == 3 && *cand.count >= cand.max_cand ? 1u : 0u;
  stage_tables<DP>(ti, FP ? t.tabq : (HM == kHashPacked ? t.tabp : t.tabi), (uint32_t)KB, (uint32_t)KB);
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
  // The particles that may pass wait in the wave's queue and are looked up and tested 64 at a time:
  // where a tenth of them reaches the test, a test in place runs with a tenth of its lanes.
  uint32_t queued = 0;
  auto cache_slot = [](uint64_t key) { return (uint32_t)(key ^ (key >> 21)) & (CE - 1u); };
  auto flush = [&]() {
    // a key was refused: the error is latched and no other can get in
    if (__builtin_amdgcn_readfirstlane(
            __hip_atomic_load(&ctl[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != 0u) {
      queued = 0;
      return;
    }
    const bool act = lane < queued;
    const uint64_t key = act ? (uint64_t)qhi[lane] << 32 | qlo[lane] : 0ull;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    queued = 0;
    // a key already in the set needs no exact test: the set only ever gains keys
    const uint64_t s0 = act ? set[(uint32_t)slot_mix(key) & slot_mask] : kEmptyKey;
    bool in = act && s0 == key, pass = false, is_new = false;
    if (act && !in && s0 != kEmptyKey) in = set_contains(set, slot_mask, key);   // a longer probe run
    if (act && !in) {
      uint32_t bk[D], ng[D];
      exact_rows(key, bk, ng);
#pragma unroll
      for (int r = 0; r < D; ++r) ng[r] &= t.cm ^ 1u;
      in = pass = rows_pass<D>(bk, ng, need, nullptr, M, t.w, theta);
    }
    if (in && !pass) __hip_atomic_store(&cache[cache_slot(key)], key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    // Of the lanes that bring a key to the cache one claims it: where all particles share a cell there
    // would be a compare-and-swap each, all to one word, until the cache shows it.
    if (pass && __hip_atomic_exchange(&cache[cache_slot(key)], key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != key) {
      const uint32_t got = set_claim(cand, key, err, [&]() {
        return __hip_atomic_load(&ctl[3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == 0u;
      });
      is_new = got == kClaimNew;
      if (got == kClaimRefused) __hip_atomic_store(&ctl[2], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    // New keys go into the list with the workgroup's others when it ends, past `hold` of them here and now:
    // one or two at a time they kept the kernel waiting for the count (about 40 ns an add, one after
    // the other over all XCDs).  The count tells then whether the set is full.
    const uint64_t who = __ballot(is_new);
    if (who == 0) return;
    const uint32_t more = (uint32_t)__popcll(who);
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u));
    uint32_t at = 0;
    if (lane == 0) at = __hip_atomic_fetch_add(&ctl[0], more, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    at = __builtin_amdgcn_readfirstlane(at);
    if (at + more <= hold) {
      if (is_new) fresh[at + rank] = key;
      return;
    }
    if (lane == 0) {
      __hip_atomic_fetch_min(&ctl[1], at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      at = atomicAdd(cand.count, more);
    }
    at = __builtin_amdgcn_readfirstlane(at);
    if (is_new && at + rank < cand.max_cand) cand.list[at + rank] = key;
    if (at + more > cand.max_cand && lane == 0) {
      atomicOr(err, kErrCapacity);
      __hip_atomic_store(&ctl[2], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  };
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
    auto hits = [&](int j) {
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
      return fp;
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
    // (no branch or && per particle, which put every one's reads and waits into a block of their own: 2^30
    // particles, d = 5, w = 2^24: 4.19 ms, 4.00 ms so)
    maybe = fine;
    if (uf) {
      maybe = 0;
#pragma unroll
      for (int j = 0; j < PPT; ++j) maybe |= (uint32_t)(hits(j) >= need) << j;
      maybe &= fine;
    }
    // The particles that may pass.  A key seen recently by this workgroup needs no look-up: heavy
    // cells repeat thousands of times.
    uint32_t todo = maybe;
#pragma unroll
    for (int j = 0; j < PPT; ++j)
      // (lanes with nothing to look up read one common slot: no bank conflicts)
      if (__hip_atomic_load(&cache[(todo >> j) & 1u ? cache_slot(keys[j]) : 0u], __ATOMIC_RELAXED,
                            __HIP_MEMORY_SCOPE_WORKGROUP) == keys[j])
        todo &= ~(1u << j);
    uint32_t some = 0;   // the particles j that some lane has to look up
#pragma unroll
    for (int j = 0; j < PPT; ++j) some |= (__ballot((todo >> j) & 1u) != 0 ? 1u : 0u) << j;
    static_assert(PPT == 8, "the selection below");
#pragma unroll 1
    for (; some != 0; some &= some - 1u) {
      const uint32_t j = (uint32_t)__builtin_ctz(some);
      uint64_t key;
      switch (j) {
        case 0: key = keys[0]; break;
        case 1: key = keys[1]; break;
        case 2: key = keys[2]; break;
        case 3: key = keys[3]; break;
        case 4: key = keys[4]; break;
        case 5: key = keys[5]; break;
        case 6: key = keys[6]; break;
        default: key = keys[7]; break;
      }
      const bool open = (todo >> j) & 1u;
      const uint64_t who = __ballot(open);
      const uint32_t more = (uint32_t)__popcll(who);
      if (queued + more > 64u) flush();
      if (open) {
        const uint32_t at = queued + __builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32),
                                                               __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u));
        qlo[at] = (uint32_t)key;
        qhi[at] = (uint16_t)(key >> 32);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      queued += more;
    }
  }
  if (queued) flush();
  __syncthreads();
  // The domain error once a workgroup: all go to one word.  (By hand, in the queues' first words, which are
  // done with: the barrier that ORs a predicate brings LDS of its own, and the dynamic part is all there is.)
  uint32_t* outside = (uint32_t*)(cache + CE);
  const bool some_bad = __any(bad);
  if (lane == 0) outside[wave] = some_bad ? 1u : 0u;
  const uint32_t nf = min(ctl[0], ctl[1]);   // the slots handed out before the first that was refused
  if (threadIdx.x == 0 && nf != 0) ctl[3] = atomicAdd(cand.count, nf);
  __syncthreads();
  const uint32_t base = ctl[3];
  for (uint32_t i = threadIdx.x; i < nf; i += kCollectThreads) {
    if (base + i < cand.max_cand) cand.list[base + i] = fresh[i];
    else atomicOr(err, kErrCapacity);
  }
  if (threadIdx.x == 0) {
    uint32_t any = 0;
    for (uint32_t i = 0; i < kWaves; ++i) any |= outside[i];
    if (any) atomicOr(err, kErrDomain);
  }
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
    if (hm == kHashMulHi && c.field) {
      launch_collect2_one<D, MM, kHashMulHi, true>(grid, block, lds, s, c);
      return;
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

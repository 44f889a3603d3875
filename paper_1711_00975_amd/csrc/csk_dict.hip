// csk_dict.hip — candidate passes over ranges of cell keys on gfx950: the whole dictionary (Count
// Sketch with Full Search, Sec. 2.2 item 1; Alg. 1) and the children of a coarse sketch's candidate
// super-items (the second layer of the hierarchical query, Alg. 3).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "csk_kernel_util.h"

namespace csk {

namespace {

constexpr uint32_t kDictThreads = 1024;
constexpr uint32_t kDictQueue = 128;   // keys a wave holds for the exact test
constexpr uint32_t kDictBlocks = 256;  // one workgroup per CU (the filter fills its LDS)

// What the two passes share.  The list (children): super-item j covers the keys
// [j group, min((j + 1) group, nkeys)); m of them, at most cap are read.
struct DictArgs {
  uint64_t nkeys;
  Tables t;
  const int32_t* M;
  int32_t theta;
  const uint32_t* filter;      // NULL: no filter
  const uint32_t* hot;
  const uint32_t* hot_table;   // may be NULL
  CandSet cand;
  uint32_t* err;
  uint32_t nch;                // key bytes that can be non-zero
  uint32_t unit;               // dictionary: 256-key blocks a wave takes at a time (a power of two <= 64)
  const uint64_t* list;
  const uint32_t* list_count;
  uint32_t list_cap;
  uint32_t group;
  uint64_t direct;             // list: no filter for at most this many keys
};

// x >> (byte B of b), the byte selected by the instruction itself.
template <int B>
__device__ __forceinline__ uint32_t shift_by(uint32_t x, uint32_t b) {
  uint32_t y;
  if constexpr (B == 0) asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_0 src1_sel:DWORD" : "=v"(y) : "v"(b), "v"(x));
  if constexpr (B == 1) asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1 src1_sel:DWORD" : "=v"(y) : "v"(b), "v"(x));
  if constexpr (B == 2) asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_2 src1_sel:DWORD" : "=v"(y) : "v"(b), "v"(x));
  if constexpr (B == 3) asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:DWORD" : "=v"(y) : "v"(b), "v"(x));
  return y;
}

// Keys are enumerated, so a key's hash need not be looked up from scratch: a tabulation hash is the
// XOR of one table entry per key byte, and the 256 keys of an aligned block differ in byte 0 only.  A
// wave takes such a block at a time; every lane keeps the byte-0 entries of its four keys in registers
// and the XOR of the other bytes' entries is a wave-uniform value, so that hashing a key is one XOR
// per word and LDS is read for the filter alone.  FP: the field-probe filter, whose probe fields are
// tabulated themselves (word address and bit positions kept apart in registers, XORed separately).
// The few keys that pass are gathered in an LDS queue per wave and take the exact test 64 at a time.
// The conflicts of the filter reads are those of the byte-0 entries (the rest of the address is the same
// for all lanes), so their order over the lanes is chosen against them when the sketch is made.  Bound by
// the VALU (4.5 instructions per row and key) and the LDS reads alike.  2000^3 keys, d = 5, w = 2^22, 88655
// hot counters: 34.8 ms with a hash of four LDS reads and a computed probe per key and row, 7.95 ms so
// with the values in their order (64 random words take 6.9 cycles), 7.03 ms in the chosen one (4.5
// cycles); 34329 super-items of 1000 keys: 3.04 ms with every row's counter read, 0.18 ms so.
template <int D, int HM, bool FP>
struct KeyWalk {
  static constexpr int TW = FP ? 4 : HashWords<D, HM>::value;   // words per table entry
  static constexpr int NR = FP ? D + (D + 1) / 2 : TW;          // registers per entry
  static constexpr uint32_t FW = FP ? kFieldFilterWords : (uint32_t)kFilterWords;

  const DictArgs& a;
  const uint32_t* filt;   // LDS
  uint64_t* queue;        // LDS, this wave's
  uint32_t queued = 0;
  uint32_t need;
  bool uh;
  uint32_t vs = 0;        // the byte-0 values of this lane's four keys
  uint32_t e0[4][NR];

  // registers of a table entry (linear: the registers of an XOR are the XOR of the registers)
  static __device__ __forceinline__ void split(const uint32_t (&q)[TW], uint32_t (&e)[NR]) {
    if constexpr (FP) {
#pragma unroll
      for (int r = 0; r < D; ++r) {
        const uint32_t f = field_bits<kFieldBits>(q, r);
        e[r] = (f >> 8) & ((kFieldFilterWords - 1u) << 2);   // byte offset of the filter word
        const uint32_t b = (f & 31u) | ((f >> 5) & 31u) << 8;    // the two bit positions, a byte each
        e[D + r / 2] = (r & 1) ? e[D + r / 2] | b << 16 : b;
      }
    } else {
#pragma unroll
      for (int i = 0; i < TW; ++i) e[i] = q[i];
    }
  }
  __device__ __forceinline__ void entry(uint32_t c, uint32_t v, uint32_t (&q)[TW]) const {
    const uint32_t* src = (FP ? a.t.tabq : (HM == kHashPacked ? a.t.tabp : a.t.tabi)) + (c * 256 + v) * TW;
#pragma unroll
    for (int i = 0; i < TW; ++i) q[i] = src[i];
  }
  // XOR of the entries of bytes first..5 of a wave-uniform key
  __device__ __forceinline__ void upper(uint64_t key, int first, uint32_t (&q)[TW]) const {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)key);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(key >> 32));
    const uint32_t byte[kChars] = {lo & 255u, (lo >> 8) & 255u, (lo >> 16) & 255u, lo >> 24, hi & 255u, (hi >> 8) & 255u};
#pragma unroll
    for (int i = 0; i < TW; ++i) q[i] = 0;
#pragma unroll
    for (int c = 1; c < kChars; ++c) {
      if (c < first) continue;
      uint32_t x[TW];
      entry((uint32_t)c, byte[c], x);
#pragma unroll
      for (int i = 0; i < TW; ++i) q[i] ^= x[i];
    }
  }

  __device__ __forceinline__ KeyWalk(const DictArgs& args, const uint32_t* lds_filter, uint64_t* lds_queue, bool hot_set)
      : a(args), filt(lds_filter), queue(lds_queue), uh(hot_set) {
    need = a.t.cm ? (uint32_t)D : (uint32_t)(D - ((D - 1) >> 1));
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      uint32_t q[TW], v = 64u * g + lane_id();
      if constexpr (FP) v = ((const uint8_t*)(a.t.tabq + kTableWords * TW))[v];   // see probe_order()
      vs |= v << (8 * g);
      entry(0, v, q);
      split(q, e0[g]);
    }
  }

  // The exact test and insertion of one key per lane.
  __device__ __forceinline__ void test(uint64_t key) {
    uint32_t bk[D], ng[D];
    rows_bucket_sign_kb<D, HM, kChars>(HM == kHashPacked ? a.t.tabp : a.t.tabi, key, a.t.w, a.t.wshift, bk, ng);
#pragma unroll
    for (int r = 0; r < D; ++r) ng[r] &= a.t.cm ^ 1u;
    if (rows_pass<D>(bk, ng, need, uh ? a.hot_table : nullptr, a.M, a.t.w, a.theta)) set_insert(a.cand, key, a.err);
  }
  __device__ __forceinline__ uint32_t value(uint32_t g) const { return (vs >> (8 * g)) & 255u; }
  // The lanes of who hold keys base + value(g) that pass the filter (who: the same in every lane).
  __device__ __forceinline__ void offer(uint64_t who, uint64_t base, uint32_t g) {
    const uint32_t at = queued + __builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32),
                                                           __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u));
    if ((who >> lane_id()) & 1u) queue[at] = base + value(g);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    queued = __builtin_amdgcn_readfirstlane(queued + (uint32_t)__popcll(who));
    if (queued >= 64u) {
      queued -= 64u;
      const uint64_t k = queue[queued + lane_id()];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      test(k);
    }
  }
  __device__ __forceinline__ void finish() {
    if (lane_id() < queued) test(queue[lane_id()]);
  }

  // The keys base + v, first <= v < end, of one aligned block; f: the uniform registers of its upper bytes.
  __device__ __forceinline__ void block(uint64_t base, uint32_t first, uint32_t end, const uint32_t (&f)[NR]) {
    uint64_t who[4];
    uint32_t x[4][D];
    if constexpr (FP) {   // all the reads of the block before any is used
      // the filter is at LDS address 0 (the kernel sees to it): the byte offset is the address
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int r = 0; r < D; ++r)
          x[g][r] = *(const __attribute__((address_space(3))) uint32_t*)(uintptr_t)(e0[g][r] ^ f[r]);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      uint32_t fp = 0;
      if constexpr (FP) {
#pragma unroll
        for (int r = 0; r < D; ++r) {
          const uint32_t b = e0[g][D + r / 2] ^ f[D + r / 2];
          fp += (r & 1 ? shift_by<2>(x[g][r], b) & shift_by<3>(x[g][r], b) : shift_by<0>(x[g][r], b) & shift_by<1>(x[g][r], b)) & 1u;
        }
      } else {
        uint32_t h[TW];
#pragma unroll
        for (int i = 0; i < TW; ++i) h[i] = e0[g][i] ^ f[i];
#pragma unroll
        for (int r = 0; r < D; ++r) {
          uint32_t bk, ng;
          if constexpr (HM == kHashPacked) {
            constexpr int F = packed_bits(D);
            const uint32_t q[4] = {h[0], h[1], h[2], h[3]};
            const uint32_t v = packed_field<F>(q, r);
            ng = v >> (F - 1);
            bk = (v << (33 - F)) >> a.t.wshift;
          } else {
            bk = bucket_of_t<HM == kHashShift>(h[r], a.t.w, a.t.wshift);
            ng = h[r] >> 31;
          }
          const FilterProbe pr = filter_probe((uint32_t)r, bk, ng & (a.t.cm ^ 1u), a.t.bnorm);
          fp += ((filt[pr.word] & pr.mask) == pr.mask) ? 1u : 0u;
        }
      }
      who[g] = __ballot(fp >= need);
    }
    if (end - first < 256u) {
#pragma unroll
      for (int g = 0; g < 4; ++g) who[g] &= __ballot(value(g) >= first && value(g) < end);
    }
    if ((who[0] | who[1] | who[2] | who[3]) == 0) return;
#pragma unroll 1
    for (uint32_t g = 0; g < 4; ++g) {
      const uint64_t w = g < 2 ? (g == 0 ? who[0] : who[1]) : (g == 2 ? who[2] : who[3]);
      if (w) offer(w, base, g);
    }
  }
};

// Without a filter: all rows hashed from the tables in LDS and the counters read.
template <int D, int HM>
__device__ __forceinline__ void direct_test(const DictArgs& a, const uint32_t* ti, uint64_t key) {
  const uint32_t need = a.t.cm ? (uint32_t)D : (uint32_t)(D - ((D - 1) >> 1));
  uint32_t bk[D], ng[D];
  rows_bucket_sign<D, HM>(ti, key, a.nch, a.t.w, a.t.wshift, bk, ng);
#pragma unroll
  for (int r = 0; r < D; ++r) ng[r] &= a.t.cm ^ 1u;
  if (rows_pass<D>(bk, ng, need, nullptr, a.M, a.t.w, a.theta)) set_insert(a.cand, key, a.err);
}

// How many of the `workers` (waves, quarter workgroups) take one of m super-items together, 256 keys in turn:
// few large ones would leave the others idle (d = 5, w = 2^18: 10 of 30000 keys, read directly: 340 us with a
// quarter workgroup each, 31 us so; 3 of 10^6 through the filter: 2.1 ms with a wave each, 42 us so).
__device__ __forceinline__ uint32_t list_share(uint32_t workers, uint32_t m, uint32_t group) {
  const uint32_t blocks = group / 256u + 1u;
  return m != 0 && m < workers ? min(workers / m, blocks) : 1u;
}

template <int D, int HM, bool FP, bool LIST>
__global__ __launch_bounds__(kDictThreads) void dict_kernel(DictArgs a) {
  using W = KeyWalk<D, HM, FP>;
  extern __shared__ __align__(16) uint32_t lds4[];
  uint32_t m = 0;
  if (LIST) {
    const uint32_t count = *a.list_count;
    m = min(count, a.list_cap);
    if (count > a.list_cap && blockIdx.x == 0 && threadIdx.x == 0) atomicOr(a.err, kErrCapacity);
  }
  bool uf = a.filter != nullptr && !(LIST && (uint64_t)m * a.group <= a.direct);
  const uint32_t nhot = uf ? *a.hot : 0xFFFFFFFFu;
  uf = uf && (FP ? (uint64_t)nhot * a.t.fspan <= kFieldFilterMaxItems : nhot <= kFilterMaxItems);
  // The walk takes byte offsets into the field-probe filter for LDS addresses.  They are, as long as the
  // dynamic LDS is all the kernel has; static LDS would come first, and every key would take the exact
  // test.  (Adding the base costs an instruction per row and key.)
  if (FP && (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint32_t*)lds4 != 0u) uf = false;
  if (!uf) {
    stage_tables<HashWords<D, HM>::value>(lds4, HM == kHashPacked ? a.t.tabp : a.t.tabi, a.nch);
    if (LIST) {
      // a quarter of a workgroup per super-item, or several where there are few of them
      const uint32_t part = blockIdx.x * 4u + (threadIdx.x >> 8), parts = gridDim.x * 4u;
      const uint32_t share = list_share(parts, m, a.group);
      for (uint32_t u = part; u < m * share; u += parts) {
        const uint32_t i = share == 1u ? u : u / share;
        const uint64_t lo = a.list[i] * a.group;
        const uint64_t hi = lo + a.group < a.nkeys ? lo + a.group : a.nkeys;
        for (uint64_t key = lo + 256u * (u - i * share) + (threadIdx.x & 255u); key < hi; key += 256u * share)
          direct_test<D, HM>(a, lds4, key);
      }
    } else {
      const uint64_t stride = (uint64_t)gridDim.x * kDictThreads;
      for (uint64_t key = (uint64_t)blockIdx.x * kDictThreads + threadIdx.x; key < a.nkeys; key += stride)
        direct_test<D, HM>(a, lds4, key);
    }
    return;
  }
  using V4 = uint32_t __attribute__((ext_vector_type(4)));
  static_assert(W::FW % 4 == 0, "16-byte pieces");
  for (uint32_t i = threadIdx.x; i < W::FW / 4; i += kDictThreads) ((V4*)lds4)[i] = ((const V4*)a.filter)[i];
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  W walk(a, lds4, (uint64_t*)(lds4 + W::FW) + wave * kDictQueue, a.hot_table != nullptr && nhot <= kHotMaxItems);
  __syncthreads();
  constexpr uint32_t kWaves = kDictThreads / 64u;
  // neighbours in the stream of work on different CUs
  const uint32_t w0 = wave * gridDim.x + blockIdx.x, nw = gridDim.x * kWaves;
  if (LIST) {
    const uint32_t share = list_share(nw, m, a.group);   // waves per super-item
    for (uint32_t u = w0; u < m * share; u += nw) {
      const uint32_t i = share == 1u ? u : u / share;
      const uint64_t lo = a.list[i] * a.group;
      const uint64_t hi = lo + a.group < a.nkeys ? lo + a.group : a.nkeys;
      for (uint64_t base = (lo & ~255ull) + 256u * (u - i * share); base < hi; base += 256u * share) {
        uint32_t q[W::TW], f[W::NR];
        walk.upper(base, 1, q);
        W::split(q, f);
        walk.block(base, base < lo ? (uint32_t)(lo - base) : 0u, hi - base < 256 ? (uint32_t)(hi - base) : 256u, f);
      }
    }
  } else {
    const uint64_t units = ((a.nkeys + 255) / 256 + a.unit - 1) / a.unit;
    for (uint64_t u = w0; u < units; u += nw) {
      // lane l: the registers of the unit's block l (byte 1 and the bytes above, which are the same for all)
      const uint64_t first = u * a.unit * 256;
      uint32_t q[W::TW], x[W::TW], f1[W::NR];
      walk.upper(first, 2, q);
      walk.entry(1, ((uint32_t)(first >> 8) & 255u) + (lane_id() & (a.unit - 1u)), x);
#pragma unroll
      for (int i = 0; i < W::TW; ++i) q[i] ^= x[i];
      W::split(q, f1);
      for (uint32_t j = 0; j < a.unit; ++j) {
        const uint64_t base = first + 256ull * j;
        if (base >= a.nkeys) break;
        const uint32_t end = a.nkeys - base < 256 ? (uint32_t)(a.nkeys - base) : 256u;
        uint32_t f[W::NR];
#pragma unroll
        for (int i = 0; i < W::NR; ++i) f[i] = __builtin_amdgcn_readlane(f1[i], j);
        walk.block(base, 0, end, f);
      }
    }
  }
  walk.finish();
}

// The dictionary for any d, with row-major tables read from global memory (d > 8).
__global__ __launch_bounds__(256) void dict_collect_generic_kernel(uint64_t nkeys, Tables t,
                                                                   const int32_t* __restrict__ M, int32_t theta,
                                                                   CandSet cand,
                                                                   uint32_t* err) {
  const uint32_t need = t.cm ? t.d : t.d - ((t.d - 1) >> 1);
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t key = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; key < nkeys; key += stride) {
    uint32_t pass = 0;
    for (uint32_t r = 0; r < t.d; ++r) {
      if (pass >= need || pass + (t.d - r) < need) break;
      if (row_estimate(t.tab + r * kTableWords, M + (uint64_t)r * t.w, t.w, t.cm, key) >= theta) ++pass;
    }
    if (pass >= need) set_insert(cand, key, err);
  }
}

// The children for any d (d > 8): one workgroup per super-item at a time.
__global__ __launch_bounds__(256) void children_generic_kernel(const uint64_t* __restrict__ list,
                                                               const uint32_t* __restrict__ count, uint32_t cap,
                                                               uint32_t group, uint64_t ncells, Tables t,
                                                               const int32_t* __restrict__ M, int32_t theta,
                                                               CandSet cand, uint32_t* err) {
  const uint32_t m = min(*count, cap);
  if (*count > cap && blockIdx.x == 0 && threadIdx.x == 0) atomicOr(err, kErrCapacity);
  for (uint32_t i = blockIdx.x; i < m; i += gridDim.x) {
    const uint64_t lo = list[i] * group;
    const uint64_t hi = (lo + group < ncells) ? lo + group : ncells;
    for (uint64_t c = lo + threadIdx.x; c < hi; c += blockDim.x)
      if (estimate_key<32>(t.tab, M, t.d, t.w, t.cm, c) >= theta) set_insert(cand, c, err);
  }
}

template <int D, int HM, bool FP>
void launch_one(const DictArgs& a, bool list, hipStream_t s) {
  const size_t tables = (size_t)kTableWords * HashWords<D, HM>::value * 4;
  const size_t filtered = KeyWalk<D, HM, FP>::FW * 4 + (kDictThreads / 64) * kDictQueue * 8;
  static_assert(KeyWalk<D, HM, FP>::FW * 4 >= (size_t)kTableWords * HashWords<D, HM>::value * 4, "tables in the filter's place");
  const size_t lds = a.filter ? filtered : tables;
  const dim3 grid(a.filter ? kDictBlocks : 2 * kDictBlocks), block(kDictThreads);
  if (list) hipLaunchKernelGGL((dict_kernel<D, HM, FP, true>), grid, block, lds, s, a);
  else hipLaunchKernelGGL((dict_kernel<D, HM, FP, false>), grid, block, lds, s, a);
}

template <int D>
void launch_d(const DictArgs& a, bool list, hipStream_t s) {
  const int hm = a.t.hash_mode();
  if constexpr (D == 5) {
    if (collect_field_form(a.t)) {
      if (hm == kHashPacked) launch_one<D, kHashPacked, true>(a, list, s);
      else launch_one<D, kHashMulHi, true>(a, list, s);
      return;
    }
  }
  if constexpr (D >= 5) {
    if (hm == kHashPacked) {
      launch_one<D, kHashPacked, false>(a, list, s);
      return;
    }
  }
  if (hm == kHashMulHi) launch_one<D, kHashMulHi, false>(a, list, s);
  else launch_one<D, kHashShift, false>(a, list, s);
}

hipError_t launch_any(const DictArgs& a, bool list, hipStream_t s) {
  switch (a.t.d) {
    case 1: launch_d<1>(a, list, s); break;
    case 2: launch_d<2>(a, list, s); break;
    case 3: launch_d<3>(a, list, s); break;
    case 4: launch_d<4>(a, list, s); break;
    case 5: launch_d<5>(a, list, s); break;
    case 6: launch_d<6>(a, list, s); break;
    case 7: launch_d<7>(a, list, s); break;
    default: launch_d<8>(a, list, s); break;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_collect_dictionary(uint64_t nkeys, const Mesh& mesh, const Tables& t, const int32_t* M,
                                     int32_t theta, const uint32_t* filter, const uint32_t* hot,
                                     const uint32_t* hot_table, const CandSet& cand, uint32_t* err, hipStream_t s) {
  if (t.d > (uint32_t)kTabLdsRows) {
    hipLaunchKernelGGL(dict_collect_generic_kernel, dim3(grid_for(nkeys, 256, 8192)), dim3(256), 0, s, nkeys, t, M,
                       theta, cand, err);
    return hipGetLastError();
  }
  DictArgs a{};
  a.nkeys = nkeys;
  a.t = t;
  a.M = M;
  a.theta = theta;
  a.filter = filter;
  a.hot = hot;
  a.hot_table = hot_table;
  a.cand = cand;
  a.err = err;
  a.nch = mesh.nch;
  // four units or more per wave where there are keys for it, so that the last ones do not run alone
  const uint64_t per = nkeys / 256 / (kDictBlocks * (kDictThreads / 64) * 4);
  a.unit = 4;
  while (a.unit < 64 && a.unit < per) a.unit *= 2;
  return launch_any(a, false, s);
}

// Reading the counters of every child against building the filter first (in us, 1000 children a
// super-item, 400, 800 and 1600 of them): d = 5, w = 2^16: 14, 17, 27 and 15, 15, 17; w = 2^20: 25, 35, 63
// and 38, 38, 39; w = 2^22: 28, 47, 85 and 52, 52, 53; w = 2^24: 30, 53, 95 and a build of 133; d = 8,
// w = 2^16: 19, 24, 40 and 22, 23, 29; d = 3, w = 2^20: 19, 22, 37 and 33, 33, 35.
uint64_t children_direct_keys(const Tables& t) {
  return t.d <= (uint32_t)kTabLdsRows ? (1ull << 19) + t.w / 10u : ~0ull;
}

hipError_t launch_collect_children(const uint64_t* list, const uint32_t* list_count, uint32_t list_cap, uint32_t group,
                                   uint64_t ncells, uint32_t nch, const Tables& t, const int32_t* M, int32_t theta,
                                   const uint32_t* filter, const uint32_t* hot, const CandSet& cand, uint32_t* err,
                                   hipStream_t s) {
  if (t.d > (uint32_t)kTabLdsRows) {
    hipLaunchKernelGGL(children_generic_kernel, dim3(2048), dim3(256), 0, s, list, list_count, list_cap, group, ncells,
                       t, M, theta, cand, err);
    return hipGetLastError();
  }
  DictArgs a{};
  a.nkeys = ncells;
  a.t = t;
  a.M = M;
  a.theta = theta;
  a.filter = filter;
  a.hot = hot;
  a.cand = cand;
  a.err = err;
  a.nch = nch;
  a.list = list;
  a.list_count = list_count;
  a.list_cap = list_cap;
  a.group = group;
  a.direct = children_direct_keys(t);
  return launch_any(a, true, s);
}

}  // namespace csk

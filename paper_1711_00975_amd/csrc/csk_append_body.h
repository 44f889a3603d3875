// csk_append_body.h — the append bin kernel of the update (Sec. 2.2 Add; Alg. 4 Update;
// Sec. 3.1 stages 1-3), shared by its translation units: csk_append.hip (the packed
// sort-word table, w = 2^lw) and csk_append_rows.hip (row-interleaved tables with
// multiply-high buckets for any w, and the router's exclusion).
//
// Per particle: the exact cell key, then the token of every row with its slice, as in
// csk_sortbin_body.h.  Tokens are not sorted: every (row, slice) bin of the sketch has a
// buffer of `ring` tokens in LDS for the whole kernel, a token is appended to its bin's buffer
// with one LDS add-with-return (its slot) and one 16-bit LDS store, and a full buffer goes to
// its region in whole 64-byte pieces.  That is 2.2 LDS operations per token where a counting
// sort takes about 5 (count, cursor, staging store, staging load, destination) and two barriers
// per phase instead of four per sorted pass.  Whole pieces are what the regions are bound by:
// the counting sort's runs of 16 tokens wrote 19.4 GiB for 10 GiB of tokens, and 32-byte stores
// scattered over the 256 x 2560 regions reach 1.3 TB/s here, 64-byte ones 3.3-4.
//
// A phase is `pp` iterations of one particle per thread, then a flush: every bin is looked at
// by its own thread (or tpb threads when there are fewer bins than threads).  The hashes of
// the next particle are computed between the flush and its closing barrier, and its key while
// the slots of the current one return.  Positions are loaded two iterations ahead.  The
// workgroups take 1024-particle pieces of the stream in turn, which spreads a structure that
// is contiguous in the stream over all regions.
//
// A token that finds its bin's buffer full goes to its counter with a global atomic, and so
// does a granule that finds its region full (equal tokens of the granule in one add): the
// same sum.
//
// Measured, bin kernel alone (the sort-word or general kernel before): 2^30 particles, d = 5,
// w = 2^24: 10.98 -> 9.15 ms (5.2 ms of it with the flush left out: LDS 39 % and VALU 33 %
// busy); 4 calls of 2^25 packed particles, w = 2^22: 1.33 -> 0.92 ms; 2^20 particles,
// w = 2^16: 44 -> 22 us; 12.3 million particles in structure order, d = 8, w = 3145733:
// 6.3 -> 1.6 ms.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "csk_kernel_util.h"

namespace csk {
namespace append {

constexpr uint32_t kNT = kBin2Threads;
using Quad = uint32_t __attribute__((ext_vector_type(4)));   // 8 tokens, one 16-byte access

// LDS layout (bytes): [EX: the exclusion's table] | tables [kb * 256 * dp words] | cnt [P + 64] |
// sent [P] (16 bits) | buffers [P * ring tokens] (16-byte aligned) | one dummy token.  Bins
// P .. P + 63 are dummies, one per lane: particles outside the stream or the domain, or counted
// otherwise, append there.  Their counts start far above any buffer, so that nothing is stored.
struct AppendLds {
  uint32_t ts, cnt, sent, ring, bytes;
};
__host__ __device__ __forceinline__ AppendLds append_lds(uint32_t dp, uint32_t kb, uint32_t P, uint32_t ring, bool ex) {
  AppendLds L;
  L.ts = ex ? kExLdsWords * 4u : 0u;
  L.cnt = L.ts + 256u * dp * kb * 4u;
  L.sent = L.cnt + 4u * (P + 64u);
  L.ring = (L.sent + 2u * P + 15u) & ~15u;
  L.bytes = L.ring + 2u * P * ring + 16u;
  return L;
}

template <int D, uint32_t MODE, bool ROWS, bool EX, int KB, bool HOLD>
__device__ __forceinline__ void append_body(const BinArgs* __restrict__ ap, const float* __restrict__ pos, uint64_t n,
                                            uint32_t g) {
  constexpr int DP = ROWS ? RowPad<D>::value : 4;
  constexpr int F = packed_bits(D);
  constexpr uint32_t GT = HOLD ? kAppendHold : kAppendGranule;   // tokens a bin gives up at a time
  static_assert(!EX || (D == 5 && MODE != kMeshPacked), "the exclusion is compiled for d = 5, float positions");
  const BinArgs& a = *ap;
  const BinPlan& pl = a.plan;
  extern __shared__ __align__(16) uint8_t ldsa[];
  const uint32_t P = pl.P, Pr = pl.Pr, cap = pl.cap, R = pl.ring;
  const AppendLds Ly = append_lds(DP, KB, P, R, EX);
  const ExLds ext = ex_lds((uint32_t*)ldsa);   // EX only
  uint32_t* ts = (uint32_t*)(ldsa + Ly.ts);
  uint32_t* cnt = (uint32_t*)(ldsa + Ly.cnt);   // tokens appended to the bin since its last flush, plus what that left
  uint16_t* sent = (uint16_t*)(ldsa + Ly.sent);  // granules of the bin in its region
  uint16_t* ring = (uint16_t*)(ldsa + Ly.ring);
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t pos_sign = a.cm ^ 1u;   // ROWS: Count-Min tokens carry no sign
  uint16_t* __restrict__ tokg = a.tok + (uint64_t)g * P * cap;   // this workgroup's regions

  for (uint32_t i = tid; i < P + 64u; i += kNT) cnt[i] = i < P ? 0u : 1u << 30;
  for (uint32_t i = tid; i < P; i += kNT) sent[i] = 0;
  stage_tables<DP>(ts, ROWS ? a.tabi : a.tabs, KB, KB);   // fold point KB >= nch; ends with a barrier
  if constexpr (EX) ex_fill(a.ex.admitted, adm_count(a.ex), ext);   // ends with a barrier

  // this workgroup's pieces of kNT particles: g, g + nwg, ...
  const uint64_t pieces = (n + kNT - 1) / kNT;
  const uint64_t mine = pieces > g ? (pieces - g + pl.nwg - 1) / pl.nwg : 0;
  // taken two at a time (a piece past the stream is all dummies), so that the loop body has
  // no condition between a load and its use two iterations later
  const uint64_t iters = (mine + 1) & ~1ull;
  const uint64_t stride = (uint64_t)pl.nwg * kNT;
  struct Pos {
    float x, y, z;
    uint32_t w0, w1;
    uint32_t count;   // particles of the piece (the same for the whole workgroup)
  };
  // a piece is read through a buffer resource of its own bytes: loads past the stream give 0
  uint64_t ahead = (uint64_t)g * kNT;   // first particle of the next piece to load
  auto load = [&](Pos& p) {
    const uint64_t first = ahead < n ? ahead : 0, left = ahead < n ? n - ahead : 0;
    p.count = left < kNT ? (uint32_t)left : kNT;
    ahead += stride;
    if constexpr (MODE == kMeshPacked) {
      const auto v = __builtin_amdgcn_raw_buffer_load_b64(byte_span((const uint64_t*)pos + first, 8u * p.count),
                                                          8u * tid, 0, 2);
      p.w0 = v[0];
      p.w1 = v[1];
    } else {
      load_xyz(byte_span(pos + 3 * first, 12u * p.count), 12u * tid, 0, p.x, p.y, p.z);
    }
  };
  uint32_t bin[D], v[D];   // bin and 16-bit token (the low half of v) of every row
  uint64_t key;            // every byte indexes its table in range, whatever the particle
  uint32_t ix, iy, iz;
  bool odd = false, ok = true, bad = false;   // odd: some particle of the wave may have to be dropped
  // first half of a particle's work, the exact cell key: arithmetic only
  auto to_key = [&](const Pos& p) {
    if constexpr (MODE == kMeshPacked) {
      ok = packed_key<false>((uint64_t)p.w0 | (uint64_t)p.w1 << 32, a.mesh, key);   // ungrouped (plan)
      odd = p.count != kNT || !__all(ok);
    } else {
      // nearly always every particle is in [0, L), which needs no wrap and no domain test
      odd = p.count != kNT || !__all(inside_box(p.x, p.y, p.z, a.mesh));
      if (!odd) {
        ix = cell_index_inside<MODE>(p.x, a.mesh);
        iy = cell_index_inside<MODE>(p.y, a.mesh);
        iz = cell_index_inside<MODE>(p.z, a.mesh);
      } else {
        int32_t jx, jy, jz;
        ok = ((int)cell_index_m<MODE>(p.x, a.mesh, jx) & (int)cell_index_m<MODE>(p.y, a.mesh, jy) &
              (int)cell_index_m<MODE>(p.z, a.mesh, jz)) != 0;
        ix = (uint32_t)jx;
        iy = (uint32_t)jy;
        iz = (uint32_t)jz;
      }
      key = cell_key_of((int32_t)ix, (int32_t)iy, (int32_t)iz, a.mesh);   // ungrouped (plan)
    }
  };
  auto to_counter = [&](uint32_t b, uint32_t t, int32_t times) {
    asm volatile("" : "+v"(b));   // keeps the division in the rare paths that need it
    const uint32_t r = b / Pr, sl = b % Pr;
    atomicAdd(&a.M[(uint64_t)r * a.w + ((sl << kSliceBits) | (t & (kSlice - 1)))], (t & 0x8000u) ? -times : times);
  };
  // second half: the row words and from them every row's bin and token
  auto to_tokens = [&](const Pos& p) {
    uint32_t h[DP];
    row_hashes_kb<DP, KB>(ts, key, h);
#pragma unroll
    for (int r = 0; r < D; ++r) {
      if constexpr (ROWS) {
        const uint32_t b = bucket_of(h[r], a.w);
        bin[r] = (b >> kSliceBits) + (uint32_t)r * Pr;
        v[r] = (b & (kSlice - 1)) | (((h[r] >> 31) & pos_sign) << 15);
      } else {
        const uint32_t q[4] = {h[0], h[1], h[2], h[3]};
        v[r] = field_bits<F>(q, r);   // token in the low half; bits above the field are ignored
        bin[r] = ((v[r] >> 16) & ((1u << (F - 16)) - 1u)) + (uint32_t)r * Pr;
      }
    }
    if (odd) {   // past the stream, or a particle outside the domain
      const bool in = tid < p.count;
      bad = bad || (in && !ok);
#pragma unroll
      for (int r = 0; r < D; ++r) bin[r] = in && ok ? bin[r] : P + lane;
    }
    if constexpr (EX) {
      if (!odd || (tid < p.count && ok)) {
        uint32_t child;
        const int32_t c = ex_find(adm_coarse((int32_t)ix, (int32_t)iy, (int32_t)iz, a.ex, child), ext);
        if (c >= 0) {   // counted exactly
          atomicAdd(&a.ex.child[(uint32_t)c * a.ex.f3 + child], 1u);
#pragma unroll
          for (int r = 0; r < D; ++r) bin[r] = P + lane;
        }
      }
    }
    // A stream in structure order: when many lanes share the cell of the first or of a middle
    // lane, the wave's repeated cells go straight to the counters, one add per row and cell.  Each
    // of them would otherwise fill its bins' buffers and send them there token by token.
    const uint32_t klo = (uint32_t)key, khi = (uint32_t)(key >> 32);
    const int like = __popcll(__ballot(klo == (uint32_t)__builtin_amdgcn_readfirstlane(klo))) +
                     __popcll(__ballot(klo == (uint32_t)__builtin_amdgcn_readlane(klo, 29)));
    if (like >= 8) {
      const bool alive = bin[0] < P;
      uint64_t todo = __ballot(alive), gone = 0;
      for (int k = 0; k < 16 && todo; ++k) {
        const uint32_t lead = (uint32_t)__ffsll((unsigned long long)todo) - 1u;
        const uint32_t lo = __builtin_amdgcn_readlane(klo, lead), hi = __builtin_amdgcn_readlane(khi, lead);
        const uint64_t same = __ballot(klo == lo && khi == hi) & todo;
        const int32_t times = (int32_t)__popcll(same);
        todo &= ~same;
        if (times < 3) continue;
        gone |= same;
        if (lane == lead) {
#pragma unroll
          for (int r = 0; r < D; ++r) to_counter(bin[r], v[r], times);
        }
      }
      if ((gone >> lane) & 1u) {
#pragma unroll
        for (int r = 0; r < D; ++r) bin[r] = P + lane;
      }
    }
  };
  // tokens [s0, s0 + c) of bin b's buffer to its counters, equal ones in one add (c <= 32)
  auto spill = [&](uint32_t b, uint32_t s0, uint32_t c) {
    const uint16_t* t = ring + b * R + s0;
    uint32_t left = 0xFFFFFFFFu >> (32u - c);
    while (left) {
      const uint32_t i = (uint32_t)__ffs((int)left) - 1u, x = t[i];
      int32_t times = 0;
      for (uint32_t j = i; j < c; ++j) {
        const bool eq = ((left >> j) & 1u) && t[j] == x;
        times += eq ? 1 : 0;
        left &= ~((eq ? 1u : 0u) << j);
      }
      to_counter(b, x, times);
    }
  };
  const uint32_t capb = 2u * cap, sent_max = cap / GT;
  const uint32_t tpb = HOLD ? 1u : pl.tpb, tj = tid & (tpb - 1u), bins = kNT / tpb, b_first = tid / tpb;
  constexpr uint32_t NB = HOLD ? 3 : 5;   // bins of one thread (the plan checks)
  Quad h0[NB] = {}, h1[NB] = {};           // HOLD: the granule that waits for its other half
  // Flush.  Memory takes whole 64-byte pieces at 3.3-4 TB/s here but 32-byte ones at 1.3 (8 GiB
  // over 256 x 2560 regions), so a bin's tokens leave 32 at a time:
  //   HOLD false  tpb threads (4..64, within one wave) per bin send its granules of 32 tokens,
  //               16 bytes each;
  //   HOLD true   more bins than LDS can buffer 32 tokens for (w = 2^24): a bin gives up 16
  //               tokens at a time to its one thread, which holds them in registers until the
  //               next 16 make the piece whole.
  // What is left moves to the front of the buffer.  A thread has at most NB bins, and their LDS
  // reads are all in flight before any is used.
  auto flush = [&](bool final) {
    uint32_t fill[NB], done[NB];
    Quad x0[NB] = {}, x1[NB] = {}, y[NB] = {};
#pragma unroll
    for (uint32_t e = 0; e < NB; ++e) {
      const uint32_t b = b_first + e * bins;
      fill[e] = done[e] = 0;
      if (b < P) {
        fill[e] = min(cnt[b], R);
        done[e] = sent[b];
      }
    }
    bool full = false;   // a region has no room
#pragma unroll
    for (uint32_t e = 0; e < NB; ++e) {
      const Quad* src = (const Quad*)(ring + (b_first + e * bins) * R);
      const uint32_t ng = fill[e] / GT;
      if constexpr (HOLD) {   // ring < 32: at most one granule
        if (ng) {
          x0[e] = src[0];
          x1[e] = src[1];
          y[e] = src[2];
        }
      } else {
        if (tj < 4 * ng) x0[e] = src[tj];
        if (8 * tj < (ng ? fill[e] % GT : 0u)) y[e] = src[4 * ng + tj];   // what is left, no more
      }
      full |= ng && done[e] + ng > sent_max;
    }
#pragma unroll
    for (uint32_t e = 0; e < NB; ++e) {
      const uint32_t ng = fill[e] / GT, room = sent_max - done[e];
      const uint32_t go = ng < room ? ng : room;   // granules that the region has room for
      uint8_t* to = (uint8_t*)tokg;
      const uint32_t at = (b_first + e * bins) * capb + 2u * GT * done[e];
      if constexpr (HOLD) {
        if (go) {
          if (done[e] & 1u) {
            Quad* q = (Quad*)(to + (at - 32u));
            q[0] = h0[e];
            q[1] = h1[e];
            q[2] = x0[e];
            q[3] = x1[e];
          }
          h0[e] = x0[e];
          h1[e] = x1[e];
        }
      } else {
        if (tj < 4 * go) *(Quad*)(to + (at + 16u * tj)) = x0[e];
        if (tj + tpb < 4 * go) {
          const Quad* src = (const Quad*)(ring + (b_first + e * bins) * R);
          for (uint32_t q = tj + tpb; q < 4 * go; q += tpb) *(Quad*)(to + (at + 16u * q)) = src[q];
        }
      }
    }
    if (full) {   // rare: what a region has no room for goes to the counters
#pragma unroll 1
      for (uint32_t b = b_first; b < P; b += bins) {
        const uint32_t ng = min(cnt[b], R) / GT, room = sent_max - sent[b];
        for (uint32_t q = tj; q < ng; q += tpb)
          if (q >= room) spill(b, GT * q, GT);
      }
    }
    __builtin_amdgcn_wave_barrier();   // granules are read before the rest moves over them
#pragma unroll
    for (uint32_t e = 0; e < NB; ++e) {
      const uint32_t b = b_first + e * bins, ng = fill[e] / GT, rest = fill[e] % GT;
      // what a full region could not take went to the counters: its count stays at the cap
      const uint32_t now = min(done[e] + ng, sent_max);
      if (ng) {
        if (8 * tj < rest) ((Quad*)(ring + b * R))[tj] = y[e];
        if (tj == 0) {
          cnt[b] = rest;
          sent[b] = (uint16_t)now;
        }
      }
      if (final && b < P) {   // the last tokens, as a partly filled granule
        __builtin_amdgcn_wave_barrier();
        uint8_t* to = (uint8_t*)tokg + (b * capb + 2u * GT * now);
        const Quad* src = (const Quad*)(ring + b * R);
        if constexpr (HOLD) {
          if (now & 1u) {
            ((Quad*)to)[-2] = h0[e];
            ((Quad*)to)[-1] = h1[e];
          }
        }
        const bool room = now < sent_max;
        if (room) {
          for (uint32_t q = tj; 8 * q < rest; q += tpb) ((Quad*)to)[q] = src[q];
        } else if (rest && tj == 0) {
          spill(b, 0, rest);
        }
        if (tj == 0) a.cnt[(uint64_t)b * pl.nwg + g] = now * GT + (room ? rest : 0u);
      }
    }
  };

  Pos pa, pb;
  load(pa);
  load(pb);
  to_key(pa);
  to_tokens(pa);
  load(pa);
  uint32_t ph = 0;
  // LDS addresses of the buffers and of the dummy bin's
  using LdsU16 = __attribute__((address_space(3))) uint16_t;
  const uint32_t ring0 = (uint32_t)(uintptr_t)(LdsU16*)ring, dummy = ring0 + 2u * P * R;   // the dummy token
  // append this particle's tokens; the next particle's key is computed while the slots return
  auto append = [&](const Pos& next) {
    uint32_t slot[D], at[D];
#pragma unroll
    for (int r = 0; r < D; ++r) slot[r] = atomicAdd(&cnt[bin[r]], 1u);
    __builtin_amdgcn_sched_barrier(0);   // all D slots are asked for before any is waited for
#pragma unroll
    for (int r = 0; r < D; ++r) at[r] = __umul24(bin[r], 2u * R) + ring0;
    to_key(next);
    __builtin_amdgcn_sched_barrier(0);
    bool over = false;
#pragma unroll
    for (int r = 0; r < D; ++r) {
      const bool full = slot[r] >= R;
      over |= full;
      const uint32_t byte = at[r] + 2u * slot[r];
      *(LdsU16*)(uintptr_t)(full ? dummy : byte) = (uint16_t)v[r];
    }
    if (over) {   // a buffer was full (rare): straight to the counter
#pragma unroll
      for (int r = 0; r < D; ++r)
        if (slot[r] >= R && bin[r] < P) to_counter(bin[r], v[r], 1);
    }
  };
  for (uint64_t it = 0; it < iters; it += 2) {
    append(pb);
    to_tokens(pb);
    load(pb);
    append(pa);
    const bool last = it + 2 == iters, end = ++ph == pl.pp / 2 || last;   // uniform
    if (end) {
      ph = 0;
      __syncthreads();   // every append of the phase is in the buffers
      flush(last);
    }
    to_tokens(pa);
    load(pa);
    if (end) __syncthreads();   // the flush is done before the next append
  }
  if (!mine)
    for (uint32_t s = tid; s < P; s += kNT) a.cnt[(uint64_t)s * pl.nwg + g] = 0;
  // The error once a workgroup: all go to one word.  (By hand, in counts that are done with: the barrier that
  // ORs a predicate brings LDS of its own, and the dynamic part may be all there is.)
  const bool some = __any(bad);
  if (lane == 0) cnt[tid >> 6] = some ? 1u : 0u;
  __syncthreads();
  if (tid == 0) {
    uint32_t any = 0;
    for (uint32_t i = 0; i < kNT / 64u; ++i) any |= cnt[i];
    if (any) atomicOr(a.err, kErrDomain);
  }
}

template <int D, uint32_t MODE, bool ROWS, bool EX, int KB, bool HOLD>
__global__ __launch_bounds__(kBin2Threads) void append_kernel(BinArgs a) {
  append_body<D, MODE, ROWS, EX, KB, HOLD>(&a, a.pos, a.n, blockIdx.x);
}

template <int D, uint32_t MODE, bool ROWS, int KB>
__global__ __launch_bounds__(kBin2Threads) void append_batch_kernel(const BinArgs* __restrict__ descs,
                                                                    const uint16_t* __restrict__ wg_sketch,
                                                                    const uint32_t* __restrict__ wg_first,
                                                                    BatchCall call) {
  const uint32_t i = wg_sketch[blockIdx.x];
  append_body<D, MODE, ROWS, false, KB, false>(descs + i, call.pos[i], call.n[i], blockIdx.x - wg_first[i]);
}

template <int D, uint32_t MODE, bool ROWS>
void launch_append_batch_kb(const AppendBatch& b, uint32_t kb, hipStream_t s) {
  const dim3 grid(b.nwg_total), block(kBin2Threads);
  if (kb == 4)
    hipLaunchKernelGGL((append_batch_kernel<D, MODE, ROWS, 4>), grid, block, b.lds_bytes, s, b.descs, b.wg_sketch,
                       b.wg_first, *b.call);
  else if (kb == 5)
    hipLaunchKernelGGL((append_batch_kernel<D, MODE, ROWS, 5>), grid, block, b.lds_bytes, s, b.descs, b.wg_sketch,
                       b.wg_first, *b.call);
  else
    hipLaunchKernelGGL((append_batch_kernel<D, MODE, ROWS, 6>), grid, block, b.lds_bytes, s, b.descs, b.wg_sketch,
                       b.wg_first, *b.call);
}

template <int D, bool ROWS>
void launch_append_batch_d(const AppendBatch& b, uint32_t mode, uint32_t kb, hipStream_t s) {
  if (mode == kMeshPow2Ratio) launch_append_batch_kb<D, kMeshPow2Ratio, ROWS>(b, kb, s);
  else if (mode == kMeshExactRatio) launch_append_batch_kb<D, kMeshExactRatio, ROWS>(b, kb, s);
  else launch_append_batch_kb<D, kMeshGeneral, ROWS>(b, kb, s);
}

template <int D, uint32_t MODE, bool ROWS, bool EX, int KB>
void launch_append_hold(const BinArgs& a, hipStream_t s) {
  const dim3 grid(a.plan.nwg), block(kBin2Threads);
  if (a.plan.hold)
    hipLaunchKernelGGL((append_kernel<D, MODE, ROWS, EX, KB, true>), grid, block, a.plan.lds_bytes, s, a);
  else
    hipLaunchKernelGGL((append_kernel<D, MODE, ROWS, EX, KB, false>), grid, block, a.plan.lds_bytes, s, a);
}

template <int D, uint32_t MODE, bool ROWS, bool EX>
void launch_append_kb(const BinArgs& a, hipStream_t s) {
  if (a.plan.kb == 4) launch_append_hold<D, MODE, ROWS, EX, 4>(a, s);
  else if (a.plan.kb == 5) launch_append_hold<D, MODE, ROWS, EX, 5>(a, s);
  else launch_append_hold<D, MODE, ROWS, EX, 6>(a, s);
}

template <int D, bool ROWS>
void launch_append_d(const BinArgs& a, uint32_t mode, hipStream_t s) {
  if (mode == kMeshPacked) launch_append_kb<D, kMeshPacked, ROWS, false>(a, s);
  else if (mode == kMeshPow2Ratio) launch_append_kb<D, kMeshPow2Ratio, ROWS, false>(a, s);
  else if (mode == kMeshExactRatio) launch_append_kb<D, kMeshExactRatio, ROWS, false>(a, s);
  else launch_append_kb<D, kMeshGeneral, ROWS, false>(a, s);
}

}  // namespace append
}  // namespace csk

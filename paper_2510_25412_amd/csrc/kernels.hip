// HIP kernels (gfx950 / CDNA4) of the pred hot path: copy-on-write page copy, KV append,
// page-table-indirected decode attention with per-lane online softmax, split merge, plus
// a file gather used by tests and two calibration kernels of known traffic.
//
// Geometry shared by all kernels (also stated in include/symphony_kv.h): a K or V row of
// one token and one kv head is 256 bytes; a (page, kv head) slab is [K|V][row half 0|1]
// [16 tokens][128 bytes], 8 KiB, so 8 tokens of one row half are 1 KiB contiguous.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <type_traits>

#include "desc.hpp"
#include "kernels.hpp"

namespace symkv {

namespace {

constexpr int kP = 16;              // tokens per page
constexpr int kRowBytes = 256;      // bytes of one K or V row (one token, one kv head)
constexpr int kHalfBytes = 128;     // a row half
constexpr int kBlk = kP * kRowBytes;   // 4096: K (or V) of one (page, head)
constexpr int kSlab = 2 * kBlk;        // 8192: K+V of one (page, head)
constexpr int kWavesPerBlock = 4;
constexpr float kTau = 8.0f;        // the running max may lag the true max by up to 2^kTau

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float as_f32(uint32_t u) { return __builtin_bit_cast(float, u); }
__device__ __forceinline__ uint32_t as_u32(float f) { return __builtin_bit_cast(uint32_t, f); }

// One word of the batch descriptor at a wavefront-uniform address, through the scalar cache.  The constant address space says
// what the compiler cannot see: nothing writes the descriptor while a kernel runs.  Without it these loads are vector loads as
// soon as the kernel stores anything, and since vector loads return in order, waiting for a page id then meant waiting for every
// K/V load in flight (s_waitcnt vmcnt(0) once per page; whole calls without / with: long contexts, 8 heads per kv head 754 / 716
// us; one file of 2000 tokens x 32 layers 494 / 473; drafts of 4 on 64 files 136.4 / 134.4; the mixed batch 1845 / 1824).
typedef const __attribute__((address_space(4))) int32_t* const_word_t;
__device__ __forceinline__ int sload(const int32_t* ptr) { return __builtin_amdgcn_readfirstlane(*(const_word_t)(uintptr_t)ptr); }

// Kernel arguments that a start needs, all requested before the first of them is waited for.  Left to itself the compiler fetches
// each where it is used, and a start is then a chain of up to six misses of the scalar cache before the first K/V load.
template <typename... T>
__device__ __forceinline__ void hold(const T&... x) {
  (..., [](auto v) __attribute__((always_inline)) { asm volatile("" ::"s"(v)); }(x));
}

// Sum over the 8 lanes of a lane octet (lanes 8k .. 8k+7): three DPP adds.
__device__ __forceinline__ float octet_sum(float x) {
  x += as_f32(__builtin_amdgcn_update_dpp(0, as_u32(x), 0xB1, 0xf, 0xf, false));    // quad_perm [1,0,3,2]
  x += as_f32(__builtin_amdgcn_update_dpp(0, as_u32(x), 0x4E, 0xf, 0xf, false));    // quad_perm [2,3,0,1]
  x += as_f32(__builtin_amdgcn_update_dpp(0, as_u32(x), 0x141, 0xf, 0xf, false));   // row_half_mirror
  return x;
}

// Value of the lane 8 away inside the 16-lane row (lane ^ 8): DPP row rotate by 8.
__device__ __forceinline__ float row_xor8(float x) {
  return as_f32(__builtin_amdgcn_update_dpp(0, as_u32(x), 0x128, 0xf, 0xf, false));   // row_ror:8
}

// max / sum of x over the lane pairs (l, l ^ 32) and (l, l ^ 16), in every lane, with the lane-swap instructions: swapping
// the upper 32 lanes of x with the lower 32 of a copy leaves one register holding the lower half twice and the other the
// upper half twice (likewise the odd and even rows of 16 lanes), so combining the two needs no select.
__device__ __forceinline__ float pair32_max(float x) {
  const auto sw = __builtin_amdgcn_permlane32_swap(as_u32(x), as_u32(x), false, false);
  return fmaxf(as_f32(sw[0]), as_f32(sw[1]));
}
__device__ __forceinline__ float pair16_max(float x) {
  const auto sw = __builtin_amdgcn_permlane16_swap(as_u32(x), as_u32(x), false, false);
  return fmaxf(as_f32(sw[0]), as_f32(sw[1]));
}
__device__ __forceinline__ float pair32_sum(float x) {
  const auto sw = __builtin_amdgcn_permlane32_swap(as_u32(x), as_u32(x), false, false);
  return as_f32(sw[0]) + as_f32(sw[1]);
}
__device__ __forceinline__ float pair16_sum(float x) {
  const auto sw = __builtin_amdgcn_permlane16_swap(as_u32(x), as_u32(x), false, false);
  return as_f32(sw[0]) + as_f32(sw[1]);
}

// Element-type traits.  A lane holds, per row half, one 16-byte chunk of a K/V row.
struct ElemBF16 {
  static constexpr int kDimsPerChunk = 8;
  // dot of one 16-byte chunk of K with the matching chunk of q, accumulated into s
  static __device__ __forceinline__ float dot(const uint4& k, const uint4& q, float s) {
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, k.x), __builtin_bit_cast(bf16x2_t, q.x), s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, k.y), __builtin_bit_cast(bf16x2_t, q.y), s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, k.z), __builtin_bit_cast(bf16x2_t, q.z), s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, k.w), __builtin_bit_cast(bf16x2_t, q.w), s, false);
    return s;
  }
  static __device__ __forceinline__ void unpack(const uint4& v, float* f) {
    f[0] = as_f32(v.x << 16); f[1] = as_f32(v.x & 0xffff0000u);
    f[2] = as_f32(v.y << 16); f[3] = as_f32(v.y & 0xffff0000u);
    f[4] = as_f32(v.z << 16); f[5] = as_f32(v.z & 0xffff0000u);
    f[6] = as_f32(v.w << 16); f[7] = as_f32(v.w & 0xffff0000u);
  }
};
struct ElemF32 {
  static constexpr int kDimsPerChunk = 4;
  static __device__ __forceinline__ float dot(const uint4& k, const uint4& q, float s) {
    s = __builtin_fmaf(as_f32(k.x), as_f32(q.x), s);
    s = __builtin_fmaf(as_f32(k.y), as_f32(q.y), s);
    s = __builtin_fmaf(as_f32(k.z), as_f32(q.z), s);
    s = __builtin_fmaf(as_f32(k.w), as_f32(q.w), s);
    return s;
  }
  static __device__ __forceinline__ void unpack(const uint4& v, float* f) {
    f[0] = as_f32(v.x); f[1] = as_f32(v.y); f[2] = as_f32(v.z); f[3] = as_f32(v.w);
  }
};

// 16 bytes of K or V.  STREAM: nontemporal, which streams a batch larger than the caches fastest; a compute unit that reads
// with few others gets its lines sooner without it.
template <bool STREAM>
__device__ __forceinline__ uint4 ld16(const uint8_t* p) {
  if constexpr (STREAM) return __builtin_bit_cast(uint4, __builtin_nontemporal_load((const u32x4_t*)p));
  else return *(const uint4*)p;
}

struct PageRegs {
  uint4 k[4];   // index = row_half * 2 + token_half
  uint4 v[4];
};

// ---------------------------------------------------------------------------------------
// Decode attention.  One wavefront per work range; lane = (r = lane/8: token slot within a
// half page, j = lane%8: which 16-byte chunk of each row half).  Every lane keeps its own
// running max / sum / accumulators over the tokens it sees (2 per page), so the page loop
// has no cross-lane traffic except the 8-lane score reduction; the 8 token slots are
// combined once, when a (row, kv head) range ends; a range that is only part of its (row, kv
// head) leaves a partial result for the merge kernel.
// ---------------------------------------------------------------------------------------
// decode_bins (below) is the form for up to 4 query heads per kv head.  decode_ranges is the form for 8
// heads per kv head on the vector units (whose 8 x 16 accumulators do not fit one wavefront's
// registers twice per SIMD): GT = query heads per kv head, G = GT / 2 = heads per wavefront, a
// workgroup of TWO wavefronts per range; wavefront 0 fetches the K half of every page,
// wavefront 1 the V half, they exchange them through LDS (written and read in the same
// lane-linear 1 KiB runs, so without bank conflicts), and every page is still read from HBM once.
// ---------------------------------------------------------------------------------------
// Decode ranges in bins (the VALU kernel for up to 4 query heads per kv head).  A workgroup of W
// wavefronts is a bin: the host hands it a list of segments (whole (row, kv head) ranges, or pieces of
// ranges too long for one bin) and cuts that list into W contiguous parts of equal cost, one per
// wavefront.  A wavefront walks its part as ONE page stream: a LOAD cursor runs two pages ahead of the
// COMPUTE cursor through the same unit sequence, across segment boundaries (starting every segment
// with its own chain of dependent loads, segment record -> page ids -> K/V, would cost several memory
// latencies per segment, a third of the time at 10 pages per range), so the K/V stream never drains;
// the query rows of the next segment are fetched one segment ahead.  At a boundary the compute side only
// combines its 8 token slots, hands the result on and switches to the next segment's registers.
// Where a result goes: a piece that is its whole segment writes the segment's destination (the final
// output rows, or a partial slot in device memory when the segment is only part of its range or the row has a
// shared prefix); a piece of a segment that the bin's cut divided goes to an LDS slot, and when all
// wavefronts of the bin are done they combine those pieces (merge_bin_pieces) into the destination.
// The append of a row's new token can ride along (segment word S_APPEND): the wavefront that reads
// the row's last page replaces the token's slot in its registers with the rows of k_new / v_new and
// writes them into the pool afterwards; nobody else reads that page in this launch.
// ---------------------------------------------------------------------------------------
template <typename E, int G>
struct BinLds {
  static constexpr int kAcc = G * 16 * E::kDimsPerChunk;      // accumulator floats of a piece: G heads x D dims
  static constexpr int kSlot = kAcc + 2 * G;                   // + (max, sum) per head
};

// What a wavefront of a bin starts with: its wave record, and the entry of the bin's merge list that it will carry out (the cut
// divides at most W - 1 segments, so there is at most one).  Both hang on the kernel arguments alone, so they are one round trip;
// the first K/V page and the records of the segments, which the wave record leads to, are the next.  (Arguments fetched one by one, the
// first page behind the segment's record and the merge list behind the barrier were eight misses of about 0.2 us each: one file of
// 2000 tokens x 32 layers 413 -> 394 us, 64 files of 512..4096 x 8 layers 786 -> 781.)
struct BinStart {
  int seg, p, units, id0, id1, head;           // first segment, page inside it, units, ids of its first two pages, kv head
  bool merges;
  int m_seg, m_slot, m_wave, m_pieces;
};
__device__ __forceinline__ BinStart bin_start(const DecodeArgs& a, const int bin, const int W, const int wib) {
  const int32_t* ww = a.waves + ((int64_t)bin * W + wib) * 8;
  const int32_t* lm = a.lmerge + (int64_t)bin * 32;
  const int32_t* en = lm + 4 + 4 * min(wib, 6);
  BinStart b;
  b.seg = sload(ww + 0);
  b.p = sload(ww + 1);
  b.units = sload(ww + 2);
  b.id0 = sload(ww + 4);
  b.id1 = sload(ww + 5);
  b.head = sload(ww + 7);
  b.merges = wib < sload(lm);
  b.m_seg = sload(en + 0);
  b.m_slot = sload(en + 1);
  b.m_wave = sload(en + 2);
  b.m_pieces = sload(en + 3);
  return b;
}

// After the barrier: the wavefront combines the pieces of the divided segment that is its own (qh, dest: words 5 and 6 of that
// segment's record, fetched while the first pages were on their way).
// Lane owns accumulator entries e * 64 + lane of the G * D values (head = entry / D).
template <typename E, int G>
__device__ __forceinline__ void merge_bin_pieces(const DecodeArgs& a, const BinStart& b, const int qh, const int dest, const float* lds) {
  constexpr int D = 16 * E::kDimsPerChunk, VL = G * D / 64, SLOT = BinLds<E, G>::kSlot, ACC = BinLds<E, G>::kAcc;
  const int lane = threadIdx.x & 63;
  if (b.merges) {
    const int s0 = b.m_slot, w0 = b.m_wave, n = b.m_pieces;
    float M[G], ls[G], o[VL];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      M[h] = -__builtin_inff();
      ls[h] = 0.f;
    }
#pragma unroll
    for (int e = 0; e < VL; ++e) o[e] = 0.f;
    for (int i = 0; i < n; ++i) {
      const float* sl = lds + (int64_t)(i == 0 ? s0 : 2 * (w0 + i)) * SLOT;
      float sc[G], wt[G];
#pragma unroll
      for (int h = 0; h < G; ++h) {
        const float mi = sl[ACC + 2 * h], li = sl[ACC + 2 * h + 1];
        const float mn = fmaxf(M[h], mi);
        sc[h] = __builtin_amdgcn_exp2f(M[h] - mn);      // 0 for the first piece (M = -inf)
        wt[h] = __builtin_amdgcn_exp2f(mi - mn);
        ls[h] = ls[h] * sc[h] + li * wt[h];
        M[h] = mn;
      }
#pragma unroll
      for (int e = 0; e < VL; ++e) o[e] = o[e] * sc[(e * 64) / D] + sl[e * 64 + lane] * wt[(e * 64) / D];
    }
    if (dest < 0) {
      float* out = a.out + (int64_t)qh * D;
#pragma unroll
      for (int e = 0; e < VL; ++e) out[e * 64 + lane] = o[e] / ls[(e * 64) / D];
    } else {
      float* pa = a.part_acc + (int64_t)dest * G * D;
#pragma unroll
      for (int e = 0; e < VL; ++e) pa[e * 64 + lane] = o[e];
      if (lane < G) {
        float mm = M[0], ll = ls[0];
#pragma unroll
        for (int hh = 1; hh < G; ++hh) {
          mm = (lane == hh) ? M[hh] : mm;
          ll = (lane == hh) ? ls[hh] : ll;
        }
        a.part_ml[((int64_t)dest * G + lane) * 2 + 0] = mm;
        a.part_ml[((int64_t)dest * G + lane) * 2 + 1] = ll;
      }
    }
  }
}

template <typename E, int G, bool STREAM>
__device__ __forceinline__ void decode_bins(const DecodeArgs& a, const int bin, const int W, float* lds) {
  constexpr int C = E::kDimsPerChunk;    // dims per 16-byte chunk
  constexpr int DPL = 2 * C;             // dims per lane
  constexpr int D = 16 * C;              // head dim
  constexpr int SLOT = BinLds<E, G>::kSlot, ACC = BinLds<E, G>::kAcc;
  hold(a.waves, a.lmerge, a.segs, a.pt, a.pool, a.page_bytes, a.q, a.out, a.part_acc, a.part_ml, a.k_new, a.v_new, a.n_bins, a.Hkv, a.scale_log2e);
  if (bin >= a.n_bins) return;           // the whole workgroup
  const int lane = threadIdx.x & 63;
  const int wib = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));      // wavefront within the bin
  const int r = lane >> 3, j = lane & 7;
  const BinStart st = bin_start(a, bin, W, wib);
  int remaining = st.units;
  int m_qh = 0, m_dest = 0;              // of the segment whose pieces it merges at the end: query row * Hq + head, destination
  auto merge_record = [&]() __attribute__((always_inline)) {
    const int32_t* msr = a.segs + (int64_t)(st.merges ? st.m_seg : 0) * 8;
    m_qh = sload(msr + 5);
    m_dest = sload(msr + 6);
  };

  if (remaining > 0) {
  // The first page, by what the wave record holds: its loads go out before the segment's record has come.
  const uint8_t* pool_lane = a.pool + lane * 16;
  auto request = [&](PageRegs& R, const uint8_t* base) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < 4; ++x) R.k[x] = ld16<STREAM>(base + x * 1024);
#pragma unroll
    for (int x = 0; x < 4; ++x) R.v[x] = ld16<STREAM>(base + kBlk + x * 1024);
  };
  PageRegs A, B;
  request(A, pool_lane + (int64_t)st.head * kSlab + (int64_t)st.id0 * a.page_bytes);
  __builtin_amdgcn_sched_barrier(0);
  merge_record();
  // Segment record: [0] page-table offset, [1] kv head, [2] first page, [3] end page (what the load side needs),
  // [4] tokens the row sees, [5] q row * Hq + first query head, [6] destination, [7] slot of the appended token or -1.
  // compute cursor: the segment being accumulated
  int seg = st.seg, p = st.p;
  const int32_t* sr = a.segs + (int64_t)seg * 8;
  int pe = sload(sr + 3), vis = sload(sr + 4), qh = sload(sr + 5);
  int dest = sload(sr + 6), app = sload(sr + 7), tbl = sload(sr + 0);
  bool from_start = p == sload(sr + 2);                  // the piece begins where its segment begins
  // load cursor: the unit whose K/V is requested next (two pages ahead of the compute cursor)
  int lseg = seg, lg = sload(sr + 1), lp = p, lpe = pe, ltbl = sload(sr + 0), lrem = remaining;
  // record of the segment after the load cursor's (fetched a whole segment ahead of its use; the list ends with spare records)
  int n_tbl = 0, n_g = 0, n_pb = 0, n_pe = 0;
  auto fetch_next_seg = [&](int ss) __attribute__((always_inline)) {
    const int32_t* q4 = a.segs + (int64_t)ss * 8;
    n_tbl = sload(q4 + 0);
    n_g = sload(q4 + 1);
    n_pb = sload(q4 + 2);
    n_pe = sload(q4 + 3);
  };
  fetch_next_seg(lseg + 1);
  // record of segment seg + 1 as the compute side needs it
  int c_pe = 0, c_vis = 0, c_qh = 0, c_dest = 0, c_app = 0, c_tbl = 0;
  auto fetch_compute_next_seg = [&]() __attribute__((always_inline)) {
    const int32_t* q8 = a.segs + (int64_t)(seg + 1) * 8;
    c_pe = sload(q8 + 3);
    c_vis = sload(q8 + 4);
    c_qh = sload(q8 + 5);
    c_dest = sload(q8 + 6);
    c_app = sload(q8 + 7);
    c_tbl = sload(q8 + 0);
  };

  // Requests the K/V of the next unit into R and advances the load cursor; past the last unit: page 0, head 0 (valid
  // memory that every wavefront touches, never used).
  // A streaming batch takes page ids as vector loads: the wait for one then drains the K/V loads before it, and without that the
  // wavefronts of a batch of equally long files run in step over the same memory channels (64 files of 4000 tokens, one
  // after the other in the pool: 190 us instead of 175; ragged or scattered files: the same within 1 %).
  auto page_id = [&](const int32_t* ptr) __attribute__((always_inline)) { return STREAM ? __builtin_amdgcn_readfirstlane(*ptr) : sload(ptr); };
  int next_pid = 0;
  auto load_next = [&](PageRegs& R) __attribute__((always_inline)) {
    const bool valid = lrem > 0;
    const uint8_t* base = pool_lane + (int64_t)(valid ? lg : 0) * kSlab + (int64_t)(valid ? next_pid : 0) * a.page_bytes;
    if (valid) {
      --lrem;
      if (++lp == lpe) {
        ++lseg;
        ltbl = n_tbl;
        lg = n_g;
        lp = n_pb;
        lpe = n_pe;
        fetch_next_seg(lseg + 1);
      }
      next_pid = lrem > 0 ? page_id(a.pt + ltbl + lp) : 0;   // id of the unit after this one, used one page later
    }
    // every load is unconditional and off one base address: no control-flow join between a load and its use, so the
    // waits can be for exactly the older page while the newer one is in flight
    request(R, base);
  };

  // q chunks of this lane for the G heads of the current segment
  u32x4_t q[G][2];
  // The append that rides along: the K and V rows of the row's new token (2 x 256 bytes in k_new / v_new) are requested
  // with the query rows, one 16-byte chunk per lane (lanes 0..15: K, 16..31: V; the upper half of the wavefront repeats
  // them), whenever a segment begins: the load is unconditional like every load of the stream (for a segment that appends
  // nothing the chunk is never used; k_new / v_new then point at the query rows, which are no smaller).
  u32x4_t nr;
  auto load_q = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const uint8_t* qp = (const uint8_t*)a.q + (int64_t)(qh + h) * kRowBytes + j * 16;
      q[h][0] = *(const u32x4_t*)qp;
      q[h][1] = *(const u32x4_t*)(qp + kHalfBytes);
    }
    nr = *(const u32x4_t*)((const uint8_t*)((lane & 16) ? a.v_new : a.k_new) + (int64_t)(qh / G) * kRowBytes + (lane & 15) * 16);
  };
  fetch_compute_next_seg();
  load_q();
  // past the first page, which is on its way; the record has the second one's id too, if that is of the same segment
  hold(m_qh, m_dest);
  next_pid = st.id1;
  --lrem;
  if (++lp == lpe) {
    ++lseg;
    ltbl = n_tbl;
    lg = n_g;
    lp = n_pb;
    lpe = n_pe;
    fetch_next_seg(lseg + 1);
    if (lrem > 0) next_pid = page_id(a.pt + ltbl + lp);
  }

  float m[G], l[G], acc[G][DPL];
  auto reset_state = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      m[h] = -1e30f;
      l[h] = 0.f;
#pragma unroll
      for (int d = 0; d < DPL; ++d) acc[h][d] = 0.f;
    }
  };
  reset_state();
  int piece = 0;                                         // pieces this wavefront has finished

  // tokens of page index pi (absolute, within the row) that exist: the row's last page may be ragged
  auto compute = [&](PageRegs& R, int pi) __attribute__((always_inline)) {
    const int nvalid = vis - pi * kP;          // >= 1; >= 16 for a full page
    if (nvalid < kP) {
      // ragged last page: slots past the file's end hold whatever was there before (possibly
      // NaN patterns); their weight is 0, but 0 * NaN is NaN, so clear their V chunks
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
        if ((hf * 8 + r) >= nvalid) {
          R.v[hf] = make_uint4(0, 0, 0, 0);
          R.v[2 + hf] = make_uint4(0, 0, 0, 0);
        }
    }
    float s[2][G];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      const bool valid = (hf * 8 + r) < nvalid;
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float x = E::dot(R.k[hf], __builtin_bit_cast(uint4, q[h][0]), 0.f);
        x = E::dot(R.k[2 + hf], __builtin_bit_cast(uint4, q[h][1]), x);
        x = octet_sum(x) * a.scale_log2e;
        s[hf][h] = valid ? x : -__builtin_inff();
      }
    }
    bool need = false;
#pragma unroll
    for (int h = 0; h < G; ++h) need |= fmaxf(s[0][h], s[1][h]) > m[h] + kTau;
    if (__builtin_amdgcn_ballot_w64(need) != 0) {     // rare after the first page
#pragma unroll
      for (int h = 0; h < G; ++h) {
        const float mn = fmaxf(m[h], fmaxf(s[0][h], s[1][h]));
        const float al = __builtin_amdgcn_exp2f(m[h] - mn);
        l[h] *= al;
#pragma unroll
        for (int d = 0; d < DPL; ++d) acc[h][d] *= al;
        m[h] = mn;
      }
    }
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      float pw[G];
#pragma unroll
      for (int h = 0; h < G; ++h) {
        pw[h] = __builtin_amdgcn_exp2f(s[hf][h] - m[h]);
        l[h] += pw[h];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        float vf[C];
        E::unpack(R.v[i * 2 + hf], vf);
#pragma unroll
        for (int h = 0; h < G; ++h)
#pragma unroll
          for (int e = 0; e < C; ++e) acc[h][i * C + e] = __builtin_fmaf(pw[h], vf[e], acc[h][i * C + e]);
      }
    }
  };

  // End of a piece: combine the 8 token slots (lanes with equal j).  Per head: common max M, rescale, total sum.  The
  // G*DPL accumulators are then reduced with a halving exchange (lane bit 5, 4, 3 in turn: keep one half of the list,
  // send the other), so lane (r, j) ends up owning the fully reduced values r*V/8 .. r*V/8 + V/8 - 1 of the list.
  // Then the compute cursor moves on.
  auto finish_piece = [&]() __attribute__((always_inline)) {
    const bool whole = from_start && p == pe;            // the piece is its whole segment
    const int64_t out_row = (int64_t)qh * D;
    const int f_dest = dest;
    // The segment after this one: its query rows are requested now, so that they arrive while the exchange
    // below runs (q is not needed any more for this piece).
    const bool more = remaining > 0;
    if (more) {
      ++seg;
      pe = c_pe;
      vis = c_vis;
      qh = c_qh;
      dest = c_dest;
      app = c_app;
      tbl = c_tbl;
      fetch_compute_next_seg();
      load_q();
    }
    constexpr int V = G * DPL;
    float vals[V];
    float lsum[G], Mh[G];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float M = m[h];
      M = fmaxf(M, row_xor8(M));
      M = pair16_max(M);
      M = pair32_max(M);
      const float f = __builtin_amdgcn_exp2f(m[h] - M);
      float ls = l[h] * f;
      ls += row_xor8(ls);
      ls = pair16_sum(ls);
      ls = pair32_sum(ls);
      lsum[h] = ls;
      Mh[h] = M;
#pragma unroll
      for (int d = 0; d < DPL; ++d) vals[h * DPL + d] = acc[h][d] * f;
    }
    {
      // lane bits 5 and 4: the lane-swap instructions do "keep one, send the other" in one go: after swapping the upper
      // 32 lanes of x with the lower 32 of y, x + y is x summed over the lane pairs (l, l + 32) in the lower half and y
      // summed in the upper half; likewise with the odd and even rows of 16 lanes
#pragma unroll
      for (int i = 0; i < V / 2; ++i) {
        const auto sw = __builtin_amdgcn_permlane32_swap(as_u32(vals[i]), as_u32(vals[i + V / 2]), false, false);
        vals[i] = as_f32(sw[0]) + as_f32(sw[1]);
      }
#pragma unroll
      for (int i = 0; i < V / 4; ++i) {
        const auto sw = __builtin_amdgcn_permlane16_swap(as_u32(vals[i]), as_u32(vals[i + V / 4]), false, false);
        vals[i] = as_f32(sw[0]) + as_f32(sw[1]);
      }
      const bool b3 = (lane & 8) != 0;
#pragma unroll
      for (int i = 0; i < V / 8; ++i) {
        const float keep = b3 ? vals[i + V / 8] : vals[i], send = b3 ? vals[i] : vals[i + V / 8];
        vals[i] = keep + row_xor8(send);
      }
    }
    // lane (r, j) now holds list entries idx = r * V/8 + t: head idx / DPL, lane-local dim idx % DPL
    if (whole && f_dest < 0) {
#pragma unroll
      for (int t = 0; t < V / 8; ++t) {
        const int idx = r * (V / 8) + t, h = idx / DPL, dl = idx % DPL;
        float ls = lsum[0];
#pragma unroll
        for (int hh = 1; hh < G; ++hh) ls = (h == hh) ? lsum[hh] : ls;
        a.out[out_row + h * D + (dl / C) * (D / 2) + j * C + (dl % C)] = vals[t] / ls;
      }
    } else {
      // unnormalised accumulator, max and sum: to the segment's partial slot in device memory, or to this wavefront's LDS
      // slot (two separate stretches of code: one pointer that may be either would make every store a flat store, and
      // with flat stores outstanding the waits for the K/V loads could no longer count)
      float mm = Mh[0], ll = lsum[0];
#pragma unroll
      for (int hh = 1; hh < G; ++hh) {
        mm = (lane == hh) ? Mh[hh] : mm;
        ll = (lane == hh) ? lsum[hh] : ll;
      }
      if (whole) {
        float* pa = a.part_acc + (int64_t)f_dest * G * D;
#pragma unroll
        for (int t = 0; t < V / 8; ++t) {
          const int idx = r * (V / 8) + t, h = idx / DPL, dl = idx % DPL;
          pa[h * D + (dl / C) * (D / 2) + j * C + (dl % C)] = vals[t];
        }
        if (lane < G) {
          a.part_ml[((int64_t)f_dest * G + lane) * 2 + 0] = mm;
          a.part_ml[((int64_t)f_dest * G + lane) * 2 + 1] = ll;
        }
      } else {
        float* pl = lds + (piece == 0 ? 2 * wib : 2 * wib + 1) * SLOT;
#pragma unroll
        for (int t = 0; t < V / 8; ++t) {
          const int idx = r * (V / 8) + t, h = idx / DPL, dl = idx % DPL;
          pl[h * D + (dl / C) * (D / 2) + j * C + (dl % C)] = vals[t];
        }
        if (lane < G) {
          pl[ACC + lane * 2 + 0] = mm;
          pl[ACC + lane * 2 + 1] = ll;
        }
      }
    }
    ++piece;
    if (more) {                                          // the next segment (the piece ended with its own)
      p = sload(a.segs + (int64_t)seg * 8 + 2);
      from_start = true;
      reset_state();
    }
  };
  // one unit: accumulate the page, move the compute cursor, close the piece at the end of the segment or of the wavefront's work
  auto do_unit = [&](PageRegs& R) __attribute__((always_inline)) {
    if (app >= 0 && p + 1 == pe) {
      // The segment's last page is the row's last page, and its slot `app` is the new token's, still unwritten in the pool:
      // the lanes that hold that slot take the token's chunks (K row halves from lanes j and 8 + j of `nr`, V from
      // 16 + j and 24 + j) and write them into the pool, where this wavefront is the page's only reader in this launch.
      const u32x4_t k0 = {(uint32_t)__shfl((int)nr.x, j), (uint32_t)__shfl((int)nr.y, j), (uint32_t)__shfl((int)nr.z, j), (uint32_t)__shfl((int)nr.w, j)};
      const u32x4_t k1 = {(uint32_t)__shfl((int)nr.x, 8 + j), (uint32_t)__shfl((int)nr.y, 8 + j), (uint32_t)__shfl((int)nr.z, 8 + j), (uint32_t)__shfl((int)nr.w, 8 + j)};
      const u32x4_t v0 = {(uint32_t)__shfl((int)nr.x, 16 + j), (uint32_t)__shfl((int)nr.y, 16 + j), (uint32_t)__shfl((int)nr.z, 16 + j), (uint32_t)__shfl((int)nr.w, 16 + j)};
      const u32x4_t v1 = {(uint32_t)__shfl((int)nr.x, 24 + j), (uint32_t)__shfl((int)nr.y, 24 + j), (uint32_t)__shfl((int)nr.z, 24 + j), (uint32_t)__shfl((int)nr.w, 24 + j)};
      uint8_t* dst = const_cast<uint8_t*>(a.pool) + (int64_t)sload(a.pt + tbl + p) * a.page_bytes + (int64_t)(qh / G % a.Hkv) * kSlab +
                     app * kHalfBytes + j * 16;
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)                     // (register indices stay compile-time constants)
        if ((app >> 3) == hf && r == (app & 7)) {
          R.k[hf] = __builtin_bit_cast(uint4, k0);
          R.k[2 + hf] = __builtin_bit_cast(uint4, k1);
          R.v[hf] = __builtin_bit_cast(uint4, v0);
          R.v[2 + hf] = __builtin_bit_cast(uint4, v1);
          *(u32x4_t*)dst = k0;
          *(u32x4_t*)(dst + kP * kHalfBytes) = k1;
          *(u32x4_t*)(dst + kBlk) = v0;
          *(u32x4_t*)(dst + kBlk + kP * kHalfBytes) = v1;
        }
    }
    compute(R, p);
    ++p;
    --remaining;
    if (p == pe || remaining == 0) finish_piece();
  };

  while (remaining > 0) {
    load_next(B);
    do_unit(A);
    load_next(A);
    if (remaining > 0) do_unit(B);
  }
  } else {
    merge_record();
  }
  __syncthreads();                                       // every piece of the bin is in LDS (or went straight to its destination)
  merge_bin_pieces<E, G>(a, st, m_qh, m_dest, lds);
}

// ---------------------------------------------------------------------------------------
// Decode bins on the matrix cores, fp32 weights (bf16 storage, 4 query heads per kv head).  The same stream of pages,
// segments, pieces and LDS merge as decode_bins above; what differs is a page's arithmetic:
//   S^T[16 tokens][16 columns] = K · Q^T     4 x v_mfma_f32_16x16x32_bf16 (exact products, two sums of 64)
//   O^T[128 dims][16 columns] += V^T · P^T   8 x v_mfma_f32_16x16x16_bf16
// A softmax weight is a 24-bit fp32 number; cut into three bf16 numbers of 8 bits each (hi, mid, lo: cutting is exact, and so is
// their sum) it takes three of the 16 columns, column = part * G + head, so ONE product per 16 dims carries the weights at full
// precision and V as it is stored.  The three columns of a head are added when a piece ends.
// Neither operand needs LDS or a transpose: a lane (col, grp) loads 64 contiguous bytes of K per token `col` and step, and of
// V the tokens 4 grp .. +3 at dims 8 col .. +7; product block e holds dims 8 i + e, so the lane's own words, the tokens of a
// dim packed by v_perm, are the operand (16 instructions a page), and the lane's four scores are the tokens it supplies.
// About 70 vector instructions a page instead of 330 (dot products on lane octets, 32 fused multiply-adds per dim chunk):
// the attention launch of 64 files of 512..4096 tokens 97.4 -> 95.1 us (6.3 TB/s), of 8 files of 4000 27.2 -> 26.1 us, the mixed
// batch's 1734 -> 1724 us.  What bounds it is HBM, and with few files the 40 GB/s that one compute unit draws.  Error against
// 64 bits 2.0e-7, the vector units' 2.2e-7.  A third page in flight: slower (96.2 us; one file of 2000 tokens 15.3 -> 17.8 us).
// ---------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

template <int N>
__device__ __forceinline__ float row_shl(float x) {     // value of the lane N further up in the 16-lane row (0 past its end)
  return as_f32(__builtin_amdgcn_update_dpp(0, as_u32(x), 0x100 + N, 0xf, 0xf, true));
}

template <int G>
__device__ __forceinline__ void decode_bins_mx(const DecodeArgs& a, const int bin, const int W, float* lds) {
  constexpr int D = 128, SLOT = BinLds<ElemBF16, G>::kSlot, ACC = BinLds<ElemBF16, G>::kAcc;
  hold(a.waves, a.lmerge, a.segs, a.pt, a.pool, a.page_bytes, a.q, a.out, a.part_acc, a.part_ml, a.k_new, a.v_new, a.n_bins, a.Hkv, a.scale_log2e);
  if (bin >= a.n_bins) return;           // the whole workgroup
  const int lane = threadIdx.x & 63;
  const int wib = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));      // wavefront within the bin
  const int col = lane & 15, grp = lane >> 4;
  const int head = col % G, part = col / G;                                      // columns from 3 G on are ignored
  const BinStart st = bin_start(a, bin, W, wib);
  int remaining = st.units;
  int m_qh = 0, m_dest = 0;
  auto merge_record = [&]() __attribute__((always_inline)) {
    const int32_t* msr = a.segs + (int64_t)(st.merges ? st.m_seg : 0) * 8;
    m_qh = sload(msr + 5);
    m_dest = sload(msr + 6);
  };

  if (remaining > 0) {
  // first page, cursors and records as in decode_bins
  const int k_off = col * kHalfBytes + grp * 16;                                 // token col, chunk 4 ks + grp of its row
  const int v_off = kBlk + (col >> 3) * (kP * kHalfBytes) + (4 * grp) * kHalfBytes + (col & 7) * 16;      // tokens 4 grp + u, chunk col
  auto request = [&](PageRegs& R, const uint8_t* base) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      R.k[ks] = __builtin_bit_cast(uint4, __builtin_nontemporal_load((const u32x4_t*)(base + k_off + (ks >> 1) * (kP * kHalfBytes) + (ks & 1) * 64)));
#pragma unroll
    for (int u = 0; u < 4; ++u) R.v[u] = __builtin_bit_cast(uint4, __builtin_nontemporal_load((const u32x4_t*)(base + v_off + u * kHalfBytes)));
  };
  PageRegs A, B;
  request(A, a.pool + (int64_t)st.head * kSlab + (int64_t)st.id0 * a.page_bytes);
  __builtin_amdgcn_sched_barrier(0);
  merge_record();
  int seg = st.seg, p = st.p;
  const int32_t* sr = a.segs + (int64_t)seg * 8;
  int pe = sload(sr + 3), vis = sload(sr + 4), qh = sload(sr + 5);
  int dest = sload(sr + 6), app = sload(sr + 7), tbl = sload(sr + 0);
  bool from_start = p == sload(sr + 2);
  int lseg = seg, lg = sload(sr + 1), lp = p, lpe = pe, ltbl = sload(sr + 0), lrem = remaining;
  int n_tbl = 0, n_g = 0, n_pb = 0, n_pe = 0;
  auto fetch_next_seg = [&](int ss) __attribute__((always_inline)) {
    const int32_t* q4 = a.segs + (int64_t)ss * 8;
    n_tbl = sload(q4 + 0);
    n_g = sload(q4 + 1);
    n_pb = sload(q4 + 2);
    n_pe = sload(q4 + 3);
  };
  fetch_next_seg(lseg + 1);
  int c_pe = 0, c_vis = 0, c_qh = 0, c_dest = 0, c_app = 0, c_tbl = 0;
  auto fetch_compute_next_seg = [&]() __attribute__((always_inline)) {
    const int32_t* q8 = a.segs + (int64_t)(seg + 1) * 8;
    c_pe = sload(q8 + 3);
    c_vis = sload(q8 + 4);
    c_qh = sload(q8 + 5);
    c_dest = sload(q8 + 6);
    c_app = sload(q8 + 7);
    c_tbl = sload(q8 + 0);
  };

  int next_pid = 0;
  auto load_next = [&](PageRegs& R) __attribute__((always_inline)) {
    const bool valid = lrem > 0;
    const uint8_t* base = a.pool + (int64_t)(valid ? lg : 0) * kSlab + (int64_t)(valid ? next_pid : 0) * a.page_bytes;
    if (valid) {
      --lrem;
      if (++lp == lpe) {
        ++lseg;
        ltbl = n_tbl;
        lg = n_g;
        lp = n_pb;
        lpe = n_pe;
        fetch_next_seg(lseg + 1);
      }
      next_pid = lrem > 0 ? sload(a.pt + ltbl + lp) : 0;
    }
    request(R, base);
  };

  bf16x8_t q[4];                         // Q^T operand: this lane's head, dims 32 ks + 8 grp .. +8
  u32x4_t nr;                            // the row's new token: K chunks in lanes 0..15, V chunks in 16..31 (decode_bins)
  auto load_q = [&]() __attribute__((always_inline)) {
    const uint8_t* qp = (const uint8_t*)a.q + (int64_t)(qh + head) * kRowBytes + grp * 16;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) q[ks] = __builtin_bit_cast(bf16x8_t, *(const u32x4_t*)(qp + ks * 64));
    nr = *(const u32x4_t*)((const uint8_t*)((lane & 16) ? a.v_new : a.k_new) + (int64_t)(qh / G) * kRowBytes + (lane & 15) * 16);
  };
  fetch_compute_next_seg();
  load_q();
  hold(m_qh, m_dest);
  next_pid = st.id1;
  --lrem;
  if (++lp == lpe) {
    ++lseg;
    ltbl = n_tbl;
    lg = n_g;
    lp = n_pb;
    lpe = n_pe;
    fetch_next_seg(lseg + 1);
    if (lrem > 0) next_pid = sload(a.pt + ltbl + lp);
  }

  f32x4_t O[8];
  float m, l;
  auto reset_state = [&]() __attribute__((always_inline)) {
    m = -1e30f;
    l = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) O[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  };
  reset_state();
  int piece = 0;
  // masks that leave a lane its part of a weight: w - (w & cut1) drops the upper 8 bits, once more the next 8
  const uint32_t cut1 = part >= 1 ? 0xffff0000u : 0u, cut2 = part >= 2 ? 0xffff0000u : 0u;

  auto compute = [&](PageRegs& R, int pi) __attribute__((always_inline)) {
    const int nvalid = vis - pi * kP;          // >= 1; >= 16 for a full page
    f32x4_t S = {0.f, 0.f, 0.f, 0.f}, S2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, R.k[ks]), q[ks], S, 0, 0, 0);
      S2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, R.k[2 + ks]), q[2 + ks], S2, 0, 0, 0);
    }
    S = S + S2;
    if (nvalid < kP) {
      // ragged last page: slots past the file's end hold whatever was there before; weight 0, but 0 * NaN is NaN
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (4 * grp + u >= nvalid) {
          S[u] = -__builtin_inff();
          R.v[u] = make_uint4(0, 0, 0, 0);
        }
    }
    const float mx = fmaxf(fmaxf(S[0], S[1]), fmaxf(S[2], S[3])) * a.scale_log2e;
    if (__builtin_amdgcn_ballot_w64(mx > m + kTau) != 0) {     // rare after the first page
      const float mn = pair32_max(pair16_max(fmaxf(m, mx)));   // the four lane groups of a column agree
      const float al = __builtin_amdgcn_exp2f(m - mn);
      l *= al;
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int v = 0; v < 4; ++v) O[e][v] *= al;
      m = mn;
    }
    uint32_t w[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      float x = __builtin_amdgcn_exp2f(__builtin_fmaf(S[v], a.scale_log2e, -m));
      l += x;
      x -= as_f32(as_u32(x) & cut1);
      x -= as_f32(as_u32(x) & cut2);
      w[v] = as_u32(x);
    }
    const s16x4_t P = __builtin_bit_cast(s16x4_t, make_uint2(__builtin_amdgcn_perm(w[1], w[0], 0x07060302), __builtin_amdgcn_perm(w[3], w[2], 0x07060302)));
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t sel = (e & 1) ? 0x07060302 : 0x05040100;
      auto word = [&](int u) { return (e >> 1) == 0 ? R.v[u].x : (e >> 1) == 1 ? R.v[u].y : (e >> 1) == 2 ? R.v[u].z : R.v[u].w; };
      const s16x4_t vt = __builtin_bit_cast(s16x4_t, make_uint2(__builtin_amdgcn_perm(word(1), word(0), sel), __builtin_amdgcn_perm(word(3), word(2), sel)));
      O[e] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vt, P, O[e], 0, 0, 0);
    }
  };

  // End of a piece: the sums of the four lane groups, the three columns of a head added up in its first; lane (col < G, grp)
  // then holds dims 32 grp .. +31 of head col.  Then the compute cursor moves on.
  auto finish_piece = [&]() __attribute__((always_inline)) {
    const bool whole = from_start && p == pe;            // the piece is its whole segment
    const int64_t out_row = (int64_t)qh * D;
    const int f_dest = dest;
    const bool more = remaining > 0;
    if (more) {
      ++seg;
      pe = c_pe;
      vis = c_vis;
      qh = c_qh;
      dest = c_dest;
      app = c_app;
      tbl = c_tbl;
      fetch_compute_next_seg();
      load_q();                                          // on its way while this piece is finished
    }
    const float ls = pair32_sum(pair16_sum(l));
    // An infinite V element: a lower part that is 0 (the maximum's weight is exactly 1) makes its column NaN, while the upper
    // part, never 0 where the weight is not, makes its own what the whole weight makes it.  So lower parts that are NaN are
    // dropped: where V is NaN, or infinities of both signs meet, the upper part's column says so by itself.
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float low = row_shl<G>(O[e][v]) + row_shl<2 * G>(O[e][v]);
        O[e][v] += low == low ? low : 0.f;
      }
    const int at = col * D + 32 * grp;                   // + 8 v + e
    if (col < G) {
      // (destinations in device memory and in LDS apart, see decode_bins)
      if (whole && f_dest < 0) {
        const float inv = 1.0f / ls;
        float* o = a.out + out_row + at;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          *(float4*)(o + 8 * v) = make_float4(O[0][v] * inv, O[1][v] * inv, O[2][v] * inv, O[3][v] * inv);
          *(float4*)(o + 8 * v + 4) = make_float4(O[4][v] * inv, O[5][v] * inv, O[6][v] * inv, O[7][v] * inv);
        }
      } else if (whole) {
        float* o = a.part_acc + (int64_t)f_dest * G * D + at;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          *(float4*)(o + 8 * v) = make_float4(O[0][v], O[1][v], O[2][v], O[3][v]);
          *(float4*)(o + 8 * v + 4) = make_float4(O[4][v], O[5][v], O[6][v], O[7][v]);
        }
        if (grp == 0) *(float2*)(a.part_ml + ((int64_t)f_dest * G + col) * 2) = make_float2(m, ls);
      } else {
        float* o = lds + (piece == 0 ? 2 * wib : 2 * wib + 1) * SLOT;
        if (grp == 0) *(float2*)(o + ACC + 2 * col) = make_float2(m, ls);
        o += at;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          *(float2*)(o + 8 * v) = make_float2(O[0][v], O[1][v]);
          *(float2*)(o + 8 * v + 2) = make_float2(O[2][v], O[3][v]);
          *(float2*)(o + 8 * v + 4) = make_float2(O[4][v], O[5][v]);
          *(float2*)(o + 8 * v + 6) = make_float2(O[6][v], O[7][v]);
        }
      }
    }
    ++piece;
    if (more) {                                          // the next segment (the piece ended with its own)
      p = sload(a.segs + (int64_t)seg * 8 + 2);
      from_start = true;
      reset_state();
    }
  };
  auto do_unit = [&](PageRegs& R) __attribute__((always_inline)) {
    if (app >= 0 && p + 1 == pe) {
      // the row's last page: slot `app` is the new token's, still unwritten in the pool.  The lanes that hold that slot take
      // the token's chunks and write them into the pool, where this wavefront is the page's only reader in this launch.
      uint8_t* dst = const_cast<uint8_t*>(a.pool) + (int64_t)sload(a.pt + tbl + p) * a.page_bytes + (int64_t)(qh / G % a.Hkv) * kSlab + app * kHalfBytes;
      auto chunk_of = [&](int from) __attribute__((always_inline)) {
        return u32x4_t{(uint32_t)__shfl((int)nr.x, from), (uint32_t)__shfl((int)nr.y, from), (uint32_t)__shfl((int)nr.z, from), (uint32_t)__shfl((int)nr.w, from)};
      };
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const u32x4_t x = chunk_of(4 * ks + grp);
        if (col == app) {
          R.k[ks] = __builtin_bit_cast(uint4, x);
          *(u32x4_t*)(dst + (ks >> 1) * (kP * kHalfBytes) + ((ks & 1) * 4 + grp) * 16) = x;
        }
      }
      const u32x4_t y = chunk_of(16 + col);
      if (grp == (app >> 2)) *(u32x4_t*)(dst + kBlk + (col >> 3) * (kP * kHalfBytes) + (col & 7) * 16) = y;
#pragma unroll
      for (int u = 0; u < 4; ++u)                        // (register indices stay compile-time constants)
        if (4 * grp + u == app) R.v[u] = __builtin_bit_cast(uint4, y);
    }
    compute(R, p);
    ++p;
    --remaining;
  };

  // One copy of the end-of-piece code for both register sets: a launch starts with a cold instruction cache, and a wavefront of
  // a small batch runs through this code once.
  bool odd = false;
  while (remaining > 0) {
    if (!odd) {
      load_next(B);
      do_unit(A);
    } else {
      load_next(A);
      do_unit(B);
    }
    odd = !odd;
    if (p == pe || remaining == 0) finish_piece();
  }
  } else {
    merge_record();
  }
  __syncthreads();                                       // every piece of the bin is in LDS (or went straight to its destination)
  merge_bin_pieces<ElemBF16, G>(a, st, m_qh, m_dest, lds);
}

// The decode bins of a shape.  With 1 or 2 query heads per kv head the vector units' page is short, and its loads take whole
// 128-byte lines of K where the matrix cores' take halves: attention launch, 64 files of 512..4096 tokens, matrix cores / vector
// units: G = 1 94.7 / 93.3 us, G = 2 98.6 / 97.9, G = 4 99.3 / 101.4; 256 files of 100..260: 37.3 / 34.7, 37.5 / 35.9, 39.1 / 39.9.
// Small batches (STREAM = false) stay with the vector units too: one file of 2000 tokens x 32 layers 473 against 501 us.
template <typename E, int G, bool STREAM>
__device__ __forceinline__ void bins_of(const DecodeArgs& a, const int bin, const int W, float* lds) {
  if constexpr (E::kDimsPerChunk == 8 && G == 4 && STREAM) decode_bins_mx<G>(a, bin, W, lds);
  else decode_bins<E, G, STREAM>(a, bin, W, lds);
}

template <typename E, int GT, int G>
__device__ __forceinline__ void decode_ranges(const DecodeArgs& a, const int block, uint8_t (*plds)[kSlab], const int wpb = kWavesPerBlock) {
  constexpr bool kPair = G < GT;
  const int hs = kPair ? (int)(threadIdx.x >> 6) : 0;      // which wavefront of the pair
  const int h0 = hs * G;                                    // first head (within the group) of this wavefront
  constexpr int C = E::kDimsPerChunk;    // dims per 16-byte chunk
  constexpr int DPL = 2 * C;             // dims per lane
  constexpr int D = 16 * C;              // head dim
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(kPair ? block : block * wpb + (int)(threadIdx.x >> 6));
  if (wv >= a.n_waves) return;
  const int r = lane >> 3, j = lane & 7;

  const int32_t* ww = a.waves + wv * 8;
  int row = sload(ww + 0);
  int g = sload(ww + 1);
  int p = sload(ww + 2);
  int remaining = sload(ww + 3);
  int part = sload(ww + 4);
  // ids of the first range's first three pages (no table lookup before the first loads)
  int pid0 = sload(ww + 5);
  int pid1 = sload(ww + 6);
  int pid2 = sload(ww + 7);
  int tbl_off = sload(a.rows + row * 4 + 0);
  int vis = sload(a.rows + row * 4 + 1);
  int qrow = sload(a.rows + row * 4 + 2);
  int pstart = sload(a.rows + row * 4 + 3);   // first page of the row's own range (pages before it
                                                                       // are a shared prefix handled by the tile kernel)
  bool first_range = true;

  while (remaining > 0) {
    const int np = (vis + kP - 1) / kP;
    const int cnt = min(remaining, np - p);
    const int32_t* tbl = a.pt + tbl_off + p;

    // q chunks of this lane for the G heads of kv head g
    uint4 q[G][2];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const uint8_t* qp = (const uint8_t*)a.q + ((int64_t)qrow * a.Hq + g * GT + h0 + h) * kRowBytes + j * 16;
      q[h][0] = *(const uint4*)qp;
      q[h][1] = *(const uint4*)(qp + kHalfBytes);
    }
    float m[G], l[G], acc[G][DPL];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      m[h] = -1e30f;
      l[h] = 0.f;
#pragma unroll
      for (int d = 0; d < DPL; ++d) acc[h][d] = 0.f;
    }

    const uint8_t* slab0 = a.pool + (int64_t)g * kSlab + lane * 16;
    // tokens of page index pi (absolute, within the row) that exist: the row's last page may be ragged
    auto compute = [&](PageRegs& R, int pi) {
      const int nvalid = vis - pi * kP;          // >= 1; >= 16 for a full page
      if (nvalid < kP) {
        // ragged last page: slots past the file's end hold whatever was there before (possibly
        // NaN patterns); their weight is 0, but 0 * NaN is NaN, so clear their V chunks
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
          if ((hf * 8 + r) >= nvalid) {
            R.v[hf] = make_uint4(0, 0, 0, 0);
            R.v[2 + hf] = make_uint4(0, 0, 0, 0);
          }
      }
      float s[2][G];
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const bool valid = (hf * 8 + r) < nvalid;
#pragma unroll
        for (int h = 0; h < G; ++h) {
          float x = E::dot(R.k[hf], q[h][0], 0.f);
          x = E::dot(R.k[2 + hf], q[h][1], x);
          x = octet_sum(x) * a.scale_log2e;
          s[hf][h] = valid ? x : -__builtin_inff();
        }
      }
      bool need = false;
#pragma unroll
      for (int h = 0; h < G; ++h) need |= fmaxf(s[0][h], s[1][h]) > m[h] + kTau;
      if (__builtin_amdgcn_ballot_w64(need) != 0) {     // rare after the first page
#pragma unroll
        for (int h = 0; h < G; ++h) {
          const float mn = fmaxf(m[h], fmaxf(s[0][h], s[1][h]));
          const float al = __builtin_amdgcn_exp2f(m[h] - mn);
          l[h] *= al;
#pragma unroll
          for (int d = 0; d < DPL; ++d) acc[h][d] *= al;
          m[h] = mn;
        }
      }
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        float pw[G];
#pragma unroll
        for (int h = 0; h < G; ++h) {
          pw[h] = __builtin_amdgcn_exp2f(s[hf][h] - m[h]);
          l[h] += pw[h];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          float vf[C];
          E::unpack(R.v[i * 2 + hf], vf);
#pragma unroll
          for (int h = 0; h < G; ++h)
#pragma unroll
            for (int e = 0; e < C; ++e) acc[h][i * C + e] = __builtin_fmaf(pw[h], vf[e], acc[h][i * C + e]);
        }
      }
    };

    // Page ids come through the scalar cache, two pages ahead of their K/V loads.  Every load in
    // the loop is unconditional, so the loop body has no control-flow join between a prefetch and
    // its use and the compiler can wait for exactly the older page while the newer one is in
    // flight.  Past the end of the range the prefetch is pointed at page 0 of the pool (valid
    // memory that every wave touches, so it stays in L2) and its data is never used.
    const int last = cnt - 1;
    if (!first_range) {
      // (page ids as vector loads: through the scalar cache 128 files of 1000..3000 tokens in fp32 take 185 us instead of 178)
      pid0 = tbl[0];
      pid1 = tbl[min(1, last)];
      pid2 = tbl[min(2, last)];
    }
    first_range = false;
    static_assert(kPair, "one wavefront per range is decode_stream's job");
    {
      // this wavefront's half (K or V) of a page: 4 lane-linear 1 KiB runs -> registers -> LDS
      const uint8_t* half0 = slab0 + hs * kBlk;
      auto load_half = [&](uint4 (&st)[4], int pid) {
        const uint8_t* base = half0 + (int64_t)pid * a.page_bytes;
#pragma unroll
        for (int x = 0; x < 4; ++x) st[x] = __builtin_bit_cast(uint4, __builtin_nontemporal_load((const u32x4_t*)(base + x * 1024)));
      };
      int id1 = cnt > 1 ? pid1 : 0, id2 = cnt > 2 ? pid2 : 0;
      uint4 sa[4], sb[4];                    // pages k and k+1 in flight
      load_half(sa, pid0);
      load_half(sb, id1);
      for (int k = 0; k < cnt; k += 2) {
        // page k
        {
          uint8_t* buf = plds[0] + hs * kBlk + lane * 16;
#pragma unroll
          for (int x = 0; x < 4; ++x) *(uint4*)(buf + x * 1024) = sa[x];
          __syncthreads();                   // both halves of page k are in LDS; the other buffer is free again
          load_half(sa, id2);
          id2 = k + 4 <= last ? tbl[k + 4] : 0;
          PageRegs R;
          const uint8_t* rb = plds[0] + lane * 16;
#pragma unroll
          for (int x = 0; x < 4; ++x) R.k[x] = *(const uint4*)(rb + x * 1024);
#pragma unroll
          for (int x = 0; x < 4; ++x) R.v[x] = *(const uint4*)(rb + kBlk + x * 1024);
          compute(R, p + k);
        }
        // page k + 1 (both wavefronts take the same branch: cnt is the same for the pair)
        {
          uint8_t* buf = plds[1] + hs * kBlk + lane * 16;
#pragma unroll
          for (int x = 0; x < 4; ++x) *(uint4*)(buf + x * 1024) = sb[x];
          __syncthreads();
          id1 = k + 3 <= last ? tbl[k + 3] : 0;
          load_half(sb, id1);
          if (k + 1 < cnt) {
            PageRegs R;
            const uint8_t* rb = plds[1] + lane * 16;
#pragma unroll
            for (int x = 0; x < 4; ++x) R.k[x] = *(const uint4*)(rb + x * 1024);
#pragma unroll
            for (int x = 0; x < 4; ++x) R.v[x] = *(const uint4*)(rb + kBlk + x * 1024);
            compute(R, p + k + 1);
          }
        }
      }
      __syncthreads();                       // the next range of this pair reuses both buffers
    }

    // ---- end of a (row, kv head) range: combine the 8 token slots (lanes with equal j).
    // Per head: common max M, rescale, total sum.  The G*DPL accumulators are then reduced with
    // a halving exchange (lane bit 5, 4, 3 in turn: keep one half of the list, send the other), so
    // lane (r, j) ends up owning the fully reduced values r*V/8 .. r*V/8 + V/8 - 1 of the list.
    const bool whole = (p == 0 && cnt == np);
    constexpr int V = G * DPL;
    float vals[V];
    float lsum[G], Mh[G];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float M = m[h];
      M = fmaxf(M, row_xor8(M));
      M = fmaxf(M, __shfl_xor(M, 16));
      M = fmaxf(M, __shfl_xor(M, 32));
      const float f = __builtin_amdgcn_exp2f(m[h] - M);
      float ls = l[h] * f;
      ls += row_xor8(ls);
      ls += __shfl_xor(ls, 16);
      ls += __shfl_xor(ls, 32);
      lsum[h] = ls;
      Mh[h] = M;
#pragma unroll
      for (int d = 0; d < DPL; ++d) vals[h * DPL + d] = acc[h][d] * f;
    }
    {
      const bool b5 = (lane & 32) != 0, b4 = (lane & 16) != 0, b3 = (lane & 8) != 0;
#pragma unroll
      for (int i = 0; i < V / 2; ++i) {
        const float keep = b5 ? vals[i + V / 2] : vals[i], send = b5 ? vals[i] : vals[i + V / 2];
        vals[i] = keep + __shfl_xor(send, 32);
      }
#pragma unroll
      for (int i = 0; i < V / 4; ++i) {
        const float keep = b4 ? vals[i + V / 4] : vals[i], send = b4 ? vals[i] : vals[i + V / 4];
        vals[i] = keep + __shfl_xor(send, 16);
      }
#pragma unroll
      for (int i = 0; i < V / 8; ++i) {
        const float keep = b3 ? vals[i + V / 8] : vals[i], send = b3 ? vals[i] : vals[i + V / 8];
        vals[i] = keep + row_xor8(send);
      }
    }
    // lane (r, j) now holds list entries idx = r * V/8 + t: head idx / DPL, lane-local dim idx % DPL
    const int64_t out_row = ((int64_t)qrow * a.Hq + g * GT + h0) * D;
    if (whole) {
#pragma unroll
      for (int t = 0; t < V / 8; ++t) {
        const int idx = r * (V / 8) + t, h = idx / DPL, dl = idx % DPL;
        float ls = lsum[0];
#pragma unroll
        for (int hh = 1; hh < G; ++hh) ls = (h == hh) ? lsum[hh] : ls;
        a.out[out_row + h * D + (dl / C) * (D / 2) + j * C + (dl % C)] = vals[t] / ls;
      }
    } else {
      float* pa = a.part_acc + ((int64_t)part * GT + h0) * D;
#pragma unroll
      for (int t = 0; t < V / 8; ++t) {
        const int idx = r * (V / 8) + t, h = idx / DPL, dl = idx % DPL;
        pa[h * D + (dl / C) * (D / 2) + j * C + (dl % C)] = vals[t];
      }
      if (lane < G) {
        float mm = Mh[0], ll = lsum[0];
#pragma unroll
        for (int hh = 1; hh < G; ++hh) {
          mm = (lane == hh) ? Mh[hh] : mm;
          ll = (lane == hh) ? lsum[hh] : ll;
        }
        a.part_ml[((int64_t)part * GT + h0 + lane) * 2 + 0] = mm;
        a.part_ml[((int64_t)part * GT + h0 + lane) * 2 + 1] = ll;
      }
    }
    if (!whole) ++part;
    remaining -= cnt;
    p += cnt;
    if (p == np) {
      if (++g == a.Hkv) {
        g = 0;
        ++row;
        if (remaining > 0) {
          tbl_off = sload(a.rows + row * 4 + 0);
          vis = sload(a.rows + row * 4 + 1);
          qrow = sload(a.rows + row * 4 + 2);
          pstart = sload(a.rows + row * 4 + 3);
        }
      }
      p = pstart;
    }
  }
}

// ---------------------------------------------------------------------------------------
// Prefill-chunk attention on the matrix cores (bf16 storage, D = 128).  One workgroup of 4
// wavefronts per tile = (LIP, kv head, TQ = 128/G consecutive new tokens): 128 query rows
// (token, head of the group), 32 per wavefront.  The file's K/V is walked in blocks of 32 tokens
// (two pages), staged through LDS and shared by the 4 wavefronts.  The same kernel serves
// shared-prefix tiles: 128 rows = the decode rows (members x heads) of LIPs whose files begin
// with the same pages; it reads those pages once for all of them and leaves partial results.
//
// Everything is computed transposed so that what belongs to one query row lives in one lane:
//   S^T[token][row] = K · Q^T      v_mfma_f32_32x32x16_bf16, A = K rows from LDS, B = Q (registers)
//   O^T[dim][row]  += V^T · P^T    v_mfma_f32_32x32x16_f16,  A = V^T from LDS, B = P (registers)
// In both results a lane's column is its query row (lane % 32), so the running max, the sum and
// the rescale factor are lane-local, and the 16 scores a lane holds are, in register order,
// exactly the 8+8 token slots it must supply as the B operand of the two PV steps.  The two
// lanes of a row (lane, lane ^ 32) hold different tokens / dims and share only the max.
// P is rounded to fp16 (2^-11; bf16's 2^-8 would not fit a 2e-3 bar on rows with few keys) and
// the softmax sum adds the rounded weights, so the output is an exact weighted mean of V rows
// for slightly perturbed weights.  The rounding is to nearest: cut off, the weights would all be low by half a unit but for each
// maximum's, which is exactly 1, and a tile cut into key chunks has a maximum per chunk (error against 64 bits, prompts of
// 16..1000 tokens on up to 5500: whole tiles, cut off 2.04e-4; chunks, cut off 2.05e-4 and up to 6 % above the whole tile's;
// chunks, to nearest 1.53e-4, nowhere above; the same time).  (The pieces of a tile split over wavefronts are still cut off.)
// V is converted bf16 -> fp16 while it is transposed into LDS:
// packing the same dim of two neighbouring tokens into one register IS the transposition.
// ---------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8_t;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

constexpr int kKvBlock = 32;              // tokens per K/V block
constexpr int kKLds = kKvBlock * kRowBytes;      // 8 KiB: K block, 16-byte chunks, xor-swizzled
constexpr int kVRow = 80;                 // bytes per dim row of V^T in LDS (64 + 16 pad: conflict-free reads)
constexpr int kVLds = 128 * kVRow;        // 10 KiB

template <int G, int TW, bool SPLIT>
__device__ __forceinline__ void tile_block(const PrefillArgs& a, const int block, uint8_t (*lds)[kKLds + kVLds]) {
  // TW = wavefronts of the workgroup (4 or 8); a tile has 32 * TW query rows that share one staging
  // of every K/V block, so K/V bytes read per flop (from L2, and written to LDS) halve with TW = 8.
  // (Two 32-row column tiles per wavefront instead, four wavefronts per 256-row tile, halve the LDS
  // reads per flop but need ~510 registers, one wavefront per SIMD: measured 1.5x slower, also with
  // the pipelined block loop below.)
  constexpr int CT = 1;
  // workgroups go round-robin over the 8 XCDs; the tile list comes in 8 shares in which tiles that read the same K/V are
  // neighbours (one L2 per XCD): of equal cost, longest first, or, where all are about equal pieces of cut tiles, of equal count
  // A start is the order table, the tile's record, then everything else at once: the offsets of the shares are kernel arguments,
  // and the record names the first block's pages, whose loads need no table lookup.  (As a chain of about ten scalar loads, 0.2 us
  // each: fork tree of 16 x 16 81.5 -> 80.7 us, three ragged prompts 72.0 -> 71.3, the mixed batch the same.)
  int tile = a.xcd_off[0], tile_end = a.xcd_off[1];
#pragma unroll
  for (int x = 1; x < 8; ++x)
    if (block % 8 == x) {
      tile = a.xcd_off[x];
      tile_end = a.xcd_off[x + 1];
    }
  tile += block / 8;
  if (tile >= tile_end) return;
  const int32_t* tw = a.tiles + (int64_t)tile * 12;
  int rec[12];
#pragma unroll
  for (int i = 0; i < 12; ++i) rec[i] = sload(tw + i);
  hold(rec[0], rec[1], rec[2], rec[3], rec[4], rec[5], rec[6], rec[7], rec[8], rec[9], rec[10], rec[11]);
  const int tbl_off = rec[0], g = rec[4], count = rec[3];
  const bool shared = rec[6] == 1;
  const bool partial = rec[6] != 0;               // shared prefixes and key chunks leave partials
  const int32_t* tbl = a.pt + tbl_off;

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int col = lane & 31, hf = lane >> 5;
  // prefill chunk: `count` new tokens from chunk offset t0 on a file of L tokens; row tl sees
  // tokens 0 .. L + t0 + tl.  shared prefix: `count` decode rows (q rows in the member list) that
  // all see the same full pages [page0, page1) of the group's first file.
  const int L = rec[1], t0 = rec[5];
  // key chunk of a prefill tile: the same rows over the blocks of pages [page0, page1) only (some rows may see none of them)
  const int lim = partial ? rec[8] * kP : 0x7fffffff;
  const int kv_end = shared ? lim : min(L + t0 + count, lim);    // tokens the tile's last row sees
  const int mask_from = shared ? lim : min(L + t0 + 1, lim);     // first token some row may not see
  const int kb0 = partial ? rec[7] / 2 : 0;                       // first 32-token block (page0 is even)
  const int nblk = (kv_end + kKvBlock - 1) / kKvBlock;
  const int last_page = max((kv_end + kP - 1) / kP - 1, 0);
  // A shared-prefix tile of four wavefronts with at most 64 live rows would keep two of them busy, each alone
  // with the whole chain of a block (operand reads, eight chained score MFMAs, weights, PV) in every step.
  // Such a tile is split by key block instead: wavefronts 0 and 1 take the rows for the even blocks,
  // wavefronts 2 and 3 the same rows for the odd blocks, and each does half of a block's chain per
  // step (scores and weights of its block in one step, PV in the next); the two halves are combined
  // through LDS at the end like two pieces of a split range.
  // (A kernel of its own, chosen by the host when every tile of the batch is such a tile: with both block
  // loops in one kernel the register allocator spills inside them.)
  static_assert(!SPLIT || TW == 4, "only four-wavefront tiles are split");
  constexpr bool split = SPLIT;
  const int pair = split ? (wv >> 1) : 0;
  const int wvr = split ? (wv & 1) : wv;                         // which 32 rows of the tile
  const int wvu = __builtin_amdgcn_readfirstlane(wv);
  const bool wave_live = (TW == 8 ? wvu : wvr) * 32 * CT < count * G;      // a wavefront whose rows are all padding only stages (eight wavefronts: a scalar)

  // ---- staging roles
  // K: thread copies chunk c = tid (and tid + 256 with four wavefronts) of the block: token c/16, dim chunk c%16
  // V: thread takes tokens (4*q4 + 2*up, +1) of page pg, dim chunk vc: VD dims x 2 tokens
  constexpr int VD = TW == 4 ? 8 : 4;                       // dims per thread
  const int up = tid & 1, q4 = (tid >> 1) & 3, vc = (tid >> 3) & (128 / VD - 1), pg = tid >> (TW == 4 ? 7 : 8);
  // K/V of the blocks in flight.  Four wavefronts: loaded three blocks ahead of their use, three register sets.  Eight: two blocks
  // ahead of their way into LDS, which is three ahead of their use; the third set serves the start alone.
  uint4 ka0, ka1, va0, va1, kb0r, kb1r, vb0, vb1, kc0, kc1, vc0, vc1;
  const uint8_t* slab = a.pool + (int64_t)g * kSlab;
  // Which of the block's two pages a thread stages is the same for its whole wavefront, so the page
  // ids come through the scalar cache and the page base is scalar arithmetic; what differs per
  // thread is a fixed offset inside the page, computed once.
  const int k_page = TW == 4 ? 0 : (wvu >> 2);            // chunk tid: page of the block (chunk tid + 256: the other one)
  const int v_page = TW == 4 ? (wvu >> 1) : (wvu >> 2);
  const int kt = (tid >> 4) & 15, kdc = tid & 15;
  const int k_off = (kdc >> 3) * (kP * kHalfBytes) + kt * kHalfBytes + (kdc & 7) * 16;
  const int dbyte = vc * VD * 2;                            // byte offset of the thread's dims in the 256-byte row
  const int v_off = kBlk + (dbyte >> 7) * (kP * kHalfBytes) + (4 * q4 + 2 * up) * kHalfBytes + (dbyte & 127);
  auto page_id = [&](int pi) { return sload(tbl + min(pi, last_page)); };
  // K/V of a block, its two pages by their ids (eight wavefronts: a wavefront needs one of them)
  auto issue_pages = [&](int id0, int id1, uint4& k0, uint4& k1, uint4& v0, uint4& v1) {
    const uint8_t* p0 = slab + (int64_t)id0 * a.page_bytes;
    const uint8_t* p1 = slab + (int64_t)id1 * a.page_bytes;
    const uint8_t* pk = k_page ? p1 : p0;
    // four-wavefront tiles are shared-prefix tiles, and each of those streams K/V of its own (nobody reads a
    // line twice): nontemporal loads.  Prefill tiles share their stream with seven neighbours through L2.
    auto ld16 = [&](const uint8_t* q16) {
      if constexpr (TW == 4) return __builtin_bit_cast(uint4, __builtin_nontemporal_load((const u32x4_t*)q16));
      else return *(const uint4*)q16;
    };
    k0 = ld16(pk + k_off);
    if constexpr (TW == 4) k1 = ld16(p1 + k_off);
    const uint8_t* p = (v_page ? p1 : p0) + v_off;
    if constexpr (TW == 4) {
      v0 = ld16(p);
      v1 = ld16(p + kHalfBytes);
    } else {
      const uint2 x0 = *(const uint2*)p, x1 = *(const uint2*)(p + kHalfBytes);
      v0.x = x0.x; v0.y = x0.y;
      v1.x = x1.x; v1.y = x1.y;
    }
  };
  auto issue_loads = [&](int kb, uint4& k0, uint4& k1, uint4& v0, uint4& v1) { issue_pages(page_id(2 * kb), page_id(2 * kb + 1), k0, k1, v0, v1); };
  int tl[CT], h[CT], qrow[CT], vis[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const int rho = (wvr * CT + ct) * 32 + col;    // query row of this lane inside the tile
    tl[ct] = rho / G;                              // token (prefill) or member (shared prefix) of the row
    h[ct] = rho % G;
    const int tlc = min(tl[ct], count - 1);        // rows past the tile's last token/member repeat it (never written)
    qrow[ct] = shared ? a.members[rec[2] + tlc] : rec[2] + tlc;
    vis[ct] = shared ? kv_end : min(L + t0 + tlc + 1, lim);   // tokens this row sees
  }
  // the first block by the record's ids; those of the blocks behind it are on their way meanwhile, all in one round trip
  constexpr int kAhead = SPLIT ? 3 : TW == 8 ? 5 : 2;
  int ids[kAhead][2];
#pragma unroll
  for (int i = 0; i < kAhead; ++i) {
    ids[i][0] = page_id(2 * (kb0 + 1 + i) + (TW == 4 ? 0 : k_page));
    ids[i][1] = TW == 4 ? page_id(2 * (kb0 + 1 + i) + 1) : ids[i][0];
  }
  issue_pages(rec[10], rec[11], ka0, ka1, va0, va1);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < kAhead; ++i) hold(ids[i][0], ids[i][1]);
  bf16x8_t q[CT][8];             // Q of this lane's rows: 8 k-steps of 16 dims, this lane supplies dims 16*ks + 8*hf .. +8
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const uint8_t* qp = (const uint8_t*)a.q + ((int64_t)qrow[ct] * a.Hq + g * G + h[ct]) * kRowBytes + hf * 16;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) q[ct][ks] = __builtin_bit_cast(bf16x8_t, *(const uint4*)(qp + ks * 32));
  }

  auto k_dst = [&](uint8_t* base, int c) {
    const int t = c >> 4, dc = c & 15;
    return base + (t * 16 + (dc ^ (t & 15))) * 16;
  };
  auto store_k = [&](uint8_t* base, const uint4& k0, const uint4& k1) {
    *(uint4*)k_dst(base, tid) = k0;
    if constexpr (TW == 4) *(uint4*)k_dst(base, tid + 256) = k1;
  };
  auto store_v = [&](int kb, uint8_t* base, const uint4& v0, const uint4& v1, bool masked) {
    // tokens past the end of what the tile may see are cleared (their weight is 0, 0 * NaN is not);
    // only the last block can hold such tokens
    const int tok = kb * kKvBlock + pg * 16 + 4 * q4 + 2 * up;
    const bool tail = masked && kb * kKvBlock + kKvBlock > kv_end;
    const bool ok0 = !tail || tok < kv_end, ok1 = !tail || tok + 1 < kv_end;
    uint8_t* vb = base + kKLds + (2 * pg + (q4 & 1)) * 16 + (q4 >> 1) * 8 + up * 4 + vc * VD * kVRow;
    auto put = [&](int e, uint32_t lo_word0, uint32_t lo_word1, bool high) {
      const uint32_t x0 = high ? (lo_word0 & 0xffff0000u) : (lo_word0 << 16);
      const uint32_t x1 = high ? (lo_word1 & 0xffff0000u) : (lo_word1 << 16);
      const float f0 = ok0 ? as_f32(x0) : 0.f, f1 = ok1 ? as_f32(x1) : 0.f;
      *(uint32_t*)(vb + e * kVRow) = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(f0, f1));
    };
    put(0, v0.x, v1.x, false); put(1, v0.x, v1.x, true);
    put(2, v0.y, v1.y, false); put(3, v0.y, v1.y, true);
    if constexpr (TW == 4) {
      put(4, v0.z, v1.z, false); put(5, v0.z, v1.z, true);
      put(6, v0.w, v1.w, false); put(7, v0.w, v1.w, true);
    }
  };
  auto store_lds = [&](int kb, uint8_t* base, const uint4& k0, const uint4& k1, const uint4& v0, const uint4& v1) {
    store_k(base, k0, k1);
    store_v(kb, base, v0, v1, true);
  };

  f32x16_t O[CT][4];
  float m[CT], l[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    m[ct] = -1e30f;
    l[ct] = 0.f;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) O[ct][db][v] = 0.f;
  }

  // Four wavefronts: the block loop is software-pipelined over three LDS buffers (eight: see below).  One step: block kb + 1 (loaded three
  // steps ago) goes from registers to LDS, the loads of block kb + 4 are issued into the same
  // registers, then the matrix cores start S^T = K Q^T of block kb + 1 while the vector units do the
  // softmax arithmetic of block kb, and O^T += V^T P^T of block kb follows.  So the MFMAs of one block
  // run under the vector work of its neighbour inside one wavefront, not only across wavefronts.
  // All loads and all blocks are unconditional: past the end the last pages are loaded again and
  // every token is masked, so the loop (unrolled by three) has no control-flow join between a load
  // and its use.  One barrier per step: the buffer a step writes was last read two steps earlier.
  auto k_operands = [&](const uint8_t* base, bf16x8_t (&kk)[8]) {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) kk[ks] = *(const bf16x8_t*)(base + (col * 16 + ((2 * ks + hf) ^ (col & 15))) * 16);
  };
  auto scores = [&](const bf16x8_t (&kk)[8]) {
    f32x16_t S;
#pragma unroll
    for (int v = 0; v < 16; ++v) S[v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk[ks], q[0][ks], S, 0, 0, 0);
    return S;
  };
  f32x16_t Sc;                   // scores of the current block (computed one step ahead)
  float mx_cur = 0.f;            // their row maximum in log2 units, both lanes of the row agreeing
  // Causal mask and row maximum of the scores in Sc (block kb), done as soon as the scores exist, at the
  // end of the step before the one that uses them: the exchange between the two lanes of a row goes
  // through the LDS pipe, and there it must not queue behind the sixteen operand reads of its own step
  // with the MFMAs waiting for the branch that needs it.
  // value v of a lane is token 8*(v/4) + 4*hf + v%4 of the block
  // scores stay unscaled; the scale (softmax scale * log2 e, positive) goes into one fma with the max
  auto mask_and_max = [&](const int kb) __attribute__((always_inline)) {
    const int tok0 = kb * kKvBlock + 4 * hf;
    const bool edge = kb * kKvBlock + kKvBlock > mask_from;      // the block reaches the causal edge of some row
    float mx = -__builtin_inff();
    if (edge) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int tok = tok0 + 8 * (v >> 2) + (v & 3);
        Sc[v] = tok < vis[0] ? Sc[v] : -__builtin_inff();
      }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) mx = fmaxf(mx, Sc[v]);
    mx_cur = fmaxf(mx, __shfl_xor(mx, 32)) * a.scale_log2e;
  };
  auto step = [&](const int kb, uint8_t* cur, uint8_t* nxt, uint4& k0, uint4& k1, uint4& v0, uint4& v1) {
    store_lds(kb + 1, nxt, k0, k1, v0, v1);
    __syncthreads();           // block kb + 1 is in LDS; everyone is done with the block that was in `nxt` before
    issue_loads(kb + 4, k0, k1, v0, v1);
    if (!wave_live) return;

    // operands of both MFMA phases are requested from LDS up front: the latency is paid once per step
    bf16x8_t kk[8];
    k_operands(nxt, kk);
    const uint8_t* vbase = cur + kKLds + col * kVRow + hf * 16;
    f16x8_t vv[4][2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int db = 0; db < 4; ++db) vv[db][ks] = *(const f16x8_t*)(vbase + db * 32 * kVRow + ks * 32);
    __builtin_amdgcn_sched_barrier(0);

    // the block's row maximum was found at the end of the step before (mask_and_max)
    const float mx = mx_cur;
    if (__builtin_amdgcn_ballot_w64(mx > m[0] + kTau) != 0) {     // rare after the first block
      const float mn = fmaxf(m[0], mx);
      const float al = __builtin_amdgcn_exp2f(m[0] - mn);
      l[0] *= al;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) O[0][db][v] *= al;
      m[0] = mn;
    }
    // From here to the end of the step there is no branch: the scores of block kb + 1 (eight MFMAs)
    // run under the exponentials of block kb; then the weights of the block's first 16 tokens, their
    // O^T += V^T P^T MFMAs (four independent accumulators), and the second 16 tokens' weights while those run.
    const f32x16_t Sn = scores(kk);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      uint32_t pw[4];
#pragma unroll
      for (int u = 0; u < 8; u += 2) {
        const int v = 8 * ks + u;
        const f16x2_t pk = {(_Float16)__builtin_amdgcn_exp2f(__builtin_fmaf(Sc[v], a.scale_log2e, -m[0])),
                            (_Float16)__builtin_amdgcn_exp2f(__builtin_fmaf(Sc[v + 1], a.scale_log2e, -m[0]))};
        l[0] = __builtin_amdgcn_fdot2(pk, f16x2_t{(_Float16)1.0f, (_Float16)1.0f}, l[0], false);
        pw[u >> 1] = __builtin_bit_cast(uint32_t, pk);
      }
      const f16x8_t P = __builtin_bit_cast(f16x8_t, make_uint4(pw[0], pw[1], pw[2], pw[3]));
#pragma unroll
      for (int db = 0; db < 4; ++db) O[0][db] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vv[db][ks], P, O[0][db], 0, 0, 0);
    }
    // issue order of this stretch: one MFMA, then a few vector instructions, sixteen times (the first
    // eight MFMAs are the scores of the next block, which depend on nothing computed here)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x402, 4, 0);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x402, 2, 0);
    }
    Sc = Sn;
    mask_and_max(kb + 1);
  };

  // A tile split by key block (see `split` above).  The pair whose block it is computes scores, maximum and
  // weights of block kb + 1 (K in `nxt`) in step kb and the PV product of that block (V^T then in `cur`) in
  // step kb + 1, while the other pair does the same one block later: the buffers are read in the same steps
  // as in the unsplit loop, so three of them and one barrier per step still do.
  uint32_t pwc[2][4] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}};
  auto first_half = [&](const int kb, const uint8_t* kbuf) {
    bf16x8_t kk[8];
    k_operands(kbuf, kk);
    Sc = scores(kk);
    mask_and_max(kb);
    const float mx = mx_cur;
    if (__builtin_amdgcn_ballot_w64(mx > m[0] + kTau) != 0) {
      const float mn = fmaxf(m[0], mx);
      const float al = __builtin_amdgcn_exp2f(m[0] - mn);
      l[0] *= al;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) O[0][db][v] *= al;
      m[0] = mn;
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int u = 0; u < 8; u += 2) {
        const int v = 8 * ks + u;
        const auto pk = __builtin_amdgcn_cvt_pkrtz(__builtin_amdgcn_exp2f(__builtin_fmaf(Sc[v], a.scale_log2e, -m[0])),
                                                   __builtin_amdgcn_exp2f(__builtin_fmaf(Sc[v + 1], a.scale_log2e, -m[0])));
        l[0] = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2_t, pk), f16x2_t{(_Float16)1.0f, (_Float16)1.0f}, l[0], false);
        pwc[ks][u >> 1] = __builtin_bit_cast(uint32_t, pk);
      }
  };
  auto second_half = [&](const uint8_t* vbuf) {
    const uint8_t* vbase = vbuf + kKLds + col * kVRow + hf * 16;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const f16x8_t P = __builtin_bit_cast(f16x8_t, make_uint4(pwc[ks][0], pwc[ks][1], pwc[ks][2], pwc[ks][3]));
#pragma unroll
      for (int db = 0; db < 4; ++db)
        O[0][db] = __builtin_amdgcn_mfma_f32_32x32x16_f16(*(const f16x8_t*)(vbase + db * 32 * kVRow + ks * 32), P, O[0][db], 0, 0, 0);
    }
  };
  auto step_split = [&](const int kb, const uint8_t* cur, uint8_t* nxt, uint4& k0, uint4& k1, uint4& v0, uint4& v1) {
    store_lds(kb + 1, nxt, k0, k1, v0, v1);
    __syncthreads();
    issue_loads(kb + 5, k0, k1, v0, v1);
    if (!wave_live) return;
    if (((kb - kb0) & 1) == pair) second_half(cur);
    else first_half(kb + 1, nxt);
  };

  if constexpr (SPLIT) {
    // This kernel has registers to spare: a fourth set of staging registers (and a fourth LDS buffer, so that
    // the loop unrolled by four addresses them statically) puts the loads four blocks ahead of their use.
    // These tiles each stream K/V of their own, and what bounds them is the bytes in flight.
    uint4 kd0, kd1, vd0, vd1;
    issue_pages(ids[0][0], ids[0][1], kb0r, kb1r, vb0, vb1);
    issue_pages(ids[1][0], ids[1][1], kc0, kc1, vc0, vc1);
    issue_pages(ids[2][0], ids[2][1], kd0, kd1, vd0, vd1);
    store_lds(kb0, lds[0], ka0, ka1, va0, va1);
    __syncthreads();
    issue_loads(kb0 + 4, ka0, ka1, va0, va1);
    if (wave_live && pair == 0) first_half(kb0, lds[0]);
    for (int kb = kb0; kb < nblk; kb += 4) {
      step_split(kb, lds[0], lds[1], kb0r, kb1r, vb0, vb1);
      step_split(kb + 1, lds[1], lds[2], kc0, kc1, vc0, vc1);
      step_split(kb + 2, lds[2], lds[3], kd0, kd1, vd0, vd1);
      step_split(kb + 3, lds[3], lds[0], ka0, ka1, va0, va1);
    }
    // the odd blocks' half (wavefronts 2, 3) goes to the even blocks' (wavefronts 0, 1) through LDS: per
    // lane maximum, sum and the 64 accumulator values
    __syncthreads();
    float* xch = (float*)lds[0] + (wvr * 66) * 64 + lane;
    if (pair == 1) {
      xch[0] = m[0];
      xch[64] = l[0];
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) xch[(2 + db * 16 + v) * 64] = O[0][db][v];
    }
    __syncthreads();
    if (pair == 1) return;
    {
      const float m1 = xch[0], l1 = xch[64];
      const float mn = fmaxf(m[0], m1);
      const float a0 = __builtin_amdgcn_exp2f(m[0] - mn), a1 = __builtin_amdgcn_exp2f(m1 - mn);
      l[0] = l[0] * a0 + l1 * a1;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) O[0][db][v] = O[0][db][v] * a0 + xch[(2 + db * 16 + v) * 64] * a1;
      m[0] = mn;
    }
  } else if constexpr (TW == 8) {
    // Eight wavefronts, two on a SIMD: while wavefronts 0..3 are in a matrix phase (scores of the next block, weights x V of this
    // one: sixteen MFMAs whose operands all lie in registers), wavefronts 4..7 are in a vector phase (operands of their next
    // matrix phase from LDS, mask, maximum, exponentials), and at the next barrier they change over.  In step with each other the two
    // want the same unit at the same time: a step took 2500 cycles for 1024 of MFMA.  Staging belongs to the matrix phase, whose issue slots are
    // free between its MFMAs; in the vector phase it makes that the longer one (1914 us against 1520 in step and 1365 now).
    // Four LDS buffers: in the matrix phase that follows block kb's weights a wavefront stores block kb + 3 over block kb - 1, which the
    // other half read last two phases before; it is complete one phase before its first reader.
    // What bounds it is the power limit: 32 chunks of 512 tokens on U{0..8192}: 3.17 M -> 2.50 M cycles, at 2.14 -> 1.91 GHz.  Whole calls:
    // that batch 1520 -> 1365 us, three ragged prompts 68.5 -> 62.7, the mixed batch 1905 -> 1708.  Without the priority of the matrix
    // phase 1387; MFMAs and vector instructions in a prescribed order 1363; page ids a phase earlier 1425 (the scheduler then puts the
    // scores behind the products with V, and the other half waits for them).
    issue_pages(ids[0][0], ids[0][0], kb0r, kb1r, vb0, vb1);
    issue_pages(ids[1][0], ids[1][0], kc0, kc1, vc0, vc1);
    store_lds(kb0, lds[0], ka0, ka1, va0, va1);
    issue_pages(ids[2][0], ids[2][0], ka0, ka1, va0, va1);
    store_lds(kb0 + 1, lds[1], kb0r, kb1r, vb0, vb1);
    issue_pages(ids[3][0], ids[3][0], kb0r, kb1r, vb0, vb1);
    store_lds(kb0 + 2, lds[2], kc0, kc1, vc0, vc1);
    int next_id = ids[4][0];                           // page of the block to be requested next, fetched a step ahead
    int k_at[8];                                       // this lane's operands in a K block: held, or each read adds its parts up again
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      k_at[ks] = (col * 16 + ((2 * ks + hf) ^ (col & 15))) * 16;
      asm volatile("" : "+v"(k_at[ks]));
    }
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) asm volatile("" : "+v"(q[0][ks]));      // Q is here: no wait for it in the loop
    __syncthreads();
    // The walk over the blocks, for a wavefront with rows and for one that only stages.
    auto walk = [&](auto live_) __attribute__((always_inline)) {
      constexpr bool live = decltype(live_)::value;
      bf16x8_t kk[8];                                  // operands of the next matrix phase
      f16x8_t vv[4][2], P[2];
      auto read_k = [&](const uint8_t* base) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) kk[ks] = *(const bf16x8_t*)(base + k_at[ks]);
      };
      if constexpr (live) {
        read_k(lds[0]);
        Sc = scores(kk);
      }
      // Block kb: its vector phase, then the matrix phase behind it.  K is of block kb + 1 in `nxt`, V^T of block kb in `cur`; block
      // kb + 3 goes from its registers to `stage`.  Returns whether block kb was the last (the scores then computed are of no use).
      auto turn = [&](const int kb, const uint8_t* cur, const uint8_t* nxt, uint8_t* stage, uint4& k0, uint4& k1, uint4& v0, uint4& v1) __attribute__((always_inline)) {
        if constexpr (live) {
          read_k(nxt);
          const uint8_t* vbase = cur + kKLds + col * kVRow + hf * 16;
#pragma unroll
          for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int db = 0; db < 4; ++db) vv[db][ks] = *(const f16x8_t*)(vbase + db * 32 * kVRow + ks * 32);
          if (kb * kKvBlock + kKvBlock > mask_from) {    // the block reaches the causal edge of some row
            const int tok0 = kb * kKvBlock + 4 * hf;
#pragma unroll
            for (int v = 0; v < 16; ++v) Sc[v] = tok0 + 8 * (v >> 2) + (v & 3) < vis[0] ? Sc[v] : -__builtin_inff();
          }
          float mx = -__builtin_inff();
#pragma unroll
          for (int v = 0; v < 16; ++v) mx = fmaxf(mx, Sc[v]);
          mx = pair32_max(mx) * a.scale_log2e;
          if (__builtin_amdgcn_ballot_w64(mx > m[0] + kTau) != 0) {     // rare after the first block
            const float mn = fmaxf(m[0], mx);
            const float al = __builtin_amdgcn_exp2f(m[0] - mn);
            l[0] *= al;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
              for (int v = 0; v < 16; ++v) O[0][db][v] *= al;
            m[0] = mn;
          }
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) {
            uint32_t pw[4];
#pragma unroll
            for (int u = 0; u < 8; u += 2) {
              const int v = 8 * ks + u;
              const f16x2_t pk = {(_Float16)__builtin_amdgcn_exp2f(__builtin_fmaf(Sc[v], a.scale_log2e, -m[0])),
                                  (_Float16)__builtin_amdgcn_exp2f(__builtin_fmaf(Sc[v + 1], a.scale_log2e, -m[0]))};
              l[0] = __builtin_amdgcn_fdot2(pk, f16x2_t{(_Float16)1.0f, (_Float16)1.0f}, l[0], false);
              pw[u >> 1] = __builtin_bit_cast(uint32_t, pk);
            }
            P[ks] = __builtin_bit_cast(f16x8_t, make_uint4(pw[0], pw[1], pw[2], pw[3]));
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
        if constexpr (live) {
          Sc = scores(kk);
#pragma unroll
          for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int db = 0; db < 4; ++db) O[0][db] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vv[db][ks], P[ks], O[0][db], 0, 0, 0);
        }
        store_k(stage, k0, k1);
        store_v(kb + 3, stage, v0, v1, false);
        if ((kb + 4) * kKvBlock > kv_end) store_v(kb + 3, stage, v0, v1, true);      // again, without the tokens past the end
        issue_pages(next_id, next_id, k0, k1, v0, v1);   // block kb + 5
        next_id = page_id(2 * (kb + 6) + k_page);
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        return kb + 1 >= nblk;
      };
      for (int kb = kb0;; kb += 4) {
        if (turn(kb, lds[0], lds[1], lds[3], ka0, ka1, va0, va1)) break;
        if (turn(kb + 1, lds[1], lds[2], lds[0], kb0r, kb1r, vb0, vb1)) break;
        if (turn(kb + 2, lds[2], lds[3], lds[1], ka0, ka1, va0, va1)) break;
        if (turn(kb + 3, lds[3], lds[0], lds[2], kb0r, kb1r, vb0, vb1)) break;
      }
    };
    if (wvu >= 4) __syncthreads();                     // half a step behind; the other half waits for it at the end
    if (wave_live) walk(std::true_type{});
    else walk(std::false_type{});
    if (wvu < 4) __syncthreads();
  } else {
  issue_pages(ids[0][0], ids[0][1], kb0r, kb1r, vb0, vb1);
  issue_pages(ids[1][0], ids[1][1], kc0, kc1, vc0, vc1);
  store_lds(kb0, lds[0], ka0, ka1, va0, va1);
  __syncthreads();
  issue_loads(kb0 + 3, ka0, ka1, va0, va1);
  if (wave_live) {
    bf16x8_t kk[8];
    k_operands(lds[0], kk);
    Sc = scores(kk);
    mask_and_max(kb0);
  }
  for (int kb = kb0; kb < nblk; kb += 3) {
    step(kb, lds[0], lds[1], kb0r, kb1r, vb0, vb1);
    step(kb + 1, lds[1], lds[2], kc0, kc1, vc0, vc1);
    step(kb + 2, lds[2], lds[0], ka0, ka1, va0, va1);
  }
  }

  // Results.  In the accumulators a lane holds 16 bytes at a time of a row of its own: stored like that, an instruction touches
  // 64 lines.  Each wavefront turns its 32 rows through LDS, 32 dims at a time (rows of 36 floats), and stores whole 128-byte
  // lines, eight rows per instruction.  Whole calls: 16 prompts of 600..1000 tokens on nothing 204 -> 199 us, 8 x 512 tokens on
  // U{0..8000} 320 -> 317.  A tile of at most two wavefronts' rows has few lines to store and would only wait for the turning: kernel
  // time, straight / through LDS, 32 rows 0.89 (on nothing) .. 0.97 (on 1500), 64 rows 0.94 .. 0.98, 128 rows 1.02, 256 rows
  // 1.05 .. 1.10 (420 shapes); fork trees, whose split tiles are always such, 0.97 .. 1.00.
  const float lt = l[0] + __shfl_xor(l[0], 32);
  const float inv = partial ? 1.0f : 1.0f / lt;
  // first partial slot of the tile, or its first q / out row
  const int64_t row0 = partial ? (int64_t)(shared ? t0 : rec[9]) : (int64_t)rec[2];
  if (partial && hf == 0 && tl[0] < count) {           // partials: unnormalised accumulator, max, sum, for the merge kernel
    float* ml = a.part_ml + ((row0 + tl[0]) * G + h[0]) * 2;
    ml[0] = m[0];
    ml[1] = lt;
  }
  if (SPLIT || count * G <= 64) {
    if (tl[0] < count) {
      float* o = (partial ? a.part_acc + ((row0 + tl[0]) * G + h[0]) * 128 : a.out + ((row0 + tl[0]) * a.Hq + g * G + h[0]) * 128) + 4 * hf;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int vb = 0; vb < 4; ++vb)
          *(float4*)(o + db * 32 + vb * 8) = make_float4(O[0][db][4 * vb] * inv, O[0][db][4 * vb + 1] * inv, O[0][db][4 * vb + 2] * inv, O[0][db][4 * vb + 3] * inv);
    }
    return;
  }
  __syncthreads();                                     // everyone is done with the block buffers
  float* const stg = (float*)lds[0] + wvr * (32 * 36);
  const int r8 = lane >> 3, c4 = (lane & 7) * 4;
#pragma unroll
  for (int db = 0; db < 4; ++db) {
#pragma unroll
    for (int vb = 0; vb < 4; ++vb)
      *(float4*)(stg + col * 36 + vb * 8 + hf * 4) = make_float4(O[0][db][4 * vb] * inv, O[0][db][4 * vb + 1] * inv, O[0][db][4 * vb + 2] * inv, O[0][db][4 * vb + 3] * inv);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = i * 8 + r8, rho = wvr * 32 + row, tlr = rho / G;
      const float4 x = *(const float4*)(stg + row * 36 + c4);
      if (tlr < count) {
        float* o = partial ? a.part_acc + ((row0 + tlr) * G + rho % G) * 128 : a.out + ((row0 + tlr) * a.Hq + g * G + rho % G) * 128;
        *(float4*)(o + db * 32 + c4) = x;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// ---------------------------------------------------------------------------------------
// Decode ranges on the matrix cores (bf16 storage).  With 8 query heads per kv head the VALU
// decode kernel above is bound by vector issue, not by HBM (8 flop per KV byte in plain fp32
// FMAs); the 8 heads of a group are a small query tile, so here one wavefront per range feeds
// them to 16x16x32 MFMAs (16 columns, GT of them used):
//   S^T[16 tokens][16 heads] = K · Q^T     A = K rows straight from global memory (64 B per token and
//                                          k-step, no LDS), B = Q (registers), per page
//   O^T[128 dims][16 heads] += V^T · P^T    per two pages (k = 32 tokens); V^T through a wavefront-private
//                                          LDS buffer, written by the wavefront itself while it converts
//                                          bf16 -> fp16 (pairs of neighbouring tokens packed = the transpose)
// A lane's column is a head in both results, so max / sum / rescale factor are lane-local; the
// four lane groups of a head hold different tokens and share only the (lagging) running max.
// No barrier anywhere: the LDS buffer is private to the wavefront.
// A row may hold nt <= 16 / GT consecutive new tokens of one LIP (a short draft being verified,
// paper section 4.1): column c is then (token c / GT, head c % GT), token t sees vis + t file
// tokens, and the page loop runs to the last token's limit: one pass over K/V for all of them.
// ---------------------------------------------------------------------------------------
constexpr int kVtRow = 80;                    // bytes per dim row of V^T (32 tokens fp16 + 16 pad)
constexpr int kVtLds = 128 * kVtRow;          // 10 KiB per wavefront

// Two plans (see the descriptor): the global cut (BINS = false: a wavefront per range of the cut, every piece of a divided range a
// partial in device memory), and bins (BINS = true), as in decode_bins: what the wavefronts of a workgroup divide is combined
// through LDS when they are done.  A row of four draft tokens leaves 8 KiB per piece, so with the global cut a batch of drafts
// wrote and read again 21 MB beside 604 MB of K/V.  Bins in a launch of their own, i.e. in batches without tiles.  Before / after:
// drafts of 4 on 64 files of 512..4096 tokens 134.3 / 121.1 us, 8 query heads per kv head on 16 files of 32 k..131 k 709 / 694; per layer,
// 64 query heads: one file of 2000 tokens 18.3 / 15.6, four of 100..300 17.1 / 12.2, 64 of 512..4096 120.7 / 113.1; drafts of 3 on 64 files of
// 500..900 52.3 / 46.3.  Eight wavefronts in 150 KiB of LDS, one workgroup per compute unit: with two of four a cut divides twice as
// many ranges (drafts 133, short drafts 55.5 against 53.5).
constexpr int kMxRow = 132;                                    // floats per query column of a piece in LDS: 128 dims, max, sum, 2 spare
constexpr int kMxSlot = 16 * kMxRow * 4;                       // a piece: 16 columns
constexpr int kMxWave = kVtLds + kMxSlot;                      // LDS of a wavefront: its V buffer, where its last piece goes when it is done, and its first piece
static_assert(kMxSlot <= kVtLds, "the last piece takes the V buffer's place");

template <int GT, bool BINS, bool STREAM>
__device__ __forceinline__ void decode_mfma_ranges(const DecodeArgs& a, const int block, const int W, uint8_t* lds) {
  const int lane = threadIdx.x & 63;
  const int wib = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wv = block * W + wib;
  if (BINS ? block >= a.n_bins : wv >= a.n_waves) return;        // (bins: the whole workgroup)
  uint8_t* const vlds = lds + wib * (BINS ? kMxWave : kVtLds);
  const int col = lane & 15, grp = lane >> 4;        // query column, lane group (tokens 4*grp .. 4*grp+3 of a page)
  const int head = col % GT;                          // columns past nt * GT repeat earlier ones; their results are ignored
  const int vq4 = lane >> 4, vc = lane & 15;          // V staging role: tokens 4*vq4 .. +3 of a page, dim chunk vc

  // As in the VALU kernel, the wavefront's units form ONE stream: a load cursor runs ahead of the compute
  // cursor through the same sequence of (row, kv head) ranges, in steps of a pair of pages (a pair never
  // straddles two ranges: the last pair of a range with an odd number of pages has one page), so the
  // K/V loads of the next range are in flight while the current one is finished and written out.
  const BinStart st = BINS ? bin_start(a, block, W, wib) : BinStart{};
  const int32_t* ww = a.waves + (int64_t)wv * 8;
  // compute cursor: the range (bins: segment, number `row`) being accumulated: pages [pstart, np), tokens its first token sees,
  // q row * Hq + first head, new tokens
  int row = BINS ? st.seg : sload(ww + 0), g = BINS ? 0 : sload(ww + 1), p = BINS ? st.p : sload(ww + 2);
  int remaining = BINS ? st.units : sload(ww + 3);
  int part = BINS ? 0 : sload(ww + 4);                // global cut: the next partial; bins: the segment's destination
  int m_g = 0, m_qh = 0, m_dest = 0;                  // of the segment whose pieces it merges at the end
  auto merge_record = [&]() __attribute__((always_inline)) {
    const int32_t* msr = a.segs + (int64_t)(st.merges ? st.m_seg : 0) * 8;
    m_g = sload(msr + 1);
    m_qh = sload(msr + 5);
    m_dest = sload(msr + 6);
  };
  if constexpr (BINS) merge_record();
  if (!BINS || remaining > 0) {
  const int32_t* sr = a.segs + (int64_t)row * 8;
  const int tbl0 = BINS ? sload(sr + 0) : sload(a.rows + row * 4 + 0);
  int vis = BINS ? sload(sr + 4) : sload(a.rows + row * 4 + 1);
  int qh = BINS ? sload(sr + 5) : sload(a.rows + row * 4 + 2) * a.Hq + g * GT;
  const int ps0 = BINS ? sload(sr + 1) : sload(a.rows + row * 4 + 3);      // (tokens - 1) << 28 | kv head (bins) or first page
  int pstart = BINS ? sload(sr + 2) : ps0 & 0x0fffffff;
  int nt = (ps0 >> 28) + 1;                           // new tokens in the row
  int np = BINS ? sload(sr + 3) : (vis + nt - 1 + kP - 1) / kP;              // bins: the segment's end; else the pages the row's last token sees
  if constexpr (BINS) part = sload(sr + 6);
  // load cursor: the pair whose K/V is requested next
  int lg = BINS ? ps0 & 0x0fffffff : g, lrow = row, lp = p, lnp = np, ltbl = tbl0, lpstart = pstart, lrem = remaining;
  // page ids of that pair (the first pair's come with the wave record; a pair of one page: the second is not used)
  int id0 = BINS ? st.id0 : sload(ww + 5), id1 = BINS ? st.id1 : sload(ww + 6);
  // record of the row (bins: segment) after the load cursor's, fetched a whole row ahead (one past the last row: valid words, never used)
  int n_tbl = 0, n_np = 0, n_pstart = 0, n_g = 0;
  auto fetch_next_row = [&](int rr) __attribute__((always_inline)) {
    if constexpr (BINS) {
      const int32_t* q4 = a.segs + (int64_t)rr * 8;
      n_tbl = sload(q4 + 0);
      n_g = sload(q4 + 1) & 0x0fffffff;
      n_pstart = sload(q4 + 2);
      n_np = sload(q4 + 3);
    } else {
      n_tbl = sload(a.rows + rr * 4 + 0);
      const int v = sload(a.rows + rr * 4 + 1), ps = sload(a.rows + rr * 4 + 3);
      n_pstart = ps & 0x0fffffff;
      n_np = (v + (ps >> 28) + kP - 1) / kP;
    }
  };
  fetch_next_row(row + 1);
  // record of row + 1 as the compute side needs it
  int c_nvis = 0, c_nqrow = 0, c_nps = 0, c_pb = 0, c_pe = 0, c_dest = 0;
  auto fetch_compute_next_row = [&]() __attribute__((always_inline)) {
    if constexpr (BINS) {
      const int32_t* q8 = a.segs + (int64_t)(row + 1) * 8;
      c_nps = sload(q8 + 1);
      c_pb = sload(q8 + 2);
      c_pe = sload(q8 + 3);
      c_nvis = sload(q8 + 4);
      c_nqrow = sload(q8 + 5);
      c_dest = sload(q8 + 6);
    } else {
      c_nvis = sload(a.rows + (row + 1) * 4 + 1);
      c_nqrow = sload(a.rows + (row + 1) * 4 + 2);
      c_nps = sload(a.rows + (row + 1) * 4 + 3);
    }
  };
  fetch_compute_next_row();

  // K of a page as the A operand: token col, chunk 4*ks + grp of its row (row half ks/2, chunk 4*(ks%2) + grp)
  const int k_off = col * kHalfBytes + grp * 16;
  // V of a page for the staging: tokens 4*vq4 + u, chunk vc
  const int v_off = kBlk + (vc >> 3) * (kP * kHalfBytes) + (4 * vq4) * kHalfBytes + (vc & 7) * 16;
  auto load_page = [&](uint4 (&kk)[4], uint4 (&vv)[4], const uint8_t* slab, int pid) __attribute__((always_inline)) {
    const uint8_t* base = slab + (int64_t)pid * a.page_bytes;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) kk[ks] = ld16<STREAM>(base + k_off + (ks >> 1) * (kP * kHalfBytes) + (ks & 1) * 64);
#pragma unroll
    for (int u = 0; u < 4; ++u) vv[u] = ld16<STREAM>(base + v_off + u * kHalfBytes);
  };
  // Requests the next pair and moves the load cursor; every load is unconditional (a page that does not
  // exist, also past the end of the wavefront's work, is page 0 of the pool and is never used).
  auto load_next_pair = [&](uint4 (&k0)[4], uint4 (&v0)[4], uint4 (&k1)[4], uint4 (&v1)[4]) __attribute__((always_inline)) {
    const int take = min(2, min(lrem, lnp - lp));
    const uint8_t* slab = a.pool + (int64_t)(take > 0 ? lg : 0) * kSlab;
    load_page(k0, v0, slab, take > 0 ? id0 : 0);
    load_page(k1, v1, slab, take > 1 ? id1 : 0);
    if (take > 0) {
      lrem -= take;
      lp += take;
      if (lp == lnp) {                                 // the range after: next head of the row, or the next row; bins: the next segment
        if (BINS || ++lg == a.Hkv) {
          lg = BINS ? n_g : 0;
          ++lrow;
          ltbl = n_tbl;
          lnp = n_np;
          lpstart = n_pstart;
          fetch_next_row(lrow + 1);
        }
        lp = lpstart;
      }
      const int t2 = min(2, min(lrem, lnp - lp));      // ids of the pair after this one, used one pair later
      id0 = t2 > 0 ? sload(a.pt + ltbl + lp) : 0;
      id1 = t2 > 1 ? sload(a.pt + ltbl + lp + 1) : 0;
    }
  };

  // state of the range being accumulated
  int tok = 0;                                        // this column's token within the row
  bf16x8_t q[4];                                      // Q^T operand: this lane's (token, head), dims 32*ks + 8*grp .. +8
  auto load_q = [&]() __attribute__((always_inline)) {
    tok = min(col / GT, nt - 1);
    const uint8_t* qp = (const uint8_t*)a.q + ((int64_t)qh + tok * a.Hq + head) * kRowBytes + grp * 16;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) q[ks] = __builtin_bit_cast(bf16x8_t, *(const uint4*)(qp + ks * 64));
  };
  f32x4_t O[8];
  float m = -1e30f, l = 0.f;
  auto reset_state = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int db = 0; db < 8; ++db) O[db] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    m = -1e30f;
    l = 0.f;
  };
  reset_state();
  load_q();
  int p_first = p;                                    // first page of the piece being accumulated
  int piece = 0;                                      // pieces this wavefront has finished

  // scores of one page: 4 tokens (4*grp + v) x this lane's head; tokens past nvalid masked
  auto scores = [&](const uint4 (&kk)[4], int nvalid, float (&sc)[4]) __attribute__((always_inline)) {
    f32x4_t S = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kk[ks]), q[ks], S, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) sc[v] = (4 * grp + v) < nvalid ? S[v] : -__builtin_inff();
  };
  // V of one page -> fp16, transposed, into the wavefront's LDS buffer (half pg of every dim row)
  auto stage_v = [&](const uint4 (&vv)[4], int nvalid, int pg) __attribute__((always_inline)) {
    const uint32_t w[4][4] = {{vv[0].x, vv[0].y, vv[0].z, vv[0].w}, {vv[1].x, vv[1].y, vv[1].z, vv[1].w},
                              {vv[2].x, vv[2].y, vv[2].z, vv[2].w}, {vv[3].x, vv[3].y, vv[3].z, vv[3].w}};
    bool ok[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) ok[u] = (4 * vq4 + u) < nvalid;      // slots past the file's end may hold anything
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float f[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t x = (e & 1) ? (w[u][e >> 1] & 0xffff0000u) : (w[u][e >> 1] << 16);
        f[u] = ok[u] ? as_f32(x) : 0.f;
      }
      const int d = vc * 8 + e;
      uint2 pk;
      pk.x = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(f[0], f[1]));
      pk.y = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(f[2], f[3]));
      *(uint2*)(vlds + d * kVtRow + ((vq4 ^ ((d >> 4) & 3)) * 16) + pg * 8) = pk;
    }
  };
  // two pages (32 tokens): scores, softmax weights, O^T += V^T P^T
  auto compute2 = [&](const uint4 (&kA)[4], const uint4 (&vA)[4], const uint4 (&kB)[4], const uint4 (&vB)[4], int piA, bool haveB) __attribute__((always_inline)) {
    // tokens of the page visible to this column's token; slots that hold file tokens at all
    const int nvA = vis + tok - piA * kP, nvB = haveB ? nvA - kP : 0;
    const int nsA = vis + nt - 1 - piA * kP, nsB = haveB ? nsA - kP : 0;
    float sA[4], sB[4];
    scores(kA, nvA, sA);
    scores(kB, nvB, sB);
    stage_v(vA, nsA, 0);
    stage_v(vB, nsB, 1);
    const float mx = fmaxf(fmaxf(fmaxf(sA[0], sA[1]), fmaxf(sA[2], sA[3])), fmaxf(fmaxf(sB[0], sB[1]), fmaxf(sB[2], sB[3]))) * a.scale_log2e;
    if (__builtin_amdgcn_ballot_w64(mx > m + kTau) != 0) {       // rare after the first pages
      float mn = fmaxf(m, mx);
      mn = fmaxf(mn, __shfl_xor(mn, 16));
      mn = fmaxf(mn, __shfl_xor(mn, 32));                        // all four lane groups of the head agree
      const float al = __builtin_amdgcn_exp2f(m - mn);
      l *= al;
#pragma unroll
      for (int db = 0; db < 8; ++db)
#pragma unroll
        for (int v = 0; v < 4; ++v) O[db][v] *= al;
      m = mn;
    }
    uint32_t pw[4];
#pragma unroll
    for (int v = 0; v < 4; v += 2) {
      const auto pa = __builtin_amdgcn_cvt_pkrtz(__builtin_amdgcn_exp2f(__builtin_fmaf(sA[v], a.scale_log2e, -m)),
                                                 __builtin_amdgcn_exp2f(__builtin_fmaf(sA[v + 1], a.scale_log2e, -m)));
      const auto pb = __builtin_amdgcn_cvt_pkrtz(__builtin_amdgcn_exp2f(__builtin_fmaf(sB[v], a.scale_log2e, -m)),
                                                 __builtin_amdgcn_exp2f(__builtin_fmaf(sB[v + 1], a.scale_log2e, -m)));
      l = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2_t, pa), f16x2_t{(_Float16)1.0f, (_Float16)1.0f}, l, false);
      l = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2_t, pb), f16x2_t{(_Float16)1.0f, (_Float16)1.0f}, l, false);
      pw[v >> 1] = __builtin_bit_cast(uint32_t, pa);
      pw[2 + (v >> 1)] = __builtin_bit_cast(uint32_t, pb);
    }
    const f16x8_t P = __builtin_bit_cast(f16x8_t, make_uint4(pw[0], pw[1], pw[2], pw[3]));
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      const f16x8_t vt = *(const f16x8_t*)(vlds + (db * 16 + col) * kVtRow + ((grp ^ (db & 3)) * 16));
      O[db] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vt, P, O[db], 0, 0, 0);
    }
  };

  // End of a piece: the four lane groups of a head add up their sums, O^T is complete; the compute cursor
  // moves to the next range first, so that its query rows are on their way while this piece is written.
  auto finish_piece = [&]() __attribute__((always_inline)) {
    const bool whole = p_first == (BINS ? pstart : 0) && p == np;
    const int64_t o_row = (int64_t)qh + tok * a.Hq + head;
    const int64_t o_slot = (int64_t)(part + tok) * GT + head;     // a piece leaves one partial per token of the row
    const bool o_live = col < nt * GT;
    const bool o_final = BINS ? part < 0 : true;                   // what a whole piece writes: the output, or (bins) a partial
    if (!BINS && !whole) part += nt;
    const bool more = remaining > 0;
    if (more) {
      if (BINS || ++g == a.Hkv) {
        g = 0;
        ++row;
        vis = c_nvis;
        nt = (c_nps >> 28) + 1;
        if constexpr (BINS) {
          qh = c_nqrow;
          pstart = c_pb;
          np = c_pe;
          part = c_dest;
        } else {
          qh = c_nqrow * a.Hq;
          pstart = c_nps & 0x0fffffff;
          np = (vis + nt - 1 + kP - 1) / kP;
        }
        fetch_compute_next_row();
      } else {
        qh += GT;
      }
      load_q();
    }
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (o_live) {
      if (BINS && !whole) {
        float* o = (float*)(piece == 0 ? vlds + kVtLds : vlds) + col * kMxRow + 4 * grp;
#pragma unroll
        for (int db = 0; db < 8; ++db) *(float4*)(o + db * 16) = make_float4(O[db][0], O[db][1], O[db][2], O[db][3]);
        if (grp == 0) *(float2*)(o + 128) = make_float2(m, l);
      } else if (whole && o_final) {
        const float inv = 1.0f / l;
        float* o = a.out + o_row * 128 + 4 * grp;
#pragma unroll
        for (int db = 0; db < 8; ++db) *(float4*)(o + db * 16) = make_float4(O[db][0] * inv, O[db][1] * inv, O[db][2] * inv, O[db][3] * inv);
      } else {
        float* o = a.part_acc + o_slot * 128 + 4 * grp;
#pragma unroll
        for (int db = 0; db < 8; ++db) *(float4*)(o + db * 16) = make_float4(O[db][0], O[db][1], O[db][2], O[db][3]);
        if (grp == 0) {
          a.part_ml[o_slot * 2 + 0] = m;
          a.part_ml[o_slot * 2 + 1] = l;
        }
      }
    }
    ++piece;
    if (more) {
      p = pstart;
      p_first = p;
      reset_state();
    }
  };
  // one pair of the stream: accumulate it, move the compute cursor, close the piece at the end of the range or of the wavefront's work
  auto do_pair = [&](const uint4 (&kA)[4], const uint4 (&vA)[4], const uint4 (&kB)[4], const uint4 (&vB)[4]) __attribute__((always_inline)) {
    const int took = max(1, min(2, min(remaining, np - p)));     // >= 1 whatever the descriptor says: the loop ends
    compute2(kA, vA, kB, vB, p, took > 1);
    p += took;
    remaining -= took;
    if (p == np || remaining == 0) finish_piece();
  };

  // pair k in registers while pair k + 1 is in flight
  uint4 kA[4], vA[4], kB[4], vB[4], kC[4], vC[4], kD[4], vD[4];
  load_next_pair(kA, vA, kB, vB);
  load_next_pair(kC, vC, kD, vD);
  while (remaining > 0) {
    do_pair(kA, vA, kB, vB);
    load_next_pair(kA, vA, kB, vB);
    if (remaining > 0) do_pair(kC, vC, kD, vD);
    load_next_pair(kC, vC, kD, vD);
  }
  }
  if constexpr (!BINS) return;
  __syncthreads();                                       // every piece of the bin is in LDS (or went straight to its destination)
  if (!st.merges) return;
  // four columns at a time: lane group `grp` has one, its lanes dims 4 (lane % 16) .. +3 and the same plus 64
  const int m_cols = ((m_g >> 28) + 1) * GT, d0 = 4 * (lane & 15);
#pragma unroll
  for (int c0 = 0; c0 < 16; c0 += 4) {
    const int c = c0 + grp;
    if (c >= m_cols) continue;
    float M = -__builtin_inff(), ls = 0.f;
    f32x4_t x = {0.f, 0.f, 0.f, 0.f}, y = x;
    for (int i = 0; i < st.m_pieces; ++i) {
      const int slot = i == 0 ? st.m_slot : 2 * (st.m_wave + i);
      const float* pc = (const float*)(lds + (slot >> 1) * kMxWave + (slot & 1 ? 0 : kVtLds)) + c * kMxRow;
      const float mi = pc[128], li = pc[129], mn = fmaxf(M, mi);
      const float sc = __builtin_amdgcn_exp2f(M - mn), wt = __builtin_amdgcn_exp2f(mi - mn);      // sc: 0 for the first piece
      ls = ls * sc + li * wt;
      M = mn;
      x = x * sc + *(const f32x4_t*)(pc + d0) * wt;
      y = y * sc + *(const f32x4_t*)(pc + d0 + 64) * wt;
    }
    const int t = c / GT, h = c % GT;
    if (m_dest < 0) {
      const float inv = 1.0f / ls;
      float* o = a.out + ((int64_t)m_qh + t * a.Hq + h) * 128 + d0;
      *(f32x4_t*)o = x * inv;
      *(f32x4_t*)(o + 64) = y * inv;
    } else {
      const int64_t o_slot = (int64_t)(m_dest + t) * GT + h;
      float* o = a.part_acc + o_slot * 128 + d0;
      *(f32x4_t*)o = x;
      *(f32x4_t*)(o + 64) = y;
      if ((lane & 15) == 0) {
        a.part_ml[o_slot * 2 + 0] = M;
        a.part_ml[o_slot * 2 + 1] = ls;
      }
    }
  }
}

template <int GT>
__global__ __launch_bounds__(256, 2) void decode_mfma_kernel(DecodeArgs da) {
  __shared__ __align__(16) uint8_t vlds[kWavesPerBlock * kVtLds];
  decode_mfma_ranges<GT, false, true>(da, blockIdx.x, kWavesPerBlock, vlds);
}
template <int GT, int W, bool STREAM>
__global__ __launch_bounds__(64 * W, 8 / W) void decode_mfma_bins_kernel(DecodeArgs da) {
  __shared__ __align__(16) uint8_t lds[W * kMxWave];
  decode_mfma_ranges<GT, true, STREAM>(da, blockIdx.x, W, lds);
}

// ---------------------------------------------------------------------------------------
// The attention launch of a batch: workgroups that run tiles (prefill chunks and shared prefixes)
// and workgroups that run decode ranges (one wavefront per range) in ONE grid, so the two kinds of
// work fill the GPU together and there is no launch boundary between them.
// ---------------------------------------------------------------------------------------
template <typename E, int G, int TW, bool SPLIT = false>
__global__ __launch_bounds__(64 * TW, 8 / TW) void attn_kernel(DecodeArgs da, PrefillArgs pa) {
  // Workgroups come in groups of eight (one per XCD, which the tile order relies on).  The host's table says what a
  // group runs: tile group g (g >= 0) or decode group ~g.  By default the decode groups are spread among the
  // first half of the tile groups, so that some CUs stream K/V from HBM for decode ranges while the others keep
  // the matrix cores busy: the two kinds of work are bound by different units.  (Measured on the mixed batch:
  // 1.85 ms against 1.91 ms with all tiles first; spread over the whole grid: 2.02 ms.  A CU that runs decode
  // ranges alone has only its eight wavefronts' loads in flight, so the gain is small.)
  if constexpr (E::kDimsPerChunk == 8)
    hold(pa.group_map, pa.tiles, pa.pt, pa.pool, pa.page_bytes, pa.q, pa.members, pa.Hq, pa.scale_log2e, pa.xcd_off[0], pa.xcd_off[1], pa.xcd_off[2], pa.xcd_off[3],
         pa.xcd_off[4], pa.xcd_off[5], pa.xcd_off[6], pa.xcd_off[7], pa.xcd_off[8], da.waves, da.lmerge, da.segs, da.n_bins);
  const uint32_t j = blockIdx.x >> 3, x = blockIdx.x & 7;
  const int32_t g = pa.group_map ? sload(pa.group_map + j) : (int32_t)j;   // no table: tiles only
  const bool is_decode = g < 0;
  // LDS: the K/V buffers of a tile workgroup, or the piece slots of a decode bin (a workgroup is one or the other)
  constexpr int kTileLds = E::kDimsPerChunk == 8 ? (SPLIT || TW == 8 ? 4 : 3) * (kKLds + kVLds) : 0;      // tiles exist for bf16 storage only
  constexpr int kBinLds = G < 8 ? 2 * TW * BinLds<E, G < 8 ? G : 1>::kSlot * 4 : 0;
  constexpr int kLds = kTileLds > kBinLds ? kTileLds : (kBinLds > 16 ? kBinLds : 16);
  __shared__ __align__(16) uint8_t lds[kLds];
  if constexpr (E::kDimsPerChunk == 8) {
    if (!is_decode) {
      tile_block<G, TW, SPLIT>(pa, (int)(g * 8 + x), (uint8_t(*)[kKLds + kVLds])lds);
      return;
    }
  }
  if constexpr (G < 8) {
    if (is_decode) bins_of<E, G, true>(da, (int)(~g * 8 + x), TW, (float*)lds);
  }
}

// A batch without tiles (plain decode): the decode bins alone, W wavefronts per bin.
template <typename E, int G, int W, bool STREAM>
__global__ __launch_bounds__(64 * W, 8 / W) void decode_only_kernel(DecodeArgs da) {
  __shared__ __align__(16) float lds[2 * W * BinLds<E, G>::kSlot];
  bins_of<E, G, STREAM>(da, (int)blockIdx.x, W, lds);
}

// Decode ranges for 8 query heads per kv head: one workgroup of two wavefronts per range.
template <typename E>
__global__ __launch_bounds__(128, 2) void decode_pair_kernel(DecodeArgs da) {
  __shared__ __align__(16) uint8_t plds[2][kSlab];
  decode_ranges<E, 8, 4>(da, blockIdx.x, plds);
}

// ---------------------------------------------------------------------------------------
// Row tiles: several new tokens of a LIP in fp32 storage (prompts, chunks of prompts, drafts) on the fp32 matrix cores.
// A workgroup = 32 query rows (32 / G tokens x G heads of one kv head) as two column tiles of 16; its eight wavefronts take
// every eighth page of the file each, on their own, and their results are combined through LDS at the end, so that even a
// prompt of a few hundred tokens gives every compute unit a short chain.  Per page and wavefront, everything transposed as in
// the bf16 kernels (a lane's column is its query row):
//   S^T[16 tokens][16 rows] = K · Q^T     16 x v_mfma_f32_16x16x4_f32: step s, lane group g supplies dim 16 g + s, so a lane
//                                          reads 64 consecutive bytes of one token's K row; Q comes from LDS
//   O^T[64 dims][16 rows]  += V^T · P^T   4 steps x 4 dim blocks: step v, lane group g supplies token 4 g + v, which is the
//                                          token whose score the lane holds in register v; block d holds dims 4 i + d, so a
//                                          lane reads 16 consecutive bytes of V per token
// K and V come straight from global memory in whole 1 KiB wavefront loads: no barrier in the loop, no transpose.  V of a page is
// requested before its scores are computed and K of the next page after them, so one set of registers each is enough and four
// wavefronts fit on a SIMD (<= 128 registers, which is why Q waits in LDS: 8 reads per page beside 128 MFMAs).  Bound: fp32 matrix
// cores (a page costs a wavefront 64 MFMAs of 32 cycles per column tile for 8 KiB of K/V).
// All sums and weights are fp32, and sums are short: a page's products are added up by themselves before they meet the
// accumulator, one rounding per page at its size instead of 16, and so are four chunks in the merge.  Error against 64 bits, 4..200
// new tokens on 0..8000, tiles / rows of the vector-unit kernel: 0.67..0.92 (products added to the accumulator one by one: 1.06
// with 4 tokens, on 500 tokens up to 1.23; short sums cost nothing: 31.6 / 31.3 us for the prompts below).
// A row must not meet what it does not see, also where that is not finite (0 * Inf is NaN): such V elements of the tile's own
// tokens are left out of the products and added at the end.
// Measured, whole calls: four prompts of 64..512 tokens on new files, 8 heads: 538 -> 31 us (as rows of the vector-unit kernel: 67 us
// of kernel that re-read the file per token, and 0.5 ms of planning for 13 500 ranges); 8 prompts of 400..500 tokens on 500, 16
// query heads: 1250 -> 138 us (77 of 157 TFLOP/s).
// ---------------------------------------------------------------------------------------
constexpr int kRowTileWaves = 8;
constexpr int kRowTileRows = 32;
constexpr int kRowTileStride = 68;            // floats per row of the exchange buffer: 64 dims + 4 (16-byte stores of 16 rows hit all banks)

template <int G>
__global__ __launch_bounds__(64 * kRowTileWaves, 4) void row_tile_kernel(PrefillArgs a) {
  __shared__ __align__(16) float xch[kRowTileWaves / 2][kRowTileRows][kRowTileStride];
  __shared__ float stat[kRowTileWaves][kRowTileRows][2];          // (max, sum) per wavefront and row
  __shared__ int left_out[kRowTileWaves];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int col = lane & 15, grp = lane >> 4;
  const int32_t* t = a.rtiles + (int64_t)blockIdx.x * 8;
  const int32_t* tbl = a.pt + sload(t + 0);
  const int vis0 = sload(t + 1), qrow = sload(t + 2), count = sload(t + 3), head = sload(t + 4);
  const int page0 = sload(t + 5), page1 = sload(t + 6), dest = sload(t + 7);
  const int kv_end = vis0 + count - 1;                             // tokens the tile's last row sees
  const bool two = count * G > 16;                                 // the second column tile holds rows

  // Q waits in the exchange buffer, where each wavefront reads it page by page: the loop has no registers to spare for it
  const int rho = threadIdx.x >> 4;
  const int64_t q_at = (int64_t)(qrow + min(rho / G, count - 1)) * a.Hq + head * G + rho % G;      // rows past the last token repeat it (never written)
  const f32x4_t q_part = ((const f32x4_t*)((const uint8_t*)a.q + q_at * kRowBytes))[threadIdx.x & 15];
  int vis[2];
#pragma unroll
  for (int ct = 0; ct < 2; ++ct) vis[ct] = vis0 + min((ct * 16 + col) / G, count - 1);
  f32x4_t O[2][4];
  float m[2], l[2];
#pragma unroll
  for (int ct = 0; ct < 2; ++ct) {
    m[ct] = -1e30f;
    l[ct] = 0.f;
#pragma unroll
    for (int db = 0; db < 4; ++db) O[ct][db] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }

  const uint8_t* slab = a.pool + (int64_t)head * kSlab;
  // a page's address in scalar registers and the lane's offset in one of its own (left to itself the compiler keeps 64-bit sums
  // and extended offsets, two registers each, through the loop, which has none to spare)
  auto at = [&](int id, int part, uint32_t off) __attribute__((always_inline)) {
    auto b = (const __attribute__((address_space(1))) uint8_t*)(slab + (int64_t)id * a.page_bytes + part);
    asm("" : "+s"(b));
    asm("" : "+v"(off));
    return (const f32x4_t*)(b + off);
  };
  const uint32_t k_off = (grp >> 1) * (kP * kHalfBytes) + col * kHalfBytes + (grp & 1) * 64;        // token col, dims 16 grp .. +15
  const uint32_t v_off = (col >> 3) * (kP * kHalfBytes) + (4 * grp) * kHalfBytes + (col & 7) * 16;   // tokens 4 grp + v, dims 4 col .. +3
  f32x4_t kk[4], vv[4];
  int p = page0 + wv;
  int pid = p < page1 ? sload(tbl + p) : 0;                        // a wavefront without pages: page 0, loaded and never used
  {
    const f32x4_t* kp = at(pid, 0, k_off);
#pragma unroll
    for (int i = 0; i < 4; ++i) kk[i] = kp[i];
  }
  *(f32x4_t*)&xch[0][rho][(threadIdx.x & 15) * 4] = q_part;
  __syncthreads();
  bool odd = false;                                                // V elements of the tile's own tokens were left out
  for (; p < page1; p += kRowTileWaves) {
    const f32x4_t* vp = at(pid, kBlk, v_off);
#pragma unroll
    for (int v = 0; v < 4; ++v) vv[v] = vp[v * (kHalfBytes / 16)];
    pid = p + kRowTileWaves < page1 ? sload(tbl + p + kRowTileWaves) : 0;
    // eight sums of 8 products each, added up as a tree: one chain of 64 would round three times as coarsely as the
    // vector units' eight lanes per score
    f32x4_t S[2];
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
      if (ct == 0 || two) {
        f32x4_t q[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) q[i] = *(const f32x4_t*)&xch[0][ct * 16 + col][grp * 16 + i * 4];
        auto part = [&](int u) __attribute__((always_inline)) {
          f32x4_t x = __builtin_amdgcn_mfma_f32_16x16x4f32(kk[u >> 1][2 * (u & 1)], q[u >> 1][2 * (u & 1)], f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
          return __builtin_amdgcn_mfma_f32_16x16x4f32(kk[u >> 1][2 * (u & 1) + 1], q[u >> 1][2 * (u & 1) + 1], x, 0, 0, 0);
        };
        S[ct] = (part(0) + part(1)) + (part(2) + part(3));
        __builtin_amdgcn_sched_barrier(0);       // (all eight at once would not fit the registers)
        S[ct] = S[ct] + ((part(4) + part(5)) + (part(6) + part(7)));
      } else {
        S[ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    {
      const f32x4_t* kp = at(pid, 0, k_off);
#pragma unroll
      for (int i = 0; i < 4; ++i) kk[i] = kp[i];
    }
    if ((p + 1) * kP > vis0) {                                     // the causal edge of some row, or the end of the file
      const int tok = p * kP + 4 * grp;                            // the lane's first token of the page
#pragma unroll
      for (int ct = 0; ct < 2; ++ct)
#pragma unroll
        for (int v = 0; v < 4; ++v) S[ct][v] = v < vis[ct] - tok ? S[ct][v] : -__builtin_inff();
      // slots past the file's end may hold anything; their weight is 0, but 0 * NaN is NaN.  Likewise elements of the tile's own
      // tokens that are not finite: V is the operand of all rows, and some don't see the token (added at the end to those that do)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (v >= kv_end - tok) vv[v] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (v >= vis0 - tok && !__builtin_isfinite(vv[v][e])) {
            vv[v][e] = 0.f;
            odd = true;
          }
      }
    }
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
      if (ct == 1 && !two) break;
      const float mx = fmaxf(fmaxf(S[ct][0], S[ct][1]), fmaxf(S[ct][2], S[ct][3])) * a.scale_log2e;
      if (__builtin_amdgcn_ballot_w64(mx > m[ct] + kTau) != 0) {   // rare after the first page
        const float mn = pair32_max(pair16_max(fmaxf(m[ct], mx))); // the four lane groups of a row agree
        const float al = __builtin_amdgcn_exp2f(m[ct] - mn);
        l[ct] *= al;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
          for (int v = 0; v < 4; ++v) O[ct][db][v] *= al;
        m[ct] = mn;
      }
      float pw[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        pw[v] = __builtin_amdgcn_exp2f(__builtin_fmaf(S[ct][v], a.scale_log2e, -m[ct]));
        l[ct] += pw[v];
      }
      // likewise: a page's products are added up by themselves, two sums of 8, before they meet the accumulator
#pragma unroll
      for (int db = 0; db < 4; ++db) {
        f32x4_t x = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[0][db], pw[0], f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        f32x4_t y = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[2][db], pw[2], f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        x = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[1][db], pw[1], x, 0, 0, 0);
        y = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[3][db], pw[3], y, 0, 0, 0);
        O[ct][db] = O[ct][db] + (x + y);
      }
    }
  }

  // (the thread's place again, from the register that brings it: nothing but the loop's own values lives through the loop)
  int tid = threadIdx.x;
  asm("" : "+v"(tid));
  const int ecol = tid & 15, egrp = (tid >> 4) & 3;
  // combine the eight wavefronts: common maximum per row, everyone's accumulators rescaled to it, added up in two stages
#pragma unroll
  for (int ct = 0; ct < 2; ++ct) {
    l[ct] = pair32_sum(pair16_sum(l[ct]));
    if (egrp == 0) {
      stat[wv][ct * 16 + ecol][0] = m[ct];
      stat[wv][ct * 16 + ecol][1] = l[ct];
    }
  }
  const bool any_odd = __builtin_amdgcn_ballot_w64(odd) != 0;
  if ((tid & 63) == 0) left_out[wv] = any_odd;
  __syncthreads();
  auto row_max = [&](int row) {
    float M = stat[0][row][0];
#pragma unroll
    for (int w = 1; w < kRowTileWaves; ++w) M = fmaxf(M, stat[w][row][0]);
    return M;
  };
#pragma unroll
  for (int ct = 0; ct < 2; ++ct) {
    const float f = __builtin_amdgcn_exp2f(m[ct] - row_max(ct * 16 + ecol));
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int v = 0; v < 4; ++v) O[ct][db][v] *= f;
  }
  // lane's values of column tile ct, register v: dims 16 egrp + 4 v .. +3 (one per dim block)
  auto cell = [&](int w, int ct, int v) { return (f32x4_t*)&xch[w][ct * 16 + ecol][16 * egrp + 4 * v]; };
  if (wv >= kRowTileWaves / 2) {
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int v = 0; v < 4; ++v) *cell(wv - kRowTileWaves / 2, ct, v) = f32x4_t{O[ct][0][v], O[ct][1][v], O[ct][2][v], O[ct][3][v]};
  }
  __syncthreads();
  if (wv < kRowTileWaves / 2) {
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        f32x4_t* c = cell(wv, ct, v);
        *c = *c + f32x4_t{O[ct][0][v], O[ct][1][v], O[ct][2][v], O[ct][3][v]};
      }
  }
  __syncthreads();
  const int row = tid >> 4, d0 = ecol * 4;   // 32 rows x 64 dims, four dims per thread
  const int tl = row / G, h = row % G;
  if (tl >= count) return;
  f32x4_t o = *(const f32x4_t*)&xch[0][row][d0];
#pragma unroll
  for (int w = 1; w < kRowTileWaves / 2; ++w) o = o + *(const f32x4_t*)&xch[w][row][d0];
  bool add = false;
#pragma unroll
  for (int w = 0; w < kRowTileWaves; ++w) add |= left_out[w] != 0;
  if (add)                                                         // rare: Inf and NaN are what they are at any weight
    for (int t = max(vis0, page0 * kP); t < min(vis0 + tl, page1 * kP); ++t) {
      const f32x4_t x = *(const f32x4_t*)(slab + (int64_t)sload(tbl + t / kP) * a.page_bytes + kBlk + (d0 >> 5) * (kP * kHalfBytes) + (t % kP) * kHalfBytes + (d0 & 31) * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (!__builtin_isfinite(x[e])) o[e] += x[e];
    }
  const float M = row_max(row);
  float L = 0.f;
#pragma unroll
  for (int w = 0; w < kRowTileWaves; ++w) L = __builtin_fmaf(stat[w][row][1], __builtin_amdgcn_exp2f(stat[w][row][0] - M), L);
  if (dest < 0) {
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = o[e] / L;
    *(f32x4_t*)(a.out + ((int64_t)(qrow + tl) * a.Hq + head * G + h) * 64 + d0) = o;
  } else {
    const int64_t slot = (int64_t)(dest + tl) * G + h;
    *(f32x4_t*)(a.part_acc + slot * 64 + d0) = o;
    if (d0 == 0) {
      a.part_ml[slot * 2 + 0] = M;
      a.part_ml[slot * 2 + 1] = L;
    }
  }
}

// Partials of tiles whose keys were cut into chunks, one wavefront per (token, kv head): the chunks of a token lie `count`
// slots apart.  Four chunks' loads are in flight together, as in merge_kernel.
template <int G, int D>
__global__ __launch_bounds__(kWavesPerBlock * 64) void tile_merge_kernel(MergeArgs a) {
  const int lane = threadIdx.x & 63;
  const int32_t* it = a.tile_items + (int64_t)blockIdx.x * 4;
  const int first = sload(it + 0), chunks = sload(it + 1);
  const int count = sload(it + 2), qh = sload(it + 3);
  const int tl = __builtin_amdgcn_readfirstlane((int)(blockIdx.y * kWavesPerBlock + (threadIdx.x >> 6)));
  if (tl >= count) return;
  constexpr int VL = G * D / 64;
  float M[G], ls[G], o[VL];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    M[h] = -__builtin_inff();
    ls[h] = 0.f;
  }
#pragma unroll
  for (int e = 0; e < VL; ++e) o[e] = 0.f;
  for (int c0 = 0; c0 < chunks; c0 += 4) {
    float mv[4][G], lv[4][G], t[4][VL];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t ii = first + (int64_t)min(c0 + u, chunks - 1) * count + tl;
#pragma unroll
      for (int h = 0; h < G; ++h) {
        mv[u][h] = a.part_ml[(ii * G + h) * 2];
        lv[u][h] = a.part_ml[(ii * G + h) * 2 + 1];
      }
#pragma unroll
      for (int e = 0; e < VL; ++e) t[u][e] = a.part_acc[ii * G * D + e * 64 + lane];
    }
    float w[4][G], sc[G];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float mn = fmaxf(fmaxf(fmaxf(mv[0][h], mv[1][h]), fmaxf(mv[2][h], mv[3][h])), M[h]);
      sc[h] = __builtin_amdgcn_exp2f(M[h] - mn);      // 0 for the first group (M = -inf)
      M[h] = mn;
      ls[h] *= sc[h];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        w[u][h] = c0 + u < chunks ? __builtin_amdgcn_exp2f(mv[u][h] - mn) : 0.f;
        ls[h] = __builtin_fmaf(lv[u][h], w[u][h], ls[h]);
      }
    }
    // the group's sum first: one rounding per group, not per chunk, at the size of the whole
    float x[VL];
#pragma unroll
    for (int e = 0; e < VL; ++e) x[e] = t[0][e] * w[0][(e * 64) / D];
#pragma unroll
    for (int u = 1; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < VL; ++e) x[e] = __builtin_fmaf(c0 + u < chunks ? t[u][e] : 0.f, w[u][(e * 64) / D], x[e]);      // (0 * Inf is NaN)
#pragma unroll
    for (int e = 0; e < VL; ++e) o[e] = __builtin_fmaf(o[e], sc[(e * 64) / D], x[e]);
  }
  float* out = a.out + ((int64_t)qh + (int64_t)tl * a.Hq) * D + lane;
#pragma unroll
  for (int e = 0; e < VL; ++e) out[e * 64] = o[e] / ls[(e * 64) / D];
}

// ---------------------------------------------------------------------------------------
// Merge of partial results of a (row, kv head) that was cut:
//   out = sum_i acc_i 2^(m_i - M) / sum_i l_i 2^(m_i - M),  M = max_i m_i.
// The G*D accumulator values of a piece form one flat list; lane owns entries e*64 + lane.  All
// loads of a group of 4 pieces are issued before any is used (indices past the end re-read the
// last piece and drop it: by a select, since under a branch the compiler moves the loads behind it, one round trip each), so the kernel costs one memory round trip per group after the entry.  A row that belongs
// to a shared-prefix group has extra pieces: the partials the tile kernel left for the prefix.
// S = wavefronts per entry.  1: four entries per workgroup.  4: wavefront w takes pieces w, w + 4, ..., so that up to 16 pieces
// are one round trip, and the four are combined through LDS: for entries of many pieces (long files, and few files cut over
// the whole chip): long contexts, 128 entries of 16 or more pieces, 14.9 -> 8.4 us by events, of which 6 are the launch.
// ---------------------------------------------------------------------------------------
template <int G, int D, int S>
__global__ __launch_bounds__(kWavesPerBlock * 64) void merge_kernel(MergeArgs a) {
  constexpr int VL = G * D / 64;
  __shared__ float s_acc[S == 1 ? 1 : S][S == 1 ? 1 : G * D], s_ml[S == 1 ? 1 : S][S == 1 ? 1 : 2 * G];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int item = S == 1 ? (int)blockIdx.x * kWavesPerBlock + wv : (int)blockIdx.x;
  if (item >= a.n_items) return;                                  // S == 4: never, the grid is the list
  const int32_t* it = a.items + item * 8;
  const int first = sload(it);
  const int own = sload(it + 1);
  const int64_t out_row = (int64_t)sload(it + 2) * D;   // (q row * Hq + first head) * D
  // pieces own .. own + xcount - 1 are the partials of the row's shared prefix: xfirst + i * xstride
  const int xfirst = sload(it + 3);
  const int xstride = sload(it + 4);
  const int pieces = own + sload(it + 5);
  const int ostride = sload(it + 6);      // distance between own pieces (tokens in the row)
  auto slot = [&](int i) -> int64_t {
    i = min(i, pieces - 1);
    return i < own ? first + (int64_t)i * ostride : xfirst + (int64_t)(i - own) * xstride;
  };
  const float* ml0 = a.part_ml;
  const float* pa0 = a.part_acc + lane;
  float Mx[G], ls[G], o[VL];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    Mx[h] = -1e30f;                               // (finite: a wavefront without pieces takes part in the combination below)
    ls[h] = 0.f;
  }
#pragma unroll
  for (int e = 0; e < VL; ++e) o[e] = 0.f;
  // groups of 4 pieces: all their loads (max, sum, accumulator) are issued together, one memory round
  // trip per group; the running maximum is carried from group to group (most rows have one group)
  for (int i0 = S == 1 ? 0 : wv; i0 < pieces; i0 += 4 * S) {
    float mv[4][G], lv[4][G], t[4][VL];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t ii = slot(i0 + u * S);
#pragma unroll
      for (int h = 0; h < G; ++h) {
        mv[u][h] = ml0[(ii * G + h) * 2];
        lv[u][h] = ml0[(ii * G + h) * 2 + 1];
      }
#pragma unroll
      for (int e = 0; e < VL; ++e) t[u][e] = pa0[ii * G * D + e * 64];
    }
    float sc[G];                                  // factor that brings what was summed so far to the new maximum
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float mn = Mx[h];
#pragma unroll
      for (int u = 0; u < 4; ++u) mn = fmaxf(mn, mv[u][h]);
      sc[h] = __builtin_amdgcn_exp2f(Mx[h] - mn);     // 0 for the first group
      Mx[h] = mn;
      ls[h] *= sc[h];
    }
#pragma unroll
    for (int e = 0; e < VL; ++e) o[e] *= sc[(e * 64) / D];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float w[G];
#pragma unroll
      for (int h = 0; h < G; ++h) {
        w[h] = (i0 + u * S < pieces) ? __builtin_amdgcn_exp2f(mv[u][h] - Mx[h]) : 0.f;
        ls[h] = __builtin_fmaf(lv[u][h], w[h], ls[h]);
      }
#pragma unroll
      for (int e = 0; e < VL; ++e) o[e] = __builtin_fmaf(i0 + u * S < pieces ? t[u][e] : 0.f, w[(e * 64) / D], o[e]);      // (0 * Inf is NaN)
    }
  }
  if constexpr (S == 1) {
#pragma unroll
    for (int e = 0; e < VL; ++e) a.out[out_row + e * 64 + lane] = o[e] / ls[(e * 64) / D];
  } else {
#pragma unroll
    for (int e = 0; e < VL; ++e) s_acc[wv][e * 64 + lane] = o[e];
    if (lane == 0)
#pragma unroll
      for (int h = 0; h < G; ++h) {
        s_ml[wv][2 * h] = Mx[h];
        s_ml[wv][2 * h + 1] = ls[h];
      }
    __syncthreads();
    for (int x = threadIdx.x; x < G * D; x += kWavesPerBlock * 64) {
      const int h = x / D;
      float M = s_ml[0][2 * h], num = 0.f, den = 0.f;
#pragma unroll
      for (int w = 1; w < S; ++w) M = fmaxf(M, s_ml[w][2 * h]);
#pragma unroll
      for (int w = 0; w < S; ++w) {
        const float f = __builtin_amdgcn_exp2f(s_ml[w][2 * h] - M);
        num = __builtin_fmaf(s_acc[w][x], f, num);
        den = __builtin_fmaf(s_ml[w][2 * h + 1], f, den);
      }
      a.out[out_row + x] = num / den;
    }
  }
}

// ---------------------------------------------------------------------------------------
// Prologue of a batch, one launch: (1) KV append, a workgroup per few tokens; (2) copy-on-write page copies, one block
// per copy: slots [0, r) of every (head, K/V, row half) of page src into page dst; (3) the batch
// descriptor copied from pinned host memory into the device workspace for the attention kernel that
// follows.  The three parts touch disjoint bytes (a copy covers slots below r, appends write slots
// from r on), so they need no ordering among themselves.  Slot map and copy list are read straight
// from the pinned host buffer: an append workgroup reads its tokens' slots once, in one line, and
// shares them through LDS (a request over the host link takes about 4.6 ns of all of them together: one for every workgroup, not for
// every thread).  The rows themselves are requested meanwhile, and the next ones before the barrier of a loop would come round.
// Few runs of consecutive slots (prompts, drafts, chunks of up to about 2000 tokens) come with the kernel's arguments instead: no request over the
// host link stands before the first store (by rocprofv3's trace 900 tokens of three prompts 5.2 -> 4.5 us, 1559 rows of 64 floats 6.4
// -> 5.3; whole calls 61.7 -> 60.0 and 23.2 -> 22.4).
// Bound: HBM, read + write.  By rocprofv3's trace, slots before the first row / now: a document of 7100 tokens 13.2 -> 11.8 us
// (4.9 TB/s read + written), the mixed batch's 16 600 tokens 34.2 -> 26.7; descriptors and few tokens (256 of drafts, 900 of
// prompts) the same.  The append workgroups come first in the grid (last: the mixed batch 31.9 us, a fork's descriptor 7.6 -> 7.5).
// Workgroups of 512 threads for both (the line: launch_prologue): 1024 threads 12.1 and 28.1 us, 256 threads 12.9 and 32.4.
// ---------------------------------------------------------------------------------------
constexpr int kAppendTokens = 16;        // most tokens per append workgroup

// The slot map of a small batch, as part of the kernel's arguments: run r is tokens first[r] .. first[r + 1] - 1 in consecutive slots
// from slot[r] (or appended elsewhere: -1).
struct PrologueRuns {
  int32_t first[kPrologueRuns + 1], slot[kPrologueRuns];
};

template <int NT, bool RUNS>
__device__ __forceinline__ void prologue(const PrologueArgs& a, const __attribute__((address_space(4))) PrologueRuns* runs) {
  __shared__ int32_t s_slot[kAppendTokens];
  int blk = blockIdx.x;
  if (blk < a.append_blocks) {
    const int t0 = blk * a.append_tokens, n = min(a.append_tokens, a.n_tokens - t0);
    const int total = n * a.Hkv * 32;       // 16-byte chunks: token, kv head, K/V, chunk within the row
    const uint8_t* k0 = (const uint8_t*)a.k_new + (int64_t)t0 * a.Hkv * kRowBytes;
    const uint8_t* v0 = (const uint8_t*)a.v_new + (int64_t)t0 * a.Hkv * kRowBytes;
    int my_slot = 0, first = 0, end = 0;    // the slot of token t0 + thread, or the run that the thread writes out
    if constexpr (RUNS) {
      if ((int)threadIdx.x < a.n_runs) {
        first = runs->first[threadIdx.x];
        end = runs->first[threadIdx.x + 1];
        my_slot = runs->slot[threadIdx.x];
      }
    } else {
      my_slot = a.slots[t0 + min((int)threadIdx.x, n - 1)];
    }
    u32x4_t v[4];
    auto request = [&](int x) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {         // past the end the last chunk is read again and not stored
        const int i = min(x + u * NT, total - 1);
        v[u] = *(const u32x4_t*)((((i >> 4) & 1) ? v0 : k0) + (i >> 5) * kRowBytes + (i & 15) * 16);
      }
    };
    request(threadIdx.x);                   // under way while the slots come over the host link
    if constexpr (RUNS) {
      for (int t = max(first, t0); t < min(end, t0 + n); ++t) s_slot[t - t0] = my_slot < 0 ? -1 : my_slot + (t - first);
    } else {
      if ((int)threadIdx.x < n) s_slot[threadIdx.x] = my_slot;
    }
    __syncthreads();
    for (int x = threadIdx.x;;) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = x + u * NT;
        const int th = min(i, total - 1) >> 5, tl = th / a.Hkv, g = th - tl * a.Hkv, slot = s_slot[tl];
        if (i < total && slot >= 0)         // negative: this token is appended by the attention kernel
          *(u32x4_t*)(a.pool + (int64_t)(slot / kP) * a.page_bytes + (int64_t)g * kSlab + ((i >> 4) & 1) * kBlk +
                      ((i & 15) >> 3) * (kP * kHalfBytes) + (slot % kP) * kHalfBytes + (i & 7) * 16) = v[u];
      }
      x += 4 * NT;
      if (x >= total) break;
      request(x);
    }
    return;
  }
  blk -= a.append_blocks;
  if (blk < a.n_cow) {
    const int src = a.cow[blk * 3 + 0], dst = a.cow[blk * 3 + 1], r = a.cow[blk * 3 + 2];
    const uint8_t* s = a.pool + (int64_t)src * a.page_bytes;
    uint8_t* d = a.pool + (int64_t)dst * a.page_bytes;
    const int per_seg = r * (kHalfBytes / 16);           // 16-byte chunks per (head, K/V, half)
    const int n_seg = a.Hkv * 4;
    for (int x = threadIdx.x; x < n_seg * per_seg; x += NT) {
      const int seg = x / per_seg, w = x % per_seg;
      const int64_t off = (int64_t)seg * (kP * kHalfBytes) + w * 16;
      *(uint4*)(d + off) = *(const uint4*)(s + off);
    }
    return;
  }
  blk -= a.n_cow;
  // 16 bytes per thread, enough blocks that the whole descriptor is one round trip to the host
  const uint4* src = (const uint4*)a.host_words;
  uint4* dst = (uint4*)a.dev_words;
  const int64_t n16 = (a.copy_words + 3) / 4;            // the staging buffer is padded to 16 bytes
  for (int64_t i = (int64_t)blk * NT + threadIdx.x; i < n16; i += (int64_t)a.copy_blocks * NT) dst[i] = src[i];
}

template <int NT>
__global__ __launch_bounds__(NT) void prologue_kernel(PrologueArgs a) {
  prologue<NT, false>(a, nullptr);
}
__global__ __launch_bounds__(256) void prologue_runs_kernel(PrologueArgs a, PrologueRuns) {
  // the runs where they lie, behind the arguments proper: named as a parameter and indexed by the thread they would be copied to scratch
  auto args = (const __attribute__((address_space(4))) uint8_t*)__builtin_amdgcn_kernarg_segment_ptr();
  static_assert(sizeof(PrologueArgs) % alignof(PrologueRuns) == 0, "the runs follow the arguments at once");
  prologue<256, true>(a, (const __attribute__((address_space(4))) PrologueRuns*)(args + sizeof(PrologueArgs)));
}

// Inverse of append for a list of token slots: pool -> contiguous [n][Hkv][row].
__global__ void gather_kernel(GatherArgs a, uint8_t* k_out, uint8_t* v_out) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)a.n_tokens * a.Hkv * 32;
  if (tid >= total) return;
  const int c = tid & 15;
  const int kv = (tid >> 4) & 1;
  const int64_t th = tid >> 5;
  const int g = (int)(th % a.Hkv);
  const int64_t t = th / a.Hkv;
  const int slot = a.slots[t];
  const int page = slot / kP, ts = slot % kP;
  const uint8_t* src = a.pool + (int64_t)page * a.page_bytes + (int64_t)g * kSlab + kv * kBlk +
                       (c >> 3) * (kP * kHalfBytes) + ts * kHalfBytes + (c & 7) * 16;
  uint8_t* dst = (kv ? v_out : k_out) + th * kRowBytes + c * 16;
  *(uint4*)dst = *(const uint4*)src;
}

// extract / merge (paper section 4.2): K and V rows of whole tokens copied into fresh pages, bit for bit.  A workgroup works on one
// page of one layer.  A thread owns one token and one of the eight 16-byte chunks of a 128-byte piece, and takes pieces (kv
// head, K/V, row half), two to a pass of the workgroup: stores are a page from end to end, loads whole 128-byte lines.  Sources are
// pages of existing files, destinations fresh pages: disjoint.  Bound: HBM, read + write.
// A list in pinned host memory: one workgroup per page and layer, since each sends requests over the host link (a wavefront's source
// slots are one line), and all its loads in flight.  About half of the tokens of 64 files of 512..4096, one layer of 8 heads: 108 us
// by rocprofv3's trace (5.6 TB/s read + written), and no launch for the list before it (as pairs of slots 16 us + 104; eight loads in
// flight 115, four 117, nontemporal stores 121; the list through LDS 110; several workgroups to a page 114 with two or four, 142 with eight).
// Slots and destination are one round trip (TOGETHER) where all workgroups start at once (the line: launch_move); behind other workgroups' copies
// the second round trip costs nothing.
// A list in device memory (brought there for what is large: many layers above all): a workgroup per pass, so that the loads
// and stores under way at one time lie close together.  The same files, 8 heads x 32 layers, 2.68 ms of kernel (6.2 TB/s) against 3.05
// ms with the pinned list and 3.1 ms with one workgroup per page and the list in device memory; one head x 32 layers 350 us against 402.
template <int U, bool TOGETHER>
__global__ __launch_bounds__(256) void move_kernel(MoveArgs a) {
  constexpr int kPiece = kP * kHalfBytes;
  const int tid = threadIdx.x, t = (tid >> 3) & (kP - 1), first = tid >> 7, chunk = (tid & 7) * 16;
  const int slot = a.src[(int64_t)blockIdx.y * kP + t], dst = a.dst[blockIdx.y];
  if constexpr (TOGETHER) asm volatile("" ::"v"(slot));             // both requests under way before the branch waits for one
  if (t > dst % kP) return;                                         // the page's last tokens do not exist
  uint8_t* pool = a.pool + (int64_t)blockIdx.z * a.layer_bytes;
  const uint8_t* s = pool + (int64_t)(slot / kP) * a.page_bytes + first * kPiece + (slot % kP) * kHalfBytes + chunk;
  uint8_t* d = pool + (int64_t)(dst / kP) * a.page_bytes + first * kPiece + t * kHalfBytes + chunk;
  for (int p = blockIdx.x * U; p < a.Hkv * 2; p += gridDim.x * U) { // two pieces per pass of the workgroup, U passes at a time
    u32x4_t v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load((const u32x4_t*)(s + (int64_t)(p + u) * (2 * kPiece)));
#pragma unroll
    for (int u = 0; u < U; ++u) *(u32x4_t*)(d + (int64_t)(p + u) * (2 * kPiece)) = v[u];
  }
}

// offload / restore (paper section 4.3): whole pages between the pool and pinned host memory, over
// the host link.  Four workgroups per page, 16 bytes per thread and pass; the list (page id, host
// address) is read from pinned memory by every workgroup for itself.
constexpr int kSwapSplit = 4;
__global__ __launch_bounds__(256) void swap_kernel(SwapArgs a) {
  const int e = blockIdx.x / kSwapSplit, part = blockIdx.x % kSwapSplit;
  const int64_t page = (int64_t)a.list[2 * e];
  uint8_t* host = (uint8_t*)a.list[2 * e + 1] + a.host_offset;
  uint8_t* dev = a.pool + page * a.page_bytes;
  const int64_t n16 = a.page_bytes / 16, per = (n16 + kSwapSplit - 1) / kSwapSplit;
  const int64_t lo = part * per, hi = min(n16, lo + per);
  const u32x4_t* src = (const u32x4_t*)(a.to_host ? dev : host);
  u32x4_t* dst = (u32x4_t*)(a.to_host ? host : dev);
  for (int64_t i = lo + threadIdx.x; i < hi; i += 4 * 256) {      // four loads in flight per thread
    u32x4_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + u * 256 < hi) v[u] = __builtin_nontemporal_load(src + i + u * 256);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + u * 256 < hi) dst[i + u * 256] = v[u];
  }
}

// ---------------------------------------------------------------------------------------
// Calibration: streaming read (reduced so that the loads are live) and plain copy.
// ---------------------------------------------------------------------------------------
// Read: every wave streams its own contiguous span with nontemporal 16-byte loads, 16 KiB in
// flight per wave (the access pattern that reads fastest on this part).
__global__ __launch_bounds__(256) void calib_read_kernel(const u32x4_t* __restrict__ src, int64_t n16, unsigned long long* out) {
  constexpr int U = 16;
  uint32_t acc = 0;
  const int lane = threadIdx.x & 63;
  const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * 4;
  const int64_t per = n16 / nwaves / (64 * U) * (64 * U);
  const u32x4_t* p = src + wave * per + lane;
  for (int64_t k = 0; k < per; k += 64 * U) {
    u32x4_t a[U];
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = __builtin_nontemporal_load(p + k + u * 64);
#pragma unroll
    for (int u = 0; u < U; ++u) acc += a[u].x ^ a[u].y ^ a[u].z ^ a[u].w;
  }
  // the tail that does not divide evenly (none when bytes is a multiple of grid * 64 KiB)
  for (int64_t i = nwaves * per + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (int64_t)gridDim.x * blockDim.x) {
    u32x4_t a0 = src[i];
    acc += a0.x ^ a0.y ^ a0.z ^ a0.w;
  }
  if (acc == 0x9e3779b9u) atomicAdd(out, 1ull);      // practically never: keeps the loads alive
}
__global__ __launch_bounds__(256) void calib_copy_kernel(uint4* dst, const uint4* src, int64_t n16) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
}

// Matrix-core rate that this part sustains: every wavefront (8 per workgroup, two per SIMD, as in the
// tile kernel) issues 16 independent-enough 32x32x16 bf16 MFMAs per iteration on four accumulators,
// operands in registers, nothing else in the loop.  flops = blocks * 8 * iters * 16 * 32768.
__global__ __launch_bounds__(512, 1) void calib_mfma_kernel(float* out, int iters) {
  const int lane = threadIdx.x & 63;
  bf16x8_t x[4], y[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      // values of mixed sign and exponent, different in every lane and register
      const uint32_t hsh = (uint32_t)(threadIdx.x * 8 + e + 131 * i + 977 * blockIdx.x) * 2654435761u;
      x[i][e] = (__bf16)(((int)(hsh >> 20) - 2048) * (1.0f / 2048.0f));
      y[i][e] = (__bf16)(((int)((hsh >> 8) & 4095) - 2048) * (1.0f / 2048.0f));
    }
  f32x16_t acc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[(i + r) & 3], y[i], acc[i], 0, 0, 0);
  }
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) sum += acc[i][v];
  out[(int64_t)blockIdx.x * 512 + threadIdx.x] = sum + (float)lane;
}

template <typename E>
hipError_t launch_attn_g(const DecodeArgs& da, const PrefillArgs& pa, int decode_mode, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  const int G = da.Hq / da.Hkv;
  // With events: they are attached to the dispatches themselves (start of the first kernel of the
  // attention launch, end of the last), so the interval holds kernel time and nothing else.
  auto launch = [&](auto kernel, dim3 g, dim3 b, hipEvent_t s, hipEvent_t e, auto... args) {
    if (s || e) hipExtLaunchKernelGGL(kernel, g, b, 0, st, s, e, 0, args...);
    else hipLaunchKernelGGL(kernel, g, b, 0, st, args...);
  };
  // decode ranges: matrix cores (mode 1), the two-wavefront VALU kernel for 8 heads (mode 2), or the
  // VALU kernel fused into the tile launch (mode 0)
  const int mode = (E::kDimsPerChunk == 8 && decode_mode == 1) ? 1 : (G == 8 ? 2 : 0);
  PrefillArgs ps = pa;
  const int tile_blocks = ps.n_tiles > 0 ? ps.tile_blocks : 0;
  // eight-wavefront workgroups when the tiles have 256 query rows (and no tile is there: four)
  const int tw = (ps.n_tiles > 0 && ps.tile_rows == 256) ? 8 : 4;
  // every tile a shared-prefix tile with at most 64 live rows: the kernel that splits them by key block
  const bool split_tiles = E::kDimsPerChunk == 8 && tw == 4 && ps.n_tiles > 0 && ps.small_shared_only != 0;
  // mode 0: one workgroup per bin; the host made the bins for workgroups of this size
  if (mode == 0 && da.n_bins > 0 && (tile_blocks > 0 ? da.bin_waves != tw : (da.bin_waves != 4 && da.bin_waves != 8))) return hipErrorInvalidValue;
  const int decode_blocks = mode == 0 ? da.n_bins : 0;
  const int tile_groups = (tile_blocks + 7) / 8, decode_groups = (decode_blocks + 7) / 8;
  const dim3 grid((tile_groups + decode_groups) * 8), block(256), block8(512);
  // tiles and bins in one grid: the host's order table must cover it; tiles alone run in list order
  if (tile_groups > 0 && decode_groups > 0 && (!ps.group_map || ps.n_groups != tile_groups + decode_groups)) return hipErrorInvalidValue;
  if (decode_groups == 0) ps.group_map = nullptr;
  if (ps.n_tiles > 0 && ps.tile_rows != 128 && ps.tile_rows != 256) return hipErrorInvalidValue;
  if (mode == 2 && da.n_bins > 0) return hipErrorInvalidValue;      // no kernel
  const bool second = da.n_waves > 0 && mode != 0;          // decode ranges in a launch of their own
  const hipEvent_t e_first = second ? nullptr : ev1;
  const hipEvent_t s_second = grid.x > 0 ? nullptr : ev0;
#define SYM_ATTN_CASE(GG) \
  case GG: \
    if (tw == 8) launch(attn_kernel<E, GG, 8>, grid, block8, ev0, e_first, da, ps); \
    else if (split_tiles) launch(attn_kernel<E, GG, 4, true>, grid, block, ev0, e_first, da, ps); \
    else launch(attn_kernel<E, GG, 4>, grid, block, ev0, e_first, da, ps); \
    break;
  if (tile_blocks == 0 && mode == 0 && da.n_bins > 0) {      // plain decode: the lean kernel
    const dim3 dgrid(da.n_bins), dblock(64 * da.bin_waves);
#define SYM_DECODE_CASE(GG) \
  case GG: \
    if (da.bin_waves == 8) launch(decode_only_kernel<E, GG, 8, true>, dgrid, dblock, ev0, ev1, da); \
    else if (da.cached) launch(decode_only_kernel<E, GG, 4, false>, dgrid, dblock, ev0, ev1, da); \
    else launch(decode_only_kernel<E, GG, 4, true>, dgrid, dblock, ev0, ev1, da); \
    break;
    switch (G) {
      SYM_DECODE_CASE(1) SYM_DECODE_CASE(2) SYM_DECODE_CASE(4)
      default: return hipErrorInvalidValue;
    }
#undef SYM_DECODE_CASE
    return hipGetLastError();
  }
  if (grid.x > 0) switch (G) {
    SYM_ATTN_CASE(1) SYM_ATTN_CASE(2) SYM_ATTN_CASE(4) SYM_ATTN_CASE(8)
    default: return hipErrorInvalidValue;
  }
#undef SYM_ATTN_CASE
  if (da.n_waves > 0 && mode == 2) launch(decode_pair_kernel<E>, dim3(da.n_waves), dim3(128), s_second, ev1, da);
  if (da.n_bins > 0 && mode == 1) {
    if (da.bin_waves != 4 && da.bin_waves != 8) return hipErrorInvalidValue;
    const dim3 dgrid(da.n_bins), dblock(64 * da.bin_waves);
#define SYM_DECODE_CASE(GG) \
  case GG: \
    if (da.bin_waves == 8) launch(decode_mfma_bins_kernel<GG, 8, true>, dgrid, dblock, s_second, ev1, da); \
    else if (da.cached) launch(decode_mfma_bins_kernel<GG, 4, false>, dgrid, dblock, s_second, ev1, da); \
    else launch(decode_mfma_bins_kernel<GG, 4, true>, dgrid, dblock, s_second, ev1, da); \
    break;
    switch (G) {
      SYM_DECODE_CASE(1) SYM_DECODE_CASE(2) SYM_DECODE_CASE(4) SYM_DECODE_CASE(8)
      default: return hipErrorInvalidValue;
    }
#undef SYM_DECODE_CASE
  } else if (da.n_waves > 0 && mode == 1) {
    const dim3 dgrid((da.n_waves + kWavesPerBlock - 1) / kWavesPerBlock);
    switch (G) {
      case 1: launch(decode_mfma_kernel<1>, dgrid, block, s_second, ev1, da); break;
      case 2: launch(decode_mfma_kernel<2>, dgrid, block, s_second, ev1, da); break;
      case 4: launch(decode_mfma_kernel<4>, dgrid, block, s_second, ev1, da); break;
      case 8: launch(decode_mfma_kernel<8>, dgrid, block, s_second, ev1, da); break;
      default: return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Scratch memory of the entry point that allocates nothing (sym_pred_batch_static): descriptor
// words + partial results live in this file-scope array instead of the caller's workspace.
// Every GPU the library runs on holds its own copy at its own address, until the process ends;
// host code never uses the array's name as an address: it asks the runtime once per device for
// the address and passes that to the kernels like any other workspace.
// ---------------------------------------------------------------------------------------
static __device__ __align__(256) uint8_t scratch[kStaticScratchBytes];

}  // namespace

hipError_t static_scratch_address(int device, uint8_t** ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static uint8_t* addr[kMaxDevices] = {};
  if (device < 0 || device >= kMaxDevices || !ptr) return hipErrorInvalidValue;
  std::lock_guard<std::mutex> lk(mu);
  if (!addr[device]) {
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != device && (e = hipSetDevice(device)) != hipSuccess) return e;
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != device) (void)hipSetDevice(cur);
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    addr[device] = (uint8_t*)p;
  }
  *ptr = addr[device];
  return hipSuccess;
}

hipError_t launch_attn(const DecodeArgs& da, const PrefillArgs& pa, int dtype, int decode_mode, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  if (pa.n_rtiles > 0) {
    if (dtype != 0) return hipErrorInvalidValue;
    const bool last = da.n_waves <= 0;
    const dim3 grid((unsigned)pa.n_rtiles), block(64 * kRowTileWaves);
    const hipEvent_t e1 = last ? ev1 : nullptr;
#define SYM_ROW_TILE_CASE(GG) \
  case GG: \
    if (ev0 || e1) hipExtLaunchKernelGGL(row_tile_kernel<GG>, grid, block, 0, st, ev0, e1, 0, pa); \
    else hipLaunchKernelGGL(row_tile_kernel<GG>, grid, block, 0, st, pa); \
    break;
    switch (da.Hq / da.Hkv) {
      SYM_ROW_TILE_CASE(1) SYM_ROW_TILE_CASE(2) SYM_ROW_TILE_CASE(4) SYM_ROW_TILE_CASE(8)
      default: return hipErrorInvalidValue;
    }
#undef SYM_ROW_TILE_CASE
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || last) return e;
    ev0 = nullptr;
  }
  if (da.n_waves <= 0 && pa.n_tiles <= 0) return hipSuccess;
  if (dtype == 0) return pa.n_tiles > 0 ? hipErrorInvalidValue : launch_attn_g<ElemF32>(da, pa, 0, st, ev0, ev1);
  return launch_attn_g<ElemBF16>(da, pa, decode_mode, st, ev0, ev1);
}

hipError_t launch_merge(const MergeArgs& a, int G, int D, hipStream_t st) {
  if (a.n_tile_items > 0) {
    const dim3 tgrid((unsigned)a.n_tile_items, (unsigned)((a.tile_tokens + kWavesPerBlock - 1) / kWavesPerBlock));
#define SYM_TILE_MERGE_CASE(GG, DD) \
  if (G == GG && D == DD) hipLaunchKernelGGL((tile_merge_kernel<GG, DD>), tgrid, dim3(kWavesPerBlock * 64), 0, st, a);
    SYM_TILE_MERGE_CASE(1, 64) SYM_TILE_MERGE_CASE(2, 64) SYM_TILE_MERGE_CASE(4, 64) SYM_TILE_MERGE_CASE(8, 64)
    SYM_TILE_MERGE_CASE(1, 128) SYM_TILE_MERGE_CASE(2, 128) SYM_TILE_MERGE_CASE(4, 128) SYM_TILE_MERGE_CASE(8, 128)
#undef SYM_TILE_MERGE_CASE
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (a.n_items <= 0) return hipSuccess;
  // four wavefronts per entry when some entry has more pieces than one group, and there are few entries
  const bool wide = a.max_pieces > 4 && a.n_items <= kWideMergeItems;
  const dim3 grid(wide ? a.n_items : (a.n_items + kWavesPerBlock - 1) / kWavesPerBlock), block(kWavesPerBlock * 64);
#define SYM_MERGE_CASE(GG, DD) \
  if (G == GG && D == DD) { \
    if (wide) hipLaunchKernelGGL((merge_kernel<GG, DD, 4>), grid, block, 0, st, a); \
    else hipLaunchKernelGGL((merge_kernel<GG, DD, 1>), grid, block, 0, st, a); \
    return hipGetLastError(); \
  }
  SYM_MERGE_CASE(1, 64) SYM_MERGE_CASE(2, 64) SYM_MERGE_CASE(4, 64) SYM_MERGE_CASE(8, 64)
  SYM_MERGE_CASE(1, 128) SYM_MERGE_CASE(2, 128) SYM_MERGE_CASE(4, 128) SYM_MERGE_CASE(8, 128)
#undef SYM_MERGE_CASE
  return hipErrorInvalidValue;
}

// A launch that completes the event `done` (or none).  The event hangs on the dispatch itself: recorded behind the launch it is a
// packet of its own, which the next kernel waits for, 3.0 us in every call whatever its size (two kernels of 10 us with an event
// recorded between them 25.4 us, with it attached and without a system fence 22.4, with no event at all 22.4; as a record without a
// system fence 23.6).  A stream that is being captured takes it as a record: a graph's kernel nodes carry no events.
template <typename K, typename... A>
hipError_t launch_done(K kernel, dim3 grid, dim3 block, hipStream_t st, hipEvent_t done, const A&... a) {
  if (done) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess) {
      (void)hipGetLastError();
      cs = hipStreamCaptureStatusActive;
    }
    if (cs == hipStreamCaptureStatusNone) {
      hipExtLaunchKernelGGL(kernel, grid, block, 0, st, nullptr, done, 0, a...);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL(kernel, grid, block, 0, st, a...);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess && done ? hipEventRecord(done, st) : e;
}

hipError_t launch_prologue(PrologueArgs a, hipStream_t st) {
  // few tokens: one per workgroup (latency); many: up to 16, while there are 512 workgroups, two per compute unit
  a.append_tokens = std::min(std::max(a.n_tokens / 512, 1), kAppendTokens);
  a.append_blocks = (a.n_tokens + a.append_tokens - 1) / a.append_tokens;
  // 512 threads where each has more than two 16-byte chunks; below, most of the four it requests at a time would be none (by events
  // around the launch, 512 / 256 threads: 8 kv heads 2500 tokens 10.6 / 10.0 us, 3000 10.8 / 11.3, 7100 13.6 / 14.3; 4 heads 2600 tokens
  // 9.8 / 9.3, 6000 10.9 / 11.5; one head 2600 tokens 9.2 / 8.8; 16 heads 2600 tokens 13.2 / 12.6, 8190 20.6 / 20.9)
  const int nt = a.append_tokens > 4 && a.append_tokens * a.Hkv > 32 ? 512 : 256;
  a.copy_blocks = a.copy_words > 0 ? (int32_t)std::min<int64_t>(((a.copy_words + 3) / 4 + nt - 1) / nt, 256) : 0;   // >= 1: also for one, two or three words
  const int64_t blocks = (int64_t)a.append_blocks + a.n_cow + a.copy_blocks;
  if (blocks <= 0) return a.done ? hipEventRecord(a.done, st) : hipSuccess;
  if (a.append_blocks > 0 && a.n_runs > 0 && a.n_runs <= kPrologueRuns) {
    static_assert(kPrologueRuns * kP / 512 <= 4 && kPrologueRuns <= 256, "workgroups of 256 threads, a run for each thread at most");
    PrologueRuns r;
    for (int i = 0; i < a.n_runs; ++i) {
      r.first[i] = a.runs[2 * i];
      r.slot[i] = a.runs[2 * i + 1];
    }
    r.first[a.n_runs] = a.n_tokens;
    return launch_done(prologue_runs_kernel, dim3((unsigned)blocks), dim3(256), st, a.done, a, r);
  }
  if (nt == 512) return launch_done(prologue_kernel<512>, dim3((unsigned)blocks), dim3(512), st, a.done, a);
  return launch_done(prologue_kernel<256>, dim3((unsigned)blocks), dim3(256), st, a.done, a);
}

hipError_t launch_gather(const GatherArgs& a, void* k_out, void* v_out, hipStream_t st) {
  if (a.n_tokens <= 0) return hipSuccess;
  const int64_t total = (int64_t)a.n_tokens * a.Hkv * 32;
  hipLaunchKernelGGL(gather_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, a, (uint8_t*)k_out, (uint8_t*)v_out);
  return hipGetLastError();
}

// One workgroup per page and layer.
template <bool TOGETHER>
hipError_t launch_move_pages(const MoveArgs& a, hipStream_t st) {
  const dim3 grid(1, (unsigned)a.n_pages, (unsigned)a.n_layers), block(256);
  if (a.Hkv % 8 == 0) return launch_done(move_kernel<16, TOGETHER>, grid, block, st, a.done, a);      // all of a page of 8 kv heads at once
  if (a.Hkv % 4 == 0) return launch_done(move_kernel<8, TOGETHER>, grid, block, st, a.done, a);
  // (two instead of four for 6 heads: 8 files of 512..4096 x 2 layers 27.0 instead of 26.2 us, 64 files x 1 layer 65.8 instead of 64.3)
  if (a.Hkv % 2 == 0) return launch_done(move_kernel<4, TOGETHER>, grid, block, st, a.done, a);
  return launch_done(move_kernel<2, TOGETHER>, grid, block, st, a.done, a);
}

hipError_t launch_move(const MoveArgs& a, hipStream_t st) {
  if (a.n_pages <= 0) return hipSuccess;
  if (a.n_pages > 65535 || a.n_layers < 1 || a.n_layers > 65535) return hipErrorInvalidValue;
  const dim3 block(256);
  if (a.near) return launch_done(move_kernel<1, false>, dim3((unsigned)a.Hkv * 2, (unsigned)a.n_pages, (unsigned)a.n_layers), block, st, a.done, a);
  // 2048 workgroups of 256 threads are all that 256 compute units hold.  By events around the launch, slots and destination in one round trip /
  // one after the other: 8 kv heads 16 pages 9.3 / 10.5 us, 128 10.3 / 11.5, 512 21.0 / 22.0, 2048 60.7 / 61.1, 512 x 4 layers 57.2 / 58.1; one head
  // 512 pages 10.3 / 10.9; but 4096 pages of 8 heads 81.9 / 81.1, of 2 heads 33.4 / 32.2, 8192 of 4 heads 82.6 / 81.4; 1024 x 4 layers 83.7 / 83.4
  if ((int64_t)a.n_pages * a.n_layers <= 2048) return launch_move_pages<true>(a, st);
  return launch_move_pages<false>(a, st);
}

hipError_t launch_swap(const SwapArgs& a, hipStream_t st) {
  if (a.n_pages <= 0) return hipSuccess;
  hipLaunchKernelGGL(swap_kernel, dim3((unsigned)a.n_pages * kSwapSplit), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_calib_read(const void* src, int64_t bytes, void* out8, hipStream_t st) {
  hipLaunchKernelGGL(calib_read_kernel, dim3(256 * 4), dim3(256), 0, st, (const u32x4_t*)src, bytes / 16, (unsigned long long*)out8);
  return hipGetLastError();
}
hipError_t launch_calib_mfma(float* out, int blocks, int iters, hipStream_t st) {
  hipLaunchKernelGGL(calib_mfma_kernel, dim3(blocks), dim3(512), 0, st, out, iters);
  return hipGetLastError();
}
hipError_t launch_calib_copy(void* dst, const void* src, int64_t bytes, hipStream_t st) {
  hipLaunchKernelGGL(calib_copy_kernel, dim3(256 * 8), dim3(256), 0, st, (uint4*)dst, (const uint4*)src, bytes / 16);
  return hipGetLastError();
}

}  // namespace symkv

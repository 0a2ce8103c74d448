// Argument blocks and launch functions of the HIP kernels (see kernels.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace symkv {

struct DecodeArgs {
  const uint8_t* pool;
  int64_t page_bytes;
  const void* q;            // [rows][Hq][D] storage dtype
  float* out;               // [rows][Hq][D]
  float* part_acc;          // [n_partials][G][D]
  float* part_ml;           // [n_partials][G][2] (max in log2 units, sum)
  const int32_t* rows;      // [n_rows][4]: page-table offset, visible tokens, q/out row, lip
  const int32_t* waves;     // [n_waves][8]: row, kv head, page, units, first partial, ids of the first
                            //   range's first three pages
  const int32_t* pt;        // flattened page tables
  int32_t n_waves, Hq, Hkv;
  float scale_log2e;        // softmax scale * log2(e)
  // bins: `waves` then holds bin_waves records per bin: first segment, first page, units, 0, ids of the first three pages, kv head | (tokens
  // in the row - 1) << 28
  const int32_t* segs;      // [n_segs + 2][8]: page-table offset, kv head | (tokens in the row - 1) << 28, first page, end page, visible
                            //   tokens, q/out row * Hq + first query head, destination (-1 output, else partial slot), slot of the appended token or -1
  const int32_t* lmerge;    // [n_bins][32]: count, then (segment, LDS slot of its first piece, that piece's wavefront,
                            //   pieces) per segment the bin's cut divided, from word 4 on
  int32_t n_bins, bin_waves;
  int32_t cached;           // bins of four wavefronts without tiles: plain loads of K/V (a small batch), not nontemporal ones
  const void* k_new;        // [rows][Hkv][D]: rows of the new tokens, for segments that append (else unused)
  const void* v_new;
};

struct PrefillArgs {
  const uint8_t* pool;
  int64_t page_bytes;
  const void* q;            // [tokens][Hq][128] bf16
  float* out;               // [tokens][Hq][128]
  const int32_t* tiles;     // [n_tiles][12]: page-table offset, length before, first q/out row (or offset
                            //   into members), tokens (or members) in the tile, kv head, token offset in the
                            //   chunk (or first partial slot), kind (0 prefill, 1 shared prefix, 2 prefill
                            //   over part of its keys), first page, end page, first partial slot of kind 2, ids
                            //   of the first two pages it walks
  const int32_t* pt;        // flattened page tables
  const int32_t* members;   // q rows of the members of shared-prefix tiles
  float* part_acc;          // partial results (shared-prefix tiles)
  float* part_ml;
  int32_t xcd_off[9];       // workgroup b runs tile xcd_off[b % 8] + b / 8 if that is below xcd_off[b % 8 + 1]
  int32_t tile_blocks;      // workgroups of the tile part of the launch (multiple of 8)
  int32_t n_tiles;
  int32_t tile_rows;             // query rows per tile: 128 (four wavefronts per workgroup) or 256 (eight)
  int32_t Hq, Hkv;
  float scale_log2e;
  int32_t small_shared_only;     // every tile is a shared-prefix tile of at most 64 query rows (members x heads per kv head)
  const int32_t* group_map;      // a launch with tiles and decode bins: per group of 8 workgroups, tile group g or ~(decode group)
  int32_t n_groups;
  // row tiles (fp32 storage, a launch of their own): a few consecutive new tokens of a LIP x one kv head
  const int32_t* rtiles;         // [n_rtiles][8]: page-table offset, tokens the first row sees, its q/out row, tokens, kv head,
                                 //   first page, end page, first partial slot (-1: the final output rows)
  int32_t n_rtiles;
};

struct MergeArgs {
  const float* part_acc;
  const float* part_ml;
  const int32_t* items;     // [n_items][8]: first partial, pieces, q row * Hq + first head, then the extra
                            //   pieces of a shared prefix: first, stride, count; 0, 0
  float* out;
  int32_t n_items, max_pieces;   // entries; the most pieces of one
  // tiles whose keys were cut into chunks (a launch of their own)
  const int32_t* tile_items;   // [n_tile_items][4]: first partial (chunk c, token t: first + c * tokens + t), chunks, tokens,
                               //   q row * Hq + first head of its first token
  int32_t n_tile_items, tile_tokens, Hq;   // ... and the most tokens one of them holds
};

struct PrologueArgs {
  uint8_t* pool;
  int64_t page_bytes;
  const void* k_new;            // device [n_tokens][Hkv][row]
  const void* v_new;
  const int32_t* slots;         // pinned host [n_tokens]: page * P + slot
  const int32_t* cow;           // pinned host [n_cow][3]: src, dst, slots
  const int32_t* host_words;    // pinned host: descriptor words to copy
  int32_t* dev_words;           // device workspace
  int64_t copy_words;
  int32_t n_tokens, Hkv, n_cow;
  int32_t append_blocks, append_tokens, copy_blocks;   // filled by launch_prologue
  hipEvent_t done;              // completed by the launch, or null
  const int32_t* runs;          // host: the slot map as (first token, slot or -1) pairs of consecutive slots, ...
  int32_t n_runs;               // ... handed to the kernel with its arguments where they are at most kPrologueRuns; 0: none given
};
// Each run saves the launch a part of a round trip over the host link and costs the call host time, used or not.  Calls with room for 64 / 128 /
// 255 runs, one after the other: 200 tokens of 8 kv heads 9.0 / 9.7 / 9.8 us, 2033 tokens 9.3 / 10.1 / 10.2; a call alone: 2033 tokens 20.4 / 18.9 /
// 19.0 us, 3000 tokens 21.5 / 21.5 / 21.1, 4064 22.1 / 22.2 / 21.8.
constexpr int kPrologueRuns = 128;

struct GatherArgs {
  const uint8_t* pool;
  int64_t page_bytes;
  const int32_t* slots;         // pinned host or device [n_tokens]
  int32_t n_tokens, Hkv;
};

struct MoveArgs {
  uint8_t* pool;
  int64_t page_bytes;
  int64_t layer_bytes;
  const int32_t* src;           // [n_pages][P]: source slots (page * P + slot) of the tokens of a destination page
  const int32_t* dst;           // [n_pages]: destination page * P + tokens - 1
  bool near;                    // src and dst are in device memory (otherwise pinned host memory)
  int32_t n_pages, n_layers, Hkv;
  hipEvent_t done;              // completed by the launch, or null
};

struct SwapArgs {
  uint8_t* pool;
  int64_t page_bytes;
  const uint64_t* list;         // pinned host [n_pages][2]: page id, address of the page's host slot
  int32_t n_pages;
  int32_t to_host;              // 1 = pool -> host slots, 0 = host slots -> pool
  int64_t host_offset;          // byte offset inside every host slot (a slot holds the page's bytes of every layer)
};

// Size of the file-scope device array that stands in for the workspace in sym_pred_batch_static, and
// its address on `device` (looked up once per device, with that device current during the lookup).
constexpr int64_t kStaticScratchBytes = 64ll << 20;
hipError_t static_scratch_address(int device, uint8_t** ptr);

// decode_mode: 0 = VALU decode kernel, 1 = decode ranges on the matrix cores (bf16 storage only)
// ev0 / ev1 (both or neither): events attached to the first / last dispatch of the launch (kernel start, kernel end)
hipError_t launch_attn(const DecodeArgs& da, const PrefillArgs& pa, int dtype, int decode_mode, hipStream_t st,
                       hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
hipError_t launch_merge(const MergeArgs& a, int G, int D, hipStream_t st);
hipError_t launch_prologue(PrologueArgs a, hipStream_t st);
hipError_t launch_gather(const GatherArgs& a, void* k_out, void* v_out, hipStream_t st);
hipError_t launch_move(const MoveArgs& a, hipStream_t st);
hipError_t launch_swap(const SwapArgs& a, hipStream_t st);
hipError_t launch_calib_read(const void* src, int64_t bytes, void* out8, hipStream_t st);
hipError_t launch_calib_copy(void* dst, const void* src, int64_t bytes, hipStream_t st);
hipError_t launch_calib_mfma(float* out, int blocks, int iters, hipStream_t st);

}  // namespace symkv

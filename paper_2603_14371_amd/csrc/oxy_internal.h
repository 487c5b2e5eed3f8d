// Internal interface between the host pool (oxy_pool.cpp) and the HIP kernels
// (oxy_kernels.hip).  Not part of the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace oxy {

constexpr int kHeads = 8;        // query heads sharing the one KV head
constexpr int kDim = 256;        // head_dim
constexpr int kPage = 16;        // tokens per page
constexpr int kPageBytes = kPage * kDim * 2;      // one K page or one V page (bf16)
constexpr int kBlockBytes = 2 * kPageBytes;       // K page + V page of one layer
constexpr int kNoCausal = 0x3fffffff;
constexpr int kWorkWords = 32;             // one 128-byte line per work record
constexpr int kWorkInlineToks = 8;         // words 8..15: query token ids of the tile
constexpr int kWorkInlinePages = 16;       // words 16..31: block ids of the first 16 pages
constexpr int kMaxInlineBlocks = 512;             // block ids passed by value to an append

// work record fields (words 0..7)
enum { W_TOK_OFF = 0, W_N_TOK, W_TBL_OFF, W_KV_BEGIN, W_KV_END, W_CAUSAL_Q0, W_PART_IDX, W_PATH };
// paths
enum { PATH_STREAM = 0,  // <=2 query tokens (16 rows)
       PATH_TILE = 1,    // up to 8 query tokens (64 rows)
       PATH_NOOP = 2 };  // padding that keeps the index -> XCD pattern of the work list intact
// The path sits in the low four bits of word W_PATH.  kPathFresh marks an own-phase tile of an
// item whose own history was empty before this step: all of its keys are rows of this step's
// k_new / v_new, row = (word >> kPathRowShift) + own position.
// kPathAppends marks a streaming work item on an item's own pages: its query tokens are the new
// rows that a folded append has to write (a streaming item on prefix pages appends nothing).
// kPathOnce (with kPathAppends) asks for non-temporal page loads.
constexpr int kPathMask = 15, kPathFresh = 16, kPathAppends = 32, kPathOnce = 64, kPathRowShift = 8;

struct InlineIds {
  int32_t v[kMaxInlineBlocks];
};

// Copies a batch descriptor from pinned host memory (16-byte aligned, as the device address is) on
// stream s; `done` is complete when the staging buffer has been read.
hipError_t launch_upload(const int32_t* pinned, int32_t* device, int32_t n_words, hipStream_t s,
                         hipEvent_t done);
// Scatter n_tokens rows of K and V (natural [token][256] bf16) into the slots of one layer.
hipError_t launch_append(const void* k_new, const void* v_new, const int32_t* d_slots,
                         int32_t n_tokens, void* layer_base, hipStream_t s);
// Same, slots = blocks.v[(pos0+t)/16]*16 + (pos0+t)%16 with the block ids passed by value.
// n_layers consecutive layers in one launch: layer i reads k_new/v_new + i*src_layer_stride and
// writes layer_base + i*pool_layer_stride (bytes).
hipError_t launch_append_inline(const void* k_new, const void* v_new, const InlineIds& blocks,
                                int32_t pos0, int32_t n_tokens, void* layer_base, int32_t n_layers,
                                size_t src_layer_stride, size_t pool_layer_stride, hipStream_t s);
// Gather rows back to natural order, at most kMaxRuns runs and kMaxGatherRows rows a launch.  Run i is
// 1..16 consecutive slots of one block: slot[i] = its first slot, where[i] = (row of k_out / v_out
// << 4) | (length - 1).  16 bits for `where` leave room for 512 runs in the 4 KiB of arguments that a
// launch takes: a list of single slots then needs no more launches than one with a slot each would.
constexpr int kMaxRuns = 512, kMaxGatherRows = 4096;
struct GatherRuns {
  int32_t slot[kMaxRuns];
  uint16_t where[kMaxRuns];
};
hipError_t launch_gather_inline(const void* layer_base, const GatherRuns& runs, int32_t n_runs,
                                void* k_out, void* v_out, hipStream_t s);

struct AttnArgs {
  const void* layer_base;   // KV of this layer
  const void* q;            // [n_q][8][256] bf16
  void* out;                // [n_q][8][256] bf16
  float* lse;               // [n_q][8] or null
  const int32_t* work;      // [n_work][32]: one 128-byte record per work item
  const int32_t* tables;
  const int32_t* part_off;  // [n_q]
  const int32_t* n_parts;   // [n_q]
  uint16_t* part_acc;       // [n_partials][8][256] fp16: accumulator * 2^(14 - exponent)
  float* part_ml;           // [n_partials][8][4]: reference max (log2 domain), sum, the exponents of
                            // the row's four 64-dim parts (int8 each), -
  int32_t n_work;
  int32_t n_q;
  float scale;
  int32_t write_through;    // split results go to memory at once (not zero) or when the L2 is flushed
  // Append folded into the work items (all three null otherwise): this step's new rows
  // [n_q][256] bf16 and their slots.  A streaming work item first writes the new rows that lie
  // in its key range into the pool; a fresh tile reads its keys from the new rows themselves
  // (the merge launch of the layer writes those rows to the pool).
  const void* k_new;
  const void* v_new;
  const int32_t* d_slots;
};
// Launches with more split results than kWriteThroughParts write them through, those with decode items
// (whose work items are short and end a launch, acknowledgement included) and two workgroups on some CU
// only beyond kWriteThroughMixed.  (What gains is that items still run when the first results leave; the rule
// goes by counts and does not look at how long they do.)  us per layer, flushed / written through, as steps that follow each other and
// (in brackets) with a read of 512 MB between them:
//   no decode items: 800 results 9.7 / 9.2 (10.4 / 9.9), 819 12.95 / 12.3 (13.9 / 14.5), 900 11.3 / 11.0 (12.0 / 11.9),
//     1050 10.4 / 9.7 (11.1 / 10.4), 1350 12.6 / 12.0 (13.6 / 13.3), 2000 18.3 / 16.6 (20.4 / 19.3), eight chunks on 832
//     tokens 20.8 / 17.8 (22.2 / 19.5), on 2048 24.9 / 24.1 (26.5 / 26.4);
//   decode items, at most 256 workgroups: 714 12.4 / 12.0 (13.4 / 13.2), 1039 13.2 / 12.5 (14.4 / 13.8);
//   decode items, more workgroups: 707 11.4 / 11.9 (12.4 / 12.9), 774 12.2 / 12.5 (12.2 / 12.7), 876 12.3 / 12.7 (13.1 / 13.4),
//     970 11.2 / 10.9 (12.4 / 12.7), 1071 10.3 / 9.8 (11.1 / 11.9), 1073 11.5 / 11.6 (12.6 / 13.4), 1172 14.3 / 15.4 (15.1 / 15.8);
//     1377 12.4 / 11.8 (13.6 / 13.7), 1608 13.8 / 12.8 (14.8 / 14.5), 64 requests and two chunks on 2048 tokens (1791)
//     24.4 / 23.6 (24.3 / 23.7).
constexpr int kWriteThroughParts = 640;    // 2.6 MB
constexpr int kWriteThroughMixed = 1280;   // 5.3 MB
hipError_t launch_attention(const AttnArgs& a, hipStream_t s);       // work items, then merge
// Split-result buffers in static device memory of the current device (kStaticMaxPartials
// entries, shared by every call on that device).  The first call on a device looks the address
// up; later calls make no HIP call other than hipGetDevice.
constexpr int kStaticMaxPartials = 2048;
hipError_t static_scratch(uint16_t** part_acc, float** part_ml);
// work items only; start/stop (may be null) receive the kernel's own begin/end timestamps
hipError_t launch_attention_work(const AttnArgs& a, hipStream_t s, hipEvent_t start = nullptr,
                                 hipEvent_t stop = nullptr);
struct AppendArgs {
  const void* k_new;
  const void* v_new;
  const int32_t* d_slots;
  int32_t n_blocks;      // workgroups: tokens, or runs
  void* layer_base;
  // null: tokens 0..n_blocks-1, a row each; else runs of up to 16 tokens in order that fill a block from
  // its first slot on, (first token << 4) | (length - 1)
  const int32_t* runs;
};
// Heads, and wavefronts, of a merge workgroup: 4, or all 8 where a launch has more tokens than the GPU has CUs.
// us per layer, 4 / 8: one request 6.70 / 6.83, 50 queries + one request 8.12 / 8.34, 78 queries 13.1 / 13.45, 164 22.8 /
// 22.7, 356 72.7 / 72.7, 400 17.8 / 17.3.  Each is a kernel of its own: a recording of one is none of the other.
constexpr int kMergeManyTokens = 256;
constexpr int merge_heads(int32_t n_q) { return n_q > kMergeManyTokens ? kHeads : kHeads / 2; }
// merge of `a`, and in the same launch the append described by `next` (may be null)
hipError_t launch_merge_append(const AttnArgs& a, const AppendArgs* next, hipStream_t s,
                               hipEvent_t start = nullptr, hipEvent_t stop = nullptr);

}  // namespace oxy

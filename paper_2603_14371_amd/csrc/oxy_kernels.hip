// HIP kernels for gfx950 (MI355X): KV append / gather and the mixed-mask paged attention.
//
// What is computed is the attention inside the paper's ActionDenoise and
// BatchedLanguageDecode passes (App. A.1, Eq. 5-6) for queries of several tasks at once,
// all reading one shared prefill cache (Sec. 3.2, cross-task KV sharing) plus their own
// tokens.  Visibility: prefix always; own tokens causally for decode queries, all of the
// chunk for action queries.
//
// Evaluation scheme.  The visible set of a query is cut into (prefix | own) and each part
// into fixed-size splits.  A work item is (query rows that share one KV source, one split of
// that source); it yields an un-normalised partial (reference max m in the log2 domain, sum
// l, accumulator acc[256]).  A second kernel merges a query's partials by the log-sum-exp
// rule.  How many queries share a work item depends on the whole batch; the splits depend on the
// pool and the item only, and a query's arithmetic is the same in a work item of any width, so its
// bits never depend on what else is in the batch.
//
// MFMA mapping (v_mfma_f32_16x16x32_bf16, lane = 16*g + n, keys taken 32 at a time = page A
// and page B of the block table):
//   S^T[key][row]  = sum_d K[key][d] * Q[row][d]      A = K chunks, B = Q rows
//       tile hf (0,1): A-row r is key 8hf + r%8 of page r/8, so lane (n = row, g) receives
//       the logits of keys 8hf + 4(g%2) + e, e < 4, of page g/2
//   O^T[d][row]   += sum_key V[key][d] * P[row][key]  A = V chunk, B = P
//       lane (g) contracts eight keys of one page, the same eight whose logits lane (g) of the
//       first product holds: its V operand is ONE 16-byte chunk of that page, and P goes from
//       wavefront to wavefront without moving between lanes.  A-row m of operand c is dim
//       64w+4m+c -> lane (n = row, g) accumulates dims 64w+16g..64w+16g+15 over four operands
// Both results keep "row = lane % 16", so the softmax state (m, l, rescale factor) is a
// per-lane scalar.  The pool pages are stored in exactly the operand order these products
// want (see oxy.h): every MFMA operand is one aligned 16-byte load.
#include "oxy_internal.h"

#include <hip/hip_ext.h>

#include <mutex>
#include <tuple>
#include <type_traits>
#include <utility>

namespace oxy {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;

__device__ __forceinline__ f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// two floats -> packed bf16 pair, round to nearest even (inputs are finite here)
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
  const f32x2 f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// two floats -> packed fp16 pair (round to nearest even)
__device__ __forceinline__ uint32_t pack_f16(float lo, float hi) {
  typedef __attribute__((__vector_size__(2 * sizeof(_Float16)))) _Float16 f16x2;
  const f32x2 f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, f16x2));
}
__device__ __forceinline__ void unpack_f16(uint32_t u, float& lo, float& hi) {
  typedef __attribute__((__vector_size__(2 * sizeof(_Float16)))) _Float16 f16x2;
  const f16x2 h = __builtin_bit_cast(f16x2, u);
  lo = (float)h[0];
  hi = (float)h[1];
}

// max over the four lanes {n, n+16, n+32, n+48} that hold one query row: two register swaps
// between lane halves (v_permlane16_swap, v_permlane32_swap), no LDS round trip
__device__ __forceinline__ float row_max4(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const uint32_t v = __float_as_uint(y);
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
// The same of G values at once: lane row g gets the maximum of value g % G.  The first swap leaves two lanes' parts of
// two values in a register, the second one those of all four lanes (of four values: three swaps, not eight).  us per
// layer, one value at a time / so: six chunks on 1500 tokens 17.55 / 17.25, on 2048 18.1 / 17.9, eight on 832 16.6 / 16.5,
// 256 requests 71.6 / 71.4.
template <int G>
__device__ __forceinline__ float row_max4_each(const float (&x)[G]) {
  if constexpr (G == 1) {
    return row_max4(x[0]);
  } else {
    float y[2];
#pragma unroll
    for (int i = 0; i < G / 2; ++i) {
      const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[2 * i]), __float_as_uint(x[2 * i + 1]), false, false);
      y[i] = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    }
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y[0]), __float_as_uint(y[G == 4]), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
  }
}
// sum over the same four lanes, same two swaps: every lane adds its own value and its partner's
__device__ __forceinline__ float row_sum4(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const uint32_t v = __float_as_uint(y);
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
// x of the lane N places on in the row of 16 lanes
template <int N>
__device__ __forceinline__ float dpp_row_ror(const float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x120 + N, 0xf, 0xf, false));
}
// f(0), f(1), .. f(N - 1) with the index as a constant
template <int N, class F, int... I>
__device__ __forceinline__ void static_for_each(const F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>()), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(const F& f) {
  static_for_each<N>(f, std::make_integer_sequence<int, N>());
}
// ------------------------------------------------------------------------------------------
// page layout (see oxy.h)
// ------------------------------------------------------------------------------------------
// K page: chunk (j, hf, g, k8) holds K[8hf+k8][32j+8g .. +7]
__device__ __forceinline__ int k_chunk_offset(int j, int hf, int g, int k8) {
  return ((((j * 2 + hf) * 4 + g) * 8) + k8) * 16;
}
// V page: chunk (w, c, gp, n) holds V[4gp..4gp+3][d] then V[8+4gp..8+4gp+3][d], d = 64w+4n+c
__device__ __forceinline__ int v_chunk_offset(int w, int c, int gp, int n) {
  return ((((w * 4 + c) * 2 + gp) * 16) + n) * 16;
}
// the chunk of dim d
__device__ __forceinline__ int v_chunk_of_dim(int d, int gp) {
  return v_chunk_offset(d >> 6, d & 3, gp, (d >> 2) & 15);
}
__device__ __forceinline__ int v_slot_of_key(int key) { return ((key >> 3) << 2) | (key & 3); }

// ------------------------------------------------------------------------------------------
// append / gather
// ------------------------------------------------------------------------------------------
// One row of K and V on its way into a page: thread t of 256 carries 16 bytes of K (t < 32)
// and one element of V.  Load and store are separate so that callers can keep several rows in
// flight before the first store.
struct RowPart {
  u32x4 k;
  uint16_t v;
};
__device__ __forceinline__ RowPart load_row(const uint16_t* __restrict__ k_row,
                                            const uint16_t* __restrict__ v_row, int t) {
  RowPart r;
  r.k = *(const u32x4*)(k_row + (t & 31) * 8);
  r.v = v_row[t];
  return r;
}
__device__ __forceinline__ void store_row(const RowPart& r, int32_t slot,
                                          char* __restrict__ layer_base, int t) {
  const int blk = slot >> 4, key = slot & 15;
  char* kp = layer_base + (size_t)blk * kBlockBytes;
  char* vp = kp + kPageBytes;
  if (t < 32) *(u32x4*)(kp + k_chunk_offset(t >> 2, key >> 3, t & 3, key & 7)) = r.k;
  *(uint16_t*)(vp + v_chunk_of_dim(t, (key >> 2) & 1) + v_slot_of_key(key) * 2) = r.v;
}
__device__ __forceinline__ void append_row(const uint16_t* __restrict__ k_row,
                                           const uint16_t* __restrict__ v_row, int32_t slot,
                                           char* __restrict__ layer_base, int t) {
  store_row(load_row(k_row, v_row, t), slot, layer_base, t);
}

__global__ __launch_bounds__(256) void append_kernel(const uint16_t* __restrict__ k_new,
                                                     const uint16_t* __restrict__ v_new,
                                                     const int32_t* __restrict__ slots,
                                                     char* __restrict__ layer_base) {
  const int tok = blockIdx.x;
  append_row(k_new + (size_t)tok * kDim, v_new + (size_t)tok * kDim, slots[tok], layer_base,
             threadIdx.x);
}

// Rows of keys key0..key0+n-1 of one block, by one workgroup: all rows are read at once, K goes out as
// 16-byte chunks and V, turned through LDS, as whole chunks where all eight keys of one are among them
// and key by key elsewhere, so that nothing else in the page is touched.  kWhole: all sixteen rows, without
// the other form's clamps and conditions (52 blocks of one layer 2.8 us, with them 3.1; 50 blocks in each of 18
// layers 6.2 / 6.4, kernel trace).
struct __align__(16) PageLds {
  uint16_t v[kPage][kDim + 8];   // +8: rows land in different banks
};
template <bool kWhole>
__device__ __forceinline__ void append_page(const uint16_t* __restrict__ k_src,
                                            const uint16_t* __restrict__ v_src, const int key0,
                                            const int n, char* __restrict__ block, PageLds& sm,
                                            const int t) {
  char* kp = block;
  char* vp = block + kPageBytes;
  u32x4 k[2], v[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int idx = t + 256 * i, cd = idx & 31;
    const int row = kWhole ? idx >> 5 : min(max((idx >> 5) - key0, 0), n - 1);
    k[i] = *(const u32x4*)(k_src + (size_t)row * kDim + cd * 8);
    v[i] = *(const u32x4*)(v_src + (size_t)row * kDim + cd * 8);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int idx = t + 256 * i, key = idx >> 5, cd = idx & 31;
    if (kWhole || (key >= key0 && key < key0 + n))
      *(u32x4*)(kp + k_chunk_offset(cd >> 2, key >> 3, cd & 3, key & 7)) = k[i];
    *(u32x4*)(&sm.v[key][cd * 8]) = v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int ci = t + 256 * i, gp = (ci >> 4) & 1, d = 64 * (ci >> 7) + 4 * (ci & 15) + ((ci >> 5) & 3);
    u32x4 out;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k0 = (e < 2 ? 4 * gp : 8 + 4 * gp) + 2 * (e & 1);
      out[e] = (uint32_t)sm.v[k0][d] | ((uint32_t)sm.v[k0 + 1][d] << 16);
    }
    if (kWhole || (key0 <= 4 * gp && key0 + n >= 12 + 4 * gp)) {
      *(u32x4*)(vp + ci * 16) = out;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int key = (e < 4 ? 4 * gp : 4 + 4 * gp) + e;
        if (key >= key0 && key < key0 + n)
          *(uint16_t*)(vp + ci * 16 + 2 * e) = (uint16_t)(out[e >> 1] >> (16 * (e & 1)));
      }
    }
  }
}
__device__ __forceinline__ void append_rows(const uint16_t* __restrict__ k_src,
                                            const uint16_t* __restrict__ v_src, const int key0,
                                            const int n, char* __restrict__ block, PageLds& sm,
                                            const int t) {
  if (n == kPage)
    append_page<true>(k_src, v_src, 0, kPage, block, sm, t);
  else
    append_page<false>(k_src, v_src, key0, n, block, sm, t);
}

// Append of a run of consecutive positions of one table (a prefix): one workgroup per block.
// blockIdx.y = layer relative to the first one: sources advance by src_layer_stride bytes, the
// pool by pool_layer_stride bytes per layer.
__global__ __launch_bounds__(256) void append_blocks_kernel(const uint16_t* __restrict__ k_new,
                                                            const uint16_t* __restrict__ v_new,
                                                            const InlineIds blocks, int32_t pos0,
                                                            int32_t n_tokens,
                                                            char* __restrict__ layer_base,
                                                            size_t src_layer_stride,
                                                            size_t pool_layer_stride) {
  __shared__ PageLds sm;
  k_new = (const uint16_t*)((const char*)k_new + blockIdx.y * src_layer_stride);
  v_new = (const uint16_t*)((const char*)v_new + blockIdx.y * src_layer_stride);
  layer_base += blockIdx.y * pool_layer_stride;
  const int page = (pos0 >> 4) + blockIdx.x;
  const int lo = max(pos0, page * kPage), hi = min(pos0 + n_tokens, (page + 1) * kPage);
  append_rows(k_new + (size_t)(lo - pos0) * kDim, v_new + (size_t)(lo - pos0) * kDim, lo & 15, hi - lo,
              layer_base + (size_t)blocks.v[blockIdx.x] * kBlockBytes, sm, threadIdx.x);
}

// Reads runs of tokens back in natural order, one workgroup per run (at most the 16 tokens of a
// block; see oxy_internal.h for the encoding).  Every V chunk holds one dim of eight keys, so a
// token alone touches all of its V page: the page is read once as whole chunks, turned through
// LDS, and only the run's rows are written; of a page the chunks with a key of the run are read (a
// single token's are half of them).  (One workgroup per token read 256 two-byte pieces per row: the
// 1337 tokens of four histories took three launches of 2.8 us, now one of 3.4 us.  A list of as many
// scattered single slots takes three launches as before; the C call waited for is 23.5 us against 21.7.)
__global__ __launch_bounds__(256) void gather_inline_kernel(const char* __restrict__ layer_base,
                                                            const GatherRuns runs,
                                                            uint16_t* __restrict__ k_out,
                                                            uint16_t* __restrict__ v_out) {
  __shared__ __align__(16) uint16_t v_s[kPage][kDim + 8];   // +8: rows start in different banks
  const int t = threadIdx.x;
  const int slot = runs.slot[blockIdx.x], where = runs.where[blockIdx.x];
  const int key0 = slot & 15, len = (where & 15) + 1;
  const size_t out0 = (size_t)(where >> 4);
  const char* kp = layer_base + (size_t)(slot >> 4) * kBlockBytes;
  const char* vp = kp + kPageBytes;
  // chunks with a key of the run: keys 4gp..4gp+3 and 8+4gp..8+4gp+3 (gp = (t >> 4) & 1 for both)
  const int lo = 4 * ((t >> 4) & 1), hi = lo + 8, end = key0 + len;
  const bool wanted = (key0 < lo + 4 && end > lo) || (key0 < hi + 4 && end > hi);
  u32x4 v[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (wanted) v[i] = *(const u32x4*)(vp + (t + 256 * i) * 16);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int idx = t + 256 * i, key = idx >> 5, cd = idx & 31;
    if (key >= key0 && key < key0 + len)
      *(u32x4*)(k_out + (out0 + key - key0) * kDim + cd * 8) =
          *(const u32x4*)(kp + k_chunk_offset(cd >> 2, key >> 3, cd & 3, key & 7));
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int ci = t + 256 * i, gp = (ci >> 4) & 1, d = 64 * (ci >> 7) + 4 * (ci & 15) + ((ci >> 5) & 3);
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (wanted) v_s[(e < 4 ? 4 * gp : 4 + 4 * gp) + e][d] = (uint16_t)(v[i][e >> 1] >> (16 * (e & 1)));
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int idx = t + 256 * i, key = idx >> 5, cd = idx & 31;
    if (key >= key0 && key < key0 + len)
      *(u32x4*)(v_out + (out0 + key - key0) * kDim + cd * 8) = *(const u32x4*)(&v_s[key][cd * 8]);
  }
}

// Descriptor upload: pinned host memory -> device memory, read over the bus by the kernel itself.
// A copy of this size (8 to 100 KiB) is bound by its hand-over: hipMemcpyAsync gives one of more
// than 16 KiB to a copy engine, and the two queues then wait for each other's signals (fixed cost of
// a step with a 33 KiB descriptor 30 us, of one with 8 KiB, which is copied by a kernel, 12 us).
__global__ __launch_bounds__(256) void upload_kernel(const int32_t* __restrict__ src,
                                                     int32_t* __restrict__ dst, int32_t n_words) {
  const int i = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (i + 4 <= n_words) {
    *(u32x4*)(dst + i) = __builtin_nontemporal_load((const u32x4*)(src + i));
  } else {
    for (int k = i; k < n_words; ++k) dst[k] = src[k];
  }
}

// The status is the launch's own (hipGetLastError would report, and clear, whatever an earlier call
// of the thread left behind), and the launch completes `done` itself: recording an event behind it
// is one more runtime call and one more packet (one-layer step 19.3 -> 18.5 us, 25.0 -> 24.0 in
// processes where the runtime's calls are slow).
hipError_t launch_upload(const int32_t* pinned, int32_t* device, int32_t n_words, hipStream_t s,
                         hipEvent_t done) {
  if (n_words <= 0) return hipErrorInvalidValue;
  void* args[] = {&pinned, &device, &n_words};
  return hipExtLaunchKernel((const void*)upload_kernel, dim3((n_words + 1023) / 1024), dim3(256),
                            args, 0, s, nullptr, done, 0);
}

hipError_t launch_append(const void* k_new, const void* v_new, const int32_t* d_slots,
                         int32_t n_tokens, void* layer_base, hipStream_t s) {
  if (n_tokens <= 0) return hipSuccess;
  append_kernel<<<n_tokens, 256, 0, s>>>((const uint16_t*)k_new, (const uint16_t*)v_new, d_slots,
                                         (char*)layer_base);
  return hipGetLastError();
}

hipError_t launch_append_inline(const void* k_new, const void* v_new, const InlineIds& blocks,
                                int32_t pos0, int32_t n_tokens, void* layer_base, int32_t n_layers,
                                size_t src_layer_stride, size_t pool_layer_stride, hipStream_t s) {
  if (n_tokens <= 0 || n_layers <= 0) return hipSuccess;
  // blocks.v[i] is the block of page (pos0 / 16 + i)
  const int32_t n_pages = ((pos0 + n_tokens + kPage - 1) >> 4) - (pos0 >> 4);
  append_blocks_kernel<<<dim3(n_pages, n_layers), 256, 0, s>>>(
      (const uint16_t*)k_new, (const uint16_t*)v_new, blocks, pos0, n_tokens, (char*)layer_base,
      src_layer_stride, pool_layer_stride);
  return hipGetLastError();
}

hipError_t launch_gather_inline(const void* layer_base, const GatherRuns& runs, int32_t n_runs,
                                void* k_out, void* v_out, hipStream_t s) {
  if (n_runs <= 0) return hipSuccess;
  gather_inline_kernel<<<n_runs, 256, 0, s>>>((const char*)layer_base, runs, (uint16_t*)k_out,
                                              (uint16_t*)v_out);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// attention work items
// ------------------------------------------------------------------------------------------
constexpr float kGrow = 8.f;  // the reference max only moves when a logit exceeds it by 2^8
constexpr int kMaxGroups = 4; // groups of 16 query rows (two tokens) in one work item

// LDS of a work item: nothing of K and V, only what the four wavefronts exchange.  Every u32x4
// entry is one lane's 16-byte MFMA operand, stored and read back at the lane's own position.
struct __align__(16) WorkLds {
  u32x4 q[kMaxGroups][8][64];      // query fragments (B operand of S^T), the same for all wavefronts
  u32x4 p[4][kMaxGroups][2][64];   // [32-key step of the round][group][hi / lo]: P of all 128 keys
  float mx[kMaxGroups][16][4];     // largest logit of a row among each wavefront's 32 keys
  int slot[2 * kMaxGroups];        // split result of each token
  float ls[kMaxGroups][64][4];     // sum of a lane's P over each wavefront's keys
};

// The descriptor is read with scalar loads: it is not written during a launch and every address
// is wave-uniform, so records, token ids and block ids land in scalar registers, take no part in
// the order in which the vector loads of queries and pages complete, and need no lane reads.
typedef const __attribute__((address_space(4))) int32_t* DescPtr;
typedef int32_t i32x8 __attribute__((ext_vector_type(8)));
typedef const __attribute__((address_space(4))) i32x8* DescPtr8;

// A record: 8 header words, 8 query token ids (the last one repeated), the block ids of the
// split's first 16 pages (the last one repeated).  All but the last eight words are requested
// at once at the start of the kernel.
struct WorkItem {
  DescPtr rec;
  i32x8 toks, pages;
  int n_tok, tbl_off, kv_begin, kv_end, q0, part_idx;
};
// What a work item needs only after its first loads, read from the argument segment there.
struct LateArgs {
  uint16_t* part_acc;
  float* part_ml;
  const int32_t* tables;
  int32_t write_through;
};
constexpr int kLateOffset = 7 * 8;   // behind the preloaded arguments (held against attn_kernel's own list below it)
__device__ __forceinline__ void take_late(AttnArgs& a) {
  auto seg = (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(seg));   // here, and not at the start of the kernel
  const auto* late = (const __attribute__((address_space(4))) LateArgs*)(seg + kLateOffset);
  a.part_acc = late->part_acc;
  a.part_ml = late->part_ml;
  a.tables = late->tables;
  a.write_through = late->write_through;
}
// query token of this lane's row in group r
__device__ __forceinline__ int token_of(const WorkItem& wi, const int r, const int second) {
  return second ? wi.toks[2 * r + 1] : wi.toks[2 * r];
}
// First split result of token lane % (2*G) of the item.  It is needed at the very end only, but
// requested at the start (a full memory latency in front of the stores otherwise) and kept in LDS
// meanwhile: four groups leave no registers for it.
template <int G>
__device__ __forceinline__ int request_slot(const AttnArgs& a, const WorkItem& wi, const int lane) {
  int tok = wi.toks[0];
#pragma unroll
  for (int i = 1; i < 2 * G; ++i) tok = lane % (2 * G) == i ? wi.toks[i] : tok;
  return a.part_off[tok];
}

// Values of keys at or beyond kv_end may be stale bits (never-written slots, freed blocks):
// they are selected to zero, not multiplied by zero.  `left` = valid keys in this step.
__device__ __forceinline__ u32x4 value_mask(const int left, const int g) {
  const int k0 = 16 * (g >> 1) + 4 * (g & 1);
  u32x4 mask;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    mask[i] = (k0 + 2 * i < left ? 0xffffu : 0u) | (k0 + 2 * i + 1 < left ? 0xffff0000u : 0u);
    mask[2 + i] = (k0 + 8 + 2 * i < left ? 0xffffu : 0u) | (k0 + 8 + 2 * i + 1 < left ? 0xffff0000u : 0u);
  }
  return mask;
}

// Softmax scale in the log2 domain, as a positive factor: the largest logit of a row is then the
// scale times its largest dot product, and one fused multiply-add takes a dot product to its
// exponent.  A negative scale goes into the sign of the queries (see query_sign); a zero one is
// taken as 2^-120, which gives the same uniform weights and keeps -inf (a masked key) what it is.
__device__ __forceinline__ float log2_scale(const AttnArgs& a) {
  const float x = fabsf(a.scale * 1.4426950408889634f);
  return x == 0.f ? 0x1p-120f : x;
}
// flips the signs of eight bf16 query elements where the scale is negative
__device__ __forceinline__ u32x4 query_sign(const AttnArgs& a, const u32x4 q) {
  const uint32_t flip = a.scale < 0.f ? 0x80008000u : 0u;
  return q ^ (u32x4){flip, flip, flip, flip};
}
// largest of a lane's eight dot products
__device__ __forceinline__ float row_max8(const f32x4 s0, const f32x4 s1) {
  return fmaxf(fmaxf(fmaxf(s0[0], s0[1]), fmaxf(s0[2], s0[3])),
               fmaxf(fmaxf(s1[0], s1[1]), fmaxf(s1[2], s1[3])));
}
// P = 2^(sl2 * s - m) of a lane's eight dot products as hi + lo bf16 (a single bf16 rounding, 2^-9
// relative, is too coarse for queries that see only a handful of keys); returns their fp32 sum.
__device__ __forceinline__ float softmax_weights(const f32x4 s0, const f32x4 s1, const float sl2,
                                                 const float m, u32x4& hi, u32x4& lo) {
  float p[8], sum = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    p[e] = fast_exp2(__builtin_fmaf(e < 4 ? s0[e & 3] : s1[e & 3], sl2, -m));
    sum += p[e];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    hi[i] = pack_bf16(p[2 * i], p[2 * i + 1]);
    lo[i] = pack_bf16(p[2 * i] - __uint_as_float(hi[i] << 16),
                      p[2 * i + 1] - __uint_as_float(hi[i] & 0xffff0000u));
  }
  return sum;
}
// A row's sum times the factor of a moved reference.  Rounded here, never contracted with the addition
// that follows: otherwise `attend`, where the two lie in different branches, and `attend_fresh`, where
// they do not, give different bits.
__device__ __forceinline__ float rescaled(const float l, const float alpha) {
#pragma clang fp contract(off)
  return l * alpha;
}
// Stores a at dst and b 64 bytes on.  A launch leaves its split results dirty in eight L2s, and the
// merge launch starts only when they have been written back: 1.4 us after the last work item of a
// launch with 9 split results, 5.8 us with 15 MB of them.  Written through (sc0 sc1) they reach
// memory while other work items run.  A work item then ends with their acknowledgement, which costs
// a small launch more than it gives, hence a flag (see kWriteThroughParts).  In inline assembly: no
// builtin takes these bits with a 64-bit address.  The wait counts that the compiler places after it are
// only ever stricter than needed, and the two wait states keep the data registers from being
// written in the cycles in which a 128-bit store still reads them.
__device__ __forceinline__ void store_piece_pair(const AttnArgs& args, u32x4* dst, const u32x4 a,
                                                 const u32x4 b) {
  if (args.write_through) {
    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\t"
                 "global_store_dwordx4 %0, %2, off offset:64 sc0 sc1\n\t"
                 "s_nop 1" ::"v"(dst), "v"(a), "v"(b) : "memory");
  } else {
    dst[0] = a;
    dst[4] = b;
  }
}
// Eight rows' 128 bytes each at (split result, offset), for both tokens of a group: see store_part.  Buffer
// stores take the cache bits of the written-through form as an argument.
__device__ __forceinline__ void store_lines(const AttnArgs& args, const int offset, const int slot_a,
                                            const u32x4 a, const bool live_a, const int slot_b,
                                            const u32x4 b, const bool live_b) {
  constexpr int kPartBytes = kHeads * kDim * (int)sizeof(uint16_t), kFlags = 0x00027000;
  constexpr int kThrough = 1 | 16;   // sc0, sc1
  // a token that is not there has a buffer of no bytes: its rows are dropped
  const auto part_a = __builtin_amdgcn_make_buffer_rsrc((char*)args.part_acc + (size_t)slot_a * kPartBytes, 0,
                                                        live_a ? kPartBytes : 0, kFlags);
  const auto part_b = __builtin_amdgcn_make_buffer_rsrc((char*)args.part_acc + (size_t)slot_b * kPartBytes, 0,
                                                        live_b ? kPartBytes : 0, kFlags);
  if (args.write_through) {
    __builtin_amdgcn_raw_buffer_store_b128(a, part_a, offset, 0, kThrough);
    __builtin_amdgcn_raw_buffer_store_b128(b, part_b, offset, 0, kThrough);
  } else {
    __builtin_amdgcn_raw_buffer_store_b128(a, part_a, offset, 0, 0);
    __builtin_amdgcn_raw_buffer_store_b128(b, part_b, offset, 0, 0);
  }
}
constexpr int kRowRor8 = 0x128;   // DPP: lane n of each 16 gets lane n^8's value
// One wavefront's 64 dims of a group's split result.  A split result leaves as (m, l, four
// exponents) and acc * 2^(14 - exponent) in fp16: half the bytes of fp32, with the exponent of the
// largest value per row and 64 dims, so that the rounding does not depend on the magnitude of the
// values.  kLines: whole lines, for items of eight tokens, whose launches write the most (us per layer, pieces /
// lines: eight chunks on 2048 tokens 24.4 / 23.6, six on 1500 22.1 / 21.6, four and 32 requests on 1024 17.9 / 17.1,
// eight on 832 17.36 / 17.32; narrower items are up to 1 % slower with it).  acc[c][e] = dim 16g + 4e + c of the 64: a lane's sixteen values are consecutive.  slot:
// split result of this lane's token.
template <bool kLines>
__device__ __forceinline__ void store_part(const AttnArgs& a, const WorkItem& wi, const int slot,
                                           const f32x4 (&acc)[4], const int group, const int wv,
                                           const int lane) {
  const int n = lane & 15, g = lane >> 4;
  float amax = 0.f;
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) amax = fmaxf(amax, fabsf(acc[c][e]));
  amax = row_max4(amax);
  // biased exponent of amax, kept where 2^(14 - exponent) is a normal number
  const int eb = max(24, min(253, (int)(__float_as_uint(amax) >> 23)));
  // an infinite value leaves no exponent for the others: all 64 are NaN then, instead of zeros (looking
  // for the largest finite one in a branch of its own cost 0.5 % of a launch of chunks)
  const float up = __uint_as_float((uint32_t)(127 + 14 + 126 - eb) << 23) + (amax - amax);
  const int ex = eb - 126;
  u32x4 o[2];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    o[e >> 1][2 * (e & 1)] = pack_f16(acc[0][e] * up, acc[1][e] * up);
    o[e >> 1][2 * (e & 1) + 1] = pack_f16(acc[2][e] * up, acc[3][e] * up);
  }
  if constexpr (kLines) {
    // Lane g of row n holds 16-byte pieces 2g and 2g+1 of the row's eight.  Rows n and n^8 (the group's two
    // tokens) trade one each, so that a store takes whole lines: eight lanes the 128 bytes of one row, a
    // token's eight rows at once.
    u32x4 first = o[0], second = o[1];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      first[i] = __builtin_amdgcn_update_dpp(o[0][i], o[1][i], kRowRor8, 0xf, 0xc, false);
      second[i] = __builtin_amdgcn_update_dpp(o[1][i], o[0][i], kRowRor8, 0xf, 0x3, false);
    }
    const int offset = (n & 7) * (kDim * 2) + 128 * wv + 32 * g + 16 * (n >> 3);
    store_lines(a, offset, __builtin_amdgcn_readlane(slot, 0), first, 2 * group < wi.n_tok,
                __builtin_amdgcn_readlane(slot, 8), second, 2 * group + 1 < wi.n_tok);
    if (g == 0 && 2 * group + (n >> 3) < wi.n_tok)
      ((int8_t*)(a.part_ml + ((size_t)slot * kHeads + (n & 7)) * 4 + 2))[wv] = (int8_t)ex;
    return;
  }
  // Lane g of a row holds 16-byte pieces 2g and 2g+1 of the row's eight: exchanged so that the
  // four lanes of a row store pieces 0..3 together and then 4..7, 64 contiguous bytes each time.
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const auto x = __builtin_amdgcn_permlane16_swap(o[0][i], o[1][i], false, false);
    const auto y = __builtin_amdgcn_permlane32_swap(x[0], x[1], false, false);
    o[0][i] = y[0];
    o[1][i] = y[1];
  }
  if (2 * group + (n >> 3) < wi.n_tok) {
    const size_t row = (size_t)slot * kHeads + (n & 7);
    u32x4* dst = (u32x4*)(a.part_acc + row * kDim + 64 * wv + 8 * g);
    store_piece_pair(a, dst, o[0], o[1]);
    if (g == 0) ((int8_t*)(a.part_ml + row * 4 + 2))[wv] = (int8_t)ex;
  }
}

// Bound by the memory pipeline of the CU where a launch is large (128 KiB of pages per workgroup and
// round, two workgroups per CU), by the length of this chain where it is small.
//
// One work item: up to 2*G query tokens (G groups of 16 rows) against one split of a KV source,
// taken in rounds of 128 keys.  In a round wavefront w
//   1. holds the K operands of keys 32w..32w+31 in registers and computes S^T for all rows,
//   2. publishes each row's largest logit, and after a barrier takes the row's largest of all 128,
//   3. writes its P (hi + lo bf16, relative to the common reference max) to LDS,
//   4. after a second barrier contracts ALL 128 keys for dims 64w..64w+63, whose V operands it
//      loaded itself.
// K and V thus go from memory to registers exactly once per work item and never through LDS; what
// the wavefronts exchange is P (2 KiB per group and step).  The accumulator is 16 registers per
// group, no combination of per-wavefront accumulators follows, and a work item of eight tokens fits
// the registers of two workgroups per CU.  (Before: work items of up to two tokens kept a
// 64-register accumulator per wavefront and combined the four through 66 KiB of LDS, 1.1 us of a
// 4 us work item, now 0.4; larger ones staged K and V in LDS, where each of the four wavefronts
// read all of both.  Work-item launch of one request on 832 tokens 5.44 -> 4.79 us, of eight requests
// and a chunk 7.8 -> 7.05, of eight chunks on 2048 tokens 23.3 -> 20.6, of 64 requests and two
// chunks on 2048-token prefixes 20.55 -> 20.27, kernel trace.)
//
// A row's arithmetic does not depend on G or on the other rows: a query may be evaluated alone or
// beside any others and gives the same bits.
//
// kOwnPages: a decode item's own pages, read by this work item alone, which also writes the item's
// new rows when the append is folded in.  Otherwise the pages are a prefix's or a multi-token item's,
// and other work items read them too.  kOnce: non-temporal page loads, for own pages that will have
// left the Infinity Cache by the next step and are not to push others out (see kOnceBytes).
//
// kSteps: 32-key steps of a round that are loaded, 4, or 2 for a split of at most 64 keys of a prefix or of a
// multi-token item (the last one of an 832-token prefix, a short observation's): wavefronts 2 and 3 load no
// K then, and all of them half of V.  A decode item's own pages always take 4.  (With every step loaded, the
// pages past the end once more, such an item took as long as one of 128 keys and kept the loads of its
// CU's other workgroup waiting: work-item launch of eight requests and a chunk 7.3 us, now 7.0, of six
// requests with 13 new tokens 10.2 / 9.6; others +-0.5 %.)
template <int G, bool kOwnPages, bool kOnce, int kSteps>
__device__ __forceinline__ void attend(const AttnArgs& early_args, const WorkItem& wi, WorkLds& sm) {
  AttnArgs a = early_args;
  int tid = threadIdx.x;
  // keeps what is computed from the thread id inside this instance: shared with the other
  // instances of the kernel it would have to live across all of them, which costs G = 4 spills
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: keep it scalar
  const int n = lane & 15, g = lane >> 4;
  const int h = n & 7, sub = n >> 3;
  const float ninf = -__builtin_inff();
  const float sl2 = log2_scale(a);
  const char* __restrict__ base = (const char*)a.layer_base;
  const int nsteps = (wi.kv_end - wi.kv_begin + 31) >> 5;
  const int rounds = (nsteps + 3) >> 2;
  const int npg = ((wi.kv_end + 15) >> 4) - (wi.kv_begin >> 4);


  u32x4 kr[16];      // kr[2j+hf]: K operand (j, hf) of this wavefront's 32 keys
  u32x4 vr[kSteps][4];    // vr[s][c]: V operand c of this wavefront's 64 dims, step s of the round
  auto page_load = [](const char* p) {
    if constexpr (kOnce) return __builtin_nontemporal_load((const u32x4*)p);
    return *(const u32x4*)p;
  };
  // A step past the split's end re-reads a page of the split; its logits are masked and its V
  // operands are not used.  The block ids of the first two rounds are in the record (no dependent
  // load in front of the first pages), those of later rounds in the block table.
  // Lane offsets are formed anew at every use (the asm statements): hoisted out of the rounds as
  // 64-bit addresses they cost four groups the registers that they do not have.
  auto load_k_of = [&](const int blk_a, const int blk_b) {
    int off = (g * 8 + (n & 7)) * 16;
    asm volatile("" : "+v"(off));
    const char* p = base + (size_t)((n >> 3) ? blk_b : blk_a) * kBlockBytes + off;
#pragma unroll
    for (int i = 0; i < 16; ++i) kr[i] = page_load(p + i * 512);
  };
  auto load_v_of = [&](const i32x8 blks) {
    int off = kPageBytes + v_chunk_offset(wv, 0, g & 1, n);
    asm volatile("" : "+v"(off));
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      const char* p = base + (size_t)((g >> 1) ? blks[2 * s + 1] : blks[2 * s]) * kBlockBytes + off;
#pragma unroll
      for (int c = 0; c < 4; ++c) vr[s][c] = page_load(p + c * 512);
    }
  };
  auto load_k = [&](const int round) {
    if (round < 2) {
      const DescPtr id = wi.rec + 16 + 8 * round + 2 * wv;
      load_k_of(id[0], id[1]);
    } else {
      const DescPtr ids = (DescPtr)a.tables + wi.tbl_off + (wi.kv_begin >> 4);
      const int pi = 8 * round + 2 * wv;
      load_k_of(ids[min(pi, npg - 1)], ids[min(pi + 1, npg - 1)]);
    }
  };
  auto load_v = [&](const int round) {
    if (round < 2) {
      load_v_of(*(DescPtr8)(wi.rec + 16 + 8 * round));
    } else {
      const DescPtr ids = (DescPtr)a.tables + wi.tbl_off + (wi.kv_begin >> 4);
      i32x8 blks;
#pragma unroll
      for (int i = 0; i < 8; ++i) blks[i] = ids[min(8 * round + i, npg - 1)];
      load_v_of(blks);
    }
  };

  // Folded append: the query tokens of an item on its own pages are its new rows.  Those inside
  // this split's key range are written to the pool by this workgroup (no other workgroup reads
  // them in this launch), and a workgroup barrier orders the writes before the page loads that
  // cover them.  The first new row sits in step `first_new`: when that step belongs to a later
  // round, its loads come after the barriers of the first one anyway; otherwise the rows go out,
  // with a barrier of their own, before the first page load.
  RowPart rows[2];
  int32_t row_slot[2] = {0, 0};
  bool row_mine[2] = {false, false};
  bool early = false;
  const bool fold = kOwnPages && a.k_new;
  if (fold) {
    const int pos0 = (wi.q0 == kNoCausal ? 0 : wi.q0);
    const int ta = wi.toks[0], tb = wi.toks[1];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int pos = pos0 + t;
      row_mine[t] = t < wi.n_tok && pos >= wi.kv_begin && pos < wi.kv_end;
      const int tk = t ? tb : ta;
      rows[t] = load_row((const uint16_t*)a.k_new + (size_t)tk * kDim,
                         (const uint16_t*)a.v_new + (size_t)tk * kDim, tid);
    }
    row_slot[0] = ((DescPtr)a.d_slots)[ta];
    row_slot[1] = ((DescPtr)a.d_slots)[tb];
    const int first_new = (max(pos0, wi.kv_begin) - wi.kv_begin) >> 5;
    early = first_new < 4;
    if (early) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
        if (row_mine[t])
          store_row(rows[t], row_slot[t], (char*)a.layer_base, tid);
      __syncthreads();
    }
  }
  // The query loads are issued BEFORE the first pages: loads complete in order per wavefront, so
  // the barrier below waits for the queries only, not for the slowest wavefront's first 32 KiB.
  int slot_req;
  {
    u32x4 qtmp[G][2];
#pragma unroll
    for (int r = 0; r < G; ++r) {
      const char* qrow = (const char*)a.q + ((size_t)token_of(wi, r, sub) * kHeads + h) * (kDim * 2);
#pragma unroll
      for (int jj = 0; jj < 2; ++jj)   // unconditional, zeroed afterwards
        qtmp[r][jj] = *(const u32x4*)(qrow + (2 * wv + jj) * 64 + g * 16);
    }
    slot_req = request_slot<G>(a, wi, lane);
    __builtin_amdgcn_sched_barrier(0);
    auto store_q = [&]() {
      __builtin_amdgcn_sched_barrier(0);
      take_late(a);
#pragma unroll
      for (int r = 0; r < G; ++r) {
        const u32x4 z = {0, 0, 0, 0};
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
          sm.q[r][2 * wv + jj][lane] = 2 * r + sub < wi.n_tok ? query_sign(a, qtmp[r][jj]) : z;
      }
    };
    // on both sides by itself: behind the join the queries would be waited for as if no K were in flight
    if (kSteps == 2 && wv >= 2) {
      load_v_of(wi.pages);
      store_q();
    } else {
      load_k_of(wi.rec[16 + 2 * wv], wi.rec[17 + 2 * wv]);
      load_v_of(wi.pages);
      store_q();
    }
  }
  if (tid < 2 * G) sm.slot[tid] = slot_req + wi.part_idx;
  if (fold && !early) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
      if (row_mine[t])
        store_row(rows[t], row_slot[t], (char*)a.layer_base, tid);
  }
  __syncthreads();

  float m[G], l[G];   // reference max (scaled log2 domain) of this lane's row, and the sum of P
  f32x4 acc[G][4];    // over this wavefront's keys; acc[r][c][e] = dim 64w + 16g + 4e + c
#pragma unroll
  for (int r = 0; r < G; ++r) {
    m[r] = ninf;
    l[r] = 0.f;
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[r][c] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }

  // kLast: the split's last round, the only one with steps past the end or a partial step.  It is
  // a copy of its own so that the loads of the other rounds sit under no condition.
  auto round_body = [&](const int round, auto last) {
    constexpr bool kLast = decltype(last)::value;
    int lane_now = tid & 63;   // likewise, for the mask limits and LDS addresses
    asm volatile("" : "+v"(lane_now));
    const int lane = lane_now, n = lane & 15, g = lane >> 4, sub = n >> 3;
    const int pos = wi.kv_begin + 32 * (4 * round + wv);
    const int left = wi.kv_end - pos;
    const bool need_mask = (kLast && left < 32) || pos + 31 > wi.q0;
    constexpr int kAhead = G == 4 ? 3 : 8;
    f32x4 s0[G], s1[G];
    // with two steps wavefronts 2 and 3 have no keys (and kr[] was never written): nothing is visible
    if (kSteps == 4 || wv < 2) {
#pragma unroll
      for (int r = 0; r < G; ++r) {
        s0[r] = (f32x4){0.f, 0.f, 0.f, 0.f};
        s1[r] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const u32x4 q = sm.q[r][j][lane];
          s0[r] = mfma16(kr[2 * j], q, s0[r]);
          s1[r] = mfma16(kr[2 * j + 1], q, s1[r]);
        }
      }
      // a few query reads ahead of the products: more would cost registers that four groups do
      // not leave, fewer make every pair of products wait a full LDS round trip (four groups with three ahead for
      // two, fewer groups with eight for four, us per layer: five chunks on 1500 tokens 16.6 / 16.4, a chunk of 300
      // 21.2 / 20.85, eight on 832 16.6 / 16.5, six and 48 requests 16.35 / 16.25)
      __builtin_amdgcn_sched_group_barrier(0x100, kAhead, 0);
#pragma unroll
      for (int i = 0; i < 8 * G - kAhead; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 2 * kAhead, 0);
      if (need_mask) {   // wave-uniform: only the end of a split or the causal diagonal
        const int k0 = pos + 16 * (g >> 1) + 4 * (g & 1);
#pragma unroll
        for (int r = 0; r < G; ++r) {
          const int end = min(wi.kv_end, wi.q0 + 2 * r + sub + 1) - k0;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            s0[r][e] = e < end ? s0[r][e] : ninf;
            s1[r][e] = 8 + e < end ? s1[r][e] : ninf;
          }
        }
      }
    } else {
#pragma unroll
      for (int r = 0; r < G; ++r) s0[r] = s1[r] = (f32x4){ninf, ninf, ninf, ninf};
    }
    {
      float mx[G];
#pragma unroll
      for (int r = 0; r < G; ++r) mx[r] = row_max8(s0[r], s1[r]) * sl2;
      const float mine = row_max4_each(mx);
      if (g < G) sm.mx[g][n][wv] = mine;
    }
    __syncthreads();
    // Online softmax.  The reference max only moves when a logit exceeds it by more than kGrow,
    // so the rescale of acc is rare; P is then at most 2^kGrow, well inside fp32/bf16 range.  P
    // travels as hi+lo bf16: a single bf16 rounding (2^-9 relative) is too coarse for queries that
    // see only a handful of keys.
    float mx[G];
    bool grow = false;   // true for the first finite logit too (m = -inf)
#pragma unroll
    for (int r = 0; r < G; ++r) {
      const f32x4 mw = *(const f32x4*)sm.mx[r][n];
      mx[r] = fmaxf(fmaxf(mw[0], mw[1]), fmaxf(mw[2], mw[3]));
      grow |= mx[r] > m[r] + kGrow;
    }
    if (__any(grow)) {
#pragma unroll
      for (int r = 0; r < G; ++r) {
        const bool up = mx[r] > m[r] + kGrow;
        const float alpha = up ? fast_exp2(m[r] - mx[r]) : 1.f;   // m = -inf gives 0
        l[r] = rescaled(l[r], alpha);
        if (round > 0) {   // acc holds zeros before
#pragma unroll
          for (int c = 0; c < 4; ++c) acc[r][c] *= alpha;
        }
        m[r] = up ? mx[r] : m[r];
      }
    }
#pragma unroll
    for (int r = 0; r < G; ++r) {
      u32x4 hi, lo;
      l[r] += softmax_weights(s0[r], s1[r], sl2, (m[r] == ninf) ? 0.f : m[r], hi, lo);
      sm.p[wv][r][0][lane] = hi;
      sm.p[wv][r][1][lane] = lo;
      if constexpr (kLast) sm.ls[r][lane][wv] = l[r];
    }
    __builtin_amdgcn_sched_barrier(0);   // the next K operands reuse kr[]
    if constexpr (!kLast) load_k(round + 1);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    // With one group all P operands are requested at once, in front of the branches of a last
    // round; with more the products of one group hide the reads of the next.
    u32x4 ph[kSteps], pl[kSteps];
    if constexpr (G == 1) {
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        ph[s] = sm.p[s][0][0][lane];
        pl[s] = sm.p[s][0][1][lane];
      }
    }
    auto contract = [&](const int s, const int r) {
      const u32x4 hi = G == 1 ? ph[s] : sm.p[s][r][0][lane];
      const u32x4 lo = G == 1 ? pl[s] : sm.p[s][r][1][lane];
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[r][c] = mfma16(vr[s][c], hi, acc[r][c]);
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[r][c] = mfma16(vr[s][c], lo, acc[r][c]);
    };
    if constexpr (!kLast) {
#pragma unroll
      for (int s = 0; s < kSteps; ++s)
#pragma unroll
        for (int r = 0; r < G; ++r) contract(s, r);
      __builtin_amdgcn_sched_barrier(0);   // likewise vr[]
      load_v(round + 1);
      __builtin_amdgcn_sched_barrier(0);
    } else {
      const int nv = nsteps - 4 * round;   // 1..4 steps
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        const int left_s = wi.kv_end - (wi.kv_begin + 32 * (4 * round + s));
        if (s < nv && left_s < 32) {
          const u32x4 mask = value_mask(left_s, g);
#pragma unroll
          for (int c = 0; c < 4; ++c) vr[s][c] &= mask;
        }
        if (G == 1 && s < nv) contract(s, 0);
      }
      // Several groups: group by group, so that a group's scaling and stores fall into the
      // products of the next (8 chunks on 2048 tokens 164.1 -> 160.2 us for six layers).
      auto finish = [&](auto full) {
#pragma unroll
        for (int r = 0; r < G; ++r) {
#pragma unroll
          for (int s = 0; s < kSteps; ++s)
            if (G > 1 && (decltype(full)::value || s < nv)) contract(s, r);
          const int slot = sm.slot[2 * r + sub];
          store_part<(G >= 4)>(a, wi, slot, acc[r], r, wv, lane);
          if (wv == r) {   // wave-uniform: the sums of the groups are shared out
            const f32x4 lw = *(const f32x4*)sm.ls[r][lane];
            const float total = row_sum4((lw[0] + lw[1]) + (lw[2] + lw[3]));
            if (g == 0 && 2 * r + sub < wi.n_tok)
              *(f32x2*)(a.part_ml + ((size_t)slot * kHeads + (n & 7)) * 4) = (f32x2){m[r], total};
          }
        }
      };
      if (G > 1 && nv == kSteps)
        finish(std::true_type());
      else
        finish(std::false_type());
    }
  };
  if constexpr (kSteps == 4)
    for (int round = 0; round + 1 < rounds; ++round) round_body(round, std::false_type());
  round_body(kSteps == 4 ? rounds - 1 : 0, std::true_type());
}

// Own phase of an item whose history was empty before the step (an action chunk): up to eight
// tokens whose keys are this step's new rows.  With the append folded in they are read from
// k_new / v_new, and the pool receives them from the merge launch of the same layer.  A split is one 32-key step
// or a few, so the wavefronts share the rows out, not the keys: wavefront w computes the logits
// and P of tokens 2w and 2w+1, with the K operands brought in by all four through LDS, and contracts
// all tokens' P for its 64 dims as in `attend`.  (Each wavefront by itself, all of K, Q and V in its
// own registers and no barrier, waits for four times the loads: 4.3 us until the logits are there
// against 1.8 us for a single wavefront.)
// Every sum is taken in the order of `attend`, rounds of 128 keys included, so that a folded
// append and a separate one give the same bits.  kOneStep: the split is one step, and everything
// it needs is requested at once; otherwise a step's operands are requested when it is their turn.
// kRows: the keys are rows of k_new / v_new (row0 + own position); otherwise (the append went
// before, one step only) they are read from the pages.  kG: groups of two tokens; every wavefront
// scales and stores its 64 dims of all of them, one after the other, which is what a tile ends with.
template <bool kOneStep, bool kRows, int kG>
__device__ __forceinline__ void attend_fresh(const AttnArgs& early_args, const WorkItem& wi, WorkLds& sm,
                                             const int row0) {
  AttnArgs a = early_args;
  static_assert(kOneStep || kRows, "several steps from pages go through attend");
  constexpr int kSteps = kOneStep ? 1 : 4;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, g = lane >> 4, h = n & 7, sub = n >> 3;
  const float ninf = -__builtin_inff();
  const float sl2 = log2_scale(a);
  const int nsteps = (wi.kv_end - wi.kv_begin + 31) >> 5, last = wi.kv_end - 1;
  const uint16_t* kn = (const uint16_t*)a.k_new + (size_t)row0 * kDim + 64 * wv + 8 * g;
  const uint16_t* vn = (const uint16_t*)a.v_new + (size_t)row0 * kDim + 64 * wv + 4 * n;
  const int blk_a = wi.pages[0], blk_b = wi.pages[1];
  const char* __restrict__ pages = (const char*)a.layer_base;
  u32x4 (*ks)[64] = &sm.q[0][0];   // K operands of the step (the query rows stay in registers)

  u32x4 kr[4], qf[8], vpage[4];
  u32x2 vr[8];   // [key]: dims 64w+4n..+3 of this lane's eight keys, as they lie in the row
  // this wavefront's quarter of the step's K operands: dims 64w..64w+63.  Positions at or beyond
  // the split's end re-read its last row and are masked.
  auto load_k = [&](const int s) {
    if constexpr (!kRows) {
      const char* p = pages + (size_t)(sub ? blk_b : blk_a) * kBlockBytes + (g * 8 + h) * 16;
#pragma unroll
      for (int i = 0; i < 4; ++i) kr[i] = *(const u32x4*)(p + (4 * wv + i) * 512);
      return;
    }
    const int pos = wi.kv_begin + 32 * s + 16 * sub + h;
    const uint16_t* r0 = kn + (size_t)min(pos, last) * kDim;
    const uint16_t* r1 = kn + (size_t)min(pos + 8, last) * kDim;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      kr[2 * j] = *(const u32x4*)(r0 + 32 * j);
      kr[2 * j + 1] = *(const u32x4*)(r1 + 32 * j);
    }
  };
  auto load_v = [&](const int s) {
    if constexpr (!kRows) {
      const char* p = pages + (size_t)((g >> 1) ? blk_b : blk_a) * kBlockBytes + kPageBytes +
                      v_chunk_offset(wv, 0, g & 1, n);
#pragma unroll
      for (int c = 0; c < 4; ++c) vpage[c] = *(const u32x4*)(p + c * 512);
      return;
    }
    const int pos = wi.kv_begin + 32 * s + 16 * (g >> 1) + 4 * (g & 1);
#pragma unroll
    for (int e = 0; e < 8; ++e)
      vr[e] = *(const u32x2*)(vn + (size_t)min(pos + (e < 4 ? e : e + 4), last) * kDim);
  };
  if constexpr (kOneStep) load_k(0);
  {   // wavefronts past the item's tokens hold its last token's rows and store nothing
    const char* qrow = (const char*)a.q + ((size_t)token_of(wi, wv, sub) * kHeads + h) * (kDim * 2);
#pragma unroll
    for (int j = 0; j < 8; ++j) qf[j] = *(const u32x4*)(qrow + j * 64 + g * 16);
  }
  const int slot_req = request_slot<kMaxGroups>(a, wi, lane);
  if constexpr (kOneStep) load_v(0);
  __builtin_amdgcn_sched_barrier(0);
  take_late(a);
#pragma unroll
  for (int j = 0; j < 8; ++j) qf[j] = query_sign(a, qf[j]);
  float m_own = ninf, l[4] = {0.f, 0.f, 0.f, 0.f};   // of this wavefront's row n
  f32x4 acc[kG][4];
#pragma unroll
  for (int r = 0; r < kG; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[r][c] = (f32x4){0.f, 0.f, 0.f, 0.f};
  for (int first = 0; first < (kOneStep ? 1 : nsteps); first += 4) {
    f32x4 s0[kSteps], s1[kSteps];
    float mx = ninf;
#pragma unroll
    for (int s = 0; s < kSteps; ++s)
      if (kOneStep || first + s < nsteps) {
        if constexpr (!kOneStep) {
          __syncthreads();   // the previous step's operands are used up, the previous round's P too
          load_k(first + s);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) ks[4 * wv + i][lane] = kr[i];
        if (kOneStep || s == 0)
          if (threadIdx.x < 8) sm.slot[lane] = slot_req + wi.part_idx;
        __syncthreads();
        s0[s] = s1[s] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          s0[s] = mfma16(ks[2 * j][lane], qf[j], s0[s]);
          s1[s] = mfma16(ks[2 * j + 1][lane], qf[j], s1[s]);
        }
        const int pos = wi.kv_begin + 32 * (first + s);
        const int end = min(wi.kv_end, wi.q0 + 2 * wv + sub + 1) - (pos + 16 * (g >> 1) + 4 * (g & 1));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s0[s][e] = e < end ? s0[s][e] : ninf;
          s1[s][e] = 8 + e < end ? s1[s][e] : ninf;
        }
        mx = fmaxf(mx, row_max4(row_max8(s0[s], s1[s]) * sl2));
      }
    const bool up = mx > m_own + kGrow;
    const float alpha = up ? fast_exp2(m_own - mx) : 1.f;
    m_own = up ? mx : m_own;
    if constexpr (!kOneStep) {
#pragma unroll
      for (int s = 0; s < 4; ++s) l[s] = rescaled(l[s], alpha);
      if (g == 0) sm.mx[wv][n][0] = alpha;
    }
#pragma unroll
    for (int s = 0; s < kSteps; ++s)
      if (kOneStep || first + s < nsteps) {
        u32x4 hi, lo;
        l[s] += softmax_weights(s0[s], s1[s], sl2, (m_own == ninf) ? 0.f : m_own, hi, lo);
        sm.p[s][wv][0][lane] = hi;
        sm.p[s][wv][1][lane] = lo;
      }
    __syncthreads();
    if constexpr (!kOneStep) {
#pragma unroll
      for (int r = 0; r < kG; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[r][c] *= sm.mx[r][n][0];
    }
#pragma unroll
    for (int s = 0; s < kSteps; ++s)
      if (kOneStep || first + s < nsteps) {
        if constexpr (!kOneStep) load_v(first + s);
        const u32x4 mask = value_mask(wi.kv_end - (wi.kv_begin + 32 * (first + s)), g);
        u32x4 v[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          if constexpr (kRows) {   // dim 64w+4n+c: halfword c of every key
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const uint32_t x = vr[2 * i][c >> 1], y = vr[2 * i + 1][c >> 1];
              v[c][i] = (c & 1) ? ((x >> 16) | (y & 0xffff0000u)) : ((x & 0xffffu) | (y << 16));
            }
          } else {
            v[c] = vpage[c];
          }
          v[c] &= mask;
        }
#pragma unroll
        for (int r = 0; r < kG; ++r) {
          const u32x4 hi = sm.p[s][r][0][lane], lo = sm.p[s][r][1][lane];
#pragma unroll
          for (int c = 0; c < 4; ++c) acc[r][c] = mfma16(v[c], hi, acc[r][c]);
#pragma unroll
          for (int c = 0; c < 4; ++c) acc[r][c] = mfma16(v[c], lo, acc[r][c]);
        }
      }
  }
  const float total = row_sum4((l[0] + l[1]) + (l[2] + l[3]));
  const int own_slot = sm.slot[2 * wv + sub];
  if (g == 0 && 2 * wv + sub < wi.n_tok) {
    *(f32x2*)(a.part_ml + ((size_t)own_slot * kHeads + h) * 4) = (f32x2){m_own, total};
  }
#pragma unroll
  for (int r = 0; r < kG; ++r) store_part<(kG >= 4)>(a, wi, sm.slot[2 * r + sub], acc[r], r, wv, lane);
}

template <bool kRows>
__device__ __forceinline__ void attend_fresh_width(const AttnArgs& a, const WorkItem& wi, WorkLds& sm,
                                                   const int row0) {
  if (wi.n_tok <= 2)
    attend_fresh<true, kRows, 1>(a, wi, sm, row0);
  else if (wi.n_tok <= 4)
    attend_fresh<true, kRows, 2>(a, wi, sm, row0);
  else
    attend_fresh<true, kRows, 4>(a, wi, sm, row0);
}

__device__ __forceinline__ void attend_fresh_any(const AttnArgs& a, const WorkItem& wi, WorkLds& sm,
                                                 const int row0) {
  if (wi.kv_end - wi.kv_begin <= 32)
    attend_fresh_width<true>(a, wi, sm, row0);
  else if (wi.n_tok <= 4)
    attend_fresh<false, true, 2>(a, wi, sm, row0);
  else
    attend_fresh<false, true, 4>(a, wi, sm, row0);
}

// The narrowest is tested last, and with it the four-step instance that every decode step runs: the compiler
// lays the instance that is tested last out first and the widest at the kernel's end.  With the narrowest tested first
// and laid out last a launch whose code has left the caches (other kernels and a read of 512 MB in front of every
// launch) took, one request on 832 tokens 7.3-7.5 us, now 6.9-7.1, three 7.1-7.2 / 7.0, one with a chunk 7.6-7.8 / 7.3-7.5;
// larger launches and launches that follow each other within 1 %.  Where code lies is worth that much for no reason that
// shows in it: the whole kernel 4 KiB further on took 0.2 us more.
__device__ __forceinline__ void attend_shared(const AttnArgs& a, const WorkItem& wi, WorkLds& sm) {
  const bool few_keys = wi.kv_end - wi.kv_begin <= 64;
  if (wi.n_tok > 4)
    attend<4, false, false, 4>(a, wi, sm);   // bound by its products and stores: no faster with half the loads
  else if (wi.n_tok > 2)
    few_keys ? attend<2, false, false, 2>(a, wi, sm) : attend<2, false, false, 4>(a, wi, sm);
  else
    few_keys ? attend<1, false, false, 2>(a, wi, sm) : attend<1, false, false, 4>(a, wi, sm);
}

// What the first loads need is preloaded into scalar registers (all 14 words there are; see build.py).  The rest is
// read from the argument segment once those loads are on their way (take_late): every workgroup of a launch
// reads that segment at the same time, and in front of the first loads it cost, us per layer, 50 queries + one
// request 7.81 / 7.58, a chunk on 100 tokens 7.31 / 7.04, three requests 6.70 / 6.57, four chunks on 832 tokens 11.39 /
// 11.22, one request 6.31 / 6.26, 64 requests and two chunks 22.29 / 22.18, 256 requests 71.6 / 71.8.
// On a page of its own start: 768 bytes further on, because a kernel in front had grown, the same code took
// 7.4-7.6 us instead of 7.0-7.2 in a cold launch of one request, and 19.8-20.1 instead of 19.3-19.5 in
// repeated ones of 64 requests and two chunks.  Multiples of 8, 16 and 32 KiB are no better.
__global__ __attribute__((aligned(4096))) __launch_bounds__(256, 2) void attn_kernel(
    const int32_t* work, const void* q, const void* layer_base, const void* k_new, const void* v_new,
    const int32_t* d_slots, const int32_t part_off, const float scale, const LateArgs) {
  __shared__ WorkLds sm;
  AttnArgs a;
  a.q = q;
  a.layer_base = layer_base;
  a.part_off = work + part_off;
  a.scale = scale;
  a.k_new = k_new;
  a.v_new = v_new;
  a.d_slots = d_slots;
  WorkItem wi;
  wi.rec = (DescPtr)work + (size_t)blockIdx.x * kWorkWords;
  const i32x8 head = ((DescPtr8)wi.rec)[0];
  wi.toks = ((DescPtr8)wi.rec)[1];
  wi.pages = ((DescPtr8)wi.rec)[2];
  // wanted here, in one go, and not one after the other where they are used first
  asm volatile("" ::"s"(head), "s"(wi.toks), "s"(wi.pages));
  wi.n_tok = head[W_N_TOK];
  wi.tbl_off = head[W_TBL_OFF];
  wi.kv_begin = head[W_KV_BEGIN];
  wi.kv_end = head[W_KV_END];
  wi.q0 = head[W_CAUSAL_Q0];
  wi.part_idx = head[W_PART_IDX];
  const int path_word = head[W_PATH];
  if ((path_word & kPathMask) == PATH_NOOP) return;   // padding record
  if (path_word & kPathAppends)                       // one or two tokens on their own pages
    path_word & kPathOnce ? attend<1, true, true, 4>(a, wi, sm) : attend<1, true, false, 4>(a, wi, sm);
  else if (a.k_new && (path_word & kPathFresh))
    attend_fresh_any(a, wi, sm, path_word >> kPathRowShift);
  else if ((path_word & kPathFresh) && wi.kv_end - wi.kv_begin <= 32)
    attend_fresh_width<false>(a, wi, sm, 0);
  else
    attend_shared(a, wi, sm);
}
// Where the argument segment holds a kernel's last argument: each lies at the next multiple of its alignment.
template <class Kernel>
struct Params;
template <class... P>
struct Params<void (*)(P...)> {
  using Last = std::tuple_element_t<sizeof...(P) - 1, std::tuple<P...>>;
  static constexpr size_t offset_of_last() {
    constexpr size_t n = sizeof...(P), size[n] = {sizeof(P)...}, align[n] = {alignof(P)...};
    size_t at = 0;
    for (size_t i = 0; i + 1 < n; ++i) at = (at + align[i] - 1) / align[i] * align[i] + size[i];
    return (at + align[n - 1] - 1) / align[n - 1] * align[n - 1];
  }
};
using AttnParams = Params<decltype(&attn_kernel)>;
static_assert(std::is_same_v<AttnParams::Last, LateArgs> && AttnParams::offset_of_last() == kLateOffset,
              "take_late reads attn_kernel's last argument at kLateOffset");

// ------------------------------------------------------------------------------------------
// merge of a query token's partials (log-sum-exp rule).  One wavefront per token and head, which has
// every load of the first sixteen partials in flight at once.
// (A merge fused into attn_kernel by "last arriver merges" was built twice and measured: with
// device-scope fences every workgroup pays a whole-L2 write-back + invalidate (165 us per
// launch); with scoped write-through stores and no fences it is correct and fence-free, but the
// tile workgroups finish last and then merge their eight tokens serially (53 us).  Hence its own
// kernel.)
// ------------------------------------------------------------------------------------------
constexpr int kMergeAhead = 16;       // partials whose loads are all issued before anything is used
struct MergeArgs {
  const uint16_t* part_acc;
  const float* part_ml;
  void* out;
  float* lse;
  const int32_t *n_parts, *part_off;
};
constexpr int kRowBcast0 = 0x150;     // DPP: all lanes of each 16 get the value of lane 0 (+ u: lane u)

// largest value / sum of a row of 16 lanes, in all of them
__device__ __forceinline__ float lanes16_max(float x) {
  x = fmaxf(x, dpp_row_ror<8>(x));
  x = fmaxf(x, dpp_row_ror<4>(x));
  x = fmaxf(x, dpp_row_ror<2>(x));
  return fmaxf(x, dpp_row_ror<1>(x));
}
__device__ __forceinline__ float lanes16_sum(float x) {
  x += dpp_row_ror<8>(x);
  x += dpp_row_ror<4>(x);
  x += dpp_row_ror<2>(x);
  return x + dpp_row_ror<1>(x);
}

// Bound by the round trip of its loads, by their bytes where tokens are many (400 tokens of 9 split results:
// 14.7 MB).  Lane 16q + i owns dims 64q + 4i..+3 of the output, and, for the weights, split result i of every
// sixteen in the 64 dims q, whose exponent it applies: sixteen weights take one exponential per wavefront, and a
// weight reaches its 16 lanes by a DPP broadcast.  (With a workgroup per token, eight dims per thread and every
// weight computed by every thread, the sums of nine split results alone took 0.7 us of a wavefront.  Layer of
// a decode step 6.80 -> 6.36 us, of 50 queries + one request 8.37 -> 7.88, of three requests 7.37 -> 6.77, of 78 queries
// with up to 15 split results 12.8 -> 11.9, of 64 requests and two chunks on 2048 tokens 23.6 -> 23.1.)
// They are read here and never again, hence the non-temporal hint (50 queries + one request 8.22 -> 8.12 us,
// 64 requests and two chunks 23.2 -> 22.8; on (m, l) too: 2 % slower).
// kAhead: split results whose loads are issued before anything is used, np rounded up to a multiple of four
// or the most: an instance for each, so that the first wait is for (m, l) only (loads under conditions are
// all waited for where the conditions meet; three requests 6.96 us a layer, now 6.77).
template <int kAhead>
__device__ __forceinline__ void merge_head(const MergeArgs& a, const size_t base, const int np, const int tok,
                                           const int h, const int lane) {
  const int i = lane & 15, q = lane >> 4;
  // wave-uniform; a lane adds 32 bits to them
  const char* ml = (const char*)(a.part_ml + (base * kHeads + h) * 4);
  const char* acc = (const char*)(a.part_acc + (base * kHeads + h) * kDim);
  constexpr uint32_t kMlStride = kHeads * 4 * sizeof(float), kAccStride = kHeads * kDim * sizeof(uint16_t);
  const float ninf = -__builtin_inff();
  u32x2 x[kAhead];
  // (m, l, exponents of the 64-dim parts, -) of this lane's split result; past the end the last one's
  auto load_ml = [&](const int p0) {
    return *(const f32x4*)(ml + (uint32_t)min(p0 + i, np - 1) * kMlStride);
  };
  auto load_x = [&](const int p0) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
      x[u] = __builtin_nontemporal_load((const u32x2*)(acc + (size_t)min(p0 + u, np - 1) * kAccStride + (uint32_t)lane * 8u));
  };
  f32x4 w = load_ml(0);
  load_x(0);
  float big = w[0];
  if constexpr (kAhead == kMergeAhead)
    for (int p0 = kAhead; p0 < np; p0 += kAhead)
      big = fmaxf(big, load_ml(p0)[0]);
  big = lanes16_max(big);
  float total = 0.f, o[4] = {0.f, 0.f, 0.f, 0.f};
  auto add = [&](const int p0) {
    const bool live = p0 + i < np && w[0] != ninf;
    const float wgt = live ? fast_exp2(w[0] - big) : 0.f;
    total += wgt * (live ? w[1] : 0.f);
    const int ex = (int32_t)(__float_as_uint(w[2]) << (24 - 8 * q)) >> 24;   // signed byte q
    const float ws = __builtin_amdgcn_ldexpf(wgt, ex - 14);
    static_for<kAhead>([&](auto u) {
      const float wu = __uint_as_float(
          __builtin_amdgcn_update_dpp(0, __float_as_uint(ws), kRowBcast0 + u.value, 0xf, 0xf, false));
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        float lo, hi;
        unpack_f16(x[u.value][k], lo, hi);
        o[2 * k] = __builtin_fmaf(wu, lo, o[2 * k]);
        o[2 * k + 1] = __builtin_fmaf(wu, hi, o[2 * k + 1]);
      }
    });
  };
  add(0);
  if constexpr (kAhead == kMergeAhead)
    for (int p0 = kAhead; p0 < np; p0 += kAhead) {
      w = load_ml(p0);
      load_x(p0);
      add(p0);
    }
  total = lanes16_sum(total);
  const float inv = 1.f / total;
  const u32x2 packed = {pack_bf16(o[0] * inv, o[1] * inv), pack_bf16(o[2] * inv, o[3] * inv)};
  *(u32x2*)((uint16_t*)a.out + ((size_t)tok * kHeads + h) * kDim + 4 * lane) = packed;
  if (a.lse && lane == 0)
    a.lse[(size_t)tok * kHeads + h] = (big + __builtin_amdgcn_logf(total)) * 0.6931471805599453f;
}
template <int kBlockHeads>
__device__ __forceinline__ void merge_block(const MergeArgs& a, const int block) {
  constexpr int kBlocks = kHeads / kBlockHeads;
  const int tok = block / kBlocks, lane = threadIdx.x & 63;
  const int h = kBlockHeads * (block % kBlocks) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int np = ((DescPtr)a.n_parts)[tok];
  const size_t base = (size_t)((DescPtr)a.part_off)[tok];
  if (np <= 4)
    merge_head<4>(a, base, np, tok, h, lane);
  else if (np <= 8)
    merge_head<8>(a, base, np, tok, h, lane);
  else if (np <= 12)
    merge_head<12>(a, base, np, tok, h, lane);
  else
    merge_head<kMergeAhead>(a, base, np, tok, h, lane);
}

// Everything a merge workgroup needs comes preloaded in scalar registers (13 of the 14 there are; see build.py):
// the argument segment is memory that every workgroup of a launch would read at once, in front of its first load.
// us per layer with the segment / preloaded: 50 queries + one request 8.02 / 7.81, eight requests and a chunk 8.92 /
// 8.76, three requests 6.80 / 6.65, eight chunks on 832 tokens 16.82 / 16.61, 64 requests and two chunks 22.66 / 22.40, one
// request (two workgroups) 6.33 / 6.36, eight chunks on 2048 22.44 / 22.49.
#define OXY_MERGE_PARAMS                                                                              \
  const uint16_t *part_acc, const float *part_ml, void *out, float *lse, const int32_t *n_parts, \
      const int32_t *part_off, const int32_t n_q
template <int kBlockHeads>
__global__ __launch_bounds__(64 * kBlockHeads) void merge_kernel(OXY_MERGE_PARAMS) {
  merge_block<kBlockHeads>({part_acc, part_ml, out, lse, n_parts, part_off}, blockIdx.x);
}

// merge of one layer and, in the same launch, an append that touches other memory than the
// merge: the next layer's new rows (cross-layer fusion), or this layer's rows of the items whose
// tiles read their keys from k_new / v_new (nx.runs names them, a block of a table each).  256 threads append.
template <int kBlockHeads>
__global__ __launch_bounds__(64 * kBlockHeads) void merge_append_kernel(OXY_MERGE_PARAMS, const AppendArgs nx) {
  __shared__ PageLds sm;
  const int n_merge = kHeads / kBlockHeads * n_q, i = (int)blockIdx.x - n_merge;
  if (i < 0) {
    merge_block<kBlockHeads>({part_acc, part_ml, out, lse, n_parts, part_off}, blockIdx.x);
    return;
  }
  if (threadIdx.x >= 256) return;   // whole wavefronts: a barrier waits for those of its workgroup that have not ended
  const int run = nx.runs ? nx.runs[i] : i << 4;
  const int tok = run >> 4, slot = nx.d_slots[tok];
  const uint16_t* k_row = (const uint16_t*)nx.k_new + (size_t)tok * kDim;
  const uint16_t* v_row = (const uint16_t*)nx.v_new + (size_t)tok * kDim;
  if (nx.runs)   // a row each: 18 layers of 50 queries + one request 167.2 us instead of 163.6
    append_rows(k_row, v_row, 0, (run & 15) + 1, (char*)nx.layer_base + (size_t)(slot >> 4) * kBlockBytes,
                sm, threadIdx.x);
  else
    append_row(k_row, v_row, slot, (char*)nx.layer_base, threadIdx.x);
}

hipError_t launch_attention_work(const AttnArgs& a, hipStream_t s, hipEvent_t start,
                                 hipEvent_t stop) {
  if (a.n_work <= 0 || a.n_q <= 0) return hipErrorInvalidValue;
  const LateArgs late = {a.part_acc, a.part_ml, a.tables, a.write_through};
  const int32_t part_off = (int32_t)(a.part_off - a.work);   // of one descriptor
  if (start || stop)
    hipExtLaunchKernelGGL(attn_kernel, dim3(a.n_work), dim3(256), 0, s, start, stop, 0, a.work, a.q, a.layer_base,
                          a.k_new, a.v_new, a.d_slots, part_off, a.scale, late);
  else
    attn_kernel<<<a.n_work, 256, 0, s>>>(a.work, a.q, a.layer_base, a.k_new, a.v_new, a.d_slots, part_off, a.scale,
                                         late);
  return hipGetLastError();
}

namespace {
template <int kBlockHeads>
void launch_merge(const AttnArgs& a, const AppendArgs* next, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  const bool timed = start || stop, appends = next && next->n_blocks > 0;
  const dim3 grid(kHeads / kBlockHeads * a.n_q + (appends ? next->n_blocks : 0)), block(64 * kBlockHeads);
  const auto launch = [&](auto kernel, auto... more) {
    if (timed)
      hipExtLaunchKernelGGL(kernel, grid, block, 0, s, start, stop, 0, a.part_acc, a.part_ml, a.out, a.lse,
                            a.n_parts, a.part_off, a.n_q, more...);
    else
      kernel<<<grid, block, 0, s>>>(a.part_acc, a.part_ml, a.out, a.lse, a.n_parts, a.part_off,
                                    a.n_q, more...);
  };
  if (appends)
    launch(merge_append_kernel<kBlockHeads>, *next);
  else
    launch(merge_kernel<kBlockHeads>);
}
}  // namespace

hipError_t launch_merge_append(const AttnArgs& a, const AppendArgs* next, hipStream_t s,
                               hipEvent_t start, hipEvent_t stop) {
  if (a.n_q <= 0) return hipErrorInvalidValue;
  if (merge_heads(a.n_q) == kHeads)
    launch_merge<kHeads>(a, next, s, start, stop);
  else
    launch_merge<kHeads / 2>(a, next, s, start, stop);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Split results in static device memory, for callers that cannot allocate (see
// oxy_mixed_attention_static in oxy.h).  Every GPU the library runs on holds its own copy of
// the array, at its own address, until the process ends; that address is looked up once per
// device, with the device current, and is what host code passes on from then.
// ------------------------------------------------------------------------------------------
constexpr size_t kStaticAccBytes = (size_t)kStaticMaxPartials * kHeads * kDim * sizeof(uint16_t);
constexpr size_t kStaticMlBytes = (size_t)kStaticMaxPartials * kHeads * 4 * sizeof(float);
static __device__ __align__(256) unsigned char scratch[kStaticAccBytes + kStaticMlBytes];

hipError_t static_scratch(uint16_t** part_acc, float** part_ml) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* ptr_of_device[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr_of_device[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    ptr_of_device[dev] = ptr;
  }
  *part_acc = (uint16_t*)ptr_of_device[dev];
  *part_ml = (float*)((char*)ptr_of_device[dev] + kStaticAccBytes);
  return hipSuccess;
}

hipError_t launch_attention(const AttnArgs& a, hipStream_t s) {
  hipError_t e = launch_attention_work(a, s);
  if (e != hipSuccess) return e;
  return launch_merge_append(a, nullptr, s);
}

}  // namespace oxy

// Internal helpers shared by the library's translation units (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdarg.h>
#include <stddef.h>
#include <atomic>
#include "usp.h"

namespace usp {

// thread-local message behind usp_last_error()
void set_error(const char* fmt, ...);
void clear_error();

#define USP_CHECK_ARG(cond, ...)                       \
  do {                                                 \
    if (!(cond)) {                                     \
      ::usp::set_error(__VA_ARGS__);                   \
      return USP_ERR_INVALID_ARG;                      \
    }                                                  \
  } while (0)

#define USP_CHECK_HIP(expr)                                                    \
  do {                                                                         \
    hipError_t e_ = (expr);                                                    \
    if (e_ != hipSuccess) {                                                    \
      ::usp::set_error("%s failed: %s", #expr, hipGetErrorString(e_));         \
      return USP_ERR_HIP;                                                      \
    }                                                                          \
  } while (0)

static inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// ---- device-side scalar type helpers ---------------------------------------------------
typedef uint16_t bf16_t;  // raw bf16 bits

__device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// fp32 -> bf16, round to nearest even (finite inputs; NaN stays NaN via the quiet bit)
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

// two fp32 -> packed bf16x2 (low half = a), hardware RNE convert
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  typedef __bf16 bf16x2_v __attribute__((ext_vector_type(2)));
  typedef float f32x2_v __attribute__((ext_vector_type(2)));
  f32x2_v f = {a, b};
  bf16x2_v r = __builtin_convertvector(f, bf16x2_v);
  return *reinterpret_cast<uint32_t*>(&r);
}

// ---- kernel launchers implemented in the .hip files ------------------------------------
// Row visiting order of the mapped FP8 kernels: row id -> (i0..i3), i3 fastest -> two offsets.
struct RowMap {
  uint32_t n1, n2, n3;       // extents of i1..i3 (i0 is what is left)
  int64_t src[4], dst[4];
};
usp_status launch_fp8_quant_mapped(const RowMap& m, int64_t rows, int64_t cols, int in_dt, const void* x,
                                   uint8_t* q, float* scales, hipStream_t st);
usp_status launch_fp8_dequant_mapped(const RowMap& m, int64_t rows, int64_t cols, int out_dt, const uint8_t* q,
                                     const float* scales, void* y, hipStream_t st);
usp_status launch_fp8_quant(int64_t rows, int64_t cols, int in_dt, const void* x, uint8_t* q,
                            float* scales, hipStream_t st);
usp_status launch_fp8_dequant(int64_t rows, int64_t cols, int out_dt, const uint8_t* q,
                              const float* scales, void* y, hipStream_t st);
usp_status launch_lse_merge(int64_t rows, int d, int dt, const void* o1, const float* lse1,
                            const void* o2, const float* lse2, void* o_out, float* lse_out,
                            hipStream_t st);

// One attention step over one KV chunk.
struct AttnStep {
  int B, H, d, Sq, Sc;
  int qo_dtype;              // USP_F32 / USP_BF16
  int kv_dtype;              // USP_F32 / USP_BF16 / USP_FP8_E4M3FN
  const void* q;
  const void* k;
  const void* v;
  const float* k_scale;      // FP8 only: [B,H,Sc]
  const float* v_scale;
  const uint8_t* key_mask;   // [B,Sc] or null
  int64_t qs[3], ks[3], os[3];
  float scale;
  // merge-in-epilogue: mode 0 = write (O_r, lse_r) to out/lse in qo_dtype (single chunk or unfused)
  //                    mode 1 = first of several chunks: write fp32 O to acc, lse to lse
  //                    mode 2 = middle chunk: merge with (acc, lse), write back fp32
  //                    mode 3 = last chunk: merge with (acc, lse), write out in qo_dtype and lse
  int mode;
  int variant;               // matrix-core kernels: 0 = pick by grid size, 1 = 256-query work-groups, 2 = key-split, 4 = mixed
  int mix_halves;            // mixed launch: blocks per XCD run as two key-split halves (set by the launcher)
  int half_d;                // matrix-core kernels: d = 64: the rows of Q, K, V, `out` and acc are 64 wide (128 bytes), the kernels
                             // run their head-dimension loops over half the slices
  float* acc;                // fp32 [B,H,Sq,d] dense carried O (modes 1-3)
  // mode 0 (general kernel: and one chunk): the keys of a query block are shared by `parts` work-groups (0 counts as 1), each
  // with its own range of tiles; their unnormalised O~ and (m in log2 units, l) per query are put together by a second launch
  int parts;
  float* part_o;             // fp32 [parts][B,H,Sq,d]
  float* part_ml;            // fp32 [parts][B,H,Sq][2]
  void* out;                 // qo_dtype by os strides (modes 0, 3)
  float* lse;                // fp32 [B,H,Sq] dense
  // Matrix-core kernels, FP8 K: per-(batch, head, 64-key tile) records of 64 floats, laid out
  // [B*H][tiles of the launch], filled by launch_attn_fp8_chunk_prepare on the same stream before the
  // attention launch or by the copy work-groups inside it
  float* ext;
  // Matrix-core kernels, several resident chunks in one launch (n_multi > 0): their 64-key tiles form one
  // stream in ring order and the running (O~, m, l) stays in registers from the first tile to the last,
  // which is the merge of section 3.4 applied tile by tile.  k, v, Sc and ks above are then unused.
  //
  // With `arrive` set the launch also plays the ring's transfers (Algorithm 2 inside one launch): its
  // first copy_wgs work-groups copy chunk c = 1, 2, .. from k_src / v_src (bytes each) into k / v, a
  // staging buffer of its own per chunk (each of copy_groups groups its own chunks), and count themselves on
  // arrive[c] when their share of chunk c is visible device-wide; an attention work-group waits for
  // arrive[c] == tag + copy_wgs / copy_groups before it loads the first tile of chunk c.  Dependencies only
  // point from the attention work-groups to the copy work-groups, which are dispatched first and wait
  // for nothing.
  //
  // multi_fp8: the sources are FP8 E4M3 chunks ([B,H,Sc,128] codes at k_src / v_src, per-(head, token)
  // scales at k_scale_src / v_scale_src; Algorithm 1 line 4 on arrival).  A copy work-group then
  // decodes while it copies: K's codes widened to bf16 as they are, V's multiplied by their scales,
  // and the per-tile records of the chunk (K's scales as per-key factors) written into `ext`.  Chunk 0 is
  // decoded by a launch of its own
  // (launch_attn_fp8_chunk_prepare) before the attention launch.
  struct Chunk {
    const void* k; const void* v; int64_t ks0, ks1; int Sc;
    const void* k_src; const void* v_src; int64_t bytes;
    const float* k_scale_src; const float* v_scale_src;
    const uint8_t* mask_src;   // key mask [B,Sc] of the chunk (nonzero = key takes part), or null
  };
  static constexpr int kMaxMulti = 16;
  int n_multi;
  int16_t multi_fp8;
  int16_t arrive_set;        // the counters have been set to `tag` by a launch in front of this one
  uint64_t* arrive;          // [kMaxMulti] counters, or null
  uint64_t tag;              // this launch's own (next_launch_tag), its lower 16 bits zero: a word whose upper bits differ is none of this
                             // launch's.  0 where a launch in front sets the counters in any case (multi_fp8)
  int16_t copy_groups;       // the copy work-groups fall into this many groups (copy_groups_of, set by the launcher)
  // what an attention work-group waits for on arrive[c], and for how long: the launcher sets the
  // count to copy_wgs / copy_groups plus arrive_need_extra and the poll limit to its default when arrive_polls is
  // 0.  Both exist so that a host-side test can make the bounded wait give up (a count that is never
  // reached, a short limit) with every kernel still running to its end.
  int16_t arrive_need_extra;
  int arrive_need;
  int arrive_polls;
  // Prefetch carried by this launch (Algorithm 2, the transfer of the next chunk): the last
  // copy_wgs work-groups of the grid copy the n_copy segments and exit; they are dispatched after
  // the attention work-groups, onto the CU slots those leave free.  The launcher fills copy_wgs (0 when n_copy == 0).
  struct CopySeg { const void* src; void* dst; int64_t bytes; };
  int n_copy;
  int copy_wgs;
  // set by the launcher, so that a work-group need not walk the chunk table first: work-groups of the grid, tiles of
  // the launch's stream, and whether some chunk has a key mask
  int grid_wgs;
  int tiles;
  int any_mask;
  Chunk chunk[kMaxMulti];
  CopySeg copy[4];
};
static_assert(sizeof(AttnStep) <= 4096, "AttnStep is passed by value as the kernels' only argument");
// touch_step has these lines on their way when a work-group begins
static_assert(offsetof(AttnStep, chunk) + sizeof(AttnStep::Chunk) <= 6 * 64, "one chunk lies in the lines that are touched");
// Copy work-groups that go with attn_wgs attention work-groups, one of which fits on a CU: the CUs the
// attention grid leaves free, as a multiple of 8 in [16, 64] (one work-group copied about 50 GB/s when this was chosen, with
// one batch of loads in flight; it has two now).
constexpr int kMostCopyWGs = 64;
inline int copy_wgs_beside(int attn_wgs) {
  const int n = (256 - attn_wgs % 256) / 8 * 8;
  return n < 16 ? 16 : (n > kMostCopyWGs ? kMostCopyWGs : n);
}
// Groups into which the copy work-groups of a launch over a ring fall, each with chunks of its own: a chunk is a
// chain of load, store, acknowledgement and count that takes 4 to 5 us however short it is, so short chunks travel
// side by side, up to eight, as long as that puts the first one off by no more than another 4 us (65 GB/s per
// work-group, as the copies were when this was chosen; `largest`: bytes read and written for the largest chunk; `later`: chunks that travel).
inline int copy_groups_of(int copy_wgs, int later, int64_t largest) {
  int g = 1;
  while (g < 8 && g < later && (double)(2 * g) * (double)largest <= 4.0 * 65e3 * copy_wgs) g *= 2;   // (copy_wgs is a multiple of 8)
  return g;
}
inline int prefetch_wg_count(const AttnStep& s, int attn_wgs) { return s.n_copy <= 0 ? 0 : copy_wgs_beside(attn_wgs); }
usp_status launch_attn_generic(const AttnStep& s, hipStream_t st);
// work-groups that share the keys of a query block in a launch of the general kernel over one chunk (AttnStep::parts)
int attn_generic_parts(bool f32, int B, int H, int Sq, int d, int keys);
usp_status launch_attn_mfma(const AttnStep& s, hipStream_t st);
bool attn_mfma_supported(const AttnStep& s);
// How the matrix-core kernels run a launch that finishes its result: variant as AttnStep::variant, and parts
struct AttnForm { int variant, parts; };
// The mixed launch of 256-query work-groups and key-split halves over `items` query blocks: all attention work-groups, the blocks of
// each XCD that are run as halves, and the copy work-groups behind them if the launch carries a transfer.  wgs = 0: not taken.
struct MixedGrid { int wgs, halves, copy_wgs; };
MixedGrid attn_mfma_mixed_grid(int items, bool forced, bool copies);
// What a launch over a ring moves while it computes: chunks that hold keys, bytes read and written for all
// but the first of them and for the largest of those, tiles of the last
struct RingTransfers { int chunks; int64_t bytes, largest, last_tiles; bool fp8; };
// ring: null for a launch over one chunk, and of that: decoded from FP8; some of its keys are dead (a mask, a ragged end); most: parts at most
AttnForm attn_mfma_form(int B, int H, int Sq, int d, int64_t tiles, const RingTransfers* ring, bool fp8, bool dead, int most);
// parts of the keys of a query block at most, of which a second launch holds all at once: matrix-core kernels, general kernel
constexpr int kMostParts = 16, kMostShares = 8;
// One launch over a ring: key-split or 256-query work-groups, and whether it is expected to beat a launch per chunk
struct RingForm { bool split, pays; };
RingForm attn_mfma_ring_form(int B, int H, int Sq, int d, int64_t tiles, int chunks, int variant, bool fp8);
// tiles a launch over several chunks takes if some of its keys are dead (a mask, a ragged chunk)
int64_t attn_mfma_max_dead_tiles();
// A value that no launch of this process has had, its lower 16 bits zero.  Of other processes' only by a chance of 2^-48 and for
// a word that is still as they left it.
uint64_t next_launch_tag();
// Is the stream being captured into a graph?  A launch that is replayed has the same tag every time, so the counters of the replay
// before have to be set back in front of it.
bool stream_is_capturing(hipStream_t st);
usp_status launch_attn_arrive_set(uint64_t* arrive, uint64_t tag, hipStream_t st);
// An FP8 chunk decoded by a launch of its own: bf16 K and V, and the records of its tiles.  (Less than 120 bytes: see PackedMap.)
struct Fp8Chunk {
  const void* k_src; const void* v_src;     // codes
  void* k; void* v;                         // bf16
  const float* k_scale_src; const float* v_scale_src;
  const uint8_t* mask_src;                  // or null
  float* ext;                               // records of the whole launch
  uint64_t* arrive;                         // arrival counters that this launch sets to zero, or null
  int Sc;
  int tile0, tiles;                         // the chunk's first tile, tiles of the whole launch
  int bh, H, ush;                           // (batch, head) pairs; log2 of the 8-code units per row
  float scale2;
  int threads;                              // of the launch
};
static_assert(sizeof(Fp8Chunk) <= 112, "a launch with more costs the host more");
// fills in the last five
usp_status launch_attn_fp8_chunk_prepare(Fp8Chunk* c, int B, int H, int d, float scale, hipStream_t st);

// More than 64 KB of dynamic LDS has to be allowed per kernel, and the setting belongs to the device
// that is current when it is made: once per (kernel, device ordinal below 64), every launch beyond.
template <void (*kKernel)(AttnStep)>
static hipError_t allow_large_lds(int bytes) {
  static std::atomic<uint64_t> done{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const bool tracked = dev >= 0 && dev < 64;
  if (tracked && ((done.load(std::memory_order_acquire) >> dev) & 1u) != 0) return hipSuccess;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(kKernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess && tracked) done.fetch_or((uint64_t)1 << dev, std::memory_order_release);
  return e;
}

// The route of a call with its full workspace, for tests: one launch over all chunks or a launch for each, whether
// that launch is key-split, and the work-groups that share the keys of a query block.  masked: some chunk comes
// with a key mask.
struct AttnRoute { bool one_launch, split; int parts; };
usp_status attn_route(const usp_attn_desc* desc, bool masked, AttnRoute* route);

// What usp_ring_attn_fwd does, with the knobs the ABI does not carry.
struct CallOptions {
  int arrive_need_extra = 0;  // see AttnStep (tests of the give-up path only)
  int arrive_polls = 0;
};
usp_status ring_attn_fwd_impl(const usp_attn_desc* desc, const void* q, const void* const* k_chunks,
                              const void* const* v_chunks, const float* const* k_scales,
                              const float* const* v_scales, const uint8_t* const* key_mask, void* out,
                              float* lse, void* workspace, size_t workspace_bytes, void* compute_stream,
                              void* copy_stream, const CallOptions& opt);

}  // namespace usp

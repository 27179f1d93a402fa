// Device-side transfers that ride in an attention launch (Algorithm 2: the transfer of chunk r+1
// overlaps the compute on chunk r).
//  * prefetch_copy: the next chunk into the idle one of two staging buffers, run by extra work-groups
//    of a per-chunk launch.  Stream order gives the two hazards for free: the launch that reads the
//    buffer starts after this one has ended, and the buffer's previous reader ended before this one
//    began.
//  * stream_chunks / stream_chunks_fp8: every later chunk of a ring into a buffer of its own, run by
//    the first work-groups of the one launch over the ring, each chunk published through an arrival
//    counter; the FP8 form decodes the chunk on the way (Algorithm 1 line 4).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "usp_common.h"

namespace usp {

// The kernel's argument lies in memory that a scalar load takes some 700 cycles to reach the first time: a word of each of
// its 64-byte lines up to the chunk table, all in flight together, so that no later use of a field waits for memory
// (they came one after another, line by line, and made a good part of the 4500 cycles in front of the first tile).
__device__ __forceinline__ void touch_step() {
  typedef const __attribute__((address_space(4))) uint32_t* words;
  const words p = (words)__builtin_amdgcn_kernarg_segment_ptr();
  static_assert(offsetof(AttnStep, chunk) > 4 * 64 && offsetof(AttnStep, chunk) <= 6 * 64, "lines of the step");
  asm volatile("" :: "s"(p[0]), "s"(p[16]), "s"(p[32]), "s"(p[48]), "s"(p[64]), "s"(p[80]));
}
// The chunk table, likewise
__device__ __forceinline__ void touch_chunks() {
  typedef const __attribute__((address_space(4))) uint32_t* words;
  const words p = (words)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(AttnStep, chunk) / 4;
  static_assert(sizeof(AttnStep::Chunk) * AttnStep::kMaxMulti == 22 * 64, "lines of the table");
  asm volatile("" :: "s"(p[0]), "s"(p[16]), "s"(p[32]), "s"(p[48]), "s"(p[64]), "s"(p[80]), "s"(p[96]), "s"(p[112]), "s"(p[128]), "s"(p[144]), "s"(p[160]));
  asm volatile("" :: "s"(p[176]), "s"(p[192]), "s"(p[208]), "s"(p[224]), "s"(p[240]), "s"(p[256]), "s"(p[272]), "s"(p[288]), "s"(p[304]), "s"(p[320]), "s"(p[336]));
}

__device__ __forceinline__ void prefetch_copy(const AttnStep& s, int wg, int tid, int nthr) {
  const int64_t stride = (int64_t)s.copy_wgs * nthr;
  const int64_t first = (int64_t)wg * nthr + tid;
  for (int c = 0; c < s.n_copy; ++c) {
    const unsigned char* src = (const unsigned char*)s.copy[c].src;
    unsigned char* dst = (unsigned char*)s.copy[c].dst;
    const int64_t bytes = s.copy[c].bytes;
    const uintptr_t both = (uintptr_t)src | (uintptr_t)dst;
    if ((both & 15) == 0) {
      const uint4* s4 = (const uint4*)src;
      uint4* d4 = (uint4*)dst;
      const int64_t n = bytes >> 4;
      int64_t i = first;
      for (; i + 3 * stride < n; i += 4 * stride) {   // four loads in flight per lane
        const uint4 a = s4[i], b = s4[i + stride], e = s4[i + 2 * stride], f = s4[i + 3 * stride];
        d4[i] = a; d4[i + stride] = b; d4[i + 2 * stride] = e; d4[i + 3 * stride] = f;
      }
      for (; i < n; i += stride) d4[i] = s4[i];
      for (int64_t j = (n << 4) + first; j < bytes; j += stride) dst[j] = src[j];
    } else if ((both & 3) == 0) {                     // per-token scales: 4-byte aligned only
      const uint32_t* s1 = (const uint32_t*)src;
      uint32_t* d1 = (uint32_t*)dst;
      const int64_t n = bytes >> 2;
      for (int64_t i = first; i < n; i += stride) d1[i] = s1[i];
      for (int64_t j = (n << 2) + first; j < bytes; j += stride) dst[j] = src[j];
    } else {
      for (int64_t j = first; j < bytes; j += stride) dst[j] = src[j];
    }
  }
}

// The transfers of a whole ring inside one launch: work-group wg of s.copy_wgs copies its share of
// chunk c = 1, 2, .. (of its group's chunks, see copy_groups_of) and then counts itself on s.arrive[c].
// The stores carry device scope (they are written through to where every XCD's loads find them; a fence
// would write back and invalidate the whole L2 under the attention work-groups), each thread waits until
// its own stores have been acknowledged, the work-group barrier collects the threads, and one thread
// publishes the count.
// The readers make no acquire of their own either: nothing reads a staging buffer or its records
// before their chunk's count is complete, and the launch starts with invalid caches, so no cache on
// the reading side can hold an older copy of those lines.
__device__ __forceinline__ void publish_chunk(int* counter, int tid) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's stores have been acknowledged (and none is moved past this)
  __syncthreads();
  if (tid == 0) __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Algorithm 1 line 4 for chunk c of a launch over FP8 chunks: unit `first`, first + stride, .. of the chunk
// (8 codes of K and of V each; then one key of the records).  The arithmetic is the dequantiser's: E4M3
// code -> fp32 (exact), times the scale in fp32, RNE to bf16; K keeps scale 1 and hands its scales to the
// records as per-key factors of the exponent.  A key that takes no part (masked, or past the end of the
// last tile) gets the plain factor instead of its scale's: its score is -inf by then and stays so under
// any positive finite factor.
template <bool kDeviceScope>
__device__ __forceinline__ void put_float(float* p, float v) {
  if (kDeviceScope) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}
__device__ __forceinline__ uint4 decode8_bf16(uint32_t w0, uint32_t w1, float sc) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  const f32x2_t a = __builtin_amdgcn_cvt_pk_f32_fp8((int)w0, false), b = __builtin_amdgcn_cvt_pk_f32_fp8((int)w0, true);
  const f32x2_t c = __builtin_amdgcn_cvt_pk_f32_fp8((int)w1, false), e = __builtin_amdgcn_cvt_pk_f32_fp8((int)w1, true);
  return make_uint4(pack_bf16x2(a.x * sc, a.y * sc), pack_bf16x2(b.x * sc, b.y * sc),
                    pack_bf16x2(c.x * sc, c.y * sc), pack_bf16x2(e.x * sc, e.y * sc));
}
template <bool kDeviceScope>
__device__ __forceinline__ void fp8_chunk_records(const AttnStep& s, int c, int64_t first, int64_t stride) {
  const AttnStep::Chunk& ch = s.chunk[c];
  int tile0 = 0, nt_total = 0;                          // first tile of the chunk, tiles of all chunks
  for (int i = 0; i < s.n_multi; ++i) {
    if (i < c) tile0 += (s.chunk[i].Sc + 63) / 64;
    nt_total += (s.chunk[i].Sc + 63) / 64;
  }
  const float scale2 = s.scale * 1.44269504088896340736f;
  const uint32_t ntc = (uint32_t)(ch.Sc + 63) / 64;
  const int64_t slots = (int64_t)s.B * s.H * ntc * 64;
  for (int64_t i = first; i < slots; i += stride) {
    const uint32_t t = (uint32_t)(i >> 6), bh = t / ntc, tile = t - bh * ntc;   // (2^32 tiles would be 32 TB of codes)
    const int key = (int)(tile * 64 + (uint32_t)(i & 63));
    const bool live = key < ch.Sc && (ch.mask_src == nullptr || ch.mask_src[(int64_t)(bh / s.H) * ch.Sc + key] != 0);
    const float f = live ? ch.k_scale_src[(int64_t)bh * ch.Sc + key] * scale2 : scale2;
    put_float<kDeviceScope>(s.ext + (((int64_t)bh * nt_total + tile0 + tile) << 6) + (i & 63), f);
  }
}
// A chunk decoded by a launch of its own.  A thread takes 8 codes at a time, so that a store instruction writes 1024
// consecutive bytes: with 16 codes and two stores each wrote every other 16 bytes.
__device__ __forceinline__ void fp8_chunk_prepare(const AttnStep& s, int c, int64_t first, int64_t stride) {
  const AttnStep::Chunk& ch = s.chunk[c];
  const int ush = s.d == 64 ? 3 : 4;                    // log2 of the 8-code units per row
  const uint2* kc = (const uint2*)ch.k_src;
  const uint2* vc = (const uint2*)ch.v_src;
  uint4* kd = (uint4*)ch.k;
  uint4* vd = (uint4*)ch.v;
  const int64_t units = ((int64_t)s.B * s.H * ch.Sc) << ush;
  int64_t u = first;
  for (; u + 3 * stride < units; u += 4 * stride) {     // the loads of four units in flight per lane
    uint2 a[4], b[4];
    float sc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) { a[i] = kc[u + i * stride]; b[i] = vc[u + i * stride]; sc[i] = ch.v_scale_src[(u + i * stride) >> ush]; }
#pragma unroll
    for (int i = 0; i < 4; ++i) { kd[u + i * stride] = decode8_bf16(a[i].x, a[i].y, 1.0f); vd[u + i * stride] = decode8_bf16(b[i].x, b[i].y, sc[i]); }
  }
  for (; u < units; u += stride) {
    const uint2 a = kc[u], b = vc[u];
    const float sc = ch.v_scale_src[u >> ush];
    kd[u] = decode8_bf16(a.x, a.y, 1.0f);
    vd[u] = decode8_bf16(b.x, b.y, sc);
  }
  fp8_chunk_records<false>(s, c, first, stride);
}
// ---- the copy work-groups of a launch over a ring ----
// They are few (the CUs that the attention leaves free) and the ring waits for them: a chunk of 24 heads x 1152 keys took
// 40 of them 21 us in bf16 and 24 in FP8, where the attention needs 15 for it.  So loads run two batches ahead of the
// stores, through registers, bounded by descriptors, so that no test and no tail stand between them; the stores are
// builtins, whose count the compiler knows (behind stores in inline asm it waited for their acknowledgement before the
// next batch could be used); and an FP8 thread takes 8 codes at a time, so that a store instruction writes whole lines
// (with 16 codes and two stores each wrote every other 16 bytes, straight through to memory).  That ring's calls
// with the transfers inside, inputs changing: bf16 84.5 -> 73 us, FP8 104 -> 82; B = 2, H = 12, Sq = 150, FP8, eight of 320
// keys 56 -> 50.
typedef uint32_t copy_u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t copy_u32x4 __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t CopyBuf;
constexpr int kCopyBatch = 2;          // units per thread and batch: 2, 3, 4 and 8 bring long chunks equally fast, and what a batch has past the end costs the address unit too
constexpr int kCopyDeviceScope = 16;   // cache policy of a buffer store: sc1
__device__ __forceinline__ CopyBuf copy_buffer(const void* p, int64_t bytes) {   // (what lies past the bytes loads as zeros, and is not stored)
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)(bytes < 0 ? 0 : bytes < 0x7fffffff ? bytes : 0x7fffffff), 0x00020000);
}
// Batches 0 .. n - 1 through `load(batch, buffer)` and `store(batch, buffer)`, buffer a constant 0, 1 or 2.  Loads of batches
// past the last are empty (their descriptors hold nothing): a branch around them would cost the others their distance, as
// the wait in front of a store has to be right for both ways.
template <class Load, class Store>
__device__ __forceinline__ void copy_pipeline(int n, Load load, Store store) {
  load(0, 0);
  load(1, 1);
  for (int i = 0; i < n; i += 3) {
    load(i + 2, 2);
    store(i, 0);
    if (i + 1 >= n) break;
    load(i + 3, 0);
    store(i + 1, 1);
    if (i + 2 >= n) break;
    load(i + 4, 1);
    store(i + 2, 2);
  }
}
// Chunk c of a launch over several FP8 chunks, decoded (fp8_chunk_prepare's arithmetic)
__device__ __forceinline__ void stream_chunk_fp8(const AttnStep& s, int c, int first, int stride) {
  constexpr int kU = kCopyBatch;                          // units of 8 codes of K and of V
  const AttnStep::Chunk& ch = s.chunk[c];
  const int ush = s.d == 64 ? 3 : 4;                      // log2 of the units per row
  const int64_t rows = (int64_t)s.B * s.H * ch.Sc, units = rows << ush;
  const int64_t span = (int64_t)stride * kU;              // (stride is a multiple of 512: a batch begins with a row)
  copy_u32x2 k[3][kU], v[3][kU];
  float sc[3][kU];
  copy_pipeline((int)((units + span - 1) / span),
      [&](int i, int buf) __attribute__((always_inline)) {
        const int64_t u0 = i * span;
        const CopyBuf kb = copy_buffer((const uint2*)ch.k_src + u0, (units - u0) * 8), vb = copy_buffer((const uint2*)ch.v_src + u0, (units - u0) * 8);
        const CopyBuf sb = copy_buffer(ch.v_scale_src + (u0 >> ush), (rows - (u0 >> ush)) * 4);
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const int at = first + u * stride;
          k[buf][u] = __builtin_amdgcn_raw_buffer_load_b64(kb, at * 8, 0, 0);
          v[buf][u] = __builtin_amdgcn_raw_buffer_load_b64(vb, at * 8, 0, 0);
          sc[buf][u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(sb, (at >> ush) * 4, 0, 0));
        }
      },
      [&](int i, int buf) __attribute__((always_inline)) {
        const int64_t u0 = i * span;
        const CopyBuf kd = copy_buffer((const uint4*)ch.k + u0, (units - u0) * 16), vd = copy_buffer((const uint4*)ch.v + u0, (units - u0) * 16);
        auto put = [](CopyBuf b, int off, const uint4& x) { __builtin_amdgcn_raw_buffer_store_b128(copy_u32x4{x.x, x.y, x.z, x.w}, b, off, 0, kCopyDeviceScope); };
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const int off = (first + u * stride) * 16;
          put(kd, off, decode8_bf16(k[buf][u][0], k[buf][u][1], 1.0f));
          put(vd, off, decode8_bf16(v[buf][u][0], v[buf][u][1], sc[buf][u]));
        }
      });
}
// Chunk c of a launch over several bf16 chunks
__device__ __forceinline__ void stream_chunk(const AttnStep& s, int c, int first, int stride) {
  constexpr int kU = kCopyBatch;                          // 16-byte units
  const int64_t bytes = s.chunk[c].bytes;                 // (the host passes 16-byte multiples, 16-byte aligned)
  const int64_t span = (int64_t)stride * kU * 16;
  const int per = (int)((bytes + span - 1) / span);       // batches of K, then of V
  copy_u32x4 r[3][kU];
  copy_pipeline(2 * per,
      [&](int i, int buf) __attribute__((always_inline)) {
        const int64_t at = (i < per ? i : i - per) * span;
        const CopyBuf b = copy_buffer((const char*)(i < per ? s.chunk[c].k_src : s.chunk[c].v_src) + at, bytes - at);
#pragma unroll
        for (int u = 0; u < kU; ++u) r[buf][u] = __builtin_amdgcn_raw_buffer_load_b128(b, (first + u * stride) * 16, 0, 0);
      },
      [&](int i, int buf) __attribute__((always_inline)) {
        const int64_t at = (i < per ? i : i - per) * span;
        const CopyBuf b = copy_buffer((const char*)(i < per ? s.chunk[c].k : s.chunk[c].v) + at, bytes - at);
#pragma unroll
        for (int u = 0; u < kU; ++u) __builtin_amdgcn_raw_buffer_store_b128(r[buf][u], b, (first + u * stride) * 16, 0, kCopyDeviceScope);
      });
}
// Copy work-group wg: its group's chunks, each counted when its stores have been acknowledged
template <bool kFp8>
__device__ __forceinline__ void stream_chunks(const AttnStep& s, int wg, int tid, int nthr) {
  const int groups = s.copy_groups;
  const int stride = s.copy_wgs / groups * nthr;
  const int first = wg / groups * nthr + tid;
  for (int c = 1 + wg % groups; c < s.n_multi; c += groups) {
    if (kFp8) {
      stream_chunk_fp8(s, c, first, stride);
      fp8_chunk_records<true>(s, c, first, stride);
    } else stream_chunk(s, c, first, stride);
    publish_chunk(s.arrive + c, tid);
  }
}

}  // namespace usp

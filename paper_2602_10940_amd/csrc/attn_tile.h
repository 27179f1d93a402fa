// Attention for every shape the bf16 d = 128 / 64 kernels do not take: fp32 inputs, other head
// dimensions (multiples of 8 up to 256), FP8 K/V with those.  fp32 arithmetic throughout, on the
// matrix cores.  For one KV chunk (FastUSP section 2.2 and 2.2.2),
//   O_r = softmax(q K^T * scale) V,   lse_r = log sum_j exp(q.k_j * scale),
// and over several chunks in one launch, each folded into the carried (O, lse) by the merge equations
// of section 3.4 with the operations a launch per chunk would perform (same bits).
//
//   * A wave owns 16 queries.  Scores are computed transposed, S^T = K Q^T, so that a lane owns one
//     query (column r = lane % 16) and four consecutive keys per 16-key block, and P^T in accumulator
//     layout is the B operand of O^T += V^T P^T as it stands.
//   * bf16 Q (engine Bf16Q): v_mfma_f32_16x16x32_bf16.  Products of bf16 values (and of E4M3 codes, which
//     are bf16 values) are exact in fp32; P is not rounded but split into three bf16 parts that add up
//     to its 24 bits, so P.V is three exact products instead of one (of finite V: a part that is 0 times
//     infinity is NaN).  fp32 Q (engine F32Q): v_mfma_f32_16x16x4_f32.
//   * Per-key factors: FP8 scales of K multiply the fp32 scores, those of V multiply P.
//   * 64-key tiles come to LDS while the one before is computed on: bf16 ones of d <= 128 directly (work-groups being few: by
//     width and mask, see attn_generic.hip), the others through registers (see Plan).  Pitches are odd multiples of 32 bytes (Bf16Q, V read transposed: no bank conflicts in the operand
//     reads), or d + 4 words (F32Q; K's reads conflict, which d + 8 words cure for nothing: fp32 is bound by its MFMAs).
//   * kKW waves share the 16 queries and take 64 / kKW keys of every tile each, their partial results
//     being combined through LDS at the end of a chunk: for calls with few query blocks, and to have eight waves on 64 queries.
//   * Where the work-groups are still few and there is one chunk, each query block's tiles are cut into ranges with a work-group
//     each (kShares, attn_generic_parts), whose O~, m and l a second launch puts together.
//
// What bounds it (bf16, d = 72): the issue of instructions and the bytes that the operand reads return.  Per wave, 16 queries
// and 32 keys: 80 VALU instructions, 21 MFMAs of 16 cycles, 16 operand reads of 11 KB; with what stands before and behind the tiles
// the VALU issues for 63 % of the launch's cycles and the matrix cores work for 36 %, mostly one after the other.
// So: one barrier per tile, tiles fetched through descriptors at places fixed per lane (directly to LDS they cost
// neither registers nor LDS writes), no test of a key outside masked and ragged tiles, no work for 16-wide blocks past the
// head dimension, O rescaled only when a maximum has outgrown a reference that was set 2^8 above it.  B=2 H=16 S=1024 d=72
// bf16, a call among others: 28.0 us (32.5 with tiles through registers and four waves; one wave per query row
// with scalar products, the first form, 857); 22 heads of 700 queries and keys 17.8 -> 15.8.
// (The exponentials against the old reference first, the maximum only where their sum does not show that none exceeds it, and
// the remainders of the split of P as dot products with -1 were no gain up to d = 128: one work-group on a CU waits for the longer chain
// of every tile.  16 heads of 1024, FP8, d = 40 29.0 us against 25.5, d = 72 34.2 against 30.7, d = 96 31.5 against 32.7; bf16,
// d = 40 20.4 against 19.7, d = 56 22.5 against 21.6, 24 heads 26.3 against 25.2.)  fp32 is bound by the fp32 matrix
// rate from about 256 work-groups on (d = 64, 32 heads: 80 us, 107 TFLOP/s).  Two chunks of 128 keys, H=2 Sq=128 d=64
// fp32: one launch, 9.6 us a call.
#pragma once
#include <type_traits>

#include "usp_common.h"
#include "prefetch_copy.h"

namespace usp {
namespace tile {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kTile = 64;          // keys per tile

// maximum / sum over the four lanes r, r + 16, r + 32, r + 48 that hold one query
__device__ __forceinline__ float group_max(float x) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float group_sum(float x) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// A tile of K or V as a buffer: what lies past its valid rows, or is asked for at kNowhere, loads as zeros.
typedef __amdgpu_buffer_rsrc_t Buf;
constexpr uint32_t kNowhere = 0xf0000000u;
__device__ __forceinline__ Buf tile_buffer(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

// Eight consecutive elements of a K / V row in flight from global memory, and their form in LDS.
struct UnitBf16 {
  typedef bf16_t elt;
  u32x4 w;
  __device__ __forceinline__ void zero() { w = u32x4{0u, 0u, 0u, 0u}; }
  __device__ __forceinline__ void load(const elt* p) { w = *reinterpret_cast<const u32x4*>(p); }
  __device__ __forceinline__ void load(Buf b, uint32_t off) { w = __builtin_amdgcn_raw_buffer_load_b128(b, off, 0, 0); }
  __device__ __forceinline__ u32x4 as_bf16() const { return w; }
};
struct UnitF8 {
  typedef uint8_t elt;
  u32x2 w;
  __device__ __forceinline__ void zero() { w = u32x2{0u, 0u}; }
  __device__ __forceinline__ void load(const elt* p) { w = *reinterpret_cast<const u32x2*>(p); }   // rows are 8-byte aligned
  __device__ __forceinline__ void load(Buf b, uint32_t off) { w = __builtin_amdgcn_raw_buffer_load_b64(b, off, 0, 0); }
  __device__ __forceinline__ void as_f32(f32x4& a, f32x4& b) const {
    const f32x2 c0 = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[0], false), c1 = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[0], true);
    const f32x2 c2 = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[1], false), c3 = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[1], true);
    a = f32x4{c0[0], c0[1], c1[0], c1[1]};
    b = f32x4{c2[0], c2[1], c3[0], c3[1]};
  }
  __device__ __forceinline__ u32x4 as_bf16() const {   // exact: every E4M3 value is a bf16 value
    f32x4 a, b;
    as_f32(a, b);
    return u32x4{pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(b[0], b[1]), pack_bf16x2(b[2], b[3])};
  }
};
struct UnitF32 {
  typedef float elt;
  f32x4 a, b;
  __device__ __forceinline__ void zero() { a = b = f32x4{0.0f, 0.0f, 0.0f, 0.0f}; }
  __device__ __forceinline__ void load(const elt* p) {
    a = *reinterpret_cast<const f32x4*>(p);
    b = *reinterpret_cast<const f32x4*>(p + 4);
  }
  __device__ __forceinline__ void load(Buf buf, uint32_t off) {
    a = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(buf, off, 0, 0));
    b = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(buf, off + 16, 0, 0));
  }
  __device__ __forceinline__ void as_f32(f32x4& x, f32x4& y) const { x = a; y = b; }
};

// p0, p1 as three bf16 pairs whose sums are p0 and p1 exactly (8 + 8 + 8 significant bits).  split3_dot: what is left of a value
// after its leading bf16 is one v_dot2_f32_bf16 with (-1, 0) or (0, -1), the same bits (compared for every fp32 value in the
// diagnostics), instead of a shift and a subtraction: two instructions less a value, a longer chain.  For d above 128, where the
// wave has the most MFMAs to hide it behind (9 heads of 1220 queries, 608 keys, d = 160 20.4 us with dots, 21.0 without; FP8, 4
// heads of 512 queries, 700 keys 20.1, 20.6; d = 256 within 1.5 %); narrower heads lose by it (see above).  The
// constants are kept in registers: the inline constant -1.0 that the compiler puts for (-1, 0) is not that pair.
struct Minus { uint32_t lo, hi; };
__device__ __forceinline__ Minus minus_one() {
  Minus m = {0x0000bf80u, 0xbf800000u};
  asm volatile("" : "+s"(m.lo), "+s"(m.hi));
  return m;
}
__device__ __forceinline__ void split3_dot(Minus one, float p0, float p1, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  auto rest = [](uint32_t pair, uint32_t c, float p) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), __builtin_bit_cast(bf16x2, c), p, false);
  };
  hi = pack_bf16x2(p0, p1);
  const float a0 = rest(hi, one.lo, p0), a1 = rest(hi, one.hi, p1);
  mid = pack_bf16x2(a0, a1);
  lo = pack_bf16x2(rest(mid, one.lo, a0), rest(mid, one.hi, a1));
}
__device__ __forceinline__ void split3(float p0, float p1, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
  hi = pack_bf16x2(p0, p1);
  const float a0 = p0 - __uint_as_float(hi << 16), a1 = p1 - __uint_as_float(hi & 0xffff0000u);
  mid = pack_bf16x2(a0, a1);
  lo = pack_bf16x2(a0 - __uint_as_float(mid << 16), a1 - __uint_as_float(mid & 0xffff0000u));
}

// kD: head dimension rounded up to the kernel's size (columns past s.d are zero); kDB: 16-wide blocks of it that
// the output has; kMB: 16-key blocks per wave
template <int kD, int kDB, int kMB>
struct Bf16Q {
  typedef bf16_t qo_elt;
  static constexpr int kSK = kD / 32, kBlocks = kDB;
  // bytes.  K: an odd multiple of 32: a 16-byte read takes the lanes 0-3, 12-15, 20-27 together (then 4-11, 16-19, 28-31, then the upper
  // half likewise), so that 8 rows of one piece must lie in the even 16-byte places of the banks and 8 of the next piece
  // in the odd ones.  (An odd multiple of 16 put two into one: d = 72, 32 heads of 1024 29.65 -> 29.1 us, from FP8 37.7 -> 36.3, d = 112 37.3 -> 36.3.)
  static constexpr int kPitchK = kD * 2 + 32, kPitchV = (kDB | 1) * 32;
  static_assert(kD % 32 == 0 && kMB % 2 == 0, "32-wide contraction steps");
  bf16x8 q[kSK];
  __device__ __forceinline__ void load_q(const bf16_t* row, int d, int g) {
#pragma unroll
    for (int ks = 0; ks < kSK; ++ks) {
      const int c = 32 * ks + 8 * g;
      u32x4 w = {0u, 0u, 0u, 0u};
      if (c < d) w = *reinterpret_cast<const u32x4*>(row + c);
      q[ks] = __builtin_bit_cast(bf16x8, w);
    }
  }
  // Q is waited for here, in front of the tiles.  Left to its first use, the wait stands at the head of the loop over them, and there
  // it waits in every tile for the next one, just asked for, too.  With tiles going to LDS directly: two chunks of 800 keys under 16 heads of
  // 800, d = 80 31.7 -> 28.8 us, 10 heads of 512, 900 keys, d = 112 19.8 -> 17.0, 22 heads of 700, d = 72 15.7 -> 14.7; fp32 ring of two of 128 under two
  // heads 9.85 -> 9.53.  Not from FP8, where the tile is converted on its way to LDS and the wait for it comes better early (d = 72, 32 heads
  // of 1024 36.4 us with that wait, 38.4 without), nor in fp32 where one wave has 16 queries for itself or d is above 64 (16 heads of 700, d = 128
  // 64.4, 65.0: kQFirst).
  __device__ __forceinline__ void landed() {
#pragma unroll
    for (int ks = 0; ks < kSK; ++ks) asm volatile("" : "+v"(q[ks]));
  }
  template <class U> static __device__ __forceinline__ void put(unsigned char* kv, int pitch, int row, int unit, const U& u) {
    *reinterpret_cast<u32x4*>(kv + row * pitch + unit * 16) = u.as_bf16();
  }
  // scores of the wave's keys: block mb holds keys 16 * mb + 4 * g + i of query r
  __device__ __forceinline__ void scores(const unsigned char* k, int r, int g, f32x4 (&s)[kMB]) const {
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb) s[mb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ks = 0; ks < kSK; ++ks)
#pragma unroll
      for (int mb = 0; mb < kMB; ++mb) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(k + (16 * mb + r) * kPitchK + (4 * ks + g) * 16);
        s[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, q[ks], s[mb], 0, 0, 0);
      }
  }
  static __device__ __forceinline__ bf16x8 v_operand(const unsigned char* v, int kk, int db, int r, int g) {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4* lds_p;
    const unsigned char* p = v + (32 * kk + 4 * g + (r >> 2)) * kPitchV + db * 32 + 8 * (r & 3);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(p + 16 * kPitchV));
    const u32x2 a = __builtin_bit_cast(u32x2, lo), b = __builtin_bit_cast(u32x2, hi);
    return __builtin_bit_cast(bf16x8, u32x4{a[0], a[1], b[0], b[1]});
  }
  // O^T += V^T P^T
  __device__ __forceinline__ void pv(const unsigned char* v, int r, int g, const float (&p)[kMB][4], f32x4 (&o)[kDB]) const {
    constexpr bool kDot = kD > 128;
    Minus one = {};
    if constexpr (kDot) one = minus_one();
    constexpr int kGrp = 4;   // head-dim blocks whose MFMAs alternate, so that none waits for its predecessor
#pragma unroll
    for (int kk = 0; kk < kMB / 2; ++kk) {
      u32x4 part[3];
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          uint32_t hi, mid, lo;
          if constexpr (kDot) split3_dot(one, p[2 * kk + a][2 * j], p[2 * kk + a][2 * j + 1], hi, mid, lo);
          else split3(p[2 * kk + a][2 * j], p[2 * kk + a][2 * j + 1], hi, mid, lo);
          part[0][2 * a + j] = hi; part[1][2 * a + j] = mid; part[2][2 * a + j] = lo;
        }
#pragma unroll
      for (int d0 = 0; d0 < kDB; d0 += kGrp) {
        bf16x8 a[kGrp];
#pragma unroll
        for (int x = 0; x < kGrp; ++x)
          if (d0 + x < kDB) a[x] = v_operand(v, kk, d0 + x, r, g);
#pragma unroll
        for (int t = 2; t >= 0; --t)   // small parts first
#pragma unroll
          for (int x = 0; x < kGrp; ++x)
            if (d0 + x < kDB) o[d0 + x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[x], __builtin_bit_cast(bf16x8, part[t]), o[d0 + x], 0, 0, 0);
      }
    }
  }
  static __device__ __forceinline__ void store4(bf16_t* p, const float (&o)[4]) {
    *reinterpret_cast<u32x2*>(p) = u32x2{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
  }
};

template <int kD, int kDB, int kMB>
struct F32Q {
  typedef float qo_elt;
  static constexpr int kSK = kD / 16, kBlocks = kDB;
  static constexpr int kPitchK = (kD + 4) * 4, kPitchV = (kD + 4) * 4;
  f32x4 q[kSK];   // head dims 16 * s + 4 * g + j: the contraction visits the head dimensions in that order on both sides
  __device__ __forceinline__ void load_q(const float* row, int d, int g) {
#pragma unroll
    for (int s = 0; s < kSK; ++s) {
      const int c = 16 * s + 4 * g;
      q[s] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      if (c < d) q[s] = *reinterpret_cast<const f32x4*>(row + c);
    }
  }
  __device__ __forceinline__ void landed() {
#pragma unroll
    for (int s = 0; s < kSK; ++s) asm volatile("" : "+v"(q[s]));
  }
  template <class U> static __device__ __forceinline__ void put(unsigned char* kv, int pitch, int row, int unit, const U& u) {
    f32x4 a, b;
    u.as_f32(a, b);
    *reinterpret_cast<f32x4*>(kv + row * pitch + unit * 32) = a;
    *reinterpret_cast<f32x4*>(kv + row * pitch + unit * 32 + 16) = b;
  }
  // kAcc sums per block, so that an MFMA does not wait for the one before it where a wave has one block
  __device__ __forceinline__ void scores(const unsigned char* k, int r, int g, f32x4 (&s)[kMB]) const {
    constexpr int kAcc = kMB >= 4 ? 1 : 4 / kMB;
    f32x4 acc[kAcc][kMB];
#pragma unroll
    for (int x = 0; x < kAcc; ++x)
#pragma unroll
      for (int mb = 0; mb < kMB; ++mb) acc[x][mb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c = 0; c < kSK; ++c) {
      f32x4 a[kMB];
#pragma unroll
      for (int mb = 0; mb < kMB; ++mb) a[mb] = *reinterpret_cast<const f32x4*>(k + (16 * mb + r) * kPitchK + (16 * c + 4 * g) * 4);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int mb = 0; mb < kMB; ++mb)
          acc[j % kAcc][mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[mb][j], q[c][j], acc[j % kAcc][mb], 0, 0, 0);
    }
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb) {
      s[mb] = acc[0][mb];
#pragma unroll
      for (int x = 1; x < kAcc; ++x) s[mb] += acc[x][mb];
    }
  }
  __device__ __forceinline__ void pv(const unsigned char* v, int r, int g, const float (&p)[kMB][4], f32x4 (&o)[kDB]) const {
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
      for (int i = 0; i < 4; ++i)   // contraction index g of the MFMA is key 16 * mb + 4 * g + i
#pragma unroll
        for (int x = 0; x < kDB; ++x) {
          const float a = *reinterpret_cast<const float*>(v + (16 * mb + 4 * g + i) * kPitchV + (16 * x + r) * 4);
          o[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, p[mb][i], o[x], 0, 0, 0);
        }
  }
  static __device__ __forceinline__ void store4(float* p, const float (&o)[4]) {
    *reinterpret_cast<float4*>(p) = make_float4(o[0], o[1], o[2], o[3]);
  }
};

// bf16 K and V whose two buffers leave room for a second work-group on the CU (kDma): the tiles go from memory to LDS
// directly.  A load instruction fills 64 consecutive 16-byte slots with what its lanes name, so the rows' padding is slots
// that name nothing (they load as zeros, as columns past d and rows past the chunk do).  Otherwise (FP8 K/V, rows further
// apart than a descriptor reaches, d above 128) through registers; so are fp32 tiles, whose waves have the time: directly,
// 6 heads of d = 96 in a ring of four chunks of 500 took 68.6 us instead of 62.8, 4 heads of d = 64 26.5 instead of 25.0.
template <class Unit> struct Directly { static constexpr bool value = std::is_same<Unit, UnitBf16>::value; };

// LDS of a work-group: one or two buffers of K tile | V tile | per-key factors of FP8 (exponent, V).  With two, a tile is
// brought while the one before it is computed on, with one barrier per tile.  The exchange of the kKW partial results reuses a
// buffer's tiles (kDma: has its own room behind them, since the next chunk's tiles are on their way).
template <class E, int kD, int kKW, int kW>
struct Plan {
  static constexpr int tiles = kTile * (E::kPitchK + E::kPitchV);
  static constexpr int xch = (kW / kKW) * (kKW - 1) * 64 * (4 * E::kBlocks + 2) * 4;
  static constexpr int fac = xch > tiles ? xch : tiles;          // offset of the per-key values
  static constexpr int one = fac + 2 * kTile * 4;
  static constexpr bool pair = 2 * one <= 80 * 1024;             // two buffers, and two work-groups on a CU
  static constexpr int direct = 2 * tiles + xch;
  static constexpr bool dma = direct <= 80 * 1024;
};

__device__ __forceinline__ void dma_slots(u32x4 desc, uint32_t lane_off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(lds), "v"(lane_off), "s"(desc) : "memory", "m0");
}

// kShares: the keys of the one chunk are shared by AttnStep::parts work-groups per query block (a template parameter: what it asks
// of the scalar registers costs launches without it 2 to 9 %).
template <template <int, int, int> class Engine, class Unit, int kD, int kDB, int kKW, int kW, bool kDma, bool kShares>
__global__ __launch_bounds__(kW * 64, kW / 4 * (kD > 160 ? 1 : 2))   // waves per SIMD the registers allow
void attn_tile_kernel(AttnStep s) {
  constexpr int kMB = 4 / kKW, kThreads = kW * 64;
  typedef Engine<kD, kDB, kMB> E;
  typedef Plan<E, kD, kKW, kW> L;
  constexpr int kBuffers = kDma || L::pair ? 2 : 1, kOne = kDma ? L::tiles : L::one;
  typedef typename Unit::elt KT;
  typedef typename E::qo_elt QT;
  constexpr bool fp8 = std::is_same<Unit, UnitF8>::value;
  constexpr bool kQFirst = !fp8 && (std::is_same<QT, float>::value ? kD <= 64 && kKW > 1 : kD <= 128);   // (see landed)
  extern __shared__ __align__(16) unsigned char smem[];
  touch_step();
  if (s.copy_wgs > 0 && blockIdx.x >= gridDim.x - s.copy_wgs) {   // prefetch work-groups end the x axis
    if (blockIdx.y == 0 && blockIdx.z == 0) prefetch_copy(s, blockIdx.x - (gridDim.x - s.copy_wgs), threadIdx.x, kThreads);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int part = wave % kKW;                                  // which keys of a tile this wave takes
  const int h = blockIdx.y, b = blockIdx.z, d = s.d;
  // work-groups that share the keys of a query block (attn_generic_parts) follow one another
  const uint32_t shares = kShares ? (uint32_t)s.parts : 1u;
  const uint32_t q_block = kShares ? blockIdx.x / shares : blockIdx.x, share = kShares ? blockIdx.x - q_block * shares : 0u;
  const int qi = ((int)q_block * (kW / kKW) + wave / kKW) * 16 + r;
  const int qc = min(qi, s.Sq - 1);                             // surplus lanes recompute the last row, store nothing
  const float scale2 = s.scale * 1.44269504088896340736f;

  E e;
  e.load_q((const QT*)s.q + b * s.qs[0] + h * s.qs[1] + (int64_t)qc * s.qs[2], d, g);

  // ---- staging.  A thread's (kDma: a lane's) places in a tile are the same in every tile, so that a tile costs the scalar unit
  // a descriptor and nothing else: with a 64-bit address, a row and a column test per unit, fetching took 140 of the
  // 500 instructions a wave issued per tile.
  constexpr int kUPR = kD / 8, kNU = kDma ? 1 : kTile * kUPR / kThreads;   // through registers: units per row; per thread and tensor (unit u: thread u % kThreads)
  constexpr int kSlotsK = E::kPitchK / 16, kSlotsV = E::kPitchV / 16;      // directly: slots per row, which is also the instructions per tensor
  constexpr int kNI = kDma ? (kSlotsK + kSlotsV + kW - 1) / kW : 1;        // a wave's instructions: wave, wave + kW, ..
  Unit ku[kNU], vu[kNU];
  float f_c = 0.0f, f_v = 0.0f;                                 // FP8, threads 0..63: the tile's per-key values
  const uint32_t rowB = (uint32_t)(s.ks[2] * sizeof(KT));
  const bool near_rows = kDma || s.ks[2] * (int64_t)sizeof(KT) * kTile < (int64_t)kNowhere;   // else: addresses of 64 bits
  uint32_t place[kDma ? kNI : kNU];
  if (kDma) {
#pragma unroll
    for (int i = 0; i < kNI; ++i) {
      const int j = wave + i * kW, is_v = j >= kSlotsK;
      const int slot = (is_v ? j - kSlotsK : j) * 64 + lane, per = is_v ? kSlotsV : kSlotsK;
      const int row = slot / per, col = (slot - row * per) * (16 / (int)sizeof(KT));
      place[i] = col < d && row < kTile ? row * rowB + col * (uint32_t)sizeof(KT) : kNowhere;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kNU; ++i) {
      const int u = tid + i * kThreads, row = u / kUPR, col = (u % kUPR) * 8;
      place[i] = col < d ? row * rowB + col * (uint32_t)sizeof(KT) : kNowhere;
    }
  }
  // this work-group's keys of the one chunk that is shared: tiles share * n / shares .. (share + 1) * n / shares - 1
  int own_from = 0, own_to = 0x7fffffff;
  if (kShares) {
    const uint32_t n = (uint32_t)(s.chunk[0].Sc + kTile - 1) / kTile;
    own_from = (int)(n * share / shares) * kTile;
    own_to = min(s.chunk[0].Sc, (int)(n * (share + 1) / shares) * kTile);
  }
  int pc = -1, first_key = 0, left = 0;                         // next tile to fetch: its chunk, first key, rows from there on
  const KT *kb = nullptr, *vb = nullptr;
  const uint8_t* mask = nullptr;                                // of that chunk and batch entry, or null
  uint8_t mask_byte = 1;                                        // key `lane` of the tile fetched last takes part
  bool masked = false;
  const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
  auto fetch = [&](uint32_t lds) {                              // lds: where a tile that goes directly lands
    if (near_rows) {
      const uint32_t bytes = (uint32_t)min(left, kTile) * rowB;
      if constexpr (kDma) {
        auto desc = [&](const void* p) {
          const uint64_t a = (uint64_t)(uintptr_t)p;
          return u32x4{(uint32_t)a, (uint32_t)(a >> 32) & 0xffffu, bytes, 0x00020000u};
        };
        const u32x4 kd = desc(kb), vd = desc(vb);
#pragma unroll
        for (int i = 0; i < kNI; ++i) {
          const int j = wave + i * kW;
          if ((i + 1) * kW > kSlotsK + kSlotsV && j >= kSlotsK + kSlotsV) continue;
          if (j < kSlotsK) dma_slots(kd, place[i], lds + j * 1024);
          else dma_slots(vd, place[i], lds + kTile * E::kPitchK + (j - kSlotsK) * 1024);
        }
      } else {
        const Buf kbuf = tile_buffer(kb, bytes), vbuf = tile_buffer(vb, bytes);
#pragma unroll
        for (int i = 0; i < kNU; ++i) ku[i].load(kbuf, place[i]);
#pragma unroll
        for (int i = 0; i < kNU; ++i) vu[i].load(vbuf, place[i]);
      }
    } else if constexpr (!kDma) {
#pragma unroll
      for (int i = 0; i < kNU; ++i) {
        const int u = tid + i * kThreads, row = u / kUPR, col = (u % kUPR) * 8;
        ku[i].zero();
        vu[i].zero();
        if (row < left && col < d) {
          ku[i].load(kb + row * s.ks[2] + col);
          vu[i].load(vb + row * s.ks[2] + col);
        }
      }
    }
    masked = mask != nullptr;
    if (masked) mask_byte = lane < left ? mask[first_key + lane] : 0;
    if (fp8 && tid < kTile) {
      const AttnStep::Chunk& ch = s.chunk[pc];
      f_c = scale2; f_v = 1.0f;
      if (tid < left) {
        const int64_t row = ((int64_t)b * s.H + h) * ch.Sc + first_key + tid;
        f_c = ch.k_scale_src[row] * scale2;
        f_v = ch.v_scale_src[row];
      }
    }
  };
  auto stage = [&](unsigned char* buf) {
    unsigned char* v_lds = buf + kTile * E::kPitchK;
    float* fac = reinterpret_cast<float*>(buf + L::fac);         // factor | V scale
#pragma unroll
    for (int i = 0; i < kNU; ++i) {
      const int u = tid + i * kThreads, row = u / kUPR, unit = u % kUPR;
      E::put(buf, E::kPitchK, row, unit, ku[i]);
      if ((unit + 1) * 8 <= kDB * 16) E::put(v_lds, E::kPitchV, row, unit, vu[i]);
    }
    if (fp8 && tid < kTile) { fac[tid] = f_c; fac[kTile + tid] = f_v; }
  };

  // carried (O, lse) of earlier chunks
  f32x4 oc[kDB];
  float lse_c = -INFINITY;
  bool carried = s.mode >= 2;
  const int64_t row = ((int64_t)b * s.H + h) * s.Sq + qc;
  float* accp = s.acc ? s.acc + row * d : nullptr;
  if (carried && part == 0) {
    lse_c = s.lse[row];
#pragma unroll
    for (int db = 0; db < kDB; ++db) {
      oc[db] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      if (16 * db + 4 * g < d) oc[db] = *reinterpret_cast<const f32x4*>(accp + 16 * db + 4 * g);
    }
  }

  bool fetched = false;                                         // a tile is on the way, or waits in registers
  auto fetch_next = [&](uint32_t lds) {
    while (left <= 0 && pc < s.n_multi) {                       // into the next chunk that holds keys
      if (++pc == s.n_multi) break;
      const AttnStep::Chunk& ch = s.chunk[pc];
      left = ch.Sc;
      first_key = 0;
      kb = (const KT*)ch.k + b * ch.ks0 + h * ch.ks1;
      vb = (const KT*)ch.v + b * ch.ks0 + h * ch.ks1;
      if (kShares) {
        left = min(left, own_to) - own_from;
        first_key = own_from;
        kb += own_from * s.ks[2];
        vb += own_from * s.ks[2];
      }
      mask = ch.mask_src ? ch.mask_src + (int64_t)b * ch.Sc : nullptr;
    }
    fetched = left > 0;
    if (!fetched) return;
    fetch(lds);
    left -= kTile;
    first_key += kTile;
    kb += kTile * s.ks[2];
    vb += kTile * s.ks[2];
  };
  // live keys of the tile fetched last (its mask has landed), bit = key
  auto live_word = [&]() -> uint64_t { return masked ? __builtin_amdgcn_ballot_w64(mask_byte != 0) : ~0ull; };
  uint64_t live = ~0ull, live_next = ~0ull;                     // of the tile computed on, and of the one behind it
  unsigned char* cur = smem;                                    // the tile computed on
  unsigned char* oth = smem + (kBuffers - 1) * kOne;            // the other buffer, if there is one
  auto lds_of = [&](const unsigned char* p) -> uint32_t { return __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(p - smem)); };
  fetch_next(lds0);
  if (kDma) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);                         // vmcnt(0)
    e.landed();
    live = live_word();
    __syncthreads();
    fetch_next(lds_of(oth));
  } else if (kBuffers == 2 && fetched) {
    stage(cur);
    if (kQFirst) e.landed();
    live = live_word();
    fetch_next(0);
    __syncthreads();
  } else if (kQFirst) {
    e.landed();
  }

  for (int c = 0; c < s.n_multi; ++c) {
    // m: a reference that is never below the maximum (so that P <= 1, as V times a larger P could leave the fp32 range)
    // and was set kAbove above the one that moved it last, so that it moves seldom.  fp32: less, because the exponents
    // are rounded at their own size (d = 32, 1000 keys: O off by 6.3e-7 with 8)
    constexpr float kAbove = std::is_same<QT, float>::value ? 2.0f : 8.0f;
    float m = -INFINITY, l = 0.0f;
    f32x4 o[kDB];
#pragma unroll
    for (int db = 0; db < kDB; ++db) o[db] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int len = kShares ? min(s.chunk[c].Sc, own_to) - own_from : s.chunk[c].Sc;
    for (int t = 0; t * kTile < len; ++t) {
      if (kBuffers == 1) {
        __syncthreads();              // the previous tile (or the exchange) has been read
        stage(cur);
        live = live_word();
        fetch_next(0);
        __syncthreads();
      }
      const float* fac = reinterpret_cast<const float*>(cur + L::fac);
      const int k0 = part * 16 * kMB;                            // first key of this wave
      f32x4 sc[kMB];
      e.scores(cur + k0 * E::kPitchK, r, g, sc);
      // exponents in log2 units are sc * f with f the uniform scale, or with FP8 K sc itself, scaled by key here
      if (fp8) {
#pragma unroll
        for (int mb = 0; mb < kMB; ++mb) sc[mb] *= *reinterpret_cast<const f32x4*>(fac + k0 + 16 * mb + 4 * g);
      }
      const int rest = len - t * kTile;
      if (rest < kTile || live != ~0ull) {                       // (uniform) the tile has dead keys
        asm volatile("" ::: "memory");                           // (kept a branch)
        const uint64_t keep = (rest < kTile ? live & ((1ull << rest) - 1ull) : live) >> (k0 + 4 * g);
#pragma unroll
        for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
          for (int i = 0; i < 4; ++i) sc[mb][i] = (keep >> (16 * mb + i)) & 1 ? sc[mb][i] : -INFINITY;
      }
      const float f = fp8 ? 1.0f : scale2;
      float tm = -INFINITY;
#pragma unroll
      for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
        for (int i = 0; i < 4; ++i) tm = fmaxf(tm, sc[mb][i]);
      tm = group_max(tm);
      if (!fp8) tm *= scale2;
      const bool jump = tm > m;                                  // m = -inf: the first live key
      if (__builtin_amdgcn_ballot_w64(jump) != 0ull) {
        const float m_new = tm + kAbove, alpha = jump ? __builtin_amdgcn_exp2f(m - m_new) : 1.0f;
        m = jump ? m_new : m;
        l *= alpha;
#pragma unroll
        for (int db = 0; db < kDB; ++db) o[db] *= alpha;
      }
      // no live key so far: every exponent is -inf and P = 0 against any finite reference
      const float ref = m == -INFINITY ? 0.0f : m;
      float p[kMB][4], ps = 0.0f;
#pragma unroll
      for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
        for (int i = 0; i < 4; ++i) { p[mb][i] = __builtin_amdgcn_exp2f(fmaf(sc[mb][i], f, -ref)); ps += p[mb][i]; }
      l += ps;
      if (fp8) {
#pragma unroll
        for (int mb = 0; mb < kMB; ++mb) {
          const f32x4 fv = *reinterpret_cast<const f32x4*>(fac + kTile + k0 + 16 * mb + 4 * g);
#pragma unroll
          for (int i = 0; i < 4; ++i) p[mb][i] *= fv[i];
        }
      }
      e.pv(cur + kTile * E::kPitchK + k0 * E::kPitchV, r, g, p, o);
      if (kBuffers == 2) {
        if (kDma) {
          asm volatile("" ::: "memory");
          __builtin_amdgcn_s_waitcnt(0x0F70);                    // the next tile, asked for a tile ago
          live_next = live_word();
          __syncthreads();
          fetch_next(lds_of(cur));
        } else {
          if (fetched) {
            stage(oth);
            live_next = live_word();
            fetch_next(0);
          }
          __syncthreads();
        }
        live = live_next;
        unsigned char* x = cur; cur = oth; oth = x;              // oth: the tile just computed on
      }
    }
    l = group_sum(l);

    if (kKW > 1 && len > 0) {   // combine the waves that share these queries: [wave][slot][lane], in the place of the last tile or behind the tiles
      constexpr int kSlots = 4 * kDB + 2;
      float* x = reinterpret_cast<float*>(kDma ? smem + 2 * kOne : oth) + ((wave / kKW) * (kKW - 1) - 1) * kSlots * 64 + lane;
      if (kBuffers == 1) __syncthreads();
      if (part > 0) {
        float* y = x + part * kSlots * 64;
#pragma unroll
        for (int db = 0; db < kDB; ++db)
#pragma unroll
          for (int i = 0; i < 4; ++i) y[(4 * db + i) * 64] = o[db][i];
        y[4 * kDB * 64] = m;
        y[(4 * kDB + 1) * 64] = l;
      }
      __syncthreads();
      if (part == 0) {
#pragma unroll
        for (int w = 1; w < kKW; ++w) {
          const float* y = x + w * kSlots * 64;
          const float mw = y[4 * kDB * 64], lw = y[(4 * kDB + 1) * 64];
          const float mm = fmaxf(m, mw), ref = mm == -INFINITY ? 0.0f : mm;
          const float wa = __builtin_amdgcn_exp2f(m - ref), wb = __builtin_amdgcn_exp2f(mw - ref);
#pragma unroll
          for (int db = 0; db < kDB; ++db)
#pragma unroll
            for (int i = 0; i < 4; ++i) o[db][i] = wa * o[db][i] + wb * y[(4 * db + i) * 64];
          l = wa * l + wb * lw;
          m = mm;
        }
      }
      if (!kDma && kBuffers == 2 && c + 1 < s.n_multi) __syncthreads();   // before the next chunk's tiles are staged over it
    }
    if (kShares) {   // left as it is for attn_tile_combine_kernel
      if (part == 0 && qi < s.Sq) {
        const int64_t at = (int64_t)share * s.B * s.H * s.Sq + row;
#pragma unroll
        for (int db = 0; db < kDB; ++db)
          if (16 * db + 4 * g < d) *reinterpret_cast<f32x4*>(s.part_o + at * d + 16 * db + 4 * g) = o[db];
        if (g == 0) *reinterpret_cast<float2*>(s.part_ml + 2 * at) = make_float2(m, l);
      }
      return;
    }
    // the chunk's result and the merge of section 3.4
    float lse_r = -INFINITY, c_cur = 0.0f, w_prev = 0.0f;
    // (log l apart from m ln 2, so that what is rounded is no larger than the result: in log2 units it would be by half)
    if (l > 0.0f) { lse_r = fmaf(m, 0.69314718055994530942f, logf(l)); c_cur = 1.0f / l; }
    float lse_new = lse_r;
    if (carried) {
      const float mm = fmaxf(lse_c, lse_r);
      if (mm == -INFINITY) { c_cur = 0.0f; lse_new = -INFINITY; }
      else {
        lse_new = mm + logf(expf(lse_c - mm) + expf(lse_r - mm));
        w_prev = expf(lse_c - lse_new);
        c_cur *= expf(lse_r - lse_new);
      }
    }
#pragma unroll
    for (int db = 0; db < kDB; ++db)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float x = o[db][i] * c_cur;
        oc[db][i] = carried ? fmaf(w_prev, oc[db][i], x) : x;
      }
    lse_c = lse_new;
    carried = true;
  }

  if (part != 0 || qi >= s.Sq) return;
  QT* outp = (QT*)s.out + b * s.os[0] + h * s.os[1] + (int64_t)qi * s.os[2];
#pragma unroll
  for (int db = 0; db < kDB; ++db) {
    const int col = 16 * db + 4 * g;
    if (col >= d) continue;
    if (s.mode == 1 || s.mode == 2) *reinterpret_cast<f32x4*>(accp + col) = oc[db];
    else {
      const float x[4] = {oc[db][0], oc[db][1], oc[db][2], oc[db][3]};
      E::store4(outp + col, x);
    }
  }
  if (g == 0) s.lse[row] = lse_c;
}

template <template <int, int, int> class Engine, class Unit, int kD, int kDB, int kKW, int kW, bool kDma, bool kShares>
usp_status launch_tile_as(const AttnStep& s, hipStream_t st) {
  typedef Plan<Engine<kD, kDB, 4 / kKW>, kD, kKW, kW> L;
  constexpr int lds = kDma ? L::direct : (L::pair ? 2 : 1) * L::one;
  constexpr int qpw = 16 * kW / kKW;   // queries per work-group
  if (lds > 64 * 1024) USP_CHECK_HIP((allow_large_lds<attn_tile_kernel<Engine, Unit, kD, kDB, kKW, kW, kDma, kShares>>(lds)));
  const dim3 grid((unsigned)((s.Sq + qpw - 1) / qpw * (kShares ? s.parts : 1) + s.copy_wgs), (unsigned)s.H, (unsigned)s.B);
  hipLaunchKernelGGL((attn_tile_kernel<Engine, Unit, kD, kDB, kKW, kW, kDma, kShares>), grid, dim3(kW * 64), lds, st, s);
  USP_CHECK_HIP(hipGetLastError());
  return USP_OK;
}
// (only few work-groups share keys: those whose waves share queries, four to a work-group)
template <template <int, int, int> class Engine, class Unit, int kD, int kDB, int kKW, int kW, bool kDma>
usp_status launch_tile_one(const AttnStep& s, hipStream_t st) {
  if constexpr (kKW > 1 && kW == 4 && kD <= 160) {
    if (s.parts > 1) return launch_tile_as<Engine, Unit, kD, kDB, kKW, kW, kDma, true>(s, st);
  }
  return launch_tile_as<Engine, Unit, kD, kDB, kKW, kW, kDma, false>(s, st);
}
// kKW, kW: waves that share queries, and waves of a work-group where the tiles go directly to LDS (otherwise four, with kKWR)
template <template <int, int, int> class Engine, class Unit, int kD, int kDB, int kKW, int kW, int kKWR>
usp_status launch_tile(const AttnStep& s, hipStream_t st) {
  if constexpr (Directly<Unit>::value && Plan<Engine<kD, kDB, 4 / kKW>, kD, kKW, kW>::dma) {
    if (s.ks[2] * (int64_t)sizeof(typename Unit::elt) * kTile < (int64_t)kNowhere) return launch_tile_one<Engine, Unit, kD, kDB, kKW, kW, true>(s, st);
  }
  return launch_tile_one<Engine, Unit, kD, kDB, kKWR, 4, false>(s, st);
}

}  // namespace tile
}  // namespace usp

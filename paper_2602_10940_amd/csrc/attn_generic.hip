// bf16 Q with head dimensions other than 64 and 128 (bf16 or FP8 K/V): attn_tile.h, and the dispatch of every
// shape that file takes.
#include "attn_tile.h"

namespace usp {

usp_status launch_attn_generic_f32(const AttnStep& s, bool few, hipStream_t st);   // attn_generic_f32.hip

namespace {
// wgs: work-groups of 64 queries
template <class Unit, int kD, int kDB>
usp_status run_bf16(const AttnStep& s, bool few, int64_t wgs, hipStream_t st) {
  if (few) {
    // Few work-groups leave one wave to a SIMD.  The narrow widths then wait longer for a tile on its way to LDS than for one in
    // their registers, and d = 81 to 96 do with half the CUs busy; bytes of a mask, and LDS writes of wider rows, turn that round
    // (d = 49 to 64 excepted).  us of launches that do not share keys, with direct tiles, through registers: 16 heads of 153 queries, 1793 keys, d = 40 21.7, 21.3 (masked
    // 23.0, 23.9), d = 56 27.8, 25.6 (29.8, 30.1), d = 72 30.0, 28.9 (32.4, 34.4), d = 96 32.3, 30.0 (34.3, 35.6), d = 112 35.4, 34.8
    // (36.7, 39.0); 2 x 5 heads of 959 queries, 634 keys, d = 56 12.7, 12.7, d = 72 13.9, 15.0, d = 96 14.9, 15.5, d = 112 16.1, 18.1;
    // 4 heads of 512 queries, 700 keys, d = 56 11.3, 10.7, d = 72 12.3, 12.4, d = 96 12.7, 12.6, d = 112 14.2, 15.1.
    bool masked = false;
    for (int c = 0; c < s.n_multi; ++c) masked = masked || s.chunk[c].mask_src != nullptr;
    if (kDB == 4 || (!masked && (kDB == 3 || (kDB == 6 && wgs <= 128)))) return tile::launch_tile_one<tile::Bf16Q, Unit, kD, kDB, 2, 4, false>(s, st);
    return tile::launch_tile<tile::Bf16Q, Unit, kD, kDB, 2, 4, 2>(s, st);
  }
  // 65 to 80 columns of output, as long as the chip takes all work-groups at once with two on a CU: eight waves share 64 queries,
  // two by two, for four waves a SIMD.  Four waves leave room for three work-groups.  d = 72, 1024 queries and keys, with eight and
  // four: 256 work-groups 22.1 us, 24.2; 272 27.5, 27.7; 384 27.9, 28.3; 512 29.0, 29.2; from 513 on eight need a second round
  // (960 queries and keys, 540: 43.5, 35.7).  The neighbours have no such line: eight waves take 2 % more for d <= 64, and for d
  // = 81 to 96 (126 registers) 3 % less at 272 to 448 work-groups and as much at 512.
  if constexpr (kDB == 5) if (wgs <= 512) return tile::launch_tile<tile::Bf16Q, Unit, kD, kDB, 2, 8, 1>(s, st);
  return tile::launch_tile<tile::Bf16Q, Unit, kD, kDB, 1, 4, 1>(s, st);
}
// 32-wide steps of the head dimension in the scores, 16-wide blocks of it in the output
template <class Unit>
usp_status run_bf16_d(const AttnStep& s, bool few, int64_t wgs, hipStream_t st) {
  if (s.d <= 48) return run_bf16<Unit, 64, 3>(s, few, wgs, st);
  if (s.d <= 64) return run_bf16<Unit, 64, 4>(s, few, wgs, st);
  if (s.d <= 80) return run_bf16<Unit, 96, 5>(s, few, wgs, st);
  if (s.d <= 96) return run_bf16<Unit, 96, 6>(s, few, wgs, st);
  if (s.d <= 112) return run_bf16<Unit, 128, 7>(s, few, wgs, st);
  if (s.d <= 128) return run_bf16<Unit, 128, 8>(s, few, wgs, st);
  if (s.d <= 160) return run_bf16<Unit, 160, 10>(s, few, wgs, st);
  return run_bf16<Unit, 256, 16>(s, few, wgs, st);
}
// The shares of a launch whose work-groups shared the keys of a query block (AttnStep::parts): per query,
// O = sum_i 2^(m_i - m) O~_i / l, l = sum_i 2^(m_i - m) l_i, m = max_i m_i, and lse = m ln 2 + log l as the kernel itself
// has it.  One thread per four head dims; the shares lie in the caches, and all of up to kParts are read together (one after the other, each
// trip waiting for the one before, fp32, 8 heads of 102 queries, 1549 keys, d = 32 took 10.2 us instead of 8.4, d = 96 18.7 instead of 17.0; bf16, 16 heads of
// 153 queries, 1793 keys, d = 40 12.9 instead of 11.2).
template <typename T, int kParts>
__global__ __launch_bounds__(256) void attn_tile_combine_kernel(const float* __restrict__ part_o, const float* __restrict__ part_ml, T* __restrict__ out,
                                                                float* __restrict__ lse, int parts, uint32_t rows, uint32_t quads, uint32_t Sq,
                                                                uint32_t H, int64_t os0, int64_t os1, int64_t os2) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  const uint32_t at = blockIdx.x * 256 + threadIdx.x, row = at / quads, c = at - row * quads;   // quads: of head dims
  if (row >= rows) return;
  float2 ml[kParts];
  f32x4 x[kParts];
#pragma unroll
  for (int i = 0; i < kParts; ++i) {
    const int64_t at = (int64_t)(i < parts ? i : 0) * rows + row;
    ml[i] = *reinterpret_cast<const float2*>(part_ml + 2 * at);
    x[i] = *reinterpret_cast<const f32x4*>(part_o + (at * quads + c) * 4);
  }
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < kParts; ++i) m = fmaxf(m, ml[i].x);   // (those past the last repeat the first)
  const float ref = m == -INFINITY ? 0.0f : m;   // (no live key: every weight and every l is 0)
  float l = 0.0f;
  f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int i = 0; i < kParts; ++i) {
    if (i < parts) {
      const float w = __builtin_amdgcn_exp2f(ml[i].x - ref);
      l = fmaf(w, ml[i].y, l);
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = fmaf(w, x[i][e], o[e]);
    }
  }
  const float inv = l > 0.0f ? 1.0f / l : 0.0f;
  const uint32_t bh = row / Sq, qi = row - bh * Sq, b = bh / H, h = bh - b * H;
  T* p = out + b * os0 + h * os1 + (int64_t)qi * os2 + 4 * c;
  if constexpr (sizeof(T) == 2) *reinterpret_cast<u32x2*>(p) = u32x2{pack_bf16x2(o[0] * inv, o[1] * inv), pack_bf16x2(o[2] * inv, o[3] * inv)};
  else *reinterpret_cast<f32x4*>(p) = o * inv;
  if (c == 0) lse[row] = l > 0.0f ? fmaf(m, 0.69314718055994530942f, logf(l)) : -INFINITY;
}
template <typename T>
usp_status launch_tile_combine(const AttnStep& s, hipStream_t st) {
  const uint32_t rows = (uint32_t)((int64_t)s.B * s.H * s.Sq), quads = (uint32_t)s.d / 4;
  const dim3 grid((unsigned)(((uint64_t)rows * quads + 255) / 256));
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, s.part_o, s.part_ml, (T*)s.out, s.lse, s.parts, rows, quads, (uint32_t)s.Sq, (uint32_t)s.H, s.os[0],
                       s.os[1], s.os[2]);
  };
  if (s.parts <= 2) launch(attn_tile_combine_kernel<T, 2>);
  else if (s.parts <= 4) launch(attn_tile_combine_kernel<T, 4>);
  else launch(attn_tile_combine_kernel<T, kMostShares>);
  USP_CHECK_HIP(hipGetLastError());
  return USP_OK;
}
// Waves share queries where 64-query work-groups would leave CUs idle: H = 4, Sq = S = 1024 (64 of them): fp32
// d = 64 53 -> 27 us, d = 128 100 -> 46 us, bf16 d = 72 30 -> 21 us.  At 192 work-groups the two are within
// 20 %, at 256 fp32 loses (30 against 36 us).  The d = 256 sizes fill a CU's LDS with one work-group, so
// sharing stops paying at half a chip of them (192: bf16 65 against 93 us, fp32 199 against 268 us).
bool few_work_groups(bool f32, int B, int H, int Sq, int d, int64_t* wgs) {
  *wgs = (int64_t)((Sq + 63) / 64) * B * H;
  return *wgs < (d > 160 || (f32 && d > 128) ? 160 : 256);
}
}  // namespace

// How many work-groups share the keys of a query block: one chunk under few query blocks leaves CUs idle, and each work-group goes
// through its tiles one after the other.  The figures of the rule are microseconds: a launch 4; a tile, in fp32 by its columns in
// steps of 32, in bf16 by d; what a tile takes longer with two work-groups on a CU, and with more than two; the second launch 2.5,
// and the shares, written and read, at 5 TB/s.  Powers of two: a share's number then says which XCDs it runs on, so that each
// L2 holds its part of K and V only (56 work-groups over 25 tiles, d = 128, shared by 3, 4, 6, 8, 12: 29.2, 23.7, 27.1, 23.8,
// 30.9 us); more than 8 gains 4 % at the most.  A share has two tiles at least.  768 work-groups are a fitted limit: where LDS takes three
// to a CU they run at once, where it takes two (fp32 d = 33 to 64 and 97 to 128, bf16 d = 65 to 128) those above 512 are a second round, and the factor 2.1 stands for that.
// Of 80 shapes, each measured with 1, 2, 4 and 8, the choice is on average 1 %, at worst 15 %, above the best and never above 1.
// us before and after: fp32, 8 heads of 102 queries, 1549 keys, d = 32, 64, 96, 128 23.5, 34.5, 45.4, 60.3 -> 11.7, 15.6, 19.3, 23.5; 4 heads of
// 512 queries, 512 keys 8.7, 13.0, 17.6, 22.7 -> 8.7 (as before), 11.4, 14.0, 17.1; bf16, 16 heads of 153 queries, 1793 keys, d = 40, 72, 112,
// 160 25.5, 30.4, 35.7, 36.7 -> 13.2, 15.5, 17.3, 21.8, d = 40, 72, 112 from FP8 35.0, 41.7, 49.2 -> 14.6, 19.1, 22.9.
// Against 64 bits, 21 random shapes, relative L2 over that of one work-group: fp32 0.56 to 0.98, bf16 1.00.
// Several chunks are merged one after another, with the operations and the bits of a launch per chunk, and are not shared; a ring of which one
// chunk alone holds keys counts as several (its workspace and its launches are those of a ring).
int attn_generic_parts(bool f32, int B, int H, int Sq, int d, int keys) {
  int64_t wgs64;
  if (d > 160 || (f32 && d > 128) || !few_work_groups(f32, B, H, Sq, d, &wgs64)) return 1;   // (the sizes of 256 fill a CU with one work-group)
  const int64_t rows = (int64_t)B * H * Sq, wgs = (int64_t)B * H * (f32 ? (Sq + 15) / 16 : (Sq + 31) / 32), tiles = ((int64_t)keys + 63) / 64;
  const double tile = f32 ? 0.1 + 0.0165 * ((d + 31) / 32 * 32) : 0.55 + 0.004 * d;
  auto cost = [&](int64_t p) {
    const double crowd = wgs * p <= 256 ? 1.0 : wgs * p <= 512 ? 1.2 : 2.1;
    return 4.0 + (double)((tiles + p - 1) / p) * tile * crowd + (p > 1 ? 2.5 + 8.0e-6 / 5.0 * (double)(d * p * rows) : 0.0);
  };
  int best = 1;
  double least = 0.93 * cost(1);
  for (int p = 2; p <= kMostShares && 2 * p <= tiles && wgs * p <= 768; p *= 2) {
    const double c = cost(p);
    if (c < least) { least = c; best = p; }
  }
  return best;
}

usp_status launch_attn_generic(const AttnStep& step, hipStream_t st) {
  AttnStep s = step;
  if (s.d > 256) {
    set_error("generic attention kernel supports d <= 256 (got %d)", s.d);
    return USP_ERR_UNSUPPORTED;
  }
  if (s.n_multi == 0) {   // one chunk
    AttnStep::Chunk& c = s.chunk[0];
    c.k = s.k; c.v = s.v; c.Sc = s.Sc; c.ks0 = s.ks[0]; c.ks1 = s.ks[1];
    c.k_scale_src = s.k_scale; c.v_scale_src = s.v_scale; c.mask_src = s.key_mask;
    s.n_multi = 1;
  }
  s.copy_wgs = s.n_copy > 0 ? 32 : 0;
  if (s.parts > 1 && (s.mode != 0 || s.n_multi != 1 || s.copy_wgs != 0 || !s.part_o || !s.part_ml)) {
    set_error("a launch that shares keys between work-groups has one chunk, finishes the result and needs room for the shares");
    return USP_ERR_INVALID_ARG;
  }
  if (s.parts > kMostShares) {
    set_error("the keys of a query block are shared by at most %d work-groups (got %d)", kMostShares, s.parts);
    return USP_ERR_INVALID_ARG;
  }
  int64_t wgs;
  const bool few = few_work_groups(s.qo_dtype == USP_F32, s.B, s.H, s.Sq, s.d, &wgs);
  usp_status r;
  if (s.qo_dtype == USP_F32) r = launch_attn_generic_f32(s, few, st);
  else r = s.kv_dtype == USP_FP8_E4M3FN ? run_bf16_d<tile::UnitF8>(s, few, wgs, st) : run_bf16_d<tile::UnitBf16>(s, few, wgs, st);
  if (r != USP_OK || s.parts <= 1) return r;
  return s.qo_dtype == USP_F32 ? launch_tile_combine<float>(s, st) : launch_tile_combine<bf16_t>(s, st);
}

}  // namespace usp

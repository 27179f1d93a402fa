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
    // (d = 49 to 64 excepted).  us with direct tiles, through registers: 16 heads of 153 queries, 1793 keys, d = 40 21.7, 21.3 (masked
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
}  // namespace

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
  // Waves share queries where 64-query work-groups would leave CUs idle: H = 4, Sq = S = 1024 (64 of them): fp32
  // d = 64 53 -> 27 us, d = 128 100 -> 46 us, bf16 d = 72 30 -> 21 us.  At 192 work-groups the two are within
  // 20 %, at 256 fp32 loses (30 against 36 us).  The d = 256 sizes fill a CU's LDS with one work-group, so
  // sharing stops paying at half a chip of them (192: bf16 65 against 93 us, fp32 199 against 268 us).
  const int64_t wgs = (int64_t)((s.Sq + 63) / 64) * s.B * s.H;
  const bool few = wgs < (s.d > 160 || (s.qo_dtype == USP_F32 && s.d > 128) ? 160 : 256);
  if (s.qo_dtype == USP_F32) return launch_attn_generic_f32(s, few, st);
  return s.kv_dtype == USP_FP8_E4M3FN ? run_bf16_d<tile::UnitF8>(s, few, wgs, st) : run_bf16_d<tile::UnitBf16>(s, few, wgs, st);
}

}  // namespace usp

// fp32 Q (fp32 or FP8 K/V): attn_tile.h on the fp32 matrix instructions.
#include "attn_tile.h"

namespace usp {
namespace {
template <class Unit, int kD>
usp_status run_f32(const AttnStep& s, bool few, hipStream_t st) {
  return few ? tile::launch_tile_one<tile::F32Q, Unit, kD, kD / 16, 4, 4, false>(s, st) : tile::launch_tile_one<tile::F32Q, Unit, kD, kD / 16, 1, 4, false>(s, st);
}
template <class Unit>
usp_status run_f32_d(const AttnStep& s, bool few, hipStream_t st) {
  if (s.d <= 32) return run_f32<Unit, 32>(s, few, st);
  if (s.d <= 64) return run_f32<Unit, 64>(s, few, st);
  if (s.d <= 96) return run_f32<Unit, 96>(s, few, st);
  if (s.d <= 128) return run_f32<Unit, 128>(s, few, st);
  return run_f32<Unit, 256>(s, few, st);
}
}  // namespace

usp_status launch_attn_generic_f32(const AttnStep& s, bool few, hipStream_t st) {
  return s.kv_dtype == USP_FP8_E4M3FN ? run_f32_d<tile::UnitF8>(s, few, st) : run_f32_d<tile::UnitF32>(s, few, st);
}

}  // namespace usp

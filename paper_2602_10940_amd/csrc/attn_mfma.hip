// bf16 MFMA attention step for gfx950 (head dimension 128 or 64): for one KV chunk,
//   O_r = softmax(Q K^T * scale) V,   lse_r = log sum_j exp(q.k_j * scale)
// (FastUSP section 2.2 and 2.2.2), with the carried (O, lse) of earlier chunks folded in
// by the merge equations of section 3.4 in the epilogue.
//
// Shape of the computation (all choices are for 64-wide wavefronts and the 16x16x32 bf16 MFMA,
// whose A and B operands hold 8 consecutive contraction-index values per lane and whose 16 x 16
// result puts column (lane % 16), rows 4 * (lane / 16) .. +3 into a lane; under a full matrix load
// the chip holds a 13 % higher clock with this shape than with 32x32x16, which moves twice the
// accumulator data per flop):
//   * A work-group owns 256 queries of one (batch, head); each of its 8 waves owns 32, as two
//     16-query blocks.
//   * Scores are computed TRANSPOSED, S^T = K Q^T (keys are MFMA rows, queries columns), so
//     a lane owns one query column per block: the row max / row sum of the online softmax are in-lane
//     reductions plus two exchanges over the four lanes r, r+16, r+32, r+48.
//   * The exponentiated tile P^T, already in registers in the accumulator layout, is cast to
//     bf16 and used directly as the B operand of O^T += V^T P^T; it never touches LDS.  (The lane
//     that holds keys 16*mb + 4*g + i of a query is the lane that must supply contraction indices
//     8*g + j of the P.V step: the keys of a step are simply taken in that order on the V side.)
//   * K and V tiles (64 keys) sit in LDS as 64-byte pieces of rows, ordered so that an operand's address is one
//     register of the lane's plus an immediate (TileLayout); the V^T operand (8 keys of one head-dim column per
//     lane) comes from the LDS transposing read.
//   * O and l are rescaled lazily: only when a row max has outgrown the exponent reference.
//   * exp is taken in base 2 with scale * log2(e) folded into one FMA.
#include "usp_common.h"
#include "prefetch_copy.h"

namespace usp {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kD = 128;          // head dimension
constexpr int kWaves = 8;
constexpr int kThreads = kWaves * 64;
constexpr int kQPerWave = 32;
constexpr int kQPerWG = kWaves * kQPerWave;   // 256
constexpr int kQPerWGSplit = 4 * kQPerWave;     // 128: split kernel, two waves per 32 queries
constexpr int kTile = 64;        // keys per LDS tile

// K and V tiles in LDS.  A tile load moves 1 KB: a group of 4 rows (kHalfD, head dimension 64: 8 rows of 128 bytes).  Inside a
// group the 64-byte quarters (halves) of its rows follow one another, first all rows' first quarter, then all rows' second, ..:
// the quarter of an operand is then an immediate offset, as its key block is, and all reads of a tensor share one address register
// (V with kHalfD two; one form keeps V's rows whole, see kRowsV).  Four consecutive lanes of a load still fetch 64 consecutive bytes, which is what the address unit counts.
// What is left is that the rows a read touches together lie in different banks (64 of 4 bytes):
//   K: a 16-byte read takes the lanes 0-3, 12-15, 20-27, then 4-11, 16-19, 28-31, then the same of the upper half (measured, lane
//      against lane).  Rows r to r + 3 (r a multiple of 4) differ by 64 bytes; the 16-byte pieces of their 64 bytes are swapped by
//      XOR with swap_k(r / 4), which gives each of those sets of (rows, piece) a place of its own.
//   V: 32 lanes read 32 bytes of 8 rows by the transposing read: two groups, which lie 32 bytes more than 1 KB apart; kHalfD: one group,
//      whose rows 4 to 7 have the halves of their 64 bytes swapped.
// With rows of 256 bytes swizzled by XOR, as they were, K took 4 address registers and V 8, each a vector addition per phase, and
// every load set m0 for itself.
template <bool kHalfD>
struct TileLayout {
  static constexpr int kGroup = kHalfD ? 8 : 4;                    // rows that one load moves
  static constexpr int kPitchK = 1024, kPitchV = 1024 + (kHalfD ? 0 : 32);   // from a group to the next
  static __device__ __forceinline__ int swap_k(int four) { return ((four ^ (four >> 1)) & 1) << 1 | ((four >> 1) & 1); }   // 0 2 3 1
  static constexpr int kQuarter = kGroup * 64;                     // from a row's 64 bytes to its next
};
// Work-group -> (batch*head, query block) with the 8 XCDs of the chip in mind: consecutive
// work-group ids go to consecutive XCDs (id % 8), each with its own L2.  The (head, query block)
// items, head-major, are cut into 8 contiguous ranges of equal length, one per XCD: the query
// blocks of a head stay on one XCD (two where a range boundary falls inside a head), so its K/V
// is fetched from HBM once or twice instead of once per XCD, and every XCD gets the same number
// of work-groups whatever the head count.  The grid holds 8 * ceil(items / 8) ids; ids past the
// last item return false.
constexpr int kXcds = 8;
constexpr int kSplitBelowWGs = 128;   // use the key-split kernel when 256-query work-groups number at most this
__device__ __forceinline__ bool wg_to_tile(int attn_wgs, int nqb, int bh_total, int& bh, int& qb, int lead = 0) {
  const int id = blockIdx.x - lead;                   // the copy work-groups are the last ids of the grid, or the first `lead` (a multiple of 8)
  const int per_xcd = attn_wgs / kXcds;
  const int item = (id % kXcds) * per_xcd + id / kXcds;
  bh = item / nqb;
  qb = item - bh * nqb;
  return bh < bh_total;
}
static inline unsigned wg_grid_size(int nqb, int bh_total) {
  return (unsigned)(kXcds * ((bh_total * nqb + kXcds - 1) / kXcds));
}

// A query's values sit in the four lanes r, r + 16, r + 32, r + 48 (r = lane % 16): maximum / sum over them,
// left in all four (two swaps: rows of 16 lanes pairwise, then the halves of the wave).
__device__ __forceinline__ float xgroup_max(float x) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float xgroup_sum(float x) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Chunk result of one query from its running state (reference m in log2 units, sum l), merged with the
// carried lse of earlier chunks by the section 3.4 equations: the factor for this chunk's O~ (c_cur), the
// weight of the carried O (w_prev) and the new lse.
// `invalid`: the rows are not to be trusted (a chunk of the ring never arrived): O and lse become NaN,
// which no valid result is (a query whose keys are all masked gets O = 0, lse = -inf).
struct RowFinish { float c_cur, w_prev, lse_new; };
__device__ __forceinline__ RowFinish finish_row(const AttnStep& s, float m, float l, int64_t lse_row, bool invalid) {
  RowFinish f;
  float lse_r = -INFINITY;
  f.c_cur = 0.0f;
  if (l > 0.0f) { lse_r = (m + log2f(l)) * 0.69314718055994530942f; f.c_cur = 1.0f / l; }
  f.w_prev = 0.0f;
  f.lse_new = lse_r;
  if (s.mode >= 2) {
    const float lse_p = s.lse[lse_row];
    const float mm = fmaxf(lse_p, lse_r);
    if (mm == -INFINITY) { f.w_prev = 0.0f; f.c_cur = 0.0f; f.lse_new = -INFINITY; }
    else {
      f.lse_new = mm + logf(expf(lse_p - mm) + expf(lse_r - mm));
      f.w_prev = expf(lse_p - f.lse_new);
      f.c_cur *= expf(lse_r - f.lse_new);
    }
  }
  if (invalid) { f.c_cur = __builtin_nanf(""); f.lse_new = f.c_cur; }
  return f;
}

// Chunk result, merge and store.  In the accumulator layout a store would touch 16 rows with 16 or 32 bytes each, and the
// CU's one address unit takes a cycle per line and quad of lanes: the key-split work-groups, which once stored so, spent
// 6400 cycles there (and as many branches on the mode as stores).  So a wave turns its O~ tile through its own LDS
// region (a row pitch 16 bytes past a multiple of 128, so that rows do not all start in the same bank) and moves whole
// rows: 16 lanes (kHalfD: 8) x 32 bytes of fp32 or 16 bytes of bf16 per row.
//   wide : a wave has its own 32 queries; only it touches its region, and the LDS operations of one wave complete in
//          order, so no barrier is needed.
//   split: waves w and w + 4 hold the same 32 queries over different keys.  Both stage, and behind a barrier wave w puts the
//          two together for the first 16 queries, wave w + 4 for the others.
// kHalfD: head dimension 64: only the first four 16-wide blocks exist, rows are 64 wide everywhere.
constexpr int kEpiInfoB = kQPerWave * 32 + 16 * 16;       // per row: m, four partial sums l, factor of O~ (split) or the row's weights (wide); split: the 16 rows' weights
template <bool kHalfD>
struct EpiLayout {
  static constexpr int kPitch = (kHalfD ? 64 : kD) * 4 + 16;       // bytes per staged row
  static constexpr int kWaveB = kQPerWave * kPitch + kEpiInfoB;
};

// Rows 0 .. rows - 1 of the wave's share, of them `valid` (may be <= 0) exist.  a, b: the staged rows (b of the other half of
// the keys, split only); info: per row {weight of a, weight of b, scale, weight of the carry}.  kCarry: fold the carried O
// in; kF32: the result is the fp32 carry (or a part), dst32, else bf16.  row0: first row in the dense fp32 tensors.
template <bool kSplit, bool kHalfD, bool kCarry, bool kF32>
__device__ __forceinline__ void store_rows(const unsigned char* a, const unsigned char* b, const f32x4* info, int lane, int valid,
                                           const float* carry, float* dst32, bf16_t* dst16, int64_t stride16) {
  constexpr int kLPR = kHalfD ? 8 : 16, kRPI = 64 / kLPR;           // lanes per row, rows per instruction
  constexpr int kRows = kSplit ? 16 : kQPerWave, kRowF = kHalfD ? 64 : kD, kEpiPitch = EpiLayout<kHalfD>::kPitch;
  const int sub = lane / kLPR, c = lane % kLPR;
#pragma unroll
  for (int it = 0; it < kRows / kRPI; ++it) {
    const int rr = it * kRPI + sub;
    if (rr >= valid) continue;
    const f32x4 w = info[rr];
    f32x4 o[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      o[u] = *reinterpret_cast<const f32x4*>(a + rr * kEpiPitch + c * 32 + u * 16);
      if (kSplit) {
        const f32x4 p = *reinterpret_cast<const f32x4*>(b + rr * kEpiPitch + c * 32 + u * 16);
        o[u] = w[0] * o[u] + w[1] * p;
      }
      o[u] = o[u] * w[2];
    }
    if (kCarry) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const f32x4 p = *reinterpret_cast<const f32x4*>(carry + (int64_t)rr * kRowF + 8 * c + 4 * u);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[u][e] = fmaf(w[3], p[e], o[u][e]);
      }
    }
    if (kF32) {
#pragma unroll
      for (int u = 0; u < 2; ++u) *reinterpret_cast<f32x4*>(dst32 + (int64_t)rr * kRowF + 8 * c + 4 * u) = o[u];
    } else {
      // the final output is not read again here: a streaming store leaves no dirty line for the end of the kernel to
      // write back (the fp32 carry above is re-read by the next step and stays cached)
      const u32x4 v = {pack_bf16x2(o[0][0], o[0][1]), pack_bf16x2(o[0][2], o[0][3]), pack_bf16x2(o[1][0], o[1][1]), pack_bf16x2(o[1][2], o[1][3])};
      __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(dst16 + rr * stride16 + 8 * c));
    }
  }
}

// q0: the wave's first query (its pair's, in the split form).  lratio: factor of O~ beside 1 / l.  Every tile read of the work-group is behind a barrier.
template <bool kSplit, bool kHalfD>
__device__ __forceinline__ void finish_and_store(const AttnStep& s, f32x4 (&oacc)[8][2], const float (&m)[2], const float (&lsum)[2], const float (&lratio)[2],
                                                 int b, int h, int q0, int wave, int lane, unsigned char* smem, bool invalid, int part) {
  constexpr int kDB = kHalfD ? 4 : 8, kRowF = kHalfD ? 64 : kD, kEpiPitch = EpiLayout<kHalfD>::kPitch, kEpiWaveB = EpiLayout<kHalfD>::kWaveB;
  const int r = lane & 15, g = lane >> 4;
  const int64_t row0 = ((int64_t)b * s.H + h) * s.Sq;     // first row of this (batch, head) in lse / acc
  unsigned char* epi = smem + wave * kEpiWaveB;
  float* info = reinterpret_cast<float*>(epi + kQPerWave * kEpiPitch);
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int db = 0; db < kDB; ++db)                       // row 16*nb + r, head dims 16*db + 4*g .. +3
      *reinterpret_cast<f32x4*>(epi + (16 * nb + r) * kEpiPitch + (16 * db + 4 * g) * 4) = oacc[db][nb];
  const unsigned char* other = epi;
  f32x4* weights;                                          // of the rows this wave stores
  int first = q0;                                          // the first of them
  if (kSplit) {
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      if (g == 0) {
        info[8 * (16 * nb + r)] = m[nb];
        info[8 * (16 * nb + r) + 5] = lratio[nb];
      }
      info[8 * (16 * nb + r) + 1 + g] = lsum[nb];
    }
    __syncthreads();
    const int half = wave >> 2;                            // which 16 of the 32 queries
    first += 16 * half;
    const unsigned char* mine = smem + (wave & 3) * kEpiWaveB;   // the even tiles' half of the keys; then the odd ones'
    const unsigned char* theirs = mine + 4 * kEpiWaveB;
    const float* ia = reinterpret_cast<const float*>(mine + kQPerWave * kEpiPitch) + 8 * (16 * half + r);
    const float* ib = reinterpret_cast<const float*>(theirs + kQPerWave * kEpiPitch) + 8 * (16 * half + r);
    // Both under one reference, the larger of what the two have summed to (in log2 units) and not of their references,
    // which say little about it: one may lag its sum by 2^60 and more, the other lie 2^32 above.
    const float mA = ia[0], mB = ib[0], lA = (ia[1] + ia[2]) + (ia[3] + ia[4]), lB = (ib[1] + ib[2]) + (ib[3] + ib[4]);
    const float mm = fmaxf(mA + __builtin_amdgcn_logf(lA), mB + __builtin_amdgcn_logf(lB));
    const float wa = (lA == 0.0f) ? 0.0f : __builtin_amdgcn_exp2f(mA - mm);
    const float wb = (lB == 0.0f) ? 0.0f : __builtin_amdgcn_exp2f(mB - mm);
    const float l = wa * lA + wb * lB;
    const int qi = first + r;
    RowFinish f = finish_row(s, mm, l, row0 + min(qi, s.Sq - 1), invalid);
    if (s.parts > 1 && !invalid) f.c_cur = 1.0f;   // a part's O~, m and l are kept as they are (attn_combine_kernel)
    weights = reinterpret_cast<f32x4*>(epi + kQPerWave * (kEpiPitch + 32));
    if (g == 0) {
      weights[r] = f32x4{wa * ia[5], wb * ib[5], f.c_cur, f.w_prev};
      if (qi < s.Sq) {
        if (s.parts > 1) *reinterpret_cast<float2*>(s.part_ml + 2 * (part * (int64_t)s.B * s.H * s.Sq + row0 + qi)) = make_float2(mm, invalid ? f.c_cur : l);
        else s.lse[row0 + qi] = f.lse_new;
      }
    }
    epi = smem + (wave & 3) * kEpiWaveB + 16 * half * kEpiPitch;
    other = epi + 4 * kEpiWaveB;
  } else {
    weights = reinterpret_cast<f32x4*>(info);
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      const float l = xgroup_sum(lsum[nb]);
      const int qi = q0 + 16 * nb + r;
      const RowFinish f = finish_row(s, m[nb], l, row0 + min(qi, s.Sq - 1), invalid);
      if (g == 0) {
        weights[16 * nb + r] = f32x4{1.0f, 0.0f, f.c_cur * lratio[nb], f.w_prev};
        if (qi < s.Sq) s.lse[row0 + qi] = f.lse_new;
      }
    }
  }
  const int valid = s.Sq - first;
  bf16_t* dst16 = (bf16_t*)s.out + b * s.os[0] + h * s.os[1] + (int64_t)first * s.os[2];
  if (kSplit && s.parts > 1) {
    float* dst = s.part_o + ((int64_t)part * s.B * s.H * s.Sq + row0 + first) * kRowF;
    store_rows<kSplit, kHalfD, false, true>(epi, other, weights, lane, valid, nullptr, dst, nullptr, 0);
    return;
  }
  float* acc = s.acc + (row0 + first) * kRowF;             // (null, and not touched, in mode 0)
  if (s.mode == 0) store_rows<kSplit, kHalfD, false, false>(epi, other, weights, lane, valid, nullptr, nullptr, dst16, s.os[2]);
  else if (s.mode == 1) store_rows<kSplit, kHalfD, false, true>(epi, other, weights, lane, valid, nullptr, acc, nullptr, 0);
  else if (s.mode == 2) store_rows<kSplit, kHalfD, true, true>(epi, other, weights, lane, valid, acc, acc, nullptr, 0);
  else store_rows<kSplit, kHalfD, true, false>(epi, other, weights, lane, valid, acc, nullptr, dst16, s.os[2]);
}

// =============================================================================================
// Ping-pong kernels.
//
// The 8 waves form two groups (waves 0-3 = A, 4-7 = B; each SIMD hosts one wave of each; the
// register budget of 32 queries x 128 head dims per wave allows no more than these two).  A
// wave alternates between a softmax phase SM(t) (VALU only: scores of tile t -> bf16 P) and a
// matrix phase MM(t) (MFMA only: O += P(t) V(t), then the scores of its next tile).  The groups
// run half a period apart and a work-group barrier separates the phases, so in every phase one
// wave of each SIMD feeds the matrix core while the other does the exponentials.
//
// Two work decompositions (template parameter kSplit):
//   wide  : 256 queries per work-group, each wave its own 32; every wave visits every tile.
//             phase 2j   : A does SM(j),  B does MM(j-1)
//             phase 2j+1 : A does MM(j),  B does SM(j)
//   split : 128 queries per work-group, waves w and w+4 share 32 queries; group A takes the even
//           tiles, group B the odd ones, and the two partial (O~, m, l) are put together through
//           LDS at the end, sixteen of the 32 queries by each wave.  Twice the work-groups for half the time each: for Q shards too
//           small to fill the chip with 256-query work-groups.
//             phase p : the owner of tile p does SM(p), the other group MM(p-1)
// K and V tiles go through three LDS stages each (K four in the split form), written by direct global->LDS loads issued
// from the softmax phases (whose critical resource, the VALU, is not the matrix core's).
//
// Template parameter kExt: per-key scales of FP8 K (Algorithm 1, line 4, applied to the fp32 scores instead
// of to K).  The launch that decodes a chunk writes, per (batch, head, tile), a record of 64 factors
// c = k_scale * softmax_scale * log2(e), and the record follows its K tile through the LDS stages.  The
// scales of FP8 V are not applied here: V is widened to bf16 as round(code * v_scale) before the kernel
// runs (the dequantise step of Algorithm 1 in the working precision), because a multiply per P element
// would make the softmax phase, which issues from a single wave per SIMD, the longer of the two phases.
// K keeps its exact codes: its scale costs nothing inside the exponent's FMA, and rounding K would move
// the scores themselves.
//
// Template parameter kDead: some keys take no part (a key mask, a chunk length that is not a multiple of
// 64).  A work-group starts by turning masks and lengths into one 64-bit word per tile in LDS (bit = key
// lives; a mask is a byte per key, so that is one load per tile, all in flight together), from which it
// knows where the live keys end and, one scan of 64 words at a time, which tile is the next with a dead
// key.  A softmax phase compares its tile index with that one and nothing else; only a tile with dead keys
// reads its word and overwrites their scores with -inf.  The per-tile records of factor, bias and flag
// this replaced (1 KB a tile, written by a launch in front) cost that launch and its gap, 4 to 5 us a
// chunk, an LDS read per block of exponentials and 5 to 10 % of the kernel.  More tiles than the words'
// room (kMaxWords): every tile looks its keys up in global memory.
//
// Template parameter kMulti lets one launch cover a whole ring (Algorithm 2): the 64-key tiles of up
// to 16 chunks (a ragged one ends in a tile with dead keys) form one stream in ring order, a cursor maps a tile index to
// its chunk's pointer, and the running (O~, m, l) stays in registers from the first tile to the
// last, which is the merge of section 3.4 applied tile by tile.  With AttnStep::arrive set the
// launch also plays the ring's transfers: its first work-groups copy the chunks into staging
// buffers and count themselves on a per-chunk arrival counter (prefetch_copy.h), and an attention
// work-group waits for a chunk's count before it loads the chunk's first tile (wait_arrival).
// FP8 chunks (AttnStep::multi_fp8) are decoded by those work-groups on the way (Algorithm 1 line 4:
// K widened, V dequantised, the records above written) and attended by the record-reading form.
//
// kHalfD: head dimension 64 (see attn_pp_body).
// =============================================================================================
// 64 lanes x 16 bytes from an address per lane: lane i's 16 bytes land at lds_base + 16*i.  Issued through inline asm so
// the compiler does not serialise later LDS reads behind it; completion is awaited with an explicit vmcnt wait before the
// barrier that publishes the tile.
__device__ __forceinline__ void lds_dma16_lanes(const void* p, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds_base), "v"(p) : "memory", "m0");
}
// Two (kPair = 0: one) such loads, numbers j and j + 1 (j = 0 or 2) of a wave's share of a tile: load i's bytes land at lds_base + i * kPitch,
// and come from gbase + off + i * kPitch (an immediate offset counts on both sides).
template <int kPitch, int kPair>
__device__ __forceinline__ void lds_dma16_pair(const void* gbase, uint32_t off0, uint32_t off1, uint32_t lds_base, int j) {
  if (!kPair) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(lds_base), "v"(off0), "s"(gbase) : "memory", "m0");
  else if (j == 0)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %3\n\tglobal_load_lds_dwordx4 %2, %3 offset:%4"
                 :: "s"(lds_base), "v"(off0), "v"(off1), "s"(gbase), "n"(kPitch) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %3 offset:%4\n\tglobal_load_lds_dwordx4 %2, %3 offset:%5"
                 :: "s"(lds_base), "v"(off0), "v"(off1), "s"(gbase), "n"(2 * kPitch), "n"(3 * kPitch) : "memory", "m0");
}
// The same through a buffer descriptor (base, 0, bytes, flags): lanes that fall outside the descriptor's bytes load zeros.
template <int kPitch, int kPair>
__device__ __forceinline__ void lds_dma16_pair_bounded(u32x4 desc, uint32_t off0, uint32_t off1, uint32_t lds_base, int j) {
  if (!kPair) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(lds_base), "v"(off0), "s"(desc) : "memory", "m0");
  else if (j == 0)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %3, 0 offen lds\n\tbuffer_load_dwordx4 %2, %3, 0 offen offset:%4 lds"
                 :: "s"(lds_base), "v"(off0), "v"(off1), "s"(desc), "n"(kPitch) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %3, 0 offen offset:%4 lds\n\tbuffer_load_dwordx4 %2, %3, 0 offen offset:%5 lds"
                 :: "s"(lds_base), "v"(off0), "v"(off1), "s"(desc), "n"(2 * kPitch), "n"(3 * kPitch) : "memory", "m0");
}
__device__ __forceinline__ void lds_dma4(const void* gbase, uint32_t lane_off, uint32_t lds_base) {
  // the same with 4 bytes per lane: lane i's dword lands at lds_base + 4*i
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
               :: "s"(lds_base), "v"(lane_off), "s"(gbase) : "memory", "m0");
}
// Waits until at most kLoads of this wave's loads are in flight (and, if lgkm, none of its LDS operations)
template <int kLoads, bool kLds = false>
__device__ __forceinline__ void wait_loads() {
  if (kLds) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(kLoads) : "memory");
  else asm volatile("s_waitcnt vmcnt(%0)" :: "n"(kLoads) : "memory");
}
constexpr int kStages = 3, kStagesSplitK = 4;   // LDS tile buffers per tensor; of K in the key-split form
constexpr int kExtTileB = kTile * 4;   // bytes of one tile's record: the factors of its 64 keys

// LDS of a work-group: K stages | V stages (each with room for a record) | four records | the words of kDead launches (188 000 keys).
// The epilogue stages each wave's O tile (eight regions from offset 0, over everything else, which is dead by then).
constexpr int kMaxWords = 2944;
constexpr int kLdsAlign = 64;   // of the dynamic LDS: d = 64 finds the other half of a row's 64 bytes of V by XOR of the address with 32 (v_operand)
template <bool kHalfD>
struct LdsPlan {
  typedef TileLayout<kHalfD> L;
  static constexpr int kTileB = kTile / L::kGroup * (L::kPitchK > L::kPitchV ? L::kPitchK : L::kPitchV);
  static constexpr int kStageB = kTileB + kExtTileB;
  static constexpr int kQRowsB = kQPerWave / L::kGroup * L::kPitchK;     // 32 rows of Q, laid out as K is
  static constexpr int kExtOff = (kStagesSplitK + kStages) * kStageB;
  static constexpr int kWordsOff = kExtOff + 4 * kExtTileB;
  static constexpr int kEpilogueB = 8 * EpiLayout<kHalfD>::kWaveB;
  static constexpr int bytes(int words) { return kEpilogueB > kWordsOff + 8 * words ? kEpilogueB : kWordsOff + 8 * words; }
  static_assert(kStageB % kLdsAlign == 0 && L::kPitchV % (kHalfD ? kLdsAlign : 16) == 0, "rows of V are told apart by address bits");
  static_assert(2 * kQRowsB <= kTileB && kWordsOff % 8 == 0 && bytes(kMaxWords) <= 159 * 1024, "LDS plan");   // (some is left to __syncthreads_or)
};

// LDS transposing read: the 16 lanes of a group each name 8 bytes; seen as a 4 x 16 matrix of
// bf16 (row i = the data of lanes 4i..4i+3), lane j of the group receives column j.
__device__ __forceinline__ u32x2 lds_read_tr3(const __attribute__((address_space(3))) unsigned char* p) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  s16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p));
  return __builtin_bit_cast(u32x2, r);
}


// Wait of an attention work-group for a chunk that the copy work-groups of the same launch are still
// writing: polls the chunk's counter with device-scope loads until it is complete.  The copy
// work-groups are dispatched before every attention work-group and wait for nothing but the first of them, so the count
// is reached; the poll limit (of the order of a second by default) only keeps a launch from spinning
// forever should that ever not hold, at the price of a result the caller can recognise as invalid:
// every row of a work-group one of whose waves gave up is returned as NaN in out and lse.
constexpr int kArrivePolls = 1 << 21;
// kTagged: bf16 chunks.  FP8 chunks have a launch in front that sets the counters to zero (their tag), so that the count alone says
// it: with the tag looked at, rings of six to eight chunks of 320 to 350 keys took 1 to 2.5 % longer.
// (The counter's halves in the even and the odd lanes: a count read ahead then lives in one register.)
template <bool kTagged>
__device__ __forceinline__ uint32_t read_count(const uint64_t* counter) {
  uint32_t half = 0;
  if (kTagged) {   // (counted here, not kept from the start of the kernel)
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0" : "=v"(half));
    half &= 1;
  }
  return __hip_atomic_load(reinterpret_cast<const uint32_t*>(counter) + half, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <bool kTagged>
__device__ __forceinline__ bool has_arrived(const AttnStep& s, uint32_t halves) {
  // (what is computed from a count read ahead is computed here: anywhere else it would wait there for the loads in flight)
  asm volatile("" : "+v"(halves));
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)halves);
  if (!kTagged) return (int)lo >= s.arrive_need;
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)halves, 1);
  return hi == (uint32_t)(s.tag >> 32) && ((lo ^ (uint32_t)s.tag) >> 16) == 0 && (int)(lo & 0xffffu) >= s.arrive_need;
}
template <bool kTagged>
__device__ __forceinline__ bool wait_arrival(const AttnStep& s, int c) {
  for (int i = 0; i < s.arrive_polls; ++i) {
    if (has_arrived<kTagged>(s, read_count<kTagged>(s.arrive + c))) {
      asm volatile("" ::: "memory");
      return true;
    }
    __builtin_amdgcn_s_sleep(4);
  }
  return false;
}
__global__ __launch_bounds__(64) void attn_arrive_set_kernel(uint64_t* arrive, uint64_t tag) {
  if (threadIdx.x < AttnStep::kMaxMulti) arrive[threadIdx.x] = tag;
}
// A chunk decoded by a launch of its own (the first of a ring, which no attention
// work-group could overlap with anything; the chunk of a launch-per-chunk step).
__global__ __launch_bounds__(256) void attn_fp8_chunk_prepare_kernel(Fp8Chunk c) {
  if (c.arrive != nullptr && blockIdx.x == 0 && threadIdx.x < AttnStep::kMaxMulti) c.arrive[threadIdx.x] = 0;
  fp8_chunk_prepare(c, (int64_t)blockIdx.x * 256 + threadIdx.x);
}

// The live keys of tile t (of a launch's tile stream) as a word, by the lanes of a wave: bit = key takes part.
__device__ __forceinline__ uint64_t live_keys(const uint8_t* mask, int Sc, int t, int lane) {
  const int key = t * kTile + lane;
  bool live = key < Sc;
  if (live && mask != nullptr) live = mask[key] != 0;
  return __builtin_amdgcn_ballot_w64(live);
}

// The key-split forms of head dimension 64 fit 128 vector registers and half of the LDS: two work-groups to a CU, four waves
// to a SIMD, where the softmax phases, the longer ones there, overlap with one another.  (24 heads of 4608: 166.8 us with one
// work-group a CU, 141.5 with two; 256-query work-groups 157.)  Not FP8 chunks with dead keys or in one launch over a ring, whose factors
// would have to be read from LDS when they are needed (ring of eight of 2112 under 12 heads 170 -> 190 us).
constexpr bool four_waves(bool split, bool ext, bool multi, bool dead, bool half_d) { return split && half_d && !(ext && (multi || dead)); }
// One work-group's share: the queries q_base .. q_base + 255 (wide) or + 127 (split) of (batch, head) bh_.
// kHalfD: head dimension 64: rows of Q, K, V and O are 128 bytes (K and V are read in place; their LDS tiles: TileLayout), the scores contract over two 32-wide slices
// of the head dimension and P.V produces four 16-wide blocks.
template <bool kSplit, bool kExt, bool kMulti, bool kDead, bool kHalfD>
__device__ __forceinline__ void attn_pp_body(const AttnStep& s, unsigned char* smem_raw, int bh_, int q_base, int part) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keep it in an SGPR
  const int r = lane & 15, g = lane >> 4;   // MFMA column (a query) and 8-wide slice of the contraction index
  constexpr int kKS = kHalfD ? 2 : 4;        // 32-wide slices of the head dimension (contraction of the scores)
  constexpr int kNV = kHalfD ? 2 : 4;        // operands of either kind per block of the matrix phase
  constexpr int kDB = kHalfD ? 4 : 8;        // 16-wide blocks of the head dimension that P.V produces
  constexpr int kStagesK = kSplit ? kStagesSplitK : kStages;
  const int h = bh_ % s.H, b = bh_ / s.H;
  // split: waves w and w+4 share their 32 queries
  const int q0 = q_base + (kSplit ? (wave & 3) : wave) * kQPerWave;
  const bool grpA = wave < 4;

  constexpr bool kFour = four_waves(kSplit, kExt, kMulti, kDead, kHalfD);
  typedef TileLayout<kHalfD> Layout;
  typedef LdsPlan<kHalfD> Lds;
  constexpr int kStageB = Lds::kStageB, kQRowsB = Lds::kQRowsB;
  constexpr int RB = kHalfD ? 128 : 256;     // bytes per row of Q, K and V
  const uint32_t lds_base = (uint32_t)(uintptr_t)smem_raw;
  // this lane's row of a group that a load moves, and its byte in that row (K and Q, V)
  const int dma_i = (lane >> 2) & (Layout::kGroup - 1), dma_q = kHalfD ? lane >> 5 : lane >> 4;
  // kRowsV: V's rows stay whole in LDS, the 32-byte chunk c of row r at chunk c ^ (r >> 1 & 3), and each of the four chunks has an address
  // register.  For the 256-query form of d = 64 from FP8 with dead keys, which V in pieces makes slower, though counters of instructions, conflicts and
  // traffic are no higher (cycles that waves wait are); us with rows and V's load behind the first block (kVLate), and with pieces: 24 heads of 2400 queries,
  // 4500 keys 96.1, 100.6, 2112 keys of which 100 masked 49.3, 51.4; rings of two of 2215 87.4, 92.8, of three of 1345, 700 masked, 104.6, 107.8.  From
  // bf16 83.1, 78.9 the other way round (4500 keys).
  constexpr bool kRowsV = !kSplit && kHalfD && kExt && kDead;
  const int dma_iv = kRowsV ? lane >> 3 : dma_i;
  auto dma_k = [&](int group) -> uint32_t {   // (of the tile)
    return (uint32_t)(64 * dma_q + 16 * ((lane & 3) ^ Layout::swap_k(kHalfD ? 2 * group + (dma_i >> 2) : group)));
  };
  const uint32_t dma_v = kRowsV ? (uint32_t)(16 * ((lane & 7) ^ ((dma_iv >> 1 & 3) << 1)))
                                : (uint32_t)(64 * dma_q + 16 * ((lane & 3) ^ (kHalfD ? dma_i >> 2 << 1 : 0)));
  // ---- Q first, the longest way to the first score.  Its operand layout (16 rows x 64 bytes an instruction) would take the
  // CU's one address unit 64 cycles a load, 4000 for a work-group, so it is moved to LDS as K is and the operands are
  // read from there.  It lands in stages that no load in front of the second barrier uses, 32 rows for each half stage: split, the
  // rows of a pair of waves, half by each, in V stages 1 and 2; wide, a wave's own 32 rows in K stage 2, V stages 1
  // and 2 and the room behind them.
  const int q_slot = kSplit ? 2 * (kStagesK + 1) + (wave & 3) : wave < 2 ? 4 + wave : 6 + wave;
  const uint32_t q_lds = lds_base + (q_slot >> 1) * kStageB + (q_slot & 1) * kQRowsB;
  {
    const bf16_t* qb = (const bf16_t*)s.q + b * s.qs[0] + h * s.qs[1];
    constexpr int kGroups = (kSplit ? kQPerWave / 2 : kQPerWave) / Layout::kGroup;
    const int first = kSplit && !grpA ? kGroups : 0;
#pragma unroll
    for (int t = 0; t < kGroups; ++t)
      lds_dma16_lanes((const unsigned char*)(qb + (int64_t)min(q0 + (first + t) * Layout::kGroup + dma_i, s.Sq - 1) * s.qs[2]) + dma_k(first + t),
                      __builtin_amdgcn_readfirstlane(q_lds + (first + t) * Layout::kPitchK));
  }
  const unsigned char* kb = (const unsigned char*)((const bf16_t*)s.k + b * s.ks[0] + h * s.ks[1]);
  const unsigned char* vb = (const unsigned char*)((const bf16_t*)s.v + b * s.ks[0] + h * s.ks[1]);
  const float scale2 = s.scale * 1.44269504088896340736f;
  // without kDead the host guarantees whole tiles and at least one; with it, the tiles up to the last live
  // key are visited, and none may be left (nt == 0)
  auto tiles_of = [](int len) { return (len + kTile - 1) / kTile; };
  const int nt_all = s.tiles;
  const bool masked = s.any_mask != 0;
  int nt = nt_all;
  typedef const __attribute__((address_space(3))) uint64_t* lds_words;
  const lds_words words = (lds_words)(uintptr_t)((uint32_t)(uintptr_t)smem_raw + Lds::kWordsOff);
  const bool in_lds = kMulti || nt_all <= kMaxWords;   // (the host keeps several chunks below that)
  // the word of tile t where the words have no room in LDS
  auto word_from_memory = [&](int t) -> uint64_t {
    return live_keys(s.key_mask ? s.key_mask + (int64_t)b * s.Sc : nullptr, s.Sc, t, lane);
  };
  auto dead_word = [&](int t) -> uint64_t {
    if (!in_lds) return word_from_memory(t);
    const uint64_t w = words[t];
    return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)w) |
           (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(w >> 32)) << 32;
  };
  // first tile >= t of the launch's stream that has a dead key (nt_all or more: none)
  auto find_dead = [&](int t) -> int {
    if (!in_lds) return t;
    for (; t < nt_all; t += 64) {
      const bool dead = t + lane < nt_all && words[t + lane] != ~0ull;
      const uint64_t any = __builtin_amdgcn_ballot_w64(dead);
      if (any != 0ull) return t + __builtin_ctzll(any);
    }
    return t;
  };
  if (kDead) {
    if (in_lds) {
      int first = 0;
      for (int c = 0; c < (kMulti ? s.n_multi : 1); ++c) {
        const int len = kMulti ? s.chunk[c].Sc : s.Sc, ntc = tiles_of(len);
        const uint8_t* mask = kMulti ? s.chunk[c].mask_src : s.key_mask;
        if (mask != nullptr) mask += (int64_t)b * len;
        for (int t0 = wave; t0 < ntc; t0 += 8 * kWaves) {   // the loads of eight tiles in flight
          uint32_t live[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int key = (t0 + u * kWaves) * kTile + lane;
            live[u] = key < len ? 1u : 0u;
            if (mask != nullptr && key < len) live[u] = mask[key];
          }
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const uint64_t w = __builtin_amdgcn_ballot_w64(live[u] != 0u);
            if (lane == 0 && t0 + u * kWaves < ntc)
              *(__attribute__((address_space(3))) uint64_t*)(words + first + t0 + u * kWaves) = w;
          }
        }
        first += ntc;
      }
    }
    if (masked) {   // where the live keys end (without a mask every tile has one); the first barrier below publishes the words otherwise
      __syncthreads();
      nt = 0;
      if (in_lds) {
        for (int t0 = (nt_all - 1) / 64 * 64; t0 >= 0 && nt_all > 0; t0 -= 64) {
          const bool any_live = t0 + lane < nt_all && words[t0 + lane] != 0ull;
          const uint64_t any = __builtin_amdgcn_ballot_w64(any_live);
          if (any != 0ull) { nt = t0 + 64 - __builtin_clzll(any); break; }
        }
      } else {
        for (int t = nt_all; t > 0; --t)
          if (word_from_memory(t - 1) != 0ull) { nt = t; break; }
      }
      nt = __builtin_amdgcn_readfirstlane(nt);
    }
  }
  // this work-group's part of the tiles, t_beg .. nt - 1; tile indices below count from t_beg
  const int nt_live = nt;
  const bool parted = kSplit && s.parts > 1;
  const int t_beg = parted ? (int)((uint32_t)nt_live * (uint32_t)part / (uint32_t)s.parts) : 0;   // (at most 2^25 tiles and 16 parts)
  if (parted) nt = (int)((uint32_t)nt_live * (uint32_t)(part + 1) / (uint32_t)s.parts) - t_beg;

  f32x4 oacc[8][2];   // O~^T: [16-wide head-dim block db][16-query block nb]: head dims 16*db + 4*g + i of query 16*nb + r
#pragma unroll
  for (int db = 0; db < 8; ++db)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) oacc[db][nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  float m[2] = {-INFINITY, -INFINITY}, lsum[2] = {0.0f, 0.0f};   // per query block
  float lhat[2] = {0.0f, 0.0f};   // heavy: sums of the weights as bf16 has them (see kRefMargin)
  bool heavy = false;             // a reference has been outgrown (wave-uniform)
  bool late = false;   // an awaited chunk never arrived (see wait_arrival): the results are replaced by NaN
  int arrived_upto = kMulti && s.arrive != nullptr ? 0 : AttnStep::kMaxMulti;   // chunks known to have arrived
  int probe_c = 0;                     // the one whose count has been read ahead
  uint32_t probe_val = 0;
  constexpr int kProbeAheadTiles = 4;

  if (!kDead || nt > 0) {   // (uniform over the work-group)
  // ---- direct global->LDS tile loads, a group of rows per instruction.  wide: wave w moves rows 8w..8w+7 of every
  // tile.  split: only the group in its softmax phase loads, its wave w & 3 the rows 16 * (w & 3) .. + 15.  The loads of a wave and
  // tensor are kPitch apart in LDS, and as far by their immediate offset, which counts in global memory too and is
  // taken off the lanes' offsets again (kBias keeps those positive, for rows of RB bytes and more).
  // kDead: a tile is loaded through a descriptor that ends with its chunk, so that the rows past the end of a
  // ragged one arrive as zeros (finite data; their P is 0).
  constexpr int kLoads = (kSplit ? 16 : 8) / Layout::kGroup;   // a wave's, per tile and tensor
  constexpr uint32_t kBias = 128;
  static_assert(kBias >= 3 * (uint32_t)(Layout::kPitchV - 1024) && kBias >= 3 * (uint32_t)(Layout::kPitchK - 1024), "lane offsets");
  const int dma_row = kSplit ? 16 * (wave & 3) : 8 * wave;
  const uint32_t rowB = (uint32_t)(s.ks[2] * 2);   // bytes between keys in global memory
  const int64_t tileB = (int64_t)kTile * rowB;
  uint32_t k_off[kLoads], v_off[kLoads];
#pragma unroll
  for (int j = 0; j < kLoads; ++j) {
    const uint32_t row = (uint32_t)(dma_row + j * Layout::kGroup + dma_i) * rowB + kBias;
    k_off[j] = row + dma_k(dma_row / Layout::kGroup + j) - j * Layout::kPitchK;
    v_off[j] = (kRowsV ? (uint32_t)(dma_row + j * Layout::kGroup + dma_iv) * rowB + kBias : row) + dma_v - j * Layout::kPitchV;
  }
  const uint32_t lds_k = __builtin_amdgcn_readfirstlane(lds_base + dma_row / Layout::kGroup * Layout::kPitchK);
  const uint32_t lds_v = __builtin_amdgcn_readfirstlane(lds_base + kStagesK * kStageB + dma_row / Layout::kGroup * Layout::kPitchV);
  // The tiles are a stream, of one chunk or (kMulti) of chunks that follow one another, and a place in it is kept in scalar
  // registers: where K's and V's tile begin (less kBias), the rows their chunk has from there on, and the chunk.  A place that
  // has run past its chunk (left <= 0) is carried into the next one by enter().
  struct Place { uint64_t k, v; int left, c; };
  auto chunk_base = [&](int c, bool is_v) -> uint64_t {
    if (!kMulti) return (uint64_t)(uintptr_t)(is_v ? vb : kb) - kBias;
    const AttnStep::Chunk& ch = s.chunk[c];
    return (uint64_t)(uintptr_t)((const bf16_t*)(is_v ? ch.v : ch.k) + b * ch.ks0 + h * ch.ks1) - kBias;
  };
  auto enter = [&](Place& p) {
    if (!kMulti) return;
    while (p.left <= 0) {
      const int over = (-p.left) / kTile;   // whole tiles of the next chunk
      ++p.c;
      p.k = chunk_base(p.c, false) + over * tileB;
      p.v = chunk_base(p.c, true) + over * tileB;
      p.left = s.chunk[p.c].Sc - over * kTile;
      if (p.c > arrived_upto) {
        // the count read a few tiles ago usually settles it; otherwise poll
        const bool seen = probe_c == p.c && has_arrived<!kExt>(s, probe_val);
        if (!seen && !wait_arrival<!kExt>(s, p.c)) late = true;
        arrived_upto = p.c;
      }
    }
  };
  auto raw_place = [&](int idx) -> Place {   // idx tiles behind this work-group's first one
    idx += t_beg;
    return Place{chunk_base(0, false) + idx * tileB, chunk_base(0, true) + idx * tileB, (kMulti ? s.chunk[0].Sc : s.Sc) - idx * kTile, 0};
  };
  auto place = [&](int idx) -> Place {
    Place p = raw_place(idx);
    enter(p);
    return p;
  };
  // kDead: bytes of a tile's descriptor, which ends with the last row, not with the step to the one after it: 64 steps of 64 MB are 2^32
  auto tile_bytes = [&](int left) -> uint32_t { return (uint32_t)min(left, kTile) * rowB - (rowB - RB) + kBias; };
  // loads j and j + 1 (kHalfD, wide: the one) of a wave's share of a tile, to the stage that begins `stage` bytes behind the first
  constexpr int kPair = kLoads < 2 ? 0 : 1;
  auto issue_k = [&](uint64_t p, uint32_t bytes, int stage, int j) {
    if (kDead)
      lds_dma16_pair_bounded<Layout::kPitchK, kPair>(u32x4{(uint32_t)p, (uint32_t)(p >> 32) & 0xffffu, bytes, 0x00020000u}, k_off[j], k_off[j + kPair], lds_k + stage, j);
    else lds_dma16_pair<Layout::kPitchK, kPair>((const void*)(uintptr_t)p, k_off[j], k_off[j + kPair], lds_k + stage, j);
  };
  auto issue_v = [&](uint64_t p, uint32_t bytes, int stage, int j) {
    if (kDead)
      lds_dma16_pair_bounded<Layout::kPitchV, kPair>(u32x4{(uint32_t)p, (uint32_t)(p >> 32) & 0xffffu, bytes, 0x00020000u}, v_off[j], v_off[j + kPair], lds_v + stage, j);
    else lds_dma16_pair<Layout::kPitchV, kPair>((const void*)(uintptr_t)p, v_off[j], v_off[j + kPair], lds_v + stage, j);
  };
  auto issue_k_tile = [&](const Place& p, int stage) {   // this wave's share
#pragma unroll
    for (int j = 0; j < kLoads; j += 2) issue_k(p.k, kDead ? tile_bytes(p.left) : 0, stage * kStageB, j);
  };
  auto issue_v_tile = [&](const Place& p, int stage) {
#pragma unroll
    for (int j = 0; j < kLoads; j += 2) issue_v(p.v, kDead ? tile_bytes(p.left) : 0, stage * kStageB, j);
  };
  // kExt: the record of a tile, one load by the first wave of the loading group, together with its K tile (kMulti: whose place says
  // that the chunk has arrived, which the copy work-groups write it with).  Records lie behind the K tiles (split) or, four of
  // them, behind all stages.
  const uint32_t lds_ext = lds_base + (kSplit ? Lds::kTileB : Lds::kExtOff);
  uint64_t xpre = kExt ? (uint64_t)(uintptr_t)s.ext + ((int64_t)bh_ * nt_all + t_beg) * kExtTileB : 0;   // the record loaded next
  auto issue_ext = [&](int stage) {
    if ((wave & 3) != 0) return;
    uint32_t l4 = lane * 4;
    if (kFour) asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0\n\tv_lshlrev_b32 %0, 2, %0" : "=v"(l4));   // (counted here, not kept)
    lds_dma4((const void*)(uintptr_t)xpre, l4, lds_ext + stage);
  };

  // Tiles needed before the first loads of the softmax phases land are fetched here.
  //   wide : A's SM(j) prefetches K(j+2) (with its record) and V(j+1); B's SM(j), one phase later,
  //          K(j+3) and V(j+2).
  //   split: the softmax phase p prefetches K(p+3) with its record and V(p+1).
  // next K / V tile this wave prefetches; split: K(p+3) / V(p+1) of its group's first softmax phase, p = 0 (A) or 1 (B)
  const int kpre_idx = (kSplit ? 3 : 2) + (wave >> 2), vpre_idx = 1 + (wave >> 2);
  if (kMulti) touch_chunks();
  auto first_record = [&](int stage) {
    if (!kExt) return;
    issue_ext(stage);
    xpre += kExtTileB;
  };
  if (!kSplit) {
    const Place first = place(0);
    if (grpA) first_record(0);
    issue_k_tile(first, 0);
    issue_v_tile(first, 0);
    if (nt > 1) {                          // (V(1) and K(2): group B, once Q has left their place)
      const Place second = place(1);
      if (grpA) first_record(kExtTileB);
      issue_k_tile(second, 1);
    }
  } else if (grpA) {                       // a group moves whole tiles: each group two of them
    const Place first = place(0);
    first_record(0);
    issue_k_tile(first, 0);
    issue_v_tile(first, 0);
    xpre += 2 * kExtTileB;                 // (its first softmax phase loads record 3, the other group's record 4)
  } else {
    xpre += kExtTileB;
    if (nt > 1) {
      const Place second = place(1);
      first_record(kStageB);
      issue_k_tile(second, 1);
    }
    if (nt > 2) {
      const Place third = place(2);
      first_record(2 * kStageB);
      issue_k_tile(third, 2);
    }
    xpre += kExtTileB;
  }
  // The K tile that this wave loads next and, for the same softmax phase, the V tile: its way through the chunks is the K
  // tile's one phase later, so that only K's is looked after (look_up).  left_look: what is left of K's chunk when there is
  // something to do: at its end, or a few tiles in front of it, where the next chunk's count is read ahead.  (A lone wave issues
  // one instruction of any kind per 5 cycles or so.  With a place for each tensor, moved on and looked at by itself, stages as
  // numbers and a place looked up per record: 24 heads of 4608 3 % more, ring of eight chunks of 2112 under 12 heads 3.4 %, ragged ring
  // of two of 2215 5 %, on a box where the first took 235 us.)
  Place pre = raw_place(kpre_idx);
  uint64_t vpre = 0;
  uint32_t vpre_bytes = 0;
  auto first_v = [&]() {
    if (vpre_idx >= nt) return;
    const Place p = place(vpre_idx);
    vpre = p.v;
    vpre_bytes = tile_bytes(p.left);
  };
  constexpr int kPreStep = kSplit ? 2 : 1;   // tiles between two softmax phases of a wave
  const int64_t pre_step = kPreStep * tileB;
  // Not where the first chunk (from FP8, a part's first chunk: the other way costs whole rings of either 1 to 2 %, by the code that the compiler makes of it) has six tiles or
  // less: looked at in the first phases, the count is rarely there yet, and the wait for the loads behind it waits for its way to memory.  us a call, transfers inside,
  // looked at and not: key-split, 24 heads, 512 queries, two of 384 19.3, 16.8; 384 queries, FP8, two of 320 22.1, 19.3; 256-query, B = 2, 14 heads of 1308, two of 256
  // 22.5, 17.9, 12 of 1660, d = 64, FP8, two of 192 21.0, 16.9.  Where the count is there early it costs up to 4 %; seven and eight tiles the other way round 0.6 % more.
  int left_look = kMulti && s.arrive != nullptr && s.chunk[0].Sc - (kExt ? t_beg * kTile : 0) > 6 * kTile ? kProbeAheadTiles * kTile : 0;
  // (A number from here on, not a condition worked out anew in the loop: the 256-query form of d = 64 from FP8 took 1 to 5 % longer, B = 2, 22 heads of 832, six of 832 87.9, 91.9.)
  if (kMulti) asm volatile("" : "+s"(left_look));
  auto look_up = [&]() {
    if (pre.left <= 0) {
      enter(pre);
      vpre = pre.v - pre_step;
    }
    // a blocking poll at the boundary would cost a round trip to memory on the critical path
    const bool ahead = pre.c + 1 < s.n_multi && pre.c + 1 > arrived_upto && probe_c <= pre.c;
    left_look = ahead ? kProbeAheadTiles * kTile : 0;
    if (ahead && pre.left <= kProbeAheadTiles * kTile) {
      probe_c = pre.c + 1;
      probe_val = read_count<!kExt>(s.arrive + probe_c);
      left_look = 0;
    }
  };

  bf16x8 qreg[2][4];   // Q^T operand (B of S^T = K Q^T): lane (r, g) holds Q[q0 + 16*nb + r][32*ks + 8*g .. +7]
  f32x4 sacc[4][2];   // scores: [16-key block mb][16-query block nb]: keys 16*mb + 4*g + i of query 16*nb + r
  u32x4 pk[2][2];     // bf16 P as the B operand of P.V: [32-key step kk][nb]: keys 32*kk + 16*(j >> 2) + 4*g + (j & 3), j = 0..7

  // per-lane LDS read addresses (see TileLayout): stage, head-dim slice and key block are added to these, the latter two as immediates
  typedef const __attribute__((address_space(3))) unsigned char* lds_cptr;
  lds_cptr k_rd, v_rd[kRowsV ? 4 : 1];          // K: row r, dims 8*g .. +7; V
  {
    const int kr = r & (Layout::kGroup - 1);
    k_rd = (lds_cptr)(uintptr_t)(lds_base + r / Layout::kGroup * Layout::kPitchK + kr * 64 + ((g ^ Layout::swap_k(r >> 2)) << 4));
    const int vrow = 4 * g + (r >> 2), vr = vrow & (Layout::kGroup - 1);   // the key this lane names in a transposing read (plus 32*kk, plus 16)
    const uint32_t v0 = lds_base + kStagesK * kStageB + vrow / Layout::kGroup * Layout::kPitchV + vr * (kRowsV ? RB : 64) + 8 * (r & 3);
    v_rd[0] = (lds_cptr)(uintptr_t)(v0 + (kHalfD && !kRowsV ? (vr >> 2) * 32 : 0));
#pragma unroll
    for (int db = 0; db < (kRowsV ? 4 : 0); ++db) v_rd[db] = (lds_cptr)(uintptr_t)(v0 + ((db ^ (vr >> 1 & 3)) << 5));
  }
  // kExt: this lane's keys of a tile are rows 16*mb + 4*g + (0..3), mb = 0..3
  const lds_cptr x_rd = (lds_cptr)(uintptr_t)(lds_ext + 16 * g);
  // (stages below are bytes behind the first stage: of K, of V, of the records)

  // LDS operands.  K: keys 16*mb .. +15 (MFMA rows), head dims 32*ks + 8*g .. +7: one 16-byte read.
  // V^T: head dims 16*db .. +15 (MFMA rows), keys of step kk in the order of pk: two transposing reads of
  // four keys each (rows 32*kk + 4*g + i and 32*kk + 16 + 4*g + i).
  auto k_operand = [&](int stage, int mb, int ks) -> bf16x8 {
    return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(k_rd + stage + 16 / Layout::kGroup * mb * Layout::kPitchK + ks * Layout::kQuarter);
  };
  auto v_operand = [&](int stage, int kk, int db) -> bf16x8 {
    // (kHalfD: the other 32 bytes of the lane's 64, whichever they are)
    const lds_cptr q = v_rd[kRowsV ? db & 3 : 0] + stage;
    const lds_cptr p = kRowsV ? q : (kHalfD && (db & 1) ? (lds_cptr)(uintptr_t)((uint32_t)(uintptr_t)q ^ 32) : q + (kHalfD ? 0 : 32 * (db & 1))) + (db >> 1) * Layout::kQuarter;
    const u32x2 lo = lds_read_tr3(p + 32 / Layout::kGroup * kk * Layout::kPitchV);
    const u32x2 hi = lds_read_tr3(p + (32 * kk + 16) / Layout::kGroup * Layout::kPitchV);
    return __builtin_bit_cast(bf16x8, u32x4{lo[0], lo[1], hi[0], hi[1]});
  };
  const f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
  // kExt: the per-key factor c replaces the uniform scale of the softmax phase.  c of the second key step is fetched while the first is computed,
  // of the first (kAhead) in the matrix phase before, so that the softmax phase, the longer one here, does not begin with a wait: FP8
  // ring of four chunks of 1152 under 24 heads 70.0 -> 67.9 us, of eight of 2112 under 12 heads, d = 64 164 -> 157.  Not where a SIMD holds four
  // waves, and not in 256-query work-groups of d = 64 (24 heads of 4608 165 -> 168).
  constexpr bool kAhead = kExt && !kFour && (kSplit || !kHalfD);
  auto x_vec = [&](int stage, int mb) -> f32x4 {   // c of keys 16*mb + 4*g + (0..3)
    return *reinterpret_cast<const __attribute__((address_space(3))) f32x4*>(x_rd + stage + 64 * mb);
  };
  f32x4 xc[2][2];
  auto x_load = [&](int kk, int xs) {
#pragma unroll
    for (int a = 0; a < 2; ++a) xc[kk][a] = x_vec(xs, 2 * kk + a);
  };
  // matrix phase: O += P V (V tile in stage sv) interleaved with the scores of the next tile (K in
  // stage sk), in four blocks of sixteen MFMAs: block b takes kNV V^T operands (key step b >> 1, head-dim
  // blocks kNV * (b & 1) ..) and kNV K operands (head-dim slice b, all key blocks; kHalfD: key block b, both slices), each
  // operand feeding two MFMAs (the wave's two 16-query blocks).  Head dimension 128: the two change their order from operand to
  // operand, so that from one MFMA to the next one of the two operands stays, which the chip, at its power limit, pays back in
  // clock (24 heads of 4608 226 -> 224.6 us, a ring of eight chunks of 2112 226.3 -> 223.6).
  // Only this wave feeds the SIMD's matrix core during the phase, so its LDS operand reads run one
  // block ahead of their use.  The order is written out and pinned (sched_barrier after every operand's
  // MFMAs and the reads issued behind them) rather than left to the instruction scheduler.
  // (The softmax phase is the one with the raised priority: what it loses to the matrix phase's issue beside it, it
  // loses in full, while the matrix core has work queued.  24 heads of 4608 queries and keys 225 -> 218 us against the other way round.)
  // (kAhead: the first factors of that tile, whose record lies in stage xs, are read while the last operands are used.)
  auto MM_full = [&](int sv, int sk, int xs) {
    __builtin_amdgcn_s_setprio(0);
    bf16x8 va[2][kNV], ka[2][kNV];
#pragma unroll
    for (int i = 0; i < kNV; ++i) va[0][i] = v_operand(sv, 0, i);
#pragma unroll
    for (int i = 0; i < kNV; ++i) ka[0][i] = kHalfD ? k_operand(sk, 0, i) : k_operand(sk, i, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int blk = 0; blk < 4; ++blk) {
      const int c = blk & 1, kk = blk >> 1;
      const bf16x8 pb0 = __builtin_bit_cast(bf16x8, pk[kk][0]), pb1 = __builtin_bit_cast(bf16x8, pk[kk][1]);
#pragma unroll
      for (int j = 0; j < kNV; ++j) {
        const int db = kNV * (blk & 1) + j;
        if (!kHalfD && (j & 1)) oacc[db][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[c][j], pb1, oacc[db][1], 0, 0, 0);
        oacc[db][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[c][j], pb0, oacc[db][0], 0, 0, 0);
        if (kHalfD || !(j & 1)) oacc[db][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[c][j], pb1, oacc[db][1], 0, 0, 0);
        if (!kHalfD) __builtin_amdgcn_sched_barrier(0);
        if (blk < 3) va[c ^ 1][j] = v_operand(sv, (blk + 1) >> 1, kNV * ((blk + 1) & 1) + j);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int j = 0; j < kNV; ++j) {             // (kNV is both the key blocks and, or for kHalfD, the head-dim slices)
        if (kAhead && blk == 3 && j == 0) x_load(0, xs);
        const int mb = kHalfD ? blk : j, ks = kHalfD ? j : blk;
        if (!kHalfD && (j & 1)) sacc[mb][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[c][j], qreg[1][ks], ks == 0 ? zero4 : sacc[mb][1], 0, 0, 0);
        sacc[mb][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[c][j], qreg[0][ks], ks == 0 ? zero4 : sacc[mb][0], 0, 0, 0);
        if (kHalfD || !(j & 1)) sacc[mb][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[c][j], qreg[1][ks], ks == 0 ? zero4 : sacc[mb][1], 0, 0, 0);
        if (!kHalfD) __builtin_amdgcn_sched_barrier(0);
        if (blk < 3) ka[c ^ 1][j] = kHalfD ? k_operand(sk, blk + 1, j) : k_operand(sk, j, blk + 1);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __builtin_amdgcn_s_setprio(1);
  };
  auto MM_last = [&](int sv) {   // last tile: no further scores; the reads run two blocks ahead
    __builtin_amdgcn_s_setprio(0);
    bf16x8 va[4][kNV];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int i = 0; i < kNV; ++i) va[blk][i] = v_operand(sv, blk >> 1, kNV * (blk & 1) + i);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int blk = 0; blk < 4; ++blk) {
      const int kk = blk >> 1;
      const bf16x8 pb0 = __builtin_bit_cast(bf16x8, pk[kk][0]), pb1 = __builtin_bit_cast(bf16x8, pk[kk][1]);
#pragma unroll
      for (int i = 0; i < kNV; ++i) {
        const int db = kNV * (blk & 1) + i;
        oacc[db][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[blk][i], pb0, oacc[db][0], 0, 0, 0);
        oacc[db][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[blk][i], pb1, oacc[db][1], 0, 0, 0);
        if (blk < 2) va[blk + 2][i] = v_operand(sv, (blk + 2) >> 1, kNV * (blk & 1) + i);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __builtin_amdgcn_s_setprio(1);
  };
  // softmax phase: sacc (scores of one tile) -> pk (bf16 P), running references m and sums l of the
  // lane's two queries.
  // Fast path: exponentials are taken against the current reference m without first looking for
  // the tile's maximum; the row sum then certifies the result: if this lane's sum of P is at most
  // 2^60, no P exceeded 2^60, and neither l (at most 2^60 per key) nor O~ (at most 2^60 |v| per key)
  // leaves the fp32 range (2^127) over 2^20 keys with |v| up to 2^40; a reference that lags the
  // maximum by D only scales P, l and O~ by 2^D, which floating point carries without loss.  Only
  // when some lane fails that test (always on a first tile with dead keys, where m = -inf makes every P inf or NaN)
  // does the wave find the true maximum, move m, rescale O and l, and redo the exponentials.
  // While it runs, the wave also issues its tile loads, spread between the exponential blocks so
  // that the waves do not hit the load path at once.
  // one block: the 8 scores of query block nb over key step kk -> pk[kk][nb]
  auto exp_block = [&](int kk, int nb, float& psum, int xs, bool fetch_ahead) {   // (key step 0 begins the sum)
    float p[8];
    if (!kExt) {
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          p[4 * a + e] = __builtin_amdgcn_exp2f(fmaf(sacc[2 * kk + a][nb][e], scale2, -m[nb]));
          psum = kk == 0 && a == 0 && e == 0 ? p[0] : psum + p[4 * a + e];
        }
    } else {
      // blocks run in the order (0,0) (0,1) (1,0) (1,1)
      if (fetch_ahead && kk == 0 && nb == (kFour ? 0 : 1)) x_load(1, xs);
#pragma unroll
      for (int a = 0; a < 2; ++a) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          p[4 * a + e] = __builtin_amdgcn_exp2f(fmaf(sacc[2 * kk + a][nb][e], xc[kk][a][e], -m[nb]));
          psum = kk == 0 && a == 0 && e == 0 ? p[0] : psum + p[4 * a + e];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) pk[kk][nb][j] = pack_bf16x2(p[2 * j], p[2 * j + 1]);
    // anchor the block here, between the tile loads that surround it in program order
    if (kFour) asm volatile("" : "+v"(pk[kk][nb]), "+v"(psum));   // (with its sum: summed later, all of the block's terms would stay in registers)
    else asm volatile("" : "+v"(pk[kk][nb]));
  };
  // largest exponent argument (before the reference is subtracted) of each of this lane's two queries over the tile
  auto tile_max = [&](int xs, float (&tmax)[2], bool do0 = true, bool do1 = true) {
    tmax[0] = tmax[1] = -INFINITY;
    if (!kExt) {
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
          for (int e = 0; e < 4; ++e) tmax[nb] = fmaxf(tmax[nb], sacc[mb][nb][e]);
      tmax[0] = xgroup_max(tmax[0]) * scale2;
      tmax[1] = xgroup_max(tmax[1]) * scale2;
      return;
    }
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
      const f32x4 c = x_vec(xs, mb);
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (nb ? do1 : do0) tmax[nb] = fmaxf(tmax[nb], sacc[mb][nb][e] * c[e]);
    }
    if (do0) tmax[0] = xgroup_max(tmax[0]);
    if (do1) tmax[1] = xgroup_max(tmax[1]);
  };
  // O~ and l of query block nb, for a reference that moves on.  (2^-126, the least factor that is not 0, takes what was summed
  // under a reference that lagged by 2^60 to 2^-34 of the 2^-32 that the new largest weight has.)
  auto rescale = [&](int nb, float alpha) {
    lsum[nb] *= alpha;
    lhat[nb] *= alpha;
#pragma unroll
    for (int db = 0; db < 8; ++db)
#pragma unroll
      for (int e = 0; e < 4; ++e) oacc[db][nb][e] *= alpha;
  };
  constexpr float kCertifiedSum = 1152921504606846976.0f;   // 2^60
  // A reference is set this far ABOVE the maximum that moved it: the largest P is then 2^-32
  // instead of 1, which fp32 sums and bf16 P carry as well (every P, l and O~ is scaled by the same
  // power of two; P V stays a normal number for |V| down to 2^-94), and a later score has to exceed the maximum seen so far
  // by 2^92, not 2^60, before the reference has to move again.  No tile looks for its maximum first, not even after a move.
  // (2^64 for the references that replace an outgrown one, as scores with heavy tails have them, x20 outliers in Q and K,
  // makes a third one rarer, but leaves nothing of O for V of 2^-90.)
  // Heavy tails also make a row mostly one key, whose weight, far from the reference, is no power of two: what it loses
  // to bf16 would be the row's error.  So O is divided by the sum of the weights as they multiply V, lhat, and lse alone
  // comes from their sum in fp32: against 64 bits 1.26e-3 of O instead of 1.84e-3 (12 heads of 4096 queries and keys with
  // such outliers; 24 heads, FP8 ring of two 1.55e-3 instead of 2.02e-3), for 8 of 113 and 18 of 436 us.  Summed here, where registers are
  // free: in the matrix phase it spills, and sums on the matrix cores take as long.
  constexpr float kRefMargin = 32.0f;
  int sm_tile = t_beg + (kSplit && !grpA ? 1 : 0);   // kDead: tile of this wave's next softmax phase
  int next_dead = 0;                         // kDead: the next tile with a dead key, as far as it has been looked up
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  // (kFarOff: what ordinary scores never reach lies outside the loop over the tiles.  FP8 ring of three chunks of 1152 keys,
  // 12 heads, d = 64, 45.8 -> 43.8 us; in the 256-query form, which has no register to spare, that spills, and the mixed
  // launch, which holds both, takes 447 us instead of 435 on 24 heads of 4096 queries, FP8 ring of two with outliers.)
  constexpr bool kFarOff = kSplit && kMulti;
  // The exponentials of the query blocks do0, do1 (constants) again if one of their lanes failed (fail0, fail1).
  // had: some lane has had a reference before this tile
  auto redo = [&](bool do0, bool do1, uint64_t fail0, uint64_t fail1, uint64_t had, int xs, float (&psum)[2]) {
    if (!heavy && had != 0ull) {
      heavy = true;
      lhat[0] = lsum[0];
      lhat[1] = lsum[1];
    }
    float tmax[2];
    tile_max(xs, tmax, do0, do1);
    if (kExt) { x_load(0, xs); x_load(1, xs); }
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      if (!(nb ? do1 : do0) || (nb ? fail1 : fail0) == 0ull) continue;
      const float m_new = tmax[nb] > m[nb] ? tmax[nb] + kRefMargin : m[nb];
      // m = -inf (first live tile) gives the factor 0; no live key so far: nothing to rescale, P = 0
      rescale(nb, m_new == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m[nb] - m_new));
      m[nb] = m_new;
      psum[nb] = 0.0f;
      if ((kExt || kDead) && m_new == -INFINITY) {
        pk[0][nb] = u32x4{0u, 0u, 0u, 0u};
        pk[1][nb] = u32x4{0u, 0u, 0u, 0u};
      } else {
        exp_block(0, nb, psum[nb], xs, false);
        exp_block(1, nb, psum[nb], xs, false);
      }
    }
  };
  auto failed = [&](float sum) -> uint64_t { return __builtin_amdgcn_ballot_w64(!(sum <= kCertifiedSum)); };
  auto has_reference = [&]() -> uint64_t { return __builtin_amdgcn_ballot_w64(m[0] != -INFINITY || m[1] != -INFINITY); };
  // SM of the tile whose record sits in stage xs; loads the next K tile into stage sk and, if do_x, its record into stage xst (if do_k), and the
  // next V tile into stage sv (if do_v)
  auto SM = [&](int xs, int sk, int sv, bool do_k, bool do_v, bool do_x, int xst) {
    float psum[2] = {0.0f, 0.0f};
    if (kExt && !kAhead) x_load(0, xs);
    if (kDead) {
      if (sm_tile >= next_dead) {
        if (next_dead < sm_tile) next_dead = find_dead(sm_tile);
        if (next_dead == sm_tile) {
          // (any positive finite factor keeps -inf, and exp2 makes it 0)
          const uint64_t live = dead_word(sm_tile) >> (4 * g);
#pragma unroll
          for (int mb = 0; mb < 4; ++mb) {
            const uint32_t bits = (uint32_t)(live >> (16 * mb));   // bit e: key 16*mb + 4*g + e
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const bool keep = (bits & (1u << e)) != 0u;
              sacc[mb][0][e] = keep ? sacc[mb][0][e] : -INFINITY;
              sacc[mb][1][e] = keep ? sacc[mb][1][e] : -INFINITY;
            }
            __builtin_amdgcn_sched_barrier(0);   // one block's lane masks at a time: sixteen pairs of scalar registers are not to be had
          }
          next_dead = find_dead(sm_tile + 1);
        }
      }
      sm_tile += kPreStep;
    }
    // sched_barrier: keep each load between two blocks of arithmetic (the scheduler would
    // otherwise hoist all of them to the top, where they queue behind one another)
    auto load_k = [&]() {
      if (!do_k) return;
      if (kMulti && pre.left <= left_look) look_up();
      if (kDead) vpre_bytes = tile_bytes(pre.left);
      issue_k(pre.k, vpre_bytes, sk, 0);
    };
    auto load_record = [&]() {
      if (kExt && do_k && do_x) issue_ext(xst);
    };
    // (kVLate: V's load stands behind the first block too.  256-query form of d = 64, bf16, us so and with that load in front: 24 heads of 2400 queries,
    // 4608 keys 79.7, 81.8, 576 keys 13.8, 14.2, 4500 keys 78.9, 81.3; ring of two of 2215 80.5, 82.9.  From FP8, whole tiles, 94.0, 90.6 the other way round.)
    constexpr bool kVLate = !kSplit && kHalfD && (!kExt || kDead);
    if (do_v && !kVLate) issue_v(vpre, vpre_bytes, sv, 0);
    if (kFour && kExt) {
      // one query block after the other: the first one's scores are done with when the second one's exponentials begin
      exp_block(0, 0, psum[0], xs, true);
      __builtin_amdgcn_sched_barrier(0);
      load_k();
      exp_block(1, 0, psum[0], xs, false);
      __builtin_amdgcn_sched_barrier(0);
      const uint64_t fail0 = failed(psum[0]);
      uint64_t had = 0ull;
      if (__builtin_expect(fail0 != 0ull, 0)) {
        had = has_reference();
        redo(true, false, fail0, 0ull, had, xs, psum);
      }
      load_record();
      exp_block(0, 1, psum[1], xs, false);
      __builtin_amdgcn_sched_barrier(0);
      exp_block(1, 1, psum[1], xs, false);
      __builtin_amdgcn_sched_barrier(0);
      const uint64_t fail1 = failed(psum[1]);
      if (__builtin_expect(fail1 != 0ull, 0)) redo(false, true, 0ull, fail1, fail0 != 0ull ? had : has_reference(), xs, psum);
    } else {
      exp_block(0, 0, psum[0], xs, true);
      __builtin_amdgcn_sched_barrier(0);
      if (do_v && (kVLate || kLoads > 2)) issue_v(vpre, vpre_bytes, sv, kVLate ? 0 : 2);
      exp_block(0, 1, psum[1], xs, true);
      __builtin_amdgcn_sched_barrier(0);
      load_k();
      exp_block(1, 0, psum[0], xs, true);
      __builtin_amdgcn_sched_barrier(0);
      if (do_k && kLoads > 2) issue_k(pre.k, vpre_bytes, sk, 2);
      load_record();
      exp_block(1, 1, psum[1], xs, true);
      __builtin_amdgcn_sched_barrier(0);
    }
    pre.k += pre_step;
    if (kMulti || kDead) pre.left -= kPreStep * kTile;
    vpre += pre_step;
    if (kExt) xpre += kPreStep * kExtTileB;
    // (per query block: a block all of whose lanes passed keeps its exponentials and its reference)
    if (!(kFour && kExt)) {
      const uint64_t fail0 = failed(psum[0]), fail1 = failed(psum[1]);
      if (kFarOff ? __builtin_expect((fail0 | fail1) != 0ull, 0) : (fail0 | fail1) != 0ull)
        redo(true, true, fail0, fail1, heavy ? 0ull : has_reference(), xs, psum);
    }
    lsum[0] += psum[0];
    lsum[1] += psum[1];
    if (kFarOff ? __builtin_expect(heavy, 0) : heavy) {
      bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3f803f80u);
      asm volatile("" : "+v"(ones));   // (as an inline constant it would not be that pair)
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
          const uint32_t w = pk[i >> 2][nb][i & 3];
          lhat[nb] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), ones, lhat[nb], false);
        }
    }
    // pin the results here: without a use in this phase the optimiser sinks the exponentials past
    // the barrier, next to their first use in the matrix phase
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) asm volatile("" : "+v"(pk[kk][nb]));
    asm volatile("" : "+v"(lsum[0]), "+v"(lsum[1]), "+v"(lhat[0]), "+v"(lhat[1]));
  };
  auto first_scores = [&](int stage) {   // (of tile `stage`)
    stage *= kStageB;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
      sacc[mb][0] = zero4;
      sacc[mb][1] = zero4;
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks) {
        const bf16x8 a = k_operand(stage, mb, ks);
        sacc[mb][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qreg[0][ks], sacc[mb][0], 0, 0, 0);
        sacc[mb][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qreg[1][ks], sacc[mb][1], 0, 0, 0);
      }
    }
  };

  // prologue: Q has landed and is read, then the tiles of the first scores
  {
    constexpr int kTL = kLoads;   // a wave's loads per tile
    if (kSplit) {
      if (grpA || nt > 2) wait_loads<2 * kTL>();
      else wait_loads<0>();
      __builtin_amdgcn_s_barrier();                  // (each wave of a pair has moved half of their rows)
      asm volatile("" ::: "memory");
    } else if (nt > 1) wait_loads<3 * kTL>();
    else wait_loads<2 * kTL>();
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks)
        qreg[nb][ks] = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(k_rd + (q_lds - lds_base) + 16 / Layout::kGroup * nb * Layout::kPitchK + ks * Layout::kQuarter);
    if (kSplit) {
      if (grpA || nt > 2) wait_loads<kTL, true>();
      else wait_loads<0, true>();
    } else if (nt > 1) wait_loads<2 * kTL, true>();
    else wait_loads<kTL, true>();
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks) asm volatile("" : "+v"(qreg[nb][ks]));
  }
  if (kDead) {
    __syncthreads();                      // (orders the words too)
    next_dead = find_dead(t_beg);
  } else {
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }
  // The reference of the first tile, unless it has dead keys (its softmax phase then finds the maximum, after the
  // exponentials against the reference -inf have failed the certification).  sm_tile: that tile.
  auto first_reference = [&](int xs) {
    if (kDead && next_dead <= sm_tile) return;
    float tmax[2];
    tile_max(xs, tmax);
    m[0] = tmax[0] + kRefMargin;
    m[1] = tmax[1] + kRefMargin;
  };

  __builtin_amdgcn_s_setprio(1);
  if (!kSplit) {
    first_scores(0);   // scores of tile 0 in both groups
    first_reference(0);
    wait_loads<0>();   // V(0), K(1): published by the barrier in front of A's matrix phase
    if (!grpA) {
      if (nt > 1) issue_v_tile(place(1), 1);
      if (nt > 2) issue_k_tile(place(2), 2);
    }
    first_v();
    // Both groups execute the same barrier sequence (two per tile index j = 0..nt); the steady-state
    // bodies are straight-line code so the accumulators stay in place.
    // sched_barrier(0): nothing may be moved across a phase boundary (the compiler would otherwise
    // sink the softmax arithmetic below the barrier, into the matrix phase of the same wave).
    // A wave waits for its own tile loads at the end of its softmax phases: the batch issued one
    // softmax phase earlier must have landed, the batch just issued (if full: 4 loads, 5 with a
    // record) may be in flight.
    // Only the barrier in front of A's matrix phase / B's softmax phase is needed (the other phase
    // boundaries pass needed = false and only order the instruction stream): with
    // three stages no load of the half-period after it overwrites what that half-period or the one
    // before the next barrier still reads, and every tile is waited for by its loaders before the
    // barrier in front of its first reader.  The second barrier only kept the groups in step, which
    // equal phase lengths do by themselves.  The key records are read in the softmax phases of both
    // halves, so they go round four stages (tile j in stage j % 4): record j+2 then replaces record
    // j-2, last read in phase 2j-3, in phase 2j, with the barrier of tile j-1 between the two.
    auto phase_barrier = [&](int wait_mode, bool needed = true) {   // 0: no wait, 1: all but the last full batch, 2: vmcnt(0)
      __builtin_amdgcn_sched_barrier(0);
      if (wait_mode == 1) {
        // a full batch is 4 loads (2 with 128-byte rows), plus the record's in the wave that loads it
        if (kExt && wave == 0) __builtin_amdgcn_s_waitcnt(kHalfD ? 0x0F73 : 0x0F75);   // vmcnt(3) / vmcnt(5)
        else __builtin_amdgcn_s_waitcnt(kHalfD ? 0x0F72 : 0x0F74);                // vmcnt(2) / vmcnt(4)
      } else if (wait_mode == 2) __builtin_amdgcn_s_waitcnt(0x0F70);
      if (needed) __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    };
    // LDS stages of tiles j, j + 1 and j + 2 (mod 3), and the record's of tile j (mod 4)
    int st = 0, s1 = kStageB, s2 = 2 * kStageB, xs = 0;
    auto next_tile = [&]() {
      const int sp = st;
      st = s1; s1 = s2; s2 = sp;
      xs = (xs + kExtTileB) & (3 * kExtTileB);
    };
    if (kAhead) x_load(0, 0);
    if (grpA) {
      // tile j: phase 2j = SM(j), prefetching K(j+2) and its record -> stage st+2, V(j+1) -> stage st+1;
      //         phase 2j+1 = MM(j) with V(j) in stage st, K(j+1) in stage st+1
      for (int j = 0; j < nt - 1; ++j) {
        SM(xs, s2, s1, j + 2 < nt, true, true, xs ^ (2 * kExtTileB));
        phase_barrier(j + 2 < nt ? 1 : 2);
        MM_full(st, s1, (xs + kExtTileB) & (3 * kExtTileB));
        phase_barrier(0, false);
        next_tile();
      }
      SM(xs, 0, 0, false, false, false, 0);
      phase_barrier(2);
      MM_last(st);
      phase_barrier(0, false);
      phase_barrier(0);
      phase_barrier(0, false);
    } else {
      // tile j: phase 2j = MM(j-1) with V(j-1) in stage st-1, K(j) in stage st;
      //         phase 2j+1 = SM(j), prefetching K(j+3) -> stage st, V(j+2) -> stage st+2
      phase_barrier(0);                                 // phase 0: nothing to do yet
      SM(0, 0, 2 * kStageB, 3 < nt, 2 < nt, false, 0);         // phase 1 (tile 0)
      phase_barrier(3 < nt ? 1 : 2, false);
      for (int j = 1; j < nt; ++j) {
        MM_full(st, s1, (xs + kExtTileB) & (3 * kExtTileB));
        phase_barrier(0);
        next_tile();
        SM(xs, st, s2, j + 3 < nt, j + 2 < nt, false, 0);
        phase_barrier(j + 3 < nt ? 1 : 2, false);
      }
      MM_last(st);
      phase_barrier(0);
      phase_barrier(0, false);
    }
  } else {
    // scores of tile 0 (group A) / tile 1 (group B)
    if (grpA || nt > 1) {
      first_scores(grpA ? 0 : 1);
      first_reference(grpA ? 0 : kStageB);
    }
    wait_loads<0>();   // V(0), K(2): published by the barrier that ends phase 0
    first_v();
    // Phases p = 0..nt, one work-group barrier each; both groups execute nt + 1 of them.
    //   reads in phase p : V(p-1) from stage (p-1)%3, K(p+1) and the first factors of record p+1 from stage (p+1)%4, the others of record p
    //   batch of phase p : K(p+3) -> stage (p+3)%4 (last read, as K(p-1), in phase p-2; a stage less, and the
    //                      batch of phase 0 would land on K(0), which the first scores read without a
    //                      barrier in between),
    //                      V(p+1) -> stage (p+1)%3 (last read, as V(p-2), in phase p-1),
    //                      record p+3 with K(p+3) (last read, as record p-1, in phase p-1)
    //   end of phase p   : the batch of phase p-1 must have landed (first read in phase p+1); its
    //                      issuers are the group now ending a matrix phase, which waits for all of
    //                      its loads; the other group has only this phase's batch in flight
    // (A stage more for each tensor and loads a phase further ahead gained nothing and cost every launch 0.5 us:
    // 4 heads of 768 17.8 -> 18.2 us, a ring of four chunks of 1152 on 24 heads 67.9 -> 68.2.)
    auto end_phase = [&](bool wait_loads) {
      __builtin_amdgcn_sched_barrier(0);
      if (wait_loads) __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    };
    int t = grpA ? 0 : 1;                  // this group's current tile; SM(t) runs in phase t
    // stages of V, of tiles t, t + 1 and t + 2 (mod 3); of K and the records, of tiles t (the record), t + 2 (read) and t + 3 (loaded), mod
    // 4: from one to the next but one and back
    int st = t * kStageB, s1 = st + kStageB, s2 = grpA ? 2 * kStageB : 0;
    int xs = t * kStageB, k_rdst = (t + 2) * kStageB, k_ldst = grpA ? 3 * kStageB : 0;
    constexpr int kFlipEven = 2 * kStageB, kFlipOdd = kStageB ^ (3 * kStageB);
    const int flip_rd = grpA ? kFlipEven : kFlipOdd, flip_ld = grpA ? kFlipOdd : kFlipEven;
    if (kAhead) x_load(0, xs);
    if (!grpA) end_phase(false);           // phase 0: group B has no scores yet
    while (t + 2 < nt) {
      SM(xs, k_ldst, s1, t + 3 < nt, true, true, k_ldst);   // phase t (t + 1 < nt holds here)
      end_phase(false);
      MM_full(st, k_rdst, k_rdst);                          // phase t + 1
      end_phase(true);
      t += 2;
      const int sp = st;
      st = s2; s2 = s1; s1 = sp;
      xs = k_rdst;
      k_rdst ^= flip_rd;
      k_ldst ^= flip_ld;
    }
    if (t < nt) {                                          // this group's last tile
      SM(xs, 0, s1, false, t + 1 < nt, false, 0);
      end_phase(false);
      MM_last(st);
      end_phase(true);
      t += 2;
    }
    // the group whose last matrix phase was phase nt-1 sits out phase nt
    if ((grpA && (nt % 2 == 0)) || (!grpA && (nt % 2 == 1))) end_phase(false);
  }
  } else {               // no live key: the loads of Q and the words' last readers are through before the epilogue reuses their place
    wait_loads<0>();
    __syncthreads();
  }
  // A wave that gave up waiting for a chunk loaded its rows of the tiles too early, and every wave of
  // the work-group has read those rows: the flag belongs to the work-group.
  if (kMulti) {
    if (s.arrive != nullptr) late = __syncthreads_or(late ? 1 : 0) != 0;
  }

  float lratio[2] = {1.0f, 1.0f};
  if (heavy) {
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      const float lh = xgroup_sum(lhat[nb]);
      if (lh > 0.0f) lratio[nb] = xgroup_sum(lsum[nb]) / lh;
    }
  }
  // every tile read of the work-group is behind a barrier here (the one after the last matrix phase)
  finish_and_store<kSplit, kHalfD>(s, oacc, m, lsum, lratio, b, h, q0, wave, lane, smem_raw, kMulti && late, part);
}

template <bool kSplit, bool kExt, bool kMulti, bool kDead, bool kHalfD>
__global__ __launch_bounds__(kThreads, four_waves(kSplit, kExt, kMulti, kDead, kHalfD) ? 4 : 2) void attn_pp_kernel(AttnStep s) {
  extern __shared__ __align__(kLdsAlign) unsigned char smem_raw[];
  touch_step();
  if (!kMulti && (int)blockIdx.x >= s.grid_wgs) {   // prefetch work-group: copy and leave
    prefetch_copy(s, blockIdx.x - s.grid_wgs, threadIdx.x, kThreads);
    return;
  }
  constexpr int kQBlock = kSplit ? kQPerWGSplit : kQPerWG;
  int bh_, qb_;
  int lead = 0;
  if (kMulti && s.arrive != nullptr) {   // the whole ring's transfers ride in this launch, in its first work-groups
    if ((int)blockIdx.x < s.copy_wgs) {
      stream_chunks<kExt>(s, blockIdx.x, threadIdx.x, kThreads);   // (several FP8 chunks: kExt, and the other way round)
      return;
    }
    lead = s.copy_wgs;
  }
  // (batch, head, part of the keys), each with its query blocks: whoever shares K and V follows one another
  const int parts = kSplit ? s.parts : 1;   // (only key-split work-groups come in parts)
  if (!wg_to_tile(s.grid_wgs, (s.Sq + kQBlock - 1) / kQBlock, s.B * s.H * parts, bh_, qb_, lead)) return;   // whole work-group
  int part = 0;
  if (parts > 1) {
    part = bh_ % parts;
    bh_ /= parts;
  }
  attn_pp_body<kSplit, kExt, kMulti, kDead, kHalfD>(s, smem_raw, bh_, qb_ * kQBlock, part);
}

// The parts of a launch whose work-groups shared the keys of a query block (AttnStep::parts): per query,
// O = sum_i 2^(m_i - m) O~_i / l, l = sum_i 2^(m_i - m) l_i, m = max_i m_i, and lse = (m + log2 l) ln 2.
// One thread per eight head dims; the parts lie in the caches, so what bounds it is the launch and one trip to them: all of up to
// kParts parts' loads are issued together (four parts 0.3 to 0.5 us less than one after the other).
template <int kRowD, int kParts>
__global__ __launch_bounds__(256) void attn_combine_kernel(const float* __restrict__ part_o, const float* __restrict__ part_ml,
                                                           bf16_t* __restrict__ out, float* __restrict__ lse, int parts,
                                                           uint32_t rows, uint32_t Sq, uint32_t H, int64_t os0, int64_t os1, int64_t os2) {
  constexpr uint32_t kLanes = kRowD / 8;
  const uint32_t row = blockIdx.x * (256 / kLanes) + threadIdx.x / kLanes, c = threadIdx.x % kLanes;
  if (row >= rows) return;
  constexpr int kBatch = kParts < 8 ? kParts : 8;   // parts whose O~ is on the way at a time
  float2 ml[kParts];
  f32x4 x[kBatch][2];
  auto load = [&](int first) {
#pragma unroll
    for (int i = 0; i < kBatch; ++i)
#pragma unroll
      for (int u = 0; u < 2; ++u)
        x[i][u] = *reinterpret_cast<const f32x4*>(part_o + ((int64_t)(first + i < parts ? first + i : 0) * rows + row) * kRowD + 8 * c + 4 * u);
  };
#pragma unroll
  for (int i = 0; i < kParts; ++i) ml[i] = *reinterpret_cast<const float2*>(part_ml + 2 * ((int64_t)(i < parts ? i : 0) * rows + row));
  load(0);
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < kParts; ++i) m = fmaxf(m, ml[i].x);   // (those past the last repeat the first)
  const float ref = m == -INFINITY ? 0.0f : m;   // (no live key: every weight and every l is 0)
  float l = 0.0f;
  f32x4 o[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
  for (int first = 0; first < kParts; first += kBatch) {
    if (first > 0) load(first);
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      if (first + i < parts) {
        const float w = __builtin_amdgcn_exp2f(ml[first + i].x - ref);
        l = fmaf(w, ml[first + i].y, l);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) o[u][e] = fmaf(w, x[i][u][e], o[u][e]);
      }
    }
  }
  const float inv = l == 0.0f ? 0.0f : 1.0f / l;   // (a part that gave up left NaN in l and O~)
  const uint32_t bh = row / Sq, qi = row - bh * Sq, b = bh / H, h = bh - b * H;
  const u32x4 v = {pack_bf16x2(o[0][0] * inv, o[0][1] * inv), pack_bf16x2(o[0][2] * inv, o[0][3] * inv),
                   pack_bf16x2(o[1][0] * inv, o[1][1] * inv), pack_bf16x2(o[1][2] * inv, o[1][3] * inv)};
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(out + b * os0 + h * os1 + (int64_t)qi * os2 + 8 * c));
  if (c == 0) lse[row] = l == 0.0f ? -INFINITY : (m + log2f(l)) * 0.69314718055994530942f;
}

// Mixed launch: when the 256-query blocks do not fill the last round of work-groups on the 256 CUs
// (one work-group per CU at a time), at least the blocks of that round, and up to half of all (attn_mfma_mixed_grid), are run
// as two key-split work-groups of 128 queries each, which take about 0.55 of a wide work-group's time.  Per XCD (ids go round
// robin) the contiguous, head-major range of blocks is dispatched wide blocks first, then the
// halves of its last s.mix_halves blocks.
template <bool kExt, bool kDead>
__global__ __launch_bounds__(kThreads, 2) void attn_pp_mixed_kernel(AttnStep s) {
  extern __shared__ __align__(kLdsAlign) unsigned char smem_raw[];
  touch_step();
  if ((int)blockIdx.x >= s.grid_wgs) {
    prefetch_copy(s, blockIdx.x - s.grid_wgs, threadIdx.x, kThreads);
    return;
  }
  const int nqb = (s.Sq + kQPerWG - 1) / kQPerWG;
  const int items = nqb * s.B * s.H;
  const int per = (items + kXcds - 1) / kXcds;
  const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
  const int first = xcd * per;
  const int count = min(per, items - first);          // blocks of this XCD (may be <= 0 on the last ones)
  const int halves = min(s.mix_halves, count);
  const int wide = count - halves;
  if (slot < wide) {
    const int item = first + slot;
    const int bh_ = item / nqb;
    attn_pp_body<false, kExt, false, kDead, false>(s, smem_raw, bh_, (item - bh_ * nqb) * kQPerWG, 0);
  } else {
    const int hs = slot - wide;
    if (hs >= 2 * halves) return;
    const int item = first + wide + (hs >> 1);
    const int bh_ = item / nqb;
    const int q_base = (item - bh_ * nqb) * kQPerWG + (hs & 1) * kQPerWGSplit;
    if (q_base >= s.Sq) return;                        // second half of a ragged last block
    attn_pp_body<true, kExt, false, kDead, false>(s, smem_raw, bh_, q_base, 0);
  }
}

}  // namespace

bool attn_mfma_supported(const AttnStep& s) {
  return s.qo_dtype == USP_BF16 && s.kv_dtype == USP_BF16 && (s.d == kD || (s.d == 64 && s.half_d)) && s.Sq > 0;
}

usp_status launch_attn_fp8_chunk_prepare(Fp8Chunk* c, int B, int H, int d, float scale, hipStream_t st) {
  if (!c->ext || !c->k || !c->v || !c->k_src || !c->v_src || !c->k_scale_src || !c->v_scale_src || (d != 64 && d != kD)) {
    set_error("FP8 chunk preparation needs the chunk, its scales, its buffers and room for its records");
    return USP_ERR_INVALID_ARG;
  }
  c->bh = B * H;
  c->H = H;
  c->ush = d == 64 ? 3 : 4;
  c->scale2 = scale * 1.44269504088896340736f;
  const int64_t units = ((int64_t)c->bh * c->Sc) << c->ush;             // 8 codes each
  const int64_t want = (units + 255) / 256;                            // one unit per thread while the chunk is small
  const int blocks = (int)(want < 1 ? 1 : want > 8192 ? 8192 : want);
  c->threads = blocks * 256;
  hipLaunchKernelGGL(attn_fp8_chunk_prepare_kernel, dim3((unsigned)blocks), dim3(256), 0, st, *c);
  USP_CHECK_HIP(hipGetLastError());
  return USP_OK;
}

usp_status launch_attn_arrive_set(uint64_t* arrive, uint64_t tag, hipStream_t st) {
  hipLaunchKernelGGL(attn_arrive_set_kernel, dim3(1), dim3(64), 0, st, arrive, tag);
  USP_CHECK_HIP(hipGetLastError());
  return USP_OK;
}

namespace {
template <bool kSplit, bool kExt, bool kMulti, bool kDead, bool kHalfD>
usp_status launch_pp(const AttnStep& s, unsigned wgs, hipStream_t st) {
  typedef LdsPlan<kHalfD> Lds;
  const int lds = Lds::bytes(kDead && s.tiles <= kMaxWords ? s.tiles : 0);
  USP_CHECK_HIP((allow_large_lds<attn_pp_kernel<kSplit, kExt, kMulti, kDead, kHalfD>>(Lds::bytes(kMaxWords))));
  hipLaunchKernelGGL((attn_pp_kernel<kSplit, kExt, kMulti, kDead, kHalfD>), dim3(wgs + s.copy_wgs), dim3(kThreads), lds, st, s);
  USP_CHECK_HIP(hipGetLastError());
  return USP_OK;
}
template <bool kExt, bool kMulti, bool kDead>
usp_status launch_pp_form(const AttnStep& s, bool split, unsigned wgs, hipStream_t st) {
  if (s.half_d) return split ? launch_pp<true, kExt, kMulti, kDead, true>(s, wgs, st) : launch_pp<false, kExt, kMulti, kDead, true>(s, wgs, st);
  return split ? launch_pp<true, kExt, kMulti, kDead, false>(s, wgs, st) : launch_pp<false, kExt, kMulti, kDead, false>(s, wgs, st);
}
template <bool kMulti>
usp_status launch_pp_any(const AttnStep& s, bool ext, bool dead, bool split, unsigned wgs, hipStream_t st) {
  if (ext) return dead ? launch_pp_form<true, kMulti, true>(s, split, wgs, st) : launch_pp_form<true, kMulti, false>(s, split, wgs, st);
  return dead ? launch_pp_form<false, kMulti, true>(s, split, wgs, st) : launch_pp_form<false, kMulti, false>(s, split, wgs, st);
}
// A launch over one chunk (or step) of head dimension 64, four waves to a SIMD (four_waves): key-split or 256-query work-groups.  In
// microseconds, over `tiles` of keys: 256-query work-groups, one to a CU, 6.1 + 1.04 each round; key-split ones 7.8 + 0.88 for two
// on a CU, 5.6 + 0.53 for one; from FP8 6.5 + 1.0, 5.0 + 0.98 and 4.0 once, and 4.6 + 0.6.  256-query, key-split: 308 blocks of 128, 128 keys 8.3, 10.1;
// 378, 448 keys 12.6, 13.2; 270, 1408 keys 27.5, 25.2; 540, 1728 keys 62.9, 44.1; 864, 4608 keys 158, 144; from FP8 375, 3136 keys 60.3, 62.4;
// 513, 192 keys 18.2, 16.9; 540, 1728 keys 67.3, 53.0; 1190, 448 keys 39.1, 35.3.  363 random launches from bf16 take 1.001 of the better one's time in the mean, 1.04 at most,
// 171 from FP8 1.001 and 1.03 (with 6.5 + 1.06, 9.5 + 0.96 and 6.6 + 0.6, fitted to 256-query work-groups as they were, 1.014 and 1.16: key-split from 30 tiles on).
bool narrow_takes_split(int64_t blocks, int64_t halves, int tiles, bool ext) {
  const int64_t rounds = (blocks + 255) / 256, per_cu = (halves + 255) / 256;
  if (per_cu <= 1) return true;
  const double n = tiles;
  const double wide = (double)rounds * (ext ? 6.5 + 1.0 * n : 6.1 + 1.04 * n);
  const double pair = ext ? 5.0 + 0.98 * n : 7.8 + 0.88 * n, one = ext ? 4.6 + 0.6 * n : 5.6 + 0.53 * n;
  return (double)(per_cu / 2) * pair + (ext ? 4.0 : 0.0) + (per_cu % 2 ? one : 0.0) < wide;
}
template <int kRowD, int kParts>
void launch_combine_as(const AttnStep& s, hipStream_t st) {
  const uint32_t rows = (uint32_t)((int64_t)s.B * s.H * s.Sq), per = 256 * 8 / kRowD;
  hipLaunchKernelGGL((attn_combine_kernel<kRowD, kParts>), dim3((rows + per - 1) / per), dim3(256), 0, st, s.part_o, s.part_ml, (bf16_t*)s.out, s.lse,
                     s.parts, rows, (uint32_t)s.Sq, (uint32_t)s.H, s.os[0], s.os[1], s.os[2]);
}
template <int kRowD>
usp_status launch_combine_d(const AttnStep& s, hipStream_t st) {
  if (s.parts <= 2) launch_combine_as<kRowD, 2>(s, st);
  else if (s.parts <= 4) launch_combine_as<kRowD, 4>(s, st);
  else if (s.parts <= 8) launch_combine_as<kRowD, 8>(s, st);
  else launch_combine_as<kRowD, kMostParts>(s, st);
  USP_CHECK_HIP(hipGetLastError());
  return USP_OK;
}
usp_status launch_combine(const AttnStep& s, hipStream_t st) { return s.half_d ? launch_combine_d<64>(s, st) : launch_combine_d<kD>(s, st); }
template <bool kExt, bool kDead>
usp_status launch_mixed(const AttnStep& s, unsigned wgs, hipStream_t st) {
  constexpr int lds = LdsPlan<false>::bytes(kMaxWords);
  USP_CHECK_HIP((allow_large_lds<attn_pp_mixed_kernel<kExt, kDead>>(lds)));
  hipLaunchKernelGGL((attn_pp_mixed_kernel<kExt, kDead>), dim3(wgs + s.copy_wgs), dim3(kThreads), lds, st, s);
  USP_CHECK_HIP(hipGetLastError());
  return USP_OK;
}
}  // namespace

int64_t attn_mfma_max_dead_tiles() { return kMaxWords; }

// Keys shared between work-groups: for Q shards whose key-split work-groups leave most of the chip idle.  In
// microseconds, a launch takes about 7.5 + tiles * t, t = 0.75 up to 128 work-groups and 0.92 at 216 and
// more; parts add 6 for the second launch and what the parts' bytes, written and read, take at 5.5 TB/s.
// Taken when that comes out at least 3 us lower.
// Over one chunk that leaves launches which gain by parts as well, since the prologue, the second launch and, for d = 64, two work-groups on a
// CU have made them cheaper: 5.5 + tiles * 0.66 (d = 64: 5.6 and 0.46), a tile up to 19 % (10 %) longer from 128 to 216 work-groups and,
// d = 64, up to 1.85 times as long from 256 to 384; parts add 2.3 + 0.35 each (1.7 + 0.25) and their bytes at 4.1 (3.4) TB/s.  46 random launches of
// 4 to 260 work-groups, each with 1, 2, 3, 4, 6 and 8 parts: 4 % rms.  us with 1 part and so: B = 2, H = 2, Sq = 3861, 3456 keys, d = 64 31.0, 25.9;
// H = 2, Sq = 1399, 1024 keys, d = 128 16.0, 14.5.  It is not asked where the first rule has taken parts: it would take fewer there, 13 of 16 tiles
// become 4, up to 20 % faster, but every part's first tile has one weight exact, and with fewer parts O is 1.03 times as far from 64
// bits in the mean of 18 launches, 1.16 at most.
// Measured, 1 against the chosen number of parts: H = 3, Sq = 4608, 4608 keys 57 -> 39 us; H = 1, Sq = 256, 4608 keys 57 -> 19 us.
// One chunk of 500 to 2600 keys, d = 64 or 128, bf16 or FP8, 35 random shapes that take parts: 0.54 to 0.97 of the time.
// At most 240 work-groups, so that the copy work-groups of the same launch (16 at least) find a CU (one chunk, which has none, is held to it too); 480 where
// two fit a CU (one chunk of d = 64, four_waves).  FP8 with dead keys has one to a CU, and beyond 240 parts would be a second round.  (From FP8, d = 64, us undivided
// and in two parts: 11 heads of 1500, 4500 keys 55.6, 64.6; 17 of 1000, 4608 keys of which 300 masked 61.4, 70.1; 8 of 2100, 3500 keys 40.9, 52.1.  Three parts
// for two rounds gain above 4000 keys, 13 of 1500, 4500 keys 56.3, 52.6, and lose below: 8 of 2100, 3500 keys 44.7; they are not taken.)
//
// (The constants of a ring are older: the prologue and the transfers have become shorter since, by 2 to 3 us and by a third.  On random launches the
// choice takes 4 to 5 % more than the best number of parts on average, 1.5 times as much at most.)
// A ring's chunks arrive inside the launch (FP8 chunks always; bf16 ones with USP_ATTN_FUSED_PREFETCH, and the plain
// call takes the same form, so that the two give the same bits): the last one 11 us after the start, plus 4 (FP8: 7)
// for each that its group of copy work-groups has to bring one after another, and the bytes moved at 50 GB/s per
// copy work-group, of which parts leave fewer.  A work-group ends no earlier than its share of that chunk's
// tiles takes from there on, nor than all its tiles take from the arrival of the chunk it begins with, and it
// spends 1 us (FP8: 2) on each chunk it enters.  With the tile times of each form this predicted 440 launches, measured
// with the longer prologue and slower transfers, within 7 % rms; parts have to gain 15 % there.  By the rule for one chunk alone short chunks
// under few queries lost: B = 2, H = 12, Sq = 150, FP8, eight of 320 keys 72 us with 1 part, 103 with 5; B = 2, H = 3,
// d = 64, Sq = 379, six of 320 34 us with 1, 50 with 10.  Long ones gain: H = 2, Sq = 108, six of 2816 202 us
// with 1, 59 with 16.
//
// One chunk under more query blocks than that is key-split where its 128-query work-groups take no second round when 256-query ones would leave
// half the chip idle (Sq that ends in the first half of a block, 129 to 250 blocks), or, for d = 64, by the estimates of attn_mfma_ring_form (three rounds
// of half the time instead of two).  us before, key-split: 136 blocks, 1024 keys 25.8, 18.2; 138 blocks, 4608 keys from FP8 128, 91; 132 blocks, 512
// keys 16.1, 12.2; d = 64, 336 blocks, 4608 keys 154, 128, 2048 keys 73.5, 63.7, 522 blocks, 4143 keys 227, 209.  Of 350 random launches, bf16, FP8 and
// masked, 30 take it, in 0.70 to 0.98 of the time; of 400 more 26, one of them (FP8, d = 64, 360 blocks, 1024 keys) in 1.02.  Their error against 64 bits is 0.96 to
// 1.00 of the other form's, with outliers, where the two forms' references differ, 0.86 to 1.05 (mean 1.00), lse 0.3 to 1.0.
AttnForm attn_mfma_form(int B, int H, int Sq, int d, int64_t tiles, const RingTransfers* ring, bool fp8, bool dead, int most) {
  const int64_t blocks = (int64_t)B * H * ((Sq + kQPerWGSplit - 1) / kQPerWGSplit), wgs = 8 * ((blocks + 7) / 8);
  AttnForm best = {0, 1};
  const bool pairs = !ring && four_waves(true, fp8, false, dead, d != kD);   // two work-groups to a CU (whose launch has a rule of its own, narrow_takes_split)
  if (wgs > 120) {
    const int64_t wide = (int64_t)B * H * ((Sq + kQPerWG - 1) / kQPerWG);
    if (!ring && !pairs && (wide <= 256 ? wgs <= 256 : d != kD)) best.variant = attn_mfma_ring_form(B, H, Sq, d, tiles, 1, 0, fp8).split ? 2 : 0;
    if (!pairs || wgs > 240) return best;
  }
  auto crowd = [](double n) { return n <= 128 ? 0.0 : n >= 216 ? 1.0 : (n - 128) / 88; };   // how far work-groups take each other's time
  // one chunk, the times as they are
  auto chunk_cost = [&](int parts) {
    const double n = (double)wgs * parts, bytes = 2.0 * 4 * d * parts * B * H * Sq;
    const double mine = (double)((tiles + parts - 1) / parts), shared = n <= 256 ? 0.0 : n >= 384 ? 0.75 : 0.75 * (n - 256) / 128;
    if (d == kD) return 5.5 + mine * 0.66 * (1.0 + 0.19 * crowd(n)) + (parts > 1 ? 2.3 + 0.35 * parts + bytes / 4.1e6 : 0.0);
    return 5.6 + mine * 0.46 * (1.0 + 0.1 * crowd(n) + shared) + (parts > 1 ? 1.7 + 0.25 * parts + bytes / 3.4e6 : 0.0);
  };
  auto cost = [&](int parts) {
    const double n = (double)wgs * parts, bytes = 2.0 * 4 * d * parts * B * H * Sq;
    const int64_t mine = (tiles + parts - 1) / parts;
    const double tile = !ring ? 0.75 : d == kD ? (ring->fp8 ? 0.82 : 0.75) : (ring->fp8 ? 0.65 : 0.58);
    const double t = tile * (1.0 + 0.17 / 0.75 * crowd(n));
    const double combine = parts > 1 ? 6.0 + bytes / 5.5e6 : 0.0;
    const double work = (double)mine * t;
    if (!ring) return 7.5 + work + combine;
    const int copy_wgs = copy_wgs_beside((int)(8 * ((blocks * parts + 7) / 8)));
    const int later = ring->chunks - 1, groups = copy_groups_of(copy_wgs, later, ring->largest);
    const double chain = (later + groups - 1) / groups * (ring->fp8 ? 7.0 : 4.0) + (double)ring->bytes / (copy_wgs * 50e3);
    const double share = (double)mine / (double)tiles, enters = share * later + 1.0 < later ? share * later + 1.0 : later;
    const double busy = 8.5 + work + enters * (ring->fp8 ? 2.0 : 1.0);
    const double from_first = 11.0 + chain * (1.0 - share) + work;
    const double from_last = 11.0 + chain + (double)(mine < ring->last_tiles ? mine : ring->last_tiles) * t;
    const double waited = from_last > from_first ? from_last : from_first;
    return (busy > waited ? busy : waited) + (parts > 1 ? combine + 1.0 : 0.0);
  };
  // (Either rule is asked only where the tiles could pay for its second launch: up to 12 tiles of 0.75 are less than 6 + 3, up to 4 of 0.66 * 1.19
  // or 0.46 * 1.1 less than 2.3 + 0.35 * 2 or 1.7 + 0.25 * 2.  Calls so short are as fast as the host issues them.)
  if (wgs <= 120 && (ring || tiles > 12)) {
    const double one = cost(1);
    double least = !ring ? one - 3.0 : 0.96 * one;
    for (int parts = 2; parts <= most && parts * wgs <= 240 && parts <= tiles; ++parts) {
      const double c = cost(parts);
      if (c < least) { least = c; best = {2, parts}; }
    }
  }
  if (ring || best.parts > 1 || tiles <= 4) return best;
  double least = 0.97 * chunk_cost(1);
  for (int parts = 2; parts <= most && parts * wgs <= (pairs ? 480 : 240) && parts <= tiles; ++parts) {
    const double c = chunk_cost(parts);
    if (c < least) { least = c; best = {2, parts}; }
  }
  return best;
}

// How one launch over a ring is decomposed, and whether it is expected to beat a launch per chunk (bf16 chunks,
// all of them at hand).  variant: as AttnStep::variant, 1 and 2 force a form and are judged by that one.  fp8: chunks decoded from FP8.
// Up to one round of 256-query blocks on the 256 CUs the one launch is always the better; key-split there where
// the blocks number at most kSplitBelowWGs or their halves, which take about 0.55 of a block's time, fit a round.  (d = 64 from bf16, two key-split
// work-groups to a CU, would gain up to 13 % with more halves than that where chunks are long and at hand, and lose up to 23 % with the
// transfers inside: 210 blocks, 40 tiles, eight chunks 64.4 us 256-query, 79.5 key-split.  It is left alone.)
// Beyond, in microseconds, with `rounds` of the work-groups over the CUs: 256-query work-groups
// rounds * (10.8 + 1.46 * tiles), d = 64 from FP8 (8.0 + 1.13 * tiles); key-split ones rounds * (9.6 + 0.73 * tiles) and 0.116
// per tile and 256 work-groups (idle CUs let the others clock higher), d = 64 from FP8 (7.1 + 0.47 * tiles) and 0.16; a launch
// per chunk 10.5 each, 5.3 per chunk and round, 1.48 per tile and round, the last round counting
// 0.6 where the mixed launch can halve its blocks (fitted when those of the last round alone were: with less than 96 of them it takes 4 % less now), and 0.115
// per MB of the carried fp32 O, out and back between two chunks.  70 rings of 260 to 864 blocks, two to eight chunks of 64 to 4096 keys, all three timed, with the
// prologue 2 to 3 us longer than it is now: each estimate within 12 % (d = 128: 9 %).  Per chunk, 256-query, key-split: B = 2, H = 24, Sq = 4608, two of 1536
// 370, 331, 363 us; H = 24, Sq = 2816, four of 1024 245, 208, 184; B = 2, H = 18, Sq = 3629, two of 3008 430, 456, 432 (left per chunk).
// d = 64 from bf16, where two key-split work-groups share a CU (four_waves): 256-query ones rounds * (5.8 + 1.04 * tiles), key-split ones
// 4.5 + 1.2 * chunks + 0.944 * tiles for two on a CU and 4.0 + 0.485 * tiles for one.  380 rings of 257 to 2200 blocks, two to twelve chunks of 64 to 4608
// keys, whole, ragged and masked, every form timed with the chunks at hand and with the transfers inside, which take the same form: 115 become key-split by
// these figures that were not by the ones for one to a CU, which stood here, in 0.87 of the time in the mean (0.76 to 0.97), with the
// transfers inside 0.90 (1.004 at most); of 130 rings that were not fitted to 20, in 0.91 (0.998) and 0.93 (1.02).  The error against 64 bits is 0.996 of the
// other form's in the mean (1.003 at most, with outliers 1.08), lse's 0.47 (with outliers 1.0).  The cost per chunk is higher than the chunks at hand ask
// for, so that many short ones stay 256-query: 408 blocks, 64 tiles, eight chunks 139.5, 132.2, with the transfers inside 148.6, 160.4.  So do less than
// six tiles in more than one round: 340 blocks, four tiles 18.9, 16.6, with the transfers inside 23.0, 26.2; six 22.5, 19.2 and 24.9, 23.3.  24 heads of 4608,
// two of 2304 154.6, 144.9.  A launch per chunk took 1.02 to 4 times the better one's time throughout (352 tiles in two chunks 525, 512).
RingForm attn_mfma_ring_form(int B, int H, int Sq, int d, int64_t tiles, int chunks, int variant, bool fp8) {
  const int64_t blocks = (int64_t)B * H * ((Sq + kQPerWG - 1) / kQPerWG), halves = (int64_t)B * H * ((Sq + kQPerWGSplit - 1) / kQPerWGSplit);
  if (blocks <= 256) {
    const int64_t w256 = (blocks + 7) / 8 * 8, w128 = (halves + 7) / 8 * 8;   // (as the grid rounds them)
    return {variant == 2 || (variant != 1 && (w256 <= kSplitBelowWGs || w128 <= 256)), true};
  }
  const int64_t r256 = (blocks + 255) / 256, r128 = (halves + 255) / 256, rem = blocks % 256;
  const double n = (double)tiles;
  if (d != kD) {
    double wide, split;
    if (four_waves(true, fp8, true, false, true)) {
      wide = (double)r256 * (5.8 + 1.04 * n);
      split = (double)(r128 / 2) * (4.5 + 1.2 * chunks + 0.944 * n) + (r128 % 2 ? 4.0 + 0.485 * n : 0.0);
      if (r128 > 2 && tiles < 6) split = wide;
    } else {
      wide = (double)r256 * (8.0 + 1.13 * n);
      split = (double)r128 * (7.1 + 0.47 * n) + 0.16 * n * (double)halves / 256.0;
    }
    return {variant == 2 || (variant != 1 && split < wide), true};
  }
  const double wide = (double)r256 * (10.8 + 1.46 * n);
  const double split = (double)r128 * (9.6 + 0.73 * n) + 0.116 * n * (double)halves / 256.0;
  const double rounds = (double)(blocks / 256) + (rem == 0 ? 0.0 : rem <= 128 ? 0.6 : 1.0);
  const double carry = 2.0 * 4 * d * B * H * Sq / 1e6;
  const double stepwise = chunks * (10.5 + 5.3 * rounds) + rounds * n * 1.48 + (chunks - 1) * carry * 0.115;
  const bool take_split = variant == 2 || (variant != 1 && split < wide);
  return {take_split, (take_split ? split : wide) < 0.97 * stepwise};
}

// The mixed launch: taken when the last round of 256-query work-groups would be at most half full, whose blocks are then run as halves.
// Up to half of all blocks are, as long as the work-groups need no round more: the CUs that begin with halves have
// gone on to the next ones when the wide work-groups end.  us with the last round's blocks alone, so: 264 blocks, 256 keys 22.7, 21.8; 272, 2048 82.4,
// 79.0; 336, 2048 84.0, 83.0; FP8, 266, 2048 97.9, 94.4; 78 random shapes of 260 to 1100 blocks, one chunk, 0.96 to 1.00 of the time; 60 rings
// of two to four chunks, a launch per chunk with carried state, 0.91 to 0.99 (mean 0.957; one of 36 us 1.06, 0.99 when repeated).  From 96 blocks in the last round on there is nothing in it (0.97 to 1.03).
// Copy work-groups, at the end of the same grid, are left their CUs (kMostCopyWGs) in the last round: in a round of their own they
// would have nothing to run beside, and the fewer there are, the longer they take.  us a call with the last round's blocks alone, with halves up to the end of the
// round, so, three chunks from HBM and from pinned host memory: 264 blocks, 640 keys 123.8, 117.0, 115.9 and 495, 488, 487; 520, 128 keys 114.4, 111.5, 109.9
// and 162.4, 165.5, 159.6; 600, 640 keys 233.6, 238.3, 231.0 and 1347, 1349, 1344; 26 such, merged in the launch or not: 0.90 to 1.01 of the time.
MixedGrid attn_mfma_mixed_grid(int items, bool forced, bool copies) {
  const int rem = items % 256, blocks = forced ? (items + 1) / 2 : rem <= 128 ? rem : 0;   // forced: the second half of the blocks
  if (blocks == 0) return {0, 0, 0};
  const int per = (items + kXcds - 1) / kXcds;
  int halves = (blocks + kXcds - 1) / kXcds;
  if (!forced && rem < 96) {
    const int rounds = (per + 256 / kXcds - 1) / (256 / kXcds), room = rounds * (256 / kXcds) - per - (copies ? kMostCopyWGs / kXcds : 0);
    const int more = (per + 1) / 2 < room ? (per + 1) / 2 : room;
    if (more > halves) halves = more;
  }
  const int wgs = kXcds * (per + halves);
  return {wgs, halves, copies ? copy_wgs_beside(wgs) : 0};
}

usp_status launch_attn_mfma(const AttnStep& step, hipStream_t st) {
  AttnStep s = step;
  if (s.parts < 1) s.parts = 1;
  if (s.parts > 1 && (s.mode != 0 || s.variant != 2 || !s.part_o || !s.part_ml || s.n_copy != 0)) {
    set_error("a launch that shares keys between work-groups finishes the result and needs room for the parts (key-split form)");
    return USP_ERR_INVALID_ARG;
  }
  if (s.parts > kMostParts) {
    set_error("the keys of a query block are shared by at most %d work-groups (got %d)", kMostParts, s.parts);
    return USP_ERR_INVALID_ARG;
  }
  if (s.n_multi > 0) {
    if (s.n_multi > AttnStep::kMaxMulti || s.mode != 0 || s.n_copy != 0 || s.key_mask || s.k_scale || s.v_scale) {   // (n_copy: the per-step form of the transfers)
      set_error("a launch over several chunks takes at most %d chunks and finishes the result", AttnStep::kMaxMulti);
      return USP_ERR_INVALID_ARG;
    }
    if (s.multi_fp8 && (!s.arrive || !s.ext)) {
      set_error("a launch over several FP8 chunks needs arrival counters and per-tile records");
      return USP_ERR_INVALID_ARG;
    }
    bool dead = false, masked = false;
    for (int c = 0; c < s.n_multi; ++c) {
      if (s.chunk[c].Sc <= 0 || !s.chunk[c].k || !s.chunk[c].v) {
        set_error("a launch over several chunks needs chunks that hold keys");
        return USP_ERR_INVALID_ARG;
      }
      masked |= s.chunk[c].mask_src != nullptr;
      dead |= masked || s.chunk[c].Sc % kTile != 0;
    }
    const unsigned w256 = wg_grid_size((s.Sq + kQPerWG - 1) / kQPerWG, s.B * s.H);
    const unsigned w128 = wg_grid_size((s.Sq + kQPerWGSplit - 1) / kQPerWGSplit, s.B * s.H * s.parts);
    // (there is no mixed form of this launch)
    int64_t tiles = 0;
    for (int c = 0; c < s.n_multi; ++c) tiles += (s.chunk[c].Sc + kTile - 1) / kTile;
    const bool split = attn_mfma_ring_form(s.B, s.H, s.Sq, s.d, tiles, s.n_multi, s.variant, s.multi_fp8).split;
    const unsigned wgs = split ? w128 : w256;
    s.grid_wgs = (int)wgs;
    s.tiles = (int)tiles;
    s.any_mask = masked;
    s.copy_wgs = 0;
    if (s.arrive != nullptr) {
      for (int c = s.multi_fp8 ? 0 : 1; c < s.n_multi; ++c)
        if (!s.chunk[c].k_src || !s.chunk[c].v_src || s.chunk[c].bytes <= 0 || s.chunk[c].bytes % 16 != 0 ||
            !aligned16(s.chunk[c].k_src) || !aligned16(s.chunk[c].v_src) || !aligned16(s.chunk[c].k) || !aligned16(s.chunk[c].v) ||
            (s.multi_fp8 && (!s.chunk[c].k_scale_src || !s.chunk[c].v_scale_src))) {
          set_error("transfers inside a launch over several chunks need 16-byte aligned sources and buffers");
          return USP_ERR_INVALID_ARG;
        }
      s.copy_wgs = copy_wgs_beside((int)wgs);
      int64_t largest = 0;
      for (int c = 1; c < s.n_multi; ++c) largest = s.chunk[c].bytes > largest ? s.chunk[c].bytes : largest;
      s.copy_groups = copy_groups_of(s.copy_wgs, s.n_multi - 1, largest * (s.multi_fp8 ? 6 : 4));   // K and V, codes or bf16 read, bf16 written
      s.arrive_need = s.copy_wgs / s.copy_groups + (s.arrive_need_extra > 0 ? s.arrive_need_extra : 0);
      if (s.arrive_polls <= 0 || s.arrive_polls > kArrivePolls) s.arrive_polls = kArrivePolls;
    }
    const usp_status r = launch_pp_any<true>(s, s.multi_fp8 != 0, dead, split, wgs, st);
    return r == USP_OK && s.parts > 1 ? launch_combine(s, st) : r;
  }
  s.tiles = (s.Sc + kTile - 1) / kTile;
  s.any_mask = s.key_mask != nullptr;
  const bool ext = s.k_scale != nullptr;
  const bool dead = s.key_mask != nullptr || s.Sc % kTile != 0 || s.Sc == 0;
  // Few query blocks (a small Q shard of a ring step): 256-query work-groups would leave CUs idle;
  // 128-query work-groups whose two wave groups split the keys fill twice as many.
  const unsigned wgs256 = wg_grid_size((s.Sq + kQPerWG - 1) / kQPerWG, s.B * s.H);
  const bool narrow_split = s.half_d && four_waves(true, ext, false, dead, true) &&
                            narrow_takes_split((int64_t)s.B * s.H * ((s.Sq + kQPerWG - 1) / kQPerWG), (int64_t)s.B * s.H * ((s.Sq + kQPerWGSplit - 1) / kQPerWGSplit), s.tiles, ext);
  const bool split = s.variant == 2 || (s.variant == 0 && ((int)wgs256 <= kSplitBelowWGs || narrow_split));
  if (ext && s.ext == nullptr) {
    set_error("attention step with FP8 scales needs its per-tile records");
    return USP_ERR_INVALID_ARG;
  }
  if (s.v_scale != nullptr) {
    set_error("the bf16 matrix-core kernels take V already multiplied by its scales");
    return USP_ERR_INVALID_ARG;
  }
  // (the mixed kernel has no half-head-dimension form, and shares no keys; variant 4 asks for it)
  const int items = (int)((s.Sq + kQPerWG - 1) / kQPerWG) * s.B * s.H;
  const MixedGrid mixed = s.half_d || s.parts > 1 || !(s.variant == 4 || (s.variant == 0 && !split))
                              ? MixedGrid{0, 0, 0} : attn_mfma_mixed_grid(items, s.variant == 4, s.n_copy > 0);
  if (mixed.wgs > 0) {
    const unsigned wgs_mixed = (unsigned)mixed.wgs;
    s.mix_halves = mixed.halves;
    s.grid_wgs = mixed.wgs;
    s.copy_wgs = mixed.copy_wgs;
    if (ext) return dead ? launch_mixed<true, true>(s, wgs_mixed, st) : launch_mixed<true, false>(s, wgs_mixed, st);
    return dead ? launch_mixed<false, true>(s, wgs_mixed, st) : launch_mixed<false, false>(s, wgs_mixed, st);
  }
  const unsigned wgs = split ? wg_grid_size((s.Sq + kQPerWGSplit - 1) / kQPerWGSplit, s.B * s.H * s.parts) : wgs256;
  s.grid_wgs = (int)wgs;
  s.copy_wgs = prefetch_wg_count(s, (int)wgs);
  const usp_status r = launch_pp_any<false>(s, ext, dead, split, wgs, st);
  return r == USP_OK && s.parts > 1 ? launch_combine(s, st) : r;
}

}  // namespace usp

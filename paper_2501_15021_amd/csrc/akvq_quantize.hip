// Write path of the AKVQ-VL cache (Section III-C of arXiv 2501.15021): rotate each new Key/Value head vector by
// the 128-point Walsh-Hadamard matrix (Eq. 7), derive per-group scale and zero-point (Eq. 5-6, with clipping),
// emit 2-bit codes (Eq. 3), pack them into the block layout decode reads, and keep salient rows as bfloat16.
//
// Mapping: one wavefront owns one 32-token block of one (batch, kv-head, tensor).  Four neighbouring lanes own a
// token pair (t, t+16): lane (r, j) holds channels e = 32*m + 8*j + i (m<4, i<8) of tokens r and r+16 of the
// block, so every global load is a 128-bit load and a quad covers 64 contiguous bytes of a row.  Butterfly
// strides 1,2,4 and 32,64 stay in registers; strides 8,16 cross the quad with DPP quad_perm.
#include "../../include/akvq.h"
#include "akvq_device.h"
#include "akvq_kernels.h"
#include "akvq_rowquant.h"

namespace akvq {

namespace {

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move_u(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}
// Running extrema, three operands at a time, and their reduction over the four lanes of a quad with the partner's
// value read through DPP by the min / max itself.  Assembly, because the compiler's fminf / fmaxf first canonicalise
// operands it cannot prove quiet (one more instruction each) and reach a partner lane through a separate move.
__device__ __forceinline__ void minmax3(float &mn, float &mx, float a, float b) {
  asm("v_min3_f32 %0, %0, %1, %2" : "+v"(mn) : "v"(a), "v"(b));
  asm("v_max3_f32 %0, %0, %1, %2" : "+v"(mx) : "v"(a), "v"(b));
}
// (the leading s_nop covers the wait states of a DPP read after a VALU write of its source and after an EXEC write)
__device__ __forceinline__ void quad_minmax(float &mn, float &mx) {
  asm volatile("s_nop 4\n\t"
               "v_min_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
               "v_max_f32_dpp %1, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
               "s_nop 1\n\t"
               "v_min_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
               "v_max_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf"
               : "+v"(mn), "+v"(mx));
}
constexpr int kRowRor4 = 0x124;  // rotate right by 4 inside a row of 16 lanes
constexpr int kRowRor8 = 0x128;

// A cross-lane butterfly level: the lane whose index bit is clear keeps a+b, its partner should keep a-b (a = the
// lower lane's value).  One DPP multiply-add per element does it: own += c * partner with c = +1 in the lower lane and
// -1 in the upper one.  The product is exact and the sum is rounded once, exactly like the add of the specification;
// the upper lane ends up with b-a, i.e. the negated result, and since every later level is linear that lane simply
// carries all its values negated from then on (rounding to nearest is symmetric in sign).  After both cross-lane
// levels lanes j = 1, 2 hold negated values; quad_sign(j) is folded into the per-lane constants that consume them.
__device__ __forceinline__ float quad_sign(int j) { return (j == 1 || j == 2) ? -1.0f : 1.0f; }

// Eight elements of one level.  The leading s_nop covers the wait states a DPP read needs after the VALU write of
// its source register (and after an EXEC write): the compiler does not track hazards of inline assembly.
#define AKVQ_DPP_FMAC8(CTRL, NOP)                                                                              \
  asm volatile("s_nop " NOP "\n\t"                                                                            \
               "v_fmac_f32_dpp %0, %0, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                            \
               "v_fmac_f32_dpp %1, %1, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                            \
               "v_fmac_f32_dpp %2, %2, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                            \
               "v_fmac_f32_dpp %3, %3, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                            \
               "v_fmac_f32_dpp %4, %4, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                            \
               "v_fmac_f32_dpp %5, %5, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                            \
               "v_fmac_f32_dpp %6, %6, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                            \
               "v_fmac_f32_dpp %7, %7, %8 " CTRL " row_mask:0xf bank_mask:0xf"                                \
               : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7]) \
               : "v"(c))
__device__ __forceinline__ void quad_level_xor1(float (&x)[8], float c, bool first) {
  if (first) AKVQ_DPP_FMAC8("quad_perm:[1,0,3,2]", "4"); else AKVQ_DPP_FMAC8("quad_perm:[1,0,3,2]", "1");
}
__device__ __forceinline__ void quad_level_xor2(float (&x)[8], float c, bool first) {
  if (first) AKVQ_DPP_FMAC8("quad_perm:[2,3,0,1]", "4"); else AKVQ_DPP_FMAC8("quad_perm:[2,3,0,1]", "1");
}
#undef AKVQ_DPP_FMAC8

// First level (stride 1) straight from the packed binary16 pair: lo + hi and lo - hi, each one mixed-precision
// multiply-add (the widening is exact, the sum is rounded once, as widening followed by an fp32 add would be).
__device__ __forceinline__ void level1_from_half2(uint32_t w, float &sum, float &diff) {
  asm("v_fma_mix_f32 %0, %1, 1.0, %1 op_sel:[0,0,1] op_sel_hi:[1,0,1]" : "=v"(sum) : "v"(w));
  asm("v_fma_mix_f32 %0, %1, 1.0, -%1 op_sel:[0,0,1] op_sel_hi:[1,0,1]" : "=v"(diff) : "v"(w));
}

// un-normalised 128-point butterfly of one row held as raw[m] (eight binary16 channels 32m+8j..+7 per m) with the j
// index spread over the quad; the result in lane j is quad_sign(j) times the transform
__device__ __forceinline__ void wht128_quad(const u32x4 (&raw)[4], float (&u)[4][8], int j) {
  // stride 1
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int w = 0; w < 4; ++w) level1_from_half2(raw[m][w], u[m][2 * w], u[m][2 * w + 1]);
  // strides 2, 4: inside i
#pragma unroll
  for (int h = 2; h < 8; h *= 2)
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if ((i & h) == 0) {
          float a = u[m][i], b = u[m][i + h];
          u[m][i] = a + b;
          u[m][i + h] = a - b;
        }
  // strides 8, 16: across the quad (j bit 0, j bit 1)
  const float c1 = (j & 1) ? -1.0f : 1.0f, c2 = (j & 2) ? -1.0f : 1.0f;
#pragma unroll
  for (int m = 0; m < 4; ++m) quad_level_xor1(u[m], c1, m == 0);
#pragma unroll
  for (int m = 0; m < 4; ++m) quad_level_xor2(u[m], c2, m == 0);
  // strides 32, 64: inside m
#pragma unroll
  for (int h = 1; h < 4; h *= 2)
#pragma unroll
    for (int m = 0; m < 4; ++m)
      if ((m & h) == 0)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          float a = u[m][i], b = u[m + h][i];
          u[m][i] = a + b;
          u[m + h][i] = a - b;
        }
}

// Rotary position embedding of one row held as raw[m] (see wht128_quad): channel e pairs with e + 64, i.e. raw[mm] with
// raw[mm + 2] word by word, both in this lane; cw / sw hold the binary16 cos / sin of channels 32*mm + 8*j .. + 7.
// Both products are exact in fp32 and the multiply-add rounds their sum once; the result is then rounded to binary16.
// The mixed-precision instructions read the binary16 halves in place (HI selects the upper half of every word); being
// assembly, they also keep the compiler from merging the two roundings into one.
template <int HI>
__device__ __forceinline__ float rope_mix(uint32_t x, uint32_t c, uint32_t xp, uint32_t sn, bool subtract) {
  float t, r;
  const float neg_zero = -0.0f;  // product + (-0) is the product itself, signed zeros included
  if (HI) asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,1,0] op_sel_hi:[1,1,0]" : "=v"(t) : "v"(xp), "v"(sn), "v"(neg_zero));
  else asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[0,0,0] op_sel_hi:[1,1,0]" : "=v"(t) : "v"(xp), "v"(sn), "v"(neg_zero));
  if (subtract) {
    if (HI) asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel:[1,1,0] op_sel_hi:[1,1,0]" : "=v"(r) : "v"(x), "v"(c), "v"(t));
    else asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel:[0,0,0] op_sel_hi:[1,1,0]" : "=v"(r) : "v"(x), "v"(c), "v"(t));
  } else {
    if (HI) asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,1,0] op_sel_hi:[1,1,0]" : "=v"(r) : "v"(x), "v"(c), "v"(t));
    else asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[0,0,0] op_sel_hi:[1,1,0]" : "=v"(r) : "v"(x), "v"(c), "v"(t));
  }
  return r;
}
// two floats -> packed binary16 pair (lo = a, hi = b), round to nearest even, one conversion instruction
__device__ __forceinline__ uint32_t pack_half2(float a, float b) {
  uint32_t r;
  asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ void rope_row_quad(u32x4 (&raw)[4], const u32x4 (&cw)[2], const u32x4 (&sw)[2]) {
#pragma unroll
  for (int mm = 0; mm < 2; ++mm)
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const uint32_t lo = raw[mm][w], hi = raw[mm + 2][w], c = cw[mm][w], sn = sw[mm][w];
      raw[mm][w] = pack_half2(rope_mix<0>(lo, c, hi, sn, true), rope_mix<1>(lo, c, hi, sn, true));
      raw[mm + 2][w] = pack_half2(rope_mix<0>(hi, c, lo, sn, false), rope_mix<1>(hi, c, lo, sn, false));
    }
}

// Packing adds the raw patterns with shifts (one shift-add per code); what the constant part of every pattern
// contributes is a compile-time constant (mod 2^32) that is subtracted once per word.
constexpr uint32_t kPack16Bias = (uint32_t)(0x4B400000ull * 0x55555555ull);   // sum over s<16 of kMagicBits << 2s
constexpr uint32_t kPack4Bias = (uint32_t)(0x4B400000ull * 0x01010101ull);    // sum over b<4 of kMagicBits << 8b

// One row as bfloat16 (u holds its sign-carrying transform, scale undoes that) into slot `slot` of row-major K rows or of
// 32-slot V tiles; zeros for a row that carries no token.
template <int TENSOR>
__device__ __forceinline__ void store_bf16_row(const float (&u)[4][8], float scale, int j, uint16_t *k_rows, uint16_t *v_plane,
                                               int slot, bool token) {
  if (TENSOR == 0) {
    uint16_t *dst = k_rows + (size_t)slot * kD;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      u32x4 o;
#pragma unroll
      for (int w = 0; w < 4; ++w)
        o[w] = token ? pack_bf16x2(scaled_row_value(u[m][2 * w], scale), scaled_row_value(u[m][2 * w + 1], scale)) : 0u;
      *reinterpret_cast<u32x4 *>(dst + 32 * m + 8 * j) = o;
    }
  } else {
    const int sb = slot >> 5, sh = (slot & 31) >> 4, sr = slot & 15, sq = sr >> 2, sii = sr & 3;
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int e = 32 * m + 8 * j + i, nb = e >> 4, n = e & 15;
        v_plane[(size_t)sb * 4096 + nb * 512 + (16 * sq + n) * 8 + 2 * sii + sh] =
            token ? (uint16_t)pack_bf16x2(scaled_row_value(u[m][i], scale), 0.0f) : (uint16_t)0;
      }
  }
}

// One token half of a block into the recent-window rings (slot = row mod win_len).  `whole`: every row of the block is new
// and inside the window; it then fills one 32-slot tile of the V ring (the prefill case).  In a tile the values of rows r
// and r+16 of one channel are neighbours; the lane owns both rows and writes its 16-bit values into the wavefront's tile in
// LDS, half 0 and then half 1, and the finished tile goes out as eight fully coalesced 1 KB stores.  (Scattered partial-line
// stores, as for the rows of other blocks, are several times slower.)
template <int TENSOR>
__device__ __forceinline__ void store_ring_half(const QuantArgs &a, const float (&u)[4][8], float scale, int h, int t0, int lane,
                                                bool inside, bool token, bool whole, uint32_t *vtile_lds) {
  const int bh = blockIdx.y, r = lane >> 2, j = lane & 3;
  uint16_t *k_ring = a.k_win + (size_t)bh * a.win_len * kD, *v_ring = a.v_win + (size_t)bh * a.win_len * kD;
  if (TENSOR == 1 && whole) {
    uint16_t *tile16 = reinterpret_cast<uint16_t *>(vtile_lds);
    const int sq = r >> 2, sii = r & 3;
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t pk = token ? pack_bf16x2(scaled_row_value(u[m][2 * w], scale), scaled_row_value(u[m][2 * w + 1], scale)) : 0u;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const int e = 32 * m + 8 * j + 2 * w + c, nb = e >> 4, n = e & 15;
          tile16[nb * 512 + (16 * sq + n) * 8 + 2 * sii + h] = (uint16_t)(c == 0 ? pk : pk >> 16);
        }
      }
    if (h == 1) {
      uint32_t *ring_out = reinterpret_cast<uint32_t *>(v_ring + (size_t)((t0 % a.win_len) >> 5) * 4096);  // (win_len: a multiple of 64)
      wave_lds_sync();
#pragma unroll
      for (int x = 0; x < 8; ++x)
        *reinterpret_cast<u32x4 *>(ring_out + 256 * x + 4 * lane) = *reinterpret_cast<const u32x4 *>(vtile_lds + 256 * x + 4 * lane);
    }
  } else if (inside) {
    store_bf16_row<TENSOR>(u, scale, j, k_ring, v_ring, (t0 + 16 * h + r) % a.win_len, token);
  }
}

// TIERED: rows carry a tier and a source-row index (akvq_quantize_append_tiered); the plain instantiation is the
// two-bit path with identity row mapping and none of the per-row tier arithmetic.
// RING: a block that holds rows of the recent window (the last win_len appended rows) also stores those to the rings.
// ROPE: K rows arrive without their rotary position embedding; it is applied here, in front of the rotation.
// (the tensor, 0 = K or 1 = V, is a template parameter of the body: the two differ in everything after the transform,
// and the kernel branches once, on blockIdx.z)
// blk_from, blk_to: the blocks (counted from a.first_blk) whose four-block groups `group` counts
template <int G, bool TIERED, bool ROPE, int TENSOR, bool RING = false, bool FLAT = false>
__device__ __forceinline__ void quantize_append_body(const QuantArgs &a, int group, int blk_from, int blk_to, int (*slot_of_lds)[kTokBlock],
                                                     uint32_t (*vtile_lds)[2048] = nullptr) {
  // the wavefront index as a scalar: the block index, its first row and every base address derived from them then
  // live in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  int bh = blockIdx.y, blk_rel = blk_from + group * 4 + wave;
  if constexpr (FLAT) {
    const uint32_t at = blockIdx.x * 4 + wave;  // of the blocks of all units
    if (at >= (uint32_t)a.groups) return;
    bh = (int)__umulhi(at, (uint32_t)a.turn);  // at / n_blk
    blk_rel = (int)at - bh * a.n_blk;
  } else {
    if (blk_rel >= blk_to) return;  // whole wavefront leaves; no block-wide barrier is used below
  }
  const int blk = a.first_blk + blk_rel;
  constexpr int tensor = TENSOR;
  const int r = lane >> 2, j = lane & 3;
  constexpr int NG = kD / G;

  const uint16_t *src = tensor == 0 ? a.k_new : a.v_new;
  const bool rotate = (tensor == 0 ? a.rotate_k : a.rotate_v) != 0;
  const float kappa = rotate ? inv_sqrt128() : 1.0f;
  const float lane_sign = rotate ? quad_sign(j) : 1.0f;  // this lane holds lane_sign * (transformed values)
  const float kappa_s = lane_sign * kappa;
  const int t0 = blk * kTokBlock;
  const int t_end = a.T_len + a.n_new;

  // ---- which tokens of this block are salient, and at which overlay slot (rank in the ascending list).
  // The list is ascending, so the block's entries are one contiguous run of at most 32.  Lane l samples entry
  // l*stride; the number of samples below the block start locates the run within one stride, and a second load of
  // 64 consecutive entries covers it.  Lists of up to 64 entries need the first load only.  Both loads are
  // independent of the row loads, which are issued in between so that all latencies overlap.
  int *slot_of = slot_of_lds[wave];
  const int32_t *sidx = a.sal_idx + (size_t)bh * a.S_cap;
  int cnt = a.sal_cnt[bh];
  cnt = min(max(cnt, 0), a.S_cap);
  const int stride = (cnt + 63) >> 6;
  int e1 = 0x7FFFFFFF;
  if (lane * stride < cnt) e1 = sidx[lane * stride];

  bool valid[2];
  int tier[2] = {AKVQ_TIER_2BIT, AKVQ_TIER_2BIT};
  u32x4 raw[2][4];
  u32x4 rope_c[ROPE ? 2 : 1][2], rope_s[ROPE ? 2 : 1][2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int t = t0 + 16 * h + r;
    valid[h] = (t >= a.T_len) && (t < t_end);
    // rows outside the appended range read a clamped (valid) address; nothing derived from them is stored
    const int rel = min(max(t - a.T_len, 0), a.n_new - 1);
    int src_row = rel;
    if constexpr (TIERED) {
      const size_t at = (size_t)(bh / a.Hkv) * a.n_new + rel;
      src_row = min(max(a.row_src[at], 0), a.n_src - 1);
      if (valid[h]) tier[h] = a.row_tier[at];
    }
    const uint16_t *row = src + ((size_t)bh * a.n_src + src_row) * kD;
#pragma unroll
    for (int m = 0; m < 4; ++m) raw[h][m] = *reinterpret_cast<const u32x4 *>(row + 32 * m + 8 * j);
    if constexpr (ROPE) {
      if (tensor == 0) {
        const size_t at = (size_t)(bh / a.Hkv) * a.rope_stride + (size_t)src_row * 64 + 8 * j;
#pragma unroll
        for (int mm = 0; mm < 2; ++mm) {
          rope_c[h][mm] = *reinterpret_cast<const u32x4 *>(a.rope_cos + at + 32 * mm);
          rope_s[h][mm] = *reinterpret_cast<const u32x4 *>(a.rope_sin + at + 32 * mm);
        }
      }
    }
  }
  if constexpr (TIERED) {
    // fine-half mask of this block (one word per batch element): lane L < 32 looks at row t0 + L
    if (tensor == 0 && bh % a.Hkv == 0) {
      const int t = t0 + (lane & 31);
      const bool in_range = lane < kTokBlock && t >= a.T_len && t < t_end;
      const bool fine = in_range && a.row_tier[(size_t)(bh / a.Hkv) * a.n_new + (t - a.T_len)] == AKVQ_TIER_4BIT_FINE;
      const uint32_t written = (uint32_t)__ballot(in_range), bits = (uint32_t)__ballot(fine);
      if (lane == 0) {
        uint32_t *w = a.fine_mask + (size_t)(bh / a.Hkv) * (a.T_cap / kTokBlock) + blk;
        *w = (written == 0xFFFFFFFFu) ? bits : ((*w & ~written) | bits);
      }
    }
  }

  // A block that is only partly new (a decode step appends one row) keeps the other tokens' bits of its V words: the
  // words this lane will rewrite are requested now, with the rows, instead of after the arithmetic.
  const size_t blk_word = ((size_t)bh * (a.T_cap / kTokBlock) + blk) * kBlockWords;
  const bool partial_blk = t0 < a.T_len || t0 + kTokBlock > t_end;  // uniform over the wavefront
  u32x2 v_old[2] = {{0u, 0u}, {0u, 0u}};
  if (tensor == 1 && partial_blk) {
    const int ii = r & 3, q = r >> 2;
#pragma unroll
    for (int c = 0; c < 2; ++c)
      v_old[c] = *reinterpret_cast<const u32x2 *>(a.v_codes + blk_word + (size_t)(16 * q + 8 * (j & 1) + 2 * ii + c) * 4 +
                                                  2 * (j >> 1));
  }

  if (lane < kTokBlock) slot_of[lane] = -1;
  wave_lds_sync();
  // (long lists out of the way of the others' code: between it, they cost launches of few workgroups up to 5 %, 12 prompts of 368 tokens,
  // 4 heads, G = 64, 5.5 -> 5.8 us, one list entry a head)
  if (__builtin_expect(stride <= 1, 1)) {
    if (e1 >= t0 && e1 < t0 + kTokBlock) slot_of[e1 - t0] = lane;
  } else if (__builtin_expect(stride <= 32, 1)) {
    const int below = __popcll(__ballot(e1 < t0));  // samples before the block: the run starts after the last of them
    const int idx = max(below - 1, 0) * stride + lane;
    const int e2 = idx < cnt ? sidx[idx] : 0x7FFFFFFF;
    if (e2 >= t0 && e2 < t0 + kTokBlock) slot_of[e2 - t0] = idx;
  } else {
    // Lists of more than 2048 entries: the stretch between two samples is sampled again until the run starts within 96
    // entries of its first, and two loads cover it.  (Reading the whole list, 64 entries a step, took longer than all the
    // rest from there on: 7 prompts of 15167 tokens, 2463 of them text, 28/4 heads, 109.6 us,
    // now 58; 1 of 20000, 32 heads, 182 -> 83.)
    int below = __popcll(__ballot(e1 < t0));  // (an int: the builtin's own type is unsigned)
    int base = max(below - 1, 0) * stride, span = stride;
    while (span > 96) {
      const int step = (span + 63) >> 6;
      const int at = base + lane * step;
      const int e = lane * step < span && at < cnt ? sidx[at] : 0x7FFFFFFF;
      below = __popcll(__ballot(e < t0));
      base += max(below - 1, 0) * step;
      span = step;
    }
    int e2[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) e2[x] = base + 64 * x + lane < cnt ? sidx[base + 64 * x + lane] : 0x7FFFFFFF;
#pragma unroll
    for (int x = 0; x < 2; ++x)
      if (e2[x] >= t0 && e2[x] < t0 + kTokBlock) slot_of[e2[x] - t0] = base + 64 * x + lane;
  }
  wave_lds_sync();

  // any row that is not a plain one: codes then go through the field extraction of code_bits_tiered, which leaves no
  // constant part behind  (uniform over the wavefront; never without tiers)
  bool no_bias = false;
  if constexpr (TIERED) no_bias = __ballot(tier[0] != AKVQ_TIER_2BIT || tier[1] != AKVQ_TIER_2BIT) != 0ull;

  uint32_t kw[2][2];         // K words of token half h: [h][group-of-64 word]
  uint32_t vcode[2][8];      // V: [mpair][i]: raw patterns of (X, Y) x (half 0, half 1) in the four byte lanes
  uint32_t vmask_part = 0;
  uint32_t meta_out[2][NG];
  int slots[2];

#pragma unroll
  for (int h = 0; h < 2; ++h) {
    slots[h] = slot_of[16 * h + r];
    if (TIERED && tier[h] != AKVQ_TIER_2BIT) slots[h] = -1;  // only plain rows can be salient
    float u[4][8];  // lane_sign times the (rotated) row
    if constexpr (ROPE) {
      if (tensor == 0) rope_row_quad(raw[h], rope_c[h], rope_s[h]);
    }
    if (rotate) {
      wht128_quad(raw[h], u, j);
    } else {
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          u[m][2 * w] = half_bits_to_float(raw[h][m][w] & 0xFFFFu);
          u[m][2 * w + 1] = half_bits_to_float(raw[h][m][w] >> 16);
        }
    }

    // ---- bfloat16 copy: the overlay slot of a salient row (Section III-C.1: salient tokens keep 16-bit precision) ----
    // (the V rows of long salient lists are stored by overlay_rows_body instead)
    if (valid[h] && slots[h] >= 0 && (tensor == 0 || !a.skip_overlay))
      store_bf16_row<TENSOR>(u, kappa_s, j, a.k_sal + (size_t)bh * a.S_cap * kD, a.v_sal + (size_t)bh * a.S_cap * kD, slots[h], true);
    if constexpr (RING) {
      if (blk >= a.win_blk) {  // uniform over the wavefront
        const int t_first = max(a.T_len, t_end - a.win_len);
        // fine halves and padding rows carry no token: their ring slots are zeroed
        const bool token = !TIERED || (tier[h] != AKVQ_TIER_4BIT_FINE && tier[h] != AKVQ_TIER_PAD);
        store_ring_half<TENSOR>(a, u, kappa_s, h, t0, lane, valid[h] && t0 + 16 * h + r >= t_first, token,
                                t0 >= t_first && t0 + kTokBlock <= t_end, TENSOR == 1 ? vtile_lds[wave] : nullptr);
      }
    }

    // ---- group extrema (quad reduction), scale, zero-point ----
    GroupQ gq[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      constexpr int MPG = 4 / NG;  // m-slices per group
      float mn = u[g * MPG][0], mx = u[g * MPG][0];
#pragma unroll
      for (int m = g * MPG; m < (g + 1) * MPG; ++m)
#pragma unroll
        for (int i = 0; i < 8; i += 2) minmax3(mn, mx, u[m][i], u[m][i + 1]);
      if (lane_sign < 0.0f) {  // extrema of the true values
        const float t = mn;
        mn = -mx;
        mx = -t;
      }
      quad_minmax(mn, mx);
      if constexpr (!TIERED) {
        gq[g] = group_params(mn, mx, kappa, a.clip, tier_two_bit());
        meta_out[h][g] = gq[g].meta | (slots[h] >= 0 ? 0x8000u : 0u);
      } else {
        const bool four = tier[h] == AKVQ_TIER_4BIT_COARSE || tier[h] == AKVQ_TIER_4BIT_FINE;
        const TierQ t2 = tier_two_bit(), t4 = tier_four_bit();
        const TierQ tq = {four ? t4.inv_levels : t2.inv_levels, four ? t4.s16_max : t2.s16_max};
        gq[g] = group_params(mn, mx, kappa, four ? a.clip4 : a.clip, tq);
        uint32_t mw = gq[g].meta | (slots[h] >= 0 ? 0x8000u : 0u);
        if (tier[h] == AKVQ_TIER_4BIT_COARSE)  // scale 4*s (exact in binary16), zero floor(z4 / 4)
          mw = float_to_half_bits_rne(4.0f * half_bits_to_float(gq[g].s16)) | ((uint32_t)((gq[g].z >> 2) & 0xFFFF) << 16);
        else if (tier[h] == AKVQ_TIER_4BIT_FINE)  // scale s, zero z4 mod 4
          mw = gq[g].s16 | ((uint32_t)(gq[g].z & 3) << 16);
        else if (tier[h] == AKVQ_TIER_PAD)  // ignored by decode: salient bit with scale bits 0, a marker no real row has
          mw = 0x8000u;
        meta_out[h][g] = mw;
      }
      gq[g].rcpu *= lane_sign;  // codes are taken from the signed values this lane holds
    }
    // per-row constants of the code extraction (tiered rows only)
    float code_top = kMagic + 3.0f;
    uint32_t code_shift = 0u, code_keep = 2u;  // field offset and width in bits
    if constexpr (TIERED) {
      if (tier[h] == AKVQ_TIER_4BIT_COARSE || tier[h] == AKVQ_TIER_4BIT_FINE) code_top = kMagic + 15.0f;
      if (tier[h] == AKVQ_TIER_4BIT_COARSE) code_shift = 2u;
      if (tier[h] == AKVQ_TIER_PAD) code_keep = 0u;
    }
    auto pack_codes = [&](auto &&row_code, uint32_t bias16) {
      if (tensor == 0) {
        // K word (m/2): slot 8*(m%2)+i at bits 2*slot; built from the top slot down by shift-adds
#pragma unroll
        for (int wq = 0; wq < 2; ++wq) {
          uint32_t word = 0;
#pragma unroll
          for (int slot = 15; slot >= 0; --slot) {
            const int m = 2 * wq + (slot >> 3), i = slot & 7;
            word = (word << 2) + row_code(u[m][i], gq[m / (4 / NG)]);
            asm("" : "+v"(word));  // keep the chain one shift-add per code (re-association costs more instructions)
          }
          kw[h][wq] = word - bias16;
        }
      } else {
        // V: byte lanes of a partial word: token half h, X (m even) / Y (m odd); biases removed after both halves
#pragma unroll
        for (int mp = 0; mp < 2; ++mp)
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const uint32_t bx = row_code(u[2 * mp][i], gq[(2 * mp) / (4 / NG)]);
            const uint32_t by = row_code(u[2 * mp + 1][i], gq[(2 * mp + 1) / (4 / NG)]);
            const uint32_t part = (by << 8) + bx;
            if (h == 0) vcode[mp][i] = part; else vcode[mp][i] = (part << 16) + vcode[mp][i];
          }
        if (valid[h]) vmask_part |= 0x0303u << (16 * h);
      }
    };
    // ---- codes ----  (a tiered block whose rows are all plain, most blocks of a prompt, takes the plain path)
    if (no_bias)
      pack_codes([&](float x, const GroupQ &q) { return code_bits_tiered(x, q, code_top, code_shift, code_keep); }, 0u);
    else
      pack_codes([&](float x, const GroupQ &q) { return code_bits(x, q); }, kPack16Bias);
  }

  // ---- meta ----
  if (j == 0) {
    uint32_t *meta = tensor == 0 ? a.k_meta : a.v_meta;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (valid[h]) {
        uint32_t *dst = meta + ((size_t)bh * a.T_cap + t0 + 16 * h + r) * NG;
#pragma unroll
        for (int g = 0; g < NG; ++g) dst[g] = meta_out[h][g];
      }
  }

  if (tensor == 0) {
    // chunk 16*j + r: words {2h, 2h+1} belong to token half h
    uint32_t *chunk = a.k_codes + blk_word + (size_t)(16 * j + r) * 4;
    if (valid[0] && valid[1]) {
      u32x4 o = {kw[0][0], kw[0][1], kw[1][0], kw[1][1]};
      *reinterpret_cast<u32x4 *>(chunk) = o;
    } else if (valid[0]) {
      u32x2 o = {kw[0][0], kw[0][1]};
      *reinterpret_cast<u32x2 *>(chunk) = o;
    } else if (valid[1]) {
      u32x2 o = {kw[1][0], kw[1][1]};
      *reinterpret_cast<u32x2 *>(chunk + 2) = o;
    }
  } else {
    // shift the byte lanes to this token's pair position (ii = r%4), then OR over the four rows that share a chunk
    const int ii = r & 3, q = r >> 2;
    uint32_t mask = vmask_part << (2 * ii);
    mask |= dpp_move_u<kRowRor4>(mask);
    mask |= dpp_move_u<kRowRor8>(mask);
    if (mask != 0u) {  // uniform over the four rows of a chunk; in practice over the wavefront
      const uint32_t shifted_bias = no_bias ? 0u : 0u - (kPack4Bias << (2 * ii));
      // all cross-lane work first, outside any divergent control flow: complete words of the lane's eight chunks
      uint32_t w[2][8];
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int mp = 0; mp < 2; ++mp) {
          // (the patterns' constant part is taken off after the shift, where both are one shift-add)
          uint32_t x = (vcode[mp][i] << (2 * ii)) + shifted_bias;
          x |= dpp_move_u<kRowRor4>(x);
          x |= dpp_move_u<kRowRor8>(x);
          w[mp][i] = x;
        }
      // Each of the four rows stores two of the eight chunks: i = 2*ii and 2*ii + 1.  The candidates are pinned to registers
      // first: left to itself the compiler makes an indexed array of the choice and moves it to LDS, 16 KB per workgroup,
      // whose addresses need the workgroup's size from the dispatch packet: a scalar load from host memory by every
      // wavefront.  Kernel time of one prompt with 32 heads, without that load: 640 tokens 13.0 -> 6.0 us, 1280 tokens
      // 18.7 -> 7.9, 5120 tokens 26.4 -> 18.6; 16 prompts of 4096 tokens 232 -> 228.
      uint32_t sel[2][2];
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int mp = 0; mp < 2; ++mp) {
          uint32_t x[4] = {w[mp][c], w[mp][2 + c], w[mp][4 + c], w[mp][6 + c]};
#pragma unroll
          for (int p = 0; p < 4; ++p) asm("" : "+v"(x[p]));
          const uint32_t lo = (ii & 1) ? x[1] : x[0], hi = (ii & 1) ? x[3] : x[2];
          sel[c][mp] = (ii & 2) ? hi : lo;
        }
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        uint32_t *dst = a.v_codes + blk_word + (size_t)(16 * q + 8 * (j & 1) + 2 * ii + c) * 4 + 2 * (j >> 1);
        uint32_t w0 = sel[c][0], w1 = sel[c][1];
        if (mask != 0xFFFFFFFFu) {  // block only partly new: keep the other tokens' bits (read at the top)
          w0 = (v_old[c][0] & ~mask) | (w0 & mask);
          w1 = (v_old[c][1] & ~mask) | (w1 & mask);
        }
        u32x2 o = {w0, w1};
        *reinterpret_cast<u32x2 *>(dst) = o;
      }
    }
  }
}

// (batch, kv-head) blockIdx.y, tensor blockIdx.z, four blocks of the appended range a workgroup.  Workgroups go to the XCDs
// in turn, so with an even number of them per unit an XCD would work on the same few ranges of every unit; a.turn (see
// launch_blocks) moves each unit's order on by one, eight in a cycle.
// ... or (FLAT) four consecutive blocks of all units' blocks, one unit after the other (a.groups of them; a.turn: 2^32 / n_blk,
// rounded up): no wavefront without a block, and no XCD with more of the units' short last groups than another.
template <int G, bool TIERED, bool ROPE>
__global__ __launch_bounds__(256) void quantize_append_flat_kernel(QuantArgs a) {
  __shared__ int slot_of_lds[4][kTokBlock];
  if (blockIdx.z == 0) quantize_append_body<G, TIERED, ROPE, 0, false, true>(a, 0, 0, 0, slot_of_lds);
  else quantize_append_body<G, TIERED, ROPE, 1, false, true>(a, 0, 0, 0, slot_of_lds);
}
template <int G, bool TIERED, bool ROPE>
__global__ __launch_bounds__(256) void quantize_append_kernel(QuantArgs a) {
  __shared__ int slot_of_lds[4][kTokBlock];
  int group = blockIdx.x + (blockIdx.y & a.turn);
  if (group >= a.groups) group -= a.groups;  // (turn < groups)
  if (blockIdx.z == 0) quantize_append_body<G, TIERED, ROPE, 0>(a, group, 0, a.n_blk, slot_of_lds);
  else quantize_append_body<G, TIERED, ROPE, 1>(a, group, 0, a.n_blk, slot_of_lds);
}

// ------------------------------------------------------------------------------------------------
// The rows of an append that fall into the recent window, as bfloat16 into their ring slots: one wavefront per 32-row block
// from win_blk on, behind the wavefronts of the unit's blocks in the same launch.  They read and transform their rows a
// second time (same butterflies and roundings), and the blocks take the body without ring stores.  The window's blocks used
// to go through bodies with them in a launch of their own at the end, or in one launch of four bodies (59 KB of code) where
// that was small.  Before and now, window W: 8 prompts of 4096 tokens, 32 heads, W 512: 136 -> 122 us; 2 of 1000, W 128: 15.8
// -> 12.7; 1 of 700, W 64: 6.9 -> 6.3; 1 of 700 with tiers, W 128: 7.8 -> 6.8; 64 of 300, 40 heads, W 128 (ring rows stored
// by the blocks, all in one launch): 169 -> 121.
// ------------------------------------------------------------------------------------------------
template <bool TIERED, bool ROPE, int TENSOR>
__device__ __forceinline__ void ring_rows_body(const QuantArgs &a, int win_rel, uint32_t *vtile_lds) {
  const int lane = threadIdx.x & 63;
  const int bh = blockIdx.y, r = lane >> 2, j = lane & 3;
  const int t0 = (a.win_blk + win_rel) * kTokBlock, t_end = a.T_len + a.n_new;
  if (t0 >= t_end) return;  // whole wavefront leaves; no block-wide barrier is used below
  const int t_first = max(a.T_len, t_end - a.win_len);
  const bool rotate = (TENSOR == 0 ? a.rotate_k : a.rotate_v) != 0;
  const float kappa_s = rotate ? quad_sign(j) * inv_sqrt128() : 1.0f;
  const uint16_t *src = TENSOR == 0 ? a.k_new : a.v_new;
  bool valid[2], token[2];
  u32x4 raw[2][4], rope_c[2][2], rope_s[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int t = t0 + 16 * h + r;
    valid[h] = t >= t_first && t < t_end;
    token[h] = true;
    // rows outside read a clamped (valid) address; nothing derived from them is stored
    const int rel = min(max(t - a.T_len, 0), a.n_new - 1);
    int src_row = rel;
    if constexpr (TIERED) {
      const size_t at = (size_t)(bh / a.Hkv) * a.n_new + rel;
      src_row = min(max(a.row_src[at], 0), a.n_src - 1);
      const int tier = a.row_tier[at];
      token[h] = tier != AKVQ_TIER_4BIT_FINE && tier != AKVQ_TIER_PAD;  // such rows carry no token: their slots are zeroed
    }
    const uint16_t *row = src + ((size_t)bh * a.n_src + src_row) * kD;
#pragma unroll
    for (int m = 0; m < 4; ++m) raw[h][m] = *reinterpret_cast<const u32x4 *>(row + 32 * m + 8 * j);
    if constexpr (ROPE && TENSOR == 0) {
      const size_t at = (size_t)(bh / a.Hkv) * a.rope_stride + (size_t)src_row * 64 + 8 * j;
#pragma unroll
      for (int mm = 0; mm < 2; ++mm) {
        rope_c[h][mm] = *reinterpret_cast<const u32x4 *>(a.rope_cos + at + 32 * mm);
        rope_s[h][mm] = *reinterpret_cast<const u32x4 *>(a.rope_sin + at + 32 * mm);
      }
    }
  }
  const bool whole = t0 >= t_first && t0 + kTokBlock <= t_end;  // (uniform over the wavefront)
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    float u[4][8];  // quad_sign(j) times the (rotated) row
    if constexpr (ROPE && TENSOR == 0) rope_row_quad(raw[h], rope_c[h], rope_s[h]);
    if (rotate) {
      wht128_quad(raw[h], u, j);
    } else {
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          u[m][2 * w] = half_bits_to_float(raw[h][m][w] & 0xFFFFu);
          u[m][2 * w + 1] = half_bits_to_float(raw[h][m][w] >> 16);
        }
    }
    store_ring_half<TENSOR>(a, u, kappa_s, h, t0, lane, valid[h], token[h], whole, vtile_lds);
  }
}
template <int G, bool TIERED, bool ROPE>
__global__ __launch_bounds__(256) void quantize_append_window_kernel(QuantArgs a) {
  __shared__ int slot_of_lds[4][kTokBlock];
  __shared__ __attribute__((aligned(16))) uint32_t vtile_lds[4][2048];  // one V tile (32 slots x 128 channels, bf16) per wavefront
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), win_rel = (int)blockIdx.x * 4 + wave - a.n_blk;
  if (blockIdx.z == 0) {
    if (win_rel >= 0) ring_rows_body<TIERED, ROPE, 0>(a, win_rel, vtile_lds[wave]);
    else quantize_append_body<G, TIERED, ROPE, 0>(a, blockIdx.x, 0, a.n_blk, slot_of_lds);
  } else {
    if (win_rel >= 0) ring_rows_body<TIERED, ROPE, 1>(a, win_rel, vtile_lds[wave]);
    else quantize_append_body<G, TIERED, ROPE, 1>(a, blockIdx.x, 0, a.n_blk, slot_of_lds);
  }
}
// ... or by the blocks themselves (see launch_blocks for which), all of a unit's through the body with the ring stores
template <int G, bool TIERED, bool ROPE>
__global__ __launch_bounds__(256) void quantize_append_ring_kernel(QuantArgs a) {
  __shared__ int slot_of_lds[4][kTokBlock];
  __shared__ __attribute__((aligned(16))) uint32_t vtile_lds[4][2048];  // one V tile (32 slots x 128 channels, bf16) per wavefront
  int group = blockIdx.x + (blockIdx.y & a.turn);
  if (group >= a.groups) group -= a.groups;
  if (blockIdx.z == 0) quantize_append_body<G, TIERED, ROPE, 0, true>(a, group, 0, a.n_blk, slot_of_lds);
  else quantize_append_body<G, TIERED, ROPE, 1, true>(a, group, 0, a.n_blk, slot_of_lds, vtile_lds);
}
// ... or the window's blocks alone, in workgroups of their own that come first, and the others through the short body
template <int G, bool TIERED, bool ROPE>
__global__ __launch_bounds__(256) void quantize_append_two_bodies_kernel(QuantArgs a) {
  __shared__ int slot_of_lds[4][kTokBlock];
  __shared__ __attribute__((aligned(16))) uint32_t vtile_lds[4][2048];
  const int n_plain = a.win_blk - a.first_blk, ring_groups = (a.n_blk - n_plain + 3) / 4, group = (int)blockIdx.x - ring_groups;
  if (group < 0) {
    if (blockIdx.z == 0) quantize_append_body<G, TIERED, ROPE, 0, true>(a, blockIdx.x, n_plain, a.n_blk, slot_of_lds);
    else quantize_append_body<G, TIERED, ROPE, 1, true>(a, blockIdx.x, n_plain, a.n_blk, slot_of_lds, vtile_lds);
  } else {
    if (blockIdx.z == 0) quantize_append_body<G, TIERED, ROPE, 0>(a, group, 0, n_plain, slot_of_lds);
    else quantize_append_body<G, TIERED, ROPE, 1>(a, group, 0, n_plain, slot_of_lds);
  }
}

// ------------------------------------------------------------------------------------------------
// The 16-bit V rows of a long salient list (text-salient layers, Section III-B.1 / III-C.1), as a pass of their own
// beside the blocks or behind them: one wavefront per 32-slot tile of the overlay.  It gathers the tile's rows through the salient
// list, transforms them exactly as the block kernel does (same butterflies, same roundings) and stores the tile through
// LDS as eight coalesced 1 KB pieces, instead of one 2-byte store per value from whichever block a row happens to sit
// in.  Slots of the tile that are not being written (rows of earlier appends, unused slots) keep their contents: unless
// every slot is new the tile is read into LDS first.
// The pass reads its rows a second time and runs at the rate of a copy (5 TB/s in and out), so K rows, which are whole
// lines wherever they come from, are left to the block kernel: 8 prompts of 4001 tokens, 1121 of them text, 32 heads:
// block kernel 134.7 -> 147.5 us, this pass (alone) 52.5 -> 28.7 us, the call 181.2 -> 168.9 us.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ void overlay_rows_body(const QuantArgs &a, int group, uint32_t (*vtile_lds)[2048]) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int bh = blockIdx.y;
  const int s0 = (group * 4 + wave) * kTokBlock;
  const int cnt = min(max(a.sal_cnt[bh], 0), a.S_cap);
  if (s0 >= cnt) return;  // whole wavefront leaves; no block-wide barrier is used below
  const int r = lane >> 2, j = lane & 3;
  const int t_end = a.T_len + a.n_new;
  const bool rotate = a.rotate_v != 0;
  const float kappa_s = rotate ? quad_sign(j) * inv_sqrt128() : 1.0f;
  const int32_t *sidx = a.sal_idx + (size_t)bh * a.S_cap;

  bool fresh[2];  // this lane's slot of half h holds a row of this append
  u32x4 raw[2][4];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int slot = s0 + 16 * h + r;
    const int t = slot < cnt ? sidx[slot] : -1;
    fresh[h] = t >= a.T_len && t < t_end;
    const int rel = min(max(t - a.T_len, 0), a.n_new - 1);  // other rows read a clamped (valid) address; nothing of them is stored
    const uint16_t *row = a.v_new + ((size_t)bh * a.n_src + rel) * kD;
#pragma unroll
    for (int m = 0; m < 4; ++m) raw[h][m] = *reinterpret_cast<const u32x4 *>(row + 32 * m + 8 * j);
  }
  const unsigned long long n_fresh = __ballot(fresh[0]) | __ballot(fresh[1]);
  if (n_fresh == 0ull) return;  // a tile of earlier rows
  const bool all_fresh = __ballot(!fresh[0]) == 0ull && __ballot(!fresh[1]) == 0ull;
  uint32_t *tile_out = reinterpret_cast<uint32_t *>(a.v_sal + (size_t)bh * a.S_cap * kD + (size_t)(s0 >> 5) * 4096);
  if (!all_fresh) {
#pragma unroll
    for (int x = 0; x < 8; ++x)
      *reinterpret_cast<u32x4 *>(vtile_lds[wave] + 256 * x + 4 * lane) =
          *reinterpret_cast<const u32x4 *>(tile_out + 256 * x + 4 * lane);
    wave_lds_sync();
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    float u[4][8];  // quad_sign(j) times the (rotated) row
    if (rotate) {
      wht128_quad(raw[h], u, j);
    } else {
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          u[m][2 * w] = half_bits_to_float(raw[h][m][w] & 0xFFFFu);
          u[m][2 * w + 1] = half_bits_to_float(raw[h][m][w] >> 16);
        }
    }
    if (fresh[h]) {
      // in a tile the values of slots r and r + 16 of one channel are neighbours (see the recent-window tiles)
      uint16_t *tile16 = reinterpret_cast<uint16_t *>(vtile_lds[wave]);
      const int sq = r >> 2, sii = r & 3;
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const uint32_t pk = pack_bf16x2(scaled_row_value(u[m][2 * w], kappa_s), scaled_row_value(u[m][2 * w + 1], kappa_s));
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const int e = 32 * m + 8 * j + 2 * w + c, nb = e >> 4, n = e & 15;
            tile16[nb * 512 + (16 * sq + n) * 8 + 2 * sii + h] = (uint16_t)(c == 0 ? pk : pk >> 16);
          }
        }
    }
  }
  wave_lds_sync();
#pragma unroll
  for (int x = 0; x < 8; ++x)
    *reinterpret_cast<u32x4 *>(tile_out + 256 * x + 4 * lane) =
        *reinterpret_cast<const u32x4 *>(vtile_lds[wave] + 256 * x + 4 * lane);
}

__global__ __launch_bounds__(256) void overlay_rows_kernel(QuantArgs a) {
  __shared__ __attribute__((aligned(16))) uint32_t vtile_lds[4][2048];
  overlay_rows_body(a, blockIdx.x, vtile_lds);
}
// ... or in the launch of the blocks, half of it beside a unit's K blocks and half beside its V blocks: the pass is bound by
// memory and the blocks by vector issue.  8 prompts of 4001 tokens, 1121 of them text, 32 heads: 169.2 -> 146.9 us the call,
// 5 of them the selection; block kernel and pass one after the other took 141 + 27.
template <int G, bool ROPE>
__global__ __launch_bounds__(256) void quantize_append_overlay_kernel(QuantArgs a) {
  __shared__ int slot_of_lds[4][kTokBlock];
  __shared__ __attribute__((aligned(16))) uint32_t vtile_lds[4][2048];
  const int groups = (a.n_blk + 3) / 4, group = blockIdx.x;
  if (group >= groups) overlay_rows_body(a, 2 * (group - groups) + blockIdx.z, vtile_lds);
  else if (blockIdx.z == 0) quantize_append_body<G, false, ROPE, 0>(a, group, 0, a.n_blk, slot_of_lds);
  else quantize_append_body<G, false, ROPE, 1>(a, group, 0, a.n_blk, slot_of_lds);
}

template <int G>
__global__ __launch_bounds__(64) void append_row_kernel(QuantArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t code_lds[kD];
  __shared__ __attribute__((aligned(16))) uint16_t row_lds[kD];
  append_row_wave<G>(a, blockIdx.x, blockIdx.y, threadIdx.x, code_lds, row_lds);
}

}  // namespace

constexpr long kCus = kAppendCus, kResidentGroups = 4 * kCus;
// Who stores the ring rows of an append (n_win of its n_blk blocks hold window rows; units: batch elements x KV heads).
enum class Ring { kWavefronts, kBlocks, kTwoBodies };
static Ring ring_by(int n_blk, int n_win, long units, bool tiered, bool rope) {
  // Wavefronts of their own leave the blocks the short body, but read and transform the window's rows a second time: that
  // costs least where they fit into the last workgroup of a unit's blocks, or into CUs that have room.  Otherwise, with the
  // window more than a quarter of the blocks, the blocks are the better place.  Us, wavefronts / blocks, 16-bit rows:
  // 64 prompts of 300 tokens, 40 heads, W 128: 140 / 121; 33 of 337, 4 heads, W 128: 12.1 / 11.7; without a workgroup more:
  // 7 of 150, 32 heads, W 64: 9.3 / 11.2; a small window: 8 of 4096, 32 heads, W 512: 122 / 125.
  const int groups = (n_blk + 3) / 4, with_ring = (n_blk + n_win + 3) / 4, extra = with_ring - groups;
  const long in_blocks = 2 * units * groups, alone = 2 * units * with_ring;  // workgroups
  if (4 * n_win <= n_blk) return Ring::kWavefronts;
  // (one or two blocks, all of the window, no workgroup more: 16 of 40 tokens, 32 heads, 9.6 / 9.0; 32 of 64, 17.6 / 18.8)
  if (extra == 0) return n_win == n_blk && in_blocks > 2 * kCus && in_blocks <= kResidentGroups ? Ring::kBlocks : Ring::kWavefronts;
  if (in_blocks <= 2 * kCus) {
    // Up to two workgroups a CU it is the rounds of workgroups that count.  Two more are never worth it: 7 of 128, 32 heads,
    // W 128 (448 or 896 workgroups) 11.2 / 9.3.  One more is not where their number doubles (33 of 128, 4 heads: 8.8 / 8.2;
    // within the first round 5.9 / 6.2) and, with the rotary embedding or tiers, where ring and block wavefronts share a
    // workgroup (rotary: 4 of 200, 32 heads, W 128: 9.3 / 8.5, but 2 of 256, 8 blocks: 6.5 / 7.4; both, 3 of 64: 7.4 / 6.6).
    const long rounds = (alone + kCus - 1) / kCus - (in_blocks + kCus - 1) / kCus;
    const bool doubled = extra >= groups, shared = n_blk % 4 != 0;
    const bool dear = tiered ? doubled && shared : (doubled && in_blocks > kCus) || (rope && shared && 2 * extra >= groups && in_blocks >= kCus);
    if (rounds == 0 || (rounds == 1 && !dear)) return Ring::kWavefronts;
  }
  // A window of up to a third of the blocks whose groups come out even, all workgroups resident: 4 of 300, 32 heads, W 64: 9.65 by
  // wavefronts, 9.24 by the body with the ring stores for all blocks, 8.78 by both bodies.
  const bool same_groups = (n_blk - n_win + 3) / 4 + (n_win + 3) / 4 == groups;
  if (3 * n_win <= n_blk && same_groups && in_blocks <= kResidentGroups) return Ring::kTwoBodies;
  return Ring::kBlocks;
}
// The blocks of an append, with the wavefronts of its window rows behind those of every unit's blocks where there is a window.
static hipError_t launch_blocks(const QuantArgs &a_in, int B, int G, hipStream_t stream) {
  QuantArgs a = a_in;
  const bool tiered = a.row_tier != nullptr, rope = a.rope_cos != nullptr, window = a.win_len > 0;
  int groups = (a.n_blk + 3) / 4;
  Ring ring = Ring::kWavefronts;
  if (window) {
    const int t_end = a.T_len + a.n_new, t_first = t_end - a.win_len > a.T_len ? t_end - a.win_len : a.T_len;
    a.win_blk = t_first / kTokBlock;
    const int n_win = a.first_blk + a.n_blk - a.win_blk;
    ring = ring_by(a.n_blk, n_win, (long)B * a.Hkv, tiered, rope);
    if (ring == Ring::kWavefronts) groups = (a.n_blk + n_win + 3) / 4;
  }
  // Turned orders in launches of ten rounds of workgroups (four per CU) and more, over units of an even number of them: 16
  // prompts of 4096 tokens (32 workgroups a unit), 32 heads, 229.5 -> 221 us; 16 of 5000 (40) 290 -> 274; 8 of 5000 145.4 ->
  // 137.6.  An odd number moves on by itself.  In shorter launches they gain nothing or cost: 2 of 4000 the same, 12 of 1000
  // 40.2 -> 41.1, 3 of 1000 13.8 -> 14.8, one of 4096 with rotary embedding 17.1 -> 18.4; so they do with the window's workgroups
  // in the launch (8 of 4096 with window 512: 119.0, 119.1) or the overlay's (8 of 1920, 576 slots: 52.3, 56.0).
  a.groups = groups;
  a.turn = (!window || ring == Ring::kBlocks) && groups >= 8 && groups % 2 == 0 && 2l * groups * B * a.Hkv >= 10 * kResidentGroups ? 7 : 0;
  const long blocks = (long)B * a.Hkv * a.n_blk;
  const bool flat = append_runs_on((long)B * a.Hkv, a.n_blk, window);
  if (flat) {
    a.groups = (int)blocks;
    a.turn = (int)reciprocal_of_blocks(a.n_blk);
  }
  const dim3 grid(flat ? (unsigned)((blocks + 3) / 4) : groups, flat ? 1 : B * a.Hkv, 2), block(256);
#define AKVQ_LAUNCH_Q(GG, TT, RR) \
  do { \
    if (flat) hipLaunchKernelGGL((quantize_append_flat_kernel<GG, TT, RR>), grid, block, 0, stream, a); \
    else if (ring == Ring::kTwoBodies) hipLaunchKernelGGL((quantize_append_two_bodies_kernel<GG, TT, RR>), grid, block, 0, stream, a); \
    else if (ring == Ring::kBlocks) hipLaunchKernelGGL((quantize_append_ring_kernel<GG, TT, RR>), grid, block, 0, stream, a); \
    else if (window) hipLaunchKernelGGL((quantize_append_window_kernel<GG, TT, RR>), grid, block, 0, stream, a); \
    else hipLaunchKernelGGL((quantize_append_kernel<GG, TT, RR>), grid, block, 0, stream, a); \
  } while (0)
#define AKVQ_LAUNCH_QR(GG, TT) do { if (rope) AKVQ_LAUNCH_Q(GG, TT, true); else AKVQ_LAUNCH_Q(GG, TT, false); } while (0)
  if (G == 128) {
    if (tiered) AKVQ_LAUNCH_QR(128, true); else AKVQ_LAUNCH_QR(128, false);
  } else {
    if (tiered) AKVQ_LAUNCH_QR(64, true); else AKVQ_LAUNCH_QR(64, false);
  }
#undef AKVQ_LAUNCH_QR
#undef AKVQ_LAUNCH_Q
  return hipGetLastError();
}

hipError_t launch_quantize_append(const QuantArgs &a, int B, int G, hipStream_t stream) {
  if (a.n_new == 1 && a.n_src == 1 && a.row_tier == nullptr) {  // the decode step: one plain row per (batch, kv-head)
    dim3 grid(B * a.Hkv, 2), block(64);
    if (G == 128) hipLaunchKernelGGL(append_row_kernel<128>, grid, block, 0, stream, a);
    else hipLaunchKernelGGL(append_row_kernel<64>, grid, block, 0, stream, a);
    return hipGetLastError();
  }
  // Long salient lists (text-salient layers) get their V overlay rows from workgroups of their own, in the launch of the
  // blocks or (beside a window's ring rows, or one or two blocks of many units) in a launch behind it; a handful of pivots
  // (and the rows of a tiered append, whose tiers the block kernel knows) are stored by the block kernel itself.
  if (a.S_cap > 64 && a.row_tier == nullptr) {
    QuantArgs blocks = a;
    blocks.skip_overlay = 1;
    const int overlay_groups = (a.S_cap / kTokBlock + 3) / 4, n_units = B * a.Hkv;
    // (Not for one or two blocks of so many units that the blocks' workgroups alone fill the card: the overlay's, most of them
    // with nothing to do, then stand in the way of the blocks.  128 prompts of 8 tokens, 8 heads, 128 slots: 10.7 us in a
    // launch behind the blocks, 15.3 in theirs.)
    if (a.win_len <= 0 && !(a.n_blk <= 2 && 2l * n_units >= kResidentGroups)) {
      // Workgroups go to the XCDs in turn: with four a unit the blocks' all sit on the same two of eight, with any even number
      // some XCDs have more of the blocks than others.  One idle workgroup a unit more, where the launch is large enough for that
      // to show, us without and with it: 16 prompts of 80 tokens, 32 heads, 576 slots, 17 rows before: 24.8, 14.1 (two
      // launches: 10.8); 32 of 300, 1152 slots: 89, 36 (42.4); below, it costs: 4 of 100, 1152 slots, 5.8, 7.5.  At exactly four
      // workgroups a CU, four a unit: 4 of 100, 576 slots, 8.6, 6.0, but 4 of 8, one block a unit, 4.7, 5.7.
      int groups = (a.n_blk + 3) / 4 + (overlay_groups + 1) / 2;
      const long launch = 2l * n_units * groups;
      const bool filled = launch > kResidentGroups || (launch == kResidentGroups && a.n_blk > 2);
      if (groups % 2 == 0 && (launch > 6 * kCus || (groups % 4 == 0 && filled))) ++groups;
      const dim3 grid(groups, n_units, 2), block(256);
      const bool rope = a.rope_cos != nullptr;
#define AKVQ_LAUNCH_O(GG, RR) hipLaunchKernelGGL((quantize_append_overlay_kernel<GG, RR>), grid, block, 0, stream, blocks)
      if (G == 128) { if (rope) AKVQ_LAUNCH_O(128, true); else AKVQ_LAUNCH_O(128, false); }
      else { if (rope) AKVQ_LAUNCH_O(64, true); else AKVQ_LAUNCH_O(64, false); }
#undef AKVQ_LAUNCH_O
      return hipGetLastError();
    }
    hipError_t e = launch_blocks(blocks, B, G, stream);
    if (e != hipSuccess) return e;
    const dim3 grid(overlay_groups, n_units), block(256);
    hipLaunchKernelGGL(overlay_rows_kernel, grid, block, 0, stream, a);
    return hipGetLastError();
  }
  return launch_blocks(a, B, G, stream);
}

}  // namespace akvq

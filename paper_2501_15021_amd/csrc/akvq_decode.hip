// Read path of the AKVQ-VL cache: decode attention straight from the packed 2-bit + bfloat16 cache
// (decode step of Section II-A over the cache of Section III-C, arXiv 2501.15021).
//
// A workgroup of four (or eight) wavefronts owns one (batch, kv-head, KV-split); the wavefronts take its 64-token (MHA)
// or 32-token (GQA) tiles round-robin and merge their partial softmaxes through LDS.  Both contractions run on the
// matrix cores with the 2-bit codes expanded in registers (see akvq_device.h):
//   scores  S = Q~ * C_K^T   : rows = the query vector as fixed-point digits, K-dim = 128 channels; the codes as int8
//                              (MHA) or as 4-bit floats (GQA),
//   output  O = W  * C_V     : rows = (softmax weight x scale) split into bfloat16 terms, K-dim = 32 tokens; the codes as
//                              bfloat16 numbers, one and-or per two codes.
// Scale, zero-point and the constants of the expansion are applied to the small side of each product
// (per token for S, per channel-class for O), so the streamed bytes are touched once.
// The cache block layout makes each lane's 128-bit load its own matrix-core operand: no shuffles.  The next
// tile's loads are issued before the current tile is consumed.
#include <mutex>
#include <type_traits>

#include "akvq_device.h"
#include "akvq_kernels.h"
#include "akvq_rowquant.h"

namespace akvq {

// Split-KV partial results for callers that may not allocate (akvq_decode_attention_static): a fixed array in the
// library's own device image, one copy per GPU, held until the process ends.  In host code this name is only a
// handle; the device address comes from decode_static_scratch() below and is what the kernels are given.
static __device__ __align__(256) unsigned char scratch[kDecodeStaticScratchBytes];

hipError_t decode_static_scratch(void **ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void *addr[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (addr[dev] == nullptr) {  // once per device, with that device current: every GPU has its own copy of the array
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

namespace {

// Wavefronts per workgroup (template parameter NW).  Four when the launch has more than one workgroup per CU; eight when
// it has one, where a wavefront walks its tiles at the latency of its own chain and the only thing that shortens the
// call is fewer tiles per wavefront (see launch_decode_stream).
constexpr int kWaves = 4, kWavesWide = 8;
constexpr int kCus = 256;

// Barrier for data exchanged through LDS: unlike __syncthreads() it does not wait for outstanding global loads, so the
// first tiles stay in flight across the staging of the query.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// ------------------------------------------------------------------------------------------------
// Orthonormal 128-point Walsh-Hadamard transform (Section III-C.2) of a vector held by one wavefront, two elements
// per lane: x0 = element `lane`, x1 = element `lane + 64`.  Strides 1..32 exchange lanes, stride 64 stays in the lane.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ void wht128_wave(float &x0, float &x1, int lane) {
#pragma unroll
  for (int h = 1; h < kWave; h *= 2) {
    const float p0 = __shfl_xor(x0, h, kWave), p1 = __shfl_xor(x1, h, kWave);
    x0 = (lane & h) ? p0 - x0 : x0 + p0;
    x1 = (lane & h) ? p1 - x1 : x1 + p1;
  }
  const float s = x0 + x1, d = x0 - x1;
  x0 = s * inv_sqrt128();
  x1 = d * inv_sqrt128();
}
// rotate a query row inside one wavefront (unless it arrives rotated): x0 = element `lane`, x1 = element `lane + 64`
// A pre-RoPE query (cos_row != null) first takes its rotary position embedding: channel i pairs with i + 64, both held
// by this lane; exact fp32 products, one rounding of their sum to fp32, then to binary16 (kept apart by the barrier).
__device__ __forceinline__ void rotate_query(const uint16_t *q_row, float &x0, float &x1, bool q_rotated,
                                             const uint16_t *cos_row, const uint16_t *sin_row, int lane) {
  x0 = half_bits_to_float(q_row[lane]);
  x1 = half_bits_to_float(q_row[lane + 64]);
  if (cos_row != nullptr) {
    const float c = half_bits_to_float(cos_row[lane]), sn = half_bits_to_float(sin_row[lane]);
    float r0 = __fmaf_rn(x0, c, -__fmul_rn(x1, sn)), r1 = __fmaf_rn(x1, c, __fmul_rn(x0, sn));
    asm("" : "+v"(r0));
    asm("" : "+v"(r1));
    x0 = half_bits_to_float(float_to_half_bits_rne(r0));
    x1 = half_bits_to_float(float_to_half_bits_rne(r1));
  }
  if (!q_rotated) wht128_wave(x0, x1, lane);
}
// position of channel e inside the 128-byte A-operand image of the int8 score product: word kc = e/64, lane group
// qd = (e%32)/8, code slot s = 8*((e/32)%2) + e%8 -> register j = s%4, byte b = s/4 -> byte 4j + b of the lane's 16
__device__ __forceinline__ int k_digit_pos(int e) {
  const int kc = e >> 6, j_lane = (e >> 3) & 3, slot = 8 * ((e >> 5) & 1) + (e & 7);
  return (4 * kc + j_lane) * 16 + 4 * (slot & 3) + (slot >> 2);
}
__device__ __forceinline__ float pow4_neg(int k) { return k == 0 ? 1.0f : (k == 1 ? 0.25f : 0.0625f); }

__device__ __forceinline__ uint32_t pack16(uint32_t lo, uint32_t hi) { return (lo & 0xFFFFu) | (hi << 16); }
__device__ __forceinline__ uint32_t hi16(float f) { return __float_as_uint(f) >> 16; }

// Keeps the wavefronts that share a SIMD in step.  Among wavefronts of equal priority the oldest one issues first, so of
// the two workgroups of a CU one ran ahead and the other then finished alone, at the latency of its own chain: with 28/4
// heads, 32 sequences of 32768 tokens and 4 splits the workgroups ended between 46 and 68 us, now between 57 and 63 us.
// A wavefront therefore lowers its priority when half, three quarters and seven eighths of its tiles are done: whoever is
// behind goes first, and what is left of a lead is part of an eighth.  It looks every third tile and goes down one level at
// a time, so a wavefront of few tiles skips the later marks (up to five tiles: all of them) and keeps the level it has
// through the 16-bit rows and the merge.  Catching up on skipped marks and ending the stream at level 0 was no faster, and
// up to 2 % slower (28/4 heads, 64 sequences of 16384 tokens, 64 tiles a wavefront: 75.1 -> 76.4 us; 12/2 heads, 100 of 8000
// tokens, 31 tiles: 35.5 -> 36.4).  Only grouped-query launches that are resident at once (launch_decode_stream): with several
// rounds of workgroups the ones that have just started would hold up the ones about to make room (32 heads, 64 sequences
// of 8192 tokens: 202 -> 221 us), and a stream that waits for memory and not for issue slots gains nothing (the one-head
// kernel, 16 sequences of 4096 tokens: 28.9 us either way; it has no such steps).
struct StreamPace {
  int at, left;  // next tile count that lowers the priority; tiles behind it
  int level;
  __device__ __forceinline__ StreamPace(int n, bool on) : at(on ? n - n / 2 : 0x7FFFFFFF), left(n / 2), level(3) {
    if (on) __builtin_amdgcn_s_setprio(3);
  }
  __device__ __forceinline__ void done(int k) {  // k tiles are done (uniform over the wavefront)
    if (k < at) return;
    if (level == 3) __builtin_amdgcn_s_setprio(2);
    else if (level == 2) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
    --level;
    at += left - left / 2;
    left /= 2;
  }
};

struct Meta {
  float scale, zero;
  bool salient;
};
__device__ __forceinline__ Meta unpack_meta(uint32_t w) {
  Meta m;
  m.scale = __builtin_fabsf(half_bits_to_float(w & 0xFFFFu));  // bit 15 is the salient flag: dropped by the abs modifier
  m.zero = (float)((int)w >> 16);
  m.salient = (w & 0x8000u) != 0;
  return m;
}

// bit 15 of a meta word marks a salient row; read as binary16 the low half is then a negative number (or -0), which one
// class test detects
__device__ __forceinline__ bool meta_is_salient(uint32_t w) {
  return __builtin_amdgcn_classh(__builtin_bit_cast(_Float16, (unsigned short)w), 0x3C | 0x3);  // any negative class or NaN
}
// w minus one bfloat16 of `pair`: pair . sel + w in one dot-product instruction, sel = (-1, 0) or (0, -1) as a bfloat16
// pair held in a register.  Exact: the remainder of a rounding to bfloat16 has at most 16 significant bits.
__device__ __forceinline__ float minus_bf16(uint32_t pair, uint32_t sel, float w) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, pair), __builtin_bit_cast(bf16x2_t, sel), w, false);
}

// two-term bfloat16 split, w ~= hi + lo (17 significant bits): hi is w rounded to bfloat16, lo the exactly representable
// remainder rounded to bfloat16; both as floats whose lower halves are zero (storing the upper half stores the term)
__device__ __forceinline__ void split2(float w, float &hif, float &lof) {
  hif = __uint_as_float(pack_bf16x2(w, 0.0f) << 16);
  lof = __uint_as_float(pack_bf16x2(w - hif, 0.0f) << 16);
}
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kLazyMax = 12.0f;  // the softmax reference is raised only when a score exceeds it by 2^12
constexpr float kNoScore = -1.0e30f;  // softmax reference of the grouped-query kernel before its first score
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }  // bare v_exp_f32

// ---- DPP reductions over the wavefront (result in every lane) ----
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float lane_bcast(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ float row_max_dpp(float v) {  // max over each row of 16 lanes
  v = fmaxf(v, dpp_f<0xB1>(v));   // quad_perm [1,0,3,2]
  v = fmaxf(v, dpp_f<0x4E>(v));   // quad_perm [2,3,0,1]
  v = fmaxf(v, dpp_f<0x141>(v));  // row_half_mirror
  v = fmaxf(v, dpp_f<0x140>(v));  // row_mirror
  return v;
}
__device__ __forceinline__ float row_sum_dpp(float v) {
  v += dpp_f<0xB1>(v);
  v += dpp_f<0x4E>(v);
  v += dpp_f<0x141>(v);
  v += dpp_f<0x140>(v);
  return v;
}
__device__ __forceinline__ float wave_max_dpp(float v) {
  v = row_max_dpp(v);
  return fmaxf(fmaxf(lane_bcast(v, 0), lane_bcast(v, 16)), fmaxf(lane_bcast(v, 32), lane_bcast(v, 48)));
}
__device__ __forceinline__ float wave_sum_dpp(float v) {
  v = row_sum_dpp(v);
  return (lane_bcast(v, 0) + lane_bcast(v, 16)) + (lane_bcast(v, 32) + lane_bcast(v, 48));
}

// Final step: one wavefront holds the merged, normalised o~ (x0 = element `lane`, x1 = element `lane + 64`); rotate it
// back (H is its own inverse) unless the caller wants it rotated, and store.
// `out` is the output array ([B][Hq][128] fp32, or binary16 when out_half), `row_index` the (batch, query-head) row.
__device__ __forceinline__ void unrotate_store_wave(float x0, float x1, void *out, size_t row_index, bool out_rotated,
                                                    bool out_half, int lane) {
  if (!out_rotated) wht128_wave(x0, x1, lane);
  if (out_half) {
    uint16_t *o = static_cast<uint16_t *>(out) + row_index * kD;
    o[lane] = (uint16_t)float_to_half_bits_rne(x0);
    o[lane + 64] = (uint16_t)float_to_half_bits_rne(x1);
  } else {
    float *o = static_cast<float *>(out) + row_index * kD;
    o[lane] = x0;
    o[lane + 64] = x1;
  }
}
// One wavefront merges the NW partial softmaxes of a workgroup for one head (m, l: per wavefront; rows: LDS, 128 floats
// each, row_stride apart) and finishes the row, or stores the split's partial result.
template <int NW>
__device__ __forceinline__ void merge_waves_and_store(const DecodeArgs &a, const float *m, const float *l, int ml_stride,
                                                      const float *rows, int row_stride, size_t bhq, int split, int lane) {
  float m_all = -INFINITY, l_all = 0.0f, o0 = 0.0f, o1 = 0.0f;
#pragma unroll
  for (int w = 0; w < NW; ++w) m_all = fmaxf(m_all, m[w * ml_stride]);
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const float mw = m[w * ml_stride];
    const float wgt = mw == -INFINITY ? 0.0f : fast_exp2(mw - m_all);  // a wavefront without rows has sums of 0
    l_all += wgt * l[w * ml_stride];
    o0 += wgt * rows[w * row_stride + lane];
    o1 += wgt * rows[w * row_stride + lane + 64];
  }
  if (a.n_split == 1) {
    if (a.lse && lane == 0) a.lse[bhq] = (m_all + __log2f(l_all)) * kLn2;
    unrotate_store_wave(o0 / l_all, o1 / l_all, a.out, bhq, a.out_rotated != 0, a.out_half != 0, lane);
  } else {
    float *dst = a.partial + (bhq * a.n_split + split) * kPartialStride;
    if (lane == 0) { dst[0] = m_all; dst[1] = l_all; }
    dst[4 + lane] = o0;
    dst[4 + lane + 64] = o1;
  }
}

// ------------------------------------------------------------------------------------------------
// MHA (one query head per KV head).  A tile is 64 tokens = two cache blocks; the query's three bfloat16 terms
// sit in rows 4g..4g+2 of the A operand used for token group g, so after the 16 products lane l holds the
// three partial dot products of token l: one token per lane for the softmax.
// ------------------------------------------------------------------------------------------------
template <int NG>
struct MhaTile {
  u32x4 kc[2], vc[2];
  uint32_t km[NG], vm[NG];
  uint32_t fm;  // fine-half mask word of this lane's 32-row block (only loaded by the PAIRS instantiations)
};

// PAIRS: the cache holds 4-bit tokens as (coarse, fine) pairs of 2-bit rows on (even, odd) rows, flagged in
// a.fine_mask: the two rows' scores add up to the token's score, the token enters the softmax sum once, and each row
// takes the token's weight times its own scale in the value product.
template <int G, bool PAIRS, int NW>
__device__ __forceinline__ void decode_mha_body(const DecodeArgs &a) {
  constexpr int NG = kD / G;
  // three signed 7-bit digits of q~[e] / U (U a power of two, |q~|/U < 2^20), as int8, in A-operand order of the
  // 16x16x64 int8 product (see k_digit_pos): the code stream's A operand, 16 bytes per lane
  __shared__ __attribute__((aligned(16))) int8_t q_digit[4][kD];  // row 3 stays zero: operand rows that carry nothing
  __shared__ float q_scal[NG + 1];  // U and, per group, the sum of the digitised query in units of U
  __shared__ __attribute__((aligned(16))) uint16_t q_plain[4][kD];  // terms of q~[e], natural order; row 3 stays zero
  __shared__ __attribute__((aligned(16))) uint16_t w_lds_all[NW][2][NG][3][kTokBlock];
  __shared__ __attribute__((aligned(16))) uint16_t zero16[64];  // 128 zero bytes: operand rows that carry nothing
  __shared__ float mrg_m[NW], mrg_l[NW];
  __shared__ float mrg_o[NW][kD];

  const int tid = threadIdx.x;
  // the wavefront index as a scalar: everything derived from it (tile indices, tile addresses) then lives in scalar
  // registers and the loads take a scalar base plus a per-lane offset
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int split = blockIdx.x;
  const int bh = blockIdx.y;  // Hq == Hkv here
  const int mrow = lane & 15, qd = lane >> 4;
  const ExpandK ex;
  auto &w_lds = w_lds_all[wave];  // [blk][group][term][slot]

  // ---- tile bookkeeping and the first two tiles' loads come first: they do not depend on the query, so their
  // latency overlaps with the query rotation below ----
  const int n_tiles = (a.t_win + kMhaTileRows - 1) / kMhaTileRows;  // rows from t_win on are read from the recent-window rings
  int tile_begin, tile_end;
  decode_split_range(n_tiles, a.n_split, split, tile_begin, tile_end);
  const size_t plane_blocks = (size_t)a.T_cap / kTokBlock;
  // Plane bases and tile indices are uniform over the wavefront (scalar registers); a lane adds a fixed 32-bit offset,
  // so every load of the stream is "scalar base + lane offset" and needs no per-lane address arithmetic.
  const gptr_u32 kc_plane = as_global(a.k_codes) + (size_t)bh * plane_blocks * kBlockWords;
  const gptr_u32 vc_plane = as_global(a.v_codes) + (size_t)bh * plane_blocks * kBlockWords;
  const gptr_u32 km_plane = as_global(a.k_meta) + (size_t)bh * a.T_cap * NG;
  const gptr_u32 vm_plane = as_global(a.v_meta) + (size_t)bh * a.T_cap * NG;
  const uint32_t *fm_base = PAIRS ? a.fine_mask + (size_t)(bh / a.Hkv) * plane_blocks + (lane >> 5) : nullptr;
  const uint32_t lane_code = (uint32_t)lane * 4u, lane_meta = (uint32_t)lane * NG;

  auto load_tile = [&](int tile, MhaTile<NG> &t) {
    if constexpr (PAIRS) t.fm = fm_base[2 * tile];
    gptr_u32 kc_t = kc_plane + (size_t)tile * (2 * kBlockWords), vc_t = vc_plane + (size_t)tile * (2 * kBlockWords);
    gptr_u32 km_t = km_plane + (size_t)tile * (64 * NG), vm_t = vm_plane + (size_t)tile * (64 * NG);
    keep_scalar(kc_t); keep_scalar(vc_t); keep_scalar(km_t); keep_scalar(vm_t);
#pragma unroll
    for (int b2 = 0; b2 < 2; ++b2) {
      t.kc[b2] = stream_load_x4(kc_t + b2 * kBlockWords + lane_code);
      t.vc[b2] = stream_load_x4(vc_t + b2 * kBlockWords + lane_code);
    }
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      t.km[g] = stream_load_x1(km_t + lane_meta + g);
      t.vm[g] = stream_load_x1(vm_t + lane_meta + g);
    }
  };

  // Three tile buffers: while tile k is consumed, the loads of tiles k+1 and k+2 are in flight.  Loads are issued
  // unconditionally (the index is clamped to the wavefront's last tile) so that the number of outstanding loads is
  // the same on every path and the waits inside the loop count exactly two tiles of loads.
  // the length of the salient list is asked for now and looked at after the stream (the append of a fused decode
  // step does not change it): the 16-bit rows then cost one memory round trip, not three dependent ones
  // (read through the constant address space: a scalar load, whose wait the compiler puts in front of the first use;
  // as a vector load of a uniform address it would be moved to a scalar register, and waited for, right here)
  const int sal_cnt_early = reinterpret_cast<const __attribute__((address_space(4))) int32_t *>(
      reinterpret_cast<uintptr_t>(a.sal_cnt))[bh];
  const int n_mine = tile_begin + wave < tile_end ? (tile_end - tile_begin - wave + NW - 1) / NW : 0;
  const int last_tile = tile_begin + wave + NW * max(n_mine - 1, 0);
  auto tile_at = [&](int k) { return min(tile_begin + wave + NW * k, last_tile); };
  MhaTile<NG> tb[3];
  // Fused decode step: the workgroups of the split that owns the row's tile first write the new row (wavefront 1
  // the K row, wavefront 2 the V row, while wavefront 0 stages the query); the barrier below orders those stores
  // before this workgroup's loads of the tile that holds the row, and no other workgroup reads that tile.  A wavefront
  // whose first two tiles include that tile asks for them after the barrier instead of here.
  const bool appends = a.fused_append != 0 && split == a.append_split;  // uniform over the workgroup
  const bool defer_loads = appends && a.t_win == a.T_len && n_mine > 0 &&
                           (tile_at(0) == n_tiles - 1 || tile_at(1) == n_tiles - 1);
  if (n_mine > 0 && !defer_loads) {
    load_tile(tile_at(0), tb[0]);
    load_tile(tile_at(1), tb[1]);
  }
  if (appends && (wave == 1 || wave == 2)) {
    __shared__ __attribute__((aligned(16))) uint8_t step_codes[2][kD];
    __shared__ __attribute__((aligned(16))) uint16_t step_row[2][kD];
    append_row_wave<G>(a.step, bh, wave - 1, lane, step_codes[wave - 1], step_row[wave - 1]);
  }

  // Wavefront 0 stages the query on its own (two channels per lane, reductions inside the wavefront); the others wait at
  // one barrier, with the loads of their first tiles in flight.
  if (wave == NW - 1) {
    zero16[lane] = 0;
    q_digit[3][lane] = 0; q_digit[3][lane + 64] = 0;
    q_plain[3][lane] = 0; q_plain[3][lane + 64] = 0;
  }
  if (wave == 0) {
    float x[2];
    rotate_query(a.q + (size_t)bh * kD, x[0], x[1], a.q_rotated != 0,
                 a.rope_cos ? a.rope_cos + (size_t)(bh / a.Hkv) * a.rope_stride : nullptr,
                 a.rope_sin ? a.rope_sin + (size_t)(bh / a.Hkv) * a.rope_stride : nullptr, lane);
    // fixed-point unit of the query: U = 2^ceil(log2 max|q~|) / 2^20 (the digits then cover it exactly, 21 bits)
    const float mx = wave_max_dpp(fmaxf(fabsf(x[0]), fabsf(x[1])));
    const uint32_t e_biased = min(max(__float_as_uint(mx) >> 23, 20u), 250u);  // mx < 2^(e_biased - 126)
    const float unit_inv = __uint_as_float((273u - e_biased) << 23);           // 2^20 / 2^(e_biased - 126)
    float n_of[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int e = lane + 64 * i;
      uint32_t hi, mid, lo;
      split3_bf16(x[i], hi, mid, lo);
      q_plain[0][e] = (uint16_t)hi; q_plain[1][e] = (uint16_t)mid; q_plain[2][e] = (uint16_t)lo;
      const int n = (int)rintf(x[i] * unit_inv);                    // |n| <= 2^20
      const int d2 = (n << 25) >> 25, n1 = (n - d2) >> 7;           // balanced base-128 digits, each in [-64, 64]
      const int d1 = (n1 << 25) >> 25, d0 = (n1 - d1) >> 7;
      const int p = k_digit_pos(e);
      q_digit[0][p] = (int8_t)d0; q_digit[1][p] = (int8_t)d1; q_digit[2][p] = (int8_t)d2;
      n_of[i] = (float)n;                                           // the value the digits represent, in units of U
    }
    if constexpr (NG == 2) {
      const float s0 = wave_sum_dpp(n_of[0]), s1 = wave_sum_dpp(n_of[1]);
      if (lane == 0) { q_scal[0] = 1.0f / unit_inv; q_scal[1] = s0; q_scal[2] = s1; }
    } else {
      const float s0 = wave_sum_dpp(n_of[0] + n_of[1]);
      if (lane == 0) { q_scal[0] = 1.0f / unit_inv; q_scal[1] = s0; }
    }
  }
  if (appends) __syncthreads();  // also orders the new row's stores before the loads below
  else lds_barrier();
  if (defer_loads) {
    load_tile(tile_at(0), tb[0]);
    load_tile(tile_at(1), tb[1]);
  }
  const float q_unit = q_scal[0];
  float qsum[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g) qsum[g] = q_scal[1 + g];

  // ---- A operands for the code stream, per token group g: row 4g+digit carries that digit, other rows are zero.
  // They stay in LDS (two 128-bit reads per product) instead of 32 registers: the kernel then fits three
  // wavefronts per SIMD instead of two, which is what keeps enough loads in flight.
  uint32_t a_off[4];  // byte offset of this lane's operand row inside q_digit, per token group
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int dig = mrow - 4 * g;
    a_off[g] = (uint32_t)(((dig >= 0 && dig < 3) ? dig : 3) * kD + qd * 16);
  }
  const ExpandI8 ex8;

  f32x4 acc_o[8];
#pragma unroll
  for (int nb = 0; nb < 8; ++nb) acc_o[nb] = (f32x4){0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.0f;  // softmax reference (base-2 domain) and this lane's share of the sum
  float swx[NG], szx[NG];                // running sums of w*cx and w*cx*zero over this lane's tokens
#pragma unroll
  for (int g = 0; g < NG; ++g) swx[g] = szx[g] = 0.0f;
  const float sm2 = a.sm_scale * kLog2e;

  const int r16 = lane & 15, half = (lane >> 4) & 1, blk_of_lane = lane >> 5;
  const int slot = 2 * r16 + half, ii = r16 & 3;
  const float cx = pow4_neg(pair_exp(ii)), rcx = 1.0f / cx;  // exact powers of two

  // online-softmax bookkeeping shared by the code stream and the bfloat16 rows.  The reference m_run is only
  // raised when some score exceeds it by more than kLazyMax, so the common tile costs one compare and one branch;
  // weights are then at most 2^kLazyMax, which fp32 sums and the bfloat16 term split absorb.
  auto softmax_step = [&](float score, bool ok, bool count, float &p) -> bool {
    const float sc = ok ? score : -INFINITY;
    if (__ballot(sc > m_run + kLazyMax) != 0ull) {
      const float m_new = wave_max_dpp(sc);
      const float alpha = (m_run == -INFINITY) ? 0.0f : fast_exp2(m_run - m_new);
#pragma unroll
      for (int nb = 0; nb < 8; ++nb) acc_o[nb] *= alpha;
      l_run *= alpha;
#pragma unroll
      for (int g = 0; g < NG; ++g) { swx[g] *= alpha; szx[g] *= alpha; }
      m_run = m_new;
    }
    if (m_run == -INFINITY) { p = 0.0f; return false; }
    p = fast_exp2(sc - m_run);
    l_run += count ? p : 0.0f;  // the fine half of a 4-bit token carries the token's weight but is not a token
    return true;
  };

  // ================= code stream =================
  auto process = [&](const MhaTile<NG> &cur, int tile) {
    const int t = tile * 64 + lane;

    // scores: lane l ends up with the three digit products of token l in acc[0..2] (exact integers)
    i32x4 acc[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) acc[g] = (i32x4){0, 0, 0, 0};
#pragma unroll
    for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const int tg = 2 * b2 + hf;
        uint32_t off = a_off[tg];
        asm volatile("" : "+v"(off));  // keep the operand reads inside the loop (see above)
        const i32x4 a0 = *reinterpret_cast<const i32x4 *>(&q_digit[0][0] + off);
        const i32x4 a1 = *reinterpret_cast<const i32x4 *>(&q_digit[0][0] + off + 64);
        acc[0] = mfma_i8(a0, ex8(cur.kc[b2][2 * hf]), acc[0]);
        acc[NG - 1] = mfma_i8(a1, ex8(cur.kc[b2][2 * hf + 1]), acc[NG - 1]);
      }
    float score = 0.0f;
    bool salient = false;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const Meta mk = unpack_meta(cur.km[g]);
      salient = salient || mk.salient;
      const float raw = (float)acc[g][0] * 16384.0f + ((float)acc[g][1] * 128.0f + (float)acc[g][2]);
      score += mk.scale * (raw - mk.zero * qsum[g]);
    }
    score *= q_unit;
    score *= sm2;
    const bool ok = (t < a.t_win) && !salient;
    bool count = true;
    if constexpr (PAIRS) {
      const uint32_t from_me = cur.fm >> (lane & 31);      // bit 0: this row is a fine half; bit 1: the next row is
      const bool fine = (from_me & 1u) != 0u, coarse = (from_me & 2u) != 0u;  // pairs start on even rows
      const float partner = dpp_f<0xB1>(score);            // lane ^ 1
      score = (fine || coarse) ? score + partner : score;
      count = !fine;
    }
    float p;
    if (softmax_step(score, ok, count, p)) {
      // weights for the value contraction: w = p * scale_V as two bfloat16 terms, pre-divided by the 4^k of its slot
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const Meta mv = unpack_meta(cur.vm[g]);
        float hix, lox;
        split2(ok ? p * (mv.scale * cx) : 0.0f, hix, lox);  // rows past T_len hold arbitrary meta
        w_lds[blk_of_lane][g][0][slot] = (uint16_t)hi16(hix);
        w_lds[blk_of_lane][g][1][slot] = (uint16_t)hi16(lox);
        const float wxr = hix + lox;
        swx[g] += wxr;
        szx[g] = __builtin_fmaf(wxr, mv.zero, szx[g]);
      }
      wave_lds_sync();
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2) {
        bf16x8 a_v[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const uint16_t *src = mrow < 2 ? &w_lds[b2][g][mrow][8 * qd] : zero16;
          a_v[g] = *reinterpret_cast<const bf16x8 *>(src);
        }
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const int g = (NG == 2) ? (w & 1) : 0;
          const int nbx = 4 * (w & 1) + (w >> 1), nby = nbx + 2;
          acc_o[nbx] = mfma_bf16(a_v[g], ex.x(cur.vc[b2][w]), acc_o[nbx]);
          acc_o[nby] = mfma_bf16(a_v[g], ex.y(cur.vc[b2][w]), acc_o[nby]);
        }
      }
      wave_lds_sync();
    }
  };
  if (n_mine > 0) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2) { settle(tb[i].kc[b2]); settle(tb[i].vc[b2]); }
#pragma unroll
      for (int g = 0; g < NG; ++g) { settle(tb[i].km[g]); settle(tb[i].vm[g]); }
    }
    for (int k = 0; k < n_mine; k += 3) {
      load_tile(tile_at(k + 2), tb[2]);
      process(tb[0], tile_at(k));
      if (k + 1 >= n_mine) break;
      load_tile(tile_at(k + 3), tb[0]);
      process(tb[1], tile_at(k + 1));
      if (k + 2 >= n_mine) break;
      load_tile(tile_at(k + 4), tb[1]);
      process(tb[2], tile_at(k + 2));
    }
  }

  // ================= bfloat16 rows: units of 32 slots =================
  // Used twice: the salient overlay (slot = rank in the salient list) and the recent-window rings (slot = row mod W).
  // All of a unit is requested at once: key rows, value rows and the rows' validity are one memory round trip.  (Units of
  // 64 rows, whose four token groups and second block of values each waited for the one before, left two of four
  // wavefronts of the appending workgroup without rows of a window of 128: a step of 4 x 3001 rows, 32 heads, 4-bit text,
  // 17.6 us, of which the window cost 3.6; now 15.5.)
  // (The kernel for plain caches of one group fits four wavefronts per SIMD, which takes asking for the second token group
  // after the first.)
  constexpr bool kBothGroups = PAIRS || NG == 2 || NW == kWavesWide;
  const int cnt_sal = min(max(sal_cnt_early, 0), a.S_cap), win_rows = min(a.win_len, a.T_len);  // (slots behind T_len hold no row)
  // In launches of a workgroup per CU and more without splits (a.row_pairs) issue takes the time and not latency: two units
  // share a softmax step, the second requested behind the first.  Us by units and by pairs of them: 512 workgroups of 400 rows,
  // window 128 (five units for four wavefronts) 13.7, 12.9; 1024 of 64 rows, 64 of them pivots, 11.2, 10.2; up to two workgroups
  // per CU, a unit or none for each wavefront: 320 of 400 rows, 64 of them pivots, 9.6, 10.5.
  const int n_units = (cnt_sal + kRowUnit - 1) / kRowUnit + (win_rows + kRowUnit - 1) / kRowUnit;
  // (eight wavefronts: no longer where the pairs take a second round: 576 salient rows, 256 workgroups of 1000 rows, 20.6, 22.0)
  const bool pairs = a.row_pairs > 0 && n_units >= a.row_pairs && (NW == kWaves || n_units <= 2 * NW + 1);
  auto bf16_units = [&](const uint16_t *ks_base, const uint16_t *vs_base, int cnt, const RowUnits units, auto &&row_ok) {
    for (int i = units.first; i < units.limit; i += units.step) {
      const int unit = pairs ? 2 * i : units.unit(i), s_lane = unit * kRowUnit + lane;
      if (unit * kRowUnit >= cnt) continue;
      const int n_grp = min(pairs ? 4 : 2, (cnt - unit * kRowUnit + 15) >> 4);  // token groups (16 slots) that hold rows
      const bool row_valid = row_ok(s_lane);  // fetched whatever cnt says (clamped address): no load behind a branch
      const bool ok = (pairs | (lane < kRowUnit)) & (s_lane < cnt) & row_valid;
      // (scalar bases and 32-bit lane offsets, as for the code stream)
      u32x4 vb[8];
      auto request_values = [&](int b2) {
#pragma unroll
        for (int half_v = 0; half_v < 2; ++half_v) {
          gptr_u32 v_unit = as_global(reinterpret_cast<const uint32_t *>(vs_base)) + (size_t)(unit + b2) * 2048 + half_v * 1024;
          keep_scalar(v_unit);
#pragma unroll
          for (int nb = 0; nb < 4; ++nb) vb[4 * half_v + nb] = *(const AKVQ_GLOBAL u32x4 *)(v_unit + nb * 256 + lane_code);
        }
      };
      request_values(0);
      auto request_group = [&](int g, bf16x8 (&kb)[4]) {
        gptr_u32 k_group = as_global(reinterpret_cast<const uint32_t *>(ks_base)) + (size_t)unit * 2048 + g * 1024;
        keep_scalar(k_group);
        const uint32_t lane_row = (uint32_t)(mrow * (kD / 2) + 4 * qd);
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) kb[kc] = __builtin_bit_cast(bf16x8, *(const AKVQ_GLOBAL u32x4 *)(k_group + 16 * kc + lane_row));
      };
      f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f};
      auto score_group = [&](int g, const bf16x8 (&kb)[4]) {
        const int term = mrow - 4 * g;
        const uint16_t *ap = &q_plain[(term >= 0 && term < 3) ? term : 3][8 * qd];
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) acc = mfma_bf16(*reinterpret_cast<const bf16x8 *>(ap + 32 * kc), kb[kc], acc);
      };
      if constexpr (kBothGroups) {
        bf16x8 kb[2][4];
        request_group(0, kb[0]);
        if (n_grp > 1) request_group(1, kb[1]);
        score_group(0, kb[0]);
        if (n_grp > 1) score_group(1, kb[1]);
#pragma unroll 1
        for (int g = 2; g < n_grp; ++g) {
          request_group(g, kb[0]);
          score_group(g, kb[0]);
        }
      } else {
#pragma unroll 1
        for (int g = 0; g < n_grp; ++g) {
          bf16x8 kb[4];
          request_group(g, kb);
          score_group(g, kb);
        }
      }
      const float score = sm2 * (acc[0] + acc[1] + acc[2]);
      float p;
      if (!softmax_step(score, ok, true, p)) continue;
      {
        // three terms here: a head that looks at one pivot has that row's rounding of the weight in its result
        const float w = ok ? p : 0.0f;
        float hif, lof;
        split2(w, hif, lof);
        w_lds[blk_of_lane][0][0][slot] = (uint16_t)hi16(hif);
        w_lds[blk_of_lane][0][1][slot] = (uint16_t)hi16(lof);
        w_lds[blk_of_lane][0][2][slot] = (uint16_t)f32_to_bf16_rne((w - hif) - lof);
      }
      wave_lds_sync();
      auto add_values = [&](int b2) {
        const uint16_t *src = mrow < 3 ? &w_lds[b2][0][mrow][8 * qd] : zero16;
        const bf16x8 a_v = *reinterpret_cast<const bf16x8 *>(src);
        // which of this lane's 8 K-slots (pair i, half) are real rows: mask the others (unwritten memory)
        uint32_t keep[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int s0 = (unit + b2) * kRowUnit + 4 * qd + e;  // half 0; half 1 is 16 slots further
          keep[e] = (s0 < cnt ? 0x0000FFFFu : 0u) | (s0 + 16 < cnt ? 0xFFFF0000u : 0u);
        }
#pragma unroll
        for (int nb = 0; nb < 8; ++nb) {
#pragma unroll
          for (int e = 0; e < 4; ++e) vb[nb][e] &= keep[e];
          acc_o[nb] = mfma_bf16(a_v, __builtin_bit_cast(bf16x8, vb[nb]), acc_o[nb]);
        }
      };
      add_values(0);
      if (n_grp > 2) {
        request_values(1);
        add_values(1);
      }
      wave_lds_sync();
    }
  };
  {
    const int32_t *sidx = a.sal_idx + (size_t)bh * a.S_cap;
    bf16_units(a.k_sal + (size_t)bh * a.S_cap * kD, a.v_sal + (size_t)bh * a.S_cap * kD, cnt_sal,
               pairs ? paired_units<NW>(cnt_sal, 0, wave) : salient_units<NW>(a, cnt_sal, split, wave, appends),
               [&](int s) { return sidx[min(s, a.S_cap - 1)] < a.t_win; });  // rows in the window are read there
  }
  if (a.win_len > 0) {
    // slot s holds the row of [t_win, T_len) congruent to s mod W; fine halves and padding rows carry no token
    const int W = a.win_len;
    bf16_units(a.k_win + (size_t)bh * W * kD, a.v_win + (size_t)bh * W * kD, win_rows,
               pairs ? paired_units<NW>(win_rows, cnt_sal, wave) : window_units<NW>(a, cnt_sal, split, wave, appends), [&](int s) {
      int d = (a.T_len - 1 - s) % W;
      d = d < 0 ? d + W : d;
      const int t = a.T_len - 1 - d;
      bool row = t >= a.t_win;
      if constexpr (PAIRS) {
        const int tc = max(t, 0);
        const bool fine = ((a.fine_mask[(size_t)(bh / a.Hkv) * plane_blocks + tc / 32] >> (tc % 32)) & 1u) != 0u;
        const bool pad = (a.k_meta[((size_t)bh * a.T_cap + tc) * NG] & 0xFFFFu) == 0x8000u;
        row = row && !fine && !pad;
      }
      return row;
    });
  }

  // ================= merge the wavefronts, then either finish (one split) or store the partial =================
  {
    const float l_tot = wave_sum_dpp(l_run);
    float corr[NG];  // what the expansion constant and the zero-points added to every channel of the group
#pragma unroll
    for (int g = 0; g < NG; ++g) corr[g] = kCodeBias * wave_sum_dpp(swx[g]) + wave_sum_dpp(szx[g] * rcx);
    if (lane == 0) { mrg_m[wave] = m_run; mrg_l[wave] = l_tot; }
    if (lane < 16) {
#pragma unroll
      for (int nb = 0; nb < 8; ++nb) {
        mrg_o[wave][16 * nb + lane] = (acc_o[nb][0] + acc_o[nb][1]) + acc_o[nb][2] - corr[(NG == 2) ? (nb >> 2) : 0];
      }
    }
  }
  lds_barrier();
  if (wave == 0) merge_waves_and_store<NW>(a, mrg_m, mrg_l, 1, &mrg_o[0][0], kD, (size_t)bh, split, lane);
}

template <int G, bool PAIRS, int NW>
__global__ __launch_bounds__(64 * NW, !PAIRS && G == 128 && NW == kWaves ? 4 : 1) void decode_mha_kernel(DecodeArgs a) { decode_mha_body<G, PAIRS, NW>(a); }

// ------------------------------------------------------------------------------------------------
// GQA (R = Hq/Hkv query heads share a KV head, 2 <= R <= 8; also valid for R = 1).  A tile is one cache block
// (32 tokens, two token groups of 16).  Rows 2h and 2h+1 of an A operand belong to head h: for the code stream they carry
// its query as base-32 digits of a 20-bit integer, for 16-bit rows and weights as two bfloat16 terms.  Lane (n, q) so
// receives heads 2q, 2q+1 of token n, and the same lanes own those heads' output rows.
// ------------------------------------------------------------------------------------------------
template <int NG>
struct GqaTile {
  u32x4 kc, vc;
  uint32_t km[2][NG], vm[2][NG];
  uint32_t fm;  // fine-half mask word of the block (only loaded by the PAIRS instantiations)
};

template <int G, bool PAIRS, int NW>
__global__ __launch_bounds__(64 * NW) void decode_gqa_kernel(DecodeArgs a) {
  constexpr int NG = kD / G;
  // With two groups per row a group's product takes zeros in the other group's slots: in the query operands, which never
  // change (half of 24 registers), or, in the kernel that also tells row pairs apart, in the code operands: it then stays
  // at 168 registers, three wavefronts per SIMD, instead of 176 and two (64/8 heads, 80 sequences of 4572 rows, 4-bit
  // text: 65.6 -> 61.6 us; 28/4 heads, 200 sequences: 85.7 -> 82.2; up to 512 workgroups, where two are enough, the same).
  constexpr bool kMaskCodes = PAIRS && NG == 2;
  __shared__ __attribute__((aligned(16))) int q_int[8][kD];           // queries as integers, in units of their head's U
  __shared__ __attribute__((aligned(16))) uint16_t q_plain[16][kD];   // row 2h+term, natural order
  __shared__ __attribute__((aligned(16))) uint32_t a_lds[2][6][kWave];  // the two operand images of the code stream
  __shared__ float q_sum[8][NG];                                      // per head and group: sum of the queries
  __shared__ uint32_t q_exp[8];                                       // biased exponent above the head's largest query
  __shared__ __attribute__((aligned(16))) uint16_t w_lds_all[NW][NG][16][kTokBlock];  // [group][row][slot]
  __shared__ float mrg_m[NW][8], mrg_l[NW][8];
  __shared__ float mrg_o[NW][8][kD];

  const int tid = threadIdx.x;
  // the wavefront index as a scalar: everything derived from it (tile indices, tile addresses) then lives in scalar
  // registers and the loads take a scalar base plus a per-lane offset
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int split = blockIdx.x;
  const int bh = blockIdx.y;  // b * Hkv + hkv
  const int R = a.Hq / a.Hkv;
  const int b = bh / a.Hkv, hkv = bh % a.Hkv;
  const int mrow = lane & 15, qd = lane >> 4;
  const ExpandK ex;
  const ExpandF4 ex4;
  auto &w_lds = w_lds_all[wave];

  // ---- tile bookkeeping and the first two tiles' loads come first: they do not depend on the queries ----
  const int n_tiles = (a.t_win + kGqaTileRows - 1) / kGqaTileRows;  // rows from t_win on are read from the recent-window rings
  int tile_begin, tile_end;
  decode_split_range(n_tiles, a.n_split, split, tile_begin, tile_end);
  const size_t plane_blocks = (size_t)a.T_cap / kTokBlock;
  // plane bases and tile indices are uniform (scalar registers); a lane adds a fixed 32-bit offset (see the MHA kernel)
  const gptr_u32 kc_plane = as_global(a.k_codes) + (size_t)bh * plane_blocks * kBlockWords;
  const gptr_u32 vc_plane = as_global(a.v_codes) + (size_t)bh * plane_blocks * kBlockWords;
  const gptr_u32 km_plane = as_global(a.k_meta) + (size_t)bh * a.T_cap * NG;
  const gptr_u32 vm_plane = as_global(a.v_meta) + (size_t)bh * a.T_cap * NG;
  const uint32_t lane_code = (uint32_t)lane * 4u, lane_meta = (uint32_t)mrow * NG;

  const uint32_t *fm_base = PAIRS ? a.fine_mask + (size_t)b * plane_blocks : nullptr;
  auto load_tile = [&](int tile, GqaTile<NG> &t) {
    if constexpr (PAIRS) t.fm = fm_base[tile];
    gptr_u32 kc_t = kc_plane + (size_t)tile * kBlockWords, vc_t = vc_plane + (size_t)tile * kBlockWords;
    gptr_u32 km_t = km_plane + (size_t)tile * (32 * NG), vm_t = vm_plane + (size_t)tile * (32 * NG);
    keep_scalar(kc_t); keep_scalar(vc_t); keep_scalar(km_t); keep_scalar(vm_t);
    t.kc = stream_load_x4(kc_t + lane_code);
    t.vc = stream_load_x4(vc_t + lane_code);
#pragma unroll
    for (int tg = 0; tg < 2; ++tg) {
      if constexpr (NG == 2) {
        const u32x2 k2 = stream_load_x2(km_t + 16 * tg * NG + lane_meta);
        const u32x2 v2 = stream_load_x2(vm_t + 16 * tg * NG + lane_meta);
        t.km[tg][0] = k2[0]; t.km[tg][1] = k2[1];
        t.vm[tg][0] = v2[0]; t.vm[tg][1] = v2[1];
      } else {
        t.km[tg][0] = stream_load_x1(km_t + 16 * tg * NG + lane_meta);
        t.vm[tg][0] = stream_load_x1(vm_t + 16 * tg * NG + lane_meta);
      }
    }
  };

  // the length of the salient list is asked for now and looked at after the stream (the append of a fused decode
  // step does not change it): the 16-bit rows then cost one memory round trip, not three dependent ones
  // (read through the constant address space: a scalar load, whose wait the compiler puts in front of the first use;
  // as a vector load of a uniform address it would be moved to a scalar register, and waited for, right here)
  const int sal_cnt_early = reinterpret_cast<const __attribute__((address_space(4))) int32_t *>(
      reinterpret_cast<uintptr_t>(a.sal_cnt))[bh];
  const int n_mine = tile_begin + wave < tile_end ? (tile_end - tile_begin - wave + NW - 1) / NW : 0;
  const int last_tile = tile_begin + wave + NW * max(n_mine - 1, 0);
  auto tile_at = [&](int k) { return min(tile_begin + wave + NW * k, last_tile); };
  GqaTile<NG> tb[3];
  // Fused decode step: the workgroups of the split that owns the row's tile first write the new row (the last wavefront
  // the K row, the one before it the V row); the barrier below orders those stores before this workgroup's loads of that
  // tile, and no other workgroup reads it.  A wavefront whose first two tiles include it asks for them after the barrier.
  // (So does the four-wavefront kernel of tiered caches with two groups, everywhere: what it keeps across the staging
  // otherwise overflows the scalar registers, and scratch memory is reserved for them; same time either way.)
  const bool appends = a.fused_append != 0 && split == a.append_split;  // uniform over the workgroup
  const bool defer_loads = (kMaskCodes && NW == kWaves && n_mine > 0) ||
                           (appends && a.t_win == a.T_len && n_mine > 0 &&
                            (tile_at(0) == n_tiles - 1 || tile_at(1) == n_tiles - 1));
  if (n_mine > 0 && !defer_loads) {
    load_tile(tile_at(0), tb[0]);
    load_tile(tile_at(1), tb[1]);
  }
  if (appends && wave >= NW - 2) {
    __shared__ __attribute__((aligned(16))) uint8_t step_codes[2][kD];
    __shared__ __attribute__((aligned(16))) uint16_t step_row[2][kD];
    append_row_wave<G>(a.step, bh, NW - 1 - wave, lane, step_codes[NW - 1 - wave], step_row[NW - 1 - wave]);
  }
  // Queries, one head per wavefront at a time, two channels (lane, lane + 64) per lane.  sm_scale * log2(e) is folded in,
  // so the products already are base-2 logits.  For the 16-bit rows: two bfloat16 terms.  For the code stream: integers
  // of up to 20 bits in units of a power of two U (2^18 U <= largest |q| < 2^19 U), and their sums per group.  Every channel
  // is off by at most U/2 <= 2^-19 of the largest one: as a vector the query is as exact as with 16 significant bits per
  // channel (2^-17 of its norm), but a channel below 1/4 of the largest one carries less than it would then.
  const float sm2 = a.sm_scale * kLog2e;
#pragma unroll
  for (int hi = 0; hi < 8 / NW; ++hi) {
    const int h = wave + NW * hi;
    float x0 = 0.0f, x1 = 0.0f;
    if (h < R)  // uniform
      rotate_query(a.q + ((size_t)b * a.Hq + hkv * R + h) * kD, x0, x1, a.q_rotated != 0,
                   a.rope_cos ? a.rope_cos + (size_t)b * a.rope_stride : nullptr,
                   a.rope_sin ? a.rope_sin + (size_t)b * a.rope_stride : nullptr, lane);
    x0 *= sm2;
    x1 *= sm2;
    float hif, lof;
    split2(x0, hif, lof);
    q_plain[2 * h][lane] = (uint16_t)hi16(hif); q_plain[2 * h + 1][lane] = (uint16_t)hi16(lof);
    split2(x1, hif, lof);
    q_plain[2 * h][lane + 64] = (uint16_t)hi16(hif); q_plain[2 * h + 1][lane + 64] = (uint16_t)hi16(lof);
    const float mx = wave_max_dpp(fmaxf(fabsf(x0), fabsf(x1)));
    const uint32_t e_biased = min(max(__float_as_uint(mx) >> 23, 20u), 250u);    // mx < 2^(e_biased - 126)
    const float unit_inv = __uint_as_float((272u - e_biased) << 23);             // 1 / U = 2^19 / 2^(e_biased - 126)
    const float n0 = rintf(x0 * unit_inv), n1 = rintf(x1 * unit_inv);
    q_int[h][lane] = (int)n0;
    q_int[h][lane + 64] = (int)n1;
    const float unit = 1.0f / unit_inv;  // exact
    if constexpr (NG == 2) {
      const float s0 = wave_sum_dpp(n0 * unit), s1 = wave_sum_dpp(n1 * unit);
      if (lane == 0) { q_sum[h][0] = s0; q_sum[h][1] = s1; q_exp[h] = e_biased; }
    } else {
      const float s0 = wave_sum_dpp(n0 * unit + n1 * unit);
      if (lane == 0) { q_sum[h][0] = s0; q_exp[h] = e_biased; }
    }
  }
  if (appends) __syncthreads();  // also orders the new row's stores before the loads below
  else lds_barrier();
  if (defer_loads) {
    load_tile(tile_at(0), tb[0]);
    load_tile(tile_at(1), tb[1]);
  }

  // Row operands of the code stream: the integer of a channel is four balanced base-32 digits, |digit| <= 16, which E2M3
  // holds exactly as digit / 8.  Image 0 holds digit 3 in row 2h and digit 2 in row 2h+1, image 1 digits 1 and 0; the
  // products of the two images accumulate on top of each other, every row weighted by its digit's power of 32, the
  // unit U and the factor 16 of the two operands' fractions through the scale operand, so row 2h + row 2h+1 is the
  // dot product.  Slot v of lane (m, q) is what ExpandF4 makes of the code words: word v / 16, field 2*(v % 8) + (v / 8) % 2.
  const uint32_t e_row = q_exp[mrow >> 1];
  uint32_t a_scale[2];
#pragma unroll
  for (int img = 0; img < 2; ++img) a_scale[img] = e_row - 14u + 5u * (uint32_t)(3 - (mrow & 1) - 2 * img);
  if (wave < 2) {
    const int shift = 5 * (3 - (mrow & 1) - 2 * wave);
    f32x16 dig[2];  // even and odd slots, as the packing conversion takes them
#pragma unroll
    for (int w = 0; w < 2; ++w)
#pragma unroll
      for (int f8 = 0; f8 < 2; ++f8) {  // fields 8*f8 .. 8*f8 + 7 of word w: channels 64*w + 32*f8 + 8*q + (0 .. 7)
        const i32x4 lo = *reinterpret_cast<const i32x4 *>(&q_int[mrow >> 1][64 * w + 32 * f8 + 8 * qd]);
        const i32x4 hi = *reinterpret_cast<const i32x4 *>(&q_int[mrow >> 1][64 * w + 32 * f8 + 8 * qd + 4]);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int n = (i < 4 ? lo[i & 3] : hi[i & 3]) + 16 * (1 + 32 + 1024);  // the lower digits offset to 0 .. 31
          const int d = shift == 15 ? n >> 15 : ((n >> shift) & 31) - 16;
          const int slot = 16 * w + 8 * (i & 1) + 4 * f8 + (i >> 1);
          dig[slot & 1][slot >> 1] = 0.125f * (float)d;
        }
      }
    const u32x6 img = __builtin_bit_cast(u32x6, __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(dig[0], dig[1], 1.0f));
#pragma unroll
    for (int i = 0; i < 6; ++i) a_lds[wave][i][lane] = img[i];
  }
  lds_barrier();
  constexpr int kOperands = kMaskCodes ? 1 : NG;
  u32x6 a_k[2][kOperands];
#pragma unroll
  for (int img = 0; img < 2; ++img)
#pragma unroll
    for (int g = 0; g < kOperands; ++g)
#pragma unroll
      for (int i = 0; i < 6; ++i) a_k[img][g][i] = (kOperands == 1 || i / 3 == g) ? a_lds[img][i][lane] : 0u;

  // this lane scores heads h0 = 2*qd and h0+1
  const int h0 = 2 * qd;
  float qsum[2][NG];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int g = 0; g < NG; ++g) qsum[hh][g] = q_sum[h0 + hh][g];

  f32x4 acc_o[8];
#pragma unroll
  for (int nb = 0; nb < 8; ++nb) acc_o[nb] = (f32x4){0.f, 0.f, 0.f, 0.f};
  // Softmax reference (base 2) per head, its trigger level, and this lane's share of the sum.  "No score yet" is a large
  // negative finite number instead of -inf: exp2(x - kNoScore) of a masked score (x = -inf) is 0 and the first real
  // score raises the reference, so neither the weights nor the rescale factor need a special case.
  float m_run[2] = {kNoScore, kNoScore}, m_trig[2] = {kNoScore, kNoScore}, l_run[2] = {0.f, 0.f};
  // Per head and group: szx = running sum of w*cx*zero over this lane's tokens; the sum of the weights themselves
  // (what the expansion constant 128 multiplies) comes out of the matrix cores: one extra product per group and tile
  // against an all-ones operand sums exactly the bfloat16 terms the value product uses, over all 32 slots.
  f32x4 acc_one[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g) acc_one[g] = (f32x4){0.f, 0.f, 0.f, 0.f};
  const bf16x8 ones = __builtin_bit_cast(bf16x8, (u32x4){0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u});
  float szx[2][NG];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int g = 0; g < NG; ++g) szx[hh][g] = 0.0f;

  // The value product wants every weight divided by the 4^k of its token's slot in the code word (k = pair_exp of
  // the token's position, a per-lane constant).  That factor rides in the exponent of the softmax: weights are taken
  // as exp2(score - (reference + 2k)), i.e. already divided; the sums kept per lane (l_run, szx) carry the same factor
  // and are multiplied by 4^k once at the end.
  const int ii = mrow & 3;  // token n = mrow of its group: pair position
  const float two_k = 2.0f * (float)pair_exp(ii);
  const float rcx = 1.0f / pow4_neg(pair_exp(ii));  // 4^k, exact
  float m_off[2] = {kNoScore, kNoScore};             // reference + 2k
  uint32_t minus_lo = 0x0000BF80u, minus_hi = 0xBF800000u;  // bfloat16 pairs (-1, 0) and (0, -1), kept in registers
  asm volatile("" : "+v"(minus_lo), "+v"(minus_hi));

  // scm[hh][tg]: scores of heads h0+hh for tokens (16*tg + mrow) of the tile, -inf where the row does not take part;
  // returns the weights p[hh][tg] (divided by 4^k).  The reference of a head is raised (and its accumulators rescaled)
  // only when one of its scores exceeds it by more than kLazyMax; the common tile pays one compare and one branch.
  auto softmax_step = [&](const float (&scm)[2][2], const bool (&count)[2], float (&p)[2][2]) {
    float top[2];
    bool need = false;
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      top[hh] = fmaxf(scm[hh][0], scm[hh][1]);
      need = need || (top[hh] > m_trig[hh]);
    }
    if (__ballot(need) != 0ull) {
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        const float mx = row_max_dpp(top[hh]);  // the 16 lanes of a row share a head
        if (mx > m_trig[hh]) {
          const float alpha = fast_exp2(m_run[hh] - mx);  // 0 while there was no score
#pragma unroll
          for (int nb = 0; nb < 8; ++nb) { acc_o[nb][2 * hh] *= alpha; acc_o[nb][2 * hh + 1] *= alpha; }
          l_run[hh] *= alpha;
#pragma unroll
          for (int g = 0; g < NG; ++g) {
            acc_one[g][2 * hh] *= alpha;
            acc_one[g][2 * hh + 1] *= alpha;
            szx[hh][g] *= alpha;
          }
          m_run[hh] = mx;
          m_trig[hh] = mx + kLazyMax;
          m_off[hh] = mx + two_k;
        }
      }
    }
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int tg = 0; tg < 2; ++tg) {
        p[hh][tg] = fast_exp2(scm[hh][tg] - m_off[hh]);
        l_run[hh] += count[tg] ? p[hh][tg] : 0.0f;  // a fine half carries its token's weight but is not a token
      }
  };
  // upper halves of two floats packed into one word (two bfloat16 values that are already exact in 16 bits)
  auto pack_hi = [](float lo, float hi) {
    return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
  };

  // ================= code stream =================
  // Only the last tile of the stream can hold rows at or beyond t_win, whose meta words are arbitrary bits.  For that
  // tile the words of such rows are replaced, in registers, by "salient, scale 0" (K) and "scale 0" (V); everything
  // below then needs no validity mask at all: a salient row gets a score of -inf, hence a weight of exactly 0, and the
  // scales of written rows are finite.
  auto process = [&](const GqaTile<NG> &cur, int tile) {
    uint32_t km[2][NG], vm[2][NG];
#pragma unroll
    for (int tg = 0; tg < 2; ++tg)
#pragma unroll
      for (int g = 0; g < NG; ++g) { km[tg][g] = cur.km[tg][g]; vm[tg][g] = cur.vm[tg][g]; }
    if (tile == n_tiles - 1) {  // uniform over the wavefront
#pragma unroll
      for (int tg = 0; tg < 2; ++tg) {
        const bool beyond = tile * 32 + 16 * tg + mrow >= a.t_win;
#pragma unroll
        for (int g = 0; g < NG; ++g) { km[tg][g] = beyond ? 0x8000u : km[tg][g]; vm[tg][g] = beyond ? 0u : vm[tg][g]; }
      }
    }
    float scm[2][2];
    bool ok[2];
#pragma unroll
    for (int tg = 0; tg < 2; ++tg) {
      f32x4 acc[NG];
      const u32x2 c0 = ex4(cur.kc[2 * tg]), c1 = ex4(cur.kc[2 * tg + 1]);
      u32x4 codes[kMaskCodes ? 2 : 1];
      if constexpr (kMaskCodes) {
        codes[0] = (u32x4){c0[0], c0[1], 0u, 0u};
        codes[1] = (u32x4){0u, 0u, c1[0], c1[1]};
      } else {
        codes[0] = (u32x4){c0[0], c0[1], c1[0], c1[1]};
      }
#pragma unroll
      for (int g = 0; g < NG; ++g)
        acc[g] = mfma_f6f4(a_k[0][g % kOperands], a_scale[0], codes[kMaskCodes ? g : 0], (f32x4){0.f, 0.f, 0.f, 0.f});
#pragma unroll
      for (int g = 0; g < NG; ++g)
        acc[g] = mfma_f6f4(a_k[1][g % kOperands], a_scale[1], codes[kMaskCodes ? g : 0], acc[g]);
      // bit 15 of every meta word of a salient row is set: as a binary16 pattern the low half is then negative
      const bool off = meta_is_salient(km[tg][0]);
      ok[tg] = !off;
      const float pen = (PAIRS || !off) ? 0.0f : -INFINITY;
      float s0 = pen, s1 = pen;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const Meta mk = unpack_meta(km[tg][g]);
        // scale * (dot - zero*sum(q))
        s0 = __builtin_fmaf(mk.scale, __builtin_fmaf(-mk.zero, qsum[0][g], acc[g][0] + acc[g][1]), s0);
        s1 = __builtin_fmaf(mk.scale, __builtin_fmaf(-mk.zero, qsum[1][g], acc[g][2] + acc[g][3]), s1);
      }
      scm[0][tg] = s0;
      scm[1][tg] = s1;
    }
    bool count[2] = {true, true};
    if constexpr (PAIRS) {
#pragma unroll
      for (int tg = 0; tg < 2; ++tg) {
        const uint32_t from_me = cur.fm >> (16 * tg + mrow);  // bit 0: this row is a fine half; bit 1: the next one is
        const bool pair = (from_me & 3u) != 0u;               // pairs start on even rows: the partner is lane ^ 1
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          const float partner = dpp_f<0xB1>(scm[hh][tg]);
          const float both = pair ? scm[hh][tg] + partner : scm[hh][tg];
          scm[hh][tg] = ok[tg] ? both : -INFINITY;
        }
        count[tg] = (from_me & 1u) == 0u;
      }
    }
    float p[2][2];
    softmax_step(scm, count, p);
    // weights: rows 4*qd + {0,1,2,3} = (head h0: hi, lo; head h0+1: hi, lo); slots 2*mrow (+1 for the second group)
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      float sv[2], zv[2];
#pragma unroll
      for (int tg = 0; tg < 2; ++tg) {
        const Meta mv = unpack_meta(vm[tg][g]);
        sv[tg] = mv.scale;
        zv[tg] = mv.zero;
      }
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        // two bfloat16 terms per weight: hi = the weight rounded to bfloat16, lo = the (exactly representable)
        // remainder rounded to bfloat16; the zero-point sum takes the fp32 weight (it differs from hi+lo by 2^-17
        // relative, on a term of the size of the result itself)
        const float w0 = p[hh][0] * sv[0], w1 = p[hh][1] * sv[1];
        szx[hh][g] = __builtin_fmaf(w0, zv[0], szx[hh][g]);
        szx[hh][g] = __builtin_fmaf(w1, zv[1], szx[hh][g]);
        const uint32_t hi = pack_bf16x2(w0, w1);
        const uint32_t lo = pack_bf16x2(minus_bf16(hi, minus_lo, w0), minus_bf16(hi, minus_hi, w1));
        const int row = 4 * qd + 2 * hh;
        reinterpret_cast<uint32_t *>(&w_lds[g][row][0])[mrow] = hi;
        reinterpret_cast<uint32_t *>(&w_lds[g][row + 1][0])[mrow] = lo;
      }
    }
    wave_lds_sync();
    bf16x8 a_v[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      a_v[g] = *reinterpret_cast<const bf16x8 *>(&w_lds[g][mrow][8 * qd]);
      acc_one[g] = mfma_bf16(a_v[g], ones, acc_one[g]);
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int g = (NG == 2) ? (w & 1) : 0;
      const int nbx = 4 * (w & 1) + (w >> 1), nby = nbx + 2;
      acc_o[nbx] = mfma_bf16(a_v[g], ex.x(cur.vc[w]), acc_o[nbx]);
      acc_o[nby] = mfma_bf16(a_v[g], ex.y(cur.vc[w]), acc_o[nby]);
    }
    wave_lds_sync();
  };
  // three tile buffers, two tiles of loads in flight (see the MHA kernel)
  if (n_mine > 0) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      settle(tb[i].kc); settle(tb[i].vc);
#pragma unroll
      for (int tg = 0; tg < 2; ++tg)
#pragma unroll
        for (int g = 0; g < NG; ++g) { settle(tb[i].km[tg][g]); settle(tb[i].vm[tg][g]); }
    }
    StreamPace pace(n_mine, a.paced != 0);
    for (int k = 0; k < n_mine; k += 3) {
      pace.done(k);
      load_tile(tile_at(k + 2), tb[2]);
      process(tb[0], tile_at(k));
      if (k + 1 >= n_mine) break;
      load_tile(tile_at(k + 3), tb[0]);
      process(tb[1], tile_at(k + 1));
      if (k + 2 >= n_mine) break;
      load_tile(tile_at(k + 4), tb[1]);
      process(tb[2], tile_at(k + 2));
    }
  }

  // ================= bfloat16 rows: units of 32 slots =================
  // Used twice: the salient overlay (slot = rank in the salient list) and the recent-window rings (slot = row mod W).
  auto bf16_units = [&](const uint16_t *ks_base, const uint16_t *vs_base, int cnt, auto &&row_ok) {
    const int n_units = (cnt + 31) / 32;
    // fused decode step: the 16-bit rows (one of which may be the new row) are read by the appending split only
    const int unit_step = a.fused_append ? NW : NW * a.n_split;
    const int first_unit = a.fused_append ? (appends ? NW - 1 - wave : n_units) : split + (NW - 1 - wave) * a.n_split;
    if (first_unit >= n_units) return;
    bf16x8 a_s[4];
#pragma unroll
    for (int kc = 0; kc < 4; ++kc)
      a_s[kc] = *reinterpret_cast<const bf16x8 *>(&q_plain[mrow][32 * kc + 8 * qd]);
    for (int unit = first_unit; unit < n_units; unit += unit_step) {
      // the value rows and the rows' validity are requested together with the key rows (one round trip for the
      // phase); a token group (16 slots) without rows is not read
      const int n_grp = min(2, (cnt - unit * 32 + 15) >> 4);
      bool lane_ok[2];
#pragma unroll
      for (int tg = 0; tg < 2; ++tg) {
        const int s_lane = unit * 32 + 16 * tg + mrow;
        const bool row_valid = row_ok(s_lane);  // fetched whatever cnt says (clamped address): no load behind a branch
        lane_ok[tg] = (s_lane < cnt) & row_valid;
      }
      u32x4 vb_all[8];
#pragma unroll
      for (int nb = 0; nb < 8; ++nb)
        vb_all[nb] = *reinterpret_cast<const u32x4 *>(vs_base + (size_t)unit * 4096 + nb * 512 + (16 * qd + mrow) * 8);
      float sc[2][2];
      bool ok[2];
#pragma unroll
      for (int tg = 0; tg < 2; ++tg) {
        f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f};
        const int s_lane = unit * 32 + 16 * tg + mrow;
        if (tg < n_grp) {
#pragma unroll
          for (int kc = 0; kc < 4; ++kc) {
            const bf16x8 kb =
                *reinterpret_cast<const bf16x8 *>(ks_base + (size_t)s_lane * kD + 32 * kc + 8 * qd);
            acc = mfma_bf16(a_s[kc], kb, acc);
          }
        }
        ok[tg] = lane_ok[tg];
        sc[0][tg] = ok[tg] ? acc[0] + acc[1] : -INFINITY;
        sc[1][tg] = ok[tg] ? acc[2] + acc[3] : -INFINITY;
      }
      float p[2][2];
      const bool count[2] = {true, true};
      softmax_step(sc, count, p);
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        float hif[2], lof[2];
#pragma unroll
        for (int tg = 0; tg < 2; ++tg) split2(p[hh][tg] * rcx, hif[tg], lof[tg]);  // these rows are plain values: undo the 4^-k
        const int row = 4 * qd + 2 * hh;
        reinterpret_cast<uint32_t *>(&w_lds[0][row][0])[mrow] = pack_hi(hif[0], hif[1]);
        reinterpret_cast<uint32_t *>(&w_lds[0][row + 1][0])[mrow] = pack_hi(lof[0], lof[1]);
      }
      wave_lds_sync();
      const bf16x8 a_v = *reinterpret_cast<const bf16x8 *>(&w_lds[0][mrow][8 * qd]);
      uint32_t keep[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int s0 = unit * 32 + 4 * qd + i;
        keep[i] = (s0 < cnt ? 0x0000FFFFu : 0u) | (s0 + 16 < cnt ? 0xFFFF0000u : 0u);
      }
#pragma unroll
      for (int nb = 0; nb < 8; ++nb) {
        u32x4 vb = vb_all[nb];
#pragma unroll
        for (int i = 0; i < 4; ++i) vb[i] &= keep[i];
        acc_o[nb] = mfma_bf16(a_v, __builtin_bit_cast(bf16x8, vb), acc_o[nb]);
      }
      wave_lds_sync();
    }
  };
  {
    const int cnt = min(max(sal_cnt_early, 0), a.S_cap);
    const int32_t *sidx = a.sal_idx + (size_t)bh * a.S_cap;
    bf16_units(a.k_sal + (size_t)bh * a.S_cap * kD, a.v_sal + (size_t)bh * a.S_cap * kD, cnt,
               [&](int s) { return sidx[min(s, a.S_cap - 1)] < a.t_win; });  // rows in the window are read there
  }
  if (a.win_len > 0) {
    // slot s holds the row of [t_win, T_len) congruent to s mod W; fine halves and padding rows carry no token
    const int W = a.win_len;
    bf16_units(a.k_win + (size_t)bh * W * kD, a.v_win + (size_t)bh * W * kD, W, [&](int s) {
      int d = (a.T_len - 1 - s) % W;
      d = d < 0 ? d + W : d;
      const int t = a.T_len - 1 - d;
      bool row = t >= a.t_win;
      if constexpr (PAIRS) {
        const int tc = max(t, 0);
        const bool fine = ((a.fine_mask[(size_t)b * plane_blocks + tc / 32] >> (tc % 32)) & 1u) != 0u;
        const bool pad = (a.k_meta[((size_t)bh * a.T_cap + tc) * NG] & 0xFFFFu) == 0x8000u;
        row = row && !fine && !pad;
      }
      return row;
    });
  }

  // ================= merge the wavefronts =================
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    const int h = h0 + hh;
    const float l_tot = row_sum_dpp(l_run[hh] * rcx);
    float corr[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g)  // acc_one already holds the sum over all slots (every column the same)
      corr[g] = kCodeBias * (acc_one[g][2 * hh] + acc_one[g][2 * hh + 1]) + row_sum_dpp(szx[hh][g] * rcx);
    if (mrow == 0) { mrg_m[wave][h] = m_run[hh]; mrg_l[wave][h] = l_tot; }
#pragma unroll
    for (int nb = 0; nb < 8; ++nb) {
      mrg_o[wave][h][16 * nb + mrow] = (acc_o[nb][2 * hh] + acc_o[nb][2 * hh + 1]) - corr[(NG == 2) ? (nb >> 2) : 0];
    }
  }
  lds_barrier();
#pragma unroll
  for (int hi = 0; hi < 8 / NW; ++hi) {
    const int h = wave + NW * hi;
    if (h < R)  // uniform
      merge_waves_and_store<NW>(a, &mrg_m[0][h], &mrg_l[0][h], 8, &mrg_o[0][h][0], 8 * kD, (size_t)b * a.Hq + hkv * R + h,
                                split, lane);
  }
}

// ------------------------------------------------------------------------------------------------
// Merge the KV splits (exact log-sum-exp merge), rotate the output back (H is its own inverse), write out.
// One workgroup per (batch, query head).  The launch is bound by memory latency, not by its few KB per head: wavefront w
// takes splits w, w + 4, ... and requests everything it needs of BATCH of them at once (two channels per lane,
// and the reference and sum of the split), none of it dependent on another load, so that up to 64 splits
// cost one or two memory round trips.  Against a loop over the splits with a wait in every round (12.3 us at 19 splits of
// 28 heads, half a KB per split) the whole decode call of that shape went from 28.9 to 19.3 us, with 4 splits of 896 heads
// from 80.8 to 79.9 us, with 3 splits of 128 heads from 19.6 to 18.7 us.
// ------------------------------------------------------------------------------------------------
constexpr int kCombineWaves = 4;
template <int BATCH>  // splits of one wavefront requested together
__global__ __launch_bounds__(64 * kCombineWaves) void decode_combine_kernel(DecodeArgs a) {
  __shared__ float of[kCombineWaves][kD];
  __shared__ float wave_m[kCombineWaves], wave_l[kCombineWaves];
  const int bhq = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const float *part = a.partial + (size_t)bhq * a.n_split * kPartialStride;
  int lane_zero = 0;
  asm volatile("" : "+v"(lane_zero));  // m and l as vector loads, in flight with the others (scalar ones are waited for first)
  float m_run = -INFINITY, l_run = 0.0f, o0 = 0.0f, o1 = 0.0f;  // this wavefront's splits, relative to m_run
  for (int first = wave; first < a.n_split; first += kCombineWaves * BATCH) {
    float m[BATCH], l[BATCH], x0[BATCH], x1[BATCH];
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {  // past the end: the last split again, taken as one without rows
      const float *src = part + (size_t)min(first + i * kCombineWaves, a.n_split - 1) * kPartialStride;
      m[i] = src[lane_zero];
      l[i] = src[lane_zero + 1];
      x0[i] = src[4 + lane];
      x1[i] = src[4 + lane + 64];
    }
    float m_new = m_run;
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      if (first + i * kCombineWaves >= a.n_split) m[i] = -INFINITY;
      m_new = fmaxf(m_new, m[i]);
    }
    const float alpha = m_run == -INFINITY ? 0.0f : fast_exp2(m_run - m_new);
    l_run *= alpha; o0 *= alpha; o1 *= alpha;
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const float wgt = m[i] == -INFINITY ? 0.0f : fast_exp2(m[i] - m_new);  // a split without rows has sums of 0
      l_run += wgt * l[i];
      o0 += wgt * x0[i];
      o1 += wgt * x1[i];
    }
    m_run = m_new;
  }
  if (lane == 0) { wave_m[wave] = m_run; wave_l[wave] = l_run; }
  of[wave][lane] = o0;
  of[wave][lane + 64] = o1;
  __syncthreads();
  if (wave != 0) return;
  float m_all = -INFINITY, l_all = 0.0f;
  o0 = o1 = 0.0f;
#pragma unroll
  for (int w = 0; w < kCombineWaves; ++w) m_all = fmaxf(m_all, wave_m[w]);
#pragma unroll
  for (int w = 0; w < kCombineWaves; ++w) {
    if (wave_m[w] == -INFINITY) continue;
    const float wgt = fast_exp2(wave_m[w] - m_all);
    l_all += wgt * wave_l[w];
    o0 += wgt * of[w][lane];
    o1 += wgt * of[w][lane + 64];
  }
  if (a.lse && lane == 0) a.lse[bhq] = (m_all + __log2f(l_all)) * kLn2;
  unrotate_store_wave(o0 / l_all, o1 / l_all, a.out, (size_t)bhq, a.out_rotated != 0, a.out_half != 0, lane);
}

}  // namespace

template <int G, bool PAIRS>
static void launch_decode_stream(DecodeArgs a, hipStream_t stream) {
  const dim3 grid(a.n_split, a.B * a.Hkv);
  const bool mha = a.Hq == a.Hkv;
  const int rows = mha ? kMhaTileRows : kGqaTileRows;
  // At most one workgroup per CU: with four wavefronts every SIMD would hold a single one, so the workgroups get eight.
  // (Beyond that, eight need more registers than two workgroups of a CU have between them: 384 of them, tiered rows,
  // took 21.7 us instead of 18.7.)
  const long workgroups = (long)a.B * a.Hkv * a.n_split;
  // Eight also where a split's few tiles would do with four, but a fused step leaves one split more 16-bit rows than those have
  // units for (the salient ones, and the window's in the grouped-query kernel): 1100 rows, 28/4 heads, window 512, 8 splits:
  // 19.2 us with four, 15.7 with eight.
  const int alone = !a.fused_append || a.n_split == 1 ? 0 : mha ? a.S_cap : a.S_cap + (a.win_len < a.T_len ? a.win_len : a.T_len);
  const bool wide = workgroups <= kCus && (decode_tiles_per_split((a.t_win + rows - 1) / rows, a.n_split) > kWaves || alone > kWaves * kRowUnit);
  // From how many units of 16-bit rows on they are taken in pairs.  Beyond two workgroups per CU always where the last round of
  // them, four or three per CU by registers, is nearly full (a short one is latency again: 1280 workgroups of 200 rows, 64 of
  // them in the window, 18.9 us by units, 20.6 by pairs).
  constexpr long kRound = (!PAIRS && G == 128 ? 4 : 3) * kCus;
  const long last_round = (workgroups - 1) % kRound + 1;
  if (!mha || a.n_split > 1 || 4 * workgroups <= 3 * kCus) a.row_pairs = 0;
  else if (workgroups <= kCus) a.row_pairs = wide ? kWavesWide + 1 : kWaves + 3;
  else if (workgroups <= 2 * kCus) a.row_pairs = kWaves + 1;
  else a.row_pairs = 8 * last_round >= 5 * kRound ? 1 : 0;
  a.paced = !mha && !wide && workgroups <= 2 * kCus;
  if (mha) {
    if (wide) hipLaunchKernelGGL((decode_mha_kernel<G, PAIRS, kWavesWide>), grid, dim3(64 * kWavesWide), 0, stream, a);
    else hipLaunchKernelGGL((decode_mha_kernel<G, PAIRS, kWaves>), grid, dim3(64 * kWaves), 0, stream, a);
  } else {
    if (wide) hipLaunchKernelGGL((decode_gqa_kernel<G, PAIRS, kWavesWide>), grid, dim3(64 * kWavesWide), 0, stream, a);
    else hipLaunchKernelGGL((decode_gqa_kernel<G, PAIRS, kWaves>), grid, dim3(64 * kWaves), 0, stream, a);
  }
}

hipError_t launch_decode_attention(const DecodeArgs &a_in, int G, hipStream_t stream) {
  DecodeArgs a = a_in;
  {
    const int rows = a.Hq == a.Hkv ? kMhaTileRows : kGqaTileRows;
    a.append_split = decode_last_tile_split((a.t_win + rows - 1) / rows, a.n_split);
  }
  if (a.fine_mask) {
    if (G == 128) launch_decode_stream<128, true>(a, stream);
    else launch_decode_stream<64, true>(a, stream);
  } else {
    if (G == 128) launch_decode_stream<128, false>(a, stream);
    else launch_decode_stream<64, false>(a, stream);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.n_split == 1) return e;
  const dim3 heads(a.B * a.Hq), lanes(64 * kCombineWaves);
  if (a.n_split <= kCombineWaves) hipLaunchKernelGGL(decode_combine_kernel<1>, heads, lanes, 0, stream, a);
  else if (a.n_split <= 2 * kCombineWaves) hipLaunchKernelGGL(decode_combine_kernel<2>, heads, lanes, 0, stream, a);
  else hipLaunchKernelGGL(decode_combine_kernel<8>, heads, lanes, 0, stream, a);
  return hipGetLastError();
}

}  // namespace akvq

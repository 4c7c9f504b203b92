// Salient-token identification (Section III-B of arXiv 2501.15021).
//   TSA layers: the salient set is the text positions -> ordered stream compaction of the modality mask.
//   PSA layers: pivot tokens are the few tokens that receive most of the attention (Section I / III-A.3); the score
//   is the attention-column mass of the last W prompt rows, computed on the matrix cores (bfloat16 operands, fp32
//   accumulate, fp32 softmax) in two streaming passes over K (row statistics, then column sums) or, where the exponentials
//   can wait in registers for the statistics, in one, followed by an exact top-k (radix select on the fp32 bit patterns, ties to the lower position).
#include <atomic>

#include "akvq_device.h"
#include "akvq_kernels.h"

namespace akvq {

namespace {

// Text positions of one batch element, listed for all of its kv-heads by one workgroup per (batch, kv-head).  Latency is
// all there is to it: a row of a few KB, scanned once.  Each thread takes kTsaBytes consecutive positions at a time, so a
// round of loads, one workgroup scan and two barriers cover 4096 positions (256 before: 4001 positions of 256 heads took
// 11.2 us, now 5.9 us), or 16384 with 1024 threads (text_threads).
constexpr int kTsaBytes = 16;
template <int NT>
__global__ __launch_bounds__(NT) void select_tsa_kernel(SelectArgs a) {
  __shared__ int wave_tot[2][NT / 64];
  const int bh = blockIdx.x, b = bh / a.Hkv;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint8_t *mask = a.is_text + (size_t)b * a.T;
  int32_t *out = a.sal_idx + (size_t)bh * a.S_cap;
  const bool aligned = (reinterpret_cast<uintptr_t>(mask) & 15u) == 0;  // uniform: whole rows of 16-byte loads
  int base_count = 0, copy = 0;
  for (int base = 0; base < a.T; base += NT * kTsaBytes, copy ^= 1) {
    const int t0 = base + threadIdx.x * kTsaBytes;
    uint32_t set = 0u;  // bit i: position t0 + i is text
    if (aligned && t0 + kTsaBytes <= a.T) {
      const u32x4 m = *reinterpret_cast<const u32x4 *>(mask + t0);
#pragma unroll
      for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int i = 0; i < 4; ++i) set |= ((m[w] >> (8 * i)) & 0xFFu) != 0u ? 1u << (4 * w + i) : 0u;
    } else {
      uint8_t m[kTsaBytes];  // positions past the end read the last one and are dropped
#pragma unroll
      for (int i = 0; i < kTsaBytes; ++i) m[i] = mask[min(t0 + i, a.T - 1)];
#pragma unroll
      for (int i = 0; i < kTsaBytes; ++i) set |= (t0 + i < a.T && m[i] != 0) ? 1u << i : 0u;
    }
    int upto = __popc(set);  // inclusive prefix over the wavefront, then over the workgroup
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const int up = __shfl_up(upto, off, kWave);
      if (lane >= off) upto += up;
    }
    if (lane == kWave - 1) wave_tot[copy][wave] = upto;
    __syncthreads();  // (two copies: the next round's totals do not overwrite these)
    int pos = base_count + upto - __popc(set);
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
      const int c = wave_tot[copy][w];
      if (w < wave) pos += c;
      base_count += c;
    }
    while (set != 0u) {
      const int i = __ffs((int)set) - 1;
      set &= set - 1u;
      if (pos < a.S_cap) out[pos] = t0 + i;
      ++pos;
    }
  }
  if (threadIdx.x == 0) a.sal_cnt[bh] = base_count;
}

// ---- pivot scoring ---------------------------------------------------------------------------------------
// Scoring windows of fewer than 64 rows (the kernels for W = 64 follow further down): each workgroup (4 wavefronts)
// owns kScoreChunk consecutive keys of one (batch, query head); its wavefronts take the groups of 16 keys in turn,
// with the next groups' loads in flight while the current one goes through the matrix cores.
// Logits are kept in the base-2 domain (sm_scale * log2(e) folded into one multiply) so that exponentials are bare
// v_exp_f32; both passes use the same domain, so the statistics carry over unchanged.
constexpr int kGroupsPerWave = kScoreChunk / (4 * 16);
constexpr int kKeyDepth = 1;  // key groups in flight ahead of the one being scored in the second pass (deeper is slower)
static_assert(kGroupsPerWave % (kKeyDepth + 1) == 0, "the scoring loop is unrolled over the key ring");

// binary16 pair (packed) -> bfloat16 pair (packed), each rounded to nearest even
__device__ __forceinline__ uint32_t half2_to_bf16x2(uint32_t hh) {
  return pack_bf16x2(half_bits_to_float(hh & 0xFFFFu), half_bits_to_float(hh >> 16));
}
__device__ __forceinline__ bf16x8 rows8_as_bf16(u32x4 raw) {
  u32x4 r = {half2_to_bf16x2(raw[0]), half2_to_bf16x2(raw[1]), half2_to_bf16x2(raw[2]), half2_to_bf16x2(raw[3])};
  return __builtin_bit_cast(bf16x8, r);
}

struct KeyGroup {
  u32x4 raw[4];  // 16 keys x 128 channels as this lane's four 8-channel pieces (binary16)
};
__device__ __forceinline__ void load_key_group(const uint16_t *k_rows, int t_first, int T, int mrow, int qd, KeyGroup &g) {
  const int t = min(t_first + mrow, T - 1);  // rows past the end repeat the last key; the causal mask removes them
#pragma unroll
  for (int kc = 0; kc < 4; ++kc)
    g.raw[kc] = *reinterpret_cast<const u32x4 *>(k_rows + (size_t)t * kD + 32 * kc + 8 * qd);
}

// The same 16 keys as they come from memory line by line: load i covers keys 4i .. 4i+3 whole, lane l taking the
// (l % 16)-th 16-byte piece of key 4i + l / 16, so every load is 1 KB of consecutive bytes (eight full cache lines, each
// fetched by one instruction only) and can carry the non-temporal hint.
__device__ __forceinline__ void load_key_lines(const uint16_t *k_rows, int t_first, int T, int lane, KeyGroup &g) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int t = min(t_first + 4 * i + (lane >> 4), T - 1);  // rows past the end repeat the last key; the causal mask removes them
    g.raw[i] = stream_load(reinterpret_cast<const u32x4 *>(k_rows + (size_t)t * kD + 8 * (lane & 15)));
  }
}
// ... turned into matrix-core operands through the wavefront's own 4 KB of LDS (converted to bfloat16 on the way in):
// piece p of key r sits at slot r * 16 + (p ^ r), which keeps both the writes (16 pieces of one key) and the reads (one
// piece of 16 keys) free of bank conflicts.  Same wavefront on both sides; its LDS instructions complete in order.
__device__ __forceinline__ void lines_to_operands(const KeyGroup &g, u32x4 *tile, int lane, bf16x8 (&kb)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 4 * i + (lane >> 4), p = lane & 15;
    tile[r * 16 + (p ^ r)] = __builtin_bit_cast(u32x4, rows8_as_bf16(g.raw[i]));
  }
  const int mrow = lane & 15, qd = lane >> 4;
#pragma unroll
  for (int kc = 0; kc < 4; ++kc) kb[kc] = __builtin_bit_cast(bf16x8, tile[mrow * 16 + ((4 * kc + qd) ^ mrow)]);
}
// products of such operands with the query rows in LDS, keys as the first operand: acc[rb][i] = key 4*qd + i of the
// group, tail row 16*rb + mrow (the query operands are re-read per group behind an opaque offset, see score_16keys)
template <int NRB>
__device__ __forceinline__ void score_operands_by_row(const u32x4 *q_lds, const bf16x8 (&kb)[4], int mrow, int qd,
                                                      f32x4 (&acc)[4]) {
  uint32_t lane_off = (uint32_t)(qd * 16 + mrow);
  asm volatile("" : "+v"(lane_off));
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    acc[rb] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < 4; ++kc)
      acc[rb] = mfma_bf16(kb[kc], __builtin_bit_cast(bf16x8, q_lds[(rb * 4 + kc) * 64 + lane_off]), acc[rb]);
  }
}
// dot products of the W tail rows of one query head with 16 keys: acc[rb][i] = row 16*rb + 4*qd + i, key = mrow
template <int NRB>
__device__ __forceinline__ void score_16keys(const u32x4 *q_lds, const KeyGroup &g, int mrow, int qd, f32x4 (&acc)[4]) {
  // The query operands live in LDS and are re-read for every key group: the offset is made opaque so the reads are
  // not hoisted out of the caller's loop into 64 registers (which would cost a wavefront of occupancy).
  uint32_t lane_off = (uint32_t)(qd * 16 + mrow);
  asm volatile("" : "+v"(lane_off));
  bf16x8 kb[4];
#pragma unroll
  for (int kc = 0; kc < 4; ++kc) kb[kc] = rows8_as_bf16(g.raw[kc]);
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    acc[rb] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < 4; ++kc)
      acc[rb] = mfma_bf16(__builtin_bit_cast(bf16x8, q_lds[(rb * 4 + kc) * 64 + lane_off]), kb[kc], acc[rb]);
  }
}
// causal visibility of key t for tail row `row` (the row sits at position T-W+row); keys past the end are never seen
__device__ __forceinline__ bool key_seen(int t, int row, int T, int W) { return t < T && t <= T - W + row; }
// a group of 16 keys starting at t_first needs per-element masking only if it reaches past position T-W
__device__ __forceinline__ bool group_has_masked(int t_first, int T, int W) { return t_first + 15 > T - W; }

// the W tail rows of one query head as matrix-core A operands in LDS: slot (rb, kc, lane) is what lane (mrow, qd)
// feeds for row block rb and channel step kc; wavefront w converts row blocks w, w+4, ...
template <int NRB>
__device__ __forceinline__ void stage_query_rows(const uint16_t *q_head, int wave, int mrow, int qd, u32x4 *q_lds) {
  for (int rb = wave; rb < NRB; rb += 4)
#pragma unroll
    for (int kc = 0; kc < 4; ++kc)
      q_lds[(rb * 4 + kc) * 64 + qd * 16 + mrow] = __builtin_bit_cast(u32x4, rows8_as_bf16(
          *reinterpret_cast<const u32x4 *>(q_head + (size_t)(16 * rb + mrow) * kD + 32 * kc + 8 * qd)));
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kStatsMost = 1152921504606846976.0f;  // 2^60: a row's sum beyond it (or infinite, or NaN) has its reference raised
constexpr float kLazyRaise = 12.0f;  // a row reference is raised only for logits this far (base 2) above it
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }  // bare v_exp_f32

// ---- row statistics of the first pass, key-major ---------------------------------------------------------------
// The products are taken with the keys as the first operand: acc[rb][i] = key 4*qd + i of the group against tail row
// row0 + 16*rb + mrow, so a lane holds four keys of ONE tail row per row block, and a row's reference m and partial sum l
// are one register each (shared with the three other lanes of the row) instead of four.
// m is a reference, not the running maximum: it is raised only when a logit exceeds it by more than kLazyRaise (or at
// the causal edge), so in the common case the sums just grow; otherwise the references are raised to the row maxima
// of the group and the sums rescaled.
struct RowStats {
  float m[4], l[4];
};
template <int NRB>
__device__ __forceinline__ void stats_raise_and_add(RowStats &s, const f32x4 (&acc)[4], float scale2, int t_first, int T,
                                                    int W, int mrow, int qd, int row0 = 0) {
  int t = t_first + 4 * qd;
  asm volatile("" : "+v"(t));  // keeps the masks from being precomputed ahead of the loop
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    float sv[4];
    bool seen[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      seen[i] = key_seen(t + i, row0 + 16 * rb + mrow, T, W);
      sv[i] = seen[i] ? scale2 * acc[rb][i] : -INFINITY;
    }
    float top = fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]));
    top = fmaxf(top, __shfl_xor(top, 16, kWave));
    top = fmaxf(top, __shfl_xor(top, 32, kWave));
    if (top > s.m[rb]) {  // uniform over the row's four lanes; a reference of -inf goes with a zero sum
      s.l[rb] *= fast_exp2(s.m[rb] - top);
      s.m[rb] = top;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (seen[i]) s.l[rb] += fast_exp2(sv[i] - s.m[rb]);
  }
}
// a group every key of which is seen by every tail row
template <int NRB>
__device__ __forceinline__ void stats_add_group(RowStats &s, const f32x4 (&acc)[4], float scale2, int t_first, int T,
                                                int W, int mrow, int qd, int row0 = 0) {
  float x[4][4];
  float top = -INFINITY;
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[rb][i] = __builtin_fmaf(acc[rb][i], scale2, -s.m[rb]);
      top = fmaxf(top, x[rb][i]);
    }
  if (__ballot(!(top <= kLazyRaise)) == 0ull) {
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
      s.l[rb] += (fast_exp2(x[rb][0]) + fast_exp2(x[rb][1])) + (fast_exp2(x[rb][2]) + fast_exp2(x[rb][3]));
  } else {
    stats_raise_and_add<NRB>(s, acc, scale2, t_first, T, W, mrow, qd, row0);
  }
}
// ... without a look at how far above the reference they are: the sums tell (kStatsMost)
template <int NRB>
__device__ __forceinline__ void stats_add_unseen(RowStats &s, const f32x4 (&acc)[4], float scale2) {
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    float e[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) e[i] = fast_exp2(__builtin_fmaf(acc[rb][i], scale2, -s.m[rb]));
    s.l[rb] += (e[0] + e[1]) + (e[2] + e[3]);
  }
}
// the row's four lanes share the reference: their sums add up (lanes of quarter 0 hold the result)
__device__ __forceinline__ float stats_row_sum(float l) {
  l += __shfl_xor(l, 16, kWave);
  l += __shfl_xor(l, 32, kWave);
  return l;
}

// pass 1: per (b, hq, chunk): reference and sum of exponentials (base 2) of every tail row
constexpr int kStatsDepth = 3;  // key groups in flight ahead of the one being scored in the first pass
static_assert(kGroupsPerWave % (kStatsDepth + 1) == 0, "the scoring loop is unrolled over the key ring");
template <int NRB>
__global__ __launch_bounds__(256, 4) void psa_row_stats_kernel(SelectArgs a) {  // 4 wavefronts per SIMD: at most 128 registers
  __shared__ float st_m[4][64], st_l[4][64];
  const int chunk = blockIdx.x, bhq = blockIdx.y;
  const int b = bhq / a.Hq, hq = bhq % a.Hq, hkv = hq / (a.Hq / a.Hkv);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, mrow = lane & 15, qd = lane >> 4;
  const uint16_t *k_rows = a.k + ((size_t)b * a.Hkv + hkv) * a.T * kD;
  const float scale2 = a.sm_scale * kLog2e;
  __shared__ u32x4 q_lds[NRB * 4 * 64];
  __shared__ u32x4 key_tile[4][256];
  // the wavefronts take the chunk's groups of 16 keys in turn, so the workgroup walks its keys front to back in 16 KB
  // windows (a quarter of the chunk per wavefront, i.e. four distant streams per workgroup, is 3-4 % slower on HBM)
  const int t_wave = chunk * kScoreChunk + wave * 16;
  // kStatsDepth groups of keys are in flight ahead of the one being scored (a ring of register buffers; loads are
  // unconditional with clamped addresses, so the wait counts the compiler derives stay exact).  The first keys are
  // requested before the query rows are staged, so the two latencies overlap.  The keys come line by line with the
  // non-temporal hint and are turned into operands through LDS (2-4 % of the pass; the second pass would lose a
  // workgroup per CU to the extra 16 KB and keeps its direct half-line loads).
  KeyGroup ring[kStatsDepth + 1];
#pragma unroll
  for (int p = 0; p < kStatsDepth; ++p) load_key_lines(k_rows, t_wave + 64 * p, a.T, lane, ring[p]);
  stage_query_rows<NRB>(a.q_tail + (size_t)bhq * a.W * kD, wave, mrow, qd, q_lds);
  __syncthreads();
  RowStats st;  // of tail row 16*rb + mrow, over the keys 4*qd .. 4*qd + 3 of every group
#pragma unroll
  for (int rb = 0; rb < 4; ++rb) { st.m[rb] = -INFINITY; st.l[rb] = 0.0f; }
  for (int g0 = 0; g0 < kGroupsPerWave; g0 += kStatsDepth + 1)
#pragma unroll
  for (int u = 0; u <= kStatsDepth; ++u) {
    const int g = g0 + u;
    const int t_first = t_wave + 64 * g;
    load_key_lines(k_rows, t_wave + 64 * min(g + kStatsDepth, kGroupsPerWave - 1), a.T, lane,
                   ring[(u + kStatsDepth) % (kStatsDepth + 1)]);
    if (t_first >= a.T) continue;  // uniform over the wavefront
    f32x4 acc[4];
    bf16x8 kb[4];
    lines_to_operands(ring[u], key_tile[wave], lane, kb);
    score_operands_by_row<NRB>(q_lds, kb, mrow, qd, acc);
    if (!group_has_masked(t_first, a.T, a.W)) stats_add_group<NRB>(st, acc, scale2, t_first, a.T, a.W, mrow, qd);
    else stats_raise_and_add<NRB>(st, acc, scale2, t_first, a.T, a.W, mrow, qd);
  }
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    const float lr = stats_row_sum(st.l[rb]);
    if (qd == 0) { st_m[wave][16 * rb + mrow] = st.m[rb]; st_l[wave][16 * rb + mrow] = lr; }
  }
  __syncthreads();
  if (threadIdx.x < a.W) {
    const int row = threadIdx.x;
    float mm = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) mm = fmaxf(mm, st_m[w][row]);
    float ll = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w)
      if (st_m[w][row] != -INFINITY) ll += st_l[w][row] * fast_exp2(st_m[w][row] - mm);
    float *dst = a.row_stats + (((size_t)bhq * a.n_chunk + chunk) * a.W + row) * 2;
    dst[0] = mm;
    dst[1] = ll;
  }
}

// Reference and reciprocal sum of one tail row over all chunks.  The chunks' statistics are requested kMergeBatch at a
// time, independent of one another: one memory round trip per batch, where a loop with a wait per load spent two per
// chunk in front of every workgroup of the second pass.
constexpr int kMergeBatch = 16;
__device__ __forceinline__ void merge_chunk_stats(const SelectArgs &a, int bhq, int row, float &m_out, float &il_out) {
  const float *src = a.row_stats + ((size_t)bhq * a.n_chunk * a.W + row) * 2;
  float mm = -INFINITY, ll = 0.0f;
  for (int c0 = 0; c0 < a.n_chunk; c0 += kMergeBatch) {
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    f32x2 ml[kMergeBatch];  // past the end: the last chunk again, left out below
#pragma unroll
    for (int i = 0; i < kMergeBatch; ++i)
      ml[i] = *reinterpret_cast<const f32x2 *>(src + (size_t)min(c0 + i, a.n_chunk - 1) * a.W * 2);
    float m_new = mm;
#pragma unroll
    for (int i = 0; i < kMergeBatch; ++i) m_new = fmaxf(m_new, ml[i][0]);
    if (mm != -INFINITY) ll *= fast_exp2(mm - m_new);
#pragma unroll
    for (int i = 0; i < kMergeBatch; ++i)
      if (c0 + i < a.n_chunk && ml[i][0] != -INFINITY) ll += ml[i][1] * fast_exp2(ml[i][0] - m_new);
    mm = m_new;
  }
  m_out = mm;
  il_out = 1.0f / ll;
}

// pass 2: per (b, hkv, chunk): mass[t] = sum over the group's heads and the tail rows of 2^(s - m_row) / l_row
template <int NRB>
__global__ __launch_bounds__(256, 4) void psa_mass_kernel(SelectArgs a) {  // registers and LDS sized for 4 workgroups per CU
  __shared__ __attribute__((aligned(16))) float row_m[64], row_il[64];
  __shared__ u32x4 q_lds[NRB * 4 * 64];
  const int chunk = blockIdx.x, bh = blockIdx.y;
  const int b = bh / a.Hkv, hkv = bh % a.Hkv, R = a.Hq / a.Hkv;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, mrow = lane & 15, qd = lane >> 4;
  const uint16_t *k_rows = a.k + (size_t)bh * a.T * kD;
  const float scale2 = a.sm_scale * kLog2e;
  const int t_wave = chunk * kScoreChunk + wave * 16;  // groups of 16 keys dealt to the wavefronts in turn
  // column sums of the chunk, one slot per (pair of row quarters, key): the two quarters of a pair are added across
  // lanes first, every slot then has a single owning lane, so the sums over key groups and over the heads of the
  // group are plain read-add-write in a fixed order
  __shared__ float col_lds[2 * kScoreChunk];
  for (int i = threadIdx.x; i < 2 * kScoreChunk; i += 256) col_lds[i] = 0.0f;
  for (int h = 0; h < R; ++h) {
    const int bhq = b * a.Hq + hkv * R + h;
    KeyGroup ring[kKeyDepth + 1];  // first keys requested before the row statistics and query rows are staged
#pragma unroll
    for (int p = 0; p < kKeyDepth; ++p) load_key_group(k_rows, t_wave + 64 * p, a.T, mrow, qd, ring[p]);
    __syncthreads();
    if (threadIdx.x < a.W) merge_chunk_stats(a, bhq, threadIdx.x, row_m[threadIdx.x], row_il[threadIdx.x]);
    stage_query_rows<NRB>(a.q_tail + (size_t)bhq * a.W * kD, wave, mrow, qd, q_lds);
    __syncthreads();
#pragma unroll
    for (int p = 0; p < kKeyDepth; ++p)
#pragma unroll
      for (int kc = 0; kc < 4; ++kc) settle(ring[p].raw[kc]);
    for (int g0 = 0; g0 < kGroupsPerWave; g0 += kKeyDepth + 1)
#pragma unroll
    for (int u = 0; u <= kKeyDepth; ++u) {
      const int g = g0 + u;
      const int t_first = t_wave + 64 * g;
      load_key_group(k_rows, t_wave + 64 * min(g + kKeyDepth, kGroupsPerWave - 1), a.T, mrow, qd,
                     ring[(u + kKeyDepth) % (kKeyDepth + 1)]);
      if (t_first >= a.T) continue;  // uniform over the wavefront
      const KeyGroup &cur = ring[u];
      f32x4 acc[4];
      score_16keys<NRB>(q_lds, cur, mrow, qd, acc);
      uint32_t row_off = (uint32_t)(4 * qd);  // opaque for the same reason as the query operands
      asm volatile("" : "+v"(row_off));
      const bool masked = group_has_masked(t_first, a.T, a.W);  // uniform over the wavefront
      float c0 = 0.0f, c1 = 0.0f;  // two chains: even and odd row blocks
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) {
        const f32x4 rm = *reinterpret_cast<const f32x4 *>(row_m + 16 * rb + row_off);
        const f32x4 ril = *reinterpret_cast<const f32x4 *>(row_il + 16 * rb + row_off);
        float &c = (rb & 1) ? c1 : c0;
        if (!masked) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            c = __builtin_fmaf(fast_exp2(__builtin_fmaf(acc[rb][i], scale2, -rm[i])), ril[i], c);
        } else {
          int t = t_first + mrow;
          asm volatile("" : "+v"(t));  // keeps the masks of all groups from being precomputed ahead of the loop
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (key_seen(t, 16 * rb + 4 * qd + i, a.T, a.W))
              c = __builtin_fmaf(fast_exp2(__builtin_fmaf(acc[rb][i], scale2, -rm[i])), ril[i], c);
        }
      }
      float c = c0 + c1;
      c += __shfl_xor(c, 16, kWave);  // quarters qd and qd ^ 1
      if ((qd & 1) == 0) {
        float *slot = col_lds + (qd >> 1) * kScoreChunk + (t_first - chunk * kScoreChunk) + mrow;
        *slot += c;
      }
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kScoreChunk; i += 256) {
    const int t = chunk * kScoreChunk + i;
    if (t < a.T)
      a.mass[(size_t)bh * a.T + t] = col_lds[i] + col_lds[kScoreChunk + i];
  }
}

// ---- pivot scoring, W = 64: scoring wavefronts with their rows in registers, keys fed through LDS -----------------
// (any number of query heads per KV head up to eight; the kernels above serve the other W)
// One workgroup per (batch, kv-head, chunk of kScoreChunk keys) with one or two wavefronts per query head of the group,
// each holding all or half of the head's W = 64 tail rows in registers as one matrix operand.  The keys are read from
// HBM and converted to bfloat16 once for the whole group: blocks of 64 keys go through LDS (two buffers, laid out as
// matrix-core operands) and every scoring wavefront multiplies all of them with its rows.  Per block: the keys of the
// block after next are requested into registers, the next block's are converted and stored to LDS, the current block
// is scored; one barrier per block orders the buffers.  With fewer than eight heads per KV head the keys are brought
// in by wavefronts of their own (feeders: two in the first pass, one in the second, which also adds up the column
// sums); with eight heads the scoring wavefronts share that work.
// The first pass runs two wavefronts per head (32 rows and under 128 registers each, four wavefronts per SIMD: 10 %
// faster than one per head at about 200 registers and two per SIMD); the second pass one per head (with two, every
// key operand is read from LDS twice for half the arithmetic each time: 17 % slower), except with a single head.
// The feeders read whole keys (1 KB of consecutive bytes per load, non-temporal); against the kernels above, whose
// wavefronts load, convert and score their own keys, that is 2-7 % per pass with one head per KV head.
constexpr int kGqaBlockGroups = 4;                                // groups of 16 keys per block
constexpr int kGqaBlockKeys = 16 * kGqaBlockGroups;               // 64
constexpr int kGqaItems = kGqaBlockGroups * 4;                    // 1 KB pieces (four whole keys each) of a block
constexpr int kGqaMaxHeads = 8;                                   // query heads per KV head
constexpr int kGqaFeederItems = kGqaItems / 2;                    // MAXIT from this on: feeder wavefronts bring in the keys
static_assert(kGqaBlockKeys == 64 && kScoreChunk % 64 == 0, "a chunk is a whole number of blocks: a multiple of 64 keys");
static_assert(kGqaBlockGroups % 2 == 0, "the first pass walks a block two groups at a time");
static_assert(kGqaItems % (2 * kGqaMaxHeads) == 0, "up to sixteen scoring wavefronts share a block's pieces evenly");

// MAXIT: pieces of a block one wavefront brings in: pieces first, first + stride, ... (all of them for the feeder;
// kGqaItems / (scoring wavefronts) each when eight heads' scoring wavefronts share the work).  The loads are unconditional and in
// straight-line code, so that they are in flight together (under per-piece branches the wait counts the compiler
// inserts serialise them).
template <int MAXIT>
struct KeyStage {
  u32x4 raw[MAXIT];
};
template <int MAXIT>
__device__ __forceinline__ void request_block(const uint16_t *k_rows, int t_block, int T, int first, int stride, int mrow,
                                              int qd, KeyStage<MAXIT> &st) {
  // piece `item` of a block = keys 4*item .. 4*item + 3 whole: lane l takes the (l % 16)-th 16 bytes of key
  // 4*item + l / 16, so a load is 1 KB of consecutive bytes and can carry the non-temporal hint (every key is read
  // once per pass)
  const int lane = qd * 16 + mrow;
#pragma unroll
  for (int it = 0; it < MAXIT; ++it) {
    const int item = first + it * stride;  // uniform over the wavefront
    const int t = min(t_block + 4 * item + (lane >> 4), T - 1);  // rows past the end repeat the last key; never scored unmasked
    st.raw[it] = stream_load(reinterpret_cast<const u32x4 *>(k_rows + (size_t)t * kD + 8 * (lane & 15)));
  }
}
template <int MAXIT>
__device__ __forceinline__ void deposit_block(const KeyStage<MAXIT> &st, u32x4 *buf, int first, int stride, int lane) {
  // LDS layout of a block: key r of the block at r * 16 slots of 16 bytes, its piece p at slot p ^ (r % 16): the
  // writes here (16 pieces of one key per 16 lanes) and the operand reads (one piece of 16 keys) are both free of
  // bank conflicts
#pragma unroll
  for (int it = 0; it < MAXIT; ++it) {
    const int r = 4 * (first + it * stride) + (lane >> 4), p = lane & 15;
    buf[r * 16 + (p ^ (r & 15))] = __builtin_bit_cast(u32x4, rows8_as_bf16(st.raw[it]));
  }
}
// NRB row blocks of one query head, from row block rb0 on, as matrix-core operands in registers: q[rb * 4 + kc] is
// what this lane feeds for row block rb0 + rb and channel step kc
template <int NRB>
__device__ __forceinline__ void load_query_rows(const uint16_t *q_head, int rb0, int mrow, int qd, bf16x8 (&q)[NRB * 4]) {
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
    for (int kc = 0; kc < 4; ++kc)
      q[rb * 4 + kc] = rows8_as_bf16(
          *reinterpret_cast<const u32x4 *>(q_head + (size_t)(16 * (rb0 + rb) + mrow) * kD + 32 * kc + 8 * qd));
}
// One group of 16 keys of a block against the wavefront's rows: the keys' operands are read from LDS
// (read_block_group) and multiplied (products_of_group) in two steps, so that loops can read a group ahead of its
// products.  Row-major: acc[rb][i] = row 16*rb + 4*qd + i of the wavefront's rows, key mrow; BY_ROW swaps the
// operands: acc[rb][i] = key 4*qd + i of the group, row 16*rb + mrow.
__device__ __forceinline__ void read_block_group(const u32x4 *buf, int g, int lane, bf16x8 (&kb)[4]) {
  const int mrow = lane & 15, qd = lane >> 4;  // key 16*g + mrow of the block, channel pieces 4*kc + qd
#pragma unroll
  for (int kc = 0; kc < 4; ++kc) kb[kc] = __builtin_bit_cast(bf16x8, buf[(16 * g + mrow) * 16 + ((4 * kc + qd) ^ mrow)]);
}
template <int NRB, bool BY_ROW>
__device__ __forceinline__ void products_of_group(const bf16x8 (&q)[NRB * 4], const bf16x8 (&kb)[4], f32x4 (&acc)[4]) {
  // channel step outermost: consecutive products belong to different row blocks, so none waits for the one before it
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) acc[rb] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kc = 0; kc < 4; ++kc)
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
      acc[rb] = BY_ROW ? mfma_bf16(kb[kc], q[rb * 4 + kc], acc[rb]) : mfma_bf16(q[rb * 4 + kc], kb[kc], acc[rb]);
}
template <int NRB, bool BY_ROW>
__device__ __forceinline__ void score_block_group(const bf16x8 (&q)[NRB * 4], const u32x4 *buf, int g, int lane,
                                                  f32x4 (&acc)[4]) {
  bf16x8 kb[4];
  read_block_group(buf, g, lane, kb);
  products_of_group<NRB, BY_ROW>(q, kb, acc);
}

// pass 1: per (b, hq, chunk): reference and sum of exponentials (base 2) of every tail row, as psa_row_stats_kernel.
// NRB: row blocks per wavefront (4: one wavefront per head; 2: two).
// LONG: chunks of 2048 keys.  Their blocks are added up without a look at the logits, branch-free, and the sums tell whether one
// lay far above its row's reference: such a block is done again, group by group.  Us per selection, without and with it:
// 32 x 32768 keys, 28/4 heads, 1207 -> 1152 (of which this pass is half), 16 x 8192, 32/8 heads, 226.5 -> 221.7; with shorter chunks
// the first references cost what it gains or more (20 x 2500, 28/4 heads, 77.6 -> 79.9).
template <int NRB, int MAXIT, bool LONG>
__global__ __launch_bounds__(64 * kGqaMaxHeads * (4 / NRB)) void psa_row_stats_gqa_kernel(SelectArgs a) {
  constexpr int kHeadWaves = 4 / NRB;                      // wavefronts per query head
  constexpr int kMaxWaves = kGqaMaxHeads * kHeadWaves;     // scoring wavefronts of a workgroup, at most
  __shared__ u32x4 kbuf[2][kGqaItems * 64];
  const int chunk = blockIdx.x, bh = blockIdx.y;
  const int R = a.Hq / a.Hkv, b = bh / a.Hkv, hkv = bh % a.Hkv;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, mrow = lane & 15, qd = lane >> 4;
  const int n_score = R * kHeadWaves;                 // scoring wavefronts
  const int head = wave / kHeadWaves, rb0 = (wave % kHeadWaves) * NRB;  // this wavefront's head and first row block
  const int bhq = b * a.Hq + hkv * R + head;
  const uint16_t *k_rows = a.k + (size_t)bh * a.T * kD;
  const float scale2 = a.sm_scale * kLog2e;
  const int t_chunk = chunk * a.chunk;
  const int n_blk = (min(a.chunk, a.T - t_chunk) + kGqaBlockKeys - 1) / kGqaBlockKeys;  // blocks that hold keys
  // feeders (kGqaItems / MAXIT wavefronts behind the scoring ones) take consecutive pieces; without feeders the
  // scoring wavefronts take pieces wave, wave + kMaxWaves, ...
  constexpr bool kFeeder = MAXIT >= kGqaFeederItems;
  const int first = kFeeder ? (wave - n_score) * MAXIT : wave, stride = kFeeder ? 1 : kMaxWaves;
  KeyStage<MAXIT> st;
  if (kFeeder && wave >= n_score) {  // a feeder: same barriers as the scoring wavefronts below
    request_block(k_rows, t_chunk, a.T, first, stride, mrow, qd, st);
    deposit_block(st, kbuf[0], first, stride, lane);
    request_block(k_rows, t_chunk + kGqaBlockKeys, a.T, first, stride, mrow, qd, st);
    __syncthreads();
    for (int j = 0; j < n_blk; ++j) {
      if (j + 1 < n_blk) deposit_block(st, kbuf[(j + 1) & 1], first, stride, lane);
      if (j + 2 < n_blk) request_block(k_rows, t_chunk + (j + 2) * kGqaBlockKeys, a.T, first, stride, mrow, qd, st);
      __syncthreads();
    }
    return;
  }
  if constexpr (!kFeeder) request_block(k_rows, t_chunk, a.T, first, stride, mrow, qd, st);
  bf16x8 q[NRB * 4];
  load_query_rows<NRB>(a.q_tail + (size_t)bhq * a.W * kD, rb0, mrow, qd, q);
  if constexpr (!kFeeder) {
    deposit_block(st, kbuf[0], first, stride, lane);
    request_block(k_rows, t_chunk + kGqaBlockKeys, a.T, first, stride, mrow, qd, st);
  }
  RowStats st_row;  // of tail row 16*(rb0 + rb) + mrow, over the keys 4*qd .. 4*qd + 3 of every group
#pragma unroll
  for (int rb = 0; rb < 4; ++rb) { st_row.m[rb] = -INFINITY; st_row.l[rb] = 0.0f; }
  __syncthreads();
  for (int j = 0; j < n_blk; ++j) {
    if constexpr (!kFeeder) {
      if (j + 1 < n_blk) deposit_block(st, kbuf[(j + 1) & 1], first, stride, lane);
      if (j + 2 < n_blk) request_block(k_rows, t_chunk + (j + 2) * kGqaBlockKeys, a.T, first, stride, mrow, qd, st);
    }
    const u32x4 *buf = kbuf[j & 1];
    const int t_block = t_chunk + j * kGqaBlockKeys;
    bool again = true;  // the block's groups one by one, references raised as needed
    if (t_block + kGqaBlockKeys - 1 <= a.T - a.W) {
      // Every key of the block is seen by every tail row (all but the last blocks of a context): no masks; keys are
      // read from LDS one group ahead of their products, the products issued one group ahead of the exponentials.
      again = false;
      f32x4 acc_a[4], acc_b[4];
      bf16x8 kb_a[4], kb_b[4];
      if (LONG && j == 0) {  // references from the chunk's first group
        score_block_group<NRB, true>(q, buf, 0, lane, acc_a);
        stats_raise_and_add<NRB>(st_row, acc_a, scale2, t_block, a.T, a.W, mrow, qd, 16 * rb0);
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) st_row.l[rb] = 0.0f;
      }
      const RowStats before = st_row;
      auto add = [&](const f32x4 (&acc)[4], int g) {
        if constexpr (LONG) stats_add_unseen<NRB>(st_row, acc, scale2);
        else stats_add_group<NRB>(st_row, acc, scale2, t_block + 16 * g, a.T, a.W, mrow, qd, 16 * rb0);
      };
      read_block_group(buf, 0, lane, kb_a);
      read_block_group(buf, 1, lane, kb_b);
      products_of_group<NRB, true>(q, kb_a, acc_a);
#pragma unroll
      for (int g = 0; g < kGqaBlockGroups; g += 2) {
        if (g + 2 < kGqaBlockGroups) read_block_group(buf, g + 2, lane, kb_a);
        products_of_group<NRB, true>(q, kb_b, acc_b);
        add(acc_a, g);
        if (g + 2 < kGqaBlockGroups) {
          read_block_group(buf, g + 3, lane, kb_b);
          products_of_group<NRB, true>(q, kb_a, acc_a);
        }
        add(acc_b, g + 1);
      }
      if constexpr (LONG) {
        bool far = false;
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) far |= !(st_row.l[rb] <= kStatsMost);
        again = __ballot(far) != 0ull;
        if (again) st_row = before;
      }
    }
    if (again) {
      for (int g = 0; g < kGqaBlockGroups; ++g) {
        const int t_first = t_block + 16 * g;
        if (t_first >= a.T) break;  // uniform over the workgroup
        f32x4 acc[4];
        score_block_group<NRB, true>(q, buf, g, lane, acc);
        stats_raise_and_add<NRB>(st_row, acc, scale2, t_first, a.T, a.W, mrow, qd, 16 * rb0);
      }
    }
    __syncthreads();
  }
  // this wavefront saw every key of the chunk for its rows: its statistics are the chunk's
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    const float lr = stats_row_sum(st_row.l[rb]);
    if (qd == 0) {
      float *dst = a.row_stats + (((size_t)bhq * a.n_chunk + chunk) * a.W + 16 * (rb0 + rb) + mrow) * 2;
      dst[0] = st_row.m[rb];
      dst[1] = lr;
    }
  }
}

// pass 2: per (b, hkv, chunk): mass[t] = sum over the group's heads and the tail rows of 2^(s - m_row) / l_row (added
// up in wavefront order, i.e. head by head, lower rows first)
template <int NRB, int MAXIT>
__global__ __launch_bounds__(64 * kGqaMaxHeads * (4 / NRB)) void psa_mass_gqa_kernel(SelectArgs a) {
  constexpr int kHeadWaves = 4 / NRB;                      // wavefronts per query head
  constexpr int kMaxWaves = kGqaMaxHeads * kHeadWaves;     // scoring wavefronts of a workgroup, at most
  __shared__ u32x4 kbuf[2][kGqaItems * 64];
  __shared__ float stat_m[kGqaMaxHeads][64], stat_il[kGqaMaxHeads][64];
  // column sums of a block: one slot per (scoring wavefront, row quarter, key), each written by one lane; two copies,
  // so that a block's slots are added up (fixed order) while the next block is being scored
  __shared__ float col_lds[2][kMaxWaves][4][kGqaBlockKeys];
  const int chunk = blockIdx.x, bh = blockIdx.y;
  const int R = a.Hq / a.Hkv, b = bh / a.Hkv, hkv = bh % a.Hkv;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, mrow = lane & 15, qd = lane >> 4;
  const int n_score = R * kHeadWaves;
  const int head = wave / kHeadWaves, rb0 = (wave % kHeadWaves) * NRB;
  const int bhq = b * a.Hq + hkv * R + head;
  const uint16_t *k_rows = a.k + (size_t)bh * a.T * kD;
  const float scale2 = a.sm_scale * kLog2e;
  const int t_chunk = chunk * a.chunk;
  const int n_blk = (min(a.chunk, a.T - t_chunk) + kGqaBlockKeys - 1) / kGqaBlockKeys;
  // feeders (kGqaItems / MAXIT wavefronts behind the scoring ones) take consecutive pieces; without feeders the
  // scoring wavefronts take pieces wave, wave + kMaxWaves, ...
  constexpr bool kFeeder = MAXIT >= kGqaFeederItems;
  const int first = kFeeder ? (wave - n_score) * MAXIT : wave, stride = kFeeder ? 1 : kMaxWaves;
  // adds up the slots of key `key` of block j (scoring wavefronts in order, quarters pairwise) and stores its mass
  auto flush_key = [&](int j, int key) {
    const int t = t_chunk + j * kGqaBlockKeys + key;
    float sum = 0.0f;
    for (int w = 0; w < n_score; ++w)
      sum += (col_lds[j & 1][w][0][key] + col_lds[j & 1][w][1][key]) +
             (col_lds[j & 1][w][2][key] + col_lds[j & 1][w][3][key]);
    if (t < a.T) a.mass[(size_t)bh * a.T + t] = sum;
  };
  KeyStage<MAXIT> st;
  if (kFeeder && wave >= n_score) {  // a feeder: same barriers as the scoring wavefronts below
    // the feeders share the keys of a block when its column sums are added up
    constexpr int kFeederKeys = kFeeder ? kGqaBlockKeys * MAXIT / kGqaItems : kGqaBlockKeys;
    const int first_key = (wave - n_score) * kFeederKeys;
    request_block(k_rows, t_chunk, a.T, first, stride, mrow, qd, st);
    deposit_block(st, kbuf[0], first, stride, lane);
    request_block(k_rows, t_chunk + kGqaBlockKeys, a.T, first, stride, mrow, qd, st);
    __syncthreads();
    for (int j = 0; j < n_blk; ++j) {
      if (j + 1 < n_blk) deposit_block(st, kbuf[(j + 1) & 1], first, stride, lane);
      if (j + 2 < n_blk) request_block(k_rows, t_chunk + (j + 2) * kGqaBlockKeys, a.T, first, stride, mrow, qd, st);
      if (j > 0 && lane < kFeederKeys) flush_key(j - 1, first_key + lane);
      __syncthreads();
    }
    if (lane < kFeederKeys) flush_key(n_blk - 1, first_key + lane);
    return;
  }
  if constexpr (!kFeeder) request_block(k_rows, t_chunk, a.T, first, stride, mrow, qd, st);
  if (lane < 16 * NRB) {
    const int row = 16 * rb0 + lane;
    merge_chunk_stats(a, bhq, row, stat_m[head][row], stat_il[head][row]);
  }
  bf16x8 q[NRB * 4];
  load_query_rows<NRB>(a.q_tail + (size_t)bhq * a.W * kD, rb0, mrow, qd, q);
  if constexpr (!kFeeder) {
    deposit_block(st, kbuf[0], first, stride, lane);
    request_block(k_rows, t_chunk + kGqaBlockKeys, a.T, first, stride, mrow, qd, st);
  }
  wave_lds_sync();  // the statistics read below were written by this wavefront
  f32x4 rm[NRB], ril[NRB];  // rows 16*(rb0 + rb) + 4*qd + i
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    rm[rb] = *reinterpret_cast<const f32x4 *>(&stat_m[head][16 * (rb0 + rb) + 4 * qd]);
    ril[rb] = *reinterpret_cast<const f32x4 *>(&stat_il[head][16 * (rb0 + rb) + 4 * qd]);
  }
  __syncthreads();
  for (int j = 0; j < n_blk; ++j) {
    if constexpr (!kFeeder) {
      if (j + 1 < n_blk) deposit_block(st, kbuf[(j + 1) & 1], first, stride, lane);
      if (j + 2 < n_blk) request_block(k_rows, t_chunk + (j + 2) * kGqaBlockKeys, a.T, first, stride, mrow, qd, st);
      if (j > 0 && threadIdx.x < kGqaBlockKeys) flush_key(j - 1, threadIdx.x);
    }
    const u32x4 *buf = kbuf[j & 1];
    const int t_block = t_chunk + j * kGqaBlockKeys;
    if (t_block + kGqaBlockKeys - 1 <= a.T - a.W) {
      // Every key of the block is seen by every tail row (all but the last blocks of a context): straight-line code,
      // keys read from LDS one group ahead of their products, the products issued one group ahead of the exponentials.
      f32x4 acc[2][4];
      bf16x8 kb[2][4];
      read_block_group(buf, 0, lane, kb[0]);
      read_block_group(buf, 1, lane, kb[1]);
      products_of_group<NRB, false>(q, kb[0], acc[0]);
#pragma unroll
      for (int g = 0; g < kGqaBlockGroups; ++g) {
        const f32x4(&cur)[4] = acc[g & 1];
        if (g + 2 < kGqaBlockGroups) read_block_group(buf, g + 2, lane, kb[g & 1]);
        if (g + 1 < kGqaBlockGroups) products_of_group<NRB, false>(q, kb[(g + 1) & 1], acc[(g + 1) & 1]);
        float c0 = 0.0f, c1 = 0.0f;  // two chains: even and odd row blocks
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
          float &cc = (rb & 1) ? c1 : c0;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            cc = __builtin_fmaf(fast_exp2(__builtin_fmaf(cur[rb][i], scale2, -rm[rb][i])), ril[rb][i], cc);
        }
        col_lds[j & 1][wave][qd][16 * g + mrow] = c0 + c1;
      }
    } else {
      for (int g = 0; g < kGqaBlockGroups; ++g) {
        const int t_first = t_block + 16 * g;
        float c = 0.0f;
        if (t_first < a.T) {  // uniform over the workgroup; groups past the end leave zeros in their slots
          f32x4 acc[4];
          score_block_group<NRB, false>(q, buf, g, lane, acc);
          float c0 = 0.0f, c1 = 0.0f;
          const int t = t_first + mrow;
#pragma unroll
          for (int rb = 0; rb < NRB; ++rb) {
            float &cc = (rb & 1) ? c1 : c0;
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (key_seen(t, 16 * (rb0 + rb) + 4 * qd + i, a.T, a.W))
                cc = __builtin_fmaf(fast_exp2(__builtin_fmaf(acc[rb][i], scale2, -rm[rb][i])), ril[rb][i], cc);
          }
          c = c0 + c1;
        }
        col_lds[j & 1][wave][qd][16 * g + mrow] = c;
      }
    }
    __syncthreads();
  }
  if constexpr (!kFeeder)
    if (threadIdx.x < kGqaBlockKeys) flush_key(n_blk - 1, threadIdx.x);
}

// inclusive prefix sum of one int per thread over a workgroup of NW wavefronts, plus the workgroup total
template <int NW>
__device__ __forceinline__ int block_inclusive_scan(int v, int *wave_tot, int &total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int up = __shfl_up(v, off, kWave);
    if (lane >= off) v += up;
  }
  __syncthreads();  // previous use of wave_tot finished
  if (lane == kWave - 1) wave_tot[wave] = v;
  __syncthreads();
  int before = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const int c = wave_tot[w];
    if (w < wave) before += c;
    tot += c;
  }
  total = tot;
  return before + v;
}

// exact top-k of non-negative fp32 keys by radix select; equal keys go to the lower position; output ascending.
// STAGED: the row of keys is copied to LDS once and every pass reads it from there.
constexpr int kTopkStageMax = 32768;  // keys (128 KB of LDS)
constexpr int kTopkListMax = 256;     // selected positions ordered through LDS when k is at most this
constexpr int kTopkCandMax = 512;     // candidates the short cut ranks among themselves
constexpr int kTopkWideFrom = 8192, kTopkWideRows = 512, kTopkWideThreads = 1024;  // see launch_topk
constexpr int kTopkBatch = 8;         // keys a thread requests together
constexpr int kTopkMaximaMax = 192;   // of the 256 maxima: beyond, the candidate bound is searched to its last bit
// NT threads per workgroup (256, or 1024 for long rows: the passes over the keys are what takes the time there)
// keys: the row of keys in LDS (STAGED; every thread's largest of the keys it wrote there is `mine`), or in memory
template <bool STAGED, int NT>
__device__ __forceinline__ void topk_row(const SelectArgs &a, int bh, const float *keys, uint32_t mine) {
  __shared__ int hist[256];
  __shared__ int wave_tot[NT / 64];
  __shared__ uint32_t sh_prefix;
  __shared__ int sh_need;
  __shared__ int list_n;
  __shared__ __attribute__((aligned(16))) int list[kTopkListMax + 8];
  __shared__ uint32_t thread_max[NT];
  __shared__ int cand_n;
  __shared__ __attribute__((aligned(16))) uint64_t cand[kTopkCandMax + 8];  // key, then the position inverted: larger comes first
  const int lane = threadIdx.x & 63;
  int32_t *out = a.sal_idx + (size_t)bh * a.S_cap;
  const int k = min(a.top_k, a.T);
  const uint32_t lowest = a.skip_zero ? 1u : 0u;  // keys below this bit pattern (i.e. +0) are never selected
  if (STAGED) {
    if (threadIdx.x == 0) { list_n = 0; cand_n = 0; }
    thread_max[threadIdx.x] = mine;
    __syncthreads();
    if (k <= 128) {
      // Short cut for the usual case (a few pivots out of thousands of keys): the k-th largest of the per-thread
      // maxima is a lower bound of the k-th largest key, and few keys reach it.  They are collected and ranked among
      // themselves (key descending, position ascending: the order of the radix path).  Too many candidates (many equal
      // keys): the radix passes below take over.  Every wavefront finds the bound for itself, bit by bit from the top:
      // the largest x with at least k of 256 maxima >= x (four per lane; with more than 256 threads each is the
      // largest of NT / 256 thread maxima, still 256 different keys).
      uint32_t mx[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t v = 0u;
#pragma unroll
        for (int jj = 0; jj < NT / 256; ++jj) v = max(v, thread_max[lane + 64 * i + 256 * jj]);
        mx[i] = v;
      }
      // Sixteen bits of it (the sign is 0: exponent and eight bits of the fraction) are mostly enough: a bound that is
      // lower by up to 2^-8 of itself lets a few more candidates through, and each bit is a step of a serial chain.  Where
      // the largest keys lie so close together that most of the 256 maxima reach that bound, the other bits are searched
      // too: at three quarters of them, keys in any order give about 256 ln 4 = 355 candidates; much beyond that they
      // overflow the list and end in the radix passes.
      uint32_t bound = 0u;
      int n_at = 256;  // maxima that reach it
      auto try_bit = [&](int bit) {
        const uint32_t x = bound | (1u << bit);
        const int n_ge = __popcll(__ballot(mx[0] >= x)) + __popcll(__ballot(mx[1] >= x)) + __popcll(__ballot(mx[2] >= x)) +
                         __popcll(__ballot(mx[3] >= x));
        if (n_ge >= k) { bound = x; n_at = n_ge; }
      };
#pragma unroll
      for (int bit = 30; bit >= 15; --bit) try_bit(bit);
      if (__builtin_expect(n_at > kTopkMaximaMax, 0))
        for (int bit = 14; bit >= 0; --bit) try_bit(bit);
      for (int t0 = threadIdx.x; t0 < a.T; t0 += kTopkBatch * NT) {
        uint32_t bits[kTopkBatch];
#pragma unroll
        for (int i = 0; i < kTopkBatch; ++i) bits[i] = __float_as_uint(keys[min(t0 + i * NT, a.T - 1)]);
#pragma unroll
        for (int i = 0; i < kTopkBatch; ++i)
          if (t0 + i * NT < a.T && bits[i] >= bound && bits[i] >= lowest) {
            const int at = atomicAdd(&cand_n, 1);
            if (at < kTopkCandMax) cand[at] = ((uint64_t)bits[i] << 32) | ~(uint32_t)(t0 + i * NT);
          }
      }
      __syncthreads();
      const int n_cand = cand_n;
      if (n_cand <= kTopkCandMax) {  // uniform
        if (threadIdx.x < 8) cand[n_cand + threadIdx.x] = 0u;  // the ranking below reads eight at a time; 0 ranks behind all
        __syncthreads();
        for (int c = threadIdx.x; c < n_cand; c += NT) {
          const uint64_t mine_key = cand[c];
          int beaten_by = 0;
          for (int j = 0; j < n_cand; j += 8)
#pragma unroll
            for (int i = 0; i < 8; ++i) beaten_by += cand[j + i] > mine_key;
          if (beaten_by < k) list[atomicAdd(&list_n, 1)] = (int)~(uint32_t)mine_key;
        }
        __syncthreads();
        const int n_kept = list_n;  // k, or fewer when zero keys are excluded
        if (threadIdx.x < 8) list[n_kept + threadIdx.x] = 0x7FFFFFFF;
        __syncthreads();
        if ((int)threadIdx.x < n_kept) {
          const int mine_pos = list[threadIdx.x];
          int rank = 0;
          for (int j = 0; j < n_kept; j += 8)
#pragma unroll
            for (int i = 0; i < 8; ++i) rank += list[j + i] < mine_pos;
          if (rank < a.S_cap) out[rank] = mine_pos;
        }
        if (threadIdx.x == 0) a.sal_cnt[bh] = n_kept;
        return;
      }
      __syncthreads();
      if (threadIdx.x == 0) list_n = 0;
      __syncthreads();
    }
  }
  uint32_t prefix = 0;
  int need = k;
  for (int pass = 3; pass >= 0; --pass) {
    if (threadIdx.x < 256) hist[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t hi_mask = pass == 3 ? 0u : (0xFFFFFFFFu << (8 * (pass + 1)));
    for (int t = threadIdx.x; t < a.T; t += NT) {
      const uint32_t bits = __float_as_uint(keys[t]);
      if ((bits & hi_mask) == (prefix & hi_mask)) {
        // the leading digits of the keys of a wavefront mostly coincide: one add for all of them then
        const int bin = (bits >> (8 * pass)) & 0xFF;
        const int first = __builtin_amdgcn_readfirstlane(bin);
        const unsigned long long active = __ballot(true), same = __ballot(bin == first);
        if (same == active) {
          if (lane == __ffsll((long long)active) - 1) atomicAdd(&hist[first], __popcll(active));
        } else {
          atomicAdd(&hist[bin], 1);
        }
      }
    }
    __syncthreads();
    // thread i looks at bin 255-i: the prefix sum over threads is the count of candidates in bins >= that bin; the
    // digit of the k-th largest key is the first bin (from the top) where that count reaches `need`
    const int bin = 255 - (int)threadIdx.x;  // (threads past the 256 bins add nothing to the sums)
    const int mine = bin >= 0 ? hist[bin] : 0;
    int total;
    const int upto = block_inclusive_scan<NT / 64>(mine, wave_tot, total);
    if (bin >= 0 && upto >= need && upto - mine < need) {
      sh_prefix = prefix | ((uint32_t)bin << (8 * pass));
      sh_need = need - (upto - mine);
      if (pass == 0) hist[0] = mine;  // number of keys equal to the k-th largest (bin 0's own count is not needed again)
    }
    __syncthreads();
    prefix = sh_prefix;
    need = sh_need;
  }
  // prefix = bit pattern of the k-th largest key; `need` of the keys equal to it are taken, lowest positions first.
  const int n_equal = hist[0];
  if (STAGED && k <= kTopkListMax && n_equal == need) {
    // every key >= prefix is taken: gather their positions in any order, then order the short list by rank
    for (int t = threadIdx.x; t < a.T; t += NT) {
      const uint32_t bits = __float_as_uint(keys[t]);
      if (bits >= prefix && bits >= lowest) list[atomicAdd(&list_n, 1)] = t;
    }
    __syncthreads();
    const int n_kept = list_n;  // k, or fewer when zero keys are excluded
    if ((int)threadIdx.x < n_kept) {
      const int mine = list[threadIdx.x];
      int rank = 0;
      for (int j = 0; j < n_kept; ++j) rank += list[j] < mine;
      if (rank < a.S_cap) out[rank] = mine;
    }
    if (threadIdx.x == 0) a.sal_cnt[bh] = n_kept;
    return;
  }
  // general case: each thread owns a contiguous run of positions, so two workgroup scans (equal keys, taken keys)
  // order the output
  const int per = (a.T + NT - 1) / NT;
  const int t0 = min((int)threadIdx.x * per, a.T), t1 = min(t0 + per, a.T);
  int n_eq = 0;
  for (int t = t0; t < t1; ++t) n_eq += __float_as_uint(keys[t]) == prefix;
  int tot_eq;
  int eq_rank = block_inclusive_scan<NT / 64>(n_eq, wave_tot, tot_eq) - n_eq;
  int n_take = 0;
  {
    int r = eq_rank;
    for (int t = t0; t < t1; ++t) {
      const uint32_t bits = __float_as_uint(keys[t]);
      n_take += (bits > prefix || (bits == prefix && r++ < need)) && bits >= lowest;
    }
  }
  int tot_take;
  int pos = block_inclusive_scan<NT / 64>(n_take, wave_tot, tot_take) - n_take;
  if (n_take > 0) {
    for (int t = t0; t < t1; ++t) {
      const uint32_t bits = __float_as_uint(keys[t]);
      if ((bits > prefix || (bits == prefix && eq_rank++ < need)) && bits >= lowest) {
        if (pos < a.S_cap) out[pos] = t;
        ++pos;
      }
    }
  }
  if (threadIdx.x == 0) a.sal_cnt[bh] = tot_take;
}
// SUM: the keys are the query heads' masses of a KV head, added up in head order (and stored)
template <bool STAGED, int NT, bool SUM = false>
__global__ __launch_bounds__(NT) void topk_kernel(SelectArgs a) {
  extern __shared__ float keys_lds[];
  const int bh = blockIdx.x;
  const float *mass = a.mass + (size_t)(a.mass_per_batch ? bh / a.Hkv : bh) * a.T;
  uint32_t mine = 0u;  // largest key this thread staged (bit patterns of non-negative floats order like the floats)
  if constexpr (SUM) {
    // four positions a thread, all heads requested together
    const int R = a.Hq / a.Hkv;
    const float *heads = a.score + (size_t)bh * R * a.score_stride;
    float *mass_out = a.mass + (size_t)bh * a.T;
    for (int t0 = 4 * threadIdx.x; t0 < a.T; t0 += 4 * NT) {
      f32x4 x[kGqaMaxHeads];
#pragma unroll
      for (int h = 0; h < kGqaMaxHeads; ++h)
        if (h < R) x[h] = *reinterpret_cast<const f32x4 *>(heads + (size_t)h * a.score_stride + t0);
      f32x4 sum = x[0];
#pragma unroll
      for (int h = 1; h < kGqaMaxHeads; ++h)
        if (h < R) sum += x[h];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (t0 + i < a.T) {
          keys_lds[t0 + i] = sum[i];
          mass_out[t0 + i] = sum[i];
          mine = max(mine, __float_as_uint(sum[i]));
        }
    }
  } else if (STAGED)
    for (int t0 = threadIdx.x; t0 < a.T; t0 += kTopkBatch * NT) {
      float x[kTopkBatch];  // requested together; positions past the end read the last key and are dropped
#pragma unroll
      for (int i = 0; i < kTopkBatch; ++i) x[i] = mass[min(t0 + i * NT, a.T - 1)];
#pragma unroll
      for (int i = 0; i < kTopkBatch; ++i)
        if (t0 + i * NT < a.T) {
          keys_lds[t0 + i * NT] = x[i];
          mine = max(mine, __float_as_uint(x[i]));
        }
    }
  topk_row<STAGED, NT>(a, bh, STAGED ? keys_lds : mass, mine);
}

// ---- selection of a short prompt in one launch ------------------------------------------------------------------
// lane exchanges in registers: within a row of 16 lanes, and between the rows
template <int CTRL>
__device__ __forceinline__ float row_dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}
// four values per lane, reduced over the lanes l, l ^ 16, l ^ 32, l ^ 48: lane 16 * i + r gets the result of v[i] for r
template <typename F>
__device__ __forceinline__ float over_rows_each(const float (&v)[4], F f) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[0]), __float_as_uint(v[2]), false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[1]), __float_as_uint(v[3]), false, false);
  const float t0 = f(__uint_as_float(a[0]), __uint_as_float(a[1])), t1 = f(__uint_as_float(b[0]), __uint_as_float(b[1]));
  const auto c = __builtin_amdgcn_permlane16_swap(__float_as_uint(t0), __float_as_uint(t1), false, false);
  return f(__uint_as_float(c[0]), __uint_as_float(c[1]));
}
// ... and back: lane r of every row gets the values of lanes r, 16 + r, 32 + r, 48 + r
__device__ __forceinline__ void to_each_row(float x, float (&v)[4]) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);  // rows 0 0 2 2, 1 1 3 3
  const auto b = __builtin_amdgcn_permlane32_swap(a[0], a[0], false, false);
  const auto c = __builtin_amdgcn_permlane32_swap(a[1], a[1], false, false);
  v[0] = __uint_as_float(b[0]); v[2] = __uint_as_float(b[1]);
  v[1] = __uint_as_float(c[0]); v[3] = __uint_as_float(c[1]);
}
// The largest of three by the builtins that become one v_maximum3_f32 (the compiler's fmaxf first quiets operands it cannot
// prove quiet).  Not by assembly: the operands are fresh matrix products and the result goes into lane swaps, and the wait
// states that both need (eight behind a product of 16 x 16 x 32, two in front of a swap) are put in for instructions the
// compiler knows, and for no others.
__device__ __forceinline__ float max3(float a, float b, float c) {
  return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c);
}
// eight values per lane, added up over the 16 lanes of a row: lanes 2 * i and 2 * i + 1 get the sum of v[i]
__device__ __forceinline__ float row_sums_each(const float (&v)[8], int mrow) {
  float x[4], y[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {  // lanes r and 15 - r
    const float keep = (mrow & 8) ? v[i + 4] : v[i], give = (mrow & 8) ? v[i] : v[i + 4];
    x[i] = keep + row_dpp<0x140>(give);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {  // r and 7 - r of each half
    const float keep = (mrow & 4) ? x[i + 2] : x[i], give = (mrow & 4) ? x[i] : x[i + 2];
    y[i] = keep + row_dpp<0x141>(give);
  }
  const float keep = (mrow & 2) ? y[1] : y[0], give = (mrow & 2) ? y[0] : y[1];
  const float z = keep + row_dpp<0x1B>(give);  // r and 3 - r of each quad
  return z + row_dpp<0xB1>(z);                 // r and r ^ 1
}

// NG groups of 16 keys against the 64 tail rows: s = products, row 16*rb + mrow, keys t_lane + GROUP_STEP * g + i;
// STEP: groups multiplied at a time (their operands take 16 registers each, but the rows are read from LDS once for each step).
template <int NG, int STEP>
__device__ __forceinline__ void score_wave_keys(const KeyGroup (&raw)[NG], u32x4 *tile, const u32x4 *q_lds, int lane, f32x4 (&s)[4][NG]) {
#pragma unroll
  for (int g0 = 0; g0 < NG; g0 += STEP) {
    bf16x8 key[STEP][4];
#pragma unroll
    for (int g = 0; g < STEP; ++g) lines_to_operands(raw[g0 + g], tile, lane, key[g]);
    uint32_t lane_off = (uint32_t)lane;
    if (STEP < NG) asm volatile("" : "+v"(lane_off));  // (not kept in registers from step to step)
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
#pragma unroll
      for (int g = 0; g < STEP; ++g) s[rb][g0 + g] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kc = 0; kc < 4; ++kc) {
        const bf16x8 rows = __builtin_bit_cast(bf16x8, q_lds[(rb * 4 + kc) * 64 + lane_off]);
#pragma unroll
        for (int g = 0; g < STEP; ++g) s[rb][g0 + g] = mfma_bf16(key[g][kc], rows, s[rb][g0 + g]);
      }
    }
    if (STEP < NG) __builtin_amdgcn_sched_barrier(0);
  }
}
// ... turned into exponentials; t_last: the last of the keys; m_row, l_row: reference and sum of row `lane`
template <int NG, int GROUP_STEP>
__device__ __forceinline__ void exponentials_of_keys(f32x4 (&s)[4][NG], int t_lane, int t_last, int T, float scale2, int lane, float &m_row,
                                                     float &l_row) {
  const int mrow = lane & 15;
  if (t_last > T - 64) {  // some key is hidden from some row, or past the end: behind position T - 64 + row
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
      int last = T - 64 + 16 * rb + mrow - t_lane;
      asm volatile("" : "+v"(last));
#pragma unroll
      for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int i = 0; i < 4; ++i) s[rb][g][i] = GROUP_STEP * g + i <= last ? s[rb][g][i] : -INFINITY;
    }
  }
  float x[4];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb) {
    x[rb] = s[rb][0][0];
#pragma unroll
    for (int g = 0; g < NG; ++g) x[rb] = max3(max3(x[rb], s[rb][g][0], s[rb][g][1]), s[rb][g][2], s[rb][g][3]);
  }
  // row `lane` of this wavefront's keys (finite where no key is seen)
  m_row = fmaxf(over_rows_each(x, [](float u, float v) { return max3(u, u, v); }) * scale2, -1e30f);
  float ref[4];
  to_each_row(m_row, ref);
#pragma unroll
  for (int rb = 0; rb < 4; ++rb) {
    x[rb] = 0.0f;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
#pragma unroll
      for (int i = 0; i < 4; ++i) s[rb][g][i] = fast_exp2(__builtin_fmaf(s[rb][g][i], scale2, -ref[rb]));
      x[rb] += (s[rb][g][0] + s[rb][g][1]) + (s[rb][g][2] + s[rb][g][3]);
    }
  }
  l_row = over_rows_each(x, [](float u, float v) { return u + v; });
}
// column sums of such exponentials, each row times its weight (row `lane`): store(t, sum), each key by one lane.  A weight that is
// infinite or no number makes the sum of every key its row sees no number, and of no other: row r sees the keys up to T - 64 + r.
template <int NG, int GROUP_STEP, typename F>
__device__ __forceinline__ void column_sums(const f32x4 (&s)[4][NG], float weight, int t_lane, int T, int lane, F store) {
  const int mrow = lane & 15;
  const bool finite = weight <= 3.4028235e38f;
  const uint64_t spoilt = __ballot(!finite);
  const int spoilt_to = T - 1 - __builtin_clzll(spoilt | 1u) - (spoilt ? 0 : T);  // (none: in front of the first key)
  float wgt[4];
  to_each_row(finite ? weight : 0.0f, wgt);
#pragma unroll
  for (int half = 0; half < NG / 2; ++half) {
    float col[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int g = 2 * half + (i >> 2);
      col[i] = s[0][g][i & 3] * wgt[0];
#pragma unroll
      for (int rb = 1; rb < 4; ++rb) col[i] = __builtin_fmaf(s[rb][g][i & 3], wgt[rb], col[i]);
    }
    const float sum = row_sums_each(col, mrow);  // lanes of mrow 2 * (4*(g - 2*half) + i): key 16*g + 4*qd + i
    const int t = t_lane + GROUP_STEP * (2 * half + (mrow >> 3)) + ((mrow >> 1) & 3);
    if ((mrow & 1) == 0) store(t, t <= spoilt_to ? __builtin_nanf("") : sum);
  }
}

// One workgroup per (batch, query head), W = 64: a wavefront holds 64 keys as operands and, in 64 registers, what they make of
// the 64 tail rows, so that every key is read, multiplied and exponentiated once; the wavefronts' row statistics meet in
// LDS.  With one query head per KV head (TOPK) the top-k takes the masses from there; several heads leave theirs to
// topk_kernel, which adds them up.  Up to kSmallKeys keys: what twelve wavefronts of 168 registers, three on a SIMD, hold.
// Three launches of 5 to 6.6 us each did this before, each waiting for the one in front of it; us per selection, 32 heads,
// then and now: 1 x 640 keys 16.3 -> 13.3, 1 x 256 15.1 -> 7.8, 16 x 512 37.7 -> 21.3, 64 x 256 72 -> 38, 64 x 768 162 -> 128;
// in two launches, several heads per KV head: 1 x 368, 32/8 heads, 20.8 -> 13.1, 16 x 275, 28/4 heads, 29.6 -> 19.5.
// Keys come line by line and are turned through LDS: loads in operand order (half lines) took 1.4 us longer at 1 x 640.
// The time is a chain: rows and keys from memory (one CU brings a head's 164 KB), products, exponentials, three barriers,
// and about 2.5 us of top-k.
// NT: threads, and the most keys (a wavefront takes 64).
template <int NT, bool TOPK>
__global__ __launch_bounds__(NT) void psa_small_kernel(SelectArgs a) {
  __shared__ u32x4 key_tile[NT / 64][256];                              // 16 keys on their way to operands
  __shared__ u32x4 q_lds[1024];                                         // the tail rows as operands: slot (rb, kc, lane)
  __shared__ float part_m[NT / 64][64], part_l[NT / 64][64];  // per wavefront and row
  __shared__ float mass_lds[NT];
  const int bh = blockIdx.x;  // (batch, query head)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, qd = lane >> 4;
  const int n_waves = (a.T + 63) / 64, t_wave = 64 * wave;
  const bool scores = wave < n_waves;
  const uint16_t *k_rows = a.k + (size_t)(TOPK ? bh : bh / (a.Hq / a.Hkv)) * a.T * kD, *q_rows = a.q_tail + (size_t)bh * 64 * kD;
  const float scale2 = a.sm_scale * kLog2e;
  // rows first: they are looked at first, and loads return in order
  // eight wavefronts: two workgroups a CU, which 128 registers allow (18 x 500 keys, 28/4 heads: 27.5 us a selection with 144, 24.5)
  constexpr int kStep = NT == 512 && !TOPK ? 2 : 4;
  constexpr int kRowPieces = (1024 + NT - 1) / NT;  // 16-byte pieces of the rows per thread; consecutive threads, consecutive pieces
  u32x4 row_piece[kRowPieces];
#pragma unroll
  for (int x = 0; x < kRowPieces; ++x)
    row_piece[x] = *reinterpret_cast<const u32x4 *>(q_rows + 8 * min((int)threadIdx.x + x * NT, 1023));
  KeyGroup raw[4];
  if (scores) {
#pragma unroll
    for (int g = 0; g < 4; ++g) load_key_lines(k_rows, t_wave + 16 * g, a.T, lane, raw[g]);  // (past the end: masked)
  }
#pragma unroll
  for (int x = 0; x < kRowPieces; ++x) {
    const int i = (int)threadIdx.x + x * NT, piece = i & 15, row = i >> 4;
    if (i < 1024)
      q_lds[((row >> 4) * 4 + (piece >> 2)) * 64 + (piece & 3) * 16 + (row & 15)] = __builtin_bit_cast(u32x4, rows8_as_bf16(row_piece[x]));
  }
  __syncthreads();
  f32x4 s[4][4];  // exponentials: row 16*rb + mrow, keys 16*g + 4*qd + i
  float m_row = -1e30f, l_row = 0.0f;
  if (scores) {
    score_wave_keys<4, kStep>(raw, key_tile[wave], q_lds, lane, s);
    exponentials_of_keys<4, 16>(s, t_wave + 4 * qd, t_wave + 63, a.T, scale2, lane, m_row, l_row);
  }
  part_m[wave][lane] = m_row;
  part_l[wave][lane] = l_row;
  __syncthreads();
  if (scores) {
    float m_all = -1e30f, l_all = 0.0f;
    float m_w[NT / 64], l_w[NT / 64];
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) { m_w[w] = part_m[w][lane]; l_w[w] = part_l[w][lane]; }
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) m_all = fmaxf(m_all, m_w[w]);
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) l_all = __builtin_fmaf(l_w[w], fast_exp2(m_w[w] - m_all), l_all);
    column_sums<4, 16>(s, fast_exp2(m_row - m_all) * (1.0f / l_all), t_wave + 4 * qd, a.T, lane, [&](int t, float sum) {
      if (t < a.T) {
        if constexpr (TOPK) mass_lds[t] = sum;
        a.score[(size_t)bh * a.score_stride + t] = sum;
      }
    });
  }
  if constexpr (TOPK) {
    __syncthreads();
    topk_row<true, NT>(a, bh, mass_lds, (int)threadIdx.x < a.T ? __float_as_uint(mass_lds[threadIdx.x]) : 0u);
  }
}

// ---- pivot scoring with every key read once, W = 64 -------------------------------------------------------------------
// As psa_small_kernel, over as many workgroups per head as its keys need: a workgroup's exponentials (512 keys, 64 registers
// a lane) wait in registers while the row statistics go around between the workgroups of a head, so that every key is read,
// converted, multiplied and exponentiated once instead of twice.
// The statistics of a chunk are 64 words (reference and sum of a row) that say themselves whether they are there: a
// published word is never zero (where the reference is 0, the key it comes from adds 1 to the sum; where no key is seen, it is
// -1e30), and a launch in front clears them; so nothing has to be ordered but the word itself.  A head's workgroups are consecutive, and
// workgroups are dispatched in order: those of the oldest unfinished head are resident together.  Where they are not after all
// (fewer places than chunks, or another kernel in them), a workgroup that has looked often enough (OnceWait) scores a missing
// chunk itself: same code, same words, so the result does not depend on it, and every wait ends.
// What bounds it: neither issue (vector unit about 45 % busy, matrix pipe 20 %) nor the exchange (without waiting for the
// words it takes as long) but the loads between: two workgroups of eight wavefronts per CU, 128 registers each, leave room to
// request half of the next head's keys ahead and no more.  They are requested as soon as the products have taken the
// registers of the present ones, in front of the exponentials: behind the first look at the words, 5 us later, 8 x 32 x 16384
// took 240 us, now 234.  (Timing builds of that one: without the arithmetic 0.94 of the time, without the loads 0.8.)  Keys are
// dealt to the wavefronts four at a time, so that all wavefronts' loads are 8 KB in a row (64 keys each, 16 KB in a row: 251
// -> 239).
// Us per selection, two passes and this: 32 heads, 8 x 16384 keys 357 -> 234, 16 x 4096 184 -> 127, 33 x 2170 314 -> 147,
// 2 x 32768 187 -> 137.  Not kept: 256 registers and 128 keys a wavefront (252 when this took 250; a
// lone wavefront per SIMD and workgroup waits for its own chains), four wavefronts a workgroup, three workgroups a CU and
// all keys requested ahead (143 at 16 x 4096), six wavefronts (they do not spread evenly over four SIMDs: one workgroup a CU),
// the other half of the keys requested between the halves of the column sums (237).
constexpr int kOnceGroups = 4;  // groups of 16 keys of a wavefront
constexpr int kOnceWaves = kOnceKeys / (16 * kOnceGroups);
constexpr int kOnceStep = 16 * kOnceWaves;  // keys from one group of a wavefront to its next
static_assert(kOnceMaxChunks <= 64, "missing chunks are the bits of a ballot");
static_assert(kOnceWaves == 8, "rows are staged by 512 threads, statistics merged for 8 wavefronts");
constexpr int kOnceBatch = 4;                // chunks whose words a wavefront requests together
constexpr int kOnceWords = (kOnceMaxChunks + kOnceWaves - 1) / kOnceWaves;  // chunks whose words it collects, at most

__global__ __launch_bounds__(256) void clear_stats_kernel(u32x4 *words, size_t n) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) words[i] = (u32x4){0u, 0u, 0u, 0u};
}

// Memory through a buffer descriptor: what lies past the end reads as zero and is not written, and a tile of accesses needs one
// address register.  Only the lane's offset is certain to be compared with the end: an access that may pass it has no scalar
// offset (those of load_x2 and store_x2 stay inside).
struct Buffer {
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ __forceinline__ Buffer(const void *p, uint32_t bytes)
      : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00027000)) {}
  static constexpr int kStream = 2;                    // non-temporal
  static constexpr int kShared = 16 | (int)0x80000000;  // with other workgroups: volatile (never merged or moved), which makes it system scope (sc0 sc1)
  template <int POLICY>
  __device__ __forceinline__ u32x4 load_x4(uint32_t lane_bytes) const {
    return __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)lane_bytes, 0, POLICY);
  }
  template <int POLICY>
  __device__ __forceinline__ u32x2 load_x2(uint32_t lane_bytes, uint32_t bytes) const {
    return __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)lane_bytes, (int)bytes, POLICY);
  }
  template <int POLICY>
  __device__ __forceinline__ void store_x2(u32x2 v, uint32_t lane_bytes, uint32_t bytes) const {
    __builtin_amdgcn_raw_buffer_store_b64(v, rsrc, (int)lane_bytes, (int)bytes, POLICY);
  }
  __device__ __forceinline__ void store(float v, uint32_t lane_bytes) const {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rsrc, (int)lane_bytes, 0, 0);
  }
};

// A workgroup barrier that orders LDS only: loads and stores in flight stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
// WORDS: chunks whose words one wavefront collects, at most; AHEAD: groups of the next head's keys that are requested ahead.
// gridDim.y workgroup rows take the heads in turn.
template <int WORDS, int AHEAD>
__global__ __launch_bounds__(64 * kOnceWaves, 4) void psa_once_kernel(SelectArgs a) {  // 4 wavefronts per SIMD: at most 128 registers
  __shared__ u32x4 key_tile[kOnceWaves][256];
  __shared__ u32x4 q_lds[2][1024];
  __shared__ float part_m[kOnceWaves][64], part_l[kOnceWaves][64], got_m[kOnceWaves][64], got_l[kOnceWaves][64];
  __shared__ uint32_t missing[kOnceWaves];
  const int own = (blockIdx.x + blockIdx.y) % gridDim.x, n_heads = a.B * a.Hq, group = a.Hq / a.Hkv;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int tid = threadIdx.x;
  const float scale2 = a.sm_scale * kLog2e;
  KeyGroup raw[kOnceGroups];
  u32x4 row_piece[2];
  auto request_keys = [&](int bhq, int c, int g0, int g1) {
    const Buffer keys(a.k + (size_t)(bhq / group) * a.T * kD, bhq < n_heads ? a.T * (kD * 2) : 0);
    int at = 16 * (tid & 63) + (c * kOnceKeys + kOnceStep * g0 + 4 * wave) * (kD * 2);
#pragma unroll
    for (int g = g0; g < g1; ++g)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        asm volatile("" : "+v"(at));  // one register, moved on from load to load
        raw[g].raw[i] = keys.load_x4<Buffer::kStream>(at);
        at += 4 * kOnceWaves * (kD * 2);
      }
  };
  auto request_first = [&](int bhq, int c) {  // the rows (consecutive threads, consecutive pieces) and half of the keys
    const Buffer rows(a.q_tail + (size_t)bhq * 64 * kD, bhq < n_heads ? 64 * kD * 2 : 0);
#pragma unroll
    for (int x = 0; x < 2; ++x) row_piece[x] = rows.load_x4<0>(16 * tid + 8192 * x);
    request_keys(bhq, c, 0, AHEAD);
  };
  auto keep_rows = [&](u32x4 *q) {  // as operands: slot (rb, kc, lane)
#pragma unroll
    for (int x = 0; x < 2; ++x)
      q[((tid >> 8) * 4 + ((tid & 15) >> 2)) * 64 + (tid & 3) * 16 + ((tid >> 4) & 15) + 512 * x] =
          __builtin_bit_cast(u32x4, rows8_as_bf16(row_piece[x]));
  };
  auto merge = [&](const float (&pm)[kOnceWaves][64], const float (&pl)[kOnceWaves][64], float &m_all, float &l_all) {
    const int lane = tid & 63;
    m_all = -1e30f;  // the wavefronts' statistics of row `lane`
    l_all = 0.0f;
#pragma unroll
    for (int w = 0; w < kOnceWaves; ++w) m_all = fmaxf(m_all, pm[w][lane]);
#pragma unroll
    for (int w = 0; w < kOnceWaves; ++w) l_all = __builtin_fmaf(pl[w][lane], fast_exp2(pm[w][lane] - m_all), l_all);
  };
  int bhq = blockIdx.y, c = own, buf = 0;
  OnceWait wait;
  request_first(bhq, c);
  keep_rows(q_lds[0]);
  lds_barrier();
  for (;;) {
    asm volatile("" : "+v"(tid));  // no address of the lane's is kept from round to round
    const int lane = tid & 63, t_lane = c * kOnceKeys + 4 * kOnceWaves * (lane >> 4) + 4 * wave;
    const Buffer words(reinterpret_cast<uint64_t *>(a.row_stats) + (size_t)bhq * a.n_chunk * 64, a.n_chunk * 512);
    request_keys(bhq, c, AHEAD, kOnceGroups);
    f32x4 s[4][kOnceGroups];
    float m_row = -1e30f, l_row = 0.0f, m_all, l_all;
    score_wave_keys<kOnceGroups, 2>(raw, key_tile[wave], q_lds[buf], lane, s);
    const int next_bhq = bhq + gridDim.y;
    request_first(next_bhq, own);
    __builtin_amdgcn_sched_barrier(0);  // (not behind the exponentials)
    exponentials_of_keys<kOnceGroups, kOnceStep>(s, t_lane, (c + 1) * kOnceKeys - 1, a.T, scale2, lane, m_row, l_row);
    part_m[wave][lane] = m_row;
    part_l[wave][lane] = l_row;
    lds_barrier();
    if (wave == 0) {
      merge(part_m, part_l, m_all, l_all);
      words.store_x2<Buffer::kShared>((u32x2){__float_as_uint(l_all), __float_as_uint(m_all)}, 8 * lane, 512 * c);
    }
    // This wavefront collects chunks wave, wave + 8, ..., kOnceBatch at a time (loads return in order: behind the keys).
    float mm = -1e30f, ll = 0.0f;
    uint32_t need_all = 0u;
#pragma unroll
    for (int b = 0; b < WORDS; b += kOnceBatch) {
      u32x2 got[kOnceBatch];
      uint32_t need = 0u;
      auto look = [&](int i) {
        got[i] = words.load_x2<Buffer::kShared>(8 * lane, 512 * min(wave + kOnceWaves * (b + i), a.n_chunk - 1));
      };
      auto is_there = [&](int i) { return __ballot((got[i][0] | got[i][1]) == 0u) == 0ull; };
#pragma unroll
      for (int i = 0; i < kOnceBatch; ++i) look(i);
#pragma unroll
      for (int i = 0; i < kOnceBatch; ++i) need |= is_there(i) ? 0u : 1u << i;
      while (need != 0u && wait.look_again()) {
        __builtin_amdgcn_s_sleep(1);
#pragma unroll
        for (int i = 0; i < kOnceBatch; ++i)
          if ((need >> i) & 1u) look(i);
#pragma unroll
        for (int i = 0; i < kOnceBatch; ++i)
          if (((need >> i) & 1u) && is_there(i)) need &= ~(1u << i);
      }
      float m_new = mm, m_got[kOnceBatch];
#pragma unroll
      for (int i = 0; i < kOnceBatch; ++i) {
        m_got[i] = wave + kOnceWaves * (b + i) < a.n_chunk ? __uint_as_float(got[i][1]) : -INFINITY;
        m_new = fmaxf(m_new, m_got[i]);
      }
      ll *= fast_exp2(mm - m_new);
#pragma unroll
      for (int i = 0; i < kOnceBatch; ++i) ll = __builtin_fmaf(__uint_as_float(got[i][0]), fast_exp2(m_got[i] - m_new), ll);
      mm = m_new;
      need_all |= need << b;
    }
    got_m[wave][lane] = mm;
    got_l[wave][lane] = ll;
    if (lane == 0) missing[wave] = need_all;
    keep_rows(q_lds[buf ^ 1]);
    lds_barrier();
    merge(got_m, got_l, m_all, l_all);
    // chunk `lane`, which wavefront lane % 8 has looked for
    const uint64_t who = __ballot(lane < a.n_chunk && ((missing[lane % kOnceWaves] >> (lane / kOnceWaves)) & 1u));
    if (__builtin_expect(who != 0ull || c != own, 0)) {
      c = own;
      if (who != 0ull) {
        wait.give_up();
        c = once_chunk_to_score(who, own);
      }
      lds_barrier();  // `missing` has been read
      request_first(bhq, c);
      continue;
    }
    const Buffer mass(a.score + (size_t)bhq * a.score_stride, a.T * 4);
    asm volatile("" : "+v"(tid));
    const int t_mass = own * kOnceKeys + 4 * kOnceWaves * ((tid >> 4) & 3) + 4 * wave;
    column_sums<kOnceGroups, kOnceStep>(s, fast_exp2(m_row - m_all) * (1.0f / l_all), t_mass, a.T, tid & 63,
                                        [&](int t, float sum) { mass.store(sum, 4 * t); });
    wait.next_head();
    bhq = next_bhq;
    buf ^= 1;
    if (bhq >= n_heads) break;
  }
}

// ---- massive-activation score (Section III-B.2): largest channel magnitude of every token's hidden state ----
// One wavefront per token; magnitudes of binary16 values order like their low 15 bits, so the row maximum is taken on
// integers; scores below the floor are written as 0 (the top-k never selects a zero key).
__global__ __launch_bounds__(256) void massive_score_kernel(SelectArgs a) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const long row = (long)blockIdx.x * 4 + wave;
  if (row >= (long)a.B * a.T) return;
  const uint16_t *src = a.hidden + (size_t)row * a.d_model;
  uint32_t m0 = 0u, m1 = 0u;  // running maxima of the low and the high binary16 of every word, as 15-bit integers
  for (int c0 = 0; c0 < a.d_model; c0 += 512) {  // 64 lanes x 8 channels
    const u32x4 v = stream_load(reinterpret_cast<const u32x4 *>(src + c0 + 8 * lane));
    const uint32_t w0 = v[0], w1 = v[1], w2 = v[2], w3 = v[3];
    m0 = max(m0, max(max(w0 & 0x7FFFu, w1 & 0x7FFFu), max(w2 & 0x7FFFu, w3 & 0x7FFFu)));
    m1 = max(m1, max(max((w0 >> 16) & 0x7FFFu, (w1 >> 16) & 0x7FFFu), max((w2 >> 16) & 0x7FFFu, (w3 >> 16) & 0x7FFFu)));
  }
  uint32_t m2 = max(m0, m1);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m2 = max(m2, (uint32_t)__shfl_xor((int)m2, off, kWave));
  if (lane == 0) {
    const float score = half_bits_to_float(m2);
    a.mass[row] = score >= a.floor ? score : 0.0f;
  }
}

}  // namespace

// Dynamic LDS above 48 KB has to be opted into, per device and process: done on the first launch that needs it on a
// device (for the largest size the kernel is ever given), not on every call.
static hipError_t topk_allow_large_lds() {
  static std::atomic<unsigned long long> done{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev >= 0 && dev < 64 && ((done.load(std::memory_order_acquire) >> dev) & 1ull)) return hipSuccess;
  const void *kernels[] = {reinterpret_cast<const void *>(&topk_kernel<true, kTopkWideThreads>),
                           reinterpret_cast<const void *>(&topk_kernel<true, 256>),
                           reinterpret_cast<const void *>(&topk_kernel<true, kTopkWideThreads, true>),
                           reinterpret_cast<const void *>(&topk_kernel<true, 256, true>)};
  for (const void *kernel : kernels)
    if (e == hipSuccess)
      e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kTopkStageMax * sizeof(float)));
  if (e == hipSuccess && dev >= 0 && dev < 64) done.fetch_or(1ull << dev, std::memory_order_release);
  return e;
}

// One workgroup per row of keys.  Few long rows (at most kTopkWideRows rows of kTopkWideFrom keys or more) get
// workgroups of 1024 threads: the time goes into the passes over the keys then, and 256-thread workgroups would leave
// most of the chip idle.  With many rows the small workgroups already fill it (and are 6 % faster at 2048 x 8192).
static hipError_t launch_topk(const SelectArgs &k, hipStream_t stream) {
  const dim3 grid(k.B * k.Hkv);
  const bool wide = k.T >= kTopkWideFrom && (long)k.B * k.Hkv <= kTopkWideRows;
  const size_t lds = k.T <= kTopkStageMax ? (size_t)k.T * sizeof(float) : 0;
  if (lds > 48 * 1024) {
    hipError_t e = topk_allow_large_lds();
    if (e != hipSuccess) return e;
  }
  if (k.score_path != kScoreTwoPasses && k.Hq > k.Hkv) {  // (of at most kTopkStageMax keys)
    if (wide) hipLaunchKernelGGL((topk_kernel<true, kTopkWideThreads, true>), grid, dim3(kTopkWideThreads), lds, stream, k);
    else hipLaunchKernelGGL((topk_kernel<true, 256, true>), grid, dim3(256), lds, stream, k);
  } else if (k.T > kTopkStageMax) {
    if (wide) hipLaunchKernelGGL((topk_kernel<false, kTopkWideThreads>), grid, dim3(kTopkWideThreads), 0, stream, k);
    else hipLaunchKernelGGL((topk_kernel<false, 256>), grid, dim3(256), 0, stream, k);
  } else {
    if (wide) hipLaunchKernelGGL((topk_kernel<true, kTopkWideThreads>), grid, dim3(kTopkWideThreads), lds, stream, k);
    else hipLaunchKernelGGL((topk_kernel<true, 256>), grid, dim3(256), lds, stream, k);
  }
  return hipGetLastError();
}

hipError_t launch_select_massive(const SelectArgs &a, hipStream_t stream) {
  const long rows = (long)a.B * a.T;
  hipLaunchKernelGGL(massive_score_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_topk(a, stream);
}

hipError_t launch_select_tsa(const SelectArgs &a, hipStream_t stream) {
  const dim3 grid(a.B * a.Hkv);
  if (text_threads((long)a.B * a.Hkv, a.T) == 256) hipLaunchKernelGGL(select_tsa_kernel<256>, grid, dim3(256), 0, stream, a);
  else hipLaunchKernelGGL(select_tsa_kernel<1024>, grid, dim3(1024), 0, stream, a);
  return hipGetLastError();
}

namespace {

// token-level pivots: the masses of a batch element's kv-heads added in head order (one thread per position)
__global__ __launch_bounds__(256) void sum_heads_kernel(SelectArgs a) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long)a.B * a.T) return;
  const int b = (int)(i / a.T), t = (int)(i % a.T);
  float sum = 0.0f;
  for (int h = 0; h < a.Hkv; ++h) sum += a.mass[((size_t)b * a.Hkv + h) * a.T + t];
  a.mass_shared[i] = sum;
}

}  // namespace

// FEEDER: fewer than eight heads per KV head (room for feeder wavefronts behind the scoring ones)
template <bool FEEDER>
static void launch_psa_gqa_passes(const SelectArgs &a, hipStream_t stream) {
  const int R = a.Hq / a.Hkv;
  const dim3 grid(a.n_chunk, a.B * a.Hkv);
  // first pass: two wavefronts per head and two feeders (one feeder would be the slowest wavefront of the workgroup:
  // about 240 vector instructions per block against 150 of a scoring wavefront); second pass: one per head, one feeder
  constexpr int kItems = FEEDER ? kGqaItems / 2 : kGqaItems / (2 * kGqaMaxHeads);
  const dim3 block(64 * (2 * R + (FEEDER ? 2 : 0)));
  if (a.chunk == kScoreChunk) hipLaunchKernelGGL((psa_row_stats_gqa_kernel<2, kItems, true>), grid, block, 0, stream, a);
  else hipLaunchKernelGGL((psa_row_stats_gqa_kernel<2, kItems, false>), grid, block, 0, stream, a);
  if (R == 1) {
    // one head: a single scoring wavefront would leave the workgroup at two wavefronts; two of 32 rows and two feeders
    hipLaunchKernelGGL((psa_mass_gqa_kernel<2, kGqaItems / 2>), grid, dim3(64 * 4), 0, stream, a);
    return;
  }
  // (two wavefronts per head and two feeders, measured with seven heads: 692 against 645 us at cfg5)
  hipLaunchKernelGGL((psa_mass_gqa_kernel<4, FEEDER ? kGqaItems : kGqaItems / kGqaMaxHeads>), grid,
                     dim3(64 * (R + (FEEDER ? 1 : 0))), 0, stream, a);
}
template <int NRB>
static void launch_psa_passes(const SelectArgs &a, hipStream_t stream) {
  if constexpr (NRB == 4) {  // the kernels with feeder wavefronts exist for W = 64 only
    const int R = a.Hq / a.Hkv;
    if (R == kGqaMaxHeads) return launch_psa_gqa_passes<false>(a, stream);
    if (R >= 1 && R < kGqaMaxHeads) return launch_psa_gqa_passes<true>(a, stream);
  }
  const dim3 block(256);
  hipLaunchKernelGGL(psa_row_stats_kernel<NRB>, dim3(a.n_chunk, a.B * a.Hq), block, 0, stream, a);
  hipLaunchKernelGGL(psa_mass_kernel<NRB>, dim3(a.n_chunk, a.B * a.Hkv), block, 0, stream, a);
}

static void launch_psa_once(const SelectArgs &a, hipStream_t stream) {
  const size_t pairs = (size_t)a.B * a.Hq * a.n_chunk * 32;  // of words
  hipLaunchKernelGGL(clear_stats_kernel, dim3((unsigned)((pairs + 255) / 256)), dim3(256), 0, stream,
                     reinterpret_cast<u32x4 *>(a.row_stats), pairs);
  // as many heads abreast as two workgroups per CU hold, in rounds of equal length
  const int heads = a.B * a.Hq, most = 2 * kScoreCus / a.n_chunk, rounds = (heads + most - 1) / most;
  const dim3 grid(a.n_chunk, (heads + rounds - 1) / rounds), block(64 * kOnceWaves);
  if (a.n_chunk <= kOnceBatch * kOnceWaves) hipLaunchKernelGGL((psa_once_kernel<kOnceBatch, 2>), grid, block, 0, stream, a);
  else hipLaunchKernelGGL((psa_once_kernel<kOnceWords, 1>), grid, block, 0, stream, a);
}

hipError_t launch_select_psa(const SelectArgs &a, hipStream_t stream) {
  if (a.score_path == kScoreSmall) {
    const dim3 grid(a.B * a.Hq);
    const bool whole = a.Hq == a.Hkv;  // with the top-k
    if (a.T <= 256) hipLaunchKernelGGL((whole ? psa_small_kernel<256, true> : psa_small_kernel<256, false>), grid, dim3(256), 0, stream, a);
    else if (a.T <= 512) hipLaunchKernelGGL((whole ? psa_small_kernel<512, true> : psa_small_kernel<512, false>), grid, dim3(512), 0, stream, a);
    else hipLaunchKernelGGL((whole ? psa_small_kernel<kSmallKeys, true> : psa_small_kernel<kSmallKeys, false>), grid, dim3(kSmallKeys), 0, stream, a);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess || whole ? e : launch_topk(a, stream);
  }
  if (a.score_path == kScoreOnce) {
    launch_psa_once(a, stream);
  } else {
    switch (a.W / 16) {
      case 1: launch_psa_passes<1>(a, stream); break;
      case 2: launch_psa_passes<2>(a, stream); break;
      case 3: launch_psa_passes<3>(a, stream); break;
      default: launch_psa_passes<4>(a, stream); break;
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  SelectArgs k = a;  // what the top-k reads
  if (a.mass_shared != nullptr) {
    hipLaunchKernelGGL(sum_heads_kernel, dim3((unsigned)(((long)a.B * a.T + 255) / 256)), dim3(256), 0, stream, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    k.mass = a.mass_shared;
    k.mass_per_batch = 1;
  }
  return launch_topk(k, stream);
}

}  // namespace akvq

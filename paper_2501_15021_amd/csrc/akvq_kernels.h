// Host-side launch interfaces of the libakvq kernels (internal; the public ABI is include/akvq.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace akvq {

struct QuantArgs {
  const uint16_t *k_new, *v_new;  // [B][Hkv][n_new][128] binary16
  uint32_t *k_codes, *v_codes, *k_meta, *v_meta;
  uint16_t *k_sal, *v_sal;
  const int32_t *sal_idx, *sal_cnt;
  int Hkv, T_cap, S_cap, T_len, n_new;
  int first_blk, n_blk;  // 32-token blocks touched by rows [T_len, T_len + n_new)
  float clip;
  int rotate_k, rotate_v;
  // tiered append (all null / zero for the plain call): source row and tier of every new cache row, per batch element
  const int32_t *row_src;   // [B][n_new]
  const uint8_t *row_tier;  // [B][n_new]
  uint32_t *fine_mask;      // [B][T_cap/32]
  int n_src;                // rows per (b, kv-head) in k_new / v_new (= n_new for the plain call)
  float clip4;
  uint16_t *k_win, *v_win;  // recent-window rings (null: none)
  int win_len;
  int win_blk;  // first block that holds window rows (set by the launcher)
  int groups, turn;  // workgroups of one unit's tensor, and by how many of them (at most) a unit's order is turned (set by the launcher)
  const uint16_t *rope_cos, *rope_sin;  // rotary tables for pre-RoPE K rows (null: rows arrive embedded), [n_src][64] binary16
  long long rope_stride;                // elements between the tables of consecutive batch elements
  int skip_overlay;  // the block kernel leaves the 16-bit V rows to the overlay pass (in its launch or behind it)
};
hipError_t launch_quantize_append(const QuantArgs &a, int B, int G, hipStream_t stream);
constexpr long kAppendCus = 256;
// Whether the groups of four blocks of an append (units: batch elements x KV heads, of n_blk blocks each; two tensors) run on from unit
// to unit.  Units whose last group is short leave wavefronts without a block, and with an even number of groups the
// short ones all fall on the same XCDs: from two workgroups a CU on, and a twelfth of the wavefronts idle, the groups run on
// from unit to unit instead (up to 33 blocks).  29 prompts of 397 tokens, 32 heads, 61.5 -> 52.3 us; 64 of 150, 75 -> 54.
// With fewer idle it gains nothing (16 of 8200, 4 heads, takes 1.1).
// Up to ten rounds of workgroups, one per CU each, there has to be a round less: a CU whose last workgroup was a short one has four
// full wavefronts instead (3 of 275, 40 heads, rotary, 720 workgroups to 540, three rounds both: 8.9 -> 9.6; 3 of 668, 40 heads, 1440
// to 1320, six both: 10.7 -> 11.7; but 5 of 144, 40 heads, 800 to 500, 11.0 -> 8.1).  From five to ten rounds more than an eighth of
// the wavefronts, and two of a unit, have to be idle as well (52 of 1051, 2 heads, a twelfth, eight rounds to seven, 13.4 -> 14.5; 3 of 659,
// 40 heads, an eighth, six to five, 11.6 -> 12.3; 110 of 91, 8 heads, rotary, one of four, seven to six, 12.8 -> 13.8).  Units of three blocks
// gain from three rounds to two (264 units 6.4 -> 5.2) and not beyond (118 of 91, 4 heads, four to three, 7.7 -> 8.1).
// 400 shapes that pass, 512 to 8000 workgroups, plain, rotary and with tiers: 0.90 of the time, three above 1.01, at most 1.04 (74 of
// 314, 4 heads, seven rounds to six, 13.2 -> 13.7).
inline bool append_runs_on(long units, int n_blk, bool window) {
  const int groups = (n_blk + 3) / 4, idle = 4 * groups - n_blk;
  const long blocks = units * n_blk, in_units = 2 * units * groups, in_row = 2 * ((blocks + 3) / 4);  // workgroups
  const auto rounds = [](long workgroups) { return (workgroups + kAppendCus - 1) / kAppendCus; };
  if (window || n_blk <= 1 || 3 * idle < groups || in_units <= 2 * kAppendCus || blocks * n_blk >= (1l << 32)) return false;
  if (in_units > 10 * kAppendCus) return true;
  if (rounds(in_row) >= rounds(in_units)) return false;
  return in_units > 5 * kAppendCus ? idle >= 2 && 2 * idle > groups : n_blk != 3 || in_row <= 2 * kAppendCus;
}
// Block `at` of such an append is one of unit (at * reciprocal_of_blocks(n_blk)) >> 32: with blocks * n_blk below 2^32 the rounding up
// does not reach the next unit.
inline uint32_t reciprocal_of_blocks(int n_blk) { return (uint32_t)(((1ull << 32) + n_blk - 1) / n_blk); }

struct DecodeArgs {
  const uint32_t *k_codes, *v_codes, *k_meta, *v_meta;
  const uint16_t *k_sal, *v_sal;
  const int32_t *sal_idx, *sal_cnt;
  const uint32_t *fine_mask;  // [B][T_cap/32] or null: fine halves of 4-bit tokens stored as row pairs
  const uint16_t *k_win, *v_win;  // recent-window rings (null: none), win_len slots
  int win_len;
  int t_win;                  // first row read from the rings (= T_len without a window)
  const uint16_t *q;  // [B][Hq][128] binary16
  float *partial;     // [B*Hq][n_split][kPartialStride] fp32
  void *out;          // [B][Hq][128] fp32, or binary16 when out_half
  float *lse;         // optional [B][Hq]
  int B, Hq, Hkv, T_cap, S_cap, T_len, n_split;
  float sm_scale;
  int q_rotated, out_rotated, out_half;
  // the decode step in one launch: row T_len - 1 is first quantized from step.k_new / step.v_new (step.T_len is that
  // row) by the workgroups of split append_split: the split whose tile range holds the tile of that row (see
  // decode_split_range), so that the row is written and read by the same workgroup.  For the same reason they are the only
  // ones to read the salient rows then, and the new row's unit of the recent window (the one-head kernel deals the window's
  // other units to all splits, the grouped-query kernel leaves the whole window to them).
  int fused_append;
  int append_split;
  // (16 bits each: with an int more in front of them the step's arguments lie 8 bytes further, and a fused step of 20011 rows,
  // 28/4 heads, window and rotary embedding, took 12.47 us instead of 12.35)
  short paced;  // grouped-query launch, all of it resident at once: wavefronts of a SIMD are kept in step (set by the launcher)
  short row_pairs;  // one-head launch: units of 16-bit rows from which on they are taken in pairs, 0: never (set by the launcher)
  QuantArgs step;
  const uint16_t *rope_cos, *rope_sin;  // rotary tables for pre-RoPE queries (null: none), one row of 64 per batch element
  long long rope_stride;
};
constexpr int kPartialStride = 132;  // m, l, 2 pad, 128 accumulators

// How the code stream's n_tiles tiles are dealt to the n_split KV splits: equal runs of ceil(n_tiles / n_split) tiles,
// so trailing splits can be short or empty.  Used by the kernels, by the host (append_split) and by the public helper
// akvq_decode_split_range, so that all three agree by construction.
__host__ __device__ inline int decode_tiles_per_split(int n_tiles, int n_split) {
  return n_tiles > 0 ? (n_tiles - 1) / n_split + 1 : 0;  // ceil(n_tiles / n_split) without overflow
}
__host__ __device__ inline void decode_split_range(int n_tiles, int n_split, int split, int &begin, int &end) {
  const int per = decode_tiles_per_split(n_tiles, n_split);
  const long long b = (long long)split * per, e = b + per;
  begin = (int)(b < n_tiles ? b : n_tiles);
  end = (int)(e < n_tiles ? e : n_tiles);
}
// the split whose range holds the last tile (the tile of the row a fused decode step appends); split 0 if there is no tile
__host__ __device__ inline int decode_last_tile_split(int n_tiles, int n_split) {
  if (n_tiles <= 0) return 0;
  return (n_tiles - 1) / decode_tiles_per_split(n_tiles, n_split);
}
// ---- how many KV splits: one workgroup per (unit, split), unit = (batch, kv-head) ----
// Two workgroups per CU, measured with workgroups of four wavefronts, which most launches of more than 64 units have.
inline int decode_splits_by_two(long units, int tiles) {
  if (units >= 512) return 1;                  // already two workgroups per CU: finish in one kernel, no merge pass
  long want = (512 + units - 1) / units;       // more splits only add merge work
  const long cap = tiles / 16 > 1 ? tiles / 16 : 1;  // keep at least 16 64-token tiles per workgroup
  if (want > cap) want = cap;
  if (want > 64) want = 64;
  // A split adds the merge launch (about 8 us end to end): with more than 128 units it only pays when every workgroup
  // still streams at least 48 tiles (measured: 256 units of 64 tiles run 19.7 us unsplit, 21.7 us in two splits).
  if (units > 128 && tiles / want < 48) want = tiles / 48 > 1 ? tiles / 48 : 1;
  return (int)want;
}
// Up to 64 units: one workgroup per CU at most, of eight wavefronts, and one merge; two tiles a workgroup at least, and up to 32
// splits, what the merge reads in one round trip (64 where 512 tiles and more make the streams longer than a second one).
// None below 1024 rows (1 x 700 rows, 28/4 heads, 9.0 us in 1, 4 or 8 splits; 640 rows, 32 heads, 6.7 in 1, 7.7 in 8).
// Us in decode_splits_by_two and so: a step of 20011 rows, 28/4 heads, with window and rotary embedding, 16.0, 12.7; 12000 rows
// 14.0, 10.9; 12/2 heads, 4000 rows 14.3, 10.2; 32 heads, 2500 rows 10.8, 8.8, 8000 rows 11.9, 11.4.  Rounding 256 / units
// down leaves up to a fifth of the CUs idle, and is still faster at 33 to 60 units: decode of 52 units, 28/4 heads, 2048 / 8192 /
// 32768 rows, 13.5 / 18.5 / 41.9 us in 2 / 8 / 10 splits and 12.5 / 17.7 / 37.1 in 4; 104 shapes of 1 to 64 units, 2048 to
// 131072 rows: nowhere slower.  (Two full rounds of four wavefronts, 512 / units, are better still on long streams that leave
// CUs idle: 52 units of 32768 rows, 9 splits, 35.3; 44 and 60 units: equal.)
inline int decode_most_splits(long units, int T_len) {
  const int tiles = (int)(((long)T_len + 63) / 64);
  if (units > 64) return decode_splits_by_two(units, tiles);
  if (T_len < 1024) return 1;
  long n = 256 / units;
  if (n > 32) n = tiles >= 512 && n >= 64 ? 64 : 32;
  return (int)(n < tiles / 2 ? n : tiles / 2);
}
// What a call without a split count gets: as many, or decode_splits_by_two where the streams are so short that the merge
// launch costs what the splits gain.  Where that is depends on how much of the work the splits share: 16-bit rows are dealt to
// them too (good from 1024 rows on: 2 x 1024 rows, 28/4 heads, window 512, 1 split or 8: 12.9 and 10.2 us), but a fused step
// of the grouped-query kernel leaves all of them, and one of either kernel the salient ones, to the split that appends (same
// shape, a step: 14.6 and 15.8).  It depends on how many splits there are: with more than 48 units four or five share what
// eight wavefronts did in one (60 x 1024, 8/1 heads: 9.6, 10.8).  Steps of 13 to 48 units with such rows pay later (4 x 1024
// rows, 32/8 heads, window 64: 11.2, 12.5).  5772 calls of 1 to 64 units, 1024 to 5000 rows, against decode_splits_by_two for
// all: with decode_most_splits for all 848 were more than 2.5 % slower, 224 of them more than 10 %; so 97 and none.
inline int decode_splits(const DecodeArgs &a, bool fused) {
  const long units = (long)a.B * a.Hkv;
  const int most = decode_most_splits(units, a.T_len);
  if (units > 64 || most == 1) return most;
  const bool mha = a.Hq == a.Hkv;
  const int win = a.T_len - a.t_win, listed = a.S_cap > 64 ? a.S_cap : 0;
  int from;  // rows from which on the splits pay
  if (!fused && win + listed >= 256) from = 1024;
  else if (mha && fused) from = units > 48 ? 1153 : 1024;
  else if (mha) from = units > 48 ? (win > 0 ? 1473 : 1985) : units > 32 && win == 0 ? 1473 : 1024;
  else if (units > 48) from = 1729;
  else if (fused) from = units > 12 && win + listed > 0 ? 1217 : 1024;
  else from = 1281;
  if (fused) {
    const int alone = (mha ? 0 : win) + listed;
    if (alone > 128) from += 5 * (alone - 128) / 2;
    if (mha && listed > 0 && units > 12) from += 256;
  }
  if (a.T_len >= from) return most;
  const int few = decode_splits_by_two(units, (a.T_len + 63) / 64);
  return few < most ? few : most;
}
// How the units of 32 16-bit rows are dealt in the one-head kernel: index i of a wavefront runs from first in steps of step while it is below
// limit, and stands for unit(i).  From the last wavefront on (when the tiles do not divide evenly, the last ones have one
// tile less), to the splits before the wavefronts.
// In a fused decode step the unit of the new row is read by the workgroups that write it, as the salient rows are (the new
// one may be among them); the other units of the recent window go to every split.  With one split there is nothing to
// deal, and both calls take the rows in the same order.
struct RowUnits {
  int first, step, limit, special;  // special: the unit that negative indices stand for; no other index does
  __host__ __device__ inline int unit(int i) const { return i < 0 ? special : i + (i >= special ? 1 : 0); }
};
constexpr int kRowUnit = 32;
template <int NW>
__host__ __device__ inline RowUnits salient_units(const DecodeArgs &a, int cnt, int split, int wave, bool appends) {
  const int n = (cnt + kRowUnit - 1) / kRowUnit, back = NW - 1 - wave;
  if (a.fused_append) return {back, NW, appends ? n : 0, n};
  return {split + back * a.n_split, NW * a.n_split, n, n};
}
template <int NW>
__host__ __device__ inline RowUnits window_units(const DecodeArgs &a, int cnt_salient, int split, int wave, bool appends) {
  const int n = a.win_len / kRowUnit, back = NW - 1 - wave, step = NW * a.n_split;
  if (a.fused_append && a.n_split > 1) {
    // the appending workgroup's last wavefront has the first salient rows, the one before it the new row
    const int p = (back + (appends ? NW - 2 : 0)) % NW;
    const int first = split + p * a.n_split;
    return {appends && wave == NW - 2 ? first - step : first, step, n - 1, ((a.T_len - 1) % a.win_len) / kRowUnit};
  }
  // behind the salient units
  const int first = split + back * a.n_split - (cnt_salient + kRowUnit - 1) / kRowUnit % step;
  return {first < 0 ? first + step : first, step, n, n};
}
// ... and in pairs of units (one split): index i stands for units 2 * i and 2 * i + 1; behind the pairs of `before` rows
template <int NW>
__host__ __device__ inline RowUnits paired_units(int rows, int before, int wave) {
  const int n = (rows + 2 * kRowUnit - 1) / (2 * kRowUnit), first = (NW - 1 - wave) - (before + 2 * kRowUnit - 1) / (2 * kRowUnit) % NW;
  return {first < 0 ? first + NW : first, NW, n, n};
}
constexpr int kMhaTileRows = 64, kGqaTileRows = 32;  // rows per code-stream tile of the two decode kernels
hipError_t launch_decode_attention(const DecodeArgs &a, int G, hipStream_t stream);
// Device address, on the current device, of the library's fixed scratch array for split-KV partials (no allocation).
constexpr size_t kDecodeStaticScratchBytes = 8u << 20;
hipError_t decode_static_scratch(void **ptr);

struct SelectArgs {
  const uint8_t *is_text;    // [B][T]
  const uint16_t *q_tail;    // [B][Hq][W][128] binary16
  const uint16_t *k;         // [B][Hkv][T][128] binary16
  int32_t *sal_idx, *sal_cnt;
  float *mass;               // [B][Hkv][T] fp32 (user buffer or workspace)
  float *row_stats;          // workspace: [B][Hq][n_chunk][W][2]
  int B, Hq, Hkv, T, W, top_k, S_cap;
  int chunk, n_chunk;        // keys per scoring workgroup (score_chunk) and how many of them cover T
  float sm_scale;
  // massive-activation mode: hidden states, one score row per batch element, zero keys are never selected
  const uint16_t *hidden;    // [B][T][d_model] binary16
  int d_model;
  float floor;
  int mass_per_batch;        // top-k reads mass[b][T] (shared by the batch element's kv-heads) instead of mass[b][hkv][T]
  int skip_zero;
  int score_path;            // ScorePath
  float *score;              // where the scoring of kScoreSmall and kScoreOnce leaves a query head's masses, rows of score_stride: mass
  int score_stride;          // itself, or workspace with several heads per KV head (16-byte aligned rows)
  float *mass_shared;        // token-level pivots: [B][T] sums of the kv-heads' masses (workspace), null: per-head lists
};
// Keys per scoring workgroup: kScoreChunk, or less where that leaves the chip idle (scoring windows of 64 rows only; the
// kernels for smaller windows have it built in, and beyond two workgroups per CU there is nothing to fill).  The prompt is
// cut into n chunks of equal length, for the n with the least time by this model: the workgroups go in rounds of one or
// two per CU, each as long as its keys plus the staging of the rows (192 keys' worth); a round of two takes 1.5, 1.75 or
// 2 times one of one, with one, two or three, and more heads per KV head (4 wavefronts a workgroup, 6 to 8, 10 to 18).
// Equal lengths, because a chunk's number decides its die (workgroup id mod 8): with 2 chunks the long ones would all go
// to four of the eight dies.  Not below two blocks of keys, nor beyond 64 chunks, whose statistics the second pass merges
// in four round trips, nor beyond four workgroups per CU.
// Over 1053 shapes (1 to 8 heads per KV head, 4 to 600 units, 258 to 32768 tokens) a selection takes 0.69 of its time with
// chunks of 2048 on average, at most 1.04 (what two runs of one length differ), and 1.03 of the best length tried.  One
// prompt, in two passes (score_path has most of those with one head per KV head read once): 32 heads, 640 tokens 29.1 -> 18.7 us,
// 4096 tokens 72.3 -> 31.0, 16384 tokens 82.4 -> 62.8; 28/4 heads, 4096
// tokens 142 -> 35, 32768 tokens 160 -> 76; 40 prompts of 1300 tokens, 28/4 heads, 100 -> 92, and 16 of 4907 142 -> 103,
// where halving the chunk until every CU has a workgroup, whatever the rounds and lengths, makes 148 and 151.
constexpr int kScoreChunk = 2048, kScoreChunkMin = 128, kScoreMaxFineChunks = 64, kScoreCus = 256;
constexpr int kSmallKeys = 768, kOnceKeys = 512, kOnceMaxChunks = 64;  // keys of the two kernels that read them once (score_path)
inline bool score_fine_chunks(int Hq, int Hkv, int W) { return W == 64 && Hq >= Hkv && Hq / Hkv <= 8; }
inline int score_chunk(int B, int Hq, int Hkv, int T, int W) {
  const long units = (long)B * Hkv, n_coarse = ((long)T + kScoreChunk - 1) / kScoreChunk;
  if (!score_fine_chunks(Hq, Hkv, W) || units * n_coarse > 2 * kScoreCus) return kScoreChunk;
  const int R = Hq / Hkv;
  const long one = 4, two = R == 1 ? 6 : R <= 3 ? 7 : 8;  // quarters of a round's time: one workgroup per CU, two
  int chunk = kScoreChunk;
  long best = 0;
  for (long n = n_coarse; n == n_coarse || (n <= kScoreMaxFineChunks && units * n <= 4 * kScoreCus); ++n) {
    const long keys = ((T + n - 1) / n + 63) / 64 * 64;
    if (n > n_coarse && keys < kScoreChunkMin) break;
    const long groups = units * ((T + keys - 1) / keys), rest = groups % (2 * kScoreCus);
    const long time = (groups / (2 * kScoreCus) * two + (rest == 0 ? 0 : rest <= kScoreCus ? one : two)) * (keys + 192);
    if (best == 0 || time < best) { best = time; chunk = (int)keys; }
  }
  return chunk;
}
// Most (batch, head, chunk) triples that score_chunk makes of any batch up to B and any prompt up to T: it grows with B
// and T, which the triples of one shape do not (a longer prompt can have fewer, larger chunks).
inline size_t score_max_triples(int B, int Hq, int Hkv, int T, int W) {
  const size_t heads = (size_t)B * Hq;
  size_t coarse = heads * (((size_t)T + kScoreChunk - 1) / kScoreChunk);
  if (!score_fine_chunks(Hq, Hkv, W)) return coarse;
  if (Hq == Hkv) {  // a prompt read once
    const size_t keys = T < kOnceKeys * kOnceMaxChunks ? T : kOnceKeys * kOnceMaxChunks;
    const size_t once = heads * ((keys + kOnceKeys - 1) / kOnceKeys);
    if (once > coarse) coarse = once;
  }
  size_t fine = heads * (((size_t)T + kScoreChunkMin - 1) / kScoreChunkMin);
  if (fine > heads * kScoreMaxFineChunks) fine = heads * kScoreMaxFineChunks;
  const size_t filled = (size_t)(4 * kScoreCus) * (Hq / Hkv);  // four workgroups per CU, of Hq / Hkv heads each
  if (fine > filled) fine = filled;
  return fine > coarse ? fine : coarse;
}
// How a prompt's pivots are scored.  Two passes over the keys serve everything; where a head's exponentials fit into registers
// until its row statistics are known, one does: one workgroup per query head (psa_small_kernel), or as many as the keys need
// (psa_once_kernel: a launch more, which clears the words they exchange).
// One head per KV head: in one pass up to kOnceKeys * kOnceMaxChunks keys (beyond, the words a workgroup collects are a
// quarter of its keys and more).  110 shapes of 513 to 768 keys: 0.76 of the time of two passes; the small kernel up to
// 512 workgroups, two rounds of them on the CUs: 16 x 640 keys, 32 heads, 33.3 us in small, 33.9 in once, 32 x 640 63.9 and 57.8.  Up
// to 64 workgroups of the once kernel and four chunks, two passes of shorter chunks are as fast: 77 such shapes 0.99 of their time, 12 of them
// 1.02 to 1.07 (16 x 971 keys 14.8 -> 15.8); 143 others of 513 to 2600 keys, up to 200 heads, 0.86, one above 1.01 (1.026).
// Several heads per KV head: each head reads and converts the keys for itself, which costs what the second pass did (64 x 768
// keys, 32/8 heads, 101 us in two passes, 112 in one; 16 x 8192, 28/4 heads, 150 and 209), so one pass pays where everything is
// resident at once: it is a launch less, or the same three with shorter ones (2 x 1000, 12/2 heads, 26.2 -> 18.2).  In the small
// kernel up to 512 keys that is 512 workgroups, two per CU, beyond one per CU; up to 256 keys with four per CU it is faster at any
// number (73 x 256, 28/4 heads, 64 -> 38), but not with eight heads, whose two passes have no feeders to wait for (32 x 256,
// 64/8 heads, 1.05 of the time).  671 shapes of 256 to 4096 keys, 2 to 8 heads: 0.87 of the time of two passes; of 240 in one pass,
// 513 to 20000 keys, 0.82, ten 1.02 to 1.046 (100 heads, four to a KV head, of 1202 keys 20.6 -> 21.3; of other shapes 18, three to one, of 7349 28.8
// -> 30.9), all with 2 to 4 heads per KV head and among others that gain as much.
enum ScorePath { kScoreTwoPasses, kScoreSmall, kScoreOnce };
inline int score_path(int B, int Hq, int Hkv, int T, int W, float sm_scale, bool shared) {
  const long heads = (long)B * Hq, chunks = ((long)T + kOnceKeys - 1) / kOnceKeys;
  if (W != 64 || Hq > 8 * Hkv || !(sm_scale > 0.0f) || chunks > kOnceMaxChunks) return kScoreTwoPasses;
  if (Hq == Hkv) {
    if (T <= 512 || (T <= kSmallKeys && heads <= 2 * kScoreCus)) return shared ? kScoreTwoPasses : kScoreSmall;
    return T <= 4 * kOnceKeys && heads * chunks <= 64 ? kScoreTwoPasses : kScoreOnce;
  }
  if (shared) return kScoreTwoPasses;  // (each KV head's mass is needed before they are added)
  const long small = T <= 256 ? (Hq < 8 * Hkv ? heads : 2 * kScoreCus) : T <= 512 ? 2 * kScoreCus : T <= kSmallKeys ? kScoreCus : 0;
  if (heads <= small) return kScoreSmall;
  return heads * chunks <= 2 * kScoreCus ? kScoreOnce : kScoreTwoPasses;
}
// How long a workgroup of psa_once_kernel waits for the statistics of its head's other chunks before it scores a missing one itself:
// kOncePolls looks for a whole head, and none any more for that head once they have run out.  The head behind one that
// ran out gets kOnceFewPolls, and kOncePolls again behind one that did not.  So a row of workgroups whose siblings are never
// resident waits 16 ms once and 64 us for each later head, and scores every chunk of its heads itself.
#ifndef AKVQ_ONCE_POLLS
#define AKVQ_ONCE_POLLS (1 << 14)
#endif
constexpr int kOncePolls = AKVQ_ONCE_POLLS;  // about a microsecond each
constexpr int kOnceFewPolls = kOncePolls < 64 ? kOncePolls : 64;
struct OnceWait {
  int left = kOncePolls;  // looks at missing words
  bool gave_up = false;
  __host__ __device__ bool look_again() { return left > 0 && left-- > 0; }
  __host__ __device__ void give_up() { left = 0; gave_up = true; }
  __host__ __device__ void next_head() { left = gave_up ? kOnceFewPolls : kOncePolls; gave_up = false; }
};
// The missing chunk (set bits) that the workgroup of chunk `own` scores: the first one from its own on, so that those who wait
// for the same chunks do not all begin with the same one.
__host__ __device__ inline int once_chunk_to_score(uint64_t missing, int own) {
  const uint64_t ahead = missing >> own << own;
  return __builtin_ctzll(ahead ? ahead : missing);
}
// Masses of single query heads, with several per KV head: elements of a shape, and the most of any batch up to B and prompt up to T
inline size_t score_stride(int T) { return ((size_t)T + 3) / 4 * 4; }
inline size_t score_head_masses(int B, int Hq, int Hkv, int T) { return Hq > Hkv ? (size_t)B * Hq * score_stride(T) : 0; }
inline size_t score_max_head_masses(int B, int Hq, int Hkv, int T, int W) {
  if (Hq <= Hkv || W != 64 || Hq > 8 * Hkv) return 0;
  const size_t heads = (size_t)B * Hq, all = heads * score_stride(T);
  const size_t resident = (size_t)2 * kScoreCus * (kOnceKeys + 4), few_keys = heads * (T < 256 ? score_stride(T) : 256);
  const size_t most = resident > few_keys ? resident : few_keys;
  return all < most ? all : most;
}
// Threads of a workgroup that lists the text positions of one row of T (rows: batch elements x KV heads): with 256 a round covers
// 4096 positions, with 1024 it covers 16384, but its barriers and scan are longer.  1024 for rows of more than two rounds where one
// workgroup per CU holds them all (us: 28 rows of 15167 positions 8.4 -> 6.3, 32 of 32768 9.7 -> 5.8; 99 such shapes 0.83 of the time, at most
// 0.99).  Not for shorter ones (160 of 6808, 6.1 and 6.4; 80 of 8020, 5.9 and 6.1), nor for more rows (352 of 20425, 11.0 and 12.7; 288 of
// 4708, 4.2 and 5.0; 2048 of 8192, 8.3 and 15.9).
inline int text_threads(long rows, int T) { return T > 8192 && rows <= kScoreCus ? 1024 : 256; }
hipError_t launch_select_tsa(const SelectArgs &a, hipStream_t stream);
hipError_t launch_select_psa(const SelectArgs &a, hipStream_t stream);
hipError_t launch_select_massive(const SelectArgs &a, hipStream_t stream);

// offline fold of H_128 into a projection matrix w [rows][cols] binary16 (axis 1: runs of 128 columns, axis 0: of rows)
hipError_t launch_fold_hadamard(const uint16_t *w, uint16_t *out, int rows, int cols, int axis, hipStream_t stream);

// measurement aid: plain 128-bit streaming read of `bytes` bytes (a multiple of 16, at least 16)
hipError_t launch_stream_read(const void *src, size_t bytes, uint32_t *sink, int non_temporal, hipStream_t stream);

}  // namespace akvq

// da_api.cpp -- the C ABI of include/delta_attn.h: argument validation,
// workspace planning and the launch sequence of the Delta Attention prefill.
#include <math.h>
#include <string.h>

#include <cmath>

#include <atomic>

#include "delta_attn.h"
#include "da_internal.hpp"

namespace da {

namespace {

constexpr int kCUs = 256;  // of a gfx950
constexpr int64_t kPartialBudget = (int64_t)8 << 30;  // bytes of the strided rows' partials

thread_local int g_last_hip_error = 0;

// Per-device answer to "is this a gfx950": 0 unknown, 1 yes, 2 no.
constexpr int kMaxDevices = 64;
std::atomic<int> g_arch_ok[kMaxDevices];
thread_local int g_cur_dev = 0;  // the device check_device() last looked at

da_status fail_hip(hipError_t e) {
  g_last_hip_error = (int)e;
  return DA_ERR_HIP;
}

da_status check_device() {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail_hip(e);
  if (dev < 0 || dev >= kMaxDevices) return DA_ERR_UNSUPPORTED;
  int st = g_arch_ok[dev].load(std::memory_order_relaxed);
  if (st == 0) {
    hipDeviceProp_t prop;
    e = hipGetDeviceProperties(&prop, dev);
    if (e != hipSuccess) return fail_hip(e);
    st = (strncmp(prop.gcnArchName, "gfx950", 6) == 0) ? 1 : 2;
    g_arch_ok[dev].store(st, std::memory_order_relaxed);
  }
  g_cur_dev = dev;
  return st == 1 ? DA_OK : DA_ERR_UNSUPPORTED;
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

}  // namespace

// Query heads of one GQA group that share an attention workgroup: the
// largest power of two dividing G, at most its wavefronts.
int heads_per_block(int G, int waves) {
  int h = 1;
  while (h * 2 <= waves && G % (h * 2) == 0) h *= 2;
  return h;
}

int fused_heads_per_block(int G, int gamma, int max_rows, int waves) {
  for (int h = heads_per_block(G, waves); h >= 1; h /= 2) {
    const int slab = kRowsPerWave * (waves / h);
    if (G % h == 0 && slab % gamma == 0 && slab <= max_rows) return h;
  }
  return 0;
}

// Key tiles all strided-row workgroups of kAttnWaves wavefronts run together:
// row tiles of rpb rows, the anchors' growing with their position, those of
// `tail` further rows reaching over the whole sequence.
static int64_t strided_tiles(int64_t B, int64_t N, int Hq, int G, int64_t gamma, int64_t tail) {
  const int hpw = heads_per_block(G);
  const int64_t rpb = kRowsPerWave * (kAttnWaves / hpw);
  const int64_t T = (N + kKeyTile - 1) / kKeyTile;
  const int64_t nA = N / gamma, ra = (nA + rpb - 1) / rpb;
  int64_t per = (int64_t)((double)ra * (ra + 1) / 2 * rpb * gamma / kKeyTile);
  if (per > ra * T) per = ra * T;
  per += ((nA + tail + rpb - 1) / rpb - ra) * T;
  return B * (Hq / hpw) * per;
}

// Workspace of the Delta path.  Dense rows of a sequence of length L are the
// floor(L/gamma) anchors plus the L mod gamma tail rows.  Their key axis is
// split into nC chunks of `chunk` keys (at least kLongChunk tiles), up to 16 of
// them.  Workgroups that run at the same time then process one key chunk each
// in step with their neighbours, which keeps them sharing that chunk's keys
// and values in L2.  (The minimum sets nC only below 40960 keys.  At 32768, 13
// chunks of 2560 keys fill just under two rounds of the CUs where 16 of 2048
// filled two and a quarter: 15 % less time on the strided rows and merge.)
// Where chunks of that size leave CUs idle, shorter ones spread the rows over
// the chip: as many tiles as give every CU one full-size workgroup's worth (two
// half-size ones), at least kShortChunk.  In a batch the lengths may lie below
// max_seqlen, so its chunks are half as long again shorter.  Measured on an
// MI355X, Delta prefill, 2560-key minimum -> this: 32 heads d 128, 1024 tokens
// 43.8 -> 27.5 us, 2048 tokens 70.9 -> 36 us, 4021 tokens 168 -> 139 us, 8192
// tokens 120 -> 96 us; 32 heads d 64, 2048 tokens 52.4 -> 27.6 us; eight packed
// prompts up to 3071 tokens 232 -> 212 us.  Against 2 tiles, a minimum of 4
// takes 29.3 us at 1024 tokens and 8 takes 34.4 us; from 2048 tokens on 2 to 4
// are alike.  Twice as many chunks cost 5 % where the grid is full already
// (12000 tokens 154 -> 166 us).  Sequences of at most 448 keys keep one chunk,
// which needs no merge, however few workgroups that makes.  One chunk -> two and
// more, whole calls, gamma 64: one d 64 head 449 tokens 22.0 -> 19.2 us, 1024 tokens
// 30.7 -> 20.4 us; 16 heads d 64 300 tokens 18.0 -> 19.3 us; 32 heads d 128 300
// tokens 24.5 -> 25.4 us, 520 tokens 30.8 -> 26.7 us.  (At 400 tokens two chunks
// would take 7-13 % less already: 26.9 -> 24.1 us, 21.4 -> 20.0 us.)
// Each chunk also costs a partial per row, written and read again.  Where the anchors'
// are many (gamma 1 to 8: 12.5 MB a chunk at d = 128, twice that at d = 64) and chunks of
// 2560 keys give the CUs 0.65 rounds of work, that outweighs what finer ones gain:
// finer -> long, 3 -> 2 chunks, 32 heads, gamma 2, 2814 tokens 125 -> 119 us; 5 -> 3, 9
// heads, 6008 tokens 112 -> 102 us; 2 -> 1, 40 heads, gamma 1, 2122 tokens 117 -> 95 us;
// packed, 6 -> 4, 12 heads, gamma 7, 8248 tokens 297 -> 256 us.  Below that: 0.49 rounds,
// 4 -> 2, 32 heads, gamma 4, 3402 tokens 82.7 -> 85.7 us; 10 MB, 6 -> 4, 8 heads, gamma 4,
// 8437 tokens 84.5 -> 93.7 us.
// Nor do chunks of fewer than 8 tiles pay where they make more workgroups than there are
// CUs, whose fixed cost is several tiles: at d = 128 there are no more chunks then than a
// round of full-size workgroups holds.  Packed, 40 heads, gamma 2, 537 + 515 tokens 51.8
// -> 41.5 us (3 chunks -> 1), ten up to 493 tokens, 16 heads 50.5 -> 41.6 us (2 -> 1); 8
// heads, gamma 7, 4776 tokens 81.8 -> 65.1 us; with d = 64 included 0.91-1.06 there.
// nC drops only when the partial results would pass kPartialBudget, or, with a nonzero
// `limit`, until the whole workspace fits `limit` bytes (false when even one
// chunk does not).  long_chunks: chunks of at least kLongChunk tiles whatever
// the launch fills (the least workspace a call takes).
bool make_plan(int B, int max_seqlen, int Hq, int Hkv, int d, int gamma, Plan* p, size_t limit,
               bool long_chunks) {
  if (B < 1 || max_seqlen < 1 || Hq < 1 || Hkv < 1 || gamma < 1 || (d != 64 && d != 128))
    return false;
  if (Hq % Hkv != 0) return false;
  const int64_t nA_max = max_seqlen / gamma;
  const int64_t nR_max = nA_max + (int64_t)((gamma - 1 < max_seqlen) ? gamma - 1 : max_seqlen);
  constexpr int64_t kLongChunk = 40, kShortChunk = 2, kFewTiles = 8;  // tiles
  const int64_t work = strided_tiles(B, max_seqlen, Hq, Hq / Hkv, gamma, nR_max - nA_max);
  const int64_t places = B == 1 ? kCUs : kCUs * 3 / 2;
  int64_t min_tiles = (work + places - 1) / places;
  min_tiles = min_tiles < kShortChunk ? kShortChunk : min_tiles > kLongChunk ? kLongChunk : min_tiles;
  // (every chunk writes a partial per row, and the merge reads it)
  const int64_t row_bytes = (int64_t)(d + 2) * 4, per_chunk_anchors = (int64_t)B * Hq * nA_max * row_bytes;
  const int64_t n_long = (max_seqlen + kKeyTile * kLongChunk - 1) / (kKeyTile * kLongChunk);
  const int64_t long_tiles = ((max_seqlen + n_long - 1) / n_long + kKeyTile - 1) / kKeyTile;
  if (per_chunk_anchors >= (int64_t)12500000 * 128 / d && work * 100 >= long_tiles * kCUs * 65)
    min_tiles = kLongChunk;
  constexpr int64_t one = 448;  // keys
  const int64_t min_keys = long_chunks ? kKeyTile * kLongChunk
                           : max_seqlen <= one ? one : kKeyTile * min_tiles;
  int64_t nC = (max_seqlen + min_keys - 1) / min_keys;
  if (nC > 16) nC = 16;
  if (nC < 1) nC = 1;
  if (d == 128 && !long_chunks) {
    // (full-size workgroups of one chunk; sequences of a batch have half the tail)
    const int hpw = heads_per_block(Hq / Hkv);
    const int64_t rpb = kRowsPerWave * (kAttnWaves / hpw);
    const int64_t rows = B == 1 ? nR_max : (nA_max + nR_max + 1) / 2;
    const int64_t blocks = (int64_t)B * (Hq / hpw) * ((rows + rpb - 1) / rpb);
    while (nC > n_long && nC * blocks > kCUs && max_seqlen < nC * kKeyTile * kFewTiles) --nC;
  }
  const int64_t per_chunk_bytes = (int64_t)B * Hq * nR_max * row_bytes;
  while (nC > 1 && per_chunk_bytes * nC > kPartialBudget) --nC;
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  auto fill = [&](int64_t want) {
    int64_t chunk = (max_seqlen + want - 1) / want;
    chunk = (chunk + kKeyTile - 1) / kKeyTile * kKeyTile;
    const int64_t n = (max_seqlen + chunk - 1) / chunk;
    p->nA_max = (int)nA_max;
    p->nR_max = (int)nR_max;
    p->nC = (int)n;
    p->chunk = (int)chunk;
    p->finer = n > (max_seqlen + kKeyTile * kLongChunk - 1) / (kKeyTile * kLongChunk);
    p->sa_floats = (size_t)B * Hq * nR_max * d;  // sparse anchor rows, or merged dense rows
    p->part_o_floats = (size_t)B * Hq * nR_max * n * d;
    p->part_ml_floats = (size_t)B * Hq * nR_max * n * 2;
    p->bytes = up(p->sa_floats * 4) + up(p->part_o_floats * 4) + up(p->part_ml_floats * 4);
  };
  fill(nC);
  while (limit && p->bytes > limit && p->nC > 1) fill(p->nC - 1);
  return !limit || p->bytes <= limit;
}

size_t correction_floats(int B, int max_seqlen, int Hq, int d, int gamma, int mode) {
  if (mode < 2 || gamma < 1) return 0;
  const size_t per = (size_t)B * Hq * (size_t)(max_seqlen / gamma) * d;
  return mode == 3 ? 2 * per : per;
}

namespace {

struct Problem {
  const void *q, *k, *v;
  void* out;
  const int32_t* cu;
  int B, N, Hq, Hkv, d;
  int window, n_sink, gamma;
  // key-block lists (nullptr: sink + window attention)
  const int32_t* blk_ptr = nullptr;
  const int32_t* blk_idx = nullptr;
  int block_q = 0;
};

// Rows per query head of one sparse workgroup; with key-block lists they must
// fit one query block.
int slab_rows(int hpw) { return kRowsPerWave * (kAttnWaves / hpw); }

// Shape/parameter checks shared by all calls; no HIP call happens here.
da_status validate(const Problem& P, bool need_window, bool need_gamma) {
  if (!P.q || !P.k || !P.v || !P.out) return DA_ERR_NULL;
  if (P.B < 1 || P.N < 1 || P.Hq < 1 || P.Hkv < 1 || P.Hq % P.Hkv != 0) return DA_ERR_SHAPE;
  if (need_window && (P.window < 1 || P.n_sink < 0)) return DA_ERR_PARAM;
  if (need_gamma && P.gamma < 1) return DA_ERR_PARAM;
  if (P.d != 64 && P.d != 128) return DA_ERR_UNSUPPORTED;
  // token indices and row-tile counts are 32-bit inside the kernels
  if (!P.cu && (int64_t)P.B * P.N > INT32_MAX) return DA_ERR_SHAPE;
  const int hpw = heads_per_block(P.Hq / P.Hkv);
  const int64_t rows_per_block = (int64_t)kRowsPerWave * (kAttnWaves / hpw);
  const int64_t blocks = (int64_t)P.B * (P.Hq / hpw) * ((P.N + rows_per_block - 1) / rows_per_block);
  if (blocks > INT32_MAX) return DA_ERR_SHAPE;
  if (P.blk_ptr || P.blk_idx) {
    if (!P.blk_ptr || !P.blk_idx) return DA_ERR_NULL;
    if (P.block_q != 64 && P.block_q != 128 && P.block_q != 256) return DA_ERR_PARAM;
    if (slab_rows(hpw) > P.block_q) return DA_ERR_UNSUPPORTED;
    if ((int64_t)P.B * P.Hkv * ((int64_t)(P.N + P.block_q - 1) / P.block_q + 1) > INT32_MAX)
      return DA_ERR_SHAPE;
  }
  if (!aligned16(P.q) || !aligned16(P.k) || !aligned16(P.v) || !aligned16(P.out))
    return DA_ERR_ALIGN;
  return DA_OK;
}

enum class Launch { kSparseRows, kDenseCausal, kStridedRows };
// Keys of a row under key-block lists, as a typical guess: the lists are on the device.
constexpr int64_t kListKeys = 2048;

// Wavefronts per attention workgroup: kAttnWaves, or half of them.  `blocks` is
// the launch in 8-wave workgroups, `work` its tiles in units of the longest of
// them, `keys` the keys of a sparse row, `shape` how long the workgroups are and how
// they come.  Outputs are bitwise the same either way: a wavefront runs the same rows
// over the same tiles.
//
// Half-size workgroups fit a CU twice at d = 128 (registers: one wavefront per
// SIMD each), so that one's first loads and last stores run beside the other's
// tiles, and spread a small launch over more CUs; each K/V tile then serves
// 128 rows instead of 256, which costs a long launch 2-4 % in L2 traffic and
// power.  At d = 64 three fit (12 wavefronts per CU in place of 8), which
// always pays.  Measured on an MI355X, 8 -> 4 wavefronts:
//   d = 64: 16-head sparse rows, window 1024, 38K tokens 282 -> 223 us; Delta
//     prefill 131K tokens, 32 heads 6.01 -> 5.34 ms; dense 16K 1.16 -> 1.06 ms;
//   d = 128, less work than the CUs hold: dense 512-2048 tokens, 32 heads
//     18.7 -> 14.3 and 52.1 -> 45.4 us, 3000 tokens 78.2 -> 75.5 us (0.73
//     rounds of the CUs), 4096 tokens 123 -> 134 us (1.0); sparse, window 2048,
//     2500 tokens 74.6 -> 69.5 us (0.7), 3000 tokens 88 -> 95 us (0.95);
//   d = 128, few keys per row (the fixed cost of a workgroup then outweighs its
//     tiles), 32K tokens, 32 heads, 64 sinks: window 64 200 -> 183 us, 256
//     275 -> 261 us, 512 383 -> 377 us, 1024 593 -> 599 us; with 8 heads (one
//     per workgroup, whose 256 rows reach further past the window) 1024
//     161 -> 156 us, 1536 215 -> 214 us, 2048 265 -> 268 us;
//   d = 128, window 2048, a few rounds of the CUs: where the last round leaves
//     many places, half-size workgroups share them better.  Uneven workgroups
//     (32 heads, whole call, rounds by work): 4021 tokens 135.7 -> 128.4 us
//     (1.46), 6000 tokens 201 -> 196 us (2.42), but 3500 tokens 111 -> 114 us
//     (1.2), 5000 tokens 153 -> 160 us (1.95).  Even ones (8 heads, rounds by
//     workgroups): 11264 tokens 120 -> 106 us (1.4), 13312 121 -> 110 us (1.6),
//     17408 150 -> 144 us (2.1), but 8192 63 -> 69 us (1.0), 15360 126 -> 132 us
//     (1.9);
//   d = 128, strided rows up to 1.4 rounds: 16384 tokens, gamma 64 220 -> 211 us
//     (0.8), 8 heads, gamma 32, 32768 tokens 208 -> 188 us (1.0); past it even
//     workgroups, of which half a round may be left: 64 heads, gamma 32, 14848
//     tokens 314 -> 322 us (1.53), 32 heads, 49945 tokens 1314 -> 1334 us (3.7).
//   d = 128, flat work below a round of the CUs, whose full-size workgroups all run at
//     once: a CU that gets two half-size ones takes as long as with a full-size one, so
//     they pay only while most CUs get one.  Sparse rows: 7791 tokens, 4 heads on 1 (0.41)
//     54.7 -> 45.4 us, 9729, 4 on 2, window 1600 (0.55) 46.6 -> 46.0 us, 6390, 8 heads
//     (0.65) 59.8 -> 64.0 us, 12800, 4 on 2, window 4096 (0.65) 104 -> 115 us, 7725, 8 on
//     4 (0.82) 64.2 -> 68.7 us; but 11382, 6 on 2, window 1600, 270 workgroups of eight
//     (0.98) 76.4 -> 62.5 us;
//   d = 128, uneven work of 16 head groups, of which each XCD runs the second after the
//     first, so that the long half-size workgroups of the one meet those of the other:
//     from 14 row tiles per head on.  Dense, 16 kv heads: 766 tokens, 64 heads (12) 24.7
//     -> 22.0 us, 3277, 16 heads (13) 74.9 us both, 3361 (14) 76.2 -> 78.8 us, 4243 (17) 95.9
//     -> 110 us, 1232, 64 heads (20) 35.8 -> 39.0 us, 2988, 32 heads (24) 0.92 of the time;
//     with four or more groups in turn neither size is the better one throughout.
struct Shape {
  bool even = false;     // nearly all workgroups are as long as the longest
  bool flat = false;     // most are
  bool in_turn = false;  // each XCD runs two head groups one after the other
  bool shared = false;   // another launch's workgroups fill what it leaves, or some of
                         // those counted are empty (packed sequences)
};
int attn_waves(Launch kind, int d, int heads, int64_t blocks, int64_t work, int64_t keys,
               Shape shape) {
  constexpr int kHalf = kAttnWaves / 2;
  if (d == 64) return kHalf;
  if (kind == Launch::kSparseRows && keys <= (heads == 1 ? 1600 : 600)) return kHalf;
  // flat work of full-size workgroups that all run at once
  const bool at_once = shape.flat && blocks <= kCUs && !shape.shared;
  if (!shape.flat && shape.in_turn && blocks * 8 >= kCUs * 7 && work < kCUs) return kAttnWaves;
  if (work * 5 < kCUs * (at_once ? 3 : 4) || (kind == Launch::kStridedRows && work <= kCUs * 11 / 8)) return kHalf;
  if (at_once) return kAttnWaves;
  if (work > 4 * kCUs || kind == Launch::kDenseCausal) return kAttnWaves;
  const int64_t part = (shape.even ? blocks : work) % kCUs * 100 / kCUs;  // of a round, in hundredths
  const int64_t least = shape.even ? 1 : 28, most = kind == Launch::kStridedRows ? 50 : 72;
  return part >= least && part <= most ? kHalf : kAttnWaves;
}

Shape shape_of(const Problem& P, int heads, bool even, bool flat, bool shared) {
  shared |= P.cu && P.B > 1;
  // (the order of the head groups: see prepare_attn; of eight heads each, whose half-size
  // workgroups take four, neither size is the better one)
  return {even, flat, !shared && heads < 8 && P.Hq / heads == 16 && P.Hkv % 16 == 0, shared};
}

// Tiling of a launch over `rows` rows per (sequence, head) by workgroups of
// `waves` wavefronts and `hpw` heads.
void set_tiling(Args& a, int waves, int hpw, int rows) {
  a.hpw = hpw;
  a.ppw = waves / hpw;
  a.n_hgroups = a.Hq / hpw;
  const int rpb = kRowsPerWave * a.ppw;
  a.n_rtiles = (int)(((int64_t)rows + rpb - 1) / rpb);
}

// Full-size workgroups of a launch over every row.
int64_t full_blocks(const Problem& P, int hpw) {
  const int64_t rpb = kRowsPerWave * (kAttnWaves / hpw);
  return (int64_t)P.B * (P.Hq / hpw) * ((P.N + rpb - 1) / rpb);
}

// Tiles the sparse launch; in the fused schedule gamma and the list blocks bind
// the row slab.  shared: it may run together with the strided rows.
void tile_sparse(Args& a, const Problem& P, bool fused, bool shared) {
  const int G = P.Hq / P.Hkv;
  const int max_rows = P.blk_ptr ? P.block_q : INT32_MAX;
  auto heads = [&](int waves) {
    return fused ? fused_heads_per_block(G, P.gamma, max_rows, waves) : heads_per_block(G, waves);
  };
  const int h8 = heads(kAttnWaves);
  const int64_t keys = P.blk_ptr ? kListKeys : (int64_t)P.window + P.n_sink;
  // rows before a whole key set grow with their position
  const int64_t blocks = full_blocks(P, h8);
  const int64_t ramp = keys < P.N ? keys : P.N;
  const int64_t work = blocks * (2 * (int64_t)P.N - ramp) / (2 * (int64_t)P.N);
  const Shape shape = shape_of(P, h8, P.N >= 4 * keys, (int64_t)P.N * 5 >= keys * 14, shared);
  int waves = attn_waves(Launch::kSparseRows, P.d, h8, blocks, work, keys, shape);
  // Two half-size workgroups share a CU's 160 KB of LDS only if each stages at most
  // 16 KB of dense rows beside its 64 KB ring: 128 / gamma rows of 512 bytes at
  // d = 128, so not at gamma 2 (3 does not divide a slab).  There they pay only while
  // each has a CU to itself.  Whole calls, gamma 2, window 512, 32 heads, 8 -> 4
  // wavefronts: 1000 tokens 54.2 -> 48.4 us (128 workgroups of eight), 1500 tokens
  // 64.1 -> 69.6 us (192; window 1024, 125 by work, 73.2 -> 64.9 us), 4096 tokens
  // 163 -> 185 us, 40000 tokens 7.30 -> 7.67 ms.
  const bool alone = fused && P.d == 128 && P.gamma > 1 && P.gamma < 4;
  if (alone && work * 2 > kCUs) waves = kAttnWaves;
  // (a slab of half the rows may hold no whole group)
  if (heads(waves) == 0) waves = kAttnWaves;
  set_tiling(a, waves, heads(waves), P.N);
}

int64_t sparse_blocks(const Args& a) { return (int64_t)a.B * a.n_hgroups * a.n_rtiles; }
int64_t strided_blocks(const Args& a) { return sparse_blocks(a) * a.nC; }

// Tiles the dense causal launch.
void tile_dense(Args& a, const Problem& P) {
  const int G = P.Hq / P.Hkv;
  const int h8 = heads_per_block(G);
  const int64_t work = full_blocks(P, h8) / 2;
  const Shape shape = shape_of(P, h8, false, false, false);
  const int waves = attn_waves(Launch::kDenseCausal, P.d, h8, 2 * work, work, 0, shape);
  set_tiling(a, waves, heads_per_block(G, waves), P.N);
}

// Strided workgroups of `waves` wavefronts that have a key to look at, in one
// sequence of P.N tokens.
int64_t strided_with_keys(const Problem& P, const Plan& plan, int64_t tail, int waves) {
  const int hpw = heads_per_block(P.Hq / P.Hkv, waves);
  const int64_t rpb = kRowsPerWave * (waves / hpw), rows = plan.nA_max + tail;
  int64_t n = 0;
  for (int64_t r0 = 0; r0 < rows; r0 += rpb) {
    const int64_t last = (r0 + rpb < rows ? r0 + rpb : rows) - 1;
    n += ((last < plan.nA_max ? last * P.gamma + 1 : P.N) + plan.chunk - 1) / plan.chunk;
  }
  return n * (P.Hq / hpw);
}

// Tiles the strided dense rows: nR_max rows, nC chunks of `chunk` keys.
// sparse_waves: of the sparse rows' workgroups, 0 where those run by themselves.
// Up to 1.4 rounds of the CUs, where attn_waves takes half-size workgroups:
//  - next to sparse rows of full-size workgroups they take full-size ones as well,
//    which lets one launch run both (moving average, 32 heads, 9000 tokens 253 -> 225
//    us; gamma 48, 12 heads, 7194 tokens 154 -> 130 us, 8 heads, 35539 429 -> 377 us);
//  - so they do where the full-size ones run all at once and the half-size ones would
//    share the CUs, as in attn_waves (2 heads, gamma 64, 175872 tokens 429 -> 378 us; 8
//    heads, gamma 2, 7036 tokens 134 -> 127 us).
void tile_strided(Args& a, const Problem& P, const Plan& plan, int sparse_waves) {
  const int G = P.Hq / P.Hkv;
  const int64_t tail = P.cu ? (int64_t)plan.nR_max - plan.nA_max : P.N % P.gamma;
  const int64_t work = strided_tiles(P.B, P.N, P.Hq, G, P.gamma, tail) / (plan.chunk / kKeyTile);
  Shape shape;
  shape.even = true;
  int waves = attn_waves(Launch::kStridedRows, P.d, heads_per_block(G), work, work, 0, shape);
  if (P.d == 128 && work <= kCUs * 11 / 8) {
    if (sparse_waves)
      waves = sparse_waves;
    else if (P.B * strided_with_keys(P, plan, tail, kAttnWaves) <= kCUs &&
             P.B * strided_with_keys(P, plan, tail, kAttnWaves / 2) * 5 > kCUs * 6)
      waves = kAttnWaves;
  }
  set_tiling(a, waves, heads_per_block(G, waves), plan.nR_max);
}

// Whether the unfused schedule runs the sparse rows `as` and the strided rows `ar`
// in one launch: up to 40 rounds of the CUs (where it pays: see attn_pair_kernel)
// and where they take workgroups of one size.
bool paired(const Args& as, const Args& ar) {
  return as.hpw * as.ppw == ar.hpw * ar.ppw &&
         sparse_blocks(as) * as.hpw * as.ppw <= 40 * kCUs * kAttnWaves &&
         strided_blocks(ar) < INT32_MAX / 2;
}

Args base_args(const Problem& P) {
  Args a;
  memset(&a, 0, sizeof a);
  a.q = (const uint16_t*)P.q;
  a.k = (const uint16_t*)P.k;
  a.v = (const uint16_t*)P.v;
  a.out = (uint16_t*)P.out;
  a.cu = P.cu;
  a.B = P.B;
  a.N = P.N;
  a.Hq = P.Hq;
  a.Hkv = P.Hkv;
  a.d = P.d;
  a.window = P.window;
  a.n_sink = P.n_sink;
  a.cover = (int64_t)P.n_sink + P.window;
  if (P.blk_ptr) {
    // the key set is the lists' tiles plus the own query block's, masked
    // causally: no sink/window test applies, and no anchor is known covered
    a.blk_ptr = P.blk_ptr;
    a.blk_idx = P.blk_idx;
    a.block_q = P.block_q;
    a.nqb = (P.N + P.block_q - 1) / P.block_q;
    a.n_sink = INT32_MAX;
    a.window = 1;
    a.cover = 0;
  }
  a.gamma = P.gamma > 0 ? P.gamma : 1;
  a.scale_log2 = (float)(1.4426950408889634 / sqrt((double)P.d));
  a.head_chunk = 8192 / P.d;
  return a;
}

da_status run_plain(const Problem& P, bool sparse, void* stream) {
  da_status st = validate(P, sparse, false);
  if (st != DA_OK) return st;
  st = check_device();
  if (st != DA_OK) return st;
  Args a = base_args(P);
  if (sparse)
    tile_sparse(a, P, false, false);
  else
    tile_dense(a, P);
  hipError_t e = sparse ? launch_sparse(a, (hipStream_t)stream) : launch_dense(a, (hipStream_t)stream);
  if (e != hipSuccess) return fail_hip(e);
  return DA_OK;
}

// Launch sequence of the Delta path.  Unfused schedule: sparse kernel (plus
// the fp32 sparse rows at anchors), strided dense rows, then the epilogue
// that merges them, forms Delta and adds it to `out` in place.  Fused
// schedule (when every group of gamma rows fits one head slab of a sparse
// workgroup, and for the Delta and recompute corrections only): strided
// dense rows, the merge into fp32 dense rows, then the sparse kernel storing
// the corrected rows.  `steps` without DA_STEP_FUSED picks the unfused
// schedule; `auto_fuse` lets the whole-path calls take the fused one.
da_status run_delta(const Problem& P, void* workspace, size_t workspace_bytes, void* stream,
                    unsigned steps, bool auto_fuse, int corr_mode = 0, float p0 = 0.f,
                    float p1 = 0.f, float p2 = 0.f, bool scratch = false) {
  da_status st = validate(P, true, true);
  if (st != DA_OK) return st;
  if ((steps & DA_STEP_ALL) == 0u || steps > (DA_STEP_ALL | DA_STEP_FUSED)) return DA_ERR_PARAM;
  if (corr_mode < DA_CORR_DELTA || corr_mode > DA_CORR_ABG) return DA_ERR_PARAM;
  if (!std::isfinite(p0) || !std::isfinite(p1) || !std::isfinite(p2)) return DA_ERR_PARAM;
  if (corr_mode == DA_CORR_EMA && (p0 < 0.f || p0 > 1.f)) return DA_ERR_PARAM;
  const int fhpw = fused_heads_per_block(P.Hq / P.Hkv, P.gamma, P.blk_ptr ? P.block_q : INT32_MAX);
  const bool can_fuse = fhpw > 0 && corr_mode <= DA_CORR_RECOMPUTE;
  if ((steps & DA_STEP_FUSED) && !can_fuse) return DA_ERR_UNSUPPORTED;
  const bool fused = (steps & DA_STEP_FUSED) || (auto_fuse && can_fuse);
  Plan plan;
  if (!make_plan(P.B, P.N, P.Hq, P.Hkv, P.d, P.gamma, &plan)) return DA_ERR_SHAPE;
  if (scratch) {
    // the static scratch array: as many key chunks as fit it
    if (!make_plan(P.B, P.N, P.Hq, P.Hkv, P.d, P.gamma, &plan, kScratchBytes))
      return DA_ERR_WORKSPACE;
  } else {
    const size_t extra = correction_floats(P.B, P.N, P.Hq, P.d, P.gamma, corr_mode) * 4;
    if (!workspace) return DA_ERR_WORKSPACE;
    if (workspace_bytes < plan.bytes + extra) {
      // Short sequences may want more chunks, and a larger workspace, than longer
      // ones.  A workspace that holds the plan with long chunks only (one laid out
      // for the longest sequence of a serving loop, say) takes as many as fit it.
      // So does one that a longer sequence's plan may fill where kPartialBudget
      // holds that to fewer chunks, n < plan.nC of them: then n + 1 chunks of its
      // rows pass the budget, and n with the d fp32 values per row beside them take
      // (n + d / (d + 2)) / (n + 1) of it at the least, which is smallest at n = 1.
      // Calls that pass partials from one to the other take the long chunks then,
      // so that calls given different sizes agree on the layout.
      Plan least;
      if (!make_plan(P.B, P.N, P.Hq, P.Hkv, P.d, P.gamma, &least, 0, true)) return DA_ERR_WORKSPACE;
      const unsigned both = DA_STEP_DENSE_ROWS | DA_STEP_CORRECT;
      const bool passed_on = (steps & both) != 0u && (steps & both) != both;
      const size_t longer = (size_t)(kPartialBudget / (P.d + 2) * (P.d + 1));
      const size_t floor = passed_on || least.bytes < longer ? least.bytes : longer;
      if (workspace_bytes < floor + extra) return DA_ERR_WORKSPACE;
      if (passed_on)
        plan = least;
      else if (!make_plan(P.B, P.N, P.Hq, P.Hkv, P.d, P.gamma, &plan, workspace_bytes - extra))
        return DA_ERR_WORKSPACE;
    }
    if (!aligned16(workspace)) return DA_ERR_ALIGN;
  }
  {
    const int hpw = heads_per_block(P.Hq / P.Hkv);
    const int64_t rows_per_block = (int64_t)kRowsPerWave * (kAttnWaves / hpw);
    const int64_t rtiles = (plan.nR_max + rows_per_block - 1) / rows_per_block;
    if ((int64_t)P.B * (P.Hq / hpw) * plan.nC * rtiles > INT32_MAX) return DA_ERR_SHAPE;
    if ((int64_t)P.B * plan.nR_max * ((P.Hq + 8192 / P.d - 1) / (8192 / P.d)) > INT32_MAX)
      return DA_ERR_SHAPE;
    if (fused) {
      const int64_t frows = (int64_t)kRowsPerWave * (kAttnWaves / fhpw);
      if ((int64_t)P.B * (P.Hq / fhpw) * ((P.N + frows - 1) / frows) > INT32_MAX)
        return DA_ERR_SHAPE;
    }
  }
  st = check_device();
  if (st != DA_OK) return st;
  if (scratch) {
    // this device's copy of the static array (its address is looked up once
    // per device, with the device current)
    const hipError_t e = scratch_address(g_cur_dev, &workspace);
    if (e != hipSuccess) return fail_hip(e);
  }

  Args a = base_args(P);
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  char* ws = (char*)workspace;
  a.sa = (float*)ws;
  a.part_o = (float*)(ws + up(plan.sa_floats * 4));
  a.part_ml = (float*)(ws + up(plan.sa_floats * 4) + up(plan.part_o_floats * 4));
  a.nA_max = plan.nA_max;
  a.nR_max = plan.nR_max;
  a.nC = plan.nC;
  a.chunk = plan.chunk;
  a.split_ref = plan.finer;
  a.corr_mode = corr_mode;
  a.corr_p[0] = p0;
  a.corr_p[1] = p1;
  a.corr_p[2] = p2;
  if (corr_mode >= DA_CORR_INTERP) {
    a.dbuf = (float*)(ws + plan.bytes);
    a.ebuf = a.dbuf + (size_t)P.B * P.Hq * (size_t)plan.nA_max * P.d;
  }
  hipStream_t s = (hipStream_t)stream;

  hipError_t e = hipSuccess;
  if (fused) {
    a.dense = a.sa;
    a.fuse = corr_mode == DA_CORR_RECOMPUTE ? 2 : 1;
    // One key chunk has nothing to merge: with both steps asked for, the strided
    // kernel writes the dense rows beside their partials (the merge's arithmetic,
    // one launch less: 300 tokens, 32 heads, gamma 64 25.4 -> 24.5 us).  The partials
    // stay for a later call that asks for the merge alone.
    const unsigned both = DA_STEP_DENSE_ROWS | DA_STEP_CORRECT;
    const bool direct = plan.nC == 1 && (steps & both) == both;
    if (steps & DA_STEP_DENSE_ROWS) {
      Args ar = a;
      tile_strided(ar, P, plan, 0);
      ar.merged = direct;
      e = launch_dense_rows(ar, s);
      if (e != hipSuccess) return fail_hip(e);
    }
    if ((steps & DA_STEP_CORRECT) && !direct) {
      e = launch_delta_epilogue(a, s);
      if (e != hipSuccess) return fail_hip(e);
    }
    if (steps & DA_STEP_SPARSE) {
      Args as = a;
      tile_sparse(as, P, true, false);
      e = launch_sparse(as, s);
      if (e != hipSuccess) return fail_hip(e);
    }
    return DA_OK;
  }
  Args as = a, ar = a;
  tile_sparse(as, P, false, true);
  tile_strided(ar, P, plan, as.hpw * as.ppw);
  const unsigned both = DA_STEP_SPARSE | DA_STEP_DENSE_ROWS;
  const bool pair = (steps & both) == both && paired(as, ar);
  if (pair) as.rows = &ar;
  // Step 1: sparse attention for every row (+ fp32 copy at anchors).
  if (steps & DA_STEP_SPARSE) {
    e = launch_sparse(as, s);
    if (e != hipSuccess) return fail_hip(e);
  }
  // Steps 2-3: dense attention at anchors and tail rows, key axis split in chunks.
  if ((steps & DA_STEP_DENSE_ROWS) && !pair) {
    e = launch_dense_rows(ar, s);
    if (e != hipSuccess) return fail_hip(e);
  }
  // Steps 4-5: merge, Delta, broadcast-add in place (or the chosen variant).
  if (steps & DA_STEP_CORRECT) {
    e = launch_delta_epilogue(a, s);
    if (e != hipSuccess) return fail_hip(e);
    e = launch_correction(a, s);
    if (e != hipSuccess) return fail_hip(e);
  }
  return DA_OK;
}

}  // namespace
}  // namespace da

using da::Problem;

extern "C" {

da_status delta_attn_prefill(const void* q, const void* k, const void* v, void* out, int B,
                             int Hq, int Hkv, int N, int d, int window, int n_sink, int gamma,
                             void* workspace, size_t workspace_bytes, void* stream) {
  Problem P{q, k, v, out, nullptr, B, N, Hq, Hkv, d, window, n_sink, gamma};
  return da::run_delta(P, workspace, workspace_bytes, stream, DA_STEP_ALL, true);
}

da_status delta_attn_prefill_varlen(const void* q, const void* k, const void* v, void* out,
                                    const int32_t* cu_seqlens, int B, int max_seqlen, int Hq,
                                    int Hkv, int d, int window, int n_sink, int gamma,
                                    void* workspace, size_t workspace_bytes, void* stream) {
  if (!cu_seqlens) return DA_ERR_NULL;
  Problem P{q, k, v, out, cu_seqlens, B, max_seqlen, Hq, Hkv, d, window, n_sink, gamma};
  return da::run_delta(P, workspace, workspace_bytes, stream, DA_STEP_ALL, true);
}

da_status delta_attn_prefill_steps(const void* q, const void* k, const void* v, void* out,
                                   const int32_t* cu_seqlens, int B, int max_seqlen, int Hq,
                                   int Hkv, int d, int window, int n_sink, int gamma,
                                   void* workspace, size_t workspace_bytes, void* stream,
                                   unsigned steps) {
  Problem P{q, k, v, out, cu_seqlens, B, max_seqlen, Hq, Hkv, d, window, n_sink, gamma};
  return da::run_delta(P, workspace, workspace_bytes, stream, steps, false);
}

da_status delta_attn_prefill_correction(const void* q, const void* k, const void* v, void* out,
                                        const int32_t* cu_seqlens, int B, int max_seqlen, int Hq,
                                        int Hkv, int d, int window, int n_sink, int gamma,
                                        int mode, float p0, float p1, float p2, void* workspace,
                                        size_t workspace_bytes, void* stream) {
  Problem P{q, k, v, out, cu_seqlens, B, max_seqlen, Hq, Hkv, d, window, n_sink, gamma};
  return da::run_delta(P, workspace, workspace_bytes, stream, DA_STEP_ALL, true, mode, p0, p1,
                       p2);
}

da_status delta_attn_prefill_noalloc(const void* q, const void* k, const void* v, void* out,
                                     const int32_t* cu_seqlens, int B, int max_seqlen, int Hq,
                                     int Hkv, int d, int window, int n_sink, int gamma,
                                     void* stream) {
  Problem P{q, k, v, out, cu_seqlens, B, max_seqlen, Hq, Hkv, d, window, n_sink, gamma};
  return da::run_delta(P, nullptr, 0, stream, DA_STEP_ALL, true, 0, 0.f, 0.f, 0.f, true);
}

size_t da_workspace_bytes_correction(int B, int max_seqlen, int Hq, int Hkv, int d, int gamma,
                                     int mode) {
  da::Plan p;
  if (mode < DA_CORR_DELTA || mode > DA_CORR_ABG) return 0;
  if (!da::make_plan(B, max_seqlen, Hq, Hkv, d, gamma, &p)) return 0;
  return p.bytes + da::correction_floats(B, max_seqlen, Hq, d, gamma, mode) * 4;
}

da_status sparse_attn_prefill(const void* q, const void* k, const void* v, void* out, int B,
                              int Hq, int Hkv, int N, int d, int window, int n_sink,
                              void* stream) {
  Problem P{q, k, v, out, nullptr, B, N, Hq, Hkv, d, window, n_sink, 1};
  return da::run_plain(P, true, stream);
}

da_status sparse_attn_prefill_varlen(const void* q, const void* k, const void* v, void* out,
                                     const int32_t* cu_seqlens, int B, int max_seqlen, int Hq,
                                     int Hkv, int d, int window, int n_sink, void* stream) {
  if (!cu_seqlens) return DA_ERR_NULL;
  Problem P{q, k, v, out, cu_seqlens, B, max_seqlen, Hq, Hkv, d, window, n_sink, 1};
  return da::run_plain(P, true, stream);
}

da_status dense_causal_attn_prefill(const void* q, const void* k, const void* v, void* out,
                                    int B, int Hq, int Hkv, int N, int d, void* stream) {
  Problem P{q, k, v, out, nullptr, B, N, Hq, Hkv, d, 1, 0, 1};
  return da::run_plain(P, false, stream);
}

da_status dense_causal_attn_prefill_varlen(const void* q, const void* k, const void* v,
                                           void* out, const int32_t* cu_seqlens, int B,
                                           int max_seqlen, int Hq, int Hkv, int d,
                                           void* stream) {
  if (!cu_seqlens) return DA_ERR_NULL;
  Problem P{q, k, v, out, cu_seqlens, B, max_seqlen, Hq, Hkv, d, 1, 0, 1};
  return da::run_plain(P, false, stream);
}

int da_fused_supported(int Hq, int Hkv, int gamma) {
  if (Hq < 1 || Hkv < 1 || Hq % Hkv != 0 || gamma < 1) return 0;
  return da::fused_heads_per_block(Hq / Hkv, gamma, INT32_MAX) > 0 ? 1 : 0;
}

int da_fused_supported_blocksparse(int Hq, int Hkv, int gamma, int block_q) {
  if (Hq < 1 || Hkv < 1 || Hq % Hkv != 0 || gamma < 1) return 0;
  if (block_q != 64 && block_q != 128 && block_q != 256) return 0;
  return da::fused_heads_per_block(Hq / Hkv, gamma, block_q) > 0 ? 1 : 0;
}

da_status blocksparse_attn_prefill(const void* q, const void* k, const void* v, void* out,
                                   const int32_t* cu_seqlens, int B, int max_seqlen, int Hq,
                                   int Hkv, int d, int block_q, const int32_t* block_ptr,
                                   const int32_t* block_idx, void* stream) {
  Problem P{q, k, v, out, cu_seqlens, B, max_seqlen, Hq, Hkv, d, 1, 0, 1};
  P.blk_ptr = block_ptr;
  P.blk_idx = block_idx;
  P.block_q = block_q;
  if (!block_ptr || !block_idx) return DA_ERR_NULL;
  return da::run_plain(P, true, stream);
}

da_status delta_attn_prefill_blocksparse(const void* q, const void* k, const void* v, void* out,
                                         const int32_t* cu_seqlens, int B, int max_seqlen,
                                         int Hq, int Hkv, int d, int block_q,
                                         const int32_t* block_ptr, const int32_t* block_idx,
                                         int gamma, void* workspace, size_t workspace_bytes,
                                         void* stream, unsigned steps) {
  Problem P{q, k, v, out, cu_seqlens, B, max_seqlen, Hq, Hkv, d, 1, 0, gamma};
  P.blk_ptr = block_ptr;
  P.blk_idx = block_idx;
  P.block_q = block_q;
  if (!block_ptr || !block_idx) return DA_ERR_NULL;
  if (steps == 0u) return da::run_delta(P, workspace, workspace_bytes, stream, DA_STEP_ALL, true);
  return da::run_delta(P, workspace, workspace_bytes, stream, steps, false);
}

da_status da_launch_plan(int B, int max_seqlen, int Hq, int Hkv, int d, int gamma, int block_q,
                         da_plan* plan) {
  if (!plan) return DA_ERR_NULL;
  if (B < 1 || max_seqlen < 1 || Hq < 1 || Hkv < 1 || Hq % Hkv != 0) return DA_ERR_SHAPE;
  if (gamma < 1) return DA_ERR_PARAM;
  if (block_q != 0 && block_q != 64 && block_q != 128 && block_q != 256) return DA_ERR_PARAM;
  if (d != 64 && d != 128) return DA_ERR_UNSUPPORTED;
  da::Plan p;
  if (!da::make_plan(B, max_seqlen, Hq, Hkv, d, gamma, &p)) return DA_ERR_SHAPE;
  const int G = Hq / Hkv;
  const int hpw = da::heads_per_block(G);
  if (block_q && da::kRowsPerWave * (da::kAttnWaves / hpw) > block_q) return DA_ERR_UNSUPPORTED;
  const int fhpw = da::fused_heads_per_block(G, gamma, block_q ? block_q : INT32_MAX);
  plan->fused = fhpw > 0 ? 1 : 0;
  plan->sparse_heads = fhpw > 0 ? fhpw : hpw;
  plan->sparse_slab_rows = da::kRowsPerWave * (da::kAttnWaves / (fhpw > 0 ? fhpw : hpw));
  plan->rows_heads = hpw;
  plan->key_chunks = p.nC;
  plan->chunk_keys = p.chunk;
  plan->key_tile = da::kKeyTile;
  plan->rows_per_wave = da::kRowsPerWave;
  plan->waves_per_block = da::kAttnWaves;
  return DA_OK;
}

da_status da_launch_workgroups(int B, int max_seqlen, int packed, int Hq, int Hkv, int d,
                               int window, int n_sink, int gamma, int block_q, int mode,
                               da_workgroups* w) {
  if (!w) return DA_ERR_NULL;
  if (packed < 0 || packed > 1 || block_q < 0) return DA_ERR_PARAM;
  if (mode < DA_CORR_DELTA || mode > DA_CORR_ABG) return DA_ERR_PARAM;
  alignas(16) static const int32_t given[4] = {};  // stands for every tensor
  Problem P{given, given, given, const_cast<int32_t*>(given), packed ? given : nullptr, B,
            max_seqlen, Hq, Hkv, d, window, n_sink, gamma};
  if (block_q) P.blk_ptr = P.blk_idx = given;
  P.block_q = block_q;
  const da_status st = da::validate(P, true, true);
  if (st != DA_OK) return st;
  da::Plan plan;
  if (!da::make_plan(B, max_seqlen, Hq, Hkv, d, gamma, &plan)) return DA_ERR_SHAPE;
  const bool fused = mode <= DA_CORR_RECOMPUTE &&
                     da::fused_heads_per_block(Hq / Hkv, gamma, block_q ? block_q : INT32_MAX) > 0;
  da::Args as = da::base_args(P), ar, base, dense;
  as.nC = plan.nC;
  ar = base = dense = as;
  da::tile_sparse(as, P, fused, !fused);
  da::tile_strided(ar, P, plan, fused ? 0 : as.hpw * as.ppw);
  da::tile_sparse(base, P, false, false);
  da::tile_dense(dense, P);
  w->sparse_waves = as.hpw * as.ppw;
  w->sparse_heads = as.hpw;
  w->rows_waves = ar.hpw * ar.ppw;
  w->rows_heads = ar.hpw;
  w->together = !fused && da::paired(as, ar);
  w->base_waves = base.hpw * base.ppw;
  w->base_heads = base.hpw;
  w->dense_waves = dense.hpw * dense.ppw;
  w->dense_heads = dense.hpw;
  return DA_OK;
}

size_t da_workspace_bytes(int B, int max_seqlen, int Hq, int Hkv, int d, int gamma) {
  da::Plan p;
  if (!da::make_plan(B, max_seqlen, Hq, Hkv, d, gamma, &p)) return 0;
  return p.bytes;
}

da_status da_check_inputs(const int32_t* cu_seqlens, int B, int max_seqlen, int Hkv,
                          int block_q, const int32_t* block_ptr, const int32_t* block_idx,
                          int64_t block_nnz, int32_t* result, void* stream) {
  if (!result || (!cu_seqlens && !block_ptr)) return DA_ERR_NULL;
  if (B < 1 || max_seqlen < 1) return DA_ERR_SHAPE;
  int nqb = 0;
  if (block_ptr) {
    if (!block_idx && block_nnz > 0) return DA_ERR_NULL;
    if (Hkv < 1 || block_nnz < 0) return DA_ERR_SHAPE;
    if (block_q != 64 && block_q != 128 && block_q != 256) return DA_ERR_PARAM;
    nqb = (max_seqlen + block_q - 1) / block_q;
  }
  if (((uintptr_t)result & 3u) != 0) return DA_ERR_ALIGN;
  da_status st = da::check_device();
  if (st != DA_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  hipError_t e = da::launch_check_inputs(cu_seqlens, B, max_seqlen, block_ptr, block_idx,
                                         block_nnz, Hkv, nqb, result, s);
  if (e != hipSuccess) return da::fail_hip(e);
  int32_t host = 0;
  e = hipMemcpyAsync(&host, result, sizeof host, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return da::fail_hip(e);
  return host == 0 ? DA_OK : DA_ERR_PARAM;
}

const char* da_status_string(da_status s) {
  switch (s) {
    case DA_OK: return "DA_OK";
    case DA_ERR_NULL: return "DA_ERR_NULL";
    case DA_ERR_SHAPE: return "DA_ERR_SHAPE";
    case DA_ERR_PARAM: return "DA_ERR_PARAM";
    case DA_ERR_UNSUPPORTED: return "DA_ERR_UNSUPPORTED";
    case DA_ERR_ALIGN: return "DA_ERR_ALIGN";
    case DA_ERR_WORKSPACE: return "DA_ERR_WORKSPACE";
    case DA_ERR_HIP: return "DA_ERR_HIP";
  }
  return "DA_ERR_UNKNOWN";
}

int da_last_hip_error(void) { return da::g_last_hip_error; }

int da_abi_version(void) { return DA_ABI_VERSION; }

}  // extern "C"

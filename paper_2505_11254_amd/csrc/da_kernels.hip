// da_kernels.hip -- gfx950 (CDNA4) kernels of the Delta Attention prefill.
//
// Delta Attention (arXiv 2505.11254, Algorithm 1) runs three steps:
//   1. sparse attention A*V for every query (StreamingLLM sinks + window, or
//      key tiles from per-query-block lists for other sparse bases),
//   2. dense causal attention A~V for every gamma-th query row (Eq. 4),
//   3. Delta = A~V - (A*V) at those rows, added to the gamma rows each covers
//      (Eq. 6); rows after the last whole group are computed densely
//      (implementation-details appendix).
// Steps 1 and 2 and the dense causal baseline share one attention kernel
// template (`attn_body`); step 3 is `delta_epilogue_kernel`.  The fused
// schedule runs step 2 first, merges its dense rows (`merge_rows_kernel`), and
// lets the sparse kernel store sparse + Delta directly, which saves the
// in-place pass over the output.
//
// Tile core (one wavefront = 32 query rows, 64-key tiles, bf16 MFMA):
//   S^T[key][row] = K Q^T   with v_mfma_f32_32x32x16_bf16: A = K rows from
//                           LDS, B = the wave's Q rows held in registers;
//   P^T = exp2(S^T * log2(e)/sqrt(d) - m)   online softmax in fp32;
//   O^T[dim][row] += V^T P^T  A = V^T read from the row-major V tile with
//                           gfx950's transposing LDS reads, B = P^T taken
//                           straight from the S^T accumulator registers.
// With this orientation a lane owns one query row in every accumulator
// (lane % 32 = row), so the row max, the normaliser and the rescale of O
// stay in the lane apart from one exchange with lane ^ 32, and P never goes
// through LDS.  K/V tiles go through a ring of LDS buffers; the waves of a
// workgroup share every K/V tile between the query heads of one GQA group.
#include "da_internal.hpp"

#include <math.h>

#include <algorithm>
#include <atomic>

namespace da {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

enum Mode { kSparse = 0, kDense = 1, kDenseRows = 2 };
// Per-element masks of a partly visible key tile (tile classes 2..5).
enum MaskKind { kMaskCausal = 2, kMaskWindow = 3, kMaskBoth = 4, kMaskAll = 5 };

// LDS layout of one pipeline stage (bf16 elements): K and V tiles of 64 keys,
// both row-major [key][dim] with unpadded rows of 2*D bytes.  Tiles arrive by
// LDS DMA, which writes 1 KB contiguous per wave instruction, so bank
// conflicts are avoided by XOR-swizzling the 16-byte chunks of each row
// instead of padding it:
//   K: chunk c of key row r sits at c ^ kswz(r), which spreads the 16-byte
//      operand reads of 16 consecutive keys over all banks;
//   V: chunk c of key row r sits at c ^ vswz(r), which spreads the transposing
//      8-byte reads (four keys x sixteen dims per 16-lane group).
template <int D, int NW>
struct Lds {
  static constexpr int kElems = kKeyTile * D;
  static constexpr int vElems = kKeyTile * D;
  static constexpr int stageElems = kElems + vElems;
  static constexpr int kRegions = kKeyTile * D * 2 / 1024;  // 1 KB DMA regions per tile
  static constexpr int kRegionsPerWave = kRegions / NW;
  __device__ static constexpr int kswz(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
  __device__ static constexpr int vswz(int r) {
    return D == 128 ? ((r & 3) << 2) : (((r >> 1) & 1) << 2);
  }
};

struct Seq {
  int64_t base;  // first token row of the sequence
  int L;         // its length
};

__device__ __forceinline__ Seq seq_of(const Args& a, int b) {
  if (a.cu) {
    const int s0 = a.cu[b], s1 = a.cu[b + 1];
    return {s0, s1 - s0};
  }
  return {(int64_t)b * a.N, a.N};
}

// Workgroups are dispatched in order, round-robin over the 8 XCDs (block i ->
// XCD i % 8), each with its own L2.
//  - When the head groups split evenly over the XCDs, XCD x takes the
//    contiguous eighth [x*n/8, (x+1)*n/8) of the logical blocks, ordered head
//    groups outermost, then sequence, [key chunk,] row tile: whole head groups,
//    each with every sequence, so the XCDs get equal work and each streams its
//    own kv heads' keys and values through its L2 while neighbouring tiles
//    share them.  Where an eighth is whole kv heads, the head groups of one kv
//    head run innermost: the workgroups that read the same keys and values run
//    side by side.
//  - Otherwise all head groups run innermost, the kv heads in turn, so that
//    the round-robin keeps as few kv heads per XCD as their number allows, the
//    XCDs get equal work and the longest rows of all heads run first.  Against
//    chunks of 64 blocks per XCD, head groups outermost, in every mode, which
//    left XCDs idle where few blocks had work: dense causal, d 128, 32 heads on
//    4 kv heads, 16K tokens 2541 -> 1807 us, 20 on 4 1269 -> 1113 us; Delta, 8
//    heads on 4, packed prompts 4-22K tokens 445 -> 319 us; 8 heads on 2, 64K
//    tokens 771 -> 681 us.
//  - Sparse rows whose head groups are so few that the round-robin would put
//    kXcdSpread rows or more between an XCD's neighbouring slabs: XCD x takes the
//    logical chunks x, x+8, x+16, ... of `chunk` consecutive blocks, so that
//    slabs whose windows overlap stay on one L2 (4 heads on 4, window 1000, 100K
//    tokens, whole call 508 -> 463 us; 16 heads on 4, 128 rows apart, 477 us
//    without and 489 us with it).  The chunk (a power of two, at most kXcdChunk)
//    leaves at least four rounds of chunks, 64 in a packed batch, where whole chunks
//    may lie past the end of their sequence and leave their XCD idle (8 heads on 2,
//    window 1024, six sequences of 1.7-11.7K tokens, four rounds 270 us, 64 rounds
//    210 us; 2 heads on 2, window 4096, 1.8-25K tokens 345 -> 291 us); blocks past
//    the last whole round of 8 chunks keep their index.
constexpr int kXcdChunk = 64, kXcdSpread = 256;
__device__ __forceinline__ uint32_t xcd_remap(uint32_t i, uint32_t n, bool contiguous,
                                              int log_chunk) {
  if (contiguous) {
    const uint32_t per = n / 8;
    return i < per * 8 ? (i % 8) * per + i / 8 : i;
  }
  const uint32_t span = 8u << log_chunk;
  if (i >= n / span * span) return i;
  const uint32_t k = i / 8;
  return (((i % 8) + 8 * (k >> log_chunk)) << log_chunk) + (k & ((1u << log_chunk) - 1));
}

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// The lanes of a wavefront exchange data through LDS here and there (each
// writes its own part, then reads what other lanes wrote).  The hardware runs
// a wave's LDS instructions in order, but the compiler knows nothing of the
// other lanes: without a fence it may move a read above another lane's write
// (into the branch that made that write conditional, say).  This orders every
// LDS access before it against every one after it, with all lanes present.
__device__ __forceinline__ void wave_lds_exchange() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef short i16x8 __attribute__((ext_vector_type(8)));

typedef int i32x4 __attribute__((ext_vector_type(4)));

// 16 bytes per lane from a buffer into LDS at byte address lds + 16*lane (LDS
// DMA; rsrc and lds are wave-uniform scalars).  Written as asm so that the
// compiler does not track the transfer: its wait-count pass would otherwise
// wait for every DMA in flight before any LDS read it cannot prove disjoint
// from the DMA's target (the V^T reads of the current tile, while the next
// tile's DMA is in flight).  The main loop waits for each tile's DMA itself
// (vmcnt) before the barrier that publishes the tile.  The host pass of the
// kernel templates sees empty bodies.
//
// The compiler inserts no wait states for an instruction inside asm, and the
// hardware does not interlock two of the operands here: a VMEM instruction
// that reads an SGPR written by a VALU instruction (v_readfirstlane, which
// builds the descriptors) needs 5 wait states, and an LDS DMA needs 1 after M0
// is written.  With fewer it can read the SGPR's previous value: a stale
// record count makes the fetch return zeros past it.  So the descriptors and
// the LDS base of a group of DMAs first pass through settle_sgprs (s_nop 4,
// which hands them back as its own outputs: every use comes after it, and
// only scalar arithmetic lies between), and each DMA then waits the one state
// M0 needs.

// A descriptor as read from the first lane (wave-uniform values in scalar
// registers: the compiler cannot hand an "s" asm operand a vector copy).
__device__ __forceinline__ i32x4 first_lane(i32x4 r) {
  return {__builtin_amdgcn_readfirstlane(r[0]), __builtin_amdgcn_readfirstlane(r[1]),
          __builtin_amdgcn_readfirstlane(r[2]), __builtin_amdgcn_readfirstlane(r[3])};
}
__device__ __forceinline__ void settle_sgprs(i32x4& r0, i32x4& r1, uint32_t& m) {
#if defined(__HIP_DEVICE_COMPILE__)
  r0 = first_lane(r0);
  r1 = first_lane(r1);
  m = (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
  asm volatile("s_nop 4" : "+s"(r0), "+s"(r1), "+s"(m));
#endif
}
__device__ __forceinline__ void settle_sgprs(i32x4& r0, uint32_t& m) {
#if defined(__HIP_DEVICE_COMPILE__)
  r0 = first_lane(r0);
  m = (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
  asm volatile("s_nop 4" : "+s"(r0), "+s"(m));
#endif
}
__device__ __forceinline__ void dma16(const i32x4& rsrc, uint32_t lds, int voff) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
               :: "v"(voff), "s"(rsrc), "{m0}"(lds) : "memory");
#endif
}

// ds_read_b64_tr_b16: inside each group of 16 lanes, lane i receives element
// k (k = 0..3) of the 8-byte row read by lane 4k + i/4, at position i%4.
__device__ __forceinline__ i16x4 lds_read_tr(const uint16_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (i16x4 __attribute__((address_space(3)))*)(p));
}

// Row index -> position of that row inside its sequence.  In the strided
// dense-row mode row r < nA is anchor r*gamma, later rows are tail rows.
template <int MODE>
__device__ __forceinline__ int row_pos(int r, int nA, int Lc, int gamma) {
  if (MODE == kDenseRows) return r < nA ? r * gamma : Lc + (r - nA);
  return r;
}

// LDS bytes of one workgroup: the K/V ring, then, for the sparse kernel, the
// fp32 dense rows of its anchors (`pre_bytes`) and the staging of the queries
// of wavefronts past the fourth.
template <int D, int MODE, int NW>
constexpr int lds_bytes(int pre_bytes) {
  return kAttnStages * Lds<D, NW>::stageElems * 2 +
         (MODE == kSparse ? pre_bytes + (NW > 4 ? (NW - 4) * kRowsPerWave * D * 2 : 0) : 0);
}

// One attention workgroup, block `bid` of the launch's `nblk`.
template <int D, int MODE, int NW>
__device__ __forceinline__ void attn_body(const Args& a, uint32_t bid, uint32_t nblk) {
  using LD = Lds<D, NW>;
  constexpr int NS = kAttnStages;
  constexpr int kThreads = 64 * NW;
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  // The sparse kernel also holds, after the K/V ring, the fp32 dense rows of
  // its block's anchors for the fused store: hpw * (slab rows / gamma) rows
  // of D floats.
  float* const dpre = (float*)(smem + NS * LD::stageElems);

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  // The sparse kernel classifies tiles per wave from wave-uniform bounds:
  // with the wave index in a scalar register those tests stay scalar.
  const int wave = MODE == kSparse ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;
  const int half = lane >> 5;
  const int col = lane & 31;

  // ---- which (sequence, head group, row tile[, key chunk]) this block owns
  // (grids hold fewer than 2^31 blocks; the divisors are the launch's)
  uint32_t lid = xcd_remap(bid, nblk, a.n_hgroups % 8 == 0, a.xcd_log);
  uint32_t q = fdiv(lid, a.fd_sub);
  const uint32_t sub_hg = lid - q * (uint32_t)a.n_sub;
  lid = q;
  q = fdiv(lid, a.fd_rtiles);
  int rt = (int)(lid - q * (uint32_t)a.n_rtiles);
  lid = q;
  int c = 0;
  if (MODE == kDenseRows) {
    q = fdiv(lid, a.fd_nC);
    c = (int)(lid - q * (uint32_t)a.nC);
    lid = q;
  }
  q = fdiv(lid, a.fd_B);
  const int b = (int)(lid - q * (uint32_t)a.B);
  // (sub_hg counts the kv heads in turn where all head groups run innermost)
  const uint32_t turn = fdiv(sub_hg, a.fd_turn);
  const int hg = (int)(q * (uint32_t)a.n_sub + (sub_hg - turn * (uint32_t)a.turn) * (uint32_t)a.turn_step + turn);
  // Longest rows first.  In the dense modes blocks dispatched together then have
  // (nearly) the same number of key tiles, start on the same tile and stay in
  // step, so they share each key/value tile in L2.  In the sparse mode the rows
  // short of a whole window come last, the longest of them first, and fill the
  // CUs' uneven ends (32K tokens, window 2048 1176 -> 1156 us the whole call; packed
  // prompts up to 3071 tokens 223 -> 213 us); those with a whole window run in
  // ascending order, as the tiles in them do, so that the keys that neighbouring
  // slabs share are still in L2.  Against descending order all through: GQA 3,
  // gamma 48, 20K tokens 408 -> 394 us; sparse rows, 8 heads, three sequences of
  // 92-182K tokens 4000 -> 3891 us; 32 heads, window 4096, five of 6-18K 4152 ->
  // 4021 us; 4 heads, 100K tokens 265 -> 255 us; 131K tokens, 32 heads 6192 -> 6181 us,
  // 32K 1181 -> 1187 us.  Over key-block lists, whose short rows the host does not
  // know, all rows run in descending order (64K tokens, vertical-slash 2805 -> 2670 us
  // against ascending; with 2048 keys taken for the ramp 2744 -> 2813 us).
  if (MODE == kDenseRows && a.dr_n1 > 0) {
    // Sequences of one length: every (row tile, chunk) pair that takes a whole
    // key chunk runs before any that takes part of one.  The whole-chunk
    // blocks all run the same number of tiles, so the blocks on one XCD stay
    // in step over a chunk's tiles from round to round of the dispatch (a
    // shorter diagonal block in between would start its CU on the next chunk
    // early and put it out of step with the others).
    int j = c * a.n_rtiles + rt;
    if (j < a.dr_n1) {
      c = 0;
      for (int f; c < a.nC - 1 && j >= (f = a.dr_nrt - a.dr_t[c]); ++c) j -= f;
      rt = a.dr_nrt - 1 - j;
    } else if ((j -= a.dr_n1) < a.dr_n2) {
      c = 0;
      for (int f; c < a.nC - 1 && j >= (f = a.dr_t[c] - a.dr_z[c]); ++c) j -= f;
      rt = a.dr_t[c] - 1 - j;
    } else {
      return;  // no key of any chunk is visible to this pair (uniform over the block)
    }
  } else if (MODE != kSparse) {
    rt = a.n_rtiles - 1 - rt;
  }

  const Seq sq = seq_of(a, b);
  const int L = sq.L;
  const int rows_per_block = kRowsPerWave * a.ppw;
  if (MODE == kSparse) {
    // (the places that a shorter sequence of a packed batch leaves empty come first)
    const int nt = min(a.n_rtiles, (L + rows_per_block - 1) >> __builtin_ctz(rows_per_block));
    rt -= a.n_rtiles - nt;
    if (rt < 0) return;  // uniform over the block
    rt = rt < nt - a.ramp ? rt + a.ramp : nt - 1 - rt;
  }
  // hpw is a power of two: head in block = wave % hpw, sub-tile = wave / hpw
  const int hpw_log = __builtin_ctz(a.hpw);
  const int h = hg * a.hpw + (wave & (a.hpw - 1));
  const int g = (int)fdiv((uint32_t)(hg * a.hpw), a.fd_G);
  const int sub = wave >> hpw_log;
  const int nA = (int)fdiv((uint32_t)L, a.fd_gamma);
  const int Lc = nA * a.gamma;
  const int n_rows = (MODE == kDenseRows) ? nA + (L - Lc) : L;

  const int R0 = rt * rows_per_block;
  if (R0 >= n_rows) return;  // uniform over the block
  const int R1 = min(R0 + rows_per_block, n_rows);
  const int bpos_lo = row_pos<MODE>(R0, nA, Lc, a.gamma);
  const int bpos_hi = row_pos<MODE>(R1 - 1, nA, Lc, a.gamma);

  // ---- key tiles the block visits: [ta0, ta1) then [tb0, tb1)
  int ta0 = 0, ta1 = 0, tb0 = 0, tb1 = 0;
  // key-block lists: [ta0, ta1) indexes the block's list, then its own query
  // block's tiles [diag0, last row's tile]
  int lst0 = 0, diag0 = 0;
  if (MODE == kSparse && a.blk_ptr) {
    const int qb = (int)fdiv((uint32_t)R0, a.fd_bq);  // the block's rows lie in one query block
    const int64_t pi = ((int64_t)b * a.Hkv + g) * (a.nqb + 1) + qb;
    lst0 = a.blk_ptr[pi];
    ta1 = max(0, a.blk_ptr[pi + 1] - lst0);
    diag0 = qb * (a.block_q / kKeyTile);
    tb0 = diag0;
    tb1 = max(tb0, bpos_hi / kKeyTile + 1);
  } else if (MODE == kSparse) {
    const int sink_end = min(a.n_sink, bpos_hi + 1);
    ta1 = (sink_end + kKeyTile - 1) / kKeyTile;
    const int ws = max(0, bpos_lo - a.window + 1);
    tb0 = max(ws / kKeyTile, ta1);
    tb1 = max(tb0, bpos_hi / kKeyTile + 1);
  } else if (MODE == kDense) {
    ta1 = bpos_hi / kKeyTile + 1;
  } else {
    const int64_t kc0 = (int64_t)c * a.chunk;
    if (kc0 > bpos_hi) return;  // this key chunk lies past every row of the block
    const int64_t kc1 = min(kc0 + a.chunk, (int64_t)bpos_hi + 1);
    ta0 = (int)(kc0 / kKeyTile);
    ta1 = (int)((kc1 + kKeyTile - 1) / kKeyTile);
  }
  // The tile range is block-uniform; the list loads above are vector loads,
  // so say so explicitly, which keeps the loop counter and the per-tile tests
  // in scalar registers.
  ta0 = __builtin_amdgcn_readfirstlane(ta0);
  tb0 = __builtin_amdgcn_readfirstlane(tb0);
  lst0 = __builtin_amdgcn_readfirstlane(lst0);
  const int n_a = __builtin_amdgcn_readfirstlane(ta1 - ta0);
  const int n_iter = __builtin_amdgcn_readfirstlane(n_a + (tb1 - tb0));

  // ---- this wave's rows; lane (col) owns row wr0 + col
  const int wr0 = R0 + sub * kRowsPerWave;
  const bool wave_has_rows = wr0 < R1;
  const int my_r = wr0 + col;
  const bool row_valid = my_r < R1;
  const int my_pos = row_valid ? row_pos<MODE>(my_r, nA, Lc, a.gamma) : -1;
  const int wpos_lo = wave_has_rows ? row_pos<MODE>(wr0, nA, Lc, a.gamma) : 0;
  const int wpos_hi = wave_has_rows ? row_pos<MODE>(min(wr0 + kRowsPerWave, R1) - 1, nA, Lc,
                                                    a.gamma) : -1;

  bf16x8 qf[D / 16];  // the wave's queries (loaded in the prologue below)
  const int64_t kv_stride = (int64_t)a.Hkv * D;  // elements between consecutive keys
  const uint16_t* kbase = a.k + (sq.base * a.Hkv + g) * (int64_t)D;
  const uint16_t* vbase = a.v + (sq.base * a.Hkv + g) * (int64_t)D;

  // ---- tile loads by LDS DMA.  buffer_load_dwordx4 ... lds writes 16 bytes per
  // lane at M0 + 16*lane, so one instruction fills one 1 KB region of a tile.
  // Wave w fills regions w*RPW .. w*RPW+RPW-1 of both tiles; lane l of region
  // n lands on key row r = (1024n + 16l) / 2D at physical chunk pc and so
  // fetches logical chunk pc ^ swizzle(r) of that key.  The descriptors are
  // re-based at the tile's first key and end at the sequence end: keys past it
  // read as zero (and every valid row masks them).
  constexpr int RPW = LD::kRegionsPerWave;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  int dma_koff[RPW], dma_voff[RPW];
#pragma unroll
  for (int i = 0; i < RPW; ++i) {
    const int byte = (wave_s * RPW + i) * 1024 + 16 * lane;
    const int r = byte / (2 * D);
    const int pc = (byte % (2 * D)) / 16;
    dma_koff[i] = (int)(r * kv_stride * 2) + (pc ^ LD::kswz(r)) * 16;
    dma_voff[i] = (int)(r * kv_stride * 2) + (pc ^ LD::vswz(r)) * 16;
  }
  // Buffer descriptors (stride 0, raw buffer): base at the tile's first key,
  // num_records up to the sequence end, at most one tile.  Everything here is
  // wave-uniform (scalar registers).
  const uint32_t key_bytes = (uint32_t)__builtin_amdgcn_readfirstlane((int)(kv_stride * 2));
  const uint32_t tile_bytes = key_bytes * kKeyTile;
  const uint64_t kaddr0 = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uintptr_t)kbase) |
                          (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)((uintptr_t)kbase >> 32)) << 32;
  const uint64_t vaddr0 = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uintptr_t)vbase) |
                          (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)((uintptr_t)vbase >> 32)) << 32;
  const int L_s = __builtin_amdgcn_readfirstlane(L);
  const uint32_t smem_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)smem;
  auto dma = [&](int tile, int stage, bool values = true) {
    if (tile < 0) return;  // a list entry the key set ignores
    const uint32_t tu = (uint32_t)__builtin_amdgcn_readfirstlane(tile);
    const uint64_t off = (uint64_t)tu * tile_bytes;
    int keys = L_s - (int)(tu * kKeyTile);
    keys = keys < 0 ? 0 : keys;
    keys = keys > kKeyTile ? kKeyTile : keys;
    const uint32_t nrec = (uint32_t)keys * key_bytes;
    const uint64_t ka = kaddr0 + off, va = vaddr0 + off;
    i32x4 kr = {(int)(uint32_t)ka, (int)((uint32_t)(ka >> 32) & 0xffffu), (int)nrec, 0x00020000};
    i32x4 vr = {(int)(uint32_t)va, (int)((uint32_t)(va >> 32) & 0xffffu), (int)nrec, 0x00020000};
    uint32_t st0 = smem_lds + (uint32_t)(stage * LD::stageElems) * 2;
    settle_sgprs(kr, vr, st0);
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
      const uint32_t region = (uint32_t)((wave_s * RPW + i) * 512) * 2;  // bytes
      dma16(kr, st0 + region, dma_koff[i]);
      if (values) dma16(vr, st0 + (uint32_t)LD::kElems * 2 + region, dma_voff[i]);
    }
  };

  // Per-lane LDS read offsets (elements, stage 0).  K operand (nb, kk): key row
  // 32nb + col, logical chunk 2kk + half.  V^T operand (t, mb): transposing
  // reads where, inside each 16-lane group, lane 4k+m points at key
  // 16t + 4h + k (and +8 for the second read) and dims 32mb + 16*g1 + 4m.
  const int ksw = LD::kswz(col);
  int kread[D / 16];
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) kread[kk] = col * D + (((2 * kk + half) ^ ksw) * 8);
  const int tr_g1 = (lane >> 4) & 1, tr_k = (lane >> 2) & 3, tr_m = lane & 3;
  const int vsw = LD::vswz(4 * half + tr_k);
  int vread[D / 32];
#pragma unroll
  for (int mb = 0; mb < D / 32; ++mb)
    vread[mb] = (4 * half + tr_k) * D + (((4 * mb + 2 * tr_g1 + (tr_m >> 1)) ^ vsw) * 8) +
                (tr_m & 1) * 4;

  // list entries outside [0, diag0) are not part of the key set (-1: skipped)
  auto tile_at = [&](int it) -> int {
    if (it >= n_a) return tb0 + (it - n_a);
    if (MODE == kSparse && a.blk_ptr) {
      const int e = __builtin_amdgcn_readfirstlane(a.blk_idx[lst0 + it]);
      return (e >= 0 && e < diag0) ? e : -1;
    }
    return ta0 + it;
  };

  // 0: no key of the tile is visible to any row of the wave; 1: every key is
  // visible to every row; otherwise the mask the tile needs per element:
  // kMaskCausal (some key lies past some row), kMaskWindow (some key lies
  // before some row's window), kMaskBoth, or kMaskAll (the window test meets
  // sink keys).  The dense modes only ever need the causal mask.
  auto classify = [&](int tile) -> int {
    if (!wave_has_rows || tile < 0) return 0;
    const int k0 = tile * kKeyTile, k1 = k0 + kKeyTile - 1;
    if (k0 > wpos_hi) return 0;
    if (MODE == kSparse) {
      if (k0 >= a.n_sink && wpos_lo - k1 >= a.window) return 0;
      const bool need_c = k1 > wpos_lo;
      const bool need_w = k1 >= a.n_sink && (int64_t)wpos_hi - k0 >= a.window;
      if (need_w && k0 < a.n_sink) return kMaskAll;
      return need_c ? (need_w ? kMaskBoth : kMaskCausal) : (need_w ? kMaskWindow : 1);
    }
    return k1 <= wpos_lo ? 1 : kMaskCausal;
  };

  f32x16 o[D / 32];
#pragma unroll
  for (int mb = 0; mb < D / 32; ++mb) o[mb] = f32x16{};
  // Reference `ref` of the base-2 logits (same in lanes l and l^32; has_ref: a
  // reference exists) and -ref / c in every register of nref, the block the
  // score accumulators start from, so that c times them is logit - ref.
  // (Scaling the queries by c ahead of the MFMA would round c q to bf16 once
  // more, an error proportional to the logits themselves.)
  const float qscale = a.scale_log2, inv_qscale = 1.f / a.scale_log2;
  float ref = 0.f;
  bool has_ref = false;
  f32x16 nref = f32x16{};
  float l = 0.f;        // this lane's share of the softmax normaliser
  // Key axis split finer than into long chunks (a.split_ref): the references of
  // chunks past the first differ from `ref0`, the one that the row takes from the
  // sequence's first tile, by whole powers of two.  Then every weight of the row
  // rounds to bf16 as it does in one chunk, and as the anchor's sparse row rounds
  // it, whose first tile is the same where the sinks cover it: the roundings of the
  // keys that both rows have cancel in Delta however finely the keys are split
  // (corrected rows against 64 bits, 2500 tokens, window 1024, 16 chunks: relative
  // error 0.00246, as in one chunk, in place of 0.00296; 4021 tokens, window 2048
  // 0.00245, 0.00274 in two long chunks).  It costs the keys of one more tile per
  // workgroup, 0-1 % of a whole call.
  const bool split = MODE == kDenseRows && a.split_ref && c > 0;
  float ref0 = 0.f;
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 ones2 = {(__bf16)1.0f, (__bf16)1.0f};

  // S^T of one tile against the wave's rows (register r of lane half h holds
  // key 8*(r/4) + 4*h + r%4 in s0, that key + 32 in s1); keys outside a row's
  // key set read -inf when `masked`.
  auto qk = [&](const uint16_t* ks, int tile, int masked, f32x16& s0, f32x16& s1) {
    s0 = nref;
    s1 = nref;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      const bf16x8 ka = *(const bf16x8*)(ks + kread[kk]);
      const bf16x8 kb = *(const bf16x8*)(ks + kread[kk] + 32 * D);
      s0 = mfma32(ka, qf[kk], s0);
      s1 = mfma32(kb, qf[kk], s1);
    }
    // issue the K reads four MFMAs ahead of their use, so the matrix phase is
    // not paced by LDS latency
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
    for (int i = 0; i < D / 8 - 4; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
    // accumulator register r of lane half h holds key kbase_t + o with the
    // constant offset o = 8*(r/4) + r%4 (+32 in s1); the tests compare o
    // against per-lane bounds: causal o <= my_pos - kbase_t, window
    // o > my_pos - kbase_t - window, sink o < n_sink - kbase_t
    if (masked) {
      const int kbase_t = tile * kKeyTile + 4 * half;
      const int lim_c = my_pos - kbase_t;
      // (64-bit: the window may be as large as INT_MAX; every offset is >= 0,
      // so a bound clamped at -1 admits the whole tile, as such a window does)
      const int lim_w = (int)max((int64_t)lim_c - (int64_t)a.window, (int64_t)-1);
      const int lim_s = a.n_sink - kbase_t;
      // one element test per mask kind (the kind is wave-uniform in the sparse
      // mode, so each is a branch of its own)
      auto apply = [&](auto ok) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int o0 = 8 * (r >> 2) + (r & 3);
          s0[r] = ok(o0) ? s0[r] : -INFINITY;
          s1[r] = ok(o0 + 32) ? s1[r] : -INFINITY;
        }
      };
      if (MODE != kSparse || masked == kMaskCausal)
        apply([&](int o) { return o <= lim_c; });
      else if (masked == kMaskWindow)
        apply([&](int o) { return o > lim_w; });
      else if (masked == kMaskBoth)
        apply([&](int o) { return o <= lim_c && o > lim_w; });
      else
        apply([&](int o) { return o <= lim_c && (o < lim_s || o > lim_w); });
    }
  };

  // The row's largest score of a tile in base-2 units (before the reference is
  // added back): over the 32 scores of this lane (a tree of 3-input max), then
  // across the lane pair l, l^32 that shares the row.
  auto row_max = [&](const f32x16& s0, const f32x16& s1) -> float {
    float t3[11];
#pragma unroll
    for (int i = 0; i < 5; ++i) t3[i] = fmaxf(s0[3 * i], fmaxf(s0[3 * i + 1], s0[3 * i + 2]));
#pragma unroll
    for (int i = 0; i < 5; ++i) t3[5 + i] = fmaxf(s1[3 * i], fmaxf(s1[3 * i + 1], s1[3 * i + 2]));
    t3[10] = fmaxf(s0[15], s1[15]);
    float mx = fmaxf(fmaxf(fmaxf(t3[0], t3[1]), fmaxf(t3[2], t3[3])),
                     fmaxf(fmaxf(t3[4], t3[5]), fmaxf(t3[6], t3[7])));
    mx = fmaxf(mx, fmaxf(t3[8], fmaxf(t3[9], t3[10])));
    const auto pr = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx),
                                                     false, false);
    return qscale * fmaxf(__uint_as_float(pr[0]), __uint_as_float(pr[1]));
  };

  // Online-softmax update with one tile's scores: the accumulators hold
  // s = q.k - ref / c, so c s = logit - ref in base-2 units, with c =
  // log2(e)/sqrt(d) applied in fp32 here (the queries stay as given); adds
  // the tile's weights to l and returns them as bf16 P^T fragments, moving
  // the reference first when it has to.
  //
  // The reference lags the true running max: weights are taken against the
  // current one, and only if some lane's share of the tile's weight sum exceeds
  // 2^13 (or some lane has no reference yet) does the wave take the row max
  // of the tile.  ref then moves up by it when a score exceeds ref by more than 8
  // (a weight above 2^8), rescaling O and l, and the weights are taken again.
  // Every weight stays below 2^13 (harmless in fp32 and bf16): a lane whose
  // scores all lie within 8 of ref sums at most 32 * 2^8 = 2^13.  The result is
  // the same either way, since numerator and normaliser share the reference;
  // the common tile pays no max reduction and no subtraction.
  auto softmax = [&](f32x16& s0, f32x16& s1, bf16x8* pf) {
    // P^T fragment t covers keys 16t..16t+15: registers 8*(t%2)..+7 of block
    // t/2.  The sum covers the bf16 weights the MFMA multiplies (dot2 with 1,1),
    // in two chains.
    auto weights = [&]() {
      f32x16 p0, p1;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        p0[i] = fast_exp2(qscale * s0[i]);
        p1[i] = fast_exp2(qscale * s1[i]);
      }
      pf[0] = __builtin_convertvector(p0.lo, bf16x8);
      pf[1] = __builtin_convertvector(p0.hi, bf16x8);
      pf[2] = __builtin_convertvector(p1.lo, bf16x8);
      pf[3] = __builtin_convertvector(p1.hi, bf16x8);
      float ta = 0.f, tb = 0.f;
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        ta = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf[f], pf[f], 0, 1), ones2, ta, false);
        tb = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf[f], pf[f], 2, 3), ones2, tb, false);
        ta = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf[f], pf[f], 4, 5), ones2, ta, false);
        tb = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf[f], pf[f], 6, 7), ones2, tb, false);
      }
      // the exponentials go two at a time with other VALU instructions (the
      // scaling multiplies, conversions, sums) between them: a wave issues one
      // exponential every ~15 clocks and fits its other VALU work into those
      // gaps
      __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
      }
      return ta + tb;
    };
    float t = INFINITY;
    if (!__any(!has_ref)) t = weights();
    if (__any(!(t <= 8192.f))) {
      const float mx = row_max(s0, s1);
      // a lane without a reference takes its tile max (if it sees any key);
      // one with a reference moves only up
      const bool seen = mx != -INFINITY;
      const bool grow = has_ref ? mx > 8.f : seen;
      if (__any(grow)) {
        float up = mx;
        if (split) up = has_ref ? ceilf(mx) : ref0 + ceilf(mx - ref0);
        const float dm = has_ref ? fmaxf(up, 0.f) : (seen ? up : 0.f);
        const float alpha = has_ref ? fast_exp2(-dm) : 0.f;  // l and O are still zero without one
        ref += dm;
        has_ref = has_ref || seen;
        l *= alpha;
#pragma unroll
        for (int mb = 0; mb < D / 32; ++mb) o[mb] *= alpha;
        const float dr = dm * inv_qscale;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          s0[i] -= dr;
          s1[i] -= dr;
          nref[i] = -ref * inv_qscale;
        }
      }
      t = weights();
    }
    l += t;
  };

  // O^T += V^T P^T for one tile.
  auto pv = [&](const uint16_t* vs, const bf16x8* pf) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
      for (int mb = 0; mb < D / 32; ++mb) {
        const i16x4 lo = lds_read_tr(vs + vread[mb] + (16 * t) * D);
        const i16x4 hi = lds_read_tr(vs + vread[mb] + (16 * t + 8) * D);
        const i16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        o[mb] = mfma32(__builtin_bit_cast(bf16x8, both), pf[t], o[mb]);
      }
    }
    // V^T reads (two per MFMA) four MFMAs ahead of their use
    __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
#pragma unroll
    for (int i = 0; i < D / 8 - 4; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
  };

  auto compute = [&](const uint16_t* ks, int tile, int masked) {
    f32x16 s0, s1;
    bf16x8 pf[4];
    qk(ks, tile, masked, s0, s1);
    softmax(s0, s1, pf);
    pv(ks + LD::kElems, pf);
  };

  // ---- prologue: the first tile's DMA, the queries and the staged dense rows
  // are all in flight before the block waits once for them.
  //
  // A stage holds the tile of its last DMA; lanes past the sequence end are
  // written as zeros.  Only a block whose first NS tiles include its last one
  // (the only tile that can end inside the sequence's last 64 keys) clears
  // the ring first, so that no stage can hold bits left by an earlier kernel.
  if (n_iter <= NS) {
    for (int i = tid; i < NS * LD::stageElems / 8; i += kThreads)
      *(u32x4*)(smem + 8 * i) = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();
  }
#pragma unroll
  for (int p = 0; p < NS - 1; ++p)
    if (p < n_iter) dma(tile_at(p), p);
  if (split) dma(0, NS - 1, false);  // (its keys, into the stage that fills last)

  // Fused store: the merged dense rows of the block's anchors whose Delta is
  // not zero (anchor slot = head in block * groups per slab + group in slab),
  // staged in LDS so the epilogue does not wait on memory.  Each thread's
  // first vector loads with the queries; gamma < 16 (d = 128) leaves more.
  const bool stage_dense = MODE == kSparse && a.fuse && a.gamma > 1;
  const int per_slab = (int)fdiv((uint32_t)(kRowsPerWave * a.ppw), a.fd_gamma);
  const int nvec = stage_dense ? a.hpw * per_slab * (D / 4) : 0;
  auto dense_src = [&](int u) -> const f32x4* {
    const int slot = u / (D / 4), dv = u % (D / 4);
    const int apos = R0 + (slot % per_slab) * a.gamma;
    if (apos >= min(R1, Lc) || (int64_t)apos < a.cover) return nullptr;
    const int hh = hg * a.hpw + slot / per_slab;
    return (const f32x4*)(a.dense + (((int64_t)b * a.Hq + hh) * a.nR_max +
                                     (int)fdiv((uint32_t)apos, a.fd_gamma)) * D + dv * 4);
  };

  // Q fragments: lane holds dims kk*16 + half*8 .. +8 of its row, for every kk.
  // Rows past the end of the block load row R1-1's query (a valid row) and are
  // never written, so no load sits behind a branch.
  //
  // The sparse kernel, whose blocks are short, fetches its queries by LDS DMA
  // instead: whole rows (four per instruction at d = 128), each lane fetching
  // the 16-byte chunk that lands, XOR-swizzled by row, at its place in LDS.
  // The staging is free LDS: ring stage 1 (filled only after the first
  // barrier) for waves 0-3, the space behind the dense rows for waves 4-7.
  // Each lane reads its fragments from there.  Read straight into the fragment layout, every load
  // instruction fetched 32 bytes of each of 32 rows, and at every block's start
  // those loads queued behind each other in the memory pipeline.
  constexpr int QCPR = D / 8;  // 16-byte chunks per query row
  constexpr bool q_lds = MODE == kSparse;
  uint16_t* const qst = smem + (wave < 4 ? LD::stageElems + wave * (kRowsPerWave * D)
                                         : NS * LD::stageElems + nvec * 8 + (wave - 4) * (kRowsPerWave * D));
  if (q_lds) {
    static_assert(NS == 2 && 4 * kRowsPerWave * D <= LD::stageElems, "query staging fits stage 1");
    constexpr int RPI = 64 / QCPR;  // rows per DMA instruction
    const int jl = lane / QCPR, pc = lane % QCPR;
    const uint32_t row_bytes = (uint32_t)__builtin_amdgcn_readfirstlane(a.Hq * D * 2);
    const uint16_t* q0 = a.q + ((sq.base + R0) * a.Hq + h) * (int64_t)D;
    const uint64_t qa = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uintptr_t)q0) |
                        (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)((uintptr_t)q0 >> 32)) << 32;
    i32x4 qr = {(int)(uint32_t)qa, (int)((uint32_t)(qa >> 32) & 0xffffu), (int)0xfffffff0u, 0x00020000};
    uint32_t qdst = smem_lds + (uint32_t)(qst - smem) * 2;
    settle_sgprs(qr, qdst);
#pragma unroll
    for (int i = 0; i < kRowsPerWave / RPI; ++i) {
      const int j = i * RPI + jl;  // row of the wave
      const int r = min(wr0 + j, R1 - 1);
      dma16(qr, qdst + i * 1024, (r - R0) * (int)row_bytes + ((pc ^ (j & (QCPR - 1))) * 16));
    }
  } else {
    const int pos_ld = row_valid ? my_pos : row_pos<MODE>(R1 - 1, nA, Lc, a.gamma);
    const uint16_t* qp = a.q + ((sq.base + pos_ld) * a.Hq + h) * (int64_t)D + half * 8;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) qf[kk] = *(const bf16x8*)(qp + kk * 16);
  }
  const f32x4* dsrc = tid < nvec ? dense_src(tid) : nullptr;
  f32x4 dreg = f32x4{};
  if (dsrc) dreg = *dsrc;
  // Everything above has landed after this wait (vmcnt(0)): the main loop's
  // MFMAs read qf every iteration and must not wait behind the DMA issued in
  // it, and the first tile is in this wave's part of stage 0.
  __builtin_amdgcn_s_waitcnt(0x0F70);
  if (q_lds) {
    // this wave's query rows have landed in its staging (each lane reads
    // chunks other lanes fetched)
    wave_lds_exchange();
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk)
      qf[kk] = *(const bf16x8*)(qst + col * D + (((2 * kk + half) ^ (col & (QCPR - 1))) * 8));
    // the fragments are in registers before the barrier after which stage 1 fills
    __builtin_amdgcn_s_waitcnt(0xC07F);
  }
  if (split) {
    // (every row that sees this chunk sees all of tile 0)
    __syncthreads();
    f32x16 s0, s1;
    qk(smem + (NS - 1) * LD::stageElems, 0, 0, s0, s1);
    const float m0 = row_max(s0, s1);
    ref0 = fabsf(m0) < 1e30f ? m0 : 0.f;
  }
  if (dsrc) *(f32x4*)(dpre + tid * 4) = dreg;
  for (int u = tid + kThreads; u < nvec; u += kThreads)
    if (const f32x4* src = dense_src(u)) *(f32x4*)(dpre + u * 4) = *src;

  // ---- main loop over a ring of NS LDS stages, one barrier per tile.  Step
  // `it` waits until this wave's DMA of tile it has landed (later tiles may
  // still be in flight), meets the other waves at the barrier (after which
  // tile it is in LDS for everyone and nobody reads stage (it-1) % NS any
  // more), starts the DMA of tile it+NS-1 into that stage, then computes
  // tile it.  Keys past the sequence end arrive as zeros from the DMA; a
  // stage is read only after a DMA has filled it.
  constexpr int kLoadsPerTile = 2 * RPW;  // vmcnt entries one tile's DMA adds per wave
  // The loop is unrolled by the ring depth so each step's stage is a constant:
  // the LDS operand addresses are then a loop-invariant per-lane register plus
  // an immediate offset, with no address arithmetic per tile.
  for (int it0 = 0; it0 < n_iter; it0 += NS) {
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      const int it = it0 + st;
      if (it >= n_iter) break;
      const int ahead = min(NS - 2, n_iter - 1 - it);  // later tiles already in flight
      if (NS >= 4 && ahead >= 2)
        __builtin_amdgcn_s_waitcnt(0x0F70 | ((2 * kLoadsPerTile) & 15) | (((2 * kLoadsPerTile) >> 4) << 14));
      else if (NS >= 3 && ahead >= 1)
        __builtin_amdgcn_s_waitcnt(0x0F70 | (kLoadsPerTile & 15) | ((kLoadsPerTile >> 4) << 14));
      else
        __builtin_amdgcn_s_waitcnt(0x0F70);
      __syncthreads();
      if (it + NS - 1 < n_iter) dma(tile_at(it + NS - 1), (st + NS - 1) % NS);
      const int tile = tile_at(it);
      const int cls = classify(tile);
      const uint16_t* ks = smem + st * LD::stageElems;
      if (MODE == kSparse) {
        // tile classes are scalar here: one copy of the tile body with the
        // mask as a branch inside it, so the accumulators keep one register
        // assignment across tiles (two copies made the compiler copy O
        // between them at every step)
        if (cls != 0) compute(ks, tile, cls == 1 ? 0 : cls);
      } else if (cls == 1) {
        compute(ks, tile, 0);
      } else if (cls != 0) {
        compute(ks, tile, kMaskCausal);
      }
    }
  }

  // ---- epilogue: output register r of block mb is dim 32*mb + 8*(r/4) + 4*half + r%4
  const float lt = l + __shfl_xor(l, 32);
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  if (MODE == kSparse) {
    const float inv = 1.f / lt;
    f32x4 val[D / 32][4];  // this lane's output row in fp32
    if (a.fuse) {
      // Fused Delta store (the dense rows were merged into a.dense beforehand).
      // Every group of gamma rows lies inside one head's row slab of this
      // block, so its anchor's sparse row is in a register of some lane here:
      // the anchor lane forms Delta = dense - sparse in fp32 over the dense row
      // the prologue staged in LDS and leaves it there for the group's other
      // rows, which store bf16(sparse + Delta), one rounding.  Anchor rows
      // store the dense row, tail rows (past the last whole group) the dense
      // row too; groups whose anchor lies below a.cover (a < n_sink + window:
      // its sparse key set is all of [0, a]) have Delta = 0 exactly and keep
      // the sparse row untouched.  Recompute (fuse 2) replaces anchors only.
      const bool in_c = row_valid && my_pos < Lc;
      // group of the row inside the block's slab (R0 is a multiple of gamma)
      const int grp = in_c ? (int)fdiv((uint32_t)(my_pos - R0), a.fd_gamma) : 0;
      const int anc = in_c ? R0 + grp * a.gamma : 0;
      const bool open = in_c && (int64_t)anc >= a.cover;
      const bool is_anchor = open && anc == my_pos;
      const bool staged = a.gamma > 1;  // anchor dense rows are in dpre
      const bool delta = a.fuse == 1 && staged;
      const int xslot = ((wave & (a.hpw - 1)) * per_slab + grp) * D;
      if (delta && is_anchor) {
#pragma unroll
        for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
          for (int jq = 0; jq < 4; ++jq) {
            const int dim = 32 * mb + 8 * jq + 4 * half;
            const f32x4 sv = {o[mb][4 * jq] * inv, o[mb][4 * jq + 1] * inv,
                              o[mb][4 * jq + 2] * inv, o[mb][4 * jq + 3] * inv};
            const f32x4 dv = *(const f32x4*)(dpre + xslot + dim);
            *(f32x4*)(dpre + xslot + dim) = dv - sv;
            val[mb][jq] = dv;
          }
      }
      // Delta of every group is in dpre, and no wave reads the K/V ring any more
      __syncthreads();
      const bool tail = row_valid && my_pos >= Lc;
      // one branch per row kind (not one per vector): corrected rows fold the
      // normalisation into the add, sparse rows only normalise, dense rows copy
      if (delta && is_anchor) {
        // val holds the dense row
      } else if (delta && open) {
#pragma unroll
        for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
          for (int jq = 0; jq < 4; ++jq) {
            const f32x4 dl = *(const f32x4*)(dpre + xslot + 32 * mb + 8 * jq + 4 * half);
#pragma unroll
            for (int e = 0; e < 4; ++e) val[mb][jq][e] = __builtin_fmaf(o[mb][4 * jq + e], inv, dl[e]);
          }
      } else if (tail || (is_anchor && !staged)) {
        // dense row in global memory: tail rows, and anchors when not staged
        const float* gdrow =
            a.dense + (((int64_t)b * a.Hq + h) * a.nR_max +
                       (in_c ? (int)fdiv((uint32_t)my_pos, a.fd_gamma) : nA + (my_pos - Lc))) * D;
#pragma unroll
        for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
          for (int jq = 0; jq < 4; ++jq) val[mb][jq] = *(const f32x4*)(gdrow + 32 * mb + 8 * jq + 4 * half);
      } else if (is_anchor) {
#pragma unroll
        for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
          for (int jq = 0; jq < 4; ++jq)
            val[mb][jq] = *(const f32x4*)(dpre + xslot + 32 * mb + 8 * jq + 4 * half);
      } else {
#pragma unroll
        for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
          for (int jq = 0; jq < 4; ++jq)
#pragma unroll
            for (int e = 0; e < 4; ++e) val[mb][jq][e] = o[mb][4 * jq + e] * inv;
      }
    } else {
#pragma unroll
      for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
        for (int jq = 0; jq < 4; ++jq)
#pragma unroll
          for (int e = 0; e < 4; ++e) val[mb][jq][e] = o[mb][4 * jq + e] * inv;
      // the unfused schedule also keeps every anchor's sparse row in fp32
      const int grp = (a.sa && row_valid) ? (int)fdiv((uint32_t)my_pos, a.fd_gamma) : 0;
      if (a.sa && row_valid && grp * a.gamma == my_pos && my_pos < Lc) {
        float* sarow = a.sa + (((int64_t)b * a.Hq + h) * a.nA_max + grp) * D;
#pragma unroll
        for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
          for (int jq = 0; jq < 4; ++jq) *(f32x4*)(sarow + 32 * mb + 8 * jq + 4 * half) = val[mb][jq];
      }
      __syncthreads();  // no wave reads the K/V ring any more
    }
    // The rows go out through LDS: each lane writes its row as bf16 into its
    // wave's 32 x D region of the idle K/V ring (16-byte chunks XOR-swizzled
    // by row), then every store instruction writes whole rows (64 lanes x 16
    // bytes: four rows at d = 128) instead of 16 bytes of each of 32 rows
    // that lie Hq * d elements apart.  The wave reads only what it wrote (its
    // lanes exchange rows through wave_lds_exchange).
    static_assert(NS * LD::stageElems >= NW * kRowsPerWave * D, "output staging fits the ring");
    constexpr int CPR = D / 8;     // 16-byte chunks per row
    constexpr int RPI = 64 / CPR;  // rows per store instruction
    uint16_t* const stg = smem + wave * (kRowsPerWave * D);
    if (row_valid) {
#pragma unroll
      for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
        for (int jq = 0; jq < 4; ++jq)
          *(bf16x4*)(stg + col * D + (((4 * mb + jq) ^ (col & (CPR - 1))) * 8) + 4 * half) =
              __builtin_convertvector(val[mb][jq], bf16x4);
    }
    wave_lds_exchange();
    // All the wave's reads first (one wait for them), then the stores: row
    // wr0 + rr of the wave lies rr * Hq * D elements past row wr0.
    const int rsub = lane / CPR, cc = lane % CPR;
    constexpr int NI = kRowsPerWave / RPI;
    u32x4 w[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int rr = i * RPI + rsub;
      w[i] = *(const u32x4*)(stg + rr * D + ((cc ^ (rr & (CPR - 1))) * 8));
    }
    uint16_t* const orow = a.out + ((sq.base + wr0 + rsub) * a.Hq + h) * (int64_t)D + cc * 8;
    const int64_t rstep = (int64_t)RPI * a.Hq * D;
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (wr0 + i * RPI + rsub < R1) *(u32x4*)(orow + i * rstep) = w[i];
    return;
  }
  if (MODE == kDenseRows) {
    // Unnormalised partial rows of this key chunk, through the idle ring like
    // the sparse rows: each lane writes its fp32 row into its wave's 16 x D
    // region (16-byte chunks XOR-swizzled by row), two passes of 16 rows, so
    // that every store instruction writes whole rows (two of 512 bytes at
    // d = 128) instead of 32 bytes of each of 32 rows nC * D floats apart.
    __syncthreads();  // no wave reads the K/V ring any more
    static_assert(NS * LD::stageElems * 2 >= NW * 16 * D * 4, "partial staging fits the ring");
    constexpr int CPR = D / 4;     // 16-byte chunks per fp32 row
    constexpr int RPI = 64 / CPR;  // rows per store instruction
    float* const stg = (float*)smem + wave * (16 * D);
    const int rsub = lane / CPR, cc = lane % CPR;
    const int64_t row0 = ((int64_t)b * a.Hq + h) * a.nR_max;
    if (a.merged) {
      // the only chunk: normalised rows, with the merge's arithmetic, which are
      // the merged rows as well (as a partial, each has a normaliser of 1)
      const float inv = 1.f / lt;
#pragma unroll
      for (int mb = 0; mb < D / 32; ++mb) o[mb] *= inv;
    }
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      if (pass) wave_lds_exchange();  // the first pass's reads are done
      if (row_valid && (col >> 4) == pass) {
        const int r16 = col & 15;
#pragma unroll
        for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
          for (int jq = 0; jq < 4; ++jq)
            *(f32x4*)(stg + r16 * D + (((8 * mb + 2 * jq + half) ^ (r16 & (CPR - 1))) * 4)) =
                f32x4{o[mb][4 * jq], o[mb][4 * jq + 1], o[mb][4 * jq + 2], o[mb][4 * jq + 3]};
      }
      wave_lds_exchange();
      // reads first, then the stores (row r lies r * nC * D floats past row 0)
      constexpr int NI = 16 / RPI;
      f32x4 w[NI];
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int rr = i * RPI + rsub;
        w[i] = *(const f32x4*)(stg + rr * D + ((cc ^ (rr & (CPR - 1))) * 4));
      }
      const int rb = wr0 + 16 * pass + rsub;
      float* const prow = a.part_o + ((row0 + rb) * a.nC + c) * D + cc * 4;
      const int64_t rstep = (int64_t)RPI * a.nC * D;
#pragma unroll
      for (int i = 0; i < NI; ++i)
        if (rb + i * RPI < R1) *(f32x4*)(prow + i * rstep) = w[i];
      if (a.merged) {
        float* const drow = a.dense + (row0 + rb) * D + cc * 4;
#pragma unroll
        for (int i = 0; i < NI; ++i)
          if (rb + i * RPI < R1) *(f32x4*)(drow + i * (RPI * D)) = w[i];
      }
    }
    if (row_valid && half == 0) {
      const int64_t slot = (row0 + my_r) * a.nC + c;
      a.part_ml[slot * 2] = has_ref ? ref : -INFINITY;  // -inf when no key of the chunk is visible
      a.part_ml[slot * 2 + 1] = a.merged ? 1.f : lt;
    }
    return;
  }
  if (!row_valid) return;
  const float inv = 1.f / lt;
  uint16_t* orow = a.out + ((sq.base + my_pos) * a.Hq + h) * (int64_t)D;
#pragma unroll
  for (int mb = 0; mb < D / 32; ++mb) {
#pragma unroll
    for (int jq = 0; jq < 4; ++jq) {
      const int dim = 32 * mb + 8 * jq + 4 * half;
      f32x4 val = {o[mb][4 * jq] * inv, o[mb][4 * jq + 1] * inv, o[mb][4 * jq + 2] * inv,
                   o[mb][4 * jq + 3] * inv};
      *(bf16x4*)(orow + dim) = __builtin_convertvector(val, bf16x4);
    }
  }
}

#define DA_ATTN_KERNEL(D, NW) \
  __global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 64 && NW == 4 ? 3 : 2)))

template <int D, int MODE, int NW>
DA_ATTN_KERNEL(D, NW) void attn_kernel(Args a) {
  attn_body<D, MODE, NW>(a, blockIdx.x, gridDim.x);
}

// The strided dense rows (`ar`, the first nr blocks: longer ones) and the sparse
// rows (`as`, from block nr8 on, nr rounded up to the XCDs' turn) of the unfused
// schedule, which do not depend on each other, in one launch: the sparse
// workgroups fill the CUs that the last strided ones leave, and a short call
// waits for the longer of the two instead of both.  Measured on an MI355X, two
// launches -> one, whole calls: interpolation, 32 heads d 128, window 512, 500
// tokens 36.0 -> 27.5 us, 4000 tokens 89 -> 77 us, 16000 tokens 302 -> 279 us;
// Delta, GQA 3, gamma 48, 20K tokens 433 -> 402 us; EMA 64K tokens 2791 -> 2763
// us; 131K tokens, 32 heads 6622 -> 6697 us (64 rounds of the CUs: not taken).
template <int D, int NW>
DA_ATTN_KERNEL(D, NW) void attn_pair_kernel(Args ar, Args as, uint32_t nr, uint32_t nr8) {
  if (blockIdx.x >= nr8)
    attn_body<D, kSparse, NW>(as, blockIdx.x - nr8, gridDim.x - nr8);
  else if (blockIdx.x < nr)
    attn_body<D, kDenseRows, NW>(ar, blockIdx.x, nr);
}
#undef DA_ATTN_KERNEL

// Log-sum-exp merge of the first nc key-chunk partials of one dense row:
// values po[cc * D] (VF floats each) under (running max, normaliser) ml[cc].
// One pass in chunk order with a running max M: chunks with no visible key
// (max -inf) are skipped, and acc, lsum move to a larger M by 2^(M - Mn).
// The loads of kU chunks go out before any of them is used.
template <int D, int kU, typename VF>
__device__ __forceinline__ VF merge_chunks(const float* po, const f32x2* ml, int nc) {
  float M = -INFINITY, lsum = 0.f;
  VF acc = VF{};
  for (int c0 = 0; c0 < nc; c0 += kU) {
    f32x2 m[kU];
    VF x[kU];
#pragma unroll
    for (int j = 0; j < kU; ++j) {
      const int cc = min(c0 + j, nc - 1);
      m[j] = ml[cc];
      x[j] = *(const VF*)(po + (int64_t)cc * D);
    }
#pragma unroll
    for (int j = 0; j < kU; ++j) {
      if (c0 + j >= nc || m[j][0] == -INFINITY) continue;
      const float Mn = fmaxf(M, m[j][0]);
      const float sc = fast_exp2(M - Mn), w = fast_exp2(m[j][0] - Mn);
      lsum = lsum * sc + w * m[j][1];
      acc = acc * sc + w * x[j];
      M = Mn;
    }
  }
  return acc * (1.f / lsum);
}

// The merge on its own.  Fused schedule, ahead of the sparse kernel: the dense
// rows it needs (tail rows and the anchors whose Delta is not zero) into a.dense
// in fp32.  Smoothing variants (DELTA), behind the unfused sparse kernel:
// Delta_i of every anchor into a.dbuf, tail rows into out.  Bound by reading the
// partials; one thread per four values of a row (a wavefront reads whole rows of
// one chunk stride), so that even a short sequence's rows give every SIMD
// several wavefronts: 4021 tokens, 32 heads 13.7 -> 5.2 us, 131K 80 -> 61 us
// against a workgroup per dense row.  U: chunks loaded together (see launch_delta_epilogue).
template <int D, bool DELTA, int U>
__global__ __launch_bounds__(kEpiThreads) void merge_rows_kernel(Args a) {
  constexpr int V = D / 4;
  const uint32_t n_rows = (uint32_t)a.B * (uint32_t)a.Hq * (uint32_t)a.nR_max;
  constexpr uint32_t kRowsPerBlock = kEpiThreads / V;
  const int dv = (int)(threadIdx.x % V) * 4;
  for (uint32_t row = blockIdx.x * kRowsPerBlock + threadIdx.x / V; row < n_rows;
       row += gridDim.x * kRowsPerBlock) {
    const uint32_t bh = fdiv(row, a.fd_nR);
    const int r = (int)(row - bh * (uint32_t)a.nR_max);
    const int b = (int)fdiv(bh, a.fd_Hq);
    const Seq sq = seq_of(a, b);
    const int nA = (int)fdiv((uint32_t)sq.L, a.fd_gamma);
    const int Lc = nA * a.gamma;
    if (r >= nA + (sq.L - Lc)) continue;
    const bool anchor = r < nA;
    const int pos = anchor ? r * a.gamma : Lc + (r - nA);
    const int64_t arow = ((int64_t)bh * a.nA_max + r) * D + dv;  // (anchors)
    if (anchor && (int64_t)pos < a.cover) {
      if (DELTA) *(f32x4*)(a.dbuf + arow) = f32x4{};  // exactly zero
      continue;
    }
    const int nc = (int)(((int64_t)pos + a.chunk) / a.chunk);  // chunks holding keys 0..pos
    const int64_t slot0 = (int64_t)row * a.nC;
    const f32x4 dense =
        merge_chunks<D, U, f32x4>(a.part_o + slot0 * D + dv, (const f32x2*)a.part_ml + slot0, nc);
    if (!DELTA) {
      *(f32x4*)(a.dense + (int64_t)row * D + dv) = dense;
    } else if (anchor) {
      *(f32x4*)(a.dbuf + arow) = dense - *(const f32x4*)(a.sa + arow);
    } else {
      typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
      const int h = (int)(bh - (uint32_t)b * (uint32_t)a.Hq);
      *(bf16x4*)(a.out + ((sq.base + pos) * a.Hq + h) * (int64_t)D + dv) =
          __builtin_convertvector(dense, bf16x4);
    }
  }
}

// Step 3 of Algorithm 1 for one dense row r of one sequence and a range of
// heads: merge the key-chunk partials of r into the dense result (log-sum-exp
// merge), then
//   anchor row a = r*gamma:  Delta = dense - sparse(a) in fp32, out[a] = dense,
//                            out[i] += Delta for i = a+1 .. a+gamma-1;
//   tail row:                out[row] = dense.
// An anchor below a.cover (a < n_sink + window: all keys 0..a are in its
// sparse set) has Delta exactly zero and the block leaves its rows untouched;
// with key-block lists no anchor is assumed covered (cover = 0).
// Epilogue modes: the Delta correction itself; "recompute" (Eq. 5: the dense
// row replaces the sparse one at anchors only).
enum Epi { kEpiDelta = 0, kEpiRecompute = 1 };

template <int D, int EPI>
__global__ __launch_bounds__(kEpiThreads) void delta_epilogue_kernel(Args a) {
  extern __shared__ __attribute__((aligned(16))) float delta[];  // [head in range][D]
  const int tid = threadIdx.x;
  int64_t lid = blockIdx.x;
  const int n_hc = (a.Hq + a.head_chunk - 1) / a.head_chunk;
  const int hc = (int)(lid % n_hc);
  lid /= n_hc;
  const int r = (int)(lid % a.nR_max);
  const int b = (int)(lid / a.nR_max);

  const Seq sq = seq_of(a, b);
  const int L = sq.L;
  const int nA = L / a.gamma;
  const int Lc = nA * a.gamma;
  const int nR = nA + (L - Lc);
  if (r >= nR) return;
  const bool anchor = r < nA;
  const int pos = anchor ? r * a.gamma : Lc + (r - nA);
  const bool covered = anchor && (int64_t)pos < a.cover;
  const int h0 = hc * a.head_chunk;
  const int h1 = min(a.Hq, h0 + a.head_chunk);
  const int nh = h1 - h0;
  constexpr int DC = D / 8;
  if (covered) return;
  const int nc = (int)(((int64_t)pos + a.chunk) / a.chunk);  // chunks holding keys 0..pos
  typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

  for (int idx = tid; idx < nh * DC; idx += kEpiThreads) {
    const int hh = idx / DC, dc = idx % DC;
    const int h = h0 + hh;
    const int64_t slot0 = (((int64_t)b * a.Hq + h) * a.nR_max + r) * a.nC;
    const f32x8 dense =
        merge_chunks<D, 8, f32x8>(a.part_o + slot0 * D + dc * 8, (const f32x2*)a.part_ml + slot0, nc);
    uint16_t* orow = a.out + ((sq.base + pos) * a.Hq + h) * (int64_t)D + dc * 8;
    *(bf16x8_t*)orow = __builtin_convertvector(dense, bf16x8_t);
    if (anchor && EPI == kEpiDelta) {
      const int64_t arow = (((int64_t)b * a.Hq + h) * a.nA_max + r) * D + dc * 8;
      *(f32x8*)(delta + hh * D + dc * 8) = dense - *(const f32x8*)(a.sa + arow);
    }
  }
  if (!anchor || EPI != kEpiDelta) return;
  __syncthreads();

  // rows pos+1 .. pos+gamma-1 for heads [h0, h1): nh*D contiguous values per
  // row.  Each thread loads kU vectors before it stores any, so that many
  // reads per thread are in flight (a load and a store of one address per
  // iteration would leave one).
  constexpr int kU = 4;
  const int per_row = nh * DC;
  const int64_t total = (int64_t)(a.gamma - 1) * per_row;
  for (int64_t u0 = tid; u0 < total; u0 += (int64_t)kU * kEpiThreads) {
    uint16_t* p[kU];
    bf16x8_t x[kU];
    int dl[kU];
#pragma unroll
    for (int j = 0; j < kU; ++j) {
      const int64_t u = min(u0 + (int64_t)j * kEpiThreads, total - 1);
      const int i = (int)(u / per_row);
      const int rem = (int)(u % per_row);
      const int hh = rem / DC, dc = rem % DC;
      p[j] = a.out + ((sq.base + pos + 1 + i) * a.Hq + h0 + hh) * (int64_t)D + dc * 8;
      dl[j] = hh * D + dc * 8;
      x[j] = *(const bf16x8_t*)p[j];
    }
#pragma unroll
    for (int j = 0; j < kU; ++j) {
      if (u0 + (int64_t)j * kEpiThreads >= total) break;
      const f32x8 y = __builtin_convertvector(x[j], f32x8) + *(const f32x8*)(delta + dl[j]);
      *(bf16x8_t*)p[j] = __builtin_convertvector(y, bf16x8_t);
    }
  }
}

// Recurrences of the smoothing variants over the anchors of one sequence, per
// (sequence, head, channel), in anchor order (a group's state needs the
// previous group's):
//   EMA (weight w): E_r = (1-w) E_{r-1} + w D_r over D = repeat(Delta, gamma),
//     E_{-1} = D_0.  Inside group i, D is constant, so with q = 1-w the value
//     entering the group, Ein_i, gives E_{a_i+k} = q^(k+1) Ein_i +
//     (1 - q^(k+1)) Delta_i; the scan stores Ein_i and steps
//     Ein_{i+1} = q^gamma Ein_i + (1 - q^gamma) Delta_i.
//   alpha-beta-gamma filter (gain p0, p1, p2; the interpolation appendix's
//     filter algorithm): a linear state-space recursion over the anchors;
//     Delta_i is replaced by the filtered position.
// Both steps are linear, x -> A x + g Delta_i, so a channel's anchors are cut
// into kScanSegs segments with a thread each: every segment runs from a zero
// state, the entry states follow one from the other through A^(segment), and
// every segment runs again from its own.  A workgroup holds kScanCh adjacent
// channels of one head (64-byte accesses), which gives B * Hq * d / kScanCh
// workgroups of 16 wavefronts; with one thread per channel the scan was one
// serial chain on 16 CUs (64K tokens, 32 heads, gamma 64: 73 -> 15 us for
// the EMA).  A diverging filter's A^(segment) may pass the range of floats, and a
// state may stop being finite; times the exact zeros of covered anchors, or of A,
// that would make NaN of rows whose correction is finite.  Such channels take their
// steps in order, one thread each, and so do the sequences of at most kScanSegs
// anchors in a longer batch, whose 64 entry states are the longer chain (whole
// calls, four sequences of 11-135 tokens, 32 heads, gamma 7, filter 42.5 -> 28.8 us,
// 50.2 us with registers for one workgroup per CU instead of two).
constexpr int kScanCh = 16, kScanSegs = 64;
constexpr double kScanMaxPower = 1e30;  // largest entry of A^(segment) that segments take
template <int CORR>
struct Scan {
  static constexpr int S = CORR == 3 ? 1 : 3;  // state size
  // the filter's state is Delta_0 at anchor 0: its steps start at anchor 1
  static constexpr int first = CORR == 3 ? 0 : 1;
  float A[S][S], g[S];
  float *dl, *ein;  // one channel's Delta_i, and its EMA values entering group i
  int64_t stride;

  // channel `ch` of all (sequence, head, d); nA: the sequence's anchors
  __device__ __forceinline__ Scan(const Args& a, int64_t ch, int& nA) : stride(a.d) {
    const int64_t bh = ch / a.d;
    nA = seq_of(a, (int)(bh / a.Hq)).L / a.gamma;
    const int64_t base = bh * a.nA_max * a.d + ch % a.d;
    dl = a.dbuf + base;
    ein = CORR == 3 ? a.ebuf + base : nullptr;
    if constexpr (CORR == 3) {
      const float q = 1.f - a.corr_p[0];
      A[0][0] = (q == 0.f) ? 0.f : fast_exp2((float)a.gamma * __log2f(q));
      g[0] = 1.f - A[0][0];
    } else {
      // x_i = A x_{i-1} + g Delta_i, A = (I - g h) F: the constant-acceleration
      // transition F (unit step) followed by the correction of the observed
      // position (h = (1, 0, 0)) with gain g
      const float g0 = a.corr_p[0], g1 = a.corr_p[1], g2 = a.corr_p[2];
      const float F[3][3] = {{1.f - g0, 1.f - g0, 0.5f * (1.f - g0)},
                             {-g1, 1.f - g1, 1.f - 0.5f * g1},
                             {-g2, -g2, 1.f - 0.5f * g2}};
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        g[i] = a.corr_p[i];
#pragma unroll
        for (int j = 0; j < 3; ++j) A[i][j] = F[i][j];
      }
    }
  }
  __device__ __forceinline__ void step(float* x, float v) const {
    float y[S];
#pragma unroll
    for (int i = 0; i < S; ++i) {
      y[i] = g[i] * v;
#pragma unroll
      for (int j = S - 1; j >= 0; --j) y[i] = __builtin_fmaf(A[i][j], x[j], y[i]);
    }
#pragma unroll
    for (int i = 0; i < S; ++i) x[i] = y[i];
  }
  // runs the anchors [i0, i1) from state x: batches of kB loads go out together
  __device__ __forceinline__ void run(float* x, int i0, int i1, bool store) const {
    constexpr int kB = 16;
    for (int i = i0; i < i1; i += kB) {
      float buf[kB];
#pragma unroll
      for (int j = 0; j < kB; ++j) buf[j] = dl[(int64_t)min(i + j, i1 - 1) * stride];
#pragma unroll
      for (int j = 0; j < kB; ++j) {
        if (i + j >= i1) break;
        if (CORR == 3 && store) ein[(int64_t)(i + j) * stride] = x[0];
        step(x, buf[j]);
        if (CORR == 4 && store) dl[(int64_t)(i + j) * stride] = x[0];
      }
    }
  }
  __device__ __forceinline__ void run_in_order(int nA) const {
    float x[S] = {};
    x[0] = dl[0];
    run(x, first, nA, true);
  }
};

// One thread per channel, in order (see scan_in_order).
template <int CORR>
__global__ __launch_bounds__(256) void corr_scan_in_order_kernel(Args a, int64_t block0) {
  const int64_t ch = (block0 + blockIdx.x) * 256 + threadIdx.x;
  if (ch >= (int64_t)a.B * a.Hq * a.d) return;
  int nA;
  const Scan<CORR> scan(a, ch, nA);
  if (nA > 0) scan.run_in_order(nA);
}

template <int CORR>
__global__ __launch_bounds__(kScanCh * kScanSegs) __attribute__((amdgpu_waves_per_eu(8)))
void corr_scan_kernel(Args a, int64_t block0) {
  constexpr int S = Scan<CORR>::S, first = Scan<CORR>::first;
  __shared__ float st[kScanSegs][S][kScanCh];
  __shared__ float Ap[S * S];
  __shared__ int in_order;  // 1: no segments
  const int cl = threadIdx.x % kScanCh, seg = threadIdx.x / kScanCh;
  int nA;
  const Scan<CORR> scan(a, (block0 + blockIdx.x) * kScanCh + cl, nA);
  if (nA == 0) return;  // uniform over the block
  const int len = (nA - first + kScanSegs - 1) / kScanSegs;
  const int i0 = min(nA, first + seg * len), i1 = min(nA, i0 + len);

  if (nA <= kScanSegs) {  // uniform over the block
    if (seg == 0) scan.run_in_order(nA);
    return;
  }
  if (threadIdx.x == kScanCh * kScanSegs - 1) {
    // A^len by repeated squaring, in 64 bits (a marginally stable filter's
    // powers cancel); entries stay finite, as products end past kScanMaxPower
    double P[S][S], Q[S][S];
    for (int i = 0; i < S; ++i)
      for (int j = 0; j < S; ++j) {
        P[i][j] = i == j ? 1.0 : 0.0;
        Q[i][j] = scan.A[i][j];
      }
    bool fits;
    double sum = 0.0;
    auto mul = [&](double (*X)[S], double (*Y)[S]) {  // X = X Y
      double Z[S][S];
      sum = 0.0;
      for (int i = 0; i < S; ++i)
        for (int j = 0; j < S; ++j) {
          Z[i][j] = 0.0;
          for (int k = 0; k < S; ++k) Z[i][j] += X[i][k] * Y[k][j];
        }
      for (int i = 0; i < S; ++i)
        for (int j = 0; j < S; ++j) {
          X[i][j] = Z[i][j];
          sum += fabs(Z[i][j]);
        }
      fits = sum <= kScanMaxPower;
    };
    for (int i = 0; i < S; ++i)
      for (int j = 0; j < S; ++j) sum += fabs(Q[i][j]);
    fits = sum <= kScanMaxPower;
    for (int n = len; n > 0 && fits; n >>= 1) {
      if (n & 1) mul(P, Q);
      if (n > 1 && fits) mul(Q, Q);
    }
    for (int i = 0; i < S; ++i)
      for (int j = 0; j < S; ++j) Ap[i * S + j] = fits ? (float)P[i][j] : 0.f;
    in_order = !fits;
  }
  float x[S] = {};
  scan.run(x, i0, i1, false);
#pragma unroll
  for (int i = 0; i < S; ++i) st[seg][i][cl] = x[i];
  __syncthreads();
  if (seg == 0 && !in_order) {
    float e[S] = {};
    e[0] = scan.dl[0];
    for (int sg = 0; sg < kScanSegs; ++sg) {
      float y[S];
#pragma unroll
      for (int i = 0; i < S; ++i) {
        y[i] = st[sg][i][cl];
        st[sg][i][cl] = e[i];
#pragma unroll
        for (int j = S - 1; j >= 0; --j) y[i] = __builtin_fmaf(Ap[i * S + j], e[j], y[i]);
      }
#pragma unroll
      for (int i = 0; i < S; ++i) e[i] = y[i];
    }
    // (every later state has a state that is not finite as a summand)
    if ((__float_as_uint(e[0]) & 0x7f800000u) == 0x7f800000u) in_order = 1;
  }
  __syncthreads();
  if (in_order) {  // uniform over the block
    if (seg == 0) scan.run_in_order(nA);
    return;
  }
#pragma unroll
  for (int i = 0; i < S; ++i) x[i] = st[seg][i][cl];
  scan.run(x, i0, i1, true);
}

// Adds the per-row correction of a smoothing variant to the gamma rows of one
// group, for a range of heads (rows a_i .. a_i+gamma-1, Hq*d contiguous values
// each):  interpolation (1-beta_k) Delta_i + beta_k Delta_{i+1} with
// beta_k = k/(gamma-1) (Delta_{i+1} = Delta_i for the last group); EMA
// q^(k+1) Ein_i + (1 - q^(k+1)) Delta_i; filter: the filtered Delta_i.
template <int D, int CORR>
__global__ __launch_bounds__(kEpiThreads) void corr_apply_kernel(Args a) {
  extern __shared__ __attribute__((aligned(16))) float c0[];  // [head in range][D], twice
  float* const c1 = c0 + a.head_chunk * D;
  const int tid = threadIdx.x;
  int64_t lid = blockIdx.x;
  const int n_hc = (a.Hq + a.head_chunk - 1) / a.head_chunk;
  const int hc = (int)(lid % n_hc);
  lid /= n_hc;
  const int i = (int)(lid % a.nA_max);
  const int b = (int)(lid / a.nA_max);
  const Seq sq = seq_of(a, b);
  const int nA = sq.L / a.gamma;
  if (i >= nA) return;
  const int h0 = hc * a.head_chunk;
  const int nh = min(a.Hq, h0 + a.head_chunk) - h0;
  constexpr int DC = D / 8;
  for (int idx = tid; idx < nh * DC; idx += kEpiThreads) {
    const int hh = idx / DC, dc = idx % DC;
    const int64_t row = (((int64_t)b * a.Hq + h0 + hh) * a.nA_max + i) * D + dc * 8;
    *(f32x8*)(c0 + hh * D + dc * 8) = *(const f32x8*)(a.dbuf + row);
    if (CORR == 2)
      *(f32x8*)(c1 + hh * D + dc * 8) = *(const f32x8*)(a.dbuf + row + (i + 1 < nA ? D : 0));
    if (CORR == 3) *(f32x8*)(c1 + hh * D + dc * 8) = *(const f32x8*)(a.ebuf + row);
  }
  __syncthreads();
  typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
  const int per_row = nh * DC;
  const int64_t total = (int64_t)a.gamma * per_row;
  const float lq = (CORR == 3) ? ((a.corr_p[0] >= 1.f) ? -INFINITY : __log2f(1.f - a.corr_p[0])) : 0.f;
  // (each thread loads kU vectors before it stores any: EMA at 64K tokens, 32
  // heads 252 -> 178 us, 6.0 TB/s of reads and writes, against one at a time)
  constexpr int kU = 4;
  for (int64_t u0 = tid; u0 < total; u0 += (int64_t)kU * kEpiThreads) {
    uint16_t* p[kU];
    bf16x8_t x[kU];
    int kk[kU], off[kU];
#pragma unroll
    for (int j = 0; j < kU; ++j) {
      const int64_t u = min(u0 + (int64_t)j * kEpiThreads, total - 1);
      kk[j] = (int)(u / per_row);
      const int rem = (int)(u % per_row);
      off[j] = rem * 8;
      p[j] = a.out + ((sq.base + (int64_t)i * a.gamma + kk[j]) * a.Hq + h0) * (int64_t)D + off[j];
      x[j] = *(const bf16x8_t*)p[j];
    }
#pragma unroll
    for (int j = 0; j < kU; ++j) {
      if (u0 + (int64_t)j * kEpiThreads >= total) break;
      const f32x8 di = *(const f32x8*)(c0 + off[j]);
      f32x8 corr;
      if (CORR == 2) {
        const float beta = a.gamma > 1 ? (float)kk[j] / (float)(a.gamma - 1) : 0.f;
        corr = (1.f - beta) * di + beta * *(const f32x8*)(c1 + off[j]);
      } else if (CORR == 3) {
        const float w = fast_exp2((float)(kk[j] + 1) * lq);  // q^(k+1)
        corr = w * *(const f32x8*)(c1 + off[j]) + (1.f - w) * di;
      } else {
        corr = di;
      }
      *(bf16x8_t*)p[j] = __builtin_convertvector(__builtin_convertvector(x[j], f32x8) + corr, bf16x8_t);
    }
  }
}

// Counts violations of what the other kernels take on trust in device-resident
// inputs (one workgroup; a debugging aid, not on the hot path):
//   cu_seqlens: starts at 0, non-decreasing, every length <= max_seqlen;
//   key-block lists, per (sequence, kv head): offsets inside [0, nnz] and
//   non-decreasing over the query blocks, each list strictly ascending.
// Every load is guarded by the checks before it, so malformed offsets are
// counted, never followed out of bounds.
__global__ __launch_bounds__(256) void check_inputs_kernel(const int32_t* cu, int B, int max_seqlen,
                                                           const int32_t* bptr,
                                                           const int32_t* bidx, int64_t nnz,
                                                           int Hkv, int nqb, int32_t* result) {
  __shared__ int32_t red[256];
  int32_t bad = 0;
  const int tid = threadIdx.x;
  if (cu) {
    if (tid == 0 && cu[0] != 0) ++bad;
    for (int i = tid; i < B; i += 256) {
      const int64_t len = (int64_t)cu[i + 1] - cu[i];
      if (len < 0 || len > max_seqlen) ++bad;
    }
  }
  if (bptr) {
    for (int64_t row = tid; row < (int64_t)B * Hkv; row += 256) {
      const int32_t* p = bptr + row * (nqb + 1);
      bool ok = p[0] >= 0 && (int64_t)p[nqb] <= nnz;
      for (int qb = 0; qb < nqb; ++qb) ok = ok && p[qb + 1] >= p[qb];
      if (!ok) {
        ++bad;
        continue;
      }
      for (int qb = 0; qb < nqb; ++qb)
        for (int64_t e = (int64_t)p[qb] + 1; e < p[qb + 1]; ++e)
          if (bidx[e] <= bidx[e - 1]) ++bad;
    }
  }
  red[tid] = bad;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) red[tid] += red[tid + w];
    __syncthreads();
  }
  if (tid == 0) *result = red[0];
}

// Fills in what a launch of `nblocks` blocks derives from its tiling.
template <int MODE>
void prepare_attn(Args& a, int64_t nblocks) {
  a.fd_rtiles = make_fastdiv((uint32_t)a.n_rtiles);
  a.fd_nC = make_fastdiv((uint32_t)(a.nC > 0 ? a.nC : 1));
  a.fd_B = make_fastdiv((uint32_t)a.B);
  a.fd_G = make_fastdiv((uint32_t)(a.Hq / a.Hkv));
  a.fd_gamma = make_fastdiv((uint32_t)a.gamma);
  a.fd_bq = make_fastdiv((uint32_t)(a.block_q > 0 ? a.block_q : 1));
  const int per_kv = a.Hq / a.Hkv / a.hpw;
  if (a.n_hgroups % 8 == 0) {
    // (an eighth that is half a kv head would be its shorter or longer rows)
    a.n_sub = a.Hkv % 8 == 0 ? per_kv : 1;
    a.turn = a.n_sub;
    a.turn_step = 1;
  } else {
    a.n_sub = a.n_hgroups;
    a.turn = a.Hkv;
    a.turn_step = per_kv;
  }
  a.fd_sub = make_fastdiv((uint32_t)a.n_sub);
  a.fd_turn = make_fastdiv((uint32_t)a.turn);
  const int64_t rpb = kRowsPerWave * a.ppw, keys = (int64_t)a.window + a.n_sink;
  a.ramp = a.blk_ptr ? a.n_rtiles : (int)std::min<int64_t>(a.n_rtiles, (keys + rpb - 1) / rpb);
  a.xcd_log = 0;
  const int64_t rounds = a.cu && a.B > 1 ? 64 : 4;
  if (MODE == kSparse && kRowsPerWave * a.ppw * 8 >= kXcdSpread * a.n_hgroups)
    while ((2 << a.xcd_log) <= kXcdChunk && nblocks >= (rounds * 8 * 2 << a.xcd_log)) ++a.xcd_log;
}

// Bytes of the dense rows a sparse workgroup stages for the fused store.
int pre_bytes(const Args& a) {
  return a.fuse && a.gamma > 1 ? a.hpw * (kRowsPerWave * a.ppw / a.gamma) * a.d * 4 : 0;
}

template <int MODE>
hipError_t launch_attn(const Args& a0, hipStream_t s, int64_t nblocks) {
  if (nblocks <= 0) return hipSuccess;
  if (nblocks > INT32_MAX) return hipErrorInvalidValue;
  Args a = a0;
  prepare_attn<MODE>(a, nblocks);
  const int pre = MODE == kSparse ? pre_bytes(a) : 0;
#define DA_ATTN(DD, W)                                                                          \
  hipLaunchKernelGGL((attn_kernel<DD, MODE, W>), dim3((unsigned)nblocks), dim3(64 * W),         \
                     (lds_bytes<DD, MODE, W>(pre)), s, a)
  const int waves = a.hpw * a.ppw;
  if (a.d == 128) {
    if (waves == 8) DA_ATTN(128, 8);
    else DA_ATTN(128, 4);
  } else {
    // (eight at d = 64: only fused sparse slabs that no half-size workgroup holds)
    if (waves == 4) DA_ATTN(64, 4);
    else if constexpr (MODE == kSparse) DA_ATTN(64, 8);
    else return hipErrorInvalidValue;
  }
#undef DA_ATTN
  return hipGetLastError();
}

constexpr int kScratchDevices = 64;
std::atomic<void*> g_scratch[kScratchDevices];

}  // namespace

// Workspace of the allocation-free entry point: each device the library runs
// on holds its own copy of this array until the process ends.  Host code
// never passes the array's name to a kernel (on the host it is a stand-in,
// not a device address): it uses the address hipGetSymbolAddress gives for
// the current device.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

hipError_t scratch_address(int dev, void** p) {
  if (dev < 0 || dev >= kScratchDevices) return hipErrorInvalidDevice;
  void* a = g_scratch[dev].load(std::memory_order_acquire);
  if (!a) {
    const hipError_t e = hipGetSymbolAddress(&a, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!a) return hipErrorInvalidSymbol;
    g_scratch[dev].store(a, std::memory_order_release);
  }
  *p = a;
  return hipSuccess;
}

hipError_t launch_check_inputs(const int32_t* cu, int B, int max_seqlen, const int32_t* bptr,
                              const int32_t* bidx, int64_t nnz, int Hkv, int nqb,
                              int32_t* result, hipStream_t s) {
  hipLaunchKernelGGL(check_inputs_kernel, dim3(1), dim3(256), 0, s, cu, B, max_seqlen, bptr, bidx,
                     nnz, Hkv, nqb, result);
  return hipGetLastError();
}

hipError_t launch_dense(const Args& a, hipStream_t s) {
  return launch_attn<kDense>(a, s, (int64_t)a.B * a.n_hgroups * a.n_rtiles);
}

// The strided rows' block order (see dr_n1 in Args).
static void order_dense_rows(Args& a) {
  a.dr_n1 = a.dr_n2 = 0;
  if (!a.cu && a.nC >= 1 && a.nC <= 16 && a.gamma >= 1) {
    // Sequences of a.N tokens: the key tiles row tile rt takes from chunk c,
    // for the dense rows (anchors r * gamma, then the tail rows) as the kernel
    // decodes them.
    const int64_t nA = a.N / a.gamma, Lc = nA * a.gamma, n_rows = nA + (a.N - Lc);
    const int rpb = kRowsPerWave * a.ppw;
    const int nrt = (int)((n_rows + rpb - 1) / rpb);
    auto end = [&](int rt) {  // one past the last row's position
      const int64_t r = std::min<int64_t>((int64_t)(rt + 1) * rpb, n_rows) - 1;
      return (r < nA ? r * a.gamma : Lc + (r - nA)) + 1;
    };
    auto tiles = [&](int rt, int c) -> int64_t {
      const int64_t kc0 = (int64_t)c * a.chunk, e = end(rt);
      if (kc0 >= e) return 0;
      return (std::min<int64_t>(kc0 + a.chunk, e) + kKeyTile - 1) / kKeyTile - kc0 / kKeyTile;
    };
    a.dr_nrt = nrt;
    for (int c = 0; c < a.nC; ++c) {
      const int64_t full = nrt > 0 ? tiles(nrt - 1, c) : 0;
      int t = nrt, z = nrt;
      if (full > 0) {
        for (t = nrt; t > 0 && tiles(t - 1, c) == full;) --t;
        for (z = t; z > 0 && tiles(z - 1, c) > 0;) --z;
      }
      a.dr_t[c] = t;
      a.dr_z[c] = z;
      a.dr_n1 += nrt - t;
      a.dr_n2 += t - z;
    }
  }
}

static int64_t dense_row_blocks(const Args& a) {
  return (int64_t)a.B * a.n_hgroups * a.nC * a.n_rtiles;
}

hipError_t launch_dense_rows(const Args& a0, hipStream_t s) {
  Args a = a0;
  order_dense_rows(a);
  return launch_attn<kDenseRows>(a, s, dense_row_blocks(a));
}

hipError_t launch_sparse(const Args& a0, hipStream_t s) {
  const int64_t ns = (int64_t)a0.B * a0.n_hgroups * a0.n_rtiles;
  if (!a0.rows) return launch_attn<kSparse>(a0, s, ns);
  // together with the strided rows: as many wavefronts per workgroup
  Args ar = *a0.rows, as = a0;
  const int64_t nr = dense_row_blocks(ar), nr8 = (nr + 7) / 8 * 8;
  const int waves = as.hpw * as.ppw;
  if (nr <= 0 || ns <= 0 || ar.hpw * ar.ppw != waves || nr8 + ns > INT32_MAX ||
      (as.d == 64 && waves != 4))
    return hipErrorInvalidValue;
  order_dense_rows(ar);
  prepare_attn<kDenseRows>(ar, nr);
  prepare_attn<kSparse>(as, ns);
  const dim3 g((unsigned)(nr8 + ns));
  const int pre = pre_bytes(as);
#define DA_PAIR(DD, W)                                                                          \
  hipLaunchKernelGGL((attn_pair_kernel<DD, W>), g, dim3(64 * W), (lds_bytes<DD, kSparse, W>(pre)), \
                     s, ar, as, (uint32_t)nr, (uint32_t)nr8)
  if (as.d == 128) {
    if (waves == 8) DA_PAIR(128, 8);
    else DA_PAIR(128, 4);
  } else {
    DA_PAIR(64, 4);
  }
#undef DA_PAIR
  return hipGetLastError();
}

// Query heads per workgroup of the in-place passes over `out`: a.head_chunk, or
// fewer where that leaves under eight workgroups per CU and each still has 16
// vectors per thread.  Measured on an MI355X, all heads -> this: Delta, 16 heads
// d 128, gamma 100, 1000 tokens 57.8 -> 39.2 us, 5000 tokens 90 -> 71 us;
// interpolation 32 heads, 5376 tokens, gamma 64 125 -> 103 us; GQA 3, 20K tokens,
// gamma 48, the epilogue alone 51 -> 46 us.  Without the second condition gamma 7
// loses: 16 heads d 64, 5000 tokens 55.7 -> 59.6 us.
int epilogue_heads(const Args& a, int64_t rows) {
  int hc = std::min(a.head_chunk, a.Hq);
  while (hc > 4 && a.B * rows * ((a.Hq + hc - 1) / hc) < 8 * 256 &&
         (int64_t)a.gamma * hc * (a.d / 8) >= 2 * 16 * kEpiThreads)
    hc = (hc + 1) / 2;
  return hc;
}

hipError_t launch_delta_epilogue(const Args& a0, hipStream_t s) {
  const dim3 t(kEpiThreads);
  if (a0.fuse || a0.corr_mode >= 2) {
    Args a = a0;
    a.fd_nR = make_fastdiv((uint32_t)a.nR_max);
    a.fd_Hq = make_fastdiv((uint32_t)a.Hq);
    a.fd_gamma = make_fastdiv((uint32_t)a.gamma);
    const int64_t rows = (int64_t)a.B * a.Hq * a.nR_max;
    if (rows <= 0) return hipSuccess;
    if (rows > INT32_MAX) return hipErrorInvalidValue;  // (over a terabyte of partials)
    const int64_t rpb = kEpiThreads / (a.d / 4);
    const dim3 g((unsigned)std::min<int64_t>((rows + rpb - 1) / rpb, 1 << 20));
    // Chunks whose loads go out together: at most those there are.  A row at half the
    // length has half of the chunks, so from five to eight of them two steps of four
    // load less for nothing, where bytes and not latency bound the pass: 16 heads,
    // three prompts of up to 13K tokens, gamma 4 (5M threads) 698 -> 691 us, 32 heads, up
    // to 11K, gamma 2 1153 -> 1126 us; 40000 tokens, 8 heads, gamma 16 (0.6M) 425 -> 429 us.
    const bool four = a.nC <= 4 || (a.nC <= 8 && rows * (a.d / 4) >= (1 << 21));
#define DA_MERGE(DD, DELTA, U) hipLaunchKernelGGL((merge_rows_kernel<DD, DELTA, U>), g, t, 0, s, a)
#define DA_MERGE_U(DD, DELTA)                \
  do {                                       \
    if (a.nC <= 2) DA_MERGE(DD, DELTA, 2);   \
    else if (four) DA_MERGE(DD, DELTA, 4);   \
    else DA_MERGE(DD, DELTA, 8);             \
  } while (0)
    if (a.d == 128) {
      if (a.fuse) DA_MERGE_U(128, false);
      else DA_MERGE_U(128, true);
    } else {
      if (a.fuse) DA_MERGE_U(64, false);
      else DA_MERGE_U(64, true);
    }
#undef DA_MERGE_U
#undef DA_MERGE
    return hipGetLastError();
  }
  Args a = a0;
  a.head_chunk = epilogue_heads(a, a.nR_max);
  const unsigned lds = (unsigned)(a.head_chunk * a.d * 4);
  const int n_hc = (a.Hq + a.head_chunk - 1) / a.head_chunk;
  const int64_t nblocks = (int64_t)a.B * a.nR_max * n_hc;
  if (nblocks <= 0) return hipSuccess;
  const dim3 g((unsigned)nblocks);
#define DA_EPI(DD, E) hipLaunchKernelGGL((delta_epilogue_kernel<DD, E>), g, t, lds, s, a)
  if (a.d == 128) {
    if (a.corr_mode == 0) DA_EPI(128, kEpiDelta);
    else DA_EPI(128, kEpiRecompute);
  } else {
    if (a.corr_mode == 0) DA_EPI(64, kEpiDelta);
    else DA_EPI(64, kEpiRecompute);
  }
#undef DA_EPI
  return hipGetLastError();
}

// Whether every channel takes its steps in order, one thread each: for few anchors,
// where the chain over the segments' entry states is the longer one, and for so
// many channels that one thread each fills the chip, where a second pass over the
// anchors only costs.  Measured on an MI355X, whole calls, segments -> in order:
// 4096 channels 73 anchors 68.4 -> 65.8 us, 151 anchors 53.1 -> 56.2 us; 16384
// channels 207 anchors 581 -> 578 us, 1076 anchors 4735 -> 4776 us; 32768 channels,
// 1667 anchors 5351 -> 5342 us; 40960, 2502 anchors 7103 -> 6882 us; 229376, up to
// 679 anchors 1429 -> 1240 us.
static bool scan_in_order(int64_t channels, int nA) {
  return nA <= kScanSegs || channels >= 32768 || nA <= channels / 64;
}

// After the merge: the scan (EMA, filter) and the apply pass of
// the smoothing variants (modes 2-4).
hipError_t launch_correction(const Args& a0, hipStream_t s) {
  Args a = a0;
  if (a.corr_mode < 2) return hipSuccess;
  if (a.corr_mode >= 3) {
    const int64_t channels = (int64_t)a.B * a.Hq * a.d;
    const bool in_order = scan_in_order(channels, a.nA_max);
    const int per_block = in_order ? 256 : kScanCh;
    const int64_t blocks = (channels + per_block - 1) / per_block;
    // (a dispatch holds fewer than 2^32 threads)
    const int64_t max_blocks = (int64_t)(1 << 28) / (in_order ? 256 : kScanCh * kScanSegs);
    for (int64_t b0 = 0; b0 < blocks; b0 += max_blocks) {
      const dim3 g((unsigned)std::min(max_blocks, blocks - b0));
      if (in_order && a.corr_mode == 3)
        hipLaunchKernelGGL(corr_scan_in_order_kernel<3>, g, dim3(256), 0, s, a, b0);
      else if (in_order)
        hipLaunchKernelGGL(corr_scan_in_order_kernel<4>, g, dim3(256), 0, s, a, b0);
      else if (a.corr_mode == 3)
        hipLaunchKernelGGL(corr_scan_kernel<3>, g, dim3(kScanCh * kScanSegs), 0, s, a, b0);
      else
        hipLaunchKernelGGL(corr_scan_kernel<4>, g, dim3(kScanCh * kScanSegs), 0, s, a, b0);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  }
  a.head_chunk = epilogue_heads(a, a.nA_max);
  const unsigned lds = (unsigned)(2 * a.head_chunk * a.d * 4);
  const int n_hc = (a.Hq + a.head_chunk - 1) / a.head_chunk;
  const int64_t nblocks = (int64_t)a.B * a.nA_max * n_hc;
  if (nblocks <= 0) return hipSuccess;
  const dim3 g((unsigned)nblocks), t(kEpiThreads);
#define DA_APPLY(DD, C) hipLaunchKernelGGL((corr_apply_kernel<DD, C>), g, t, lds, s, a)
  if (a.d == 128) {
    if (a.corr_mode == 2) DA_APPLY(128, 2);
    else if (a.corr_mode == 3) DA_APPLY(128, 3);
    else DA_APPLY(128, 4);
  } else {
    if (a.corr_mode == 2) DA_APPLY(64, 2);
    else if (a.corr_mode == 3) DA_APPLY(64, 3);
    else DA_APPLY(64, 4);
  }
#undef DA_APPLY
  return hipGetLastError();
}

}  // namespace da

// Chunked prefill of TreeKV for gfx950.
//
// A chunk of L tokens attends the cache as it was before the chunk plus the chunk's own tokens
// up to and including itself; every row's probabilities are added to the scores; the averaged
// scores are then frozen and Algorithm 1's append / compare / evict / advance
// is replayed for the L tokens.  L = 1 gives the decode step.
//
// Three launches per chunk, two for short ones (with re-assigned positions a fourth before them, which turns keys and queries):
//   attend   grid row tiles x G x U (ids remapped so that a unit's row tiles share an XCD's L2).  Two passes
//            over all visible columns with MFMA (16x16x32 bf16): the first finds the row statistics, the
//            second forms the final probabilities, O^T += V^T P^T with P split into two bf16 halves
//            (hi + lo) so that rounding P costs 2^-16, not 2^-9, and the probabilities' sums down the
//            workgroup's rows.  Writes O; the column sums go, as 64-bit fixed point, into one accumulator
//            per column of the unit with integer atomic adds (which commute exactly: whatever order the
//            workgroups arrive in, the sum is the same to the bit).  Up to 2560 visible columns (and, at
//            plain head_dim 64, while row tiles are few) a workgroup of 32 rows keeps their logits in registers and passes
//            over the columns once.
//   replay   grid U.  Adds the accumulated column sums to the scores (Algorithm 1's S update) and clears the
//            accumulators, then Algorithm 1's eviction for the chunk's tokens with frozen scores.  Inside one
//            sweep of idx over the tree region the scopes are disjoint pairs, so a sweep is one
//            parallel pass; sweeps run one after the other.  Then surviving chunk tokens are
//            matched with freed slots (ballot ranks), the order arrays are rewritten and the retained
//            positions emitted.
//   scatter  one wave per chunk token: the surviving rows are copied into their slots (short chunks: by the replay).
//
// Token ids during the replay: a slot number (< cap) for a cached token, cap + i for chunk
// token i that has no slot yet.

#include <type_traits>

#include "treekv_internal.h"

namespace tkv {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

constexpr int ROW_TILE = 64;     // query rows per attend workgroup
constexpr float NEG_BIG = -1.0e30f;
constexpr float COLSUM_FIX = 1099511627776.0f;      // 2^40: column sums cross kernels as 64-bit fixed point

__device__ inline f32x4_t mfma16(const uint4& a, const uint4& b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

struct ChunkInfo {
  int n;        // tokens cached before the chunk
  int fslot;    // the free slot (a hole among slots [0, n] once the cache is full)
  int t0;       // position of the chunk's first token
};

__device__ inline ChunkInfo load_chunk_info(const int* meta) {
  ChunkInfo c;
  c.n = meta[META_N];
  c.fslot = meta[META_FREE];
  c.t0 = meta[META_T];
  return c;
}

// ---------------------------------------------------------------------------------------------
// attend
// ---------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;

// two floats -> two bf16 (round to nearest even) packed in one dword, first value in the low half
__device__ inline unsigned pack_bf16(float a, float b) {
  f32x2_t v = {a, b};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2_t));
}

constexpr int AT_THREADS = 512;   // 8 waves
constexpr int AT_COLS = 128;      // columns per staged tile of the attend kernel

typedef short short4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4_t lds_short4_t;

// LDS of the attend kernel: K and V tiles exactly as they lie in memory (row-major, 128 rows each),
// two stages of each; the 16-byte pieces of a row are XOR-swizzled (see the kernel).
template <int D>
struct AttendLds {
  static constexpr int TILE_ELEMS = AT_COLS * D;                 // bf16 elements of one staged tile
  static constexpr int COLBUF_FLOATS = 2 * 2 * AT_COLS;          // column sums on their way out: [2 tiles][2 row groups][128]
  static constexpr size_t BYTES = 4 * (size_t)TILE_ELEMS * sizeof(uint16_t) + COLBUF_FLOATS * sizeof(float);
};

// Sum over the 16 lanes of a DPP row; every lane gets the total.
__device__ inline float row16_sum(float v) { return group_sum<16>(v); }
// Sums of eight values over the 16 lanes of a DPP row, shared out: lane lr gets those of x[2 (lr / 4)] and x[2 (lr / 4) + 1].
// Halving the values with the lanes (a masked add writes one value's sum into half of the lanes, another value's into
// the other half) takes 16 adds where eight full sums take 32.  One statement, because the instructions' distances are
// part of it: two wait states between the write of a register and its use through DPP.
__device__ inline float2 row16_sum8(const float (&x)[8]) {
  float s0, s1, r0, r1, r2, r3;
  asm("s_nop 1\n\t"
      "v_add_f32_dpp %2, %6, %6 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %3, %7, %7 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %4, %8, %8 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %5, %9, %9 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %2, %10, %10 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %3, %11, %11 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %4, %12, %12 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %5, %13, %13 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %0, %2, %2 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %1, %3, %3 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %0, %4, %4 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %1, %5, %5 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "s_nop 0\n\t"
      "v_add_f32_dpp %0, %0, %0 quad_perm:[3,2,1,0] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %1, %1, %1 quad_perm:[3,2,1,0] row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_add_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %1, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
      : "=&v"(s0), "=&v"(s1), "=&v"(r0), "=&v"(r1), "=&v"(r2), "=&v"(r3)
      : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]));
  return make_float2(s0, s1);
}
// Neither an infinity nor a NaN.  From the bits: this file is compiled with -fno-honor-nans.
__device__ inline int is_finite(float v) { return (__float_as_uint(v) & 0x7f800000u) != 0x7f800000u; }
// max of three.  This file is compiled with -fno-honor-nans: otherwise every fmaxf operand that comes out of
// an MFMA costs an extra instruction that quiets signalling NaNs, and the pair is not fused into v_max3_f32.
__device__ inline float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// Max over the four lanes (16 apart) that hold the same row; every lane gets it.
__device__ inline float row_max(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// The same with the source given as a wave-uniform base and a per-lane byte offset.
__device__ inline void async_copy16_offset(const void* uniform_base, unsigned lane_offset, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(lane_offset), "s"(uniform_base), "s"(lds_base) : "memory");
}
// A run of copies whose sources and LDS images are both contiguous, 1 KB apart: one M0 write, and the instruction
// offset (which is added to the global and to the LDS address alike) steps both sides.  One statement, so that
// nothing can come between the M0 write and its readers.
__device__ inline void async_copy16_run(const void* uniform_base, unsigned lds_base, unsigned off0, unsigned off1) {
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\t"
               "global_load_lds_dwordx4 %0, %2\n\t"
               "global_load_lds_dwordx4 %1, %2 offset:1024"
               :: "v"(off0), "v"(off1), "s"(uniform_base), "s"(lds_base) : "memory");
}
__device__ inline void async_copy16_run(const void* uniform_base, unsigned lds_base, unsigned off0, unsigned off1,
                                        unsigned off2, unsigned off3) {
  asm volatile("s_mov_b32 m0, %5\n\ts_nop 0\n\t"
               "global_load_lds_dwordx4 %0, %4\n\t"
               "global_load_lds_dwordx4 %1, %4 offset:1024\n\t"
               "global_load_lds_dwordx4 %2, %4 offset:2048\n\t"
               "global_load_lds_dwordx4 %3, %4 offset:3072"
               :: "v"(off0), "v"(off1), "v"(off2), "v"(off3), "s"(uniform_base), "s"(lds_base) : "memory");
}

// One workgroup owns 64 query rows of one head and passes over the visible columns twice, in tiles of 128.
//
// Staging.  Tiles go from global memory into LDS with asynchronous 16-byte loads (global_load_lds): no
// registers, no LDS store instructions, and the next tiles are in flight while the current one is used.
// One such instruction fills 1 KB of LDS in lane order, so a staged tile is row-major like the source; what
// a lane is free to choose is which 16-byte piece of its row it fetches, and that gives the swizzle: slot s
// of row r holds piece s ^ KSWZ(r) (K tiles) or s ^ VSWZ(r) (V tiles), chosen so that the operand reads
// below touch every LDS bank once.
//
// Sweep 1 finds every row's softmax statistics (max, sum).  Wave w takes the 16-column block w of every
// tile against all 64 rows (four 16-row MFMA blocks): S^T = K Q^T, K rows from LDS as A operands.  Each
// lane keeps a (reference, sum) for its own columns of its four rows, the reference raised lazily; lanes and waves are
// merged once, at the end.  Four K stages, so tiles are requested three iterations before they are used.
//
// Sweep 2 recomputes the logits and, knowing the statistics, forms the normalised probabilities
// directly: p = exp2(s*scale - max - log2(sum)), no running maximum and nothing to rescale.  They feed
// O^T += V^T P^T and, summed down the rows, the per-column score increments (Algorithm 1's S update).
// The 8 waves are 2 row groups (32 rows = two 16-row MFMA blocks) x 4 column quarters (32 columns of
// every tile).  S^T comes out of the MFMA with a lane holding 8 columns of one row, which is the B
// operand layout of P^T, so P never leaves the registers; it is split into two bf16 halves (hi + lo) so that
// rounding P costs 2^-16, not 2^-9.  The A operand V^T[d][8 columns] is read from the row-major V tile with
// the transposing LDS read (ds_read_b64_tr_b16: 16 lanes fetch a 4 x 16 block and each gets one column).
// Sweep 1 is software pipelined: the logits of tile t+1 are formed (matrix pipe) while the statistics of tile t are
// worked out (vector ALU).  The four quarters of a row group add their O through LDS at the end.
// Bound by instruction issue: two waves per SIMD (four at head_dim 64) issue every address, conversion and wait.
//
// Column sums: a wave adds its two row blocks, reduces over the 16 lanes that hold the 16 rows and
// leaves the 32 sums of its columns in LDS.  During the next tile two of the waves add the two row groups
// and add the tile's 128 sums to the unit's accumulators (the atomics then have a whole iteration to
// complete before anything waits on the memory counter).  A workgroup touches the accumulators of the columns
// of the tiles it visits (masked entries add zero; cache columns past the last cached token are left alone).
//
// ROPE (positions re-assigned to cache ranks): queries and keys come, already turned to their ranks and split into
// two bf16 parts each, from the scratch prefill_turn_kernel fills (pf_qrot, pf_krot; the chunk's own keys lie behind
// the cache rows there), and a logit is k_hi.q_hi + k_lo.q_hi + k_hi.q_lo (what is left out, lo.lo, is 2^-18 of the
// product).  The staging memory then holds one tile pair (hi, lo) where the plain kernel holds two tiles: sweep 1
// requests two tiles ahead instead of three, and sweep 2 has a second barrier per tile (the K pair is requested once
// every wave has formed its logits from it).  Everything after the logits is unchanged.
//
// head_dim 64 leaves room for two workgroups per compute unit (66 KB of LDS each) if the registers are held to 128: two
// sequences of 6000 tokens, 8 KV heads x 4, into 4096 slots take 956 us in chunks of 512 (1406 with one workgroup of 165
// registers and the longer instruction stream).  With ROPE 128 registers are not enough: 28 spill, and the wait for a reload
// in sweep 1 waits for the tiles requested ahead too.  One workgroup of 150 registers: 74.5 us a call at 32 heads, 512 into
// 2048 slots (87.7 with two of 128), 36.7 at 8 heads, 17 into 1024 (45.1), 468 at batch 8 (479); one case is slower, two
// sequences of 8 KV heads x 4 into 1024 slots, 86.3 (84.4).
template <int D, bool ROPE>
__global__ __launch_bounds__(AT_THREADS, D == 64 && !ROPE ? 4 : 2) void prefill_attend_kernel(Params p, const uint16_t* __restrict__ Q,
                                                                    const uint16_t* __restrict__ Kc,
                                                                    const uint16_t* __restrict__ Vc, int L,
                                                                    int row_tiles, float* __restrict__ out) {
  using Lds = AttendLds<D>;
  constexpr int KS = D / 32;          // k-steps of the q.k contraction
  constexpr int DB = D / 16;          // 16-wide blocks of the head dimension
  constexpr int PARTS = D / 8;        // 16-byte pieces per row
  constexpr int ROWB = D * 2;         // bytes per row
  constexpr int RPC = 1024 / ROWB;    // rows per 1 KB async-load instruction (4 at d=128, 8 at d=64)
  constexpr int CPW = AT_COLS / RPC / 8;               // such instructions per wave and tile (4 or 2)
  static_assert(D == 64 || D == 128, "swizzles are written for head_dim 64 and 128");
  extern __shared__ __attribute__((aligned(1024))) uint16_t pf_smem[];
  uint16_t* sK = pf_smem;                               // sweep 2: [2][TILE_ELEMS]; sweep 1: all four stages
  uint16_t* sV = pf_smem + 2 * Lds::TILE_ELEMS;         // [2][TILE_ELEMS]
  float* sC = reinterpret_cast<float*>(pf_smem + 4 * Lds::TILE_ELEMS);   // [2][2][128]

  // swizzles of the 16-byte slots of tile row r
  auto kswz = [](int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); };
  auto vswz = [](int r) { return D == 128 ? ((r & 7) << 1) : (((r >> 1) & 3) << 1); };

  // Workgroups are dealt to the 8 XCDs round robin by their linear id, and each XCD has its own L2.
  // The row tiles of one unit read the same K and V, so give them ids that land on one XCD:
  // workgroup w works on item (w % 8) * (n/8) + w / 8 of the (row tile fastest) item list.
  const int n_items = row_tiles * p.G * p.U, per_xcd = (n_items + 7) / 8;
  const int item = ((int)blockIdx.x % 8) * per_xcd + (int)blockIdx.x / 8;
  if (item >= n_items) return;
  const int row_tile = item % row_tiles, g = (item / row_tiles) % p.G, unit = item / (row_tiles * p.G);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, q4 = lane >> 4;
  const int rg = wave & 1;                                 // sweep 2: rows 32*rg .. +31 of the workgroup's 64
  const int cq = wave >> 1;                                // sweep 2: column quarter of every tile
  const int kvh = unit % p.Hkv, b = unit / p.Hkv;
  const int h = kvh * p.G + g;
  ChunkInfo ci = load_chunk_info(p.meta + (size_t)unit * META_STRIDE);
  ci.n = __builtin_amdgcn_readfirstlane(ci.n);             // tile addresses are scalar arithmetic on these two
  ci.fslot = __builtin_amdgcn_readfirstlane(ci.fslot);
  const int rbase = row_tile * ROW_TILE;                   // first chunk row of the workgroup

  // B operands: the Q rows of the four 16-row blocks (rows past the chunk repeat its last row)
  constexpr int QL = ROPE ? KS : 1;          // the second bf16 part of the queries exists only with ROPE
  uint4 qa[4][KS], qlo[4][QL];
  const uint16_t* Qsrc = ROPE ? p.pf_qrot : Q;
  const size_t q_part = (size_t)p.B * p.max_chunk * p.H * D;      // pf_qrot: [hi, lo][B][max_chunk][H][D]
  const int q_rows = ROPE ? p.max_chunk : L;
#pragma unroll
  for (int rb = 0; rb < 4; ++rb) {
    const uint16_t* qp = Qsrc + (((size_t)b * q_rows + min(rbase + rb * 16 + lr, L - 1)) * p.H + h) * D + q4 * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qa[rb][ks] = *reinterpret_cast<const uint4*>(qp + ks * 32);
    if constexpr (ROPE) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) qlo[rb][ks] = *reinterpret_cast<const uint4*>(qp + q_part + ks * 32);
    }
  }

  const size_t krot_rows = (size_t)p.cap + p.max_chunk;            // pf_krot: [U][hi, lo][cap + max_chunk][D]
  const uint16_t* Ku = ROPE ? p.pf_krot + (size_t)unit * 2 * krot_rows * D : (const uint16_t*)p.K + (size_t)unit * p.cap * D;
  const uint16_t* Vu = (const uint16_t*)p.V + (size_t)unit * p.cap * D;
  const int chunk_row_stride = p.Hkv * D;
  const int kchunk_row_stride = ROPE ? D : chunk_row_stride;
  const uint16_t* Kcu = ROPE ? Ku + (size_t)p.cap * D : Kc + ((size_t)b * L * p.Hkv + kvh) * D;
  const uint16_t* Vcu = Vc + ((size_t)b * L * p.Hkv + kvh) * D;
  const size_t klo_off = krot_rows * D;                            // from a key's hi part to its lo part (ROPE)

  // Cache columns are the n cached tokens' slots in slot order with the free slot left out: column j is slot
  // j + (j >= fslot).  (Walking slots [0, n] and masking the free one would cost a full cache of 2048 a 17th tile
  // for its one last slot.)
  const int cache_tiles = (ci.n + AT_COLS - 1) / AT_COLS;
  const int last_row = min(rbase + ROW_TILE, L) - 1;                   // last chunk row of the workgroup
  const int chunk_tiles = last_row / AT_COLS + 1;                      // causal: columns <= last_row
  const int ntiles = cache_tiles + chunk_tiles;
  const float sc = p.scale_log2e;
  const int last_cached = ci.n - 1, fslot = ci.fslot;                   // last visible cache column
  const int cache_lim = p.cap - 1, chunk_lim = L - 1;                   // last row that exists

  // ---- asynchronous tile loads: this wave's CPW instructions of 1 KB each ----
  // Instruction x of wave w fills LDS block c = w*CPW + x, i.e. tile rows c*RPC + a_lrow.  w*CPW*RPC is a
  // multiple of 16 rows, so the swizzle of a lane's row depends on x and a_lrow only.
  static_assert(CPW * RPC == 16, "a wave covers 16 rows of every tile");
  const int a_lrow = lane / PARTS, a_slot = lane % PARTS;
  // A tile wholly inside the cache, whose 16 rows for this wave do not straddle the free slot, is one run of requests from
  // one scalar base: nearly every tile, so its address costs some 20 scalar instructions (47 when all cases shared one
  // computation; two waves per SIMD issue them all, and with the shorter column sums that is 64.8 -> 59.4 us for the
  // kernel at 512 tokens into 2048 slots).
  const int full_tiles = ci.n / AT_COLS;
  const int fw = fslot - wave * 16;                        // the wave's columns reach the free slot ..
  const int shift_tile = (fw + AT_COLS - 1) >> 7;          // .. before this tile,
  const int straddle_tile = ((fw - 1) & (AT_COLS - 1)) < 15 ? fw >> 7 : -1;   // .. inside this one, or between two
  static_assert(AT_COLS == 128, "shifts by 7");
  const unsigned lds_wave = __builtin_amdgcn_readfirstlane(lds_address(pf_smem)) + wave * CPW * 1024;
  auto issue_tile = [&](const uint16_t* cache_src, const uint16_t* chunk_src, int chunk_stride, int tile, int stage,
                        auto swz) {
    const unsigned m0 = lds_wave + stage * (Lds::TILE_ELEMS * 2);
    auto piece = [&](int x) { return (unsigned)((a_slot ^ swz(x * RPC + a_lrow)) * 16); };
    if (tile < full_tiles && tile != straddle_tile) {
      // Cache rows are contiguous, like their LDS image: one scalar base and one M0 for the run of requests;
      // the per-lane offsets differ only in the swizzled piece.
      const unsigned lane_row = (unsigned)a_lrow * ROWB;
      const int row = __builtin_amdgcn_readfirstlane(tile * AT_COLS + wave * 16 + (tile >= shift_tile ? 1 : 0));
      const char* sbase = reinterpret_cast<const char*>(cache_src) + (size_t)row * ROWB;
      if constexpr (CPW == 4) async_copy16_run(sbase, m0, lane_row + piece(0), lane_row + piece(1), lane_row + piece(2), lane_row + piece(3));
      else async_copy16_run(sbase, m0, lane_row + piece(0), lane_row + piece(1));
      return;
    }
    const bool is_cache = tile < cache_tiles;
    const int col_w = (is_cache ? tile : tile - cache_tiles) * AT_COLS + wave * 16;    // first of this wave's 16 columns
    const uint16_t* base = is_cache ? cache_src : chunk_src;
    const int rstride = is_cache ? D : chunk_stride;
    const int lim = is_cache ? cache_lim : chunk_lim;
    if (!is_cache && col_w + 15 <= lim) {
      // every row exists: a scalar base per instruction plus a per-lane byte offset
      const unsigned lane_row = (unsigned)(a_lrow * rstride) * 2;
#pragma unroll
      for (int x = 0; x < CPW; ++x)
        async_copy16_offset(base + (size_t)(col_w + x * RPC) * rstride, lane_row + piece(x), m0 + x * 1024);
    } else {
      // cache columns at and after the free slot sit one row further on; rows past the last one repeat it (they are
      // masked later; what they must not be is unreadable)
#pragma unroll
      for (int x = 0; x < CPW; ++x) {
        const int col = col_w + x * RPC + a_lrow;
        const int row = col + ((is_cache && col >= fslot) ? 1 : 0);
        async_copy16(base + (size_t)min(row, lim) * rstride + piece(x) / 2, m0 + x * 1024);
      }
    }
  };

  // ------------------------------------------------------------------------------------------
  // sweep 1: row statistics
  // ------------------------------------------------------------------------------------------
  float neg_ml0, neg_ml1;              // -(max + log2(sum)) in the scaled log2 domain, rows of the two sweep-2 blocks
  {
    float m_run[4], l_run[4];          // this lane's columns of row rb*16 + lr: max of the scaled logits, sum of exp2
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) { m_run[rb] = NEG_BIG; l_run[rb] = 0.f; }
    // S^T of this wave's 16 columns of a staged tile against the 64 rows
    const int k1_row = wave * 16 + lr;
    const int k1_off = k1_row * D;
    const int k1_swz = kswz(k1_row);
    auto qk = [&](f32x4_t (&s)[4], int stage) {
      const uint16_t* kp = sK + stage * Lds::TILE_ELEMS + k1_off;
      uint4 k[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) k[ks] = *reinterpret_cast<const uint4*>(kp + ((ks * 4 + q4) ^ k1_swz) * 8);
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) s[rb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) s[rb] = mfma16(k[ks], qa[rb][ks], s[rb]);
      if constexpr (ROPE) {          // stage holds the keys' hi parts, stage + 1 their lo parts
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int rb = 0; rb < 4; ++rb) s[rb] = mfma16(k[ks], qlo[rb][ks], s[rb]);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) k[ks] = *reinterpret_cast<const uint4*>(kp + Lds::TILE_ELEMS + ((ks * 4 + q4) ^ k1_swz) * 8);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int rb = 0; rb < 4; ++rb) s[rb] = mfma16(k[ks], qa[rb][ks], s[rb]);
      }
    };
    // Masked logits become -inf: their exp2 is 0 against any finite running max, and a lane that has seen
    // nothing yet keeps its (finite) initial max, so no probability needs a guard.
    auto stats = [&](f32x4_t (&s)[4], int tile) {
      const bool is_cache = tile < cache_tiles;
      const int c0 = (is_cache ? tile * AT_COLS : (tile - cache_tiles) * AT_COLS) + wave * 16;   // this wave's 16 columns
      // only tiles that touch the end of the cache, the free slot or the causal diagonal need a mask (wave uniform)
      const bool need_mask = is_cache ? (c0 + 15 > last_cached) : (c0 + 15 > rbase);
      if (need_mask) {
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) {
          const int lim = is_cache ? last_cached : rbase + rb * 16 + lr;   // last visible column of this lane's row
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int col = c0 + q4 * 4 + i;
            s[rb][i] = col <= lim ? s[rb][i] : -INFINITY;
          }
        }
      }
      // The reference m_run of a lane's sums need not be their maximum, so it is raised lazily: when some lane's sum
      // passes 2^16 (or its exponentials overflow: the first tile it sees), the tile is taken again with the reference
      // 2^4 above the row's maximum in this tile.  The common path has no maxima, no rescaling and one exp2 per logit.
      // Not later than at 2^16, because log2(sum) and the exponents lose a bit each time they double: with 2^64 a row
      // whose logits rise by 40 had its normaliser off by 1.4e-6 instead of 0.7e-6.  2^4 above, and above the whole row's,
      // so that fewer tiles are taken twice: a sequence of 6000 tokens x 2 takes 956 us, 974 with every lane's own maximum
      // (941 with 2^64); the sums then lie nearer to 1, which costs no accuracy.
      float l_new[4];
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) {
        const float e0 = fast_exp2(fmaf(s[rb][0], sc, -m_run[rb])), e1 = fast_exp2(fmaf(s[rb][1], sc, -m_run[rb]));
        const float e2 = fast_exp2(fmaf(s[rb][2], sc, -m_run[rb])), e3 = fast_exp2(fmaf(s[rb][3], sc, -m_run[rb]));
        l_new[rb] = l_run[rb] + ((e0 + e1) + (e2 + e3));
      }
      if (__any(max3(l_new[0], l_new[1], fmaxf(l_new[2], l_new[3])) > 0x1p16f)) {
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) {
          const float m_new = row_max(fmaxf(m_run[rb], max3(s[rb][0], s[rb][1], fmaxf(s[rb][2], s[rb][3])) * sc + 4.0f));
          const float e0 = fast_exp2(fmaf(s[rb][0], sc, -m_new)), e1 = fast_exp2(fmaf(s[rb][1], sc, -m_new));
          const float e2 = fast_exp2(fmaf(s[rb][2], sc, -m_new)), e3 = fast_exp2(fmaf(s[rb][3], sc, -m_new));
          l_new[rb] = fmaf(l_run[rb], fast_exp2(m_run[rb] - m_new), (e0 + e1) + (e2 + e3));
          m_run[rb] = m_new;
        }
      }
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) l_run[rb] = l_new[rb];
    };
    // Iteration t: request tile t+3, form the logits of tile t+1 while the statistics of tile t are updated.
    // Stage (t+3)&3 held tile t-1, last read in iteration t-2.  In this sweep a wave reads exactly the 16 rows
    // of every tile that it requested itself, so the waves need no barrier between tiles: each runs on its own
    // count of outstanding requests.
    f32x4_t sa[4], sb[4];
    // ROPE: tile t sits in the stage pair (t & 1) * 2 (hi), + 1 (lo) and is requested two tiles ahead
    auto issue_k1 = [&](int t) {
      if constexpr (ROPE) {
        issue_tile(Ku, Kcu, kchunk_row_stride, t, (t & 1) * 2, kswz);
        issue_tile(Ku + klo_off, Kcu + klo_off, kchunk_row_stride, t, (t & 1) * 2 + 1, kswz);
      } else {
        issue_tile(Ku, Kcu, kchunk_row_stride, t, t & 3, kswz);
      }
    };
    constexpr int AHEAD = ROPE ? 2 : 3;     // how many tiles ahead of the one being finished the requests run
#pragma unroll
    for (int t = 0; t < AHEAD; ++t)
      if (t < ntiles) issue_k1(t);
    wait_vmcnt<0>();
    __syncthreads();
    qk(sa, 0);
    auto step = [&](f32x4_t (&cur)[4], f32x4_t (&nxt)[4], int t) {
      const bool more = t + AHEAD < ntiles;
      if constexpr (ROPE) {
        // the pair of tile t+2 goes where tile t was (its logits were formed in iteration t-1) and is read in the
        // next iteration: everything must have landed by then
        if (more) issue_k1(t + 2);
        if (t + 1 < ntiles) qk(nxt, ((t + 1) & 1) * 2);
        stats(cur, t);
        wait_vmcnt<0>();
      } else {
        if (more) issue_k1(t + 3);
        if (t + 1 < ntiles) qk(nxt, (t + 1) & 3);
        stats(cur, t);
        // tile t+2 must have landed before the next iteration reads it; only this iteration's requests may stay out
        if (more) wait_vmcnt<CPW>(); else wait_vmcnt<0>();
      }
    };
    for (int t = 0; t < ntiles; t += 2) {
      step(sa, sb, t);
      if (t + 1 < ntiles) step(sb, sa, t + 1);
    }
    __syncthreads();                   // the statistics below reuse the staging memory other waves may still read
    // merge the four lanes that share a row, then the eight waves through LDS
    float* st = reinterpret_cast<float*>(pf_smem);       // [8 waves][64 rows][2]
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
#pragma unroll
      for (int off = 16; off <= 32; off <<= 1) {
        const float mo = __shfl_xor(m_run[rb], off, 64), lo = __shfl_xor(l_run[rb], off, 64);
        const float mn = fmaxf(m_run[rb], mo);
        l_run[rb] = l_run[rb] * fast_exp2(m_run[rb] - mn) + lo * fast_exp2(mo - mn);
        m_run[rb] = mn;
      }
      if (q4 == 0) {
        st[(wave * 64 + rb * 16 + lr) * 2] = m_run[rb];
        st[(wave * 64 + rb * 16 + lr) * 2 + 1] = l_run[rb];
      }
    }
    __syncthreads();
    auto final_of = [&](int r) {       // r: row inside the workgroup's 64
      float mx = NEG_BIG;
#pragma unroll
      for (int w = 0; w < 8; ++w) mx = fmaxf(mx, st[(w * 64 + r) * 2]);
      float l = 0.f;
#pragma unroll
      for (int w = 0; w < 8; ++w) l += st[(w * 64 + r) * 2 + 1] * fast_exp2(st[(w * 64 + r) * 2] - mx);
      // rows past the chunk get probabilities of zero: they must not reach the column sums
      return rbase + r < L ? -(mx + __log2f(l)) : NEG_BIG;
    };
    neg_ml0 = final_of(rg * 32 + lr);
    neg_ml1 = final_of(rg * 32 + 16 + lr);
    __syncthreads();                   // the staging below reuses this LDS
  }

  // ------------------------------------------------------------------------------------------
  // sweep 2: outputs and column sums
  // ------------------------------------------------------------------------------------------
  const int row0 = rbase + rg * 32;                        // first chunk row of this wave
  const int my_row0 = row0 + lr, my_row1 = row0 + 16 + lr; // the query rows this lane's results belong to
  uint4 qa0[KS], qa1[KS], ql0[QL], ql1[QL];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const uint4 a0 = qa[0][ks], a1 = qa[1][ks], a2 = qa[2][ks], a3 = qa[3][ks];   // values, not addresses, into the select
    qa0[ks] = rg ? a2 : a0;
    qa1[ks] = rg ? a3 : a1;
  }
  if constexpr (ROPE) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint4 a0 = qlo[0][ks], a1 = qlo[1][ks], a2 = qlo[2][ks], a3 = qlo[3][ks];
      ql0[ks] = rg ? a2 : a0;
      ql1[ks] = rg ? a3 : a1;
    }
  }

  // operand read offsets inside one stage (bf16 elements), tile independent
  // K: row cq*32 + bk*16 + lr, piece ks*4 + q4
  const int k2_off = (cq * 32 + lr) * D;                                 // + bk*16 rows
  const int k2_swz0 = kswz(cq * 32 + lr), k2_swz1 = kswz(cq * 32 + 16 + lr);
  // V: the lane hands the transposing read the address of 4 dims of one row: row cq*32 + hh*16 + q4*4 + lr/4,
  // dims db*16 + (lr%4)*4 .. +3, i.e. half (lr%4)%2 of piece db*2 + (lr%4)/2
  const int v_row0 = cq * 32 + q4 * 4 + (lr >> 2), v_row1 = v_row0 + 16;
  const int v_off0 = v_row0 * D + (lr & 1) * 4, v_off1 = v_row1 * D + (lr & 1) * 4;
  const int v_swz0 = vswz(v_row0) ^ ((lr >> 1) & 1), v_swz1 = vswz(v_row1) ^ ((lr >> 1) & 1);   // piece db*2 ^ this

  f32x4_t o0[DB], o1[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d) { o0[d] = f32x4_t{0.f, 0.f, 0.f, 0.f}; o1[d] = f32x4_t{0.f, 0.f, 0.f, 0.f}; }

  // the unit's column-sum accumulators: [cache columns rounded up to a tile | chunk columns]
  const int cap_cols = (p.cap + AT_COLS - 1) / AT_COLS * AT_COLS;
  const int cs_stride = cap_cols + (p.max_chunk + AT_COLS - 1) / AT_COLS * AT_COLS;
  unsigned long long* cs_acc = p.pf_colacc + (size_t)unit * cs_stride;
  // lanes lr = 0, 4, 8, 12 leave columns 0-1, 2-3 of block 0 and 0-1, 2-3 of block 1 of their lane group's four
  float* cs_lds = sC + rg * AT_COLS + cq * 32 + (lr >> 3) * 16 + q4 * 4 + ((lr >> 2) & 1) * 2;   // + (tile & 1) * 2 * AT_COLS
  // the waves of column quarter t & 3 pass tile t's sums on (during tile t+1): thread j of the pair owns column j
  auto drain = [&](int tile) {
    const bool is_cache = tile < cache_tiles;
    const int col0 = is_cache ? tile * AT_COLS : (tile - cache_tiles) * AT_COLS;
    const float* src = sC + (tile & 1) * 2 * AT_COLS + (tid & 127);
    // Integer adds commute exactly, so the row tiles (and query heads) of a unit can meet in one accumulator per
    // column in any order and the result is still the same to the bit.  A tile's sum is below 64; 2^-40 resolves it
    // far finer than fp32 does.
    const long long fix = (long long)((src[0] + src[AT_COLS]) * COLSUM_FIX + 0.5f);
    const int col = col0 + (tid & 127);
    if (is_cache) {             // the accumulators are indexed by slot
      if (col <= last_cached) atomicAdd(cs_acc + col + (col >= fslot ? 1 : 0), (unsigned long long)fix);
    } else {
      atomicAdd(cs_acc + cap_cols + col, (unsigned long long)fix);
    }
  };

  // S^T blocks of a staged K tile: rows = columns cq*32 + bk*16 + q4*4 + i, column = the lane's query row of block 0 / 1
  auto qk2 = [&](f32x4_t (&s0)[2], f32x4_t (&s1)[2], int stage) {
    const uint16_t* kp = sK + stage * Lds::TILE_ELEMS + k2_off;
    uint4 ka[2][KS];
#pragma unroll
    for (int bk = 0; bk < 2; ++bk)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        ka[bk][ks] = *reinterpret_cast<const uint4*>(kp + bk * 16 * D + ((ks * 4 + q4) ^ (bk ? k2_swz1 : k2_swz0)) * 8);
#pragma unroll
    for (int bk = 0; bk < 2; ++bk) { s0[bk] = f32x4_t{0.f, 0.f, 0.f, 0.f}; s1[bk] = f32x4_t{0.f, 0.f, 0.f, 0.f}; }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int bk = 0; bk < 2; ++bk) {
        s0[bk] = mfma16(ka[bk][ks], qa0[ks], s0[bk]);
        s1[bk] = mfma16(ka[bk][ks], qa1[ks], s1[bk]);
      }
    if constexpr (ROPE) {            // `stage` holds the keys' hi parts, the stage after it their lo parts
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int bk = 0; bk < 2; ++bk) {
          s0[bk] = mfma16(ka[bk][ks], ql0[ks], s0[bk]);
          s1[bk] = mfma16(ka[bk][ks], ql1[ks], s1[bk]);
        }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int bk = 0; bk < 2; ++bk) {
          const uint4 kl = *reinterpret_cast<const uint4*>(kp + Lds::TILE_ELEMS + bk * 16 * D +
                                                           ((ks * 4 + q4) ^ (bk ? k2_swz1 : k2_swz0)) * 8);
          s0[bk] = mfma16(kl, qa0[ks], s0[bk]);
          s1[bk] = mfma16(kl, qa1[ks], s1[bk]);
        }
    }
  };
  // bf16 pairs (-1, 0) and (0, -1).  Kept opaque in scalar registers: as immediates, the second has the bit
  // pattern of the fp32 inline constant -1.0, which a packed 16-bit operand does not read as these two halves.
  unsigned minus_one_lo = 0x0000BF80u, minus_one_hi = 0xBF800000u;
  asm volatile("" : "+s"(minus_one_lo), "+s"(minus_one_hi));
  // probabilities in place of one row block's 8 logits
  auto probs = [&](f32x4_t (&s)[2], float neg_ml) {
#pragma unroll
    for (int bk = 0; bk < 2; ++bk)
#pragma unroll
      for (int i = 0; i < 4; ++i) s[bk][i] = fast_exp2(fmaf(s[bk][i], sc, neg_ml));
  };
  // ... as the packed hi / lo P^T operands (k-slots 0-3 = block 0, i = 0..3; k-slots 4-7 = block 1); the values are used up.
  // p - hi is one instruction each, a bf16 dot product against (-1, 0) / (0, -1) added to p.  One statement of the
  // three-operand form: left to itself the compiler takes the two-operand one and a copy of p for each.  Three wait
  // states between such a product and the first use of its result.
  auto split = [&](const f32x4_t (&s)[2], uint4& phi, uint4& plo) {
    phi = make_uint4(pack_bf16(s[0][0], s[0][1]), pack_bf16(s[0][2], s[0][3]), pack_bf16(s[1][0], s[1][1]),
                     pack_bf16(s[1][2], s[1][3]));
    if constexpr (D == 128) {
      float l0 = s[0][0], l1 = s[0][1], l2 = s[0][2], l3 = s[0][3], l4 = s[1][0], l5 = s[1][1], l6 = s[1][2], l7 = s[1][3];
      asm("v_dot2_f32_bf16 %0, %8, %12, %0\n\t"
          "v_dot2_f32_bf16 %1, %8, %13, %1\n\t"
          "v_dot2_f32_bf16 %2, %9, %12, %2\n\t"
          "v_dot2_f32_bf16 %3, %9, %13, %3\n\t"
          "v_dot2_f32_bf16 %4, %10, %12, %4\n\t"
          "v_dot2_f32_bf16 %5, %10, %13, %5\n\t"
          "v_dot2_f32_bf16 %6, %11, %12, %6\n\t"
          "v_dot2_f32_bf16 %7, %11, %13, %7\n\t"
          "s_nop 2"
          : "+v"(l0), "+v"(l1), "+v"(l2), "+v"(l3), "+v"(l4), "+v"(l5), "+v"(l6), "+v"(l7)
          : "v"(phi.x), "v"(phi.y), "v"(phi.z), "v"(phi.w), "s"(minus_one_lo), "s"(minus_one_hi));
      plo = make_uint4(pack_bf16(l0, l1), pack_bf16(l2, l3), pack_bf16(l4, l5), pack_bf16(l6, l7));
    } else {                                  // (at head_dim 64 the statement's eight live values do not fit the registers)
      const unsigned h[4] = {phi.x, phi.y, phi.z, phi.w};
      unsigned lo[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bf16x2_t hv = __builtin_bit_cast(bf16x2_t, h[e]);
        const float l0 = __builtin_amdgcn_fdot2_f32_bf16(hv, __builtin_bit_cast(bf16x2_t, minus_one_lo), s[e >> 1][(e & 1) * 2], false);
        const float l1 = __builtin_amdgcn_fdot2_f32_bf16(hv, __builtin_bit_cast(bf16x2_t, minus_one_hi), s[e >> 1][(e & 1) * 2 + 1], false);
        lo[e] = pack_bf16(l0, l1);
      }
      plo = make_uint4(lo[0], lo[1], lo[2], lo[3]);
    }
  };
  // the two row blocks' probabilities added, per column
  auto add_blocks = [&](const f32x4_t (&s0)[2], const f32x4_t (&s1)[2], float (&x)[8]) {
#pragma unroll
    for (int bk = 0; bk < 2; ++bk)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[bk * 4 + i] = s0[bk][i] + s1[bk][i];
  };
  // what follows the logits of tile t, in three pieces: mask + probabilities, O^T += V^T P^T, column sums
  auto mask_tile = [&](f32x4_t (&s0)[2], f32x4_t (&s1)[2], int tile) {
    if (tile < full_tiles) return;
    const bool is_cache = tile < cache_tiles;
    const int col0 = is_cache ? tile * AT_COLS : (tile - cache_tiles) * AT_COLS;
    // only tiles that touch the end of the cache or the causal diagonal need a mask (wave uniform)
    const bool need_mask = is_cache ? (col0 + AT_COLS - 1 > last_cached) : (col0 + AT_COLS - 1 > row0);
    if (need_mask) {
      const int cbase = col0 + cq * 32 + q4 * 4;
      const int lim0 = is_cache ? last_cached : my_row0, lim1 = is_cache ? last_cached : my_row1;   // last visible column
#pragma unroll
      for (int bk = 0; bk < 2; ++bk)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int col = cbase + bk * 16 + i;
          s0[bk][i] = col <= lim0 ? s0[bk][i] : -INFINITY;   // exp2 gives exactly 0
          s1[bk][i] = col <= lim1 ? s1[bk][i] : -INFINITY;
        }
    }
  };
  // O^T += V^T P^T : A = V^T[d][the quarter's 8 k-slot columns of this lane group], B = P^T (hi and lo parts)
  auto read_v = [&](uint4 (&va)[DB], int tile) {
    const uint16_t* vp = sV + (tile & 1) * Lds::TILE_ELEMS;
#pragma unroll
    for (int d = 0; d < DB; ++d) {
      const short4_t t0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_t*)(vp + v_off0 + ((d * 2) ^ v_swz0) * 8));
      const short4_t t1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_t*)(vp + v_off1 + ((d * 2) ^ v_swz1) * 8));
      const uint2 a0 = __builtin_bit_cast(uint2, t0), a1 = __builtin_bit_cast(uint2, t1);
      va[d] = make_uint4(a0.x, a0.y, a1.x, a1.y);
    }
  };
  auto pv = [&](const uint4 (&va)[DB], const uint4& phi0, const uint4& plo0, const uint4& phi1, const uint4& plo1) {
#pragma unroll
    for (int d = 0; d < DB; ++d) { o0[d] = mfma16(va[d], phi0, o0[d]); o1[d] = mfma16(va[d], phi1, o1[d]); }
#pragma unroll
    for (int d = 0; d < DB; ++d) { o0[d] = mfma16(va[d], plo0, o0[d]); o1[d] = mfma16(va[d], plo1, o1[d]); }
  };
  // column sums over this wave's 32 rows
  auto colsums = [&](const float (&x)[8], int tile) {
    const float2 c = row16_sum8(x);
    if ((lr & 3) == 0) *reinterpret_cast<float2*>(cs_lds + (tile & 1) * 2 * AT_COLS) = c;
  };

  // what follows the logits of tile t.  All of V's operands are requested before the probabilities are worked out, which
  // hides their way from LDS (read as they are needed, two blocks at a time, they cost a wait each).
  auto finish_tile = [&](f32x4_t (&s0)[2], f32x4_t (&s1)[2], int t) {
    uint4 va[DB], phi0, plo0, phi1, plo1;
    float x[8];
    read_v(va, t);
    mask_tile(s0, s1, t);
    probs(s0, neg_ml0);
    probs(s1, neg_ml1);
    add_blocks(s0, s1, x);
    colsums(x, t);
    split(s0, phi0, plo0);
    split(s1, phi1, plo1);
    pv(va, phi0, plo0, phi1, plo1);
  };
  f32x4_t s0[2], s1[2];
  if constexpr (!ROPE) {
    // Iteration t: request K and V of tile t+1 into the other stages, then take tile t from its logits to its column sums.
    // (Forming the logits a tile ahead took 254 registers instead of 204, left none for V's operands and was slower: 57.9 us
    // against 55.5 at 512 tokens into 2048 slots; at head_dim 64 it spilled: 77.0 against 72.5.)
    issue_tile(Ku, Kcu, kchunk_row_stride, 0, 0, kswz);
    issue_tile(Vu, Vcu, chunk_row_stride, 0, 2, vswz);
    wait_vmcnt<0>();
    __syncthreads();
    for (int t = 0; t < ntiles; ++t) {
      if (t > 0 && cq == ((t - 1) & 3)) drain(t - 1);
      if (t + 1 < ntiles) {
        issue_tile(Ku, Kcu, kchunk_row_stride, t + 1, (t + 1) & 1, kswz);
        issue_tile(Vu, Vcu, chunk_row_stride, t + 1, 2 + ((t + 1) & 1), vswz);
      }
      qk2(s0, s1, t & 1);
      finish_tile(s0, s1, t);
      wait_vmcnt<0>();                   // this iteration's requests are the next one's operands
      __syncthreads();
    }
  } else {
    // ROPE: one K pair (hi in K stage 0, lo in K stage 1) and two V stages.  Iteration t: with the pair of tile t landed,
    // form its logits; once every wave has done so, request the pair of tile t+1 into the same two stages and V of tile
    // t+1 into V stage (t+1)&1, which held tile t-1, and finish tile t while they are on their way.
    auto issue_pair = [&](int t) {
      issue_tile(Ku, Kcu, kchunk_row_stride, t, 0, kswz);
      issue_tile(Ku + klo_off, Kcu + klo_off, kchunk_row_stride, t, 1, kswz);
      issue_tile(Vu, Vcu, chunk_row_stride, t, 2 + (t & 1), vswz);
    };
    issue_pair(0);
    for (int t = 0; t < ntiles; ++t) {
      wait_vmcnt<0>();                   // the pair and V of tile t
      __syncthreads();                   // ... for every wave; and every wave is done with V of tile t-1 and tile t-1's sums
      if (t > 0 && cq == ((t - 1) & 3)) drain(t - 1);
      qk2(s0, s1, 0);
      __syncthreads();                   // every wave has read the pair
      if (t + 1 < ntiles) issue_pair(t + 1);
      finish_tile(s0, s1, t);
    }
    __syncthreads();                     // the last tile's sums are in LDS
  }
  if (cq == ((ntiles - 1) & 3)) drain(ntiles - 1);     // the last tile's sums (its barrier has passed)

  // ---- add the four column quarters of every row group through LDS ----
  float* xch = reinterpret_cast<float*>(pf_smem);           // [6 waves][2 blocks][DB*4][64 lanes]
  constexpr int XN = DB * 4;
  if (cq > 0) {
    float* dst = xch + (((cq - 1) * 2 + rg) * 2 * XN) * 64 + lane;
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int i = 0; i < 4; ++i) { dst[(d * 4 + i) * 64] = o0[d][i]; dst[(XN + d * 4 + i) * 64] = o1[d][i]; }
  }
  __syncthreads();
  if (cq > 0) return;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const float* src = xch + ((c * 2 + rg) * 2 * XN) * 64 + lane;
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int i = 0; i < 4; ++i) { o0[d][i] += src[(d * 4 + i) * 64]; o1[d][i] += src[(XN + d * 4 + i) * 64]; }
  }
  auto finish = [&](int my_row, const f32x4_t (&oacc)[DB]) {
    if (my_row < L) {
      float* op = out + (((size_t)b * L + my_row) * p.H + h) * D;
#pragma unroll
      for (int d = 0; d < DB; ++d)
        *reinterpret_cast<float4*>(op + d * 16 + q4 * 4) = make_float4(oacc[d][0], oacc[d][1], oacc[d][2], oacc[d][3]);
    }
  };
  finish(my_row0, o0);
  finish(my_row1, o1);
}

// ---------------------------------------------------------------------------------------------
// attend with the logits kept in registers
// ---------------------------------------------------------------------------------------------
// One workgroup owns 32 query rows of one head and keeps all their logits: a wave takes 32-column blocks w, w + 8, .. of
// the visible columns, up to ten of them, 16 registers each.  Queries meet keys once and every logit has one exponential,
// where the two-sweep kernel above does both twice.  What is left of its structure:
//   logits   S^T = K Q^T with v_mfma_f32_32x32x16_bf16, a lane holding 16 columns of one row.  The exponentials of block t
//            are taken while the products of block t + 1 run, against the lane's running maximum; what each block's are
//            relative to is kept (ref) instead of rescaling them.
//   merge    maxima and sums: two lanes of a row, then eight waves through LDS; one barrier.
//   O^T      += V^T P^T.  A lane's logits are the B operand as they lie (with the columns of a k-step in the order the
//            transposing reads of V fetch them in); P is split into two bf16 halves as above.
//   sums     of a block's columns over the 32 rows stay inside the wave and go straight to the unit's accumulators.
// A wave reads only what it requested itself, two blocks ahead, so the blocks take no barrier.  Lane-dependent addresses
// are worked out anew where they are used: held, they would spill at head_dim 128 (255 registers of 256 are in use there, 256
// with ROPE; 227 at head_dim 64).
//
// Bound by the vector ALU's issue (a block costs a wave some 440 cycles of it for the logits and 500 for O, the products
// of which take 270 and 550 of the matrix pipe) and by the path from L2: a workgroup takes in every K and V row, 604 MB
// for 512 tokens into 2048 slots at 32 heads, 5.3 us for a workgroup's keys alone, where 8.3 are measured with the
// arithmetic and 5.0 for the arithmetic alone; for O 5.0, 9.6 and 8.1.  Starting up, merging and writing out take 7 us of a
// workgroup's 26, which is why short chunks gain most: one sequence of 8 KV heads, 100 tokens into 1024 slots, 38.9 ->
// 23.0 us a call; 32 heads, 32 into 2048, 53.4 -> 31.6; 512 into 2048 71.4 -> 66.1, with re-assigned positions 110.3 -> 94.3.
// Measured and not kept: v_dot2 for the remainder of the split (it runs on the matrix pipe: 5 % longer), twelve waves of
// seven blocks at head_dim 64 (no change), wave priorities around the products or by wave (no change).
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

constexpr int RES_ROWS = 32;                       // query rows of a workgroup
constexpr int RES_WAVES = AT_THREADS / 64;
constexpr int RES_BLOCKS = 10;                     // 32-column blocks of logits a wave holds: 160 registers
typedef unsigned uint4v_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const uint4v_t lds_uint4_t;

template <int D, bool ROPE>
struct ResidentLds {
  static constexpr int STAGE = 32 * D * 2;                          // one block of K (one part of it with ROPE) or V rows
  static constexpr int STAGES = 2;
  static constexpr int RING = RES_WAVES * STAGES * STAGE;                   // every wave its own stages
  static_assert(STAGES * STAGE == RES_ROWS * D * 4, "a wave's stages hold its outputs at the end");
  static constexpr int STATS = RING;                                // [waves][32 rows] (max, sum)
  static constexpr int QLO = STATS + RES_WAVES * RES_ROWS * 8;              // the queries' second parts, as operands (ROPE)
  static constexpr int BYTES = QLO + (ROPE ? RES_ROWS * D * 2 : 0);
};

__device__ inline f32x16_t mfma32(const uint4& a, const uint4& b, const f32x16_t& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// the same address, in scalar registers
__device__ inline const char* scalar_ptr(const void* ptr) {
  const uint64_t a = (uint64_t)(uintptr_t)ptr;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a), hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
  return reinterpret_cast<const char*>((uintptr_t)((uint64_t)hi << 32 | lo));
}

template <int D, bool ROPE>
__global__ __launch_bounds__(AT_THREADS, 2) void prefill_attend_resident_kernel(Params p, const uint16_t* __restrict__ Q,
                                                                             const uint16_t* __restrict__ Kc,
                                                                             const uint16_t* __restrict__ Vc, int L,
                                                                             int row_tiles, float* __restrict__ out) {
  using Lds = ResidentLds<D, ROPE>;
  constexpr int KS = D / 16;                         // k-steps of the q.k contraction
  constexpr int DB = D / 32;                         // 32-wide blocks of the head dimension
  constexpr int PARTS = D / 8, ROWB = D * 2;         // 16-byte pieces, bytes of a row
  constexpr int RPC = 1024 / ROWB;                   // rows per 1 KB request
  constexpr int REQ = 32 / RPC;                      // requests per block
  constexpr int KPARTS = ROPE ? 2 : 1;
  extern __shared__ __attribute__((aligned(1024))) uint16_t pf_smem[];
  char* smem = reinterpret_cast<char*>(pf_smem);

  // a unit's row tiles share one XCD's L2 (see the two-sweep kernel); the longest row tiles first
  const int n_items = row_tiles * p.G * p.U, per_xcd = (n_items + 7) / 8;
  const int item = ((int)blockIdx.x % 8) * per_xcd + (int)blockIdx.x / 8;
  if (item >= n_items) return;
  const int row_tile = __builtin_amdgcn_readfirstlane(row_tiles - 1 - item % row_tiles);
  const int head = __builtin_amdgcn_readfirstlane(item / row_tiles);                 // (unit, query head of its group)
  const int unit = __builtin_amdgcn_readfirstlane(head / p.G), g = head - unit * p.G;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r32 = lane & 31, half = lane >> 5, lr = lane & 15, g1 = (lane >> 4) & 1;
  const int b = __builtin_amdgcn_readfirstlane(unit / p.Hkv), kvh = unit - b * p.Hkv, h = kvh * p.G + g;
  // B operands: query row r32, dims 16 ks + 8 half .. + 7 (rows past the chunk repeat its last row)
  const uint16_t* Qsrc = ROPE ? p.pf_qrot : Q;
  const size_t q_part = (size_t)p.B * p.max_chunk * p.H * D;      // pf_qrot: [hi, lo][B][max_chunk][H][D]
  const int q_rows = ROPE ? p.max_chunk : L;
  const uint16_t* qp = Qsrc + (((size_t)b * q_rows + min(row_tile * RES_ROWS + r32, L - 1)) * p.H + h) * D + half * 8;
  uint4 qa[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qa[ks] = *reinterpret_cast<const uint4*>(qp + ks * 16);
  const int* meta = p.meta + (size_t)unit * META_STRIDE;
  const int n = __builtin_amdgcn_readfirstlane(meta[META_N]), fslot = __builtin_amdgcn_readfirstlane(meta[META_FREE]);
  const int rbase = row_tile * RES_ROWS, my_row = rbase + r32;
  // columns: the cached tokens' slots in slot order without the free one, then the chunk's tokens; blocks of 32 of either
  const int cache_blk = (n + 31) / 32, nblk = cache_blk + row_tile + 1;
  const int cnt = (nblk - wave + RES_WAVES - 1) / RES_WAVES;                           // this wave's blocks: wave, wave + RES_WAVES, ..

  const size_t krot_rows = (size_t)p.cap + p.max_chunk;            // pf_krot: [U][hi, lo][cap + max_chunk][D]
  const uint16_t* Ku = ROPE ? p.pf_krot + (size_t)unit * 2 * krot_rows * D : (const uint16_t*)p.K + (size_t)unit * p.cap * D;
  const uint16_t* Vu = (const uint16_t*)p.V + (size_t)unit * p.cap * D;
  const int vstride = p.Hkv * D, kstride = ROPE ? D : vstride;     // of the chunk's own rows
  const uint16_t* Kcu = ROPE ? Ku + (size_t)p.cap * D : Kc + ((size_t)b * L * p.Hkv + kvh) * D;
  const uint16_t* Vcu = Vc + ((size_t)b * L * p.Hkv + kvh) * D;
  const size_t klo_off = krot_rows * D;

  // ---- requests: the wave's blocks of K (with ROPE the hi, then the lo part of each), then its blocks of V ----
  // slot s of row r of a staged block holds 16-byte piece s ^ KSWZ(r) or s ^ VSWZ(r), so that the operand reads touch
  // every bank once
  auto kswz = [](int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); };
  auto vswz = [](int r) { return D == 128 ? ((r & 3) << 2) : (((r >> 1) & 1) << 2); };
  const int a_lrow = lane / PARTS, a_slot = lane % PARTS;
  const unsigned k_from = a_lrow * ROWB + (a_slot ^ kswz(a_lrow)) * 16;        // of request x: ^ (x % 4) * 64 or (x % 2) * 64
  static_assert(D == 64 || D == 128, "swizzles are written for head_dim 64 and 128");
  const unsigned ring = __builtin_amdgcn_readfirstlane(lds_address(pf_smem)) + wave * (Lds::STAGES * Lds::STAGE);
  // bit i: the wave's i-th block is a run of cache rows / one that starts a row further on, behind the free slot / reaches
  // past what the first row sees
  unsigned run_blocks, moved_blocks, mask_blocks;
  {
    const int blk = wave + lane * RES_WAVES;
    const bool is_cache = blk < cache_blk;
    const int col0 = (is_cache ? blk : blk - cache_blk) * 32, from = fslot - col0;
    run_blocks = (unsigned)__ballot(is_cache && col0 + 32 <= n && (from <= 0 || from >= 32));
    moved_blocks = (unsigned)__ballot(from <= 0);
    mask_blocks = (unsigned)__ballot(col0 + 31 > (is_cache ? n - 1 : rbase));
  }
  auto request_rows = [&](const uint16_t* cache_src, const uint16_t* chunk_src, int stride, int i, unsigned m0, auto is_k) {
    int l = lane;
    asm volatile("" : "+v"(l));                      // worked out anew each time: held, this would take the logits' registers
    const unsigned v_from = l / PARTS * ROWB + (l % PARTS ^ vswz(l / PARTS)) * 16;            // the same for every request
    auto from_of = [&](int x) { return decltype(is_k)::value ? k_from ^ (unsigned)((D == 128 ? x & 3 : x & 1) * 64) : v_from; };
    if (run_blocks >> i & 1) {
      const char* base = scalar_ptr(reinterpret_cast<const char*>(cache_src) + (unsigned)((wave + i * RES_WAVES) * 32 * ROWB) +
                                    (moved_blocks >> i & 1) * ROWB);
#pragma unroll
      for (int x = 0; x < REQ; x += 4)
        async_copy16_run(base + x * 1024, m0 + x * 1024, from_of(x), from_of(x + 1), from_of(x + 2), from_of(x + 3));
    } else {                                         // rows past the last one that exists repeat it (they are masked)
      const int blk = wave + i * RES_WAVES;
      const bool is_cache = blk < cache_blk;
      const int col0 = (is_cache ? blk : blk - cache_blk) * 32;
      const int rstride = is_cache ? D : stride;
      const char* base = scalar_ptr((is_cache ? cache_src : chunk_src) + (size_t)col0 * rstride);
      const int lim = (is_cache ? p.cap : L) - 1 - col0, moved_from = is_cache ? fslot - col0 : 32;
#pragma unroll 1
      for (int x = 0; x < REQ; ++x) {
        const int c = x * RPC + l / PARTS, row = min(c + (c >= moved_from ? 1 : 0), lim);
        async_copy16_offset(base, (unsigned)(row * rstride) * 2 + (from_of(x) & (ROWB - 1)), m0 + x * 1024);
      }
    }
  };
  const int nk = cnt * KPARTS;
  auto request_k = [&](int u) {                      // u-th part-block of K
    const size_t off = ROPE && (u & 1) ? klo_off : 0;
    request_rows(Ku + off, Kcu + off, kstride, ROPE ? u >> 1 : u, ring + (u & 1) * Lds::STAGE, std::true_type{});
  };
  auto request_v = [&](int i) {                      // i-th block of V
    if (i < cnt) request_rows(Vu, Vcu, vstride, i, ring + ((nk + i) & 1) * Lds::STAGE, std::false_type{});
  };
  auto request_after_k = [&](int u) { if (u < nk) request_k(u); else request_v(u - nk); };
  // block u of K and V together has landed: of what was requested after it, only block u + 1 may be out
  auto landed = [&](int u) { if (u + 1 < nk + cnt) wait_vmcnt<REQ>(); else wait_vmcnt<0>(); };
  // a staged block's operand reads have returned: its stage can be requested anew
  auto reads_done = [&]() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };

  const uint4* qlo = reinterpret_cast<const uint4*>(smem + Lds::QLO) + lane;      // [KS][64 lanes]
  if constexpr (ROPE) {
    static_assert(KS <= 8, "one k-step per wave");
    if (wave < KS) reinterpret_cast<uint4*>(smem + Lds::QLO)[wave * 64 + lane] = *reinterpret_cast<const uint4*>(qp + q_part + wave * 16);
    __syncthreads();
  }
  if (cnt > 0) {
    request_k(0);
    request_after_k(1);
  }

  // ------------------------------------------------------------------------------------------
  // logits, and their exponentials against the running maximum of the lane
  // ------------------------------------------------------------------------------------------
  const float sc = p.scale_log2e;
  f32x16_t s[RES_BLOCKS];            // S^T: component e is column 8 (e / 4) + 4 half + e % 4 of row r32
  float ref[RES_BLOCKS];             // what block t's exponentials are relative to (scaled log2 domain)
  float m_run = NEG_BIG, l_run = 0.f;
  const unsigned stages = lds_address(pf_smem) + wave * (Lds::STAGES * Lds::STAGE);
  const unsigned k_lane = stages + r32 * ROWB + (half ^ kswz(r32)) * 16;       // k-step ks: piece 2 ks + half
  auto mask = [&](f32x16_t& x, int t) {
    if (mask_blocks >> t & 1) {
      const int blk = wave + t * RES_WAVES;
      const bool is_cache = blk < cache_blk;
      const int lim = (is_cache ? n - 1 - blk * 32 : my_row - (blk - cache_blk) * 32) - half * 4;
#pragma unroll
      for (int e = 0; e < 16; ++e) x[e] = (e >> 2) * 8 + (e & 3) <= lim ? x[e] : -INFINITY;
    }
  };
  auto exps = [&](f32x16_t& x, int t) {
    float mx = fmaxf(x[0], x[1]);
#pragma unroll
    for (int e = 2; e < 16; e += 2) mx = max3(mx, x[e], x[e + 1]);
    const float m_new = fmaxf(m_run, mx * sc);
#pragma unroll
    for (int e = 0; e < 16; ++e) x[e] = fast_exp2(fmaf(x[e], sc, -m_new));
    const float s0 = (x[0] + x[1]) + (x[2] + x[3]), s1 = (x[4] + x[5]) + (x[6] + x[7]);
    const float s2 = (x[8] + x[9]) + (x[10] + x[11]), s3 = (x[12] + x[13]) + (x[14] + x[15]);
    l_run = fmaf(l_run, fast_exp2(m_run - m_new), (s0 + s1) + (s2 + s3));
    m_run = m_new;
    ref[t] = m_new;
  };
  auto read_k = [&](uint4 (&k)[KS], int u) {
    unsigned a = k_lane;
    asm volatile("" : "+v"(a));
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) k[ks] = __builtin_bit_cast(uint4, *(lds_uint4_t*)(uintptr_t)((a ^ (ks * 32)) + (u & 1) * Lds::STAGE));
  };
#pragma unroll
  for (int t = 0; t < RES_BLOCKS; ++t) {
    if (t < cnt) {
      f32x16_t acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      uint4 k[KS];
      landed(t * KPARTS);
      read_k(k, t * KPARTS);
      reads_done();
      request_after_k(t * KPARTS + 2);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) acc = mfma32(k[ks], qa[ks], acc);
      if constexpr (ROPE) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) acc = mfma32(k[ks], qlo[ks * 64], acc);
        landed(t * 2 + 1);
        read_k(k, t * 2 + 1);
        reads_done();
        request_after_k(t * 2 + 3);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) acc = mfma32(k[ks], qa[ks], acc);
      }
      s[t] = acc;
      if (t > 0) exps(s[t - 1 < 0 ? 0 : t - 1], t - 1);          // while the products run
      mask(s[t], t);
    }
  }
#pragma unroll
  for (int t = 0; t < RES_BLOCKS; ++t)
    if (t == cnt - 1) exps(s[t], t);

  // ---- row statistics: the two lanes of a row, then the waves ----
  float* st = reinterpret_cast<float*>(smem + Lds::STATS);
  {
    const float mo = __shfl_xor(m_run, 32, 64), lo = __shfl_xor(l_run, 32, 64);
    const float mn = fmaxf(m_run, mo);
    const float l = l_run * fast_exp2(m_run - mn) + lo * fast_exp2(mo - mn);
    if (half == 0) *reinterpret_cast<float2*>(st + (wave * RES_ROWS + r32) * 2) = make_float2(mn, l);
  }
  // (not __syncthreads, which would wait for the blocks of V on their way; here and below only LDS passes between waves)
  auto block_sync = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  block_sync();
  float mx = NEG_BIG, sum = 0.f;
  {
    float2 w[RES_WAVES];
#pragma unroll
    for (int i = 0; i < RES_WAVES; ++i) w[i] = *reinterpret_cast<const float2*>(st + (i * RES_ROWS + r32) * 2);
#pragma unroll
    for (int i = 0; i < RES_WAVES; ++i) mx = fmaxf(mx, w[i].x);
#pragma unroll
    for (int i = 0; i < RES_WAVES; ++i) sum += w[i].y * fast_exp2(w[i].x - mx);
  }
  const float inv = my_row < L ? 1.0f / sum : 0.f;                 // rows past the chunk must not reach the column sums
  // to probabilities: the first blocks while the matrix pipe works on the block before them, the others here, because there
  // is no register for their references later
  constexpr int LATE = 4;
  auto scale = [&](int t) {
    const float f = fast_exp2(ref[t] - mx) * inv;
#pragma unroll
    for (int e = 0; e < 16; ++e) s[t][e] *= f;
  };
#pragma unroll
  for (int t = LATE; t < RES_BLOCKS; ++t)
    if (t < cnt) scale(t);

  // ------------------------------------------------------------------------------------------
  // O^T += V^T P^T, column sums
  // ------------------------------------------------------------------------------------------
  f32x16_t o[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[d][e] = 0.f;
  // the lane's address for the transposing read: row 4 half + lr / 4 of a k-step's 16 (second read: 8 rows on), dims
  // 32 db + 16 g1 + 4 (lr % 4) ..
  const int v_row = half * 4 + (lr >> 2);
  const unsigned v_lane = stages + v_row * ROWB + (lr & 1) * 8 + ((g1 * 2 + ((lr >> 1) & 1)) ^ vswz(v_row)) * 16;
  // one k-step's eight probabilities as P^T operands, two bf16 parts each (see the two-sweep kernel)
  auto split = [&](const f32x16_t& x, int k, uint4& phi, uint4& plo) {
    phi = make_uint4(pack_bf16(x[k], x[k + 1]), pack_bf16(x[k + 2], x[k + 3]), pack_bf16(x[k + 4], x[k + 5]), pack_bf16(x[k + 6], x[k + 7]));
    const unsigned h[4] = {phi.x, phi.y, phi.z, phi.w};
    unsigned l[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      l[e] = pack_bf16(x[k + e * 2] - __uint_as_float(h[e] << 16), x[k + e * 2 + 1] - __uint_as_float(h[e] & 0xffff0000u));
    plo = make_uint4(l[0], l[1], l[2], l[3]);
  };
  // the sums of a block's 32 columns over the 32 rows; the probabilities are used up
  auto column_sums = [&](f32x16_t& x) {
    float y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {                    // the two 16-lane halves of the rows: lanes g1 = 0 take column e, g1 = 1 column e + 8
      const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[e]), __float_as_uint(x[e + 8]), false, false);
      y[e] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    }
    const float2 c = row16_sum8(y);
    return lr & 1 ? c.y : c.x;
  };
  // integer adds commute exactly: the sums are the same to the bit whatever order a unit's row tiles and heads arrive in
  const int cap_cols = (p.cap + AT_COLS - 1) / AT_COLS * AT_COLS;
  const int cs_stride = cap_cols + (p.max_chunk + AT_COLS - 1) / AT_COLS * AT_COLS;
  unsigned long long* cs_acc = p.pf_colacc + (size_t)unit * cs_stride;
  auto add_columns = [&](int t, float sum) {         // lanes lr % 4 < 2 hold one column each
    const int blk = wave + t * RES_WAVES;
    const bool is_cache = blk < cache_blk;
    int l = lane;
    asm volatile("" : "+v"(l));
    const int c = (l >> 4 & 1) * 8 + (l >> 2 & 3) * 2 + (l & 1);         // the accumulator whose sum column_sums left here
    const int col = (is_cache ? blk : blk - cache_blk) * 32 + (c >> 2) * 8 + (l >> 5) * 4 + (c & 3);
    const int at = is_cache ? col + (col >= fslot ? 1 : 0) : cap_cols + col;
    const float x = sum * 256.f, whole = floorf(x);  // 2^40 times the sum, in two 32-bit words
    const unsigned long long fix = (unsigned long long)(unsigned)whole << 32 | (unsigned)rintf((x - whole) * 0x1p32f);
    if ((l & 2) == 0 && col < (is_cache ? n : L)) atomicAdd(cs_acc + (unsigned)at, fix);
  };
  float csum;
  uint4 phi[2], plo[2];
  auto prepare = [&](int t) {
    if (t < LATE) scale(t);
    split(s[t], 0, phi[0], plo[0]);
    split(s[t], 8, phi[1], plo[1]);
    csum = column_sums(s[t]);
  };
  if (cnt > 0) prepare(0);
#pragma unroll
  for (int t = 0; t < RES_BLOCKS; ++t) {
    if (t < cnt) {
      const int u = nk + t;
      landed(u);
      unsigned va0 = v_lane + (u & 1) * Lds::STAGE;
      asm volatile("" : "+v"(va0));
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        uint4 va[DB];
#pragma unroll
        for (int d = 0; d < DB; ++d) {
          const unsigned a = (va0 ^ (d * 64)) + ks * 16 * ROWB;
          const short4_t t0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_t*)(uintptr_t)a);
          const short4_t t1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_t*)(uintptr_t)(a + 8 * ROWB));
          const uint2 a0 = __builtin_bit_cast(uint2, t0), a1 = __builtin_bit_cast(uint2, t1);
          va[d] = make_uint4(a0.x, a0.y, a1.x, a1.y);
        }
        if (ks == 1) {
          add_columns(t, csum);                      // (ahead of the requests, which are waited for later than it)
          reads_done();
          request_v(t + 2);
        }
#pragma unroll
        for (int d = 0; d < DB; ++d) o[d] = mfma32(va[d], phi[ks], o[d]);
#pragma unroll
        for (int d = 0; d < DB; ++d) o[d] = mfma32(va[d], plo[ks], o[d]);
      }
      if (t + 1 < RES_BLOCKS) prepare(t + 1);        // (of no use behind the last one, and of no harm)
    }
  }

  // ---- add the waves' outputs ----
  // a wave's own stages take its outputs; 16-byte piece x of row r sits in slot x ^ r
  constexpr int OP = D / 4;
  float4* xo = reinterpret_cast<float4*>(smem + wave * (Lds::STAGES * Lds::STAGE));
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      xo[r32 * OP + ((d * 8 + q * 2 + half) ^ (r32 & (OP - 1)))] = make_float4(o[d][q * 4], o[d][q * 4 + 1], o[d][q * 4 + 2], o[d][q * 4 + 3]);
  block_sync();
  for (int y = tid; y < RES_ROWS * OP; y += AT_THREADS) {
    const int row = y / OP, x = y % OP;
    if (rbase + row >= L) break;                     // rows ascend with y
    const float4* src = reinterpret_cast<const float4*>(smem) + row * OP + (x ^ (row & (OP - 1)));
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < RES_WAVES; ++w) {
      const float4 v = src[w * RES_ROWS * OP];
      a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w;
    }
    *reinterpret_cast<float4*>(out + (((size_t)b * L + rbase + row) * p.H + h) * D + x * 4) = a;
  }
}

// ---------------------------------------------------------------------------------------------
// attend for fp32 storage
// ---------------------------------------------------------------------------------------------
// The same four steps (logits, row softmax, output, column sums) with v_mfma_f32_16x16x4_f32: fp32 operands, fp32
// multiply-adds, so the results are held to 1e-5 as the vector ALU's would be.  A workgroup takes 16 query rows of
// one head, wave w the 16-column blocks w, w + 8, ..; operands come straight from global memory in 16-byte lane loads,
// because the order of a contraction is free as long as both operands agree on it:
//   S^T = K Q^T    lane (lr, q4) loads dims 16 s + 4 q4 .. + 3 of K row lr and of Q row lr; component j of the four is
//                  k-slot q4 of the j-th instruction.
//   O^T += V^T P^T S^T's accumulator i of a lane is column 4 q4 + i of row lr, which is k-slot q4 of the B operand of the
//                  instruction for those columns; its A operand is V[column 4 q4 + i][64 x + 4 lr + e], one component of
//                  a 16-byte lane load for each of four instructions (so a lane's accumulators are 4 adjacent dims).
// Sweep 1 forms the logits, parks them in LDS (a wave reads only what it wrote) and keeps a running (max, sum) per lane;
// sweep 2 turns them into probabilities.  The first `park_blocks` blocks are parked (all of them up to 2048 columns); the
// logits of the rest are formed again.
// Bound by matrix issue (one 16x16x4 instruction is 32 cycles: 7.7 us here) and by the latency of the first blocks.
// Measured at 8 heads x 200 tokens into 512 slots, head_dim 64: 17.9 us, against 380 us for one query row at a time on
// the vector ALUs with shuffled dot products; the whole call 27 us against 397.
constexpr int F32_THREADS = 512;
constexpr int F32_WAVES = F32_THREADS / 64;
constexpr int F32_ROWS = 16;
constexpr int F32_PARK_BLOCKS = 128;               // 1 KB of LDS each
constexpr int F32_MAX_COLS = 10240;                // visible columns the call accepts

template <int D>
constexpr size_t f32_merge_bytes() { return (size_t)F32_WAVES * F32_ROWS * (D + 4) * sizeof(float); }

// ROPE (positions re-assigned to cache ranks): queries and keys are read, already turned to their ranks, from the scratch
// prefill_turn_f32_kernel fills (the same memory the bf16 path keeps its two-part copies in).
template <int D, bool ROPE>
__global__ __launch_bounds__(F32_THREADS) void prefill_attend_f32_kernel(Params p, const float* __restrict__ Q,
                                                                         const float* __restrict__ Kc,
                                                                         const float* __restrict__ Vc, int L,
                                                                         int park_blocks, float* __restrict__ out) {
  constexpr int KQ = D / 16, VX = D / 64;          // 16-byte pieces per lane of a K row block, and of one V row
  extern __shared__ __attribute__((aligned(16))) float f32_smem[];      // parked logits; at the end the waves' outputs
  __shared__ float st[F32_WAVES][F32_ROWS][2];
  const int unit = blockIdx.z, g = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, q4 = lane >> 4;
  const int kvh = unit % p.Hkv, b = unit / p.Hkv, h = kvh * p.G + g;
  const ChunkInfo ci = load_chunk_info(p.meta + (size_t)unit * META_STRIDE);
  const int r0 = blockIdx.x * F32_ROWS, my_row = r0 + lr;
  const int n = ci.n, fslot = ci.fslot;
  const int ncols = n + min(L, r0 + F32_ROWS);     // columns any of these rows sees: cached tokens, then the chunk's
  const int nblk = (ncols + 15) / 16;
  const size_t krot_rows = (size_t)p.cap + p.max_chunk;          // turned keys: [U][cap + max_chunk][D] fp32
  const float* Ku = ROPE ? reinterpret_cast<const float*>(p.pf_krot) + (size_t)unit * krot_rows * D
                         : (const float*)p.K + (size_t)unit * p.cap * D;
  const float* Vu = (const float*)p.V + (size_t)unit * p.cap * D;
  const float* Kcu = ROPE ? Ku + (size_t)p.cap * D : Kc + ((size_t)b * L * p.Hkv + kvh) * D;
  const float* Vcu = Vc + ((size_t)b * L * p.Hkv + kvh) * D;
  const size_t cstride = (size_t)p.Hkv * D;
  const size_t kcstride = ROPE ? (size_t)D : cstride;
  const float* Qsrc = ROPE ? reinterpret_cast<const float*>(p.pf_qrot) : Q;   // turned queries: [B][max_chunk][H][D] fp32
  const int q_rows = ROPE ? p.max_chunk : L;

  // row of column j (past the last one: the last one, masked later); cache columns are the slots without the free one
  auto row_of = [&](const float* cache, const float* chunk, size_t stride, int j) -> const float* {
    j = min(j, ncols - 1);
    return j < n ? cache + (size_t)(j + (j >= fslot ? 1 : 0)) * D : chunk + (size_t)(j - n) * stride;
  };
  float4 qv[KQ], kv[KQ], kn[KQ], vv[4][VX], vn[4][VX];
  auto load_k = [&](float4 (&k)[KQ], int blk) {
    const float* row = row_of(Ku, Kcu, kcstride, blk * 16 + lr) + q4 * 4;
#pragma unroll
    for (int s = 0; s < KQ; ++s) k[s] = *reinterpret_cast<const float4*>(row + s * 16);
  };
  auto load_v = [&](float4 (&v)[4][VX], int blk) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* row = row_of(Vu, Vcu, cstride, blk * 16 + q4 * 4 + i) + lr * 4;
#pragma unroll
      for (int x = 0; x < VX; ++x) v[i][x] = *reinterpret_cast<const float4*>(row + x * 64);
    }
  };
  const int first = min(wave, nblk - 1);           // (a wave without a block loads one it does not use)
  load_k(kv, first);
  {
    const float* qp = Qsrc + (((size_t)b * q_rows + min(my_row, L - 1)) * p.H + h) * D + q4 * 4;
#pragma unroll
    for (int s = 0; s < KQ; ++s) qv[s] = *reinterpret_cast<const float4*>(qp + s * 16);
  }
  // scaled logits of block `blk`: component i is column 16 blk + 4 q4 + i of row lr; what the row does not see is -inf
  auto logits = [&](const float4 (&k)[KQ], int blk) -> f32x4_t {
    f32x4_t a = {0.f, 0.f, 0.f, 0.f}, c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < KQ; ++s) {
      a = __builtin_amdgcn_mfma_f32_16x16x4f32(k[s].x, qv[s].x, a, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_16x16x4f32(k[s].y, qv[s].y, c, 0, 0, 0);
      a = __builtin_amdgcn_mfma_f32_16x16x4f32(k[s].z, qv[s].z, a, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_16x16x4f32(k[s].w, qv[s].w, c, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      a[i] = blk * 16 + q4 * 4 + i <= n + my_row ? (a[i] + c[i]) * p.scale_log2e : -INFINITY;
    return a;
  };
  f32x4_t* park = reinterpret_cast<f32x4_t*>(f32_smem) + lane;

  // ---- sweep 1: logits and row statistics ----
  float m_run = NEG_BIG, l_run = 0.f;
  for (int blk = wave; blk < nblk; blk += F32_WAVES) {
    load_k(kn, min(blk + F32_WAVES, nblk - 1));
    const f32x4_t s = logits(kv, blk);
    if (blk < park_blocks) park[blk * 64] = s;
    const float m_new = max3(m_run, fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
    l_run = fmaf(l_run, fast_exp2(m_run - m_new), (fast_exp2(s[0] - m_new) + fast_exp2(s[1] - m_new)) +
                                                      (fast_exp2(s[2] - m_new) + fast_exp2(s[3] - m_new)));
    m_run = m_new;
#pragma unroll
    for (int x = 0; x < KQ; ++x) kv[x] = kn[x];
  }
  load_v(vv, first);                               // on their way while the statistics are merged
#pragma unroll
  for (int off = 16; off <= 32; off <<= 1) {       // the four lanes of a row, then the eight waves
    const float mo = __shfl_xor(m_run, off, 64), lo = __shfl_xor(l_run, off, 64);
    const float mn = fmaxf(m_run, mo);
    l_run = l_run * fast_exp2(m_run - mn) + lo * fast_exp2(mo - mn);
    m_run = mn;
  }
  if (q4 == 0) { st[wave][lr][0] = m_run; st[wave][lr][1] = l_run; }
  __syncthreads();
  float M = NEG_BIG, sum = 0.f;
#pragma unroll
  for (int w = 0; w < F32_WAVES; ++w) M = fmaxf(M, st[w][lr][0]);
#pragma unroll
  for (int w = 0; w < F32_WAVES; ++w) sum += st[w][lr][1] * fast_exp2(st[w][lr][0] - M);
  const float inv = my_row < L ? 1.0f / sum : 0.f;         // rows past the chunk must not reach the column sums

  // ---- sweep 2: probabilities, output, column sums ----
  const int cap_cols = (p.cap + AT_COLS - 1) / AT_COLS * AT_COLS;
  const int cs_stride = cap_cols + (p.max_chunk + AT_COLS - 1) / AT_COLS * AT_COLS;
  unsigned long long* cs_acc = p.pf_colacc + (size_t)unit * cs_stride;
  f32x4_t o[VX][4];                                // [x][e]: component i is dim 64 x + 16 q4 + 4 i + e of row lr
#pragma unroll
  for (int x = 0; x < VX; ++x)
#pragma unroll
    for (int e = 0; e < 4; ++e) o[x][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int blk = wave; blk < nblk; blk += F32_WAVES) {
    load_v(vn, min(blk + F32_WAVES, nblk - 1));
    f32x4_t s;
    if (blk < park_blocks) {
      s = park[blk * 64];
    } else {
      load_k(kv, blk);
      s = logits(kv, blk);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = fast_exp2(s[i] - M) * inv;
    // A block that reaches past what the tile's first row sees: a column some row does not see must stay without effect
    // on that row whatever the inputs hold, and 0 times an infinity or a NaN is a NaN.  The probabilities are cleared
    // (a NaN row has none that are 0), and if some v is not finite the block is taken without the matrix instructions.
    bool matrix = true;
    if (blk * 16 + 15 > n + r0) {
      int finite = 1;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (blk * 16 + q4 * 4 + i > n + my_row) s[i] = 0.f;
#pragma unroll
        for (int x = 0; x < VX; ++x)
          finite &= is_finite(vv[i][x].x) & is_finite(vv[i][x].y) & is_finite(vv[i][x].z) & is_finite(vv[i][x].w);
      }
      matrix = __all(finite);
    }
    if (matrix) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int x = 0; x < VX; ++x) {
          o[x][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[i][x].x, s[i], o[x][0], 0, 0, 0);
          o[x][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[i][x].y, s[i], o[x][1], 0, 0, 0);
          o[x][2] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[i][x].z, s[i], o[x][2], 0, 0, 0);
          o[x][3] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[i][x].w, s[i], o[x][3], 0, 0, 0);
        }
    } else {
      for (int c = 0; c < 16; ++c) {
        const int i = c & 3;
        const float pc = __shfl(i == 0 ? s[0] : i == 1 ? s[1] : i == 2 ? s[2] : s[3], (c >> 2) * 16 + lr, 64);
        const float* row = row_of(Vu, Vcu, cstride, blk * 16 + c) + q4 * 16;
        if (blk * 16 + c > n + my_row) continue;
#pragma unroll
        for (int x = 0; x < VX; ++x)
#pragma unroll
          for (int y = 0; y < 4; ++y) {
            const float4 v = *reinterpret_cast<const float4*>(row + x * 64 + y * 4);
            o[x][0][y] = fmaf(pc, v.x, o[x][0][y]);
            o[x][1][y] = fmaf(pc, v.y, o[x][1][y]);
            o[x][2][y] = fmaf(pc, v.z, o[x][2][y]);
            o[x][3][y] = fmaf(pc, v.w, o[x][3][y]);
          }
      }
    }
    // lane lr < 4 of every lane group passes on column 4 q4 + lr (integer adds: the order does not matter)
    const float c0 = row16_sum(s[0]), c1 = row16_sum(s[1]), c2 = row16_sum(s[2]), c3 = row16_sum(s[3]);
    const float cs = lr == 0 ? c0 : lr == 1 ? c1 : lr == 2 ? c2 : c3;
    const int j = blk * 16 + q4 * 4 + lr;
    if (lr < 4 && j < ncols && cs != 0.f) {
      const long long fix = (long long)(cs * COLSUM_FIX + 0.5f);
      atomicAdd(cs_acc + (j < n ? j + (j >= fslot ? 1 : 0) : cap_cols + (j - n)), (unsigned long long)fix);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int x = 0; x < VX; ++x) vv[i][x] = vn[i][x];
  }
  // ---- add the waves' outputs ----
  __syncthreads();                                 // the parked logits are done with
  constexpr int OS = D + 4;                        // row stride: 16 lanes' 16-byte stores fall into different banks
  float* xo = f32_smem + (size_t)(wave * F32_ROWS + lr) * OS + q4 * 16;
#pragma unroll
  for (int x = 0; x < VX; ++x)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<float4*>(xo + x * 64 + i * 4) = make_float4(o[x][0][i], o[x][1][i], o[x][2][i], o[x][3][i]);
  __syncthreads();
  for (int y = tid; y < F32_ROWS * D; y += F32_THREADS) {
    const int row = y / D, col = y % D;
    if (r0 + row >= L) break;                      // rows ascend with y
    float a = 0.f;
#pragma unroll
    for (int w = 0; w < F32_WAVES; ++w) a += f32_smem[(size_t)(w * F32_ROWS + row) * OS + col];
    out[(((size_t)b * L + r0 + row) * p.H + h) * D + col] = a;
  }
}

// ---------------------------------------------------------------------------------------------
// positions re-assigned to cache ranks: the chunk's queries and every key it attends, turned and split
// ---------------------------------------------------------------------------------------------
// A chunk is scored before anything of it is evicted, so the n0 cached tokens are at the positions 0 .. n0-1 of
// their logical order and chunk token i (and its query) at n0 + i.  The rotary encoding turns plane (2i, 2i+1) of
// a row by position * base^(-2i/d); here that is done once per call, in fp32 with the (cos, sin) table, and the
// result is left as two bf16 parts (hi = the rounded value, lo = the rounded remainder) for the matrix pipe.
// One thread turns 8 dimensions (4 planes, one 16-byte piece) of one row.  Rows of a unit: n0 cached keys (by
// logical index, written at their slot), L chunk keys (written behind the cache rows), L * G queries.
template <int D>
__global__ __launch_bounds__(256) void prefill_turn_kernel(Params p, const uint16_t* __restrict__ Q,
                                                           const uint16_t* __restrict__ Kc, int L) {
  constexpr int PARTS = D / 8;
  const int unit = blockIdx.y, kvh = unit % p.Hkv, b = unit / p.Hkv;
  const int* meta = p.meta + (size_t)unit * META_STRIDE;
  const int n0 = meta[META_N], j = meta[META_J], rhead = meta[META_RHEAD];
  const int rows = n0 + L + L * p.G;
  const int x = blockIdx.x * 256 + threadIdx.x;
  const int row = x / PARTS, part = x % PARTS;
  if (row >= rows) return;
  const size_t krot_rows = (size_t)p.cap + p.max_chunk;
  uint16_t* khi = p.pf_krot + (size_t)unit * 2 * krot_rows * D;
  const uint16_t* src;
  uint16_t* dst;
  size_t lo_off;
  int pos;
  if (row < n0) {                                   // cached key at logical index `row`
    const int* Eu = p.E + (size_t)unit * 2 * p.m;
    const int* Ru = p.R + (size_t)unit * max(p.n_recent, 1);
    const int slot = n0 < p.budget ? row : logical_to_slot(p, Eu, Ru, rhead, j, row);
    src = (const uint16_t*)p.K + ((size_t)unit * p.cap + slot) * D;
    dst = khi + (size_t)slot * D;
    lo_off = krot_rows * D;
    pos = row;
  } else if (row < n0 + L) {                        // the chunk's own key i
    const int i = row - n0;
    src = Kc + (((size_t)b * L + i) * p.Hkv + kvh) * D;
    dst = khi + ((size_t)p.cap + i) * D;
    lo_off = krot_rows * D;
    pos = row;
  } else {                                          // query i of head g of the group
    const int i = (row - n0 - L) / p.G, g = (row - n0 - L) % p.G;
    const int h = kvh * p.G + g;
    src = Q + (((size_t)b * L + i) * p.H + h) * D;
    dst = p.pf_qrot + (((size_t)b * p.max_chunk + i) * p.H + h) * D;
    lo_off = (size_t)p.B * p.max_chunk * p.H * D;
    pos = n0 + i;
  }
  const uint4 raw = *reinterpret_cast<const uint4*>(src + part * 8);
  const float4* cs = reinterpret_cast<const float4*>(p.rope_tab + (size_t)pos * (D / 2) + part * 4);
  const float4 c01 = cs[0], c23 = cs[1];            // (cos, sin) of planes 4 part .. 4 part + 3
  const unsigned w[4] = {raw.x, raw.y, raw.z, raw.w};
  const float co[4] = {c01.x, c01.z, c23.x, c23.z}, si[4] = {c01.y, c01.w, c23.y, c23.w};
  unsigned hi[4], lo[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float x0 = __uint_as_float(w[e] << 16), x1 = __uint_as_float(w[e] & 0xffff0000u);
    const float y0 = x0 * co[e] - x1 * si[e], y1 = x0 * si[e] + x1 * co[e];
    hi[e] = pack_bf16(y0, y1);
    lo[e] = pack_bf16(y0 - __uint_as_float(hi[e] << 16), y1 - __uint_as_float(hi[e] & 0xffff0000u));
  }
  *reinterpret_cast<uint4*>(dst + part * 8) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
  *reinterpret_cast<uint4*>(dst + lo_off + part * 8) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
}

// ---------------------------------------------------------------------------------------------
// replay (and the copy of the surviving chunk rows into their slots)
// ---------------------------------------------------------------------------------------------
constexpr int RP_THREADS = 1024;
constexpr int RP_WAVES = RP_THREADS / 64;

// Rank of this thread's flag among the set flags of the threads before it, and the number of set flags in the
// workgroup: one ballot per wave, the waves' counts through LDS.
__device__ inline int block_rank(bool flag, int* sm_wave, int& total) {
  const unsigned long long b = __ballot(flag);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int within = __popcll(b & ((1ull << lane) - 1ull));
  if (lane == 0) sm_wave[wave] = __popcll(b);
  __syncthreads();
  int before = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < RP_WAVES; ++w) {
    const int c = sm_wave[w];
    before += w < wave ? c : 0;
    tot += c;
  }
  __syncthreads();                 // sm_wave is free again
  total = tot;
  return before + within;
}

// Words of LDS the replay needs to keep a unit's order arrays, scores, the chunk's scores, flags and lists on chip.
__host__ __device__ inline size_t replay_lds_words(int m, int cap, int r, int L) {
  return (size_t)4 * m + cap + 4 * (size_t)L + 4 + (r > 0 ? r : 1);
}

// One workgroup per unit.  IN_LDS: the unit's E, PE, R, S and the chunk's scores, flags and lists live in LDS (generic
// pointers, so the code below is the same either way) and the live parts are written back at the end.  Without it
// (budgets too large for LDS) the replay runs in place, with its lists in the workspace's prefill scratch.
//
// Tokens that lose a scope: a cached token frees its slot, a chunk token that has no slot yet just disappears.  The
// k-th slot freed (in the order of the eviction steps, the slot that was free before the chunk first) goes to the
// k-th surviving chunk token without a slot (in chunk order); the one slot left over is the next call's free slot.
//
// HELD > 0: the kernel also copies the surviving rows into their slots.  A thread asks for HELD 16-byte pieces of the
// chunk's K and of its V at the start, holds them while the evictions are worked out and stores those whose token lives:
// the loads cost nothing beside the replay's own round trips, and the launch of the scatter kernel is saved.
template <bool IN_LDS, int HELD>
__global__ __launch_bounds__(RP_THREADS) void prefill_replay_kernel(Params p, int L, const uint4* __restrict__ Kc,
                                                                    const uint4* __restrict__ Vc, int row_vec,
                                                                    int32_t* __restrict__ retained,
                                                                    int32_t* __restrict__ n_retained,
                                                                    int32_t* __restrict__ evicted) {
  __shared__ int sm_wave[RP_WAVES];
  extern __shared__ __attribute__((aligned(16))) int rp_smem[];
  const int unit = blockIdx.x, tid = threadIdx.x;
  int* meta = p.meta + (size_t)unit * META_STRIDE;
  float* Sg = p.S + (size_t)unit * p.cap;
  int* Eg = p.E + (size_t)unit * 2 * p.m;
  int* PEg = p.PE + (size_t)unit * 2 * p.m;
  int* Rg = p.R + (size_t)unit * max(p.n_recent, 1);
  int32_t* evu = evicted ? evicted + (size_t)unit * L : nullptr;
  const int cap = p.cap, c = p.budget, m = p.m, r = p.n_recent;

  float* Su = Sg;
  int *Eu = Eg, *PEu = PEg, *Ru = Rg;
  float* snew = p.pf_snew + (size_t)unit * p.max_chunk;                  // [L] the chunk tokens' scores
  int* dest = p.pf_flag + (size_t)unit * (cap + p.max_chunk) + cap;     // [L] 1: the token lost a scope; later: its slot or -1
  int* loser = p.pf_list + (size_t)unit * (cap + p.max_chunk);          // [L] slot freed at eviction step e, or -1
  int* free_list = loser + L;                                           // [L + 1] freed slots in the order they are handed out
  if constexpr (IN_LDS) {
    int* w = rp_smem;
    Eu = w; w += 2 * m;
    PEu = w; w += 2 * m;
    Su = reinterpret_cast<float*>(w); w += cap;
    snew = reinterpret_cast<float*>(w); w += L;
    dest = w; w += L;
    loser = w; w += L;
    free_list = w; w += L + 1;
    Ru = w;
  }

  // Everything the kernel reads from global memory is requested here in one go (what a unit's replay costs is
  // memory round trips: its data was last touched a whole chunk ago): the bookkeeping words, the old scores and
  // the chunk's column sums of the first PRE * 1024 columns, and, for the LDS variant, the order arrays.
  const int cap_cols = (cap + AT_COLS - 1) / AT_COLS * AT_COLS;
  const int cs_stride = cap_cols + (p.max_chunk + AT_COLS - 1) / AT_COLS * AT_COLS;
  unsigned long long* acc = p.pf_colacc + (size_t)unit * cs_stride;
  constexpr int PRE = 3;
  const int n0 = meta[META_N], f0 = meta[META_FREE], j0 = meta[META_J], rhead0 = meta[META_RHEAD], t0 = meta[META_T];
  float s_pre[PRE];
  unsigned long long a_pre[PRE], n_pre[PRE];
#pragma unroll
  for (int u = 0; u < PRE; ++u) {
    const int x = u * RP_THREADS + tid;
    s_pre[u] = Sg[min(x, cap - 1)];
    a_pre[u] = acc[min(x, cap - 1)];
    n_pre[u] = acc[cap_cols + min(x, L - 1)];
  }
  // The order arrays are read whole, dead entries too: which are live hangs on a bookkeeping word, one round trip more (32 heads,
  // 512 tokens into 2048 slots 66.1 -> 65.1 us a call; short chunks the same, 8 heads, 100 into 1024 23.0).
  constexpr int PRE_E = 4;
  int e_pre[PRE_E], pe_pre[PRE_E], r_pre = 0;
  if constexpr (IN_LDS) {
#pragma unroll
    for (int u = 0; u < PRE_E; ++u) {
      const int x = min(u * RP_THREADS + tid, 2 * m - 1);
      e_pre[u] = Eg[x];
      pe_pre[u] = PEg[x];
    }
    r_pre = Rg[min(tid, max(r, 1) - 1)];
  }
  constexpr int HOLD = HELD > 0 ? HELD : 1;
  uint4v_t k_held[HOLD], v_held[HOLD];                // pieces u * 1024 + tid of the unit's L rows of row_vec pieces
  if constexpr (HELD > 0) {
    const int kvh = unit % p.Hkv, b = unit / p.Hkv;
#pragma unroll
    for (int u = 0; u < HELD; ++u) {
      const int x = min(u * RP_THREADS + tid, L * row_vec - 1), i = x / row_vec, e = x - i * row_vec;
      const size_t src = (((size_t)b * L + i) * p.Hkv + kvh) * row_vec + e;
      k_held[u] = reinterpret_cast<const uint4v_t*>(Kc)[src];
      v_held[u] = reinterpret_cast<const uint4v_t*>(Vc)[src];
    }
  }
  if constexpr (IN_LDS) {
#pragma unroll
    for (int u = 0; u < PRE_E; ++u) {
      const int x = u * RP_THREADS + tid;
      if (x < 2 * m) { Eu[x] = e_pre[u]; PEu[x] = pe_pre[u]; }
    }
    for (int x = PRE_E * RP_THREADS + tid; x < 2 * m; x += RP_THREADS) { Eu[x] = Eg[x]; PEu[x] = PEg[x]; }
    if (tid < r) Ru[tid] = r_pre;
    for (int i = RP_THREADS + tid; i < r; i += RP_THREADS) Ru[i] = Rg[i];
  }

  // ---- Algorithm 1's S update for the whole chunk: add the column sums the attend kernel left in the accumulators ----
  {
    // every accumulator that is read is also cleared for the next chunk (the others only ever received zeros)
    auto cache_col = [&](int x, float v, unsigned long long a) {
      if (x <= n0 && x != f0) {                                      // the columns every row tile visited
        v += (float)(long long)a * (1.0f / COLSUM_FIX);
        Sg[x] = v;
        acc[x] = 0;
      }
      if constexpr (IN_LDS) Su[x] = v;
    };
    auto chunk_col = [&](int x, unsigned long long a) {
      snew[x] = (float)(long long)a * (1.0f / COLSUM_FIX);
      acc[cap_cols + x] = 0;
    };
#pragma unroll
    for (int u = 0; u < PRE; ++u) {
      const int x = u * RP_THREADS + tid;
      if (x < cap) cache_col(x, s_pre[u], a_pre[u]);
      if (x < L) chunk_col(x, n_pre[u]);
    }
    for (int x = PRE * RP_THREADS + tid; x < cap; x += RP_THREADS) cache_col(x, Sg[x], acc[x]);
    for (int x = PRE * RP_THREADS + tid; x < L; x += RP_THREADS) chunk_col(x, acc[cap_cols + x]);
  }
  const int F = min(L, c - n0);            // tokens that still fit without eviction (they take slots n0 ..)
  const int Lev = L - F;                   // tokens that each trigger one eviction
  const int t_end = t0 + L - 1;            // every count C is t_end - position + 1 once the chunk is in
  const int tev = t0 + F;                  // position of the first evicting token
  for (int i = tid; i < L; i += RP_THREADS) { dest[i] = 0; loser[i] = -1; }
  __syncthreads();

  // ---- tokens that got slots while filling ----
  for (int i = tid; i < F; i += RP_THREADS) {
    Su[n0 + i] = snew[i];
    if constexpr (IN_LDS) Sg[n0 + i] = snew[i];
    if (evu) evu[i] = -1;
  }
  __syncthreads();

  int j_final = j0, rhead_final = rhead0, f_final = n0 + F, n_final = n0 + F;
  if (Lev > 0) {
    n_final = c;
    const int fstart = F > 0 ? c : f0;     // the one free slot when the evictions start
    auto score_of = [&](int id) -> float { return id < cap ? Su[id] : snew[id - cap]; };
    auto chunk_id = [&](int i) -> int { return i < F ? n0 + i : cap + i; };   // id of chunk token i

    // sweeps of idx over the tree region: eviction steps [e_a, e_b) share one sweep
    int e_a = 0;
    while (e_a < Lev) {
      const int j_a = (j0 + e_a) % m;
      const int e_b = min(Lev, e_a + (m - j_a));
      const int cnt = e_b - e_a;
      // (1) the tokens that enter the tree region at these steps
      for (int x = tid; x < cnt; x += RP_THREADS) {
        const int e = e_a + x;
        const int pos_nc = tev + e - r;    // r == 0: the new token itself
        int id;
        if (pos_nc >= t0) id = chunk_id(pos_nc - t0);
        else id = Ru[(rhead0 + e) % r];    // still the ring's entry from before the chunk (e < r here)
        Eu[m + j_a + x] = id;
        PEu[m + j_a + x] = pos_nc;
      }
      __syncthreads();
      // (2) all scopes of the sweep are disjoint pairs: decide them in parallel, then write
      for (int x0 = 0; x0 < cnt; x0 += RP_THREADS) {
        const int x = x0 + tid;
        int surv_id = 0, surv_pos = 0, lose_id = 0, lose_pos = 0;
        if (x < cnt) {
          const int j = j_a + x;
          const int idl = Eu[2 * j], idr = Eu[2 * j + 1];
          const int pl = PEu[2 * j], pr = PEu[2 * j + 1];
          const bool averaged = !(p.flags & TREEKV_SCORE_ACCUMULATED);
          const float bl = averaged ? score_of(idl) / (float)(t_end - pl + 1) : score_of(idl);
          const float br = averaged ? score_of(idr) / (float)(t_end - pr + 1) : score_of(idr);
          const bool drop_right = (p.flags & TREEKV_KEEP_LEFT) || (bl > br);
          surv_id = drop_right ? idl : idr; surv_pos = drop_right ? pl : pr;
          lose_id = drop_right ? idr : idl; lose_pos = drop_right ? pr : pl;
        }
        __syncthreads();
        if (x < cnt) {
          const int j = j_a + x;
          Eu[j] = surv_id; PEu[j] = surv_pos;
          if (lose_id >= cap) dest[lose_id - cap] = 1;                       // a chunk token without a slot is gone
          else {
            loser[e_a + x] = lose_id;                                        // a slot that is free now
            if (lose_id >= n0 && lose_id < n0 + F) dest[lose_id - n0] = 1;   // ... which a token of this chunk had taken
          }
          if (evu) evu[F + e_a + x] = lose_pos;
        }
        __syncthreads();
      }
      e_a = e_b;
    }
    j_final = (j0 + Lev) % m;

    // ---- the recent window: the last r chunk tokens (or fewer) take over ring entries ----
    if (r > 0) {
      for (int x = tid; x < r; x += RP_THREADS) {
        // ring index (rhead0 + e) % r is written by steps e = x, x + r, ...; the last one below Lev stays
        if (x < Lev) {
          const int e_last = x + ((Lev - 1 - x) / r) * r;
          Ru[(rhead0 + x) % r] = chunk_id(F + e_last);
        }
      }
      rhead_final = (rhead0 + Lev) % r;
    }

    // ---- freed slots in the order they are handed out: the slot free before the chunk, then by eviction step ----
    if (tid == 0) free_list[0] = fstart;
    int n_free = 1;
    for (int e0 = 0; e0 < Lev; e0 += RP_THREADS) {
      const int e = e0 + tid;
      const int slot = e < Lev ? loser[e] : -1;
      int total;
      const int rank = block_rank(slot >= 0, sm_wave, total);
      if (slot >= 0) free_list[n_free + rank] = slot;
      n_free += total;
    }
    __syncthreads();
    // ---- surviving chunk tokens without a slot take them in chunk order ----
    int n_alive = 0;
    for (int i0 = F; i0 < L; i0 += RP_THREADS) {
      const int i = i0 + tid;
      const bool alive = i < L && dest[i] == 0;
      int total;
      const int rank = block_rank(alive, sm_wave, total);
      if (i < L) dest[i] = alive ? free_list[n_alive + rank] : -1;
      n_alive += total;
    }
    f_final = free_list[n_alive < n_free ? n_alive : n_free - 1];      // n_free == n_alive + 1: one slot stays free
    __syncthreads();

    // ---- rewrite ids that still name chunk tokens, hand their scores to their slots ----
    for (int k = tid; k < m; k += RP_THREADS) {
      const int x = tree_index(k, j_final);
      const int id = Eu[x];
      if (id >= cap) Eu[x] = dest[id - cap];
    }
    for (int x = tid; x < r; x += RP_THREADS) {
      const int id = Ru[x];
      if (id >= cap) Ru[x] = dest[id - cap];
    }
    for (int i = F + tid; i < L; i += RP_THREADS) {
      const int slot = dest[i];
      if (slot >= 0) Sg[slot] = snew[i];
    }
  }
  // tokens that arrived while filling sit in slots n0 + i unless the chunk also evicted them
  for (int i = tid; i < F; i += RP_THREADS) dest[i] = dest[i] ? -1 : n0 + i;
  __syncthreads();
  if constexpr (IN_LDS) {          // write back what later calls read: the live entries
    if (Lev > 0) {
      for (int k = tid; k < m; k += RP_THREADS) { const int x = tree_index(k, j_final); Eg[x] = Eu[x]; PEg[x] = PEu[x]; }
      for (int i = tid; i < r; i += RP_THREADS) Rg[i] = Ru[i];
    }
  }

  // ---- retained positions, bookkeeping words ----
  int32_t* ret = retained + (size_t)unit * c;
  for (int i = tid; i < c; i += RP_THREADS) {
    int pv = -1;
    if (i < n_final) {
      pv = i;
      if (n_final == c) {
        const int k = i - p.n_sink;
        if (k >= 0 && k < m) pv = PEu[tree_index(k, j_final)];
        else if (k >= m) pv = t_end + 1 - r + (k - m);
      }
    }
    ret[i] = pv;
  }
  if (tid == 0) {
    meta[META_N] = n_final;
    meta[META_FREE] = f_final;
    meta[META_J] = j_final;
    meta[META_RHEAD] = rhead_final;
    meta[META_T] = t0 + L;
    if (n_retained) n_retained[unit] = n_final;
  }

  if constexpr (HELD > 0) {
#pragma unroll
    for (int u = 0; u < HELD; ++u) {
      const int x = u * RP_THREADS + tid, i = x / row_vec, e = x - i * row_vec;
      const int slot = x < L * row_vec ? dest[i] : -1;
      if (slot >= 0) {
        const size_t dst = ((size_t)unit * cap + slot) * row_vec + e;
        reinterpret_cast<uint4v_t*>(p.K)[dst] = k_held[u];
        reinterpret_cast<uint4v_t*>(p.V)[dst] = v_held[u];
      }
    }
  } else if constexpr (IN_LDS) {
    int* dest_g = p.pf_flag + (size_t)unit * (cap + p.max_chunk) + cap;
    for (int i = tid; i < L; i += RP_THREADS) dest_g[i] = dest[i];
  }
}

// ---------------------------------------------------------------------------------------------
// scatter: chunk rows that survived go to their slots
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void prefill_scatter_kernel(Params p, const uint4* __restrict__ Kc,
                                                              const uint4* __restrict__ Vc, int L, int row_vec) {
  // row_vec lanes (16-byte pieces of a row: 16 at d=128, 8 at d=64) per token, 256 / row_vec tokens per workgroup
  const int per_wg = 256 / row_vec;
  const int i = blockIdx.x * per_wg + threadIdx.x / row_vec, e = threadIdx.x % row_vec, unit = blockIdx.y;
  if (i >= L) return;
  const int kvh = unit % p.Hkv, b = unit / p.Hkv;
  const int slot = p.pf_flag[(size_t)unit * (p.cap + p.max_chunk) + p.cap + i];
  if (slot < 0) return;
  const size_t src = (((size_t)b * L + i) * p.Hkv + kvh) * row_vec + e;
  const size_t dst = ((size_t)unit * p.cap + slot) * row_vec + e;
  reinterpret_cast<uint4*>(p.K)[dst] = Kc[src];
  reinterpret_cast<uint4*>(p.V)[dst] = Vc[src];
}

// What follows the attend kernel, whatever the storage type: replay, then the surviving rows' copy.
int launch_replay(const Params& p, const void* K, const void* V, int L, int32_t* retained, int32_t* n_retained,
                  int32_t* evicted, hipStream_t s) {
  const size_t rp_lds = replay_lds_words(p.m, p.cap, p.n_recent, L) * sizeof(int);
  const int row_vec = p.D * (p.dtype == TREEKV_BF16 ? 2 : 4) / 16;
  // Pieces of a unit's K rows per thread.  Beyond four, one workgroup's copies outlast the launch they save: 32 heads x 512
  // tokens of head_dim 128 into 2048 slots 68.0 us a call with eight, 67.3 with the scatter kernel; the same of head_dim 64,
  // four pieces, 49.1 and 50.1; of head_dim 128, 8 heads, 100 tokens into 1024 slots 21.3 and 23.0; 4 heads, 8 into 300 14.6
  // and 16.2.
  constexpr int HELD_MAX = 4;
  const int held = (int)(((size_t)L * row_vec + RP_THREADS - 1) / RP_THREADS);
  if (rp_lds <= 140 * 1024) {
    auto replay = held <= 1 ? prefill_replay_kernel<true, 1> : held <= 2 ? prefill_replay_kernel<true, 2>
                : held <= HELD_MAX ? prefill_replay_kernel<true, HELD_MAX>
                : prefill_replay_kernel<true, 0>;
    if (rp_lds > 48 * 1024 &&
        hip_failed(hipFuncSetAttribute((const void*)replay, hipFuncAttributeMaxDynamicSharedMemorySize, (int)rp_lds)))
      return TREEKV_EHIP;
    hipLaunchKernelGGL(replay, dim3(p.U), dim3(RP_THREADS), rp_lds, s, p, L, (const uint4*)K, (const uint4*)V, row_vec,
                       retained, n_retained, evicted);
    if (held <= HELD_MAX) return finish_launch();
  } else {
    if (2 * (size_t)L + 1 > (size_t)p.cap + p.max_chunk) return TREEKV_EUNSUPPORTED;   // its lists live in pf_list
    hipLaunchKernelGGL((prefill_replay_kernel<false, 0>), dim3(p.U), dim3(RP_THREADS), 0, s, p, L, (const uint4*)K,
                       (const uint4*)V, row_vec, retained, n_retained, evicted);
  }
  hipLaunchKernelGGL(prefill_scatter_kernel, dim3((L + 256 / row_vec - 1) / (256 / row_vec), p.U), dim3(256), 0, s, p, (const uint4*)K, (const uint4*)V, L, row_vec);
  return finish_launch();
}

template <int D>
int launch_prefill_d(const Params& p, const void* Q, const void* K, const void* V, int L, float* out,
                     int32_t* retained, int32_t* n_retained, int32_t* evicted, hipStream_t s) {
  const uint16_t* q = (const uint16_t*)Q;
  const uint16_t* k = (const uint16_t*)K;
  const uint16_t* v = (const uint16_t*)V;
  const bool rope = (p.flags & TREEKV_POSITION_RERANK) != 0;
  if (rope) {
    const int rows = p.budget + L + L * p.G;           // at most: every cached key, the chunk's keys and queries
    hipLaunchKernelGGL(prefill_turn_kernel<D>, dim3((rows * (D / 8) + 255) / 256, p.U), dim3(256), 0, s, p, q, k, L);
  }
  // Logits in registers where a workgroup's fit: the fixed part of the call is shorter by far and the keys are multiplied once.
  // Plain head_dim 64, where four waves of the two-sweep kernel share a SIMD, only while that leaves compute units idle or
  // nearly so: one 32-row workgroup for each of the 256, or up to three where long chunks make their lengths uneven.  us a call,
  // two sweeps / registers, 512 tokens into 2048 slots: 24 heads 52 / 45, 32 heads 54 / 49, 48 heads 73 / 63, 64 heads 76 / 76,
  // 128 heads 134 / 143; 256 heads: 32 tokens 40 / 25, 64 tokens 42 / 41, 100 tokens 62 / 70.  The number of slots changes how
  // much is won, not by which: over 16 to 2048 slots, 8 to 1024 heads and 8 to 2000 tokens the ratio of the two is 0.97 to 1.95
  // at head_dim 128 (below 1 by 1-3 % for some calls of 2000 row tiles and more), 1.01 to 2.0 with re-assigned positions, and at
  // plain head_dim 64 1.14 to 1.8 up to 256 row tiles, 0.99 to 1.36 up to 768, and beyond, where two sweeps are kept, 0.75 to 1.0
  // (1.2 for the shortest chunks).
  // The row tiles are those of the whole call, so at plain head_dim 64 a sequence's last bits can depend on how many share it.
  const int res_tiles = (L + RES_ROWS - 1) / RES_ROWS, res_items = res_tiles * p.G * p.U;
  const bool resident = (p.budget + 31) / 32 + (L + 31) / 32 <= RES_WAVES * RES_BLOCKS &&
                        (D == 128 || rope || res_items <= 256 || (res_items <= 768 && res_tiles >= 4));
  auto attend = resident ? (rope ? prefill_attend_resident_kernel<D, true> : prefill_attend_resident_kernel<D, false>)
                         : (rope ? prefill_attend_kernel<D, true> : prefill_attend_kernel<D, false>);
  const int row_tiles = resident ? res_tiles : (L + ROW_TILE - 1) / ROW_TILE;
  const size_t lds = !resident ? AttendLds<D>::BYTES : rope ? ResidentLds<D, true>::BYTES : ResidentLds<D, false>::BYTES;
  if (lds > 48 * 1024 &&
      hip_failed(hipFuncSetAttribute((const void*)attend, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)))
    return TREEKV_EHIP;
  const int n_items = row_tiles * p.G * p.U;
  hipLaunchKernelGGL(attend, dim3((n_items + 7) / 8 * 8), dim3(AT_THREADS), lds, s, p, q, k, v, L, row_tiles, out);
  return launch_replay(p, K, V, L, retained, n_retained, evicted, s);
}

// The same for fp32 storage: one thread turns 4 dimensions (2 planes) of one row and stores them as fp32; the keys go
// to [U][cap + max_chunk][D] (cache rows at their slot, the chunk's behind them), the queries to [B][max_chunk][H][D].
template <int D>
__global__ __launch_bounds__(256) void prefill_turn_f32_kernel(Params p, const float* __restrict__ Q,
                                                               const float* __restrict__ Kc, int L) {
  constexpr int PARTS = D / 4;
  const int unit = blockIdx.y, kvh = unit % p.Hkv, b = unit / p.Hkv;
  const int* meta = p.meta + (size_t)unit * META_STRIDE;
  const int n0 = meta[META_N], j = meta[META_J], rhead = meta[META_RHEAD];
  const int rows = n0 + L + L * p.G;
  const int x = blockIdx.x * 256 + threadIdx.x;
  const int row = x / PARTS, part = x % PARTS;
  if (row >= rows) return;
  const size_t krot_rows = (size_t)p.cap + p.max_chunk;
  float* kturned = reinterpret_cast<float*>(p.pf_krot) + (size_t)unit * krot_rows * D;
  const float* src;
  float* dst;
  int pos;
  if (row < n0) {                                   // cached key at logical index `row`
    const int* Eu = p.E + (size_t)unit * 2 * p.m;
    const int* Ru = p.R + (size_t)unit * max(p.n_recent, 1);
    const int slot = n0 < p.budget ? row : logical_to_slot(p, Eu, Ru, rhead, j, row);
    src = (const float*)p.K + ((size_t)unit * p.cap + slot) * D;
    dst = kturned + (size_t)slot * D;
    pos = row;
  } else if (row < n0 + L) {                        // the chunk's own key i
    const int i = row - n0;
    src = Kc + (((size_t)b * L + i) * p.Hkv + kvh) * D;
    dst = kturned + ((size_t)p.cap + i) * D;
    pos = row;
  } else {                                          // query i of head g of the group
    const int i = (row - n0 - L) / p.G, g = (row - n0 - L) % p.G;
    const int h = kvh * p.G + g;
    src = Q + (((size_t)b * L + i) * p.H + h) * D;
    dst = reinterpret_cast<float*>(p.pf_qrot) + (((size_t)b * p.max_chunk + i) * p.H + h) * D;
    pos = n0 + i;
  }
  const float4 xv = *reinterpret_cast<const float4*>(src + part * 4);
  const float4 cs = *reinterpret_cast<const float4*>(p.rope_tab + (size_t)pos * (D / 2) + part * 2);   // (cos, sin) x 2 planes
  float4 y;
  y.x = xv.x * cs.x - xv.y * cs.y;
  y.y = xv.x * cs.y + xv.y * cs.x;
  y.z = xv.z * cs.z - xv.w * cs.w;
  y.w = xv.z * cs.w + xv.w * cs.z;
  *reinterpret_cast<float4*>(dst + part * 4) = y;
}

// fp32 storage: the fp32 matrix attend, then the same replay.
template <int D>
int launch_prefill_f32(const Params& p, const void* Q, const void* K, const void* V, int L, float* out,
                       int32_t* retained, int32_t* n_retained, int32_t* evicted, hipStream_t s) {
  const size_t ncols = (size_t)p.cap + L;
  if (ncols > (size_t)F32_MAX_COLS) return TREEKV_EUNSUPPORTED;
  const int blocks = (int)((ncols + 15) / 16), park = blocks < F32_PARK_BLOCKS ? blocks : F32_PARK_BLOCKS;
  const size_t lds = (size_t)park * 1024 > f32_merge_bytes<D>() ? (size_t)park * 1024 : f32_merge_bytes<D>();
  const bool rope = (p.flags & TREEKV_POSITION_RERANK) != 0;
  if (rope) {
    const int rows = p.budget + L + L * p.G;           // at most: every cached key, the chunk's keys and queries
    hipLaunchKernelGGL(prefill_turn_f32_kernel<D>, dim3((rows * (D / 4) + 255) / 256, p.U), dim3(256), 0, s, p,
                       (const float*)Q, (const float*)K, L);
  }
  auto attend = rope ? prefill_attend_f32_kernel<D, true> : prefill_attend_f32_kernel<D, false>;
  if (lds > 48 * 1024 &&
      hip_failed(hipFuncSetAttribute((const void*)attend, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)))
    return TREEKV_EHIP;
  hipLaunchKernelGGL(attend, dim3((L + F32_ROWS - 1) / F32_ROWS, p.G, p.U), dim3(F32_THREADS), lds, s, p, (const float*)Q,
                     (const float*)K, (const float*)V, L, park, out);
  return launch_replay(p, K, V, L, retained, n_retained, evicted, s);
}

}  // namespace

int launch_prefill(const Params& p, const void* Q, const void* K, const void* V, int len, float* out,
                   int32_t* retained, int32_t* n_retained, int32_t* evicted, hipStream_t s) {
  if (p.dtype == TREEKV_F32) {
    if (p.D == 128) return launch_prefill_f32<128>(p, Q, K, V, len, out, retained, n_retained, evicted, s);
    if (p.D == 64) return launch_prefill_f32<64>(p, Q, K, V, len, out, retained, n_retained, evicted, s);
    return TREEKV_EUNSUPPORTED;
  }
  if (p.D == 128) return launch_prefill_d<128>(p, Q, K, V, len, out, retained, n_retained, evicted, s);
  if (p.D == 64) return launch_prefill_d<64>(p, Q, K, V, len, out, retained, n_retained, evicted, s);
  return TREEKV_EUNSUPPORTED;
}

}  // namespace tkv

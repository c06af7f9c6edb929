// bf16 MFMA GEMM for gfx950:  C = epilogue(A W^T), A [M,K] and W [N,K] both K-contiguous.
//
// One workgroup owns a BM x BN tile of C and walks K in slices of 64.  Each slice of A and W is
// brought into LDS with 16-byte LDS-direct loads (no staging registers, no LDS store
// instructions) into two to four stage buffers: the loads of a later slice are issued one by one between the
// MFMAs of the current one (main_loop).
//
// LDS layout: rows of 128 bytes (64 bf16), the 16-byte chunk at position c of row r holds chunk
// c ^ ((r/2) % 8) of that row.  Measured on gfx950, ds_read_b128 serves 16 lanes per pass and the
// lanes of a pass are not consecutive (rows {0-3,12-15,20-23,24-27} of a 32-row operand read share
// one); this XOR is conflict-free for the operand reads, a plain row%8 XOR is 2-way conflicted.
// An LDS-direct load writes 64 lanes x 16 bytes in lane order, so the XOR is applied to the global
// address each lane fetches.
//
// Waves are laid out WGM x WGN over the tile; a wave accumulates (BM/WGM) x (BN/WGN) in fp32 with
// v_mfma_f32_16x16x32_bf16.  The products are formed transposed (W rows as the first operand), so
// that a lane owns rows m of C and its accumulator registers walk the
// columns in groups of four consecutive n: bias, activations, rotary pairs and 8/16-byte stores
// all work on registers of one lane.
#include <stdio.h>
#include <stdlib.h>

#include <atomic>

#include "common.h"

namespace cs {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void lds_void;

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// All products run on v_mfma_f32_16x16x32_bf16.  The 32x32x16 shape does the same 1024 FLOP per SIMD and clock, but on
// random operands at the board's power limit a bare loop of 16x16x32 sustains about 12 % more (cs_mfma_ceiling).
//
// A wave's accumulators are kept per 32 x 32 block of C^T (or C) as 4 groups q of 4 consecutive columns of one row
// ("row" is the second operand's index, "column" the first operand's): four MFMAs per block, group q of a lane holds
// row 16 (q / 2) + lane % 16, columns 16 (q % 2) + 4 (lane / 16) ...
// (Each group is a register quad of its own: kept as one 16-register vector per block, a four-wave workgroup's
// accumulators were copied between register files around every MFMA.)
__device__ __forceinline__ int blk_row(int q, int lane) { return 16 * (q >> 1) + (lane & 15); }
__device__ __forceinline__ int blk_col(int q, int lane) { return 16 * (q & 1) + 4 * (lane >> 4); }
// four floats -> four bf16 (v_cvt_pk_bf16_f32, round to nearest even), as 8 bytes
__device__ __forceinline__ u32x2 pack4(float a, float b, float c, float d) {
  const f32x4 v = {a, b, c, d};
  const bf16x4 h = __builtin_convertvector(v, bf16x4);
  return __builtin_bit_cast(u32x2, h);
}
// z * sigmoid(z) with the hardware exp2 and reciprocal (1 ulp each): five instructions, where the
// IEEE division costs a dozen, and this runs for every element of the widest GEMM's epilogue
__device__ __forceinline__ float silu_f(float z) {
  return z * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * z));
}

// ---- epilogue through LDS.  A lane of an accumulator block owns one row and 4-column groups of
// it, so storing from registers writes 16-byte pieces of 32 different rows per instruction: measured,
// that way the stores cost a quarter of a K = 1280 launch.  Instead every wave passes its blocks
// through a private 32-row LDS chunk and writes them out as whole 64- or 128-byte row segments,
// 16 bytes per lane.  LDS serves one wave's instructions in order, so no wait is needed between a
// chunk's writes and reads beyond keeping the compiler from reordering them.
// What a tile may use behind its stage buffers: 1 KB of per-column values, then the waves' per-row partial
// sums of a folded normalisation, [2][WGN][BM] floats (sums of squares, plain sums).  (The 128 x 160 tiles, of
// which the four-wave one must fit a CU twice, have 128 rows and two waves along N: 2 KB of sums.)
constexpr int EXTRA_LDS_BYTES = 1024 + 2 * 4 * 256 * 4;
constexpr int EXTRA_LDS_BYTES_PAIR = 1024 + 4 * 256 * 4;
template <int BM, int BN, int NWAVES = 0, int EPI = -1>
constexpr int extra_lds_bytes() {
  return BM == 128 && BN == 160 ? EXTRA_LDS_BYTES_PAIR : EXTRA_LDS_BYTES;
}
// Stage buffers of the K loop, where the launcher does not say otherwise (its one-round tiles have three or four).  Two
// (a slice's MFMAs cover the next slice's loads where the tile is
// large, and more would not fit) except on the eight-wave 128 x 160 tile, which runs one workgroup per CU in
// launches that do not fill the chip: its slice of MFMAs is much shorter than the loads' latency, so it keeps
// CS_GEMM_SMALL_STAGES - 1 slices in flight, four stages being what 160 KB of LDS hold (build-time switch for
// measurement: 2 is the plain double buffer.  Measured on one box, 3072 tokens, 2 / 3 / 4 stages: out projection
// 31.4 / 32.1 / 28.5 us, down projection 60.3 / 61.8 / 52.0 us, the step 6.78 / 6.85 / 6.40 ms).
#ifndef CS_GEMM_SMALL_STAGES
#define CS_GEMM_SMALL_STAGES 4
#endif
template <int BM, int BN, int NWAVES>
constexpr int default_stages() { return BM == 128 && BN == 160 && NWAVES == 8 ? CS_GEMM_SMALL_STAGES : 2; }
template <int BM, int BN, int NWAVES, int EPI, int STAGES>
constexpr int tile_lds_bytes() {   // (the epilogue chunks have room of their own where the idle stage buffers are too small for them)
  return STAGES * (BM + BN) * 128 + extra_lds_bytes<BM, BN, NWAVES, EPI>() +
         (NWAVES * 32 * 144 > (BM + BN) * 128 * (STAGES == 4 ? 2 : 1) ? NWAVES * 32 * 144 : 0);
}
constexpr int CHUNK_STRIDE = 144;               // bytes between chunk rows: 128 of data + 16 of padding
constexpr int CHUNK_BYTES_ = 32 * CHUNK_STRIDE;
// The 64-row tiles of a ragged last tile row run behind the full tiles, eight of them or so on an otherwise idle
// chip, each alone on its CU with next to no MFMA work per slice: their K loop goes at the pace of the loads
// (measured on 8224 x 1024 x 4096: the 32 extra rows cost 29 us on top of 65, 0.45 us per slice).  With eight
// waves they take as many stage buffers, up to four, as 160 KB of LDS hold (CS_GEMM_LIGHT_STAGES=2 at build time:
// two): 21 us, 0.33 us per slice, which is 75 GB/s, about what one CU draws; the 8-tile class-token step 9.82 ->
// 9.51 ms.
#ifndef CS_GEMM_LIGHT_STAGES
#define CS_GEMM_LIGHT_STAGES 4
#endif
template <int BN, int NWAVES, int EPI>
constexpr int light_lds_need(int st) {
  const int stage = (64 + BN) * 128, chunks = NWAVES * CHUNK_BYTES_;
  return st * stage + extra_lds_bytes<64, BN, NWAVES, EPI>() + (chunks > stage ? chunks : 0);
}
template <int BN, int NWAVES, int EPI>
constexpr int light_stages() {
  if (NWAVES != 8) return 2;
  for (int st = CS_GEMM_LIGHT_STAGES; st > 2; --st)
    if (light_lds_need<BN, NWAVES, EPI>(st) <= 160 * 1024) return st;
  return 2;
}
constexpr int CHUNK_BYTES = 32 * CHUNK_STRIDE;

// v[b][q] holds columns b*32 + blk_col(q) .. +3 of row blk_row(q) of a 32 x (NB*32) block.
// The block's element (r, c) goes to out[rowmap(row0 + r) * ld + col0 + c] for row0 + r < row_end,
// col0 + c < col_end (col_end - col0 a multiple of 4); ACCUM adds to what is there (fp32 only).
// Producer side of a folded RMSNorm: what the residual epilogue writes beside the updated stream.
struct NormFold {
  bf16_t* xg;             // [*, ld_xg] bf16(x_new * gain)
  int64_t ld_xg;
  const float* gain_lds;  // gain of the tile's columns, staged in LDS; index = column - n0
  int n0;
  float ssacc[4];         // this lane's sums of x_new^2, one per 8-row group of the 32-row block
  float s1acc[4];         // ... and of x_new (a LayerNorm needs the mean too)
};

template <int NB, typename T, bool ACCUM, bool SUMS = false>
__device__ __forceinline__ void store_block(unsigned char* chunk, const f32x4 (&v)[NB][4], T* out, int64_t ld,
                                            const int32_t* row_map, int row0, int row_end, int col0, int col_end,
                                            bool wide, bool wt, const f32x4* held = nullptr, NormFold* fold = nullptr) {
  constexpr int ES = (int)sizeof(T);
  static_assert(NB * 32 * ES <= 128, "a chunk row holds 128 bytes");
  static_assert(!ACCUM || ES == 4, "accumulation is for fp32 outputs");
  const int lane = threadIdx.x & 63;
  asm volatile("" ::: "memory");
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      unsigned char* p = chunk + blk_row(q, lane) * CHUNK_STRIDE + (b * 32 + blk_col(q, lane)) * ES;
      if constexpr (ES == 2) *reinterpret_cast<u32x2*>(p) = pack4(v[b][q][0], v[b][q][1], v[b][q][2], v[b][q][3]);
      else *reinterpret_cast<f32x4*>(p) = v[b][q];
    }
  asm volatile("" ::: "memory");
  constexpr int LPR = NB * 32 * ES / 16;          // lanes per row
  constexpr int RPI = 64 / LPR;                   // rows per instruction
  constexpr int EPL = 16 / ES;                    // elements per lane
#pragma unroll
  for (int it = 0; it < 32 / RPI; ++it) {
    const int r = it * RPI + lane / LPR, c = (lane % LPR) * EPL;
    const f32x4 piece = *reinterpret_cast<const f32x4*>(chunk + r * CHUNK_STRIDE + (lane % LPR) * 16);
    const int m = row0 + r, n = col0 + c;
    if (m >= row_end || n >= col_end) continue;
    int64_t row = m;
    if (row_map) {
      row = row_map[m];
      if (row < 0) continue;
    }
    T* dst = out + row * ld + n;
    if constexpr (ES == 4) {
      f32x4* d4 = reinterpret_cast<f32x4*>(dst);
      if constexpr (ACCUM) {
        const f32x4 nx = (held ? held[it] : *d4) + piece;
        store16(d4, nx, wt);
        if constexpr (NB == 1) {
          if (fold) {
            const f32x4 gg = *reinterpret_cast<const f32x4*>(fold->gain_lds + (n - fold->n0));
            *reinterpret_cast<u32x2*>(fold->xg + row * fold->ld_xg + n) = pack4(nx[0] * gg[0], nx[1] * gg[1], nx[2] * gg[2], nx[3] * gg[3]);
            fold->ssacc[it] += (nx[0] * nx[0] + nx[1] * nx[1]) + (nx[2] * nx[2] + nx[3] * nx[3]);
            if constexpr (SUMS) fold->s1acc[it] += (nx[0] + nx[1]) + (nx[2] + nx[3]);
          }
        }
      } else {
        store16(d4, piece, wt);
      }
    } else {
      if (wide && n + 8 <= col_end) {
        store16(dst, piece, wt);
      } else {
        const f32x2 lo = {piece[0], piece[1]}, hi = {piece[2], piece[3]};
        *reinterpret_cast<f32x2*>(dst) = lo;
        if (n + 8 <= col_end) *reinterpret_cast<f32x2*>(dst + 4) = hi;
      }
    }
  }
  asm volatile("" ::: "memory");
}

// Cache-policy bits of the operand loads (build-time switches for measurement: -DCS_GEMM_W_AUX=2 marks the
// W loads non-temporal, 1 = sc0, 16 = sc1; likewise CS_GEMM_A_AUX for the A loads).
#ifndef CS_GEMM_W_AUX
#define CS_GEMM_W_AUX 0
#endif
#ifndef CS_GEMM_RESADD_WT     // 1: the residual-add epilogue stores write-through like the others
#define CS_GEMM_RESADD_WT 1
#endif
#ifndef CS_GEMM_A_AUX
#define CS_GEMM_A_AUX 0
#endif

template <int V>
struct int_tag { static constexpr int value = V; };
template <bool V>
struct bool_tag { static constexpr bool value = V; };

// The operands of a tile as buffer resources: base = first row of the tile, and per load the lane's byte offset
// from it (row and swizzled chunk).  LDS-direct loads go through buffer instructions, not global_load_lds: the
// compiler counts the latter in both wait counters without a known order, so that every wait for an LDS read in the
// loop became "all of them" (lgkmcnt(0)); buffer loads count in vmcnt alone and the LDS waits are exact.
// FAR: rows that lie too far apart for 32-bit offsets from the tile's first one (gemm_rows_addressable) are addressed by
// a 64-bit pointer per load and lane, and fetched with global_load_lds: slower, for pitches that nothing ordinary has.
template <int A_LOADS, int B_LOADS, bool FAR>
struct Operands {
  const bf16_t* a;            // uniform
  const bf16_t* w;
  uint32_t a_off[A_LOADS], b_off[B_LOADS];
};
template <int A_LOADS, int B_LOADS>
struct Operands<A_LOADS, B_LOADS, true> {
  const bf16_t* a[A_LOADS];
  const bf16_t* w[B_LOADS];
};
template <int AUX>
__device__ __forceinline__ void load_lds16(const bf16_t* base, uint32_t byte_off, unsigned char* lds) {
#ifdef __HIP_DEVICE_COMPILE__   // (the builtin's resource type does not exist in the host pass)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base), 0, 0xFFFFFFFFu, 0x00020000),
                                           (lds_void*)(uintptr_t)lds, 16, byte_off, 0, 0, AUX);
#endif
}
template <int AUX>
__device__ __forceinline__ void load_lds16_far(const bf16_t* src, unsigned char* lds) {
  __builtin_amdgcn_global_load_lds(src, (lds_void*)(uintptr_t)lds, 16, 0, AUX);
}

// Issues the LDS-direct loads of one 64-wide K slice: every wave instruction moves 64 x 16 bytes
// from the lanes' global addresses to 1 KB of LDS starting at a wave-uniform address, in lane order.
// (A wave whose share of the W rows lies beyond the tile, where BN is not a multiple of 8 rows per wave,
// skips that load: wave-uniform.)
// One of the A_LOADS + B_LOADS loads of a slice, by index.
template <int A_LOADS, int B_LOADS, int NWAVES, int BM, int BN, bool FAR>
__device__ __forceinline__ void issue_one(const Operands<A_LOADS, B_LOADS, FAR>& op, int l, int kt, unsigned char* stage, int wave) {
  if (l < A_LOADS) {
    if constexpr (FAR) load_lds16_far<CS_GEMM_A_AUX>(op.a[l] + (int64_t)kt * 64, stage + (l * NWAVES + wave) * 1024);
    else load_lds16<CS_GEMM_A_AUX>(op.a + (int64_t)kt * 64, op.a_off[l], stage + (l * NWAVES + wave) * 1024);
  } else if (BN % (8 * NWAVES) == 0 || ((l - A_LOADS) * NWAVES + wave) * 8 < BN) {
    if constexpr (FAR) load_lds16_far<CS_GEMM_W_AUX>(op.w[l - A_LOADS] + (int64_t)kt * 64, stage + BM * 128 + ((l - A_LOADS) * NWAVES + wave) * 1024);
    else load_lds16<CS_GEMM_W_AUX>(op.w + (int64_t)kt * 64, op.b_off[l - A_LOADS], stage + BM * 128 + ((l - A_LOADS) * NWAVES + wave) * 1024);
  }
}
template <int A_LOADS, int B_LOADS, int NWAVES, int BM, int BN, bool FAR>
__device__ __forceinline__ void issue_slice(const Operands<A_LOADS, B_LOADS, FAR>& op, int kt, unsigned char* stage, int wave) {
#pragma unroll
  for (int l = 0; l < A_LOADS + B_LOADS; ++l) issue_one<A_LOADS, B_LOADS, NWAVES, BM, BN>(op, l, kt, stage, wave);
}

// The K loop, pipelined across the slices: every LDS read is issued three fragment rows of MFMAs ahead of its use,
// also over the boundary of a slice, and a slice has one barrier, three rows before its end.  (With the barrier
// between the slices all waves met there with nothing to multiply and waited out the latency of their first reads.
// With exact waits and the pipelined boundary, 8192 rows, bf16 out: N = 6912, K = 1280 131.3 -> 119.7 us, N = 3840
// 68.7 -> 63.3 us, N = 8192, K = 5120 510 -> 477 us.  The latter runs at 1.6 GHz, the board's power limit, with the
// MFMA pipes busy 76 % of the cycles.)
// W_FIRST: accumulate C^T blocks (lane = row m, registers = columns n); otherwise C blocks (lane = column n,
// registers = rows m).
// On return the stage buffer that does not hold the last slice is idle: every wave passed the last barrier after
// reading it and nothing was loaded into it since.
// before_last() runs ahead of the last slice's MFMAs and in_last() in the middle of them, where the fragments of the
// first k-step have left their registers: global loads they issue are in flight while those execute.
//
// Fragment i of A (16 rows) pairs with fragment j of W into quarter 2 (i % 2) + j % 2 of block (i / 2, j / 2).  The
// operand with fewer fragments per wave is held for a k-step of 32 (double-buffered over the two k-steps of a slice);
// the other is streamed through a ring of registers, row r of the 2 NO rows of a slice requested at row r - 3.
// The loads of slice s + STAGES go out one at a time between MFMAs, from the barrier of slice s (which frees that
// slice's buffer) to the middle of the first k-step of slice s + 1: in one burst they queue in the texture-address
// unit (16 clocks each, all waves at once) and every wave sits in the issue stall.
template <int BM, int BN, int WGM, int WGN, bool W_FIRST, int STAGES, bool FAR, typename F, typename G>
__device__ __forceinline__ void main_loop(const GemmArgs& g, unsigned char* smem, int m0, int n0,
                                          f32x4 (&acc)[BM / WGM / 32][(BN / WGN + 31) / 32][4], F&& before_last, G&& in_last) {
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 32, TN = (WN + 31) / 32;
  constexpr int STAGE_BYTES = (BM + BN) * 128;
  constexpr int NWAVES = WGM * WGN;
  constexpr int A_LOADS = BM / (8 * NWAVES), B_LOADS = (BN + 8 * NWAVES - 1) / (8 * NWAVES), LT = A_LOADS + B_LOADS;
  static_assert(BM % (8 * NWAVES) == 0 && BN % 8 == 0, "tile vs waves");
  static_assert(WM % 32 == 0 && WN % 16 == 0, "wave tile vs MFMA shape");
  static_assert(STAGES >= 2 && STAGES <= 4 && 2 * LT < 64, "the waits below cover up to two newer slices; vmcnt is a 6-bit counter");
  constexpr int TM16 = WM / 16, TN16 = WN / 16;   // a wave's columns may end in the middle of its last 32-block
  constexpr bool STREAM_A = TM16 >= TN16;
  constexpr int NO = STREAM_A ? TM16 : TN16;      // streamed fragments per k-step
  constexpr int NI = STREAM_A ? TN16 : TM16;      // held fragments per k-step
  constexpr int ROWS = 2 * NO, SYNC_ROW = ROWS - 3;
  constexpr int RING = ROWS % 4 == 0 ? 4 : 5;     // divides ROWS: a row sits in the same registers in every slice
  static_assert(ROWS % RING == 0 && SYNC_ROW >= 1, "fragment ring");
  constexpr int HEAD_ROWS = STAGES == 2 && NO < 8 ? 0 : NO / 2, SLOTS = (3 + HEAD_ROWS) * NI;   // MFMAs over which a slice's loads are spread
  constexpr int L0 = (3 * NI * LT + SLOTS - 1) / SLOTS;             // ... the first so many in the slice that frees the buffer
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int M = g.M, N = g.N, K = g.K;
  // the lane's row inside an operand fragment and its 16-byte piece of a k-step; sw = the row's share of the LDS
  // chunk swizzle
  const int lrow = lane & 15, lhi = lane >> 4;
  const int a_rd = (wm * WM + lrow) * 128;
  const int b_rd = BM * 128 + (wn * WN + lrow) * 128;
  const int sw = (lrow >> 1) & 7;
  const int s_rd = STREAM_A ? a_rd : b_rd, h_rd = STREAM_A ? b_rd : a_rd;
  const int coff0 = (lhi ^ sw) << 4, coff1 = ((4 + lhi) ^ sw) << 4;

#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[i][j][q] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int lr = lane >> 3;  // row inside an 8-row group
  Operands<A_LOADS, B_LOADS, FAR> op;
  if constexpr (!FAR) {
    op.a = g.A + (int64_t)m0 * g.lda;
    op.w = g.W + (int64_t)n0 * g.ldw;
  }
#pragma unroll
  for (int i = 0; i < A_LOADS; ++i) {
    const int rt = (i * NWAVES + wave) * 8 + lr;  // row inside the tile
    const int r = m0 + rt < M ? rt : M - 1 - m0;
    if constexpr (FAR) op.a[i] = g.A + (int64_t)(m0 + r) * g.lda + (((lane & 7) ^ ((rt >> 1) & 7)) << 3);
    else op.a_off[i] = (uint32_t)r * (uint32_t)(g.lda * 2) + (((lane & 7) ^ ((rt >> 1) & 7)) << 4);
  }
#pragma unroll
  for (int i = 0; i < B_LOADS; ++i) {
    const int rt = (i * NWAVES + wave) * 8 + lr;
    const int r = n0 + rt < N ? rt : N - 1 - n0;
    if constexpr (FAR) op.w[i] = g.W + (int64_t)(n0 + r) * g.ldw + (((lane & 7) ^ ((rt >> 1) & 7)) << 3);
    else op.b_off[i] = (uint32_t)r * (uint32_t)(g.ldw * 2) + (((lane & 7) ^ ((rt >> 1) & 7)) << 4);
  }
  const int KT = K >> 6;

  // A wave's loads complete in the order it issued them: at most n * L of them outstanding (L = its loads per slice)
  // means that everything older than the newest n slices has landed.
  const bool all_loads = BN % (8 * NWAVES) == 0 || ((B_LOADS - 1) * NWAVES + wave) * 8 < BN;
  auto wait_newer = [&](int n) {
    if (n <= 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if (all_loads) {
      if (n == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LT) : "memory");
      else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * LT) : "memory");
    } else {
      if (n == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LT - 1) : "memory");
      else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * (LT - 1)) : "memory");
    }
  };
  // A bare barrier: __syncthreads() carries a fence that waits for every outstanding load, newer slices' included.
  auto barrier = [&] {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  bf16x8 hf[2][NI], sf[RING];
  auto read_streamed = [&](const unsigned char* stage, int r) {
    return *reinterpret_cast<const bf16x8*>(stage + s_rd + (r % NO) * 16 * 128 + (r < NO ? coff0 : coff1));
  };
  // One slice in `cur`.  HEAD: it issues the rest of the loads of slice kt_head into `head`; SYNC: it waits for the
  // next slice (in `nxt`; `newer` slices behind that one may still be in flight) and reads its first fragments;
  // TAIL: behind that it issues the first loads of slice kt_tail into `cur`.
  auto slice = [&](auto HEAD, auto SYNC, auto TAIL, int newer, unsigned char* cur, const unsigned char* nxt,
                   unsigned char* head, int kt_head, int kt_tail) {
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      const int ks = r / NO, o = r % NO;
      if constexpr (!SYNC.value) {
        if (r == NO) in_last();
      }
      if constexpr (SYNC.value) {
        if (r == SYNC_ROW) {
          wait_newer(newer);   // this wave's part of the next slice has landed
          barrier();           // ... and everyone's; nobody reads this slice's buffer any more
        }
      }
#pragma unroll
      for (int in = 0; in < NI; ++in) {
        const int i = STREAM_A ? o : in, j = STREAM_A ? in : o;
        const bf16x8 fa = STREAM_A ? sf[r % RING] : hf[ks][in], fw = STREAM_A ? hf[ks][in] : sf[r % RING];
        f32x4& c = acc[i >> 1][j >> 1][2 * (i & 1) + (j & 1)];
        if (W_FIRST) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw, fa, c, 0, 0, 0);
        else c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fw, c, 0, 0, 0);
        const int slot = r >= SYNC_ROW ? (r - SYNC_ROW) * NI + in : 3 * NI + r * NI + in;
#pragma unroll
        for (int l = 0; l < LT; ++l) {
          if (l * SLOTS / LT != slot) continue;
          if constexpr (TAIL.value) {
            if (r >= SYNC_ROW) issue_one<A_LOADS, B_LOADS, NWAVES, BM, BN>(op, l, kt_tail, cur, wave);
          }
          if constexpr (HEAD.value) {
            if (r < HEAD_ROWS) issue_one<A_LOADS, B_LOADS, NWAVES, BM, BN>(op, l, kt_head, head, wave);
          }
        }
        if (in == 0) {
          if (r + 3 < ROWS) sf[(r + 3) % RING] = read_streamed(cur, r + 3);
          else if constexpr (SYNC.value) sf[(r + 3) % RING] = read_streamed(nxt, r + 3 - ROWS);
        }
        if (r == 0) hf[1][in] = *reinterpret_cast<const bf16x8*>(cur + h_rd + in * 16 * 128 + coff1);
        if constexpr (SYNC.value) {
          if (r == SYNC_ROW) hf[0][in] = *reinterpret_cast<const bf16x8*>(nxt + h_rd + in * 16 * 128 + coff0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  // the first STAGES - 1 slices, and of the next one the loads that a slice's tail would have issued
#pragma unroll
  for (int st = 0; st < STAGES - 1; ++st)
    if (st < KT) issue_slice<A_LOADS, B_LOADS, NWAVES, BM, BN>(op, st, smem + st * STAGE_BYTES, wave);
  if (STAGES - 1 < KT) {
#pragma unroll
    for (int l = 0; l < L0; ++l) issue_one<A_LOADS, B_LOADS, NWAVES, BM, BN>(op, l, STAGES - 1, smem + (STAGES - 1) * STAGE_BYTES, wave);
  }
  // slice 0 has landed (everything, where a short K loop issued less than the pipeline holds)
  if (KT < STAGES) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  else if (all_loads) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((STAGES - 2) * LT + L0) : "memory");
  else asm volatile("s_waitcnt vmcnt(%0)" ::"n"((STAGES - 2) * (LT - 1) + (L0 < LT ? L0 : LT - 1)) : "memory");
  barrier();
#pragma unroll
  for (int in = 0; in < NI; ++in) hf[0][in] = *reinterpret_cast<const bf16x8*>(smem + h_rd + in * 16 * 128 + coff0);
#pragma unroll
  for (int r = 0; r < 3; ++r) sf[r] = read_streamed(smem, r);

  constexpr bool_tag<true> YES{};
  constexpr bool_tag<false> NO_{};
  int s = 0, stage = 0;   // slice, and the buffer it is in
  auto next_of = [&](int st) { return st + 1 == STAGES ? 0 : st + 1; };
  auto prev_of = [&](int st) { return st == 0 ? STAGES - 1 : st - 1; };   // of slice s - 1, and of slice s - 1 + STAGES
  for (; s + STAGES < KT; ++s) {
    const int nx = next_of(stage);
    slice(YES, YES, YES, STAGES - 2, smem + stage * STAGE_BYTES, smem + nx * STAGE_BYTES, smem + prev_of(stage) * STAGE_BYTES,
          s - 1 + STAGES, s + STAGES);
    stage = nx;
  }
  if (KT >= STAGES) {   // s == KT - STAGES: the loads of the last slice are still to be completed
    const int nx = next_of(stage);
    slice(YES, YES, NO_, STAGES - 2, smem + stage * STAGE_BYTES, smem + nx * STAGE_BYTES, smem + prev_of(stage) * STAGE_BYTES, KT - 1, 0);
    stage = nx;
    ++s;
  }
  if constexpr (STAGES > 2) {
    for (; s < KT - 1; ++s) {
      const int nx = next_of(stage);
      slice(NO_, YES, NO_, KT - 2 - s, smem + stage * STAGE_BYTES, smem + nx * STAGE_BYTES, nullptr, 0, 0);
      stage = nx;
    }
  }
  before_last();
  slice(NO_, NO_, NO_, 0, smem + stage * STAGE_BYTES, nullptr, nullptr, 0, 0);
}


// A 64-row tile for the rows behind the last full tile row exists when every wave can own whole
// 32-column blocks of it (and the epilogue has no pairing of column blocks).
template <int BN, int WGM, int WGN, int EPI>
constexpr bool light_tail() {
  constexpr int WN = BN / (WGM * WGN);                           // columns per wave of the 64-row tile
  return EPI != EPI_SWIGLU_BF16 && WN % 16 == 0 && WN >= 16 && (EPI != EPI_QKV || WN % 32 == 0);   // (a wave may own half a 32-column block)
}

// One output tile: K loop and epilogue.
// LDS_ALLOC: bytes of LDS the launch has (that of its largest tile shape).
template <int BM, int BN, int WGM, int WGN, int EPI, int STAGES, int LDS_ALLOC, bool FAR = false>
__device__ __forceinline__ void tile_body(const GemmArgs& g, unsigned char* smem, const int m0, const int n0) {
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 32, TN = (WN + 31) / 32;
  constexpr int STAGE_BYTES = (BM + BN) * 128;
  constexpr int NWAVES = WGM * WGN;
  static_assert((EPI != EPI_SWIGLU_BF16 && EPI != EPI_QKV) || WN % 32 == 0, "these epilogues work on whole 32-column blocks");
  static_assert(EPI != EPI_SWIGLU_BF16 || (TN % 2 == 0), "gate/up pairs need an even number of column tiles");
  // the epilogue chunks live in the idle stage buffer; where that is too small for them (a 64-row tail tile of a
  // narrow launch) they go behind everything else this tile uses, inside what the launch's main tile shape allocated
  // (of four stages two neighbouring ones are idle whichever holds the last slice)
  constexpr bool CHUNKS_IN_TWO = STAGES == 4 && NWAVES * CHUNK_BYTES > STAGE_BYTES && NWAVES * CHUNK_BYTES <= 2 * STAGE_BYTES;
  constexpr bool CHUNKS_BEHIND = NWAVES * CHUNK_BYTES > STAGE_BYTES && !CHUNKS_IN_TWO;
  constexpr int XTRA = extra_lds_bytes<BM, BN, NWAVES, EPI>();
  // (QKV: behind the K loop the rotary table and the chunks above it take the space of the stage buffers)
  static_assert(!CHUNKS_BEHIND || (STAGES * STAGE_BYTES + XTRA + NWAVES * CHUNK_BYTES <= LDS_ALLOC && EPI != EPI_QKV),
                "no room for the epilogue chunks");

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int M = g.M, N = g.N;
  // The extra LDS behind the stage buffers.  Consumer of a folded normalisation: BM row scales, BM row shifts
  // (LayerNorm: mean times scale) and BN column values of norm_shift.  Producer: the gain of the tile's columns
  // and, from float 256 on, the waves' sums of squares [WGN][BM] and plain sums [WGN][BM].
  float* extra_lds = reinterpret_cast<float*>(smem + STAGES * STAGE_BYTES);
  // consumer: thread t < BM gathers the partial sums of squares of row m0 + t while the last K slice runs
  // (thread BM + t the partial plain sums, for a LayerNorm), they are turned into 1 / rms (or 1 / sigma and
  // mean / sigma) behind the K loop and left in LDS for every wave
  constexpr bool CONSUMES_NORM = EPI == EPI_QKV || EPI == EPI_SWIGLU_BF16 || EPI == EPI_GELU_BF16;
  constexpr bool CONSUMES_LAYERNORM = EPI == EPI_QKV || EPI == EPI_GELU_BF16;
  static_assert(!CONSUMES_NORM || 64 * NWAVES >= BM, "one thread per tile row gathers its scale");
  static_assert(!CONSUMES_LAYERNORM || 64 * NWAVES >= 2 * BM || NWAVES <= 4, "a second thread per tile row gathers its sum");
  static_assert(!CONSUMES_NORM || (2 * BM + BN) * 4 <= XTRA, "extra LDS layout of a consumer");
  constexpr bool TWO_GATHERERS = 64 * NWAVES >= 2 * BM;
  [[maybe_unused]] float ss_part[8];
  [[maybe_unused]] float s1_part[(CONSUMES_LAYERNORM && !TWO_GATHERERS) ? 8 : 1];
  [[maybe_unused]] const bool layer_norm = CONSUMES_LAYERNORM && g.s1_in != nullptr;
  [[maybe_unused]] auto gather_scale = [&] {
    if (!g.ss_in) return;
    const int t = (int)threadIdx.x;
    if (t < BM) {
      int m = m0 + t;
      m = m < M ? m : M - 1;
#pragma unroll
      for (int k = 0; k < 8; ++k) ss_part[k] = k < g.ss_parts ? g.ss_in[(int64_t)k * g.ss_stride + m] : 0.f;
      if constexpr (CONSUMES_LAYERNORM && !TWO_GATHERERS) {
        if (layer_norm) {
#pragma unroll
          for (int k = 0; k < 8; ++k) s1_part[k] = k < g.ss_parts ? g.s1_in[(int64_t)k * g.ss_stride + m] : 0.f;
        }
      }
    } else if constexpr (CONSUMES_LAYERNORM && TWO_GATHERERS) {
      if (layer_norm && t < 2 * BM) {
        int m = m0 + t - BM;
        m = m < M ? m : M - 1;
#pragma unroll
        for (int k = 0; k < 8; ++k) ss_part[k] = k < g.ss_parts ? g.s1_in[(int64_t)k * g.ss_stride + m] : 0.f;
      }
    }
  };
  [[maybe_unused]] auto publish_scale = [&] {
    if (!g.ss_in) return;
    const int t = (int)threadIdx.x;
    const float tot = ((ss_part[0] + ss_part[1]) + (ss_part[2] + ss_part[3])) + ((ss_part[4] + ss_part[5]) + (ss_part[6] + ss_part[7]));
    if constexpr (CONSUMES_LAYERNORM) {
      if (layer_norm) {
        // the shift vector of the tile's columns, and the rows' statistics
        for (int c = t * 4; c < BN; c += 64 * NWAVES * 4) {
          int n = n0 + c;
          n = n < N ? n : N - 4;
          *reinterpret_cast<f32x4*>(extra_lds + 2 * BM + c) = *reinterpret_cast<const f32x4*>(g.norm_shift + n);
        }
        float sum1;
        if constexpr (TWO_GATHERERS) {
          if (t >= BM && t < 2 * BM) extra_lds[t] = tot;   // thread BM + r: the plain sum of row r
          __syncthreads();
          sum1 = t < BM ? extra_lds[BM + t] : 0.f;
        } else {
          sum1 = ((s1_part[0] + s1_part[1]) + (s1_part[2] + s1_part[3])) + ((s1_part[4] + s1_part[5]) + (s1_part[6] + s1_part[7]));
        }
        if (t < BM) {
          const float inv_d = 1.0f / (float)g.norm_dim;
          const float mean = sum1 * inv_d;
          const float var = fmaxf(tot * inv_d - mean * mean, 0.f);
          const float rs = rsqrtf(var + g.norm_eps);
          extra_lds[t] = rs;
          extra_lds[BM + t] = mean * rs;
        }
        __syncthreads();
        return;
      }
    }
    if (t < BM) extra_lds[t] = rsqrtf(tot / (float)g.norm_dim + g.norm_eps);
    __syncthreads();
  };

  f32x4 acc[TM][TN][4];
  // this wave's epilogue chunk, in the stage buffer the last K slice did not use
  unsigned char* chunk = CHUNKS_BEHIND ? smem + STAGES * STAGE_BYTES + XTRA + wave * CHUNK_BYTES
                         : CHUNKS_IN_TWO ? smem + (((g.K >> 6) - 1) % STAGES < 2 ? 2 * STAGE_BYTES : 0) + wave * CHUNK_BYTES
                                         : smem + ((g.K >> 6) % STAGES) * STAGE_BYTES + wave * CHUNK_BYTES;

  if constexpr (EPI == EPI_QKV) {
    if (n0 >= 2 * g.hidden) {
      // v columns (the whole workgroup: 2*hidden is a multiple of BN).  Untransposed blocks: a lane's
      // group holds one v dimension n (the block "row" here) and four consecutive tokens; written as
      // rows of the transposed v buffer, 64 tokens of one dimension per chunk row.  With the roles of
      // the operands swapped the two halves of a 16x16x32 group index swap too (vsub).
      constexpr int VB = TM % 2 == 0 ? 2 : 1;   // row blocks of 32 tokens that leave together
      float bv[TN][4];
      main_loop<BM, BN, WGM, WGN, false, STAGES, FAR>(g, smem, m0, n0, acc, [&] {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int n = n0 + wn * WN + j * 32 + blk_row(q, lane);
            bv[j][q] = (g.bias && n < N) ? g.bias[n] : 0.f;
          }
        gather_scale();
      }, [] {});
      publish_scale();
      const bool wide = (g.ld_vt & 7) == 0;
      const bool wt_v = lines_exclusive(g.vt, g.ld_vt * 2);   // a workgroup writes runs of 128 bytes or more of a v^T row
#pragma unroll
      for (int j = 0; j < TN; ++j) {
#pragma unroll
        for (int i = 0; i < TM; i += VB) {
          f32x4 v[VB][4];
#pragma unroll
          for (int ii = 0; ii < VB; ++ii)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int vsub = ((q & 1) << 1) | (q >> 1);
              // the group's four values are four consecutive tokens: their row scales
              f32x4 rs = {1.f, 1.f, 1.f, 1.f}, sh = {0.f, 0.f, 0.f, 0.f};
              float cn = 0.f;   // LayerNorm: the shift of this v dimension
              if (g.ss_in) rs = *reinterpret_cast<const f32x4*>(extra_lds + wm * WM + (i + ii) * 32 + blk_col(q, lane));
              if (layer_norm) {
                sh = *reinterpret_cast<const f32x4*>(extra_lds + BM + wm * WM + (i + ii) * 32 + blk_col(q, lane));
                cn = extra_lds[2 * BM + wn * WN + j * 32 + blk_row(q, lane)];
              }
#pragma unroll
              for (int e = 0; e < 4; ++e) v[ii][q][e] = acc[i + ii][j][vsub][e] * rs[e] - sh[e] * cn + bv[j][q];
            }
          store_block<VB, bf16_t, false>(chunk, v, g.vt, g.ld_vt, nullptr, n0 + wn * WN + j * 32 - 2 * g.hidden,
                                        N - 2 * g.hidden, m0 + wm * WM + i * 32, M, wide, wt_v);
        }
      }
      return;
    }
  }

  // Residual add: the old values are needed in the epilogue, where a load's latency would be
  // paid once per chunk (the stores in between keep the compiler from hoisting the loads), so every lane fetches
  // the 16-byte pieces it will update ahead of their use.
  // There is room for one row block before the last K slice; the second row block is
  // requested right behind the K loop, into the registers the operands leave, and from then on the pieces of
  // row block i + 2 are requested as soon as those of row block i are stored (into the same registers), so two
  // row blocks of x are in flight all through the epilogue (the narrow tiles: out projection 559 -> 575, down
  // projection 838 -> 870 TFLOP/s on 8192 tokens; the 256 x 256 tile, whose four row blocks per wave leave no
  // registers for it, stays with one: with two it spills more and gains nothing).
  constexpr bool RESADD = EPI == EPI_RESADD_F32 || EPI == EPI_RESADD_SCALED_F32 || EPI == EPI_RESADD_SUMS_F32;
  constexpr bool HOLD_TWO = RESADD && TM > 1 && BN < 256;
  // (the 256 x 256 tile has registers for that one only in the second half of the last slice: requested ahead of it,
  // 28 registers of accumulators were spilled around the slice; 110 940 x 1280 x 1280 585 -> 533 us, x 3456 1006 -> 955,
  // 24 000 x 1280 x 1280 129 -> 119)
  constexpr bool HELD_LATE = RESADD && BN == 256;
  [[maybe_unused]] f32x4 held[HOLD_TWO ? 2 : 1][RESADD ? TN : 1][4];
  [[maybe_unused]] auto fetch_old = [&](int i, int j, f32x4 (&dst)[4]) {
    const int r = lane >> 3, c = (lane & 7) * 4;
    int n = n0 + wn * WN + j * 32 + c;
    n = n < N ? n : N - 4;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      int m = m0 + wm * WM + i * 32 + it * 8 + r;
      m = m < M ? m : M - 1;
      int64_t row = m;
      if (g.row_map) {
        row = g.row_map[m];
        row = row < 0 ? 0 : row;
      }
      dst[it] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(g.out) + row * g.ldo + n);
    }
  };
  // The bias of the lane's columns is fetched there too (a load inside the epilogue waits out its
  // latency once per chunk).
  // (groups q and q + 2 hold the same columns: two distinct column groups per block)
  constexpr int CQ = 2;
  f32x4 bias_r[TN][CQ];
  [[maybe_unused]] unsigned char* const rope_lds = smem + LDS_ALLOC;   // the rotary table by position, and the rows' positions
  [[maybe_unused]] int32_t row_pos[3] = {0, 0, 0};   // of row m0 + threadIdx.x, as loaded: to pack them here would wait for every load
  [[maybe_unused]] f32x4 scale_r[EPI == EPI_RESADD_SCALED_F32 ? TN : 1][CQ];
  main_loop<BM, BN, WGM, WGN, true, STAGES, FAR>(g, smem, m0, n0, acc, [&] {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < CQ; ++q) {
        const int n = n0 + wn * WN + j * 32 + blk_col(q, lane);
        bias_r[j][q] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (g.bias && n < N) bias_r[j][q] = *reinterpret_cast<const f32x4*>(g.bias + n);
        if constexpr (EPI == EPI_RESADD_SCALED_F32) {
          scale_r[j][q] = f32x4{0.f, 0.f, 0.f, 0.f};
          if (n < N) scale_r[j][q] = *reinterpret_cast<const f32x4*>(g.col_scale + n);
        }
      }
    if constexpr (RESADD && !HELD_LATE) {
#pragma unroll
      for (int j = 0; j < TN; ++j) fetch_old(0, j, held[0][j]);
    }
    if constexpr (CONSUMES_NORM) gather_scale();
    if constexpr (EPI == EPI_QKV) {
      if (g.rope.tab) {
        for (int u = wave; u < g.rope.bytes >> 10; u += NWAVES)
          load_lds16<0>(reinterpret_cast<const bf16_t*>(g.rope.tab), (uint32_t)(u * 1024 + lane * 16), rope_lds + u * 1024);
        int m = m0 + (int)threadIdx.x;
        m = m < M ? m : M - 1;
#pragma unroll
        for (int a = 0; a < 3; ++a) row_pos[a] = g.rope.pos[3 * (int64_t)m + a];
      }
    }
  }, [&] {
    if constexpr (HELD_LATE) {
#pragma unroll
      for (int j = 0; j < TN; ++j) fetch_old(0, j, held[0][j]);
    }
  });
  if constexpr (EPI == EPI_QKV) {
    if (g.rope.tab) {
      asm volatile("" : "+v"(row_pos[0]), "+v"(row_pos[1]), "+v"(row_pos[2]));   // (keeps the packing from moving up to the loads)
      if (threadIdx.x < BM)
        *reinterpret_cast<uint32_t*>(rope_lds + g.rope.bytes + 4 * threadIdx.x) = (row_pos[0] & 255) | (row_pos[1] & 255) << 8 | (row_pos[2] & 255) << 16;
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's part of the table
      if (!g.ss_in) __syncthreads();                     // (publish_scale ends with one)
    }
  }
  if constexpr (CONSUMES_NORM) publish_scale();
  if constexpr (HOLD_TWO) {
    if (m0 + wm * WM + 32 < M) {   // wave-uniform
#pragma unroll
      for (int j = 0; j < TN; ++j) fetch_old(1, j, held[1][j]);
    }
  }
  // producer of a folded RMSNorm: the gain of the tile's columns goes to LDS, from where the epilogue's
  // row-segment lanes read it
  constexpr bool FOLDS_NORM = RESADD;
  constexpr bool FOLDS_SUMS = (EPI == EPI_RESADD_SCALED_F32 || EPI == EPI_RESADD_SUMS_F32) && 1024 + 2 * WGN * BM * 4 <= XTRA;
  static_assert(!FOLDS_NORM || (BN <= 256 && 1024 + WGN * BM * 4 <= XTRA), "extra LDS layout");
  [[maybe_unused]] const bool folding = FOLDS_NORM && g.ss_out != nullptr;
  [[maybe_unused]] const bool folding_sums = FOLDS_SUMS && folding && g.s1_out != nullptr;
  if constexpr (FOLDS_NORM) {
    if (folding) {
      for (int c = threadIdx.x * 4; c < BN; c += 64 * NWAVES * 4) {
        int n = n0 + c;
        n = n < N ? n : N - 4;
        *reinterpret_cast<f32x4*>(extra_lds + c) = *reinterpret_cast<const f32x4*>(g.norm_gain + n);
      }
      __syncthreads();
    }
  }

  // QKV.  With the angles by position the table (some 6 - 22 KB) has a place behind everything else that a tile keeps in
  // LDS and lands under the last K slice; a row of the tile is then one word, its positions.
  // Otherwise the (cos, sin) rows of this tile's BM tokens are staged in LDS (free after the K loop)
  // with coalesced 16-byte loads; read per lane from global they are 16-byte pieces of 32 different
  // rows per instruction, which cost 18 us of a 110 us launch.  The table sits at the bottom of
  // LDS and the epilogue chunks move to the top.
  [[maybe_unused]] int rope_stride = g.rope.pitch;
  if constexpr (EPI == EPI_QKV) {
    if (!g.rope.tab && g.rope_cs) {
      const int half = g.head_dim >> 1;
      const int cpr = half >> 1;                       // 16-byte pieces per token row (two pairs each)
      const int upr = (cpr + 1) | 1;                   // ... per padded LDS row: odd, so rows spread over the banks
      rope_stride = upr * 16;
      chunk = smem + STAGES * STAGE_BYTES - (NWAVES - wave) * CHUNK_BYTES;
      static_assert((BM * 21 + 64) * 16 + NWAVES * CHUNK_BYTES <= STAGES * STAGE_BYTES, "rotary table and chunks");
      __syncthreads();                                 // every wave is done reading the last K slice
      // LDS-direct loads, all in flight at once: piece u of the padded table comes from row u / upr
      // (the padding pieces repeat the row's last one; the tail of the last instruction runs up to
      // 1 KB past the table, below the chunks)
      for (int base = wave * 64; base < BM * upr; base += 64 * NWAVES) {
        const int u = base + lane;
        int r = u / upr, c = u - r * upr;
        c = c < cpr ? c : cpr - 1;
        r = m0 + r < M ? m0 + r : M - 1;
        __builtin_amdgcn_global_load_lds(g.rope_cs + ((int64_t)r * cpr + c) * 4, (lds_void*)(uintptr_t)(smem + base * 16), 16, 0, 0);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
    }
  }

  // ---- epilogue.  Register 4q+e of lane l in block (i,j) is the element
  //      (row m = i*32 + blk_row(q, l), column n = j*32 + blk_col(q, l) + e).
  const int nw = n0 + wn * WN;               // first column of this wave
  const int n_end = nw + WN < N ? nw + WN : N;   // one past its last (the wave's last 32-block may be half used)
  const bool wide = (g.ldo & 7) == 0;
  // write-through stores only where no 128-byte line of the output is shared with another workgroup:
  // aligned rows, and a tile's column extent in bytes a multiple of 128
  constexpr int OUT_ES = (EPI == EPI_F32 || EPI == EPI_GELU_F32 || RESADD) ? 4 : 2;
  constexpr int TILE_OUT_BYTES = (EPI == EPI_SWIGLU_BF16 ? BN / 2 : BN) * OUT_ES;
  const bool wt = TILE_OUT_BYTES % 128 == 0 && lines_exclusive(g.out, g.ldo * OUT_ES);
  // QKV: byte offset of the first (cos, sin) pair of every 4-column group, once per lane (the
  // divisions by run-time sizes must not be redone for every row block)
  // (and by position: the place of the axis among the row's positions)
  [[maybe_unused]] int rope_off[TN][CQ], rope_axis[TN][CQ];
  [[maybe_unused]] const unsigned char* rope_base = g.rope.tab ? rope_lds : smem;
  if constexpr (EPI == EPI_QKV) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < CQ; ++q) {
        const int n = nw + j * 32 + blk_col(q, lane);
        const int pair = (((n < g.hidden ? n : n - g.hidden)) % g.head_dim) >> 1;
        rope_off[j][q] = pair * 8;
        rope_axis[j][q] = 0;
        if (g.rope.tab) {
          const int axis = pair < g.rope.end[0] ? 0 : pair < g.rope.end[1] ? 1 : 2;
          rope_off[j][q] = (pair + (axis == 0 ? g.rope.first[0] : axis == 1 ? g.rope.first[1] : g.rope.first[2])) * 8;
          rope_axis[j][q] = 8 * axis;
        }
      }
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int mrow = m0 + wm * WM + i * 32;  // first row of the block
    if (mrow >= M) continue;                 // wave-uniform
    // folded RMSNorm, consumer side: 1 / rms of the row each group q of this block holds
    [[maybe_unused]] float rsq[4] = {1.f, 1.f, 1.f, 1.f};
    [[maybe_unused]] float msq[CONSUMES_LAYERNORM ? 4 : 1] = {};   // LayerNorm: mean / sigma of those rows
    if constexpr (CONSUMES_NORM) {
      if (g.ss_in) {
#pragma unroll
        for (int q = 0; q < 4; ++q) rsq[q] = extra_lds[mrow - m0 + blk_row(q, lane)];
      }
    }
    if constexpr (CONSUMES_LAYERNORM) {
      if (layer_norm) {
#pragma unroll
        for (int q = 0; q < 4; ++q) msq[q] = extra_lds[BM + mrow - m0 + blk_row(q, lane)];
      }
    }
    // rotary: the positions of the two rows of a lane, or their numbers in the tile
    [[maybe_unused]] uint32_t rope_row[2];
    if constexpr (EPI == EPI_QKV) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int r = mrow - m0 + blk_row(2 * h, lane);
        rope_row[h] = g.rope.tab ? *reinterpret_cast<const uint32_t*>(rope_lds + g.rope.bytes + 4 * r) : (uint32_t)r;
      }
    }
    // ... producer side: sums of squares of the updated rows, gathered by the residual store
    [[maybe_unused]] NormFold fold = {g.xg, g.ld_xg, extra_lds, n0, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    if constexpr (EPI == EPI_SWIGLU_BF16) {
      // output column p*32 + c of the wave pairs gate column 2p*32 + c with up column (2p+1)*32 + c
      auto emit = [&](auto tag, int p0) {
        constexpr int NB = decltype(tag)::value;
        f32x4 v[NB][4];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int j = 2 * (p0 + b);
            const f32x4 bg = bias_r[j][q % CQ], bu = bias_r[j + 1][q % CQ];
#pragma unroll
            for (int e = 0; e < 4; ++e)
              v[b][q][e] = silu_f(acc[i][j][q][e] * rsq[q] + bg[e]) * (acc[i][j + 1][q][e] * rsq[q] + bu[e]);
          }
        store_block<NB, bf16_t, false>(chunk, v, static_cast<bf16_t*>(g.out), g.ldo, g.row_map, mrow, M,
                                       (nw >> 1) + p0 * 32, N >> 1, wide, wt);
      };
      constexpr int NP = TN / 2;
#pragma unroll
      for (int p0 = 0; p0 + 1 < NP; p0 += 2) emit(int_tag<2>{}, p0);
      if constexpr (NP & 1) emit(int_tag<1>{}, NP - 1);
    } else {
      constexpr bool OUT_F32 = EPI == EPI_F32 || EPI == EPI_GELU_F32 || RESADD;
      auto emit = [&](auto tag, int j0) {
        constexpr int NB = decltype(tag)::value;
        f32x4 v[NB][4];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int j = j0 + b;
            const int n = nw + j * 32 + blk_col(q, lane);
            f32x4 t;
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = acc[i][j][q][e];
            if constexpr (CONSUMES_NORM && EPI != EPI_SWIGLU_BF16) t *= rsq[q];
            if constexpr (CONSUMES_LAYERNORM) {
              if (layer_norm) t -= msq[q] * *reinterpret_cast<const f32x4*>(extra_lds + 2 * BM + (n - n0));
            }
            t += bias_r[j][q % CQ];
            if constexpr (EPI == EPI_RESADD_SCALED_F32) t *= scale_r[j][q % CQ];
            if constexpr (EPI == EPI_GELU_BF16 || EPI == EPI_GELU_F32 || EPI == EPI_GELU_SPLIT) {
#pragma unroll
              for (int e = 0; e < 4; ++e) t[e] = gelu_erf(t[e]);
            }
            if constexpr (EPI == EPI_QKV) {
              // q and k columns: rotary on neighbouring columns (2p, 2p+1), both held by this lane
              if (g.rope.tab || g.rope_cs) {
                const uint32_t at = __umul24((rope_row[q >> 1] >> rope_axis[j][q % CQ]) & 255, rope_stride) + rope_off[j][q % CQ];
                const f32x4 cs = *reinterpret_cast<const f32x4*>(rope_base + at);  // cos,sin,cos,sin
                const float r0 = t[0] * cs[0] - t[1] * cs[1], r1 = t[1] * cs[0] + t[0] * cs[1];
                const float r2 = t[2] * cs[2] - t[3] * cs[3], r3 = t[3] * cs[2] + t[2] * cs[3];
                t[0] = r0; t[1] = r1; t[2] = r2; t[3] = r3;
              }
              t *= n < g.hidden ? g.q_scale : 1.0f;
            }
            v[b][q] = t;
          }
        const int col0 = nw + j0 * 32;
        if constexpr (RESADD) {
          store_block<NB, float, true, FOLDS_SUMS>(chunk, v, static_cast<float*>(g.out), g.ldo, g.row_map, mrow, M, col0, n_end, true,
                                       wt && CS_GEMM_RESADD_WT && !g.plain_stores,
                                       HOLD_TWO ? held[i & 1][j0] : held[0][j0],
                                       folding ? &fold : nullptr);
          if constexpr (HOLD_TWO) {
            if (i + 2 < TM) fetch_old(i + 2, j0, held[i & 1][j0]);
          } else {
            if (i + 1 < TM) fetch_old(i + 1, j0, held[0][j0]);
          }
        } else if constexpr (OUT_F32) {
          store_block<NB, float, false>(chunk, v, static_cast<float*>(g.out), g.ldo, g.row_map, mrow, M, col0, n_end, true, wt);
        } else if constexpr (EPI == EPI_QKV) {
          store_block<NB, bf16_t, false>(chunk, v, static_cast<bf16_t*>(g.out), g.ldo, g.row_map, mrow, M, col0,
                                         2 * g.hidden, wide, wt);
        } else {
          store_block<NB, bf16_t, false>(chunk, v, static_cast<bf16_t*>(g.out), g.ldo, g.row_map, mrow, M, col0, n_end, wide, wt);
          if constexpr (EPI == EPI_GELU_SPLIT) {
            // second half of the row: what the bf16 rounding of the first half dropped
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const bf16x4 h = __builtin_convertvector(v[b][q], bf16x4);
                v[b][q] -= __builtin_convertvector(h, f32x4);
              }
            store_block<NB, bf16_t, false>(chunk, v, static_cast<bf16_t*>(g.out) + N, g.ldo, g.row_map, mrow, M, col0, n_end,
                                           wide && (N & 7) == 0, wt && (N & 63) == 0);
          }
        }
      };
      constexpr int PER = OUT_F32 ? 1 : 2;   // 32-column blocks per 128-byte chunk row
      if constexpr (PER == 2) {
#pragma unroll
        for (int j0 = 0; j0 + 1 < TN; j0 += 2) emit(int_tag<2>{}, j0);
        if constexpr (TN & 1) emit(int_tag<1>{}, TN - 1);
      } else {
#pragma unroll
        for (int j0 = 0; j0 < TN; ++j0) emit(int_tag<1>{}, j0);
      }
      if constexpr (FOLDS_NORM) {
        if (folding) {
          // eight lanes share a row of a 32-column fp32 block: their sums over the wave's columns, added
          // in a fixed order, are the tile's contribution to the row's sum of squares
#pragma unroll
          for (int it = 0; it < 4; ++it) {
            float s = fold.ssacc[it];
            s += __shfl_xor(s, 1);
            s += __shfl_xor(s, 2);
            s += __shfl_xor(s, 4);
            if ((lane & 7) == 0) extra_lds[256 + wn * BM + wm * WM + i * 32 + it * 8 + (lane >> 3)] = s;
          }
          if constexpr (FOLDS_SUMS) {
            if (folding_sums) {
#pragma unroll
              for (int it = 0; it < 4; ++it) {
                float s = fold.s1acc[it];
                s += __shfl_xor(s, 1);
                s += __shfl_xor(s, 2);
                s += __shfl_xor(s, 4);
                if ((lane & 7) == 0) extra_lds[256 + (WGN + wn) * BM + wm * WM + i * 32 + it * 8 + (lane >> 3)] = s;
              }
            }
          }
        }
      }
    }
  }
  if constexpr (FOLDS_NORM) {
    if (folding) {
      // the waves' sums over their columns, added in wave order: the tile's share of each row's sum of squares
      __syncthreads();
      const int t = threadIdx.x;
      if (t < BM && m0 + t < M) {
        float s = extra_lds[256 + t];
#pragma unroll
        for (int w2 = 1; w2 < WGN; ++w2) s += extra_lds[256 + w2 * BM + t];
        g.ss_out[(int64_t)(n0 / BN) * g.ss_stride + m0 + t] = s;
        if constexpr (FOLDS_SUMS) {
          if (folding_sums) {
            float s1 = extra_lds[256 + WGN * BM + t];
#pragma unroll
            for (int w2 = 1; w2 < WGN; ++w2) s1 += extra_lds[256 + (WGN + w2) * BM + t];
            g.s1_out[(int64_t)(n0 / BN) * g.ss_stride + m0 + t] = s1;
          }
        }
      }
    }
  }
}

// What a launch does with the tiles that would leave the chip mostly idle:
//  TAIL_LIGHT (M not a multiple of BM): the workgroups behind those of the full tile rows take the
//    remaining rows in 64-row tiles (same threads, every wave a 64 x BN/waves strip): they stream the
//    same W slices but do a quarter of the MFMAs, so that tile row costs microseconds instead of a round
//    of the chip.
//  TAIL_SPLIT (no light tail, the last round of the chip at most half full): the tiles of that
//    last round are cut in two along M and run as BM/2-row tiles by twice as many workgroups, so the
//    round takes little more than half as long.  A round costs the same however few of its tiles are
//    there (measured: 864 tiles of 256 x 256 take as long as 1024), and 8192 x 6912 is 3 3/8 rounds.
//  A 256 x 256 launch with a light tail splits its last round as well, where its halves and the light tiles make one
//    round (GemmArgs::half_tiles; the tiles counted are the full ones, the light tiles run behind the halves):
//    5128 x 3840 x 1280, 300 tiles and 15 light ones, 72 -> 64 us, 9300 rows 105 -> 98, 14 000 rows 140 -> 133.
enum { TAIL_NONE = 0, TAIL_LIGHT = 1, TAIL_SPLIT = 2 };
constexpr int CHIP_CUS = 256;
template <int BM, int BN, int TAIL>
constexpr bool tail_splits() { return TAIL == TAIL_SPLIT || (TAIL == TAIL_LIGHT && BM == 256 && BN == 256); }

// tile id -> first row / column.  Ids walk the tile grid in bands of GROUP_M tile rows, row index
// fastest, so the ~32 tiles an XCD runs at a time form a GROUP_M x 8 block that shares GROUP_M slices
// of A and 8 slices of W per k-step (an L2 miss on every W byte otherwise: measured 427 clocks average
// L2 read latency and the L1 miss queue full 58 % of the time).
// A workgroup's way to its first load is a chain of scalar work that nothing hides, a tenth of a small launch, so no
// division is left in that of a whole or a half tile (the 64-row tiles of a light tail divide by their number): x / d = high 64 bits of x * reciprocal(d), exact for all x < 2^32, 2 <= d < 2^32 (the reciprocal
// exceeds 2^64 / d by at most one, which adds less than x / 2^64 < 1 / d to the quotient).  With the launch's tile counts in
// the arguments and the arguments in two lines: 256 x 3840 x 1280 10.8 -> 10.4 us, 256 x 1280 x 3456 in three parts 8.4 ->
// 8.1, a lone 64 x 64 x 64 tile 3.4 -> 3.0.
constexpr int GROUP_M = 4;   // (2: the same within noise; 8: 1 % slower on the 32-image batch; 16: 4 % slower)
static uint64_t reciprocal(uint32_t d) { return d >= 2 ? ~0ull / d + 1 : 0; }   // (2^64 / d rounded up)
__device__ __forceinline__ int divide(int x, uint64_t recip) {
  const uint64_t lo = (uint64_t)(uint32_t)x * (uint32_t)recip, hi = (uint64_t)(uint32_t)x * (uint32_t)(recip >> 32);
  return (int)((hi + (lo >> 32)) >> 32);
}
template <int BM, int BN>
__device__ __forceinline__ void tile_origin(const GemmArgs& g, int id, int& m0, int& n0) {
  const int band_tiles = GROUP_M * g.tiles_n, band = divide(id, g.band_recip), in_band = id - band * band_tiles;
  const int rows = g.tiles_m - band * GROUP_M;   // of the band; the last one may have fewer than four
  // (a third: 2^32 / 3 rounded up times in_band < 2^31 is exact)
  const int col = rows >= GROUP_M ? in_band >> 2 : rows == 3 ? (int)__umulhi((uint32_t)in_band, 0x55555556u) : rows == 2 ? in_band >> 1 : in_band;
  m0 = (band * GROUP_M + in_band - col * (rows < GROUP_M ? rows : GROUP_M)) * BM;
  n0 = col * BN;
}

// the b-th of n workgroups, b % 8 its XCD -> its place in the order in which every XCD has a contiguous run
__device__ __forceinline__ int xcd_run(int b, int n) {
  const int xcd = b & 7, idx = b >> 3, per = n >> 3, rem = n & 7;
  return xcd * per + (xcd < rem ? xcd : rem) + idx;
}

// LDS of a launch: that of its main tile, or what the deeper pipeline of its 64-row tail tiles needs.
template <int BM, int BN, int NWAVES, int EPI, int TAIL, int STAGES>
constexpr int launch_lds_bytes() {
  const int main_tile = tile_lds_bytes<BM, BN, NWAVES, EPI, STAGES>();
  if (TAIL != 1 /* TAIL_LIGHT */) return main_tile;
  const int light = light_lds_need<BN, NWAVES, EPI>(light_stages<BN, NWAVES, EPI>());
  return light > main_tile ? light : main_tile;
}

template <int BM, int BN, int WGM, int WGN, int EPI, int TAIL, int STAGES, bool FAR>
__global__ __launch_bounds__(64 * WGM * WGN)
// (the four-wave 128 x 160 tile must leave room for a second workgroup on the CU: 256 registers, not 512)
__attribute__((amdgpu_waves_per_eu(2))) void gemm_kernel(GemmArgs g) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int LDS = launch_lds_bytes<BM, BN, WGM * WGN, EPI, TAIL, STAGES>();
  if (g.splits > 1) {   // split K (plain fp32 partial sums only): this workgroup's K slices of A and W, its partial sums
    const int kt = g.K >> 6, part = (int)blockIdx.y;
    const int first = divide(part * kt, g.split_recip), last = divide((part + 1) * kt, g.split_recip);
    g.A += (int64_t)first * 64;
    g.W += (int64_t)first * 64;
    g.K = (last - first) * 64;
    g.out = static_cast<float*>(g.out) + (int64_t)part * g.split_stride;
  }
  constexpr bool LIGHT = TAIL == TAIL_LIGHT, SPLIT = tail_splits<BM, BN, TAIL>();
  static_assert(!LIGHT || light_tail<BN, WGM, WGN, EPI>(), "no 64-row tile for this shape");
  static_assert(!FAR || TAIL == TAIL_NONE, "far rows: whole tiles only");
  static_assert(!SPLIT || (BM / 2 / WGM) % 32 == 0, "half tiles need whole 32-row blocks per wave");
  // workgroups [0, grid_tiles) run whole tiles
  if constexpr (TAIL != TAIL_NONE) {
    int t = (int)blockIdx.x - g.grid_tiles;
    if (t >= 0) {
      if constexpr (SPLIT) {   // the next each take half of a tile of the last round
        if (t < g.half_tiles) {
          // (the half tiles get the same treatment as the tiles: consecutive workgroups run on different XCDs,
          // so every XCD takes a contiguous run of half tiles, both halves of a tile among them)
          t = xcd_run(t, g.half_tiles);
          int m0, n0;
          tile_origin<BM, BN>(g, g.grid_tiles + (t >> 1), m0, n0);
          m0 += (t & 1) * (BM / 2);
          if (m0 >= g.M) return;   // the lower half of a tile of a ragged last tile row may be empty
          tile_body<BM / 2, BN, WGM, WGN, EPI, 2, LDS>(g, smem, m0, n0);
          return;
        }
        t -= g.half_tiles;
      }
      if constexpr (LIGHT) {   // the others take the rows behind the full tile rows in 64-row tiles
        const int full = g.tiles_m * BM, tail_m = (g.M - full + 63) / 64;
        tile_body<64, BN, 1, WGM * WGN, EPI, light_stages<BN, WGM * WGN, EPI>(), LDS>(
            g, smem, full + (t % tail_m) * 64, (t / tail_m) * BN);
      }
      return;
    }
  }
  // workgroup -> tile.  Consecutive workgroups land on different XCDs (b % 8), each with its own
  // L2, so every XCD gets a contiguous range of tile ids.
  int m0, n0;
  tile_origin<BM, BN>(g, xcd_run((int)blockIdx.x, g.grid_tiles), m0, n0);
  tile_body<BM, BN, WGM, WGN, EPI, STAGES, LDS, FAR>(g, smem, m0, n0);
}

// Measurement switch: CS_GEMM_NO_TAIL_SPLIT=1 in the environment keeps whole tiles in the last round, so
// the effect of the half tiles can be measured from the committed tree (read once).
static bool tail_split_off() {
  static const bool off = [] {
    const char* v = getenv("CS_GEMM_NO_TAIL_SPLIT");
    return v && *v && *v != '0';
  }();
  return off;
}

template <int BM, int BN, int WGM, int WGN, int EPI, int TAIL, int STAGES, bool FAR = false>
static cs_status launch_one(const GemmArgs& g, hipStream_t stream) {
  constexpr int NT = 64 * WGM * WGN;
  constexpr int LDS = launch_lds_bytes<BM, BN, WGM * WGN, EPI, TAIL, STAGES>();
  static_assert(LDS <= 160 * 1024, "LDS of a CU");
  auto kern = gemm_kernel<BM, BN, WGM, WGN, EPI, TAIL, STAGES, FAR>;
  GemmArgs ga = g;
  const int tiles_n = (g.N + BN - 1) / BN;
  // the tiles that are run whole or in halves: with a light tail those of the full tile rows
  ga.tiles_n = tiles_n;
  ga.tiles_m = TAIL == TAIL_LIGHT ? g.M / BM : (g.M + BM - 1) / BM;
  const int whole = ga.tiles_m * tiles_n, light = TAIL == TAIL_LIGHT ? ((g.M % BM + 63) / 64) * tiles_n : 0;
  int tiles = whole + light;   // workgroups
  ga.half_tiles = 0;
  if constexpr (tail_splits<BM, BN, TAIL>()) {   // the tiles of a last round that is at most half full twice, as half tiles
    // (beside a light tail only where halves and light tiles make one round together: a third one costs what the split
    // saves, 8224 x 3072 x 1024 61 -> 65 us with 256 halves and 12 light tiles)
    const int rest = whole % CHIP_CUS;
    if (TAIL == TAIL_SPLIT || (whole > CHIP_CUS && 2 * rest + light <= CHIP_CUS && g.splits <= 1 && !tail_split_off())) {
      ga.half_tiles = 2 * rest;
      tiles += rest;
    }
  }
  // LDS for a rotary table by position behind the launch's own: what a CU has left, for two workgroups where two fit
  constexpr int POS_BYTES = 256 * 4, PER_CU = NT == 256 && STAGES == 2 && 2 * LDS <= 160 * 1024 ? 2 : 1;
  constexpr int ROPE_ROOM = EPI == EPI_QKV && 160 * 1024 / PER_CU >= LDS + POS_BYTES ? (160 * 1024 / PER_CU - LDS - POS_BYTES) / 1024 * 1024 : 0;
  const int lds = LDS + (g.rope.tab ? g.rope.bytes + POS_BYTES : 0);
  if (g.rope.tab && (g.rope.bytes > ROPE_ROOM || (g.rope.bytes & 1023) || g.rope.pitch % 32 != 16))
    return fail(CS_ERR_INVALID_ARG, "gemm: no room for the rotary table");
  if (g.rope_room) *g.rope_room = ROPE_ROOM;
  if (g.describe) {
    const int n = snprintf(g.describe, 96, "gemm_kernel<%d, %d, %d, %d, %d, %d> 16x16x32%s", BM, BN, WGM, WGN, EPI, TAIL, FAR ? ", far rows" : "");
    if (ga.half_tiles > 0) snprintf(g.describe + n, 96 - n, ", %d half tiles", ga.half_tiles);
    return CS_OK;
  }
  // one attribute call per instantiation (two threads that both see `false` repeat a harmless call)
  static std::atomic<bool> attr_set{false};
  if (!attr_set.load(std::memory_order_acquire)) {
    CS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, EPI == EPI_QKV ? 160 * 1024 : LDS));
    attr_set.store(true, std::memory_order_release);
  }
  ga.grid_tiles = whole - ga.half_tiles / 2;
  ga.band_recip = reciprocal((uint32_t)(GROUP_M * tiles_n));
  ga.split_recip = reciprocal((uint32_t)(g.splits > 1 ? g.splits : 0));
  // The residual epilogue's stores are write-through except in launches of the narrow tiles that run more than
  // one round: there the next round's operand loads queue behind the first round's burst of stores, and stores
  // that stay in the L2's write-back do better (16 384 tokens: out projection 487 -> 521, down projection
  // 757 -> 775 TFLOP/s; one round and the 256 x 256 tile: 1 - 4 % worse).  CS_GEMM_RESADD_PLAIN in the environment
  // (read once) overrides the rule for measurement: 0 never plain, 1 always.
  {
    static const int mode = [] { const char* v = getenv("CS_GEMM_RESADD_PLAIN"); return v && *v >= '0' && *v <= '1' ? *v - '0' : 2; }();
    ga.plain_stores = mode == 1 || (mode == 2 && BN < 256 && tiles > CHIP_CUS);
  }
  hipLaunchKernelGGL(kern, dim3(tiles, g.splits > 1 ? g.splits : 1), dim3(NT), lds, stream, ga);
  CS_HIP(hipGetLastError());
  return CS_OK;
}

template <int BM, int BN, int WGM, int WGN, int EPI, int STAGES = default_stages<BM, BN, WGM * WGN>()>
static cs_status launch_cfg(const GemmArgs& g, hipStream_t stream) {
  // the light-tail variant where the last, partly empty tile row is at least 1/64 of the tile rows
  if constexpr (BM > 64 && light_tail<BN, WGM, WGN, EPI>()) {
    if (g.M % BM != 0 && (g.M + BM - 1) / BM <= 64) return launch_one<BM, BN, WGM, WGN, EPI, TAIL_LIGHT, STAGES>(g, stream);
  }
  // half tiles for a last round that is at most half full (the big tile only: that is where a round is long)
  if constexpr (BM == 256 && BN == 256) {
    const int tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN), tail = tiles % CHIP_CUS;
    if (g.splits <= 1 && tiles > CHIP_CUS && tail > 0 && tail <= CHIP_CUS / 2 && !tail_split_off())
      return launch_one<BM, BN, WGM, WGN, EPI, TAIL_SPLIT, STAGES>(g, stream);
  }
  return launch_one<BM, BN, WGM, WGN, EPI, TAIL_NONE, STAGES>(g, stream);
}

// The fewest 256 x 256 tiles beyond one round of the chip for which a launch takes that tile: 257.  With the half
// tiles of a split last round such a launch never runs below 2/3 full (257 tiles: a round and a half round),
// which beats what the 128 x 128 tiles lose inside the CU (3072 tokens: gate|up 731 -> 872 TFLOP/s, the step 7.30
// -> 6.98 ms; 6144 tokens: 10.74 -> 10.33 ms).  CS_GEMM_BIG_MIN in the environment (read once) sets another
// threshold for measurement; 384, a round and a half, was the rule before the half tiles existed.
static int64_t big_tile_min() {
  static const int64_t v = [] {
    const char* e = getenv("CS_GEMM_BIG_MIN");
    const long x = e ? atol(e) : 0;
    return (int64_t)(x > 256 && x <= 4096 ? x : 257);
  }();
  return v;
}

static int small_resadd_pair() {
  static const int mode = [] {
    const char* v = getenv("CS_GEMM_SMALL_PAIR");
    return v && *v >= '0' && *v <= '2' ? *v - '0' : 2;
  }();
  return mode;
}

static bool narrow_resadd() {
  static const bool on = [] {
    const char* v = getenv("CS_GEMM_NARROW_RESADD");
    return v && *v && *v != '0';
  }();
  return on;
}

// Launches that fit one round of the chip: one workgroup per CU, several K slices in flight, and as many CUs at work as
// the shape allows.  Such a launch waits for its operands: measured with weights that come from HBM, a slice takes the
// times below whatever the number of workgroups (a lone CU draws 45 - 60 B/ns), so the smallest tile that still makes
// at most one round is the fastest (256 x 3840 x 1280: 64 x 64 9.4 us, 64 x 128 12.8, 128 x 128 16.9, and 20.4 with two
// slices in flight; 1024 x 3840 x 1280: 128 x 128 16.0, two per CU 20.2; 512 x 6912 x 1280: 17.2 against 23.0 for one
// and a half rounds of 64 x 128).  More slices in flight change nothing (eight for 64 x 64: 10.0 against 9.5 us), nor do
// weights that are already in the memory-side cache (7.8 us).
struct SmallTile {
  int bm, bn;
};
static constexpr SmallTile SMALL_TILES[] = {{64, 64}, {64, 128}, {128, 128}, {128, 256}};
enum { TILE_64 = 0, TILE_64x128, TILE_128, TILE_128x256, N_SMALL_TILES };
// The last stands in where 128 x 128 needs more than a round: 1100 - 2048 rows, N = 3584 - 5120, K = 1280 take 20 - 23 us
// on it, against 20 - 28 on two-stage 128 x 128 tiles, two per CU, which are ahead by up to 2 us where they number 260 -
// 420 and behind by up to 5 beyond.

static bool one_round(int64_t M, int64_t N, int64_t parts, int bm, int bn) {
  return ((M + bm - 1) / bm) * ((N + bn - 1) / bn) * parts <= CHIP_CUS;
}
// the first of those tiles from `first` on that makes at most one round of the chip, N_SMALL_TILES if none does
static int small_tile(int64_t M, int64_t N, int64_t parts, int first) {
  int t = first;
  while (t < N_SMALL_TILES && !one_round(M, N, parts, SMALL_TILES[t].bm, SMALL_TILES[t].bn)) ++t;
  return t;
}

// (as launch_epi takes it for EPI_F32)
bool gemm_split_tile(int64_t M, int64_t N, int64_t parts, int32_t* bm, int32_t* bn) {
  const int t = small_tile(M, N, parts, TILE_64);
  if (t == N_SMALL_TILES) return false;
  *bm = SMALL_TILES[t].bm;
  *bn = t == TILE_128x256 && N % 32 == 0 && one_round(M, N, parts, 128, 160) ? 160 : SMALL_TILES[t].bn;
  return true;
}

template <int EPI>
static cs_status launch_epi(const GemmArgs& g, hipStream_t stream) {
  // rows whose offsets inside a tile do not fit 32 bits
  if (!gemm_rows_addressable(g.M, g.lda) || !gemm_rows_addressable(g.N, g.ldw))
    return launch_one<128, 128, 2, 2, EPI, TAIL_NONE, 2, true>(g, stream);
  // Tile choice by the number of workgroups it yields for the 256 CUs.
  constexpr bool RESADD = EPI == EPI_RESADD_F32 || EPI == EPI_RESADD_SUMS_F32 || EPI == EPI_RESADD_SCALED_F32;
  // At most one round of small tiles.  (A residual GEMM stays on tiles of which a row has at most eight, so that the
  // next normalisation folds: N = 1280 on its 128 x 160 tiles below.)
  if (!(RESADD && g.N % 160 == 0)) {
    const int t = small_tile(g.M, g.N, g.splits > 1 ? g.splits : 1,
                             EPI == EPI_SWIGLU_BF16 || (RESADD && g.N > 8 * 64) ? TILE_64x128 : TILE_64);
    constexpr int SW = EPI == EPI_SWIGLU_BF16 ? 2 : 4;   // (gate | up pairs need 64 columns per wave)
    if constexpr (EPI != EPI_SWIGLU_BF16) {
      if (t == TILE_64) return launch_one<64, 64, 2, 2, EPI, TAIL_NONE, 4>(g, stream);
    }
    if (t == TILE_64x128) return launch_one<64, 128, 2, SW, EPI, TAIL_NONE, 4>(g, stream);
    if (t == TILE_128) return launch_one<128, 128, 4, 2, EPI, TAIL_NONE, 4>(g, stream);
    // 128 x 160 (eight waves, four stages) before 128 x 256, where whole 32-column blocks fill it: more CUs at work and
    // fewer bytes for each.  1028 x 3840 x 1280 21.5 -> 18.4 us, 1028 x 4096 x 1024 (GELU) 20.0 -> 18.2, 1024 x 5120 x 1280
    // (GELU, folded norm) 26.0 -> 23.0, 1028 x 1024 x 4096 in four parts 17.3 -> 16.0, 1024 x 1280 x 1280 in four 10.0 ->
    // 9.4, 256 x 5120 x 10240 in four 49 -> 42.  (QKV and gate | up pairs need waves of whole 32 or 64 columns.)
    if constexpr (EPI != EPI_SWIGLU_BF16 && EPI != EPI_QKV && !RESADD) {
      if (t == TILE_128x256 && g.N % 32 == 0 && one_round(g.M, g.N, g.splits > 1 ? g.splits : 1, 128, 160))
        return launch_one<128, 160, 4, 2, EPI, TAIL_NONE, 4>(g, stream);
    }
    // Gate | up pairs take it in small batches (512 < M <= 1152 at N = 6912): 1024 x 6912 x 1280, 216 workgroups, 20.1 us
    // against 25.7 on 432 of 128 x 128, two per CU: 983 KB a CU in one queue instead of two of 655.  A step of the 7B-style
    // tower: 576 tokens 2379 -> 2346 us, 676 2470 -> 2377, 900 2672 -> 2564, 1024 2916 -> 2731, 1088 3159 -> 3108.
    if constexpr (!RESADD) {
      if (t == TILE_128x256 && (EPI != EPI_QKV || (2 * g.hidden) % 256 == 0) && (EPI != EPI_SWIGLU_BF16 || g.small_batch))
        return launch_one<128, 256, 2, 4, EPI, TAIL_NONE, 3>(g, stream);
    }
  }
  // (The thresholds from here on, and the figures beside them, were measured on a K loop with a barrier between its slices.)
  const int64_t tm = (g.M + 255) / 256;
  const int64_t big = tm * ((g.N + 255) / 256);
  const bool big_ok = EPI != EPI_QKV || (2 * g.hidden) % 256 == 0;
  // (the scaled residual epilogue spills registers with eight waves and with 160-wide wave tiles: it
  // takes the 256 x 128 or 128 x 128 tiles)
  constexpr bool EIGHT_WAVES_OK = EPI != EPI_RESADD_SCALED_F32;
  if constexpr (EIGHT_WAVES_OK) {
    // 256 x 256 for more than a round of the chip (CS_GEMM_NARROW_RESADD=1 in the environment makes the
    // residual add take the narrow tile below at any size, for measurement: the 32-image batch 166.5 -> 177.4 ms)
    const bool narrow_first = EPI == EPI_RESADD_F32 && g.N % 160 == 0 && narrow_resadd();
    // (the residual GEMMs keep a round and a half: below it their narrow tiles make whole rounds, e.g. two at 16 384 tokens)
    constexpr bool RES = EPI == EPI_RESADD_F32 || EPI == EPI_RESADD_SUMS_F32;
    if (big >= (RES ? 384 : big_tile_min()) && big_ok && !narrow_first) return launch_cfg<256, 256, 2, 4, EPI>(g, stream);
  }
  // 192 x 256 (eight waves of 96 x 64; two stages, three do not fit) where 128 x 256 need more than a round of the chip and
  // these make one: K loops of one-round launches go at the pace of a CU's operand loads, 1147 KB at K = 1280 instead of 1311
  // for 256 x 256, with three quarters of the products behind each slice and, at most widths, more CUs at work.  Without them such
  // a launch runs on 256 x 256 where those fill 5/8 of a round, on 128 x 128, two per CU, where they do not, or in more than a round
  // of 256 x 160 or 256 x 128: N = 5120 and 4096, and from 8193 rows on N = 1280 (to 9792: first convolution, patch embedding)
  // and 1024 (to 12 288).  us, those -> 192 x 256: 8196 x 1280 x 1280 50.1 -> 32.3, 9792 rows 48.2 -> 30.8, 8224 x 1280 x 3840 115
  // -> 74, 8224 x 1024 x 640 18.3 -> 16.2, 12 288 rows 24.9 -> 19.2, 2052 x 5120 x 5120 154 -> 101, 3072 x 4096 x 4096 112 -> 81, 1300 x
  // 9216 x 1280 44.6 -> 31.4, 3264 x 3840 x 1280 46 -> 30, the least 2310 x 3584 x 5120 106 -> 102.  A step: 7B-style tower, gate|up of
  // 1280 tokens 3715 -> 3547 us, 1428 3875 -> 3740, QKV of 2392 5955 -> 5590, of 3072 5790 -> 5661, patches and merger of 8196 13.82 ->
  // 13.65 ms; audio tower, QKV and fc1 of 2200 6367 -> 5404 us, QKV of 2512 6928 -> 6646; class-token tower, QKV of 3084 3983 -> 3780,
  // both ends of 9252 10.55 -> 10.35 ms.  Also where 256 x 256 make as many tiles (255 of 576 x 21 760, gate|up: eight layers 1002 -> 970).
  // (256 x 160 in one round are as fast: fc1 of 1600 - 2048 audio tokens within 1 %.)
  const bool one_192 = !RESADD && big_ok && g.splits <= 1 && !one_round(g.M, g.N, 1, 128, 256) && one_round(g.M, g.N, 1, 192, 256);
  if constexpr (EPI != EPI_QKV && EPI != EPI_SWIGLU_BF16) {
    // narrow outputs (N = hidden = 1280): 256 x 160 tiles, eight waves of 64 x 80 (a wave's third 32-column block
    // half used), give M/256 * 8 workgroups, one round of the chip at M = 8192
    if constexpr (EIGHT_WAVES_OK) {
      if (g.N % 160 == 0 && tm * (g.N / 160) >= 192 && !(one_192 && tm * (g.N / 160) > CHIP_CUS)) {
        return launch_cfg<256, 160, 4, 2, EPI>(g, stream);
      }
    }
    // the same for N = 1024: 256 x 128 tiles (eight waves of 64 x 64 leave room for the scaled residual epilogue too)
    // (not for N = 1280, which it would cut into ten column tiles, too many for the next normalisation to fold:
    // 5120 tokens, 9.73 -> 9.35 ms per step on the 128 x 160 tiles below)
    if (g.N % 128 == 0 && g.N % 160 != 0 && tm * (g.N / 128) >= 192 && !(one_192 && tm * (g.N / 128) > CHIP_CUS)) {
      return launch_cfg<256, 128, 4, 2, EPI>(g, stream);
    }
  }
  if constexpr (!RESADD) {
    if (one_192) return launch_one<192, 256, 2, 4, EPI, TAIL_NONE, 2>(g, stream);
  }
  if constexpr (EIGHT_WAVES_OK) {
    // 256 x 256 also when it fills one round to 5/8 or more (batches of 2 - 4 images: 2 - 7 % faster than
    // 128 x 128 tiles; at 120 workgroups it loses)
    if (big >= 160 && big <= 256 && big_ok) return launch_cfg<256, 256, 2, 4, EPI>(g, stream);
  }
  // a residual GEMM with N = 1280 too small for the tiles above: 128 x 160 tiles rather than 128 x 128, which makes
  // eight column tiles instead of ten, so the next normalisation still folds into it (vision tower, 4096 tokens:
  // 8.32 -> 7.77 ms per step; audio tower, 3000 tokens: 8.08 -> 7.94 ms).  Up to one tile per CU they run with eight waves of 32 x 80, so that every SIMD has two waves to
  // alternate between (3072 tokens: 6.91 -> 6.73 ms, 4096: 7.58 -> 7.44); beyond that with four waves of 64 x 80,
  // two workgroups per CU.  CS_GEMM_SMALL_PAIR in the environment, for measurement: 0 keeps the 128 x 128 tiles,
  // 1 takes four waves at any size.
  if constexpr (EPI == EPI_RESADD_F32 || EPI == EPI_RESADD_SUMS_F32) {
    if (g.N % 160 == 0 && g.splits <= 1 && small_resadd_pair() > 0) {
      // 64 x 160, four waves of 32 x 80 and three K slices in flight, from half a chip of them to a whole one (N = 1280: 961 -
      // 2048 rows): such a launch goes at the pace of its operand loads, of which a CU then pulls 573 KB at K = 1280 instead of
      // 737, and twice as many CUs work.  A step of the 7B-style tower, out projections on 64 x 160 against 128 x 160: 2048 tokens
      // 4172 / 4297 us (1520 3791 / 3921 and 1760 4052 / 4198, unsplit for the measurement).
      // (Fewer of them lie in batches whose residual GEMMs run split over K, or in narrow towers.)
      if (one_round(g.M, g.N, 1, 64, 160) && (int64_t)((g.M + 63) / 64) * (g.N / 160) >= CHIP_CUS / 2)
        return launch_one<64, 160, 2, 2, EPI, TAIL_NONE, 4>(g, stream);
      const int64_t tiles = ((g.M + 127) / 128) * (g.N / 160);
      // Beyond one round of 128 x 160, up to where 256 x 160 fill the chip (N = 1280: 4097 - 5888 rows): one round of 192 x 160, six
      // waves of 64 x 80, three stages, 901 KB of operands a CU at K = 1280.  As 128 x 160, two workgroups on some CUs and one on
      // others, those with two pulled 1475 KB.  A step of the 7B-style tower: 4100 tokens 7064 -> 6787 us, 4232 7571 -> 7335, 5120
      // 8632 -> 8420, 5888 8987 -> 8732; of the audio tower: 4500 9519 -> 9084, 5128 9165 -> 8780.
      if (g.small_batch && tiles > CHIP_CUS && one_round(g.M, g.N, 1, 192, 160))
        return launch_one<192, 160, 3, 2, EPI, TAIL_NONE, 3>(g, stream);
      if (small_resadd_pair() == 2 && tiles <= CHIP_CUS) return launch_cfg<128, 160, 4, 2, EPI>(g, stream);
      return launch_cfg<128, 160, 2, 2, EPI>(g, stream);
    }
  }
  return launch_cfg<128, 128, 2, 2, EPI>(g, stream);
}

int32_t gemm_rope_room(int64_t M, int32_t hidden, int32_t head_dim, int64_t K, int64_t lda, int64_t ldw) {
  // (the launcher says so itself)
  if (M <= 0 || M > 0x7fffffff) return 0;
  char name[96] = {0};
  int32_t room = 0;
  GemmArgs g = {};
  g.M = (int32_t)M; g.N = 3 * hidden; g.K = (int32_t)K; g.lda = lda; g.ldw = ldw; g.ldo = 2 * (int64_t)hidden; g.hidden = hidden; g.head_dim = head_dim;
  g.ld_vt = round_up(M, 64); g.describe = name; g.rope_room = &room;
  return launch_gemm(EPI_QKV, g, nullptr) == CS_OK ? room : 0;
}

int32_t gemm_norm_fold_parts(int64_t M, int64_t N, int64_t K, int64_t pitch, bool scaled, bool sums) {
  // ask the launcher itself which tile such a residual GEMM runs on: one partial sum per column tile
  if (M <= 0 || M > 0x7fffffff || N <= 0 || K <= 0 || (N & 3) || (K & 63)) return 0;
  char name[96] = {0};
  GemmArgs g = {};
  g.M = (int32_t)M; g.N = (int32_t)N; g.K = (int32_t)K; g.lda = g.ldw = pitch; g.ldo = N; g.describe = name;
  g.col_scale = scaled ? reinterpret_cast<const float*>(uintptr_t(16)) : nullptr;   // only its alignment is looked at
  g.s1_out = sums ? reinterpret_cast<float*>(uintptr_t(16)) : nullptr;              // a LayerNorm tower: sums as well
  int bm = 0, bn = 0;
  if (launch_gemm(scaled ? EPI_RESADD_SCALED_F32 : EPI_RESADD_F32, g, nullptr) != CS_OK ||
      sscanf(name, "gemm_kernel<%d, %d", &bm, &bn) != 2 || bn <= 0) return 0;
  const int64_t parts = (N + bn - 1) / bn;
  return parts <= 8 ? (int32_t)parts : 0;
}

cs_status launch_gemm(int epilogue, const GemmArgs& g_in, hipStream_t stream) {
  GemmArgs g = g_in;
  if (g.M <= 0 || g.N <= 0) return CS_OK;
  if (g.ldw == 0) g.ldw = g.K;
  if (g.ldw < g.K || (g.ldw & 7)) return fail(CS_ERR_INVALID_ARG, "gemm: ldw must be at least K and a multiple of 8");
  if (g.splits > 1 && (epilogue != EPI_F32 || g.bias || g.row_map || g.splits > 16 || g.splits > g.K >> 6 ||
                       g.split_stride < (int64_t)g.M * g.ldo || (g.split_stride & 3)))
    return fail(CS_ERR_UNSUPPORTED, "gemm: split K writes plain fp32 partial sums (no bias, no row map), at most 16 parts of whole K slices");
  if (g.K <= 0 || (g.K & 63)) return fail(CS_ERR_UNSUPPORTED, "gemm: K must be a positive multiple of 64");
  // lda < K is allowed: rows may overlap (a k=3 convolution reads three consecutive frames per row)
  if ((g.lda & 7) || (reinterpret_cast<uintptr_t>(g.A) & 15) || (reinterpret_cast<uintptr_t>(g.W) & 15))
    return fail(CS_ERR_INVALID_ARG, "gemm: A and W rows must be 16-byte aligned");
  if ((g.N & 3) || (g.ldo & 3) || (reinterpret_cast<uintptr_t>(g.out) & 15) || (reinterpret_cast<uintptr_t>(g.bias) & 15))
    return fail(CS_ERR_UNSUPPORTED, "gemm: N and the output row stride must be multiples of 4, out and bias 16-byte aligned");
  switch (epilogue) {
    case EPI_BF16: return launch_epi<EPI_BF16>(g, stream);
    case EPI_F32: return launch_epi<EPI_F32>(g, stream);
    case EPI_GELU_BF16: return launch_epi<EPI_GELU_BF16>(g, stream);
    case EPI_GELU_F32: return launch_epi<EPI_GELU_F32>(g, stream);
    case EPI_GELU_SPLIT: return launch_epi<EPI_GELU_SPLIT>(g, stream);
    case EPI_RESADD_F32:
    case EPI_RESADD_SUMS_F32:
      return g.s1_out ? launch_epi<EPI_RESADD_SUMS_F32>(g, stream) : launch_epi<EPI_RESADD_F32>(g, stream);
    case EPI_RESADD_SCALED_F32:
      if (!g.col_scale || (reinterpret_cast<uintptr_t>(g.col_scale) & 15))
        return fail(CS_ERR_INVALID_ARG, "gemm: the scaled residual epilogue needs a 16-byte aligned col_scale");
      return launch_epi<EPI_RESADD_SCALED_F32>(g, stream);
    case EPI_SWIGLU_BF16:
      if (g.N & 63) return fail(CS_ERR_UNSUPPORTED, "gemm: swiglu needs N % 64 == 0");
      return launch_epi<EPI_SWIGLU_BF16>(g, stream);
    case EPI_QKV:
      if ((g.M & 3) || (g.hidden & 63) || (g.head_dim & 3) || g.N != 3 * g.hidden || (g.ld_vt & 3) ||
          (reinterpret_cast<uintptr_t>(g.vt) & 7))
        return fail(CS_ERR_UNSUPPORTED, "gemm: qkv epilogue needs M % 4 == 0, hidden % 64 == 0, head_dim % 4 == 0, N == 3 hidden");
      // the (cos, sin) table of a tile's tokens and the epilogue chunks share LDS behind the K loop
      if ((g.rope_cs || g.rope.tab) && g.head_dim > 80) return fail(CS_ERR_UNSUPPORTED, "gemm: rotary epilogue needs head_dim <= 80");
      return launch_epi<EPI_QKV>(g, stream);
    default: return fail(CS_ERR_INVALID_ARG, "gemm: unknown epilogue");
  }
}

}  // namespace cs

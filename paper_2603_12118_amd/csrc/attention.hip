// Variable-length attention for gfx950, one kernel for window layers and full layers.
//
// A work item names a block of queries [q0,q1) and the keys [kv0,kv1) they attend to (both in
// token indices of the packed batch); a window layer has one item per window, a full layer
// cuts every sequence into query blocks.  Inside a workgroup every wave owns 32 queries and
// all waves walk the same 64-key tiles, which are staged in LDS once per workgroup.
//
// Scores are computed transposed, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16: a lane then holds
// one query column (lane % 32) and 16 of the 32 key rows of a tile, so the online-softmax state
// (running max, running sum, rescale factor) is per lane, and the exponentiated scores are
// already laid out as the B operand of the second product O^T = V^T P^T.  V is consumed
// transposed (token-contiguous), which is how the QKV projection stores it.  q arrives
// pre-multiplied by softmax_scale * log2(e); probabilities are exp2 of score differences.
#include "common.h"

namespace cs {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

typedef float f32x2_a __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_a __attribute__((ext_vector_type(2)));
// two floats -> packed bf16 pair (v_cvt_pk_bf16_f32, round to nearest even)
__device__ __forceinline__ uint32_t pack2_a(float a, float b) {
  const f32x2_a v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_a));
}

// v as a value the compiler knows nothing about: what is computed from it is not kept in registers from an earlier time
__device__ __forceinline__ int afresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Window layers launch thousands of two-wave workgroups, each a short chain load -> stage ->
// MFMA -> store: latency is hidden only by residency, so the single-tile variant is held to 168 registers
// (three waves per SIMD, six workgroups per CU, which is also what their LDS tiles allow).
// SINGLE: every work item has at most 64 keys (windows of up to 64 tokens): one tile, nothing to
// prefetch, so the staging registers are dead before the accumulators come alive.
// KG > 1: the key tiles of an item are dealt to KG groups of NW / KG waves, each with tiles of its own in LDS; the
// groups' running maxima, sums and outputs are merged at the end.  For launches whose items do not fill the chip, where
// the time is the number of tiles one workgroup walks (1.4 us each, mostly waiting): 1025 keys, 16 heads 43 us in two
// launches -> 18.6 us; 1500 keys, 20 heads 34.2 -> 26.2 us.  (Four groups of 64 queries draw twice the bytes: 20.5 and
// 28.2 us.)  plan.cpp says which batches take it.
// (Waves per SIMD: four groups are taken for at most one workgroup per CU (plan.cpp), so they have the registers of two.)
constexpr int attn_waves(int nw, bool single, int kg) { return single ? 3 : nw == 8 && kg < 4 ? 4 : 2; }
template <int DH, int NW, int QT, bool SINGLE, int KG = 1>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(attn_waves(NW, SINGLE, KG), attn_waves(NW, SINGLE, KG))))
void attn_kernel(AttnArgs a) {
  constexpr int NWG = NW / KG;           // waves of a key group
  constexpr int NT = 64 * NWG;
  static_assert((NT & (NT - 1)) == 0, "threads of a key group");
  constexpr bool Q_SPLIT = NW == 2 && !SINGLE;   // may run a quarter of a 256-query item
  constexpr int KS = DH / 16;            // k-steps of the score product
  constexpr int DT = (DH + 31) / 32;     // 32-row tiles of O^T
  constexpr int KSTR = DH * 2 + 16;      // LDS row stride of the K tile, bytes
  constexpr int VSTR = 64 * 2 + 16;      // LDS row stride of the V^T tile, bytes
  constexpr int KCH = DH / 8;            // 16-byte chunks per K row
  // Head dimension 80, eight waves: the query fragments wait in LDS (each lane's own 16-byte pieces, read
  // back in lane order: no conflicts) instead of 20 registers, which brings the kernel under 128 registers
  // and a second workgroup onto the CU.
  // (Key groups: the groups have the same queries and write the same bytes.)
  constexpr bool Q_IN_LDS = (DH > 64 && NW == 8) || KG > 1;
  // There the addresses of the batch's last, partly filled tile are computed where that tile is loaded, too: what of them
  // does not change from tile to tile was kept, and eight registers spilled to scratch by every workgroup (36 bytes a
  // lane) for a tile that most never load.  110 940 tokens x 16 heads: 389 002 -> 276 621 KiB written a launch, of which
  // 277 350 are the output; 8 x 1024 tokens 58.4 -> 57.5 us, 2 x 8192 738 -> 733.
  constexpr bool LAST_TILE_AFRESH = DH > 64 && NW == 8;
  static_assert(KG == 1 || (!SINGLE && QT == 1 && DH % 32 == 0), "key groups: one 32-query block per wave");
  constexpr int K_BYTES = 64 * KSTR, V_BYTES = DT * 32 * VSTR;
  __shared__ __align__(16) unsigned char tiles[KG * (K_BYTES + V_BYTES)];
  __shared__ __align__(16) unsigned char q_lds[Q_IN_LDS ? QT * KS * NT * 16 : 16];

  const int group = KG > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT) : 0;
  const int tid = threadIdx.x & (NT - 1), lane = tid & 63, wave = tid >> 6;   // inside the key group
  unsigned char* const k_lds = tiles + group * (K_BYTES + V_BYTES);
  unsigned char* const v_lds = k_lds + K_BYTES;
  const int l31 = lane & 31, lhi = lane >> 5;
  // Workgroup -> (work item, head).  Consecutive workgroups run on different XCDs (id % 8), each with its own L2.
  int head, item;
  {
    const int xcd = blockIdx.x & 7, r = blockIdx.x >> 3;
    if constexpr (SINGLE) {
      // window layers: an XCD takes every eighth window with all its heads one after the other, so the heads of a
      // window, which share the 128-byte lines of its token rows (a head is 128 or 160 bytes of a row), meet in one L2
      item = (r / a.n_heads) * 8 + xcd;
      head = r % a.n_heads;
      if (item >= a.n_work) return;   // (whole workgroup, before any barrier)
    } else {
      // full layers: the (head, item) pairs in head-major order, cut into eight equal runs: the query blocks of one
      // (item, head), which all read that head's K and V^T, run on one XCD at about the same time instead of on
      // all eight (the 32-image batch fetched 10.5 GB per full-attention layer for 0.85 GB of operands)
      const int blocks = a.n_work * (Q_SPLIT ? a.q_split : 1), pairs = blocks * a.n_heads, per = pairs >> 3, rem = pairs & 7;
      if (r >= per + (xcd < rem ? 1 : 0)) return;
      const int p = xcd * per + (xcd < rem ? xcd : rem) + r;
      head = p / blocks;
      item = p - head * blocks;
    }
  }
  AttnWork w;
  if (Q_SPLIT && a.q_split > 1) {   // this workgroup's 64 queries of the item, if it has so many
    w = a.work[item >> 2];
    w.q0 += 64 * (item & 3);
    w.q1 = w.q1 < w.q0 + 64 ? w.q1 : w.q0 + 64;
    if (w.q0 >= w.q1) return;       // (whole workgroup, before any barrier)
  } else {
    w = a.work[item];
  }
  const int hidden = a.n_heads * DH;
  const int64_t ldq = 2 * (int64_t)hidden;
  const bf16_t* qbase = a.qk + head * DH;
  const bf16_t* kbase = a.qk + hidden + head * DH;
  const bf16_t* vbase = a.vt + (int64_t)head * DH * a.ld_vt;
  const int last_tok = a.n_tok - 1;
  const int vt_last = ((a.n_tok + 3) & ~3) - 4;   // last 4-token chunk of a V^T row that was written

  // ---- this wave's queries as B operands: lane = query column, 8 consecutive dims per k-step
  const int qw = w.q0 + wave * (32 * QT);
  bf16x8 qf[QT][KS];
#pragma unroll
  for (int it = 0; it < QT; ++it) {
    int row = qw + it * 32 + l31;
    row = row < last_tok ? row : last_tok;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      qf[it][ks] = *reinterpret_cast<const bf16x8*>(qbase + (int64_t)row * ldq + ks * 16 + lhi * 8);
  }
  if constexpr (Q_IN_LDS) {
#pragma unroll
    for (int it = 0; it < QT; ++it)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) *reinterpret_cast<bf16x8*>(q_lds + ((it * KS + ks) * NT + tid) * 16) = qf[it][ks];
  }

  f32x16 o[QT][DT];
#pragma unroll
  for (int it = 0; it < QT; ++it)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[it][dt][r] = 0.f;
  float mrun[QT], lrun[QT];
#pragma unroll
  for (int it = 0; it < QT; ++it) {
    mrun[it] = -INFINITY;
    lrun[it] = 0.f;
  }

  // ---- K / V^T tile staging: global -> registers (all loads of a tile in flight together, issued
  // before the MFMAs of the previous tile) -> LDS.
  constexpr int K_PT = (64 * KCH + NT - 1) / NT;   // 16-byte chunks of the K tile per thread
  constexpr int V_PT = (DH * 16 + NT - 1) / NT;    // 8-byte chunks of the V^T tile per thread
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  u32x4 kreg[K_PT];
  u32x2 vreg[V_PT];
  // The vector unit and the chain of one tile bound these kernels (full layers: ~100 vector instructions and 32
  // exponentials per wave beside 512 clocks of MFMA), so a tile's addresses cost no vector instructions: a tile that ends
  // inside the batch has a scalar base and 32-bit offsets which a thread keeps.  With 64-bit products per thread and tile,
  // the row maximum exchanged between the halves in every tile and V^T read in 8-byte pieces: 16 x 1500 tokens, 20 heads
  // of 64 222 -> 216 us, 2 x 8192, 16 of 80 761 -> 718, 4 x 3467 320 -> 299, 2000 windows of 64 tokens 379 -> 336.
  // The batch's last, partly filled tile, whose rows and pieces beyond the end must not be read, and pitches that the
  // offsets do not reach go the long way.
  uint32_t koff[K_PT];
#pragma unroll
  for (int u = 0; u < K_PT; ++u) {
    int c = tid + u * NT;
    c = c < 64 * KCH ? c : 64 * KCH - 1;
    koff[u] = (uint32_t)(c / KCH) * (uint32_t)(ldq * 2) + (c % KCH) * 16;
  }
  const uint32_t voff = (uint32_t)(tid >> 4) * (uint32_t)(a.ld_vt * 2) + (tid & 15) * 8;
  const bool near = 64 * ldq * 2 <= 0x7fffffff && (int64_t)(DH + NT / 16) * a.ld_vt * 2 <= 0x7fffffff;
  auto load_tile = [&](int kv) {
    if constexpr (KG > 1) {
      // by 32-bit offsets from the item's first key throughout (attention_groups_addressable)
      const unsigned char* kb = reinterpret_cast<const unsigned char*>(kbase + (int64_t)w.kv0 * ldq);
      const unsigned char* vb = reinterpret_cast<const unsigned char*>(vbase + w.kv0);
#pragma unroll
      for (int u = 0; u < K_PT; ++u) {
        const int c = tid + u * NT;
        int row = kv - w.kv0 + c / KCH;
        row = row < last_tok - w.kv0 ? row : last_tok - w.kv0;
        kreg[u] = *reinterpret_cast<const u32x4*>(kb + ((uint32_t)row * (uint32_t)(ldq * 2) + (c % KCH) * 16));
      }
      int tok = kv - w.kv0 + (tid & 15) * 4;
      tok = tok < vt_last - w.kv0 ? tok : vt_last - w.kv0;
      const uint32_t v0 = (uint32_t)(tid >> 4) * (uint32_t)(a.ld_vt * 2) + tok * 2;
#pragma unroll
      for (int u = 0; u < V_PT; ++u) vreg[u] = *reinterpret_cast<const u32x2*>(vb + (v0 + (uint32_t)u * (uint32_t)(NT / 16 * 2 * a.ld_vt)));
      return;
    }
    if (near && kv + 64 <= a.n_tok) {
      const unsigned char* kb = reinterpret_cast<const unsigned char*>(kbase + (int64_t)kv * ldq);
      const unsigned char* vb = reinterpret_cast<const unsigned char*>(vbase + kv);
#pragma unroll
      for (int u = 0; u < K_PT; ++u) kreg[u] = *reinterpret_cast<const u32x4*>(kb + koff[u]);
#pragma unroll
      for (int u = 0; u < V_PT; ++u) {
        if ((u + 1) * (NT / 16) <= DH || (tid >> 4) + u * (NT / 16) < DH)   // (rows of V^T beyond the head's)
          vreg[u] = *reinterpret_cast<const u32x2*>(vb + (int64_t)u * (NT / 16) * a.ld_vt * 2 + voff);
      }
      return;
    }
    const int t = LAST_TILE_AFRESH ? afresh(tid) : tid;
#pragma unroll
    for (int u = 0; u < K_PT; ++u) {
      int c = t + u * NT;
      c = c < 64 * KCH ? c : 64 * KCH - 1;
      const int r = c / KCH, ch = c % KCH;
      int row = kv + r;
      row = row < last_tok ? row : last_tok;
      kreg[u] = *reinterpret_cast<const u32x4*>(kbase + (int64_t)row * ldq + ch * 8);
    }
#pragma unroll
    for (int u = 0; u < V_PT; ++u) {
      int c = t + u * NT;
      c = c < DH * 16 ? c : DH * 16 - 1;
      const int d = c >> 4, ch = c & 15;
      int tok = kv + ch * 4;
      tok = tok < vt_last ? tok : vt_last;
      vreg[u] = *reinterpret_cast<const u32x2*>(vbase + (int64_t)d * a.ld_vt + tok);
    }
  };
  auto store_tile = [&]() {
#pragma unroll
    for (int u = 0; u < K_PT; ++u) {
      const int c = tid + u * NT;
      if (c < 64 * KCH) *reinterpret_cast<u32x4*>(k_lds + (c / KCH) * KSTR + (c % KCH) * 16) = kreg[u];
    }
#pragma unroll
    for (int u = 0; u < V_PT; ++u) {
      const int c = tid + u * NT;
      // (pieces 1 and 2 of every four change places: the eight keys of a lane's fragment are then 16 bytes side by side)
      const int ch = c & 15, at = (ch & 12) | ((ch & 1) << 1) | ((ch >> 1) & 1);
      if (c < DH * 16) *reinterpret_cast<u32x2*>(v_lds + (c >> 4) * VSTR + at * 8) = vreg[u];
    }
  };

  // a wave whose queries lie beyond the item (the last query block of a sequence) only helps to stage the tiles
  const bool live = qw < w.q1;
  const int kv_first = w.kv0 + 64 * group;   // this group's first tile
  load_tile(kv_first);
  for (int kv = kv_first; kv - 64 * group < (SINGLE ? w.kv0 + 1 : w.kv1); kv += 64 * KG) {
    if (!SINGLE) __syncthreads();  // previous tile fully consumed
    store_tile();
    __syncthreads();
    // (a key group's waves stage four times as much each: their next tile is requested behind the softmax, when the
    // scores' registers are free)
    const bool more = !SINGLE && kv + 64 * KG < w.kv1;
    if (KG == 1 && more) load_tile(kv + 64 * KG);
    __builtin_amdgcn_sched_barrier(0);
    if (!SINGLE && (!live || (KG > 1 && kv >= w.kv1))) {   // (or no tile is left for this group)
      if (KG > 1 && more) load_tile(kv + 64 * KG);
      continue;
    }

    // ---- S^T tiles: s[it][jt] covers keys kv + jt*32 .. +31 (rows) x queries it*32 .. +31 (lanes)
    // The accumulators start at minus the query's running maximum (a lane's scores all belong to one
    // query), so the products come out as score - maximum and the common case below needs no subtraction.
    // `first`: there is no maximum yet.  (With key groups per query: the first tiles of a group may hold nothing but
    // scores of -inf, which another group's keys outweigh.)
    bool first[QT];
    f32x16 s[QT][2];
#pragma unroll
    for (int it = 0; it < QT; ++it) {
      first[it] = KG > 1 ? mrun[it] == -INFINITY : kv == kv_first;
      const float init = first[it] ? 0.f : -mrun[it];
#pragma unroll
      for (int jt = 0; jt < 2; ++jt)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[it][jt][r] = init;
    }
    // (these products first: a wave in its exponentials then does not hold up one that is about to have work for them;
    // 4 x 3467 tokens x 16 heads of 80 304 -> 297 us, 2 x 8192 721 -> 713, three tiles in key groups 28.7 -> 27.1)
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int jt = 0; jt < 2; ++jt) {
        const bf16x8 kf = *reinterpret_cast<const bf16x8*>(k_lds + (jt * 32 + l31) * KSTR + ks * 32 + lhi * 16);
#pragma unroll
        for (int it = 0; it < QT; ++it) {
          bf16x8 q = qf[it][ks];
          if constexpr (Q_IN_LDS) q = *reinterpret_cast<const bf16x8*>(q_lds + ((it * KS + ks) * NT + tid) * 16);
          s[it][jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, q, s[it][jt], 0, 0, 0);
        }
      }
    }
    __builtin_amdgcn_s_setprio(0);
    // register r of a tile holds key row 8*(r/4) + 4*lhi + r%4
    if (kv + 64 > w.kv1) {
#pragma unroll
      for (int jt = 0; jt < 2; ++jt)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = kv + jt * 32 + 8 * (r >> 2) + 4 * lhi + (r & 3);
          if (key >= w.kv1) {
#pragma unroll
            for (int it = 0; it < QT; ++it) s[it][jt][r] = -INFINITY;
          }
        }
    }
    // ---- online softmax, per query column.  The running maximum is moved only when a tile's largest score
    // exceeds it by more than MAX_SLACK (in the log2 domain): probabilities are then at most 2^MAX_SLACK
    // instead of 1, which changes nothing in the quotient (softmax is invariant under a common shift, and
    // bf16 and fp32 keep their relative precision over that range), and the accumulators are rescaled
    // only on the first tile and on such a jump instead of on nearly every tile.
    constexpr float MAX_SLACK = 8.0f;
    bf16x8 pf[QT][4];
#pragma unroll
    for (int it = 0; it < QT; ++it) {
      float mx = s[it][0][0];
#pragma unroll
      for (int jt = 0; jt < 2; ++jt)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[it][jt][r]);
      // v_exp_f32 directly: arguments are bounded above and results that would be denormal may flush to 0,
      // so the library exp2f's range scaling (four more instructions per score) buys nothing here
      if (__any(first[it] || mx > MAX_SLACK)) {    // some query of this wave takes a new maximum
        // (the halves of a wave hold the same queries: only where a maximum moves is the other half's needed)
        mx = fmaxf(mx, __shfl_xor(mx, 32));        // the tile's largest score minus the running maximum
        const bool jump = first[it] || mx > MAX_SLACK;   // (every tile holds at least one valid key)
        const float base = first[it] ? 0.f : mrun[it];
        const float mnew = jump ? mx + base : mrun[it];
        const float alpha = first[it] ? 0.f : __builtin_amdgcn_exp2f(mrun[it] - mnew);
        float shift = mnew - base;                 // 0 in the lanes whose query keeps its maximum
        if (KG > 1 && mnew == -INFINITY) shift = 0.f;   // no key with weight yet: the probabilities are exp2(-inf)
        mrun[it] = mnew;
        lrun[it] *= alpha;
#pragma unroll
        for (int jt = 0; jt < 2; ++jt)
#pragma unroll
          for (int r = 0; r < 16; ++r) s[it][jt][r] -= shift;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[it][dt][r] *= alpha;
      }
      float sum = 0.f;
#pragma unroll
      for (int jt = 0; jt < 2; ++jt)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          uint32_t pk[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float p0 = __builtin_amdgcn_exp2f(s[it][jt][8 * u + 2 * e]);
            const float p1 = __builtin_amdgcn_exp2f(s[it][jt][8 * u + 2 * e + 1]);
            sum += p0 + p1;
            pk[e] = pack2_a(p0, p1);
          }
          uint4 t = make_uint4(pk[0], pk[1], pk[2], pk[3]);
          pf[it][jt * 2 + u] = *reinterpret_cast<bf16x8*>(&t);
        }
      lrun[it] += sum;
    }
    if constexpr (KG > 1) {
      if (more) load_tile(kv + 64 * KG);
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- O^T += V^T P^T.  k-slot e of lane-half lhi in step (jt,u) is key jt*32 + 16u + 8*(e/4) + 4*lhi + e%4
#pragma unroll
    for (int ku = 0; ku < 4; ++ku) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const bf16x8 vf = *reinterpret_cast<const bf16x8*>(v_lds + (dt * 32 + l31) * VSTR + ku * 32 + lhi * 16);
#pragma unroll
        for (int it = 0; it < QT; ++it)
          o[it][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[it][ku], o[it][dt], 0, 0, 0);
      }
    }
  }

  if constexpr (KG > 1) {
    // ---- merge: every group but the first leaves its state in LDS (lane order, 4-byte words: no conflicts), the first
    // adds the groups in order, each scaled to the common maximum
    constexpr int STATE = 16 * DT + 2;     // words per lane
    static_assert((KG - 1) * NWG * STATE * 256 <= KG * (K_BYTES + V_BYTES), "the states fit where the tiles were");
    __syncthreads();
    float* st = reinterpret_cast<float*>(tiles) + wave * STATE * 64 + lane;
    if (group > 0) {
      float* mine = st + (group - 1) * NWG * STATE * 64;
      mine[0] = mrun[0];
      mine[64] = lrun[0];
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) mine[(2 + 16 * dt + r) * 64] = o[0][dt][r];
    }
    __syncthreads();
    if (group > 0) return;
    float m = mrun[0];
#pragma unroll
    for (int k = 1; k < KG; ++k) m = fmaxf(m, st[(k - 1) * NWG * STATE * 64]);
    const float a0 = __builtin_amdgcn_exp2f(mrun[0] - m);
    lrun[0] *= a0;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[0][dt][r] *= a0;
#pragma unroll
    for (int k = 1; k < KG; ++k) {
      const float* other = st + (k - 1) * NWG * STATE * 64;
      const float ak = __builtin_amdgcn_exp2f(other[0] - m);   // 0 for a group without a tile, or without a key of weight (its maximum is -inf)
      lrun[0] += ak * other[64];
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[0][dt][r] += ak * other[(2 + 16 * dt + r) * 64];
    }
  }

  // ---- normalise and store: register r of o[it][dt] is dim dt*32 + 8*(r/4) + 4*lhi + r%4 of query it*32 + lane%32
#pragma unroll
  for (int it = 0; it < QT; ++it) {
    const float l = lrun[it] + __shfl_xor(lrun[it], 32);
    const float inv = 1.0f / l;
    const int q = qw + it * 32 + l31;
    if (q >= w.q1) continue;
    bf16_t* orow = a.out + (int64_t)q * hidden + head * DH;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int d = dt * 32 + 8 * g + 4 * lhi;
        if (d < DH) {
          uint2 pk;
          pk.x = pack2_a(o[it][dt][4 * g + 0] * inv, o[it][dt][4 * g + 1] * inv);
          pk.y = pack2_a(o[it][dt][4 * g + 2] * inv, o[it][dt][4 * g + 3] * inv);
          *reinterpret_cast<uint2*>(orow + d) = pk;
        }
      }
  }
}

cs_status launch_attention(const AttnArgs& a, hipStream_t stream) {
  if (a.n_work <= 0) return CS_OK;
  if (a.n_tok < 4 || a.ld_vt < ((a.n_tok + 3) & ~3)) return fail(CS_ERR_INVALID_ARG, "attention: ld_vt too small");
  if (a.ld_vt & 3) return fail(CS_ERR_INVALID_ARG, "attention: ld_vt must be a multiple of 4");
  AttnArgs args = a;
  args.q_split = a.q_split > 1 ? a.q_split : 1;
  if (args.q_split > 1 && (args.q_split != 4 || a.q_per_block != 256 || a.key_groups > 1 || a.single_tile))
    return fail(CS_ERR_INVALID_ARG, "attention: only 256-query items run as four workgroups");
  const int64_t pairs = (int64_t)a.n_work * args.q_split * a.n_heads;
  if (pairs + 8 * (int64_t)a.n_heads > 0x7fffffff) return fail(CS_ERR_UNSUPPORTED, "attention: too many work items");
  // (see the kernel: window layers give an XCD every eighth window, full layers an eighth of the (head, item) pairs)
  dim3 grid(a.single_tile ? (unsigned)(8 * ((a.n_work + 7) / 8) * a.n_heads) : (unsigned)(8 * ((pairs + 7) / 8)));
  // every wave owns 32 queries: two waves per 64-query work item (window layers), eight per 256-query item,
  // two waves per SIMD so that one wave's softmax arithmetic runs under the other's MFMAs
  if (a.single_tile && a.q_per_block != 64) return fail(CS_ERR_INVALID_ARG, "attention: single-tile items are 64-query items");
  if (a.q_per_block == 128 ? a.key_groups != 2 : a.key_groups > 1 && (a.key_groups != 4 || a.q_per_block != 64))
    return fail(CS_ERR_INVALID_ARG, "attention: key groups are two of 128-query items or four of 64-query items");
  if (a.key_groups > 1 && (a.head_dim != 64 || a.single_tile || a.max_keys <= 0 || !attention_groups_addressable(a)))
    return fail(CS_ERR_UNSUPPORTED, "attention: key groups need head_dim 64 and items whose keys 32-bit offsets reach");
  const int q = args.q_split > 1 ? 64 : a.q_per_block;   // queries per workgroup
  if (a.head_dim == 80 && a.q_per_block == 64 && a.single_tile) hipLaunchKernelGGL((attn_kernel<80, 2, 1, true>), grid, dim3(128), 0, stream, args);
  else if (a.head_dim == 80 && q == 64) hipLaunchKernelGGL((attn_kernel<80, 2, 1, false>), grid, dim3(128), 0, stream, args);
  else if (a.head_dim == 80 && q == 256) hipLaunchKernelGGL((attn_kernel<80, 8, 1, false>), grid, dim3(512), 0, stream, args);
  else if (a.head_dim == 64 && a.q_per_block == 64 && a.single_tile) hipLaunchKernelGGL((attn_kernel<64, 2, 1, true>), grid, dim3(128), 0, stream, args);
  else if (a.head_dim == 64 && a.q_per_block == 64 && a.key_groups > 1) hipLaunchKernelGGL((attn_kernel<64, 8, 1, false, 4>), grid, dim3(512), 0, stream, args);
  else if (a.head_dim == 64 && a.q_per_block == 128) hipLaunchKernelGGL((attn_kernel<64, 8, 1, false, 2>), grid, dim3(512), 0, stream, args);
  else if (a.head_dim == 64 && q == 64) hipLaunchKernelGGL((attn_kernel<64, 2, 1, false>), grid, dim3(128), 0, stream, args);
  else if (a.head_dim == 64 && q == 256) hipLaunchKernelGGL((attn_kernel<64, 8, 1, false>), grid, dim3(512), 0, stream, args);
  else return fail(CS_ERR_UNSUPPORTED, "attention: head_dim must be 64 or 80 and q_per_block 64, 128 or 256");
  CS_HIP(hipGetLastError());
  return CS_OK;
}

}  // namespace cs

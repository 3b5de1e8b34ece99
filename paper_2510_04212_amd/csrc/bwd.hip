// Flash-attention backward for gfx950 (Alg. 2 of arXiv 2510.04212), as two kernels so that no
// gradient needs a cross-work-group reduction (no atomics, deterministic):
//
//   attn_bwd_dkdv_kernel  one work-group per (batch, head, 128-key block; 64 on small grids) -- under the causal mask
//                         per pair of mirrored blocks, one after the other, unless the grid is
//                         small (then one block each, in a balanced order); K_j / V_j fragments
//                         stay in registers (V_j in LDS at D = 128), query tiles (Q_i, dO_i, L_i,
//                         delta_i; 64 rows, 32 at D = 128) stream through LDS.  Per tile:  S = Q_i K_j^T,  P = exp(S - L),  dP = dO_i V_j^T,
//                         dS = P o (dP - delta),  dV_j^T += dO_i^T P,  dK_j^T += Q_i^T dS.
//   attn_bwd_dq_kernel    one work-group per (batch, head, 128-query block; 64 on small grids); Q_i / dO_i fragments,
//                         L_i and delta_i stay in registers, key tiles (K_j, V_j; 64 rows) stream
//                         through LDS.  Per tile:  S^T = K_j Q_i^T,  dP^T = V_j dO_i^T,
//                         dS^T = P^T o (dP^T - delta),  dQ_i^T += K_j^T dS^T.
//
// S and dP are recomputed in the second kernel (7 matrix products per tile pair instead of
// Alg. 2's 5); in exchange every contraction finds its operands already in fragment layout:
// the accumulator-layout P / dS tiles are fed back as B operands unchanged, and the operands
// whose contraction index runs along tile rows come from transposing LDS reads.
//
// Rounding points: P (float32) -> bf16 as the operand of dO^T P; dS = P o (dP - delta) is formed
// from the float32 P and rounded to bf16 as an operand; accumulators are float32; alpha
// multiplies the float32 dQ / dK accumulators once; outputs are rounded to bf16 when stored.
#include "common.hpp"

#include <atomic>
#include <type_traits>

namespace {

constexpr int kKeysPerWG = 128;   // dK/dV kernel: keys per work-group (32 per wave); 64 with four wave groups
constexpr int kQPerWG = 128;      // dQ kernel: queries per work-group (32 per wave); 64 with wave groups

template <int NDB>
DEVI void store_acc_T(bf16_t* dst_row, const f32x16 (&acc)[NDB], float scale, int h) {
  // acc[db][i] = X^T[d = 32db + 8(i/4) + 4h + (i%4)][row of this lane]; 4 consecutive d -> 8 bytes
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      bf16x4 o4;
#pragma unroll
      for (int e = 0; e < 4; ++e) o4[e] = (bf16_t)(acc[db][4 * g + e] * scale);
      *reinterpret_cast<bf16x4*>(dst_row + 32 * db + 8 * g + 4 * h) = o4;
    }
}

// GROUPED: grouped-query attention (lay.group > 1): the work-group serves several query heads.
// Kept out of the ordinary kernel so that its tile loop has a fixed head and no bookkeeping.
// At D = 256 the two accumulator sets of a full key block would not fit the register file next
// to the K / V fragments: a work-group then owns 128 of the 256 columns of dK and dV (kDSplit
// work-groups per key block, each recomputing S and dP).
template <int D> constexpr int kDSplit = D > 128 ? 2 : 1;
// The kernel wants two waves on every SIMD: one wave alone leaves the matrix cores idle whenever
// any of its instructions waits.  That means at most 256 registers per lane (some instantiations
// at D = 128 under the mask spill two to nine, outside their tile loops).  At D = 128 the
// accumulators (128) and the K fragments (32) leave no room for the V fragments: V_j is kept in LDS
// for the whole block (8 more fragment reads per 32 queries to 48) and the query tiles shrink to 32
// rows per wave group, so that two work-groups fit a CU.  Measured against one wave per SIMD with
// 430 registers and a hand-made four-phase pipeline (us, bit-identical): B4 H32 N4096 d128 causal
// 1043 -> 990, B4 H16 N2048 d128 full 281 -> 234, B4 H16 N1999 d128 causal 157 -> 132 and full
// 602 -> 235 (that one spilled), B4 H16 N4096 d96 causal 484 -> 369.  At D = 256 (one wave per SIMD all
// the same) the single code path for masked and unmasked blocks alone took 140 -> 109.
template <int D> constexpr bool kVInLds = D == 128;
template <int D> constexpr int kWavesPerSimd = D <= 128 ? 2 : 1;
// G: wave groups.  G = 2 (512 threads) is for grids that give a CU only one work-group:
// the groups share the work-group's keys and take alternate 32-query blocks, each into accumulators
// of its own, which are added through LDS at the end.  G = 4 splits further: 64 keys (two waves) per
// group, so that a grid has twice the work-groups of half the length; a query tile is then read
// from L2 for half as many keys.
template <int G> constexpr int kKeyWaves = G == 4 ? 2 : 4;               // waves per group, 32 keys each
template <int D, int G> constexpr int kQTile = D == 128 || G == 4 ? 32 * G : 64;   // query rows per streamed tile
// LDS fragments are read this many matrix instructions before their use.
// (At D = 128 what the registers allow: the fragments of V_j come from LDS too.  Four wave groups at small D: us, four ahead ->
// two, B1 H4 N4096 d64 causal 41.1 -> 40.1, B1 H1 38.5 -> 37.7, B1 H2 N8192 d32 causal 54.0 -> 53.4, full 51.2 -> 50.5, B1 H8
// N2000 d32 16.7 -> 16.4; d64 full even to 2 % slower: not there.)
template <int D, int G, bool CAUSAL, bool DENSE> constexpr int kReadAhead =
    DENSE || (G == 4 && (D == 32 || (D == 64 && CAUSAL))) ? 2 : D == 256 ? 6 : D == 128 ? 2 : 4;
// dK / dV rows leave through a per-wave LDS staging area (store_rows_staged) where the row width
// allows it; it overlays the tile buffers where it would otherwise cost a resident work-group, and
// is left out at D = 256 (no room).
template <int D> constexpr bool kStagedDkDv = kCanStage<D / 32 / kDSplit<D>> && D <= 128;
template <int D, int G> constexpr bool kStageOverTiles = D == 128 || G > 1;
// LDS: V_j (kVInLds), Q buffers [2], dO buffers [2], L [2][kQTile], delta [2][kQTile], staging.  With two
// wave groups the start of the array serves the exchange of partial sums (and the staging) at the end.
template <int D, int G> constexpr int kVBytes = kVInLds<D> ? 32 * kKeyWaves<G> * D * 2 : 0;
template <int D, int G> constexpr int kTilesEnd = kVBytes<D, G> + 4 * kQTile<D, G> * D * 2 + 4 * kQTile<D, G> * 4;
template <int D> constexpr int kStageBytes = kStagedDkDv<D> ? 4 * 32 * kStagePitch<D / 32 / kDSplit<D>> : 0;
template <int D, int G> constexpr int kExchangeBytes = G > 1 ? 2 * 4 * (D / 32) * 4096 : 0;
constexpr int max_int(int a, int b) { return a > b ? a : b; }
template <int D, int G> constexpr int kSmemDkDv =
    G > 1 ? max_int(kTilesEnd<D, G>, kExchangeBytes<D, G>)
          : kStageOverTiles<D, G> ? max_int(kTilesEnd<D, G>, kVBytes<D, G> + kStageBytes<D>) : kTilesEnd<D, G> + kStageBytes<D>;

// DENSE (D <= 64): three waves on every SIMD at the price of a shorter read-ahead, for grids that have the work-groups
// (launch_dkdv).
template <int D, bool DENSE> constexpr int kDkDvWaves = DENSE ? 3 : kWavesPerSimd<D>;
template <int D, bool CAUSAL, bool RAGGED, bool GROUPED, int G, bool DENSE>
__global__ __launch_bounds__(64 * kKeyWaves<G> * G)
__attribute__((amdgpu_waves_per_eu(kDkDvWaves<D, DENSE>, kDkDvWaves<D, DENSE>))) void attn_bwd_dkdv_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    const bf16_t* __restrict__ dO, const float* __restrict__ LSE, const float* __restrict__ delta,
    bf16_t* __restrict__ dK, bf16_t* __restrict__ dV, int N, float alpha, Layout lay, int pairs,
    BlockOrder ord) {
  constexpr int QT = kQTile<D, G>;
  constexpr int TILE_BYTES = QT * D * 2, GT = TILE_BYTES / G;
  constexpr int T0 = kVBytes<D, G>;                    // the tile buffers follow V_j: per wave group Q [2][GT], dO [2][GT]
  constexpr int KW = kKeyWaves<G>, KEYS = 32 * KW;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  char* ldsQ = smem + T0;
  char* ldsdO = ldsQ + 2 * GT;
  float* ldsL = reinterpret_cast<float*>(smem + T0 + 4 * TILE_BYTES);
  float* ldsD = ldsL + 2 * QT;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = (tid >> 6) % KW;                    // which 32 keys
  const int grp = G > 1 ? __builtin_amdgcn_readfirstlane(tid / (64 * KW)) : 0;   // which 32-query blocks
  const int r = lane & 31, h = lane >> 5;

  // RAGGED: the bounds-checking instantiation: N queries and NK keys, neither need be a multiple
  // of the block; causal mask  key <= query + shift.
  const int NK = RAGGED ? lay.Nk : N;
  const int shift = RAGGED ? NK - N : 0;
  const int nkt = (NK + KEYS - 1) / KEYS;
  // Under the causal mask key block kt meets nkt - kt query blocks' worth of tiles.  pairs != 0: a
  // work-group takes block kt and then its mirror image nkt - 1 - kt, so that all work-groups
  // carry the same load (and there are half as many to start and drain).  pairs == 0 (grids so
  // small that equal but few work-groups would leave compute units idle): one block per
  // work-group, in the order the table `ord` gives.
  const int npw = pairs ? (nkt + 1) / 2 : nkt;         // work-groups per key/value head and column part
  constexpr int DS = kDSplit<D>;
  constexpr int NDB = D / 32 / DS;                     // 32-column blocks of dK / dV this work-group owns
  const int wg_all = logical_wg(ord, blockIdx.x, gridDim.x);
  const int db0 = (DS > 1) ? (wg_all % DS) * NDB : 0;  // first of them
  const int wg = wg_all / DS;
  // with grouped queries a work-group serves the `group` query heads that share its key/value
  // head, one after the other
  const int bhk = wg / npw;
  const int group = GROUPED ? lay.group : 1;
  const int Hkv = lay.H / group;
  const int bq0 = (bhk / Hkv) * lay.H + (bhk % Hkv) * group;   // first of those query heads
  const int kt_first = wg % npw;
  const int sn = lay.sn;
  const size_t head_off = head_base_kv(lay, bq0);              // K, V, dK, dV
  const float c2 = alpha * kLog2e;
  FragOffsets<D> fo;
  init_frag_offsets<D>(fo, lane, lds_address(smem));
  FragOffsets<D> fo_v = fo;                            // V_j fragments of this wave's keys
  FragOffsets<D> fo_upd = fo;                          // update products: columns from block db0 on
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    if (kVInLds<D>) fo_v.row[p] += 2 * wave * kRowBlockBytes<D>;
    if (DS > 1) fo_upd.col[p] += 1024 * db0;
    if (G > 1) {
      fo.row[p] += 4 * grp * GT;
      fo_upd.col[p] += 4 * grp * GT;
    }
  }
  // Group g reads the g-th 32 rows of a tile, which are the rows that its own waves fetch.  Its four buffers lie next
  // to one another (tiles as a whole would not), within the 64 KB that the immediate offset of an LDS read reaches:
  // one base register for all of them, which is what leaves the registers for the stream of qblocks below at D = 128 (with
  // whole tiles it spills 33 to 55, now 6 to 9, outside the loop).  us, whole tiles and phase after phase -> now, same
  // bits: B2 H16 N2048 d128 causal 95.5 -> 88.1, B2 H8 N2048 d128 full 71.6 -> 67.2, B1 H4 N4096 d128 causal 69.2 -> 66.0,
  // B2 H32/8 N2048 d128 causal 176 -> 172; at D <= 96, where only the layout changes, within 2 % either way.
  TileLoader<D, QT, KW * G> loader;
  loader.init(tid, sn);
  if (G > 1) {
    static_assert(G == 1 || GT == 2 * kRowBlockBytes<D>, "32 rows per group");
    loader.lds_wave += 3 * grp * GT;
  }

  // Three waves per SIMD at D = 64 under the mask: what depends on the lane is formed where it is used, from copies of the
  // thread index that the compiler cannot see through.  Formed ahead of the loops it was spilled (eight or nine registers), and
  // short problems waited for the reloads: us, 400 heads N200 23.2 -> 18.9, 472 heads N300 41.5 -> 34.3, B8 H12 N1000
  // 39.0 -> 34.5, N1024 37.1 -> 36.2, B4 H32 N4000 526 -> 512.  (Elsewhere nothing is spilled, and it costs 2 %.)
  constexpr bool FORM_LATE = DENSE && D == 64 && CAUSAL;
  auto late = [](int x) {
    if (FORM_LATE) asm volatile("" : "+v"(x));
    return x;
  };

  for (int part = 0; part < (CAUSAL ? 2 : 1); ++part) {
    const int kt = (part == 0) ? kt_first : nkt - 1 - kt_first;
    if (part == 1 && (!pairs || kt == kt_first)) break;   // no partner: one block per work-group, or the middle one of an odd number
    if (kStageOverTiles<D, G> && part > 0) __syncthreads();   // the first block's staging is done with the tile buffers
    const int k0 = kt * KEYS;
    const int kw = k0 + 32 * (FORM_LATE ? late(tid) >> 6 : wave);

    if constexpr (kVInLds<D>) {
      TileLoader<D, KEYS, KW * G> v_loader;
      v_loader.init(tid, sn);
      v_loader.template load_rows<RAGGED>(smem, V + head_off, k0, NK);
    }
    // K_j^T / V_j^T fragments (B operands): lane (r,h) holds K[kw + r][16kc + 8h .. +7]
    // (keys past the sequence end read the last row; their gradients are not stored)
    const int keyc = (RAGGED && kw + r >= NK) ? NK - 1 : kw + r, hk = late(h);
    bf16x8 kf[D / 16], vf[kVInLds<D> ? 1 : D / 16];
#pragma unroll
    for (int kc = 0; kc < D / 16; ++kc) {
      kf[kc] = *reinterpret_cast<const bf16x8*>(K + head_off + (size_t)keyc * sn + 16 * kc + 8 * hk);
      if constexpr (!kVInLds<D>) vf[kc] = *reinterpret_cast<const bf16x8*>(V + head_off + (size_t)keyc * sn + 16 * kc + 8 * hk);
    }
    f32x16 dVt[NDB], dKt[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) { dVt[db][i] = 0.f; dKt[db][i] = 0.f; }

    // first query tile that sees any key of this block (the last query sees every key: t0 < nt)
    const int t0 = !CAUSAL ? 0 : !RAGGED ? k0 / QT : max(0, k0 - shift) / QT;
    const int nt = RAGGED ? (N + QT - 1) / QT : N / QT;
    // Q_i / dO_i tiles go global -> LDS asynchronously; L_i (pre-multiplied by log2 e) and -delta_i
    // (QT floats each) pass through one register of the first 2 QT threads.  The dP accumulator starts
    // from -delta, so that the matrix instructions deliver dP - delta directly (Alg. 2 step 12).
    float sreg = 0.f;
    // Current query head: its first element in Q / dO and in LSE / delta.  With GROUPED the
    // work-group moves on to the next head of its group (at distance lay.sh and N) after tile
    // nt - 1, without breaking the double buffering: `step` counts tiles over all heads.
    const bf16_t* Qh = Q + head_base(lay, bq0);
    const bf16_t* dOh = dO + head_base(lay, bq0);
    const float* Lh = LSE + (size_t)bq0 * N;
    const float* Dh = delta + (size_t)bq0 * N;
    const int total = group * (nt - t0);
    auto load_stats = [&](const float* Lp, const float* Dp, int t) {
      const int tl = late(tid);
      const int row = t * QT + (tl & (QT - 1));
      const int rowc = (RAGGED && row >= N) ? N - 1 : row;
      if (tl < QT) {
        sreg = Lp[rowc];
      } else if (tl < 2 * QT) sreg = Dp[rowc];
      // (The loaded values are not touched before store_stats: any arithmetic on them here would
      // make the wave wait, at the start of the tile, for these loads and for the tile transfer
      // issued just before them.)
    };
    auto store_stats = [&](int buf, int tn) {      // tn: the tile they belong to
      const int tl = late(tid);
      if (tl < QT) {
        float l = sreg * kLog2e;
        if (RAGGED && l == -INFINITY) l = 0.f;         // a query that sees no key: all its scores are masked below
        if (RAGGED && tn * QT + tl >= N) l = INFINITY;    // a row past the sequence end: P = exp(-inf) = 0, so it adds nothing to dK, dV
        ldsL[buf * QT + tl] = l;
      } else if (tl < 2 * QT) ldsD[buf * QT + tl - QT] = -sreg;   // LDS holds -delta
    };
    loader.template load_rows<RAGGED>(ldsQ, Qh, t0 * QT, N);
    loader.template load_rows<RAGGED>(ldsdO, dOh, t0 * QT, N);
    load_stats(Lh, Dh, t0);
    store_stats(0, t0);
    wait_vmem();
#pragma unroll
    for (int kc = 0; kc < D / 16; ++kc) {
      settle(kf[kc]);
      if constexpr (!kVInLds<D>) settle(vf[kc]);
    }
    __syncthreads();

    // One query tile; BUF (which LDS buffer holds it) is a compile-time constant so that every LDS
    // address is a precomputed per-lane offset plus an immediate.
    auto tile_step = [&](auto buf_c, int t, int step) {
      constexpr int buf = decltype(buf_c)::value;
      const bool has_next = (step + 1 < total);
      // The next tile (after the last one: this tile once more, harmlessly) goes into the other
      // buffer.  Its transfer instructions are issued between the matrix instructions of the first
      // score products instead of in one burst behind the barrier.
      int tn = has_next ? t + 1 : t;
      if (GROUPED && has_next && t + 1 == nt) {   // on to the next query head of the group
        Qh += lay.sh; dOh += lay.sh; Lh += N; Dh += N;
        tn = t0;
      }
      constexpr int NLD = decltype(loader)::NI;
      const auto pendQ = loader.template prepare<RAGGED>(ldsQ + (buf ^ 1) * GT, Qh, tn * QT, N);
      const auto pendD = loader.template prepare<RAGGED>(ldsdO + (buf ^ 1) * GT, dOh, tn * QT, N);
      auto issue_part = [&](int i) {
        if (i < NLD) loader.issue(pendQ, i);
        else if (i < 2 * NLD) loader.issue(pendD, i - NLD);
      };
      bool issued = false;
      if (has_next) load_stats(Lh, Dh, tn);
      constexpr int tQ = T0 + buf * GT;             // byte offsets of this tile's Q and dO in smem
      constexpr int tdO = T0 + (2 + buf) * GT;
      const float* tL = ldsL + buf * QT;
      const float* tD = ldsD + buf * QT;
      const int qt0 = t * QT;
      // The NB 32-query blocks of a tile that belong to this wave's group against its 32 keys, as one stream of matrix
      // instructions ("slots"):  S (D/16 slots) | dP | dV (2 NDB) | dK, block after block.  The vector work of a
      // block lies under its own matrix instructions: P = exp(S - L) under dP, dS = P o (dP - delta) under dV,
      // and every LDS fragment is read AHEAD slots before its use (a fence per slot keeps that order).  Same bits as
      // phase after phase; us, whole kernel: B2 H8 N2048 d256 causal 120 -> 116, B1 H8 N1000 d256 causal 74 -> 59,
      // B2 H16 N2048 d96 causal 68 -> 66, B4 H32 N4096 d64 causal 519 -> 510, B32 H12 N512 d64 full 67.5 -> 66.0;
      // d128, the whole training step: B4 H32 N4096 causal 2374 -> 2309, B1 H16 N16384 causal 4561 -> 4470,
      // B4 H16 N1999 causal 334 -> 329.
      // The next tile's transfer is issued on the way.
      // MASKED: a block crosses the diagonal.
      auto qblocks = [&](auto masked_c, auto nb_c, auto qb_c) {
        constexpr bool MASKED = decltype(masked_c)::value;
        constexpr int NB = decltype(nb_c)::value, qb = decltype(qb_c)::value;
        constexpr int NS = D / 16, NU = 2 * NDB, PB = 2 * NS + 2 * NU;    // slots of S or dP, of dV or dK, of a block
        constexpr int AHEAD = kReadAhead<D, G, CAUSAL, DENSE>, RING = AHEAD + 1;
        constexpr int AHEAD_V = 1, RING_V = AHEAD_V + 1;       // kVInLds: V_j's fragments
        auto fragment = [&](int i) -> bf16x8 {
          const int b = qb + i / PB, u = i % PB;
          if (u < NS) return lds_row8<D>(tQ, fo, 32 * b, u);
          if (u < 2 * NS) return lds_row8<D>(tdO, fo, 32 * b, u - NS);
          const int w = (u - 2 * NS) % NU;
          return lds_col8<D>(u < 2 * NS + NU ? tdO : tQ, fo_upd, 32 * b + 16 * (w / NDB), w % NDB);
        };
        bf16x8 ring[RING], ring_v[kVInLds<D> ? RING_V : 1];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) ring[i] = fragment(i);
        f32x16 s, dp;
        f32x4 l4[4];
        bf16x8 pf[2], dsf[2];
        int first_seen = 0;              // MASKED: entry c = 8 (i / 4) + i % 4 counts if c >= first_seen
        static_for<NB * PB>([&](auto slot) {
          constexpr int sl = decltype(slot)::value, u = sl % PB, b = qb + sl / PB;
          const int stat = 32 * (b + grp) + 4 * h;
          if (sl + AHEAD < NB * PB) ring[(sl + AHEAD) % RING] = fragment(sl + AHEAD);
          constexpr int uv = u + AHEAD_V - NS;
          if constexpr (kVInLds<D> && uv >= 0 && uv < NS) ring_v[uv % RING_V] = lds_row8<D>(0, fo_v, 0, uv);
          if (u == 0) {
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = 0.f;
            if (MASKED) {
              int ln = lane;
              constexpr bool LATE = DENSE || kVInLds<D>;         // formed here, not ahead of the tile loop: registers
              if (LATE) asm volatile("" : "+v"(ln));
              first_seen = (LATE ? __builtin_amdgcn_readfirstlane(kw) : kw) + (ln & 31) - shift - qt0 - 32 * (b + grp) - 4 * (ln >> 5);
            }
          }
          // -delta_i seeds the dP accumulator; L_i of the rows a lane sees
#pragma unroll
          for (int g = 0; g < 4; ++g)
            if (u == g * (NS < 4 ? NS : 4) / 4) {
              const f32x4 d4 = *reinterpret_cast<const f32x4*>(tD + stat + 8 * g);
#pragma unroll
              for (int e = 0; e < 4; ++e) dp[4 * g + e] = d4[e];
            }
#pragma unroll
          for (int g = 0; g < 4; ++g)
            if (u == NS + g * NS / 4) l4[g] = *reinterpret_cast<const f32x4*>(tL + stat + 8 * g);
          const bf16x8 a = ring[sl % RING];
          if constexpr (u < NS) {
            s = mfma32(a, kf[u], s);
          } else if constexpr (u < 2 * NS) {
            if constexpr (kVInLds<D>) dp = mfma32(a, ring_v[(u - NS) % RING_V], dp);
            else dp = mfma32(a, vf[u - NS], dp);
          } else if constexpr (u < 2 * NS + NU) {
            constexpr int w = u - 2 * NS;
            dVt[w % NDB] = mfma32(a, pf[w / NDB], dVt[w % NDB]);
          } else {
            constexpr int w = u - 2 * NS - NU;
            dKt[w % NDB] = mfma32(a, dsf[w / NDB], dKt[w % NDB]);
          }
          if (b == 0) issue_part(sl);
          if (u > NS && u <= 2 * NS) {           // P = exp(S - L) (step 9)
#pragma unroll
            for (int i = 16 * (u - NS - 1) / NS; i < 16 * (u - NS) / NS; ++i) {
              float x = __builtin_fmaf(s[i], c2, -l4[i >> 2][i & 3]);
              const int c = 8 * (i >> 2) + (i & 3);
              if (MASKED && c < first_seen) x = -INFINITY;
              s[i] = __builtin_amdgcn_exp2f(x);
              pf[i >> 3][i & 7] = (bf16_t)s[i];
            }
          }
          if (u > 2 * NS && u <= 2 * NS + NU) {  // dS = P o (dP - delta) (step 12); dp already holds dP - delta
#pragma unroll
            for (int i = 16 * (u - 2 * NS - 1) / NU; i < 16 * (u - 2 * NS) / NU; ++i) {
              float ds = s[i] * dp[i];
              // a masked entry contributes exactly nothing, whatever its row holds
              const int c = 8 * (i >> 2) + (i & 3);
              if (MASKED && c < first_seen) ds = 0.f;
              dsf[i >> 3][i & 7] = (bf16_t)ds;
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        });
      };
      constexpr int NBT = QT / 32 / G;                       // blocks of this wave's group in a tile
      const int q_first = qt0 + 32 * grp, q_last = q_first + 32 * NBT - 1;     // first and last query of them
      // Blocks past the sequence end are left out as if they saw no key.  (Not with three waves per SIMD at D = 64, which then
      // spills 96 registers, and not without a mask, where it would take a second instance of qblocks.  us, computed -> left out: 801
      // heads N65 d64 15.3 -> 14.6, 401 heads N200 d64 20.7 -> 19.6, d32 14.8 -> 14.3, B8 H12 N450 d96 21.3 -> 20.6, B2 H8 N200 d256 30.3 -> 28.8.)
      constexpr bool SKIP_PADDING = RAGGED && CAUSAL && NBT > 1 && !(DENSE && D == 64);
      if ((CAUSAL && q_last + shift < kw) || (RAGGED && q_first >= N)) {
        // no query sees a key of the wave, or nothing but padding
      } else if (!CAUSAL || q_first + shift >= (SKIP_PADDING && q_last - 31 >= N ? 0x7fffffff : kw + 31)) {
        asm volatile("; every entry counts");                // (differs from the other path: nothing is merged in front of the branch)
        qblocks(std::false_type{}, std::integral_constant<int, NBT>{}, std::integral_constant<int, 0>{});
        issued = true;
      } else {
        asm volatile("; masked");
        static_for<NBT>([&](auto qb) {
          const int first = q_first + 32 * decltype(qb)::value;
          if (first + 31 + shift < (SKIP_PADDING && first >= N ? 0x7fffffff : kw)) return;     // no query of the block sees a key of the wave
          qblocks(std::true_type{}, std::integral_constant<int, 1>{}, qb);
          if (decltype(qb)::value == 0) issued = true;
        });
      }
      if (!issued) {      // a wave that skipped the tile's first block still has its share of the transfer to issue
#pragma unroll
        for (int i = 0; i < 2 * NLD; ++i) issue_part(i);
      }
      if (has_next) store_stats(buf ^ 1, tn);
      wait_vmem();
      __syncthreads();
    };
    if (!GROUPED) {
      for (int t = t0; t < nt; t += 2) {
        tile_step(std::integral_constant<int, 0>{}, t, t - t0);
        if (t + 1 < nt) tile_step(std::integral_constant<int, 1>{}, t + 1, t + 1 - t0);
      }
    } else {
      int t = t0;
      for (int step = 0; step < total; step += 2) {
        tile_step(std::integral_constant<int, 0>{}, t, step);
        t = (t + 1 == nt) ? t0 : t + 1;
        if (step + 1 < total) {
          tile_step(std::integral_constant<int, 1>{}, t, step + 1);
          t = (t + 1 == nt) ? t0 : t + 1;
        }
      }
    }
    const int rows_valid = RAGGED ? NK - kw : 32;
    auto rounded = [&](const f32x16 (&acc)[NDB], float scale) {
      return [&acc, scale](int db, int g) {
        bf16x4 o4;
#pragma unroll
        for (int e = 0; e < 4; ++e) o4[e] = (bf16_t)(acc[db][4 * g + e] * scale);
        return o4;
      };
    };
    if constexpr (G > 1) {
      // The groups add their partial sums: group 1 hands over its dV, group 0 its dK, each through an
      // area of its own per wave (16 bytes per lane, lanes consecutive), and group 0 finishes dV,
      // group 1 dK; before that groups 2 and 3 hand both over to groups 0 and 1.  Every wave is past
      // the last tile's barrier: the whole array is free.
      // (the lane index passes through an empty asm: addresses formed from the kernel's own copy would
      // be hoisted above the tile loop and held in registers through it)
      constexpr int AREA = NDB * 4096;
      int ln = lane;
      asm volatile("" : "+v"(ln));
      auto put = [&](const f32x16 (&acc)[NDB], char* give) {
#pragma unroll
        for (int i = 0; i < 4 * NDB; ++i) {
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = acc[i >> 2][4 * (i & 3) + e];
          *reinterpret_cast<f32x4*>(give + (i * 64 + ln) * 16) = v;
        }
      };
      auto add = [&](f32x16 (&acc)[NDB], const char* take) {
#pragma unroll
        for (int i = 0; i < 4 * NDB; ++i) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(take + (i * 64 + ln) * 16);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[i >> 2][4 * (i & 3) + e] += v[e];
        }
      };
      if constexpr (G == 4) {
        char* area = smem + ((grp & 1) * KW + wave) * 2 * AREA;
        if (grp >= 2) { put(dVt, area); put(dKt, area + AREA); }
        __syncthreads();
        if (grp < 2) { add(dVt, area); add(dKt, area + AREA); }
        __syncthreads();
      }
      char* give = smem + (grp * KW + wave) * AREA;
      char* take = smem + ((grp ^ 1) * KW + wave) * AREA;
      // one output per group; the wave's `take` area, read out by then, serves as its staging area
      auto finish = [&](f32x16 (&acc)[NDB], float scale, bf16_t* out) {
        add(acc, take);
        if constexpr (kStagedDkDv<D>)
          store_rows_staged<NDB>(take, rounded(acc, scale), out + head_off + (size_t)kw * sn, sn, rows_valid, ln);
        else if (!RAGGED || kw + r < NK)
          store_acc_T<NDB>(out + head_off + (size_t)(kw + r) * sn, acc, scale, h);
      };
      if (grp == 0) put(dKt, give); else if (grp == 1) put(dVt, give);
      __syncthreads();
      if (grp == 0) finish(dVt, 1.0f, dV); else if (grp == 1) finish(dKt, alpha, dK);
    } else if constexpr (kStagedDkDv<D>) {
      char* stage = smem + T0 + (kStageOverTiles<D, G> ? 0 : 4 * TILE_BYTES + 4 * QT * (int)sizeof(float));
      store_rows_staged<NDB>(stage, rounded(dVt, 1.0f), dV + 32 * db0 + head_off + (size_t)kw * sn, sn, rows_valid, tid);
      store_rows_staged<NDB>(stage, rounded(dKt, alpha), dK + 32 * db0 + head_off + (size_t)kw * sn, sn, rows_valid, tid);
    } else if (!RAGGED || kw + r < NK) {
      store_acc_T<NDB>(dV + 32 * db0 + head_off + (size_t)(kw + r) * sn, dVt, 1.0f, h);
      store_acc_T<NDB>(dK + 32 * db0 + head_off + (size_t)(kw + r) * sn, dKt, alpha, h);
    }
  }
}

// MODE of the dQ kernel:
//   kGivenDelta     delta is read from `delta` (Alg. 2 with delta computed by attn_delta);
//   kRecomputeDelta instead of dQ the kernel forms delta = rowsum(P o dP) (the recomputed,
//                   float32 form of delta of Sec. 3.2: mathematically rowsum(dO o O), but free of the
//                   forward's bf16 roundings of O); `delta` is not read, `delta_out` receives the
//                   result, dQ is not touched;
//   kOwnDelta       the kernel forms delta = rowsum(dO o O) (Alg. 2 step 4) itself, for the rows it
//                   holds anyway, from `O`, writes it to `delta_out` for the dK/dV kernel that
//                   follows, and goes on as kGivenDelta.  The sum is taken in the order of the
//                   stand-alone delta kernel (8-element chains per 16-byte chunk, then a binary tree
//                   over chunks at distances D/16 ... 1), so both give the same bits.
constexpr int kGivenDelta = 0, kRecomputeDelta = 1, kOwnDelta = 2;

// G: wave groups, for grids that leave the SIMDs with a wave or less each.  The groups share a
// work-group's queries, take alternate 32-key blocks of every tile and add their sums through LDS at the
// end.  kQueryWaves waves of 32 queries per group; a tile has as many 32-key blocks as there are groups
// (two with one group).
template <int G> constexpr int kQueryWaves = G == 1 ? 4 : 2;
template <int G> constexpr int kKeysPerTile = G == 4 ? 128 : 64;
template <int D, int G> constexpr int kSmemDq = 4 * kKeysPerTile<G> * D * 2;
// Small head sizes need more waves per SIMD next to one another (four at D = 32, three at D = 64) than a long
// read-ahead: dQ at D = 64 with two waves and fragments read four slots ahead -> three and two (us): B8 H12 N1024
// causal 33.1 -> 30.9, B4 H32 N4096 causal 395 -> 379, B16 H16 N999 full 114 -> 109.
template <int D, int G> constexpr int kDqWavesPerSimd = D == 32 && G == 1 ? 4 : D == 64 && G == 1 ? 3 : kWavesPerSimd<D>;
template <int D> constexpr int kReadAheadDq = D <= 64 ? 2 : D == 256 ? 6 : 4;

template <int D, bool CAUSAL, bool RAGGED, int MODE, int G>
__global__ __launch_bounds__(64 * kQueryWaves<G> * G)
__attribute__((amdgpu_waves_per_eu(kDqWavesPerSimd<D, G>))) void attn_bwd_dq_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    const bf16_t* __restrict__ dO, const float* __restrict__ LSE, const float* __restrict__ delta,
    const bf16_t* __restrict__ O, bf16_t* __restrict__ dQ, float* __restrict__ delta_out, int N,
    float alpha, Layout lay, int pairs, BlockOrder ord) {
  constexpr bool DELTA_MODE = MODE == kRecomputeDelta;
  constexpr int QW = kQueryWaves<G>, QUERIES = 32 * QW, KT = kKeysPerTile<G>;
  constexpr int TILE_BYTES = KT * D * 2;
  constexpr int NDB = D / 32;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  char* ldsK = smem;
  char* ldsV = smem + 2 * TILE_BYTES;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = (tid >> 6) % QW;                   // which 32 queries
  const int grp = G > 1 ? __builtin_amdgcn_readfirstlane(tid / (64 * QW)) : 0;   // which 32-key blocks
  const int r = lane & 31, h = lane >> 5;

  const int NK = RAGGED ? lay.Nk : N;                 // bounds-checking instantiation: N queries, NK keys,
  const int shift = RAGGED ? NK - N : 0;              // causal mask  key <= query + shift
  const int nqt = (N + QUERIES - 1) / QUERIES;
  // pairs != 0 (causal problems with enough work-groups): a work-group takes query block
  // nqt-1-idx and then its mirror image idx; together they always meet the same number of key
  // tiles, so every work-group carries the same load and the grid has no tail of heavy blocks.
  // pairs == 0: one block per work-group, for causal grids in the order the table `ord` gives.
  const int wg = logical_wg(ord, blockIdx.x, gridDim.x);
  const int npw = pairs ? (nqt + 1) / 2 : nqt;          // work-groups per head
  const int bh = wg / npw;
  const int idx = wg % npw;
  const size_t head_off = head_base(lay, bh);
  const int sn = lay.sn;
  const bf16_t* Kh = K + head_base_kv(lay, bh);
  const bf16_t* Vh = V + head_base_kv(lay, bh);
  const float c2 = alpha * kLog2e;
  TileLoader<D, KT, QW * G> loader;
  loader.init(tid, sn);
  FragOffsets<D> fo;
  init_frag_offsets<D>(fo, lane, lds_address(smem));
  if (G > 1) {                                        // group g reads the g-th 32 rows of a tile
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      fo.row[p] += 2 * grp * kRowBlockBytes<D>;
      fo.col[p] += 2 * grp * kRowBlockBytes<D>;
    }
  }

  for (int part = 0; part < (pairs ? 2 : 1); ++part) {
  if (part > 0) __syncthreads();                      // the first block's output staging is done with the tile buffers
  const int qt = pairs ? (part == 0 ? nqt - 1 - idx : idx)
                       : nqt - 1 - (idx + (CAUSAL && ord.n == 0 ? small_grid_rotation(bh, nqt, gridDim.x, D == 128 ? 768 : 1152) : 0)) % nqt;
  if (part == 1 && qt == nqt - 1 - idx) break;        // odd number of blocks: the middle one has no partner
  const int q0 = qt * QUERIES;
  const int qw = q0 + 32 * wave;

  // Q_i^T / dO_i^T fragments (B operands): lane (r,h) holds Q[qw + r][16kc + 8h .. +7]
  // (rows past the sequence end read the last row; their dQ is not stored)
  const int qc = (RAGGED && qw + r >= N) ? N - 1 : qw + r;
  bf16x8 qf[D / 16], dof[D / 16];
#pragma unroll
  for (int kc = 0; kc < D / 16; ++kc) {
    qf[kc] = *reinterpret_cast<const bf16x8*>(Q + head_off + (size_t)qc * sn + 16 * kc + 8 * h);
    dof[kc] = *reinterpret_cast<const bf16x8*>(dO + head_off + (size_t)qc * sn + 16 * kc + 8 * h);
  }
  float l2 = LSE[(size_t)bh * N + qc] * kLog2e;
  if (RAGGED && l2 == -INFINITY) l2 = 0.f;             // a query that sees no key: all its scores are masked below
  float dl = 0.f;
  if (MODE == kGivenDelta) dl = delta[(size_t)bh * N + qc];
  if (MODE == kOwnDelta) {
    // this lane holds chunks 2kc + h of its row: the chains of its chunks, the tree levels that
    // stay inside one parity class, and the last level (chunk 0 + chunk 1 classes) across the
    // two lanes of the row
    constexpr int NCS = kPow2D<D> / 16;     // D = 96: the tree of a 128-wide row whose last chunks are zero
    float cs[NCS];
#pragma unroll
    for (int kc = 0; kc < NCS; ++kc) cs[kc] = 0.f;
#pragma unroll
    for (int kc = 0; kc < D / 16; ++kc) {
      const bf16x8 o8 = *reinterpret_cast<const bf16x8*>(O + head_off + (size_t)qc * sn + 16 * kc + 8 * h);
      float c = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) c = __builtin_fmaf((float)o8[e], (float)dof[kc][e], c);
      cs[kc] = c;
    }
#pragma unroll
    for (int off = NCS / 2; off >= 1; off >>= 1)
#pragma unroll
      for (int kc = 0; kc < off; ++kc) cs[kc] += cs[kc + off];
    dl = sum_with_partner32(cs[0]);
    if (h == 0 && grp == 0 && (!RAGGED || qw + r < N)) delta_out[(size_t)bh * N + qw + r] = dl;
  }
  float pdp = 0.f;                                   // DELTA_MODE: this lane's share of sum_k P dP
  // -delta_i in all 16 accumulator slots of the lane: the third operand of the first dP^T matrix
  // instruction of every key block, which then delivers dP - delta with no vector instruction
  // (Alg. 2: dS = P o (dP - delta)).  Kept opaque so that it stays resident instead of being
  // rebuilt per block.
  f32x16 neg_delta;
#pragma unroll
  for (int i = 0; i < 16; ++i) neg_delta[i] = -dl;
  asm volatile("" : "+v"(neg_delta));
  f32x16 dQt[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) dQt[db][i] = 0.f;

  const int kend = !CAUSAL ? NK : !RAGGED ? q0 + QUERIES : max(0, min(NK, q0 + QUERIES + shift));
  const int ntiles = RAGGED || KT > QUERIES ? (kend + KT - 1) / KT : kend / KT;

  loader.template load_rows<RAGGED>(ldsK, Kh, 0, NK);
  loader.template load_rows<RAGGED>(ldsV, Vh, 0, NK);
  wait_vmem();
#pragma unroll
  for (int kc = 0; kc < D / 16; ++kc) { settle(qf[kc]); settle(dof[kc]); }
  settle(l2);
  __syncthreads();

  // One key tile; BUF (which LDS buffer holds it) is a compile-time constant so that every LDS
  // address is a precomputed per-lane offset plus an immediate.
  auto tile_step = [&](auto buf_c, int j) {
    constexpr int buf = decltype(buf_c)::value;
    constexpr int tK = buf * TILE_BYTES;            // byte offsets of this tile's K and V in smem
    constexpr int tV = (2 + buf) * TILE_BYTES;
    // The next tile lands in the other buffer while this one is being processed; its transfer
    // instructions are issued one per step of the first block's score products rather than in one
    // burst behind the barrier.  After the last tile the current one is fetched once more into the
    // idle buffer (harmless; keeps the instruction stream free of branches).
    const int jn = (j + 1 < ntiles) ? j + 1 : j;
    constexpr int NLD = decltype(loader)::NI;
    const auto pendK = loader.template prepare<RAGGED>(smem + (buf ^ 1) * TILE_BYTES, Kh, jn * KT, NK);
    const auto pendV = loader.template prepare<RAGGED>(smem + (2 + (buf ^ 1)) * TILE_BYTES, Vh, jn * KT, NK);
    auto issue_part = [&](int i) {
      if (i < NLD) loader.issue(pendK, i);
      else if (i < 2 * NLD) loader.issue(pendV, i - NLD);
    };
    bool issued = false;
    const int kt0 = j * KT;
    // The NB 32-key blocks of a tile that belong to this wave's group against its 32 queries, as one stream of matrix
    // instructions ("slots") in phases of D/16:  S^T, dP^T of each block, then the dQ products.  The vector work
    // lies under matrix instructions: P = exp(S - L) under the block's dP^T, dS = P o (dP - delta) under the next
    // phase (with one block only its second half), and every LDS fragment is read AHEAD slots
    // before its use (a fence per slot keeps that order).  The next tile's transfer is issued on the way.  Same bits as
    // block after block and phase after phase; us, whole kernel: B4 H32 N4096 d128 causal 716 -> 682, B2 H16 N2048 d96
    // causal 52.3 -> 50.0, B2 H8 N2048 d256 causal 89 -> 80, B4 H12 N1024 d64 causal 22.0 -> 19.9, B8 H12 N1024 d64
    // causal 32.4 -> 30.7.
    // MASKED: a block crosses the diagonal or the sequence end.
    constexpr int NBT = KT / 32 / G;                         // blocks of this wave's group in a tile
    auto kblocks = [&](auto masked_c, auto nb_c, auto kb_c) {
      constexpr bool MASKED = decltype(masked_c)::value;
      constexpr int NB = decltype(nb_c)::value;
      constexpr int kb = decltype(kb_c)::value;
      constexpr int NS = D / 16, SLOTS = (DELTA_MODE ? 2 : 3) * NB * NS;
      constexpr int AHEAD = kReadAheadDq<D>, RING = AHEAD + 1;
      auto fragment = [&](int i) -> bf16x8 {
        const int phase = i / NS, u = i % NS;
        if (phase < 2 * NB) return lds_row8<D>(phase % 2 ? tV : tK, fo, 32 * (kb + phase / 2), u);
        return lds_col8<D>(tK, fo, 32 * (kb + phase - 2 * NB) + 16 * (u / NDB), u % NDB);
      };
      bf16x8 ring[RING], dsf[NB][2];
      f32x16 s[NB], dp[NB];
      int lim[NB];                       // MASKED: last visible entry, c = 8 (i / 4) + i % 4
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) ring[i] = fragment(i);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
#pragma unroll
        for (int i = 0; i < 16; ++i) s[b][i] = 0.f;
        const int kb0 = kt0 + 32 * (kb + b + grp);
        // (formed here and not ahead of the tile loop, which costs registers: at D = 64, causal, with bounds checks six were
        // spilled.  us: 800 heads N65 15.0 -> 13.2, 400 heads N200 19.8 -> 17.6, B8 H12 N1000 29.6 -> 28.0)
        int ln = lane;
        if (MASKED) asm volatile("" : "+v"(ln));
        lim[b] = CAUSAL ? __builtin_amdgcn_readfirstlane(qw) + (ln & 31) + shift - kb0 - 4 * (ln >> 5) : 0x7fffffff;
        if (RAGGED) lim[b] = min(lim[b], NK - 1 - kb0 - 4 * (ln >> 5));
      }
      // P of entries i0 .. i1 - 1 of block b: keys in this lane's future and keys past the sequence end get
      // S = -inf, P = exp(-inf) = 0
      auto form_p = [&](int b, int i0, int i1) {
#pragma unroll
        for (int i = i0; i < i1; ++i) {
          if (MASKED && 8 * (i >> 2) + (i & 3) > lim[b]) s[b][i] = -INFINITY;
          s[b][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[b][i], c2, -l2));
        }
      };
      // dS of the same; dp already holds dP - delta
      auto form_ds = [&](int b, int i0, int i1) {
#pragma unroll
        for (int i = i0; i < i1; ++i) {
          if (DELTA_MODE) pdp = __builtin_fmaf(s[b][i], dp[b][i], pdp);
          else dsf[b][i >> 3][i & 7] = (bf16_t)(s[b][i] * dp[b][i]);
        }
      };
      static_for<SLOTS>([&](auto slot) {
        constexpr int sl = decltype(slot)::value, phase = sl / NS, u = sl % NS;
        if (sl + AHEAD < SLOTS) ring[(sl + AHEAD) % RING] = fragment(sl + AHEAD);
        if (NB == 1 && sl == 2 * NS) form_ds(0, 0, 8);
        const bf16x8 a = ring[sl % RING];
        if constexpr (phase >= 2 * NB) dQt[u % NDB] = mfma32(a, dsf[phase - 2 * NB][u / NDB], dQt[u % NDB]);   // step 13
        else if constexpr (phase % 2 == 0) s[phase / 2] = mfma32(a, qf[u], s[phase / 2]);
        else dp[phase / 2] = mfma32(a, dof[u], u == 0 ? neg_delta : dp[phase / 2]);
        // (One transfer instruction per two slots at D = 256: four waves that issue one each per slot ask for 128 bytes a clock
        // where the load path takes 64, and stall.  us, one slot -> two: B1 H8 N2048 d256 full 59.0 -> 57.4, causal 51.0 -> 47.5.
        // d <= 128: even, and 0.1 to 0.2 us slower where a problem is one tile long, as the transfer ends later.)
        constexpr int EVERY = D == 256 ? 2 : 1;
        static_assert(2 * NLD * EVERY <= 2 * NS, "all of the transfer is issued under S and dP");
        if (kb == 0 && sl % EVERY == 0) issue_part(sl / EVERY);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const int e = sl - 2 * NS * b - NS - 1;            // P of block b lies under the slots after its first dP^T
          if (e >= 0 && e < NS) form_p(b, 16 * e / NS, 16 * (e + 1) / NS);
          const int f = e - NS;                              // dS of block b
          if (NB > 1 && !DELTA_MODE && f >= 0 && f < NS) form_ds(b, 16 * f / NS, 16 * (f + 1) / NS);
        }
        if (NB == 1 && sl == 2 * NS) form_ds(0, 8, 16);
        __builtin_amdgcn_sched_barrier(0);
      });
      if (DELTA_MODE) {
        form_p(NB - 1, 16 * (NS - 1) / NS, 16);              // (the slot these would lie under is a dQ product)
#pragma unroll
        for (int b = 0; b < NB; ++b) form_ds(b, 0, 16);
      }
    };
    int k0 = kt0 + 32 * grp;                                 // first key of them
    // (in a vector register: behind a branch that the compiler knows to be uniform it needs 30 registers more)
    if (RAGGED && !CAUSAL) asm volatile("" : "+v"(k0));
    const int last = k0 + 32 * NBT - 1;
    if ((!CAUSAL || last <= qw + shift) && (!RAGGED || last < NK)) {
      asm volatile("; every key counts");                    // (differs from the other path: nothing is merged in front of the branch)
      constexpr int NB = D == 32 ? 1 : NBT;
      static_for<NBT / NB>([&](auto i) { kblocks(std::false_type{}, std::integral_constant<int, NB>{}, std::integral_constant<int, NB * decltype(i)::value>{}); });
      issued = true;
    } else {
      asm volatile("; masked");
      static_for<NBT>([&](auto kb) {
        const int kb0 = k0 + 32 * decltype(kb)::value;
        if ((CAUSAL && kb0 > qw + shift + 31) || (RAGGED && kb0 >= NK)) return;    // nothing to see in the block
        kblocks(std::true_type{}, std::integral_constant<int, 1>{}, kb);
        if (decltype(kb)::value == 0) issued = true;
      });
    }
    if (!issued) {      // a wave that skipped the tile's first block still has its share of the transfer to issue
#pragma unroll
      for (int i = 0; i < 2 * NLD; ++i) issue_part(i);
    }
    wait_vmem();
    __syncthreads();
  };
  for (int j = 0; j < ntiles; j += 2) {
    tile_step(std::integral_constant<int, 0>{}, j);
    if (j + 1 < ntiles) tile_step(std::integral_constant<int, 1>{}, j + 1);
  }
  if (DELTA_MODE) {
    static_assert(!DELTA_MODE || G == 1, "the recomputed delta has no wave groups");
    const float dsum = sum_with_partner32(pdp);      // the partner lane holds the other keys of every block
    if (h == 0 && (!RAGGED || qw + r < N)) delta_out[(size_t)bh * N + qw + r] = dsum;
    continue;
  }
  if constexpr (G > 1) {
    // The upper half of the groups hands its sums to the lower half, until group 0 has the total;
    // every wave is past the last tile's barrier, the tile buffers are free.  (Opaque lane index:
    // see the dK/dV kernel.)
    int ln = lane;
    asm volatile("" : "+v"(ln));
#pragma unroll
    for (int half = G / 2; half >= 1; half >>= 1) {
      if (grp < 2 * half) {
        char* area = smem + ((grp % half) * QW + wave) * (NDB * 4096);
        if (grp >= half) {
#pragma unroll
          for (int i = 0; i < 4 * NDB; ++i) {
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = dQt[i >> 2][4 * (i & 3) + e];
            *reinterpret_cast<f32x4*>(area + (i * 64 + ln) * 16) = v;
          }
        }
      }
      __syncthreads();
      if (grp < half) {
        const char* area = smem + (grp * QW + wave) * (NDB * 4096);
#pragma unroll
        for (int i = 0; i < 4 * NDB; ++i) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(area + (i * 64 + ln) * 16);
#pragma unroll
          for (int e = 0; e < 4; ++e) dQt[i >> 2][4 * (i & 3) + e] += v[e];
        }
      }
      __syncthreads();
    }
    if (grp != 0) continue;
  }
  if constexpr (kCanStage<D / 32>) {
    // the tile buffers are free now (every wave is past the last tile's barrier): they serve as
    // the staging areas of store_rows_staged; the barrier at the top of the part loop keeps the
    // next block's tile transfers from overwriting an area a slower wave is still reading
    auto piece = [&](int db, int g) {
      bf16x4 o4;
#pragma unroll
      for (int e = 0; e < 4; ++e) o4[e] = (bf16_t)(dQt[db][4 * g + e] * alpha);
      return o4;
    };
    store_rows_staged<D / 32>(smem, piece, dQ + head_off + (size_t)qw * sn, sn, RAGGED ? N - qw : 32, tid);
  } else if (!RAGGED || qw + r < N) {
    store_acc_T<D / 32>(dQ + head_off + (size_t)(qw + r) * sn, dQt, alpha, h);
  }
  }   // part
}

template <typename KernT>
static hipError_t set_smem(KernT kern, int smem, std::atomic<bool>& done) {
  if (done.load(std::memory_order_acquire)) return hipSuccess;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  if (e == hipSuccess) done.store(true, std::memory_order_release);
  return e;
}

template <int D, bool CAUSAL, bool RAGGED, bool GROUPED, int G, bool DENSE = false>
static hipError_t launch_dkdv_g(const void* Q, const void* K, const void* V, const void* dO,
                                const float* LSE, const float* delta, void* dK, void* dV, int BH,
                                int N, float alpha, Layout lay, hipStream_t st) {
  constexpr int smem = kSmemDkDv<D, G>;
  static std::atomic<bool> set{false};
  auto k = attn_bwd_dkdv_kernel<D, CAUSAL, RAGGED, GROUPED, G, DENSE>;
  hipError_t e;
  if ((e = set_smem(k, smem, set)) != hipSuccess) return e;
  constexpr int KEYS = 32 * kKeyWaves<G>, THREADS = 64 * kKeyWaves<G> * G;
  const int nkt = ((RAGGED ? lay.Nk : N) + KEYS - 1) / KEYS;
  // Under the causal mask: one block per work-group in a balanced order when that grid is at most
  // one and a half rounds of work-groups (measured: beyond that, mirrored pairs of blocks are as
  // fast or 2 % faster for this kernel), mirrored pairs otherwise.
  static std::atomic<int> resident{0};
  static thread_local OrderCache cache;
  const BlockOrder* ord = &kNoOrder;
  if (CAUSAL && kDSplit<D> == 1) {
    const int res = resident_per_cu(k, smem, resident, THREADS);
    ord = &small_grid_order(cache, (BH / lay.group) * nkt, nkt, res, 3LL * kNumCUs * res / 2);
  }
  const int pairs = (CAUSAL && ord->n == 0) ? 1 : 0;
  hipLaunchKernelGGL(k, dim3((BH / lay.group) * (pairs ? (nkt + 1) / 2 : nkt) * kDSplit<D>), dim3(THREADS), smem, st, (const bf16_t*)Q,
                     (const bf16_t*)K, (const bf16_t*)V, (const bf16_t*)dO, LSE, delta,
                     (bf16_t*)dK, (bf16_t*)dV, N, alpha, lay, pairs, *ord);
  return hipGetLastError();
}

template <int D, bool CAUSAL, bool RAGGED, bool GROUPED>
static hipError_t launch_dkdv(const void* Q, const void* K, const void* V, const void* dO,
                              const float* LSE, const float* delta, void* dK, void* dV, int BH,
                              int N, float alpha, Layout lay, hipStream_t st) {
  // Wave groups where one-group work-groups would leave the SIMDs with a single wave each.  Short
  // sequences do not pay for the final exchange.
  // Four groups on 64 keys, up to one 128-key block per CU (half of that without a mask, where all
  // blocks are equal and two per CU would run one after the other).  Measured, two groups -> four (us): B2
  // H32/8 N2048 d128 causal 200 -> 149, B2 H8 N2048 d128 causal 54.8 -> 48.8, d96 45.0 -> 37.6, d64 35.3 -> 28.5, B1 H4 N4096
  // d128 causal 93 -> 62, B1 H8 N2048 d128 full 50.4 -> 39.1, B1 H1 N1024 d64 full 17.1 -> 11.5; beyond the
  // limits: B2 H12 N2048 d128 causal 62 -> 89, B4 H12 N1024 d64 causal 26.0 -> 37.5.
  // Two groups on 128 keys up to one block per CU; up to two under the causal mask at D >= 96, where the
  // blocks differ in work and the CU with the heaviest one decides (at D = 64 two work-groups with 64-row tiles on a
  // CU do as well).  Measured, one group -> two (us): B2 H12 N2048 d128 causal 70.8 -> 62.6, d96 53.2 -> 48.5, B2 H8 N2048
  // d128 full 74.4 -> 66.5, at the limit of two per CU B2 H16 N2048 d128 causal 79.4 -> 76.6, d96 60.5 -> 61.9; beyond the
  // limits: B5 H8 N2048 d128 causal 93 -> 129, B3 H8 N2048 d128 full 108 -> 114, B4 H12 N1024 d64 causal 24.5 -> 26.0.
  if constexpr (D <= 128) {
    const int NK = RAGGED ? lay.Nk : N;      // (the rule looks at the keys only: a chunk of queries gets the sums of the square problem)
    const long long blocks = (long long)(BH / lay.group) * ((NK + kKeysPerWG - 1) / kKeysPerWG);
    if (NK >= 512) {
      if (blocks <= (CAUSAL ? kNumCUs : kNumCUs / 2))
        return launch_dkdv_g<D, CAUSAL, RAGGED, GROUPED, 4>(Q, K, V, dO, LSE, delta, dK, dV, BH, N, alpha, lay, st);
      if constexpr (!CAUSAL || D >= 96)
        if (blocks <= (CAUSAL ? 2 : 1) * kNumCUs)
          return launch_dkdv_g<D, CAUSAL, RAGGED, GROUPED, 2>(Q, K, V, dO, LSE, delta, dK, dV, BH, N, alpha, lay, st);
    }
  }
  // More than two 128-key blocks per CU at D <= 64: three waves per SIMD.  Measured, two -> three (us): B8 H12 N1024 d64
  // causal 39.1 -> 35.7, B32 H12 N512 d64 full 62.5 -> 58.6, B4 H32 N4096 d64 causal 557 -> 535, B8 H12 N1000 d64 full
  // 60.7 -> 56.4, causal 40.1 -> 36.5, B8 H12 N1024 d32 causal 28.2 -> 23.4, B8 H16 N1001 d32 full 52.7 -> 51.2; just above the
  // limit 400 heads N200 d64 causal 19.0 -> 19.2, B2 H16 N2050 47.8 -> 50.1; below it: B4 H12 N1024 d64 causal 24.5 -> 25.4, in pairs
  // B1 H33 N2040 d64 even, B5 H13 N1024 d32 27.7 -> 27.9; with grouped queries B4 H32/8 N2048 d64 causal 164 -> 170.
  if constexpr (D <= 64 && !GROUPED) {
    const int NK = RAGGED ? lay.Nk : N;
    // (head counts the order table does not take run as pairs of blocks: half as many work-groups)
    if ((long long)BH * ((NK + kKeysPerWG - 1) / kKeysPerWG) > (CAUSAL && BH % 8 != 0 ? 4 : 2) * kNumCUs)
      return launch_dkdv_g<D, CAUSAL, RAGGED, GROUPED, 1, true>(Q, K, V, dO, LSE, delta, dK, dV, BH, N, alpha, lay, st);
  }
  return launch_dkdv_g<D, CAUSAL, RAGGED, GROUPED, 1>(Q, K, V, dO, LSE, delta, dK, dV, BH, N, alpha, lay, st);
}

template <int D, bool CAUSAL, bool RAGGED, int MODE, int G>
static hipError_t launch_dq_g(const void* Q, const void* K, const void* V, const void* dO,
                              const float* LSE, const float* delta, const void* O, void* dQ,
                              float* delta_out, int BH, int N, float alpha, Layout lay, hipStream_t st) {
  constexpr int smem = kSmemDq<D, G>;
  constexpr int QUERIES = 32 * kQueryWaves<G>, THREADS = 64 * kQueryWaves<G> * G;
  static std::atomic<bool> set{false};
  auto k = attn_bwd_dq_kernel<D, CAUSAL, RAGGED, MODE, G>;
  hipError_t e;
  if ((e = set_smem(k, smem, set)) != hipSuccess) return e;
  // as in the forward: mirrored pairs of query blocks under the causal mask when that still
  // leaves at least two full rounds of work-groups
  const int nqt = (N + QUERIES - 1) / QUERIES;
  const int pairs = (CAUSAL && (long long)BH * ((nqt + 1) / 2) >= 1024) ? 1 : 0;
  const int grid = BH * (pairs ? (nqt + 1) / 2 : nqt);
  static std::atomic<int> resident{0};
  static thread_local OrderCache cache;
  const BlockOrder& ord = (CAUSAL && !pairs)
      ? small_grid_order(cache, grid, nqt, resident_per_cu(k, smem, resident, THREADS), 8 * kMaxOrder) : kNoOrder;
  hipLaunchKernelGGL(k, dim3(grid), dim3(THREADS), smem, st, (const bf16_t*)Q,
                     (const bf16_t*)K, (const bf16_t*)V, (const bf16_t*)dO, LSE, delta,
                     (const bf16_t*)O, (bf16_t*)dQ, delta_out, N, alpha, lay, pairs, ord);
  return hipGetLastError();
}

template <int D, bool CAUSAL, bool RAGGED, int MODE>
static hipError_t launch_dq(const void* Q, const void* K, const void* V, const void* dO,
                            const float* LSE, const float* delta, const void* O, void* dQ,
                            float* delta_out, int BH, int N, float alpha, Layout lay, hipStream_t st) {
  // Wave groups on small grids, as in launch_dkdv: up to one 128-query block per CU under the causal mask,
  // half of that without one, from 512 keys on.  Measured, one group -> four groups on 64 queries (us): B2 H8
  // N2048 d128 causal 50 -> 45, B1 H8 the same 44 -> 30, d64 30 -> 18, B1 H4 N4096 d128 79 -> 48, B1 H8
  // N2048 d128 full 44 -> 32, B1 H1 N8192 d64 101 -> 47; beyond the limits: B2 H12 N2048 d128 causal 52 -> 66,
  // B2 H8 N2048 d128 full 57 -> 64.  At D = 256 (one wave per SIMD) two groups on 64 queries are what fits:
  // B1 H8 N2048 full 73 -> 57, beyond the limit B2 H8 95 -> 109.  There the causal mask takes the limit to one block per CU
  // only where the order table balances the halved blocks (head counts in eights), in square problems (with more keys than
  // queries the blocks differ less) and from 1500 keys on: B2 H8 N2048 85 -> 79, B1 H8 N4000 145 -> 124, B1 H16 N1900 78 -> 73,
  // B2 H8 N1500 61 -> 54; not taken: B1 H15 N2048 82 -> 98, B1 H24 N1280 57 -> 60, B4 H8 N1024 51 -> 53, B2 H12 N2048 91 -> 116.
  if constexpr (MODE != kRecomputeDelta) {
    const long long blocks = (long long)BH * ((N + kQPerWG - 1) / kQPerWG);
    const bool balanced = CAUSAL && (D <= 128 || (BH % 8 == 0 && lay.Nk == N && N >= 1500));
    if ((RAGGED ? lay.Nk : N) >= 512 && blocks <= (balanced ? kNumCUs : kNumCUs / 2)) {
      // (two groups without a mask: here the aligned kernel is the faster one and spills nothing, unlike that of one group; us,
      // bounds-checking -> aligned: B1 H8 N2048 57.4 -> 56.2, B1 H4 N4096 100.7 -> 98.5, B1 H8 N512 20.8 -> 20.0)
      if constexpr (D == 256 && !CAUSAL)
        if (lay.Nk == N && N % kQPerWG == 0)
          return launch_dq_g<D, CAUSAL, false, MODE, 2>(Q, K, V, dO, LSE, delta, O, dQ, delta_out, BH, N, alpha, lay, st);
      return launch_dq_g<D, CAUSAL, RAGGED, MODE, (D <= 128 ? 4 : 2)>(Q, K, V, dO, LSE, delta, O, dQ, delta_out, BH, N, alpha, lay, st);
    }
  }
  return launch_dq_g<D, CAUSAL, RAGGED, MODE, 1>(Q, K, V, dO, LSE, delta, O, dQ, delta_out, BH, N, alpha, lay, st);
}

}  // namespace

hipError_t attn_bwd_dkdv_dispatch(const void* Q, const void* K, const void* V, const void* dO,
                                  const float* LSE, const float* delta, void* dK, void* dV,
                                  int BH, int N, int d, int causal, float alpha, Layout lay,
                                  hipStream_t st) {
  // The aligned kernels carry no bounds handling.  At D = 256 without a mask there is none but dQ with two wave groups: with
  // nothing that parts the tile from what follows, the stream of matrix instructions spills 14 and 126 registers there (us, B2 H8
  // N2048, phase after phase -> aligned stream -> bounds-checking stream: dK/dV 228 -> 232 -> 190, dQ 94 -> 194 -> 92).
  const bool ragged = (N % kKeysPerWG) != 0 || lay.Nk != N || (d == 256 && !causal);
  if (lay.group > 1) {   // grouped queries: the bounds-checking instantiation serves every N
#define CASEG(DD, CC)                                 \
  if (d == DD && (causal != 0) == CC)                 \
    return launch_dkdv<DD, CC, true, true>(Q, K, V, dO, LSE, delta, dK, dV, BH, N, alpha, lay, st);
    CASEG(32, false) CASEG(32, true) CASEG(64, false) CASEG(64, true) CASEG(128, false) CASEG(128, true)
    CASEG(256, false) CASEG(256, true) CASEG(96, false) CASEG(96, true)
#undef CASEG
    return hipErrorInvalidValue;
  }
#define CASE(DD, CC, RR)                                                \
  if (d == DD && (causal != 0) == CC && ragged == RR)                   \
    return launch_dkdv<DD, CC, RR, false>(Q, K, V, dO, LSE, delta, dK, dV, BH, N, alpha, lay, st);
  CASE(32, false, false) CASE(32, false, true) CASE(32, true, false) CASE(32, true, true)
  CASE(64, false, false) CASE(64, false, true) CASE(64, true, false) CASE(64, true, true)
  CASE(128, false, false) CASE(128, false, true) CASE(128, true, false) CASE(128, true, true)
  CASE(256, false, true) CASE(256, true, false) CASE(256, true, true)
  CASE(96, false, false) CASE(96, false, true) CASE(96, true, false) CASE(96, true, true)
#undef CASE
  return hipErrorInvalidValue;
}

// O == nullptr: delta is given.  Otherwise delta is formed by the kernel from O and dO and also
// written to delta_out (which must then be non-null).
hipError_t attn_bwd_dq_dispatch(const void* Q, const void* K, const void* V, const void* dO,
                                const float* LSE, const float* delta, const void* O, void* dQ,
                                float* delta_out, int BH, int N, int d, int causal, float alpha,
                                Layout lay, hipStream_t st) {
  const bool ragged = (N % kQPerWG) != 0 || lay.Nk != N || (d == 256 && !causal);   // (see attn_bwd_dkdv_dispatch)
  const bool own = O != nullptr;
#define CASE(DD, CC, RR)                                                \
  if (d == DD && (causal != 0) == CC && ragged == RR)                   \
    return own ? launch_dq<DD, CC, RR, kOwnDelta>(Q, K, V, dO, LSE, nullptr, O, dQ, delta_out, BH, N, alpha, lay, st) \
               : launch_dq<DD, CC, RR, kGivenDelta>(Q, K, V, dO, LSE, delta, nullptr, dQ, nullptr, BH, N, alpha, lay, st);
  CASE(32, false, false) CASE(32, false, true) CASE(32, true, false) CASE(32, true, true)
  CASE(64, false, false) CASE(64, false, true) CASE(64, true, false) CASE(64, true, true)
  CASE(128, false, false) CASE(128, false, true) CASE(128, true, false) CASE(128, true, true)
  CASE(256, false, true) CASE(256, true, false) CASE(256, true, true)
  CASE(96, false, false) CASE(96, false, true) CASE(96, true, false) CASE(96, true, true)
#undef CASE
  return hipErrorInvalidValue;
}

// delta = rowsum(P o dP) recomputed from Q, K, V, dO and LSE (always the bounds-checking kernels).
hipError_t attn_delta_recompute_dispatch(const void* Q, const void* K, const void* V,
                                         const void* dO, const float* LSE, float* delta_out,
                                         int BH, int N, int d, int causal, float alpha,
                                         Layout lay, hipStream_t st) {
#define CASE(DD, CC)                                  \
  if (d == DD && (causal != 0) == CC)                 \
    return launch_dq<DD, CC, true, kRecomputeDelta>(Q, K, V, dO, LSE, nullptr, nullptr, nullptr, delta_out, BH, N, alpha, lay, st);
  CASE(32, false) CASE(32, true) CASE(64, false) CASE(64, true) CASE(128, false) CASE(128, true)
  CASE(256, false) CASE(256, true) CASE(96, false) CASE(96, true)
#undef CASE
  return hipErrorInvalidValue;
}

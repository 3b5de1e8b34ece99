// Flash-attention backward for gfx950 (Alg. 2 of arXiv 2510.04212), as two kernels so that no
// gradient needs a cross-work-group reduction (no atomics, deterministic):
//
//   attn_bwd_dkdv_kernel  one work-group per (batch, head, 128-key block; 64 or 32 on small grids) -- under the causal mask
//                         per pair of mirrored blocks, one after the other, unless the grid is
//                         small (then one block each, in a balanced order); K_j / V_j fragments
//                         stay in registers (V_j in LDS at D = 128), query tiles (Q_i, dO_i, L_i,
//                         delta_i; 64 rows, 32 at D = 128) stream through LDS.  Per tile:  S = Q_i K_j^T,  P = exp(S - L),  dP = dO_i V_j^T,
//                         dS = P o (dP - delta),  dV_j^T += dO_i^T P,  dK_j^T += Q_i^T dS.
//   attn_bwd_dq_kernel    one work-group per (batch, head, 128-query block; 64 or 32 on small grids); Q_i / dO_i fragments,
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
#include "bwd_forms.hpp"
#include "common.hpp"

#include <atomic>
#include <type_traits>

namespace {

constexpr int kKeysPerWG = 128;   // dK/dV kernel: keys per work-group (32 per wave); 64 or 32 with four or eight wave groups
constexpr int kQPerWG = 128;      // dQ kernel: queries per work-group (32 per wave); 64 or 32 with wave groups

// GROUPED: grouped-query attention (lay.group > 1): the work-group serves several query heads.
// Kept out of the ordinary kernel so that its tile loop has a fixed head and no bookkeeping.
// At D = 256 the two accumulator sets of a full key block would not fit the register file next
// to the K / V fragments: a work-group then owns 128 of the 256 columns of dK and dV (kDSplit
// work-groups per key block, each recomputing S and dP).
template <int D> constexpr int kDSplit = D > 128 ? 2 : 1;
// The kernel wants two waves on every SIMD: one wave alone leaves the matrix cores idle whenever
// any of its instructions waits.  That means at most 256 registers per lane (some instantiations
// at D = 128 under the mask spill three to nine, kHalf's bounds-checking one at D = 64 under the mask three,
// all outside their tile loops).  At D = 128 the
// accumulators (128) and the K fragments (32) leave no room for the V fragments: V_j is kept in LDS
// for the whole block (8 more fragment reads per 32 queries to 48) and the query tiles shrink to 32
// rows per wave group, so that two work-groups fit a CU.  Measured against one wave per SIMD with
// 430 registers and a hand-made four-phase pipeline (us, bit-identical): B4 H32 N4096 d128 causal
// 1043 -> 990, B4 H16 N2048 d128 full 281 -> 234, B4 H16 N1999 d128 causal 157 -> 132 and full
// 602 -> 235 (that one spilled), B4 H16 N4096 d96 causal 484 -> 369.  At D = 256 (one wave per SIMD all
// the same) the single code path for masked and unmasked blocks alone took 140 -> 109.
template <int D> constexpr bool kVInLds = D == 128;
template <int D> constexpr int kWavesPerSimd = D <= 128 ? 2 : 1;
// FORM: how many wave groups a work-group has.  2 (512 threads) is for grids that give a CU only one work-group:
// the groups share the work-group's keys and take alternate 32-query blocks, each into accumulators
// of its own, which are added through LDS at the end.  4 splits further: 64 keys (two waves) per
// group, so that a grid has twice the work-groups of half the length; a query tile is then read
// from L2 for half as many keys.  The smallest grids take 32 keys, one wave per group: 8 groups at D <= 64, and four, kNarrow,
// where the tiles of eight would not fit the LDS.  kHalf (dK/dV at D <= 96): two groups on 64 keys, 256 threads.  bwd_forms.hpp has the
// rules that choose.
template <int FORM> constexpr int kGroups = FORM == kNarrow ? 4 : FORM == kHalf ? 2 : FORM;
// waves per group, 32 keys each
template <int FORM> constexpr int kKeyWaves = FORM == 8 || FORM == kNarrow ? 1 : FORM == 4 || FORM == kHalf ? 2 : 4;
template <int D, int FORM> constexpr int kQTile = D == 128 || FORM >= 4 ? 32 * kGroups<FORM> : 64;   // query rows per streamed tile
// LDS fragments are read this many matrix instructions before their use.
// (At D = 128 what the registers allow: the fragments of V_j come from LDS too.  Four wave groups at small D: us, four ahead ->
// two, B1 H4 N4096 d64 causal 41.1 -> 40.1, B1 H1 38.5 -> 37.7, B1 H2 N8192 d32 causal 54.0 -> 53.4, full 51.2 -> 50.5, B1 H8
// N2000 d32 16.7 -> 16.4; d64 full even to 2 % slower: not there.)
template <int D, int G, bool CAUSAL, bool DENSE> constexpr int kReadAhead =
    DENSE || (G >= 4 && (D == 32 || (D == 64 && CAUSAL))) ? 2 : D == 256 ? 6 : D == 128 ? 2 : 4;
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
template <int D, int G> constexpr int kExchangeBytes = G > 1 ? kGroups<G> * kKeyWaves<G> * (D / 32) * 4096 : 0;
constexpr int max_int(int a, int b) { return a > b ? a : b; }
template <int D, int G> constexpr int kSmemDkDv =
    G > 1 ? max_int(kTilesEnd<D, G>, kExchangeBytes<D, G>)
          : kStageOverTiles<D, G> ? max_int(kTilesEnd<D, G>, kVBytes<D, G> + kStageBytes<D>) : kTilesEnd<D, G> + kStageBytes<D>;

// DENSE (D <= 64): three waves on every SIMD at the price of a shorter read-ahead, for grids that have the work-groups
// (bwd_forms.hpp).
template <int D, bool DENSE> constexpr int kDkDvWaves = DENSE ? 3 : kWavesPerSimd<D>;
template <int D, bool CAUSAL, bool RAGGED, bool GROUPED, int FORM, bool DENSE>
__global__ __launch_bounds__(64 * kKeyWaves<FORM> * kGroups<FORM>)
__attribute__((amdgpu_waves_per_eu(kDkDvWaves<D, DENSE>, kDkDvWaves<D, DENSE>))) void attn_bwd_dkdv_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    const bf16_t* __restrict__ dO, const float* __restrict__ LSE, const float* __restrict__ delta,
    bf16_t* __restrict__ dK, bf16_t* __restrict__ dV, int N, float alpha, Layout lay, int pairs,
    BlockOrder ord) {
  constexpr int G = kGroups<FORM>, QT = kQTile<D, FORM>;
  constexpr int TILE_BYTES = QT * D * 2, GT = TILE_BYTES / G;
  constexpr int T0 = kVBytes<D, FORM>;                    // the tile buffers follow V_j: per wave group Q [2][GT], dO [2][GT]
  constexpr int KW = kKeyWaves<FORM>, KEYS = 32 * KW;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  char* ldsQ = smem + T0;
  char* ldsdO = ldsQ + 2 * GT;
  float* ldsL = reinterpret_cast<float*>(smem + T0 + 4 * TILE_BYTES);
  float* ldsD = ldsL + 2 * QT;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = (tid >> 6) % KW;                    // which 32 keys
  const int grp = G > 1 ? __builtin_amdgcn_readfirstlane(tid / (64 * KW)) : 0;   // which 32-query blocks
  const int r = lane & 15, g = lane >> 4;

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
  constexpr int NKC = D / 32;                          // 32-column blocks of a row
  constexpr int NDT = D / 16 / DS;                     // 16-column tiles of dK / dV this work-group owns
  const int wg_all = logical_wg(ord, blockIdx.x, gridDim.x);
  const int dt0 = (DS > 1) ? (wg_all % DS) * NDT : 0;  // first of them
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
  TileFrags fo;
  init_tile_frags(fo, lane, lds_address(smem));
  int v_row = fo.row;                                  // V_j fragments of this wave's keys
  if (kVInLds<D>) v_row += 2 * wave * kRowBlockBytes<D>;
  if (G > 1) {
    fo.row += 4 * grp * GT;
    fo.col[0] += 4 * grp * GT;
    fo.col[1] += 4 * grp * GT;
  }
  if (DS > 1) {                                        // update products: columns from tile dt0 on (an even one)
    fo.col[0] += 512 * dt0;
    fo.col[1] += 512 * dt0;
  }
  // D = 256: the dO buffers lie beyond the 64 KB that the immediate offset of an LDS read reaches, and have base registers of
  // their own (one addition per read otherwise, which counts where a SIMD has one wave).
  constexpr int FAR = 4 * GT > 65536 ? 2 * GT : 0;
  TileFrags fo_dO = fo;
  if (FAR) {
    fo_dO.row += FAR;
    fo_dO.col[0] += FAR;
    fo_dO.col[1] += FAR;
    asm volatile("" : "+v"(fo_dO.row), "+v"(fo_dO.col[0]), "+v"(fo_dO.col[1]));
  }
  // Group g reads the g-th 32 rows of a tile, which are the rows that its own waves fetch.  Its four buffers lie next
  // to one another (tiles as a whole would not), within the 64 KB that the immediate offset of an LDS read reaches:
  // one base register for all of them, which is what leaves the registers for the stream of qblocks below at D = 128 (with
  // whole tiles it spills 33 to 55, now three to nine, outside the loop).  us, whole tiles and phase after phase -> now, same
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
  // 39.0 -> 34.5, N1024 37.1 -> 36.2, B4 H32 N4000 526 -> 512.  (Elsewhere it costs 2 %, also at D = 128, where it takes away the
  // few spills outside the tile loop: B4 H32 N4096 causal 900 -> 933.)
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
    int kw = k0 + 32 * (FORM_LATE ? (late(tid) >> 6) % KW : wave);
    // (in a vector register: behind a branch that the compiler knows to be uniform it spills hundreds)
    if (KW == 1) asm volatile("" : "+v"(kw));

    if constexpr (kVInLds<D>) {
      TileLoader<D, KEYS, KW * G> v_loader;
      v_loader.init(tid, sn);
      v_loader.template load_rows<RAGGED>(smem, V + head_off, k0, NK);
    }
    // K_j^T / V_j^T fragments (B operands): lane (r, g) holds K[kw + 16n + r][32kc + 8g .. +7], n = 0, 1
    // (keys past the sequence end read the last row; their gradients are not stored)
    const int gk = late(g);
    bf16x8 kf[2][NKC], vf[2][kVInLds<D> ? 1 : NKC];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const int keyc = RAGGED ? min(kw + 16 * n + r, NK - 1) : kw + 16 * n + r;
#pragma unroll
      for (int kc = 0; kc < NKC; ++kc) {
        kf[n][kc] = *reinterpret_cast<const bf16x8*>(K + head_off + (size_t)keyc * sn + 32 * kc + 8 * gk);
        if constexpr (!kVInLds<D>) vf[n][kc] = *reinterpret_cast<const bf16x8*>(V + head_off + (size_t)keyc * sn + 32 * kc + 8 * gk);
      }
    }
    f32x4 dVt[NDT][2], dKt[NDT][2];
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int n = 0; n < 2; ++n) dVt[dt][n] = dKt[dt][n] = f32x4{0.f, 0.f, 0.f, 0.f};

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
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int kc = 0; kc < NKC; ++kc) {
        settle(kf[n][kc]);
        if constexpr (!kVInLds<D>) settle(vf[n][kc]);
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
      constexpr int tdO = T0 + (2 + buf) * GT - FAR;       // (from fo_dO)
      const float* tL = ldsL + buf * QT;
      const float* tD = ldsD + buf * QT;
      const int qt0 = t * QT;
      // The NB 32-query blocks of a tile that belong to this wave's group against its 32 keys, as one stream of matrix
      // instructions ("slots"):  S (D/16 slots) | dP | dV (NDT) | dK, block after block.  The vector work of a
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
        constexpr int NS = D / 16, NU = NDT, PB = 2 * NS + 2 * NU;        // slots of S or dP, of dV or dK, of a block
        constexpr int AHEAD = MASKED && DENSE ? 1 : kReadAhead<D, FORM, CAUSAL, DENSE>;       // (1: two would spill)
        // PAIRED: reads are issued two at a time, the later one first, so that one wait serves two slots.  Pays for the one wave
        // of a SIMD at D = 256: B2 H8 N2048 causal 97.2 -> 95.3 us, B1 H8 90.7 -> 89.2; at smaller D even, or to 2 % slower.
        constexpr bool PAIRED = D == 256;
        static_assert(!PAIRED || AHEAD % 2 == 0, "pairs");
        constexpr int RING = AHEAD + (PAIRED ? 2 : 1);
        // S and dP: slot u is the 16-query tile u % 2 against 32-column block u / 2; dV and dK: column tile u
        auto fragment = [&](int i) -> bf16x8 {
          const int b = qb + i / PB, u = i % PB;
          if (u < 2 * NS) return lds_row16<D>(u < NS ? tQ : tdO, u < NS ? fo : fo_dO, 32 * b + 16 * (u % 2), u % NS / 2);
          return lds_col16<D>(u < 2 * NS + NU ? tdO : tQ, u < 2 * NS + NU ? fo_dO : fo, 32 * b, (u - 2 * NS) % NU);
        };
        auto v_fragment = [&](int n, int kc) -> bf16x8 {     // kVInLds: V_j's
          TileFrags at;
          at.row = v_row;
          return lds_row16<D>(0, at, 16 * n, kc);
        };
        bf16x8 ring[RING], v_ring[2][2];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) ring[PAIRED ? i ^ 1 : i] = fragment(PAIRED ? i ^ 1 : i);
        f32x4 s[2][2], dp[2][2];         // [16-query tile][16-key tile]
        f32x4 l4[2];
        bf16x8 pf[2], dsf[2];
        int first_seen = 0;              // MASKED: entry 16m + i of 16-key tile n counts if 16 (m - n) + i >= first_seen
        static_for<NB * PB>([&](auto slot) {
          constexpr int sl = decltype(slot)::value, u = sl % PB, b = qb + sl / PB;
          const int stat = 32 * (b + grp) + 4 * g;
          if (PAIRED) {
            if (sl % 2 == 0 && sl + AHEAD < NB * PB) {
              ring[(sl + AHEAD + 1) % RING] = fragment(sl + AHEAD + 1);
              ring[(sl + AHEAD) % RING] = fragment(sl + AHEAD);
            }
          } else if (sl + AHEAD < NB * PB) ring[(sl + AHEAD) % RING] = fragment(sl + AHEAD);
          if constexpr (kVInLds<D>) {      // two slots ahead of their use
            constexpr int uv = u + 2 - NS;
            if constexpr (uv >= 0 && uv < NS) v_ring[uv % 2][uv / 2 % 2] = v_fragment(uv % 2, uv / 2);
          }
          if (u == 0) {
#pragma unroll
            for (int n = 0; n < 2; ++n) s[0][n] = s[1][n] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (MASKED) {
              int ln = lane;
              constexpr bool LATE = DENSE || kVInLds<D>;         // formed here, not ahead of the tile loop: registers
              if (LATE) asm volatile("" : "+v"(ln));
              first_seen = (LATE ? __builtin_amdgcn_readfirstlane(kw) : kw) + (ln & 15) - shift - qt0 - 32 * (b + grp) - 4 * (ln >> 4);
            }
          }
          // -delta_i seeds the dP accumulator; L_i of the rows a lane sees
#pragma unroll
          for (int m = 0; m < 2; ++m)
            if (u == m * NS / 2) {
              const f32x4 d4 = *reinterpret_cast<const f32x4*>(tD + stat + 16 * m);
              dp[m][0] = dp[m][1] = d4;
            }
#pragma unroll
          for (int m = 0; m < 2; ++m)
            if (u == NS / 2 + m * NS / 2) l4[m] = *reinterpret_cast<const f32x4*>(tL + stat + 16 * m);
          const bf16x8 a = ring[sl % RING];
#pragma unroll
          for (int n = 0; n < 2; ++n) {
            if constexpr (u < NS) {
              s[u % 2][n] = mfma16(a, kf[n][u / 2], s[u % 2][n]);
            } else if constexpr (u < 2 * NS) {
              constexpr int w = u - NS;
              if constexpr (kVInLds<D>) dp[w % 2][n] = mfma16(a, v_ring[n][w / 2 % 2], dp[w % 2][n]);
              else dp[w % 2][n] = mfma16(a, vf[n][w / 2], dp[w % 2][n]);
            } else if constexpr (u < 2 * NS + NU) {
              dVt[u - 2 * NS][n] = mfma16(a, pf[n], dVt[u - 2 * NS][n]);
            } else {
              dKt[u - 2 * NS - NU][n] = mfma16(a, dsf[n], dKt[u - 2 * NS - NU][n]);
            }
          }
          if (b == 0) issue_part(sl);
          // Entry e of a lane's 16: row (e & 3) of 16-query tile m = e / 8, 16-key tile n = (e >> 2) & 1.  Query tile by query
          // tile, so that L of one tile at a time is live (key tile by key tile the three-wave kernels spilled two registers, one
          // of them reloaded for every tile: 1120 heads N268 d64 causal 64.9 -> 60.9 us, B8 H12 N1000 35.2 -> 33.7).
          if constexpr (u >= NS && u < 2 * NS) {                  // P = exp(S - L) (step 9)
            constexpr int f = u - NS;
#pragma unroll
            for (int e = 16 * f / NS; e < 16 * (f + 1) / NS; ++e) {
              const int m = e >> 3, n = (e >> 2) & 1, i = e & 3;
              float x = __builtin_fmaf(s[m][n][i], c2, -l4[m][i]);
              if (MASKED && 16 * (m - n) + i < first_seen) x = -INFINITY;
              s[m][n][i] = __builtin_amdgcn_exp2f(x);
              pf[n][4 * m + i] = (bf16_t)s[m][n][i];
            }
          }
          if constexpr (u >= 2 * NS && u < 2 * NS + NU) {         // dS = P o (dP - delta) (step 12); dp already holds dP - delta
            constexpr int f = u - 2 * NS;
#pragma unroll
            for (int e = 16 * f / NU; e < 16 * (f + 1) / NU; ++e) {
              const int m = e >> 3, n = (e >> 2) & 1, i = e & 3;
              float ds = s[m][n][i] * dp[m][n][i];
              // a masked entry contributes exactly nothing, whatever its row holds
              if (MASKED && 16 * (m - n) + i < first_seen) ds = 0.f;
              if (MASKED) asm("" : "+v"(ds));      // (the compiler would convert first and select 16 bits at a time)
              dsf[n][4 * m + i] = (bf16_t)ds;
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
    auto rounded = [&](const f32x4 (&acc)[NDT][2], float scale) {
      return [&acc, scale](int dt, int n) {
        bf16x4 o4;
#pragma unroll
        for (int e = 0; e < 4; ++e) o4[e] = (bf16_t)(acc[dt][n][e] * scale);
        return o4;
      };
    };
    if constexpr (G > 1) {
      // The groups add their partial sums: group 1 hands over its dV, group 0 its dK, each through an
      // area of its own per wave (16 bytes per lane, lanes consecutive), and group 0 finishes dV,
      // group 1 dK; before that the upper half of the groups hands both over to the lower half, until two are left.  Every wave is past
      // the last tile's barrier: the whole array is free.
      // (the lane index passes through an empty asm: addresses formed from the kernel's own copy would
      // be hoisted above the tile loop and held in registers through it)
      constexpr int AREA = NDT * 2048;
      int ln = lane;
      asm volatile("" : "+v"(ln));
      auto put = [&](const f32x4 (&acc)[NDT][2], char* give) {
#pragma unroll
        for (int i = 0; i < 2 * NDT; ++i) *reinterpret_cast<f32x4*>(give + (i * 64 + ln) * 16) = acc[i >> 1][i & 1];
      };
      auto add = [&](f32x4 (&acc)[NDT][2], const char* take) {
#pragma unroll
        for (int i = 0; i < 2 * NDT; ++i) acc[i >> 1][i & 1] += *reinterpret_cast<const f32x4*>(take + (i * 64 + ln) * 16);
      };
#pragma unroll
      for (int half = G / 2; half >= 2; half >>= 1) {
        char* area = smem + ((grp % half) * KW + wave) * 2 * AREA;
        if (grp >= half && grp < 2 * half) { put(dVt, area); put(dKt, area + AREA); }
        __syncthreads();
        if (grp < half) { add(dVt, area); add(dKt, area + AREA); }
        __syncthreads();
      }
      char* give = smem + (grp * KW + wave) * AREA;
      char* take = smem + ((grp ^ 1) * KW + wave) * AREA;
      // one output per group; the wave's `take` area, read out by then, serves as its staging area
      auto finish = [&](f32x4 (&acc)[NDT][2], float scale, bf16_t* out) {
        add(acc, take);
        bf16_t* dst = out + head_off + (size_t)kw * sn;
        if constexpr (kStagedDkDv<D>) store_rows16_staged<NDT>(take, rounded(acc, scale), dst, sn, rows_valid, ln);
        else store_rows16<NDT>(rounded(acc, scale), dst, sn, rows_valid, ln);
      };
      if (grp == 0) put(dKt, give); else if (grp == 1) put(dVt, give);
      __syncthreads();
      if (grp == 0) finish(dVt, 1.0f, dV); else if (grp == 1) finish(dKt, alpha, dK);
    } else {
      const size_t at = 16 * dt0 + head_off + (size_t)kw * sn;
      if constexpr (kStagedDkDv<D>) {
        char* stage = smem + T0 + (kStageOverTiles<D, G> ? 0 : 4 * TILE_BYTES + 4 * QT * (int)sizeof(float));
        store_rows16_staged<NDT>(stage, rounded(dVt, 1.0f), dV + at, sn, rows_valid, tid);
        store_rows16_staged<NDT>(stage, rounded(dKt, alpha), dK + at, sn, rows_valid, tid);
      } else {
        store_rows16<NDT>(rounded(dVt, 1.0f), dV + at, sn, rows_valid, lane);
        store_rows16<NDT>(rounded(dKt, alpha), dK + at, sn, rows_valid, lane);
      }
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
template <int FORM> constexpr int kQueryWaves = FORM == 1 ? 4 : FORM == 8 || FORM == kNarrow ? 1 : 2;
template <int FORM> constexpr int kKeysPerTile = FORM >= 4 ? 32 * kGroups<FORM> : 64;
template <int D, int G> constexpr int kSmemDq = 4 * kKeysPerTile<G> * D * 2;
// Small head sizes need more waves per SIMD next to one another (four at D = 32, three at D = 64) than a long
// read-ahead: dQ at D = 64 with two waves and fragments read four slots ahead -> three and two (us): B8 H12 N1024
// causal 33.1 -> 30.9, B4 H32 N4096 causal 395 -> 379, B16 H16 N999 full 114 -> 109.
template <int D, int G> constexpr int kDqWavesPerSimd = D == 32 && G == 1 ? 4 : D == 64 && G == 1 ? 3 : kWavesPerSimd<D>;
template <int D> constexpr int kReadAheadDq = D <= 64 ? 2 : D == 256 ? 6 : 4;

template <int D, bool CAUSAL, bool RAGGED, int MODE, int FORM>
__global__ __launch_bounds__(64 * kQueryWaves<FORM> * kGroups<FORM>)
__attribute__((amdgpu_waves_per_eu(kDqWavesPerSimd<D, FORM>))) void attn_bwd_dq_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    const bf16_t* __restrict__ dO, const float* __restrict__ LSE, const float* __restrict__ delta,
    const bf16_t* __restrict__ O, bf16_t* __restrict__ dQ, float* __restrict__ delta_out, int N,
    float alpha, Layout lay, int pairs, BlockOrder ord) {
  constexpr bool DELTA_MODE = MODE == kRecomputeDelta;
  constexpr int G = kGroups<FORM>, QW = kQueryWaves<FORM>, QUERIES = 32 * QW, KT = kKeysPerTile<FORM>;
  constexpr int TILE_BYTES = KT * D * 2;
  constexpr int NKC = D / 32, NDT = D / 16;            // 32-column blocks of a row, 16-column tiles of dQ
  extern __shared__ __attribute__((aligned(16))) char smem[];
  char* ldsK = smem;
  char* ldsV = smem + 2 * TILE_BYTES;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = (tid >> 6) % QW;                   // which 32 queries
  const int grp = G > 1 ? __builtin_amdgcn_readfirstlane(tid / (64 * QW)) : 0;   // which 32-key blocks
  const int r = lane & 15, g = lane >> 4;

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
  TileFrags fo;
  init_tile_frags(fo, lane, lds_address(smem));
  if (G > 1) {                                        // a group reads its own 32 rows of a tile
    fo.row += 2 * grp * kRowBlockBytes<D>;
    fo.col[0] += 2 * grp * kRowBlockBytes<D>;
    fo.col[1] += 2 * grp * kRowBlockBytes<D>;
  }
  constexpr int FAR = 4 * TILE_BYTES > 65536 ? 2 * TILE_BYTES : 0;      // see the dK/dV kernel
  TileFrags fo_v = fo;
  if (FAR) {
    fo_v.row += FAR;
    asm volatile("" : "+v"(fo_v.row));
  }

  for (int part = 0; part < (pairs ? 2 : 1); ++part) {
  if (part > 0) __syncthreads();                      // the first block's output staging is done with the tile buffers
  const int qt = pairs ? (part == 0 ? nqt - 1 - idx : idx)
                       : nqt - 1 - (idx + (CAUSAL && ord.n == 0 ? small_grid_rotation(bh, nqt, gridDim.x, D == 128 ? 768 : 1152) : 0)) % nqt;
  if (part == 1 && qt == nqt - 1 - idx) break;        // odd number of blocks: the middle one has no partner
  const int q0 = qt * QUERIES;
  const int qw = q0 + 32 * wave;

  // Q_i^T / dO_i^T fragments (B operands): lane (r, g) holds Q[qw + 16n + r][32kc + 8g .. +7], n = 0, 1
  // (rows past the sequence end read the last row; their dQ is not stored)
  bf16x8 qf[2][NKC], dof[2][NKC];
  int qc[2];
  float l2[2], dl[2] = {0.f, 0.f};
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    qc[n] = RAGGED ? min(qw + 16 * n + r, N - 1) : qw + 16 * n + r;
    const size_t at = head_off + (size_t)qc[n] * sn + 8 * g;
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) {
      qf[n][kc] = *reinterpret_cast<const bf16x8*>(Q + at + 32 * kc);
      dof[n][kc] = *reinterpret_cast<const bf16x8*>(dO + at + 32 * kc);
    }
    l2[n] = LSE[(size_t)bh * N + qc[n]] * kLog2e;
    if (RAGGED && l2[n] == -INFINITY) l2[n] = 0.f;       // a query that sees no key: all its scores are masked below
    if (MODE == kGivenDelta) dl[n] = delta[(size_t)bh * N + qc[n]];
  }
  if (MODE == kOwnDelta) {
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      // this lane holds chunks 4kc + g of its row: the chains of its chunks, the tree levels that stay inside one
      // residue class, and the last two levels across the four lanes of the row
      constexpr int NCS = kPow2D<D> / 32;     // D = 96: the tree of a 128-wide row whose last chunks are zero
      float cs[NCS];
#pragma unroll
      for (int kc = 0; kc < NCS; ++kc) cs[kc] = 0.f;
#pragma unroll
      for (int kc = 0; kc < NKC; ++kc) {
        const bf16x8 o8 = *reinterpret_cast<const bf16x8*>(O + head_off + (size_t)qc[n] * sn + 32 * kc + 8 * g);
        float c = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) c = __builtin_fmaf((float)o8[e], (float)dof[n][kc][e], c);
        cs[kc] = c;
      }
#pragma unroll
      for (int off = NCS / 2; off >= 1; off >>= 1)
#pragma unroll
        for (int kc = 0; kc < off; ++kc) cs[kc] += cs[kc + off];
      dl[n] = sum_over_groups(cs[0]);
      if (g == 0 && grp == 0 && (!RAGGED || qw + 16 * n + r < N)) delta_out[(size_t)bh * N + qw + 16 * n + r] = dl[n];
    }
  }
  float pdp[2] = {0.f, 0.f};                         // DELTA_MODE: this lane's share of sum_k P dP
  // -delta_i in all accumulator slots of the lane: the third operand of the first dP^T matrix
  // instructions of every key block, which then deliver dP - delta with no vector instruction
  // (Alg. 2: dS = P o (dP - delta)).  Kept opaque so that it stays resident instead of being
  // rebuilt per block.
  f32x4 neg_delta[2];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
#pragma unroll
    for (int i = 0; i < 4; ++i) neg_delta[n][i] = -dl[n];
    asm volatile("" : "+v"(neg_delta[n]));
  }
  f32x4 dQt[NDT][2];
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int n = 0; n < 2; ++n) dQt[dt][n] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int kend = !CAUSAL ? NK : !RAGGED ? q0 + QUERIES : max(0, min(NK, q0 + QUERIES + shift));
  const int ntiles = RAGGED || KT > QUERIES ? (kend + KT - 1) / KT : kend / KT;

  loader.template load_rows<RAGGED>(ldsK, Kh, 0, NK);
  loader.template load_rows<RAGGED>(ldsV, Vh, 0, NK);
  wait_vmem();
#pragma unroll
  for (int n = 0; n < 2; ++n) {
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) { settle(qf[n][kc]); settle(dof[n][kc]); }
    settle(l2[n]);
  }
  __syncthreads();

  // One key tile; BUF (which LDS buffer holds it) is a compile-time constant so that every LDS
  // address is a precomputed per-lane offset plus an immediate.
  auto tile_step = [&](auto buf_c, int j) {
    constexpr int buf = decltype(buf_c)::value;
    constexpr int tK = buf * TILE_BYTES;            // byte offsets of this tile's K and V in smem
    constexpr int tV = (2 + buf) * TILE_BYTES - FAR;          // (from fo_v)
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
      constexpr bool HOLD = NB == 1 && !DELTA_MODE && (D <= 64 || (G > 1 && D <= 128));
      constexpr int NS = D / 16, READS = (DELTA_MODE ? 2 : 3) * NB * NS, SLOTS = READS + (HOLD ? NS : 0);
      constexpr int AHEAD = NB == 1 && D <= 64 ? 4 : kReadAheadDq<D>;
      // PAIRED: see the dK/dV kernel.  us: B4 H12 N1024 d64 causal 19.0 -> 18.5, B1 H4 N2048 d96 causal 19.4 -> 19.0; without wave
      // groups, and at D >= 128, even or slower (B1 H8 N2048 d256 causal 47.0 -> 48.2).
      constexpr bool PAIRED = G > 1 && D <= 96;
      static_assert(!PAIRED || AHEAD % 2 == 0, "pairs");
      constexpr int RING = AHEAD + (PAIRED ? 2 : 1);
      // phases of S^T and dP^T: slot u is the 16-key tile u % 2 against 32-column block u / 2; of dQ: column tile u
      auto fragment = [&](int i) -> bf16x8 {
        const int phase = i / NS, u = i % NS;
        if (phase < 2 * NB) return lds_row16<D>(phase % 2 ? tV : tK, phase % 2 ? fo_v : fo, 32 * (kb + phase / 2) + 16 * (u % 2), u / 2);
        return lds_col16<D>(tK, fo, 32 * (kb + phase - 2 * NB), u);
      };
      // HOLD: with one block to a tile, dS has no other block's products to lie under.  The dQ products of the first 16 queries
      // go first, with dS of the other 16 under them, and the fragments stay for those.  us: B1 H8 N2048 d64 causal 17.3 -> 16.9,
      // d128 27.0 -> 26.5, B1 H1 N5120 d64 32.0 -> 30.9.
      bf16x8 ring[RING], held[HOLD ? NS : 1], dsf[NB][2];
      auto read = [&](int i) {
        if (HOLD && i >= 2 * NS) held[HOLD ? i - 2 * NS : 0] = fragment(i);
        else ring[i % RING] = fragment(i);
      };
      f32x4 s[NB][2][2], dp[NB][2][2];   // [block][16-key tile][16-query tile]
      int lim[NB][2];                    // MASKED: last visible entry 16m + i of a 16-query tile
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) read(PAIRED ? i ^ 1 : i);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int kb0 = kt0 + 32 * (kb + b + grp);
        // (formed here and not ahead of the tile loop, which costs registers: at D = 64, causal, with bounds checks six were
        // spilled.  us: 800 heads N65 15.0 -> 13.2, 400 heads N200 19.8 -> 17.6, B8 H12 N1000 29.6 -> 28.0)
        int ln = lane;
        if (MASKED) asm volatile("" : "+v"(ln));
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          s[b][0][n] = s[b][1][n] = f32x4{0.f, 0.f, 0.f, 0.f};
          lim[b][n] = CAUSAL ? __builtin_amdgcn_readfirstlane(qw) + 16 * n + (ln & 15) + shift - kb0 - 4 * (ln >> 4) : 0x7fffffff;
          if (RAGGED) lim[b][n] = min(lim[b][n], NK - 1 - kb0 - 4 * (ln >> 4));
        }
      }
      // P of entries e0 .. e1 - 1 of a lane's 16 of block b (entry e: row (e & 3) of 16-key tile m = e / 8, 16-query tile
      // n = (e >> 2) & 1): keys in this lane's future and keys past the sequence end get S = -inf, P = exp(-inf) = 0
      auto form_p = [&](int b, int e0, int e1) {
#pragma unroll
        for (int e = e0; e < e1; ++e) {
          const int m = e >> 3, n = (e >> 2) & 1, i = e & 3;
          if (MASKED && 16 * m + i > lim[b][n]) s[b][m][n][i] = -INFINITY;
          s[b][m][n][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[b][m][n][i], c2, -l2[n]));
        }
      };
      // dS of the same (of one block, query tile by query tile: see HOLD); dp already holds dP - delta
      auto form_ds = [&](int b, int e0, int e1) {
#pragma unroll
        for (int e = e0; e < e1; ++e) {
          const int m = NB > 1 ? e >> 3 : (e >> 2) & 1, n = NB > 1 ? (e >> 2) & 1 : e >> 3, i = e & 3;
          if (DELTA_MODE) pdp[n] = __builtin_fmaf(s[b][m][n][i], dp[b][m][n][i], pdp[n]);
          else dsf[b][n][4 * m + i] = (bf16_t)(s[b][m][n][i] * dp[b][m][n][i]);
        }
      };
      static_for<SLOTS>([&](auto slot) {
        constexpr int sl = decltype(slot)::value, phase = sl / NS, u = sl % NS;
        if (PAIRED) {
          if (sl % 2 == 0 && sl + AHEAD < READS) {
            read(sl + AHEAD + 1);
            read(sl + AHEAD);
          }
        } else if (sl + AHEAD < READS) read(sl + AHEAD);
        const bf16x8 a = HOLD && phase >= 2 ? held[HOLD ? u : 0] : ring[sl % RING];
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          if (HOLD && phase >= 2 && n != phase - 2) continue;
          if (NB == 1 && sl == 2 * NS) form_ds(0, 8 * n, 8 * n + 8);
          if constexpr (phase >= 2 * NB) dQt[u][n] = mfma16(a, dsf[HOLD ? 0 : phase - 2 * NB][n], dQt[u][n]);   // step 13
          else if constexpr (phase % 2 == 0) s[phase / 2][u % 2][n] = mfma16(a, qf[n][u / 2], s[phase / 2][u % 2][n]);
          else dp[phase / 2][u % 2][n] = mfma16(a, dof[n][u / 2], u < 2 ? neg_delta[n] : dp[phase / 2][u % 2][n]);
        }
        // (One transfer instruction per two slots at D = 256: four waves that issue one each per slot ask for 128 bytes a clock
        // where the load path takes 64, and stall.  us, one slot -> two: B1 H8 N2048 d256 full 59.0 -> 57.4, causal 51.0 -> 47.5.
        // d <= 128: even, and 0.1 to 0.2 us slower where a problem is one tile long, as the transfer ends later.)
        constexpr int EVERY = D == 256 ? 2 : 1;
        static_assert(2 * NLD * EVERY <= 2 * NS, "all of the transfer is issued under S and dP");
        if (kb == 0 && sl % EVERY == 0) issue_part(sl / EVERY);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          // P of block b lies under its dP^T, dS under the phase after; both are whole when the phase ends
          const int e = sl - 2 * NS * b - NS, f = e - NS;
          if (e >= 0 && e < NS) form_p(b, 16 * e / NS, 16 * (e + 1) / NS);
          if (HOLD && phase == 2) form_ds(0, 8 + 8 * u / NS, 8 + 8 * (u + 1) / NS);
          if (NB > 1 && !DELTA_MODE && f >= 0 && f < NS) form_ds(b, 16 * f / NS, 16 * (f + 1) / NS);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      if (DELTA_MODE) {
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
      static_for<NBT / NB>([&](auto i) {
        kblocks(std::false_type{}, std::integral_constant<int, NB>{}, std::integral_constant<int, NB * decltype(i)::value>{});
      });
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
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const float dsum = sum_over_groups(pdp[n]);    // the other three lanes of a row hold the other keys of every block
      if (g == 0 && (!RAGGED || qw + 16 * n + r < N)) delta_out[(size_t)bh * N + qw + 16 * n + r] = dsum;
    }
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
        char* area = smem + ((grp % half) * QW + wave) * (NDT * 2048);
        if (grp >= half) {
#pragma unroll
          for (int i = 0; i < 2 * NDT; ++i) *reinterpret_cast<f32x4*>(area + (i * 64 + ln) * 16) = dQt[i >> 1][i & 1];
        }
      }
      __syncthreads();
      if (grp < half) {
        const char* area = smem + (grp * QW + wave) * (NDT * 2048);
#pragma unroll
        for (int i = 0; i < 2 * NDT; ++i) dQt[i >> 1][i & 1] += *reinterpret_cast<const f32x4*>(area + (i * 64 + ln) * 16);
      }
      __syncthreads();
    }
    if (grp != 0) continue;
  }
  auto piece = [&](int dt, int n) {
    bf16x4 o4;
#pragma unroll
    for (int e = 0; e < 4; ++e) o4[e] = (bf16_t)(dQt[dt][n][e] * alpha);
    return o4;
  };
  bf16_t* dst = dQ + head_off + (size_t)qw * sn;
  // the tile buffers are free now (every wave is past the last tile's barrier): they serve as
  // the staging areas of store_rows16_staged; the barrier at the top of the part loop keeps the
  // next block's tile transfers from overwriting an area a slower wave is still reading
  if constexpr (kCanStage<D / 32>) store_rows16_staged<NDT>(smem, piece, dst, sn, RAGGED ? N - qw : 32, tid);
  else store_rows16<NDT>(piece, dst, sn, RAGGED ? N - qw : 32, lane);
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
  constexpr int KEYS = 32 * kKeyWaves<G>, THREADS = 64 * kKeyWaves<G> * kGroups<G>;
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

// calls f(integral_constant<FORM>) for every form
template <class F> static void each_form(F&& f) {
  f(std::integral_constant<int, 1>{}); f(std::integral_constant<int, 2>{}); f(std::integral_constant<int, 4>{}); f(std::integral_constant<int, 8>{});
  f(std::integral_constant<int, kNarrow>{}); f(std::integral_constant<int, kHalf>{}); f(std::integral_constant<int, kDense>{});
}

template <int D, bool CAUSAL, bool RAGGED, bool GROUPED>
static hipError_t launch_dkdv(const void* Q, const void* K, const void* V, const void* dO,
                              const float* LSE, const float* delta, void* dK, void* dV, int BH,
                              int N, float alpha, Layout lay, hipStream_t st) {
  const int form = dkdv_form(D, CAUSAL, GROUPED, BH / lay.group, RAGGED ? lay.Nk : N);
  hipError_t e = hipErrorInvalidValue;
  each_form([&](auto f) {
    constexpr int ANY = decltype(f)::value, FORM = ANY == kDense ? 1 : ANY;
    constexpr bool DENSE = ANY == kDense || (ANY == kHalf && D <= 64);      // three waves per SIMD
    if constexpr (dkdv_has_form(D, CAUSAL, GROUPED, ANY))
      if (form == ANY)       // (the aligned kernels want whole tiles)
        e = RAGGED || N % kQTile<D, FORM> != 0
                ? launch_dkdv_g<D, CAUSAL, true, GROUPED, FORM, DENSE>(Q, K, V, dO, LSE, delta, dK, dV, BH, N, alpha, lay, st)
                : launch_dkdv_g<D, CAUSAL, RAGGED, GROUPED, FORM, DENSE>(Q, K, V, dO, LSE, delta, dK, dV, BH, N, alpha, lay, st);
  });
  return e;
}

template <int D, bool CAUSAL, bool RAGGED, int MODE, int G>
static hipError_t launch_dq_g(const void* Q, const void* K, const void* V, const void* dO,
                              const float* LSE, const float* delta, const void* O, void* dQ,
                              float* delta_out, int BH, int N, float alpha, Layout lay, hipStream_t st) {
  constexpr int smem = kSmemDq<D, G>;
  constexpr int QUERIES = 32 * kQueryWaves<G>, THREADS = 64 * kQueryWaves<G> * kGroups<G>;
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
  const int form = MODE == kRecomputeDelta ? 1 : dq_form(D, CAUSAL, BH, N, RAGGED ? lay.Nk : N);
  hipError_t e = hipErrorInvalidValue;
  each_form([&](auto f) {
    constexpr int FORM = decltype(f)::value;
    // At D = 256 without a mask the bounds-checking kernels serve aligned sizes too (attn_bwd_dq_dispatch), but for two groups, where
    // the aligned one is the faster and spills nothing: us, bounds-checking -> aligned: B1 H8 N2048 57.4 -> 56.2, B1 H4 N4096
    // 100.7 -> 98.5, B1 H8 N512 20.8 -> 20.0.
    constexpr bool ALIGNED_256 = D == 256 && !CAUSAL && FORM == 2;
    if constexpr (dq_has_form(D, FORM) && (MODE != kRecomputeDelta || FORM == 1)) {
      if (form != FORM) return;
      const bool aligned = ALIGNED_256 ? lay.Nk == N && N % kQPerWG == 0 : !RAGGED && N % kKeysPerTile<FORM> == 0;
      e = aligned ? launch_dq_g<D, CAUSAL, RAGGED && !ALIGNED_256, MODE, FORM>(Q, K, V, dO, LSE, delta, O, dQ, delta_out, BH, N, alpha, lay, st)
                  : launch_dq_g<D, CAUSAL, true, MODE, FORM>(Q, K, V, dO, LSE, delta, O, dQ, delta_out, BH, N, alpha, lay, st);
    }
  });
  return e;
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

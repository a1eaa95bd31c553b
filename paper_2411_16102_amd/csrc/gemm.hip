// bf16 "NT" GEMM  C[M,N] = A[M,K] * B[N,K]^T  for gfx950, fp32 accumulation on
// v_mfma_f32_16x16x32_bf16, tiles staged through LDS, fused epilogues.  (The chip lowers its
// clock under matrix load; at that limit the 16x16x32 shape, which moves fewer accumulator
// registers per flop, sustains 1.87 PFLOP/s on random operands where 32x32x16 sustains
// 1.7, and this kernel gained 10 to 24 % from the change.)
//
// Operand roles are swapped with respect to the usual picture: the weight rows
// feed the MFMA "A" operand and the activation rows the "B" operand, so an
// accumulator block holds C^T: a lane owns ONE activation row (m = lane % 16) and
// a run of four consecutive output features (n = 4 * (lane / 16) ..).  Every fused epilogue is then
// lane-local: the RMSNorm factor of a row is one scalar per lane, a RoPE pair
// (i, i + dh/2) and a SwiGLU (gate, up) pair sit in two accumulator blocks of the
// same lane; all but gate/up then turn round in LDS on their way out.
//
// Tiles travel global -> LDS directly (global_load_lds_dwordx4), so no VGPRs are spent
// on staging.  A k-tile is BK = 64 wide: a tile row is then one whole 128-byte cache
// line, which the memory pipeline delivers about 1.5 times faster than the two 64-byte
// halves fetched separately (measured: 41 against 26 B/clk/CU into LDS).  LDS holds two
// rings of panels, three weight panels and two activation panels of one k-tile each for a 256x256
// tile: while tile kt is multiplied, tile kt+1 has landed or is landing and the weight panel of
// tile kt+2 is in flight; 160x256 and 128x256 tiles have room for a third activation panel.
// (Of at most 256 rows, what the few-row kernel leaves, gate/up and plain products and the
// k-ranges of the others, uses a second pipeline where it pays, DEEP in the kernel below: one row
// of tiles, a few slots for the activation panel and all other LDS for the weight
// panel, the two kinds of panel requested by different wavefronts.)  Rows are 128 B whose eight 16-byte chunks are XOR-swizzled with
// ((row >> 1) & 7): two consecutive rows fill the 256-byte bank row, so the swizzle
// must change every two rows for the ds_read_b128 of a fragment (16 rows by four chunk
// columns) to be conflict-free.  Waits on the LDS-DMA loads are placed by hand
// (s_waitcnt vmcnt + s_barrier); the compiler does not track them.
#include <algorithm>
#include <numeric>
#include <utility>
#include "gemm.hpp"
#include "attn_device.hpp"
#include "k_order.hpp"
#include "common.hpp"

namespace bs {

// sixteen bytes of zeros: the source of tile chunks that lie beyond K
__device__ __align__(16) uint16_t g_gemm_zero_chunk[8];

namespace {

constexpr int BK = K_TILE;  // k-extent of one k-tile: rows of 128 bytes
constexpr int LDS_CU = 160 * 1024;
// the panel ring of a workgroup: all of a CU's LDS, or half where two workgroups of four wavefronts share a CU; three
// weight panels, as many activation panels as fit beside them (three are enough), and what is left to weights again
constexpr int ring_bytes(int waves) { return waves > 4 ? LDS_CU : LDS_CU / 2; }
constexpr int ring_x_slots(int bm, int bn, int waves) {
  const int n = (ring_bytes(waves) - 3 * bn * BK * 2) / (bm * BK * 2);
  return n < 3 ? n : 3;
}
constexpr int ring_w_slots(int bm, int bn, int waves) { return (ring_bytes(waves) - ring_x_slots(bm, bn, waves) * bm * BK * 2) / (bn * BK * 2); }
constexpr int XCDS = 8;

struct TileCoord { int tm, tn; };
struct Yes { static constexpr bool value = true; };
struct No { static constexpr bool value = false; };

// Workgroup ids are dealt round-robin to the 8 XCDs; give each XCD a contiguous
// range of tiles and walk that range in groups of GM tile rows, so the tiles in
// flight on one XCD share activation and weight panels in that XCD's L2.
__device__ __forceinline__ TileCoord map_tile(int pid, int n_tiles, int tiles_m, int tiles_n) {
  const int per = n_tiles / XCDS, rem = n_tiles % XCDS;
  const int xcd = pid % XCDS, idx = pid / XCDS;
  const int lin = xcd * per + (xcd < rem ? xcd : rem) + idx;
  constexpr int GM = 4;
  const int group = GM * tiles_n;
  const int g = lin / group;
  const int first_m = g * GM;
  const int gm = (tiles_m - first_m) < GM ? (tiles_m - first_m) : GM;
  const int in = lin - g * group;
  TileCoord t;
  t.tm = first_m + in % gm;
  t.tn = in / gm;
  return t;
}

__device__ __forceinline__ void store_bf16x4(uint16_t *p, float a, float b, float c, float d) {
  u32x2_t v;
  v.x = pack_bf16x2(a, b);
  v.y = pack_bf16x2(c, d);
  *reinterpret_cast<u32x2_t *>(p) = v;
}

// Columns of the fused projection enter the tiles in groups of 64: 32 features of a head and those dh/2 behind them, so
// that rotation pairs meet in a lane.  Groups of value heads are dealt evenly between the others: the rows of
// decode sequences store them two bytes at a time, one lane per clock, 28 us for a 256x256 tile of nothing else
// (QKV of 1093 prefill and 487 decode rows 111 -> 106 us against the columns in their own order).
struct QkvGroup { int head, i0; };  // features i0 .. i0 + 31 and i0 + dh/2 .. of the head; head >= all of them: beyond the last
__device__ __forceinline__ QkvGroup qkv_group(int p, const GemmArgs &a, int dh) {
  const int per_head = dh / 64, n_v = a.n_kv_heads * per_head, n_rot = (a.n_q_heads + a.n_kv_heads) * per_head, n = n_rot + n_v;
  const int v = (int)((unsigned)(p * n_v) / (unsigned)n);
  const int g = p >= n ? n : (int)((unsigned)((p + 1) * n_v) / (unsigned)n) > v ? n_rot + v : p - v;
  return QkvGroup{g / per_head, g % per_head * 32};
}

// s_waitcnt immediate (gfx9 encoding): wait until at most `vm` vector-memory
// operations are outstanding and, if lgkm0, until all LDS reads have returned
constexpr int waitcnt_imm(int vm, bool lgkm0) {
  return (vm & 0xF) | ((vm >> 4) << 14) | 0x70 | (lgkm0 ? 0 : 0xF00);
}

// Shared tiles.  A launch of G persistent workgroups takes the tiles [0, n_dp) of the launch's
// tile order whole, workgroup w the tiles w, w + G, ...; the k-tiles of the other n_sk tiles
// form one line of n_sk * nk iterations that the first g_sk workgroups cut into equal
// consecutive ranges, so a tile at a cut is computed by two or more workgroups, each over a
// part of K.  Every such workgroup leaves its partial tile in the workspace and counts itself
// in; the one that arrives last adds the parts up (always in the order of their k-ranges,
// its own part re-read like the others, so the sum does not depend on who was last) and runs
// the epilogue.  Nobody waits for anybody.
struct SkPlan {
  int n_dp, n_sk, g_sk, nk;
  float *ws;      // [2 * G][BM * BN]: slot 2 w of workgroup w for its first segment, 2 w + 1 for its last
  unsigned *cnt;  // [n_sk] arrivals at each shared tile; zero between launches
};
struct SkSeg {
  int pid, kt0, kt1;  // tile, k-tiles [kt0, kt1)
  int j;              // index of the tile among the shared ones
  int parts;          // workgroups that hold a part of the tile (1: this one has all of it)
  int w_first;        // the first of them; they are consecutive
  int my_slot;
};
constexpr int SK_SNAP = 4;      // a cut this close to a tile boundary moves onto it
constexpr int SK_MIN_ITERS = 16;  // shortest range worth a workgroup of its own

// first iteration of workgroup w's range (w = g_sk: the end of the line)
__device__ __forceinline__ int sk_bound(const SkPlan &p, int w) {
  const int total = p.n_sk * p.nk;
  int b = (int)((long)total * w / p.g_sk);
  const int r = b % p.nk;
  if (r < SK_SNAP) b -= r;
  else if (p.nk - r < SK_SNAP) b += p.nk - r;
  return b;
}
// the workgroups whose ranges meet shared tile j
__device__ __forceinline__ void sk_tile_span(const SkPlan &p, int j, int *w_first, int *parts) {
  const int lo = j * p.nk, hi = lo + p.nk;
  int w = (int)((long)lo * p.g_sk / (p.n_sk * p.nk));
  while (w + 1 < p.g_sk && sk_bound(p, w + 1) <= lo) ++w;
  while (w > 0 && sk_bound(p, w) > lo) --w;
  int n = 1;
  while (w + n < p.g_sk && sk_bound(p, w + n) < hi) ++n;
  *w_first = w;
  *parts = n;
}

// One workgroup's tile; `bid` is the workgroup's number among the GEMM workgroups of the launch
// (SK: the tile and the k-range come from `seg` instead).
template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int DH, int DEEP = 0, bool SK = false>
__device__ __forceinline__ void gemm_tile(const GemmArgs &a, const int bid, const SkPlan *sp = nullptr, const SkSeg seg = SkSeg{}) {
  static_assert(!SK || (!DEEP && EPI != EPI_PARTIAL), "shared tiles use the two rings of whole tiles and a real epilogue");
  constexpr int NW = WAVES_M * WAVES_N;
  // DEEP: the pipeline for one round of tiles over few rows, where every CU streams a weight
  // panel of its own from HBM; the first half of the wavefronts requests the activation
  // panels, the second half the weight panels (see the pipeline below)
  constexpr int XW = DEEP ? NW / 2 : NW, WW = DEEP ? NW / 2 : NW;  // wavefronts that share the loads of a panel
  constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
  constexpr int MI = WTM / 16, NI = WTN / 16;  // 16x16 accumulator blocks of a wavefront's tile
  constexpr int OUT_BN = (EPI == EPI_SWIGLU) ? BN / 2 : BN;
  constexpr int ROWB = BK * 2;                       // bytes of one tile row
  constexpr int LDS_BYTES = DEEP ? LDS_CU : ring_bytes(NW);
  constexpr int GA = BM / 8, GB = BN / 8;            // 8-row groups = one 1 KB wavefront load each
  constexpr int LA = (GA + XW - 1) / XW, LB = (GB + WW - 1) / WW;  // loads per thread per panel
  static_assert(!DEEP || NW % 2 == 0, "two halves of the workgroup share the loads");
  static_assert(BK == 64, "swizzle and fragment addressing assume 128-byte tile rows");
  static_assert(WTM % 16 == 0 && WTN % 16 == 0, "tiles are made of 16x16 MFMA blocks");
  static_assert(EPI != EPI_SWIGLU || WTN % 64 == 0, "32 gate rows and their 32 up rows pair up inside a wave");
  static_assert(EPI != EPI_QKV || (WTN % 64 == 0 && BN % DH == 0), "32 pairs of a head's features meet inside a wave");
  static_assert(2 * LA + 2 * LB < 64, "outstanding loads must fit the vmcnt field");

  extern __shared__ __align__(16) unsigned char smem[];

  const int n_lim = a.n_count ? a.n_begin + a.n_count : a.N;  // end of the output columns of this launch
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (n_lim - a.n_begin + OUT_BN - 1) / OUT_BN;
  // split-K: consecutive workgroups are the k-ranges of one tile
  const int split = (EPI == EPI_PARTIAL) ? bid % a.k_splits : 0;
  const int tile_id = SK ? seg.pid : (EPI == EPI_PARTIAL) ? bid / a.k_splits : bid;
  const TileCoord tc = map_tile(tile_id, tiles_m * tiles_n, tiles_m, tiles_n);
  const int m0 = tc.tm * BM, n0 = a.n_begin + tc.tn * OUT_BN;

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm0 = (wave / WAVES_N) * WTM, wn0 = (wave % WAVES_N) * WTN;
  const int lr = lane & 15, lg = lane >> 4;  // row of a 16-row block; k-chunk of a fragment, feature group of an accumulator

  // ---- global -> LDS, without passing through registers ---------------------------
  // One wavefront load moves 8 tile rows (1 KB): lane i lands at LDS byte 16 i of the
  // group, i.e. row i/8, 16-byte slot i%8, and fetches the chunk that the XOR swizzle
  // assigns to that slot, so the eight lanes of a row cover one whole cache line.  Rows
  // past the matrix edge are clamped to the last row (their accumulators are never
  // stored); chunks past K read a block of zeros instead.
  const int g_row = lane >> 3, g_slot = lane & 7;
  // byte offsets from the matrix base (the host checks that they fit 32 bits): the address
  // of a load is then a uniform 64-bit base, advanced per k-tile by scalar code, plus a
  // per-lane offset that never changes
  uint32_t off_a[LA], off_b[LB];
  int ka[LA], kb[LB];        // element offset of this lane's chunk inside a k-tile
  int dst_a[LA], dst_b[LB];  // LDS byte offset of the group inside a unit
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    // when the groups do not divide over the wavefronts the surplus loads repeat the last
    // group (same bytes to the same place), so every wavefront issues LA loads per panel
    const int grp = (wave % XW + i * XW) < GA ? (wave % XW + i * XW) : GA - 1;
    const int row = grp * 8 + g_row;
    const int chunk = g_slot ^ ((row >> 1) & 7);
    ka[i] = chunk * 8;
    dst_a[i] = grp * 1024;
    int gm = m0 + row;
    gm = gm < a.M ? gm : a.M - 1;
    off_a[i] = (uint32_t)(((size_t)gm * a.lda + chunk * 8) * 2);
  }
#pragma unroll
  for (int i = 0; i < LB; ++i) {
    const int grp = (wave % WW + i * WW) < GB ? (wave % WW + i * WW) : GB - 1;
    const int wr = grp * 8 + g_row;
    const int chunk = g_slot ^ ((wr >> 1) & 7);
    kb[i] = chunk * 8;
    dst_b[i] = grp * 1024;
    int gn;
    if (EPI == EPI_SWIGLU) {
      const int blk = wr >> 5;
      int col = n0 + (blk >> 1) * 32 + (wr & 31);
      col = col < a.N ? col : a.N - 1;
      gn = col + ((blk & 1) ? a.N : 0);
    } else if (EPI == EPI_QKV) {
      const QkvGroup q = qkv_group((n0 + wr) >> 6, a, DH);
      gn = q.head * DH + q.i0 + (wr & 31) + ((wr & 32) ? DH / 2 : 0);
      gn = gn < a.N ? gn : a.N - 1;
    } else {
      gn = n0 + wr;
      gn = gn < a.N ? gn : a.N - 1;
    }
    off_b[i] = (uint32_t)(((size_t)gn * a.ldb + chunk * 8) * 2);
  }
  constexpr bool TURNED = DEEP && EPI != EPI_PARTIAL && BM <= 128;
  const int nk_whole = (a.K + BK - 1) / BK;
  const int first_kt = TURNED ? first_k_tile(tile_id, a.K, a.ldb) : 0;
  auto turned_kt = [&](int kt) {
    if (!TURNED || kt >= nk_whole) return kt;
    return kt + first_kt >= nk_whole ? kt + first_kt - nk_whole : kt + first_kt;
  };
  // load number i of panel X(kt) / W(kt) to LDS byte offset `lds_off`; `checked` handles chunks past K.  Buffer loads take the
  // k-tile as a scalar offset: no address arithmetic per load, and 16 registers less than 64-bit addresses.
#ifdef __HIP_DEVICE_COMPILE__
  const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.A), 0, 0xffffffff, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.B), 0, 0xffffffff, 0x00020000);
#else
  const int rsrc_a = 0, rsrc_b = 0;
#endif
  auto dma = [&](const uint16_t *mat, auto rsrc, int kt, uint32_t off, int ke, int lds_off, auto checked) {
    kt = turned_kt(kt);
#ifdef __HIP_DEVICE_COMPILE__
    auto *dst = (__attribute__((address_space(3))) void *)(smem + lds_off);
    if constexpr (decltype(checked)::value) {
      const void *p = reinterpret_cast<const unsigned char *>(mat) + (size_t)kt * ROWB + off;
      if (kt * BK + ke >= a.K) p = g_gemm_zero_chunk;
      __builtin_amdgcn_global_load_lds(p, dst, 16, 0, 0);
    } else {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, dst, 16, off, kt * ROWB, 0, 0);
    }
#endif
  };
  auto dma_a = [&](int kt, int lds_off, int i, auto checked) { dma(a.A, rsrc_a, kt, off_a[i], ka[i], lds_off + dst_a[i], checked); };
  auto dma_b = [&](int kt, int lds_off, int i, auto checked) { dma(a.B, rsrc_b, kt, off_b[i], kb[i], lds_off + dst_b[i], checked); };

  f32x4_t acc[NI][MI];
#pragma unroll
  for (int ni = 0; ni < NI; ++ni)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) acc[ni][mi] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // fragment addresses: tile row of the lane, chunk 4*ks + lg swizzled by ((row >> 1) & 7)
  const int sw = (lr >> 1) & 7;
  const int xfrag = (wm0 + lr) * ROWB;
  const int wfrag = (wn0 + lr) * ROWB;

  const int nk_all = (a.K + BK - 1) / BK;
  // this workgroup's k-tiles [kt0, kt1): all of them, or one of k_splits nearly equal ranges
  const int kt0 = SK ? seg.kt0 : (EPI == EPI_PARTIAL) ? (int)((long)nk_all * split / a.k_splits) : 0;
  const int kt1 = SK ? seg.kt1 : (EPI == EPI_PARTIAL) ? (int)((long)nk_all * (split + 1) / a.k_splits) : nk_all;
  constexpr int NF = MI + NI;   // fragment reads per 32-wide k-step
  constexpr int NMF = MI * NI;  // MFMAs per 32-wide k-step
  // read number o of k-step ks (32 wide, two per tile) of the panels in ring slots sa, sb
  // (xo, wo: LDS byte offsets of the two panels)
  auto frag = [&](int xo, int wo, int ks, int o, bf16x8_t (&xf)[MI], bf16x8_t (&wf)[NI]) {
    const int ch = ((ks * 4 + lg) ^ sw) << 4;
    if (o < MI)
      xf[o] = as_bf16x8(*reinterpret_cast<const u32x4_t *>(smem + xo + xfrag + o * 16 * ROWB + ch));
    else
      wf[o - MI] = as_bf16x8(*reinterpret_cast<const u32x4_t *>(smem + wo + wfrag + (o - MI) * 16 * ROWB + ch));
  };
  // One k-step: its NMF MFMAs in program order, with `n_ops` side operations (LDS reads of the next k-step, DMA
  // requests) dealt out between them, operation o behind MFMA at(o), so that the matrix pipe is never left idle
  // behind a run of memory instructions.
  auto step = [&](const bf16x8_t (&xf)[MI], const bf16x8_t (&wf)[NI], int n_ops, auto &&at, auto &&op) {
#pragma unroll
    for (int j = 0; j < NMF; ++j) {
      const int ni = j / MI, mi = j % MI;
      acc[ni][mi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[ni], xf[mi], acc[ni][mi], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int o = 0; o < n_ops; ++o)
        if (at(o) == j) op(o);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Where the operations of a k-step go: NF reads, then `n_dma` requests.  A request keeps the CU's address unit busy for
  // 16 to 24 clocks, and eight wavefronts that ask for eight KB each without a pause stand still behind one another, MFMAs
  // and all: a request every third MFMA (every second where a step is short), reads in between.
  // (The deep ring, bound by its weight stream, asks as early as it can: 256 rows, N = 4096, K = 14336 43.4 against 44.8 us.)
  constexpr auto place = [](int o, int n_dma) {
    if (DEEP) return o * NMF / (NF + n_dma > NMF ? NF + n_dma : NMF);
    const int pitch = 3 * n_dma - 1 <= NMF ? 3 : 2;
    const int j = o >= NF ? pitch - 1 + pitch * (o - NF) : pitch == 3 ? o + o / 2 : o;
    return j < NMF ? j : NMF - 1;
  };
  // LDS -> registers: the fragments of the next 32-wide k-step are requested while the MFMAs of the current one are
  // issued, across tile boundaries too, so the matrix pipe never waits for a whole LDS read phase.
  // The compiler counts an LDS-DMA load as a pending LDS operation of unknown order, so
  // every wait it places before an MFMA is lgkmcnt(0); waiting explicitly at the start of
  // a k-step, for reads issued during the first MFMAs of the previous one, keeps those
  // waits from covering reads that were only just issued.
  constexpr int LGKM0 = waitcnt_imm(63, true);
  constexpr int UX = BM * ROWB, UW = BN * ROWB;  // bytes of a panel
  bf16x8_t xa[MI], wa[NI], xb[MI], wb[NI];
  if constexpr (!DEEP) {
    // Panel X(kt) lives in activation slot kt % NXS, W(kt) in weight slot kt % NWS.  Once the last fragments of tile kt
    // are in registers, at the one barrier of the iteration, X(kt+NXS) and W(kt+NWS) are requested into the two slots
    // that tile kt frees: the weight panel, which in a layer streams from HBM, has two k-tiles of look-ahead, and the
    // activation panel, which the previous kernel has just left in the caches, one, or two where three slots fit.
    constexpr int NXS = ring_x_slots(BM, BN, NW), NWS = ring_w_slots(BM, BN, NW), W_BASE = NXS * UX;
    constexpr int AHEAD = NXS > NWS ? NXS : NWS;
    // loads requested after both panels of the next tile, and so still in flight when these have landed
    constexpr int YOUNG = NXS < NWS ? (NXS - 2) * (LA + LB) + LB : (NWS - 2) * (LA + LB);
    static_assert(NXS >= 2 && NWS >= 2 && W_BASE + NWS * UW <= LDS_BYTES && NXS * LA + NWS * LB < 64, "slots and the vmcnt field");
#pragma unroll
    for (int r = -AHEAD; r < 0; ++r) {
      if (r + NXS >= 0)
#pragma unroll
        for (int i = 0; i < LA; ++i) dma_a(kt0 + r + NXS, (r + NXS) * UX, i, Yes{});
      if (r + NWS >= 0)
#pragma unroll
        for (int i = 0; i < LB; ++i) dma_b(kt0 + r + NWS, W_BASE + (r + NWS) * UW, i, Yes{});
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(YOUNG + LA + LB, true));  // tile 0 has landed
    __builtin_amdgcn_s_barrier();
    int xo = 0, wo = W_BASE;  // slots of the tile being multiplied
#pragma unroll
    for (int o = 0; o < NF; ++o) frag(xo, wo, 0, o, xa, wa);
    auto tile = [&](int kt, auto checked) {
      __builtin_amdgcn_s_waitcnt(LGKM0);
      step(xa, wa, NF, [&](int o) { return place(o, 0); }, [&](int o) { frag(xo, wo, 1, o, xb, wb); });
      // Every fragment of tile kt is in registers once the LDS reads have returned, and
      // tile kt+1 has landed once this wavefront's loads other than the YOUNG last ones
      // are done; after the barrier both hold for every wavefront, so the two
      // slots of tile kt can be refilled and tile kt+1 can be read.
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(YOUNG, true));
      __builtin_amdgcn_s_barrier();
      const int nx = xo == (NXS - 1) * UX ? 0 : xo + UX, nw = wo == W_BASE + (NWS - 1) * UW ? W_BASE : wo + UW;
      step(xb, wb, NF + LA + LB, [&](int o) { return place(o, LA + LB); }, [&](int o) {
        if (o < NF)
          frag(nx, nw, 0, o, xa, wa);
        else if (o < NF + LA)
          dma_a(kt + NXS, xo, o - NF, checked);
        else
          dma_b(kt + NWS, wo, o - NF - LA, checked);
      });
      xo = nx;
      wo = nw;
    };
    int kt = kt0;
    const int n_plain = a.K / BK - AHEAD;  // tiles kt for which X(kt+NXS) and W(kt+NWS) lie wholly inside K
    for (; kt < n_plain && kt < kt1; ++kt) tile(kt, No{});
    for (; kt < kt1; ++kt) tile(kt, Yes{});
  } else {
    // One round of tiles over few rows: every CU streams a weight panel of its own from HBM,
    // and the rings above give it two k-tiles of look-ahead at most.  Here LDS
    // holds NXS = DEEP + 1 slots for the activation panel (shared by all tiles, served by the
    // L2: NXS - 1 k-tiles of look-ahead) and all the rest, NWS slots, for the weight panel:
    // NWS - 1 k-tiles of look-ahead.  The memory counter of a wavefront retires its loads in
    // order, so a wait for an activation panel would also wait for every weight panel
    // requested before it; the two kinds of request therefore come from different wavefronts:
    // the first half of the workgroup loads activations and waits until its NXS - 2 youngest
    // panels remain, the second half loads weights and waits until its NWS - 2 youngest remain.
    constexpr int NXS = DEEP + 1;  // activation slots
    constexpr int W_BASE = NXS * UX;
    constexpr int NWS = (LDS_BYTES - W_BASE) / UW;
    static_assert(NWS >= 3 && (NWS - 1) * LB < 64 && (NXS - 1) * LA < 64, "slots and the vmcnt field");
    const bool loads_x = wave < XW;  // uniform
    if (loads_x) {
#pragma unroll
      for (int sl = 0; sl < NXS; ++sl)
#pragma unroll
        for (int i = 0; i < LA; ++i) dma_a(kt0 + sl, sl * UX, i, Yes{});
      __builtin_amdgcn_s_waitcnt(waitcnt_imm((NXS - 1) * LA, true));
    } else {
#pragma unroll
      for (int sl = 0; sl < NWS; ++sl)
#pragma unroll
        for (int i = 0; i < LB; ++i) dma_b(kt0 + sl, W_BASE + sl * UW, i, Yes{});
      __builtin_amdgcn_s_waitcnt(waitcnt_imm((NWS - 1) * LB, true));
    }
    __builtin_amdgcn_s_barrier();  // tile 0 has landed
    int xs = 0, ws = 0;            // activation and weight slot numbers of the tile being multiplied
#pragma unroll
    for (int o = 0; o < NF; ++o) frag(xs * UX, W_BASE + ws * UW, 0, o, xa, wa);
    auto tile = [&](int kt, auto checked) {
      const int wo = W_BASE + ws * UW, xo = xs * UX;
      __builtin_amdgcn_s_waitcnt(LGKM0);
      step(xa, wa, NF, [&](int o) { return place(o, 0); }, [&](int o) { frag(xo, wo, 1, o, xb, wb); });
      // after the barrier: every wavefront holds all fragments of tile kt, X(kt+1) has landed
      // (the activation half waited until only X(kt+2) .. X(kt+NXS-1) were outstanding) and so
      // has W(kt+1) (the weight half: only W(kt+2) .. W(kt+NWS-1))
      if (loads_x)
        __builtin_amdgcn_s_waitcnt(waitcnt_imm((NXS - 2) * LA, true));
      else
        __builtin_amdgcn_s_waitcnt(waitcnt_imm((NWS - 2) * LB, true));
      __builtin_amdgcn_s_barrier();
      const int nxs = xs + 1 == NXS ? 0 : xs + 1, nws = ws + 1 == NWS ? 0 : ws + 1;
      const int nxo = nxs * UX;
      const int nwo = W_BASE + nws * UW;
      if (loads_x)
        step(xb, wb, NF + LA, [&](int o) { return place(o, LA); }, [&](int o) {
          if (o < NF)
            frag(nxo, nwo, 0, o, xa, wa);
          else
            dma_a(kt + NXS, xo, o - NF, checked);
        });
      else
        step(xb, wb, NF + LB, [&](int o) { return place(o, LB); }, [&](int o) {
          if (o < NF)
            frag(nxo, nwo, 0, o, xa, wa);
          else
            dma_b(kt + NWS, wo, o - NF, checked);
        });
      xs = nxs;
      ws = nws;
    };
    int kt = kt0;
    const int n_plain = a.K / BK - (NWS > NXS ? NWS : NXS);  // tiles kt for which X(kt+NXS) and W(kt+NWS) lie wholly inside K
    for (; kt < n_plain && kt < kt1; ++kt) tile(kt, No{});
    for (; kt < kt1; ++kt) tile(kt, Yes{});
  }
  // drain the look-ahead loads (zeros or clamped rows) before the LDS is released
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, true));
  if (EPI != EPI_SWIGLU) __syncthreads();  // results pass through LDS on their way out: nobody may still be reading panels there

  if constexpr (SK) {
    if (seg.parts > 1) {
      constexpr int NT = NW * 64;
      constexpr size_t TILE = (size_t)BM * BN;
      // The register image of the accumulators, 16 bytes per thread and block (whoever adds the
      // parts up has the same layout).  The eight XCDs keep L2 caches of their own, so parts
      // written and read with ordinary accesses would need the whole-cache write-back and
      // invalidation of a device-wide fence at every cut (measured: a quarter of a millisecond
      // per launch); the parts travel with the device-scope cache policy instead (sc1: to and
      // from the point where all XCDs agree), which touches nothing else.
      typedef unsigned int u4_t __attribute__((ext_vector_type(4)));
      constexpr int SC1 = 16;
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(sp->ws, 0, 0x7fffffff, 0x00020000);
      const unsigned voff = (unsigned)t * 16u;
      {
        const unsigned soff = (unsigned)seg.my_slot * (unsigned)(TILE * 4);
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
          for (int mi = 0; mi < MI; ++mi) {
            const f32x4_t c = acc[ni][mi];
            const u4_t v = {__float_as_uint(c[0]), __float_as_uint(c[1]), __float_as_uint(c[2]), __float_as_uint(c[3])};
            __builtin_amdgcn_raw_buffer_store_b128(v, rs, voff + (unsigned)((ni * MI + mi) * NT * 16), soff, SC1);
          }
      }
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, true));  // the part has arrived there before the workgroup counts itself in
      __syncthreads();
      volatile unsigned *flag = reinterpret_cast<volatile unsigned *>(smem + LDS_BYTES - 16);
      if (t == 0) *flag = atomicAdd(sp->cnt + seg.j, 1u);
      __syncthreads();
      if (*flag + 1u != (unsigned)seg.parts) return;
      if (t == 0) atomicExch(sp->cnt + seg.j, 0u);  // as the next launch expects it
      for (int q = 0; q < seg.parts; ++q) {
        const int w2 = seg.w_first + q;
        const int slot = 2 * w2 + (sk_bound(*sp, w2) / sp->nk == seg.j ? 0 : 1);
        const unsigned soff = (unsigned)slot * (unsigned)(TILE * 4);
        // sixteen blocks at a time: the loads of a batch are all in flight before the first is
        // used (each is a round trip past the L2; the registers of the fragments are free now)
        constexpr int NB = NI * MI, BATCH = NB < 16 ? NB : 16;
        static_assert(NB % BATCH == 0, "whole batches");
#pragma unroll
        for (int b0 = 0; b0 < NB; b0 += BATCH) {
          u4_t v[BATCH];
#pragma unroll
          for (int b = 0; b < BATCH; ++b)
            v[b] = __builtin_amdgcn_raw_buffer_load_b128(rs, voff + (unsigned)((b0 + b) * NT * 16), soff, SC1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int b = 0; b < BATCH; ++b) {
            const int ni = (b0 + b) / MI, mi = (b0 + b) % MI;
            const f32x4_t c = {__uint_as_float(v[b].x), __uint_as_float(v[b].y), __uint_as_float(v[b].z), __uint_as_float(v[b].w)};
            acc[ni][mi] = q == 0 ? c : acc[ni][mi] + c;
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  }

  // ---- epilogues ---------------------------------------------------------------
  // accumulator element e of block (ni, mi): m = m0 + wm0 + mi*16 + lr, n = n_tile + wn0 + ni*16 + 4*lg + e.
  // Neighbouring lanes hold neighbouring ROWS, and a CU serves loads and stores of such lanes at about one lane per
  // clock.  The wavefront therefore turns its 64 columns round in LDS, CM blocks of 16 rows at a time, and comes back with
  // sixteen lanes along a row: 16 tiles of 256x256 with K = 64, launch included, output projection 28 -> 17 us, down
  // projection 15.8 -> 12.5, QKV 15.8 -> 12.7; 8192 rows of the 8B layer 287 -> 248, 756 -> 737, 353 -> 333.
  static_assert(WTN == 64, "an epilogue hands 64 columns to 16 lanes");
  constexpr int CM = MI <= 4 ? MI : (MI + 1) / 2;
  constexpr int RS = 64 * 4 + 16;  // bytes of a row of 64 floats: rows four banks apart
  static_assert(NW * CM * 16 * RS <= LDS_BYTES, "the turned blocks fit the panel ring");
  unsigned char *turned = smem + wave * (CM * 16 * RS);
  // blocks [c, c + CM) of rows into LDS (read and written by this wavefront alone, whose LDS operations complete in order)
  auto turn = [&](int c) {
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < CM; ++j)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
        if (c + j < MI) *reinterpret_cast<f32x4_t *>(turned + (j * 16 + lr) * RS + (ni * 16 + 4 * lg) * 4) = acc[ni][c + j];
    __builtin_amdgcn_wave_barrier();
  };
  constexpr auto rows_in = [](int c) { return (MI - c < CM ? MI - c : CM) * 16; };
  const int r16 = lane >> 4, c16 = 4 * (lane & 15);  // four rows of 64 columns per step

  if constexpr (EPI == EPI_PARTIAL || EPI == EPI_PLAIN || EPI == EPI_RESID || EPI == EPI_RESID_NORM) {
    const int n = n0 + wn0 + c16;
    const bool n_ok = n < n_lim;
    const int nc = min(n, a.N - 4);  // loads beyond an edge repeat the last column or row
    constexpr int U = 4;             // steps of four rows whose residuals are in flight
    float *ws = a.sk_ws + (size_t)split * a.M * a.N;
    f32x4_t gain = {0.f, 0.f, 0.f, 0.f};
    auto bf16x4 = [](u32x2_t v) {
      return f32x4_t{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u), __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xFFFF0000u)};
    };
    if constexpr (EPI == EPI_RESID_NORM) gain = bf16x4(*reinterpret_cast<const u32x2_t *>(a.gain + nc));
    auto resid = [&](int row) -> f32x4_t {
      const size_t at = (size_t)min(m0 + wm0 + row, a.M - 1) * a.ldr + nc;
      if (EPI == EPI_RESID && a.resid32) return *reinterpret_cast<const f32x4_t *>(a.resid32 + at);
      return bf16x4(*reinterpret_cast<const u32x2_t *>(a.resid + at));
    };
    constexpr bool ADDS = EPI == EPI_RESID || EPI == EPI_RESID_NORM;
    f32x4_t r[U];
    if constexpr (ADDS) {
#pragma unroll
      for (int u = 0; u < U; ++u) r[u] = resid(4 * u + r16);
    }
#pragma unroll
    for (int c = 0; c < MI; c += CM) {
      turn(c);
#pragma unroll 1
      for (int g = 0; g < rows_in(c); g += 4 * U) {
        f32x4_t v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          v[u] = *reinterpret_cast<const f32x4_t *>(turned + (g + 4 * u + r16) * RS + c16 * 4);
          if constexpr (ADDS) v[u] += r[u];
        }
        if constexpr (ADDS) {  // the next rows, ahead of the stores: a load does not pass a store that may write what it reads
#pragma unroll
          for (int u = 0; u < U; ++u) r[u] = resid(c * 16 + g + 4 * U + 4 * u + r16);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int m = m0 + wm0 + c * 16 + g + 4 * u + r16;
          const bool ok = n_ok && m < a.M;
          if constexpr (EPI == EPI_PARTIAL) {
            if (ok) *reinterpret_cast<f32x4_t *>(ws + (size_t)m * a.N + n) = v[u];
          } else if constexpr (EPI == EPI_RESID_NORM) {
            float ss = ok ? v[u][0] * v[u][0] + v[u][1] * v[u][1] + v[u][2] * v[u][2] + v[u][3] * v[u][3] : 0.f;
            if (ok) {
              // x1 stays in fp32 for the second residual add; the next GEMM reads bf16(x1 * gain)
              *reinterpret_cast<f32x4_t *>(a.C32 + (size_t)m * a.ldc + n) = v[u];
              store_bf16x4(a.C_gain + (size_t)m * a.ldc + n, v[u][0] * gain[0], v[u][1] * gain[1], v[u][2] * gain[2], v[u][3] * gain[3]);
            }
            // the sixteen lanes of the row add up: one partial sum per wavefront column
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) ss += __shfl_xor(ss, o, 64);
            if (c16 == 0 && m < a.M) a.ss_out[(size_t)(tc.tn * WAVES_N + (wave % WAVES_N)) * a.ss_stride + m] = ss;
          } else {
            if (ok) store_bf16x4(a.C + (size_t)m * a.ldc + n, v[u][0], v[u][1], v[u][2], v[u][3]);
          }
        }
      }
    }
  }

  float rstd[MI];
  if constexpr (EPI == EPI_QKV || EPI == EPI_SWIGLU) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) rstd[mi] = a.rstd[min(m0 + wm0 + mi * 16 + lr, a.M - 1)];
  }

  if constexpr (EPI == EPI_SWIGLU) {
    // the weight tile interleaves 32 gate rows with the matching 32 up rows: blocks 0, 1 are gate
    // features, blocks 2, 3 their up features.  A quarter of the output projection's bytes, straight from the
    // registers (turned round in LDS as well: 1580 rows of the 8B layer 351 -> 357 us)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
      const int m = m0 + wm0 + mi * 16 + lr;
      const float s = rstd[mi];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int n = n0 + (wn0 >> 1) + h * 16 + 4 * lg;
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float g = acc[h][mi][e] * s;
          const float u = acc[2 + h][mi][e] * s;
          v[e] = g / (1.f + __expf(-g)) * u;
        }
        if (m < a.M && n < n_lim) store_bf16x4(a.C + (size_t)m * a.ldc + n, v[0], v[1], v[2], v[3]);
      }
    }
  }

  if constexpr (EPI == EPI_QKV) {
    // the 64 tile columns of a wavefront: features i0 .. i0 + 31 of a head (blocks 0, 1) and i0 + dh/2 .. (blocks 2, 3)
    constexpr int HALF = DH / 2;
    const size_t tile_elems = (size_t)16 * DH;  // one K or V tile of a (page, head)
    const QkvGroup group = qkv_group((n0 + wn0) >> 6, a, DH);
    const int head = group.head, i0 = group.i0;
    const bool is_q = head < a.n_q_heads;
    const bool is_k = !is_q && head < a.n_q_heads + a.n_kv_heads;
    if (head >= a.n_q_heads + 2 * a.n_kv_heads) {
      // a wavefront beyond the last head
    } else if (is_q || is_k) {
      // eight rows per step, eight lanes with four rotation pairs each along a row
      const int r8 = lane >> 3, p8 = 4 * (lane & 7), i = i0 + p8;
      constexpr int U = 2;  // steps at a time; the angles of the next ones and the positions of those behind are under way
      int pos[U], page[U], slot[U], page_n[U] = {}, slot_n[U] = {};
      float s[U], s_n[U];
      f32x4_t cs[U], sn[U];
      auto ask_rows = [&](int row) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int m = min(m0 + wm0 + row + 8 * u + r8, a.M - 1);
          pos[u] = a.row_pos[m];
          s_n[u] = a.rstd[m];
          if (is_k) {
            page_n[u] = a.row_page[m];
            slot_n[u] = a.row_slot[m];
          }
        }
      };
      auto ask_angles = [&]() {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          cs[u] = *reinterpret_cast<const f32x4_t *>(a.rope_cos + (size_t)pos[u] * HALF + i);
          sn[u] = *reinterpret_cast<const f32x4_t *>(a.rope_sin + (size_t)pos[u] * HALF + i);
          s[u] = s_n[u];
          page[u] = page_n[u];
          slot[u] = slot_n[u];
        }
      };
      ask_rows(0);
      ask_angles();
      ask_rows(8 * U);
#pragma unroll
      for (int c = 0; c < MI; c += CM) {
        turn(c);
#pragma unroll 1
        for (int g = 0; g < rows_in(c); g += 8 * U) {
          f32x4_t lo[U], hi[U];
          uint16_t *dst[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const unsigned char *row = turned + (g + 8 * u + r8) * RS;
            const f32x4_t l = *reinterpret_cast<const f32x4_t *>(row + p8 * 4) * s[u];
            const f32x4_t h = *reinterpret_cast<const f32x4_t *>(row + (32 + p8) * 4) * s[u];
            lo[u] = l * cs[u] - h * sn[u];
            hi[u] = h * cs[u] + l * sn[u];
            const int m = m0 + wm0 + c * 16 + g + 8 * u + r8;
            dst[u] = is_q ? a.q_out + (size_t)m * (a.n_q_heads * DH) + head * DH + i
                          : a.kv_pool + (((size_t)page[u] * 2 + 0) * a.n_kv_heads + (head - a.n_q_heads)) * tile_elems +
                                (size_t)slot[u] * DH + i;
          }
          ask_angles();
          ask_rows(c * 16 + g + 16 * U);
#pragma unroll
          for (int u = 0; u < U; ++u) {
            if (m0 + wm0 + c * 16 + g + 8 * u + r8 >= a.M) continue;
            store_bf16x4(dst[u], lo[u][0], lo[u][1], lo[u][2], lo[u][3]);
            store_bf16x4(dst[u] + HALF, hi[u][0], hi[u][1], hi[u][2], hi[u][3]);
          }
        }
      }
    } else {
      // V^T tiles hold, per feature, the 16 slots of a page side by side, while a lane
      // holds four features of one row: the wavefront turns its block round in LDS
      // (feature-major, FS bytes per feature: the row count padded so that neither the
      // 2-byte writes nor the 8-byte reads below collide on banks)
      constexpr int FS = (WTM + 4) * 2;
      static_assert(64 * FS <= CM * 16 * RS, "the features of a wavefront fit its part of the ring");
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            *reinterpret_cast<uint16_t *>(turned + (b * 16 + 4 * lg + e) * FS + (mi * 16 + lr) * 2) = f32_to_bf16(acc[b][mi][e] * rstd[mi]);
      // Back out of LDS: lane = 4 * feature + quad reads rows 4 quad .. 4 quad + 3 of a 16-row block for one
      // feature.  Inside a prefill segment these are four adjacent slots of one page, and the 64 lanes then
      // cover 512 contiguous bytes of the page's V^T tile; they go out as one 8-byte store (or two
      // 4-byte ones) where the address allows.  Rows of different sequences, or on either
      // side of a page boundary, take a 2-byte store each.
      __builtin_amdgcn_wave_barrier();
      const int vh = head - a.n_q_heads - a.n_kv_heads;
      const int fl = lane >> 2, rq = lane & 3;
      int pg[4], sl[4], pn[4], ln[4];
      auto ask = [&](int mi, int (&p)[4], int (&l)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int m = min(m0 + wm0 + mi * 16 + rq * 4 + e, a.M - 1);
          p[e] = a.row_page[m];
          l[e] = a.row_slot[m];
        }
      };
      ask(0, pg, sl);
#pragma unroll 1
      for (int mi = 0; mi < MI; ++mi) {
        const int ml = mi * 16 + rq * 4, mb = m0 + wm0 + ml;
        ask(mi + 1, pn, ln);
        bool run = mb + 3 < a.M;
#pragma unroll
        for (int e = 1; e < 4; ++e) run = run && pg[e] == pg[0] && sl[e] == sl[0] + e;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int ei = (b >> 1) * HALF + i0 + (b & 1) * 16 + fl;
          const u32x2_t v = *reinterpret_cast<const u32x2_t *>(turned + (b * 16 + fl) * FS + ml * 2);
          uint16_t *d0 = a.kv_pool + (((size_t)pg[0] * 2 + 1) * a.n_kv_heads + vh) * tile_elems + ei * 16 + sl[0];
          if (run && (reinterpret_cast<uintptr_t>(d0) & 7) == 0) {
            *reinterpret_cast<u32x2_t *>(d0) = v;
          } else if (run && (reinterpret_cast<uintptr_t>(d0) & 3) == 0) {
            reinterpret_cast<uint32_t *>(d0)[0] = v.x;
            reinterpret_cast<uint32_t *>(d0)[1] = v.y;
          } else {
            const uint16_t ve[4] = {(uint16_t)(v.x & 0xFFFFu), (uint16_t)(v.x >> 16), (uint16_t)(v.y & 0xFFFFu), (uint16_t)(v.y >> 16)};
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (mb + e < a.M) a.kv_pool[(((size_t)pg[e] * 2 + 1) * a.n_kv_heads + vh) * tile_elems + ei * 16 + sl[e]] = ve[e];
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          pg[e] = pn[e];
          sl[e] = ln[e];
        }
      }
    }
  }
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int DH, int DEEP = 0>
__global__ __launch_bounds__(WAVES_M *WAVES_N * 64, 2) void gemm_kernel(const GemmArgs a) {
  gemm_tile<BM, BN, WAVES_M, WAVES_N, EPI, DH, DEEP>(a, (int)blockIdx.x);
}

// (All 256 registers are in use: 36 to 66 spill, around the loop over k-tiles and never in it, as do 4 to 7 of the whole
// 256x256 tiles of the QKV projection.)
template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int DH>
__global__ __launch_bounds__(WAVES_M *WAVES_N * 64) void gemm_sk_kernel(const GemmArgs a, const SkPlan p) {
  const int w = (int)blockIdx.x, G = (int)gridDim.x;
  int pid = w;
  int i = 0, i1 = 0, j0 = 0;
  if (w < p.g_sk) {
    i = sk_bound(p, w);
    i1 = sk_bound(p, w + 1);
    j0 = i / p.nk;
  }
  bool again = false;
  for (;;) {
    SkSeg s;
    if (pid < p.n_dp) {
      s = SkSeg{pid, 0, p.nk, 0, 1, 0, 0};
      pid += G;
    } else if (i < i1) {
      const int j = i / p.nk, kt0 = i - j * p.nk;
      const int kt1 = (i1 - j * p.nk) < p.nk ? (i1 - j * p.nk) : p.nk;
      s = SkSeg{p.n_dp + j, kt0, kt1, j, 1, 0, 0};
      if (kt0 > 0 || kt1 < p.nk) {
        sk_tile_span(p, j, &s.w_first, &s.parts);
        s.my_slot = 2 * w + (j == j0 ? 0 : 1);
      }
      i = j * p.nk + kt1;
    } else {
      break;
    }
    if (again) __syncthreads();  // the panel ring and the flag word change hands
    again = true;
    gemm_tile<BM, BN, WAVES_M, WAVES_N, EPI, DH, 0, true>(a, 0, &p, s);
  }
}

// A GEMM launch that carries decode attention (Section 3.3: a step whose compute-bound and
// memory-bound operators overlap costs the larger of their times; Section 2.2, operator-level
// overlapping).  Grid: `head` attention workgroups, the GEMM tiles, `tail` attention
// workgroups.  A workgroup of either kind takes a whole CU (the tile all of its LDS, either
// kind half of every SIMD's registers per wavefront), so the two kinds never share one: the
// head workgroups hold their CUs for as long as the GEMM runs and stream KV pages beside it,
// the tail workgroups start on the CUs that the last, partly filled round of tiles leaves
// idle.  The attention wavefronts draw 16-row units from the step's queue; the tile that
// brings the count of finished tiles to `close_at` closes the queue for this launch and
// hands its position to the next one, so nobody starts a unit that would outlast the GEMM
// by more than its own length.  No workgroup ever waits for another.
template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int DH, int ADH>
__global__ __launch_bounds__(WAVES_M *WAVES_N * 64) void gemm_attn_kernel(const GemmArgs a, const GemmRide r, const int n_tiles,
                                                                              const unsigned close_at) {
  static_assert(WAVES_M * WAVES_N == 8, "attention workgroups are written for eight wavefronts");
  const int b = (int)blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint64_t *rec = r.q.trace ? r.q.trace + (size_t)TRACE_WORDS * (8 * b + wave) : nullptr;
  if (b < r.head || b >= r.head + n_tiles) {
    attn_dev::decode_queue_worker<ADH>(r.q, wave, threadIdx.x & 63, rec);
    return;
  }
  const uint64_t t0 = rec ? wall_clock64() : 0;
  gemm_tile<BM, BN, WAVES_M, WAVES_N, EPI, DH>(a, b - r.head);
  if (threadIdx.x == 0) {
    const unsigned before = atomicAdd(r.done, 1u);
    if (before + 1 == close_at) {
      const unsigned pos = atomicAdd(r.q.ticket, DECODE_QUEUE_CLOSED);
      const unsigned capped = pos < (unsigned)r.q.n_units ? pos : (unsigned)r.q.n_units;
      atomicExch(r.ticket_next, capped);
      if (r.closed_at) *r.closed_at = capped;
    }
    if (rec) attn_dev::trace_record(rec, t0, TRACE_TILE, before + 1 == close_at ? 1u : 0u, 0u);
  }
}

constexpr int MAX_SPLITS = 8;

// four consecutive columns of one row, summed over the k-ranges in a fixed order; the loads are
// independent of one another and go out together
__device__ __forceinline__ f32x4_t splitk_sum(const float *p, size_t plane, int k_splits) {
  f32x4_t part[MAX_SPLITS];
#pragma unroll
  for (int s = 0; s < MAX_SPLITS; ++s)
    part[s] = s < k_splits ? *reinterpret_cast<const f32x4_t *>(p + s * plane) : f32x4_t{0.f, 0.f, 0.f, 0.f};
  f32x4_t v = part[0];
#pragma unroll
  for (int s = 1; s < MAX_SPLITS; ++s) v += part[s];
  return v;
}

// Second half of a split-K product: adds the k_splits partial rows and applies the epilogue.
// RESID: y = resid + sum, one thread per four columns.
__global__ __launch_bounds__(256) void splitk_reduce_resid_kernel(const GemmArgs a) {
  const int m = blockIdx.x, n = (blockIdx.y * 256 + threadIdx.x) * 4;
  if (n >= a.N) return;
  f32x4_t v = splitk_sum(a.sk_ws + (size_t)m * a.N + n, (size_t)a.M * a.N, a.k_splits);
  if (a.resid32) {
    v += *reinterpret_cast<const f32x4_t *>(a.resid32 + (size_t)m * a.ldr + n);
  } else {
    const u32x2_t rr = *reinterpret_cast<const u32x2_t *>(a.resid + (size_t)m * a.ldr + n);
    v[0] += __uint_as_float(rr.x << 16);
    v[1] += __uint_as_float(rr.x & 0xFFFF0000u);
    v[2] += __uint_as_float(rr.y << 16);
    v[3] += __uint_as_float(rr.y & 0xFFFF0000u);
  }
  store_bf16x4(a.C + (size_t)m * a.ldc + n, v[0], v[1], v[2], v[3]);
}

// RESID_NORM: x1 = resid + sum in fp32, bf16(x1 * gain), and the row's sum of squares, complete,
// in ss_out slot 0; one workgroup per row, of as many threads as the row has groups of four columns
// (up to 1024), so that a row is one round trip to memory.
__global__ __launch_bounds__(1024) void splitk_reduce_resid_norm_kernel(const GemmArgs a) {
  const int m = blockIdx.x;
  float ss = 0.f;
  for (int n = threadIdx.x * 4; n < a.N; n += (int)blockDim.x * 4) {
    f32x4_t v = splitk_sum(a.sk_ws + (size_t)m * a.N + n, (size_t)a.M * a.N, a.k_splits);
    const u32x2_t rr = *reinterpret_cast<const u32x2_t *>(a.resid + (size_t)m * a.ldr + n);
    v[0] += __uint_as_float(rr.x << 16);
    v[1] += __uint_as_float(rr.x & 0xFFFF0000u);
    v[2] += __uint_as_float(rr.y << 16);
    v[3] += __uint_as_float(rr.y & 0xFFFF0000u);
    const u32x2_t gg = *reinterpret_cast<const u32x2_t *>(a.gain + n);
    const float g0 = __uint_as_float(gg.x << 16), g1 = __uint_as_float(gg.x & 0xFFFF0000u);
    const float g2 = __uint_as_float(gg.y << 16), g3 = __uint_as_float(gg.y & 0xFFFF0000u);
    ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
    *reinterpret_cast<f32x4_t *>(a.C32 + (size_t)m * a.ldc + n) = v;
    store_bf16x4(a.C_gain + (size_t)m * a.ldc + n, v[0] * g0, v[1] * g1, v[2] * g2, v[3] * g3);
  }
  __shared__ float part[16];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
  __syncthreads();
  if (threadIdx.x == 0) {
    float row = 0.f;
    for (int w = 0; w < ((int)blockDim.x + 63) / 64; ++w) row += part[w];
    a.ss_out[m] = row;
    if (a.rstd_out) a.rstd_out[m] = rsqrtf(row / (float)a.N + a.rstd_eps);
  }
}

// QKV: scale by the row's RMSNorm factor, rotate the q and k heads (pairs i, i + dh/2), store q
// to its buffer, k and v into the row's page slot (v transposed).  One thread per four
// consecutive pairs (q and k heads) or four consecutive v elements.
__global__ __launch_bounds__(256) void splitk_reduce_qkv_kernel(const GemmArgs a, int dh) {
  const int m = blockIdx.x;
  const int item = blockIdx.y * 256 + threadIdx.x;
  const size_t plane = (size_t)a.M * a.N;
  const float *ws = a.sk_ws + (size_t)m * a.N;
  const float rs = a.rstd[m];
  const int half = dh / 2, q4 = half / 4;
  const size_t page = a.row_page[m];
  const int slot = a.row_slot[m];
  const size_t tile_elems = (size_t)16 * dh;
  const int n_rot = (a.n_q_heads + a.n_kv_heads) * q4;
  if (item < n_rot) {
    const int head = item / q4, i = (item % q4) * 4, pos = a.row_pos[m];
    const f32x4_t l = splitk_sum(ws + head * dh + i, plane, a.k_splits) * rs;
    const f32x4_t h = splitk_sum(ws + head * dh + half + i, plane, a.k_splits) * rs;
    const f32x4_t c = *reinterpret_cast<const f32x4_t *>(a.rope_cos + (size_t)pos * half + i);
    const f32x4_t sn = *reinterpret_cast<const f32x4_t *>(a.rope_sin + (size_t)pos * half + i);
    uint16_t *dst = head < a.n_q_heads
                        ? a.q_out + (size_t)m * (a.n_q_heads * dh) + head * dh
                        : a.kv_pool + ((page * 2 + 0) * a.n_kv_heads + (head - a.n_q_heads)) * tile_elems + (size_t)slot * dh;
    const f32x4_t lo = l * c - h * sn, hi = h * c + l * sn;
    store_bf16x4(dst + i, lo[0], lo[1], lo[2], lo[3]);
    store_bf16x4(dst + half + i, hi[0], hi[1], hi[2], hi[3]);
  } else if (item < n_rot + a.n_kv_heads * (dh / 4)) {
    const int w = (item - n_rot) * 4, head = w / dh, e = w % dh;
    const f32x4_t v = splitk_sum(ws + (a.n_q_heads + a.n_kv_heads) * dh + w, plane, a.k_splits) * rs;
    uint16_t *dst = a.kv_pool + ((page * 2 + 1) * a.n_kv_heads + head) * tile_elems + slot;
#pragma unroll
    for (int j = 0; j < 4; ++j) dst[(e + j) * 16] = f32_to_bf16(v[j]);
  }
}

// Few rows: a product is the stream of its weights.  One workgroup of eight wavefronts per CU takes items, 16 NI weight
// rows by 16 MI activation rows, in turn and cuts K among its wavefronts, k-tiles of 64 dealt round (together they walk
// 1 KB of every weight row at a time).  A wavefront has a ring of S k-tiles of its own in LDS, both panels, filled by its
// own requests and read by nobody else: no barrier while it streams, and the ring runs on across items.  At the end of
// an item the eight partial sums of a value meet in LDS, one wavefront adds them in the order of the wavefronts and runs
// the epilogue while the others stream on: no partial products in memory, no second kernel.
// The 16 rows of a weight block are two units of eight where the epilogue pairs rows: gate and up rows, or the lower and
// upper half of a head's rotation pairs.
// Measured, cold weights, second kernels included, 8B layer at 8 rows: QKV 17.1 -> 12.9 us, output projection
// 14.9 -> 9.1, gate/up 53.8 -> 39.5 (5.9 TB/s), down 27.9 -> 22.9; K = N = 256 7.7 -> 3.4.  Not depth but the order of
// the requests makes the difference: 128x128 tiles with as many bytes in flight take 54 us for gate/up, every workgroup
// at the same column of 128 rows 8 KB apart.  Loads straight into registers (a lane's operand: 16 bytes of a row
// 8 KB from its neighbour's) reach 16 bytes per clock and CU: 56 us.
constexpr int ROWS_MAX_M = 256;
// blocks of 16 weight rows of a product (of pairs of eight where the epilogue pairs rows)
constexpr long rows_blocks(int n, int epi) { return epi == EPI_QKV ? n / 16 : epi == EPI_SWIGLU ? n / 8 : (n + 15) / 16; }
template <int MI, int NI>  // blocks of 16 activation rows, blocks of 16 weight rows
struct RowsKernel {
  static constexpr int L = 2 * (MI + NI), STAGE = L * 1024;  // loads and bytes of a k-tile
  static constexpr int RED = 8 * MI * 1024, META = ROWS_MAX_M * 16;
  static constexpr int S = (160 * 1024 - RED - META) / 8 / STAGE;
  static constexpr int LDS = 8 * S * STAGE + RED + META;
};

// waits until at most J * L vector-memory operations are outstanding, for the J that equals `left`
template <int L, int... J>
__device__ __forceinline__ void wait_for_all_but(int left, std::integer_sequence<int, J...>) {
  ((left == J ? __builtin_amdgcn_s_waitcnt(waitcnt_imm(J * L, false)) : (void)0), ...);
}

template <int MI, int NI>
__global__ __launch_bounds__(512) void gemm_rows_kernel(const GemmArgs a, const int epi, const int dh, const int tiles_m, const int n_items) {
  typedef RowsKernel<MI, NI> R;
  constexpr int S = R::S, L = R::L;
  static_assert(S >= 2 && (S - 1) * L < 64, "look-ahead, and the vmcnt field");
  extern __shared__ __align__(16) unsigned char smem[];
  f32x4_t *red = reinterpret_cast<f32x4_t *>(smem + 8 * S * R::STAGE);  // [8][MI][64]
  float *meta_rs = reinterpret_cast<float *>(smem + 8 * S * R::STAGE + R::RED);  // [ROWS_MAX_M] per row: norm factor, position, page, slot
  int *meta_pos = reinterpret_cast<int *>(meta_rs + ROWS_MAX_M), *meta_page = meta_pos + ROWS_MAX_M, *meta_slot = meta_page + ROWS_MAX_M;
  const bool paired = epi == EPI_QKV || epi == EPI_SWIGLU;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  unsigned char *ring = smem + wave * S * R::STAGE;

  // requests: 8 lanes per row of 128 bytes, chunks swizzled as in gemm_tile
  const int g_row = lane >> 3, g_slot = lane & 7;
  const int chunk[2] = {g_slot ^ (g_row >> 1), g_slot ^ ((g_row + 8) >> 1)};  // rows g_row and g_row + 8 of a block
  uint32_t off_x[2 * MI], off_w[2 * NI];
  const int per_head = dh / 16;
  auto first_row = [&](int blk) { return epi == EPI_QKV ? blk / per_head * dh + blk % per_head * 8 : paired ? blk * 8 : blk * 16; };
  const int second = epi == EPI_QKV ? dh / 2 : a.N;  // from a paired unit's first eight rows to its second
  // items: the row tiles of a weight block one after the other
  auto set_item = [&](int item) {
    const int blk = item / tiles_m, m0 = item % tiles_m * 16 * MI;
#pragma unroll
    for (int i = 0; i < 2 * MI; ++i) off_x[i] = (uint32_t)(((size_t)min(m0 + i * 8 + g_row, a.M - 1) * a.lda + chunk[i & 1] * 8) * 2);
#pragma unroll
    for (int i = 0; i < 2 * NI; ++i) {
      // rows beyond the last repeat it (a unit of eight is whole or beyond it altogether)
      const int row = min(first_row(blk * NI + i / 2) + (paired ? 0 : 8 * (i & 1)) + g_row, a.N - 1 - (epi == EPI_QKV ? second : 0)) +
                      (paired ? (i & 1) * second : 0);
      off_w[i] = (uint32_t)(((size_t)row * a.ldb + chunk[i & 1] * 8) * 2);
    }
  };
  const int nk = (a.K + BK - 1) / BK;
  const int n = nk > wave ? (nk - wave + 7) / 8 : 0;  // k-tiles of this wavefront per item
  const int mine = (n_items - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;
  const int total = n * mine;                       // k-tiles it will see
  int i_item = (int)blockIdx.x, i_k = 0, i_slot = 0, issued = 0;
  auto dma = [](const void *p, unsigned char *lds) {
    __builtin_amdgcn_global_load_lds(p, (__attribute__((address_space(3))) void *)lds, 16, 0, 0);
  };
  auto issue = [&]() __attribute__((always_inline)) {
    const int kt = wave + 8 * i_k;
    const unsigned char *bw = reinterpret_cast<const unsigned char *>(a.B) + (size_t)kt * 128;
    const unsigned char *bx = reinterpret_cast<const unsigned char *>(a.A) + (size_t)kt * 128;
    unsigned char *dst = ring + i_slot * R::STAGE;
    const int beyond = (kt + 1) * BK > a.K ? a.K - kt * BK : BK;  // first element of the k-tile that lies beyond K
    if (beyond == BK) {
#pragma unroll
      for (int i = 0; i < 2 * NI; ++i) dma(bw + off_w[i], dst + i * 1024);
#pragma unroll
      for (int i = 0; i < 2 * MI; ++i) dma(bx + off_x[i], dst + (2 * NI + i) * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < 2 * NI; ++i) dma(chunk[i & 1] * 8 >= beyond ? (const void *)g_gemm_zero_chunk : bw + off_w[i], dst + i * 1024);
#pragma unroll
      for (int i = 0; i < 2 * MI; ++i) dma(chunk[i & 1] * 8 >= beyond ? (const void *)g_gemm_zero_chunk : bx + off_x[i], dst + (2 * NI + i) * 1024);
    }
    ++issued;
    i_slot = i_slot + 1 == S ? 0 : i_slot + 1;
    if (++i_k == n) {
      i_k = 0;
      i_item += (int)gridDim.x;
      if (i_item < n_items) set_item(i_item);
    }
  };
  if (total > 0) set_item(i_item);
  for (int s = 0; s < S && issued < total; ++s) issue();

  // what the epilogue asks per row
  const int rows = tiles_m * 16 * MI;  // at most ROWS_MAX_M
  if (t < rows) {
    const int m = min(t, a.M - 1);
    if (epi == EPI_QKV) {
      meta_pos[t] = a.row_pos[m];
      meta_page[t] = a.row_page[m];
      meta_slot[t] = a.row_slot[m];
    }
    if (paired && !a.ss_in_parts) meta_rs[t] = a.rstd[m];
  }
  if (paired && a.ss_in_parts) {
    // the second norm's factor from the output projection's partial row sums: 512 / rows threads per row
    const int per_row = 512 / rows, r = t % rows, q = t / rows;
    float s = 0.f;
    if (q < per_row) {
#pragma unroll 8
      for (int p = q; p < a.ss_in_parts; p += per_row) s += a.ss_in[(size_t)p * a.ss_stride + min(r, a.M - 1)];
    }
    float *part = reinterpret_cast<float *>(red);
    part[t] = s;
    __syncthreads();
    if (t < rows) {
      s = 0.f;
      for (int i = 0; i < per_row; ++i) s += part[t + rows * i];
      meta_rs[t] = rsqrtf(s / (float)a.K + a.rstd_eps);
    }
    __syncthreads();
  }

  const int sw = (lr >> 1) & 7;
  int slot = 0, left = total, turn = 0;
  for (int item = (int)blockIdx.x; item < n_items; item += (int)gridDim.x, ++turn) {
    const int blk = item / tiles_m, m0 = item % tiles_m * 16 * MI;
    f32x4_t acc[NI][MI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) acc[ni][mi] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < n; ++k) {
      --left;  // k-tiles behind this one
      if (left >= S - 1) {
        __builtin_amdgcn_s_waitcnt(waitcnt_imm((S - 1) * L, false));
      } else {
        wait_for_all_but<L>(left, std::make_integer_sequence<int, S - 1>{});
      }
      const unsigned char *st = ring + slot * R::STAGE;
      bf16x8_t w[2][NI], x[2][MI];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const int ch = ((ks * 4 + lg) ^ sw) << 4;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) w[ks][ni] = as_bf16x8(*reinterpret_cast<const u32x4_t *>(st + ni * 2048 + lr * 128 + ch));
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) x[ks][mi] = as_bf16x8(*reinterpret_cast<const u32x4_t *>(st + (NI + mi) * 2048 + lr * 128 + ch));
      }
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(63, true));  // the slot may be filled again
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
          for (int mi = 0; mi < MI; ++mi) acc[ni][mi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][ni], x[ks][mi], acc[ni][mi], 0, 0, 0);
      if (left >= S) issue();
      slot = slot + 1 == S ? 0 : slot + 1;
    }
    // the partial sums of 16 weight rows at a time meet; the requests in flight are left alone
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(63, true));
      __builtin_amdgcn_s_barrier();  // nobody reads the sums before these any more
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) red[(wave * MI + mi) * 64 + lane] = acc[ni][mi];
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(63, true));
      __builtin_amdgcn_s_barrier();
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) {
        if (wave != ((turn * NI + ni) * MI + mi) % 8) continue;
        auto total_of = [&](int l) {
          f32x4_t s = red[mi * 64 + l];
#pragma unroll
          for (int v = 1; v < 8; ++v) s += red[(v * MI + mi) * 64 + l];
          return s;
        };
        const int ml = m0 + 16 * mi + lr;  // (at most ROWS_MAX_M - 1)
        const bool ok = ml < a.M;
        if (paired) {
          const int u = first_row(blk * NI + ni) + 4 * (lg & 1);  // first of this lane's four rows of the lower unit
          const f32x4_t lo = total_of(lane & 31) * meta_rs[ml], hi = total_of((lane & 31) + 32) * meta_rs[ml];
          if (!ok || lg > 1 || u >= a.N) continue;
          if (epi == EPI_SWIGLU) {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = lo[e] / (1.f + __expf(-lo[e])) * hi[e];
            store_bf16x4(a.C + (size_t)ml * a.ldc + u, v[0], v[1], v[2], v[3]);
          } else {
            const int head = u / dh, i0 = u % dh, half = dh / 2;
            const size_t tile_elems = (size_t)16 * dh, page = meta_page[ml];
            const int slot_in = meta_slot[ml];
            if (head < a.n_q_heads + a.n_kv_heads) {
              const size_t at = (size_t)meta_pos[ml] * half + i0;
              const f32x4_t cs = *reinterpret_cast<const f32x4_t *>(a.rope_cos + at), sn = *reinterpret_cast<const f32x4_t *>(a.rope_sin + at);
              const f32x4_t l = lo * cs - hi * sn, h = hi * cs + lo * sn;
              uint16_t *dst = head < a.n_q_heads
                                  ? a.q_out + (size_t)ml * (a.n_q_heads * dh) + head * dh
                                  : a.kv_pool + ((page * 2 + 0) * a.n_kv_heads + (head - a.n_q_heads)) * tile_elems + (size_t)slot_in * dh;
              store_bf16x4(dst + i0, l[0], l[1], l[2], l[3]);
              store_bf16x4(dst + half + i0, h[0], h[1], h[2], h[3]);
            } else {
              uint16_t *dst = a.kv_pool + ((page * 2 + 1) * a.n_kv_heads + (head - a.n_q_heads - a.n_kv_heads)) * tile_elems + slot_in;
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                dst[(i0 + e) * 16] = f32_to_bf16(lo[e]);
                dst[(i0 + half + e) * 16] = f32_to_bf16(hi[e]);
              }
            }
          }
        } else {
          f32x4_t v = total_of(lane);
          const int n0 = (blk * NI + ni) * 16 + 4 * lg;
          const bool in = ok && n0 < a.N;
          const size_t at = (size_t)ml * a.ldr + n0;
          if (in && epi == EPI_RESID && a.resid32) {
            v += *reinterpret_cast<const f32x4_t *>(a.resid32 + at);
          } else if (in && epi != EPI_PLAIN) {
            const u32x2_t rr = *reinterpret_cast<const u32x2_t *>(a.resid + at);
            v += f32x4_t{__uint_as_float(rr.x << 16), __uint_as_float(rr.x & 0xFFFF0000u), __uint_as_float(rr.y << 16), __uint_as_float(rr.y & 0xFFFF0000u)};
          }
          if (epi == EPI_RESID_NORM) {
            float ss = 0.f;
            if (in) {
              const u32x2_t gg = *reinterpret_cast<const u32x2_t *>(a.gain + n0);
              ss = v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
              *reinterpret_cast<f32x4_t *>(a.C32 + (size_t)ml * a.ldc + n0) = v;
              store_bf16x4(a.C_gain + (size_t)ml * a.ldc + n0, v[0] * __uint_as_float(gg.x << 16), v[1] * __uint_as_float(gg.x & 0xFFFF0000u),
                           v[2] * __uint_as_float(gg.y << 16), v[3] * __uint_as_float(gg.y & 0xFFFF0000u));
            }
            ss += __shfl_xor(ss, 16, 64);
            ss += __shfl_xor(ss, 32, 64);
            if (lg == 0 && in) a.ss_out[(size_t)(blk * NI + ni) * a.ss_stride + ml] = ss;
          } else if (in) {
            store_bf16x4(a.C + (size_t)ml * a.ldc + n0, v[0], v[1], v[2], v[3]);
          }
        }
    }
    }
  }
}

template <int MI, int NI>
hipError_t launch_rows_one(const GemmArgs &a, int epi, int dh, hipStream_t stream) {
  typedef RowsKernel<MI, NI> R;
  const int n_cu = a.n_cu > 0 ? a.n_cu : 256, tiles_m = (a.M + 16 * MI - 1) / (16 * MI);
  if (tiles_m * 16 * MI > ROWS_MAX_M || a.N % 8) return hipErrorInvalidValue;
  const long items = (long)tiles_m * ((rows_blocks(a.N, epi) + NI - 1) / NI), rounds = (items + n_cu - 1) / n_cu;
  if (items <= 0 || items >= (1L << 30)) return hipErrorInvalidValue;
  auto kern = gemm_rows_kernel<MI, NI>;
  static OncePerDevice once;
  if (const hipError_t e = allow_lds(once, reinterpret_cast<const void *>(kern), R::LDS)) return e;
  // as many workgroups as give each the same number of items
  hipLaunchKernelGGL(kern, dim3((unsigned)((items + rounds - 1) / rounds)), dim3(512), R::LDS, stream, a, epi, dh, tiles_m, (int)items);
  return hipGetLastError();
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int DH, int DEEP = 0>
hipError_t launch_one(const GemmArgs &a, hipStream_t stream) {
  constexpr int OUT_BN = (EPI == EPI_SWIGLU) ? BN / 2 : BN;
  constexpr int LDS = DEEP ? LDS_CU : ring_bytes(WAVES_M * WAVES_N);
  auto kern = gemm_kernel<BM, BN, WAVES_M, WAVES_N, EPI, DH, DEEP>;
  static OncePerDevice once;
  if (const hipError_t e = allow_lds(once, reinterpret_cast<const void *>(kern), LDS)) return e;
  const int n_cols = a.n_count ? a.n_count : a.N;
  const int tiles = ((a.M + BM - 1) / BM) * ((n_cols + OUT_BN - 1) / OUT_BN) * (EPI == EPI_PARTIAL ? a.k_splits : 1);
  if (tiles <= 0) return hipSuccess;
  hipLaunchKernelGGL(kern, dim3(tiles), dim3(WAVES_M * WAVES_N * 64), LDS, stream, a);
  return hipGetLastError();
}

constexpr int SK_MAX_G = 256;  // workgroups of a shared-tile launch at most: one per CU

template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int DH>
hipError_t launch_sk(const GemmArgs &a, hipStream_t stream) {
  constexpr int OUT_BN = (EPI == EPI_SWIGLU) ? BN / 2 : BN;
  constexpr int LDS = ring_bytes(WAVES_M * WAVES_N);
  static_assert(BM == 256 && BN == 256, "the workspace slots are sized for 256x256 tiles");
  if (!a.sk_ws || !a.sk_cnt || a.n_count || a.k_splits > 1) return hipErrorInvalidValue;
  auto kern = gemm_sk_kernel<BM, BN, WAVES_M, WAVES_N, EPI, DH>;
  static OncePerDevice once;
  if (const hipError_t e = allow_lds(once, reinterpret_cast<const void *>(kern), LDS)) return e;
  const long tiles = (long)((a.M + BM - 1) / BM) * ((a.N + OUT_BN - 1) / OUT_BN);
  if (tiles <= 0) return hipSuccess;
  const int G = a.n_cu > 0 && a.n_cu < SK_MAX_G ? a.n_cu : SK_MAX_G;
  SkPlan p{};
  p.nk = (a.K + BK - 1) / BK;
  p.ws = a.sk_ws;
  p.cnt = a.sk_cnt;
  if (tiles % G == 0) {
    p.n_dp = (int)tiles;
  } else {
    // (with more than one round the last whole round is shared too: every workgroup then has more
    // than a tile's worth of iterations and at most two cuts)
    p.n_sk = tiles > G ? (int)(tiles % G) + G : (int)tiles;
    p.n_dp = (int)tiles - p.n_sk;
    const long total = (long)p.n_sk * p.nk;
    p.g_sk = (int)std::min<long>(G, std::max<long>(1, total / SK_MIN_ITERS));
    if (total * p.g_sk >= (1L << 31)) return hipErrorInvalidValue;
  }
  const int grid = (int)std::min<long>(G, std::max<long>(p.g_sk, p.n_dp));
  hipLaunchKernelGGL(kern, dim3(grid), dim3(WAVES_M * WAVES_N * 64), LDS, stream, a, p);
  return hipGetLastError();
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int ADH>
hipError_t launch_ride(const GemmArgs &a, const GemmRide &r, hipStream_t stream) {
  constexpr int OUT_BN = (EPI == EPI_SWIGLU) ? BN / 2 : BN;
  constexpr int LDS = ring_bytes(WAVES_M * WAVES_N);
  static_assert(LDS == LDS_CU, "a workgroup of either kind must take the whole LDS of its CU");
  auto kern = gemm_attn_kernel<BM, BN, WAVES_M, WAVES_N, EPI, 64, ADH>;
  static OncePerDevice once;
  if (const hipError_t e = allow_lds(once, reinterpret_cast<const void *>(kern), LDS)) return e;
  const int tiles = ((a.M + BM - 1) / BM) * ((a.N + OUT_BN - 1) / OUT_BN);
  if (tiles <= 0) return hipErrorInvalidValue;
  // (a negative margin: no tile closes the queue, the launch drains it)
  const int close_at = r.close_margin < 0 ? tiles + 1 : (tiles - r.close_margin > 1 ? tiles - r.close_margin : 1);
  hipLaunchKernelGGL(kern, dim3(r.head + tiles + r.tail), dim3(WAVES_M * WAVES_N * 64), LDS, stream, a, r, tiles,
                     (unsigned)close_at);
  return hipGetLastError();
}

// Tile shapes.  BIG: 256x256, 8 wavefronts.  TALL: 160x256, 8 wavefronts of 80x64: 2560 (and
// 5120) rows by 4096 (8192) columns then make exactly one (four) full rounds of 256
// workgroups where 256x256 tiles leave 38 % (17 %) of the CUs idle.  SMALL: 128x128.
// S128 / S256: 128x256 and 256x128 tiles on the deep weight ring, for at most 128 / 256 rows; D64 / D128: 64x128 and
// 128x128 tiles on it, for whole products of at most 64 / 128 rows.  MID: 192x256, 8 wavefronts of 96x64; WIDE: 128x256, 8 of 64x64.
// activation slots of the short-row pipeline, minus one: three slots leave four weight slots of 16 KB
// (256x128) or three of 32 KB (128x256); measured against two slots (six / four weight slots) on the
// 256-row gate/up GEMM of the 8B layer: 0.075 against 0.078 ms, the other GEMMs the same
constexpr int DEEP_X = 2;
enum { V_AUTO = 0, V_BIG = 1, V_TALL = 2, V_SMALL = 3, V_S128 = 4, V_S256 = 5, V_SHARED = 6, V_ROWS = 7, V_D64 = 8, V_D128 = 9, V_MID = 10, V_WIDE = 11 };
constexpr int N_CU = 256;

thread_local int g_forced_variant = V_AUTO;  // set by the calling entry point from its context, for the launches of that call

long n_tiles(int m, int n, int bm, int bn) { return (long)((m + bm - 1) / bm) * ((n + bn - 1) / bn); }

// few rows: one tile row on the deep weight ring (0 where the rows do not fit one tile, or a shape is forced)
int short_variant(int m) {
  if (g_forced_variant != V_AUTO || m > 256) return 0;
  return m <= 128 ? V_S128 : V_S256;
}

// The few-row kernel's item, as 10 MI + NI (0: the tiles are the better choice, or a shape is forced).  Up to 16 rows it is
// ahead everywhere (70B down projection at 16 rows 88 against 86 us, the one exception).  Beyond, the activation rows of an
// item outweigh its weights: it needs one round of items (gate/up two, which saves nothing else) over a short K, or its
// eight wavefronts hold too little of K in flight.  Measured at 32 rows against the tiles, both with cold
// weights: N = 3072, K = 2048 QKV 7.2 against 12.2 us, N = K = 4096 output projection 11.3 against 15.9, N = 2048,
// K = 8192 down 16.3 against 17.7; N = 4096, K = 14336 31 against 28.5; gate/up of 2 x 8192 columns, K = 2048 17 against 24.8,
// of 2 x 14336, K = 4096 51.5 against 54 for shallow tiles.  Above 64 rows only where a wavefront has one k-tile or two:
// 136 rows, N = 512, K = 256 5 against 10.5 us; N = 256, K = 688 5 against 12.
int rows_item(int m, int n, int k, int epilogue, int n_cu) {
  if (g_forced_variant != V_AUTO || m > ROWS_MAX_M || n % 8) return 0;
  const long nk = (k + BK - 1) / BK, blocks = rows_blocks(n, epilogue);
  if (m <= 16) return 11;
  const long tiles_m = (m + 31) / 32, longest = m <= 64 ? 128 : 12;
  if (nk > longest) return 0;
  if (tiles_m * blocks <= n_cu) return 21;
  const long rounds = epilogue == EPI_SWIGLU && m <= 32 ? 2 : 1;
  return tiles_m * ((blocks + 1) / 2) <= rounds * n_cu ? 22 : 0;
}

// Estimated time of a product in microseconds.  A k-tile costs between `lo` (few workgroups on the chip) and `hi` (all of
// them: the clock falls under matrix load); 128x128 tiles, two to a CU, cost `lo` up to one per CU.  A round of whole tiles
// has its start and its epilogue (`round`), a cut product the second kernel and the partial products once out and once back
// in (most of it the last-level cache); the output projection whole needs the pass that closes the second norm.
// Fitted on MI355X to the products of eight layers (QKV, output, gate/up and down projections, 1024 to 57344 columns, K 1024
// to 28672) at 26 row counts each, those above 512, weights cold, every shape and cut timed: 2.7 % from the times that matter.
struct Shape {
  int v, bm, bn, per_cu;
  double hi, lo, round[4];  // QKV, output projection, down projection, gate/up
};
constexpr Shape SHAPES[5] = {{V_BIG, 256, 256, 1, 1.44, 0.81, {11.6, 19.7, 18.5, 9.5}},
                             {V_TALL, 160, 256, 1, 0.97, 0.65, {8.6, 11.7, 7.7, 6.6}},
                             {V_SMALL, 128, 128, 2, 0.95, 0.51, {6.5, 8.4, 5.0, 4.0}},
                             {V_MID, 192, 256, 1, 1.13, 0.72, {9.2, 13.7, 11.3, 7.6}},
                             {V_WIDE, 128, 256, 1, 0.85, 0.58, {7.6, 10.1, 5.9, 5.9}}};
constexpr double TWO_PER_CU = 0.65, CLOSING_US = 4.5, SECOND_US[3] = {10.4, 10.3, 7.3}, PARTIAL_BYTES_US = 7.0e6;
constexpr int FIT_MIN_K = 1024;

// k-tiles of one workgroup after the other over `tiles` workgroups of the shape, in microseconds
double rounds_us(const Shape &c, long tiles, double hi, double lo, double two, int n_cu) {
  const long slots = (long)n_cu * c.per_cu, full = tiles / slots, rem = tiles % slots;
  double part = 0.0;
  if (rem && c.per_cu == 1) part = lo + (hi - lo) * (double)rem / (double)slots;
  else if (rem) part = rem <= n_cu ? lo : lo + (hi - lo) * (two + (1.0 - two) * (double)(rem - n_cu) / (double)n_cu);
  return (double)full * hi + part;
}
int epi_column(int epilogue) { return epilogue == EPI_QKV ? 0 : epilogue == EPI_RESID_NORM ? 1 : epilogue == EPI_SWIGLU ? 3 : 2; }
double whole_us(const Shape &c, int m, int n, int k, int n_cu, int epilogue) {
  const long tiles = n_tiles(m, n, c.bm, c.bn), slots = (long)n_cu * c.per_cu;
  return (double)((k + BK - 1) / BK) * rounds_us(c, tiles, c.hi, c.lo, TWO_PER_CU, n_cu) +
         c.round[epi_column(epilogue)] * (double)((tiles + slots - 1) / slots) + (epilogue == EPI_RESID_NORM ? CLOSING_US : 0.0);
}
double cut_us(const Shape &c, int m, int n, int k, int s, int n_cu, int epilogue) {
  const long nk = (k + BK - 1) / BK;
  return (double)((nk + s - 1) / s) * rounds_us(c, n_tiles(m, n, c.bm, c.bn) * s, c.hi, c.lo, TWO_PER_CU, n_cu) +
         SECOND_US[epi_column(epilogue)] + 8.0 * s * m * n / PARTIAL_BYTES_US;
}

// Columns of 256x256 tiles that fill whole rounds where the last round leaves more than a quarter of the chip idle, else 0.
long round_split_columns(long tm, long tn, int n_cu) {
  const long tiles = tm * tn, full = tiles / n_cu, idle = (full + 1) * n_cu - tiles, cols = full * n_cu / tm;
  return full < 1 || tiles % n_cu == 0 || idle * 4 <= n_cu || cols < 1 || cols >= tn ? 0 : cols;
}

// What the second launch of a product in two costs beside its rounds.  Of 386 gate/up products of eight layers, timed in steps whole and
// in two launches, the choice is 0.3 % off the best on average and 4 % at most with 2 to 3; with none, products of 45 to 80 us
// went out as two launches for an expected 2 us and took 3 to 6 more (K = 1024, 2 x 4096 columns, 2056 rows: 48.0 us, whole 42.3).
constexpr double SECOND_LAUNCH_US = 2.0;

// Gate/up of more than 512 rows: the shape with the smallest estimate, and that estimate.  *cols: 0, or the columns of 256x256 tiles
// that go out in whole rounds of their own, the rest behind them on 128x128 tiles, where that is expected to be shorter than whole
// (timed both ways, 8B layer: 1160 rows 254 us whole, 237 in two launches; 3300 rows 553 and 570).  Of 182 products of seven layers timed
// with cold weights it is 0.6 % off the best on average.  1580 rows of the 8B layer: 192x256 tiles 330 us, 160x256 tiles, faster
// since they have three activation panels, 316.  (Below K = 1024, where nothing was fitted, the relation of rounds in choose_variant.)
double gate_up_us(int m, int n_b_rows, int k, int n_cu, int *v, int *cols) {
  double best_t = 1e300;
  auto offer = [&](double t, int variant, int columns) {
    if (t < best_t) { best_t = t; *v = variant; *cols = columns; }
  };
  for (const Shape &c : SHAPES) offer(whole_us(c, m, n_b_rows, k, n_cu, EPI_SWIGLU), c.v, 0);
  const int split = (int)round_split_columns((m + 255) / 256, (n_b_rows + 255) / 256, n_cu);
  if (split)
    offer(whole_us(SHAPES[0], m, split * 256, k, n_cu, EPI_SWIGLU) + whole_us(SHAPES[2], m, n_b_rows - split * 256, k, n_cu, EPI_SWIGLU) +
              SECOND_LAUNCH_US, V_BIG, split);
  return best_t;
}

// Two shapes for one product: whole rounds of one of the 256-wide shapes over the first `cols` tile columns, another shape, whose
// rounds the rest happens to fill, over the others.  Taken where the estimate of the two launches is 3 % below the best single
// choice, about its own error.  Measured in steps, 8B layer: 776 rows 192 us on one shape, 170 as one round of 160x256 tiles and
// 256x256 ones for the rest; 1288 rows 269 -> 251.
bool gate_up_pair(int m, int n_b_rows, int k, int n_cu, int *head, int *tail, int *cols) {
  int single, single_cols;
  double best_t = 0.97 * gate_up_us(m, n_b_rows, k, n_cu, &single, &single_cols);
  bool found = false;
  for (const Shape &c : SHAPES) {
    if (c.bn != 256) continue;
    const long tm = (m + c.bm - 1) / c.bm, tn = (n_b_rows + 255) / 256, full = tm * tn / n_cu;
    for (long f = std::max(1L, full - 2); f <= full; ++f) {
      const long n = f * n_cu / tm;
      if (n < 1 || n >= tn) continue;
      const double t = whole_us(c, m, (int)n * 256, k, n_cu, EPI_SWIGLU) + SECOND_LAUNCH_US;
      for (const Shape &c2 : SHAPES) {
        const double t2 = t + whole_us(c2, m, n_b_rows - (int)n * 256, k, n_cu, EPI_SWIGLU);
        if (t2 >= best_t) continue;
        best_t = t2;
        *head = c.v;
        *tail = c2.v;
        *cols = (int)n;
        found = true;
      }
    }
  }
  return found;
}

// Tile shape of a gate/up or plain product, or of any with a forced shape (QKV, output and down projection:
// gemm_plan).
// Gate/up of more than 512 rows goes by the estimate in microseconds (gate_up_us), the others by that of a launch in
// units of one full round of 256x256 tiles: full rounds of
// workgroups (the 128x128 tile runs two per CU) cost T each; a last, partly filled round costs
// T (a + (1 - a) fill): workgroups that share the chip with fewer others run faster, but not in
// proportion.  T and a were fitted on MI355X to the four GEMM shapes of the 8B layer at 384 to
// 2560 rows (the 160x256 tile: 0.072 ms per full round at K = 4096 where the 256x256 tile takes
// 0.100 and 512 tiles of 128x128 take 0.075).
// share_k: the contraction length if the launch may share tiles between workgroups (it has the
// workspace for it and covers all columns), else 0
int choose_variant(int m, int n_b_rows, int k, int epilogue, int dh, int n_cu, int share_k = 0) {
  if (n_cu <= 0) n_cu = N_CU;
  if (g_forced_variant != V_AUTO && !(g_forced_variant == V_TALL && epilogue == EPI_QKV)) return g_forced_variant;
  (void)dh;
  // Few rows that the few-row kernel leaves: measured, cold weights, against 128x128 tiles on the shallow ring, 64 (90, 128)
  // rows: 2 x 14336 columns, K = 4096 54.9 -> 44.1 (55.9 -> 48.9, 57.2 -> 52.4) us; 2 x 8192, K = 3072 34.9 -> 31.0
  // (35.9 -> 35.0, 37.8 -> 37.5); 2 x 13824, K = 5120 60.9 -> 55.7 (62.5 -> 61.5, 66.3 -> 66.1); 2 x 4096, K = 1024
  // 13.7 -> 11.8 (14.0 -> 13.5, 14.4 -> 14.3); of more than one round only at 64 rows: 2 x 28672, K = 8192 165 -> 162
  // (128x128 tiles 179 against 162 of 128x256).
  if (g_forced_variant == V_AUTO && m <= 128 && (epilogue == EPI_SWIGLU || epilogue == EPI_PLAIN)) {
    if (m <= 64) return V_D64;
    if (n_tiles(m, n_b_rows, 128, 128) <= n_cu) return V_D128;
  }
  if (const int sv = short_variant(m); sv && (epilogue == EPI_SWIGLU || epilogue == EPI_PLAIN)) {
    // worth it once the single row of tiles fills at least half the chip
    if (2 * n_tiles(m, n_b_rows, sv == V_S128 ? 128 : 256, sv == V_S128 ? 256 : 128) >= n_cu) return sv;
  }
  const bool estimated = epilogue == EPI_SWIGLU && g_forced_variant == V_AUTO && k >= FIT_MIN_K;
  if (estimated && m > 512) {
    int best, cols;
    gate_up_us(m, n_b_rows, k, n_cu, &best, &cols);
    return best;
  }
  struct Cand { int v, bm, bn, per_cu; double T, a; };
  // 192x256 tiles (gate/up) fetch a tenth less per flop than 160x256 ones, and waste fewer rows than 256x256 where the
  // rows end early in a tile.  T and a from the gate/up products of three layers at 44 row counts from 257 to 4096,
  // every shape timed with cold weights, before 160x256 tiles had a third activation panel.  2 x 14336 columns, K = 4096:
  // 359 rows 97 -> 91 us (256x256); 2 x 8192, K = 2048: 359 rows 43 against 36 of 128x128.
  const Cand cands[4] = {{V_BIG, 256, 256, 1, 1.00, 0.72}, {V_TALL, 160, 256, 1, 0.76, 0.65}, {V_SMALL, 128, 128, 2, 0.75, 0.60},
                         {V_MID, 192, 256, 1, 0.85, 0.75}};
  int best = V_SMALL;
  double best_t = 1e300;
  for (const Cand &c : cands) {
    if (c.v == V_TALL && epilogue == EPI_QKV) continue;  // (QKV comes here for forced shapes alone, which do not force it to 160x256)
    if (c.v == V_MID && epilogue != EPI_SWIGLU) continue;
    const long tiles = n_tiles(m, n_b_rows, c.bm, c.bn);
    const long slots = (long)n_cu * c.per_cu;
    const long full = tiles / slots, rem = tiles % slots;
    const double t = (double)full * c.T + (rem ? c.T * (c.a + (1.0 - c.a) * (double)rem / (double)slots) : 0.0);
    if (t < best_t) { best_t = t; best = c.v; }
  }
  // Up to 512 rows 128x256 tiles where the estimate puts them ahead of that choice: 2 x 8192 columns, K = 2048 at 359 rows
  // 37.1 us on 128x128 tiles, 33.5 on these; 5 % on average over 51 products of 257 to 512 rows, and none slower than that
  // choice, though 128x128 tiles would be ahead of both where N and K are small (2 x 4096, K = 1024 at 308 rows 13.1 us
  // against 17.9, and 20.7 on 160x256 ones).
  if (estimated && m > 256) {
    for (const Shape &c : SHAPES)
      if (c.v == best && whole_us(SHAPES[4], m, n_b_rows, k, n_cu, EPI_SWIGLU) < whole_us(c, m, n_b_rows, k, n_cu, EPI_SWIGLU)) return V_WIDE;
  }
  // Shared 256x256 tiles: the chip's worth of k-tile iterations with nothing idle, 3 % for the
  // persistent loop, and what the cuts cost: a workgroup passes up to two partial tiles through
  // memory, about 0.08 ms per launch whatever its size (measured on the GEMMs of the 8B and 70B
  // layers), i.e. 53 k-tiles' worth of a round.  It pays only where K is long.
  if (share_k >= 4096 && m > 256) {
    const long tiles = n_tiles(m, n_b_rows, 256, 256);
    const long g = std::min<long>(n_cu, N_CU);
    if (tiles % g) {
      const double t = (double)tiles / (double)g * 1.03 + 53.0 / (double)((share_k + BK - 1) / BK);
      if (t < best_t) { best_t = t; best = V_SHARED; }
    }
  }
  return best;
}

template <int EPI>
hipError_t launch_variant(const GemmArgs &a, int v, hipStream_t stream) {
  if (v == V_BIG) return launch_one<256, 256, 2, 4, EPI, 64>(a, stream);
  if (v == V_SHARED) return launch_sk<256, 256, 2, 4, EPI, 64>(a, stream);
  if (v == V_TALL) return launch_one<160, 256, 2, 4, EPI, 64>(a, stream);
  if constexpr (EPI == EPI_SWIGLU || EPI == EPI_PLAIN) {
    if (v == V_D64) return launch_one<64, 128, 4, 2, EPI, 64, DEEP_X>(a, stream);
    if (v == V_D128) return launch_one<128, 128, 4, 2, EPI, 64, DEEP_X>(a, stream);
    if (v == V_S128) return launch_one<128, 256, 2, 4, EPI, 64, DEEP_X>(a, stream);
    if (v == V_S256) return launch_one<256, 128, 4, 2, EPI, 64, DEEP_X>(a, stream);
  }
  if constexpr (EPI != EPI_PLAIN) {  // (no plain product is given these)
    if (v == V_MID) return launch_one<192, 256, 2, 4, EPI, 64>(a, stream);
    if (v == V_WIDE) return launch_one<128, 256, 2, 4, EPI, 64>(a, stream);
  }
  return launch_one<128, 128, 2, 2, EPI, 64>(a, stream);
}

template <int DH>
hipError_t launch_qkv(const GemmArgs &a, int v, hipStream_t stream) {
  if (v == V_SHARED) return launch_sk<256, 256, 2, 4, EPI_QKV, DH>(a, stream);
  if (v == V_BIG) return launch_one<256, 256, 2, 4, EPI_QKV, DH>(a, stream);
  if (v == V_TALL) return launch_one<160, 256, 2, 4, EPI_QKV, DH>(a, stream);
  if (v == V_MID) return launch_one<192, 256, 2, 4, EPI_QKV, DH>(a, stream);
  if (v == V_WIDE) return launch_one<128, 256, 2, 4, EPI_QKV, DH>(a, stream);
  return launch_one<128, 128, 2, 2, EPI_QKV, DH>(a, stream);
}

}  // namespace

void gemm_force_variant(int v) { g_forced_variant = v; }
size_t gemm_sk_workspace_floats() { return (size_t)2 * SK_MAX_G * 256 * 256; }
int gemm_sk_counters() { return 2 * SK_MAX_G; }

bool gemm_streams_weights(const GemmArgs &a, int epilogue) {
  return !a.n_count && a.k_splits <= 1 && rows_item(a.M, a.N, a.K, epilogue, a.n_cu > 0 ? a.n_cu : N_CU) != 0;
}

bool gemm_round_split(const GemmArgs &a, int epilogue, int dh, GemmArgs *head, GemmArgs *tail) {
  if (epilogue != EPI_SWIGLU || g_forced_variant != V_AUTO || a.k_splits > 1) return false;
  const int n_cols = a.n_count ? a.n_count : a.N;
  if (gemm_streams_weights(a, epilogue)) return false;
  const int n_cu = a.n_cu > 0 ? a.n_cu : N_CU;
  int first, rest, cols;
  const bool estimated = a.M > 512 && a.K >= FIT_MIN_K;
  if (!estimated || !gate_up_pair(a.M, 2 * n_cols, a.K, n_cu, &first, &rest, &cols)) {
    if (estimated) {
      gate_up_us(a.M, 2 * n_cols, a.K, n_cu, &first, &cols);
    } else {
      if (choose_variant(a.M, 2 * n_cols, a.K, epilogue, dh, a.n_cu) != V_BIG) return false;
      cols = (int)round_split_columns((a.M + 255) / 256, (n_cols + 127) / 128, n_cu);  // a 256x256 tile yields 128 output columns
    }
    if (!cols) return false;
    first = V_BIG;
    rest = V_SMALL;  // two workgroups per CU fill the chip best with what is left of a round
  }
  *head = a;
  *tail = a;
  head->n_count = cols * 128;
  tail->n_begin = a.n_begin + head->n_count;
  tail->n_count = n_cols - head->n_count;
  head->tile_variant = first;
  tail->tile_variant = rest;
  return true;
}

void gemm_plan(GemmArgs &a, int epilogue) {
  a.k_splits = 1;
  const int n_cu = std::min(a.n_cu > 0 ? a.n_cu : N_CU, N_CU);
  if (gemm_streams_weights(a, epilogue)) {
    a.tile_variant = V_ROWS;
    return;
  }
  const long nk = (a.K + BK - 1) / BK;
  const size_t room = a.sk_ws && a.N % 4 == 0 ? gemm_sk_workspace_floats() : 0;
  // k-ranges of at least eight k-tiles, one round of workgroups, partial products that fit the workspace
  auto max_splits = [&](long tiles, long slots) {
    long s = std::min<long>(std::min<long>(MAX_SPLITS, nk / 8), slots / tiles);
    while (s > 1 && (size_t)s * a.M * a.N > room) --s;
    return std::max<long>(s, 1);
  };
  const bool may_share = a.sk_ws && a.sk_cnt && !a.n_count;
  if (g_forced_variant != V_AUTO) {
    a.tile_variant = choose_variant(a.M, a.N, a.K, epilogue, 0, a.n_cu, may_share ? a.K : 0);
    if (a.tile_variant == V_SMALL) a.k_splits = (int)max_splits(n_tiles(a.M, a.N, 128, 128), 2L * n_cu);
    return;
  }
  // At most 256 rows: the weights stream from HBM, so what counts is how many workgroups ask for them.
  // One row of tiles on the deep weight ring, cut along K until there is one workgroup per CU; of 128
  // rows and less, 128x128 tiles where MAX_SPLITS ranges of the 256-wide ones would leave a quarter of
  // the CUs without one (measured with cold weights, 64 rows, reduction included: K = 14336, N = 4096,
  // 128 workgroups of 128x256 35 us, 256 of 128x128 30; K = N = 8192, 192 of 128x256 34, 128x128 37).
  if (a.M <= 256) {
    const bool s128 = a.M <= 128;
    const long tiles = s128 ? n_tiles(a.M, a.N, 128, 256) : n_tiles(a.M, a.N, 256, 128);
    const long s = max_splits(tiles, n_cu);
    if (s >= 2 && (!s128 || 4 * s * tiles > 3 * n_cu)) {
      a.tile_variant = s128 ? V_S128 : V_S256;
      a.k_splits = (int)s;
      return;
    }
    const long small = n_tiles(a.M, a.N, 128, 128), ss = max_splits(small, n_cu);
    if (s128 && ss >= 2) {
      a.tile_variant = V_SMALL;
      a.k_splits = (int)ss;
      return;
    }
  }
  // Above, up to 1024 rows: the estimate of an earlier fit (the same terms, 256x256, 160x256 and 128x128 tiles, the products
  // of twelve layers of 256 to 12288 columns and K 256 to 28672, before the requests of the main loop were dealt out).  With the
  // present kernels its choices are 3.5 % off the best of all shapes and cuts on average over 293 products, 74 of them by more than
  // 5 % and the worst by 33 (down projection, N = 3072, K = 8192 at 667 rows: 256x256 tiles in seven ranges 60.8 us, 45.7 on 160x256
  // tiles in four).  The present fit over these three shapes gives no more; 192x256 and 128x256 tiles, cut, are not offered here.
  struct Earlier { double round, second, closing; };
  const Earlier ep = epilogue == EPI_QKV ? Earlier{7.1, 5.2, 0.0} : epilogue == EPI_RESID_NORM ? Earlier{6.7, 7.4, 4.0} : Earlier{5.7, 4.0, 0.0};
  constexpr double PARTIAL_ROUND = 5.0, PARTIAL_BYTES_PER_US = 6.4e6, HI[3] = {1.35, 1.05, 1.03}, LO[3] = {1.09, 1.06, 0.63};
  double best = 1e300;
  auto offer = [&](double t, int v, long s) {
    if (t < best) { best = t; a.tile_variant = v; a.k_splits = (int)s; }
  };
  const bool few = a.M <= 1024;
  for (int i = 0; few && i < 3; ++i) {
    const Shape &c = SHAPES[i];
    const long tiles = n_tiles(a.M, a.N, c.bm, c.bn), slots = (long)n_cu * c.per_cu;
    for (long s = 1; s <= max_splits(tiles, slots); ++s) {
      if (s == 1 && c.v == V_TALL && epilogue == EPI_QKV) continue;
      double t = (double)((nk + s - 1) / s) * rounds_us(c, tiles * s, HI[i], LO[i], 0.59, n_cu) +
                 (s > 1 ? PARTIAL_ROUND : ep.round) * (double)((tiles * s + slots - 1) / slots);
      t += s > 1 ? ep.second + 8.0 * (double)s * a.M * a.N / PARTIAL_BYTES_PER_US : ep.closing;
      offer(t, c.v, s);
    }
  }
  // QKV of 513 to 1024 rows: whole 160x256, 192x256 and 128x256 tiles against that choice by the present fit (8B layer,
  // 1024 rows: 256x256 tiles in two ranges 64.8 us, 128x256 whole 55.4; 3.4 % on average over 49 products, 2.8 % slower at worst).
  // Above 1024 rows every shape, whole and cut: against the earlier fit's choices QKV is 6.2 % faster on average over 136 products (5.3 %
  // slower at worst, 41.4 -> 43.6 us), output projection 3.5 % over 135 (9 %, 19.6 -> 21.4), down projection 4.9 % over 134 (2 %), and
  // 1.3, 0.3 and 0.2 % off the best (8B layer, 1580 rows: QKV 80 us on 256x256 tiles, 68 on 160x256; output projection 69.5 on
  // 256x256 tiles in two ranges, 61 on 128x256 whole.  70B layer, 5120 rows: QKV 721 on shared tiles, 636 on 160x256).  Of more
  // than one round QKV stays off 192x256 and 128x256 tiles, which would be ahead in 13 of the 136 by more than 5 % (70B layer,
  // 2207 rows 332 us against 309; 8B layer, 3644 rows 183 against 159; N = 3072, K = 2048 at 7000 rows 103 against 86): a
  // test holds the division of 2200 rows of the 70B layer to whole 256x256 tiles.
  if (!few || (epilogue == EPI_QKV && a.M > 512)) {
    if (few) {
      const Shape &c = SHAPES[a.tile_variant - V_BIG];  // one of the first three, numbered alike
      best = a.k_splits > 1 ? cut_us(c, a.M, a.N, a.K, a.k_splits, n_cu, epilogue) : whole_us(c, a.M, a.N, a.K, n_cu, epilogue);
    }
    for (const Shape &c : SHAPES) {
      const long tiles = n_tiles(a.M, a.N, c.bm, c.bn), slots = (long)n_cu * c.per_cu;
      const bool added = c.v == V_MID || c.v == V_WIDE;
      if (epilogue == EPI_QKV && added && tiles > slots) continue;
      if (few && !added && c.v != V_TALL) continue;
      offer(whole_us(c, a.M, a.N, a.K, n_cu, epilogue), c.v, 1);
      for (long s = 2; !few && s <= max_splits(tiles, slots); ++s) offer(cut_us(c, a.M, a.N, a.K, (int)s, n_cu, epilogue), c.v, s);
    }
  }
  // Shared 256x256 tiles: the chip's worth of k-tile iterations with nothing idle, and 22 us for the cuts (a
  // workgroup passes up to two partial tiles through memory).  Only where K is long, more than one round of tiles cannot be
  // cut evenly, and the tiles beyond whole rounds are a multiple of a quarter round: else the workgroups walk K in
  // eight and more phases and share few panels in L2 (QKV of 12288 columns, K = 4096, 5600 rows: 522 us, 461 on whole
  // 256x256 tiles; down projection of the 70B layer, 6695 rows: 2847 against 2581; of 124 such products two are
  // ahead of the best other choice, by 1 %, and all are 31 % behind it on average).  Four phases cost 4 % more per k-tile than one
  // or two.  Fitted to the 67 products of up to four phases in steps of six layers; it takes the eleven on which these tiles
  // are ahead: 70B down projection of 5120 rows 1760 us (1828 on the best other tiles), of 7012 rows 2454 (2608), N = 5120,
  // K = 13824 at 4029 rows 452 (484).
  if (may_share && a.K >= 4096 && a.M > 256) {
    const long tiles = n_tiles(a.M, a.N, 256, 256), rem = tiles % n_cu, phases = rem ? n_cu / std::gcd((long)n_cu, rem) : 1;
    const double t = (double)nk * (phases <= 2 ? 1.49 : 1.545) * (double)tiles / (double)n_cu + 22.0 +
                     SHAPES[0].round[epi_column(epilogue)] * (double)((tiles + n_cu - 1) / n_cu);
    if (rem && tiles > n_cu && phases <= 4 && t < best) { a.tile_variant = V_SHARED; a.k_splits = 1; }
  }
}

int gemm_shape(const GemmArgs &a, int epilogue, int dh) {
  if (a.tile_variant) return a.tile_variant;
  if ((epilogue == EPI_SWIGLU || epilogue == EPI_PLAIN) && gemm_streams_weights(a, epilogue)) return V_ROWS;
  const int n_cols = a.n_count ? a.n_count : a.N;
  return choose_variant(a.M, epilogue == EPI_SWIGLU ? 2 * n_cols : n_cols, a.K, epilogue, dh, a.n_cu, a.sk_ws && a.sk_cnt && !a.n_count ? a.K : 0);
}

int gemm_ss_parts(const GemmArgs &a, int epilogue, int dh) {
  if (a.k_splits > 1) return 1;  // the split-K reduction leaves whole row sums
  const int v = a.tile_variant ? a.tile_variant
                               : choose_variant(a.M, a.N, a.K, epilogue, dh, a.n_cu, a.sk_ws && a.sk_cnt && !a.n_count ? a.K : 0);
  if (v == V_ROWS) return (a.N + 15) / 16;  // one per block of 16 columns
  // partial row sums: one per (column tile, wavefront column)
  return v == V_SMALL ? ((a.N + 127) / 128) * 2 : ((a.N + 255) / 256) * 4;
}

int gemm_ride_variant(int m, int n_b_rows, int n_cu) {
  // the eight-wavefront tiles only: 256x256 or 160x256, by the same cost model of rounds
  struct Cand { int v, bm; double T, a; };
  const Cand cands[2] = {{V_BIG, 256, 1.00, 0.72}, {V_TALL, 160, 0.76, 0.65}};
  if (n_cu <= 0) n_cu = N_CU;
  int best = V_BIG;
  double best_t = 1e300;
  for (const Cand &c : cands) {
    const long tiles = n_tiles(m, n_b_rows, c.bm, 256);
    const long full = tiles / n_cu, rem = tiles % n_cu;
    const double t = (double)full * c.T + (rem ? c.T * (c.a + (1.0 - c.a) * (double)rem / (double)n_cu) : 0.0);
    if (t < best_t) { best_t = t; best = c.v; }
  }
  return best;
}

int gemm_ride_tiles(const GemmArgs &a, int epilogue) {
  const int bm = a.tile_variant == V_TALL ? 160 : 256, out_bn = epilogue == EPI_SWIGLU ? 128 : 256;
  return ((a.M + bm - 1) / bm) * ((a.N + out_bn - 1) / out_bn);
}

hipError_t launch_gemm_with_attention(const GemmArgs &a, int epilogue, int dh, const GemmRide &r, hipStream_t stream) {
  (void)dh;
  if (a.k_splits > 1 || a.n_count || r.head < 0 || r.head % XCDS || r.tail < 0 || !r.done || !r.ticket_next || !r.q.ticket)
    return hipErrorInvalidValue;
  const int b_rows = (epilogue == EPI_SWIGLU) ? 2 * a.N : a.N;
  if ((size_t)a.M * a.lda * 2 >= ((size_t)1 << 32) || (size_t)b_rows * a.ldb * 2 >= ((size_t)1 << 32))
    return hipErrorInvalidValue;
  const int v = a.tile_variant ? a.tile_variant : gemm_ride_variant(a.M, b_rows, N_CU - r.head);
  if (v != V_BIG && v != V_TALL) return hipErrorInvalidValue;
  const int adh = r.q.d.s.head_dim;
  if (adh != 64 && adh != 128) return hipErrorInvalidValue;
#define BS_RIDE(EPI)                                                                                  \
  return v == V_BIG ? (adh == 128 ? launch_ride<256, 256, 2, 4, EPI, 128>(a, r, stream)               \
                                  : launch_ride<256, 256, 2, 4, EPI, 64>(a, r, stream))               \
                    : (adh == 128 ? launch_ride<160, 256, 2, 4, EPI, 128>(a, r, stream)               \
                                  : launch_ride<160, 256, 2, 4, EPI, 64>(a, r, stream))
  switch (epilogue) {
    case EPI_RESID_NORM: BS_RIDE(EPI_RESID_NORM);
    case EPI_SWIGLU: BS_RIDE(EPI_SWIGLU);
    case EPI_RESID: BS_RIDE(EPI_RESID);
    default: return hipErrorInvalidValue;
  }
#undef BS_RIDE
}

hipError_t launch_gemm(const GemmArgs &a, int epilogue, int dh, hipStream_t stream) {
  // the kernels address operand rows with 32-bit byte offsets from the matrix base
  if ((size_t)a.M * a.lda * 2 >= ((size_t)1 << 32) ||
      (size_t)((epilogue == EPI_SWIGLU) ? 2 * a.N : a.N) * a.ldb * 2 >= ((size_t)1 << 32))
    return hipErrorInvalidValue;
  if (a.k_splits > 1) {
    if ((epilogue != EPI_RESID && epilogue != EPI_RESID_NORM && epilogue != EPI_QKV) || !a.sk_ws || a.N % 4)
      return hipErrorInvalidValue;
    if (a.k_splits > MAX_SPLITS || (size_t)a.k_splits * a.M * a.N > gemm_sk_workspace_floats() ||
        ((a.tile_variant == V_S128 || a.tile_variant == V_S256) && a.M > (a.tile_variant == V_S128 ? 128 : 256)))
      return hipErrorInvalidValue;
    hipError_t e;
    switch (a.tile_variant) {
      case V_S128: e = launch_one<128, 256, 2, 4, EPI_PARTIAL, 64, DEEP_X>(a, stream); break;
      case V_S256: e = launch_one<256, 128, 4, 2, EPI_PARTIAL, 64, DEEP_X>(a, stream); break;
      case V_BIG: e = launch_one<256, 256, 2, 4, EPI_PARTIAL, 64>(a, stream); break;
      case V_TALL: e = launch_one<160, 256, 2, 4, EPI_PARTIAL, 64>(a, stream); break;
      case V_SMALL: e = launch_one<128, 128, 2, 2, EPI_PARTIAL, 64>(a, stream); break;
      case V_MID: e = launch_one<192, 256, 2, 4, EPI_PARTIAL, 64>(a, stream); break;
      case V_WIDE: e = launch_one<128, 256, 2, 4, EPI_PARTIAL, 64>(a, stream); break;
      default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    if (epilogue == EPI_QKV) {
      const int items = ((a.n_q_heads + a.n_kv_heads) * (dh / 2) + a.n_kv_heads * dh) / 4;
      hipLaunchKernelGGL(splitk_reduce_qkv_kernel, dim3(a.M, (items + 255) / 256), dim3(256), 0, stream, a, dh);
    } else if (epilogue == EPI_RESID) {
      hipLaunchKernelGGL(splitk_reduce_resid_kernel, dim3(a.M, (a.N / 4 + 255) / 256), dim3(256), 0, stream, a);
    } else {
      const int threads = std::min(1024, (a.N / 4 + 63) / 64 * 64);
      hipLaunchKernelGGL(splitk_reduce_resid_norm_kernel, dim3(a.M), dim3(threads), 0, stream, a);
    }
    return hipGetLastError();
  }
  if (a.n_count && epilogue != EPI_SWIGLU && epilogue != EPI_PLAIN) return hipErrorInvalidValue;
  const int v = gemm_shape(a, epilogue, dh);
  if (v == V_ROWS) {
    switch (rows_item(a.M, a.N, a.K, epilogue, a.n_cu > 0 ? a.n_cu : N_CU)) {
      case 11: return launch_rows_one<1, 1>(a, epilogue, dh, stream);
      case 21: return launch_rows_one<2, 1>(a, epilogue, dh, stream);
      case 22: return launch_rows_one<2, 2>(a, epilogue, dh, stream);
      default: return hipErrorInvalidValue;
    }
  }
  switch (epilogue) {
    case EPI_PLAIN: return launch_variant<EPI_PLAIN>(a, v, stream);
    case EPI_RESID: return launch_variant<EPI_RESID>(a, v, stream);
    case EPI_RESID_NORM: return launch_variant<EPI_RESID_NORM>(a, v, stream);
    case EPI_SWIGLU: return launch_variant<EPI_SWIGLU>(a, v, stream);
    case EPI_QKV:
      if (dh == 128) return launch_qkv<128>(a, v, stream);
      if (dh == 64) return launch_qkv<64>(a, v, stream);
      return hipErrorInvalidValue;
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace bs

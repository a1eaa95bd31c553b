// Paged attention kernels for gfx950.
//
// KV page layout (per page, per KV head): a K tile [16 slots][dh] and a
// TRANSPOSED V tile [dh][16 slots].  Both contractions then read their MFMA
// operands straight from global memory with the contracted index contiguous:
// scores contract over dh (K rows), outputs contract over tokens (V^T rows).
//
// Both kernels compute transposed products, S^T = K Q^T and O^T = V^T P^T, so that
// a lane owns ONE query row (its accumulator column): the running maximum, the
// running sum and the rescale factor of the online softmax are per-lane scalars,
// and the probabilities leave the score accumulators already in the register
// layout the second MFMA wants for its P^T operand (the token order inside a
// k-group is permuted the same way on the V^T side, which a contraction allows).
//
// Decode attention is prefix-aware (BlendServe Appendix A.2, intra-batch prefix
// sharing; Section 4.1, decode attention is the memory-bound operator whose time
// is the bytes of KV it loads): the pages of a prefix node are read once for all
// member sequences of the node, whose query rows are stacked along the MFMA N
// dimension; every (node chunk | private tail chunk) leaves a partial softmax
// state (m, l, acc) per query row and head, and a second kernel merges a
// sequence's states along its root-to-leaf path.
#include <type_traits>

#include "attn.hpp"
#include "attn_device.hpp"
#include "common.hpp"

namespace bs {
namespace {
using namespace attn_dev;


// One launch for both kinds of item, one wavefront per SIMD (the 16-row items stream as fast
// with one wavefront per SIMD as with two) and per workgroup: a CU streams about 36 GB/s of pages
// however many of its wavefronts ask, so a step with few units wants each on a CU of its own.
// Measured (this launch, 8B heads) against workgroups of four wavefronts and chunks of 64 pages: one sequence
// of 4000 tokens 48 -> 7 us, 7 of 2000 63 -> 14, 64 of 2000 86 -> 85, 256 of 1024 180 -> 179.
// Grid order: wide workgroups first, narrow ones
// after, longest first within a kind; but one wide workgroup alternates with two narrow ones to the last wide one
// where there are at least two narrow ones for each and, alone, the launch is long (three and a half rounds of 1024 wavefronts) with wide
// units for half the SIMDs, beside prefill workgroups wide units for one and a half rounds: a wavefront with 64 query rows is bound by its
// own issue, the narrow ones beside it use the bandwidth it leaves, and many wide units of their own at the head of the launch leave memory
// idle.  Few wide units leave SIMDs to the narrow ones anyway, and in a short launch, or among few narrow ones, the last wide ones begin too late.
// Measured, alone: 640 sequences in a two-level tree (1792 wide, 5264 narrow units, 70B heads) 375 -> 326 us, 960 and 7592 units
// 137 -> 125; 608 and 2648 (24 heads) 49.6 wide first, 52.6 in turn; beside prefill rows: 3072 and 8192 units (70B layer,
// step) 7087 -> 7022; 1504 and 7248 (8B) 1361 wide first, 1374 in turn; 64-wide heads behind 23 prefixes 32.5 and 40.1.  Of 4482 launches of
// decode units and 1452 beside prefill rows, timed in both orders, the choice is 0.3 and 0.4 % off the better one on average and 11 and 13 % at
// worst (in turn from two rounds of units of either kind or a third of them wide, from a quarter beside prefill rows: 0.9 and 1.2 %, 27 and 32 %).
// Periods of two and four, turned over the XCDs, cost up to a fifth.
// The period is odd on purpose: workgroups go to the eight XCDs in turn, and a period of
// four would send every wide workgroup to the same two of them.
template <int DH, int WPW, bool NT_NARROW>
__device__ __forceinline__ void decode_workgroup(const DecodeArgs &a, int n_wide_units, int n_narrow_units, int b, int wave,
                                                 int lane, uint16_t *q_sh) {
  constexpr int WQB = 4;  // blocks of 16 query rows of a wide item
  const int hkv = a.s.n_kv_heads;
  const int nw = (n_wide_units + WPW - 1) / WPW, nn = (n_narrow_units + WPW - 1) / WPW;  // workgroups of each kind
  const bool mix = 2 * nw <= nn && (WPW == 1 ? nw >= 512 && nw + nn >= 3584 : nw >= 384);
  bool wide;
  int wg;  // index of this workgroup within its kind
  if (mix && b < 3 * nw) {
    const int per = b / 3, pos = b % 3;
    wide = pos == 0;
    wg = wide ? per : 2 * per + pos - 1;
  } else {
    wide = !mix && b < nw;
    wg = wide ? b : b - nw;
  }
  const int unit = wg * WPW + wave;
  if (wide) {
    if (unit < n_wide_units) decode_unit<DH, WQB, false, true>(a, unit / hkv, unit % hkv, wave, lane, q_sh);
  } else {
    if (unit < n_narrow_units) decode_unit<DH, 1, NT_NARROW, true>(a, n_wide_units / hkv + unit / hkv, unit % hkv, wave, lane, q_sh);
  }
}

constexpr int DECODE_Q_LDS(int dh, int waves) { return dh > 64 ? waves * 4 * 16 * (dh + 8) : 8; }  // bf16 elements: queries of a wide unit per wavefront

template <int DH>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, 1))) void decode_attn_kernel(const DecodeArgs a, int n_wide_units, int n_narrow_units) {
  __shared__ __align__(16) uint16_t q_sh[DECODE_Q_LDS(DH, 1)];
  // a launch of decode units alone: non-temporal loads for the 16-row units (see ld16_kv)
  decode_workgroup<DH, 1, true>(a, n_wide_units, n_narrow_units, blockIdx.x, 0, threadIdx.x & 63, q_sh);
}

// 16-row units alone (no prefix node with more than 16 member rows): under half of a SIMD's registers,
// so two wavefronts share a SIMD, and no accumulator has to be copied.
template <int DH>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void decode_narrow_kernel(const DecodeArgs a) {
  const int unit = (int)blockIdx.x;
  decode_unit<DH, 1, true>(a, unit / a.s.n_kv_heads, unit % a.s.n_kv_heads, 0, threadIdx.x & 63, nullptr);
}

// ------------------------------------------------------------------------------
// merge: dh/4 lanes per (decode sequence, query head), four output elements per lane
//   M = max_p m_p;  w_p = 2^(m_p - M);  out = sum_p w_p acc_p / sum_p w_p l_p
// ------------------------------------------------------------------------------
// A wavefront covers 256/dh heads of one sequence, so its loads of the partial outputs are
// 16 bytes per lane, and the partial states are added eight at a time with all their loads
// issued together: the kernel is a chain of a few memory round trips, not bandwidth.
template <int DH>
__device__ __forceinline__ void merge_decode_unit(const MergeArgs &a, int unit, int lane) {
  constexpr int LPH = DH / 4;    // lanes per head
  constexpr int HPW = 64 / LPH;  // heads per wavefront
  const int hq = a.s.n_q_heads;
  const int units_per_seq = (hq + HPW - 1) / HPW;
  const int seq = a.n_prefill + unit / units_per_seq;
  const int sub = lane / LPH, li = lane % LPH;
  const int head_raw = (unit % units_per_seq) * HPW + sub;
  const bool ok = head_raw < hq;
  const int head = ok ? head_raw : hq - 1;  // lanes past the last head repeat it and store nothing
  const int s0 = a.part_start[seq], n = a.part_start[seq + 1] - s0;
  float mx = NEG_BIG, ls = 0.f;
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  // A batch of states in one round trip: exponents, sums and outputs are requested together and
  // weighted against the largest exponent so far (places past the last state repeat it with weight 0).
  auto batch = [&](int p, auto count) __attribute__((always_inline)) {
    constexpr int B = decltype(count)::value;
    float m[B], l[B];
    f32x4_t v[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const size_t at = (size_t)(s0 + min(p + u, n - 1)) * hq + head;
      m[u] = a.part_m[at];
      l[u] = a.part_l[at];
      v[u] = *reinterpret_cast<const f32x4_t *>(a.part_acc + at * DH + li * 4);
    }
    float m_new = mx;
#pragma unroll
    for (int u = 0; u < B; ++u) m_new = fmaxf(m_new, m[u]);
    const float alpha = fast_exp2(mx - m_new);
    mx = m_new;
    ls *= alpha;
    acc *= alpha;
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const float w = p + u < n ? fast_exp2(m[u] - mx) : 0.f;
      ls += w * l[u];
      acc += w * v[u];
    }
  };
  int p = 0;
  for (; p + 4 < n; p += 8) batch(p, std::integral_constant<int, 8>{});
  if (p < n) batch(p, std::integral_constant<int, 4>{});
  if (!ok) return;
  const float inv = 1.f / ls;
  u32x2_t o2;
  o2.x = pack_bf16x2(acc[0] * inv, acc[1] * inv);
  o2.y = pack_bf16x2(acc[2] * inv, acc[3] * inv);
  *reinterpret_cast<u32x2_t *>(a.out + (size_t)a.row_start[seq] * (hq * DH) + head * DH + li * 4) = o2;
}

// The same for prefill work whose context is cut: a wavefront merges, of 32 query rows and one head, the 8 output columns
// that lie in one accumulator register group of the ring kernel's wavefront, in that kernel's layout.
template <int DH>
__device__ __forceinline__ void merge_prefill_unit(const MergeArgs &a, int unit, int lane) {
  constexpr int GROUPS = DH / 8;  // register groups of a block of 32 rows
  const int wg_per_work = a.s.n_q_heads / a.cut_heads;
  const int group = unit % GROUPS, qb = unit / GROUPS % 2, region = unit / (2 * GROUPS);
  const int wave = region % 4, wg = region / 4 % wg_per_work;
  const int32_t *cut = a.cut + 4 * (region / (4 * wg_per_work));
  const int r0 = a.row_start[cut[0]], q_len = a.row_start[cut[0] + 1] - r0;
  const int row0 = cut[1] * a.cut_rows + 64 * (wave / a.cut_heads) + 32 * qb;  // of the segment
  const int head = wg * a.cut_heads + wave % a.cut_heads, lr = lane & 31;
  if (row0 >= q_len) return;
  const int n = cut[3];
  float mx = NEG_BIG, ls = 0.f;
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int B = 8;
  for (int p = 0; p < n; p += B) {
    float m[B], l[B];
    f32x4_t v[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const size_t at = ((size_t)(cut[2] + min(p + u, n - 1)) * wg_per_work + wg) * 4 + wave;
      m[u] = a.cut_m[at * 64 + 32 * qb + lr];
      l[u] = a.cut_l[at * 64 + 32 * qb + lr];
      v[u] = *reinterpret_cast<const f32x4_t *>(a.cut_acc + at * (64 * DH) + qb * (32 * DH) + group * 256 + lane * 4);
    }
    float m_new = mx;
#pragma unroll
    for (int u = 0; u < B; ++u) m_new = fmaxf(m_new, m[u]);
    const float alpha = fast_exp2(mx - m_new);
    mx = m_new;
    ls *= alpha;
    acc *= alpha;
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const float w = p + u < n ? fast_exp2(m[u] - mx) : 0.f;
      ls += w * l[u];
      acc += w * v[u];
    }
  }
  if (row0 + lr >= q_len) return;
  const float inv = 1.f / ls;
  u32x2_t o2;
  o2.x = pack_bf16x2(acc[0] * inv, acc[1] * inv);
  o2.y = pack_bf16x2(acc[2] * inv, acc[3] * inv);
  *reinterpret_cast<u32x2_t *>(a.out + (size_t)(r0 + row0 + lr) * (a.s.n_q_heads * DH) + head * DH + group * 8 + 4 * (lane >> 5)) = o2;
}

template <int DH>
__global__ __launch_bounds__(256) void merge_kernel(const MergeArgs a, int n_decode_units, int n_units) {
  const int unit = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (unit < n_decode_units)
    merge_decode_unit<DH>(a, unit, lane);
  else if (unit < n_units)
    merge_prefill_unit<DH>(a, unit - n_decode_units, lane);
}

// ------------------------------------------------------------------------------
// prefill attention, the ring kernel: a workgroup of four wavefronts, each (64 query rows, one query
// head); the four share a KV head and walk the same pages
// ------------------------------------------------------------------------------
// Keys and values of a block of 32 tokens (two pages) travel global -> LDS once per workgroup, each
// wavefront requesting one of the four tiles, into a ring of PF_RING blocks; fragments then come
// out of LDS.  (Read straight from global memory by every wavefront, 24 loads of 64 scattered pieces
// per block and wavefront, a block took 3300 clocks of a CU; its MFMAs need 1024.)  It takes 2200
// now: issue 1200, of that 900 vector-ALU; 600 waiting for a pipe, 400 for LDS and barriers.
// Measured, 8B heads: 28 x 64 rows behind 6000 tokens 307 -> 207 us, 8 x 1024 rows 137 -> 111, 32 rows
// behind 8000 tokens 327 -> 216 (35 with the context cut into ranges, see prefill_cut in api.hip), 128 x 64 rows 70 -> 65,
// where starting workgroups is most of it.
//
// What then bounds a block is the issue of one wavefront per SIMD (the accumulators of 64 rows x dh
// 128 leave no room for two): 32 MFMAs of 32 clocks against about 900 clocks of softmax arithmetic.
// They overlap by software pipelining: while block t's scores turn into probabilities, the scores of
// block t+1 are computed, then the PV product of block t, one MFMA at a time with its share of the
// arithmetic behind it; the key fragments of block t+2 and the value fragments of block t are read
// from LDS in between.  One barrier per two blocks.
//
// LDS: a key tile is [16 tokens][dh], its 16-byte chunks XOR-swizzled by score row so that a
// fragment read (16 rows, two chunks) touches every bank once; a value tile is [dh][16 tokens], the
// two chunks of a row exchanged in every other group of eight rows, for the same reason.  Keys enter
// the score product in the order that leaves a lane eight adjacent tokens of one page (token bits 2
// and 3 exchanged), so a value fragment is one 16-byte read.
constexpr int PF_RING = 8;  // blocks of 32 tokens: while blocks t, t+1 are computed, t-2, t-1 make room for t+6, t+7; t+3 must have landed
constexpr int PF_LDS(int dh) { return PF_RING * 4 * 16 * dh * 2; }

// 16 bytes per lane, lane i to `lds` + 16 i, without passing through registers
__device__ __forceinline__ void dma_to_lds(const void *src, unsigned char *lds) {
  __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)lds, 16, 0, 0);
}
__device__ __forceinline__ int swap_bits_2_3(int v) { return (v & ~12) | ((v & 4) << 1) | ((v & 8) >> 1); }

// s = k q^T + s (FIRST: + 0) with the accumulators in ordinary registers, where the softmax reads them
// (left to the compiler, a kernel of more than 256 registers keeps every MFMA result in accumulation
// registers and copies it out: 130 copies per block).  The compiler does not see the latency: whoever
// reads s leaves at least four further MFMAs, which execute in order (two would cover the 12 wait states of
// this one), or mfma_settle between.
template <bool FIRST>
__device__ __forceinline__ void score_mfma(f32x16_t &s, bf16x8_t k, bf16x8_t q) {
  if constexpr (FIRST)
    asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(k), "v"(q));
  else
    asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(k), "v"(q));
}

// out = o / l of 64 query rows (two blocks of 32, of which the first n_q exist) from row `row` on, one head
template <int DH>
__device__ __forceinline__ void store_prefill_rows(const PrefillArgs &a, const f32x16_t (&o)[2][DH / 32], const float (&l)[2],
                                                   const int (&n_q)[2], int row, int head, int lr, int g2) {
  const int hq = a.s.n_q_heads;
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    float ls = l[qb];
    ls += __shfl_xor(ls, 32, 64);
    if (lr < n_q[qb]) {
      const float inv = 1.f / ls;
      uint16_t *dst = a.out + (size_t)(row + qb * 32 + lr) * (hq * DH) + head * DH;
#pragma unroll
      for (int db = 0; db < DH / 32; ++db)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          u32x2_t v;
          v.x = pack_bf16x2(o[qb][db][4 * q + 0] * inv, o[qb][db][4 * q + 1] * inv);
          v.y = pack_bf16x2(o[qb][db][4 * q + 2] * inv, o[qb][db][4 * q + 3] * inv);
          *reinterpret_cast<u32x2_t *>(dst + 32 * db + 8 * q + 4 * g2) = v;
        }
    }
  }
}

// The partial softmax state of the same rows: the accumulators as the lanes hold them (1 KB per store; row by row a CU
// would store one lane per clock), maxima and sums per row.  `at`: number of the wavefront's part of the state.
template <int DH>
__device__ __forceinline__ void store_prefill_state(const PrefillArgs &a, const f32x16_t (&o)[2][DH / 32], const float (&m)[2],
                                                    const float (&l)[2], const int (&n_q)[2], size_t at, int lane) {
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    float ls = l[qb];
    ls += __shfl_xor(ls, 32, 64);
    if (n_q[qb] <= 0) continue;  // wave-uniform
    float *acc = a.part_acc + at * (64 * DH) + qb * (32 * DH) + lane * 4;
#pragma unroll
    for (int db = 0; db < DH / 32; ++db)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<f32x4_t *>(acc + (db * 4 + q) * 256) =
            f32x4_t{o[qb][db][4 * q], o[qb][db][4 * q + 1], o[qb][db][4 * q + 2], o[qb][db][4 * q + 3]};
    if (lane < 32) {
      a.part_m[at * 64 + qb * 32 + lane] = m[qb];
      a.part_l[at * 64 + qb * 32 + lane] = ls;
    }
  }
}

template <int DH>
__device__ __forceinline__ void prefill_workgroup(const PrefillArgs &a, int heads_per_wg, int b, int wave, int lane, unsigned char *smem) {
  constexpr int KC = DH / 16;  // k-steps of the 32x32x16 score MFMA
  constexpr int DB = DH / 32;  // 32-row blocks of the output
  constexpr int NQ = 2;        // blocks of 32 query rows per wavefront
  constexpr int TILE = 16 * DH * 2;     // bytes of one K or V tile of a (page, head)
  constexpr int CPR = DH / 8;           // 16-byte chunks of a key row
  constexpr int LD = TILE / 1024;       // loads of 1 KB per tile
  constexpr int BLK = 4 * TILE;         // K, V of the first page, K, V of the second
  const int hkv = a.s.n_kv_heads, hq = a.s.n_q_heads, grp = hq / hkv;
  const int wg_per_work = hq / heads_per_wg;
  const int w = b / wg_per_work;
  const int32_t *work = a.work + (a.cut ? 4 : 2) * w;
  const int seq = work[0], qblk = work[1];  // block of 64 * (4 / heads_per_wg) query rows
  // blocks of 32 tokens [t0, t1) of the context (t1 = 0: to its end)
  const int t0 = a.cut ? work[2] & 0xFFFF : 0, t1 = a.cut ? (int)((unsigned)work[2] >> 16) : 0, state = a.cut ? work[3] : -1;
  const int head = (b % wg_per_work) * heads_per_wg + wave % heads_per_wg;
  const int kvh = head / grp;
  const int r0 = a.row_start[seq], q_len = a.row_start[seq + 1] - r0;
  // tokens are counted from the range's first one: the range ends at kv_len, row 0 of the segment stands at `before`
  const int whole_len = a.kv_len[seq], before = whole_len - q_len - 32 * t0;
  const int kv_len = (t1 ? 32 * t1 : whole_len) - 32 * t0;
  const int lr = lane & 31, g2 = lane >> 5;
  // (through the constant address space: nobody writes the page table, and its loads stay on the scalar
  // unit, where a wait for one does not wait for the tiles in flight)
  const auto *pages = (const __attribute__((address_space(4))) int32_t *)(a.page_ids + a.page_start[seq]) + 2 * t0;
  const int n_pg = (kv_len + 15) >> 4;
  const int wg_row0 = qblk * 64 * (4 / heads_per_wg);
  const int row_w = wg_row0 + 64 * (wave / heads_per_wg);  // first row of this wavefront

  // blocks of 32 tokens that the workgroup walks, and those that this wavefront needs
  const int wg_rows = min(64 * (4 / heads_per_wg), q_len - wg_row0);
  const int n_wg = t1 ? t1 - t0 : (before + wg_row0 + wg_rows - 1) / 32 + 1;
  const int n_tb = row_w >= q_len ? 0 : t1 ? t1 - t0 : (before + min(row_w + 64, q_len) - 1) / 32 + 1;

  // ---- global -> LDS: wavefront w requests tile w of a block (page w / 2; keys or values) ----
  uint32_t src[LD];  // byte offset within the tile of the chunk that this lane's LDS place holds
#pragma unroll
  for (int i = 0; i < LD; ++i) {
    const int p = i * 64 + lane;  // place in the tile, in chunks
    if (wave & 1) {
      const int dh = p >> 1;
      src[i] = (uint32_t)(dh * 32 + (((p & 1) ^ ((dh >> 3) & 1)) << 4));
    } else {
      const int tok = p / CPR, rho = swap_bits_2_3(tok), f = CPR == 16 ? rho : rho >> 1;
      src[i] = (uint32_t)(tok * DH * 2 + (((p % CPR) ^ f) << 4));
    }
  }
  auto page_of = [&](int tb) __attribute__((always_inline)) { return pages[min(2 * tb + (wave >> 1), n_pg - 1)]; };
  const unsigned char *tiles = reinterpret_cast<const unsigned char *>(a.kv_pool) + (size_t)((wave & 1) * hkv + kvh) * TILE;
  const uint32_t page_stride = (uint32_t)(2 * hkv * TILE);
  auto request = [&](int page, int slot) __attribute__((always_inline)) {
    const unsigned char *t0 = tiles + (uint64_t)(uint32_t)page * page_stride;
#pragma unroll
    for (int i = 0; i < LD; ++i)
      dma_to_lds(t0 + src[i], smem + slot * BLK + wave * TILE + i * 1024);
  };

  int n_q[NQ], my_pos[NQ], first_pos[NQ];
  bf16x8_t qf[NQ][KC];
  f32x16_t o[NQ][DB];
  float m[NQ], l[NQ];
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
    const int row0 = row_w + qb * 32;
    n_q[qb] = min(32, q_len - row0);                       // <= 0: the block does not exist
    first_pos[qb] = before + row0;
    my_pos[qb] = min(first_pos[qb] + lr, kv_len - 1);
    const bool ok = lr < n_q[qb];
    const uint16_t *p = a.q + (size_t)(r0 + (ok ? row0 + lr : 0)) * (hq * DH) + head * DH + 8 * g2;
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      u32x4_t v = {0u, 0u, 0u, 0u};
      if (ok) v = ld16(p + 16 * c);
      qf[qb][c] = as_bf16x8(v);
    }
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[qb][db][r] = 0.f;
    m[qb] = NEG_BIG;
    l[qb] = 0.f;
  }

#pragma unroll
  for (int i = 0; i < PF_RING - 2; ++i) request(page_of(min(i, n_wg - 1)), i);

  // ---- LDS -> registers ----
  const int tok = swap_bits_2_3(lr & 15), kf_sw = CPR == 16 ? (lr & 15) : ((lr & 15) >> 1);
  const uint32_t k_off = (uint32_t)((lr >> 4) * 2 * TILE + tok * DH * 2 + ((g2 ^ kf_sw) << 4));
  const uint32_t v_off = (uint32_t)(TILE + lr * 32 + ((g2 ^ ((lr >> 3) & 1)) << 4));
  u32x4_t kf[KC], va[DB][2];
  auto read_k = [&](uint32_t blk, int c) __attribute__((always_inline)) {
    kf[c] = *reinterpret_cast<const u32x4_t *>(smem + ((blk + k_off) ^ (uint32_t)(c << 5)));
  };
  auto read_v = [&](uint32_t blk, int i) __attribute__((always_inline)) {  // i = 2 db + page
    va[i >> 1][i & 1] = *reinterpret_cast<const u32x4_t *>(smem + blk + v_off + (i & 1) * 2 * TILE + (i >> 1) * 1024);
  };

  // Element r of s: token tb*32 + 16*(r/8) + 8*g2 + r%8 against the query at my_pos.  The running
  // maximum, lazily, as in the decode kernel: rescale only when somebody's maximum has grown by more
  // than 2^TAU.  `mx`: this lane's maximum over s before masking.
  auto max_of = [&](const f32x16_t &s) __attribute__((always_inline)) {
    float mx = fmaxf(s[0], s[1]);
#pragma unroll
    for (int r = 2; r < 16; r += 2) mx = fmaxf(fmaxf(mx, s[r]), s[r + 1]);
    return mx;
  };
  auto settle = [&](f32x16_t &s, float mx, int tb, int qb) __attribute__((always_inline)) {
    if (tb * 32 + 31 > first_pos[qb]) {  // wave-uniform: the block holds tokens some query must not see
      const int lim = my_pos[qb] - tb * 32 - 8 * g2;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (16 * (r >> 3) + (r & 7) > lim) s[r] = NEG_BIG;
      mx = max_of(s);
    }
    mx *= a.s.scale_log2e;  // the scale is positive: the maximum commutes with it
    if (__builtin_amdgcn_ballot_w64(mx > m[qb] + TAU) != 0) {
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float m_new = fmaxf(m[qb], mx);
      const float alpha = fast_exp2(m[qb] - m_new);
      m[qb] = m_new;
      l[qb] *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db) scale_acc(o[qb][db], alpha);
    }
  };
  f32x16_t s_a[NQ], s_b[NQ];  // scores of two successive blocks

  constexpr int AHEAD = PF_RING - 6;  // at the top of block t, t even: blocks t+4 .. t+PF_RING-3 may still be in flight
  constexpr auto wait_vm = [](int n) { return (n & 0xF) | ((n >> 4) << 14) | 0xF70; };  // s_waitcnt vmcnt(n)
  constexpr int FIRST_WAIT = wait_vm((PF_RING - 4) * LD), WAIT_AHEAD = wait_vm(AHEAD * LD);
  static_assert(PF_RING == 8 && (PF_RING - 4) * LD < 64, "outstanding loads must fit the vmcnt field");

  // blocks 0 and 1 (and the queries, requested before them) have landed: scores of block 0, key fragments of block 1
  __builtin_amdgcn_s_waitcnt(FIRST_WAIT);
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int c = 0; c < KC; ++c) read_k(0, c);
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
    score_mfma<true>(s_a[qb], as_bf16x8(kf[0]), qf[qb][0]);
#pragma unroll
    for (int c = 1; c < KC; ++c) score_mfma<false>(s_a[qb], as_bf16x8(kf[c]), qf[qb][c]);
  }
  mfma_settle(s_a[0], s_a[1]);
#pragma unroll
  for (int c = 0; c < KC; ++c) read_k(BLK, c);
  settle(s_a[0], max_of(s_a[0]), 0, 0);
  settle(s_a[1], max_of(s_a[1]), 0, 1);
  // Probabilities, two at a time: pair e (of 16) is elements 2 (e % 8), + 1 of query block e / 8.  The
  // first EARLY of query block 0 are taken one block ahead, beside the last PV MFMAs of the block before.
  constexpr int EARLY = 4;
  u32x4_t pw[NQ][2];
  float ps[NQ] = {0.f, 0.f};  // sums of the block's probabilities so far
  float ex[2];  // exponentials of the pair before: summed and packed one pair later, when they have arrived
  auto exps = [&](const f32x16_t (&s)[NQ], int e, float (&x)[2]) __attribute__((always_inline)) {
    const int qb = e >> 3, r = (e & 7) * 2;
    x[0] = fast_exp2(__builtin_fmaf(s[qb][r], a.s.scale_log2e, -m[qb]));
    x[1] = fast_exp2(__builtin_fmaf(s[qb][r + 1], a.s.scale_log2e, -m[qb]));
    asm volatile("" : "+v"(x[0]), "+v"(x[1]));  // here, and not where the compiler would first need them
  };
  auto take = [&](int e) __attribute__((always_inline)) {
    const int qb = e >> 3;
    ps[qb] += ex[0];
    ps[qb] += ex[1];
    uint32_t two = pack_bf16x2(ex[0], ex[1]);
    asm volatile("" : "+v"(two), "+v"(ps[qb]));
    pw[qb][(e & 7) >> 2][e & 3] = two;
  };
  // pair e: its exponentials; the pair before it is taken
  auto weight = [&](const f32x16_t (&s)[NQ], int e) __attribute__((always_inline)) {
    float x[2];
    exps(s, e, x);
    if (e > 0) take(e - 1);
    ex[0] = x[0];
    ex[1] = x[1];
  };
#pragma unroll
  for (int e = 0; e < EARLY; ++e) weight(s_a, e);

  int page0 = page_of(min(PF_RING - 2, n_wg - 1)), page1 = page_of(min(PF_RING - 1, n_wg - 1));
  auto block = [&](int tb, f32x16_t (&s_cur)[NQ], f32x16_t (&s_nxt)[NQ], bool first, auto last) __attribute__((always_inline)) {
    if (first) {  // the first block of a pair
      // this wavefront's tiles up to block tb+3 have landed, after the barrier everybody's, and nobody reads blocks tb-2, tb-1 any more
      __builtin_amdgcn_s_waitcnt(WAIT_AHEAD);
      __builtin_amdgcn_s_barrier();
      request(page0, (tb + PF_RING - 2) % PF_RING);
      request(page1, (tb + PF_RING - 1) % PF_RING);
      page0 = page_of(min(tb + PF_RING, n_wg - 1));
      page1 = page_of(min(tb + PF_RING + 1, n_wg - 1));
    }
    const uint32_t v_blk = (uint32_t)(tb % PF_RING * BLK), k_blk = (uint32_t)((tb + 2) % PF_RING * BLK);
    if (tb >= n_tb) return;  // wave-uniform: a wavefront of earlier rows is done, it only feeds the ring

    // One MFMA and its share of the other work: scores of block tb+1 (N_QK MFMAs), then PV of block tb
    // for query block 0 and for query block 1.  Pairs of probabilities EARLY .. 15 go beside the scores and
    // the first PV product; beside the second, query block 0 of block tb+1 settles and gives its first pairs.
    constexpr int N_QK = NQ * KC, N_PV = 2 * DB, N_W = N_QK + N_PV;
    static_assert(N_PV >= 4, "the scores of block tb+1 are read behind the first PV product alone (see score_mfma)");
    constexpr bool LAST = decltype(last)::value;  // nothing follows; the only block that can run past the context
    auto weights_of = [&](int j) __attribute__((always_inline)) {  // slot j of N_W
#pragma unroll
      for (int e = EARLY + j * (16 - EARLY) / N_W; e < EARLY + (j + 1) * (16 - EARLY) / N_W; ++e) weight(s_cur, e);
      if (j == N_W - 1) take(15);
    };
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < N_QK; ++j) {
      const int c = j / NQ, qb = j % NQ;
      if constexpr (!LAST) {
        if (c == 0) score_mfma<true>(s_nxt[qb], as_bf16x8(kf[c]), qf[qb][c]);
        else score_mfma<false>(s_nxt[qb], as_bf16x8(kf[c]), qf[qb][c]);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (j < 2 * DB) read_v(v_blk, j);
      weights_of(j);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (LAST) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int h = 0; h < 2; ++h) va[db][h] = mask_tokens8(va[db][h], tb * 32 + 16 * h + 8 * g2, kv_len);
    }
    float mx0 = 0.f, mx1 = 0.f;  // maxima of s_nxt: its last MFMA is N_PV MFMAs old when they are taken
    auto pv = [&](int qb, int j) __attribute__((always_inline)) {
      const int db = j % DB, h = j / DB;
      o[qb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(va[db][h]), as_bf16x8(pw[qb][h]), o[qb][db], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int j = 0; j < N_PV; ++j) {
      pv(0, j);
      if (!LAST && j < KC) read_k(k_blk, j);
      weights_of(N_QK + j);
      __builtin_amdgcn_sched_barrier(0);
    }
    l[0] += ps[0];
    ps[0] = 0.f;
    const bool more = !LAST && tb + 1 < n_tb;  // (if not, what is taken of block tb+1 below is never used)
    if constexpr (!LAST) {
      mx0 = max_of(s_nxt[0]);
      if (more) settle(s_nxt[0], mx0, tb + 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < N_PV; ++j) {
      pv(1, j);
      if constexpr (!LAST) {
        if (j == 0) mx1 = max_of(s_nxt[1]);
        if (j >= N_PV - EARLY) weight(s_nxt, j - (N_PV - EARLY));
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    l[1] += ps[1];
    ps[1] = 0.f;
    if (more) settle(s_nxt[1], mx1, tb + 1, 1);
  };
  int tb = 0;
  for (; tb + 2 < n_wg; tb += 2) {
    block(tb, s_a, s_b, true, std::false_type{});
    block(tb + 1, s_b, s_a, false, std::false_type{});
  }
  if (tb + 1 < n_wg) {
    block(tb, s_a, s_b, true, std::false_type{});
    s_a[0] = s_b[0];
    s_a[1] = s_b[1];
  }
  block(n_wg - 1, s_a, s_b, n_wg % 2 == 1, std::true_type{});
  __builtin_amdgcn_s_waitcnt(0x0F70);  // the look-ahead loads have landed before the LDS is released
  if (state >= 0)
    store_prefill_state<DH>(a, o, m, l, n_q, ((size_t)state * wg_per_work + b % wg_per_work) * 4 + wave, lane);
  else
    store_prefill_rows<DH>(a, o, l, n_q, r0 + row_w, head, lr, g2);
}

// 64-wide heads: 236 registers and a ring of 64 KB, so two workgroups share a CU (one against two, 32 heads in 8
// groups, 128 segments: 16 rows 24 against 17 us, 64 rows 36 against 30, 64 rows behind 500 tokens 86 against 65).
template <int DH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, DH == 64 ? 2 : 1))) void prefill_attn_kernel(const PrefillArgs a, int heads_per_wg) {
  extern __shared__ __align__(256) unsigned char attn_smem[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  prefill_workgroup<DH>(a, heads_per_wg, blockIdx.x, wave, threadIdx.x & 63, attn_smem);
}

// The same without the ring, for groups of heads that are not a multiple of four: a wavefront takes 64 query
// rows of one head, its keys and values straight from global memory, and a workgroup is the one or two heads
// of a KV group that walk the same pages.  With one head per workgroup the ring kernel needs 256 rows of a
// segment to give its four wavefronts work, and its workgroups have a CU to themselves (two, 64-wide heads);
// here a CU holds four such wavefronts (eight).  A lane's key fragment is 16 bytes of a 256-byte row, so
// a load touches 32 cache lines: a full CU is bound by its L1, 3.6 us per block of 32 tokens of four
// 128-wide heads, where the ring kernel takes 1.2 us for one wavefront with rows and 1.7 for four.
// Which one a step takes: prefill_route.
template <int DH>
__device__ __forceinline__ void prefill_direct_workgroup(const PrefillArgs &a, int heads_per_wg, int b, int wave, int lane) {
  constexpr int KC = DH / 16;  // k-steps of the 32x32x16 score MFMA
  constexpr int DB = DH / 32;  // 32-row blocks of the output
  constexpr int NQ = 2;        // blocks of 32 query rows per wavefront
  const int hkv = a.s.n_kv_heads, hq = a.s.n_q_heads, grp = hq / hkv;
  const int wg_per_work = hq / heads_per_wg;
  const int w = b / wg_per_work;
  const int seq = a.work[2 * w], qblk = a.work[2 * w + 1];  // block of 64 query rows
  const int head = (b % wg_per_work) * heads_per_wg + wave;
  const int kvh = head / grp;
  const int r0 = a.row_start[seq], q_len = a.row_start[seq + 1] - r0;
  const int kv_len = a.kv_len[seq];
  const int lr = lane & 31, g2 = lane >> 5;
  const size_t tile = (size_t)16 * DH;
  const int32_t *pages = a.page_ids + a.page_start[seq];
  const int n_pg = (kv_len + 15) >> 4;
  const uint32_t v_off = lr * 16 + 4 * g2;  // this lane's element within a value tile [dh][16 tokens]

  int n_q[NQ], my_pos[NQ], last_tb[NQ], first_pos[NQ];
  bf16x8_t qf[NQ][KC];
  f32x16_t o[NQ][DB];
  float m[NQ], l[NQ];
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
    const int row0 = qblk * 64 + qb * 32;
    n_q[qb] = min(32, q_len - row0);                       // <= 0: the block does not exist
    first_pos[qb] = kv_len - q_len + row0;
    my_pos[qb] = min(first_pos[qb] + lr, kv_len - 1);
    last_tb[qb] = n_q[qb] > 0 ? (first_pos[qb] + n_q[qb] - 1) / 32 : -1;  // last block of 32 tokens it attends to
    const bool ok = lr < n_q[qb];
    const uint16_t *p = a.q + (size_t)(r0 + (ok ? row0 + lr : 0)) * (hq * DH) + head * DH + 8 * g2;
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      u32x4_t v = {0u, 0u, 0u, 0u};
      if (ok) v = ld16(p + 16 * c);
      qf[qb][c] = as_bf16x8(v);
    }
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[qb][db][r] = 0.f;
    m[qb] = NEG_BIG;
    l[qb] = 0.f;
  }

  const int n_tb = max(last_tb[0], last_tb[1]) + 1;
  // Software pipeline, one block of 32 tokens deep: while block tb is computed, the values of
  // block tb+1 travel into the second value buffer, its keys into the key registers (as soon
  // as the score MFMAs of block tb have read them) and the page ids of block tb+2 into scalar
  // registers.  Steps past the end re-read the last block (never used).
  struct PagePair { int p0, p1; };
  auto page_pair = [&](int tb) __attribute__((always_inline)) {
    const int t = tb < n_tb ? tb : n_tb - 1;
    PagePair pp;
    pp.p0 = pages[2 * t];
    pp.p1 = (2 * t + 1 < n_pg) ? pages[2 * t + 1] : pp.p0;
    return pp;
  };
  auto load_k = [&](PagePair pp, u32x4_t (&kf)[KC]) __attribute__((always_inline)) {
    const size_t pk = (lr < 16) ? pp.p0 : pp.p1;
    const uint16_t *kp = a.kv_pool + ((pk * 2 + 0) * hkv + kvh) * tile + (lr & 15) * DH + 8 * g2;
#pragma unroll
    for (int c = 0; c < KC; ++c) kf[c] = ld16(kp + 16 * c);
  };
  // values of a block as loaded: [32-row block of dh][16-token half of the block][8 tokens]
  auto load_v = [&](PagePair pp, u32x2_t (&r)[DB][4]) __attribute__((always_inline)) {
    const uint16_t *v0 = a.kv_pool + (((size_t)pp.p0 * 2 + 1) * hkv + kvh) * tile;  // wave-uniform bases,
    const uint16_t *v1 = a.kv_pool + (((size_t)pp.p1 * 2 + 1) * hkv + kvh) * tile;  // lane offset v_off
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      r[db][0] = ld8(v0 + v_off + 512 * db);
      r[db][1] = ld8(v0 + v_off + 512 * db + 8);
      r[db][2] = ld8(v1 + v_off + 512 * db);
      r[db][3] = ld8(v1 + v_off + 512 * db + 8);
    }
  };
  // block tb: keys in kf and values in vr have been requested; `next` holds the pages of block tb+1
  auto block = [&](int tb, u32x4_t (&kf)[KC], u32x2_t (&vr)[DB][4], u32x2_t (&vn)[DB][4], PagePair &next, auto two) __attribute__((always_inline)) {
    const PagePair after = page_pair(tb + 2);
    load_v(next, vn);
    if (tb * 32 + 32 > kv_len) {  // wave-uniform: the block runs past the context
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int h = 0; h < 4; ++h) vr[db][h] = mask_tokens(vr[db][h], tb * 32 + 8 * h + 4 * g2, kv_len);
    }
    u32x4_t va[DB][2];
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      va[db][0] = u32x4_t{vr[db][0].x, vr[db][0].y, vr[db][1].x, vr[db][1].y};
      va[db][1] = u32x4_t{vr[db][2].x, vr[db][2].y, vr[db][3].x, vr[db][3].y};
    }
    // Order of issue: both score products, then softmax of the first query block (its VALU
    // work runs while the matrix pipe is still busy with the second product), its PV product,
    // softmax of the second block under that product, and the second PV product.
    auto scores = [&](int qb) {
      f32x16_t s;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
      for (int c = 0; c < KC; ++c)
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kf[c]), qf[qb][c], s, 0, 0, 0);
      return s;
    };
    // element r of s: token tb*32 + 8*(r/4) + 4*g2 + r%4 against the query at my_pos
    // softmax of one query block in two parts.  `prepare` (mask, running maximum, the rare
    // rescale) branches; `weights` (exponentials, row sums, bf16 packing) does not, so that
    // the scheduler may slide it under the MFMAs of the other query block.
    auto prepare = [&](f32x16_t &s, int qb) __attribute__((always_inline)) {
      if (tb * 32 + 31 > first_pos[qb]) {  // wave-uniform: the block holds tokens some query must not see
        const int lim = my_pos[qb] - tb * 32 - 4 * g2;
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (8 * (r >> 2) + (r & 3) > lim) s[r] = NEG_BIG;
      }
      float mx = fmaxf(s[0], s[1]);
#pragma unroll
      for (int r = 2; r < 16; r += 2) mx = fmaxf(fmaxf(mx, s[r]), s[r + 1]);
      mx *= a.s.scale_log2e;  // the scale is positive: the maximum commutes with it
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      // lazy reference exponent, as in the decode kernel: rescale only when somebody's maximum
      // has grown by more than 2^TAU
      if (__builtin_amdgcn_ballot_w64(mx > m[qb] + TAU) != 0) {
        const float m_new = fmaxf(m[qb], mx);
        const float alpha = fast_exp2(m[qb] - m_new);
        m[qb] = m_new;
        l[qb] *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db) scale_acc(o[qb][db], alpha);
      }
    };
    auto weights = [&](f32x16_t &s, int qb, u32x4_t &pw0, u32x4_t &pw1) __attribute__((always_inline)) {
      const float neg_m = -m[qb];
      float ps = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[r] = fast_exp2(__builtin_fmaf(s[r], a.s.scale_log2e, neg_m));
        ps += s[r];
      }
      l[qb] += ps;
      pw0.x = pack_bf16x2(s[0], s[1]);
      pw0.y = pack_bf16x2(s[2], s[3]);
      pw0.z = pack_bf16x2(s[4], s[5]);
      pw0.w = pack_bf16x2(s[6], s[7]);
      pw1.x = pack_bf16x2(s[8], s[9]);
      pw1.y = pack_bf16x2(s[10], s[11]);
      pw1.z = pack_bf16x2(s[12], s[13]);
      pw1.w = pack_bf16x2(s[14], s[15]);
    };
    auto pv = [&](int qb, const u32x4_t &pw0, const u32x4_t &pw1) __attribute__((always_inline)) {
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        o[qb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(va[db][0]), as_bf16x8(pw0), o[qb][db], 0, 0, 0);
        o[qb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(va[db][1]), as_bf16x8(pw1), o[qb][db], 0, 0, 0);
      }
    };
    u32x4_t pa0, pa1, pb0, pb1;
    if constexpr (decltype(two)::value) {  // the second query block exists
      // (past the first block's last position its scores are all masked and add nothing)
      f32x16_t s0 = scores(0);
      f32x16_t s1 = scores(1);
      load_k(next, kf);
      prepare(s0, 0);
      prepare(s1, 1);
      __builtin_amdgcn_sched_barrier(0);
      weights(s0, 0, pa0, pa1);
      __builtin_amdgcn_sched_barrier(0);
      // the first PV product, one MFMA at a time, with the second block's weights in between
      pv(0, pa0, pa1);
      weights(s1, 1, pb0, pb1);
#pragma unroll
      for (int i = 0; i < 2 * DB; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);           // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, 56 / (2 * DB), 0);  // its share of the VALU work
      }
      __builtin_amdgcn_sched_barrier(0);
      pv(1, pb0, pb1);
    } else {
      f32x16_t s0 = scores(0);
      load_k(next, kf);
      prepare(s0, 0);
      weights(s0, 0, pa0, pa1);
      pv(0, pa0, pa1);
    }
    next = after;
  };
  u32x4_t kf[KC];
  u32x2_t v_a[DB][4], v_b[DB][4];
  {
    const PagePair first = page_pair(0);
    load_k(first, kf);
    load_v(first, v_a);
  }
  PagePair next = page_pair(1);
  auto run = [&](auto two) __attribute__((always_inline)) {
    for (int tb = 0; tb < n_tb; tb += 2) {
      block(tb, kf, v_a, v_b, next, two);
      if (tb + 1 < n_tb) block(tb + 1, kf, v_b, v_a, next, two);
    }
  };
  if (n_q[1] > 0)  // wave-uniform: the second block of query rows exists
    run(std::true_type{});
  else
    run(std::false_type{});
  store_prefill_rows<DH>(a, o, l, n_q, r0 + qblk * 64, head, lr, g2);
}

template <int DH>
__global__ __launch_bounds__(256) void prefill_direct_kernel(const PrefillArgs a, int heads_per_wg) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  prefill_direct_workgroup<DH>(a, heads_per_wg, blockIdx.x, wave, threadIdx.x & 63);
}

// Prefill and decode attention of one step in one launch.  A prefill workgroup is bound by the
// matrix and vector pipes and leaves the memory system idle, a decode workgroup is the
// opposite, and each needs a CU to itself (one wavefront per SIMD), so the two kinds blend
// across CUs: the grid deals one prefill workgroup per `period` workgroups (an odd number, so
// that they rotate over the XCDs) for as long as both kinds last, each kind in its own order
// (longest first).  Workgroups of four wavefronts only (four query heads of a KV group).
// Measured against the two launches one after the other: 0.520 -> 0.498 ms on the 8B blended
// shape (2048 prefill rows, 1024 decode sequences), 0.746 -> 0.717 ms on the 70B one.
template <int DH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void blended_attn_kernel(
    const DecodeArgs d, int n_wide_units, int n_narrow_units, const PrefillArgs pf, int n_pf_wgs, int period) {
  extern __shared__ __align__(256) unsigned char attn_smem[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int n_dec = ((n_wide_units + 3) >> 2) + ((n_narrow_units + 3) >> 2);
  const int mixed = min(n_pf_wgs, n_dec / (period - 1));  // periods of one prefill + (period - 1) decode workgroups
  const int b = blockIdx.x;
  bool prefill;
  int idx;
  if (b < period * mixed) {
    const int per = b / period, pos = b % period;
    prefill = pos == 0;
    idx = prefill ? per : (period - 1) * per + pos - 1;
  } else {
    const int r = b - period * mixed;
    prefill = r < n_pf_wgs - mixed;
    idx = prefill ? mixed + r : (period - 1) * mixed + r - (n_pf_wgs - mixed);
  }
  if (prefill)
    prefill_workgroup<DH>(pf, 4, idx, wave, lane, attn_smem);
  else
    decode_workgroup<DH, 4, false>(d, n_wide_units, n_narrow_units, idx, wave, lane, reinterpret_cast<uint16_t *>(attn_smem));
}

// What the GEMM launches of a step have left of its queue of 16-row units, on the whole chip:
// workgroups of eight wavefronts (two per SIMD: a 16-row unit needs under half of a SIMD's
// registers), every wavefront drawing units until the queue is empty.
template <int DH>
__global__ __launch_bounds__(512) void decode_queue_kernel(const DecodeQueue q) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  decode_queue_worker<DH>(q, wave, threadIdx.x & 63,
                          q.trace ? q.trace + (size_t)TRACE_WORDS * (8 * blockIdx.x + wave) : nullptr);
}

// LDS of a blended launch: the ring of a prefill workgroup or the queries of four wide decode units
constexpr int BLENDED_LDS(int dh) {
  return PF_LDS(dh) > 2 * DECODE_Q_LDS(dh, 4) ? PF_LDS(dh) : 2 * DECODE_Q_LDS(dh, 4);
}

// a launch of 256-thread workgroups with `lds` bytes of dynamic LDS (`once`: one per kernel)
template <class Kernel, class... Args>
hipError_t launch_with_lds(Kernel kernel, OncePerDevice &once, int grid, int lds, hipStream_t stream, Args... args) {
  if (const hipError_t e = allow_lds(once, reinterpret_cast<const void *>(kernel), lds)) return e;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), lds, stream, args...);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_decode_queue(const DecodeQueue &q, int n_workgroups, hipStream_t stream) {
  if (q.n_units <= 0 || n_workgroups <= 0) return hipSuccess;
  if (q.d.s.head_dim == 128)
    hipLaunchKernelGGL((decode_queue_kernel<128>), dim3(n_workgroups), dim3(512), 0, stream, q);
  else if (q.d.s.head_dim == 64)
    hipLaunchKernelGGL((decode_queue_kernel<64>), dim3(n_workgroups), dim3(512), 0, stream, q);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_decode_attn(const DecodeArgs &a, int n_wide, int n_narrow, hipStream_t stream) {
  const int n_wide_units = n_wide * a.s.n_kv_heads, n_narrow_units = n_narrow * a.s.n_kv_heads;
  const dim3 grid(n_wide_units + n_narrow_units), block(64);
  if (grid.x == 0) return hipSuccess;
  if (n_wide <= 0 && a.s.head_dim == 128)
    hipLaunchKernelGGL((decode_narrow_kernel<128>), grid, block, 0, stream, a);
  else if (n_wide <= 0 && a.s.head_dim == 64)
    hipLaunchKernelGGL((decode_narrow_kernel<64>), grid, block, 0, stream, a);
  else if (a.s.head_dim == 128)
    hipLaunchKernelGGL((decode_attn_kernel<128>), grid, block, 0, stream, a, n_wide_units, n_narrow_units);
  else if (a.s.head_dim == 64)
    hipLaunchKernelGGL((decode_attn_kernel<64>), grid, block, 0, stream, a, n_wide_units, n_narrow_units);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_merge(const MergeArgs &a, hipStream_t stream) {
  const int dh = a.s.head_dim, hpw = 256 / dh;  // heads per wavefront
  const int n_decode_units = a.n_decode * ((a.s.n_q_heads + hpw - 1) / hpw);
  const int n_units = n_decode_units + (a.n_cut > 0 ? a.n_cut * (a.s.n_q_heads / a.cut_heads) * 4 * 2 * (dh / 8) : 0);
  if (n_units <= 0) return hipSuccess;
  if (dh == 128)
    hipLaunchKernelGGL((merge_kernel<128>), dim3((n_units + 3) / 4), dim3(256), 0, stream, a, n_decode_units, n_units);
  else if (dh == 64)
    hipLaunchKernelGGL((merge_kernel<64>), dim3((n_units + 3) / 4), dim3(256), 0, stream, a, n_decode_units, n_units);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

bool blended_attn_possible(const AttnShape &s) { return (s.n_q_heads / s.n_kv_heads) % 4 == 0; }

hipError_t launch_blended_attn(const DecodeArgs &d, int n_wide, int n_narrow, const PrefillArgs &pf, hipStream_t stream) {
  if (!blended_attn_possible(d.s)) return hipErrorInvalidValue;
  const int n_wide_units = n_wide * d.s.n_kv_heads, n_narrow_units = n_narrow * d.s.n_kv_heads;
  const int n_dec = (n_wide_units + 3) / 4 + (n_narrow_units + 3) / 4;
  const int n_pf = pf.n_work * (pf.s.n_q_heads / 4);
  if (n_dec <= 0 || n_pf <= 0) return hipErrorInvalidValue;
  // one workgroup in five is a prefill one until they run out (periods of 3 to 17 measured on the 8B and
  // 70B shapes: 3 and 5 are the fastest, the long ones cost 1-3 % of the launch); odd, so that the prefill
  // workgroups visit every XCD in turn
  const int period = n_dec >= 4 * n_pf ? 5 : 3;
  static OncePerDevice once[2];
  if (d.s.head_dim == 128)
    return launch_with_lds(blended_attn_kernel<128>, once[0], n_dec + n_pf, BLENDED_LDS(128), stream, d, n_wide_units, n_narrow_units, pf, n_pf, period);
  if (d.s.head_dim == 64)
    return launch_with_lds(blended_attn_kernel<64>, once[1], n_dec + n_pf, BLENDED_LDS(64), stream, d, n_wide_units, n_narrow_units, pf, n_pf, period);
  return hipErrorInvalidValue;
}

// Ring or direct: the shorter of two estimates (us), fitted to 332 launches of 4 to 64 heads in groups of 1,
// 2, 3, 5 and 6, 1 to 178 segments of 4 to 2048 rows behind 0 to 4000 tokens, each timed both ways: the launch
// is as long as its longest workgroup or as all of them on 256 CUs, whichever is more, and a fifth
// of the other.  A block of 32 tokens costs a ring workgroup a fixed part and one per wavefront that has rows;
// a direct wavefront 1.2 us alone and 0.45 of a full CU (128-wide heads), half that with at most 32 rows.
// Within 0.5 % of the faster kernel on average; the ring alone is 11 % off (up to 2.8 times: 128 segments of 16
// rows, 32 heads, 30 against 83 us), the direct kernel alone 10 %.  On 220 other launches: 7 % faster than the
// direct kernel alone on average, in three of them 5 to 8 % slower.
PrefillRoute prefill_route(const AttnShape &s, int n_prefill, const int32_t *row_start, const int32_t *kv_len) {
  const int grp = s.n_q_heads / s.n_kv_heads;
  if (grp % 4 == 0) return {false, 4, 64};  // four heads share every tile
  const int hpw = grp % 2 == 0 ? 2 : 1, ring_rows = 64 * (4 / hpw);
  const bool wide = s.head_dim == 128;
  const double alone = wide ? 1.2 : 0.88, shared = wide ? 0.45 : 0.21, fixed = wide ? 0.73 : 0.49, per_wave = wide ? 0.083 : 0.045,
               full = wide ? 1.2 : 1.0, start = wide ? 3.6 : 1.7;
  double d_long = 0, d_all = 0, r_long = 0, r_all = 0;
  for (int q = 0; q < n_prefill; ++q) {
    const int rows = row_start[q + 1] - row_start[q], before = kv_len[q] - rows;
    for (int r = 0; r < rows; r += 64) {
      const int n = std::min(64, rows - r);
      const double blocks = ((before + r + n - 1) / 32 + 1) * (n <= 32 ? 0.51 : 1.0);
      d_long = std::max(d_long, blocks * alone + 1.7);
      d_all += blocks * shared * hpw + 1.1;
    }
    for (int r = 0; r < rows; r += ring_rows) {
      const int n = std::min(ring_rows, rows - r);
      const double t = ((before + r + n - 1) / 32 + 1) * (fixed + per_wave * ((n + 63) / 64 * hpw));
      r_long = std::max(r_long, t + 1.8);
      r_all += t * full + start;
    }
  }
  const double wgs = (double)(s.n_q_heads / hpw) / 256.0;
  d_all *= wgs;
  r_all *= wgs;
  const bool direct = std::max(d_long, d_all) + 0.2 * std::min(d_long, d_all) <= std::max(r_long, r_all) + 0.2 * std::min(r_long, r_all);
  return {direct, hpw, direct ? 64 : ring_rows};
}

hipError_t launch_prefill_attn(const PrefillArgs &a, const PrefillRoute &route, hipStream_t stream) {
  if (a.n_work <= 0) return hipSuccess;
  if (a.cut && route.direct) return hipErrorInvalidValue;
  const int hpw = route.heads, grid = a.n_work * (a.s.n_q_heads / hpw);
  if (route.direct) {
    if (hpw > 2) return hipErrorInvalidValue;
    if (a.s.head_dim == 128) hipLaunchKernelGGL(prefill_direct_kernel<128>, dim3(grid), dim3(64 * hpw), 0, stream, a, hpw);
    else if (a.s.head_dim == 64) hipLaunchKernelGGL(prefill_direct_kernel<64>, dim3(grid), dim3(64 * hpw), 0, stream, a, hpw);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  }
  static OncePerDevice once[2];
  if (a.s.head_dim == 128) return launch_with_lds(prefill_attn_kernel<128>, once[0], grid, PF_LDS(128), stream, a, hpw);
  if (a.s.head_dim == 64) return launch_with_lds(prefill_attn_kernel<64>, once[1], grid, PF_LDS(64), stream, a, hpw);
  return hipErrorInvalidValue;
}

}  // namespace bs

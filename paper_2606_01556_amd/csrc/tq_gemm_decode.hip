// Fused dual-component W4A4 layer (paper Sec. 4.3) for decode-sized token
// counts (m <= 16): the residual 4-bit GEMM, the stage-1 product
// H = Q(X) Q(L1), its on-chip re-quantization, stage 2 Q_H Q(L2) and one
// epilogue, in one kernel.  Nothing of the layer leaves the chip but Y.
//
// Work decomposition.  One work-group of sixteen wavefronts per CU owns CT
// 16-column tiles of Y and streams their packed weights once.  H is small
// (m x r) and every work-group forms all of it itself, so no work-group waits
// for another; the price is that each CU reads all of L1 (from L2, where the
// first reader leaves it) in addition to its columns.
//  * K is cut into pairs of 64-wide blocks, and a wavefront takes whole pairs:
//    it reads the pair's activation operand once and multiplies it with the
//    pair's operands of every rank tile and every column tile (or S of them
//    share a pair, each with its part of the tiles).  So all sixteen wavefronts
//    carry the same work whatever the rank, and the activation operand is shared
//    by all tiles of a wavefront.
//  * The residual sums stay in the wavefront's registers; the partial sums of
//    the wavefronts are added in a fixed order at the end (the order of Y's
//    fp32 accumulation is free; H's is not).
//  * H is a chain over K: one fma per K-group, ascending.  The products that
//    feed it come from different wavefronts, so they pass through LDS: a
//    wavefront leaves I s_x (an exact fp32 value) of its pair there, and behind
//    a barrier one thread per element of H walks the chunk's groups in
//    ascending order with fma(I s_x, s_L1, h) -- the oracle's chain, so H is
//    bit-identical.  A chunk is the pairs the sixteen wavefronts hold at once.
//    The chain of one phase runs beside the products of the next (two buffers,
//    where LDS holds them).
//  * Weight and L1 operands stream from global memory straight into registers,
//    one chunk (two for few tiles) ahead.  The activation codes (a few KiB at
//    these sizes) are copied to LDS once, or, for the fp16 entry point,
//    quantized into LDS by the work-group itself (Sec. 4.3: the activation tile
//    is quantized once and reused by both branches), with the same arithmetic
//    as the quantizer kernel.
//
// Products.  v_mfma_scale_f32_16x16x128_f8f6f4 on codes as fp8 subnormals
// (block scales 2^9: exact integer sums).  A pair spans the 128 K of one
// product, and its two blocks need separate sums: rows 0-7 (up to 8 tokens)
// take block A's codes in k < 64 and rows 8-15 block B's in k >= 64 (zeros
// elsewhere), so one product yields both blocks' sums (A in lanes 0-31, B in
// lanes 32-63).  Only the accumulator rows that hold real tokens (MV of the
// four per lane) are rescaled.  9 to 16 tokens are two token blocks of half
// of them each in the grid.
//
// What bounds it.  No unit alone.  For 28672 -> 8192, r = 128, one token, the
// vector ALU is active 45 % of a SIMD's cycles (a 4-bit operand takes 12 integer
// instructions of four cycles to expand, three quarters of a tile's work), a CU's
// load path about 40 % (2.3 MB), the matrix cores 12 %; the rest is loads and
// chunk barriers waited for.  Before, each rank tile of H was one wavefront's own
// chain, ~48 instructions per pair one after the other, and its wavefront alone
// set the time.  us per launch from codes, weights in the memory-side cache (from
// HBM), one token unless said, before -> now: 4096 -> 4096, r = 64 9.4 -> 8.1 (11.4
// -> 9.5); 14336 -> 4096, r = 64 20.4 -> 14.9 (23.9 -> 18.5); 28672 -> 8192, r = 128,
// fp16 in 55.9 -> 49.8; 8192 -> 28672, r = 128 5 tokens 34.8 -> 28.9 (40.6 -> 35.0);
// 14336 -> 4096, r = 64 8 tokens 38.1 -> 21.6.  Slower than before: one and two
// tokens with the weights in the cache, N > 24576 (8192 -> 28672, r = 128 25.2 ->
// 27.2; from HBM 37.3 -> 35.6) and N > 16384 at K ~ 1280 (1280 -> 28672, r = 32 7.3 ->
// 8.2, from HBM even); 9 to
// 16 tokens, N > 24576, at K <= 1280 (10.7 -> 11.4 at 1280, r = 64), and from HBM at
// K >= 8192 with r <= 64 (14336 -> 28672, r = 64 57.7 -> 64.3; r = 128 faster): there
// two token blocks of sixteen tiles fetch more than the one of eight did.
// Tried and not kept: two pairs of a wavefront between barriers (no
// change), non-temporal weight or L1 loads (2-20 % slower), the chain after the
// products instead of ahead of them (8 % slower), a 16-token layout of two
// products per tile (44 us where two token blocks take 23: its products and
// codes fill the LDS, so nothing is double-buffered), three or four chunks of
// operands in flight (2-10 % slower: longer code), a test for pairs past K
// around the products (3-5 % slower on long K), and the kernel of before where N >
// 16384 (faster with the weights in the cache, 5-9 % slower from HBM).

#include <type_traits>

#include "tq_device.hpp"
#include "tq_kernels.hpp"

namespace tq {
namespace {

constexpr int DW = 16;                     // wavefronts per work-group
constexpr int kDecodeXBytes = 112 * 1024;  // LDS for the activation codes
constexpr int kDecodeLds = 160 * 1024;

// Token layouts: MODE tokens (1, 2, or 4: up to 8) with MV = MODE live
// accumulator rows per lane.
template <int MODE>
struct DMode {
  static constexpr int MV = MODE;
  // LDS copy of the activation codes: fp8 operand bytes for one or two tokens,
  // TQ4 words (unpacked at use) otherwise; MX token slots per K-group
  static constexpr bool XFP8 = MODE <= 2;
  static constexpr int MX = MODE <= 2 ? MODE : 8;
  static constexpr int XB = XFP8 ? 64 : 32;   // bytes per (group, token)
  // rank tiles of a wavefront whose products share one phase's buffer (16 or 32 KiB)
  static constexpr int PTM = 8 / MODE;
};

// R rank tiles and CT column tiles of a work-group.  S wavefronts share a pair,
// each with its part of the tiles.
constexpr int split_hs(int r, int s) { return r == 0 || r > s ? s : r; }   // of these, with rank tiles of their own (the others repeat them)
constexpr int split_ht(int r, int s) { return r / split_hs(r, s); }        // rank tiles of a wavefront
constexpr int split_cw(int ct, int s) { return ct > s ? ct / s : 1; }      // column tiles (fewer than S: kept by the first)
// The fewest wavefronts whose operands and sums fit their 128 registers (one
// token, eight column tiles, r = 32 in one wavefront spilled 24: 8192 -> 28672
// 28.9 us, 22.9 with two), or that are ever the fastest (the last line); and the
// most that still divide the tiles.
constexpr int split_min(int mode, int r, int ct) {
  if (ct >= 12 || (mode > 2 && r >= 4 && r + ct > 10)) return 4;
  if (r + ct > (mode == 1 ? 10 : (mode == 2 ? 8 : 5)) || ct == 8 || ct == 6) return 2;
  return mode > 2 && r == 4 ? 2 : 1;
}
constexpr int split_max(int mode, int r, int ct) {
  if (ct == 6) return 2;   // (three tiles each)
  const int tiles = r > ct ? r : ct, s = ct == 16 ? 8 : (tiles < 4 ? tiles : 4);
  return s > split_min(mode, r, ct) ? s : split_min(mode, r, ct);
}

// LDS layout (bytes).  K loop: the activation codes, their fp16 scales, NB
// buffers of H products [rank tile][block][16 ranks][MX tokens] fp32, and NB of
// L1 scales [group of the chunk][rank] fp16.  Epilogue, from the start: the
// residual partials, H, Q_H and s_H.
template <int MODE, int R, int CT, int S_>
struct DCfg {
  using MD = DMode<MODE>;
  static constexpr int S = S_;
  static constexpr int HS = split_hs(R, S), HT = split_ht(R, S), CW = split_cw(CT, S);
  static constexpr bool H = HT > 0;
  static constexpr int PCH = DW / S;                     // pairs of a chunk
  static constexpr int GL = 2 * PCH;                     // 64-wide blocks of a chunk
  static constexpr int NT = HT + CW;                     // tiles of a wavefront
  static constexpr int PD = NT + CW <= (MODE <= 2 ? 6 : 5) ? 2 : 1;   // chunks of operands in flight
  static constexpr int PT = HT < MD::PTM ? HT : MD::PTM; // rank tiles of a phase
  static constexpr int NPHASE = HT ? HT / PT : 0;
  static constexpr int EPT = 16 * MD::MX;                // elements of a rank tile
  static constexpr int EPS = PT * HS * EPT;              // elements of H of a phase
  // H products: up to two tokens [element][block] (each thread of the chain
  // reads its row 16 bytes at a time; rows padded so that neither side's lanes
  // meet in a bank), else [block][element]; L1 scales [rank][row] or [row][rank]
  static constexpr bool TR = MODE <= 2;
  static constexpr int PS = TR ? GL + 4 : 1, PG = TR ? 1 : EPT;   // element and block strides, floats
  static constexpr int SLS = GL < 8 ? 16 : GL + 8;        // rank stride of the transposed scales
  static constexpr int PBUF = PT * HS * EPT * (TR ? PS : GL) * 4;
  static constexpr int NH = HT && NPHASE * EPS > 64 * DW ? NPHASE * EPS / (64 * DW) : 1;   // per thread
  static constexpr int HSTR = kMaxRank + 1;              // fp32 per H row
  static constexpr int QSTR = kMaxRank + 16;             // bytes per Q_H row
  static constexpr int E_H = PCH * CT * 512;            // after the partials [PCH][CT][8][16] fp32
  static constexpr int E_Q = E_H + 16 * HSTR * 4;
  static constexpr int E_SH = E_Q + 16 * QSTR;
  static constexpr int E_END = E_SH + 2 * 16 * 4;
  static_assert(E_END <= kDecodeLds, "the epilogue fits");
};
struct DLayout {
  int xs, p, sl, nb, total;
  template <typename C>
  __host__ __device__ static DLayout make(int kg, int r_pad32) {
    const int kgp = (kg + 1) / 2 * 2;
    DLayout L;
    L.xs = (kgp * C::MD::MX * C::MD::XB + 32 + 15) / 16 * 16;   // + a 32-byte zero pad
    L.p = (L.xs + (kgp + 1) * C::MD::MX * 2 + 15) / 16 * 16;   // + a row of zeros
    const int buf = C::PBUF + (C::H ? r_pad32 * (C::TR ? C::SLS : C::GL) * 2 : 0);
    L.nb = L.p + 2 * buf <= kDecodeLds ? 2 : 1;
    L.sl = L.p + L.nb * C::PBUF;
    const int k_end = L.p + L.nb * buf;
    L.total = k_end > C::E_END ? k_end : C::E_END;
    return L;
  }
};

__host__ __device__ inline int rank_tiles(int r) { return (r + 15) / 16; }

// max over runs of n = 8, 16 or 32 aligned lanes, in every lane of the run
__device__ __forceinline__ float dpp_max(float a, int ctrl_sel) {
  int b;
  switch (ctrl_sel) {
    case 0: b = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, a), 0xB1, 0xF, 0xF, false); break;
    case 1: b = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, a), 0x4E, 0xF, 0xF, false); break;
    case 2: b = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, a), 0x141, 0xF, 0xF, false); break;
    default: b = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, a), 0x140, 0xF, 0xF, false); break;
  }
  return fmaxf(a, __builtin_bit_cast(float, b));
}
__device__ __forceinline__ float run_max(float a, int n, int lane) {
  a = dpp_max(a, 0);   // lane ^ 1
  a = dpp_max(a, 1);   // lane ^ 2
  a = dpp_max(a, 2);   // half-row mirror: 8 lanes
  if (n >= 16) a = dpp_max(a, 3);   // row mirror: 16 lanes
  if (n >= 32) {
    const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, a), 0));
    const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, a), 16));
    const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, a), 32));
    const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, a), 48));
    a = lane < 32 ? fmaxf(r0, r1) : fmaxf(r2, r3);
  }
  return a;
}

// lanes 0-31 receive lanes 32-63 of v (lanes 32-63 get their own values back)
__device__ __forceinline__ float upper_half(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, v),
                                                  __builtin_bit_cast(uint32_t, v), false, false);
  return __builtin_bit_cast(float, (uint32_t)r[1]);
}

__device__ __forceinline__ v8i lds_v8i(const uint8_t *p) {
  const u32x4 lo = *reinterpret_cast<const u32x4 *>(p);
  const u32x4 hi = *reinterpret_cast<const u32x4 *>(p + 16);
  return v8i{(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
}

__device__ __forceinline__ _Float16 half_of(uint32_t w, int hi) {
  return __builtin_bit_cast(_Float16, (uint16_t)(hi ? w >> 16 : w & 0xffffu));
}

// every LDS access of this wavefront so far has completed, then the work-group
// barrier (global loads into registers stay in flight across it)
__device__ __forceinline__ void d_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Raw buffer of `bytes` bytes at a wave-uniform address: loads past its end
// return zeros (and read nothing), so operands past K need no test.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t d_buffer(const uint8_t *p, uint32_t bytes) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(((uint64_t)hi << 32) | lo), 0,
                                           __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}
__device__ __forceinline__ u32x4 d_load16(__amdgpu_buffer_rsrc_t rsrc, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0);
}
__device__ __forceinline__ uint32_t d_load2(__amdgpu_buffer_rsrc_t rsrc, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b16(rsrc, off, 0, 0);
}

template <int MODE, int R, int CT, int S>
__global__ __launch_bounds__(64 * DW) void dual_gemm_decode_kernel(GemmArgs a,
                                                                   const uint16_t *__restrict__ xh, int mb) {
  using C = DCfg<MODE, R, CT, S>;
  using MD = DMode<MODE>;
  constexpr int MX = MD::MX, MV = MD::MV, XB = MD::XB, PCH = C::PCH, GL = C::GL;
  constexpr int HT = C::HT, CW = C::CW;
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  const Geometry &geo = a.geo;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, c16 = lane & 15, qh = q & 1, gq = q >> 1;
  const int KG = geo.k / kGroup, NP = (KG + 1) / 2, NCH = (NP + PCH - 1) / PCH;
  // Column block and token block (mb tokens from m0 on, m of them live).  Two
  // token blocks read the same weights: work-groups are dealt round-robin to
  // the 8 XCDs, so the two of a column block are placed on one, whose L2 then
  // serves the second -- if the two run in step, so they get half the tokens
  // each: with 8 + 1 the block with one token to quantize ran ahead and the
  // weights were fetched twice (8192 -> 28672 r = 0 from fp16, 9 tokens: 38 us;
  // 5 + 4: 26.5).
  // (One and two tokens are one block, and with a low-rank part go without this code:
  // it made the scalar registers of r = 64 with eight column tiles spill 48
  // against 11.  At r = 0 nothing spills either way, and the form with it
  // measured 2 to 7 % faster with the weights in HBM.)
  int cblk = blockIdx.x, m0 = 0, m = a.m;
  if constexpr (MODE > 2 || R == 0) {
    if (a.m > 8) {
      const int nwg = gridDim.x, per = nwg / 8, rem = nwg % 8, x = blockIdx.x % 8, i = blockIdx.x / 8;
      const int logical = (x < rem ? x * (per + 1) : rem * (per + 1) + (x - rem) * per) + i;
      cblk = logical / 2;
      m0 = logical % 2 * mb;
    }
    m = min(a.m - m0, mb);
  }
  const int r = geo.r, gk = geo.gk;
  const int ct16 = geo.n_pad / 16;
  const int c0 = cblk * CT;
  const DLayout LY = DLayout::make<C>(KG, geo.r_pad32);
  uint8_t *XA = smem;
  uint16_t *XS = reinterpret_cast<uint16_t *>(smem + LY.xs);
  const uint16_t *l2scales = reinterpret_cast<const uint16_t *>(a.packed + geo.off_l2s);

  // ---- this wavefront's pairs (pl of every chunk) and tiles ----
  const int sub = wave % S, pl = wave / S;
  const int hsub = sub % C::HS;
  const int rt0 = hsub * HT;                     // first rank tile
  const int ctw0 = c0 + sub % CT * CW;           // first column tile
  // Lane quarters q < 2 take block A = 2p of a pair, q >= 2 block B.  On an
  // odd tail (2p + 1 == KG), and past K, the loads return zeros.
  __amdgpu_buffer_rsrc_t tbuf[C::NT];
#pragma unroll
  for (int j = 0; j < HT; j++) {
    const int t = rt0 + j, half = (t & 1) * 256;
    tbuf[j] = d_buffer(a.packed + geo.off_l1 + (int64_t)(t >> 1) * KG * 1024 + half, (uint32_t)KG * 1024u - half);
  }
  uint32_t ws_lane[CW];
#pragma unroll
  for (int j = 0; j < CW; j++) {
    const int ct = min(ctw0 + j, ct16 - 1), half = (ct & 1) * 256;   // past the last tile: never stored
    tbuf[HT + j] = d_buffer(a.packed + geo.off_w + (int64_t)(ct >> 1) * KG * 1024 + half, (uint32_t)KG * 1024u - half);
    ws_lane[j] = (uint32_t)(16 * ct + c16) * 2;
  }
  // scale rows: one per quantization group (gk blocks)
  const int KQ = KG / gk;
  const auto wsbuf = d_buffer(a.packed + geo.off_ws, (uint32_t)KQ * (uint32_t)geo.n_pad * 2u);
  const uint32_t ws_row = (uint32_t)geo.n_pad * 2u;
  struct Slot {
    u32x4 b[C::NT];
    uint32_t sw[CW];   // fp16 weight scales of the lane's own block
  };
  const uint32_t code_lane = (uint32_t)(gq * 1024 + qh * 512 + c16 * 16);
  // offsets of the next pair to load, which advance chunk by chunk
  uint32_t code_off = (uint32_t)pl * 2048u + code_lane;
  const uint32_t ws_b = gk == 1 ? ws_row : 0u;   // block B's row: the next one, or the same group's
  uint32_t ws_off = (uint32_t)(2 * pl / gk) * ws_row + (gq ? ws_b : 0u);
  const uint32_t ws_step = (uint32_t)(GL / gk) * ws_row;
  auto load_tile = [&](Slot &Q, int j) { Q.b[j] = d_load16(tbuf[j], code_off); };
  auto load_scales = [&](Slot &Q) {   // and on to the next pair
#pragma unroll
    for (int j = 0; j < CW; j++) Q.sw[j] = d_load2(wsbuf, ws_off + ws_lane[j]);
    code_off += PCH * 2048u;
    ws_off += ws_step;
  };

  // ---- L1 scales of a chunk: its GL / gk rows, 16 bytes (8 ranks) a thread,
  // as they lie or transposed (lanes along the rows then) ----
  const int sl_rows = GL / gk;
  const int sl_row = C::TR ? tid % GL : tid / (geo.r_pad32 / 8 > 0 ? geo.r_pad32 / 8 : 1);
  const int sl_part = C::TR ? tid / GL : tid % (geo.r_pad32 / 8 > 0 ? geo.r_pad32 / 8 : 1);
  const bool sl_live = HT && sl_row < sl_rows && sl_part < geo.r_pad32 / 8;
  const auto slbuf = d_buffer(a.packed + geo.off_l1s, HT ? (uint32_t)KQ * (uint32_t)geo.r_pad32 * 2u : 0u);
  u32x4 slreg = {0u, 0u, 0u, 0u};
  uint32_t sl_off = (uint32_t)sl_row * (uint32_t)geo.r_pad32 * 2u + (uint32_t)sl_part * 16u;
  auto sl_load = [&]() {   // and on to the next chunk
    slreg = d_load16(slbuf, sl_off);
    sl_off += (uint32_t)(sl_rows * geo.r_pad32 * 2);
  };
  const int sl_buf = geo.r_pad32 * (C::TR ? C::SLS : GL) * 2;
  auto sl_write = [&](int c) {
    if (sl_live) {
      uint8_t *B = smem + LY.sl + (LY.nb == 2 ? (c & 1) * sl_buf : 0);
      if constexpr (C::TR) {
        uint16_t *D = reinterpret_cast<uint16_t *>(B) + sl_part * 8 * C::SLS + sl_row;
#pragma unroll
        for (int e = 0; e < 4; e++) {
          D[2 * e * C::SLS] = (uint16_t)(slreg[e] & 0xffffu);
          D[(2 * e + 1) * C::SLS] = (uint16_t)(slreg[e] >> 16);
        }
      } else {
        *reinterpret_cast<u32x4 *>(B + (sl_row * geo.r_pad32 + sl_part * 8) * 2) = slreg;
      }
    }
  };

  // ---- fp16 activations to quantize: eight lanes per (token, quantization
  // group), eight values of each of its blocks, XI items of a thread ahead.
  // Their loads go first: loads return in order, and the first barrier waits
  // for these ----
  constexpr int XI = 2;
  const int nitem = m * KQ, xe = lane & 7;
  constexpr int XSTEP = 64 * DW / 8;              // items of one pass of the work-group
  // (token, quantization group) of this thread's next item to load and to
  // quantize, stepped without a division
  const int xdt = XSTEP / KQ, xdg = XSTEP % KQ;
  struct XPos {
    int t, g;
  };
  auto x_next = [&](XPos &p) {
    p.t += xdt;
    p.g += xdg;
    if (p.g >= KQ) {
      p.g -= KQ;
      p.t++;
    }
  };
  u32x4 xr0[XI], xr1[XI];
  XPos xl = {tid / 8 / KQ, tid / 8 % KQ}, xq = xl;
  auto x_load = [&](int it0) {   // past the last item: item 0, not written
#pragma unroll
    for (int i = 0; i < XI; i++) {
      if (it0 + i * XSTEP >= nitem) break;
      const bool live = xl.t < m;
      const uint16_t *src = xh + (int64_t)(m0 + (live ? xl.t : 0)) * geo.k + (live ? xl.g * gk : 0) * kGroup + 8 * xe;
      xr0[i] = *reinterpret_cast<const u32x4 *>(src);
      if (gk == 2) xr1[i] = *reinterpret_cast<const u32x4 *>(src + kGroup);
      x_next(xl);
    }
  };
  // quantized activations: a thread's first 16-byte fragment (block, token,
  // half) of tile 0's TQ4 blocks and its first scale, ahead likewise
  const int nfrag = KG * m * 2, nxs = (2 * NP + 1) * MX;
  auto frag = [&](int f) {
    const int g = f / (2 * m), t = (f / 2) % m, h = f & 1;
    return *reinterpret_cast<const u32x4 *>(reinterpret_cast<const uint8_t *>(a.xc) + ((int64_t)g * 64 + 32 * h + m0 + t) * 16);
  };
  auto xscale = [&](int idx) {   // zeros past m and past K
    const int g = idx / MX, t = idx % MX;
    return g < KG && t < m ? a.xs[(int64_t)(g / gk) * a.ms + m0 + t] : (uint16_t)0;
  };
  u32x4 frag0 = {0u, 0u, 0u, 0u};
  uint16_t xscale0 = 0;
  if (xh != nullptr) {
    x_load(0);
  } else {
    if (tid < nfrag) frag0 = frag(tid);
    if (tid < nxs) xscale0 = xscale(tid);
  }

  // ---- first loads: operands of the first chunks, stage-2 operands of the
  // storing wavefronts, L1 scales ----
  Slot ring[C::PD];
#pragma unroll
  for (int u = 0; u < C::PD; u++) {
#pragma unroll
    for (int j = 0; j < C::NT; j++) load_tile(ring[u], j);
    load_scales(ring[u]);
  }
  if constexpr (HT > 0) sl_load();
  const int RB = (r + 63) / 64;   // 64-rank blocks of stage 2 (<= 2)
  const int ct_out = min(c0 + (wave < CT ? wave : 0), ct16 - 1);
  u32x4 l2raw = {0u, 0u, 0u, 0u};
  uint32_t l2sa = 0, l2sb = 0;
  const int hg1 = r > 0 ? 64 / geo.gr : 0;   // rank group of the second 64-rank block (0 if gr = 128)
  if (HT > 0 && wave < CT) {
    const int rbq = min(gq, RB - 1), L = qh * 32 + (ct_out & 1) * 16 + c16;
    l2raw = *reinterpret_cast<const u32x4 *>(
        a.packed + geo.off_l2 + (((int64_t)(ct_out >> 1) * (geo.r_pad64 / 64) + rbq) * 64 + L) * 16);
    l2sa = l2scales[ct_out * 16 + c16];
    l2sb = RB > 1 ? l2scales[(int64_t)hg1 * geo.n_pad + ct_out * 16 + c16] : 0u;
  }

  // ---- the activation codes and scales into LDS ----
  const int KGP = 2 * NP;
  if (xh != nullptr) {
    // the steps of the quantizer kernel, so the codes and scales are the same bits
    for (int it0 = 0; it0 < nitem; it0 += XI * XSTEP) {
      if (it0 > 0) x_load(it0);
#pragma unroll
      for (int i = 0; i < XI; i++) {
        if (it0 + i * XSTEP >= nitem) break;
        const int t = xq.t, g0 = xq.g * gk;
        const bool live = t < m;
        x_next(xq);
        float v0[8], v1[8];
#pragma unroll
        for (int e = 0; e < 4; e++) {
          v0[2 * e] = half_bits_to_float((uint16_t)(xr0[i][e] & 0xffffu));
          v0[2 * e + 1] = half_bits_to_float((uint16_t)(xr0[i][e] >> 16));
        }
        float amax = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; e++) amax = fmaxf(amax, fabsf(v0[e]));
        if (gk == 2) {
#pragma unroll
          for (int e = 0; e < 4; e++) {
            v1[2 * e] = half_bits_to_float((uint16_t)(xr1[i][e] & 0xffffu));
            v1[2 * e + 1] = half_bits_to_float((uint16_t)(xr1[i][e] >> 16));
          }
#pragma unroll
          for (int e = 0; e < 8; e++) amax = fmaxf(amax, fabsf(v1[e]));
        }
        amax = max8_dpp(amax);
        uint16_t s16;
        const float sc = q4_scale(amax, s16);
        const float y = sc == 0.0f ? 0.0f : __builtin_amdgcn_rcpf(sc);
        auto put = [&](const float (&v)[8], int g) {
          uint32_t b0, b1;
          quant8_fp8(v, sc, y, b0, b1);
          if (live) {
            uint8_t *dst = XA + (g * MX + t) * XB;
            if constexpr (MD::XFP8)
              *reinterpret_cast<uint2 *>(dst + 8 * xe) = make_uint2(b0, b1);
            else
              *reinterpret_cast<uint32_t *>(dst + 4 * xe) = b0 | __builtin_amdgcn_alignbit(b1, b1, 28);
            if (xe == 0) XS[g * MX + t] = s16;
          }
        };
        put(v0, g0);
        if (gk == 2) put(v1, g0 + 1);
      }
    }
    for (int idx = tid; idx < (KGP + 1) * MX; idx += 64 * DW)
      if (idx / MX >= KG || idx % MX >= m) XS[idx] = 0;
  } else {
    for (int f = tid; f < nfrag; f += 64 * DW) {
      const int g = f / (2 * m), t = (f / 2) % m, h = f & 1;
      const u32x4 raw = f < 64 * DW ? frag0 : frag(f);
      uint8_t *dst = XA + (g * MX + t) * XB;
      if constexpr (MD::XFP8) {
        const v8i o = unpack32(raw);
        *reinterpret_cast<u32x4 *>(dst + 32 * h) = u32x4{(uint32_t)o[0], (uint32_t)o[1], (uint32_t)o[2], (uint32_t)o[3]};
        *reinterpret_cast<u32x4 *>(dst + 32 * h + 16) = u32x4{(uint32_t)o[4], (uint32_t)o[5], (uint32_t)o[6], (uint32_t)o[7]};
      } else {
        *reinterpret_cast<u32x4 *>(dst + 16 * h) = raw;
      }
    }
    for (int idx = tid; idx < nxs; idx += 64 * DW) XS[idx] = idx < 64 * DW ? xscale0 : xscale(idx);
  }
  // zero codes for the token slots past m, the odd tail block and the pad that
  // lanes outside the operand's live rows read
  for (int idx = tid; idx < KGP * MX * XB / 16 + 2; idx += 64 * DW) {
    const int e = idx * 16;
    const int g = e / (MX * XB), t = (e / XB) % MX;
    if (idx >= KGP * MX * XB / 16 || g >= KG || t >= m)
      *reinterpret_cast<u32x4 *>(XA + e) = u32x4{0u, 0u, 0u, 0u};
  }
  d_barrier();

  // Activation operand of pair p: lanes outside the operand's live rows (block
  // A lives in rows 0-7 of quarters 0-1, block B in rows 8-15 of quarters 2-3;
  // one and two tokens twice in each eight), past the MX token slots or past K
  // read the zero pad after the codes; the others their (block 2p + gq, token,
  // half) slot, zero past m.
  const int arow = lane & 15;
  const int atok = MODE <= 2 ? (arow & 3) : (arow & 7);
  const int xpad = KGP * MX * XB;
  auto act_op = [&](int p) -> v8i {
    const bool alive = (arow < 8) == (q < 2) && atok < MX && p < NP;
    const uint8_t *src = XA + (alive ? ((2 * p + gq) * MX + atok) * XB + qh * (XB / 2) : xpad);
    if constexpr (MD::XFP8) return lds_v8i(src);
    else return unpack32(*reinterpret_cast<const u32x4 *>(src));
  };
  // the fp16 activation scales of this lane's accumulator rows (consecutive
  // tokens) for block g, as one or two words; zero past K
  struct Sx {
    uint32_t w0, w1;
  };
  auto xs_row = [&](int g) -> Sx {
    const uint16_t *p = XS + min(g, KGP) * MX + (4 * qh < MX ? 4 * qh : 0);
    Sx s = {0u, 0u};
    if constexpr (MV == 1) {
      s.w0 = *p;
    } else if constexpr (MV == 2) {
      s.w0 = *reinterpret_cast<const uint32_t *>(p);
    } else {
      const uint2 t = *reinterpret_cast<const uint2 *>(p);
      s.w0 = t.x;
      s.w1 = t.y;
    }
    return s;
  };
  // I s_x of the lane's rows: exact in fp32 (|I| < 2^12 times an 11-bit
  // significand), so fma(I s_x, s_L1, h) rounds the same exact value once as
  // fma(I, s_x s_L1, h) does
  auto times_sx = [&](v4f I, Sx s) -> v4f {
    v4f t = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int v = 0; v < MV; v++) t[v] = fmaf(I[v], (float)half_of(v < 2 ? s.w0 : s.w1, v & 1), 0.0f);
    return t;
  };

  v4f acc[CW];
#pragma unroll
  for (int j = 0; j < CW; j++) acc[j] = v4f{0, 0, 0, 0};
  float h[C::NH];
#pragma unroll
  for (int e = 0; e < C::NH; e++) h[e] = 0.0f;

  // One phase's part of the chain: thread e of the phase's EPS (over all
  // wavefronts, a different start per phase) walks the blocks of chunk c.
  auto h_thread = [&](int k) { return ((wave - k * C::EPS / 64) & (DW - 1)) * 64 + lane; };
  auto h_rank = [&](int k, int e) {   // rank of thread e's element in phase k
    const int bt = e / C::EPT;
    return (bt / (C::PT > 0 ? C::PT : 1) * HT + k * C::PT + bt % (C::PT > 0 ? C::PT : 1)) * 16 + e % C::EPT / MX;
  };
  auto chain = [&](int k, int buf, int c, float &hv) {
    int e = h_thread(k);
    asm volatile("" : "+v"(e));   // its addresses are formed here, not kept over the K loop
    if (e < C::EPS) {
      const float *P = reinterpret_cast<const float *>(smem + LY.p + buf * C::PBUF) +
                       (C::TR ? e * C::PS : e / C::EPT * GL * C::EPT + e % C::EPT);
      const uint16_t *sl = reinterpret_cast<const uint16_t *>(smem + LY.sl + (LY.nb == 2 ? (c & 1) * sl_buf : 0)) +
                           (C::TR ? h_rank(k, e) * C::SLS : h_rank(k, e));
      const int rs = geo.r_pad32;
      float t = hv;
      // NG groups' products (128-wide groups: a group's two blocks' products
      // with s_x add exactly, |I| < 2^13, into its one step) and scales, in
      // batches of B
      auto walk = [&](auto NGC, auto GKC) {
        constexpr int NG = decltype(NGC)::value, GK = decltype(GKC)::value, B = NG < 8 ? NG : 8;
#pragma unroll
        for (int g0 = 0; g0 < NG; g0 += B) {
          if (g0 > 0 && c * NG + g0 >= KQ) break;   // the rest of the last chunk adds zeros
          float p8[B];
          _Float16 s8[B];
          if constexpr (C::TR) {
            const u32x4 w = *reinterpret_cast<const u32x4 *>(sl + g0);
#pragma unroll
            for (int i = 0; i < B; i++) s8[i] = half_of(w[i / 2], i & 1);
#pragma unroll
            for (int i = 0; i < B * GK / 4; i++) {
              const v4f w4 = *reinterpret_cast<const v4f *>(P + g0 * GK + 4 * i);
              if constexpr (GK == 1) {
#pragma unroll
                for (int j = 0; j < 4; j++) p8[4 * i + j] = w4[j];
              } else {
                p8[2 * i] = w4[0] + w4[1];
                p8[2 * i + 1] = w4[2] + w4[3];
              }
            }
          } else {
#pragma unroll
            for (int i = 0; i < B; i++) {
              s8[i] = half_of(sl[(g0 + i) * rs], 0);
              const float *pg = P + (g0 + i) * GK * C::PG;
              p8[i] = GK == 1 ? pg[0] : pg[0] + pg[C::PG];
            }
          }
#pragma unroll
          for (int i = 0; i < B; i++) t = fmaf(p8[i], (float)s8[i], t);
          if (!C::TR) __builtin_amdgcn_sched_barrier(0);   // a batch at a time: registers
        }
      };
      if (gk == 1) walk(std::integral_constant<int, GL>{}, std::integral_constant<int, 1>{});
      else walk(std::integral_constant<int, GL / 2>{}, std::integral_constant<int, 2>{});
      hv = t;
    }
  };

  // ---- K loop ----
  // the chain's few wavefronts (up to two tokens) end last: theirs go first
  if (HT > 0 && MODE <= 2 && wave * 64 < C::EPS) __builtin_amdgcn_s_setprio(2);
  int phase = 0;
  auto chunk = [&](int c, Slot &Q) {
    const int p = c * PCH + pl;   // this wavefront's pair
    const v8i av = act_op(p);
    const Sx sx = xs_row(2 * p + gq);
    auto h_tile = [&](int j, int pt, float *P) {
      const v8i b = unpack32(Q.b[j]);
      load_tile(Q, j);
      float *D = C::TR ? P + ((hsub * C::PT + pt) * C::EPT + c16 * MX) * C::PS + 2 * pl
                       : P + ((hsub * C::PT + pt) * GL + 2 * pl) * C::EPT + c16 * MX;
      // (one and two tokens: rows 4-7 repeat rows 0-3, so lanes 16-31 and 48-63
      // write their neighbours' values to the same place)
      const v4f t = times_sx(mfma_codes_16x16x128(av, b), sx);
      if constexpr (MODE == 1) {
        D[gq] = t[0];
      } else if constexpr (MODE == 2) {
        D[gq] = t[0];
        D[gq + C::PS] = t[1];
      } else {
        *reinterpret_cast<v4f *>(D + gq * C::EPT + 4 * qh) = t;
      }
    };
    auto residual = [&]() {
#pragma unroll
      for (int j = 0; j < CW; j++) {
        if (MODE > 2) __builtin_amdgcn_sched_barrier(0);
        const v8i b = unpack32(Q.b[HT + j]);
        load_tile(Q, HT + j);
        const v4f t = times_sx(mfma_codes_16x16x128(av, b), sx);
        const float sw = (float)half_of(Q.sw[j], 0);
#pragma unroll
        for (int v = 0; v < MV; v++) acc[j][v] = fmaf(t[v], sw, acc[j][v]);
      }
    };
    if constexpr (HT == 0) {
      residual();
      load_scales(Q);
    } else {
#pragma unroll
      for (int k = 0; k < C::NPHASE; k++, phase++) {
        const int buf = LY.nb == 2 ? phase & 1 : 0;
        // the chain of the phase before (its products are behind the last
        // barrier), ahead of this phase's products: its few wavefronts wait on
        // LDS and on their own fmas while the others multiply; with one buffer
        // it must end before the products are overwritten
        const int kp = k > 0 ? k - 1 : C::NPHASE - 1;
        if (phase > 0) {
          chain(kp, LY.nb == 2 ? buf ^ 1 : 0, k > 0 ? c : c - 1, h[kp * C::EPS / (64 * DW)]);
          if (LY.nb == 1) d_barrier();
        }
        float *P = reinterpret_cast<float *>(smem + LY.p + buf * C::PBUF);
#pragma unroll
        for (int pt = 0; pt < C::PT; pt++) h_tile(k * C::PT + pt, pt, P);
        if (MODE > 2) __builtin_amdgcn_sched_barrier(0);   // (more operands at once would not fit the registers)
        if (k == 0) {
          sl_write(c);
          sl_load();
          residual();
        }
        if (k == C::NPHASE - 1) load_scales(Q);
        d_barrier();
      }
    }
  };
  for (int c = 0; c < NCH; c += C::PD) {
#pragma unroll
    for (int u = 0; u < C::PD; u++)
      if (C::PD == 1 || c + u < NCH) chunk(c + u, ring[u]);
  }
  if constexpr (HT > 0)
    chain(C::NPHASE - 1, LY.nb == 2 ? (phase - 1) & 1 : 0, NCH - 1, h[(C::NPHASE - 1) * C::EPS / (64 * DW)]);
  __builtin_amdgcn_s_setprio(0);
  d_barrier();   // every wavefront is done with the K loop's LDS

  // ---- epilogue: residual partials, H, re-quantization, stage 2, store ----
  float *RES = reinterpret_cast<float *>(smem);                // [PCH][CT][8 tokens][16 columns]
  float *HS = reinterpret_cast<float *>(smem + C::E_H);        // [16][HSTR]
  uint8_t *QS = smem + C::E_Q;                                  // [16][QSTR] fp8 codes
  float *SHS = reinterpret_cast<float *>(smem + C::E_SH);      // [2][16]
  constexpr int HSTR = C::HSTR, QSTR = C::QSTR;
#pragma unroll
  for (int j = 0; j < CW; j++)
#pragma unroll
    for (int v = 0; v < MV; v++) {
      const float val = acc[j][v] + upper_half(acc[j][v]);   // block A + block B partials
      const int t = 4 * qh + v;
      if (lane < 32 && (S == 1 || sub * CW + j < CT)) RES[((pl * CT + sub * CW + j) * 8 + t) * 16 + c16] = val;
    }
  if constexpr (HT > 0) {
#pragma unroll
    for (int k = 0; k < C::NPHASE; k++) {
      const int e = h_thread(k);
      if (e < C::EPS) HS[e % MX * HSTR + h_rank(k, e)] = h[k * C::EPS / (64 * DW)];
    }
    for (int idx = tid; idx < 16 * RB * 64; idx += 64 * DW) {
      const int row = idx / (RB * 64), j = idx % (RB * 64);
      if (j >= r) QS[row * QSTR + j] = 0;
    }
  }
  d_barrier();

  if constexpr (HT > 0) {
    // Re-quantize H per token and rank group (s_H stays fp32).  Half a
    // wavefront per token row (wavefront w < 8: rows 2w, 2w + 1); lane j of
    // the half takes ranks epl j .. epl j + epl - 1, so a rank group is a run
    // of gr / epl lanes and its max is a shuffle reduction over them.
    if (wave < 8) {
      const int gr = geo.gr, rg = r / gr;
      const int epl = r >= 32 ? r / 32 : 1;      // ranks per lane: 1, 2 or 4
      const int row = 2 * wave + (lane >> 5), j = lane & 31;
      const int lpg = gr / epl;                  // lanes per rank group (<= 32)
      const int hg = j / lpg;
      const bool valid = j * epl < r;
      const bool live = valid && row < m;
      const bool dbg = a.dbg_h != nullptr && cblk == 0;
      float hv[4];
      float amax = 0.0f;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        hv[e] = live && e < epl ? HS[row * HSTR + j * epl + e] : 0.0f;
        amax = fmaxf(amax, fabsf(hv[e]));
      }
      amax = run_max(amax, lpg, lane);
      const float sh = amax / 7.0f;   // IEEE division
      if (valid) {
        uint32_t w = 0;
#pragma unroll
        for (int e = 0; e < 4; e++) {
          if (e < epl) {
            int qv = 0;
            if (sh != 0.0f) {
              float tq = __builtin_rintf(hv[e] / sh);
              tq = tq > 7.0f ? 7.0f : (tq < -7.0f ? -7.0f : tq);
              qv = (int)tq;
            }
            w |= code_to_fp8(qv) << (8 * e);
            if (dbg && row < m) {
              a.dbg_h[(int64_t)(m0 + row) * r + j * epl + e] = hv[e];
              a.dbg_qh[(int64_t)(m0 + row) * r + j * epl + e] = (int8_t)qv;
            }
          }
        }
        uint8_t *qd = QS + row * QSTR + j * epl;
        if (epl == 4) *reinterpret_cast<uint32_t *>(qd) = w;
        else if (epl == 2) *reinterpret_cast<uint16_t *>(qd) = (uint16_t)w;
        else *qd = (uint8_t)w;
        if (j % lpg == 0) {
          SHS[hg * 16 + row] = sh;
          if (dbg && row < m) a.dbg_sh[(int64_t)(m0 + row) * rg + hg] = sh;
        }
      }
    }
    d_barrier();
  }

  // ---- stage 2 and the single epilogue: wavefront j < CT stores tile j ----
  const v8i z8 = {0, 0, 0, 0, 0, 0, 0, 0};
  if (wave < CT) {
    const int j = wave;
    const int ct = c0 + j;
    if (ct < ct16) {
      v4f ylr = v4f{0, 0, 0, 0};
      const int orow0 = 4 * q;   // output rows 4q .. 4q + 3 of this lane
      if constexpr (HT > 0) {
        const float s2a = half_bits_to_float((uint16_t)l2sa), s2b = half_bits_to_float((uint16_t)l2sb);
        const v8i qa = lds_v8i(QS + c16 * QSTR + min(gq, RB - 1) * 64 + qh * 32);
        const v8i lb = unpack32(l2raw);
        {
          const v4f cb = mfma_codes_16x16x128(q < 2 ? qa : z8, lb);
#pragma unroll
          for (int v = 0; v < 4; v++) ylr[v] = fmaf(cb[v], SHS[orow0 + v] * s2a, ylr[v]);
        }
        if (RB > 1) {
          const v4f cb = mfma_codes_16x16x128(q < 2 ? z8 : qa, lb);
#pragma unroll
          for (int v = 0; v < 4; v++) ylr[v] = fmaf(cb[v], SHS[16 * hg1 + orow0 + v] * s2b, ylr[v]);
        }
      }
      // the matrix-core products above read operands from every lane: keep
      // them out of the per-lane store branch below
      asm volatile("" : "+v"(ylr));
      const int col = ct * 16 + c16;
      if (col < geo.n) {
#pragma unroll
        for (int v = 0; v < 4; v++) {
          const int row = orow0 + v;
          if (row < m) {
            float yres = 0.0f;
#pragma unroll
            for (int w2 = 0; w2 < PCH; w2++) yres += RES[((w2 * CT + j) * 8 + row) * 16 + c16];
            const float yv = yres + ylr[v];
            const uint16_t bits = a.bf16_out ? float_to_bf16_bits(yv) : float_to_half_bits(yv);
            reinterpret_cast<uint16_t *>(a.y)[(int64_t)(m0 + row) * geo.n + col] = bits;
          }
        }
      }
    }
  }
}

// tokens of a token block
int decode_block_tokens(int m) { return m <= 8 ? 8 : (m + 1) / 2; }

template <int MODE, int R, int CT, int S>
hipError_t launch_decode(const GemmArgs &a, const uint16_t *xh, hipStream_t s) {
  using C = DCfg<MODE, R, CT, S>;
  const DLayout LY = DLayout::make<C>(a.geo.k / kGroup, a.geo.r_pad32);
  const int tiles16 = a.geo.n_pad / 16;
  if (a.geo.gk != 1 && a.geo.gk != 2) return hipErrorInvalidValue;
  auto kern = dual_gemm_decode_kernel<MODE, R, CT, S>;
  hipError_t e = allow_lds(reinterpret_cast<const void *>(kern), LY.total);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((tiles16 + CT - 1) / CT * ((a.m + 7) / 8)), dim3(64 * DW), LY.total, s, a, xh,
                     decode_block_tokens(a.m));
  return hipGetLastError();
}

// Wavefronts per pair.  A chunk takes a wavefront its tiles' time (a rank tile
// 0.7 of a column tile, which has scales of its own) and about one tile's more
// for the barrier and the chain; filling the first chunk and the epilogue take
// about 1.5 times the tiles.  So a K of few pairs, whose only chunk would leave
// most wavefronts without one, is split wide (512 -> 4096 r = 128, one token:
// four per pair 6.7 us, one 8.4), and one that fills whole chunks as little as
// the registers allow (28672 -> 8192 r = 128: one per pair 39 us, two 41, four
// 52).  A wider split has to be 4 % cheaper: its chunks are shorter, which
// costs 3 to 5 % where the weights come from HBM.  The choice is within 5 % of
// the fastest at 98 % of 2200 calls timed (K 512 to 28672, N 512 to 28672, r 0
// to 128, both group widths).
constexpr int split_cost(int r, int ct, int s, int pairs) {
  const int pch = DW / s, chunks = (pairs + pch - 1) / pch;
  const int tiles = 7 * split_ht(r, s) + 10 * split_cw(ct, s);
  return 2 * chunks * (tiles + 10) + 3 * tiles;
}

template <int MODE, int R, int CT, int S>
hipError_t launch_decode_s(int split, const GemmArgs &a, const uint16_t *xh, hipStream_t s) {
  if constexpr (S < split_max(MODE, R, CT)) {
    if (split > S) return launch_decode_s<MODE, R, CT, 2 * S>(split, a, xh, s);
  }
  return launch_decode<MODE, R, CT, S>(a, xh, s);
}

template <int MODE, int R, int CT>
hipError_t launch_decode_ct(const GemmArgs &a, const uint16_t *xh, hipStream_t s) {
  constexpr int lo = split_min(MODE, R, CT), hi = split_max(MODE, R, CT);
  const int pairs = (a.geo.k / kGroup + 1) / 2;
  int split = lo;
  for (int c = 2 * lo; c <= hi; c *= 2)
    if (25 * split_cost(R, CT, c, pairs) < 24 * split_cost(R, CT, split, pairs)) split = c;
  return launch_decode_s<MODE, R, CT, lo>(split, a, xh, s);
}

template <int MODE, int R>
hipError_t launch_decode_r(int ct, const GemmArgs &a, const uint16_t *xh, hipStream_t s) {
  if constexpr (MODE <= 2) {
    if (ct == 6) return launch_decode_ct<MODE, R, 6>(a, xh, s);
  } else {
    if (ct == 12) return launch_decode_ct<MODE, R, 12>(a, xh, s);
  }
  switch (ct) {
    case 1: return launch_decode_ct<MODE, R, 1>(a, xh, s);
    case 2: return launch_decode_ct<MODE, R, 2>(a, xh, s);
    case 4: return launch_decode_ct<MODE, R, 4>(a, xh, s);
    case 8: return launch_decode_ct<MODE, R, 8>(a, xh, s);
    default: return launch_decode_ct<MODE, R, 16>(a, xh, s);
  }
}

// The fewest 16-column tiles per work-group that keep the grid within one
// work-group per CU.  Where a power of two would leave up to half of the CUs
// without one, also twelve from three tokens on (14336 -> 16416, 16 tokens, from
// HBM r = 0 47.7 -> 38.3 us, the kernel of before 36.8; r = 64 59.5 -> 49.1, 53.4) and
// six for one and two (8192 -> 18944, r = 128, one token 22.9 -> 21.3 us, before 21.9;
// from HBM 32.1 -> 29.8, 33.6) -- these from K = 2048, since six are shared by two
// wavefronts only and a short K is faster shared out wider (1280 -> 18944, r = 128
// 8.9 against 9.5 us).  Sixteen for one and two tokens, N > 32768, are far ahead
// of before as they are.
int decode_tiles(const GemmArgs &a) {
  const int tiles16 = a.geo.n_pad / 16 * ((a.m + 7) / 8);
  if (a.m > 2 && tiles16 > 2048 && tiles16 <= 3072) return 12;
  if (a.m <= 2 && tiles16 > 1024 && tiles16 <= 1536 && a.geo.k >= 2048) return 6;
  return tiles16 <= 256 ? 1 : (tiles16 <= 512 ? 2 : (tiles16 <= 1024 ? 4 : (tiles16 <= 2048 ? 8 : 16)));
}

template <int MODE>
hipError_t launch_decode_mode(const GemmArgs &a, const uint16_t *xh, hipStream_t s) {
  const int ct = decode_tiles(a);
  switch (rank_tiles(a.geo.r)) {
    case 0: return launch_decode_r<MODE, 0>(ct, a, xh, s);
    case 1: return launch_decode_r<MODE, 1>(ct, a, xh, s);
    case 2: return launch_decode_r<MODE, 2>(ct, a, xh, s);
    case 4: return launch_decode_r<MODE, 4>(ct, a, xh, s);
    case 8: return launch_decode_r<MODE, 8>(ct, a, xh, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// K for which the decode kernel takes m tokens: 112 KiB of codes, as fp8 bytes
// for one or two tokens, 4-bit for 8 or (two token blocks, each with its own)
// 16
bool decode_fits(int m, int k) {
  if (m < 1 || m > kDecodeMaxTokens) return false;
  const int bytes = m <= 2 ? m * 64 : (m <= 8 ? 8 : 16) * 32;   // per 64-wide block
  const int64_t kgp = (int64_t)(k / kGroup + 1) / 2 * 2;
  return kgp * bytes <= kDecodeXBytes;
}

int dual_gemm_decode_block(const GemmArgs &a) { return decode_block_tokens(a.m) << 16 | 16 * decode_tiles(a); }

// xh: fp16 activations to quantize in the kernel, or NULL: codes from a.xc / a.xs
hipError_t launch_dual_gemm_decode(const GemmArgs &a, const uint16_t *xh, hipStream_t s) {
  if (a.m == 1) return launch_decode_mode<1>(a, xh, s);
  if (a.m == 2) return launch_decode_mode<2>(a, xh, s);
  return launch_decode_mode<4>(a, xh, s);
}

}  // namespace tq

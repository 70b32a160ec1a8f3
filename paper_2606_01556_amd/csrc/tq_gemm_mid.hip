// Fused dual-component W4A4 layer (paper Sec. 4.3) for mid-sized token
// counts (tens to about a thousand tokens): the residual 4-bit GEMM, the
// stage-1 product H = Q(X) Q(L1) kept on chip, its on-the-fly
// re-quantization, stage 2 Q_H Q(L2) and one epilogue, in one kernel.
//
// Work decomposition.  A workgroup of 8 wavefronts owns one block of TB
// 32-token tiles and CT output tiles of 32 columns.  Since every output tile
// needs all of H for its tokens, each workgroup forms the H of its tokens.
//  * H wavefronts (wavefronts 0 .. RT-1, RT = r/32 rounded up) each own one
//    column of TB 32 x 32 tiles of H and walk all K-groups in ascending order,
//    so H and Q_H are bit-identical to the oracle's.
//  * the other wavefronts own one column of TB residual tiles each.  Where
//    there are fewer column tiles than residual wavefronts, NPH wavefronts
//    share a column and take NPH-th parts of every chunk of K; their partial
//    sums are added in a fixed order at the end (only Y's fp32 summation order
//    then differs from the oracle's).
// Per tile and group (Eq. 2): v_mfma_scale_f32_32x32x64_f8f6f4 returns half
// of the exact integer group sum (codes as fp8 subnormals), v_mfma_f32_32x32x8
// f16 twice the exact scale product, and one fma per element applies their
// product, exactly I * s_x * s_w.
//
// Data movement.  A weight or L1 block is the operand of one wavefront alone,
// so it streams from global memory straight into that wavefront's registers,
// a chunk of K ahead (raw buffer loads: one instruction each, zeros past K).
// The activation operands and all scales are shared: K runs in chunks of MCG
// blocks, which the workgroup loads two chunks ahead into registers and writes
// one chunk ahead into a double buffer in LDS (the activation codes as fp8
// operand bytes, expanded there once).  One workgroup barrier per chunk;
// between barriers the wavefronts run freely, so one wavefront's matrix
// products overlap another's vector work.
//
// What bounds it.  With 32 tokens, the H wavefront of a SIMD: its own stream of
// ~36 instructions per K block, 110 ns.  (Bound before by its chunk of four
// blocks: a barrier, an LDS round trip of every operand and ~59 instructions
// per block; 16 blocks per chunk and operands in registers instead took
// 4096 -> 4096, r = 64, M = 128 from 19.8 to 13.7 us, 28672 -> 8192, r = 128,
// M = 32 from 91 to 63 us.)  Where 32-token blocks need more than one round
// over the CUs, a wavefront takes two token tiles: one weight operand loaded
// and expanded for both, and H formed once for twice the columns: four
// tile-groups per SIMD and K block in 310 ns, 4096 -> 12288, r = 64, M = 256
// from 61.7 to 27.3 us.  Sixteen wavefronts of one tile each instead of eight
// of two were slower (32 us: 128 registers leave no room to hold a tile's
// products while the next one's are formed).

#include <type_traits>

#include "tq_device.hpp"
#include "tq_kernels.hpp"

namespace tq {
namespace {

typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int MW = 8;                  // wavefronts per workgroup
constexpr int M_LDS = 160 * 1024;      // LDS of a CU

// TB token tiles, RT rank tiles, CT column tiles; GK 64-wide blocks per
// quantization group
template <int TB, int RT, int CT, int GK>
struct MCfg {
  static constexpr int MCG = TB == 1 ? 16 : 8;          // 64-wide K blocks per chunk
  static constexpr int NRES = MW - RT;                  // residual wavefronts
  static constexpr int CI = MCG / GK;                   // quantization groups of a chunk
  // groups of a chunk per wavefront of a column tile: whole quads (the scale
  // operands hold four groups), and the wavefronts that share the tile
  static constexpr int PMAX = NRES / CT;
  static constexpr int IPC = CI >= 16 && PMAX >= 4 ? CI / 4 : (CI >= 8 && PMAX >= 2 ? CI / 2 : CI);
  static constexpr int NPH = CI / IPC;
  static constexpr int NT = TB + RT + CT;               // rows of scale tiles: x, L1, W
  static constexpr int NP = NT * CI * 4;                // 16-byte scale pieces of a chunk
  static constexpr int SPT = (NP + 64 * MW - 1) / (64 * MW);   // pieces per thread
  static constexpr int APW = MCG / MW;                  // activation blocks per wavefront and chunk
  // chunk buffer: activation operands [TB][MCG] x 2 KiB (two 1 KiB halves),
  // scales [NT][32][CI] fp16 (a row's groups together: one read per chunk)
  static constexpr int S_S = TB * MCG * 2048;
  static constexpr int BUF = (S_S + NP * 16 + 1023) / 1024 * 1024;
  static constexpr int RB = (RT + 1) / 2;               // 64-rank blocks
  // epilogue (aliases the chunk buffers)
  static constexpr int ROWS = 32 * TB;
  static constexpr int HSTR = RT * 32 + 1;
  static constexpr int QSTR = (RB > 0 ? RB : 1) * 64 + 16;
  static constexpr int E_HS = 0;                                  // [ROWS][HSTR] fp32
  static constexpr int E_QS = (E_HS + ROWS * HSTR * 4 + 15) / 16 * 16;   // [ROWS][QSTR] fp8 codes
  static constexpr int E_SH = E_QS + ROWS * QSTR;                 // [RB][ROWS] fp32
  static constexpr int E_RES = (E_SH + (RB > 0 ? RB : 1) * ROWS * 4 + 255) / 256 * 256;
  // partial sums of the wavefronts ph > 0 of each column: [CT][NPH - 1][TB][64][16] fp32
  static constexpr int E_END = E_RES + CT * (NPH - 1) * TB * 4096;
  static constexpr int LDS = E_END > 2 * BUF ? E_END : 2 * BUF;
  static_assert(CT * NPH <= NRES, "a wavefront per column tile and part of K");
  static_assert(IPC % 4 == 0, "whole quads");
  static_assert(LDS <= M_LDS, "fits the 160 KiB LDS of a CU");
};

// Residual rank of wavefront w (w >= RT): wavefronts on SIMDs (w % 4) without
// an H wavefront come first, so they take the larger shares.
__host__ __device__ constexpr int res_index(int rt, int w) {
  int i = 0;
  for (int pass = 0; pass < 2; pass++)
    for (int v = rt; v < MW; v++) {
      const bool no_h = (v % 4) >= rt;
      if ((pass == 0) == no_h) {
        if (v == w) return i;
        i++;
      }
    }
  return -1;
}

// every LDS access of this wavefront so far has completed, then the workgroup
// barrier (global loads into registers stay in flight across it)
__device__ __forceinline__ void m_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// a wave-uniform pointer, kept in scalar registers
__device__ __forceinline__ const uint8_t *m_uniform(const uint8_t *p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const uint8_t *>(((uint64_t)hi << 32) | lo);
}

// Raw buffer of `bytes` bytes at a wave-uniform address: loads past its end
// return zeros (and read nothing), so a block past K needs no test.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t m_buffer(const uint8_t *base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(m_uniform(base)), 0, bytes, 0x00020000);
}
__device__ __forceinline__ u32x4 m_load16(__amdgpu_buffer_rsrc_t rsrc, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0);
}

__device__ __forceinline__ v8i m_join(u32x4 lo, u32x4 hi) {
  return v8i{(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
}

// 2 * s_row * s_col of a 32x32 tile for group J % 4 of four: sa and sb hold the
// four groups' fp16 scales of the lane's row and column (in k = 0..3 and
// k = 4..7); all but the group's are cleared in sb, so the other groups' row
// scales meet zeros
__device__ __forceinline__ v16f m_outer2(u32x2 sa, u32x2 sb, int j) {
  const v16f z = {0};
  const uint32_t w = (j & 2 ? sb.y : sb.x) & (j & 1 ? 0xffff0000u : 0xffffu);
  const u32x2 b2 = j & 2 ? u32x2{0u, w} : u32x2{w, 0u};
  return __builtin_amdgcn_mfma_f32_32x32x8f16(__builtin_bit_cast(v4h, sa),
                                              __builtin_bit_cast(v4h, b2), z, 0, 0, 0);
}

// half of the exact integer group sum of a 32x32 tile of code products
__device__ __forceinline__ v16f m_codes_half(v8i a, v8i b) {
  const v16f z = {0};
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, z, 0, 0, 0, kScale2p9 - 1, 0,
                                                         kScale2p9);
}
// the same added to c (exact: half sums of a 128-wide group stay below 2^13)
__device__ __forceinline__ v16f m_codes_half_acc(v8i a, v8i b, v16f c) {
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, kScale2p9 - 1, 0,
                                                         kScale2p9);
}

template <int TB, int RT, int CT, int GK, bool FP8>
__global__ __launch_bounds__(64 * MW, 2) void dual_gemm_mid_kernel(GemmArgs a, int n_rb) {
  using C = MCfg<TB, RT, CT, GK>;
  constexpr int MCG = C::MCG;
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  const Geometry &geo = a.geo;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int KG = geo.k / kGroup, KQ = KG / GK, NCH = (KG + MCG - 1) / MCG;
  const int ct32 = geo.n_pad / 32;
  const int m = a.m, ms = a.ms;

  // Workgroups are dealt round-robin to the 8 XCDs: give each XCD a
  // contiguous run of logical ids, token blocks fastest, so the workgroups of
  // an XCD share weight columns in its L2.
  int logical;
  {
    const int nwg = gridDim.x, per = nwg / 8, rem = nwg % 8;
    const int x = blockIdx.x % 8, s = blockIdx.x / 8;
    logical = (x < rem ? x * (per + 1) : rem * (per + 1) + (x - rem) * per) + s;
  }
  const int cb = logical / n_rb, tb = logical % n_rb;   // column block, token block

  // ---- roles: wavefront w < RT column w of the H tiles; residual wavefront
  // ri column tile ri % CT, part ri / CT of every chunk ----
  const bool hw = wave < RT;
  const int ri = hw ? 0 : res_index(RT, wave);
  const int jt = ri % CT, ph = hw ? 0 : ri / CT;
  const bool rbusy = !hw && ph < C::NPH;
  const int ct = min(cb * CT + jt, ct32 - 1);   // column tile (past the last: never stored)
  const int stile = hw ? TB + wave : TB + RT + jt;   // this wavefront's column of scales
  const auto bbuf = m_buffer(hw ? a.packed + geo.off_l1 + (int64_t)wave * KG * 1024
                                : a.packed + geo.off_w + (int64_t)ct * KG * 1024, (uint32_t)KG * 1024u);
  const uint32_t lane16 = lane * 16;

  // ---- staging: wavefront w the activation blocks w + 8 q of every chunk (TB
  // tiles), thread t the 16-byte scale pieces t + 512 q: 8 consecutive rows of
  // one group, written to LDS with a row's groups together ----
  constexpr int XB = FP8 ? 2048 : 1024, XR = FP8 ? 2 : 1;
  __amdgpu_buffer_rsrc_t abuf[TB];
#pragma unroll
  for (int t = 0; t < TB; t++)
    abuf[t] = m_buffer(reinterpret_cast<const uint8_t *>(a.xc) +
                       (int64_t)min(tb * TB + t, ms / 32 - 1) * KG * XB, (uint32_t)KG * XB);
  // (threads past the last piece repeat one: same bytes, same place)
  const uint8_t *sbase[C::SPT];
  uint32_t sstride[C::SPT], spiece[C::SPT];
#pragma unroll
  for (int q = 0; q < C::SPT; q++) {
    const int p0 = tid + 64 * MW * q, p = p0 < C::NP ? p0 : p0 % C::NP;
    spiece[q] = p;
    const int tile = p / (4 * C::CI), part = p % 4;
    if (tile < TB) {
      sbase[q] = reinterpret_cast<const uint8_t *>(a.xs) +
                 (int64_t)(32 * min(tb * TB + tile, ms / 32 - 1) + 8 * part) * 2;
      sstride[q] = (uint32_t)ms * 2;
    } else if (tile < TB + RT) {
      sbase[q] = a.packed + geo.off_l1s + (32 * (tile - TB) + 8 * part) * 2;
      sstride[q] = (uint32_t)geo.r_pad32 * 2;
    } else {
      sbase[q] = a.packed + geo.off_ws +
                 (int64_t)(32 * min(cb * CT + tile - TB - RT, ct32 - 1) + 8 * part) * 2;
      sstride[q] = (uint32_t)geo.n_pad * 2;
    }
  }
  u32x4 areg[C::APW][TB][XR], sreg[C::SPT];
  auto stage_load = [&](int c) {   // blocks past K read zeros, scale rows past it the last row
#pragma unroll
    for (int w = 0; w < C::APW; w++) {
      const uint32_t off = (uint32_t)(c * MCG + w * MW + wave) * XB + lane16;
#pragma unroll
      for (int t = 0; t < TB; t++)
#pragma unroll
        for (int x = 0; x < XR; x++) areg[w][t][x] = m_load16(abuf[t], off + x * 1024);
    }
#pragma unroll
    for (int q = 0; q < C::SPT; q++) {
      const uint32_t row = min((uint32_t)(c * C::CI) + spiece[q] / 4 % C::CI, (uint32_t)(KQ - 1));
      sreg[q] = *(const __attribute__((address_space(1))) u32x4 *)(sbase[q] + (uint64_t)row * sstride[q]);
    }
  };
  auto stage_write = [&](int c) {
    uint8_t *B = smem + (c & 1) * C::BUF;
#pragma unroll
    for (int w = 0; w < C::APW; w++) {
#pragma unroll
      for (int t = 0; t < TB; t++) {
        u32x4 lo, hi;
        if constexpr (FP8) {
          lo = areg[w][t][0];
          hi = areg[w][t][1];
        } else {
          const v8i u = unpack32(areg[w][t][0]);
          lo = u32x4{(uint32_t)u[0], (uint32_t)u[1], (uint32_t)u[2], (uint32_t)u[3]};
          hi = u32x4{(uint32_t)u[4], (uint32_t)u[5], (uint32_t)u[6], (uint32_t)u[7]};
        }
        uint8_t *A = B + (t * MCG + w * MW + wave) * 2048 + lane16;
        *reinterpret_cast<u32x4 *>(A) = lo;
        *reinterpret_cast<u32x4 *>(A + 1024) = hi;
      }
    }
#pragma unroll
    for (int q = 0; q < C::SPT; q++) {
      const uint32_t p = spiece[q];
      uint16_t *S = reinterpret_cast<uint16_t *>(B + C::S_S) + (p / (4 * C::CI) * 32 + p % 4 * 8) * C::CI + p / 4 % C::CI;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        S[2 * e * C::CI] = (uint16_t)(sreg[q][e] & 0xffffu);
        S[(2 * e + 1) * C::CI] = (uint16_t)(sreg[q][e] >> 16);
      }
    }
  };

  v16f acc[TB];
#pragma unroll
  for (int t = 0; t < TB; t++) acc[t] = v16f{0};

  // The K loop of one role: IP groups of every chunk (from group ph IP on),
  // with the blocks of PC chunks in flight.
  auto k_loop = [&](auto IPCC, auto PCC) {
    constexpr int IP = decltype(IPCC)::value, PC = decltype(PCC)::value, D = IP * PC;
    u32x4 ring[D][GK];
    uint32_t boff = (uint32_t)(ph * IP * GK) * 1024u + lane16;
    auto load = [&](int s, uint32_t off) {   // slot s: group s % IP of this wavefront's part of a chunk
#pragma unroll
      for (int u = 0; u < GK; u++) ring[s][u] = m_load16(bbuf, off + (s % IP * GK + u) * 1024);
    };
    stage_load(0);
#pragma unroll
    for (int s = 0; s < D; s++) load(s, boff + s / IP * (MCG * 1024));
    boff += PC * MCG * 1024;
    stage_write(0);
    stage_load(1);
    m_barrier();
    // products waiting for their fmas: those of the tile before, so that the
    // matrix core works on one tile while the vector ALU rescales another
    v16f pc = v16f{0}, pp = v16f{0};
    v8i bu[GK];
#pragma unroll
    for (int b = 0; b < GK; b++) bu[b] = unpack32(ring[0][b]);
    for (int c0 = 0; c0 < NCH; c0 += PC) {
#pragma unroll
      for (int u = 0; u < PC; u++) {
        const int c = c0 + u;
        if (PC == 1 || c < NCH) {
        const uint8_t *A = smem + (c & 1) * C::BUF + ph * IP * GK * 2048 + lane16;
        const uint8_t *S = smem + (c & 1) * C::BUF + C::S_S + (l32 * C::CI + ph * IP) * 2;
        v8i av[2][TB][GK];
        auto read_a = [&](int i) {
#pragma unroll
          for (int t = 0; t < TB; t++)
#pragma unroll
            for (int b = 0; b < GK; b++) {
              const uint8_t *p = A + (t * MCG + i * GK + b) * 2048;
              av[i & 1][t][b] = m_join(*reinterpret_cast<const u32x4 *>(p), *reinterpret_cast<const u32x4 *>(p + 1024));
            }
        };
        u32x2 sa[TB][IP / 4], sb[IP / 4];
        read_a(0);
#pragma unroll
        for (int q = 0; q < IP / 4; q++) {
#pragma unroll
          for (int t = 0; t < TB; t++)
            sa[t][q] = *reinterpret_cast<const u32x2 *>(S + (t * 32 * C::CI + 4 * q) * 2);
          sb[q] = *reinterpret_cast<const u32x2 *>(S + (stile * 32 * C::CI + 4 * q) * 2);
        }
#pragma unroll
        for (int i = 0; i < IP; i++) {
          // the rest of the last chunk lies past K (the scale operands hold four
          // groups).  Walked to its end, its zeros cost a K of 128 fourteen
          // blocks' time and one of 1280 twelve: 1280 -> 4096, r = 128,
          // M = 128 10.3 us, 9.5 without
          if (i > 0 && i % 4 == 0 && c * C::CI + ph * IP + i >= KQ) break;
          const int s = u * IP + i;
#pragma unroll
          for (int t = 0; t < TB; t++) {
            // the short scale product first: the code product behind it waits
            // half as long for the matrix core as in the other order
            const v16f cp = m_outer2(sa[t][i / 4], sb[i / 4], i);
            __builtin_amdgcn_sched_barrier(0);
            v16f cc = m_codes_half(av[i & 1][t][0], bu[0]);
            if constexpr (GK == 2) cc = m_codes_half_acc(av[i & 1][t][1], bu[1], cc);
            __builtin_amdgcn_sched_barrier(0);
            if (t == 0) {
              load(s, boff);
              if (i + 1 < IP) read_a(i + 1);
              if (i == 1) stage_write(c + 1);
              if (i == 2) stage_load(c + 2);
            }
            v16f &d = acc[(t + TB - 1) % TB];
#pragma unroll
            for (int v = 0; v < 16; v++) d[v] = fmaf(pc[v], pp[v], d[v]);
            if (t == TB - 1) {
#pragma unroll
              for (int b = 0; b < GK; b++) bu[b] = unpack32(ring[(s + 1) % D][b]);
            }
            __builtin_amdgcn_sched_barrier(0);
            pc = cc;
            pp = cp;
          }
        }
        boff += MCG * 1024;
        m_barrier();
        }
      }
    }
#pragma unroll
    for (int v = 0; v < 16; v++) acc[TB - 1][v] = fmaf(pc[v], pp[v], acc[TB - 1][v]);
  };
  // a wavefront without tiles: staging and barriers only
  auto k_idle = [&]() {
    stage_load(0);
    stage_write(0);
    stage_load(1);
    m_barrier();
    for (int c = 0; c < NCH; c++) {
      stage_write(c + 1);
      stage_load(c + 2);
      m_barrier();
    }
  };

  // stage-2 operands of this wavefront's column tile, loaded ahead of the K loop
  u32x4 l2raw[C::RB > 0 ? C::RB : 1];
  uint32_t l2s[C::RB > 0 ? C::RB : 1];
  if constexpr (RT > 0) {
    const uint16_t *l2scales = reinterpret_cast<const uint16_t *>(a.packed + geo.off_l2s);
#pragma unroll
    for (int rb = 0; rb < C::RB; rb++) {
      const int hg = rb * 64 / geo.gr;   // rank group of 64-rank block rb
      l2raw[rb] = *reinterpret_cast<const u32x4 *>(a.packed + geo.off_l2 + ((int64_t)ct * C::RB + rb) * 1024 + lane16);
      l2s[rb] = l2scales[(int64_t)hg * geo.n_pad + 32 * ct + l32];
    }
  }

  if (C::IPC == C::CI && (hw || rbusy)) {
    k_loop(std::integral_constant<int, C::CI>{}, std::integral_constant<int, 1>{});
  } else if (hw) {
    if constexpr (RT > 0) k_loop(std::integral_constant<int, C::CI>{}, std::integral_constant<int, 1>{});
  } else if (rbusy) {
    k_loop(std::integral_constant<int, C::IPC>{}, std::integral_constant<int, C::IPC == 4 && GK == 1 ? 2 : 1>{});
  } else {
    k_idle();
  }

  // ---- H tiles and residual partials -> LDS (after the last barrier every
  // wavefront is done with the chunk buffers) ----
  float *HS = reinterpret_cast<float *>(smem + C::E_HS);
  uint8_t *QS = smem + C::E_QS;
  float *SHS = reinterpret_cast<float *>(smem + C::E_SH);
  float *RES = reinterpret_cast<float *>(smem + C::E_RES);
  if (hw) {
#pragma unroll
    for (int t = 0; t < TB; t++)
#pragma unroll
      for (int v = 0; v < 16; v++)
        HS[(32 * t + row_of_32x32(lane, v)) * C::HSTR + 32 * wave + l32] = acc[t][v];
  } else if (C::NPH > 1 && rbusy && ph > 0) {
    float *P = RES + (jt * (C::NPH - 1) + ph - 1) * TB * 1024 + lane * 4;
#pragma unroll
    for (int t = 0; t < TB; t++)
#pragma unroll
      for (int v = 0; v < 16; v += 4)
        *reinterpret_cast<v4f *>(P + t * 1024 + v * 64) = v4f{acc[t][v], acc[t][v + 1], acc[t][v + 2], acc[t][v + 3]};
  }
  if constexpr (RT > 0) {
    const int r = geo.r;
    if (r < C::RB * 64)
      for (int idx = tid; idx < C::ROWS * C::RB * 64; idx += 64 * MW) {
        const int row = idx / (C::RB * 64), j = idx % (C::RB * 64);
        if (j >= r) QS[row * C::QSTR + j] = 0;
      }
  }
  m_barrier();

  // ---- re-quantize H per token and rank group (s_H stays fp32) ----
  if constexpr (RT > 0) {
    const int r = geo.r, gr = geo.gr, rg = r / gr;
    const int subs = gr / 8;                // lanes per (token, rank group): 1, 2, 4, 8 or 16
    const int work = C::ROWS * rg * subs;   // <= 512 TB
    const bool dbg = a.dbg_h != nullptr && cb == 0;
#pragma unroll
    for (int base = 0; base < 64 * MW * TB; base += 64 * MW) {
      const int idx = base + tid;
      const bool valid = idx < work;
      const int pair = idx / subs, sub = idx % subs;
      const int row = pair / rg, hg = pair % rg;
      const int j0 = hg * gr + sub * 8;
      const int grow = C::ROWS * tb + row;
      float hv[8];
      float amax = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; e++) {
        hv[e] = valid ? HS[row * C::HSTR + j0 + e] : 0.0f;
        amax = fmaxf(amax, fabsf(hv[e]));
      }
      for (int msk = 1; msk < subs; msk <<= 1) amax = fmaxf(amax, __shfl_xor(amax, msk));
      const float shv = amax / 7.0f;   // IEEE division
      if (valid) {
        uint32_t w0 = 0, w1 = 0;
#pragma unroll
        for (int e = 0; e < 8; e++) {
          int qv = 0;
          if (shv != 0.0f) {
            float tq = __builtin_rintf(hv[e] / shv);
            tq = tq > 7.0f ? 7.0f : (tq < -7.0f ? -7.0f : tq);
            qv = (int)tq;
          }
          const uint32_t bq = code_to_fp8(qv);
          if (e < 4) w0 |= bq << (8 * e); else w1 |= bq << (8 * (e - 4));
          if (dbg && grow < m) {
            a.dbg_h[(int64_t)grow * r + j0 + e] = hv[e];
            a.dbg_qh[(int64_t)grow * r + j0 + e] = (int8_t)qv;
          }
        }
        *reinterpret_cast<uint32_t *>(QS + row * C::QSTR + j0) = w0;
        *reinterpret_cast<uint32_t *>(QS + row * C::QSTR + j0 + 4) = w1;
        if (sub == 0) {
          SHS[hg * C::ROWS + row] = shv;
          if (dbg && grow < m) a.dbg_sh[(int64_t)grow * rg + hg] = shv;
        }
      }
    }
    m_barrier();
  }

  // ---- stage 2 and the single epilogue: the first wavefront of each column ----
  if (!hw && ph == 0 && cb * CT + jt < ct32) {
#pragma unroll
    for (int t = 0; t < TB; t++) {
      v16f ylr = v16f{0};
      if constexpr (RT > 0) {
        // one fma per rank group (the oracle's step): a 128-rank group (r = 128
        // in 128-wide groups) first adds its two 64-rank blocks' exact sums
        constexpr int BPG = RT == 4 && GK == 2 ? 2 : 1;   // 64-rank blocks per rank group
#pragma unroll
        for (int hg = 0; hg < C::RB / BPG; hg++) {
          v16f cbv = v16f{0};
#pragma unroll
          for (int q = 0; q < BPG; q++) {
            const int rb = hg * BPG + q;
            const uint8_t *qrow = QS + (32 * t + l32) * C::QSTR + rb * 64 + (lane >> 5) * 32;
            const v8i qa = m_join(*reinterpret_cast<const u32x4 *>(qrow), *reinterpret_cast<const u32x4 *>(qrow + 16));
            const v8i lb = unpack32(l2raw[rb]);
            cbv = q == 0 ? mfma_codes_32x32x64(qa, lb) : mfma_codes_32x32x64_acc(qa, lb, cbv);
          }
          const float sl2 = half_bits_to_float((uint16_t)l2s[hg * BPG]);
#pragma unroll
          for (int v = 0; v < 16; v++)
            ylr[v] = fmaf(cbv[v], SHS[hg * C::ROWS + 32 * t + row_of_32x32(lane, v)] * sl2, ylr[v]);
        }
      }
      v16f yres = acc[t];
#pragma unroll
      for (int p = 0; p < C::NPH - 1; p++) {
        const float *rp = RES + ((jt * (C::NPH - 1) + p) * TB + t) * 1024 + lane * 4;
#pragma unroll
        for (int v = 0; v < 16; v += 4) {
          const v4f r4 = *reinterpret_cast<const v4f *>(rp + v * 64);
          yres[v] += r4[0]; yres[v + 1] += r4[1]; yres[v + 2] += r4[2]; yres[v + 3] += r4[3];
        }
      }
#pragma unroll
      for (int v = 0; v < 16; v++) yres[v] += ylr[v];
      store_tile_32x32(a.y, a.bf16_out, m, geo.n, C::ROWS * tb + 32 * t, ct * 32, lane, yres);
    }
  }
}

template <int TB, int RT, int CT, int GK, bool FP8>
hipError_t launch_mid(const GemmArgs &a, hipStream_t s) {
  using C = MCfg<TB, RT, CT, GK>;
  const int n_rb = (a.ms / 32 + TB - 1) / TB;
  const int n_cb = (a.geo.n_pad / 32 + CT - 1) / CT;
  auto kern = dual_gemm_mid_kernel<TB, RT, CT, GK, FP8>;
  hipError_t e = allow_lds(reinterpret_cast<const void *>(kern), C::LDS);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(n_rb * n_cb), dim3(64 * MW), C::LDS, s, a, n_rb);
  return hipGetLastError();
}

template <int RT, int GK, bool FP8>
hipError_t launch_mid_tiles(int tb, int ct, const GemmArgs &a, hipStream_t s) {
  if (tb == 2) return launch_mid<2, RT, MW - RT, GK, FP8>(a, s);
  if (ct == 1) return launch_mid<1, RT, 1, GK, FP8>(a, s);
  return ct == 4 ? launch_mid<1, RT, 4, GK, FP8>(a, s) : launch_mid<1, RT, 2, GK, FP8>(a, s);
}

template <int GK, bool FP8>
hipError_t launch_mid_rt(int tb, int ct, const GemmArgs &a, hipStream_t s) {
  switch (a.geo.r_pad32 / 32) {
    case 0: return launch_mid_tiles<0, GK, FP8>(tb, ct, a, s);
    case 1: return launch_mid_tiles<1, GK, FP8>(tb, ct, a, s);
    case 2: return launch_mid_tiles<2, GK, FP8>(tb, ct, a, s);
    case 4: return launch_mid_tiles<4, GK, FP8>(tb, ct, a, s);
    default: return hipErrorInvalidValue;
  }
}


// Tile choices.  A workgroup runs one serial K loop, so a launch takes the
// rounds of workgroups over the 256 CUs times a round's time: a part that does
// not depend on K (filling the pipeline, H's re-quantization, stage 2) and a
// time per 64-wide K block.  Measured on one round at K = 2048 and 8192 (ns
// per block, 64-wide groups, ranks 0 / up to 64 / 128): 32 tokens x 1 or 2
// column tiles 70 / 112 / 130 (the H wavefront's own chain; r = 0: the column
// tiles), x 4 tiles 107 / 156 / 190; 64 tokens x all eight columns of tiles
// 320 at every rank (four tile-groups per SIMD).  128-wide groups take 0.85
// of that (one rescale per two blocks).
struct MidPlan {
  int tb, ct;   // token tiles, column tiles (TB = 2: all columns that hold no H)
  int64_t ns;   // time
};

int64_t mid_rounds(const GemmArgs &a, int tb, int ct) {
  const int64_t n_wg = (int64_t)((a.ms / 32 + tb - 1) / tb) * ((a.geo.n_pad / 32 + ct - 1) / ct);
  return (n_wg + 255) / 256;
}

MidPlan mid_cost(const GemmArgs &a, int tb, int ct) {
  const int rt = a.geo.r_pad32 / 32, c = rt == 0 ? 0 : (rt <= 2 ? 1 : 2);
  constexpr int kBlock[3][3] = {{70, 112, 130}, {107, 156, 190}, {320, 320, 310}};
  int block = kBlock[tb == 2 ? 2 : (ct == 4 ? 1 : 0)][c];
  if (a.geo.gk == 2) block = block * 85 / 100;
  const int64_t round = (tb == 2 ? 6000 : 3500) + (int64_t)block * (a.geo.k / 64);
  return MidPlan{tb, ct, 3000 + mid_rounds(a, tb, ct) * round};
}

// The same for the plans whose wavefronts own their column tiles alone, fitted
// past 512 tokens (fp8 codes) to 2600 calls with K 512 to 16384, N 256 to 16384
// and M 513 to 4096, 95 % of them within 10 %: a launch, a round, a 64-wide
// block of K by group width, token tiles and rank (0, up to 64, 128).
MidPlan mid_exact_cost(const GemmArgs &a, int tb, int ct) {
  const int rt = a.geo.r_pad32 / 32, c = rt == 0 ? 0 : (rt <= 2 ? 1 : 2);
  constexpr int kNs[2][2][3][3] = {
      {{{2260, 2370, 105}, {2200, 4280, 162}, {1900, 5620, 188}},
       {{1840, 4500, 285}, {1520, 6320, 293}, {2380, 7360, 292}}},
      {{{2250, 2840, 92}, {2120, 4490, 132}, {1840, 5450, 149}},
       {{1510, 4000, 245}, {1820, 6410, 250}, {2320, 7060, 251}}}};
  const int *t = kNs[a.geo.gk - 1][tb - 1][c];
  return MidPlan{tb, ct, t[0] + mid_rounds(a, tb, ct) * (t[1] + (int64_t)t[2] * (a.geo.k / 64))};
}

// the plan of least time; exact: only those whose wavefronts own their column
// tiles alone, so that Y is summed in ascending group order
MidPlan mid_plan(const GemmArgs &a, bool exact) {
  const int rt = a.geo.r_pad32 / 32;
  if (a.mid_ct > 0) return MidPlan{1, a.mid_ct, 0};   // forced by the test entry (1, 2 or 4, validated there)
  if (exact) {
    const MidPlan wide = mid_exact_cost(a, 2, MW - rt);
    if (rt == 0) return wide;   // (32 tokens x four column tiles share K there)
    const MidPlan p = mid_exact_cost(a, 1, 4);
    return p.ns < wide.ns ? p : wide;
  }
  MidPlan best = mid_cost(a, 2, MW - rt);
  for (int ct : {1, 2, 4}) {
    const MidPlan p = mid_cost(a, 1, ct);
    if (p.ns < best.ns) best = p;
  }
  return best;
}

}  // namespace

int64_t dual_gemm_mid_ns(const GemmArgs &a) { return mid_plan(a, true).ns; }

int dual_gemm_mid_block(const GemmArgs &a, bool exact) {
  const MidPlan p = mid_plan(a, exact);
  return 32 * p.tb << 16 | 32 * p.ct;
}

hipError_t launch_dual_gemm_mid(const GemmArgs &a, bool exact, hipStream_t s) {
  const MidPlan p = mid_plan(a, exact);
  if (a.geo.gk == 2)
    return act_codes_fp8(a.m) ? launch_mid_rt<2, true>(p.tb, p.ct, a, s) : launch_mid_rt<2, false>(p.tb, p.ct, a, s);
  return act_codes_fp8(a.m) ? launch_mid_rt<1, true>(p.tb, p.ct, a, s) : launch_mid_rt<1, false>(p.tb, p.ct, a, s);
}

}  // namespace tq

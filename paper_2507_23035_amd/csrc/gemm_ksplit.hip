// Look-ahead WAQ LUT-GEMM (Sec. III-C1) for a few dozen to a few hundred
// tokens: the main branch on the matrix cores with the reduction split over
// the waves of a workgroup.
//
// Between the few-token kernel (one tile of 16 or 32 tokens) and the
// many-token one (256 x 128 output tiles) a layer has too few output tiles to
// fill 256 CUs: at 64 x 4096 x 4096 the many-token kernel runs 16 workgroups.
// Here every wave of a workgroup owns the same output tile (32*CW columns x
// 32*FT tokens) and every NW-th block of 64 input channels; the waves are
// independent until the end, where their sums meet in LDS in a fixed order.
// A tile then costs 1 / (4 SIMDs) of its MFMAs per CU however small it is, so
// it can be cut until the grid covers the CUs.
//
// What bounds it: per 16 channels a 128 x 64 tile has 8 MFMAs of 32 clk on a
// SIMD against 24 table reads of 2 clk on the CU's LDS, a 32 x 32 tile one MFMA
// against 8 reads.  By counters the matrix cores are busy 53 % of the time with
// 128 x 128 tiles (2048 x 11008 x 4096), 40 % with 128 x 64 (200 x 8192 x 8192)
// and 22 % with 64 x 64 (777 x 5000 x 3001), the LDS active 29, 36 and 27 %; the
// rest is the fixed part (launch, decode table, reduction: a + f of plan_ks) and
// waiting, a quarter to two fifths of the wave time.
// Measured against the many-token kernel (us): 64 x 4096 x 4096 55.4 -> 7.4,
// 200 x 8192 x 8192 109 -> 33, 512 x 4096 x 4096 57 -> 20, 2048 x 11008 x 4096
// 185 -> 155, and, for d_in not a multiple of 64, 777 x 5000 x 3001 71 -> 40.
#include "common.h"
#include "decode_table.h"

namespace oasis {

// Codes of one block of 8 words (64 channels): lane (r, h) (r = lane mod 32,
// h = lane / 32) takes words 4h .. 4h + 3 of column 32 c + r and token 32 f + r.
template <int CW, int FT>
struct KsCodes {
  uint32_t w[4][CW];
  uint4_t a[FT];
};

// MASK: d_in is not a multiple of 64; the words past it are masked in the last
// block, and the whole offset of a load sits in the per-lane operand, which
// the descriptor's size check covers (otherwise the block's part is in
// soffset).
// PERCOL: a weight codebook per column (A.cb_cols): the weight half of the
// decode table holds column r's own pairs at position r.
// HV: after the codes, the blocks of the value operand A.hv with the codes
// A.hw (the heavy channels of the split compensation), dealt to the waves
// where the code blocks end.
template <int CW, int FT, int NW, bool MASK, bool PERCOL, bool HV>
__global__ void __launch_bounds__(NW * 64, NW / 4) k_gemm_mfma_ks(GemmArgs A, int ncx, int nty) {
  constexpr int PF = 2;  // blocks in flight per wave (four measured slower at 32 x 32)
  // expand a step's operands during the MFMAs of the step before it: faster
  // by 2 to 8 % with several tiles a wave, slower by 2 to 5 % with one, where
  // four waves a SIMD hide the table reads
  constexpr bool PIPE = CW * FT > 1;
  static_assert(!PERCOL || CW == 1, "the weight half of the table holds 32 columns");
  constexpr int NT = NW * 64;
  constexpr int PT = 16 / NW;  // 32 x 32 tiles reduced at a time: 64 KiB of LDS
  static_assert((CW * FT) % PT == 0, "whole pieces");
  static_assert(32 * (CW + FT) <= NT, "one scale a thread");
  // one struct, so that the table starts at LDS address 0 and a lookup's
  // address is its v_perm_b32 alone
  struct Lds {
    uint32_t tab[256 * 64];
    float4_t red[NW * PT * 256];
    float sc[32 * (CW + FT)];  // s_j, then t_i of the tile
  };
  __shared__ Lds lds;
  uint32_t* tab = lds.tab;
  float4_t* red = lds.red;
  float* sc = lds.sc;
  const char* tb = reinterpret_cast<const char*>(tab);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r32 = lane & 31, h = lane >> 5;
  const int T = ncx * nty;
  const uint32_t KB = (uint32_t)(A.d_in >> 3), d_out = (uint32_t)A.d_out;
  const int nblk = (int)(KB + 7u) / 8;
  const uint32_t arow = KB * 4u, wrow = d_out * 4u, wblk = 8u * wrow;

  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(A.idx_w), 0, (int)(KB * d_out * 4u), 0x00020000);
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(A.idx_act), 0, (int)((uint32_t)A.n * arow), 0x00020000);
  // blocks past the last one are requested too (the refills are
  // unconditional): a descriptor of size 0 returns zeros without an access
  const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(A.idx_w), 0, 0, 0x00020000);

  int j0 = 0, t0 = 0;
  uint32_t woff[CW], aoff[FT];
  float scl = 0.0f;  // this thread's scale of the tile
  // columns and tokens past the end read the last one (never stored)
  auto place = [&](int u) {
    const int r = xcd_tile(u, T);
    j0 = r / nty * 32 * CW;
    t0 = r % nty * 32 * FT;
#pragma unroll
    for (int c = 0; c < CW; ++c)
      woff[c] = ((uint32_t)(4 * h) * d_out + (uint32_t)min(j0 + 32 * c + r32, A.d_out - 1)) * 4u;
#pragma unroll
    for (int f = 0; f < FT; ++f)
      aoff[f] = (uint32_t)min(t0 + 32 * f + r32, A.n - 1) * arow + 16u * (uint32_t)h;
  };
  auto load_scale = [&]() {
    const float* src = tid < 32 * CW ? A.w_scale + min(j0 + tid, A.d_out - 1)
                                     : A.act_scale + min(t0 + tid - 32 * CW, A.n - 1);
    scl = *src;
  };
  auto load = [&](int blk, KsCodes<CW, FT>& kc) {
    const bool in = blk < nblk;
    const uint32_t b = in ? (uint32_t)blk : 0u;
    const __amdgpu_buffer_rsrc_t rwx = in ? rw : rz, rax = in ? ra : rz;
#pragma unroll
    for (int f = 0; f < FT; ++f) {
      const uint32_t o = b * 32u;
      kc.a[f] = __builtin_bit_cast(
          uint4_t, MASK ? __builtin_amdgcn_raw_buffer_load_b128(rax, (int)(aoff[f] + o), 0, 0)
                        : __builtin_amdgcn_raw_buffer_load_b128(rax, (int)aoff[f], (int)o, 0));
    }
#pragma unroll
    for (int st = 0; st < 4; ++st)
#pragma unroll
      for (int c = 0; c < CW; ++c) {
        const uint32_t o = b * wblk + (uint32_t)st * wrow;
        kc.w[st][c] = MASK ? __builtin_amdgcn_raw_buffer_load_b32(rwx, (int)(woff[c] + o), 0, 0)
                           : __builtin_amdgcn_raw_buffer_load_b32(rwx, (int)woff[c], (int)o, 0);
      }
  };

  const uint32_t l4w = (uint32_t)r32 * 4u, l4a = l4w + 128u;
  // PERCOL: two sums an output, for the steps in turn.  A wave's chain of d_in /
  // (16 NW) MFMAs is what its rounding error grows with: against 64 bits one
  // chain was off by 1.6e-7 at 4096 channels and 2.3e-7 at 11008, the GEMV
  // launches that this tile replaced (chains of d_in / 512) by 1.4e-7 and
  // 1.8e-7, two chains by 1.3e-7 and 1.75e-7; the time grows by under 2 %
  constexpr int NA = PERCOL ? 2 : 1;
  float16_t acc[NA][CW][FT];
  // operands of step st of block blk
  auto operands = [&](const KsCodes<CW, FT>& kc, int blk, int st, half8_t (&a)[CW],
                      half8_t (&b)[FT]) {
    auto bop = [&](int f) {
      b[f] = expand_dual(kc.a[f][st], tb, l4a);
      if (MASK && (uint32_t)(8 * blk + 4 * h + st) >= KB) b[f] = half8_t{0, 0, 0, 0, 0, 0, 0, 0};
    };
    a[0] = expand_dual(kc.w[st][0], tb, l4w);
    bop(0);
#pragma unroll
    for (int c = 1; c < CW; ++c) a[c] = expand_dual(kc.w[st][c], tb, l4w);
#pragma unroll
    for (int f = 1; f < FT; ++f) bop(f);
  };
  auto mma = [&](const half8_t (&a)[CW], const half8_t (&b)[FT], int st) {
    auto& s = acc[st % NA];
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
      for (int c = 0; c < CW; ++c)
        s[c][f] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[c], b[f], s[c][f], 0, 0, 0);
  };
  constexpr int NM = CW * FT;                   // MFMAs per step
  constexpr int PX = (4 * (CW + FT) + NM - 1) / NM;  // perms (= table reads) per MFMA
  constexpr int NL = FT + 4 * CW;               // loads per block
  auto interleave = [&](bool with_loads) {
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
      __builtin_amdgcn_sched_group_barrier(0x002, PX, 0);  // VALU
      __builtin_amdgcn_sched_group_barrier(0x100, PX, 0);  // DS read
      if (with_loads) __builtin_amdgcn_sched_group_barrier(0x020, (NL + NM - 1) / NM, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  half8_t a0[CW], b0[FT], a1[CW], b1[FT];
  auto mma_block = [&](const KsCodes<CW, FT>& kc, int blk) {
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      operands(kc, blk, st, a0, b0);
      mma(a0, b0, st);
    }
  };
  // one block; a0 / b0 hold its step 0 operands on entry and those of the
  // wave's next block (in nxt) on exit
  auto pipe_block = [&](KsCodes<CW, FT>& cur, const KsCodes<CW, FT>& nxt, int blk) {
    operands(cur, blk, 1, a1, b1);
    mma(a0, b0, 0);
    interleave(false);
    operands(cur, blk, 2, a0, b0);
    mma(a1, b1, 1);
    interleave(false);
    operands(cur, blk, 3, a1, b1);
    mma(a0, b0, 2);
    interleave(false);
    operands(nxt, blk + NW, 0, a0, b0);
    load(blk + 2 * NW, cur);
    mma(a1, b1, 3);
    interleave(true);
  };

  // HV: ceil(2 nh / 64) blocks of 64 positions
  const int nhb = HV ? (2 * __builtin_amdgcn_readfirstlane(*A.nheavy) + 63) / 64 : 0;
  const uint32_t hrow = 2u * kSplitPos;  // bytes per token row of hv
  const __amdgpu_buffer_rsrc_t rhw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(A.hw), 0, HV ? (int)((uint32_t)(kSplitPos / 8) * wrow) : 0,
      0x00020000);
  const __amdgpu_buffer_rsrc_t rhv = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(A.hv), 0, HV ? (int)((uint32_t)A.n * hrow) : 0, 0x00020000);

  KsCodes<CW, FT> buf[PF];
  place(blockIdx.x);
  load_scale();
#pragma unroll
  for (int d = 0; d < PF; ++d) load(wave + d * NW, buf[d]);
  if (wave < 4) {
    DualTableLoader dt;
    dt.load(A.lut, (uint32_t)wave);
    dt.store<PERCOL>(tab, (uint32_t)wave, lane);
  }
  if constexpr (PERCOL) {
    // thread t: column t mod 32 of the tile, byte rows t / 32 + i NT / 32
    constexpr int STEP = NT / 32;
    static_assert(STEP % 16 == 0, "a thread's rows share their low code");
    const int cl = tid & 31, e = tid >> 5;
    const uint16_t* cb = A.cb_cols + (size_t)min(j0 + cl, A.d_out - 1) * 16;
    const uint32_t lo = cb[e & 15];
#pragma unroll
    for (int i = 0; i < 256 / STEP; ++i)
      tab[(e + STEP * i) * 64 + cl] = lo | ((uint32_t)cb[(e + STEP * i) >> 4] << 16);
  }
  __syncthreads();  // decode table

  const bool vec = (d_out & 3u) == 0 && (reinterpret_cast<uintptr_t>(A.y) & 15u) == 0;
  for (int u = blockIdx.x; u < T; u += gridDim.x) {
#pragma unroll
    for (int s = 0; s < NA; ++s)
#pragma unroll
      for (int c = 0; c < CW; ++c)
#pragma unroll
        for (int f = 0; f < FT; ++f)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[s][c][f][v] = 0.0f;
    if constexpr (PIPE) {
      operands(buf[0], wave, 0, a0, b0);
      int blk = wave;
      for (; blk + NW < nblk; blk += 2 * NW) {
        pipe_block(buf[0], buf[1], blk);
        pipe_block(buf[1], buf[0], blk + NW);
      }
      if (blk < nblk) pipe_block(buf[0], buf[1], blk);
    } else {
      for (int blk = wave; blk < nblk; blk += PF * NW) {
#pragma unroll
        for (int d = 0; d < PF; ++d) {
          const int b = blk + d * NW;
          if (b < nblk) {
            mma_block(buf[d], b);
            load(b + PF * NW, buf[d]);
          }
        }
      }
    }
    if constexpr (HV) {
      // a step's registers are refilled with the wave's next heavy block as
      // soon as the step is multiplied: three steps hide the loads
      uint4_t va[4][FT];
      uint32_t vw[4][CW];
      auto hload = [&](int hb, int st) {
        const bool in = hb < nhb;  // past the last: zeros, never multiplied
        const uint32_t b = in ? (uint32_t)hb : 0u;
        const __amdgpu_buffer_rsrc_t rv = in ? rhv : rz, rc = in ? rhw : rz;
#pragma unroll
        for (int f = 0; f < FT; ++f) {
          const uint32_t o = (uint32_t)min(t0 + 32 * f + r32, A.n - 1) * hrow + 64u * (uint32_t)h;
          va[st][f] = __builtin_bit_cast(
              uint4_t, __builtin_amdgcn_raw_buffer_load_b128(
                           rv, (int)o, (int)(b * 128u + 16u * (uint32_t)st), 0));
        }
#pragma unroll
        for (int c = 0; c < CW; ++c)
          vw[st][c] = __builtin_amdgcn_raw_buffer_load_b32(
              rc, (int)woff[c], (int)(b * wblk + (uint32_t)st * wrow), 0);
      };
      int hb = (wave - nblk % NW + NW) % NW;
      if (hb < nhb) {
#pragma unroll
        for (int st = 0; st < 4; ++st) hload(hb, st);
        for (; hb < nhb; hb += NW) {
#pragma unroll
          for (int st = 0; st < 4; ++st) {
            half8_t a[CW], b[FT];
#pragma unroll
            for (int c = 0; c < CW; ++c) a[c] = expand_dual(vw[st][c], tb, l4w);
#pragma unroll
            for (int f = 0; f < FT; ++f) b[f] = __builtin_bit_cast(half8_t, va[st][f]);
            mma(a, b, 0);
            hload(hb + NW, st);
          }
        }
      }
    }
    if constexpr (NA > 1) {
#pragma unroll
      for (int c = 0; c < CW; ++c)
#pragma unroll
        for (int f = 0; f < FT; ++f) acc[0][c][f] += acc[1][c][f];
    }
    const int jt = j0, tt = t0;
    const float scu = scl;
    if (u + (int)gridDim.x < T) {  // the next tile's first blocks, under the reduction
      place(u + (int)gridDim.x);
      load_scale();
#pragma unroll
      for (int d = 0; d < PF; ++d) load(wave + d * NW, buf[d]);
    }

    // ---- sum over the waves and store, PT tiles of 32 columns x 32 tokens at
    // a time.  Lane (r, h), registers 4q .. 4q + 3 of a tile hold columns
    // 4 (2q + h) .. + 3 of token r; column quad x of token r sits at
    // 32 x + (r ^ x), so that both the writes (32 tokens of one quad) and the
    // reads (the 8 quads of a token in consecutive lanes) hit distinct banks.
#pragma unroll
    for (int p0 = 0; p0 < CW * FT; p0 += PT) {
      // the previous piece (of this tile or the last) has been read
      if (p0 > 0 || u != (int)blockIdx.x) __syncthreads();
      if (p0 == 0 && tid < 32 * (CW + FT)) sc[tid] = scu;
#pragma unroll
      for (int t = 0; t < PT; ++t) {
        const int c = (p0 + t) % CW, f = (p0 + t) / CW;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int x = 2 * q + h;
          red[(wave * PT + t) * 256 + 32 * x + (r32 ^ x)] =
              float4_t{acc[0][c][f][4 * q], acc[0][c][f][4 * q + 1], acc[0][c][f][4 * q + 2],
                       acc[0][c][f][4 * q + 3]};
        }
      }
      __syncthreads();
      for (int o = tid; o < PT * 256; o += NT) {
        const int t = o >> 8, x = o & 7, rt = (o >> 3) & 31;
        const int c = (p0 + t) % CW, f = (p0 + t) / CW;
        const int tok = tt + 32 * f + rt, j = jt + 32 * c + 4 * x;
        if (tok >= A.n || j >= A.d_out) continue;
        const float ts = sc[32 * CW + 32 * f + rt];
        const float4_t sw = *reinterpret_cast<const float4_t*>(&sc[32 * c + 4 * x]);
        float4_t v = {0.f, 0.f, 0.f, 0.f};
        if constexpr (PERCOL) {  // in pairs: three roundings instead of seven (the
          // pass of 332 x 1152 x 2560 9.8e-8 -> 9.2e-8, in GEMV launches 9.7e-8)
          float4_t p[NW];
#pragma unroll
          for (int w = 0; w < NW; ++w) p[w] = red[(w * PT + t) * 256 + 32 * x + (rt ^ x)];
#pragma unroll
          for (int d = NW / 2; d > 0; d /= 2)
#pragma unroll
            for (int w = 0; w < d; ++w) p[w] += p[w + d];
          v = p[0];
        } else {
#pragma unroll
          for (int w = 0; w < NW; ++w) v += red[(w * PT + t) * 256 + 32 * x + (rt ^ x)];
        }
        float* dst = A.y + (size_t)tok * d_out + j;
        if (vec) {
          v = ts * sw * v;
          float4_t* d4 = reinterpret_cast<float4_t*>(dst);
          *d4 = A.accumulate ? *d4 + v : v;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (j + e >= A.d_out) continue;
            const float s = ts * sw[e] * v[e];
            dst[e] = A.accumulate ? dst[e] + s : s;
          }
        }
      }
    }
  }
}

template <int CW, int FT, int NW, bool PERCOL, bool HV = false>
static hipError_t launch_ks_one(const GemmArgs& a, hipStream_t s) {
  const int ncx = (a.d_out + 32 * CW - 1) / (32 * CW), nty = (a.n + 32 * FT - 1) / (32 * FT);
  // the per-column table belongs to one tile
  const int grid = PERCOL ? ncx * nty : min(ncx * nty, device_cus());
  if (HV || a.d_in % 64 == 0)
    hipLaunchKernelGGL((k_gemm_mfma_ks<CW, FT, NW, false, PERCOL, HV>), dim3(grid),
                       dim3(NW * 64), 0, s, a, ncx, nty);
  else if constexpr (HV || CW * FT == 16)  // whole blocks only (plan_ks)
    return hipErrorInvalidValue;
  else
    hipLaunchKernelGGL((k_gemm_mfma_ks<CW, FT, NW, true, PERCOL, false>), dim3(grid),
                       dim3(NW * 64), 0, s, a, ncx, nty);
  return hipGetLastError();
}

// The tile by its estimated time: a + b k4 + rounds (f + p k4) us, k4 = d_in /
// 4096, a round being one tile per CU.  Fitted to every tile at 91 sizes (n 64
// to 4000, d_out 2080 to 20000, d_in 256 to 8192) and, for the masked kernels
// (d_in not a multiple of 64: offsets per load), at 116 (n 40 to 4000, d_out 700
// to 20000, d_in 136 to 8200); b < 0 because a first round is shorter than the
// ones that start under another tile's reduction.  With many_token_us the
// choice takes 0.4 % (masked 0.2 %) more than the fastest kernel on average,
// 8 % at most, and at one size more than the many-token kernel where that is
// faster (2.5 % at 1000 x 8200 x 8100).
// Small tiles fill the CUs, large ones expand fewer operands per MFMA; the
// masked 128 x 128 tile was never the fastest and is not built.
KsPlan plan_ks(int n, int d_in, int d_out, bool heavy) {
  struct Tile { int cols, toks; float a, b, f, p; };
  static const Tile whole[4] = {{32, 32, 2.9f, 0.0f, 1.3f, 3.0f},
                                {64, 64, 2.5f, -0.7f, 2.4f, 7.6f},
                                {128, 64, 2.5f, -2.7f, 4.5f, 13.1f},
                                {128, 128, 2.8f, -6.7f, 6.5f, 27.4f}};
  static const Tile masked[3] = {{32, 32, 2.7f, 0.1f, 1.4f, 3.1f},
                                 {64, 64, 2.7f, -1.0f, 2.6f, 8.7f},
                                 {128, 64, 2.9f, -2.5f, 4.5f, 15.2f}};
  const bool mask = d_in % 64 != 0;
  const Tile* tiles = mask ? masked : whole;
  const float k4 = (float)d_in / 4096.0f;
  const long cus = device_cus();
  KsPlan best{0, 0.0f};
  const int v0 = heavy ? 3 : 0;  // heavy blocks: 128 x 128 only
  for (int v = v0; v < (mask ? 3 : 4); ++v) {
    const Tile& q = tiles[v];
    const long t = (long)((d_out + q.cols - 1) / q.cols) * ((n + q.toks - 1) / q.toks);
    const long rounds = (t + cus - 1) / cus;
    const float us = q.a + q.b * k4 + (float)rounds * (q.f + q.p * k4);
    if (v == v0 || us < best.us) best = KsPlan{v, us};
  }
  return best;
}

// 32 columns x 128 tokens: the table holds 32 columns' codebooks, the tokens
// make up for it (512 x 4096 x 4096, one sum an output: 35.5 us against 54 at
// 32 x 64)
hipError_t launch_gemm_ks_percol(const GemmArgs& a, hipStream_t s) {
  return launch_ks_one<1, 4, 8, true>(a, s);
}

hipError_t launch_gemm_ks_heavy(const GemmArgs& a, hipStream_t s) {
  return launch_ks_one<4, 4, 4, false, true>(a, s);
}

hipError_t launch_gemm_ks(const GemmArgs& a, int variant, hipStream_t s) {
  switch (variant) {
    case 0: return launch_ks_one<1, 1, 16, false>(a, s);
    case 1: return launch_ks_one<2, 2, 8, false>(a, s);
    case 2: return launch_ks_one<4, 2, 8, false>(a, s);
    default: return launch_ks_one<4, 4, 4, false>(a, s);
  }
}

}  // namespace oasis

// Error compensation of the outlier branch (Sec. III-C2):
//   Y'[i][j] = s_j * sum_e r_ie * C_W[w(p_ie, j)].
// Each listed outlier channel p fetches input channel p of the weight codes
// (one contiguous row of words in the input-channel-major layout), the codes
// are dequantized with the weight codebook (the Dequant Unit) and multiplied
// by the residual (the MAC units), then merged into the main-branch output.
//
// k_compensate (up to 32 tokens, or long lists over few columns): one workgroup
// per (token, 64 output columns); its 4 waves split the token's 2k listed
// channels and are summed through LDS.  A lane owns a column and issues the
// word loads of 16 listed channels before using any of them.  Channel ids and
// residuals are wave-uniform; zero residuals (channels already compensated
// through the max list) are skipped.  k_compensate_cols (more tokens): a wave
// per token and 64 or 256 columns.  k_compensate_wr: the row layout.
#include "common.h"

namespace oasis {

constexpr int CMP_BATCH = 16;

__global__ void __launch_bounds__(256) k_compensate(CompArgs A) {
  __shared__ float cw[16];
  __shared__ float red[4][64];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  if (tid < 16) cw[tid] = h2f(A.lut->cb_wgt[tid]);
  const int i = blockIdx.x;
  const int j = blockIdx.y * 64 + lane;
  const int k = A.k, E = 2 * k;
  const int d_out = A.d_out, d_in = A.d_in;
  const size_t kr = (size_t)i * k;
  const float* res = A.residual + (size_t)i * E;
  // this wave's share of the listed channels
  const int per = (E + 3) / 4;
  const int e_beg = min(E, wave * per), e_end = min(E, e_beg + per);
  __syncthreads();

  float acc = 0.0f;
  for (int e0 = e_beg; e0 < e_end; e0 += CMP_BATCH) {
    int sh[CMP_BATCH];
    float r[CMP_BATCH];
    uint32_t w[CMP_BATCH];
#pragma unroll
    for (int u = 0; u < CMP_BATCH; ++u) {
      const int e = e0 + u;
      int p = -1;
      r[u] = 0.0f;
      if (e < e_end) {
        p = e < k ? A.max_idx[kr + e] : A.min_idx[kr + (e - k)];
        r[u] = res[e];
      }
      const bool live = p >= 0 && p < d_in && r[u] != 0.0f;  // wave-uniform
      if (!live) r[u] = 0.0f;
      // (no select on `live`: one made every entry a branch of its own, 12.6 ->
      // 13.3 us at 4 x 4096 x 1024, k = 128)
      sh[u] = 4 * (p & 7);
      w[u] = 0u;
      if (live && j < d_out) w[u] = A.idx_w[(size_t)(p >> 3) * d_out + j];
    }
#pragma unroll
    for (int u = 0; u < CMP_BATCH; ++u) acc += r[u] * cw[(w[u] >> sh[u]) & 15u];
  }
  red[wave][lane] = acc;
  __syncthreads();
  if (wave == 0 && j < d_out) {
    const float v = A.w_scale[j] * (red[0][lane] + red[1][lane] + red[2][lane] + red[3][lane]);
    float* dst = A.y + (size_t)i * d_out + j;
    *dst = A.accumulate ? *dst + v : v;
  }
}

// ----------------------------------------------------------------------------
// Many tokens, GEMM layout: a wave takes one token and 64 * CPL columns (CPL
// consecutive ones per lane).  The token's listed entries are wave-uniform:
// lane e holds entry e, readlane hands out its channel and residual, and
// COL_U entries' words (CPL per lane, one contiguous piece of a word row per
// wave) are in flight while COL_U others are consumed: per column a bit field,
// the address of the centroid in a lane's own copy of the codebook (fp32 in
// LDS, bank = lane) and one v_fma_f32.  COL_W waves of a workgroup, and the
// workgroups of a CU, work on other tokens of the same columns, so the
// channels that most tokens list are read from the CU's L1.
// PERCOL: the LDS holds every column's own codebook.
//
// Entries alternate between the two lists from their last, smallest, ones on,
// and each place of a unit has a sum of its own: at 512 x 4096 x 4096 with
// per-column codebooks Y' is off by 6.5e-8 against 64 bits (9.2e-8 with the
// compensation inside the GEMV kernel), at the time of one sum in list order.
//
// Bound by VALU issue (3.5 instructions per entry and column at CPL = 4: half of
// the SIMDs' cycles at 777 x 5000 x 3001, where waves wait to issue 47 % of
// their time; LDS active 22 %) and by the word reads, 4 bytes per entry and
// column.  It replaced a kernel that
// sorted the entries of 4 tokens by word row first: 512 x 4096 x 11008, k = 32
// 87 -> 64 us, 777 x 5000 x 3001, k = 50 171 -> 52, 512 x 4096 x 4096 70 -> 25,
// 2048 x 4096 x 11008 266 -> 219.  (16 tokens' rows as an MFMA operand: 92, 85
// and 34 us, the list work per workgroup taking longer than the products.)
// ----------------------------------------------------------------------------
constexpr int COL_W = 8;  // waves (tokens) per workgroup
constexpr int COL_U = 4;  // entries per unit of word loads, each with a sum of its own

template <int CPL, bool PERCOL>
__global__ void __launch_bounds__(64 * COL_W) k_compensate_cols(CompArgs A, const uint16_t* cb_cols,
                                                                int ntile, int ncol) {
  constexpr int COLS = 64 * CPL;
  // [code][lane], or [code][column c of each lane][lane]
  __shared__ float cw[16 * (PERCOL ? COLS : 64)];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = xcd_tile(blockIdx.x, ntile * ncol);  // token tiles of a column slab on one XCD
  const int tok = b % ntile * COL_W + wave, j0 = b / ntile * COLS;
  const int j = j0 + CPL * lane;
  const int k = A.k, E = 2 * k, d_in = A.d_in, d_out = A.d_out;

  const size_t i = (size_t)min(tok, A.n - 1);
  // entries e0 .. e0 + 63, one per lane; none, or out of range: channel 0, residual 0
  auto lists = [&](int e0, int& p, float& r) {
    const int e = min(e0 + lane, E - 1), h = k - 1 - (e >> 1);
    p = *((e & 1) ? A.min_idx + i * k + h : A.max_idx + i * k + h);
    r = A.residual[i * E + ((e & 1) ? k + h : h)];
    if (e0 + lane >= E || p < 0 || p >= d_in) {
      p = 0;
      r = 0.0f;
    }
  };
  int pl;
  float rl;
  lists(0, pl, rl);
  if constexpr (PERCOL) {
    for (int x = tid; x < 16 * COLS; x += 64 * COL_W) {
      const int c = x % COLS;  // place c: column c / 64 of lane c mod 64
      const int col = min(j0 + CPL * (c & 63) + c / 64, d_out - 1);
      cw[x] = h2f(cb_cols[(size_t)col * 16 + x / COLS]);
    }
  } else {
    for (int x = tid; x < 16 * 64; x += 64 * COL_W) cw[x] = h2f(A.lut->cb_wgt[x >> 6]);
  }
  __syncthreads();
  if (tok >= A.n) return;

  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(A.idx_w), 0, (int)((uint32_t)(d_in / 8) * (uint32_t)d_out * 4u),
      0x00020000);
  // the whole offset sits in the per-lane operand, which the size check
  // covers: columns past d_out read the next row or, past the codes, zeros
  const uint32_t voff = (uint32_t)j * 4u, row_bytes = (uint32_t)d_out * 4u;
  const char* tb = reinterpret_cast<const char*>(cw);
  const uint32_t l4 = (uint32_t)lane * 4u;
  float part[COL_U][CPL];
#pragma unroll
  for (int u = 0; u < COL_U; ++u)
#pragma unroll
    for (int c = 0; c < CPL; ++c) part[u][c] = 0.0f;

  auto issue = [&](int e, uint32_t (&w)[COL_U][CPL]) {
#pragma unroll
    for (int u = 0; u < COL_U; ++u) {
      const uint32_t p = (uint32_t)__builtin_amdgcn_readlane(pl, e + u);
      const int o = (int)((p >> 3) * row_bytes + voff);
      if constexpr (CPL == 4) {
        const uint4_t v = __builtin_bit_cast(uint4_t, __builtin_amdgcn_raw_buffer_load_b128(rw, o, 0, 0));
#pragma unroll
        for (int c = 0; c < CPL; ++c) w[u][c] = v[c];
      } else {
        w[u][0] = __builtin_amdgcn_raw_buffer_load_b32(rw, o, 0, 0);
      }
    }
  };
  auto consume = [&](int e, const uint32_t (&w)[COL_U][CPL]) {
#pragma unroll
    for (int u = 0; u < COL_U; ++u) {
      const uint32_t sh = ((uint32_t)__builtin_amdgcn_readlane(pl, e + u) & 7u) * 4u;
      const float r = __builtin_bit_cast(
          float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, rl), e + u));
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const uint32_t code = __builtin_amdgcn_ubfe(w[u][c], sh, 4u);
        const float cv = *reinterpret_cast<const float*>(
            tb + (PERCOL ? code * (COLS * 4u) + (256u * (uint32_t)c + l4) : ((code << 8) | l4)));
        part[u][c] = fmaf(r, cv, part[u][c]);
      }
    }
  };
  for (int e0 = 0; e0 < E; e0 += 64) {
    if (e0 > 0) lists(e0, pl, rl);
    const int ne = min(64, (E - e0 + COL_U - 1) / COL_U * COL_U);  // dead ones fill the last unit
    uint32_t w0[COL_U][CPL], w1[COL_U][CPL];
    issue(0, w0);
    for (int e = 0; e < ne; e += 2 * COL_U) {
      if (e + COL_U < ne) issue(e + COL_U, w1);
      consume(e, w0);
      if (e + COL_U < ne) {
        if (e + 2 * COL_U < ne) issue(e + 2 * COL_U, w0);
        consume(e + COL_U, w1);
      }
    }
  }

  // ---- merge: y (+)= s_j * acc
  float acc[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) acc[c] = (part[0][c] + part[1][c]) + (part[2][c] + part[3][c]);
  float* dst = A.y + i * d_out + j;
  if (CPL == 4 && (d_out & 3) == 0 && (reinterpret_cast<uintptr_t>(A.y) & 15u) == 0) {
    if (j >= d_out) return;
    float4_t* d4 = reinterpret_cast<float4_t*>(dst);
    float4_t v = A.accumulate ? *d4 : float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < CPL; ++c) v[c] = fmaf(A.w_scale[j + c], acc[c], v[c]);
    *d4 = v;
  } else {
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      if (j + c >= d_out) continue;
      dst[c] = fmaf(A.w_scale[j + c], acc[c], A.accumulate ? dst[c] : 0.0f);
    }
  }
}

// ----------------------------------------------------------------------------
// Compensation from the row layout: idx_wr uint32 [d_in][wn], wn =
// ceil(d_out / 8), word m of row p holds the codes of input channel p for
// output columns 8m .. 8m + 7 (column 8m + c in bits 4c .. 4c + 3).  One
// listed outlier reads exactly its own row, d_out / 2 bytes.
//
// Workgroup = 16 waves over a slab of 64 words (512 columns) and a tile of
// tt tokens; wave w takes tokens w, w + 16, ... of the tile.  Lane l owns
// word 64 * slab + l and 8 fp32 accumulators per token.  A token's listed
// entries are wave-uniform: lane e holds entry e, readlane hands out the
// channels and a broadcast LDS read the residuals, in list order, and each
// entry fetches one word per lane (one contiguous
// 256-byte piece of row p per wave, 3 * WR_U entries in flight).  A word's four
// bytes become four pairs of weight centroids through a 64 KiB LDS table -
// row `byte` holds 32 copies of the pair as two fp32 values, lane l reads
// copy l mod 32, so the 8-byte reads are conflict free and the offset is one
// v_perm_b32 - and each centroid meets the residual in one v_fma_f32 (the
// fp16-operand v_fma_mix_f32 issues at half its rate; fp32 pairs: 712 ->
// 680 us at 4096 x 8192 x 28672).  Sixteen waves share the table (128 KiB of LDS with their
// lists): four waves per SIMD hide the row loads, where 4-wave workgroups
// with their own table fit two (64 copies) or three (32 copies, one more
// shift per lookup) on a CU.
// ----------------------------------------------------------------------------
constexpr int WR_U = 16;    // entries per unit of word loads
constexpr int WR_C = 512;   // list entries per wave held in LDS at a time
constexpr int WR_W = 16;    // waves per workgroup

__global__ void __launch_bounds__(64 * WR_W) k_compensate_wr(CompArgs A, int wn, int nslab,
                                                        int ntile, int tt) {
  // the pair table at a fixed LDS address; dynamic LDS: per wave WR_C
  // channels and WR_C residuals of its lists
  __shared__ uint32_t tab[256 * 64];
  extern __shared__ __align__(16) unsigned char smem_wr[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int* lp = reinterpret_cast<int*>(smem_wr) + wave * WR_C;
  float* lr = reinterpret_cast<float*>(smem_wr + 4 * WR_W * WR_C) + wave * WR_C;
  const int r = xcd_tile(blockIdx.x, nslab * ntile);
  const int slab = r / ntile, tile = r % ntile;  // token tiles of a slab on one XCD
  const int k = A.k, E = 2 * k, d_in = A.d_in, d_out = A.d_out;

  // ---- this wave's tokens, in units of WR_U entries
  const int tok0 = tile * tt;
  const int tw = tok0 + wave;  // first token of this wave; then every WR_W-th
  const int tend = min(A.n, tok0 + tt);
  const int ntw = tw < tend ? (tend - tw + WR_W - 1) / WR_W : 0;
  // units per token: the whole list, or with compacted lists the token's own
  // entries (at least one unit when y is overwritten: a token's last unit
  // writes y; none for a token without entries when adding into y).  Lane
  // j < ntw holds the first unit past token tw + 4j (inclusive prefix sum);
  // units are numbered over the wave's tokens in order.
  const int nch = (E + WR_U - 1) / WR_U;
  int nu = 0;
  if (lane < ntw) {
    nu = nch;
    if (A.cnt) {
      nu = (min(max(A.cnt[tw + WR_W * lane], 0), E) + WR_U - 1) / WR_U;
      if (!A.accumulate) nu = max(1, nu);
    }
  }
  const int uend = (int)wave_incl_scan((uint32_t)nu);
  const int U = __builtin_amdgcn_readlane(uend, 63);
  // token slot j of unit u (the first j whose end exceeds u) and its first unit
  auto unit_token = [&](int u, int& j, int& ubeg) {
    j = 0;
    ubeg = 0;
    for (int q = 0; q + 1 < ntw; ++q) {
      const int endq = __builtin_amdgcn_readlane(uend, q);
      if (u >= endq) {
        j = q + 1;
        ubeg = endq;
      }
    }
  };
  // copy the lists of units [c0, c1) into this wave's LDS area, validated:
  // dead entries (past the lists, duplicates with residual 0, channels out of
  // range) get channel -1 and residual 0.  LDS operations of one wave run in
  // order, so the wave reads its area without a barrier.
  auto fill = [&](int c0, int c1) {
    constexpr int PER = WR_C / 64;
    int pv[PER];
    float rv[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {  // every load first, then the checks
      const int f = lane + 64 * j;
      const int u = c0 + f / WR_U;
      int slot_j, ubeg;
      unit_token(u, slot_j, ubeg);
      const int i = tw + WR_W * slot_j, e = WR_U * (u - ubeg) + f % WR_U;
      pv[j] = -1;
      rv[j] = 0.0f;
      if (f < (c1 - c0) * WR_U && e < E) {
        if (A.cnt) {  // compacted: max_idx rows hold the channels, 2k long
          if (e < A.cnt[i]) {
            pv[j] = A.max_idx[(size_t)i * E + e];
            rv[j] = A.residual[(size_t)i * E + e];
          }
        } else {
          const int32_t* src =
              e < k ? A.max_idx + (size_t)i * k + e : A.min_idx + (size_t)i * k + (e - k);
          pv[j] = *src;
          rv[j] = A.residual[(size_t)i * E + e];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const bool live = pv[j] >= 0 && pv[j] < d_in && rv[j] != 0.0f;
      lp[lane + 64 * j] = live ? pv[j] : -1;
      lr[lane + 64 * j] = live ? rv[j] : 0.0f;
    }
  };
  fill(0, min(U, WR_C / WR_U));  // the first chunk's loads overlap the table build

  // pair table, 64 KiB: row `byte` holds 32 copies of the fp32 pair
  // (C_W[byte & 15], C_W[byte >> 4]).  Thread t writes chunks c = t + 1024 s
  // (s < 4) of 16 bytes: row c / 16 (low code (t / 16) mod 16, high code
  // t / 256 + 4 s), copies 2 (c mod 16) and 2 (c mod 16) + 1
  {
    static_assert(WR_W == 16, "the table build takes 1024 threads");
    const uint16_t* cb = A.lut->cb_wgt;
    const uint32_t lo = __builtin_bit_cast(uint32_t, h2f(cb[(tid >> 4) & 15]));
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const uint32_t hi = __builtin_bit_cast(uint32_t, h2f(cb[(tid >> 8) + 4 * s]));
      const uint32_t c = (uint32_t)tid + 1024u * (uint32_t)s;
      *reinterpret_cast<uint4_t*>(&tab[(c >> 4) * 64u + (c & 15u) * 4u]) = uint4_t{lo, hi, lo, hi};
    }
  }

  const uint32_t m = (uint32_t)slab * 64u + (uint32_t)lane;  // this lane's word
  // lanes past the row end read its last word (never stored), so a load stays
  // inside its row whatever part of the offset the size check covers
  const uint32_t voff = min(m, (uint32_t)wn - 1u) * 4u;
  const uint32_t row_bytes = (uint32_t)wn * 4u;
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(A.idx_w), 0, (int)((uint32_t)d_in * row_bytes), 0x00020000);
  // the offset of byte b's entry, b * 256 + (lane mod 32) * 8, is one
  // v_perm_b32 (a ds_read_b64 serves 16 lanes at a time: 32 copies keep
  // every group of 16 on distinct banks)
  const uint32_t loff = (uint32_t)(lane & 31) * 8u;
  const char* tb = reinterpret_cast<const char*>(tab);
  float sw[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const uint32_t j = 8u * m + (uint32_t)c;
    sw[c] = j < (uint32_t)d_out ? A.w_scale[j] : 0.0f;
  }
  const bool vec = (d_out & 3) == 0 && ((reinterpret_cast<uintptr_t>(A.y) & 15u) == 0) &&
                   8u * m + 8u <= (uint32_t)d_out;
  __syncthreads();  // pair table

  // ---- chunks of WR_C entries; inside a chunk three units of word loads
  // stay in flight: step v reads the lists of unit v + 2 from LDS, requests
  // its words (one per lane per entry), then consumes unit v.  Only word
  // loads are in flight, and they retire in order, so each wait covers just
  // the unit consumed.
  auto issue = [&](int pl, uint32_t (&w)[WR_U]) {
#pragma unroll
    for (int e = 0; e < WR_U; ++e) {
      const int pe = __builtin_amdgcn_readlane(pl, e);
      // a dead entry reads row 0 (in bounds); its residual is 0
      const int soff = pe >= 0 ? (int)((uint32_t)pe * row_bytes) : 0;
      w[e] = __builtin_amdgcn_raw_buffer_load_b32(rw, (int)voff, soff, 0);
    }
  };
  float acc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = 0.0f;
  // adding into y: the token's y words are requested at its first unit and
  // used at its last (a load right before the store would wait for memory)
  float4 yv[2] = {make_float4(0.f, 0.f, 0.f, 0.f), make_float4(0.f, 0.f, 0.f, 0.f)};
  // rl: the unit's residuals, lane e holding entry e (for the skip test);
  // lrv: the same in LDS, read as one broadcast word per entry (a readlane
  // per entry was one VALU instruction of about fourteen: 747 -> 710 us at
  // 4096 x 8192 x 28672)
  auto consume = [&](int u, float rl, const uint32_t (&w)[WR_U], const float* lrv) {
    int slot_j, ubeg;
    unit_token(u, slot_j, ubeg);
    if (A.accumulate && vec && u == ubeg) {
      const float4* s4 = reinterpret_cast<const float4*>(A.y + (size_t)(tw + WR_W * slot_j) * d_out + 8u * m);
      yv[0] = s4[0];
      yv[1] = s4[1];
    }
    // a unit without a live entry (the unused places of OASIS-S lists sit at
    // the end of each list) adds nothing: skip its products
    if (__ballot(rl != 0.0f) != 0) {
#pragma unroll
      for (int e = 0; e < WR_U; ++e) {
        const float re = lrv[e];  // the same LDS word in every lane
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const uint32_t off = __builtin_amdgcn_perm(w[e], loff, 0x0C0C0000u | ((4u + b) << 8));
          const uint2 pr = *reinterpret_cast<const uint2*>(tb + off);
          acc[2 * b] = fmaf(re, __builtin_bit_cast(float, pr.x), acc[2 * b]);
          acc[2 * b + 1] = fmaf(re, __builtin_bit_cast(float, pr.y), acc[2 * b + 1]);
        }
      }
    }
    if (u != __builtin_amdgcn_readlane(uend, slot_j) - 1) return;
    // the token's last unit: y (+)= s_j * acc
    const int i = tw + WR_W * slot_j;
    float* dst = A.y + (size_t)i * d_out + 8u * m;
    if (vec) {
      float4* d4 = reinterpret_cast<float4*>(dst);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float4 o = make_float4(sw[4 * h] * acc[4 * h], sw[4 * h + 1] * acc[4 * h + 1],
                               sw[4 * h + 2] * acc[4 * h + 2], sw[4 * h + 3] * acc[4 * h + 3]);
        if (A.accumulate) {
          o.x += yv[h].x;
          o.y += yv[h].y;
          o.z += yv[h].z;
          o.w += yv[h].w;
        }
        d4[h] = o;
      }
    } else {
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        if (8u * m + (uint32_t)c < (uint32_t)d_out) {
          const float v = sw[c] * acc[c];
          dst[c] = A.accumulate ? dst[c] + v : v;
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] = 0.0f;
  };

  for (int c0 = 0; c0 < U; c0 += WR_C / WR_U) {
    const int c1 = min(U, c0 + WR_C / WR_U), V = c1 - c0;
    if (c0 > 0) fill(c0, c1);
    __builtin_amdgcn_wave_barrier();
    // lane e < WR_U: entry e of chunk unit v
    auto rd = [&](int v, int& pl, float& rl) {
      pl = -1;
      rl = 0.0f;
      if (v < V && lane < WR_U) {
        pl = lp[v * WR_U + lane];
        rl = lr[v * WR_U + lane];
      }
    };
    int p0, p1, p2;
    float r0, r1, r2;
    uint32_t w0[WR_U], w1[WR_U], w2[WR_U];
    rd(0, p0, r0);
    rd(1, p1, r1);
    issue(p0, w0);
    if (V > 1) issue(p1, w1);
    // (ra, wa): unit v; unit v + 2's lists go to (pc, rc), its words to wc
    auto step = [&](int v, float& ra, uint32_t (&wa)[WR_U], int& pc, float& rc,
                    uint32_t (&wc)[WR_U]) {
      const float ru = ra;
      rd(v + 2, pc, rc);
      if (v + 2 < V) issue(pc, wc);
      consume(c0 + v, ru, wa, lr + v * WR_U);
    };
    for (int v = 0; v < V; v += 3) {
      step(v, r0, w0, p2, r2, w2);
      if (v + 1 < V) step(v + 1, r1, w1, p0, r0, w0);
      if (v + 2 < V) step(v + 2, r2, w2, p1, r1, w1);
    }
    __builtin_amdgcn_wave_barrier();  // the next fill overwrites the area
  }
}

// tokens per wave and tile of k_compensate_wr: every wave's lists fit its LDS
// area at once (one copy, no pipeline drain) when 2k <= WR_C / 8 ... WR_C; at
// most 8 per wave
static int wr_tokens(int k) { return max(1, min(8, WR_C / (2 * k))); }

// in list order
hipError_t launch_compensate_wr(const CompArgs& a, hipStream_t s) {
  if (a.n == 0 || a.d_out == 0) return hipSuccess;
  if (a.k == 0) {
    if (a.accumulate) return hipSuccess;
    return launch_fill_zero(a.y, (size_t)a.n * a.d_out, s);
  }
  const int wn = (a.d_out + 7) / 8, tt = WR_W * wr_tokens(a.k);
  const int nslab = (wn + 63) / 64, ntile = (a.n + tt - 1) / tt;
  const size_t lds = 8 * WR_W * WR_C;  // dynamic part: the lists
  hipError_t e = hipFuncSetAttribute((const void*)k_compensate_wr,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_compensate_wr, dim3(nslab * ntile), dim3(64 * WR_W), lds, s, a, wn, nslab,
                     ntile, tt);
  return hipGetLastError();
}

// in an order of the sizes' choosing
hipError_t launch_compensate_lists(const CompArgs& a, hipStream_t s) {
  if (a.n == 0 || a.d_out == 0 || a.k == 0) return launch_compensate_wr(a, s);
  const int per = wr_tokens(a.k), tt = WR_W * per;
  const long wgs = (long)((a.d_out + 511) / 512) * ((a.n + tt - 1) / tt);
  const long rounds = (wgs + device_cus() - 1) / device_cus();
  // (compacted lists have few entries of the 2k)
  if (a.cnt || compensate_mm_fits(a.n, a.d_out, a.k, per, rounds))
    return launch_compensate_mm(a, s);
  return launch_compensate_wr(a, s);
}

template <bool PERCOL>
static hipError_t launch_compensate_cols(const CompArgs& a, const uint16_t* cb_cols,
                                         hipStream_t s) {
  const int ntile = (a.n + COL_W - 1) / COL_W;
  auto go = [&](auto kern, int cols) {
    const int ncol = (a.d_out + cols - 1) / cols;
    hipLaunchKernelGGL(kern, dim3((unsigned)(ntile * ncol)), dim3(64 * COL_W), 0, s, a, cb_cols,
                       ntile, ncol);
    return hipGetLastError();
  };
  // one column a lane while four would give a CU fewer than 8 waves
  if ((long)a.n * ((a.d_out + 255) / 256) < 8l * device_cus()) return go(k_compensate_cols<1, PERCOL>, 64);
  return go(k_compensate_cols<4, PERCOL>, 256);
}

hipError_t launch_compensate_percol(const CompArgs& a, const uint16_t* cb_cols, hipStream_t s) {
  return launch_compensate_cols<true>(a, cb_cols, s);
}

hipError_t launch_compensate(const CompArgs& a, hipStream_t s) {
  if (a.n == 0 || a.d_out == 0) return hipSuccess;
  if (a.k == 0) {
    if (a.accumulate) return hipSuccess;
    return launch_fill_zero(a.y, (size_t)a.n * a.d_out, s);
  }
  // More than 32 tokens: a wave per token and column slab, unless lists of 12
  // and more leave its chain of entries longer than five workgroups a CU of
  // k_compensate, whose waves take a quarter of the list each.  There and here
  // (us): 64 x 64, k = 4 3.6 and 2.7, k = 32 4.7 and 6.5, k = 128 12.7 and 20.4;
  // k = 32, 64 x 1024 (1024 workgroups) 6.0 and 6.6, 33 x 2048 (1056) 6.4 and
  // 6.6, 64 x 1536 (1536) 7.2 and 6.7, 64 x 4096 20.1 and 8.5
  const dim3 grid(a.n, (a.d_out + 63) / 64);
  if (a.n > 32 && (a.k < 12 || (long)grid.x * grid.y > 5l * device_cus()))
    return launch_compensate_cols<false>(a, nullptr, s);
  hipLaunchKernelGGL(k_compensate, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace oasis

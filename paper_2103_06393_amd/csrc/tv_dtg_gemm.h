// The GEMMs of the decompress-then-GEMM products (gfx950): split-bf16 MFMA
// with FP32 accumulation, one kernel for both directions.
//
//   forward  Y^k_(1)[:, slab] = A_k B_k      (A_k = [U1_1 ... U1_m], K = the
//            stacked rows with their Re / Im parts, N = the slab's columns)
//   adjoint  Z_k = Y^k_(1) B_k^*             (A = the packed y, K = the
//            slab's columns with their Re / Im parts, N = the stacked rows)
//
// Operands are split into NS bf16 planes, x = h + m + l with h = rn(x),
// m = rn(x - h), l = rn(x - h - m):
//   NS = 3 (FP32 plans): the 24 bits of an FP32 value exactly, and of the nine
//     partial products the six of weight 2^-16 and above: hh, hm, mh, hl, mm, lh.
//     The dropped ml + lm + ll is below 2^-23 |ab|, 2^-25 rms: under the
//     rounding of one FP32 product and sum.  v_mfma_f32_32x32x16_bf16 rounds
//     to FP32 after every 8 products (measured: K = 16 has the error of two
//     roundings), so six of them per 16 k-steps on the running sum would round
//     it 12 times; a chunk is summed from zero instead and then added, one
//     rounding of the running sum per 16 k-steps (CHUNK_SUM).  The MFMA cuts
//     the bits of smaller addends towards minus infinity, a bias that adds up
//     where the terms' signs are random and U1 is smooth; odd chunks form the
//     negated products and are subtracted, which cancels it (adjoint of 512
//     dipole columns on 128^3, random y: error 3.2e-6 without, 4.9e-7 with).
//     The low plane runs out of exponent below 2^-110: the plan's operand (U1;
//     the adjoint's B) is brought up to 2^-40, each tensor by itself, and what a
//     call brings (y; B with x in it) is split as 2^17 times itself, which the
//     running sum takes back as it adds a chunk.  A wave whose sums are not
//     finite (an infinity or NaN among its operands, or products from about
//     2^110 on) forms them again on v_mfma_f32_32x32x2f32 from the FP32
//     operands (128^3 x 256 adjoint: 1.1 ms, 3.9 with one infinity in y, 8.3
//     where every wave does).
//   NS = 2 (BF16X3 plans): hh, hl, lh.
//
// One LDS stage is a chunk of 16 real k-steps (8 stacked rows, or 8 columns,
// each Re and Im).  A comes split and in operand order (lane 32 h + r%32 of a
// 32-row block: k-steps 8 h .. 8 h + 7), plane after plane.  B is the FP32
// slab; every value is split once, by the thread that carries it from global
// memory to LDS, and lands in operand order ([plane][h][column], 16 bytes:
// every LDS access of the loop is a conflict-free 16-byte one).  Chunk c + 2
// is loaded into registers while chunk c is multiplied and chunk c + 1 goes
// from registers to the other LDS buffer about half way through c's products; one
// barrier per chunk.
//
// Tile: MT = WM MBW blocks of 32 rows (all of 2 n1 rows in ceil(n1/128)
// equal tiles, so short grids pad by less than one block per tile) x 256 or
// 128 columns, WM x WN waves of MBW x NBW blocks.  At most 128 accumulators
// per lane: two waves per SIMD hide each other's LDS reads and barriers.
//
// Bound by the matrix cores and their power: torch's bf16 product reaches
// 1378 TFLOP/s on this card (230 after the six products); counters at 256^3 x
// 2048: matrix cores 68 % (forward) and 65 % busy at 1.73 to 1.75 GHz, waves 23 %
// of their time waiting, 15.8 and 16.9 GB fetched for a slab of 13.1.  Against
// the FP32 MFMA GEMM (v_mfma_f32_32x32x2f32, 1/16 of the bf16 rate) that this
// one replaced: 256^3 x 2048 columns, adjoint GEMM 56.4 -> 34.8 ms (205
// TFLOP/s; 31.2 ms without CHUNK_SUM), relative error against 64 bits 1.2e-6
// -> 4.4e-7 (1.5e-6 without CHUNK_SUM, 7.7e-7 without the negated chunks);
// 205 x 109 x 270 x 287 forward GEMM 7.5 -> 4.4 ms, error 1.8e-6 -> 4.9e-7;
// BF16X3 256^3 x 256 forward 3.0 -> 2.6, adjoint 3.1 -> 2.8 ms.
#pragma once

#include "tv_internal.h"

namespace tv {

constexpr int DTG_MAXQ = 12;
constexpr int DTG_KC = 16;      // stacked rows (columns) per K range unit
constexpr int DTG_LW_F = 8;     // log2 columns per block of B, forward
constexpr int DTG_LW_A = 5;     // and adjoint

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// B: the slab of component k, complex64 in blocks of 2^lw columns: entry
// (row, n) at boff[k] + ((n >> lw) rpad[k] + row) 2^lw + n % 2^lw, with zeros
// where K is padded (forward rows up to rpad, adjoint columns up to 16).  lw = 8
// forward (a workgroup streams whole rows of its columns), lw = 5 adjoint (a
// chunk reads 64 bytes of every row; at 256^3 x 512 the decompression writes
// blocks of 8 columns, 64 bytes, in 2.2 ms, of 16 or 32 in 1.3 ms, and the
// GEMM takes 9.2 and 9.4 ms).
struct SplitGemmParams {
  const uint4* a;           // chunk c, block b, plane p, lane l at
                            // aoff[k] + ((c nbtp + b) NS + p) 64 + l
  const float2* b;
  float2* out;              // forward: y or split partials; adjoint: Z partials
  int64_t out_stride;       // complex per split
  int64_t aoff[DTG_MAXQ];
  int64_t boff[DTG_MAXQ];
  int64_t ooff[DTG_MAXQ];   // complex offset of component k in out
  int32_t rk[DTG_MAXQ];     // stacked rows
  int32_t rpad[DTG_MAXQ];   // and padded to 16
  int32_t ntb[DTG_MAXQ + 1];  // prefix sum over components of the N tiles
  int q, nbtp, mtiles, S;
  int order;                // 0: row tiles fastest, 1: N tiles fastest
  int n1;
  const float2* y;          // adjoint: y of the slab's first column, and per component
  int64_t nv;
  int64_t ncols;            // columns of the slab
  int vec4;
  int64_t nitems;
};

typedef void (*split_gemm_fn)(SplitGemmParams);
// row blocks mt (1..8, or 10, 12, 14, 16 with 128 columns) x 128 or 256 columns
split_gemm_fn split_gemm_pick_f32(bool adj, int mt, int ncol);
split_gemm_fn split_gemm_pick_bf16(bool adj, int mt, int ncol);
inline int split_gemm_threads(int mt, int ncol) { return mt > 8 ? 512 : 2 * ncol; }
inline size_t split_gemm_lds(int ns, int mt, int ncol) {
  return 2 * sizeof(uint4) * (size_t)(mt * ns * 64 + ns * 2 * (ncol + 8));
}

// scale of a call's operand as it is split into three planes
constexpr float SPLIT_UP = 131072.f;

__device__ __forceinline__ v8bf as_v8bf(v4u v) { return __builtin_bit_cast(v8bf, v); }
__device__ __forceinline__ uint32_t bf_pack(float a, float b) {
  const v2bf h = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, h);
}
// (a, b) -> NS words of bf16 pairs, high part first (with two planes, the high
// part of floats above the largest bf16 is that one, not infinity)
template <int NS>
__device__ __forceinline__ void bf_split(float a, float b, uint32_t (&w)[NS]) {
  const float top = __builtin_bit_cast(float, 0x7F7F0000u);
#pragma unroll
  for (int p = 0; p < NS; ++p) {
    w[p] = NS == 2 && p == 0 ? bf_pack(__builtin_amdgcn_fmed3f(a, -top, top),
                                       __builtin_amdgcn_fmed3f(b, -top, top))
                             : bf_pack(a, b);
    a -= __builtin_bit_cast(float, w[p] << 16);
    b -= __builtin_bit_cast(float, w[p] & 0xFFFF0000u);
  }
}

#ifdef TV_SPLIT_GEMM_KERNELS
namespace {

template <int NS, int MBW, int NBW, int WM, int WN, bool ADJ>
__global__ __launch_bounds__(64 * WM * WN, 2) void dtg_split_gemm(SplitGemmParams P) {
  constexpr int T = 64 * WM * WN;
  constexpr int MT = WM * MBW, N = 32 * WN * NBW;
  constexpr int HS = N + 8;                      // 16-byte units between the halves h of B
  constexpr int A_ST = MT * NS * 64, B_ST = NS * 2 * HS, ST = A_ST + B_ST;
  constexpr int NA = (A_ST + T - 1) / T;         // 16-byte loads of A per thread and chunk
  constexpr bool AFULL = A_ST % T == 0;
  constexpr int BT = 2 * N;                      // threads that stage B
  constexpr bool CHUNK_SUM = NS == 3;
  // the row block after which the next chunk goes to LDS.  This and the two
  // scheduling fences of step are measured (3 x 96^2 x 256 columns, both
  // directions): without them 7 blocks take 8% longer, 1 and 5 blocks 2 to 4%,
  // and fences in the others cost up to 7%.
  constexpr int SWAP = MBW == 7 ? 4 : (MBW - 1) / 2;
  static_assert(BT <= T, "one (half, column) of B per thread");
  extern __shared__ v4u lds[];
  // consecutive logical tiles on one XCD (workgroups go round-robin over 8)
  const int64_t nwg = gridDim.x;
  const int64_t L = (int64_t)(blockIdx.x % 8) * (nwg / 8) + blockIdx.x / 8;
  if (L >= P.nitems) return;
  const int ntot = P.ntb[P.q];
  int mt, ntg;
  int64_t rest;
  if (P.order == 0) {
    mt = (int)(L % P.mtiles);
    rest = L / P.mtiles;
    ntg = (int)(rest % ntot);
    rest /= ntot;
  } else {
    ntg = (int)(L % ntot);
    rest = L / ntot;
    mt = (int)(rest % P.mtiles);
    rest /= P.mtiles;
  }
  const int s = (int)rest;
  int k = 0;
  while (ntg >= P.ntb[k + 1]) ++k;
  const int nt = ntg - P.ntb[k];
  const int rk = P.rk[k], rpad = P.rpad[k];
  // chunk ranges of the splits start and end on even chunks
  const int64_t kext = ADJ ? P.ncols : (int64_t)rk;
  const int64_t nst = (kext + DTG_KC - 1) / DTG_KC;
  const int c0 = 2 * (int)(nst * s / P.S), c1 = 2 * (int)(nst * (s + 1) / P.S);

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wm = w / WN, wn = w % WN, h = lane >> 5, ln = lane & 31;

  const v4u* Ag = (const v4u*)P.a + P.aoff[k] + (int64_t)mt * A_ST;
  const int64_t astep = (int64_t)P.nbtp * NS * 64;  // per chunk
  int aidx[NA];
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    aidx[j] = j * T + tid;
    if (!AFULL) aidx[j] = min(aidx[j], A_ST - 1);   // repeats: same value, same place
  }
  // this thread's share of B: forward, column col of half bh (rows 4 bh .. of
  // a chunk); adjoint, stacked row col, columns 4 bh .. of a chunk
  const bool stager = BT == T || tid < BT;
  const int bh = ADJ ? (tid & 1) : tid / N;
  const int bcol = ADJ ? (tid >> 1) & (N - 1) : tid % N;
  const float2* Bg;
  int64_t bstep;
  if (ADJ) {
    // rows past the component's repeat its last one (their sums are not stored)
    const int row = min(nt * N + bcol, rpad - 1);
    Bg = P.b + P.boff[k] + ((int64_t)row << DTG_LW_A) + 4 * bh;
    bstep = (int64_t)rpad << DTG_LW_A;
  } else {
    const int64_t n = (int64_t)nt * N + bcol;
    Bg = P.b + P.boff[k] + (((n >> DTG_LW_F) * rpad + 4 * bh) << DTG_LW_F) +
         (n & ((1 << DTG_LW_F) - 1));
    bstep = 8 << DTG_LW_F;
  }
  const int bdst = A_ST + bh * HS + bcol;

  v4u ra[NA];
  float2 rb[4];
  // global loads of chunk c (past the end: the last one again, instead of a
  // branch)
  auto gload = [&](int c) {
    c = min(c, c1 - 1);
    const v4u* ac = Ag + (int64_t)c * astep;
#pragma unroll
    for (int j = 0; j < NA; ++j) ra[j] = ac[aidx[j]];
    if (stager) {
      const float2* bc =
          ADJ ? Bg + (int64_t)(c >> (DTG_LW_A - 3)) * bstep + 8 * (c & ((1 << (DTG_LW_A - 3)) - 1))
              : Bg + (int64_t)c * bstep;
      if (ADJ) {
        const v4f u = *(const v4f*)bc, v = *(const v4f*)(bc + 2);
        rb[0] = make_float2(u[0], u[1]);
        rb[1] = make_float2(u[2], u[3]);
        rb[2] = make_float2(v[0], v[1]);
        rb[3] = make_float2(v[2], v[3]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) rb[e] = bc[e << DTG_LW_F];
      }
    }
  };
  // the loaded chunk c to LDS buffer buf (k-steps past the stacked rows or
  // columns, up to a chunk's end, are zeros in both operands)
  auto lstore = [&](int buf) {
    v4u* S = lds + buf * ST;
#pragma unroll
    for (int j = 0; j < NA; ++j) S[aidx[j]] = ra[j];
    if (stager) {
      uint32_t wd[4][NS];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float2 v = rb[e];
        // odd chunks negated, see step
        if (CHUNK_SUM && buf) v = make_float2(-v.x, -v.y);
        if (NS == 3 && !ADJ) v = make_float2(v.x * SPLIT_UP, v.y * SPLIT_UP);
        bf_split<NS>(v.x, v.y, wd[e]);
      }
#pragma unroll
      for (int p = 0; p < NS; ++p)
        S[bdst + p * 2 * HS] = v4u{wd[0][p], wd[1][p], wd[2][p], wd[3][p]};
    }
  };

  v16f acc[MBW][NBW];
#pragma unroll
  for (int i = 0; i < MBW; ++i)
#pragma unroll
    for (int j = 0; j < NBW; ++j) acc[i][j] = v16f{0.f};

  // chunk c from LDS buffer (c - c0) % 2; half way through, chunk c + 1 goes
  // to the other buffer and chunk c + 2 is loaded
  auto step = [&](int c, int buf) {
    const v4u* S = lds + buf * ST;
    v8bf b[NBW][NS];
#pragma unroll
    for (int j = 0; j < NBW; ++j)
#pragma unroll
      for (int p = 0; p < NS; ++p)
        b[j][p] = as_v8bf(S[A_ST + (p * 2 + h) * HS + (wn * NBW + j) * 32 + ln]);
#pragma unroll
    for (int i = 0; i < MBW; ++i) {
      v8bf a[NS];
#pragma unroll
      for (int p = 0; p < NS; ++p) a[p] = as_v8bf(S[((wm * MBW + i) * NS + p) * 64 + lane]);
      // partial products of weight 2^-8 (pa + pb), the smallest first
      v16f t[NBW];
#pragma unroll
      for (int j = 0; j < NBW; ++j) t[j] = CHUNK_SUM ? v16f{0.f} : acc[i][j];
#pragma unroll
      for (int d = NS - 1; d >= 0; --d)
#pragma unroll
        for (int pa = 0; pa <= d; ++pa)
#pragma unroll
          for (int j = 0; j < NBW; ++j)
            t[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[pa], b[j][d - pa], t[j], 0, 0, 0);
#pragma unroll
      for (int j = 0; j < NBW; ++j) {
        if (CHUNK_SUM) {
#pragma unroll
          for (int r = 0; r < 16; ++r)
            acc[i][j][r] = fmaf(t[j][r], (buf ? -1.f : 1.f) / SPLIT_UP, acc[i][j][r]);
        } else {
          acc[i][j] = t[j];
        }
      }
      if (i == SWAP) {
        if (MBW == 1) __builtin_amdgcn_sched_barrier(0);
        lstore(buf ^ 1);
        gload(c + 2);
      }
    }
    if (NBW == 1 && (MBW == 1 || MBW > 3)) __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
  };

  if (c0 < c1) {
    gload(c0);
    lstore(0);
    gload(c0 + 1);
  }
  __syncthreads();
  for (int c = c0; c < c1; c += 2) {
    step(c, 0);
    step(c + 1, 1);
  }

  // accumulator register r of lane l is row 8 (r/4) + 4 (l/32) + r%4, column
  // l%32 of its block; rows are (i1, Re/Im) pairs: registers 4g .. 4g + 3 hold
  // (Re, Im) of i1 and i1 + 1
  float2* out = P.out + (int64_t)s * P.out_stride + P.ooff[k];
  const int64_t nlim = ADJ ? (int64_t)rk : P.ncols;
  const auto store = [&](const v16f& d, int i, int j) {
    const int64_t n = (int64_t)nt * N + (wn * NBW + j) * 32 + ln;
    if (n >= nlim) return;
    float2* col = out + (int64_t)P.n1 * n;
    const int blk = mt * MT + wm * MBW + i;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int i1 = blk * 16 + 4 * g + 2 * h;
      const v4f v = {d[4 * g], d[4 * g + 1], d[4 * g + 2], d[4 * g + 3]};
      if (i1 + 1 < P.n1 && P.vec4) {
        *(v4f*)(col + i1) = v;
      } else {
        if (i1 < P.n1) col[i1] = make_float2(v[0], v[1]);
        if (i1 + 1 < P.n1) col[i1 + 1] = make_float2(v[2], v[3]);
      }
    }
  };
  if constexpr (NS == 3) {
    // of columns that are stored: the others hold what the workspace held
    bool odd = false;
#pragma unroll
    for (int j = 0; j < NBW; ++j) {
      float z = 0.f;
#pragma unroll
      for (int i = 0; i < MBW; ++i)
#pragma unroll
        for (int r = 0; r < 16; r += 2)  // v_maximum3_f32: NaN if any is
          z = __builtin_elementwise_maximum(
              __builtin_elementwise_maximum(fabsf(acc[i][j][r]), fabsf(acc[i][j][r + 1])), z);
      odd = odd || (!(z < __builtin_inff()) &&
                    (int64_t)nt * N + (wn * NBW + j) * 32 + ln < nlim);
    }
    if (__any(odd)) {
      // block by block, a k-step (stacked row or column, part h) an operand
#pragma unroll 1
      for (int b = 0; b < MBW * NBW; ++b) {
        const int i = b / NBW, j = b % NBW, blk = mt * MT + wm * MBW + i;
        const int i1 = blk * 16 + (ln >> 1), im = ln & 1;
        const int64_t n = (int64_t)nt * N + (wn * NBW + j) * 32 + ln;
        const uint16_t* ap = (const uint16_t*)((const v4u*)P.a + P.aoff[k] + (int64_t)blk * NS * 64);
        const float* yp = (const float*)(P.y + k * P.nv + i1);
        const float* bp = (const float*)(P.b + P.boff[k]) + h;
        v16f sum = v16f{0.f};
#pragma unroll 1
        for (int c = c0; c < c1; ++c) {
          v16f t = v16f{0.f};
#pragma unroll 1
          for (int e = 0; e < 8; ++e) {
            const int64_t kk = 8 * (int64_t)c + e;
            float av = 0.f, bv = 0.f;
            if (kk < kext) {
              if (ADJ) {
                // rows (i1, Re): Re y, Im y; (i1, Im): Im y, -Re y
                if (i1 < P.n1) av = yp[2 * kk * P.n1 + (im ^ h)];
                if (im & h) av = -av;
                const int64_t row = min(n, (int64_t)rpad - 1);
                bv = bp[2 * ((((kk >> DTG_LW_A) * rpad + row) << DTG_LW_A) +
                             (kk & ((1 << DTG_LW_A) - 1)))];
              } else {
                const uint16_t* a8 = ap + (int64_t)c * astep * 8 +
                                     (32 * (e >> 2) + ln) * 8 + 2 * (e & 3) + h;
#pragma unroll
                for (int p = NS - 1; p >= 0; --p)
                  av += __builtin_bit_cast(float, (uint32_t)a8[p * 64 * 8] << 16);
                bv = bp[2 * ((((n >> DTG_LW_F) * rpad + kk) << DTG_LW_F) +
                             (n & ((1 << DTG_LW_F) - 1)))];
              }
            }
            t = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv, t, 0, 0, 0);
          }
          sum += t;
        }
        store(sum, i, j);
      }
      return;
    }
  }
#pragma unroll
  for (int j = 0; j < NBW; ++j)
#pragma unroll
    for (int i = 0; i < MBW; ++i) store(acc[i][j], i, j);
}

// waves: even row-block counts as 2 x WN of MT/2 x 2 blocks (less LDS traffic
// per MFMA), odd ones and 2 as 1 x 2 WN of MT x 1
template <int NS, bool ADJ, int WN>
split_gemm_fn split_pick_w(int mt) {
  switch (mt) {
    case 1: return dtg_split_gemm<NS, 1, 1, 1, 2 * WN, ADJ>;
    case 2: return dtg_split_gemm<NS, 2, 1, 1, 2 * WN, ADJ>;
    case 3: return dtg_split_gemm<NS, 3, 1, 1, 2 * WN, ADJ>;
    case 4: return dtg_split_gemm<NS, 2, 2, 2, WN, ADJ>;
    case 5: return dtg_split_gemm<NS, 5, 1, 1, 2 * WN, ADJ>;
    case 6: return dtg_split_gemm<NS, 3, 2, 2, WN, ADJ>;
    case 7: return dtg_split_gemm<NS, 7, 1, 1, 2 * WN, ADJ>;
    case 8: return dtg_split_gemm<NS, 4, 2, 2, WN, ADJ>;
  }
  return nullptr;
}
// all rows of a grid of 129 to 256 voxels along i1 in one workgroup
template <int NS, bool ADJ>
split_gemm_fn split_pick_full(int mt) {
  switch (mt) {
    case 10: return dtg_split_gemm<NS, 5, 1, 2, 4, ADJ>;
    case 12: return dtg_split_gemm<NS, 6, 1, 2, 4, ADJ>;
    case 14: return dtg_split_gemm<NS, 7, 1, 2, 4, ADJ>;
    case 16: return dtg_split_gemm<NS, 8, 1, 2, 4, ADJ>;
  }
  return nullptr;
}

}  // namespace
#endif

}  // namespace tv

// Decompress-then-GEMM form of Algorithm 1 (gfx950), for large voxel grids.
//
// Per slab of i3 values, every tensor of every component is decompressed in
// modes 3 and 2 into the stacked operand B_k = [x_1 M_1; ...; x_m M_m]
// (M_j = G_j x2 U2_j x3 U3_j unfolded along mode 1, r1 x (n2 n3)), written
// to HBM, and the mode-1 product of the whole component is then one complex
// GEMM Y^k_(1)[:, slab] = A_k B_k with A_k = [U1_1 ... U1_m] (eq. 6/7,
// Sec. III.B).  Against the fused kernels this spends the HBM traffic of B
// (written once, read once per 256-row tile) to run the dominant product as
// a plain, well-fed MFMA GEMM with long K loops.
//
// The GEMM, its operands and their layouts are in tv_dtg_gemm.h; this file
// holds the decompression that writes B, the packing of A (the plan's U1,
// the adjoint's y), the adjoint's final sum and the host side.
#include <algorithm>

#include "tv_dtg_gemm.h"

namespace tv {

namespace {

struct DecompParams {
  const TensorMeta* meta;
  const float2* cores;
  const float2* u2t;
  const float2* u3t;
  const float2* x;   // x_j scaling (forward) or null
  const float2* scale;  // see dtg_scale_kernel
  const int32_t* drow;  // first stacked row of each tensor [k * m + j]
  float2* B;         // layout as SplitGemmParams::b
  int64_t boff[DTG_MAXQ];
  int32_t rk[DTG_MAXQ], rpad[DTG_MAXQ];
  int lw;
  int64_t m;
  int q, n2, n3, i30, s3, nsub;
  int t3w;           // i3 values per decompression workgroup
  int64_t nitems;
};

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// 1 / v of a power of two between 2^-126 and 2^126
__device__ __forceinline__ float pow2_inv(float v) {
  return __builtin_bit_cast(float, 0x7F000000u - __builtin_bit_cast(uint32_t, v));
}

// The powers of two that bring a tensor's operands of the GEMMs up to 2^-40
// where they are smaller (above that a bf16's range holds the three planes of
// entries down to 2^-70 of the largest), from the largest real or imaginary
// parts of its factors, at plan set-up, a wave a factor: scale[k + q j] = (of
// modes 2 and 3, 1 / of U1).  The adjoint's B is decompressed with the first
// and the final sum takes it back; U1 is packed divided by the second, and the
// forward's B decompressed with it.
__global__ __launch_bounds__(256) void dtg_scale_kernel(const TensorMeta* meta, const float2* cores,
                                                        const float2* u1t, const float2* u2t,
                                                        const float2* u3t, float2* scale, int q,
                                                        int64_t m, int64_t j0, int n1, int n2,
                                                        int n3) {
  __shared__ int ex[4];
  const int64_t j = j0 + blockIdx.x;
  const int k = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const TensorMeta t = meta[(int64_t)k * m + j];
  const float2* v = wave == 0 ? cores + t.g_off
                    : wave == 1 ? u1t + t.u1_off : wave == 2 ? u2t + t.u2_off : u3t + t.u3_off;
  const int n = wave == 0 ? t.r1 * t.r2 * t.r3
                : wave == 1 ? n1 * t.r1 : wave == 2 ? n2 * t.r2 : n3 * t.r3;
  int top = 0;
  for (int i = lane; i < n; i += 64) {
    const float2 u = v[i];
    top = max(top, max(__builtin_bit_cast(int, u.x) & 0x7FFFFFFF,
                       __builtin_bit_cast(int, u.y) & 0x7FFFFFFF));
  }
  for (int off = 32; off > 0; off >>= 1) top = max(top, __shfl_xor(top, off));
  if (lane == 0) ex[wave] = top ? (top >> 23) - 127 : 0;
  __syncthreads();
  if (threadIdx.x) return;
  // 2^-e of an exponent below -40
  const auto up = [](int e) { return min(max(-40 - e, 0), 100); };
  scale[k + q * j] =
      make_float2(__builtin_bit_cast(float, (127 + up(ex[0] + ex[2] + ex[3])) << 23),
                  __builtin_bit_cast(float, (127 - up(ex[1])) << 23));
}

// B rows of one tensor for cnt <= t3w values of i3, two small products:
//   mode 3 (VALU):  H[p][b] = x_j sum_c G[a,b,c] U3[i3,c], p = i3l r1 + a
//   mode 2 (v_mfma_f32_32x32x2f32):  B[p][i2] = sum_b H[p][b] U2[i2,b]
// H sits in LDS as its Re and Im planes (row stride = 4 mod 8 floats: the
// 16-byte reads of four b by 32 rows are free of bank conflicts); K is (b,
// Re/Im) and the complex product's signs are in the U2 operands, which a wave
// holds in registers for its 32 columns i2 (ure: Ur, -Ui; uim: Ui, Ur for the
// two k), so rows of every i3 share them and one H operand feeds both parts.
// The waves share the (column block, row block) tiles, column block first.
// 16 i3 per workgroup fill the row blocks (8 i3 take 15% longer at 256^3) and
// 32 KB of LDS keep four workgroups on a CU.  Write-bound where ranks are
// small: 256^3 x 512 columns, 6.8 GB in 1.32 ms (5.2 TB/s; a fill reaches
// 6.9), 1.75 ms with mode 2 on the VALU; 205 x 109 x 270 x 287, ranks 15 to
// 18, 3.4 GB in 1.31 ms, where that kernel, whose threads were one i2 each,
// took 4.0; 64^3 x 256 58 us, from 110.
constexpr int DEC_T = 256;
// floats per H row: b padded to fours, 4 mod 8
__host__ __device__ inline int dec_rb(int r2) {
  const int p = (r2 + 3) & ~3;
  return (p & 7) ? p : p + 4;
}
__host__ __device__ inline int dec_rows(int r1, int t3w) { return (r1 * t3w + 31) & ~31; }
// LDS: H planes, then {column offset, row offset} of every row p
inline size_t dec_lds(int r1, int r2, int t3w) {
  const size_t rows = dec_rows(r1, t3w);
  return rows * (2 * sizeof(float) * dec_rb(r2) + sizeof(int2));
}

template <int NG>  // groups of four b, 4 NG >= r2 of every tensor
__global__ __launch_bounds__(DEC_T) void dtg_decomp_kernel(DecompParams P) {
  extern __shared__ v4f dsm[];
  const int64_t item = blockIdx.x;
  if (item >= P.nitems) return;
  const int64_t kt = item / P.nsub;           // k * m + j
  const int sub = (int)(item - kt * P.nsub);
  const int k = (int)(kt / P.m);
  const int64_t j = kt - (int64_t)k * P.m;
  const TensorMeta t = P.meta[kt];
  const int r1 = t.r1, r2 = t.r2, r3 = t.r3;
  const int i3a = P.i30 + sub * P.t3w;
  const int cnt = min(P.t3w, P.i30 + P.s3 - i3a);
  const int np = r1 * cnt, nrow = dec_rows(r1, cnt), rb = dec_rb(r2);
  float* Hs = reinterpret_cast<float*>(dsm);          // [part][p][b]
  int2* tab = reinterpret_cast<int2*>(Hs + (size_t)2 * nrow * rb);
  const int row0 = P.drow[kt];
  const float2 sc = P.scale[k + P.q * j];
  const float2 xj = P.x ? P.x[j] : make_float2(sc.x, 0.f);
  const float su = P.x ? sc.y : 1.f;
  const float2* G = P.cores + t.g_off;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r12 = r1 * r2;
  // the waves' first U2 operands are in flight during mode 3
  const int h = lane >> 5, ln = lane & 31;
  const int npb = nrow >> 5, ntask = ((P.n2 + 31) >> 5) * npb;
  const int task0 = ntask * wave / 4, task1 = ntask * (wave + 1) / 4;
  float ure[4 * NG], uim[4 * NG];
  const auto load_u2 = [&](int i2) {
    const float2* u2 = P.u2t + t.u2_off + (int64_t)min(i2, P.n2 - 1) * r2;
#pragma unroll
    for (int b = 0; b < 4 * NG; ++b) {
      const float2 u = b < r2 ? u2[b] : make_float2(0.f, 0.f);
      ure[b] = h ? -u.y : u.x;
      uim[b] = h ? u.x : u.y;
    }
  };
  int cb = task0 / npb, i2 = 32 * cb + ln;
  load_u2(i2);
  // a lane per (a, b) and 8 i3 per wave: the core fibre is read once for them,
  // coalesced over a; U3's rows are uniform (scalar loads, constant for the
  // kernel's lifetime)
  typedef const __attribute__((address_space(4))) float CF;
  CF* U3 = reinterpret_cast<CF*>(reinterpret_cast<uintptr_t>(P.u3t + t.u3_off + (int64_t)i3a * r3));
  const int ni = (cnt + 7) >> 3;
  for (int task = wave; task < ni * ((r12 + 63) >> 6); task += 4) {
    const int i0 = 8 * (task % ni), ab = 64 * (task / ni) + lane;
    if (ab >= r12) continue;
    const int b = ab / r1, a = ab - b * r1;
    const float2* g = G + ab;
    float2 s[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] = make_float2(0.f, 0.f);
#pragma unroll 4
    for (int c = 0; c < r3; ++c) {
      const float2 gv = g[(int64_t)r12 * c];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        CF* u = U3 + 2 * (min(i0 + i, cnt - 1) * r3 + c);
        const float ux = u[0], uy = u[1];
        s[i].x = fmaf(gv.x, ux, fmaf(-gv.y, uy, s[i].x));
        s[i].y = fmaf(gv.x, uy, fmaf(gv.y, ux, s[i].y));
      }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i0 + i >= cnt) break;
      float2 v = cmul(xj, s[i]);
      if (su != 1.f) v = make_float2(v.x * su, v.y * su);
      float* d = Hs + ((i0 + i) * r1 + a) * rb + b;
      d[0] = v.x;
      d[(size_t)nrow * rb] = v.y;
    }
  }
  // zeros up to the next group of four b (0 times whatever LDS held could be NaN)
  const int r2p = (r2 + 3) & ~3;
  for (int e = tid; e < np * (r2p - r2); e += DEC_T) {
    const int p = e % np, b = r2 + e / np;
    Hs[p * rb + b] = 0.f;
    Hs[(size_t)(nrow + p) * rb + b] = 0.f;
  }
  // zeros where the GEMM's K is padded: forward the rows past the last tensor's
  // (the workgroup's columns of every m-th one), adjoint this tensor's columns
  // past the slab's last
  if (P.x) {
    for (int64_t row = P.rk[k] + j; row < P.rpad[k]; row += P.m)
      for (int e = tid; e < cnt * P.n2; e += DEC_T) {
        const int n = (i3a - P.i30) * P.n2 + e;
        P.B[P.boff[k] + (((int64_t)(n >> P.lw) * P.rpad[k] + row) << P.lw) +
            (n & ((1 << P.lw) - 1))] = make_float2(0.f, 0.f);
      }
  } else if (sub == P.nsub - 1) {
    const int64_t n0 = (int64_t)P.s3 * P.n2, pad = (n0 + DTG_KC - 1) / DTG_KC * DTG_KC - n0;
    for (int e = tid; e < pad * r1; e += DEC_T) {
      const int64_t n = n0 + e / r1;
      P.B[P.boff[k] + (((n >> P.lw) * P.rpad[k] + row0 + e % r1) << P.lw) +
          (n & ((1 << P.lw) - 1))] = make_float2(0.f, 0.f);
    }
  }
  for (int p = tid; p < np; p += DEC_T) {
    const int i3l = p / r1;
    tab[p] = make_int2((i3a - P.i30 + i3l) * P.n2, (p - i3l * r1) << P.lw);
  }
  __syncthreads();

  float2* Bk = P.B + P.boff[k] + ((int64_t)row0 << P.lw);
  const uint64_t bblk = (uint64_t)P.rpad[k] << P.lw;  // one block of columns
  const int nmask = (1 << P.lw) - 1;
  for (int task = task0; task < task1; ++task) {
    const int c = task / npb, pb = task - c * npb;
    if (c != cb) {
      cb = c;
      i2 = 32 * cb + ln;
      load_u2(i2);
    }
    const float* hp = Hs + (size_t)(h * nrow + 32 * pb + ln) * rb;
    v16f re = v16f{0.f}, im = v16f{0.f};
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      if (4 * g < r2) {
        const v4f a = *(const v4f*)(hp + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          re = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], ure[4 * g + e], re, 0, 0, 0);
          im = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], uim[4 * g + e], im, 0, 0, 0);
        }
      }
    }
    if (i2 >= P.n2) continue;
    // register r: row p = 32 pb + 8 (r/4) + 4 h + r%4, column i2
    const auto put = [&](int r) {
      const int2 o = tab[32 * pb + 8 * (r >> 2) + 4 * h + (r & 3)];
      const int n = i2 + o.x;
      float2* dst = Bk + ((uint32_t)(n >> P.lw) * bblk + (uint32_t)((n & nmask) + o.y));
      __builtin_nontemporal_store(v2f{re[r], im[r]}, reinterpret_cast<v2f*>(dst));
    };
    if (32 * pb + 32 <= np) {
#pragma unroll
      for (int r = 0; r < 16; ++r) put(r);
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (32 * pb + 8 * (r >> 2) + 4 * h + (r & 3) < np) put(r);
    }
  }
}

// A_k of the forward GEMM from the plan's U1 (row-major [i1][a] per tensor),
// at plan set-up: one workgroup per chunk of 8 stacked rows, a thread per
// 16-byte operand: lane 32 h + r%32 of block blk holds, for the embedded row r
// = 2 i1 + s of A_emb = [[Ur, -Ui], [Ui, Ur]], the k-steps (stacked row
// 8 c + 4 h + e, part t); rows past n1 and past the stacked rows are zeros.
struct APackParams {
  const TensorMeta* meta;
  const float2* scale;
  const int32_t* drow;
  const float2* u1t;
  uint4* a;
  int64_t aoff[DTG_MAXQ];
  int32_t rk[DTG_MAXQ];
  int32_t cpre[DTG_MAXQ + 1];  // prefix sum over components of the chunks
  int64_t m;
  int q, n1, nbtp;
};
template <int NS>
__global__ __launch_bounds__(256) void dtg_apack_kernel(APackParams P) {
  __shared__ const float2* src[8];  // U1 column of each stacked row of the chunk
  __shared__ int ld[8];
  __shared__ float up[8];
  int k = 0;
  while ((int)blockIdx.x >= P.cpre[k + 1]) ++k;
  const int c = (int)blockIdx.x - P.cpre[k];
  if (threadIdx.x < 8) {
    const int row = 8 * c + threadIdx.x;
    src[threadIdx.x] = nullptr;
    ld[threadIdx.x] = 0;
    up[threadIdx.x] = 0.f;
    if (row < P.rk[k]) {
      // the last tensor whose first stacked row is at or before this one
      const int32_t* d = P.drow + (int64_t)k * P.m;
      int64_t lo = 0, hi = P.m;
      while (hi - lo > 1) {
        const int64_t mid = (lo + hi) / 2;
        if (d[mid] <= row) lo = mid;
        else hi = mid;
      }
      const TensorMeta t = P.meta[(int64_t)k * P.m + lo];
      src[threadIdx.x] = P.u1t + t.u1_off + (row - d[lo]);
      ld[threadIdx.x] = t.r1;
      up[threadIdx.x] = pow2_inv(P.scale[k + P.q * lo].y);
    }
  }
  __syncthreads();
  for (int u = threadIdx.x; u < P.nbtp * 64; u += 256) {
    const int blk = u >> 6, lane = u & 63, h = lane >> 5;
    const int r = 32 * blk + (lane & 31), i1 = r >> 1, s = r & 1;
    uint32_t w[4][NS];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float2* col = src[4 * h + e];
      float2 v = make_float2(0.f, 0.f);
      if (col && i1 < P.n1) v = col[(int64_t)i1 * ld[4 * h + e]];
      v = make_float2(v.x * up[4 * h + e], v.y * up[4 * h + e]);
      bf_split<NS>(s ? v.y : v.x, s ? v.x : -v.y, w[e]);
    }
    uint4* dst = P.a + P.aoff[k] + ((int64_t)c * P.nbtp + blk) * NS * 64 + lane;
#pragma unroll
    for (int p = 0; p < NS; ++p) dst[p * 64] = make_uint4(w[0][p], w[1][p], w[2][p], w[3][p]);
  }
}

// ---- adjoint as a GEMM over voxel columns ---------------------------------
// Algorithm 2's inner products with the sum over the columns (i2, i3) taken
// first: Z_k = Y^k_(1) B_k^* (n1 x stacked rows, contraction over the slab's
// columns, one partial per slab and column split), then x'_j = sum_k
// sum_{a of j} sum_i1 conj(U1_j[i1][a]) Z_k[i1][row of a] with the partials
// summed in FP64.  Z is a plain GEMM with the forward kernel's tile and stage
// structure; the final sum is a small pass.
//
// A operand (ypack, per slab): y^k real-embedded, M = (i1, s) rows
// interleaved as in the forward, K = (column n, t = Re/Im):
// [(i1,Re)][(n,Re)] = Re y, [(i1,Re)][(n,Im)] = Im y, [(i1,Im)][(n,Re)] =
// Im y, [(i1,Im)][(n,Im)] = -Re y (so the accumulator holds Re and Im of
// y conj(b)), split into NS bf16 planes in the GEMM's operand order: lane
// 32 h + m%32 of a block holds columns 8c + 4h .. 8c + 4h + 3 of row m.
// Columns past the slab's are zeros up to a multiple of 16.
struct YPackParams {
  const float2* y;
  uint4* yp;
  int64_t ystride;          // 16-byte units per component
  int64_t nv;
  int64_t col0, ncols, nchk;  // slab's first column, width, 8-column chunks packed
  int n1, nbtp, q;
};
template <int NS>
__global__ void dtg_ypack_kernel(YPackParams P) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)P.q * P.nchk * P.nbtp * 64;
  if (idx >= total) return;
  const int lane = (int)(idx & 63);
  int64_t rest = idx >> 6;
  const int blk = (int)(rest % P.nbtp);
  rest /= P.nbtp;
  const int64_t c = rest % P.nchk;
  const int k = (int)(rest / P.nchk);
  const int mrow = 32 * blk + (lane & 31), i1 = mrow >> 1, sr = mrow & 1, h = lane >> 5;
  uint32_t w[4][NS];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int64_t n = 8 * c + 4 * h + j;
    float v0 = 0.f, v1 = 0.f;                      // k = 2j (Re part), 2j + 1 (Im part)
    if (n < P.ncols && i1 < P.n1) {
      const float2 y = P.y[(int64_t)k * P.nv + (P.col0 + n) * P.n1 + i1];
      v0 = sr == 0 ? y.x : y.y;
      v1 = sr == 0 ? y.y : -y.x;
    }
    if (NS == 3) {
      v0 *= SPLIT_UP;
      v1 *= SPLIT_UP;
    }
    bf_split<NS>(v0, v1, w[j]);
  }
  uint4* dst = P.yp + (int64_t)k * P.ystride + (c * P.nbtp + blk) * NS * 64 + lane;
#pragma unroll
  for (int p = 0; p < NS; ++p) dst[p * 64] = make_uint4(w[0][p], w[1][p], w[2][p], w[3][p]);
}

// x'_j = sum_k sum_{a < r1} sum_i1 conj(U1_j[i1][a]) sum_s Z_s[row a][i1]
// over the partials s of every slab and split, in FP64 and a fixed order: one
// workgroup per column j, its 16 waves share the rows (k, a), a lane per i1.
// Where not all slabs' partials are held at once, a launch per group of slabs
// carries the FP64 sum of column j on in acc.
// Bound by the reads of Z (and by their latency where m is below the CUs:
// eight partials' loads are in flight a lane).  128^3, q = 12, 128 columns, 16
// partials (214 MB): 690 -> 57 us against
// one thread per i1 over all rows; 64^3 x 256 39 -> 7 us.
struct ColReduceParams {
  const TensorMeta* meta;
  const float2* scale;
  const int32_t* drow;
  const float2* u1t;
  const float2* z;
  float2* x;
  double2* acc;             // null: all partials are in this launch
  int64_t brow[DTG_MAXQ];
  int64_t zsplit, m;
  int q, S, n1;
  bool first, last;         // group of slabs
};
constexpr int RED_T = 1024;
__global__ __launch_bounds__(RED_T) void dtg_colgemm_reduce_kernel(ColReduceParams P) {
  __shared__ double red[2][RED_T / 64];
  const int64_t j = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double sr = 0.0, si = 0.0;
  int turn = 0;  // rows go round the waves
  for (int k = 0; k < P.q; ++k) {
    const TensorMeta t = P.meta[(int64_t)k * P.m + j];
    const float2* zk = P.z + (P.brow[k] + P.drow[(int64_t)k * P.m + j]) * P.n1;
    const double up = pow2_inv(P.scale[k + P.q * j].x);  // Z is of the scaled tensor
    for (int a = (wave - turn) & (RED_T / 64 - 1); a < t.r1; a += RED_T / 64) {
      for (int i1 = lane; i1 < P.n1; i1 += 64) {
        const float2 u = P.u1t[t.u1_off + (int64_t)i1 * t.r1 + a];
        const float2* z = zk + (int64_t)a * P.n1 + i1;
        double zr = 0.0, zi = 0.0;
        int s = 0;
        for (; s + 8 <= P.S; s += 8) {
          float2 v[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = z[(int64_t)(s + e) * P.zsplit];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            zr += v[e].x;
            zi += v[e].y;
          }
        }
        for (; s < P.S; ++s) {
          const float2 v = z[(int64_t)s * P.zsplit];
          zr += v.x;
          zi += v.y;
        }
        const double ur = u.x * up, ui = u.y * up;
        sr += ur * zr + ui * zi;
        si += ur * zi - ui * zr;
      }
    }
    turn = (turn + t.r1) & (RED_T / 64 - 1);
  }
  for (int off = 32; off > 0; off >>= 1) {
    sr += __shfl_xor(sr, off);
    si += __shfl_xor(si, off);
  }
  if (lane == 0) {
    red[0][wave] = sr;
    red[1][wave] = si;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < RED_T / 64; ++w) {
      sr += red[0][w];
      si += red[1][w];
    }
    if (P.acc) {
      if (!P.first) {
        sr += P.acc[j].x;
        si += P.acc[j].y;
      }
      if (!P.last) {
        P.acc[j] = make_double2(sr, si);
        return;
      }
    }
    P.x[j] = make_float2((float)sr, (float)si);
  }
}

typedef void (*decomp_fn)(DecompParams);

decomp_fn decomp_pick(int r2max) {
  switch ((r2max + 3) / 4) {
    case 1:
    case 2: return dtg_decomp_kernel<2>;
    case 3: return dtg_decomp_kernel<3>;
    case 4: return dtg_decomp_kernel<4>;
    case 5: return dtg_decomp_kernel<5>;
    case 6: return dtg_decomp_kernel<6>;
    case 7:
    case 8: return dtg_decomp_kernel<8>;
  }
  return dtg_decomp_kernel<16>;
}

}  // namespace

// ---- host side -----------------------------------------------------------

// 32-row blocks of a GEMM workgroup tile along the voxel rows: the 2 n1 real
// rows in the fewest equal tiles of at most 8 blocks (128 accumulators a lane)
int dtg_mt(const tv_plan_s* p) {
  const int nbt = (p->grid.n1 + 15) / 16, tiles = (nbt + 7) / 8;
  return (nbt + tiles - 1) / tiles;
}
// all blocks, padded to whole tiles
int dtg_blocks(const tv_plan_s* p) {
  const int mt = dtg_mt(p), nbt = (p->grid.n1 + 15) / 16;
  return (nbt + mt - 1) / mt * mt;
}
// a BF16X3 plan's rows fit one workgroup of two tiles (row_cap 8)
bool dtg_full_row(const tv_plan_s* p) {
  return p->precision == TV_PREC_BF16X3 && dtg_blocks(p) == 2 * dtg_mt(p);
}
// for op 0 / 1 as configured
static int dtg_mt_op(const tv_plan_s* p, int op) {
  return p->dtg_mbw[op] == 8 ? p->dtg_nbtp : dtg_mt(p);
}
// bf16 planes of the split operands
static int dtg_planes(const tv_plan_s* p) { return p->precision == TV_PREC_BF16X3 ? 2 : 3; }

// Layout of A_k for the forward GEMM (called at plan finalisation; the planes
// are written on the device from the uploaded U1 by launch_dtg_pack).
tv_status dtg_layout(tv_plan_s* p, const std::vector<TensorMeta>& meta) {
  const tv_grid& g = p->grid;
  if (g.q > DTG_MAXQ) return TV_OK;
  const int nbtp = dtg_blocks(p), ns = dtg_planes(p);
  p->dtg_nbtp = nbtp;
  p->dtg_rpad.assign(g.q, 0);
  p->dtg_abfoff.assign(g.q + 1, 0);
  p->dtg_rows = 0;
  for (int k = 0; k < g.q; ++k) {
    p->dtg_rpad[k] = (p->sum_r1_k[k] + DTG_KC - 1) / DTG_KC * DTG_KC;
    p->dtg_abfoff[k + 1] = p->dtg_abfoff[k] + p->dtg_rpad[k] / 8 * nbtp * ns * 64;
    p->dtg_rows += p->dtg_rpad[k];
  }
  // stacked row of each tensor's first U1 column in A_k (the fused BF16X3
  // kernels pad tensors to 8-row chunks in their own packing; this one does not)
  std::vector<int32_t> drow((size_t)g.q * g.m);
  for (int k = 0; k < g.q; ++k) {
    int64_t r = 0;
    for (int64_t j = 0; j < g.m; ++j) {
      drow[(size_t)k * g.m + j] = (int32_t)r;
      r += meta[(size_t)k * g.m + j].r1;
    }
  }
  p->hp.drow = std::move(drow);
  p->dtg_packed = true;
  return TV_OK;
}

tv_status launch_dtg_scale(const tv_plan_s* p, int64_t j0, hipStream_t st) {
  const tv_grid& g = p->grid;
  hipLaunchKernelGGL(dtg_scale_kernel, dim3((unsigned)(g.m - j0), g.q), dim3(256), 0, st,
                     p->d_meta, p->d_cores, p->d_u1t, p->d_u2t, p->d_u3t, p->d_scale, g.q, g.m, j0,
                     g.n1, g.n2, g.n3);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? TV_OK : hip_error(e, "operand scale launch");
}

tv_status launch_dtg_pack(const tv_plan_s* p, hipStream_t st) {
  const tv_grid& g = p->grid;
  APackParams P;
  P.meta = p->d_meta;
  P.scale = p->d_scale;
  P.drow = p->d_drow;
  P.u1t = p->d_u1t;
  P.a = p->d_abf;
  P.cpre[0] = 0;
  for (int k = 0; k < g.q; ++k) {
    P.aoff[k] = p->dtg_abfoff[k];
    P.rk[k] = (int32_t)p->sum_r1_k[k];
    P.cpre[k + 1] = P.cpre[k] + (int32_t)(p->dtg_rpad[k] / 8);
  }
  P.m = g.m;
  P.q = g.q;
  P.n1 = g.n1;
  P.nbtp = p->dtg_nbtp;
  hipLaunchKernelGGL(dtg_planes(p) == 2 ? dtg_apack_kernel<2> : dtg_apack_kernel<3>,
                     dim3((unsigned)P.cpre[g.q]), dim3(256), 0, st, P);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? TV_OK : hip_error(e, "U1 operand packing launch");
}

bool dtg_supported(const tv_plan_s* p) { return p->dtg_packed && p->grid.q <= DTG_MAXQ; }

// The path of a new plan's products, as created (tv_autotune and
// tv_plan_configure override it).  A call of this path is three or four
// launches and streams a slab through memory; the fused kernels take one or
// two and win on the smallest plans only.  Measured (us, fused / this path,
// FP32): forward 32^3 x 16 (0.11 GFLOP of mode 1) 22 / 23, 32^3 x 64 (0.45)
// 42 / 35, 81x44x108 x 250 (38) 1673 / 563; adjoint 32^3 x 16 21 / 33, 64^3 x
// 16 (0.86, 136 stacked rows) 53 / 55, 32^3 x 64 42 / 38, 256x64x64 x 8 (1.5)
// 90 / 83, 81x44x108 x 250 1890 / 592.
// tv_rmatvec_noalloc gives tv_rmatvec's result bit for bit, so where it could
// run the fused adjoint in its static scratch and not this path, tv_rmatvec
// stays on the fused adjoint until told otherwise; tv_aca_rmatvec has no such
// twin and goes by the size alone (aca_dtg).
// Forward tile 256 columns, k-step splits towards one workgroup per CU with 8
// chunks each at least (64^3 x 256: 317 -> 165, best of all splits and tiles
// 163).  Adjoint tiles of 256 stacked rows, or 128 where those pad a seventh
// less or the rows fit one (two workgroups then share a CU), column splits
// towards a full chip, 48 columns each at least, 32 at most.
// FP32 plans' adjoint: FP32 chains of 256 columns (512 where all partials of Z
// would pass 2 GiB at that), since the fused adjoint sums little in FP32 before
// its FP64 sum (81x44x108 x 250: error against 64 bits 2.7e-7 there, 2.4e-7
// with chains of 256 columns, which take 2.57 ms, 2.95 with 128); up to 1024
// columns where 64 splits of a slab leave no shorter ones (256^3 x 40, two
// seeds: 2.3 and 2.4e-7 in 1.45 ms; 1.9 and 2.0e-7 in 1.79 with slabs for chains
// of 256; fused 2.3 and 3.0e-7 in 3.6).
// Slabs as high as that and a workspace of 6 GiB in all allow (at 4 GiB 256^3 x
// 512 takes 2% longer, in BF16X3 x 256 6%); a plan whose single i3 needs more
// stays on the fused kernels.
void dtg_default(tv_plan_s* p) {
  if (!dtg_supported(p)) return;
  const tv_grid& g = p->grid;
  constexpr size_t bound = (size_t)6 << 30;
  const double gflop = 8e-9 * (double)p->sum_r1 * g.n1 * g.n2 * g.n3;
  const int64_t rows_k = p->dtg_rows / g.q;
  const auto pow2 = [](int64_t n, int64_t most) {
    int s = 1;
    while (2 * s <= std::min(n, most)) s *= 2;
    return s;
  };
  bool fits[2] = {false, false};
  p->dtg_nbw = 4;
  for (int nslab = 1; nslab <= g.n3 && !fits[0]; ++nslab) {
    p->dtg_s3 = (g.n3 + nslab - 1) / nslab;
    p->dtg_split = pow2(std::min(256 / std::max<int64_t>(1, dtg_launch_tiles(p, p->dtg_s3, 4)),
                                 rows_k / 8 / 8), 16);
    fits[0] = dtg_workspace_bytes(p, 0) <= bound;
  }
  const int64_t t4 = dtg_colgemm_tiles(p, 4), t2 = dtg_colgemm_tiles(p, 2);
  p->dtg_nbw_a = rows_k <= 256 || 16 * t4 > 9 * t2 ? 2 : 4;
  const int64_t tiles = p->dtg_nbw_a == 4 ? t4 : t2, slots = p->dtg_nbw_a == 4 ? 256 : 512;
  const int64_t z = p->dtg_rows * g.n1 * (int64_t)sizeof(float2);
  for (int nslab = 1; nslab <= g.n3 && !fits[1]; ++nslab) {
    p->dtg_s3_a = (g.n3 + nslab - 1) / nslab;
    const int64_t cols = (int64_t)g.n2 * p->dtg_s3_a;
    int64_t split = pow2(std::min(slots / std::max<int64_t>(1, tiles), cols / (3 * DTG_KC)), 32);
    if (dtg_planes(p) == 3) {
      const int64_t chain = z * nslab * ((cols + 255) / 256) <= (int64_t)2 << 30 ? 256 : 512;
      split = std::max(split, (cols + chain - 1) / chain);
      if (cols > 64 * 1024 && p->dtg_s3_a > 1) continue;
    }
    p->dtg_split_a = (int)std::min<int64_t>(split, 64);
    fits[1] = dtg_workspace_bytes(p, 1) <= bound;
  }
  p->dtg_order_a = 0;
  p->fresh[0] = p->fresh[1] = true;
  p->use_dtg[0] = fits[0] && gflop >= 0.3;
  p->aca_dtg = fits[1] && gflop >= (rows_k >= 256 ? 0.4 : 1.2);
  p->use_dtg[1] = p->aca_dtg && (fused_adjoint_ws(p) > TV_STATIC_SCRATCH_BYTES ||
                                 dtg_workspace_bytes(p, 1) <= TV_STATIC_SCRATCH_BYTES);
}

// columns of one slab's B (a multiple of the widest tile)
static int64_t dtg_ldcols(const tv_plan_s* p, int s3) {
  const int64_t cols = (int64_t)p->grid.n2 * s3;
  return (cols + 255) / 256 * 256;
}

// i3 values per decompression workgroup: 16 (small ranks still fill blocks of
// 32 rows), fewer where H would take over 32 KB of LDS
static int dtg_t3w(const tv_plan_s* p) {
  int t = 16;
  while (t > 1 && dec_lds(p->max_r[0], p->max_r[1], t) > 32 * 1024) t /= 2;
  return t;
}

int64_t dtg_launch_tiles(const tv_plan_s* p, int s3, int nbw) {
  const int64_t cols = (int64_t)p->grid.n2 * std::min(s3, p->grid.n3);
  return (int64_t)p->grid.q * (p->dtg_nbtp / dtg_mt(p)) * ((cols + 64 * nbw - 1) / (64 * nbw));
}

int64_t dtg_colgemm_tiles(const tv_plan_s* p, int nbw) {
  int64_t nt = 0;
  for (int k = 0; k < p->grid.q; ++k) nt += (p->sum_r1_k[k] + 64 * nbw - 1) / (64 * nbw);
  return nt * (p->dtg_nbtp / dtg_mt(p));
}

// the column-contraction adjoint: packed y in 16-byte units per component,
// z complex per split
static int64_t col_ystride(const tv_plan_s* p, int s3) {
  const int64_t cols = (int64_t)p->grid.n2 * s3;
  return (cols + DTG_KC - 1) / DTG_KC * 2 * p->dtg_nbtp * dtg_planes(p) * 64;
}
static int64_t col_zsplit(const tv_plan_s* p) { return p->dtg_rows * p->grid.n1; }

// column splits of the adjoint GEMM per slab of s3 values of i3: the
// configured count, raised so that no FP32 accumulation chain spans more than
// 2048 columns (BF16X3) or 4096 (FP32, which rounds its running sum once per 8
// columns, not after every product); the partials meet in FP64
static int chain_splits(const tv_plan_s* p, int s3, int splits) {
  const int64_t nst = ((int64_t)p->grid.n2 * s3 + DTG_KC - 1) / DTG_KC;
  const int64_t chain = (dtg_planes(p) == 2 ? 2048 : 4096) / DTG_KC;
  return (int)std::max<int64_t>(std::max(1, splits), (nst + chain - 1) / chain);
}
int dtg_colgemm_splits(const tv_plan_s* p, int s3) { return chain_splits(p, s3, p->dtg_split_a); }

// slabs of s3 values of i3, and how many of them have their partials of Z held
// at once: all where those take at most 2 GiB, else as many as do
static int64_t adjoint_slabs(const tv_plan_s* p, int s3) { return (p->grid.n3 + s3 - 1) / s3; }
static int64_t adjoint_group(const tv_plan_s* p, int s3, int splits) {
  const int64_t one = chain_splits(p, s3, splits) * col_zsplit(p) * (int64_t)sizeof(float2);
  return std::min(adjoint_slabs(p, s3), std::max<int64_t>(1, ((int64_t)2 << 30) / one));
}

// adjoint workspace at slabs of s3 values of i3 and a column split count
static size_t adjoint_ws(const tv_plan_s* p, int s3, int splits) {
  s3 = std::min(s3, p->grid.n3);
  const int64_t group = adjoint_group(p, s3, splits);
  return (size_t)p->dtg_rows * dtg_ldcols(p, s3) * sizeof(float2) +
         (size_t)p->grid.q * col_ystride(p, s3) * sizeof(uint4) +
         (size_t)group * chain_splits(p, s3, splits) * col_zsplit(p) * sizeof(float2) +
         (group < adjoint_slabs(p, s3) ? p->grid.m * sizeof(double2) : 0);
}

size_t dtg_workspace_bytes(const tv_plan_s* p, int op) {
  if (!dtg_supported(p)) return 0;
  if (op == 1) return adjoint_ws(p, p->dtg_s3_a, p->dtg_split_a);
  const int s3 = std::min(p->dtg_s3, p->grid.n3);
  const int64_t rows = (int64_t)p->grid.q * p->grid.n1 * p->grid.n2 * p->grid.n3;
  const size_t part = p->dtg_split > 1 ? (size_t)8 * p->dtg_split * rows : 0;
  return (size_t)p->dtg_rows * dtg_ldcols(p, s3) * sizeof(float2) + part;
}

// Slab and split count of the adjoint within a fixed scratch: as configured
// when that fits; an FP32 plan whose packed y (three bf16 planes) alone takes
// it past `cap` runs in slabs half as high with half the splits each, again
// and again, as long as FP32 y would have fitted.  False: too large.
bool dtg_adjoint_within(const tv_plan_s* p, size_t cap, int* s3, int* splits) {
  *s3 = std::min(p->dtg_s3_a, p->grid.n3);
  *splits = p->dtg_split_a;
  if (adjoint_ws(p, *s3, *splits) <= cap) return true;
  if (dtg_planes(p) == 2) return false;
  const size_t y48 = (size_t)p->grid.q * col_ystride(p, *s3) * sizeof(uint4);
  if (adjoint_ws(p, *s3, *splits) - y48 / 3 > cap) return false;
  while (*s3 > 1) {
    *s3 = (*s3 + 1) / 2;
    *splits = std::max(1, *splits / 2);
    if (adjoint_ws(p, *s3, *splits) <= cap) return true;
  }
  return false;
}

// The decompression of slabs of s3 values of i3 into B (blocks of 2^lw
// columns), unscaled or by x: its parameters and kernel.
static tv_status decomp_setup(const tv_plan_s* p, const float2* x, float2* B, int s3, int lw,
                              DecompParams* D, decomp_fn* fn, size_t* lds) {
  const tv_grid& g = p->grid;
  D->meta = p->d_meta;
  D->cores = p->d_cores;
  D->u2t = p->d_u2t;
  D->u3t = p->d_u3t;
  D->x = x;
  D->scale = p->d_scale;
  D->drow = p->d_drow;
  D->B = B;
  D->lw = lw;
  const int64_t ldcols = dtg_ldcols(p, s3);
  int64_t acc = 0;
  for (int k = 0; k < g.q; ++k) {
    D->boff[k] = acc;
    D->rk[k] = (int32_t)p->sum_r1_k[k];
    D->rpad[k] = (int32_t)p->dtg_rpad[k];
    acc += p->dtg_rpad[k] * ldcols;
  }
  D->q = g.q;
  D->m = g.m;
  D->n2 = g.n2;
  D->n3 = g.n3;
  D->t3w = dtg_t3w(p);
  *lds = dec_lds(p->max_r[0], p->max_r[1], D->t3w);
  *fn = decomp_pick(p->max_r[1]);
  hipError_t e = hipFuncSetAttribute((const void*)*fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)*lds);
  return e == hipSuccess ? TV_OK : hip_error(e, "hipFuncSetAttribute");
}

static tv_status launch_decomp(DecompParams& D, decomp_fn fn, size_t lds, int q, int i30, int s3a,
                               hipStream_t st) {
  D.i30 = i30;
  D.s3 = s3a;
  D.nsub = (s3a + D.t3w - 1) / D.t3w;
  D.nitems = (int64_t)q * D.m * D.nsub;
  hipLaunchKernelGGL(fn, dim3((unsigned)D.nitems), dim3(256), lds, st, D);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? TV_OK : hip_error(e, "slab decompression launch");
}

// The GEMM of one direction: tile mt blocks x ncol columns, its instance and
// the parameters that do not change from slab to slab.
static tv_status gemm_setup(const tv_plan_s* p, const DecompParams& D, bool adj, int ncol,
                            SplitGemmParams* G, split_gemm_fn* fn, int* threads, size_t* lds) {
  const tv_grid& g = p->grid;
  const bool bf16 = p->precision == TV_PREC_BF16X3;
  const int mt = dtg_mt_op(p, adj ? 1 : 0);
  *fn = bf16 ? split_gemm_pick_bf16(adj, mt, ncol) : split_gemm_pick_f32(adj, mt, ncol);
  if (!*fn) return set_error(TV_ERR_NOT_SUPPORTED, "no GEMM instance for this tile");
  *threads = split_gemm_threads(mt, ncol);
  *lds = split_gemm_lds(dtg_planes(p), mt, ncol);
  G->b = D.B;
  for (int k = 0; k < g.q; ++k) {
    G->boff[k] = D.boff[k];
    G->rk[k] = (int32_t)p->sum_r1_k[k];
    G->rpad[k] = (int32_t)p->dtg_rpad[k];
  }
  G->y = nullptr;
  G->nv = (int64_t)g.n1 * g.n2 * g.n3;
  G->q = g.q;
  G->nbtp = p->dtg_nbtp;
  G->mtiles = p->dtg_nbtp / mt;
  G->n1 = g.n1;
  hipError_t e = hipFuncSetAttribute((const void*)*fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)*lds);
  return e == hipSuccess ? TV_OK : hip_error(e, "hipFuncSetAttribute");
}

static tv_status launch_split_gemm(SplitGemmParams& G, split_gemm_fn fn, int threads, size_t lds,
                                   hipStream_t st) {
  G.nitems = (int64_t)G.mtiles * G.ntb[G.q] * G.S;
  const int64_t grid = (G.nitems + 7) / 8 * 8;
  hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(threads), lds, st, G);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? TV_OK : hip_error(e, "stacked GEMM launch");
}

tv_status launch_dtg_forward(const tv_plan_s* p, const float2* x, float2* y, void* ws,
                             hipStream_t st) {
  if (!dtg_supported(p)) return set_error(TV_ERR_NOT_SUPPORTED, "decompress-then-GEMM not packed");
  const tv_grid& g = p->grid;
  const int s3 = std::min(p->dtg_s3, g.n3);
  const int64_t rows = (int64_t)g.q * g.n1 * g.n2 * g.n3;
  const size_t bbytes = (size_t)p->dtg_rows * dtg_ldcols(p, s3) * sizeof(float2);
  const int S = std::max(1, p->dtg_split), ncol = 64 * p->dtg_nbw;
  float2* out = S > 1 ? (float2*)((char*)ws + bbytes) : y;
  DecompParams D;
  decomp_fn dfn;
  size_t dlds, glds;
  SplitGemmParams G;
  split_gemm_fn gfn;
  int threads;
  tv_status r = decomp_setup(p, x, (float2*)ws, s3, DTG_LW_F, &D, &dfn, &dlds);
  if (r == TV_OK) r = gemm_setup(p, D, false, ncol, &G, &gfn, &threads, &glds);
  if (r != TV_OK) return r;
  G.a = p->d_abf;
  G.out_stride = rows;
  G.S = S;
  G.order = 0;
  const int64_t nv = (int64_t)g.n1 * g.n2 * g.n3;
  for (int k = 0; k < g.q; ++k) G.aoff[k] = p->dtg_abfoff[k];
  G.vec4 = (g.n1 % 2 == 0) && ((uintptr_t)out % 16 == 0);
  for (int i30 = 0; i30 < g.n3; i30 += s3) {
    const int s3a = std::min(s3, g.n3 - i30);
    if ((r = launch_decomp(D, dfn, dlds, g.q, i30, s3a, st)) != TV_OK) return r;
    G.ncols = (int64_t)g.n2 * s3a;
    const int ntiles = (int)((G.ncols + ncol - 1) / ncol);
    for (int k = 0; k <= g.q; ++k) G.ntb[k] = k * ntiles;
    G.out = out;
    for (int k = 0; k < g.q; ++k) G.ooff[k] = k * nv + (int64_t)g.n1 * g.n2 * i30;
    if ((r = launch_split_gemm(G, gfn, threads, glds, st)) != TV_OK) return r;
  }
  if (S > 1) return launch_sum_partials(out, S, rows, y, st);
  return TV_OK;
}

// Adjoint by the column contraction: per slab, the unscaled B_k, y packed as
// the GEMM's A operand, the slab's partials of Y B^*; then the FP64 sum of
// all partials against conj(U1) per column.
tv_status launch_dtg_adjoint(const tv_plan_s* p, const float2* y, float2* x, void* ws, int s3,
                             int splits, hipStream_t st) {
  if (!dtg_supported(p)) return set_error(TV_ERR_NOT_SUPPORTED, "decompress-then-GEMM not packed");
  const tv_grid& g = p->grid;
  s3 = std::min(s3, g.n3);
  const size_t bbytes = (size_t)p->dtg_rows * dtg_ldcols(p, s3) * sizeof(float2);
  const int64_t ystride = col_ystride(p, s3);
  uint4* yp = (uint4*)((char*)ws + bbytes);
  float2* z = (float2*)(yp + (size_t)g.q * ystride);
  const int S = chain_splits(p, s3, splits), ncol = 64 * p->dtg_nbw_a;
  const bool bf16 = p->precision == TV_PREC_BF16X3;
  DecompParams D;
  decomp_fn dfn;
  size_t dlds, glds;
  SplitGemmParams G;
  split_gemm_fn gfn;
  int threads;
  tv_status r = decomp_setup(p, nullptr, (float2*)ws, s3, DTG_LW_A, &D, &dfn, &dlds);
  if (r == TV_OK) r = gemm_setup(p, D, true, ncol, &G, &gfn, &threads, &glds);
  if (r != TV_OK) return r;

  YPackParams Y;
  Y.y = y;
  Y.yp = yp;
  Y.ystride = ystride;
  Y.nv = (int64_t)g.n1 * g.n2 * g.n3;
  Y.n1 = g.n1;
  Y.nbtp = p->dtg_nbtp;
  Y.q = g.q;

  const int64_t zsplit = col_zsplit(p);
  G.a = yp;
  G.out_stride = zsplit;
  G.S = S;
  G.order = p->dtg_order_a;
  G.ntb[0] = 0;
  int64_t brow[DTG_MAXQ], acc = 0;
  for (int k = 0; k < g.q; ++k) {
    G.aoff[k] = k * ystride;
    G.ntb[k + 1] = G.ntb[k] + (int)((p->sum_r1_k[k] + ncol - 1) / ncol);
    brow[k] = acc;
    G.ooff[k] = acc * g.n1;
    acc += p->dtg_rpad[k];
  }
  G.vec4 = (g.n1 % 2 == 0) && ((uintptr_t)z % 16 == 0);
  const int64_t group = adjoint_group(p, s3, splits);
  ColReduceParams R;
  R.meta = p->d_meta;
  R.scale = p->d_scale;
  R.drow = p->d_drow;
  R.u1t = p->d_u1t;
  R.z = z;
  R.x = x;
  R.acc = group < adjoint_slabs(p, s3) ? (double2*)(z + group * S * zsplit) : nullptr;
  for (int k = 0; k < g.q; ++k) R.brow[k] = brow[k];
  R.zsplit = zsplit;
  R.m = g.m;
  R.q = g.q;
  R.n1 = g.n1;
  R.first = true;
  int slab = 0;  // of the group
  for (int i30 = 0; i30 < g.n3; i30 += s3) {
    const int s3a = std::min(s3, g.n3 - i30);
    if ((r = launch_decomp(D, dfn, dlds, g.q, i30, s3a, st)) != TV_OK) return r;
    Y.col0 = (int64_t)g.n2 * i30;
    Y.ncols = G.ncols = (int64_t)g.n2 * s3a;
    G.y = y + Y.col0 * g.n1;
    Y.nchk = (Y.ncols + DTG_KC - 1) / DTG_KC * 2;
    const int64_t yth = (int64_t)g.q * Y.nchk * Y.nbtp * 64;
    hipLaunchKernelGGL(bf16 ? dtg_ypack_kernel<2> : dtg_ypack_kernel<3>,
                       dim3((unsigned)((yth + 255) / 256)), dim3(256), 0, st, Y);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "adjoint operand packing launch");
    G.out = z + (int64_t)slab++ * S * zsplit;
    if ((r = launch_split_gemm(G, gfn, threads, glds, st)) != TV_OK) return r;
    R.last = i30 + s3 >= g.n3;
    if (slab < group && !R.last) continue;
    R.S = slab * S;
    hipLaunchKernelGGL(dtg_colgemm_reduce_kernel, dim3((unsigned)g.m), dim3(RED_T), 0, st, R);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "adjoint reduction launch");
    R.first = false;
    slab = 0;
  }
  return TV_OK;
}

}  // namespace tv

// float32 GEMM of the float32 MLP on the float32 matrix instructions
// (v_mfma_f32_16x16x4_f32 and 32x32x2_f32: full float32 products and sums).
//
// The MLP's products are a few MFLOP (32 x 256 x 512), so what bounds them is
// the chain of dependent memory round trips along K, not arithmetic: 64 x 64
// tiles put 32 x 256 x 512 on 4 workgroups that walked K in 32 barrier steps
// (48 us).  Here a workgroup owns a small output tile and its NW waves split
// K between them: each wave loads its operand fragments straight from global
// memory into registers, four 16-deep K chunks in flight, and the waves'
// partial tiles are added through LDS in wave order (deterministic).  No LDS
// staging: an operand element is read by one tile row or column, from L2;
// larger products take larger tiles.
#include "layup_internal.h"

namespace layup {

namespace {

struct F32Args {
  const float* A;
  const float* B;
  float* C;
  const float* bias;
  const float* aux;
  const float* mask;
  float* rowsum;
  int64_t M, N, K, lda, ldb, ldc;
  int32_t relu, vec_a, vec_b;
};

// Four consecutive k (k0..k0+3) of row r of an operand, zero past K.
// k-major: element (r, k) at p[r*ld + k]; m-major: at p[k*ld + r].
template <bool KMAJOR>
__device__ __forceinline__ f32x4 load4(const float* p, int64_t ld, int64_t r, int64_t k0, int64_t K, bool vec) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (KMAJOR && vec && k0 + 4 <= K) return *reinterpret_cast<const f32x4*>(p + r * ld + k0);
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (k0 + e < K) v[e] = KMAJOR ? p[r * ld + k0 + e] : p[(k0 + e) * ld + r];
  return v;
}

// T x T blocks of BS x BS outputs per workgroup (BS 16 or 32); wave w takes
// the K chunks w, w + NW, ... of 4 x 64 / BS.  Fragment layout: lane l holds
// row (column) l % BS and the four k of group l / BS; instruction e multiplies
// the k 4 g + e of the groups g, the same set for both operands.
template <bool AK, bool BKM, int T, int NW, int BS>
__device__ __forceinline__ void gemm_f32_tile(const F32Args& P, int bx, int by) {
  static_assert(BS == 16 || BS == 32, "a float32 matrix instruction");
  constexpr int KC = 4 * 64 / BS;                 // k of a chunk
  constexpr int R = BS * BS / 64;                 // outputs of a block per lane
  constexpr int UN = T == 1 && BS == 16 ? 4 : 2;  // K chunks in flight
  using Acc = float __attribute__((ext_vector_type(R)));
  __shared__ float red[NW > 1 ? NW : 1][T * T][R][64];
  __shared__ float rred[NW][T][BS];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int g = lane / BS, r = lane % BS;
  const int64_t m0 = (int64_t)by * (BS * T), n0 = (int64_t)bx * (BS * T);
  int64_t ar[T], br[T];
#pragma unroll
  for (int i = 0; i < T; ++i) {
    ar[i] = min(m0 + BS * i + r, P.M - 1);
    br[i] = min(n0 + BS * i + r, P.N - 1);
  }
  Acc acc[T][T];
  float rs[T];
#pragma unroll
  for (int i = 0; i < T; ++i) {
    rs[i] = 0.f;
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
      for (int e = 0; e < R; ++e) acc[i][j][e] = 0.f;
  }
  for (int64_t c0 = KC * w; c0 < P.K; c0 += KC * NW * UN) {
    f32x4 a[UN][T], b[UN][T];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int64_t k = c0 + (int64_t)KC * NW * u + 4 * g;
#pragma unroll
      for (int i = 0; i < T; ++i) {
        a[u][i] = load4<AK>(P.A, P.lda, ar[i], k, P.K, P.vec_a);
        b[u][i] = load4<BKM>(P.B, P.ldb, br[i], k, P.K, P.vec_b);
      }
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
          for (int j = 0; j < T; ++j) {
            if constexpr (BS == 16)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][i][e], b[u][j][e], acc[i][j], 0, 0, 0);
            else
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u][i][e], b[u][j][e], acc[i][j], 0, 0, 0);
          }
#pragma unroll
      for (int i = 0; i < T; ++i) rs[i] += (a[u][i][0] + a[u][i][1]) + (a[u][i][2] + a[u][i][3]);
    }
  }
  const bool rowsum = P.rowsum && bx == 0;
  if (rowsum) {
#pragma unroll
    for (int i = 0; i < T; ++i) {
      float s = rs[i];
#pragma unroll
      for (int o = BS; o < 64; o *= 2) s += __shfl_xor(s, o, 64);
      if (lane < BS) rred[w][i][lane] = s;
    }
  }
  if (NW > 1) {
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
      for (int j = 0; j < T; ++j)
#pragma unroll
        for (int e = 0; e < R; ++e) red[w][i * T + j][e][lane] = acc[i][j][e];
  }
  __syncthreads();
  if (rowsum) {
    for (int x = threadIdx.x; x < BS * T; x += 64 * NW) {
      float s = rred[0][x / BS][x % BS];
      for (int k = 1; k < NW; ++k) s += rred[k][x / BS][x % BS];
      if (m0 + x < P.M) P.rowsum[m0 + x] = s;
    }
  }
  // wave w finishes output registers w, w + NW, ... of the tile's T*T*R;
  // register e of lane l is row 4 g + e % 4 (+ 8 (e / 4) of a 32 x 32 block)
#pragma unroll
  for (int x = 0; x < T * T * R; ++x) {
    if (x % NW != w) continue;
    const int blk = x / R, e = x % R;
    float v = NW > 1 ? red[0][blk][e][lane] : acc[blk / T][blk % T][e];
    if (NW > 1)
      for (int k = 1; k < NW; ++k) v += red[k][blk][e][lane];
    const int64_t m = m0 + BS * (blk / T) + 8 * (e / 4) + 4 * g + e % 4, n = n0 + BS * (blk % T) + r;
    if (m >= P.M || n >= P.N) continue;
    const int64_t off = m * P.ldc + n;
    if (P.bias) v += P.bias[n];
    if (P.aux) v += P.aux[off];
    if (P.relu) v = v > 0.f ? v : 0.f;
    if (P.mask) v = P.mask[off] > 0.f ? v : 0.f;
    P.C[off] = v;
  }
}

template <bool AK, bool BKM, int T, int NW, int BS>
__global__ __launch_bounds__(64 * NW) void gemm_f32_kernel(const F32Args P) {
  gemm_f32_tile<AK, BKM, T, NW, BS>(P, blockIdx.x, blockIdx.y);
}

// dW and dX of a layer: the first workgroups take dW's 16 x 16 tiles, the
// others dX's, row by row.
struct F32Pair {
  F32Args dw, dx;
  int32_t dw_n, dw_items, dx_n, pad;  // tile columns of each, tiles of dW
};
template <int NW>
__global__ __launch_bounds__(64 * NW) void gemm_f32_backward_kernel(const F32Pair P) {
  const int b = blockIdx.x;
  if (b < P.dw_items) gemm_f32_tile<false, false, 1, NW, 16>(P.dw, b % P.dw_n, b / P.dw_n);
  else gemm_f32_tile<true, false, 1, NW, 16>(P.dx, (b - P.dw_items) % P.dx_n, (b - P.dw_items) / P.dx_n);
}

template <int T, int NW, int BS = 16>
hipError_t launch_tile(const Gemm& g, const F32Args& P, hipStream_t s) {
  const int64_t gy = cdiv(P.M, BS * T);
  // grid.y holds 65535 row tiles: taller products go in bands of rows
  constexpr int64_t BAND = 65535;
  for (int64_t y = 0; y < gy; y += BAND) {
    F32Args Q = P;
    const int64_t r0 = y * BS * T;
    Q.M = std::min<int64_t>(P.M - r0, BAND * BS * T);
    if (Q.A) Q.A += g.a_kmajor ? r0 * P.lda : r0;
    Q.C += r0 * P.ldc;
    if (Q.aux) Q.aux += r0 * P.ldc;
    if (Q.mask) Q.mask += r0 * P.ldc;
    if (Q.rowsum) Q.rowsum += r0;
    // a band's first row keeps the vector loads' alignment (k-major: lda a
    // multiple of 4; m-major operands are read element by element)
    const dim3 grid((unsigned)cdiv(P.N, BS * T), (unsigned)cdiv(Q.M, BS * T));
    if (g.a_kmajor && g.b_kmajor) gemm_f32_kernel<true, true, T, NW, BS><<<grid, 64 * NW, 0, s>>>(Q);
    else if (g.a_kmajor) gemm_f32_kernel<true, false, T, NW, BS><<<grid, 64 * NW, 0, s>>>(Q);
    else if (g.b_kmajor) gemm_f32_kernel<false, true, T, NW, BS><<<grid, 64 * NW, 0, s>>>(Q);
    else gemm_f32_kernel<false, false, T, NW, BS><<<grid, 64 * NW, 0, s>>>(Q);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

static F32Args f32_args(const Gemm& g) {
  F32Args P;
  P.A = (const float*)g.A;
  P.B = (const float*)g.B;
  P.C = (float*)g.C;
  P.bias = g.bias;
  P.aux = (const float*)g.aux;
  P.mask = g.mask;
  P.rowsum = g.rowsum;
  P.M = g.M;
  P.N = g.N;
  P.K = g.K;
  P.lda = g.lda;
  P.ldb = g.ldb;
  P.ldc = g.ldc;
  P.relu = g.relu;
  P.vec_a = g.lda % 4 == 0 && ((uintptr_t)g.A & 15) == 0;
  P.vec_b = g.ldb % 4 == 0 && ((uintptr_t)g.B & 15) == 0;
  return P;
}

// 16 x 16 tiles while they do not fill the chip a few times over (each of
// the 256 CUs holds four 8-wave workgroups); beyond that 32 x 32 tiles read
// each operand half as often.  From 1024 tiles of 64 x 64 on, and K = 256
// (below it the sum over the waves costs more than it saves), 64 x 64 tiles of
// 32 x 32 blocks: half the operand reads again, and an m-major operand's lines
// are read whole.  4096 x 4096 x 4096: 1490 to 1620 us in the four layouts,
// 32 x 32 tiles 2090 to 2260, the first, LDS-staged kernel 1990 to 2070;
// 4096 x 4096 x 256: 124 to 131, 130 to 136, 130 to 134; x 64: 57, 42 to 45, 45.
constexpr int64_t F32_SMALL_TILES = 4096, F32_LARGE_TILES = 1024, F32_LARGE_K = 256;
static int64_t tiles16(const Gemm& g) { return cdiv(g.M, 16) * cdiv(g.N, 16); }

hipError_t launch_gemm_f32(const Gemm& g, hipStream_t s) {
  if (g.M == 0 || g.N == 0) return hipSuccess;
  if (g.batch != 1) return hipErrorInvalidValue;
  const F32Args P = f32_args(g);
  if (g.K >= F32_LARGE_K && cdiv(g.M, 64) * cdiv(g.N, 64) >= F32_LARGE_TILES) return launch_tile<2, 4, 32>(g, P, s);
  // eight (four) waves where K gives each of them more than one chunk, two
  // (one) for the short K of dW (the batch)
  if (tiles16(g) > F32_SMALL_TILES) return g.K > 64 ? launch_tile<2, 4>(g, P, s) : launch_tile<2, 1>(g, P, s);
  return g.K > 64 ? launch_tile<1, 8>(g, P, s) : launch_tile<1, 2>(g, P, s);
}

// A launch costs more than either product of the tiny MLP's layers (4 us), so
// the pair shares one while both stay on small tiles.
hipError_t launch_gemm_f32_backward(const Gemm& dw, const Gemm& dx, hipStream_t s) {
  const int64_t a = tiles16(dw), b = tiles16(dx);
  if (a < 1 || b < 1 || a + b > F32_SMALL_TILES || dw.batch != 1 || dx.batch != 1 || dw.a_kmajor || dw.b_kmajor ||
      !dx.a_kmajor || dx.b_kmajor) {
    const hipError_t e = launch_gemm_f32(dw, s);
    return e != hipSuccess ? e : launch_gemm_f32(dx, s);
  }
  const F32Pair P{f32_args(dw), f32_args(dx), (int)cdiv(dw.N, 16), (int)a, (int)cdiv(dx.N, 16), 0};
  gemm_f32_backward_kernel<8><<<(unsigned)(a + b), 512, 0, s>>>(P);
  return hipGetLastError();
}

}  // namespace layup

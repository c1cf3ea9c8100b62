// bfloat16 GEMM on the CDNA4 matrix cores (v_mfma_f32_32x32x16_bf16), float32
// accumulation.  This is the one dense contraction of the layer-wise step:
// the dX = dY W and dW = dY^T X products of every linear layer's backward
// (LayUp Algorithm 1, "Backward pass at layer l"), plus the forward and the
// attention products that produce what the backward reads.
//
// Structure: a BM x BN block tile computed by a WGM x WGN grid of wave64s,
// each wave a (BM/WGM) x (BN/WGN) tile of 32x32 MFMA blocks with float32
// accumulators in registers.  K advances in steps of 32 or 64 through a ring of LDS
// stages filled by direct-to-LDS loads (see the pipeline notes below), so
// several K steps of both operands are in flight while one is multiplied and
// no registers stage the copy.  An operand that is k-contiguous in HBM stays
// k-contiguous in LDS and is read with 128-bit LDS reads; an m/n-contiguous
// operand (the transposed operands of dW = dY^T X) stays m-contiguous and is
// read with the transposing LDS read (ds_read_b64_tr_b16), so neither layout
// is transposed in registers.
//
// The grid is one flat list of (batch or split, tile) work items dealt out
// XCD-aware: workgroups are dispatched round-robin over the 8 XCDs (each with
// its own L2), so consecutive work items are mapped onto one XCD and tiles
// sharing an operand band hit the same L2.  Split-K (float32 partials + a
// fixed-order reduction, deterministic) fills the 256 CUs when the output has
// too few tiles.  Causal attention products skip the tiles and K ranges that
// the mask makes zero.  Epilogues fuse bias, residual add, GELU (storing the
// pre-activation and the activation) and the GELU backward.
#include "layup_internal.h"

namespace layup {

namespace {


struct KArgs {
  const bf16_t* A;
  const bf16_t* B;
  void* C;
  void* C2;
  const void* aux;
  const float* bias;
  float* partial;
  int64_t M, N, K, lda, ldb, ldc;
  int64_t a_outer, a_inner, b_outer, b_inner, c_outer, c_inner;
  int32_t inner, splits, tiles_m, tiles_n;
  int32_t causal, nz;      // nz: batch count
  int64_t k_per_split;
  UpdArgs upd;             // EPI_UPDATE
  float* rowsum;           // row sums of an m-major A (split-K: partials after the C partials)
  int64_t run;             // FL: the longest run of products of one accumulator
};

// GELU, tanh form: 0.5 x (1 + tanh(u)), u = sqrt(2/pi) (x + 0.044715 x^3).
// Since 0.5 (1 + tanh(u)) = sigmoid(2u), it is x s with s = 1 / (1 + e),
// e = e^(-2u): one exponential and a reciprocal instead of tanh.  1 - s = e s
// keeps its relative accuracy where s is close to 1.
// e is 2^t, t = x (K1 + K2 x^2): an error of t counts in e in proportion to
// |t|, so the last product's rounding error is taken from a second fma and
// put back as e (1 + ln2 lo).  Relative error of GELU over [-5, -2], rms:
// 3.0e-7, against 4.2e-7 with u rounded and the argument of the exponential
// reduced exactly (five instructions more) and 4.7e-7 with 2^(-2u log2(e)).
// x is clamped to where it matters: 2^t stays finite, with a normal
// reciprocal, down to x = -10 (beyond it GELU is below 2e-37) and is 0 from
// x = 13 on.
__device__ __forceinline__ float gelu_sig(float x, float& e) {
  const float K1 = -2.3022081981443251f;   // -2 sqrt(2/pi) log2(e)
  const float K2 = -0.10294323958002350f;  // 0.044715 K1
  const float xc = __builtin_amdgcn_fmed3f(x, -10.0f, 13.0f);
  const float k = fmaf(K2, xc * xc, K1);
  const float t = xc * k;
  const float lo = fmaf(xc, k, -t);
  const float p = __builtin_amdgcn_exp2f(t);
  e = fmaf(p, lo * 0.69314718055994531f, p);
  return __builtin_amdgcn_rcpf(1.0f + e);
}

__device__ __forceinline__ float gelu_tanh_f(float x) {
  float e;
  return x * gelu_sig(x, e);
}

// d/dx GELU = s + x s (1 - s) 2 sqrt(2/pi) (1 + 3 0.044715 x^2)
__device__ __forceinline__ float gelu_tanh_grad_f(float x) {
  float e;
  const float s = gelu_sig(x, e);
  const float c2 = 2.0f * 0.7978845608028654f;
  return fmaf(x * s * (e * s), c2 * fmaf(3.0f * 0.044715f, x * x, 1.0f), s);
}

// Sum of the 8 bfloat16 values of an MFMA operand register quad, in order.
__device__ __forceinline__ float sum_bf16x8(const u32x4& u) {
  float s = __builtin_bit_cast(float, u[0] << 16);
  s += __builtin_bit_cast(float, u[0] & 0xffff0000u);
#pragma unroll
  for (int e = 1; e < 4; ++e) {
    s += __builtin_bit_cast(float, u[e] << 16);
    s += __builtin_bit_cast(float, u[e] & 0xffff0000u);
  }
  return s;
}

// Split of K: none, one for the launch, or each product of a group its own
// (P.splits, which may be 1).
enum SplitMode : int { SPLIT_NO = 0, SPLIT_YES = 1, SPLIT_OWN = 2 };

// Epilogue of W consecutive columns n..n+W-1 of row m (columns >= N
// skipped); W = 4 for float32 results, 8 for bfloat16 ones.  vec: every
// access 16-byte aligned and n + W <= N.
template <int EPI, int SPLIT, int W>
__device__ __forceinline__ void epi_store(const KArgs& P, int split, int64_t c_off, int64_t m, int64_t n,
                                          float (&v)[W], bool vec) {
  const int64_t rem = P.N - n;
  const int ne = vec ? W : (int)(rem < W ? rem : W);
  if constexpr (SPLIT || EPI == EPI_F32 || EPI == EPI_UPDATE) {
    static_assert(W == 4, "float32 results go four columns at a time");
    const f32x4 v4{v[0], v[1], v[2], v[3]};
    if constexpr (SPLIT != SPLIT_NO) {
      if (SPLIT == SPLIT_YES || P.splits > 1) {
        float* dst = P.partial + (int64_t)split * P.M * P.N + m * P.N + n;
        if (vec) *reinterpret_cast<f32x4*>(dst) = v4;
        else for (int e = 0; e < ne; ++e) dst[e] = v[e];
        return;
      }
    }
    if constexpr (SPLIT == SPLIT_YES) {
    } else if constexpr (EPI == EPI_UPDATE) {
      const int64_t off = m * P.ldc + n;
      if (vec) apply_update4(P.upd, off, v4);
      else for (int e = 0; e < ne; ++e) apply_update(P.upd, off + e, v[e]);
    } else {
      const int64_t off = c_off + m * P.ldc + n;
      float* dst = reinterpret_cast<float*>(P.C) + off;
      const float* aux = reinterpret_cast<const float*>(P.aux);
      if (vec) {
        f32x4 o = v4;
        if (P.bias) o += *reinterpret_cast<const f32x4*>(P.bias + n);
        if (aux) o += *reinterpret_cast<const f32x4*>(aux + off);
        *reinterpret_cast<f32x4*>(dst) = o;
      } else {
        for (int e = 0; e < ne; ++e) {
          float o = v[e];
          if (P.bias) o += P.bias[n + e];
          if (aux) o += aux[off + e];
          dst[e] = o;
        }
      }
    }
  } else {
    static_assert(W == 8, "bfloat16 results go eight columns at a time");
    const int64_t off = c_off + m * P.ldc + n;
    if (P.bias && (EPI == EPI_BF16 || EPI == EPI_GELU)) {
      if (vec) {
        const f32x4 b0 = *reinterpret_cast<const f32x4*>(P.bias + n);
        const f32x4 b1 = *reinterpret_cast<const f32x4*>(P.bias + n + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] += b0[e];
          v[e + 4] += b1[e];
        }
      } else {
        for (int e = 0; e < ne; ++e) v[e] += P.bias[n + e];
      }
    }
    float w[8];
    if constexpr (EPI == EPI_DGELU) {
      const bf16_t* pre = reinterpret_cast<const bf16_t*>(P.aux) + off;
      float f[8];
      if (vec) {
        const u32x4 u = *reinterpret_cast<const u32x4*>(pre);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          f[2 * e] = __builtin_bit_cast(float, u[e] << 16);
          f[2 * e + 1] = __builtin_bit_cast(float, u[e] & 0xffff0000u);
        }
      } else {
        for (int e = 0; e < 8; ++e) f[e] = e < ne ? bf2f(pre[e]) : 0.f;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] *= gelu_tanh_grad_f(f[e]);
    }
    if constexpr (EPI == EPI_GELU) {
#pragma unroll
      for (int e = 0; e < 8; ++e) w[e] = gelu_tanh_f(v[e]);
    }
    bf16_t* dst = reinterpret_cast<bf16_t*>(P.C) + off;
    bf16_t* dst2 = EPI == EPI_GELU ? reinterpret_cast<bf16_t*>(P.C2) + off : nullptr;
    if (vec) {
      const u32x4 o{pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7])};
      // the pre-activation is next read in the backward: past the caches
      if (EPI == EPI_GELU) __builtin_nontemporal_store(o, reinterpret_cast<u32x4*>(dst));
      else *reinterpret_cast<u32x4*>(dst) = o;
      if (EPI == EPI_GELU)
        *reinterpret_cast<u32x4*>(dst2) =
            u32x4{pack_bf2(w[0], w[1]), pack_bf2(w[2], w[3]), pack_bf2(w[4], w[5]), pack_bf2(w[6], w[7])};
    } else {
      for (int e = 0; e < ne; ++e) {
        dst[e] = f2bf(v[e]);
        if (EPI == EPI_GELU) dst2[e] = f2bf(w[e]);
      }
    }
  }
}

// ------------------------------------------------------------ pipeline
// K advances in steps of BKV (32 or 64) through rings of LDS stages.  Every
// operand tile is copied HBM -> LDS by direct-to-LDS loads
// (global_load_lds_dwordx4: each lane's 16 bytes land at LDS base + 16*lane,
// one 1 KB block per wave instruction), so no registers stage the data and
// the tiles of the next stages are in flight while one is multiplied.  Rows
// are clamped into the operand (rows >= R read row R-1: they only feed
// discarded outputs); the last, partial K step also clamps k, and its tail is
// zeroed in LDS before use.
//
// LDS layouts (per tile, byte offsets):
//  k-major operand, ROWS x 32: row r = 64 B = four 16-byte chunks; chunk c at
//    r*64 + 16*(c ^ ((r >> 2) & 3)).  Sixteen lanes reading one chunk of 16
//    consecutive rows (the MFMA operand read, ds_read_b128) cover all banks.
//  m-major operand, 32 x ROWS (k rows of ROWS elements): chunk c of k-row kk at
//    kk*2*ROWS + 16*(c ^ sw(kk)).  The operand is read with ds_read_b64_tr_b16:
//    within each 16-lane group, lane s supplies 4 consecutive m of k-row
//    kb + s/4 and receives, transposed, 4 consecutive k of one m, so four
//    consecutive k-rows are read at one chunk position.  sw spreads those rows
//    over the 256-byte bank cycle: ((kk & 3) << 2) & (ROWS/8 - 1) for
//    power-of-two ROWS; none for ROWS = 96 (a 192-byte row stride already
//    staggers them); 4 on the odd pairs for ROWS = 192 (384-byte stride).
__device__ __forceinline__ constexpr int kswz(int r, int bkv) {
  // 16 consecutive rows of 2*bkv bytes must cover the 256-byte bank cycle once
  return (r / (128 / bkv)) % (bkv / 8);
}
template <int BKV>
__device__ __forceinline__ int km_off(int r, int c) { return r * 2 * BKV + 16 * (c ^ kswz(r, BKV)); }
template <int ROWS>
__device__ __forceinline__ int mm_sw(int kk) {
  static_assert(ROWS % 32 == 0 && (ROWS & (ROWS - 1)) == 0 || ROWS == 96 || ROWS == 192,
                "m-major tile width without a bank swizzle");
  if (ROWS == 96) return 0;
  if (ROWS == 192) return (kk & 2) << 1;
  return ((kk & 3) << 2) & (ROWS / 8 - 1);
}
template <int ROWS>
__device__ __forceinline__ int mm_off(int kk, int c) { return kk * 2 * ROWS + 16 * (c ^ mm_sw<ROWS>(kk)); }

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef short v8i16 __attribute__((ext_vector_type(8)));
#define LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

// Issue copy i (of BLOCKS / NWAVES) of this wave's share of the
// direct-to-LDS copies of one ROWS x BKV tile: one 1 KB block.
template <int ROWS, bool KMAJOR, int BKV, int NWAVES>
__device__ __forceinline__ void issue_block(const bf16_t* base, int64_t ld, int64_t r0, int64_t k0,
                                            int64_t R, int64_t K, char* lds, int wave, int lane, int i) {
  constexpr int BLOCKS = ROWS * BKV * 2 / 1024;  // 1 KB blocks per tile
  static_assert(BLOCKS % NWAVES == 0, "copies must split evenly over the waves");
  constexpr int PER_WAVE = BLOCKS / NWAVES;
  {
    const int blk = wave * PER_WAVE + i;
    const bf16_t* src;
    if (KMAJOR) {
      constexpr int KCH = BKV / 8;           // 16-byte chunks per row
      const int row = blk * (64 / KCH) + lane / KCH;
      const int c = (lane % KCH) ^ kswz(row, BKV);
      const int64_t gr = min(r0 + row, R - 1);
      const int64_t gk = min(k0 + 8 * c, K - 8);
      src = base + gr * ld + gk;
    } else {
      constexpr int LPR = ROWS / 8;           // 16-byte chunks per k-row
      const int q = blk * 64 + lane;           // chunk slot in the tile
      const int kk = q / LPR;
      const int c = (q % LPR) ^ mm_sw<ROWS>(kk);
      const int64_t gk = min(k0 + kk, K - 1);
      const int64_t gm = min(r0 + 8 * c, R - 8);
      src = base + gk * ld + gm;
    }
    __builtin_amdgcn_global_load_lds(src, LDS_PTR(lds + blk * 1024), 16, 0, 0);
  }
}

// Where this lane's 16 bytes of copy i of a wave's share come from, for the
// whole K steps from k0 on (rows clamped as above, k in range): the next
// step's are a fixed number of bytes further.
template <int ROWS, bool KMAJOR, int BKV, int NWAVES>
__device__ __forceinline__ const char* block_src(const bf16_t* base, int64_t ld, int64_t r0, int64_t k0,
                                                 int64_t R, int wave, int lane, int i) {
  const int blk = wave * (ROWS * BKV * 2 / 1024 / NWAVES) + i;
  if (KMAJOR) {
    constexpr int KCH = BKV / 8;
    const int row = blk * (64 / KCH) + lane / KCH;
    const int c = (lane % KCH) ^ kswz(row, BKV);
    return reinterpret_cast<const char*>(base + min(r0 + row, R - 1) * ld + k0 + 8 * c);
  } else {
    constexpr int LPR = ROWS / 8;
    const int q = blk * 64 + lane;
    const int kk = q / LPR;
    const int c = (q % LPR) ^ mm_sw<ROWS>(kk);
    return reinterpret_cast<const char*>(base + (k0 + kk) * ld + min(r0 + 8 * c, R - 8));
  }
}

// One 1 KB block, 16 bytes per lane.  (A function template: the builtin's
// width is checked against the target, and the host pass has none.)
template <int>
__device__ __forceinline__ void copy_block(const char* src, char* lds) {
  __builtin_amdgcn_global_load_lds(src, LDS_PTR(lds), 16, 0, 0);
}

// Zero the k >= krem part of a tile (last, partial K step).
template <int ROWS, bool KMAJOR, int BKV>
__device__ __forceinline__ void zero_tail(char* lds, int krem) {
  if (KMAJOR) {
    constexpr int KCH = BKV / 8;
    for (int e = threadIdx.x; e < ROWS * KCH; e += blockDim.x) {
      const int r = e / KCH, c = e % KCH;
      if (8 * c >= krem) *reinterpret_cast<u32x4*>(lds + km_off<BKV>(r, c)) = u32x4{0, 0, 0, 0};
    }
  } else {
    for (int e = threadIdx.x; e < BKV * (ROWS / 8); e += blockDim.x) {
      const int kk = e / (ROWS / 8), c = e % (ROWS / 8);
      if (kk >= krem) *reinterpret_cast<u32x4*>(lds + mm_off<ROWS>(kk, c)) = u32x4{0, 0, 0, 0};
    }
  }
}

// ---- operand fragments.  One 32x32x16 MFMA operand fragment holds rows
// rb..rb+31 (lane % 32) and k values ks*16 + 8*(lane/32) .. +7 of the tile.
// The LDS reads are issued as inline assembly with explicit lgkmcnt waits:
// the compiler cannot tell an LDS read apart from the direct-to-LDS copies in
// flight into other stages, and before a transposing read it would wait for
// every outstanding copy (vmcnt(0)), which serializes the copy pipeline.
// Offsets are compile-time immediates where they are lane-independent.
template <int N>
struct IntC { static constexpr int value = N; };
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(IntC<I>{});
    static_for<I + 1, N>(f);
  }
}

__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

template <int OFF>
__device__ __forceinline__ u32x4 lds_read_b128(uint32_t a) {
  static_assert(OFF >= 0 && OFF < 65536, "LDS immediate offset");
  u32x4 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(a), "n"(OFF));
  return v;
}

template <int OFF>
__device__ __forceinline__ u32x2 lds_read_tr(uint32_t a) {
  static_assert(OFF >= 0 && OFF < 65536, "LDS immediate offset");
  u32x2 v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(a), "n"(OFF));
  return v;
}

// Wait until at most N LDS reads are outstanding (LDS reads return in order).
template <int N>
__device__ __forceinline__ void lgkm_wait() {
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N < 15 ? N : 15));
}

// Make the MFMA that consumes v depend on the preceding wait.
__device__ __forceinline__ void after_wait(u32x4& v) { asm volatile("" : "+v"(v)); }

// Per-lane part of the LDS offset of a fragment.  k-major: one value per
// K sub-step (the 32-row blocks are whole-row multiples apart, which the
// swizzle leaves alone); m-major: one value per 32-column block (the sub-step
// and the second half of the k range are whole k-rows apart).
template <int ROWS, bool KMAJOR, int BKV>
__device__ __forceinline__ uint32_t frag_lane_off(int rb, int idx, int lane) {
  if (KMAJOR) {
    return km_off<BKV>(rb + (lane & 31), 2 * idx + (lane >> 5));
  } else {
    const int g = lane >> 4, s = lane & 15;
    const int kb = 8 * (g >> 1) + (s >> 2);
    const int m = rb + 32 * idx + 16 * (g & 1) + 4 * (s & 3);
    return mm_off<ROWS>(kb, m >> 3) + (m & 7) * 2;
  }
}

// Issue the LDS reads of the T fragments of sub-step KSI of one operand.
// sb: stage base + operand base; off: frag_lane_off values.
template <int ROWS, bool KMAJOR, int BKV, int T, int KSI>
__device__ __forceinline__ void read_frags(uint32_t sb, const uint32_t* off, u32x4* f) {
  static_for<0, T>([&](auto I) {
    constexpr int i = decltype(I)::value;
    if constexpr (KMAJOR) {
      f[i] = lds_read_b128<i * 32 * 2 * BKV>(sb + off[KSI]);
    } else {
      const u32x2 lo = lds_read_tr<KSI * 16 * 2 * ROWS>(sb + off[i]);
      const u32x2 hi = lds_read_tr<KSI * 16 * 2 * ROWS + 4 * 2 * ROWS>(sb + off[i]);
      f[i] = u32x4{lo.x, lo.y, hi.x, hi.y};
    }
  });
}

// s_waitcnt vmcnt(n), expcnt and lgkmcnt left alone (gfx9 encoding).
#define WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | (7 << 4) | (15 << 8))

// Workgroup barrier without the release fence of __syncthreads(): the fence
// would make the compiler drain every outstanding direct-to-LDS load
// (vmcnt(0)) at each K step; the exact wait is issued by hand before it.
__device__ __forceinline__ void barrier_only() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

// WGM x WGN waves per workgroup; each wave owns a (BM/WGM) x (BN/WGN) block of
// 32x32 MFMA tiles.  STAGES LDS stages of the BM x BKV and BN x BKV operand
// tiles.  This is the work of one workgroup: item `lid` of P's flat list of
// (batch or split, tile) work items.
// FL: the accumulators take at most P.run products in a row.
template <int BM, int BN, int WGM, int WGN, int STAGES, bool AK, bool BKM, int EPI, int SPLIT, int BKV, bool FL>
__device__ __forceinline__ void gemm_item(const KArgs& P, int lid) {
  constexpr int NW = WGM * WGN;
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int S = STAGES;
  static_assert(S >= 2, "the copies of a stage run while another is multiplied");
  constexpr int A_BYTES = BM * BKV * 2, B_BYTES = BN * BKV * 2;
  constexpr int A_BLK = A_BYTES / 1024, B_BLK = B_BYTES / 1024;
  // direct-to-LDS instructions per wave per K step (same count on every wave)
  constexpr int LOADS_A = A_BLK / NW, LOADS_B = B_BLK / NW, NPIECE = LOADS_A + LOADS_B;
  static_assert(A_BLK % NW == 0 && B_BLK % NW == 0, "copies must split evenly over the waves");
  static_assert((S - 2) * NPIECE <= 63, "vmcnt field");
  constexpr int KS = BKV / 16;
  static_assert(KS % 2 == 0, "the fragment buffers alternate by sub-step");
  __shared__ __attribute__((aligned(1024))) char smem[S * (A_BYTES + B_BYTES)];

  // tiles go in groups of 8 tile-rows for L2 reuse of B
  const int n_tiles = P.tiles_m * P.tiles_n;
  const int zz = lid / n_tiles, id = lid % n_tiles;
  constexpr int GROUP = 8;
  const int width = GROUP * P.tiles_n;
  const int grp = id / width;
  const int first_m = grp * GROUP;
  const int gsz = min(P.tiles_m - first_m, GROUP);
  const int tm = first_m + (id % width) % gsz;
  const int tn = (id % width) / gsz;

  const int z = SPLIT ? 0 : zz;
  const int split = SPLIT ? zz : 0;
  const int zo = z / P.inner, zi = z % P.inner;
  const bf16_t* Ab = P.A + zo * P.a_outer + zi * P.a_inner;
  const bf16_t* Bb = P.B + zo * P.b_outer + zi * P.b_inner;
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  int64_t kb = 0, ke = P.K;
  if (SPLIT) {
    kb = split * P.k_per_split;
    ke = min(P.K, kb + P.k_per_split);
  }
  if (P.causal == CAUSAL_OUT_LOWER && n0 > m0 + BM - 1) return;  // whole tile above the diagonal
  if (P.causal == CAUSAL_A_LOWER) ke = min(ke, m0 + BM);
  if (P.causal == CAUSAL_A_UPPER) kb = max(kb, m0);

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WGN, wn = wave % WGN;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // Row sums of an m-major A (bias gradient of dW = dY^T X): the waves of
  // the first wave column in the first tile column add up the A fragments
  // they feed to the MFMAs (lane l: row l % 32 of block i, 8 of every 16 k).
  const bool rs_on = !AK && P.rowsum && tn == 0 && wn == 0;
  float rsum[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) rsum[i] = 0.f;

  // FL: after every P.run products the accumulators (and row sums) are added
  // into a second set and start again from zero.  A float32 sum of K products
  // has an error that grows with the square root of the run: over K = 8192 it
  // is 5.7e-7 of the result in one run, 2.7e-7 in runs of 2048 (or as the sum
  // of four split-K partials) and 1.5e-7 in runs of 512.  Runs of 512 cost 1
  // to 3 % of the K loop.  The second set fits the register file up to 64
  // accumulators a thread; row sums keep theirs in LDS, each lane its own.
  static_assert(!FL || TM * TN <= 4, "registers for two sets of accumulators");
  f32x16 tot[FL ? TM : 1][FL ? TN : 1];
  __shared__ float rs_tot[FL && !AK ? WGM * TM * 64 : 1];
  if constexpr (FL) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) tot[i][j][r] = 0.f;
      if (rs_on) rs_tot[(wm * TM + i) * 64 + lane] = 0.f;
    }
  }
  auto flush = [&]() {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          tot[i][j][r] += acc[i][j][r];
          acc[i][j][r] = 0.f;
        }
      if (rs_on) rs_tot[(wm * TM + i) * 64 + lane] += rsum[i];
      rsum[i] = 0.f;
    }
  };

  // per-lane fragment offsets inside a stage (B after A)
  constexpr int NA = AK ? KS : TM, NB = BKM ? KS : TN;
  uint32_t a_off[NA], b_off[NB];
#pragma unroll
  for (int x = 0; x < NA; ++x) a_off[x] = frag_lane_off<BM, AK, BKV>(wm * WM, x, lane);
#pragma unroll
  for (int x = 0; x < NB; ++x) b_off[x] = frag_lane_off<BN, BKM, BKV>(wn * WN, x, lane);
  // LDS reads issued per sub-step
  constexpr int NREAD = TM * (AK ? 1 : 2) + TN * (BKM ? 1 : 2);
  const uint32_t lds0 = lds_addr(smem);

  const int nk = (int)((ke - kb + BKV - 1) / BKV);
  const int krem = (int)((ke - kb) - (int64_t)(nk - 1) * BKV);  // valid k in the last step
  const int n_full = krem < BKV ? nk - 1 : nk;                   // steps whose copies need no clamped k
  char* const smem_b = smem + S * A_BYTES;
  const char* src_a[LOADS_A];
  const char* src_b[LOADS_B];
#pragma unroll
  for (int i = 0; i < LOADS_A; ++i) src_a[i] = block_src<BM, AK, BKV, NW>(Ab, P.lda, m0, kb, P.M, wave, lane, i);
#pragma unroll
  for (int i = 0; i < LOADS_B; ++i) src_b[i] = block_src<BN, BKM, BKV, NW>(Bb, P.ldb, n0, kb, P.N, wave, lane, i);
  const int64_t adv_a = AK ? 2 * BKV : 2 * BKV * P.lda, adv_b = BKM ? 2 * BKV : 2 * BKV * P.ldb;
  // copy p of the next whole K step into ring slot `slot`
  auto issue = [&](int slot, int p) {
    if (p < LOADS_A) {
      copy_block<0>(src_a[p], smem + slot * A_BYTES + (wave * LOADS_A + p) * 1024);
      src_a[p] += adv_a;
    } else {
      const int q = p - LOADS_A;
      copy_block<0>(src_b[q], smem_b + slot * B_BYTES + (wave * LOADS_B + q) * 1024);
      src_b[q] += adv_b;
    }
  };
  // all copies of K step t, which may be the partial last one or past the end
  auto issue_step = [&](int t, int slot) {
    if (t < n_full) {
#pragma unroll
      for (int p = 0; p < NPIECE; ++p) issue(slot, p);
    } else if (t < nk) {
#pragma unroll
      for (int p = 0; p < LOADS_A; ++p)
        issue_block<BM, AK, BKV, NW>(Ab, P.lda, m0, kb + (int64_t)t * BKV, P.M, ke, smem + slot * A_BYTES, wave,
                                     lane, p);
#pragma unroll
      for (int p = 0; p < LOADS_B; ++p)
        issue_block<BN, BKM, BKV, NW>(Bb, P.ldb, n0, kb + (int64_t)t * BKV, P.N, ke, smem_b + slot * B_BYTES, wave,
                                      lane, p);
    }
  };
  // Fragments of sub-step ks live in buffer ks % 2.  K step kt begins with
  // the last sub-step of step kt - 1 still to be multiplied (zeros before the
  // first): its fragments are in registers, so the one barrier of a step
  // both publishes the copies of step kt and frees the stage of step kt - 1,
  // and the MFMAs of that sub-step cover the latency of the new stage's first
  // fragment reads and carry the copies of step kt + S - 1 between them.
  // (Reading a stage's first fragments behind the barrier and the copies
  // behind those cost 2 x 0.15 us of each ~1.5 us step of a 256 x 256 x 64
  // tile.)  The scheduling fences keep a cluster's MFMAs ahead of the next
  // wait: the compiler otherwise sinks them below it, and they then wait for
  // fragments they do not need.  What bounds the loop now is the rate of the
  // operand copies per CU (45-75 GB/s whatever the number of stages and of
  // active CUs; L2 prefetching raised it and moved nothing) and how little
  // of it the MFMAs hide: 8192 x 8192 x 8192 takes 880 us (before: 1001),
  // its copies alone 733, its reads and MFMAs alone 565.
  u32x4 af[2][TM], bfr[2][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) af[1][i] = u32x4{0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < TN; ++j) bfr[1][j] = u32x4{0, 0, 0, 0};
  auto read_sub = [&](auto KSI, int slot) {
    constexpr int ks = decltype(KSI)::value;
    read_frags<BM, AK, BKV, TM, ks>(lds0 + (uint32_t)(slot * A_BYTES), a_off, af[ks & 1]);
    read_frags<BN, BKM, BKV, TN, ks>(lds0 + (uint32_t)(S * A_BYTES + slot * B_BYTES), b_off, bfr[ks & 1]);
  };
  auto landed = [&](auto CB) {  // the buffer's reads have been waited for
    constexpr int cb = decltype(CB)::value;
#pragma unroll
    for (int i = 0; i < TM; ++i) after_wait(af[cb][i]);
#pragma unroll
    for (int j = 0; j < TN; ++j) after_wait(bfr[cb][j]);
  };
  // the MFMAs (and row sums) of one buffer; COPY: with the copies of a whole
  // K step into slot `slot` spread between them
  auto multiply = [&](auto CB, auto COPY, int slot) {
    constexpr int cb = decltype(CB)::value;
    constexpr bool copy = decltype(COPY)::value != 0;
    constexpr int PER = (NPIECE + TM * TN - 1) / (TM * TN);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[cb][i]),
                                                            __builtin_bit_cast(bf16x8, bfr[cb][j]),
                                                            acc[i][j], 0, 0, 0);
        if constexpr (copy) {
#pragma unroll
          for (int p = (i * TN + j) * PER; p < (i * TN + j + 1) * PER; ++p)
            if (p < NPIECE) issue(slot, p);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    if constexpr (!AK) {
      if (rs_on) {
#pragma unroll
        for (int i = 0; i < TM; ++i) rsum[i] += sum_bf16x8(af[cb][i]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // MAIN: step kt + S - 1 is a whole one.  The only branch while reads are in
  // flight is the row sums' (multiply): the compiler could move a register of
  // one there, and the tests follow the built code's paths to see that no
  // instruction touches one before its wait.
  auto k_step = [&](auto MAIN, int kt, int slot) {
    constexpr bool main = decltype(MAIN)::value != 0;
    const int pslot = slot == 0 ? S - 1 : slot - 1;  // of steps kt - 1 and kt + S - 1
    if constexpr (main) {
      WAIT_VMCNT((S - 2) * NPIECE);  // loads complete in order: step kt has landed
      barrier_only();
    } else {
      const int left = min(S - 2, nk - 1 - kt);  // younger steps still in flight
      static_for<0, S - 1>([&](auto D) {
        constexpr int d = decltype(D)::value;
        if (left == d) WAIT_VMCNT(d * NPIECE);
      });
      barrier_only();
      if (kt == nk - 1 && krem < BKV) {
        zero_tail<BM, AK, BKV>(smem + slot * A_BYTES, krem);
        zero_tail<BN, BKM, BKV>(smem_b + slot * B_BYTES, krem);
        __syncthreads();
      }
    }
    if constexpr (!main) issue_step(kt + S - 1, pslot);  // its branches before the reads
    read_sub(IntC<0>{}, slot);
    multiply(IntC<1>{}, IntC<main ? 1 : 0>{}, pslot);
    static_for<0, KS - 1>([&](auto KSI) {
      constexpr int ks = decltype(KSI)::value;
      read_sub(IntC<ks + 1>{}, slot);
      lgkm_wait<NREAD>();
      landed(IntC<ks & 1>{});
      multiply(IntC<ks & 1>{}, IntC<0>{}, 0);
    });
    // the last sub-step's fragments are complete before the back edge (no
    // register of a read in flight crosses it) and before the next barrier
    lgkm_wait<0>();
    landed(IntC<1>{});
  };
  for (int t = 0; t < S - 1; ++t) issue_step(t, t);
  int kt = 0, slot = 0;
  const int run = FL ? (int)min(P.run / BKV, (int64_t)1 << 30) : 0;  // K steps
  int left = run;
  auto end_step = [&]() {
    slot = slot + 1 == S ? 0 : slot + 1;
    if constexpr (FL) {
      if (--left == 0) {
        flush();
        left = run;
      }
    }
  };
  for (; kt + S - 1 < n_full; ++kt) {
    k_step(IntC<1>{}, kt, slot);
    end_step();
  }
  for (; kt < nk; ++kt) {
    k_step(IntC<0>{}, kt, slot);
    end_step();
  }
  multiply(IntC<1>{}, IntC<0>{}, 0);
  if constexpr (FL) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] += tot[i][j][r];
      if (rs_on) rsum[i] += rs_tot[(wm * TM + i) * 64 + lane];
    }
  }

  // ---- epilogue.  32x32 accumulator layout: lane l, register r holds
  // row (r/4)*8 + (l/32)*4 + r%4, column l%32 of the 32x32 block.  Each block
  // passes through a wave-private LDS buffer, after which every lane owns EW
  // consecutive columns of one row (4 for float32 results, 8 for bfloat16):
  // the outputs and the operands the epilogue reads (bias, residual,
  // pre-activation, optimizer state) move in 16-byte accesses, consecutive
  // lanes covering a row's columns contiguously.  LDS requests of one wave
  // are served in order, so the reads see the wave's own writes without a
  // barrier.
  constexpr int EW = (SPLIT || EPI == EPI_F32 || EPI == EPI_UPDATE) ? 4 : 8;
  if constexpr (!AK) {
    if (rs_on) {
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const float tot = rsum[i] + __shfl_xor(rsum[i], 32, 64);  // the two k halves
        const int64_t m = m0 + wm * WM + i * 32 + lane;
        if (lane < 32 && m < P.M) {
          if (SPLIT == SPLIT_YES || (SPLIT == SPLIT_OWN && P.splits > 1))
            P.partial[(int64_t)P.splits * P.M * P.N + (int64_t)split * P.M + m] = tot;
          else P.rowsum[m] = tot;
        }
      }
    }
  }
  constexpr int LDW = 40;  // floats per staged row: rows r and r + 4 sit 32 banks apart
  static_assert(NW * 32 * LDW * 4 <= S * (A_BYTES + B_BYTES), "staging fits in the stages");
  __syncthreads();  // every wave has finished reading the stages
  float* const stg = reinterpret_cast<float*>(smem) + wave * 32 * LDW;
  const int64_t c_off = zo * P.c_outer + zi * P.c_inner;
  uintptr_t ptrs = (uintptr_t)P.C | (uintptr_t)P.C2 | (uintptr_t)P.aux | (uintptr_t)P.bias |
                   (uintptr_t)P.partial;
  if (EPI == EPI_UPDATE)
    ptrs |= (uintptr_t)P.upd.p | (uintptr_t)P.upd.m | (uintptr_t)P.upd.v | (uintptr_t)P.upd.q |
            ((uintptr_t)P.upd.p16 << 1);
  const bool vec = (ptrs & 15) == 0 && ((P.ldc | P.c_outer | P.c_inner | P.N) & 7) == 0;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        stg[((r >> 2) * 8 + (lane >> 5) * 4 + (r & 3)) * LDW + (lane & 31)] = acc[i][j][r];
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int it = 0; it < 16 / EW; ++it) {
        const int item = lane + 64 * it;  // row item/(32/EW), columns (item%(32/EW))*EW .. +EW-1
        const int rr = item / (32 / EW), cc = (item % (32 / EW)) * EW;
        float v[EW];
#pragma unroll
        for (int q = 0; q < EW / 4; ++q) {
          const f32x4 x4 = *reinterpret_cast<const f32x4*>(stg + rr * LDW + cc + 4 * q);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[4 * q + e] = x4[e];
        }
        const int64_t m = m0 + wm * WM + i * 32 + rr;
        const int64_t n = n0 + wn * WN + j * 32 + cc;
        if (m < P.M && n < P.N)
          epi_store<EPI, SPLIT, EW>(P, split, c_off, m, n, v, vec && n + EW <= P.N);
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
}

// The logical work item of a hardware workgroup.  The grid is one dimension
// of n work items, padded to a multiple of 8.  Workgroups are dealt round-robin
// over the 8 XCDs (each with its own L2), so hardware id h runs on XCD h % 8:
// the remap gives every XCD a contiguous range of logical ids, i.e. whole
// bands of tiles of one batch/split that share operand rows.
__device__ __forceinline__ int work_item(int n, int h) {
  return (h & 7) * ((n + 7) >> 3) + (h >> 3);
}

// OCC: workgroups per CU.
template <int BM, int BN, int WGM, int WGN, int STAGES, int OCC, bool AK, bool BKM, int EPI, int SPLIT, int BKV,
          bool FL>
__global__ __launch_bounds__(64 * WGM * WGN, FL ? OCC * WGM * WGN / 4 : OCC) void gemm_bf16_kernel(const KArgs P) {
  const int n = P.tiles_m * P.tiles_n * (SPLIT ? P.splits : P.nz);
  const int lid = work_item(n, blockIdx.x);
  if (lid >= n) return;
  gemm_item<BM, BN, WGM, WGN, STAGES, AK, BKM, EPI, SPLIT, BKV, FL>(P, lid);
}

// Several products dW = dY^T X in one launch (GemmGroup): the work items of
// all of them numbered one product after the other, the products without a
// split of K first.  Their items and the others, shorter ones are dealt to the
// XCDs each by themselves, the longer first.
constexpr int MAX_GROUP = GEMM_GROUP_MAX;
struct GroupArgs {
  int32_t n, n_whole;             // products; those without a split
  int32_t first[MAX_GROUP + 1];   // first work item of each product
  int32_t rfirst[MAX_GROUP + 1];  // first workgroup of each product's split-K sum
  int32_t n_ln, ln_blocks;        // LayerNorm gradient sums riding along: blocks of each
  LnSum ln[2];
  KArgs p[MAX_GROUP];
};

template <int BM, int BN, int WGM, int WGN, int STAGES, int OCC, int EPI, int BKV>
__global__ __launch_bounds__(64 * WGM * WGN, OCC * WGM * WGN / 4) void gemm_bf16_group_kernel(const GroupArgs G) {
  const int n = G.first[G.n], n1 = G.first[G.n_whole];
  const int g1 = (n1 + 7) / 8 * 8, ng = g1 + (n - n1 + 7) / 8 * 8;
  const int h = blockIdx.x;
  if (h >= ng) {
    // the LayerNorm sums follow the products: they run on the CUs the last round leaves free
    constexpr int NT = 64 * WGM * WGN;
    static_assert(NT % LN_SUM_THREADS == 0, "whole teams of the LayerNorm sum");
    __shared__ f32x4 red[NT];
    const int b = h - ng, sub = (int)threadIdx.x / LN_SUM_THREADS;
    ln_sum_item(G.ln[b / G.ln_blocks], (b % G.ln_blocks) * (NT / LN_SUM_THREADS) + sub,
                (int)threadIdx.x % LN_SUM_THREADS, red + sub * LN_SUM_THREADS);
    return;
  }
  const int lid = h < g1 ? work_item(n1, h) : n1 + work_item(n - n1, h - g1);
  if (lid >= (h < g1 ? n1 : n)) return;
  int i = 0;
  while (i + 1 < G.n && lid >= G.first[i + 1]) ++i;
  gemm_item<BM, BN, WGM, WGN, STAGES, false, false, EPI, SPLIT_OWN, BKV, BM * BN <= 256 * 128>(G.p[i],
                                                                                              lid - G.first[i]);
}

// Sum over the splits, in split order, of the partials of four consecutive
// columns (ne of them valid; one 128-bit load per split when vec).  The
// loads of up to eight splits are issued before the first add, so a thread
// waits one memory round trip per eight splits instead of one per split;
// the additions keep the order p0 + p1 + ... of a plain loop.
__device__ __forceinline__ f32x4 sum_partials4(const float* src, int64_t total, int splits, int ne, bool vec) {
  f32x4 v{0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < splits; s0 += 8) {
    f32x4 t[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (s0 + k < splits) {
        const float* p = src + (int64_t)(s0 + k) * total;
        if (vec) {
          t[k] = *reinterpret_cast<const f32x4*>(p);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) t[k][e] = e < ne ? p[e] : 0.f;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (s0 + k < splits) v = s0 + k == 0 ? t[k] : v + t[k];
  }
  return v;
}

// Fixed-order sum of split-K partials plus the epilogue: float32 output
// (bias, residual) or the fused weight update.  One thread per four
// consecutive columns of a row, threads numbered row-major over the M x N/4
// groups (no idle lanes when N is not a multiple of 1024), with 128-bit
// accesses when N and ldc are multiples of 4 and every pointer is 16-byte
// aligned.  The thread of a row's first group also sums the row-sum partials.
template <int EPI>
__device__ __forceinline__ void splitk_reduce_item(const KArgs& P, int64_t idx) {
  static_assert(EPI == EPI_F32 || EPI == EPI_UPDATE, "split-K only with the float32 or update epilogue");
  const int64_t nq = (P.N + 3) / 4;
  if (idx >= P.M * nq) return;
  const int64_t m = idx / nq;
  const int64_t n = (idx - m * nq) * 4;
  const int ne = P.N - n < 4 ? (int)(P.N - n) : 4;
  const int64_t total = P.M * P.N;
  if (P.rowsum && n == 0) {
    const float* rp = P.partial + P.splits * total + m;
    float r = 0.f;
    for (int s0 = 0; s0 < P.splits; s0 += 8) {
      float t[8];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (s0 + k < P.splits) t[k] = rp[(int64_t)(s0 + k) * P.M];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (s0 + k < P.splits) r = s0 + k == 0 ? t[k] : r + t[k];
    }
    P.rowsum[m] = r;
  }
  const float* src = P.partial + m * P.N + n;
  if (EPI == EPI_UPDATE) {
    const int64_t off = m * P.ldc + n;
    const bool vec = ((P.N | P.ldc) & 3) == 0 && ((uintptr_t)P.partial & 15) == 0 &&
                     (((uintptr_t)P.upd.p | (uintptr_t)P.upd.m | (uintptr_t)P.upd.v | (uintptr_t)P.upd.q) & 15) == 0 &&
                     ((uintptr_t)P.upd.p16 & 7) == 0;
    const f32x4 v = sum_partials4(src, total, P.splits, ne, vec);
    if (vec) {
      apply_update4(P.upd, off, v);
    } else {
      for (int e = 0; e < ne; ++e) apply_update(P.upd, off + e, v[e]);
    }
    return;
  }
  float* dst = reinterpret_cast<float*>(P.C) + m * P.ldc + n;
  const float* aux = P.aux ? reinterpret_cast<const float*>(P.aux) + m * P.ldc + n : nullptr;
  const bool vec = ((P.N | P.ldc) & 3) == 0 &&
                   (((uintptr_t)P.C | (uintptr_t)P.aux | (uintptr_t)P.bias | (uintptr_t)P.partial) & 15) == 0;
  f32x4 v = sum_partials4(src, total, P.splits, ne, vec);
  if (vec) {
    if (P.bias) v += *reinterpret_cast<const f32x4*>(P.bias + n);
    if (aux) v += *reinterpret_cast<const f32x4*>(aux);
    *reinterpret_cast<f32x4*>(dst) = v;
  } else {
    for (int e = 0; e < ne; ++e) {
      float o = v[e];
      if (P.bias) o += P.bias[n + e];
      if (aux) o += aux[e];
      dst[e] = o;
    }
  }
}

__global__ __launch_bounds__(256) void splitk_reduce_kernel(const KArgs P) {
  splitk_reduce_item<EPI_F32>(P, (int64_t)blockIdx.x * 256 + threadIdx.x);
}

template <int EPI>
__global__ __launch_bounds__(256) void splitk_reduce_group_kernel(const GroupArgs G) {
  const int b = blockIdx.x;
  int i = 0;
  while (i + 1 < G.n && b >= G.rfirst[i + 1]) ++i;
  splitk_reduce_item<EPI>(G.p[i], (int64_t)(b - G.rfirst[i]) * 256 + threadIdx.x);
}

template <int BM, int BN, int WGM, int WGN, int STG, int OCC, bool AK, bool BKM, int EPI, int BKV, bool FL = false>
hipError_t launch_tiles(const KArgs& P, int batch, hipStream_t s) {
  const int64_t n_log = (int64_t)P.tiles_m * P.tiles_n * (P.splits > 1 ? P.splits : batch);
  if (n_log >= (1ll << 31) - 8) return hipErrorInvalidValue;
  dim3 grid((unsigned)((n_log + 7) / 8 * 8));
  constexpr int NT = 64 * WGM * WGN;
  if constexpr (EPI == EPI_F32) {
    if (P.splits > 1) {
      gemm_bf16_kernel<BM, BN, WGM, WGN, STG, OCC, AK, BKM, EPI, SPLIT_YES, BKV, FL><<<grid, NT, 0, s>>>(P);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      const int64_t groups = P.M * cdiv(P.N, 4);
      if (groups >= (1ll << 31) * 256ll) return hipErrorInvalidValue;
      splitk_reduce_kernel<<<(unsigned)cdiv(groups, 256), 256, 0, s>>>(P);
      return hipGetLastError();
    }
  }
  gemm_bf16_kernel<BM, BN, WGM, WGN, STG, OCC, AK, BKM, EPI, SPLIT_NO, BKV, FL><<<grid, NT, 0, s>>>(P);
  return hipGetLastError();
}

// Which products can be summed in short runs (FL): float32 results, tiles
// whose two sets of accumulators fit the registers.  (128 x 128, two a CU, has
// 128 registers a thread: enough for the addresses of m-major operands only.)
constexpr int64_t ANY_RUN = 1ll << 62;
constexpr bool can_flush(int bm, int bn, bool a_kmajor) {
  return bm * bn <= 256 * 128 && !(a_kmajor && bm == 128 && bn == 128);
}

template <int BM, int BN, int WGM, int WGN, int STG, int OCC, int BKV, int EPI, bool AK, bool BKM>
hipError_t dispatch_flush(const Gemm& g, const KArgs& P, hipStream_t s) {
  const bool flush = P.run < (P.splits > 1 ? P.k_per_split : P.K);
  if constexpr (EPI == EPI_F32 && can_flush(BM, BN, AK))
    if (flush) return launch_tiles<BM, BN, WGM, WGN, STG, OCC, AK, BKM, EPI, BKV, true>(P, g.batch, s);
  if (flush) return hipErrorInvalidValue;
  return launch_tiles<BM, BN, WGM, WGN, STG, OCC, AK, BKM, EPI, BKV>(P, g.batch, s);
}

template <int BM, int BN, int WGM, int WGN, int STG, int OCC, int BKV, int EPI>
hipError_t dispatch_layout(const Gemm& g, const KArgs& P, hipStream_t s) {
  if (g.a_kmajor && g.b_kmajor)
    return dispatch_flush<BM, BN, WGM, WGN, STG, OCC, BKV, EPI, true, true>(g, P, s);
  if (g.a_kmajor && !g.b_kmajor)
    return dispatch_flush<BM, BN, WGM, WGN, STG, OCC, BKV, EPI, true, false>(g, P, s);
  if (!g.a_kmajor && !g.b_kmajor)
    return dispatch_flush<BM, BN, WGM, WGN, STG, OCC, BKV, EPI, false, false>(g, P, s);
  return hipErrorInvalidValue;  // m-major A with k-major B: no caller needs it
}

template <int BM, int BN, int WGM, int WGN, int STG, int OCC, int BKV>
hipError_t dispatch_epi(const Gemm& g, const KArgs& P, hipStream_t s) {
  switch (g.epi) {
    case EPI_F32: return dispatch_layout<BM, BN, WGM, WGN, STG, OCC, BKV, EPI_F32>(g, P, s);
    case EPI_BF16: return dispatch_layout<BM, BN, WGM, WGN, STG, OCC, BKV, EPI_BF16>(g, P, s);
    case EPI_GELU:  // forward products
      if (!g.a_kmajor || !g.b_kmajor) return hipErrorInvalidValue;
      return launch_tiles<BM, BN, WGM, WGN, STG, OCC, true, true, EPI_GELU, BKV>(P, g.batch, s);
    case EPI_DGELU:  // dX products
      if (!g.a_kmajor || g.b_kmajor) return hipErrorInvalidValue;
      return launch_tiles<BM, BN, WGM, WGN, STG, OCC, true, false, EPI_DGELU, BKV>(P, g.batch, s);
    default: return hipErrorInvalidValue;  // the weight update: group launches only
  }
}

KArgs make_args(const Gemm& g) {
  KArgs P;
  memset(&P, 0, sizeof(P));
  P.A = (const bf16_t*)g.A;
  P.B = (const bf16_t*)g.B;
  P.C = g.C;
  P.C2 = g.C2;
  P.aux = g.aux;
  P.bias = g.bias;
  P.M = g.M;
  P.N = g.N;
  P.K = g.K;
  P.lda = g.lda;
  P.ldb = g.ldb;
  P.ldc = g.ldc;
  P.a_outer = g.a_outer;
  P.a_inner = g.a_inner;
  P.b_outer = g.b_outer;
  P.b_inner = g.b_inner;
  P.c_outer = g.c_outer;
  P.c_inner = g.c_inner;
  P.inner = g.inner;
  P.splits = 1;
  P.causal = g.causal;
  P.nz = g.batch;
  P.upd = g.upd;
  P.rowsum = g.rowsum;
  P.run = ANY_RUN;
  return P;
}

}  // namespace

std::string gemm_check(const Gemm& g, bool f32_operands) {
  if (g.M < 0 || g.N < 0 || g.K < 0) return "negative GEMM dimension";
  if (!f32_operands && !g.a_kmajor && g.b_kmajor) return "m-major A with k-major B is not supported";
  if (g.batch < 1 || g.inner < 1) return "batch and inner must be >= 1";
  // an operand is needed only when it is read (A: M, K > 0; B: N, K > 0) or
  // written (C: M, N > 0); with K = 0 the result is the bias (or zero)
  const bool reads = g.K > 0;
  if ((reads && g.M > 0 && !g.A) || (reads && g.N > 0 && !g.B) ||
      (g.M > 0 && g.N > 0 && !g.C && g.epi != EPI_UPDATE))
    return "null GEMM operand";
  if (g.epi == EPI_UPDATE) {
    if (!g.upd.p || !g.upd.m || !g.upd.q || (g.upd.adamw && !g.upd.v)) return "update epilogue needs p, m, (v) and q";
    if (g.a_kmajor || g.b_kmajor || g.batch != 1) return "update epilogue only for dW = dY^T X";
  }
  if (g.rowsum && (g.a_kmajor || g.batch != 1)) return "row sums of A only for an m-major A, batch 1";
  if (g.epi == EPI_GELU && !g.C2) return "GELU epilogue needs a second output";
  if (g.epi == EPI_DGELU && !g.aux) return "GELU-backward epilogue needs the pre-activation";
  const int64_t a_contig0 = g.a_kmajor ? g.K : g.M;
  const int64_t b_contig0 = g.b_kmajor ? g.K : g.N;
  if (g.lda < a_contig0 || g.ldb < b_contig0 || g.ldc < g.N) return "leading dimension smaller than the row";
  if (f32_operands) return "";  // scalar loads: no alignment rules
  const int64_t q = 8;
  // contiguous dimension of each operand and all leading dims multiples of 8
  const int64_t a_contig = g.a_kmajor ? g.K : g.M;
  const int64_t b_contig = g.b_kmajor ? g.K : g.N;
  if (a_contig % q || b_contig % q) return "contiguous GEMM dimensions must be multiples of 8 (bf16)";
  if (g.lda % q || g.ldb % q) return "leading dimensions of A and B must be multiples of 8 (bf16)";
  if (((uintptr_t)g.A | (uintptr_t)g.B) & 15) return "A and B must be 16-byte aligned";
  if ((g.a_outer | g.a_inner | g.b_outer | g.b_inner) % q) return "batch strides must keep 16-byte alignment";
  return "";
}

// Tile configurations.  Larger tiles read fewer operand bytes per FLOP,
// smaller ones fill the chip and overlap one workgroup's epilogue with
// another's products.  step: us per 64 k of a workgroup, alone on a quarter
// of the CUs or fewer (lo) and with every CU's slots full (hi); fix: us
// besides (first copies, epilogue arithmetic, launch).  Measured on the
// linear layers of the GPT-2-small, GPT-2-medium and 1.3B stacks with random
// operands from HBM.
struct TileCfg {
  int bm, bn, occ;
  float step_lo, step_hi, fix;
  float dw;  // steps of dW = dY^T X (both operands m-major, twice the LDS reads) take this much longer
  float fl;  // and those in short runs (FL)
};
enum TileId { T256x256 = 0, T256x192, T256x128, T128x192, T128x128, T128x64, T64x64, kNumCfg };
static const TileCfg kCfgs[kNumCfg] = {
    {256, 256, 1, 1.30f, 1.75f, 3.0f, 1.12f, 1.00f},  // 2x4 waves (each 128x64), 2 stages of K 64
    {256, 192, 1, 1.25f, 1.55f, 3.0f, 1.12f, 1.00f},  // 4x2 waves (each 64x96),  2 stages of K 64
    {256, 128, 1, 0.85f, 1.10f, 3.0f, 1.05f, 1.02f},  // 4x2 waves (each 64x64),  3 stages of K 64
    {128, 192, 1, 0.70f, 0.90f, 3.0f, 1.12f, 1.03f},  // 4x2 waves (each 32x96),  3 stages of K 64
    {128, 128, 2, 0.70f, 1.15f, 3.0f, 1.12f, 1.02f},  // 2x4 waves (each 64x32),  2 stages of K 64
    {128, 64, 3, 0.41f, 1.10f, 2.5f, 1.12f, 1.10f},   // 2x2 waves (each 64x32),  4 stages of K 32
    {64, 64, 4, 0.38f, 0.72f, 2.0f, 1.12f, 1.15f},    // 2x2 waves (each 32x32),  2 stages of K 64
};

namespace {
template <int BM, int BN, int WGM, int WGN, int STG, int OCC, int BKV, int EPI>
hipError_t launch_group_epi(const GroupArgs& G0, hipStream_t s) {
  constexpr int NT = 64 * WGM * WGN;
  GroupArgs G = G0;
  if (G.n_ln) G.ln_blocks = (int)cdiv(ln_sum_teams(G.ln[0].d), NT / LN_SUM_THREADS);
  const int n1 = G.first[G.n_whole], n2 = G.first[G.n] - n1;
  const dim3 grid((unsigned)((n1 + 7) / 8 * 8 + (n2 + 7) / 8 * 8 + G.n_ln * G.ln_blocks));
  gemm_bf16_group_kernel<BM, BN, WGM, WGN, STG, OCC, EPI, BKV><<<grid, NT, 0, s>>>(G);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || G.rfirst[G.n] == 0) return e;
  splitk_reduce_group_kernel<EPI><<<(unsigned)G.rfirst[G.n], 256, 0, s>>>(G);
  return hipGetLastError();
}

template <int BM, int BN, int WGM, int WGN, int STG, int OCC, int BKV>
hipError_t launch_group(const GroupArgs& G, int epi, hipStream_t s) {
  return epi == EPI_UPDATE ? launch_group_epi<BM, BN, WGM, WGN, STG, OCC, BKV, EPI_UPDATE>(G, s)
                           : launch_group_epi<BM, BN, WGM, WGN, STG, OCC, BKV, EPI_F32>(G, s);
}
}  // namespace

// The longest run of products that one accumulator of a float32 result may
// take.  Splitting K to fill the chip (at least 512 k each, at most 8 splits,
// two 128 x 128 tiles a CU) also shortens the runs, and with them the rounding
// error of a gradient; a plan that fills the chip without the split, by a
// smaller tile or by grouping products, keeps the sums as accurate by the
// FL form.  No limit where K would not be split: enough tiles, a
// short K, forward products, too little workspace.
static int64_t run_limit(const Gemm& g) {
  auto tiles = [&](int t) { return cdiv(g.M, t) * cdiv(g.N, t); };
  if ((g.epi != EPI_F32 && g.epi != EPI_UPDATE) || g.batch != 1 || !g.splitk_ws || g.K < 1536 || g.M > 65535 ||
      g.N <= 64 || (g.M >= 2048 && g.N >= 2048 && tiles(256) >= 256))
    return ANY_RUN;
  int64_t splits = 8;
  if (!g.a_kmajor || g.K < 16384) {
    if (g.b_kmajor || tiles(128) > 256) return ANY_RUN;
    splits = std::min<int64_t>(512 / tiles(128), std::min<int64_t>(8, g.K / 512));
  }
  splits = std::min<int64_t>(splits, g.splitk_ws_bytes / ((g.M * g.N + (g.rowsum ? g.M : 0)) * 4));
  return splits < 2 ? ANY_RUN : cdiv(cdiv(g.K, splits), 32) * 32;
}

// Splits of K that keep a product within its limit, and the workspace of split
// products: partial sums and row sums, each product's 256-byte aligned.
static int own_splits(const Gemm& g) {
  const int64_t limit = run_limit(g);
  return limit < g.K ? (int)cdiv(g.K, limit) : 1;
}
static size_t product_bytes(const Gemm& g, int splits) {
  return (((size_t)g.M * g.N + (g.rowsum ? g.M : 0)) * 4 * splits + 255) / 256 * 256;
}
// splits = 0: each product's own
static size_t group_bytes(const Gemm* g, int n, int splits) {
  size_t b = 0;
  for (int i = 0; i < n; ++i) {
    const int sp = splits ? splits : own_splits(g[i]);
    if (sp > 1) b += product_bytes(g[i], sp);
  }
  return b;
}

// The products share K, the epilogue (float32 or the weight update) and the
// split-K workspace, which has room for `splits` of each product; splits = 0:
// each as many as its run limit asks for.
hipError_t launch_gemm_bf16_group_cfg(const Gemm* g, int n, const LnSum* ln, int n_ln, int cfg, int splits,
                                      hipStream_t s) {
  if (n_ln < 0 || n_ln > 2 || (n_ln == 2 && ln[0].d != ln[1].d)) return hipErrorInvalidValue;
  if (n < 1 || n > MAX_GROUP || cfg < 0 || cfg >= kNumCfg) return hipErrorInvalidValue;
  GroupArgs G;
  memset(&G, 0, sizeof(G));
  G.n = n;
  G.n_ln = n_ln;
  for (int i = 0; i < n_ln; ++i) G.ln[i] = ln[i];
  const int BM = kCfgs[cfg].bm, BN = kCfgs[cfg].bn;
  const int64_t K = g[0].K;
  for (int i = 0; i < n; ++i)
    if (g[i].K != K || g[i].epi != g[0].epi || g[i].a_kmajor || g[i].b_kmajor || g[i].batch != 1 || g[i].M < 1 ||
        g[i].N < 1 || (g[i].epi != EPI_F32 && g[i].epi != EPI_UPDATE))
      return hipErrorInvalidValue;
  const size_t room = g[0].splitk_ws ? g[0].splitk_ws_bytes : 0;
  while (splits > 1 && group_bytes(g, n, splits) > room) --splits;
  char* part = (char*)g[0].splitk_ws;
  int64_t items = 0, rblocks = 0;
  int at = 0;
  for (int pass = 0; pass < 2; ++pass) {  // whole products, then split ones
    for (int i = 0; i < n; ++i) {
      const int sp = splits ? splits : own_splits(g[i]);
      if ((sp > 1) != (pass == 1)) continue;
      KArgs& P = G.p[at];
      P = make_args(g[i]);
      P.tiles_m = (int)cdiv(P.M, BM);
      P.tiles_n = (int)cdiv(P.N, BN);
      P.run = run_limit(g[i]);
      P.k_per_split = K;
      if (sp > 1) {
        P.k_per_split = cdiv(cdiv(K, sp), 32) * 32;
        P.splits = (int)cdiv(K, P.k_per_split);
        P.partial = (float*)part;
        part += product_bytes(g[i], P.splits);
        if (part > (char*)g[0].splitk_ws + room) return hipErrorInvalidValue;
      }
      G.first[at] = (int)items;
      G.rfirst[at] = (int)rblocks;
      items += (int64_t)P.tiles_m * P.tiles_n * P.splits;
      if (P.splits > 1) rblocks += cdiv(P.M * cdiv(P.N, 4), 256);
      if (items >= (1ll << 31) - 16 || rblocks >= (1ll << 31)) return hipErrorInvalidValue;
      ++at;
    }
    if (pass == 0) G.n_whole = at;
  }
  G.first[n] = (int)items;
  G.rfirst[n] = (int)rblocks;
  switch (cfg) {
    case T256x256: return launch_group<256, 256, 2, 4, 2, 1, 64>(G, g[0].epi, s);
    case T256x128: return launch_group<256, 128, 4, 2, 3, 1, 64>(G, g[0].epi, s);
    case T128x128: return launch_group<128, 128, 2, 4, 2, 2, 64>(G, g[0].epi, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_gemm_bf16_cfg(const Gemm& g, int cfg, int splits, int64_t run, hipStream_t s) {
  if (g.M == 0 || g.N == 0) return hipSuccess;
  if (cfg < 0 || cfg >= kNumCfg) return hipErrorInvalidValue;
  KArgs P = make_args(g);
  const int BM = kCfgs[cfg].bm, BN = kCfgs[cfg].bn;
  P.tiles_m = (int)cdiv(g.M, BM);
  P.tiles_n = (int)cdiv(g.N, BN);
  if (splits > 1 && g.batch == 1 && g.splitk_ws && g.epi == EPI_F32 && g.M <= 65535) {
    const size_t per_split = (size_t)g.M * g.N * 4 + (g.rowsum ? (size_t)g.M * 4 : 0);
    while (splits > 1 && splits * per_split > g.splitk_ws_bytes) --splits;
    if (splits > 1) {
      P.k_per_split = cdiv(cdiv(g.K, splits), 32) * 32;
      P.splits = (int)cdiv(g.K, P.k_per_split);
      P.partial = g.splitk_ws;
    }
  }
  P.run = run;
  switch (cfg) {
    case T256x256: return dispatch_epi<256, 256, 2, 4, 2, 1, 64>(g, P, s);
    case T256x192: return dispatch_epi<256, 192, 4, 2, 2, 1, 64>(g, P, s);
    case T256x128: return dispatch_epi<256, 128, 4, 2, 3, 1, 64>(g, P, s);
    case T128x192: return dispatch_epi<128, 192, 4, 2, 3, 1, 64>(g, P, s);
    case T128x128: return dispatch_epi<128, 128, 2, 4, 2, 2, 64>(g, P, s);
    case T128x64: return dispatch_epi<128, 64, 2, 2, 4, 3, 32>(g, P, s);
    default: return dispatch_epi<64, 64, 2, 2, 2, 4, 64>(g, P, s);
  }
}

// Estimated time (us) of `items` work items of `steps` K steps of 64 each on
// one tile configuration, with `bytes` of epilogue traffic per output
// element: whole rounds of the chip's slots, then a last round whose steps
// and epilogue are faster the emptier it is.
static float est_items(const TileCfg& t, int64_t items, float steps, float bytes) {
  const int64_t slots = 256 * (int64_t)t.occ;
  // 25 KB/us of epilogue traffic per CU with all CUs writing (6.4 TB/s);
  // workgroups that share a CU hide part of it behind the next round's products
  const float epi = bytes * t.bm * t.bn * t.occ / 25e3f;
  const float round = steps * t.step_hi + t.fix + epi * (t.occ > 1 ? 0.6f : 1.0f);
  const int64_t full = (items - 1) / slots, rest = items - full * slots;  // rest: the last round, 1..slots
  float us = full * round;
  if (rest > 0) {
    // the last round takes as long as its fullest CU (one workgroup per CU:
    // the operand stream slows with the share of CUs that are busy)
    const float f = t.occ > 1 ? (float)(cdiv(rest, 256) - 1) / (float)(t.occ - 1) : (float)rest / slots;
    us += steps * (t.step_lo + (t.step_hi - t.step_lo) * f) + t.fix + epi * (float)rest / slots;
  }
  return us;
}

// Tile and split of K for a product or a group of products with the same K:
// the smallest estimate over the configurations and splits, the split's
// partial sums written and read back at 4.5 TB/s by a second launch (8 us).
// A split leaves at least 512 k each, at most 8 of them.  A tile that would
// exceed the run limit takes its FL form or is left out.  (Over 568 products of
// 64 to 8192 a side that have a limit, the plan takes 0.96 of the time of the
// plan without one, 1.06 at the 90th percentile, 1.27 at most.)
// beside: the launch shares the chip with another stream's kernels, and what it
// takes from them counts besides its own time: tiles of several workgroups a CU
// leave them no CU, nor do many workgroups, and a split adds work.  Where there is
// a limit, these count a tenth more: the GPT-2-small step takes 11.65 ms with 128 x 128 and
// 11.42 with 256 x 128, four blocks of GPT-2-medium's width 7.85 ms with 128 x
// 128, 7.87 with 256 x 128 and K split in two, and 7.73 with 256 x 128.
struct Plan {
  int cfg = T128x128, splits = 1;  // 0: each product of a group its own split
  int64_t run = ANY_RUN;
  float us = 3.4e38f;
};
static Plan choose(const Gemm* g, int n, bool group, bool beside, int only_split = -1) {
  const bool splittable = g[0].batch == 1 && (g[0].epi == EPI_F32 || g[0].epi == EPI_UPDATE) && g[0].splitk_ws;
  double outputs = 0.0;
  size_t per_split = 0;
  int64_t limit = ANY_RUN;
  for (int i = 0; i < n; ++i) {
    outputs += (double)g[i].M * g[i].N;
    per_split += ((size_t)g[i].M * g[i].N + (g[i].rowsum ? g[i].M : 0)) * 4 + 256;
    limit = std::min(limit, run_limit(g[i]));
  }
  float bytes = g[0].epi == EPI_F32 ? 4.f : g[0].epi == EPI_BF16 ? 2.f : g[0].epi == EPI_UPDATE ? 30.f : 4.f;
  if (g[0].epi == EPI_F32 && g[0].aux) bytes += 4.f;
  const int64_t max_split = splittable ? std::min<int64_t>(8, g[0].K / 512) : 1;
  // a single product that has a limit is split more often than not: 5 us and
  // 6 TB/s are what its sums cost on average (over the 568 products above)
  const bool tight = !group && limit < g[0].K;
  const float sum_fix = tight ? 5.f : 8.f, sum_rate = tight ? 6e6f : 4.5e6f;
  Plan best;
  auto tiles_of = [&](const TileCfg& t) {
    int64_t tiles = 0;
    for (int i = 0; i < n; ++i) tiles += cdiv(g[i].M, t.bm) * cdiv(g[i].N, t.bn) * g[i].batch;
    return tiles;
  };
  auto consider = [&](int c, int sp, int64_t items, float us) {
    if (beside && limit < g[0].K && (kCfgs[c].occ > 1 || sp != 1 || items > 384)) us *= 1.1f;
    if (us < best.us) best = Plan{c, sp, limit, us};
  };
  for (int c = 0; c < kNumCfg; ++c) {
    if (group && c != T256x256 && c != T256x128 && c != T128x128) continue;
    const TileCfg& t = kCfgs[c];
    const int64_t tiles = tiles_of(t);
    for (int sp = 1; sp <= std::max<int64_t>(1, max_split); ++sp) {
      if (sp > 1 && (sp * per_split > g[0].splitk_ws_bytes || g[0].M > 65535)) break;
      if (only_split >= 0 && sp != only_split) continue;
      const int64_t run = sp > 1 ? cdiv(cdiv(g[0].K, sp), 32) * 32 : g[0].K;
      const bool flush = run > limit;
      if (flush && !can_flush(t.bm, t.bn, g[0].a_kmajor)) continue;
      const float steps = (float)cdiv(cdiv(g[0].K, sp), 64) * (g[0].a_kmajor ? 1.0f : t.dw) * (flush ? t.fl : 1.0f);
      float us = est_items(t, tiles * sp, steps, sp > 1 ? 4.f : bytes);
      if (sp > 1) us += sum_fix + (float)(outputs * (4.0 * sp + bytes) / sum_rate);
      consider(c, sp, tiles * sp, us);
    }
  }
  // 256 x 256 with only the limited products of the group split, as far as
  // their limits ask for: the attention projection alone from about 1100
  // features on
  if (group && limit < g[0].K && only_split <= 0 && group_bytes(g, n, 0) <= g[0].splitk_ws_bytes) {
    const TileCfg& t = kCfgs[T256x256];
    const int64_t tiles = tiles_of(t);
    float us = est_items(t, tiles, (float)cdiv(g[0].K, 64) * t.dw, bytes) + 8.f;
    for (int i = 0; i < n; ++i) {
      const int sp = own_splits(g[i]);
      if (sp > 1) us += (float)((double)g[i].M * g[i].N * (8.0 * sp + bytes) / 4.5e6);
    }
    consider(T256x256, 0, tiles, us);
  }
  return best;
}

hipError_t launch_gemm_bf16_group(const Gemm* g, int n, const LnSum* ln, int n_ln, bool beside, hipStream_t s) {
  // The split of K and the run limit fix the order of the sums, the tile does
  // not: with the split chosen as for the launch beside another stream, the
  // results are the same bit for bit on one stream and on two.
  Plan p = choose(g, n, true, true);
  if (!beside) p = choose(g, n, true, false, p.splits);
  return launch_gemm_bf16_group_cfg(g, n, ln, n_ln, p.cfg, p.splits, s);
}

hipError_t launch_gemm_bf16(const Gemm& g, hipStream_t s) {
  if (g.M == 0 || g.N == 0) return hipSuccess;
  const Plan p = choose(&g, 1, false, false);
  return launch_gemm_bf16_cfg(g, p.cfg, p.splits, p.run, s);
}

namespace {
__global__ __launch_bounds__(256) void gelu_test_kernel(const float* x, float* y, float* dy, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  y[i] = gelu_tanh_f(x[i]);
  dy[i] = gelu_tanh_grad_f(x[i]);
}
}  // namespace

}  // namespace layup

extern "C" int layup_test_gelu(const float* x, float* y, float* dy, int64_t n, void* stream) {
  if (!x || !y || !dy || n < 1 || n > (1ll << 31)) return LAYUP_ERR_INVALID_ARG;
  layup::gelu_test_kernel<<<(unsigned)cdiv(n, 256), 256, 0, (hipStream_t)stream>>>(x, y, dy, n);
  return hipGetLastError() == hipSuccess ? LAYUP_OK : LAYUP_ERR_HIP;
}

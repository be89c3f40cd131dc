// GEMM for products with few output tiles (bf16): C(m,n) = sum_k A(m,k) B(n,k), A k-contiguous, B either way.
// The step's products at small batches, and the head's and the top layer's on the predicted rows only, give the
// 128- and 256-wide kernels 3 to 100 workgroups for 256 compute units, each with a serial chain of k tiles behind it.
//
// Here a workgroup owns a TM x TN tile of C (32x32 or 64x64) and its W wavefronts split the contraction among them:
// wavefront w multiplies the 64-wide k groups w, w + W, ... of the whole tile into accumulators of its own, and the W
// partial tiles are added in order of w in LDS before the shared epilogue.  So a long contraction is a short chain in
// every wavefront, with no second launch and no partial sums in memory.  A k group of a row is one 128-byte cache line,
// loaded by eight lanes (fragments loaded straight into registers, half a line per row, took 13.3 instead of 8.4 us at
// 128x768x3072: the vector memory path is what bounds this kernel); D groups are in flight per wavefront in registers.
// They pass through a patch of LDS that only their own wavefront uses, so there is no barrier in the k loop:
// k-contiguous operands as [rows][64 k] with the 16-byte chunks XOR-swizzled by the row, a k-strided B (the weight in dX = dY W) as [64 k][TN],
// read back through the transposing read (sixteen lanes that fetch four consecutive n of four k receive four
// consecutive k of one n).
// The product is formed transposed (n in the accumulator's row index), so a lane holds four consecutive columns.
//
// Tiles are numbered down a column of tiles first and the numbers handed out in contiguous ranges, one per XCD, so
// that each XCD reads its own part of the weights and the few rows of A.
// Whole steps: BERT-Base 9 frozen + 3 trainable layers 1x128 2144 -> 1195 us (25 products of three workgroups took 817),
// with the next-sentence head and dropout 64x128 4.21 -> 4.15 ms, 128-wide model 4x64 458 -> 410 us.
#include "common.h"
#include "gemm_epilogue.h"

namespace mslt {

namespace few {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

struct Params {
  const bf16 *A, *B;
  int M, N, K, lda, ldb, tiles_m, tiles_n;
  Epilogue epi;
};

// RAGGED: M is no multiple of TM.  (The clamped row addresses cost 1.5 to 2 us of 13 at 512x1024x1024, so whole tiles keep
// theirs: one offset a lane, everything else uniform.)
template <int TM, int TN, int W, int D, bool B_KC, bool RAGGED>
__global__ void __launch_bounds__(64 * W, 2) k_gemm_few(Params p) {
  constexpr int RM = TM / 16, RN = TN / 16;
  constexpr int LDR = TN + 4;                       // floats per row of a partial tile
  constexpr int LDB = TN + 8;                       // bf16 per k row of a k-strided B patch
  constexpr int PATCH_A = TM * 128, PATCH = PATCH_A + (B_KC ? TN * 128 : 64 * LDB * 2);   // bytes
  constexpr int LDS = W * TM * LDR * 4 > W * PATCH ? W * TM * LDR * 4 : W * PATCH;
  constexpr int NA = TM / 8, NB = TN / 8;           // 16-byte chunks per lane and group
  __shared__ __attribute__((aligned(16))) unsigned char lds[LDS];

  const int total = p.tiles_m * p.tiles_n, per = (total + 7) / 8;
  const int t = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || t >= total) return;
  const int n0 = (t / p.tiles_m) * TN, m0 = (t % p.tiles_m) * TM;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, q = lane >> 4;
  const int ngroups = p.K / 64;
  const int n = wave < ngroups ? (ngroups - wave + W - 1) / W : 0;   // this wavefront's groups: wave + W * i

  f32x4_t acc[RM][RN];
#pragma unroll
  for (int i = 0; i < RM; ++i)
#pragma unroll
    for (int j = 0; j < RN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  if (n > 0) {
    // eight lanes per 128-byte row of a k-contiguous operand; TN / 8 lanes per k row of a k-strided one
    constexpr int LB = TN / 8;
    const int lr = lane >> 3, lc = lane & 7;
    // (the lane's part of an address is one 32-bit offset, everything else of it uniform)
    // (rows past the end of A, of a last tile that is not full, repeat the last one; their results are not written)
    unsigned oa[RAGGED ? NA : 1];
#pragma unroll
    for (int a = 0; a < (RAGGED ? NA : 1); ++a) oa[a] = (unsigned)((RAGGED ? min(8 * a + lr, p.M - 1 - m0) : lr) * p.lda + 8 * lc);
    const unsigned ob = B_KC ? (unsigned)(lr * p.ldb + 8 * lc) : (unsigned)((lane / LB) * p.ldb + (lane % LB) * 8);
    const bf16* ua = p.A + (size_t)m0 * p.lda;
    const bf16* ub = B_KC ? p.B + (size_t)n0 * p.ldb : p.B + n0;
    u32x4_t fa[D][NA], fb[D][NB];
    auto load = [&](int slot, int i) {               // i-th group of this wavefront
      const int k = 64 * (wave + W * i);
#pragma unroll
      for (int a = 0; a < NA; ++a) fa[slot][a] = *reinterpret_cast<const u32x4_t*>(RAGGED ? ua + k + oa[RAGGED ? a : 0] : ua + (size_t)(8 * a) * p.lda + k + oa[0]);
#pragma unroll
      for (int b = 0; b < NB; ++b)
        fb[slot][b] = *reinterpret_cast<const u32x4_t*>((B_KC ? ub + (size_t)(8 * b) * p.ldb + k : ub + (size_t)(k + b * (64 / LB)) * p.ldb) + ob);
    };
    unsigned char *patch_a = lds + wave * PATCH, *patch_b = patch_a + PATCH_A;
    auto multiply = [&](int slot) {
#pragma unroll
      for (int a = 0; a < NA; ++a) *reinterpret_cast<u32x4_t*>(patch_a + (8 * a + lr) * 128 + ((lc ^ lr) << 4)) = fa[slot][a];
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        if constexpr (B_KC) *reinterpret_cast<u32x4_t*>(patch_b + (8 * b + lr) * 128 + ((lc ^ lr) << 4)) = fb[slot][b];
        else *reinterpret_cast<u32x4_t*>(patch_b + ((lane / LB + b * (64 / LB)) * LDB + (lane % LB) * 8) * 2) = fb[slot][b];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // LDS keeps one wavefront's order; so must the compiler
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int chunk = ((4 * h + q) ^ (r16 & 7)) << 4;
        bf16x8_t va[RM], vb[RN];
#pragma unroll
        for (int i = 0; i < RM; ++i) va[i] = *reinterpret_cast<const bf16x8_t*>(patch_a + (16 * i + r16) * 128 + chunk);
#pragma unroll
        for (int j = 0; j < RN; ++j) {
          if constexpr (B_KC) {
            vb[j] = *reinterpret_cast<const bf16x8_t*>(patch_b + (16 * j + r16) * 128 + chunk);
          } else {
            // this lane's address: k row 32 h + 8 q + r16 / 4 (the second read four rows on), n 16 j + 4 (r16 % 4)
            unsigned char* at = patch_b + ((32 * h + 8 * q + (r16 >> 2)) * LDB + 16 * j + 4 * (r16 & 3)) * 2;
            struct { s16x4_t lo, hi; } v;
            v.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)at);
            v.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(at + 4 * LDB * 2));
            vb[j] = __builtin_bit_cast(bf16x8_t, v);
          }
        }
#pragma unroll
        for (int i = 0; i < RM; ++i)
#pragma unroll
          for (int j = 0; j < RN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vb[j], va[i], acc[i][j], 0, 0, 0);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
#pragma unroll
    for (int s = 0; s < D; ++s)
      if (s < n) load(s, s);
    int g = 0;
    for (; g + 2 * D <= n; g += D) {                 // every load of this turn lies inside the range
#pragma unroll
      for (int s = 0; s < D; ++s) {
        multiply(s);
        load(s, g + s + D);
      }
    }
#pragma unroll
    for (int s = 0; s < 2 * D - 1; ++s) {            // at most 2 D - 1 groups are left, D of them on their way
      if (g + s < n) multiply(s % D);
      if (s < D - 1 && g + s + D < n) load(s, g + s + D);
    }
  }

  __syncthreads();                                   // the partial tiles lie over the patches
  float* part = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int i = 0; i < RM; ++i)
#pragma unroll
    for (int j = 0; j < RN; ++j)
      *reinterpret_cast<f32x4_t*>(part + (wave * TM + 16 * i + r16) * LDR + 16 * j + 4 * q) = acc[i][j];
  const Epilogue& e = p.epi;
  constexpr int SPANS = TM * TN / 8;                 // runs of eight columns
  constexpr int TURNS = (SPANS + 64 * W - 1) / (64 * W);
  uint4 raw[TURNS];
  if (epilogue_reads_aux(e)) {
#pragma unroll
    for (int u = 0; u < TURNS; ++u) {
      const int x = (int)threadIdx.x + u * 64 * W;
      if (x < SPANS && (!RAGGED || m0 + x / (TN / 8) < p.M)) raw[u] = load_aux8(e, m0 + x / (TN / 8), n0 + (x % (TN / 8)) * 8);
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < TURNS; ++u) {
    const int x = (int)threadIdx.x + u * 64 * W;
    if (x >= SPANS) break;
    const int row = x / (TN / 8), col = (x % (TN / 8)) * 8;
    if (RAGGED && m0 + row >= p.M) continue;
    float v[8] = {0, 0, 0, 0, 0, 0, 0, 0}, bias[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const f32x4_t a = *reinterpret_cast<const f32x4_t*>(part + (w * TM + row) * LDR + col);
      const f32x4_t b = *reinterpret_cast<const f32x4_t*>(part + (w * TM + row) * LDR + col + 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) { v[i] += a[i]; v[4 + i] += b[i]; }
    }
    if (e.bias) {
#pragma unroll
      for (int i = 0; i < 8; ++i) bias[i] = e.bias[n0 + col + i];
    }
    if (e.drop.thr || e.accumulate) epilogue8<true>(e, m0 + row, n0 + col, v, bias, raw[u]);
    else epilogue8<false>(e, m0 + row, n0 + col, v, bias, raw[u]);
  }
}

template <int TM, int TN, int W, int D>
static void launch(const GemmDesc& d, const Params& p, hipStream_t s) {
  const dim3 grid((unsigned)(((p.tiles_m * p.tiles_n + 7) / 8) * 8)), block(64 * W);
  if (d.M % TM) {
    if (d.b_kcontig) k_gemm_few<TM, TN, W, D, true, true><<<grid, block, 0, s>>>(p);
    else k_gemm_few<TM, TN, W, D, false, true><<<grid, block, 0, s>>>(p);
  } else {
    if (d.b_kcontig) k_gemm_few<TM, TN, W, D, true, false><<<grid, block, 0, s>>>(p);
    else k_gemm_few<TM, TN, W, D, false, false><<<grid, block, 0, s>>>(p);
  }
}

}  // namespace few

bool gemm_few_supported(const GemmDesc& d) { return d.a_kcontig && gemm_rows_supported(d); }

// Tile edge for a product, 0 when another kernel should take it.  The chip holds 256 workgroups of the 32-wide form and
// 512 of the 64-wide one at a time; past one such round the wide kernels' fewer bytes per FLOP win, and within it the
// small tile gives a product twice the wavefronts.  Measured, microseconds, this kernel / the best of the other two
// kernels and their split factors, k-contiguous B:
//   128x768x3072 8.4 (32-wide; 64-wide 13.7) / 13.4; 512x768x768 6.7 / 12.0; 1024x768x3072 15.1 / 21.9;
//   512x3072x768 9.0 / 12.4 and 2048x768x3072 24.8 / 25.1, 384 workgroups; 2048x1024x1024 11.6 / 14.7, 512;
//   past one round 1024x2304x768 12.7 / 12.6, 1536x2304x768 15.8 / 13.1.
// At the longest contractions a layer has, this kernel / what the step would take instead: forward (never split over
// workgroups) 2048x1024x4096, 512 tiles, 33.2 / 40.0, 1024x1024x4096 19.7 / 39.8; the data gradient, which may be split, one
// workgroup per compute unit 1024x1024x4096 20.5 / 24.4 and 1024x768x3072 16.8 / 20.7, but with two, from K = 3072 on, about
// even: 1536x768x3072 22.3 / 21.0, 2688x768x3072 27.7 / 26.5, 1280x1024x4096 28.0 / 24.9, 2048x1024x4096 33.9 / 36.8,
// 2048x1024x3072 25.5 / 31.4.  The 32-wide form meets a split by 8 near K = 8192 (data gradient 128x768: 8192 18.7 / 18.9,
// 12288 26.4 / 22.7) and the 64-wide one between 6144 and 8192 (forward 1024x1024x6144 25.6 / 28.9, 1024x768x8192 30.8 / 26.9);
// past 4096 only products over the vocabulary are that long.
// Two 64-wide workgroups on a compute unit with one group in flight beat one with two in flight: 512x3072x768 9.0
// against 13.7.  A long contraction is better split over workgroups: at 512x768x30592 the 64-wide form took 154, a
// split by 8 of the 128-wide kernel 53.
int gemm_few_edge(int rows, int N, int K) {
  const long long tiles = (long long)((rows + 63) / 64) * (N / 64);
  if (4 * tiles <= 256 && K <= 8192) return 32;
  if (tiles <= 512 && K <= 4096) return 64;
  return 0;
}
int gemm_few_tile(const GemmDesc& d, int rows) { return gemm_few_supported(d) ? gemm_few_edge(rows, d.N, d.K) : 0; }

hipError_t gemm_few(const GemmDesc& d, int tile, hipStream_t s) {
  if (!gemm_few_supported(d) || (tile != 32 && tile != 64)) return hipErrorInvalidValue;
  few::Params p{reinterpret_cast<const bf16*>(d.A), reinterpret_cast<const bf16*>(d.B), d.M, d.N, d.K, d.lda, d.ldb,
                (d.M + tile - 1) / tile, d.N / tile, d.epi};
  if (tile == 32) few::launch<32, 32, 8, 3>(d, p, s);
  else few::launch<64, 64, 4, 1>(d, p, s);
  return hipGetLastError();
}

}  // namespace mslt

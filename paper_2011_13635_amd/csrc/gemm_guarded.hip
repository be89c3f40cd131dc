// Guarded matrix-core GEMM: C(m,n) = sum_k A(m,k) B(n,k) with the shared epilogue, any shape, any leading
// dimension, fp32 accumulation.  It takes the fp32 products that gemm_f32.hip does not (v_mfma_f32_32x32x2_f32) and the bf16
// products whose sizes the 128-wide kernels do not fit (v_mfma_f32_32x32x16_bf16: next-sentence head, hidden
// sizes that are no multiple of 128).
//
// A 256-thread workgroup owns a 64x64 tile of C, each wavefront a 32x32 block.  The fp32 matrix instruction does
// 256 FLOP per clock and compute unit, so a 64x64 tile needs 16 bytes of operands per clock, a quarter of what L2
// delivers: a larger tile would buy nothing and leave compute units idle at the row counts fp32 mode is used with.
// Slabs of 128 bytes of k per row (32 fp32 or 64 bf16) travel global -> registers -> LDS, one slab ahead, two LDS
// buffers, one barrier per slab.  In LDS an operand is [64 rows][128 bytes] with 16-byte chunks XOR-swizzled by the
// row, and a lane's fragment is one 16-byte read: 8 bf16 for one MFMA, or 4 fp32 for four, the contraction order
// inside a group of eight k being (j, 4 + j).  A k-strided fp32 operand lies as [32 k][64 rows] and is read four
// bytes at a time in the same order (the 64-cycle MFMA hides the extra reads); a k-strided bf16 operand is
// transposed on its way into LDS.  Rows and k past the end are read as zeros; whole chunks inside the matrix are
// 16-byte loads when base and leading dimension allow it.
//
// With few tiles the contraction is split (guarded_splitk) and a second kernel adds the parts in fixed order.
// What bounds it: the fp32 matrix pipes (157 TFLOP/s; a BERT-Base 3+3 layer step on 1024 rows, 171 GFLOP, spends 2.83 ms
// of launches in it: 60, the rest is the partly empty last round of workgroups and the first slab's latency).  Measured, whole step in fp32 mode
// against the kernel with 4x4 outputs per thread in vector FMAs that was here before: BERT-Base 3 frozen + 3
// trainable layers 8x128 21.4 -> 4.4 ms, 128-wide 3-layer model 11x50 2.77 -> 0.74 ms; BERT-Base with the
// next-sentence head in bf16 4.54 -> 4.16 ms (five products of 64 rows, 446 us before).
#include "common.h"
#include "gemm_epilogue.h"

namespace mslt {

namespace guarded {

constexpr int TILE = 64, SLAB_BYTES = 128, OPERAND_BYTES = TILE * SLAB_BYTES;

// One operand's slab: two 16-byte chunks per thread.
//   k-contiguous: chunk tid%8 of row tid/8 + 32 i;   k-strided: E = 16/sizeof(AT) rows of k number tid/(64/E) + i*BK/2
template <typename AT, bool KC>
struct Operand {
  static constexpr int E = 16 / (int)sizeof(AT), BK = SLAB_BYTES / (int)sizeof(AT), RG = TILE / E;
  u32x4_t v[2];
  // rows: logical rows of the matrix; vec: base and leading dimension are multiples of 16 bytes
  __device__ __forceinline__ void load(const AT* __restrict__ p, int ld, int r0, int rows, int k0, int K, int tid, bool vec) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = KC ? r0 + (tid >> 3) + 32 * i : r0 + (tid % RG) * E;
      const int k = KC ? k0 + (tid & 7) * E : k0 + tid / RG + i * (BK / 2);
      const size_t at = KC ? (size_t)r * ld + k : (size_t)k * ld + r;
      const bool whole = KC ? (r < rows && k + E <= K) : (k < K && r + E <= rows);
      if (vec && whole) {
        v[i] = *reinterpret_cast<const u32x4_t*>(p + at);
      } else {
        uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const bool in = KC ? (r < rows && k + e < K) : (k < K && r + e < rows);
          if (in) {
            if constexpr (sizeof(AT) == 4) w[e] = __float_as_uint(ldf(p + at + e));
            else w[e >> 1] |= (uint32_t)reinterpret_cast<const uint16_t*>(p)[at + e] << (16 * (e & 1));
          }
        }
        v[i] = u32x4_t{w[0], w[1], w[2], w[3]};
      }
    }
  }
  __device__ __forceinline__ void store(unsigned char* lds, int tid) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if constexpr (KC) {
        const int row = (tid >> 3) + 32 * i;
        *reinterpret_cast<u32x4_t*>(lds + row * SLAB_BYTES + (((tid & 7) ^ ((row >> 1) & 7)) << 4)) = v[i];
      } else if constexpr (sizeof(AT) == 4) {
        *reinterpret_cast<u32x4_t*>(lds + ((tid / RG + i * (BK / 2)) * TILE + (tid % RG) * E) * 4) = v[i];
      } else {
        const int k = tid / RG + i * (BK / 2);
        const uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int row = (tid % RG) * E + e;
          *reinterpret_cast<uint16_t*>(lds + row * SLAB_BYTES + (((k >> 3) ^ ((row >> 1) & 7)) << 4) + (k & 7) * 2) =
              (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
        }
      }
    }
  }
  // group g (0..3) of the slab for this lane's row: eight k of fp32 or sixteen of bf16, this lane's half of them
  static __device__ __forceinline__ u32x4_t frag(const unsigned char* lds, int row, int g, int half) {
    if constexpr (KC || sizeof(AT) == 2) {
      return *reinterpret_cast<const u32x4_t*>(lds + row * SLAB_BYTES + (((2 * g + half) ^ ((row >> 1) & 7)) << 4));
    } else {
      const uint32_t* q = reinterpret_cast<const uint32_t*>(lds) + (8 * g + 4 * half) * TILE + row;
      return u32x4_t{q[0], q[TILE], q[2 * TILE], q[3 * TILE]};
    }
  }
};

template <typename AT, bool A_KC, bool B_KC>
__global__ void __launch_bounds__(256) k_gemm_guarded(GemmDesc d, int tiles_m, int tiles_n, int splitk, float* __restrict__ partials,
                                                      int vec_a, int vec_b) {
  typedef Operand<AT, A_KC> OpA;
  typedef Operand<AT, B_KC> OpB;
  constexpr int BK = OpA::BK;
  __shared__ __attribute__((aligned(16))) unsigned char lds[2][2][OPERAND_BYTES];
  const AT* A = reinterpret_cast<const AT*>(d.A);
  const AT* B = reinterpret_cast<const AT*>(d.B);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
  const int split = blockIdx.x / (tiles_m * tiles_n), tile = blockIdx.x % (tiles_m * tiles_n);
  const int m0 = (tile / tiles_n) * TILE, n0 = (tile % tiles_n) * TILE;
  const int nslab = (d.K + BK - 1) / BK;
  const int lo = (int)((long long)split * nslab / splitk), hi = (int)((long long)(split + 1) * nslab / splitk);
  const int arow = 32 * (wave >> 1) + (lane & 31), brow = 32 * (wave & 1) + (lane & 31);

  f32x16_t acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  OpA a;
  OpB b;
  a.load(A, d.lda, m0, d.M, lo * BK, d.K, tid, vec_a);
  b.load(B, d.ldb, n0, d.N, lo * BK, d.K, tid, vec_b);
  for (int s = lo; s < hi; ++s) {
    unsigned char* la = lds[s & 1][0];
    unsigned char* lb = lds[s & 1][1];
    a.store(la, tid);       // (this buffer was last read two slabs ago, behind the barrier of the slab in between)
    b.store(lb, tid);
    __syncthreads();
    if (s + 1 < hi) {
      a.load(A, d.lda, m0, d.M, (s + 1) * BK, d.K, tid, vec_a);
      b.load(B, d.ldb, n0, d.N, (s + 1) * BK, d.K, tid, vec_b);
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const u32x4_t fa = OpA::frag(la, arow, g, half), fb = OpB::frag(lb, brow, g, half);
      if constexpr (sizeof(AT) == 4) {
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(fa.x), __uint_as_float(fb.x), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(fa.y), __uint_as_float(fb.y), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(fa.z), __uint_as_float(fb.z), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(fa.w), __uint_as_float(fb.w), acc, 0, 0, 0);
      } else {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, fa), __builtin_bit_cast(bf16x8_t, fb), acc, 0, 0, 0);
      }
    }
  }

  const int n = n0 + 32 * (wave & 1) + (lane & 31);
  const int mb = m0 + 32 * (wave >> 1) + 4 * half;
  if (n >= d.N) return;
  if (splitk > 1) {
    float* out = partials + (size_t)split * d.M * d.N;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = mb + 8 * (r >> 2) + (r & 3);
      if (m < d.M) out[(size_t)m * d.N + n] = acc[r];
    }
    return;
  }
  const Epilogue& e = d.epi;
  const float bias = e.bias ? e.bias[n] : 0.f;
  float x[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = mb + 8 * (r >> 2) + (r & 3);
    x[r] = m < d.M ? load_aux<AT>(e, m, n) : 0.f;
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = mb + 8 * (r >> 2) + (r & 3);
    if (m < d.M) finish_one<AT>(e, m, n, acc[r] + bias, x[r]);
  }
}

// adds the parts in split order and applies the epilogue; one element per thread
template <typename AT>
__global__ void __launch_bounds__(256) k_guarded_reduce(const float* __restrict__ partials, int splitk, int M, int N, Epilogue e) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x, total = (size_t)M * N;
  if (i >= total) return;
  const int m = (int)(i / N), n = (int)(i % N);
  const float x = load_aux<AT>(e, m, n);
  float v = 0.f;
#pragma unroll 4
  for (int s = 0; s < splitk; ++s) v += partials[(size_t)s * total + i];
  finish_one<AT>(e, m, n, v + (e.bias ? e.bias[n] : 0.f), x);
}

template <typename AT>
static void launch(const GemmDesc& d, int splitk, float* partials, hipStream_t s) {
  const int tm = (d.M + TILE - 1) / TILE, tn = (d.N + TILE - 1) / TILE;
  constexpr int E = 16 / (int)sizeof(AT);
  const int va = d.lda % E == 0 && reinterpret_cast<uintptr_t>(d.A) % 16 == 0;
  const int vb = d.ldb % E == 0 && reinterpret_cast<uintptr_t>(d.B) % 16 == 0;
  const dim3 grid((unsigned)(tm * tn * splitk)), block(256);
  if (d.a_kcontig && d.b_kcontig) k_gemm_guarded<AT, true, true><<<grid, block, 0, s>>>(d, tm, tn, splitk, partials, va, vb);
  else if (d.a_kcontig) k_gemm_guarded<AT, true, false><<<grid, block, 0, s>>>(d, tm, tn, splitk, partials, va, vb);
  else if (d.b_kcontig) k_gemm_guarded<AT, false, true><<<grid, block, 0, s>>>(d, tm, tn, splitk, partials, va, vb);
  else k_gemm_guarded<AT, false, false><<<grid, block, 0, s>>>(d, tm, tn, splitk, partials, va, vb);
  if (splitk > 1)
    k_guarded_reduce<AT><<<dim3((unsigned)(((size_t)d.M * d.N + 255) / 256)), block, 0, s>>>(partials, splitk, d.M, d.N, d.epi);
}

}  // namespace guarded

// Few tiles and a long contraction: split k.  A workgroup's slab takes about 0.5 us on a compute unit of its own
// (16 fp32 MFMAs of 64 cycles per wavefront), the parts cost a second launch of about 4 us.
int guarded_splitk(int M, int N, int K, int dtype, size_t partial_floats) {
  const int tiles = ((M + guarded::TILE - 1) / guarded::TILE) * ((N + guarded::TILE - 1) / guarded::TILE);
  const int slabs = (K * (dtype ? 2 : 4) + guarded::SLAB_BYTES - 1) / guarded::SLAB_BYTES;
  double best = 0.0;
  int pick = 1;
  for (int s = 1; s <= 64 && (s == 1 || slabs / s >= 4); ++s) {
    if (s > 1 && ((long long)tiles * s > 1024 || (size_t)s * M * N > partial_floats)) break;
    const double t = (double)((tiles * s + 255) / 256) * ((slabs + s - 1) / s) * 0.5 + (s > 1 ? 4.0 + (double)s * M * N * 8.0 / 4.0e6 : 0.0);
    if (s == 1 || t < best) { best = t; pick = s; }
  }
  return pick;
}

hipError_t guarded_reduce_f32(const float* partials, int splitk, int M, int N, const Epilogue& e, hipStream_t s) {
  guarded::k_guarded_reduce<float><<<dim3((unsigned)(((size_t)M * N + 255) / 256)), dim3(256), 0, s>>>(partials, splitk, M, N, e);
  return hipGetLastError();
}

hipError_t gemm_guarded(int dtype, const GemmDesc& d, int splitk, float* partials, hipStream_t s) {
  if (d.M <= 0 || d.N <= 0) return hipSuccess;
  if (splitk < 1 || (splitk > 1 && partials == nullptr)) return hipErrorInvalidValue;
  if (dtype == 0) guarded::launch<float>(d, splitk, partials, s);
  else guarded::launch<bf16>(d, splitk, partials, s);
  return hipGetLastError();
}

}  // namespace mslt

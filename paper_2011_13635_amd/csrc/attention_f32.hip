// fp32 attention on the matrix cores (v_mfma_f32_32x32x2_f32), head width 64, any sequence length; scores, softmax
// and all sums in fp32.  A workgroup owns 32 queries (forward, dQ) or 32 keys (dK, dV) of one (batch, head) and its four
// wavefronts share the blocks of 32 rows on the other side, then add their results in LDS in a fixed order: a head of 128
// tokens is 4 workgroups of one block per wavefront, a short chain each, which is what counts at the batch sizes
// fp32 mode is used with.
//
// As in the bf16 kernels the products are formed transposed so that the softmax index sits in a lane's registers, and
// an accumulator register is the B operand of the next product as it stands: with two contraction indices per
// instruction, register r of the lower and the upper half-wave are rows k and k + 4 of its block, and the A operand
// for them is one row of V (K, Q, dC) each, 32 consecutive floats as they lie in memory.  In the first products a lane
// takes 16 bytes of its row, and the contraction order inside eight d is (j, 4 + j).  So nothing is transposed or
// staged; operands come from L2 by loads of whole cache lines.
// What bounds them is the latency of that chain, then the fp32 matrix pipes.  Per launch at 8x128x12 heads, against one
// wavefront per row in vector arithmetic: forward 75 -> 13 us, query side 204 -> 23, key side 215 -> 22; the
// BERT-Base 3+3 layer fp32 step 8x128 went from 4.43 to 2.87 ms.
// Rows past the end of the sequence re-read the last one; such keys get a bias of -inf, such queries a
// log-sum-exp of +inf, either of which makes their probabilities exact zeros.
#include "common.h"

namespace mslt {

namespace f32attn {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

constexpr int DH = 64, BLK = 32, WAVES = 4, LDO = DH + 4;

__device__ __forceinline__ f32x16_t zero16() {
  f32x16_t z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}
// row of a 32-row block that register r of this half-wave holds
__device__ __forceinline__ int acc_row(int r, int half) { return 8 * (r >> 2) + 4 * half + (r & 3); }

// this lane's half of one row: d = 8 g + 4 half + 0..3
struct RowFrag {
  f32x4_t v[8];
  __device__ __forceinline__ void load(const float* __restrict__ row, int half) {
#pragma unroll
    for (int g = 0; g < 8; ++g) v[g] = *reinterpret_cast<const f32x4_t*>(row + 8 * g + 4 * half);
  }
};
// acc[row of a, row of b] over the 64 d
__device__ __forceinline__ f32x16_t dot_rows(const RowFrag& a, const RowFrag& b) {
  f32x16_t acc = zero16();
#pragma unroll
  for (int g = 0; g < 8; ++g)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.v[g][j], b.v[g][j], acc, 0, 0, 0);
  return acc;
}
// acc[d, column] += sum over the block's rows of x[row][d] * p[row, column]; x: first column of this lane's rows
struct ColFrag {
  float v[16][2];
  __device__ __forceinline__ void load(const float* __restrict__ x, size_t ld, int r0, int last, int half, int col) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float* p = x + (size_t)min(r0 + acc_row(r, half), last) * ld + col;
      v[r][0] = p[0];
      v[r][1] = p[32];
    }
  }
};
__device__ __forceinline__ void add_outer(f32x16_t (&acc)[2], const ColFrag& x, const f32x16_t& p) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(x.v[r][0], p[r], acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(x.v[r][1], p[r], acc[1], 0, 0, 0);
  }
}
// accumulators [d, column] -> LDS [column][d]
__device__ __forceinline__ void put_tile(float* __restrict__ lds, const f32x16_t (&acc)[2], int half, int col) {
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<f32x4_t*>(lds + col * LDO + 32 * b + 8 * g + 4 * half) =
          f32x4_t{acc[b][4 * g], acc[b][4 * g + 1], acc[b][4 * g + 2], acc[b][4 * g + 3]};
}
// sum of the four wavefronts' tiles at (row, d .. d + 7), times scale, to memory
__device__ __forceinline__ void store_sum(const float* __restrict__ lds, float* __restrict__ out, int row, int d, float scale) {
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    f32x4_t s = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < WAVES; ++w) s += *reinterpret_cast<const f32x4_t*>(lds + (w * BLK + row) * LDO + d + 4 * c);
    *reinterpret_cast<f32x4_t*>(out + d + 4 * c) = s * scale;
  }
}
// keep factors of four consecutive keys of one query; aligned: the first element's index is a multiple of four
__device__ __forceinline__ void drop4(const DropSpec& drop, uint64_t e, bool aligned, float (&f)[4]) {
  if (aligned) {
    const uint64_t h = drop_quad(drop, e >> 2);
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = drop_field(drop, h, i);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = drop_factor(drop, e + i);
  }
}

template <bool DROP>
__global__ void __launch_bounds__(256) k_attn_f32_fwd(const float* __restrict__ qkv, float* __restrict__ ctx, float* __restrict__ ctx2,
                                                      float* __restrict__ lse, const int32_t* __restrict__ am, int S, int nh,
                                                      float scale, float mask_bias, DropSpec drop) {
  __shared__ __attribute__((aligned(16))) float tile[WAVES * BLK * LDO];
  __shared__ float sm_m[WAVES][BLK], sm_l[WAVES][BLK];
  const int h = blockIdx.y, b = blockIdx.z, q0 = blockIdx.x * BLK;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, half = lane >> 5;
  const int H = nh * DH;
  const size_t ld = 3 * (size_t)H;
  const float* Q = qkv + (size_t)b * S * ld + h * DH;
  const float *K = Q + H, *V = K + H;
  const int last = S - 1, q = min(q0 + col, last);
  RowFrag fq;
  fq.load(Q + (size_t)q * ld, half);
  f32x16_t o[2] = {zero16(), zero16()};
  float m = -INFINITY, l = 0.f;
  for (int k0 = wave * BLK; k0 < S; k0 += WAVES * BLK) {
    RowFrag fk;
    fk.load(K + (size_t)min(k0 + col, last) * ld, half);
    ColFrag fv;
    fv.load(V, ld, k0, last, half, col);
    float bias[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + acc_row(r, half);
      bias[r] = key > last ? -INFINITY : (am[b * S + min(key, last)] ? 0.f : mask_bias);
    }
    f32x16_t s = dot_rows(fk, fq);
    float mb = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = s[r] * scale + bias[r];
      mb = fmaxf(mb, s[r]);
    }
    mb = fmaxf(mb, __shfl_xor(mb, 32));
    const float mn = fmaxf(m, mb), ms = mn == -INFINITY ? 0.f : mn;
    const float rescale = __expf(m - ms);
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = __expf(s[r] - ms);
      sum += s[r];
    }
    sum += __shfl_xor(sum, 32);
    l = l * rescale + sum;
    m = mn;
#pragma unroll
    for (int r = 0; r < 16; ++r) { o[0][r] *= rescale; o[1][r] *= rescale; }
    if (DROP) {       // the normaliser is that of the undropped probabilities
      const uint64_t row = (((uint64_t)b * nh + h) * S + q) * S;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float f[4];
        drop4(drop, row + k0 + 8 * g + 4 * half, (S & 3) == 0, f);
#pragma unroll
        for (int i = 0; i < 4; ++i) s[4 * g + i] *= f[i];
      }
    }
    add_outer(o, fv, s);
  }
  put_tile(tile + wave * BLK * LDO, o, half, col);
  if (half == 0) { sm_m[wave][col] = m; sm_l[wave][col] = l; }
  __syncthreads();
  const int row = threadIdx.x >> 3, d = (threadIdx.x & 7) * 8;
  if (q0 + row > last) return;
  float mx = -INFINITY, den = 0.f, w[WAVES];
#pragma unroll
  for (int i = 0; i < WAVES; ++i) mx = fmaxf(mx, sm_m[i][row]);
#pragma unroll
  for (int i = 0; i < WAVES; ++i) {
    w[i] = __expf(sm_m[i][row] - mx);
    den += w[i] * sm_l[i][row];
  }
  const float inv = 1.0f / den;
  const size_t at = ((size_t)b * S + q0 + row) * H + h * DH + d;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    f32x4_t s = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < WAVES; ++i) s += w[i] * *reinterpret_cast<const f32x4_t*>(tile + (i * BLK + row) * LDO + d + 4 * c);
    s *= inv;
    *reinterpret_cast<f32x4_t*>(ctx + at + 4 * c) = s;
    if (ctx2 != nullptr) *reinterpret_cast<f32x4_t*>(ctx2 + at + 4 * c) = s;
  }
  if (lse != nullptr && d == 0) lse[((size_t)b * nh + h) * S + q0 + row] = mx + __logf(den);
}

// delta = dC . C ; dA = P (dC . v - delta) ; dQ = scale dA K
template <bool DROP>
__global__ void __launch_bounds__(256) k_attn_f32_bwd_q(const float* __restrict__ qkv, const float* __restrict__ ctx,
                                                        const float* __restrict__ dctx, const float* __restrict__ lse,
                                                        float* __restrict__ delta, float* __restrict__ dqkv,
                                                        const int32_t* __restrict__ am, int S, int nh, float scale,
                                                        float mask_bias, DropSpec drop) {
  __shared__ __attribute__((aligned(16))) float tile[WAVES * BLK * LDO];
  const int h = blockIdx.y, b = blockIdx.z, q0 = blockIdx.x * BLK;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, half = lane >> 5;
  const int H = nh * DH;
  const size_t ld = 3 * (size_t)H;
  const float* Q = qkv + (size_t)b * S * ld + h * DH;
  const float *K = Q + H, *V = K + H;
  const int last = S - 1, q = min(q0 + col, last);
  const size_t crow = ((size_t)b * S + q) * H + h * DH, li = ((size_t)b * nh + h) * S + q;
  RowFrag fq, fc, fo;
  fq.load(Q + (size_t)q * ld, half);
  fc.load(dctx + crow, half);
  fo.load(ctx + crow, half);
  const float lq = lse[li];
  float dl = 0.f;
#pragma unroll
  for (int g = 0; g < 8; ++g)
#pragma unroll
    for (int j = 0; j < 4; ++j) dl += fc.v[g][j] * fo.v[g][j];
  dl += __shfl_xor(dl, 32);
  if (wave == 0 && half == 0 && q0 + col <= last) delta[li] = dl;
  f32x16_t dq[2] = {zero16(), zero16()};
  for (int k0 = wave * BLK; k0 < S; k0 += WAVES * BLK) {
    const size_t krow = (size_t)min(k0 + col, last) * ld;
    RowFrag fk, fv;
    fk.load(K + krow, half);
    fv.load(V + krow, half);
    ColFrag kc;
    kc.load(K, ld, k0, last, half, col);
    float bias[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + acc_row(r, half);
      bias[r] = key > last ? -INFINITY : (am[b * S + min(key, last)] ? 0.f : mask_bias);
    }
    const f32x16_t s = dot_rows(fk, fq);
    f32x16_t da = dot_rows(fv, fc);
    if (DROP) {
      const uint64_t row = (((uint64_t)b * nh + h) * S + q) * S;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float f[4];
        drop4(drop, row + k0 + 8 * g + 4 * half, (S & 3) == 0, f);
#pragma unroll
        for (int i = 0; i < 4; ++i) da[4 * g + i] *= f[i];
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) da[r] = __expf(s[r] * scale + bias[r] - lq) * (da[r] - dl);
    add_outer(dq, kc, da);
  }
  put_tile(tile + wave * BLK * LDO, dq, half, col);
  __syncthreads();
  const int row = threadIdx.x >> 3;
  if (q0 + row <= last)
    store_sum(tile, dqkv + ((size_t)b * S + q0 + row) * ld + h * DH, row, (threadIdx.x & 7) * 8, scale);
}

// dV = P^T dC (dropped P) ; dK = scale dA^T Q
template <bool DROP>
__global__ void __launch_bounds__(256) k_attn_f32_bwd_kv(const float* __restrict__ qkv, const float* __restrict__ dctx,
                                                         const float* __restrict__ lse, const float* __restrict__ delta,
                                                         float* __restrict__ dqkv, const int32_t* __restrict__ am, int S, int nh,
                                                         float scale, float mask_bias, DropSpec drop) {
  __shared__ __attribute__((aligned(16))) float tile[WAVES * BLK * LDO];
  const int h = blockIdx.y, b = blockIdx.z, k0 = blockIdx.x * BLK;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, half = lane >> 5;
  const int H = nh * DH;
  const size_t ld = 3 * (size_t)H;
  const float* Q = qkv + (size_t)b * S * ld + h * DH;
  const float *K = Q + H, *V = K + H;
  const float* C = dctx + (size_t)b * S * H + h * DH;
  const int last = S - 1, key = min(k0 + col, last);
  RowFrag fk, fv;
  fk.load(K + (size_t)key * ld, half);
  fv.load(V + (size_t)key * ld, half);
  const float bias = am[b * S + key] ? 0.f : mask_bias;
  const size_t l0 = ((size_t)b * nh + h) * S;
  f32x16_t dv[2] = {zero16(), zero16()}, dk[2] = {zero16(), zero16()};
  for (int q0 = wave * BLK; q0 < S; q0 += WAVES * BLK) {
    const int q = min(q0 + col, last);
    RowFrag fq, fc;
    fq.load(Q + (size_t)q * ld, half);
    fc.load(C + (size_t)q * H, half);
    ColFrag qc, cc;
    cc.load(C, H, q0, last, half, col);
    qc.load(Q, ld, q0, last, half, col);
    float lq[16], dl[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = q0 + acc_row(r, half);
      lq[r] = i > last ? INFINITY : lse[l0 + min(i, last)];
      dl[r] = delta[l0 + min(i, last)];
    }
    f32x16_t p = dot_rows(fq, fk);
    f32x16_t da = dot_rows(fc, fv);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float e = __expf(p[r] * scale + bias - lq[r]);
      const float kf = DROP ? drop_factor(drop, (l0 + min(q0 + acc_row(r, half), last)) * S + key) : 1.f;
      p[r] = e * kf;
      da[r] = e * (da[r] * kf - dl[r]);
    }
    add_outer(dv, cc, p);
    add_outer(dk, qc, da);
  }
  const int row = threadIdx.x >> 3;
  float* out = dqkv + ((size_t)b * S + min(k0 + row, last)) * ld + h * DH;
  put_tile(tile + wave * BLK * LDO, dv, half, col);
  __syncthreads();
  if (k0 + row <= last) store_sum(tile, out + 2 * H, row, (threadIdx.x & 7) * 8, 1.f);
  __syncthreads();
  put_tile(tile + wave * BLK * LDO, dk, half, col);
  __syncthreads();
  if (k0 + row <= last) store_sum(tile, out + H, row, (threadIdx.x & 7) * 8, scale);
}

}  // namespace f32attn

bool attention_f32_supported(int dh) { return dh == f32attn::DH; }

hipError_t attention_fwd_f32(const AttnDesc& a, hipStream_t s) {
  const dim3 grid((a.S + f32attn::BLK - 1) / f32attn::BLK, a.nh, a.B), block(64 * f32attn::WAVES);
  auto* k = a.drop.thr ? f32attn::k_attn_f32_fwd<true> : f32attn::k_attn_f32_fwd<false>;
  k<<<grid, block, 0, s>>>((const float*)a.qkv, (float*)a.ctx, a.ctx_f32, a.lse, a.attn_mask, a.S, a.nh,
                           1.0f / sqrtf((float)a.dh), a.mask_bias, a.drop);
  return hipGetLastError();
}

hipError_t attention_bwd_f32(const AttnBwdDesc& a, hipStream_t s) {
  const dim3 grid((a.S + f32attn::BLK - 1) / f32attn::BLK, a.nh, a.B), block(64 * f32attn::WAVES);
  const float scale = 1.0f / sqrtf((float)a.dh);
  auto* kq = a.drop.thr ? f32attn::k_attn_f32_bwd_q<true> : f32attn::k_attn_f32_bwd_q<false>;
  kq<<<grid, block, 0, s>>>((const float*)a.qkv, a.ctx_f32 ? a.ctx_f32 : (const float*)a.ctx, (const float*)a.dctx, a.lse,
                            a.delta, (float*)a.dqkv, a.attn_mask, a.S, a.nh, scale, a.mask_bias, a.drop);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  auto* kkv = a.drop.thr ? f32attn::k_attn_f32_bwd_kv<true> : f32attn::k_attn_f32_bwd_kv<false>;
  kkv<<<grid, block, 0, s>>>((const float*)a.qkv, (const float*)a.dctx, a.lse, a.delta, (float*)a.dqkv, a.attn_mask, a.S,
                             a.nh, scale, a.mask_bias, a.drop);
  return hipGetLastError();
}

}  // namespace mslt

// bf16 MFMA attention for gfx950, head width 64, any sequence length.
//
// Forward: softmax(Q K^T / sqrt(d) + key mask) V with the scale, mask and softmax fused between
// the two products; the S x S scores never leave registers.  Backward: scores are recomputed
// from Q, K and the stored row log-sum-exp, in two kernels that each keep one operand family
// resident: a query-side kernel (dQ, and delta = rowsum(dC * C)) and a key-side kernel (dK, dV).
//
// All products are v_mfma_f32_32x32x16_bf16 and are arranged transposed, so that the index the
// softmax runs along sits in a lane's registers:
//   query side:  S^T[key,q] = K Q^T      -> a lane owns one query column, its registers the keys
//                O^T[d,q]   = V^T P^T    -> P^T feeds the second product straight from registers
//   key side:    S[q,key]   = Q K^T      -> a lane owns one key column, its registers the queries
//                dV^T[d,key] = dC^T P,  dK^T[d,key] = Q^T dS
// The accumulator layout of one product is used directly as the B operand of the next one by
// agreeing on a permuted order of the contraction index (the order in which a lane's registers
// hold it); the A operand (V^T, K^T, Q^T, dC^T) is written to LDS transposed and in that order.
// One 256-thread workgroup handles 128 queries (or keys) of one (batch, head): 32 per wavefront.
// Lengths that are no multiple of 128 run through the same kernels (RAG below).  Before, they went to one wavefront per
// row in fp32 vector arithmetic: BERT-Base 9+3 layers, 27x203, dropout: attention 12.6 -> 0.74 ms of a step, the step
// 15.9 -> 4.0 ms.
#include "common.h"

namespace mslt {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;

constexpr int DH = 64;        // head width
constexpr int TILE = 128;     // rows per LDS tile
constexpr int TLD = 136;      // row stride (elements) of a transposed tile [64][128+8]

__device__ __forceinline__ int swz8(int row) { return ((row >> 1) & 7) ^ ((row >> 4) & 7); }

// A sequence whose length is no multiple of 128 leaves its last tile partly empty (RAG).  Loads of the rows past
// the end re-read the last row, so that they stay unconditional and in bounds; such keys get a bias of -inf and
// such queries a log-sum-exp of +inf, either of which makes their probabilities exact zeros, and nothing is stored
// for them.  Blocks of 32 rows (forward: 64 keys) of the side a wavefront walks that lie past the end altogether are
// skipped.  A wavefront whose own 32 rows do is skipped by the forward and the one-tile backward; in the two-kernel
// backward it computes on copies of the last row beside the others and stores nothing.
template <bool RAG>
__device__ __forceinline__ int tile_row(int row, int last) { return RAG ? min(row, last) : row; }

// Row-major tile [128][64] from global rows of stride ld, 16-byte chunks XOR-swizzled per row; last: last valid row.
template <bool RAG>
__device__ __forceinline__ void load_tile_rows(bf16* __restrict__ lds, const bf16* __restrict__ g, size_t ld, int tid, int last) {
  int c = tid & 7, r = tid >> 3;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    int row = r + 32 * p;
    u32x4_t v = *reinterpret_cast<const u32x4_t*>(g + (size_t)tile_row<RAG>(row, last) * ld + 8 * c);
    *reinterpret_cast<u32x4_t*>(lds + row * DH + 8 * (c ^ swz8(row))) = v;
  }
}
__device__ __forceinline__ bf16x8_t frag_rows(const bf16* __restrict__ lds, int row, int chunk) {
  return *reinterpret_cast<const bf16x8_t*>(lds + row * DH + 8 * (chunk ^ swz8(row)));
}

// Position of row r (0..127) of a tile along the contraction axis of a transposed tile: within
// each block of 32 the order is the one in which an accumulator lane holds its 16 rows, i.e.
// slot s of lane-half h in the c-th 16-wide MFMA step is row 8*(2c + s/4) + 4h + s%4.
__device__ __forceinline__ int perm_pos(int r) {
  int blk = r & ~31, o = r & 31;
  int c = o >> 4, s4 = (o >> 3) & 1, h = (o >> 2) & 1, j = o & 3;
  return blk + c * 16 + h * 8 + s4 * 4 + j;
}

// Transposed tile [64 d][128 rows permuted] from global rows of stride ld: each thread takes 4
// consecutive rows x 8 d, transposes in registers and writes eight 8-byte pieces.
__device__ __forceinline__ void put4(bf16* __restrict__ lds, int d, int pos, uint32_t a, uint32_t b, uint32_t c,
                                     uint32_t e, uint32_t sel) {
  u32x2_t o;
  o.x = __builtin_amdgcn_perm(b, a, sel);
  o.y = __builtin_amdgcn_perm(e, c, sel);
  *reinterpret_cast<u32x2_t*>(lds + d * TLD + pos) = o;
}
template <bool RAG>
__device__ __forceinline__ void load_tile_transposed(bf16* __restrict__ lds, const bf16* __restrict__ g, size_t ld,
                                                     int tid, int last) {
  int rg = tid >> 3, dg = tid & 7;  // rows 4rg..4rg+3, d 8dg..8dg+7
  const bf16* q = g + (size_t)(RAG ? 0 : 4 * rg) * ld + 8 * dg;
  auto at = [&](int i) { return q + (size_t)(RAG ? min(4 * rg + i, last) : i) * ld; };
  u32x4_t v0 = *reinterpret_cast<const u32x4_t*>(at(0));
  u32x4_t v1 = *reinterpret_cast<const u32x4_t*>(at(1));
  u32x4_t v2 = *reinterpret_cast<const u32x4_t*>(at(2));
  u32x4_t v3 = *reinterpret_cast<const u32x4_t*>(at(3));
  int pos = perm_pos(4 * rg), d = 8 * dg;
  const uint32_t LO = 0x05040100u, HI = 0x07060302u;
  put4(lds, d + 0, pos, v0.x, v1.x, v2.x, v3.x, LO);
  put4(lds, d + 1, pos, v0.x, v1.x, v2.x, v3.x, HI);
  put4(lds, d + 2, pos, v0.y, v1.y, v2.y, v3.y, LO);
  put4(lds, d + 3, pos, v0.y, v1.y, v2.y, v3.y, HI);
  put4(lds, d + 4, pos, v0.z, v1.z, v2.z, v3.z, LO);
  put4(lds, d + 5, pos, v0.z, v1.z, v2.z, v3.z, HI);
  put4(lds, d + 6, pos, v0.w, v1.w, v2.w, v3.w, LO);
  put4(lds, d + 7, pos, v0.w, v1.w, v2.w, v3.w, HI);
}
// A-operand fragment of a transposed tile: row d, the 8 contraction slots of (block kb, step c, half h)
__device__ __forceinline__ bf16x8_t frag_transposed(const bf16* __restrict__ lds, int d, int kb, int c, int half) {
  return *reinterpret_cast<const bf16x8_t*>(lds + d * TLD + kb * 32 + c * 16 + half * 8);
}

__device__ __forceinline__ uint32_t pack2(float a, float b) { return pack_bf16x2(a, b); }
// registers 8c..8c+7 of an accumulator block -> B operand of the c-th 16-wide step
__device__ __forceinline__ bf16x8_t pack_frag(const f32x16_t& p, int c) {
  u32x4_t u;
  u.x = pack2(p[8 * c + 0], p[8 * c + 1]);
  u.y = pack2(p[8 * c + 2], p[8 * c + 3]);
  u.z = pack2(p[8 * c + 4], p[8 * c + 5]);
  u.w = pack2(p[8 * c + 6], p[8 * c + 7]);
  return __builtin_bit_cast(bf16x8_t, u);
}
__device__ __forceinline__ f32x16_t zero16() {
  f32x16_t z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}
#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16((a), (b), (c), 0, 0, 0)

// The leading eight bits of the values in registers 8c..8c+7 as a B operand, by truncation; they are taken off the
// registers.  Three in a row hold an fp32 value exactly (24 bits of significand).
__device__ __forceinline__ bf16x8_t take_frag(f32x16_t& p, int c) {
  uint32_t u[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t a = __float_as_uint(p[8 * c + 2 * i]), b = __float_as_uint(p[8 * c + 2 * i + 1]);
    u[i] = __builtin_amdgcn_perm(b, a, 0x07060302u);
    p[8 * c + 2 * i] -= __uint_as_float(a & 0xffff0000u);
    p[8 * c + 2 * i + 1] -= __uint_as_float(b & 0xffff0000u);
  }
  return __builtin_bit_cast(bf16x8_t, u32x4_t{u[0], u[1], u[2], u[3]});
}
// 4 consecutive d of 32 rows: accumulator block (lane = row index n, registers = d) to global
// out[(row0 + n)*ld + d0 + 8g + 4half + j] with optional scale, 8-byte stores
__device__ __forceinline__ void store_acc_T(bf16* __restrict__ out, size_t ld, int n, int half, const f32x16_t& a,
                                            float scale) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    u32x2_t o;
    o.x = pack2(a[4 * g] * scale, a[4 * g + 1] * scale);
    o.y = pack2(a[4 * g + 2] * scale, a[4 * g + 3] * scale);
    *reinterpret_cast<u32x2_t*>(out + (size_t)n * ld + 8 * g + 4 * half) = o;
  }
}

__device__ __forceinline__ void store_acc_T_f32(float* __restrict__ out, size_t ld, int n, int half, const f32x16_t& a,
                                                float scale) {
#pragma unroll
  for (int g = 0; g < 4; ++g)
    *reinterpret_cast<float4*>(out + (size_t)n * ld + 8 * g + 4 * half) =
        make_float4(a[4 * g] * scale, a[4 * g + 1] * scale, a[4 * g + 2] * scale, a[4 * g + 3] * scale);
}
// 8 consecutive values of the context row for delta: from the fp32 copy when there is one
__device__ __forceinline__ void load_ctx8(const bf16* __restrict__ ctx, const float* __restrict__ ctx32, size_t o,
                                          float (&c)[8]) {
  if (ctx32 != nullptr) {
    float4 a = *reinterpret_cast<const float4*>(ctx32 + o), b = *reinterpret_cast<const float4*>(ctx32 + o + 4);
    c[0] = a.x; c[1] = a.y; c[2] = a.z; c[3] = a.w; c[4] = b.x; c[5] = b.y; c[6] = b.z; c[7] = b.w;
  } else {
    bf16x8_t v = *reinterpret_cast<const bf16x8_t*>(ctx + o);
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = (float)v[i];
  }
}

// acc0, acc1 (d 0..31, 32..63) += rows of the transposed tile times the c-th 16 rows of p (probabilities or their
// gradients).  Lengths that are a multiple of 128 multiply them in bf16.  The others (RAG) keep the fp32 values, as the
// wave-per-row kernels that took those lengths before did: three bf16 parts, exact together, for three times the matrix
// instructions of the second products.  Largest error of the context against float64, as a share of the sum of its
// terms' magnitudes, 3x203x2 heads: bf16 2^-9.3, in three parts 2^-20.9 (wave-per-row kernels 2^-20).  Per launch at
// 27x203x12 heads with dropout, bf16 / three parts: forward 36 / 41 us, query side 33 / 37, key side 38 / 46.
template <bool RAG>
__device__ __forceinline__ void add_product(f32x16_t& acc0, f32x16_t& acc1, const bf16* tile_t, int n, int blk, int c, int half,
                                            f32x16_t& p) {
  const bf16x8_t x0 = frag_transposed(tile_t, n, blk, c, half), x1 = frag_transposed(tile_t, 32 + n, blk, c, half);
  if constexpr (RAG) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const bf16x8_t f = take_frag(p, c);
      acc0 = MFMA(x0, f, acc0);
      acc1 = MFMA(x1, f, acc1);
    }
  } else {
    const bf16x8_t f = pack_frag(p, c);
    acc0 = MFMA(x0, f, acc0);
    acc1 = MFMA(x1, f, acc1);
  }
}

// Keep bits of the four consecutive elements from index e on, as drop_quad gives them for a whole quad: when a row
// of the probabilities does not start on a multiple of four, two quads are joined.
template <bool RAG>
__device__ __forceinline__ uint64_t drop_four(const DropSpec& d, uint64_t e) {
  const uint64_t lo = drop_quad(d, e >> 2);
  if constexpr (!RAG) return lo;
  const int sh = 16 * (int)(e & 3);
  if (sh == 0) return lo;
  return (lo >> sh) | (drop_quad(d, (e >> 2) + 1) << (64 - sh));
}

// The key side holds one key per lane and the queries in registers, so the four elements of a quad sit in four
// neighbouring lanes.  Each lane draws the quad of one of four consecutive query rows (row e0/S + lane%4; e0: element
// index of that row at the first key of the lane's four) and the lanes exchange them: a quarter of the hashes.
// keep[j]: factor of this lane's key for the j-th of the four rows.
template <int J>
__device__ __forceinline__ float quad_field(const DropSpec& d, uint32_t lo, uint32_t hi, int lane) {
  const uint32_t a = (uint32_t)__builtin_amdgcn_mov_dpp((int)lo, J * 0x55, 0xf, 0xf, true);
  const uint32_t b = (uint32_t)__builtin_amdgcn_mov_dpp((int)hi, J * 0x55, 0xf, 0xf, true);
  const uint32_t w = (lane & 2) ? b : a;
  return ((lane & 1) ? w >> 16 : w & 0xffffu) >= d.thr ? d.scale : 0.f;
}
template <bool RAG>
__device__ __forceinline__ void drop_rows(const DropSpec& d, uint64_t e0, int lane, float (&keep)[4]) {
  const uint64_t r = drop_four<RAG>(d, e0);
  const uint32_t lo = (uint32_t)r, hi = (uint32_t)(r >> 32);
  keep[0] = quad_field<0>(d, lo, hi, lane);
  keep[1] = quad_field<1>(d, lo, hi, lane);
  keep[2] = quad_field<2>(d, lo, hi, lane);
  keep[3] = quad_field<3>(d, lo, hi, lane);
}

// ---- forward --------------------------------------------------------------------------------
// The K and V^T tiles of one step (one key tile of one work item) as they sit in registers between the
// global loads and the LDS writes: issued one step ahead, so that the loads of step i+1 are in flight
// while step i computes.
struct KvRegs {
  u32x4_t k[4], v[4];
  float bias;
};
template <bool RAG>
__device__ __forceinline__ void fetch_kv(KvRegs& r, const bf16* __restrict__ kbase, const bf16* __restrict__ vbase,
                                         size_t ld, const int32_t* __restrict__ am_row, float mask_bias, int tid, int last) {
  const int c = tid & 7, rr = tid >> 3;
#pragma unroll
  for (int p = 0; p < 4; ++p)
    r.k[p] = *reinterpret_cast<const u32x4_t*>(kbase + (size_t)tile_row<RAG>(rr + 32 * p, last) * ld + 8 * c);
#pragma unroll
  for (int p = 0; p < 4; ++p)      // rows 4rr..4rr+3, d 8c..8c+7
    r.v[p] = *reinterpret_cast<const u32x4_t*>(vbase + (size_t)(RAG ? 0 : 4 * rr) * ld + 8 * c + (size_t)(RAG ? min(4 * rr + p, last) : p) * ld);
  r.bias = (tid < TILE) ? (am_row[tile_row<RAG>(tid, last)] ? 0.f : mask_bias) : 0.f;
  if (RAG && tid > last) r.bias = -INFINITY;
}
__device__ __forceinline__ void commit_kv(const KvRegs& r, bf16* __restrict__ Ks, bf16* __restrict__ Vt,
                                          float* __restrict__ bias, int tid) {
  const int c = tid & 7, rr = tid >> 3;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    int row = rr + 32 * p;
    *reinterpret_cast<u32x4_t*>(Ks + row * DH + 8 * (c ^ swz8(row))) = r.k[p];
  }
  const int pos = perm_pos(4 * rr), d = 8 * c;
  const uint32_t LO = 0x05040100u, HI = 0x07060302u;
  put4(Vt, d + 0, pos, r.v[0].x, r.v[1].x, r.v[2].x, r.v[3].x, LO);
  put4(Vt, d + 1, pos, r.v[0].x, r.v[1].x, r.v[2].x, r.v[3].x, HI);
  put4(Vt, d + 2, pos, r.v[0].y, r.v[1].y, r.v[2].y, r.v[3].y, LO);
  put4(Vt, d + 3, pos, r.v[0].y, r.v[1].y, r.v[2].y, r.v[3].y, HI);
  put4(Vt, d + 4, pos, r.v[0].z, r.v[1].z, r.v[2].z, r.v[3].z, LO);
  put4(Vt, d + 5, pos, r.v[0].z, r.v[1].z, r.v[2].z, r.v[3].z, HI);
  put4(Vt, d + 6, pos, r.v[0].w, r.v[1].w, r.v[2].w, r.v[3].w, LO);
  put4(Vt, d + 7, pos, r.v[0].w, r.v[1].w, r.v[2].w, r.v[3].w, HI);
  if (tid < TILE) bias[tid] = r.bias;
}

constexpr int FWD_BUF_ELEMS = TILE * DH + DH * TLD;                     // K rows + V^T of one step
constexpr int FWD_LDS_BYTES = 2 * (FWD_BUF_ELEMS * 2 + TILE * 4);       // two steps

// One workgroup takes `per_wg` consecutive work items (item = 128 queries of one (batch, head), numbered
// query tile fastest, then head, then batch) and walks their key tiles as one sequence of steps over two
// LDS buffers: while step i runs on one buffer, the K/V rows (and, at an item's first step, the Q
// fragments) of step i+1 are already on their way from memory.
template <bool DROP, bool RAG>
__global__ void __launch_bounds__(256, 2) k_attn_fwd_mfma(const bf16* __restrict__ qkv, bf16* __restrict__ ctx,
                                                       float* __restrict__ lse, const int32_t* __restrict__ am, int S,
                                                       int nh, float scale, float mask_bias, DropSpec drop,
                                                       float* __restrict__ ctx32, int n_items, int per_wg) {
  extern __shared__ __attribute__((aligned(16))) unsigned char fwd_lds[];
  bf16* const tiles = reinterpret_cast<bf16*>(fwd_lds);
  float* const biases = reinterpret_cast<float*>(fwd_lds + 2 * FWD_BUF_ELEMS * 2);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = lane & 31, half = lane >> 5;
  const int H = nh * DH, nkt = RAG ? (S + TILE - 1) / TILE : S / TILE;
  const size_t ld = 3 * (size_t)H;
  const int first = blockIdx.x * per_wg;
  const int count = min(per_wg, n_items - first);
  if (count <= 0) return;
  const int steps = count * nkt;
  // scores, running maximum and sum live in the base-2 domain: exp(x) = 2^(x log2 e) with the factor folded
  // into the score scale and the mask bias, so that a probability costs one subtraction and one v_exp_f32
  constexpr float LOG2E = 1.4426950408889634f, LN2 = 0.6931471805599453f;
  const float scale2 = scale * LOG2E;
  mask_bias *= LOG2E;

  // addresses of a step
  auto item_of = [&](int step, int& b, int& h, int& qt, int& kt) {
    const int it = first + step / nkt;
    kt = step % nkt;
    qt = it % nkt;
    h = (it / nkt) % nh;
    b = it / (nkt * nh);
  };
  KvRegs regs;
  bf16x8_t qn[4];
  auto fetch = [&](int step) {
    int b, h, qt, kt;
    item_of(step, b, h, qt, kt);
    const bf16* base = qkv + (size_t)b * S * ld + h * DH;
    fetch_kv<RAG>(regs, base + H + (size_t)kt * TILE * ld, base + 2 * H + (size_t)kt * TILE * ld, ld,
                  am + (size_t)b * S + kt * TILE, mask_bias, tid, S - 1 - kt * TILE);
    if (kt == 0) {
      const int q = tile_row<RAG>(qt * TILE + wave * 32 + n, S - 1);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        qn[ks] = *reinterpret_cast<const bf16x8_t*>(base + (size_t)q * ld + 16 * ks + 8 * half);
    }
  };

  fetch(0);
  commit_kv(regs, tiles, tiles + TILE * DH, biases, tid);
  __syncthreads();

  bf16x8_t qf[4];
  float m_run = -INFINITY, l_run = 0.f;
  f32x16_t o0 = zero16(), o1 = zero16();
#pragma unroll 1
  for (int step = 0; step < steps; ++step) {
    int b, h, qt, kt;
    item_of(step, b, h, qt, kt);
    const bf16* Ks = tiles + (step & 1) * FWD_BUF_ELEMS;
    const bf16* Vt = Ks + TILE * DH;
    const float* bias = biases + (step & 1) * TILE;
    const int q = qt * TILE + wave * 32 + n;  // this lane's query inside the sequence
    if (kt == 0) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) qf[ks] = qn[ks];
      m_run = -INFINITY;
      l_run = 0.f;
      o0 = zero16();
      o1 = zero16();
    }
    if (step + 1 < steps) fetch(step + 1);

    // the tile's keys go through the running softmax in two halves of 64: half the score registers
    const int halves = !RAG ? 2 : qt * TILE + wave * 32 >= S ? 0 : S - kt * TILE <= TILE / 2 ? 1 : 2;
#pragma unroll 1
    for (int kh = 0; kh < halves; ++kh) {
      f32x16_t s[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        s[j] = zero16();
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) s[j] = MFMA(frag_rows(Ks, (2 * kh + j) * 32 + n, 2 * ks + half), qf[ks], s[j]);
      }
      float tmax = -INFINITY;
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          float4 bb = *reinterpret_cast<const float4*>(&bias[(2 * kh + j) * 32 + 8 * g + 4 * half]);
          s[j][4 * g + 0] = s[j][4 * g + 0] * scale2 + bb.x;
          s[j][4 * g + 1] = s[j][4 * g + 1] * scale2 + bb.y;
          s[j][4 * g + 2] = s[j][4 * g + 2] * scale2 + bb.z;
          s[j][4 * g + 3] = s[j][4 * g + 3] * scale2 + bb.w;
          tmax = fmaxf(tmax, fmaxf(fmaxf(s[j][4 * g], s[j][4 * g + 1]), fmaxf(s[j][4 * g + 2], s[j][4 * g + 3])));
        }
      tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
      float m_new = fmaxf(m_run, tmax);
      float alpha = __builtin_amdgcn_exp2f(m_run - m_new);   // 0 on an item's first half tile (m_run = -inf)
      float psum = 0.f;
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float p = __builtin_amdgcn_exp2f(s[j][r] - m_new);
          s[j][r] = p;
          psum += p;
        }
      l_run = l_run * alpha + psum;
      m_run = m_new;
      if constexpr (DROP) {   // the row sum above is of the undropped probabilities; the product below uses the kept ones
        const uint64_t rowbase = (((uint64_t)b * nh + h) * S + q) * S + (uint64_t)kt * TILE;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const uint64_t r = drop_four<RAG>(drop, rowbase + (2 * kh + j) * 32 + 8 * g + 4 * half);
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) s[j][4 * g + jj] *= drop_field(drop, r, jj);
          }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        o0[r] *= alpha;
        o1[r] *= alpha;
      }
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int c = 0; c < 2; ++c) add_product<RAG>(o0, o1, Vt, n, 2 * kh + j, c, half, s[j]);
    }
    // (a ragged tile: the swap between the halves below is between lanes of one query, so they leave together)
    if (kt == nkt - 1 && (!RAG || q < S)) {
      float l_tot = l_run + __shfl_xor(l_run, 32, 64);
      float inv = 1.0f / l_tot;
      bf16* out = ctx + ((size_t)b * S + qt * TILE + wave * 32) * H + h * DH;
      store_acc_T(out, H, n, half, o0, inv);
      store_acc_T(out + 32, H, n, half, o1, inv);
      if (ctx32 != nullptr) {
        float* out32 = ctx32 + ((size_t)b * S + qt * TILE + wave * 32) * H + h * DH;
        store_acc_T_f32(out32, H, n, half, o0, inv);
        store_acc_T_f32(out32 + 32, H, n, half, o1, inv);
      }
      if (lse != nullptr && half == 0) lse[((size_t)b * nh + h) * S + q] = (m_run + __builtin_amdgcn_logf(l_tot)) * LN2;
    }
    if (step + 1 < steps) {
      bf16* Kn = tiles + ((step + 1) & 1) * FWD_BUF_ELEMS;
      commit_kv(regs, Kn, Kn + TILE * DH, biases + ((step + 1) & 1) * TILE, tid);
    }
    __syncthreads();
  }
}

// ---- backward, query side: delta and dQ -----------------------------------------------------
// (The four key blocks of a tile stay a loop: 154 registers and three wavefronts per SIMD, 45 us at 16x512x12 heads;
//  unrolled 252 registers, 55 us.)
template <bool DROP, bool RAG>
__global__ void __launch_bounds__(256, 2) k_attn_bwd_q_mfma(const bf16* __restrict__ qkv, const bf16* __restrict__ ctx,
                                                         const bf16* __restrict__ dctx, const float* __restrict__ lse,
                                                         float* __restrict__ delta, bf16* __restrict__ dqkv,
                                                         const int32_t* __restrict__ am, int S, int nh, float scale,
                                                         float mask_bias, DropSpec drop,
                                                         const float* __restrict__ ctx32) {
  __shared__ __attribute__((aligned(16))) bf16 Ks[TILE * DH];
  __shared__ __attribute__((aligned(16))) bf16 Vs[TILE * DH];
  __shared__ __attribute__((aligned(16))) bf16 Kt[DH * TLD];
  __shared__ __attribute__((aligned(16))) float bias[TILE];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = lane & 31, half = lane >> 5;
  const int qt = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int H = nh * DH;
  const size_t ld = 3 * (size_t)H;
  const bf16* base = qkv + (size_t)b * S * ld + h * DH;
  const int q_own = qt * TILE + wave * 32 + n, q = tile_row<RAG>(q_own, S - 1);
  const bool q_in = !RAG || q_own < S;
  const size_t tok = (size_t)b * S + q;
  const uint64_t rowbase = (((uint64_t)b * nh + h) * S + q) * S;   // element index of P[b, h, q, 0]

  bf16x8_t qf[4], gf[4];
  float dl = 0.f;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    qf[ks] = *reinterpret_cast<const bf16x8_t*>(base + (size_t)q * ld + 16 * ks + 8 * half);
    gf[ks] = *reinterpret_cast<const bf16x8_t*>(dctx + tok * H + h * DH + 16 * ks + 8 * half);
    float cf[8];
    load_ctx8(ctx, ctx32, tok * H + h * DH + 16 * ks + 8 * half, cf);
#pragma unroll
    for (int i = 0; i < 8; ++i) dl += (float)gf[ks][i] * cf[i];
  }
  dl += __shfl_xor(dl, 32, 64);
  const float l = lse[((size_t)b * nh + h) * S + q];
  if (half == 0 && q_in) delta[((size_t)b * nh + h) * S + q] = dl;

  f32x16_t dq0 = zero16(), dq1 = zero16();
  const int nkt = RAG ? (S + TILE - 1) / TILE : S / TILE;
  for (int kt = 0; kt < nkt; ++kt) {
    if (kt > 0) __syncthreads();
    const bf16* kbase = base + H + (size_t)kt * TILE * ld;
    const int last = S - 1 - kt * TILE;
    load_tile_rows<RAG>(Ks, kbase, ld, tid, last);
    load_tile_rows<RAG>(Vs, base + 2 * H + (size_t)kt * TILE * ld, ld, tid, last);
    load_tile_transposed<RAG>(Kt, kbase, ld, tid, last);
    if (tid < TILE) bias[tid] = RAG && tid > last ? -INFINITY : am[b * S + kt * TILE + tid] ? 0.f : mask_bias;
    __syncthreads();
#pragma unroll 1
    for (int kb = 0; kb < 4; ++kb) {
      if (RAG && kb * 32 > last) break;
      f32x16_t s = zero16(), dp = zero16();
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        s = MFMA(frag_rows(Ks, kb * 32 + n, 2 * ks + half), qf[ks], s);
        dp = MFMA(frag_rows(Vs, kb * 32 + n, 2 * ks + half), gf[ks], dp);
      }
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float4 bb = *reinterpret_cast<const float4*>(&bias[kb * 32 + 8 * g + 4 * half]);
        float bv[4] = {bb.x, bb.y, bb.z, bb.w};
        float kf4[4] = {1.f, 1.f, 1.f, 1.f};
        if constexpr (DROP) {
          const uint64_t r = drop_four<RAG>(drop, rowbase + (uint64_t)kt * TILE + kb * 32 + 8 * g + 4 * half);
#pragma unroll
          for (int j = 0; j < 4; ++j) kf4[j] = drop_field(drop, r, j);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float p = __expf(s[4 * g + j] * scale + bv[j] - l);
          s[4 * g + j] = p * (dp[4 * g + j] * kf4[j] - dl);   // dS^T (dP passes through the dropout mask)
        }
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) add_product<RAG>(dq0, dq1, Kt, n, kb, c, half, s);
    }
  }
  if (!q_in) return;
  bf16* out = dqkv + ((size_t)b * S + qt * TILE + wave * 32) * ld + h * DH;
  store_acc_T(out, ld, n, half, dq0, scale);
  store_acc_T(out + 32, ld, n, half, dq1, scale);
}

// ---- backward, key side: dK and dV ----------------------------------------------------------
// (Two wavefronts per SIMD asked for: the accumulators then stay in VGPRs, where the softmax arithmetic reads them
//  without v_accvgpr moves, and two workgroups share a compute unit.  Unrolled over its four query blocks the plain
//  kernel takes 53 us at 16x512x12 heads, as a loop 70; the dropout variant spills when unrolled and took 512 registers
//  with one hash per element: as a loop with shared hashes 46 us at 27x203x12 heads, before 142.)
template <bool DROP, bool RAG>
__global__ void __launch_bounds__(256, 2) k_attn_bwd_kv_mfma(const bf16* __restrict__ qkv, const bf16* __restrict__ dctx,
                                                          const float* __restrict__ lse,
                                                          const float* __restrict__ delta, bf16* __restrict__ dqkv,
                                                          const int32_t* __restrict__ am, int S, int nh, float scale,
                                                          float mask_bias, DropSpec drop) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_kv[];   // KV_LDS_BYTES
  bf16* Qs = reinterpret_cast<bf16*>(smem_kv);
  bf16* Gs = Qs + TILE * DH;
  bf16* Qt = Gs + TILE * DH;
  bf16* Gt = Qt + DH * TLD;
  float* lse_s = reinterpret_cast<float*>(Gt + DH * TLD);
  float* dl_s = lse_s + TILE;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = lane & 31, half = lane >> 5;
  const int kt = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int H = nh * DH;
  const size_t ld = 3 * (size_t)H;
  const bf16* base = qkv + (size_t)b * S * ld + h * DH;
  const int key_own = kt * TILE + wave * 32 + n, key = tile_row<RAG>(key_own, S - 1);  // this lane's key
  const uint64_t headbase = ((uint64_t)b * nh + h) * S;          // row index of P[b, h, 0, :]

  bf16x8_t kf[4], vf[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    kf[ks] = *reinterpret_cast<const bf16x8_t*>(base + H + (size_t)key * ld + 16 * ks + 8 * half);
    vf[ks] = *reinterpret_cast<const bf16x8_t*>(base + 2 * H + (size_t)key * ld + 16 * ks + 8 * half);
  }
  const float kbias = am[b * S + key] ? 0.f : mask_bias;

  f32x16_t dk0 = zero16(), dk1 = zero16(), dv0 = zero16(), dv1 = zero16();
  const int nqt = RAG ? (S + TILE - 1) / TILE : S / TILE;
  for (int qt = 0; qt < nqt; ++qt) {
    if (qt > 0) __syncthreads();
    const bf16* qbase = base + (size_t)qt * TILE * ld;
    const bf16* gbase = dctx + ((size_t)b * S + qt * TILE) * H + h * DH;
    const int last = S - 1 - qt * TILE;
    load_tile_rows<RAG>(Qs, qbase, ld, tid, last);
    load_tile_rows<RAG>(Gs, gbase, H, tid, last);
    load_tile_transposed<RAG>(Qt, qbase, ld, tid, last);
    load_tile_transposed<RAG>(Gt, gbase, H, tid, last);
    if (tid < TILE) {
      const bool in = !RAG || tid <= last;
      lse_s[tid] = in ? lse[((size_t)b * nh + h) * S + qt * TILE + tid] : INFINITY;
      dl_s[tid] = in ? delta[((size_t)b * nh + h) * S + qt * TILE + tid] : 0.f;
    }
    __syncthreads();
#pragma unroll(DROP ? 1 : 4)
    for (int qb = 0; qb < 4; ++qb) {
      if (RAG && qb * 32 > last) break;
      f32x16_t s = zero16(), dp = zero16();   // S[q,key] and dP[q,key]: lane = key, registers = queries
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        s = MFMA(frag_rows(Qs, qb * 32 + n, 2 * ks + half), kf[ks], s);
        dp = MFMA(frag_rows(Gs, qb * 32 + n, 2 * ks + half), vf[ks], dp);
      }
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float4 ll = *reinterpret_cast<const float4*>(&lse_s[qb * 32 + 8 * g + 4 * half]);
        float4 dd = *reinterpret_cast<const float4*>(&dl_s[qb * 32 + 8 * g + 4 * half]);
        float lv[4] = {ll.x, ll.y, ll.z, ll.w}, dv[4] = {dd.x, dd.y, dd.z, dd.w};
        float keep[4] = {1.f, 1.f, 1.f, 1.f};
        if constexpr (DROP)
          drop_rows<RAG>(drop, (headbase + (uint64_t)qt * TILE + qb * 32 + 8 * g + 4 * half + (lane & 3)) * S + (key_own & ~3), lane, keep);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float p = __expf(s[4 * g + j] * scale + kbias - lv[j]);
          const float kf1 = keep[j];
          s[4 * g + j] = p * kf1;                                   // dropped P (for dV)
          dp[4 * g + j] = p * (dp[4 * g + j] * kf1 - dv[j]);        // dS
        }
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        add_product<RAG>(dv0, dv1, Gt, n, qb, c, half, s);
        add_product<RAG>(dk0, dk1, Qt, n, qb, c, half, dp);
      }
    }
  }
  if (RAG && key_own >= S) return;
  bf16* out = dqkv + ((size_t)b * S + kt * TILE + wave * 32) * ld + h * DH;
  store_acc_T(out + H, ld, n, half, dk0, scale);
  store_acc_T(out + H + 32, ld, n, half, dk1, scale);
  store_acc_T(out + 2 * H, ld, n, half, dv0, 1.0f);
  store_acc_T(out + 2 * H + 32, ld, n, half, dv1, 1.0f);
}

// ---- backward for one-tile sequences (S <= 128): both sides in one launch ---------------------
// One 512-thread workgroup per (batch, head).  All eight wavefronts first stage Q, K, V and dC
// (row tiles for the first products, transposed tiles for the second ones), the row log-sum-exp,
// the key bias and delta = rowsum(dC * C) in LDS; then wavefronts 0..3 run the query side (dQ)
// and wavefronts 4..7 the key side (dK, dV) next to each other, with the same arithmetic as the
// two kernels above.  Every operand is read from memory once and delta never leaves the chip.
constexpr int ONE_LDS_BYTES = (4 * TILE * DH + 3 * DH * TLD) * 2 + 3 * TILE * 4;

template <bool DROP, bool RAG>
__global__ void __launch_bounds__(512) k_attn_bwd_one_tile(const bf16* __restrict__ qkv, const bf16* __restrict__ ctx,
                                                           const bf16* __restrict__ dctx,
                                                           const float* __restrict__ lse, bf16* __restrict__ dqkv,
                                                           const int32_t* __restrict__ am, int seq, int nh, float scale,
                                                           float mask_bias, DropSpec drop,
                                                           const float* __restrict__ ctx32) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_one[];   // ONE_LDS_BYTES
  bf16* Ks = reinterpret_cast<bf16*>(smem_one);
  bf16* Vs = Ks + TILE * DH;
  bf16* Qs = Vs + TILE * DH;
  bf16* Gs = Qs + TILE * DH;
  bf16* Kt = Gs + TILE * DH;
  bf16* Qt = Kt + DH * TLD;
  bf16* Gt = Qt + DH * TLD;
  float* lse_s = reinterpret_cast<float*>(Gt + DH * TLD);
  float* dl_s = lse_s + TILE;
  float* bias = dl_s + TILE;
  const int S = RAG ? seq : TILE, last = S - 1;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = lane & 31, half = lane >> 5;
  const int h = blockIdx.x, b = blockIdx.y;
  const int H = nh * DH;
  const size_t ld = 3 * (size_t)H;
  const bf16* base = qkv + (size_t)b * S * ld + h * DH;
  const bf16* gbase = dctx + (size_t)b * S * H + h * DH;

  // staging: the two halves of the workgroup take different tiles
  if (tid < 256) {
    load_tile_rows<RAG>(Ks, base + H, ld, tid, last);
    load_tile_rows<RAG>(Vs, base + 2 * H, ld, tid, last);
    load_tile_transposed<RAG>(Kt, base + H, ld, tid, last);
    load_tile_rows<RAG>(Gs, gbase, H, tid, last);
  } else {
    load_tile_rows<RAG>(Qs, base, ld, tid - 256, last);
    load_tile_transposed<RAG>(Qt, base, ld, tid - 256, last);
    load_tile_transposed<RAG>(Gt, gbase, H, tid - 256, last);
  }
  {
    // delta[q] = sum_d dC[q,d] * C[q,d]: four threads per query, 16 d each
    const int q = tid >> 2, part = tid & 3;
    const size_t o = ((size_t)b * S + tile_row<RAG>(q, last)) * H + h * DH + 16 * part;
    float dl = 0.f;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      bf16x8_t g = *reinterpret_cast<const bf16x8_t*>(dctx + o + 8 * j);
      float c[8];
      load_ctx8(ctx, ctx32, o + 8 * j, c);
#pragma unroll
      for (int i = 0; i < 8; ++i) dl += (float)g[i] * c[i];
    }
    dl += __shfl_xor(dl, 1, 64);
    dl += __shfl_xor(dl, 2, 64);
    if (part == 0) dl_s[q] = dl;
  }
  if (tid < TILE) lse_s[tid] = RAG && tid > last ? INFINITY : lse[((size_t)b * nh + h) * S + tid];
  else if (tid < 2 * TILE) bias[tid - TILE] = RAG && tid - TILE > last ? -INFINITY : am[b * S + tid - TILE] ? 0.f : mask_bias;
  __syncthreads();

  if (wave < 4) {
    // query side: lane owns query q, registers run over keys
    if (RAG && wave * 32 > last) return;
    const int q_own = wave * 32 + n, q = tile_row<RAG>(q_own, last);
    const uint64_t rowbase = (((uint64_t)b * nh + h) * S + q) * S;
    bf16x8_t qf[4], gf[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      qf[ks] = *reinterpret_cast<const bf16x8_t*>(base + (size_t)q * ld + 16 * ks + 8 * half);
      gf[ks] = *reinterpret_cast<const bf16x8_t*>(gbase + (size_t)q * H + 16 * ks + 8 * half);
    }
    const float l = lse_s[q], dl = dl_s[q];
    f32x16_t dq0 = zero16(), dq1 = zero16();
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      if (RAG && kb * 32 > last) break;
      f32x16_t s = zero16(), dp = zero16();
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        s = MFMA(frag_rows(Ks, kb * 32 + n, 2 * ks + half), qf[ks], s);
        dp = MFMA(frag_rows(Vs, kb * 32 + n, 2 * ks + half), gf[ks], dp);
      }
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float4 bb = *reinterpret_cast<const float4*>(&bias[kb * 32 + 8 * g + 4 * half]);
        float bv[4] = {bb.x, bb.y, bb.z, bb.w};
        float kf4[4] = {1.f, 1.f, 1.f, 1.f};
        if constexpr (DROP) {
          const uint64_t r = drop_four<RAG>(drop, rowbase + kb * 32 + 8 * g + 4 * half);
#pragma unroll
          for (int j = 0; j < 4; ++j) kf4[j] = drop_field(drop, r, j);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float p = __expf(s[4 * g + j] * scale + bv[j] - l);
          s[4 * g + j] = p * (dp[4 * g + j] * kf4[j] - dl);   // dS^T (dP passes through the dropout mask)
        }
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) add_product<RAG>(dq0, dq1, Kt, n, kb, c, half, s);
    }
    if (RAG && q_own > last) return;
    bf16* out = dqkv + ((size_t)b * S + wave * 32) * ld + h * DH;
    store_acc_T(out, ld, n, half, dq0, scale);
    store_acc_T(out + 32, ld, n, half, dq1, scale);
  } else {
    // key side: lane owns a key, registers run over queries
    const int w = wave - 4;
    if (RAG && w * 32 > last) return;
    const int key_own = w * 32 + n, key = tile_row<RAG>(key_own, last);
    const uint64_t headbase = ((uint64_t)b * nh + h) * S;
    bf16x8_t kf[4], vf[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      kf[ks] = *reinterpret_cast<const bf16x8_t*>(base + H + (size_t)key * ld + 16 * ks + 8 * half);
      vf[ks] = *reinterpret_cast<const bf16x8_t*>(base + 2 * H + (size_t)key * ld + 16 * ks + 8 * half);
    }
    const float kbias = bias[key];
    f32x16_t dk0 = zero16(), dk1 = zero16(), dv0 = zero16(), dv1 = zero16();
#pragma unroll
    for (int qb = 0; qb < 4; ++qb) {
      if (RAG && qb * 32 > last) break;
      f32x16_t s = zero16(), dp = zero16();
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        s = MFMA(frag_rows(Qs, qb * 32 + n, 2 * ks + half), kf[ks], s);
        dp = MFMA(frag_rows(Gs, qb * 32 + n, 2 * ks + half), vf[ks], dp);
      }
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float4 ll = *reinterpret_cast<const float4*>(&lse_s[qb * 32 + 8 * g + 4 * half]);
        float4 dd = *reinterpret_cast<const float4*>(&dl_s[qb * 32 + 8 * g + 4 * half]);
        float lv[4] = {ll.x, ll.y, ll.z, ll.w}, dv[4] = {dd.x, dd.y, dd.z, dd.w};
        float keep[4] = {1.f, 1.f, 1.f, 1.f};
        if constexpr (DROP)
          drop_rows<RAG>(drop, (headbase + qb * 32 + 8 * g + 4 * half + (lane & 3)) * S + (key_own & ~3), lane, keep);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float p = __expf(s[4 * g + j] * scale + kbias - lv[j]);
          const float kf1 = keep[j];
          s[4 * g + j] = p * kf1;                                   // dropped P (for dV)
          dp[4 * g + j] = p * (dp[4 * g + j] * kf1 - dv[j]);        // dS
        }
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        add_product<RAG>(dv0, dv1, Gt, n, qb, c, half, s);
        add_product<RAG>(dk0, dk1, Qt, n, qb, c, half, dp);
      }
    }
    if (RAG && key_own > last) return;
    bf16* out = dqkv + ((size_t)b * S + w * 32) * ld + h * DH;
    store_acc_T(out + H, ld, n, half, dk0, scale);
    store_acc_T(out + H + 32, ld, n, half, dk1, scale);
    store_acc_T(out + 2 * H, ld, n, half, dv0, 1.0f);
    store_acc_T(out + 2 * H + 32, ld, n, half, dv1, 1.0f);
  }
}

constexpr int KV_LDS_BYTES = (2 * TILE * DH + 2 * DH * TLD) * 2 + 2 * TILE * 4;

bool attention_mfma_supported(int S, int dh) { return dh == DH && S >= 1; }

static hipError_t allow_lds(const void* kernel, int bytes) {
  return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

template <bool DROP, bool RAG>
static hipError_t attention_fwd_mfma_t(const AttnDesc& a, hipStream_t s) {
  static const hipError_t attr = allow_lds(reinterpret_cast<const void*>(k_attn_fwd_mfma<DROP, RAG>), FWD_LDS_BYTES);
  if (attr != hipSuccess) return attr;
  // two workgroups fit a compute unit (LDS and registers); up to that many, one item each keeps the most
  // units busy, beyond it a workgroup walks several items so that loads run ahead of the arithmetic
  const int n_items = a.B * a.nh * ((a.S + TILE - 1) / TILE);
  const int slots = 2 * 256;
  const int per_wg = (n_items + slots - 1) / slots;
  const int n_wg = (n_items + per_wg - 1) / per_wg;
  k_attn_fwd_mfma<DROP, RAG><<<dim3(n_wg), dim3(256), FWD_LDS_BYTES, s>>>(
      (const bf16*)a.qkv, (bf16*)a.ctx, a.lse, a.attn_mask, a.S, a.nh, 1.0f / sqrtf((float)a.dh), a.mask_bias, a.drop,
      a.ctx_f32, n_items, per_wg);
  return hipGetLastError();
}
// Dropout and ragged lengths are compile-time variants so that the plain kernels carry none of their registers.
hipError_t attention_fwd_mfma(const AttnDesc& a, hipStream_t s) {
  if (!attention_mfma_supported(a.S, a.dh)) return hipErrorInvalidValue;
  if (a.S % TILE) return a.drop.thr ? attention_fwd_mfma_t<true, true>(a, s) : attention_fwd_mfma_t<false, true>(a, s);
  return a.drop.thr ? attention_fwd_mfma_t<true, false>(a, s) : attention_fwd_mfma_t<false, false>(a, s);
}

template <bool DROP, bool RAG>
static hipError_t attention_bwd_mfma_t(const AttnBwdDesc& a, hipStream_t s) {
  dim3 grid((a.S + TILE - 1) / TILE, a.nh, a.B);
  float scale = 1.0f / sqrtf((float)a.dh);
  if (a.S <= TILE) {
    static const hipError_t attr1 = allow_lds(reinterpret_cast<const void*>(k_attn_bwd_one_tile<DROP, RAG>), ONE_LDS_BYTES);
    if (attr1 != hipSuccess) return attr1;
    k_attn_bwd_one_tile<DROP, RAG><<<dim3(a.nh, a.B), dim3(512), ONE_LDS_BYTES, s>>>(
        (const bf16*)a.qkv, (const bf16*)a.ctx, (const bf16*)a.dctx, a.lse, (bf16*)a.dqkv, a.attn_mask, a.S, a.nh, scale,
        a.mask_bias, a.drop, a.ctx_f32);
    return hipGetLastError();
  }
  k_attn_bwd_q_mfma<DROP, RAG><<<grid, dim3(256), 0, s>>>((const bf16*)a.qkv, (const bf16*)a.ctx, (const bf16*)a.dctx, a.lse,
                                                          a.delta, (bf16*)a.dqkv, a.attn_mask, a.S, a.nh, scale, a.mask_bias,
                                                          a.drop, a.ctx_f32);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  static const hipError_t attr2 = allow_lds(reinterpret_cast<const void*>(k_attn_bwd_kv_mfma<DROP, RAG>), KV_LDS_BYTES);
  if (attr2 != hipSuccess) return attr2;
  k_attn_bwd_kv_mfma<DROP, RAG><<<grid, dim3(256), KV_LDS_BYTES, s>>>((const bf16*)a.qkv, (const bf16*)a.dctx, a.lse, a.delta,
                                                                      (bf16*)a.dqkv, a.attn_mask, a.S, a.nh, scale,
                                                                      a.mask_bias, a.drop);
  return hipGetLastError();
}
hipError_t attention_bwd_mfma(const AttnBwdDesc& a, hipStream_t s) {
  if (!attention_mfma_supported(a.S, a.dh)) return hipErrorInvalidValue;
  if (a.S % TILE) return a.drop.thr ? attention_bwd_mfma_t<true, true>(a, s) : attention_bwd_mfma_t<false, true>(a, s);
  return a.drop.thr ? attention_bwd_mfma_t<true, false>(a, s) : attention_bwd_mfma_t<false, false>(a, s);
}

}  // namespace mslt

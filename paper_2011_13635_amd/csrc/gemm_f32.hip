// fp32 matrix-core GEMM for gfx950: C(m,n) = sum_k A(m,k) B(n,k) with the shared epilogue, fp32 throughout
// (v_mfma_f32_32x32x2_f32).  Any M and N, operands in any layout with 16-byte aligned rows; K a multiple of 4 where an
// operand is k-contiguous.
//
// A 512-thread workgroup owns a 64x64 tile of C.  Its eight wavefronts are two groups of four, a 32x32 block each, and
// the groups take the slabs of 32 k in turn, so that on every SIMD one wavefront multiplies (sixteen matrix instructions
// of 64 cycles) while the other reads its next slab's fragments and queues loads; the two sums are added in LDS at the
// end.  The matrix pipes need only 16 bytes of operands per clock and compute unit, a quarter of what L2 delivers, so a
// larger tile would buy nothing; what a wavefront alone on its SIMD loses is the latency of its slab, barrier to barrier.
// The matrix pipes alone reach 134 TFLOP/s here, this kernel 92 where its rounds are full; against the guarded kernel
// (four wavefronts, registers between global memory and LDS), us: 1024x768x768 22 / 27, 1024x768x3072 55 / 54 (both in
// four parts, which go to the guarded kernel: gemm_f32_pays), weight gradient 2304x768x1024 43 / 48, 1024x3072x768 52 / 53, 544x128x128 7.4 / 8.9.
// Slabs go global memory -> LDS directly through a ring of five slots (16 KB: 64 rows of either operand), two workgroups on
// a compute unit.  LDS and fragments are as in the guarded kernel: k-contiguous operands as [64 rows][32 k] with the
// 16-byte chunks XOR-swizzled by the row, a lane's fragment being one 16-byte read for four matrix instructions, the
// contraction order inside a group of eight k (j, 4 + j); k-strided ones as [32 k][64 rows], read four bytes at a time, the
// chunks of every other four k rows moved by half a row so that the two halves of a wavefront use different banks.
// Rows past the end and k past the end are read as zeros: the operand's view ends with its last element, and lanes
// whose k lies past the end of a k-contiguous row are sent outside it.
#include "common.h"
#include "gemm_epilogue.h"

namespace mslt {

namespace f32 {

constexpr int TILE = 64, BK = 32, OPERAND = TILE * BK * 4, SLOT = 2 * OPERAND, SLOTS = 5;
constexpr int waitcnt_imm(int vm, int lgkm) { return (vm & 15) | 0x70 | ((vm >> 4) << 14) | (lgkm << 8); }

// One operand's part of a slot: eight pieces of 1 KB, of which wavefront w of a group moves 2 w and 2 w + 1.
//   k-contiguous: piece q is rows 8q .. 8q+7; lane -> row 8q + lane/8, place lane%8, which holds chunk place ^ ((row>>1)&7)
//   k-strided: piece q is k rows 4q .. 4q+3; lane -> k row 4q + lane/16, place lane%16, which holds chunk place ^ 8 (q&1)
template <bool KC>
struct Operand {
  const float* base;
  int bytes, ld;
  int voff[2];      // per-lane byte offset of even / odd pieces
  int kk[2];        // k-contiguous: k of the lane's chunk inside the slab
  unsigned frag;    // lane part of a fragment address
  __device__ __forceinline__ void init(const float* p, int ld_, int row0, int rows, int K, int lane, int block) {
    ld = ld_;
    base = KC ? p + (size_t)row0 * ld : p + row0;
    const long long left = (KC ? (long long)(rows - row0 - 1) * ld + K : (long long)(K - 1) * ld + rows - row0) * 4;
    bytes = (int)(left < 0x7fffffff ? left : 0x7fffffff);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      kk[j] = 4 * ((lane & 7) ^ ((4 * j + (lane >> 4)) & 7));
      voff[j] = KC ? ((lane >> 3) * ld + kk[j]) * 4 : (lane >> 4) * ld * 4 + (((lane & 15) ^ (8 * j)) << 4);
    }
    const int row = 32 * block + (lane & 31), half = lane >> 5;
    frag = KC ? row * 128 + (((row >> 1) & 7) << 4) : half * 1024 + (((row >> 2) ^ (8 * half)) << 4) + (row & 3) * 4;
  }
  __device__ __forceinline__ void issue(int k0, int K, bool in_range, int w, unsigned char* lds) const {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, in_range ? bytes : 0, 0x00020000);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int q = 2 * w + j;
      const int soff = KC ? (q * 8 * ld + k0) * 4 : (k0 + q * 4) * ld * 4;
      const int v = KC && k0 + kk[j] >= K ? 0x7fffff00 : voff[j];
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)(lds + q * 1024), 16, v, soff, 0, 0);
    }
  }
  // group g (0..3) of the slab: eight k, this lane's half of them
  __device__ __forceinline__ void read(unsigned lds, int half, float (&f)[4][4]) const {
    if constexpr (KC) {
      u32x4_t v[4];
      asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
                   : "v"((frag ^ ((0 + half) << 4)) + lds), "v"((frag ^ ((2 + half) << 4)) + lds), "v"((frag ^ ((4 + half) << 4)) + lds),
                     "v"((frag ^ ((6 + half) << 4)) + lds) : "memory");
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f[g][0] = __uint_as_float(v[g].x); f[g][1] = __uint_as_float(v[g].y);
        f[g][2] = __uint_as_float(v[g].z); f[g][3] = __uint_as_float(v[g].w);
      }
    } else {      // k = 8 g + 4 half + j, 256 bytes a k row
      asm volatile("ds_read_b32 %0, %16\n\tds_read_b32 %1, %16 offset:256\n\tds_read_b32 %2, %16 offset:512\n\tds_read_b32 %3, %16 offset:768\n\t"
                   "ds_read_b32 %4, %16 offset:2048\n\tds_read_b32 %5, %16 offset:2304\n\tds_read_b32 %6, %16 offset:2560\n\tds_read_b32 %7, %16 offset:2816\n\t"
                   "ds_read_b32 %8, %16 offset:4096\n\tds_read_b32 %9, %16 offset:4352\n\tds_read_b32 %10, %16 offset:4608\n\tds_read_b32 %11, %16 offset:4864\n\t"
                   "ds_read_b32 %12, %16 offset:6144\n\tds_read_b32 %13, %16 offset:6400\n\tds_read_b32 %14, %16 offset:6656\n\tds_read_b32 %15, %16 offset:6912\n\t"
                   "s_waitcnt lgkmcnt(0)"
                   : "=&v"(f[0][0]), "=&v"(f[0][1]), "=&v"(f[0][2]), "=&v"(f[0][3]), "=&v"(f[1][0]), "=&v"(f[1][1]), "=&v"(f[1][2]), "=&v"(f[1][3]),
                     "=&v"(f[2][0]), "=&v"(f[2][1]), "=&v"(f[2][2]), "=&v"(f[2][3]), "=&v"(f[3][0]), "=&v"(f[3][1]), "=&v"(f[3][2]), "=&v"(f[3][3])
                   : "v"(frag + lds) : "memory");
    }
  }
};
__device__ __forceinline__ void meet() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

template <bool A_KC, bool B_KC>
__global__ void __launch_bounds__(512, 4) k_gemm_f32(GemmDesc d, int tiles_m, int tiles_n, int splitk, float* __restrict__ partials) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const unsigned lds_base = (unsigned)(uintptr_t)(lds_void_t*)smem;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  const int group = wave >> 2, w = wave & 3, wm = w >> 1, wn = w & 1;
  const int tiles = tiles_m * tiles_n, split = (int)blockIdx.x / tiles, tile = (int)blockIdx.x % tiles;
  const int m0 = (tile / tiles_n) * TILE, n0 = (tile % tiles_n) * TILE;
  const int nslab = (d.K + BK - 1) / BK;
  const int lo = (int)((long long)split * nslab / splitk), n = (int)((long long)(split + 1) * nslab / splitk) - lo;
  Operand<A_KC> a;
  Operand<B_KC> b;
  a.init(reinterpret_cast<const float*>(d.A), d.lda, m0, d.M, d.K, lane, wm);
  b.init(reinterpret_cast<const float*>(d.B), d.ldb, n0, d.N, d.K, lane, wn);
  // slab i (of this split) lies in slot i % SLOTS; group i % 2 loads, reads and multiplies it
  auto issue = [&](int i, unsigned slot) {
    a.issue((lo + i) * BK, d.K, i < n, w, smem + slot);
    b.issue((lo + i) * BK, d.K, i < n, w, smem + slot + OPERAND);
  };
  // The group's first slabs: 0 and 2 or 1 and 3.  From then on it queues slab i + 4 (slot (i - 1) % SLOTS, which the
  // other group has read) when it reads slab i; the next one it reads has landed when four loads are in flight.
  for (int i = group; i < SLOTS - 1; i += 2) issue(i, i * SLOT);
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(4, 15));
  meet();
  f32x16_t acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  if (group) meet();
  unsigned rd = group * SLOT, wr = group ? 0 : (SLOTS - 1) * SLOT;
  auto adv = [](unsigned& x) { x += 2 * SLOT; if (x >= SLOTS * SLOT) x -= SLOTS * SLOT; };
  const int turns = (n + 1) / 2;      // the same for both groups: a slab past the end multiplies zeros
  for (int t = 0; t < turns; ++t) {
    const int i = 2 * t + group;
    issue(i + SLOTS - 1, wr); adv(wr);
    float fa[4][4], fb[4][4];
    a.read(lds_base + rd, half, fa);
    b.read(lds_base + rd + OPERAND, half, fb);
    adv(rd);
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(4, 15));
    meet();
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[g][j], fb[g][j], acc, 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    meet();
  }
  if (!group) meet();
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
  __syncthreads();

  // each group finishes eight of a lane's sixteen elements and gets the other group's sums of them
  float* share = reinterpret_cast<float*>(smem) + wave * 512 + lane;
#pragma unroll
  for (int r = 0; r < 8; ++r) share[64 * r] = group ? acc[r] : acc[8 + r];
  __syncthreads();
  const float* other = reinterpret_cast<const float*>(smem) + (wave ^ 4) * 512 + lane;
  float v[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) v[r] = (group ? acc[8 + r] : acc[r]) + other[64 * r];
  const int col = n0 + 32 * wn + (lane & 31);
  const int mb = m0 + 32 * wm + 16 * group + 4 * half;
  if (col >= d.N) return;
  if (splitk > 1) {
    float* out = partials + (size_t)split * d.M * d.N;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int m = mb + 8 * (r >> 2) + (r & 3);
      if (m < d.M) out[(size_t)m * d.N + col] = v[r];
    }
    return;
  }
  const Epilogue& e = d.epi;
  const float bias = e.bias ? e.bias[col] : 0.f;
  float x[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int m = mb + 8 * (r >> 2) + (r & 3);
    x[r] = m < d.M ? load_aux<float>(e, m, col) : 0.f;
  }
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int m = mb + 8 * (r >> 2) + (r & 3);
    if (m < d.M) finish_one<float>(e, m, col, v[r] + bias, x[r]);
  }
}
template <bool A_KC, bool B_KC>
static hipError_t launch(const GemmDesc& d, int splitk, float* partials, hipStream_t s) {
  static bool set = false;
  if (!set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_gemm_f32<A_KC, B_KC>), hipFuncAttributeMaxDynamicSharedMemorySize, SLOTS * SLOT);
    if (e != hipSuccess) return e;
    set = true;
  }
  const int tm = (d.M + TILE - 1) / TILE, tn = (d.N + TILE - 1) / TILE;
  k_gemm_f32<A_KC, B_KC><<<dim3((unsigned)(tm * tn * splitk)), dim3(512), SLOTS * SLOT, s>>>(d, tm, tn, splitk, partials);
  return hipGetLastError();
}

}  // namespace f32

bool gemm_f32_supported(const GemmDesc& d) {
  if (d.M <= 0 || d.N <= 0 || d.K <= 0) return false;
  if (d.lda % 4 || d.ldb % 4 || reinterpret_cast<uintptr_t>(d.A) % 16 || reinterpret_cast<uintptr_t>(d.B) % 16) return false;
  if ((d.a_kcontig || d.b_kcontig) && d.K % 4) return false;
  // byte offsets of a tile inside its operands' views stay below 2^31
  const long long a_span = d.a_kcontig ? (long long)f32::TILE * d.lda + d.K : (long long)(d.K + 8 * f32::BK) * d.lda + f32::TILE;
  const long long b_span = d.b_kcontig ? (long long)f32::TILE * d.ldb + d.K : (long long)(d.K + 8 * f32::BK) * d.ldb + f32::TILE;
  return 4 * a_span < 0x7fffff00LL && 4 * b_span < 0x7fffff00LL;
}

// Few tiles and a long contraction: split k.  A slab takes about 0.69 us while a compute unit has one workgroup and 0.60
// per workgroup once it has more; the parts cost a second launch of about 4 us and their way through memory.  Measured, us,
// by parts 1 / 2 / 3 / 4: 1024x768x3072 68 / 64 / 69 / 55, 1024x768x768 22 / 25 / 29 / 25, 1024x3072x768 52 / 63 / 69 / 74.
int f32_splitk(int M, int N, int K, size_t partial_floats) {
  const int tiles = ((M + f32::TILE - 1) / f32::TILE) * ((N + f32::TILE - 1) / f32::TILE), slabs = (K + f32::BK - 1) / f32::BK;
  double best = 0.0;
  int pick = 1;
  for (int s = 1; s <= 64 && (s == 1 || slabs / s >= 4); ++s) {
    if (s > 1 && ((long long)tiles * s > 1024 || (size_t)s * M * N > partial_floats)) break;
    const int turns = (tiles * s + 255) / 256 * ((slabs + s - 1) / s);
    const double t = turns * (tiles * s <= 256 ? 0.69 : 0.60) + (s > 1 ? 4.0 + (double)s * M * N * 8.0 / 4.0e6 : 0.0);
    if (s == 1 || t < best) { best = t; pick = s; }
  }
  return pick;
}

// Where the guarded kernel is the faster one.  512 workgroups of this kernel are resident (80 KB of LDS each) and five or
// more of the guarded one to a compute unit; a workgroup here starts with a ring to fill and ends with two sums to add.  So many
// tiles of a short contraction run longer here, and so do parts of a split that hold a few slabs or start a second round.
// This kernel / guarded, us: 3072x768, contraction 32 13.7 / 9.3, 128 17.5 / 15.5, 256 24.7 / 23.6, 304 (30592x768) 179 / 162,
// 384 32 / 32; 30592x768x20 77 / 44; 2304x768x32 (432 tiles) 9.6 / 8.2; in parts, 256x768x768 in five 12.6 / 11.5,
// 128x128x512 in four 8.9 / 8.5, 4x768x30592 in 64 51 / 41.  On the other side: 2304x768x128 11.8 / 12.3, 768x768x128 7.9 / 8.6,
// 1536x512x2048 43 / 57 (the guarded rule leaves it whole).
bool gemm_f32_pays(const GemmDesc& d, int splitk, int guarded_splitk) {
  const int tiles = ((d.M + f32::TILE - 1) / f32::TILE) * ((d.N + f32::TILE - 1) / f32::TILE), slabs = (d.K + f32::BK - 1) / f32::BK;
  if (splitk == 1) return !(tiles > 512 && slabs <= 10) && !(tiles > 384 && slabs == 1);
  return splitk != guarded_splitk || ((long long)tiles * splitk <= 512 && (slabs + splitk - 1) / splitk > 5);
}

hipError_t gemm_f32(const GemmDesc& d, int splitk, float* partials, hipStream_t s) {
  if (!gemm_f32_supported(d) || splitk < 1 || (splitk > 1 && !partials)) return hipErrorInvalidValue;
  hipError_t e;
  if (d.a_kcontig && d.b_kcontig) e = f32::launch<true, true>(d, splitk, partials, s);
  else if (d.a_kcontig) e = f32::launch<true, false>(d, splitk, partials, s);
  else if (d.b_kcontig) e = f32::launch<false, true>(d, splitk, partials, s);
  else e = f32::launch<false, false>(d, splitk, partials, s);
  if (e != hipSuccess || splitk == 1) return e;
  return guarded_reduce_f32(partials, splitk, d.M, d.N, d.epi, s);
}

}  // namespace mslt

// Large-tile bf16 MFMA GEMMs for gfx950 whose wavefronts take turns: C(m,n) = sum_k A(m,k) B(n,k), fp32 accumulation,
// shared epilogue.
//
// Eight wavefronts own a tile, two on each SIMD, as two groups one half step apart: while one group multiplies, the
// other fetches its next fragments from LDS and queues loads, so that a SIMD's matrix core and its memory pipes are both
// in use at any time.  A step of a wavefront is [queue loads, read fragments, wait for both the fragments and the loads
// the next step reads] barrier [multiply] barrier, and the second group starts one barrier late.  In the kernel where
// all wavefronts do the same thing at the same time (gemm_ring.hip) the matrix cores wait for every fragment read: there
// 8192x8192x8192 takes 842 us, here 757 (weight gradient 4096x3072x8192 183 and 169).
//
// Operands go global memory -> LDS directly (16 bytes per lane), into slots of 128 rows x 64 k (16 KB) that are refilled
// as soon as both groups have read them, so that the loads in flight cover one and a half k tiles or more.  In LDS a
// k-contiguous operand is [rows][64 k] with the 16-byte chunks of a row XOR-swizzled by the row; a k-strided one (the
// weight in dX = dY W, both operands in dW = dY^T X) is [64 k][rows] as it lies, read through the transposing read.
// Fragments are read in inline assembly: through the compiler every read would wait for the loads into LDS in flight.
// Each block of reads ends with its own wait.
//
// Products are formed transposed, so that a lane holds four consecutive columns of a row: bias (it is what the
// accumulators start from: as part of the epilogue its loads took 9 us per tile; a step's products with a bias have bf16
// results, whose error is 1.66e-3 either way), GELU and dropout work on registers, and
// a result goes through LDS in its final type, 16 bytes per lane and whole cache lines per store (stores straight from
// the registers, 32 bytes per row, took 4 us longer per tile).
//
// Tiles, and what they are for (us, this tile / the best tile of gemm_ring.hip; all shapes and tiles side by side stand at
// tile_plan in model.hip):
//   256x256 (k_gemm_phase): 8192x4096x1024 64 / 69; any operand layout.
//   256x384 (k_gemm_wide): one round of workgroups where 256x256 tiles leave a second one half empty: 8192x3072x768 38 / 48,
//     8192x3072x1024 47 / 58, 8192x2304x768 33 / 42.
//   256x128, four wavefronts, two workgroups on a compute unit (k_gemm_pair): outputs no multiple of 256 wide, 1280x30592x768 64 / 75.
//   128x192 (k_gemm_slim): narrow outputs beside another chain of kernels.
// M need not be a multiple of the tile (of anything, when A is k-contiguous): rows past the end are neither read nor written.
#include "common.h"
#include "gemm_epilogue.h"
#include <type_traits>

namespace mslt {

namespace phase {

typedef __attribute__((ext_vector_type(4))) short s16x4_t;

struct Params {
  const bf16* A;
  const bf16* B;
  int M, N, K;       // K = contraction length of this launch (all splits together)
  int lda, ldb;
  int splitk;
  int tiles_m, tiles_n;
  float* partials;   // [splitk][M][N] when splitk > 1
  Epilogue epi;
};

constexpr int SLOT = 16384;            // 128 rows x 64 k
constexpr int PHASE_SLOTS = 8, PAIR_SLOTS = 5, WIDE_SLOTS = 10;
// s_waitcnt immediate: vmcnt <= vm, the other counters as given (15: untouched)
constexpr int waitcnt_imm(int vm, int lgkm) { return (vm & 15) | 0x70 | ((vm >> 4) << 14) | (lgkm << 8); }

// ---- which tile ---------------------------------------------------------------------------------
// wg: the workgroup's index among the product's workgroups (a range of a grouped launch starts at a multiple of 8, so
// wg % 8 is the XCD in either case).  Each XCD gets a contiguous range of tiles, ordered in bands of 8 tile rows, column
// by column inside a band: the tiles that run together on an XCD share few operand panels in its L2.
struct Place {
  int m0, n0, split, kbeg, nk;
};
template <int TM, int TN>
__device__ __forceinline__ bool place(const Params& p, int wg, Place* o) {
  const int total = p.tiles_m * p.tiles_n * p.splitk;
  if (wg >= total) return false;      // padding of a grouped launch
  const int per = (total + 7) >> 3, tall = (total & 7) ? total & 7 : 8;
  const int xcd = wg & 7, local = wg >> 3;
  const int pid = xcd < tall ? xcd * per + local : tall * per + (xcd - tall) * (per - 1) + local;
  const int tiles = p.tiles_m * p.tiles_n;
  o->split = pid / tiles;
  const int tile = pid - o->split * tiles;
  constexpr int G = 8;
  const int band = tile / (G * p.tiles_n), first = band * G;
  const int rows = p.tiles_m - first < G ? p.tiles_m - first : G;
  const int in_band = tile - band * G * p.tiles_n;
  o->m0 = (first + in_band % rows) * TM;
  o->n0 = in_band / rows * TN;
  const int nkt = p.K / 64;
  const int lo = (int)((long long)o->split * nkt / p.splitk);
  o->kbeg = lo * 64;
  o->nk = (int)((long long)(o->split + 1) * nkt / p.splitk) - lo;
  return true;
}

// ---- operands: global memory -> LDS ---------------------------------------------------------------
// A view of one operand from the tile's first row (k-contiguous: [rows][ld]; k-strided: column row0 of [k][ld]).  Its
// size ends with the operand's last element, so rows past the end are read as zeros and cost no traffic; a k tile past
// the end is loaded through a view of size 0, which keeps the count of loads in flight the same in every step.
struct View {
  const bf16* base;
  int bytes;
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(bool in_range) const {
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, in_range ? bytes : 0, 0x00020000);
  }
};
template <bool KC>
__device__ __forceinline__ View view(const bf16* p, int ld, int row0, int rows, int K) {
  const long long bytes = KC ? ((long long)(rows - row0 - 1) * ld + K) * 2 : ((long long)(K - 1) * ld + rows - row0) * 2;
  return View{KC ? p + (size_t)row0 * ld : p + row0, (int)(bytes < 0x7fffffff ? bytes : 0x7fffffff)};
}
// One load moves 64 lanes x 16 bytes into 1024 consecutive LDS bytes (lane i lands at base + 16 i); which chunk a lane
// fetches is free, which is where the swizzles live.  Of a slot, wavefront w moves the IPW pieces IPW w .. IPW w + IPW - 1.
//   k-contiguous, [128 rows][64 k]: piece q is rows 8q .. 8q+7; lane -> row 8q + lane/8, place lane%8, which holds chunk
//     place ^ ((row>>1)&7).
//   k-strided, [64 k][128 rows]: piece q is k rows 4q .. 4q+3; chunk c of k row k sits in place c ^ ((k&3)<<2).
template <bool KC, int IPW = 2>
struct Mover {
  int voff[2];     // per-lane byte offset of even / odd pieces
  __device__ __forceinline__ void init(int lane, int ld) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if constexpr (KC) voff[j] = ((lane >> 3) * ld + 8 * ((lane & 7) ^ ((4 * j + (lane >> 4)) & 7))) * 2;
      else voff[j] = (lane >> 4) * ld * 2 + (((lane & 15) ^ ((lane >> 4) << 2)) << 4);
    }
  }
  // rows 128 half .. +127, k0 .. k0 + 63 of the view into `slot`
  __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t rsrc, int ld, int half, int k0, int wave, unsigned char* slot) const {
    static_assert(IPW % 2 == 0, "piece parity follows j");
#pragma unroll
    for (int j = 0; j < IPW; ++j) {
      const int q = wave * IPW + j;
      const int soff = KC ? ((q * 8 + 128 * half) * ld + k0) * 2 : ((k0 + q * 4) * ld + 128 * half) * 2;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_t*)(slot + q * 1024), 16, voff[j & 1], soff, 0, 0);
    }
  }
};

// ---- LDS -> fragments -----------------------------------------------------------------------------
// Fragment of v_mfma_f32_32x32x16_bf16: lane l holds row l%32, k = 8*(l/32) .. +7 of a 32 x 16 block.
__device__ __forceinline__ bf16x8_t join(s16x4_t lo, s16x4_t hi) {
  struct { s16x4_t lo, hi; } w{lo, hi};
  return __builtin_bit_cast(bf16x8_t, w);
}
// lane part of the address of 16-wide step s of row row_base + lane % 32 (rows of 128 bytes)
__device__ __forceinline__ unsigned kc_off(int lane, int row_base, int s) {
  return (unsigned)((row_base + (lane & 31)) * 128 + (((2 * s + (lane >> 5)) ^ ((lane >> 1) & 7)) << 4));
}
// the same of the 32 rows from `row_base` for the transposing read (k rows of 256 bytes): sixteen lanes that fetch four
// consecutive rows of four k receive four consecutive k of one row
__device__ __forceinline__ unsigned tr_off(int lane, int row_base) {
  const int blk = lane >> 4, j = lane & 15;
  const int e = row_base + 16 * (blk & 1) + 4 * (j & 3);      // first of this lane's four rows
  return (unsigned)(2 * ((8 * (blk >> 1) + (j >> 2)) * 128 + (((e >> 3) ^ ((j >> 2) << 2)) << 3) + (e & 7)));
}
// NBLK blocks of 32 rows x 64 k of a slot: f[block][16-wide step]
template <bool KC, int NBLK>
struct Frags {
  unsigned off[KC ? 4 : NBLK];
  __device__ __forceinline__ void init(int lane, int row_base, unsigned lds_base) {
#pragma unroll
    for (int i = 0; i < (KC ? 4 : NBLK); ++i) off[i] = lds_base + (KC ? kc_off(lane, row_base, i) : tr_off(lane, row_base + 32 * i));
  }
  __device__ __forceinline__ void read(unsigned slot, bf16x8_t (&f)[NBLK][4]) const {
    if constexpr (KC && NBLK == 1) {
      asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(f[0][0]), "=&v"(f[0][1]), "=&v"(f[0][2]), "=&v"(f[0][3])
                   : "v"(off[0] + slot), "v"(off[1] + slot), "v"(off[2] + slot), "v"(off[3] + slot) : "memory");
    } else if constexpr (KC) {
      asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %4, %8 offset:4096\n\tds_read_b128 %1, %9\n\tds_read_b128 %5, %9 offset:4096\n\t"
                   "ds_read_b128 %2, %10\n\tds_read_b128 %6, %10 offset:4096\n\tds_read_b128 %3, %11\n\tds_read_b128 %7, %11 offset:4096\n\t"
                   "s_waitcnt lgkmcnt(0)"
                   : "=&v"(f[0][0]), "=&v"(f[0][1]), "=&v"(f[0][2]), "=&v"(f[0][3]),
                     "=&v"(f[NBLK - 1][0]), "=&v"(f[NBLK - 1][1]), "=&v"(f[NBLK - 1][2]), "=&v"(f[NBLK - 1][3])
                   : "v"(off[0] + slot), "v"(off[1] + slot), "v"(off[2] + slot), "v"(off[3] + slot) : "memory");
    } else if constexpr (NBLK == 1) {
      s16x4_t v[8];
      asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:1024\n\t"
                   "ds_read_b64_tr_b16 %2, %8 offset:4096\n\tds_read_b64_tr_b16 %3, %8 offset:5120\n\t"
                   "ds_read_b64_tr_b16 %4, %8 offset:8192\n\tds_read_b64_tr_b16 %5, %8 offset:9216\n\t"
                   "ds_read_b64_tr_b16 %6, %8 offset:12288\n\tds_read_b64_tr_b16 %7, %8 offset:13312\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                   : "v"(off[0] + slot) : "memory");
#pragma unroll
      for (int s = 0; s < 4; ++s) f[0][s] = join(v[2 * s], v[2 * s + 1]);
    } else {
      s16x4_t v[2][8];
      asm volatile("ds_read_b64_tr_b16 %0, %16\n\tds_read_b64_tr_b16 %1, %16 offset:1024\n\t"
                   "ds_read_b64_tr_b16 %8, %17\n\tds_read_b64_tr_b16 %9, %17 offset:1024\n\t"
                   "ds_read_b64_tr_b16 %2, %16 offset:4096\n\tds_read_b64_tr_b16 %3, %16 offset:5120\n\t"
                   "ds_read_b64_tr_b16 %10, %17 offset:4096\n\tds_read_b64_tr_b16 %11, %17 offset:5120\n\t"
                   "ds_read_b64_tr_b16 %4, %16 offset:8192\n\tds_read_b64_tr_b16 %5, %16 offset:9216\n\t"
                   "ds_read_b64_tr_b16 %12, %17 offset:8192\n\tds_read_b64_tr_b16 %13, %17 offset:9216\n\t"
                   "ds_read_b64_tr_b16 %6, %16 offset:12288\n\tds_read_b64_tr_b16 %7, %16 offset:13312\n\t"
                   "ds_read_b64_tr_b16 %14, %17 offset:12288\n\tds_read_b64_tr_b16 %15, %17 offset:13312\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(v[0][0]), "=&v"(v[0][1]), "=&v"(v[0][2]), "=&v"(v[0][3]), "=&v"(v[0][4]), "=&v"(v[0][5]), "=&v"(v[0][6]), "=&v"(v[0][7]),
                     "=&v"(v[1][0]), "=&v"(v[1][1]), "=&v"(v[1][2]), "=&v"(v[1][3]), "=&v"(v[1][4]), "=&v"(v[1][5]), "=&v"(v[1][6]), "=&v"(v[1][7])
                   : "v"(off[0] + slot), "v"(off[KC ? 0 : NBLK - 1] + slot) : "memory");
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int s = 0; s < 4; ++s) f[i][s] = join(v[i][2 * s], v[i][2 * s + 1]);
    }
  }
};

__device__ __forceinline__ void meet() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// ---- how a tile ends ------------------------------------------------------------------------------
// chosen once per workgroup, so that a strip carries the code of one way only
enum { FIN_PLAIN, FIN_GELU, FIN_GELU_GRAD, FIN_DROP, FIN_STAGED, FIN_STAGED_EXTRAS };
constexpr int strip_bytes(int NBLK) {      // LDS of a wavefront: one fp32 strip, or two in bf16 (value and GELU derivative)
  const int f32 = 32 * (32 * NBLK + 4) * 4, b16 = 2 * 32 * (32 * NBLK + 8) * 2;
  return f32 > b16 ? f32 : b16;
}
// 32 rows x 32 NBLK columns from transposed accumulators: lane = row m + lane % 32, register r of block j = column
// n + 32 j + 8 (r / 4) + 4 (lane / 32) + r % 4; rows from m_end on are left alone
template <int FIN, int NBLK>
__device__ __forceinline__ void finish_strip(const Epilogue& e, const f32x16_t (&c)[NBLK], int m, int n, int m_end, int lane, unsigned char* stage) {
  constexpr int CHUNKS = 4 * NBLK;      // eight columns each
  const int half = lane >> 5, r32 = lane & 31;
  if constexpr (FIN <= FIN_DROP) {
    constexpr int LD = 32 * NBLK + 8;
    bf16* st = reinterpret_cast<bf16*>(stage);
#pragma unroll
    for (int j = 0; j < NBLK; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int col = 32 * j + 8 * g + 4 * half;
        float v[4] = {c[j][4 * g], c[j][4 * g + 1], c[j][4 * g + 2], c[j][4 * g + 3]};
        if constexpr (FIN == FIN_DROP) {
          const uint64_t q = drop_quad(e.drop, ((uint64_t)(m + r32) * e.drop_ld + n + col) >> 2);
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] *= drop_field(e.drop, q, i);
        }
        if constexpr (FIN == FIN_GELU_GRAD) {
          float d[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) gelu_both_fast(v[i], v[i], d[i]);
          *reinterpret_cast<u32x2_t*>(st + (32 + r32) * LD + col) =
              u32x2_t{enc_dgelu(d[0]) | (enc_dgelu(d[1]) << 16), enc_dgelu(d[2]) | (enc_dgelu(d[3]) << 16)};
        } else if constexpr (FIN == FIN_GELU) {
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = gelu_fast(v[i]);
        }
        *reinterpret_cast<u32x2_t*>(st + r32 * LD + col) = u32x2_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
      }
#pragma unroll
    for (int i = 0; i < 2 * NBLK; ++i) {
      const int x = 64 * i + lane, row = x / CHUNKS, cc = 8 * (x % CHUNKS);
      if (m + row >= m_end) continue;
      const size_t o = (size_t)(m + row) * e.ldo + n + cc;
      if constexpr (FIN == FIN_GELU_GRAD)
        *reinterpret_cast<u32x4_t*>(reinterpret_cast<bf16*>(e.out2) + o) = *reinterpret_cast<const u32x4_t*>(st + (32 + row) * LD + cc);
      *reinterpret_cast<u32x4_t*>(reinterpret_cast<bf16*>(e.out) + o) = *reinterpret_cast<const u32x4_t*>(st + row * LD + cc);
    }
  } else {
    constexpr int LD = 32 * NBLK + 4;
    float* st = reinterpret_cast<float*>(stage);
    uint4 raw[2 * NBLK];
#pragma unroll
    for (int i = 0; i < 2 * NBLK; ++i) raw[i] = make_uint4(0, 0, 0, 0);
    if (epilogue_reads_aux(e)) {
#pragma unroll
      for (int i = 0; i < 2 * NBLK; ++i) {
        const int x = 64 * i + lane, row = m + x / CHUNKS;
        if (row < m_end) raw[i] = load_aux8(e, row, n + 8 * (x % CHUNKS));
      }
    }
#pragma unroll
    for (int j = 0; j < NBLK; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<float4*>(st + r32 * LD + 32 * j + 8 * g + 4 * half) =
            make_float4(c[j][4 * g], c[j][4 * g + 1], c[j][4 * g + 2], c[j][4 * g + 3]);
    const float bias[8] = {0, 0, 0, 0, 0, 0, 0, 0};      // already in the accumulators
#pragma unroll
    for (int i = 0; i < 2 * NBLK; ++i) {
      const int x = 64 * i + lane, row = x / CHUNKS, cc = 8 * (x % CHUNKS);
      if (m + row >= m_end) continue;
      const float4 x0 = *reinterpret_cast<const float4*>(st + row * LD + cc), x1 = *reinterpret_cast<const float4*>(st + row * LD + cc + 4);
      float v[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
      epilogue8<FIN == FIN_STAGED_EXTRAS>(e, m + row, n + cc, v, bias, raw[i]);
    }
  }
}
// start value of the accumulators of a 32-column block: the bias of the lane's columns, or zero
__device__ __forceinline__ void start_block(const float* bias, int n, int lane, f32x16_t& c) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    float4 b = make_float4(0.f, 0.f, 0.f, 0.f);
    if (bias) b = *reinterpret_cast<const float4*>(bias + n + 8 * g + 4 * (lane >> 5));
    c[4 * g] = b.x; c[4 * g + 1] = b.y; c[4 * g + 2] = b.z; c[4 * g + 3] = b.w;
  }
}
// the epilogue of this launch, or the plain store of a split's partial sums
__device__ __forceinline__ Epilogue epilogue_of(const Params& p, int split) {
  if (p.splitk == 1) return p.epi;
  Epilogue e;
  e.out = p.partials + (size_t)split * p.M * p.N;
  e.ldo = p.N;
  e.out_f32 = 1;
  return e;
}
// calls strips(tag) with the way this epilogue ends a strip; EXTRAS: also accumulation and dropout in other places than
// before a plain bf16 result, which only the weight-gradient form carries (accumulation is what a step asks of it)
template <bool EXTRAS, typename F>
__device__ __forceinline__ void finish_tile(const Epilogue& e, F strips) {
  const bool direct = !e.out_f32 && (e.act == EPI_NONE || (e.act == EPI_GELU && !e.drop.thr));
  if (direct && e.act == EPI_GELU) {
    if (e.out2) strips(std::integral_constant<int, FIN_GELU_GRAD>());
    else strips(std::integral_constant<int, FIN_GELU>());
  } else if (direct) {
    if (e.drop.thr) strips(std::integral_constant<int, FIN_DROP>());
    else strips(std::integral_constant<int, FIN_PLAIN>());
  } else {
    if constexpr (EXTRAS) {
      if (e.drop.thr || e.accumulate) return strips(std::integral_constant<int, FIN_STAGED_EXTRAS>());
    }
    strips(std::integral_constant<int, FIN_STAGED>());
  }
}

// ---- 256 x 256 ------------------------------------------------------------------------------------
// (A step takes this tile with a k-contiguous A, and in the grouped launch.  The split of the contraction and the layout with
// only B k-contiguous serve the measurements and tests that pick a tile themselves.)
// Wavefront (wm, wn) of 4 x 2 owns rows 32 wm .. of both A halves and columns 64 wn .. of both B halves.  Halves are used
// in the order A0 B0 A1 B1 (tile 0), A0 B0 ... (tile 1); half number s lies in slot s % 8.  Step 2 t reads B0, A1 and
// multiplies B0 with both A halves, step 2 t + 1 reads B1 and the next tile's A0 and multiplies B1 with both: sixteen
// matrix instructions behind twelve 16-byte reads each time.  (Eight behind eight and four: 3 % slower at K = 1024, 2 %
// faster at K = 8192; ten slots: 5 % slower.)
template <bool A_KC, bool B_KC>
__device__ __forceinline__ void phase_tile(const Params& p, const int wg) {
  constexpr int R = PHASE_SLOTS;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const unsigned lds_base = (unsigned)(uintptr_t)(lds_void_t*)smem;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  Place at;
  if (!place<256, 256>(p, wg, &at)) return;
  const View va = view<A_KC>(p.A, p.lda, at.m0, p.M, p.K), vb = view<B_KC>(p.B, p.ldb, at.n0, p.N, p.K);
  Mover<A_KC> ma; ma.init(lane, p.lda);
  Mover<B_KC> mb; mb.init(lane, p.ldb);
  Frags<A_KC, 1> fa; fa.init(lane, 32 * wm, lds_base);
  Frags<B_KC, 2> fb; fb.init(lane, 64 * wn, lds_base);

  f32x16_t acc[2][2][2];     // [A half][B half][32-column block]
  const float* const bias = p.splitk > 1 ? nullptr : p.epi.bias;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      start_block(bias, at.n0 + 128 * j + 64 * wn + 32 * b, lane, acc[0][j][b]);
      acc[1][j][b] = acc[0][j][b];
    }

  auto issue = [&](int kind, int t, unsigned slot) {
    if ((kind & 1) == 0) ma.issue(va.rsrc(t < at.nk), p.lda, kind >> 1, at.kbeg + t * 64, wave, smem + slot);
    else mb.issue(vb.rsrc(t < at.nk), p.ldb, kind >> 1, at.kbeg + t * 64, wave, smem + slot);
  };
  bf16x8_t a0[2][1][4], a1[1][4], b[2][4];
  auto mfma = [&](const bf16x8_t (&a)[1][4], f32x16_t (&c)[2]) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int j = 0; j < 2; ++j) c[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j][s], a[0][s], c[j], 0, 0, 0);
  };
#pragma unroll
  for (int q = 0; q < R - 1; ++q) issue(q & 3, q >> 2, q * SLOT);
  // Entering a step's fetch all halves up to the two it reads have landed; of the R - 4 behind them some may be in
  // flight (two loads a half and wavefront).  A slot is refilled one step after it was read, when both groups are done.
  constexpr int WAIT = waitcnt_imm(2 * (R - 4), 15);
  __builtin_amdgcn_s_waitcnt(WAIT);
  meet();
  fa.read(0, a0[0]);
  meet();
  unsigned wr = (R - 1) * SLOT, rd = SLOT;
  auto adv = [](unsigned& x) { x = x == (R - 1) * SLOT ? 0 : x + SLOT; };
  const bool second = wave >= 4;
  if (second) meet();
  auto k_tile = [&](int t, bf16x8_t (&ac)[1][4], bf16x8_t (&an)[1][4]) {
    issue((R + 3) & 3, t + ((R + 3) >> 2) - 1, wr); adv(wr);
    issue(R & 3, t + (R >> 2), wr); adv(wr);
    fb.read(rd, b); adv(rd);
    fa.read(rd, a1); adv(rd);
    __builtin_amdgcn_s_waitcnt(WAIT);
    meet();
    __builtin_amdgcn_s_setprio(1);
    mfma(ac, acc[0][0]);
    mfma(a1, acc[1][0]);
    __builtin_amdgcn_s_setprio(0);
    meet();
    issue((R + 1) & 3, t + ((R + 1) >> 2), wr); adv(wr);
    issue((R + 2) & 3, t + ((R + 2) >> 2), wr); adv(wr);
    fb.read(rd, b); adv(rd);
    fa.read(rd, an); adv(rd);
    __builtin_amdgcn_s_waitcnt(WAIT);
    meet();
    __builtin_amdgcn_s_setprio(1);
    mfma(a1, acc[1][1]);
    mfma(ac, acc[0][1]);
    __builtin_amdgcn_s_setprio(0);
    meet();
  };
  int t = 0;
  for (; t + 2 <= at.nk; t += 2) {
    k_tile(t, a0[0], a0[1]);
    k_tile(t + 1, a0[1], a0[0]);
  }
  if (t < at.nk) k_tile(t, a0[0], a0[1]);
  if (!second) meet();
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));   // the loads past the end still write zeros
  __syncthreads();

  const Epilogue e = epilogue_of(p, at.split);
  unsigned char* stage = smem + wave * strip_bytes(2);
  finish_tile<!A_KC && !B_KC>(e, [&](auto fin) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int m = at.m0 + 128 * i + 32 * wm;
      if (m < p.M) {
#pragma unroll
        for (int j = 0; j < 2; ++j) finish_strip<decltype(fin)::value, 2>(e, acc[i][j], m, at.n0 + 128 * j + 64 * wn, p.M, lane, stage);
      }
    }
  });
}
template <bool A_KC, bool B_KC>
__global__ void __launch_bounds__(512) k_gemm_phase(Params p) { phase_tile<A_KC, B_KC>(p, (int)blockIdx.x); }

// Several weight-gradient products (both operands k-strided) in one launch: product g owns the workgroups
// first[g] .. first[g+1]-1.  Products too small to fill the chip one by one then need no split of their contraction.
constexpr int GROUP_MAX = 4;
struct GroupParams {
  Params p[GROUP_MAX];
  int first[GROUP_MAX + 1];
  int n;
};
__global__ void __launch_bounds__(512) k_gemm_phase_grouped(GroupParams gp) {
  int g = 0;
  while (g + 1 < gp.n && (int)blockIdx.x >= gp.first[g + 1]) ++g;
  phase_tile<false, false>(gp.p[g], (int)blockIdx.x - gp.first[g]);
}

// ---- 256 x 384 ------------------------------------------------------------------------------------
// Wavefront (wm, wn) of 4 x 2 owns rows 32 wm .. of both A halves and columns 64 wn .. of the three B thirds, 192
// accumulator registers; what is left holds the fragments of 32 k of 64 rows of either operand.  A k tile is the slots
// A0 A1 B0 B1 B2, two k tiles fill the LDS.  It is gone through twice, k 0..31 and 32..63: in a pass the A fragments are
// read with the first third.  Slots are refilled in the second pass, behind the step that reads them last.
template <bool KC>
struct HalfFrags {      // two 32-row blocks, `apart` bytes from each other, x 32 k: f[block][step]
  unsigned off[KC ? 4 : 2];
  __device__ __forceinline__ void init(int lane, int row0, int row1, int apart, unsigned lds_base) {
    if constexpr (KC) {
#pragma unroll
      for (int s = 0; s < 4; ++s) off[s] = lds_base + kc_off(lane, row0, s);
    } else {
      off[0] = lds_base + tr_off(lane, row0);
      off[1] = lds_base + tr_off(lane, row1) + apart;
    }
  }
  template <int PASS, int APART>      // APART: bytes between the blocks when k-contiguous
  __device__ __forceinline__ void read(unsigned slot, bf16x8_t (&f)[2][2]) const {
    if constexpr (KC) {
      asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %4 offset:%6\n\tds_read_b128 %3, %5 offset:%6\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(f[0][0]), "=&v"(f[0][1]), "=&v"(f[1][0]), "=&v"(f[1][1])
                   : "v"(off[2 * PASS] + slot), "v"(off[2 * PASS + 1] + slot), "n"(APART) : "memory");
    } else {
      s16x4_t v[8];
      asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:1024\n\tds_read_b64_tr_b16 %2, %8 offset:4096\n\tds_read_b64_tr_b16 %3, %8 offset:5120\n\t"
                   "ds_read_b64_tr_b16 %4, %9\n\tds_read_b64_tr_b16 %5, %9 offset:1024\n\tds_read_b64_tr_b16 %6, %9 offset:4096\n\tds_read_b64_tr_b16 %7, %9 offset:5120\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                   : "v"(off[0] + slot + 8192 * PASS), "v"(off[1] + slot + 8192 * PASS) : "memory");
#pragma unroll
      for (int i = 0; i < 4; ++i) f[i >> 1][i & 1] = join(v[2 * i], v[2 * i + 1]);
    }
  }
};
template <bool B_KC>
__global__ void __launch_bounds__(512) k_gemm_wide(Params p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const unsigned lds_base = (unsigned)(uintptr_t)(lds_void_t*)smem;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  Place at;
  if (!place<256, 384>(p, (int)blockIdx.x, &at)) return;
  const View va = view<true>(p.A, p.lda, at.m0, p.M, p.K), vb = view<B_KC>(p.B, p.ldb, at.n0, p.N, p.K);
  Mover<true> ma; ma.init(lane, p.lda);
  Mover<B_KC> mb; mb.init(lane, p.ldb);
  HalfFrags<true> fa; fa.init(lane, 32 * wm, 0, 0, lds_base);
  HalfFrags<B_KC> fb; fb.init(lane, 64 * wn, 64 * wn + 32, 0, lds_base);

  f32x16_t acc[2][3][2];     // [A half][B third][32-column block]
#pragma unroll
  for (int j = 0; j < 3; ++j)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      start_block(p.epi.bias, at.n0 + 128 * j + 64 * wn + 32 * b, lane, acc[0][j][b]);
      acc[1][j][b] = acc[0][j][b];
    }

  auto issue = [&](int what, int t, unsigned buf) {     // 0, 1: A halves; 2 .. 4: B thirds
    if (what < 2) ma.issue(va.rsrc(t < at.nk), p.lda, what, t * 64, wave, smem + buf + what * SLOT);
    else mb.issue(vb.rsrc(t < at.nk), p.ldb, what - 2, t * 64, wave, smem + buf + what * SLOT);
  };
  bf16x8_t a[2][2], b[2][2];
  auto multiply = [&](int j) {
    meet();
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int x = 0; x < 2; ++x) acc[i][j][x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[x][s], a[i][s], acc[i][j][x], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    meet();
  };
  constexpr unsigned BUF = 5 * SLOT;
#pragma unroll
  for (int w = 0; w < 5; ++w) issue(w, 0, 0);
#pragma unroll
  for (int w = 0; w < 4; ++w) issue(w, 1, BUF);
  // what the next step reads has landed when at most so many loads are in flight (two a slot and wavefront)
  constexpr int SIX = waitcnt_imm(12, 15), FIVE = waitcnt_imm(10, 15);
  __builtin_amdgcn_s_waitcnt(SIX);
  meet();
  const bool second = wave >= 4;
  if (second) meet();
  unsigned cur = 0;
  int t = 0;
  do {
    issue(4, t + 1, BUF - cur);
    fa.template read<0, SLOT>(cur, a);
    fb.template read<0, 4096>(cur + 2 * SLOT, b);
    __builtin_amdgcn_s_waitcnt(SIX);
    multiply(0);
    fb.template read<0, 4096>(cur + 3 * SLOT, b);
    __builtin_amdgcn_s_waitcnt(FIVE);
    multiply(1);
    fb.template read<0, 4096>(cur + 4 * SLOT, b);
    multiply(2);
    fa.template read<1, SLOT>(cur, a);
    fb.template read<1, 4096>(cur + 2 * SLOT, b);
    multiply(0);
    issue(0, t + 2, cur);
    issue(1, t + 2, cur);
    fb.template read<1, 4096>(cur + 3 * SLOT, b);
    multiply(1);
    issue(2, t + 2, cur);
    issue(3, t + 2, cur);
    fb.template read<1, 4096>(cur + 4 * SLOT, b);
    __builtin_amdgcn_s_waitcnt(SIX);
    multiply(2);
    cur = BUF - cur;
  } while (++t < at.nk);
  if (!second) meet();
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
  __syncthreads();

  unsigned char* stage = smem + wave * strip_bytes(2);
  finish_tile<false>(p.epi, [&](auto fin) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int m = at.m0 + 128 * i + 32 * wm;
      if (m < p.M) {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          finish_strip<decltype(fin)::value, 2>(p.epi, acc[i][j], m, at.n0 + 128 * j + 64 * wn, p.M, lane, stage);
          __builtin_amdgcn_sched_barrier(0);       // one strip's registers at a time: the accumulators leave few
        }
      }
    }
  });
}

// ---- 256 x 128, two workgroups on a compute unit ----------------------------------------------------
// Four wavefronts, each 64 rows of both A halves x 64 columns; a k tile is the halves B A0 A1, five slots.  The groups
// that take turns are the two workgroups, so one barrier a step is enough here.
template <bool A_KC, bool B_KC>
__global__ void __launch_bounds__(256, 2) k_gemm_pair(Params p) {
  constexpr int R = PAIR_SLOTS;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const unsigned lds_base = (unsigned)(uintptr_t)(lds_void_t*)smem;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  Place at;
  if (!place<256, 128>(p, (int)blockIdx.x, &at)) return;
  const View va = view<A_KC>(p.A, p.lda, at.m0, p.M, p.K), vb = view<B_KC>(p.B, p.ldb, at.n0, p.N, p.K);
  Mover<A_KC, 4> ma; ma.init(lane, p.lda);
  Mover<B_KC, 4> mb; mb.init(lane, p.ldb);
  Frags<A_KC, 2> fa; fa.init(lane, 64 * wm, lds_base);
  Frags<B_KC, 2> fb; fb.init(lane, 64 * wn, lds_base);
  f32x16_t acc[2][2][2];     // [A half][32-row block][32-column block]
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    start_block(p.epi.bias, at.n0 + 64 * wn + 32 * x, lane, acc[0][0][x]);
    acc[0][1][x] = acc[1][0][x] = acc[1][1][x] = acc[0][0][x];
  }
  auto issue = [&](int kind, int t, unsigned slot) {      // 0: B; 1, 2: A halves
    if (kind == 0) mb.issue(vb.rsrc(t < at.nk), p.ldb, 0, t * 64, wave, smem + slot);
    else ma.issue(va.rsrc(t < at.nk), p.lda, kind - 1, t * 64, wave, smem + slot);
  };
  bf16x8_t a[2][4], b[2][4];
  auto gate = [&]() {      // the halves the next step reads have landed, with two more (four loads each) in flight
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(8, 15));
    meet();
  };
  auto multiply = [&](f32x16_t (&c)[2][2]) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int x = 0; x < 2; ++x) c[i][x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[x][s], a[i][s], c[i][x], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int q = 0; q < 4; ++q) issue(q % 3, q / 3, q * SLOT);
  unsigned wr = 4 * SLOT, rd = 0;
  auto adv = [](unsigned& x) { x = x == (R - 1) * SLOT ? 0 : x + SLOT; };
  for (int t = 0; t < at.nk; ++t) {
    gate();
    issue(1, t + 1, wr); adv(wr);
    fb.read(rd, b); adv(rd);
    fa.read(rd, a); adv(rd);
    multiply(acc[0]);
    gate();
    issue(2, t + 1, wr); adv(wr);
    issue(0, t + 2, wr); adv(wr);
    fa.read(rd, a); adv(rd);
    multiply(acc[1]);
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
  __syncthreads();

  unsigned char* stage = smem + wave * strip_bytes(2);
  finish_tile<false>(p.epi, [&](auto fin) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int m = at.m0 + 128 * h + 64 * wm + 32 * i;
        if (m < p.M) finish_strip<decltype(fin)::value, 2>(p.epi, acc[h][i], m, at.n0 + 64 * wn, p.M, lane, stage);
      }
  });
}

// ---- 128 x 192 ------------------------------------------------------------------------------------
// Wavefront (wm, wn) of 4 x 2 owns 32 rows x 96 columns; one step is a whole k tile (A 16 KB, B 24 KB), four of which
// fill the LDS and three are on their way.  Narrow tiles are bound by the loads that miss L2, about 50 GB/s a compute unit
// (128x256 tiles at 8192x768x3072, operands from memory: 47 us; with their k tiles in L2, as in launches repeated on the
// same operands, 39, without any load 29, the loads alone 45), so covering more compute units is worth more than a wider tile.  A k-strided B lies as three pieces of 64
// columns, [64 k][64], chunk c of k row k in place c ^ (2 ((k>>1)&1)).
constexpr int SLIM_C = 3, SLIM_TILE = SLOT + 8192 * SLIM_C, SLIM_BUFS = 4;
template <bool B_KC>
__global__ void __launch_bounds__(512) k_gemm_slim(Params p) {
  constexpr int C = SLIM_C, BUFS = SLIM_BUFS, TILE = SLIM_TILE;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const unsigned lds_base = (unsigned)(uintptr_t)(lds_void_t*)smem;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave & 3, wn = wave >> 2;
  Place at;
  if (!place<128, 64 * C>(p, (int)blockIdx.x, &at)) return;
  const View va = view<true>(p.A, p.lda, at.m0, p.M, p.K), vb = view<B_KC>(p.B, p.ldb, at.n0, p.N, p.K);
  Mover<true> ma; ma.init(lane, p.lda);
  int vob[2];        // even / odd pieces of this wavefront (its first piece is C wave)
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int odd = (j + C * wave) & 1;
    vob[j] = B_KC ? ((lane >> 3) * p.ldb + 8 * ((lane & 7) ^ ((4 * odd + (lane >> 4)) & 7))) * 2
                  : (lane >> 3) * p.ldb * 2 + (((lane & 7) ^ (2 * ((lane >> 4) & 1))) << 4);
  }
  auto issue = [&](int t, unsigned buf) {
    const int k0 = t * 64;
    ma.issue(va.rsrc(t < at.nk), p.lda, 0, k0, wave, smem + buf);
    const __amdgpu_buffer_rsrc_t rb = vb.rsrc(t < at.nk);
#pragma unroll
    for (int j = 0; j < C; ++j) {
      const int q = C * wave + j;
      const int soff = B_KC ? (q * 8 * p.ldb + k0) * 2 : ((k0 + 8 * (q & 7)) * p.ldb + 64 * (q >> 3)) * 2;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void_t*)(smem + buf + SLOT + q * 1024), 16, vob[j & 1], soff, 0, 0);
    }
  };
  unsigned oa[4], ob[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) oa[s] = lds_base + kc_off(lane, 32 * wm, s);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (B_KC) {
      ob[i] = lds_base + SLOT + kc_off(lane, 32 * C * wn, i);
    } else {
      const int col = 32 * C * wn + 32 * (i < C ? i : 0), blk = lane >> 4, j = lane & 15;
      const int e = (col & 63) + 16 * (blk & 1) + 4 * (j & 3);
      ob[i] = lds_base + SLOT + (col >> 6) * 8192 + (8 * (blk >> 1) + (j >> 2)) * 128 + (((e >> 3) ^ (2 * (j >> 3))) << 4) + (e & 7) * 2;
    }
  }
  f32x16_t acc[C];
#pragma unroll
  for (int x = 0; x < C; ++x) start_block(p.epi.bias, at.n0 + 32 * C * wn + 32 * x, lane, acc[x]);

#pragma unroll
  for (int q = 0; q < BUFS - 1; ++q) issue(q, q * TILE);
  constexpr int WAIT = waitcnt_imm((BUFS - 2) * (2 + C), 15);      // the next k tile has landed
  __builtin_amdgcn_s_waitcnt(WAIT);
  meet();
  const bool second = wave >= 4;
  if (second) meet();
  unsigned cur = 0, wr = (BUFS - 1) * TILE;
  auto adv = [](unsigned& x) { x = x == (BUFS - 1) * TILE ? 0 : x + TILE; };
  bf16x8_t a[4], b[C][4];
  // one 32-column block of a k-strided B: eight transposing reads
  auto read_strided = [&](int x) {
    s16x4_t v[8];
    asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:512\n\tds_read_b64_tr_b16 %2, %8 offset:2048\n\tds_read_b64_tr_b16 %3, %8 offset:2560\n\t"
                 "ds_read_b64_tr_b16 %4, %8 offset:4096\n\tds_read_b64_tr_b16 %5, %8 offset:4608\n\tds_read_b64_tr_b16 %6, %8 offset:6144\n\tds_read_b64_tr_b16 %7, %8 offset:6656\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7]) : "v"(ob[x] + cur) : "memory");
#pragma unroll
    for (int s = 0; s < 4; ++s) b[x][s] = join(v[2 * s], v[2 * s + 1]);
  };
  for (int t = 0; t < at.nk; ++t) {
    issue(t + BUFS - 1, wr); adv(wr);
    asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3])
                 : "v"(oa[0] + cur), "v"(oa[1] + cur), "v"(oa[2] + cur), "v"(oa[3] + cur) : "memory");
    if constexpr (B_KC) {
      asm volatile("ds_read_b128 %0, %12\n\tds_read_b128 %4, %12 offset:4096\n\tds_read_b128 %8, %12 offset:8192\n\t"
                   "ds_read_b128 %1, %13\n\tds_read_b128 %5, %13 offset:4096\n\tds_read_b128 %9, %13 offset:8192\n\t"
                   "ds_read_b128 %2, %14\n\tds_read_b128 %6, %14 offset:4096\n\tds_read_b128 %10, %14 offset:8192\n\t"
                   "ds_read_b128 %3, %15\n\tds_read_b128 %7, %15 offset:4096\n\tds_read_b128 %11, %15 offset:8192\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(b[0][0]), "=&v"(b[0][1]), "=&v"(b[0][2]), "=&v"(b[0][3]), "=&v"(b[1][0]), "=&v"(b[1][1]), "=&v"(b[1][2]), "=&v"(b[1][3]),
                     "=&v"(b[2][0]), "=&v"(b[2][1]), "=&v"(b[2][2]), "=&v"(b[2][3])
                   : "v"(ob[0] + cur), "v"(ob[1] + cur), "v"(ob[2] + cur), "v"(ob[3] + cur) : "memory");
    } else {
#pragma unroll
      for (int x = 0; x < C; ++x) read_strided(x);
    }
    adv(cur);
    __builtin_amdgcn_s_waitcnt(WAIT);
    meet();
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int x = 0; x < C; ++x) acc[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[x][s], a[s], acc[x], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    meet();
  }
  if (!second) meet();
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
  __syncthreads();

  unsigned char* stage = smem + wave * strip_bytes(C);
  const int m = at.m0 + 32 * wm;
  if (m < p.M) finish_tile<false>(p.epi, [&](auto fin) { finish_strip<decltype(fin)::value, C>(p.epi, acc, m, at.n0 + 32 * C * wn, p.M, lane, stage); });
}

// ---- launches ---------------------------------------------------------------------------------------
static_assert(8 * strip_bytes(2) <= PHASE_SLOTS * SLOT && 4 * strip_bytes(2) <= PAIR_SLOTS * SLOT && 8 * strip_bytes(2) <= WIDE_SLOTS * SLOT &&
              8 * strip_bytes(SLIM_C) <= SLIM_BUFS * SLIM_TILE, "the strips lie over the slots");
static_assert(SLIM_BUFS * SLIM_TILE <= 160 * 1024 && WIDE_SLOTS * SLOT <= 160 * 1024 && 2 * PAIR_SLOTS * SLOT <= 160 * 1024, "LDS of a compute unit");
template <typename F>
static hipError_t lds_limit(F* kernel, int bytes, bool* set) {
  if (*set) return hipSuccess;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  *set = e == hipSuccess;
  return e;
}
#define MSLT_LAUNCH(kernel, threads, bytes)                                                              \
  do {                                                                                                   \
    static bool set = false;                                                                             \
    if (hipError_t e = lds_limit(kernel, bytes, &set)) return e;                                         \
    kernel<<<dim3((unsigned)(p.tiles_m * p.tiles_n * p.splitk)), dim3(threads), bytes, s>>>(p);          \
    return hipGetLastError();                                                                            \
  } while (0)
static Params params(const GemmDesc& d, int tile_m, int tile_n, int splitk, float* partials) {
  return Params{reinterpret_cast<const bf16*>(d.A), reinterpret_cast<const bf16*>(d.B), d.M, d.N, d.K, d.lda, d.ldb, splitk,
                (d.M + tile_m - 1) / tile_m, d.N / tile_n, partials, d.epi};
}
static hipError_t launch(const GemmDesc& d, int tile_m, int tile_n, const Params& p, hipStream_t s) {
  if (tile_m == 256 && tile_n == 256) {
    if (d.a_kcontig && d.b_kcontig) MSLT_LAUNCH((k_gemm_phase<true, true>), 512, PHASE_SLOTS * SLOT);
    if (d.a_kcontig) MSLT_LAUNCH((k_gemm_phase<true, false>), 512, PHASE_SLOTS * SLOT);
    if (d.b_kcontig) MSLT_LAUNCH((k_gemm_phase<false, true>), 512, PHASE_SLOTS * SLOT);
    MSLT_LAUNCH((k_gemm_phase<false, false>), 512, PHASE_SLOTS * SLOT);
  }
  if (tile_n == 384) {
    if (d.b_kcontig) MSLT_LAUNCH(k_gemm_wide<true>, 512, WIDE_SLOTS * SLOT);
    MSLT_LAUNCH(k_gemm_wide<false>, 512, WIDE_SLOTS * SLOT);
  }
  if (tile_m == 128) {
    if (d.b_kcontig) MSLT_LAUNCH(k_gemm_slim<true>, 512, SLIM_BUFS * SLIM_TILE);
    MSLT_LAUNCH(k_gemm_slim<false>, 512, SLIM_BUFS * SLIM_TILE);
  }
  if (d.b_kcontig) MSLT_LAUNCH((k_gemm_pair<true, true>), 256, PAIR_SLOTS * SLOT);
  MSLT_LAUNCH((k_gemm_pair<true, false>), 256, PAIR_SLOTS * SLOT);
}
#undef MSLT_LAUNCH

}  // namespace phase

bool gemm_phase_supported(const GemmDesc& d, int tile_m, int tile_n) {
  const bool square = tile_m == 256 && tile_n == 256;
  const bool other = d.a_kcontig && ((tile_m == 256 && (tile_n == 384 || tile_n == 128)) || (tile_m == 128 && tile_n == 192));
  if (!square && !other) return false;
  if (d.M <= 0 || d.N <= 0 || d.K <= 0 || d.N % tile_n || d.K % 64) return false;
  if (!d.a_kcontig && d.M % 256) return false;       // (rows past the end of a k-strided A are the next k's)
  if (d.lda % 8 || d.ldb % 8 || d.epi.ldo % 8) return false;
  if ((d.epi.act == EPI_MUL || d.epi.act == EPI_ADD) && d.epi.ldaux % 8) return false;
  if (d.epi.drop.thr && d.epi.drop_ld % 4) return false;
  if (d.epi.accumulate && !d.epi.out_f32) return false;
  const bool plain_drop = !d.epi.out_f32 && d.epi.act == EPI_NONE;      // (see finish_tile)
  if ((d.epi.accumulate || (d.epi.drop.thr && !plain_drop)) && (d.a_kcontig || d.b_kcontig)) return false;
  auto al = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
  if (!al(d.A) || !al(d.B) || !al(d.epi.out) || !al(d.epi.out2) || !al(d.epi.aux) || !al(d.epi.bias)) return false;
  // byte offsets of a tile inside its operands' views stay below 2^31, those of the loads queued past the last k tile (up to
  // three more) among them
  const long long k_end = d.K + 4 * 64;
  const long long a_span = d.a_kcontig ? (long long)tile_m * d.lda + k_end : k_end * d.lda + tile_m;
  const long long b_span = d.b_kcontig ? (long long)tile_n * d.ldb + k_end : k_end * d.ldb + tile_n;
  return 2 * a_span < 0x7fffffffLL && 2 * b_span < 0x7fffffffLL;
}
hipError_t gemm_phase(const GemmDesc& d, int tile_m, int tile_n, int splitk, float* partials, hipStream_t s) {
  if (!gemm_phase_supported(d, tile_m, tile_n)) return hipErrorInvalidValue;
  if (splitk < 1 || splitk > d.K / 64 || (splitk > 1 && (!partials || tile_m != 256 || tile_n != 256))) return hipErrorInvalidValue;
  hipError_t e = phase::launch(d, tile_m, tile_n, phase::params(d, tile_m, tile_n, splitk, partials), s);
  if (e != hipSuccess || splitk == 1) return e;
  const size_t n8 = (size_t)d.M * d.N / 8;
  k_splitk_reduce<<<dim3((unsigned)((n8 + 255) / 256)), dim3(256), 0, s>>>(partials, splitk, d.M, d.N, d.epi);
  return hipGetLastError();
}
hipError_t gemm_phase_grouped_tn(const GemmDesc* d, int n, hipStream_t s) {
  using namespace phase;
  if (n < 1 || n > GROUP_MAX) return hipErrorInvalidValue;
  GroupParams gp;
  gp.n = n;
  int at = 0;
  for (int i = 0; i < n; ++i) {
    if (d[i].a_kcontig || d[i].b_kcontig || !gemm_phase_supported(d[i], 256, 256)) return hipErrorInvalidValue;
    gp.p[i] = params(d[i], 256, 256, 1, nullptr);
    gp.first[i] = at;
    at += (gp.p[i].tiles_m * gp.p[i].tiles_n + 7) & ~7;      // every product starts on XCD 0
  }
  for (int i = n; i <= GROUP_MAX; ++i) gp.first[i] = at;
  static bool set = false;
  if (hipError_t e = lds_limit(k_gemm_phase_grouped, PHASE_SLOTS * SLOT, &set)) return e;
  k_gemm_phase_grouped<<<dim3((unsigned)at), dim3(512), PHASE_SLOTS * SLOT, s>>>(gp);
  return hipGetLastError();
}

}  // namespace mslt

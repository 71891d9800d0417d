// MXFP4 projections (4-bit weight-only variant): P[split][M][N] = X[M][K] . W[N][K]^T with
//   W[n][k] = 2^(E[n][k/32] - 127) * e2m1(code[n][k])
//
// MXFP4 is the OCP microscaling format: 4-bit e2m1 elements (sign, 2 exponent bits,
// 1 mantissa bit: 0, 0.5, 1, 1.5, 2, 3, 4, 6 and their negatives), one 8-bit power-of-two
// scale (e8m0) per 32 consecutive elements along K.  The codes and scales go to the matrix
// cores as they are (gfx950's scaled fp4 x fp6 product, 16x16x128), against activations in
// four fp6 parts (the a6 tiles of common.hpp): every product is exact, and the four parts
// together take half the matrix-core time of two bf16 halves, with no dequantization.
//
// Tiled layout (pack_weight_fp4), per 16 rows x one 128-element step of K:
//   * a 1 KB code block: lane l = 16 g + r (row r, group g) holds 16 bytes, dword c =
//     the codes of row r at k = 32 c + 8 g + 0..7, byte b = (k = 2b, 2b+1) with the even
//     k in the low nibble.  The product wants row r's 32 codes at k = 32 g .. 32 g + 31 in
//     lane 16 g + r: a transposition of 4x4 dwords between the four 16-lane groups and the
//     four registers (to_operand);
//   * a 64-byte scale block: dword r = the four e8m0 scales of row r over the step;
// both ordered time-major like the bf16 layout (the blocks that the workgroups of a
// launch stream at the same moment are adjacent).
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace spp {
namespace {

constexpr int kFp4Step = 128;                 // K elements per step

// Tiled codes <- row-major codes [N][K/2] (byte j of a row: k = 2j in the low nibble).
// Destination 16-byte unit t: lane l = t % 64 of the block at position t / 64, which
// holds row block cb and step ks (the inverse of the GEMM's block map); its dword c is the source
// dword of row 16 cb + l % 16 at byte 64 ks + 16 c + 4 (l / 16).
__global__ __launch_bounds__(256) void pack_codes_kernel(const uint32_t* __restrict__ src,
                                                         uint4* __restrict__ dst, int N, int K,
                                                         int slab) {
  const int ksteps = K / kFp4Step, nslab = ksteps / slab, nblk = N / 16;
  const int64_t total = (int64_t)N * K / 32;   // 16-byte units
  const int row_words = K / 8;                 // source dwords per row
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < total; t += (int64_t)gridDim.x * 256) {
    const int lane = (int)(t & 63);
    const int64_t pos = t >> 6;
    const int cb = (int)(pos % nblk);
    const int64_t q = pos / nblk;
    const int sl = (int)(q % nslab), ts = (int)(q / nslab);
    const int ks = sl * slab + ts;
    const int64_t n = (int64_t)cb * 16 + (lane & 15);
    const uint32_t* s = src + n * row_words + ks * 16 + (lane >> 4);
    dst[t] = make_uint4(s[0], s[4], s[8], s[12]);
  }
}

// Tiled scales <- row-major e8m0 scales [N][K/32]: block dword r = row 16 cb + r's four
// scales of step ks (one source dword).
__global__ __launch_bounds__(256) void pack_scales_kernel(const uint32_t* __restrict__ src,
                                                          uint32_t* __restrict__ dst, int N, int K,
                                                          int slab) {
  const int ksteps = K / kFp4Step, nslab = ksteps / slab, nblk = N / 16;
  const int64_t total = (int64_t)N * ksteps;   // dwords
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < total; t += (int64_t)gridDim.x * 256) {
    const int r = (int)(t & 15);
    const int64_t pos = t >> 4;
    const int cb = (int)(pos % nblk);
    const int64_t q = pos / nblk;
    const int sl = (int)(q % nslab), ts = (int)(q / nslab);
    const int ks = sl * slab + ts;
    dst[t] = src[((int64_t)cb * 16 + r) * ksteps + ks];
  }
}

constexpr int kCodeBlock = 1024, kScaleBlock = 64;  // bytes per 16 rows x step

// A block as stored -> the operand of a 16x16x128 product (see the layout above): dword j of
// group g takes dword g of group j.
__device__ __forceinline__ uint4 to_operand(const uint4& w) {
  const auto p = __builtin_amdgcn_permlane32_swap(w.x, w.z, false, false);
  const auto q = __builtin_amdgcn_permlane32_swap(w.y, w.w, false, false);
  const auto lo = __builtin_amdgcn_permlane16_swap(p[0], q[0], false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(p[1], q[1], false, false);
  return make_uint4(lo[0], lo[1], hi[0], hi[1]);
}

// Part PART of the activations of 16 rows, as the lane's operand.
struct A6Frag {
  uint4 a;
  uint2 b;
};
template <int PART>
__device__ __forceinline__ A6Frag a6_frag(const char* tile, int unit) {
  A6Frag f;
  f.a = *reinterpret_cast<const uint4*>(tile + PART * 1024 + unit * 16);
  f.b = *reinterpret_cast<const uint2*>(tile + kA6Low + PART * 512 + unit * 8);
  return f;
}

// c[n][row] += W[n][k] x[row][k] over 128 elements: lane 16 g + r holds weight row r and
// activation row r at k = 32 g + 0..31, the weights' scale in byte WSEL of ws, the parts' scales
// in the bytes of xs; c is weight rows 4 g .. 4 g + 3 of activation row r.
template <int PART, int WSEL = 0>
__device__ __forceinline__ f32x4 mma_w4(const uint4& w, const A6Frag& x, f32x4 c, int ws, int xs) {
  typedef int i32x8 __attribute__((ext_vector_type(8)));
  const i32x8 a = {(int)w.x, (int)w.y, (int)w.z, (int)w.w, 0, 0, 0, 0};
  const i32x8 b = {(int)x.a.x, (int)x.a.y, (int)x.a.z, (int)x.a.w, (int)x.b.x, (int)x.b.y, 0, 0};
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 4, 2, WSEL, ws, PART, xs);
}

// Where 16-row block `n / 16` of the concatenated matrices lies: its matrix's codes and
// scales and the address of its block at step position 0 (block index within the matrix).
struct Block4 {
  const char* code;
  const char* scale;
  int cb, nblk;
  bool ok;
};
__device__ __forceinline__ Block4 block_of(const WeightCat& w, int n) {
  // past the last column: block 0 of the first matrix (always there), whose result is not kept
  const bool ok = n < w.nbeg[3];
  const int nn = ok ? n : 0;
  const int mi = nn >= w.nbeg[2] ? 2 : (nn >= w.nbeg[1] ? 1 : 0);
  // (explicit selects: a dynamic index into the by-value argument would go to scratch)
  const void* code = mi == 2 ? w.mat[2] : (mi == 1 ? w.mat[1] : w.mat[0]);
  const void* scale = mi == 2 ? w.scale[2] : (mi == 1 ? w.scale[1] : w.scale[0]);
  const int nb = mi == 2 ? w.nbeg[2] : (mi == 1 ? w.nbeg[1] : w.nbeg[0]);
  const int ne = mi == 2 ? w.nbeg[3] : (mi == 1 ? w.nbeg[2] : w.nbeg[1]);
  return Block4{static_cast<const char*>(code), static_cast<const char*>(scale), (nn - nb) / 16,
                (ne - nb) / 16, ok};
}

// A walk over the K-steps ks, ks + 1, ...: `pos` is the step's position in the time-major order
// (in units of the matrix's row blocks).  All of it is uniform.
struct StepWalk {
  int slab, nslab, t, sl, pos;
  __device__ __forceinline__ StepWalk(int slab_, int ksteps, int ks)
      : slab(slab_), nslab(ksteps / slab_), t(ks % slab_), sl(ks / slab_) {
    pos = t * nslab + sl;
  }
  // (selects, not branches: the caller's loop body stays one block)
  __device__ __forceinline__ void next(bool go = true) {
    const bool wrap = t + 1 == slab;
    sl += go && wrap ? 1 : 0;
    pos = go ? (wrap ? sl : pos + nslab) : pos;
    t = go ? (wrap ? 0 : t + 1) : t;
  }
};

struct SwigluOut4 {
  const float* ss;
  int nb, d;
  float eps;
  char* act;
  int F;
};

// silu(inv g) * (inv u) of four columns
__device__ __forceinline__ float4 swiglu4(const f32x4& gt, const f32x4& up, float inv) {
  float o[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float a = gt[i] * inv;
    o[i] = a / (1.f + __expf(-a)) * (up[i] * inv);
  }
  return make_float4(o[0], o[1], o[2], o[3]);
}

// ---- few rows (up to 64): bound by the weight stream.  NW waves of CB column blocks each, the
// weights of the next step in flight in registers while the matrix cores work on this one, the
// activations of a step shared by the waves in double-buffered LDS.  The K-range of a split
// need not be the same for all.  One 70B layer (M = 32 / 1, against the bf16 halves with the
// weights dequantized): QKV 18.4 -> 14.5 / 12.4 -> 10.3 us, O 13.1 -> 11.8 / 10.4 -> 8.8,
// gate/up + SwiGLU 69.4 -> 58.2 / 65.2 -> 45.1 (5.3 / 6.5 TB/s), down 35.1 -> 29.5 / 29.8 -> 23.7;
// 64 rows: 34.5 -> 22.4, 21.0 -> 18.8, 130.8 -> 98, 55.8 -> 45.
template <int NW, int MT, int CB>
__global__ __launch_bounds__(64 * NW) void stream4_kernel(const char* __restrict__ A, int M, int ksteps,
                                                          WeightCat w, int N, float* __restrict__ P,
                                                          int splits) {
  constexpr int THREADS = 64 * NW;
  constexpr int UPT = kA6Tile / 16;           // 16-byte units per row tile and step
  constexpr int UNITS = MT * UPT, AU = (UNITS + THREADS - 1) / THREADS;
  __shared__ __attribute__((aligned(16))) char lds[2][UNITS * 16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r = lane & 15, unit = a6_unit(r, g);
  const int split = blockIdx.x, cgroup = blockIdx.y;
  const int i0 = (int)((int64_t)split * ksteps / splits), i1 = (int)((int64_t)(split + 1) * ksteps / splits);
  const int iters = i1 - i0, row_tiles = (M + 15) / 16;
  StepWalk walk(w.slab, ksteps, i0);

  Block4 blk[CB];
  int n0[CB];
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    n0[c] = (cgroup * NW * CB + c * NW + wave) * 16;
    blk[c] = block_of(w, n0[c]);
  }

  f32x4 acc[MT][CB];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int c = 0; c < CB; ++c) acc[t][c] = f32x4{0.f, 0.f, 0.f, 0.f};

  struct Tile {
    uint4 code[CB];
    int scale[CB];
  };
  Tile w0, w1;
  uint4 ar[AU];
  // step by step in order: uniform bases that advance, and offsets that stay
  const char* an = A + (int64_t)i0 * kA6Tile;
  uint32_t aoff[AU];
#pragma unroll
  for (int q = 0; q < AU; ++q) {
    // (a unit past the step repeats the last one, a row tile past M the last one)
    const int u = min(tid + q * THREADS, UNITS - 1), t = u / UPT;
    aoff[q] = (uint32_t)(min(t, row_tiles - 1) * ksteps) * kA6Tile + (u - t * UPT) * 16;
  }
  auto load_a = [&] {
#pragma unroll
    for (int q = 0; q < AU; ++q) ar[q] = ld_global(an + aoff[q]);
    an += kA6Tile;
  };
  auto store_a = [&](char* buf) {
#pragma unroll
    for (int q = 0; q < AU; ++q)
      *reinterpret_cast<uint4*>(buf + min(tid + q * THREADS, UNITS - 1) * 16) = ar[q];
  };
  auto load_w = [&](Tile& x) {
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      const int64_t b = (int64_t)walk.pos * blk[c].nblk + blk[c].cb;
      x.code[c] = ld_global(blk[c].code + b * kCodeBlock + (uint32_t)lane * 16);
      x.scale[c] = *(const __attribute__((address_space(1))) uint8_t*)(blk[c].scale + b * kScaleBlock +
                                                                       (uint32_t)(r * 4 + g));
    }
    walk.next();
  };
  auto compute = [&](const char* buf, const Tile& x) {
    uint4 wf[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) wf[c] = to_operand(x.code[c]);
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const char* tile = buf + t * kA6Tile;
      const int xs = *reinterpret_cast<const int*>(tile + kA6Scale + unit * 4);
      const A6Frag x0 = a6_frag<0>(tile, unit), x1 = a6_frag<1>(tile, unit);
      const A6Frag x2 = a6_frag<2>(tile, unit), x3 = a6_frag<3>(tile, unit);
#pragma unroll
      for (int c = 0; c < CB; ++c) acc[t][c] = mma_w4<0>(wf[c], x0, acc[t][c], x.scale[c], xs);
#pragma unroll
      for (int c = 0; c < CB; ++c) acc[t][c] = mma_w4<1>(wf[c], x1, acc[t][c], x.scale[c], xs);
#pragma unroll
      for (int c = 0; c < CB; ++c) acc[t][c] = mma_w4<2>(wf[c], x2, acc[t][c], x.scale[c], xs);
#pragma unroll
      for (int c = 0; c < CB; ++c) acc[t][c] = mma_w4<3>(wf[c], x3, acc[t][c], x.scale[c], xs);
    }
  };

  load_a();
  load_w(w0);
  store_a(lds[0]);
  int i = 0;
  // two steps per trip, every load unconditional; the scheduling barriers keep a step's loads
  // ahead of the products before it
  for (; i + 2 < iters; i += 2) {
    __syncthreads();  // lds[0] holds step i; lds[1] is free
    load_a();
    load_w(w1);
    __builtin_amdgcn_sched_barrier(0);
    compute(lds[0], w0);
    store_a(lds[1]);
    __syncthreads();
    load_a();
    load_w(w0);
    __builtin_amdgcn_sched_barrier(0);
    compute(lds[1], w1);
    store_a(lds[0]);
  }
  __syncthreads();
  if (i + 1 < iters) {
    load_a();
    load_w(w1);
    __builtin_amdgcn_sched_barrier(0);
    compute(lds[0], w0);
    store_a(lds[1]);
    __syncthreads();
    compute(lds[1], w1);
  } else {
    compute(lds[0], w0);
  }

#pragma unroll
  for (int c = 0; c < CB; ++c)
    if (blk[c].ok)
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        const int row = t * 16 + r;
        if (row < M)
          *reinterpret_cast<f32x4*>(P + ((int64_t)split * M + row) * N + n0[c] + 4 * g) = acc[t][c];
      }
}

// ---- many rows (more than 64): 8 waves of 16 rows x 256 columns each.  A wave's activations
// belong to it alone, so they go from memory straight to its registers (an a6 tile is in operand
// order); only the weights, which every wave needs, pass through LDS, in a ring of four steps of
// which two are computed while the next two are filled (one barrier per two steps).  A step of
// 128 costs a SIMD with two waves 2048 cycles of products and the CU 139 KB of LDS reads, 17 KB
// of LDS writes and 68 KB from L2.  SW: 8 of a wave's 16 column blocks are of the gate and the
// same 8 of the up matrix (F is a multiple of 128).
// 700 rows of one 70B layer, same box: gate/up + SwiGLU 1385 -> 707 us (930 TFLOP/s of the
// projection), QKV 353 -> 120, O 181 -> 107, down 606 -> 325; with 128 rows in place of 16 per
// wave's LDS share, that is with both operands in LDS, the gate/up took 808 (this form 685 there).
constexpr int kBigRows = 128, kBigCols = 256;

// One step's activations of a wave, as operands.
struct A6Regs {
  A6Frag x[4];
  int scale;
};

template <bool SW>
__global__ __launch_bounds__(512, 2) void tile4_kernel(const char* __restrict__ A, int M, int ksteps,
                                                       WeightCat w, int N, float* __restrict__ P,
                                                       SwigluOut4 so, int splits, int groups,
                                                       int row_tiles, int band) {
  constexpr int NW = kBigRows / 16;
  constexpr int CB = kBigCols / 16, PER = CB / NW;              // column blocks; loaded per wave
  constexpr int WBYTES = CB * kCodeBlock, STAGE = WBYTES + CB * kScaleBlock, RING = 4;
  constexpr int XCH = SW ? NW * 64 * kA6Pitch * 4 : 0;
  __shared__ __attribute__((aligned(16))) char lds[RING * STAGE > XCH ? RING * STAGE : XCH];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r = lane & 15, unit = a6_unit(r, g);

  // Workgroup id goes to XCD id % 8, slot id / 8.  An XCD's consecutive slots take `band` row
  // tiles of one (split, column group) and then the next group: the activations of a band and
  // the weights of a group are both shared in its L2.
  const int slot = blockIdx.x >> 3, xcd = blockIdx.x & 7;
  const int octs = (splits * groups + 7) / 8, per_band = octs * band;
  const int rb = slot / per_band, in = slot - rb * per_band;
  const int xy = in / band * 8 + xcd, tile_m = rb * band + in % band;
  if (xy >= splits * groups || tile_m >= row_tiles) return;
  const int split = xy % splits, cgroup = xy / splits;
  const int k0 = (int)((int64_t)split * ksteps / splits), k1 = (int)((int64_t)(split + 1) * ksteps / splits);
  const int rt = tile_m * NW + wave, rts = (M + 15) / 16;       // this wave's 16 rows

  auto column = [&](int b) {  // first column of block b, in the concatenated matrices
    if constexpr (SW) {
      const int f = (cgroup * (CB / 2) + b % (CB / 2)) * 16;
      return f < so.F ? (b < CB / 2 ? f : so.F + f) : w.nbeg[3];
    } else {
      return (cgroup * CB + b) * 16;
    }
  };
  // the blocks this wave brings in: wave, wave + NW, ...
  Block4 blk[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) blk[i] = block_of(w, column(wave + i * NW));

  // Both operands are walked step by step: uniform bases that advance, and offsets that stay.
  // Past the range the last step is loaded again and never used.
  StepWalk walk(w.slab, ksteps, k0);
  int wleft = k1 - k0, aleft = k1 - k0;
  const char* an = A + ((int64_t)min(rt, rts - 1) * ksteps + k0) * kA6Tile;
  uint4 wr[PER];
  uint32_t sr[PER];
  auto load_w = [&] {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int64_t p = (int64_t)walk.pos * blk[i].nblk + blk[i].cb;
      wr[i] = ld_global(blk[i].code + p * kCodeBlock + (uint32_t)lane * 16);
      sr[i] = *(const __attribute__((address_space(1))) uint8_t*)(blk[i].scale + p * kScaleBlock + (uint32_t)(r * 4 + g));
    }
    walk.next(wleft > 1);
    wleft -= wleft > 1 ? 1 : 0;
  };
  // In LDS a block is in operand order, and lane 16 g + r finds the scales of four blocks in the
  // four bytes of one dword: 20 reads per wave and step, where the stored order took 48 and the
  // reads alone 3100 cycles of the CU's LDS.
  auto store_w = [&](char* buf) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int b = wave + i * NW;
      // (the empty statement keeps the copies that the swaps need here, behind the wait for the
      // loads: hoisted to the end of the step before, they waited for loads just issued)
      uint4 t = wr[i];
      asm volatile("" : "+v"(t.x), "+v"(t.y), "+v"(t.z), "+v"(t.w));
      *reinterpret_cast<uint4*>(buf + b * kCodeBlock + lane * 16) = to_operand(t);
      *reinterpret_cast<uint8_t*>(buf + WBYTES + (b >> 2) * 256 + (r * 4 + g) * 4 + (b & 3)) = (uint8_t)sr[i];
    }
  };
  auto load_a = [&](A6Regs& a) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      a.x[p].a = ld_global(an + (uint32_t)(unit * 16) + p * 1024);
      typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
      const u32x2 v = *(const __attribute__((address_space(1))) u32x2*)(an + (uint32_t)(unit * 8) + kA6Low + p * 512);
      a.x[p].b = make_uint2(v.x, v.y);
    }
    a.scale = (int)ld_global_u32(an + (uint32_t)(unit * 4) + kA6Scale);
    an += aleft > 1 ? kA6Tile : 0;
    aleft -= aleft > 1 ? 1 : 0;
  };

  f32x4 acc[CB];
#pragma unroll
  for (int c = 0; c < CB; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](const char* buf, const A6Regs& a) {
    const char* wb = buf + lane * 16;
    const char* sb = buf + WBYTES + (r * 4 + g) * 4;
#pragma unroll
    for (int c = 0; c < CB; c += 4) {
      uint4 q[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) q[j] = *reinterpret_cast<const uint4*>(wb + (c + j) * kCodeBlock);
      const int ws = *reinterpret_cast<const int*>(sb + c / 4 * 256);
#define SPP_PART(p)                                                   \
  acc[c] = mma_w4<p, 0>(q[0], a.x[p], acc[c], ws, a.scale);             \
  acc[c + 1] = mma_w4<p, 1>(q[1], a.x[p], acc[c + 1], ws, a.scale);     \
  acc[c + 2] = mma_w4<p, 2>(q[2], a.x[p], acc[c + 2], ws, a.scale);     \
  acc[c + 3] = mma_w4<p, 3>(q[3], a.x[p], acc[c + 3], ws, a.scale)
      SPP_PART(0);
      SPP_PART(1);
      SPP_PART(2);
      SPP_PART(3);
#undef SPP_PART
    }
  };

  A6Regs a0, a1;
  // (loads in the order of the loop's, so that its waits name the same ones from both sides)
  load_w();
  store_w(lds);
  load_w();
  store_w(lds + STAGE);
  __builtin_amdgcn_sched_barrier(0);
  load_a(a0);
  __builtin_amdgcn_sched_barrier(0);
  load_w();
  __builtin_amdgcn_sched_barrier(0);
  load_a(a1);
  __builtin_amdgcn_sched_barrier(0);
  int at = 0;  // ring position of the pair of steps being computed
  for (int ks = k0; ks < k1; ks += 2) {
    __syncthreads();  // this pair of steps is in LDS; the other pair is free
    const char* buf = lds + at * STAGE;
    char* fill = lds + (at ^ 2) * STAGE;
    store_w(fill);
    load_w();
    __builtin_amdgcn_sched_barrier(0);
    compute(buf, a0);
    load_a(a0);
    __builtin_amdgcn_sched_barrier(0);
    if (ks + 1 == k1) break;
    store_w(fill + STAGE);
    load_w();
    __builtin_amdgcn_sched_barrier(0);
    compute(buf + STAGE, a1);
    load_a(a1);
    __builtin_amdgcn_sched_barrier(0);
    at ^= 2;
  }

  const int row = rt * 16 + r;
  if constexpr (SW) {
    __syncthreads();  // every wave is done with the ring
    float* xs = reinterpret_cast<float*>(lds) + wave * 64 * kA6Pitch;  // [row][4 blocks of 32]
    const float inv = row_inv(so.ss, min(row, M - 1), so.nb, so.d, so.eps);
#pragma unroll
    for (int c = 0; c < CB / 2; ++c)
      *reinterpret_cast<float4*>(xs + (r * 4 + c / 2) * kA6Pitch + (c & 1) * 16 + 4 * g) =
          swiglu4(acc[c], acc[c + CB / 2], inv);
    __syncthreads();
    const int orow = rt * 16 + lane / 4, f = cgroup * (CB / 2) * 16 + (lane & 3) * 32;
    if (orow < M && f < so.F) a6_store(so.act, so.F / kA6Step, orow, f / 32, xs + lane * kA6Pitch);
  } else {
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      const int n = (cgroup * CB + c) * 16;
      if (n < w.nbeg[3] && row < M)
        *reinterpret_cast<f32x4*>(P + ((int64_t)split * M + row) * N + n + 4 * g) = acc[c];
    }
  }
}

template <int NW, int MT, int CB>
hipError_t launch_stream(const k::GemmPlan& p, const void* A, int M, int K, const WeightCat& w, int N,
                         float* P, hipStream_t st) {
  const int groups = (N + 16 * NW * CB - 1) / (16 * NW * CB);
  SPP_LAUNCH((stream4_kernel<NW, MT, CB>), dim3(p.splits, groups), dim3(64 * NW), 0, st,
             static_cast<const char*>(A), M, K / kFp4Step, w, N, P, p.splits);
  return hipGetLastError();
}

template <bool SW>
hipError_t launch_tile(const k::GemmPlan& p, const void* A, int M, int K, const WeightCat& w, int N,
                       float* P, const SwigluOut4& so, hipStream_t st) {
  if (p.row_tiles != (M + kBigRows - 1) / kBigRows) return hipErrorInvalidValue;
  const int groups = (N + kBigCols - 1) / kBigCols, band = std::min(p.row_tiles, 8);
  const int bands = (p.row_tiles + band - 1) / band, octs = (p.splits * groups + 7) / 8;
  SPP_LAUNCH((tile4_kernel<SW>), dim3((unsigned)(bands * band * octs * 8)), dim3(512), 0, st,
             static_cast<const char*>(A), M, K / kFp4Step, w, N, P, so, p.splits, groups,
             p.row_tiles, band);
  return hipGetLastError();
}

}  // namespace

namespace k {

// K-steps per slab of the stored layout.  It is part of the format of packed weights, so it
// does not follow the launch shapes below: the fewest K-splits (dividing the steps, two steps
// each at least) that fill 256 workgroups of 256 columns, or for a wide MLP (N >= 32768) the
// most that keep 512-column workgroups within 256.
int pack_slab_steps_fp4(const Shape& s, int N, int K) {
  (void)s;
  const int steps = K / kFp4Step;
  const bool wide = N >= 32768;
  const int cols = wide ? 512 : 256, groups = (N + cols - 1) / cols;
  int best = 1;
  for (int sp = 1; sp <= steps; ++sp) {
    if (steps % sp || (sp > 1 && steps / sp < 2)) continue;
    if (wide && sp > 1 && sp * groups > 256) break;
    best = sp;
    if (sp * groups >= 256) break;
  }
  return steps / best;
}
// (the gate and up matrices of a narrow MLP: one slab)
int pack_slab_steps_gateup_fp4(const Shape& s, int F, int K) {
  return 2 * F < 32768 && 32 * res_blocks(s) <= 512 ? K / kFp4Step : pack_slab_steps_fp4(s, 2 * F, K);
}

// The tile kernel's plan: without K-splits, or (split) the count whose estimated time is least --
// rounds of 256 workgroups at 2 us per step, and the fp32 partials written and read at 4 TB/s.
static GemmPlan tile4_plan(int M, int N, int K, bool split) {
  GemmPlan p{};
  const int ksteps = K / kFp4Step, groups = (N + kBigCols - 1) / kBigCols;
  p.row_tiles = (M + kBigRows - 1) / kBigRows;
  p.splits = 1;
  double best = 0;
  for (int sp = 1; split && sp <= 8 && (sp == 1 || sp * 4 <= ksteps); ++sp) {
    const int64_t wgs = (int64_t)p.row_tiles * groups * sp;
    const double t = (double)((wgs + 255) / 256) * ((ksteps + sp - 1) / sp) * 2.0 +
                     (double)sp * M * N * 8.0 / 4.0e6;
    if (sp == 1 || t < best) {
      best = t;
      p.splits = sp;
    }
  }
  return p;
}

// Up to 64 rows the weight stream bounds the kernel (stream4_kernel), beyond the products do
// (tile4_kernel; a 65-row launch takes 13% longer than a 64-row one).  8 waves of two column
// blocks, or of four where that still gives 100 workgroups per split (N >= 32768: the 70B
// gate/up, 56.7 -> 51.6 us at 32 rows); past 32 rows 4 waves of four, within the registers.
// The K-range is split as finely as keeps the grid within one workgroup per CU, two steps
// each at least: twice as many workgroups took 10-25% longer at 32 rows.
GemmPlan gemm_plan_fp4(const Shape& s, int M, int N, int K) {
  (void)s;
  if (M > 64) return tile4_plan(M, N, K, true);
  GemmPlan p{};
  p.mt = M <= 16 ? 1 : (M <= 32 ? 2 : 4);
  p.nw = p.mt == 4 ? 4 : 8;
  p.cb = p.mt == 4 || N >= 32768 ? 4 : 2;
  const int ksteps = K / kFp4Step, groups = (N + 16 * p.nw * p.cb - 1) / (16 * p.nw * p.cb);
  p.splits = std::max(1, std::min(256 / groups, ksteps / 2));
  return p;
}

hipError_t gemm_fp4(const Shape& s, const GemmPlan& p, const void* X, const void*, int M, int K,
                    const WeightCat& w, int N, float* partials, hipStream_t st) {
  if (M <= 0 || p.splits < 1 || !s.a6 || w.slab < 1 || K % kFp4Step || (K / kFp4Step) % w.slab ||
      p.splits > K / kFp4Step || w.nbeg[3] != N)
    return hipErrorInvalidValue;
  if (p.row_tiles > 0) return launch_tile<false>(p, X, M, K, w, N, partials, SwigluOut4{}, st);
  if (M > 16 * p.mt) return hipErrorInvalidValue;
  const bool wide = p.cb == 4;
  switch (p.mt) {
    case 1:
      return wide ? launch_stream<8, 1, 4>(p, X, M, K, w, N, partials, st)
                  : launch_stream<8, 1, 2>(p, X, M, K, w, N, partials, st);
    case 2:
      return wide ? launch_stream<8, 2, 4>(p, X, M, K, w, N, partials, st)
                  : launch_stream<8, 2, 2>(p, X, M, K, w, N, partials, st);
    case 4:
      return launch_stream<4, 4, 4>(p, X, M, K, w, N, partials, st);
  }
  return hipErrorInvalidValue;
}

// Fused past 64 rows.  Up to 64 rows the K-splits that the unfused form allows are worth more
// than its SwiGLU launch (70B, 32 rows: 58 us against 61; 1 row: 45 against 47).
GemmPlan gemm_plan_swiglu_fp4(const Shape& s, int M, int F, int K) {
  (void)s;
  if (M <= 64 || F % kFp4Step || K % kFp4Step) return GemmPlan{};
  return tile4_plan(M, 2 * F, K, false);
}

hipError_t gemm_swiglu_fp4(const Shape& s, const GemmPlan& p, const void* X, const void*, int M, int K,
                           const WeightCat& w, int F, const float* ss, void* act, void*,
                           hipStream_t st) {
  if (M <= 0 || p.splits != 1 || !s.a6 || w.slab < 1 || K % kFp4Step || (K / kFp4Step) % w.slab ||
      F % kFp4Step || w.nbeg[1] != F || w.nbeg[2] != 2 * F || w.nbeg[3] != 2 * F)
    return hipErrorInvalidValue;
  const SwigluOut4 so{ss, res_blocks(s), s.d, s.eps, static_cast<char*>(act), F};
  return launch_tile<true>(p, X, M, K, w, 2 * F, nullptr, so, st);
}

hipError_t pack_weight_fp4(const void* codes_src, const void* scales_src, void* codes_dst,
                           void* scales_dst, int N, int K, int slab, hipStream_t st) {
  if (N % 16 || K % kFp4Step || slab < 1 || (K / kFp4Step) % slab) return hipErrorInvalidValue;
  const int64_t units = (int64_t)N * K / 32, words = (int64_t)N * (K / kFp4Step);
  int64_t b1 = (units + 255) / 256, b2 = (words + 255) / 256;
  if (b1 > 65536) b1 = 65536;
  if (b2 > 65536) b2 = 65536;
  SPP_LAUNCH(pack_codes_kernel, dim3((unsigned)b1), dim3(256), 0, st,
                     static_cast<const uint32_t*>(codes_src), static_cast<uint4*>(codes_dst), N, K,
                     slab);
  SPP_LAUNCH(pack_scales_kernel, dim3((unsigned)b2), dim3(256), 0, st,
                     static_cast<const uint32_t*>(scales_src), static_cast<uint32_t*>(scales_dst),
                     N, K, slab);
  return hipGetLastError();
}

}  // namespace k
}  // namespace spp

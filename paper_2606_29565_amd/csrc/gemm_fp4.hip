// MXFP4 projections (4-bit weight-only variant): P[split][M][N] = X[M][K] . W[N][K]^T with
//   W[n][k] = 2^(E[n][k/32] - 127) * e2m1(code[n][k]),  X = hi + lo
//
// MXFP4 is the OCP microscaling format: 4-bit e2m1 elements (sign, 2 exponent bits,
// 1 mantissa bit: 0, 0.5, 1, 1.5, 2, 3, 4, 6 and their negatives), one 8-bit power-of-two
// scale (e8m0) per 32 consecutive elements along K.  Every product of an e2m1 value and
// a power of two is exact in bf16, so gfx950's packed fp4 -> bf16 conversion with a scale
// operand (one instruction per two weights) dequantizes without rounding, and the
// matrix cores multiply the exact weights by the (hi, lo) bf16 activations as in the
// bf16 kernels.  The weight stream shrinks to 0.53 bytes per weight (codes + scales).
//
// The matrix cores also multiply fp4 by fp6 directly, at four times the bf16 rate, but an fp6
// part holds 5 bits under one scale per 32 elements: four parts lost the small elements of a
// block with an outlier (an element 1000 times below the block's largest kept 9 bits, where the
// halves keep 16 of every element), and the seven that keep them took as long as the halves
// (70B, 32 rows over 4 layers: 1153 us; the halves in a kernel of gemm.hip 1084).
//
// Tiled layout (pack_weight_fp4), per 16 rows x one 128-element step of K:
//   * a 1 KB code block: lane l = 16 g + r (row r, group g) holds 16 bytes, dword c =
//     the codes of row r at k = 32 c + 8 g + 0..7, byte b = (k = 2b, 2b+1) with the even
//     k in the low nibble -- exactly the weight operand of four 16x16x32 products;
//   * a 64-byte scale block: dword r = the four e8m0 scales of row r over the step;
// both ordered time-major like the bf16 layout (the blocks that the workgroups of a
// launch stream at the same moment are adjacent).
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace spp {
namespace {

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
  __device__ __forceinline__ void next() {
    const bool wrap = t + 1 == slab;
    sl += wrap ? 1 : 0;
    pos = wrap ? sl : pos + nslab;
    t = wrap ? 0 : t + 1;
  }
};

// ---- few rows: bound by the weight stream.  NW waves of CB column blocks each, the weights of
// the next step in flight in registers while the matrix cores work on this one, the activations
// of a step (both halves) shared by the waves in double-buffered LDS, in rows padded to an odd
// multiple of 32 bytes (fragment reads then run at the full LDS rate).  The K-range of a split
// need not be the same for all.  Appends over 3 layers of the 70B shape, us, by the launch shapes
// this replaces (gemm.hip, even splits, two column blocks, fused SwiGLU up to 64 rows) and by
// this: 1 row 442 -> 364, 32 rows 534 -> 505, 64 rows 846 -> 759, 128 rows 1493 -> 1371.
constexpr int kPitch = kFp4Step * 2 + 32;  // LDS bytes per staged row

template <int NW, int MT, int CB>
__global__ __launch_bounds__(64 * NW) void stream4_kernel(const bf16_t* __restrict__ X,
                                                          const bf16_t* __restrict__ Xlo, int M, int K,
                                                          WeightCat w, int N, float* __restrict__ P,
                                                          int splits) {
  constexpr int THREADS = 64 * NW, ROWS = 16 * MT;
  constexpr int UPR = kFp4Step * 2 / 16;          // 16-byte units per row and step
  constexpr int HALF = ROWS * UPR, AU = 2 * HALF / THREADS;
  static_assert(2 * HALF % THREADS == 0 && HALF % 64 == 0, "whole units per thread, one half per wave and unit");
  __shared__ __attribute__((aligned(16))) char lds[2][2 * ROWS * kPitch];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r = lane & 15;
  const int split = blockIdx.x, cgroup = blockIdx.y, ksteps = K / kFp4Step;
  const int i0 = (int)((int64_t)split * ksteps / splits), i1 = (int)((int64_t)(split + 1) * ksteps / splits);
  const int iters = i1 - i0;
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
    uint32_t scale[CB];
  };
  Tile w0, w1;
  uint4 ar[AU];
  // step by step in order: uniform bases that advance, and offsets that stay
  const char *ah = reinterpret_cast<const char*>(X) + (int64_t)i0 * kFp4Step * 2;
  const char *al = reinterpret_cast<const char*>(Xlo) + (int64_t)i0 * kFp4Step * 2;
  uint32_t aoff[AU], loff[AU];
#pragma unroll
  for (int q = 0; q < AU; ++q) {
    const int u = tid + q * THREADS, row = u / UPR % ROWS, off = u % UPR * 16;
    aoff[q] = (uint32_t)min(row, M - 1) * (uint32_t)K * 2u + off;  // (a row past M: the last one)
    loff[q] = (uint32_t)(u / UPR * kPitch + off);
  }
  auto load_a = [&] {
#pragma unroll
    for (int q = 0; q < AU; ++q)
      ar[q] = ld_global((wave * 64 + q * THREADS < HALF ? ah : al) + aoff[q]);  // (uniform)
    ah += kFp4Step * 2;
    al += kFp4Step * 2;
  };
  auto store_a = [&](char* buf) {
#pragma unroll
    for (int q = 0; q < AU; ++q) *reinterpret_cast<uint4*>(buf + loff[q]) = ar[q];
  };
  auto load_w = [&](Tile& x) {
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      const int64_t b = (int64_t)walk.pos * blk[c].nblk + blk[c].cb;
      x.code[c] = ld_global(blk[c].code + b * kFp4Code + (uint32_t)lane * 16);
      x.scale[c] = ld_global_u32(blk[c].scale + b * kFp4Scale + (uint32_t)r * 4);
    }
    walk.next();
  };
  // c[n][row] += W[n][k] x[row][k]: lane 16 g + r holds weight row r and activation row r at k =
  // 32 J + 8 g + 0..7; the sum is weight rows 4 g .. 4 g + 3 of activation row r
  auto compute = [&](const char* buf, const Tile& x) {
    const char* a = buf + r * kPitch + g * 16;
#define SPP_CHUNK(J, D)                                                                           \
  {                                                                                               \
    uint4 wf[CB];                                                                                 \
    _Pragma("unroll") for (int c = 0; c < CB; ++c) wf[c] = fp4_frag(x.code[c].D, e8m0<J>(x.scale[c])); \
    _Pragma("unroll") for (int p = 0; p < 2; ++p)                                                 \
        _Pragma("unroll") for (int t = 0; t < MT; ++t) {                                          \
      const uint4 xf = *reinterpret_cast<const uint4*>(a + (p * ROWS + t * 16) * kPitch + J * 64); \
      _Pragma("unroll") for (int c = 0; c < CB; ++c)                                              \
          acc[t][c] = mma_frag(wf[c], xf, acc[t][c], bf16_t{});                                   \
    }                                                                                             \
  }
    SPP_CHUNK(0, x)
    SPP_CHUNK(1, y)
    SPP_CHUNK(2, z)
    SPP_CHUNK(3, w)
#undef SPP_CHUNK
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

template <int NW, int MT, int CB>
hipError_t launch_stream(const k::GemmPlan& p, const void* X, const void* Xlo, int M, int K,
                         const WeightCat& w, int N, float* P, hipStream_t st) {
  const int groups = (N + 16 * NW * CB - 1) / (16 * NW * CB);
  SPP_LAUNCH((stream4_kernel<NW, MT, CB>), dim3(p.splits, groups), dim3(64 * NW), 0, st,
             static_cast<const bf16_t*>(X), static_cast<const bf16_t*>(Xlo), M, K, w, N, P, p.splits);
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

// Up to kFp4Stream rows one pass over the weights serves all rows (stream4_kernel); beyond, the
// products bound the projections and go to the tile kernel of gemm_tile.hip.  Appends over 3
// layers of the 70B shape, us, streaming / tiles: 65 rows 1266 / 1385, 128 rows 1404 / 1480.
//
// 8 waves of two column blocks, or of four, so that an LDS read feeds more products, where the
// matrices are wide enough: at 33-64 rows from 8192 columns (33 rows 778 -> 735, 64 rows 816 ->
// 789; all widths with four against this line, 40 rows over 3 or 4 layers: d 256 252 -> 207, d
// 1024 286 -> 236, d 2048 324 -> 289, d 4096 359 -> 336), at up to 32 rows from 32768, where
// four still give 100 workgroups per split (17 and 32 rows with four everywhere: 486 -> 489,
// 514 -> 524).  Past 64 rows four do not fit the registers.  The K-range is split as finely as
// keeps the grid within one workgroup per CU, two steps each at least (twice as many: 368 ->
// 375 at 1 row, 514 -> 547 at 32).
constexpr int kFp4Stream = 128;
GemmPlan gemm_plan_fp4(const Shape& s, int M, int N, int K) {
  (void)s;
  if (M > kFp4Stream) return gemm_plan_tile(M, N, K, true);
  GemmPlan p{};
  p.mt = M <= 16 ? 1 : (M <= 32 ? 2 : (M <= 64 ? 4 : 8));
  p.nw = 8;
  p.cb = p.mt < 8 && N >= (p.mt == 4 ? 8192 : 32768) ? 4 : 2;
  const int ksteps = K / kFp4Step, groups = (N + 16 * p.nw * p.cb - 1) / (16 * p.nw * p.cb);
  p.splits = std::max(1, std::min(256 / groups, ksteps / 2));
  return p;
}

hipError_t gemm_fp4(const Shape& s, const GemmPlan& p, const void* X, const void* Xlo, int M, int K,
                    const WeightCat& w, int N, float* partials, hipStream_t st) {
  if (M <= 0 || p.splits < 1 || !s.bf16 || !Xlo || w.slab < 1 || K % kFp4Step ||
      (K / kFp4Step) % w.slab || p.splits > K / kFp4Step || w.nbeg[3] != N || !w.scale[0])
    return hipErrorInvalidValue;
  if (p.row_tiles > 0) return gemm_tile(p, X, Xlo, M, K, w, N, partials, st);
  if (M > 16 * p.mt) return hipErrorInvalidValue;
  const bool wide = p.cb == 4;
  switch (p.mt) {
    case 1:
      return wide ? launch_stream<8, 1, 4>(p, X, Xlo, M, K, w, N, partials, st)
                  : launch_stream<8, 1, 2>(p, X, Xlo, M, K, w, N, partials, st);
    case 2:
      return wide ? launch_stream<8, 2, 4>(p, X, Xlo, M, K, w, N, partials, st)
                  : launch_stream<8, 2, 2>(p, X, Xlo, M, K, w, N, partials, st);
    case 4:
      return wide ? launch_stream<8, 4, 4>(p, X, Xlo, M, K, w, N, partials, st)
                  : launch_stream<8, 4, 2>(p, X, Xlo, M, K, w, N, partials, st);
    case 8:
      return launch_stream<8, 8, 2>(p, X, Xlo, M, K, w, N, partials, st);
  }
  return hipErrorInvalidValue;
}

// Fused past kFp4Stream rows, from kTileFused workgroups on or where K is too short to split (4
// layers of d 2048, F 5632, 200 rows: fused 677 us, split 606; of d 256, F 512, 600 rows: 375, split
// without a split 399).  Up to kFp4Stream rows the K-splits that the unfused form allows are worth
// more than its SwiGLU launch (the former forms at stream4_kernel were fused up to 16 rows).
GemmPlan gemm_plan_swiglu_fp4(const Shape& s, int M, int F, int K) {
  (void)s;
  if (M <= kFp4Stream || F % 16 || K % kFp4Step ||
      ((M + 127) / 128 * ((2 * F + 255) / 256) < kTileFused && gemm_plan_tile(M, 2 * F, K, true).splits > 1))
    return GemmPlan{};
  return gemm_plan_tile(M, 2 * F, K, false);
}

hipError_t gemm_swiglu_fp4(const Shape& s, const GemmPlan& p, const void* X, const void* Xlo, int M, int K,
                           const WeightCat& w, int F, const float* ss, void* act, void* act_lo,
                           hipStream_t st) {
  if (M <= 0 || p.splits != 1 || !s.bf16 || !Xlo || !w.scale[0] || !w.scale[1])
    return hipErrorInvalidValue;
  return gemm_tile_swiglu(s, p, X, Xlo, M, K, w, F, ss, act, act_lo, st);
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

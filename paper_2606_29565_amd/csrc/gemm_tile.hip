// Projections over many rows (more than 128), of bf16 and of MXFP4 weights:
//   P[split][M][N] = X[M][K-range of split] . W[N][K-range]^T,  X = hi + lo
// where the products, not the weight stream, bound the kernel: every weight meets two bf16
// halves of each activation.
//
// A workgroup of 4 waves takes 128 rows x 256 columns; two workgroups share a CU, and while one
// waits the other multiplies.  A wave owns 32 rows and all the columns.  Its activations belong
// to it alone, so they go from memory straight to its registers as operands; only the weights,
// which the four waves share, pass through LDS (the stored tiles are in operand order, so LDS
// is written and read in whole linear kilobytes), in two buffers, with one barrier per
// 64-element step and the step after next in flight in registers.  An operand read from LDS
// feeds four products (two row tiles, two halves).  A step takes 1.6 us of a CU; its products
// alone take 1.3 at the 1.63 PFLOP/s that the matrix cores sustain from registers.
// 8B shape, us per layer, same box, before (64-row tiles with the activations in LDS; at 203 rows
// 128-row passes over all weights, SwiGLU apart) and now:
//                   QKV            O              gate/up + SwiGLU    down
//   2467 rows   237.0 -> 210.6   161.6 -> 162.5   1035.9 -> 903.4   476.3 -> 464.1
//   1000 rows    99.7 -> 110.3    58.8 ->  60.6    442.3 -> 381.0   185.0 -> 196.1
//    600 rows    58.4 ->  60.2    54.3 ->  44.6    322.9 -> 285.7   137.6 -> 127.9
//    300 rows    34.9 ->  45.3    31.7 ->  31.2    209.8 -> 184.4    92.3 ->  82.9
//    203 rows    38.8 ->  32.0    28.2 ->  24.1    142.4 -> 112.8    67.4 ->  56.3
// The larger tile leaves part of the chip idle where 128 x 256 divides badly (QKV at 300 and 1000
// rows, down at 1000): past 256 rows gemm_plan takes the 64-row tiles where they are estimated
// shorter.
// MXFP4 weights take the same tiles: a block of codes holds two steps, and the wave that brings
// it in makes the bf16 operands on the way to LDS.  Appends over one layer of the 70B shape, us,
// 128-row passes over all weights and now: 129 rows 865 -> 774, 300 rows 1343 -> 1132, 640 rows
// 2353 -> 1865, 1100 rows 4246 -> 3248.
// 128-column tiles (twice the activation traffic per product) took 1.2-1.4 times as long at 2467
// rows.  At 128 rows and fewer the passes of gemm.hip stay ahead (128 rows: 166 us per layer, 174
// with 128-column tiles, 204 with 256).
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace spp {
namespace {

constexpr int kRows = 128;        // rows of a workgroup
constexpr int CB = 16;            // its column blocks of 16
constexpr int kStep = 64;         // elements of a step
constexpr int kBlock = 2048;      // bytes of a weight block: 16 rows x one step, two 1 KB operands

struct SwigluTile {
  const float* ss;
  int nb, d;
  float eps;
  bf16_t* act;
  bf16_t* act_lo;
  int F;
};

struct TileBlock {
  const char* base;   // the matrix (bf16 blocks, or MXFP4 codes)
  const char* scale;  // its MXFP4 scales
  int cb, nblk;
};
__device__ __forceinline__ TileBlock tile_block(const WeightCat& w, int n) {
  // past the last column: block 0 of the first matrix (always there), whose result is not kept
  const int nn = n < w.nbeg[3] ? n : 0;
  const int mi = nn >= w.nbeg[2] ? 2 : (nn >= w.nbeg[1] ? 1 : 0);
  const void* mat = mi == 2 ? w.mat[2] : (mi == 1 ? w.mat[1] : w.mat[0]);
  const void* scale = mi == 2 ? w.scale[2] : (mi == 1 ? w.scale[1] : w.scale[0]);
  const int nb = mi == 2 ? w.nbeg[2] : (mi == 1 ? w.nbeg[1] : w.nbeg[0]);
  const int ne = mi == 2 ? w.nbeg[3] : (mi == 1 ? w.nbeg[2] : w.nbeg[1]);
  return TileBlock{static_cast<const char*>(mat), static_cast<const char*>(scale), (nn - nb) / 16,
                   (ne - nb) / 16};
}

// The weights that a wave brings in for one step: both operands of its blocks, or (MXFP4) the
// codes and scales of the blocks that hold the step, whose operands are made on the way to LDS.
template <bool Q4, int PER>
struct TileWeights {
  uint4 f[PER][2];
};
template <int PER>
struct TileWeights<true, PER> {
  uint4 code[PER];
  uint32_t scale[PER];
};

// c[n][row] += W[n][k] x[row][k] over 32 elements: lane 16 g + r holds weight row r and
// activation row r at k = 8 g + 0..7; c is weight rows 4 g .. 4 g + 3 of activation row r.
__device__ __forceinline__ f32x4 mma(const uint4& w, const uint4& x, f32x4 c) {
  return mma_frag(w, x, c, bf16_t{});
}

template <bool SW, bool Q4>
__global__ __launch_bounds__(256, 2) void tile_kernel(const bf16_t* __restrict__ X,
                                                      const bf16_t* __restrict__ Xlo, int M, int K,
                                                      WeightCat w, int N, float* __restrict__ P,
                                                      SwigluTile so, int splits, int groups,
                                                      int row_tiles, int band) {
  constexpr int NW = 4, PER = CB / NW, STAGE = CB * kBlock;
  __shared__ __attribute__((aligned(16))) char lds[2][STAGE];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r = lane & 15;

  // Workgroup id goes to XCD id % 8, slot id / 8.  An XCD's consecutive slots take `band` row
  // tiles of one (split, column group) and then the next group: the activations of a band and
  // the weights of a group are both shared in its L2.  Bands are alike and have no empty slots: as
  // 8 + 1 or 8 + 2 tiles, with the second band filled up by workgroups that returned, appends of
  // 1025-1280 rows over 2 layers of the 8B shape took 2475-2700 us (1200 rows 2656; by the 64-row
  // tiles 2406), now 2003-2192 (2181).
  const int slot = blockIdx.x >> 3, xcd = blockIdx.x & 7;
  const int octs = (splits * groups + 7) / 8, per_band = octs * band;
  const int rb = slot / per_band, in = slot - rb * per_band;
  const int rows = min(band, row_tiles - rb * band);  // row tiles of this band (the last may be short)
  const int xy = in / rows * 8 + xcd, tile_m = rb * band + in % rows;
  if (xy >= splits * groups) return;
  const int split = xy % splits, cgroup = xy / splits;
  // the stored blocks: one step each, or (MXFP4) two
  constexpr int SPB = Q4 ? kFp4Step / kStep : 1;
  const int kblocks = K / (kStep * SPB);
  const int b0 = (int)((int64_t)split * kblocks / splits), b1 = (int)((int64_t)(split + 1) * kblocks / splits);
  const int k0 = b0 * SPB, k1 = b1 * SPB;
  const int row0 = tile_m * kRows + wave * 32;

  auto column = [&](int b) {  // first column of block b, in the concatenated matrices
    if constexpr (SW) {       // CB / 2 blocks of the gate and the same of the up matrix
      const int f = (cgroup * (CB / 2) + b % (CB / 2)) * 16;
      return f < so.F ? (b < CB / 2 ? f : so.F + f) : w.nbeg[3];
    } else {
      return (cgroup * CB + b) * 16;
    }
  };
  TileBlock blk[PER];  // the blocks this wave brings in: wave, wave + NW, ...
#pragma unroll
  for (int i = 0; i < PER; ++i) blk[i] = tile_block(w, column(wave + i * NW));

  // Both operands are walked step by step: uniform bases that advance, and offsets that stay.
  // Past the range the last step is loaded again and never used.
  const int nslab = kblocks / w.slab;
  int ts = b0 % w.slab, sl = b0 / w.slab, pos = ts * nslab + sl;  // (time-major position)
  int wleft = b1 - b0, aleft = k1 - k0;
  using Weights = TileWeights<Q4, PER>;
  bool second = false, second_st = false;  // (MXFP4) the half of its block that comes next
  auto load_w = [&](Weights& x) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int64_t p = (int64_t)pos * blk[i].nblk + blk[i].cb;
      if constexpr (Q4) {
        x.code[i] = ld_global(blk[i].base + p * kFp4Code + (uint32_t)lane * 16);
        x.scale[i] = ld_global_u32(blk[i].scale + p * kFp4Scale + (uint32_t)r * 4);
      } else {
        x.f[i][0] = ld_global(blk[i].base + p * kBlock + (uint32_t)lane * 16);
        x.f[i][1] = ld_global(blk[i].base + p * kBlock + (uint32_t)lane * 16 + 1024);
      }
    }
    const bool go = wleft > 1 && (!Q4 || second), wrap = ts + 1 == w.slab;
    second = !second;
    wleft -= go ? 1 : 0;
    sl += go && wrap ? 1 : 0;
    pos = go ? (wrap ? sl : pos + nslab) : pos;
    ts = go ? (wrap ? 0 : ts + 1) : ts;
  };
  auto store_w = [&](char* buf, const Weights& x) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      char* p = buf + (wave + i * NW) * kBlock + lane * 16;
      if constexpr (Q4) {
        const uint32_t c0 = second_st ? x.code[i].z : x.code[i].x, c1 = second_st ? x.code[i].w : x.code[i].y;
        const uint32_t sc = second_st ? x.scale[i] >> 16 : x.scale[i];
        *reinterpret_cast<uint4*>(p) = fp4_frag(c0, e8m0<0>(sc));
        *reinterpret_cast<uint4*>(p + 1024) = fp4_frag(c1, e8m0<1>(sc));
      } else {
        *reinterpret_cast<uint4*>(p) = x.f[i][0];
        *reinterpret_cast<uint4*>(p + 1024) = x.f[i][1];
      }
    }
    second_st = !second_st;
  };
  struct Act {
    uint4 x[2][2][2];  // [operand of 32 elements][row tile][hi, lo]
  };
  const int64_t base = (int64_t)min(row0, M - 1) * K + (int64_t)k0 * kStep;  // uniform
  const char *ah = reinterpret_cast<const char*>(X + base), *al = reinterpret_cast<const char*>(Xlo + base);
  uint32_t aoff[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)  // (rows past M read row M - 1)
    aoff[t] = (uint32_t)(min(row0 + t * 16 + r, M - 1) - min(row0, M - 1)) * (uint32_t)K * 2u + g * 16;
  auto load_half = [&](Act& a, int j) {  // operand j of a step; the second one advances
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      a.x[j][t][0] = ld_global(ah + aoff[t] + j * 64);
      a.x[j][t][1] = ld_global(al + aoff[t] + j * 64);
    }
    if (j == 1) {
      const int adv = aleft > 1 ? kStep * 2 : 0;
      ah += adv;
      al += adv;
      aleft -= aleft > 1 ? 1 : 0;
    }
  };

  f32x4 acc[2][CB];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int c = 0; c < CB; ++c) acc[t][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](const char* buf, const Act& a, int j) {
    const char* wb = buf + lane * 16 + j * 1024;
#pragma unroll
    for (int c = 0; c < CB; c += 2) {
      const uint4 q0 = *reinterpret_cast<const uint4*>(wb + c * kBlock);
      const uint4 q1 = *reinterpret_cast<const uint4*>(wb + (c + 1) * kBlock);
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          acc[t][c] = mma(q0, a.x[j][t][p], acc[t][c]);
          acc[t][c + 1] = mma(q1, a.x[j][t][p], acc[t][c + 1]);
        }
    }
  };
  // One step: the weights of the step after go from registers to the other buffer, and their
  // registers take the next step not yet requested; an operand's registers are reloaded as soon
  // as its products are issued, for the next step that uses them.  The barriers keep that order,
  // which the waits rely on (a prologue in another order made every step wait for its newest
  // loads).
  auto step = [&](const char* buf, char* next, Act& a, Weights& x) {
    __syncthreads();  // buf holds this step; next is free
    store_w(next, x);
    load_w(x);
    __builtin_amdgcn_sched_barrier(0);
    compute(buf, a, 0);
    __builtin_amdgcn_sched_barrier(0);
    load_half(a, 0);
    __builtin_amdgcn_sched_barrier(0);
    compute(buf, a, 1);
    __builtin_amdgcn_sched_barrier(0);
    load_half(a, 1);
    __builtin_amdgcn_sched_barrier(0);
  };
  Weights w0;
  Act a0;
  load_w(w0);
  store_w(lds[0], w0);
  __builtin_amdgcn_sched_barrier(0);
  load_w(w0);
  __builtin_amdgcn_sched_barrier(0);
  load_half(a0, 0);
  load_half(a0, 1);
  __builtin_amdgcn_sched_barrier(0);
  // (rolled: two copies of the body did not fit the registers)
#pragma unroll 1
  for (int ks = k0, at = 0; ks < k1; ++ks, at ^= 1) step(lds[at], lds[at ^ 1], a0, w0);

#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int row = row0 + t * 16 + r;
    if (row >= M) continue;
    if constexpr (SW) {
      const float inv = row_inv(so.ss, row, so.nb, so.d, so.eps);
#pragma unroll
      for (int c = 0; c < CB / 2; ++c) {
        const int f = (cgroup * (CB / 2) + c) * 16;
        if (f >= so.F) continue;
        float o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float a = acc[t][c][i] * inv;
          o[i] = a / (1.f + __expf(-a)) * (acc[t][c + CB / 2][i] * inv);
        }
        store_act4(so.act, so.act_lo, (int64_t)row * so.F + f + 4 * g, make_float4(o[0], o[1], o[2], o[3]));
      }
    } else {
#pragma unroll
      for (int c = 0; c < CB; ++c) {
        const int n = (cgroup * CB + c) * 16;
        if (n < w.nbeg[3])
          *reinterpret_cast<f32x4*>(P + ((int64_t)split * M + row) * N + n + 4 * g) = acc[t][c];
      }
    }
  }
}

template <bool SW, bool Q4>
hipError_t launch_t(const k::GemmPlan& p, const void* X, const void* Xlo, int M, int K, const WeightCat& w,
                    int N, float* P, const SwigluTile& so, hipStream_t st) {
  const int groups = (N + 16 * CB - 1) / (16 * CB), octs = (p.splits * groups + 7) / 8;
  const int bands = (p.row_tiles + 7) / 8, band = (p.row_tiles + bands - 1) / bands;
  SPP_LAUNCH((tile_kernel<SW, Q4>), dim3((unsigned)(p.row_tiles * octs * 8)), dim3(256), 0, st,
             static_cast<const bf16_t*>(X), static_cast<const bf16_t*>(Xlo), M, K, w, N, P, so, p.splits,
             groups, p.row_tiles, band);
  return hipGetLastError();
}
template <bool SW>
hipError_t launch(const k::GemmPlan& p, const void* X, const void* Xlo, int M, int K, const WeightCat& w,
                  int N, float* P, const SwigluTile& so, hipStream_t st) {
  const bool q4 = w.scale[0] != nullptr;
  const int blocks = K / (q4 ? kFp4Step : kStep);  // stored blocks along K: what the splits divide
  if (M <= 0 || p.row_tiles != (M + kRows - 1) / kRows || K % (q4 ? kFp4Step : kStep) || p.splits < 1 ||
      p.splits > blocks || w.slab < 1 || blocks % w.slab)
    return hipErrorInvalidValue;
  return q4 ? launch_t<SW, true>(p, X, Xlo, M, K, w, N, P, so, st)
            : launch_t<SW, false>(p, X, Xlo, M, K, w, N, P, so, st);
}

}  // namespace

namespace k {

// The time of the kernel, estimated from the workgroups that the busiest CU takes: an XCD gets
// whole (split, column group) pairs, each with all the row tiles, and has 32 CUs.  Within 8% of
// the QKV, O and down projections of the 8B and 32B shapes and of d = 4096, F = 11008 at 321 to 2000
// rows; estimating from the chip's workgroups instead (32B down, 550 rows: 500 of them, but 65 on
// some XCDs) had picked splits 20% slower than the best.
double tile_us(int row_tiles, int groups, int splits, int steps) {
  const int busiest = ((groups * splits + 7) / 8 * row_tiles + 31) / 32;
  return busiest == 1 ? 1.95 * steps + 8.5 : busiest * (1.64 * steps + 3.5) + 5;
}

// The K-split count whose estimated time is least, with the fp32 partials at kPartialRate.
GemmPlan gemm_plan_tile(int M, int N, int K, bool split) {
  GemmPlan p{};
  const int ksteps = K / kStep, groups = (N + 16 * CB - 1) / (16 * CB);
  p.row_tiles = (M + kRows - 1) / kRows;
  p.splits = p.iters = 1;
  double best = 0;
  for (int sp = 1; split && sp <= 8 && (sp == 1 || sp * 4 <= ksteps); ++sp) {
    const double t = tile_us(p.row_tiles, groups, sp, (ksteps + sp - 1) / sp) +
                     (double)sp * M * N * 8.0 / kPartialRate;
    if (sp == 1 || t < best) {
      best = t;
      p.splits = sp;
    }
  }
  return p;
}

hipError_t gemm_tile(const GemmPlan& p, const void* X, const void* Xlo, int M, int K,
                     const WeightCat& w, int N, float* partials, hipStream_t st) {
  if (w.nbeg[3] != N) return hipErrorInvalidValue;
  return launch<false>(p, X, Xlo, M, K, w, N, partials, SwigluTile{}, st);
}

hipError_t gemm_tile_swiglu(const Shape& s, const GemmPlan& p, const void* X, const void* Xlo, int M,
                            int K, const WeightCat& w, int F, const float* ss, void* act, void* act_lo,
                            hipStream_t st) {
  if (p.splits != 1 || F % 16 || w.nbeg[1] != F || w.nbeg[3] != 2 * F) return hipErrorInvalidValue;
  const SwigluTile so{ss, res_blocks(s), s.d, s.eps, static_cast<bf16_t*>(act),
                      static_cast<bf16_t*>(act_lo), F};
  return launch<true>(p, X, Xlo, M, K, w, 2 * F, nullptr, so, st);
}

}  // namespace k
}  // namespace spp

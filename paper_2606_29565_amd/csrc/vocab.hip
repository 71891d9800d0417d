// Vocabulary-sized work: the LM head at the decision point with its reductions
// fused in, and the serve-time scan of a cached distribution.
//
// lmhead_gemv: one row z = rmsnorm(x_last) * g_final against W_lm[V][d] (the largest
// single weight stream of the step).  Each lane keeps its slice of z in registers
// and streams two weight rows at a time (all loads of both rows in flight; the rows
// are dealt to the waves of the whole grid in turn, so that together they read one
// compact window of W_lm), a butterfly shuffle sums each row, and the same wave keeps
// a running top-2 (value desc, index asc), a running (max, sum of exp) for the
// log-sum-exp and a nonfinite flag.  A second kernel merges the workgroup partials in
// a fixed tree order, so the result is deterministic.
//
// scan: the same reductions over already computed fp32 distributions (the gate's
// vocabulary scan, and the batched LM head's), one grid column per distribution, merged
// by the last workgroup of each.
#include "common.hpp"
#include "kernels.hpp"

namespace spp {
namespace {

struct Acc {  // running reductions
  Top2 t;
  float m, s;
  uint32_t nonfinite;
};

__device__ __forceinline__ void acc_init(Acc& a) {
  top2_init(a.t);
  a.m = -INFINITY;
  a.s = 0.f;
  a.nonfinite = 0;
}

__device__ __forceinline__ void lse_merge(float& m, float& s, float m2, float s2) {
  const float M = fmaxf(m, m2);
  if (M == -INFINITY) return;
  s = (m == -INFINITY ? 0.f : s * __expf(m - M)) + (m2 == -INFINITY ? 0.f : s2 * __expf(m2 - M));
  m = M;
}

template <bool LSE>
__device__ __forceinline__ void acc_push(Acc& a, float v, int i) {
  a.nonfinite |= !(fabsf(v) < INFINITY);
  top2_push(a.t, v, i);
  if constexpr (LSE) {
    if (fabsf(v) < INFINITY) {
      if (v > a.m) {
        a.s = a.s * __expf(a.m - v) + 1.f;
        a.m = v;
      } else {
        a.s += __expf(v - a.m);
      }
    }
  }
}

template <bool LSE>
__device__ __forceinline__ void acc_merge(Acc& a, const Acc& b) {
  top2_merge(a.t, b.t);
  if constexpr (LSE) lse_merge(a.m, a.s, b.m, b.s);
  a.nonfinite |= b.nonfinite;
}

// All 64 lanes' accumulators merged, in every lane.
template <bool LSE>
__device__ __forceinline__ Acc wave_acc(Acc a) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    Acc b = a;
    b.t.v1 = __shfl_xor(a.t.v1, o, 64);
    b.t.v2 = __shfl_xor(a.t.v2, o, 64);
    b.t.i1 = __shfl_xor(a.t.i1, o, 64);
    if constexpr (LSE) {
      b.m = __shfl_xor(a.m, o, 64);
      b.s = __shfl_xor(a.s, o, 64);
    }
    acc_merge<LSE>(a, b);
  }
  a.nonfinite = __builtin_amdgcn_ballot_w64(a.nonfinite != 0) ? 1u : 0u;
  return a;
}

__device__ __forceinline__ ScanPartial to_partial(const Acc& a) {
  return ScanPartial{a.t.v1, a.t.v2, a.t.i1, a.nonfinite, a.m, a.s, {0, 0}};
}

__device__ __forceinline__ Acc from_partial(const ScanPartial& p) {
  return Acc{Top2{p.v1, p.v2, p.i1}, p.m, p.s, p.nonfinite};
}

// Block-level: merge the 4 waves' accumulators (wave order), the result in every thread.
template <bool LSE>
__device__ __forceinline__ Acc block_acc(Acc a, ScanPartial* red) {
  a = wave_acc<LSE>(a);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();
  if (lane == 0) red[wave] = to_partial(a);
  __syncthreads();
  Acc r = from_partial(red[0]);
  for (int w = 1; w < 4; ++w) acc_merge<LSE>(r, from_partial(red[w]));
  return r;
}

// ---- the last workgroup of a launch merges: records handed over between workgroups
//
// The workgroups of a distribution sit on different XCDs, whose L2s are not coherent within a
// kernel.  A record is stored and read with device-scope atomic accesses, which go past the
// L2s; the store's completion is waited for before the arrival is counted, so whoever sees the
// full count reads complete records.  A device-scope fence per workgroup would order the same
// but writes the whole L2 back (it cost more than the second launch that this replaces).
template <typename R>
__device__ __forceinline__ void put_record(R* dst, const R& v) {
  static_assert(sizeof(R) == 32 && alignof(R) <= 8, "four 8-byte stores");
  unsigned long long w[4];
  __builtin_memcpy(w, &v, 32);
#pragma unroll
  for (int i = 0; i < 4; ++i)
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(dst) + i, w[i], __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
template <typename R>
__device__ __forceinline__ R get_record(const R* src) {
  unsigned long long w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    w[i] = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(src) + i, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
  R v;
  __builtin_memcpy(&v, w, 32);
  return v;
}
// Counts one arrival after this thread's stores have completed; true for the last of `total`,
// which leaves the counter at zero for the next launch.
__device__ __forceinline__ bool last_arrival(uint32_t* counter, uint32_t total) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");  // (compiler order)
  __builtin_amdgcn_s_waitcnt(0);
  const bool last = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == total - 1;
  if (last) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  return last;
}
__device__ __forceinline__ uint32_t* scan_counter(ScanPartial* parts, int i) {
  return reinterpret_cast<uint32_t*>(parts + k::kScanParts) + i * k::kScanCounterWords;
}
static_assert(k::kScanCounters * sizeof(ScanPartial) == (k::kScanMax + 1) * k::kScanCounterWords * 4, "");
__device__ __forceinline__ ScanResult* scan_results(ScanPartial* parts) {
  return reinterpret_cast<ScanResult*>(parts + k::kScanParts + k::kScanCounters);
}

template <bool LSE>
__device__ __forceinline__ ScanResult make_result(const Acc& a, const uint32_t* bitmap, uint32_t range,
                                                  uint32_t seq) {
  uint32_t flags = a.nonfinite ? 1u : 0u;
  if (bitmap && a.t.i1 >= 0 && a.t.i1 != 0x7FFFFFFF)
    flags |= ((bitmap[a.t.i1 >> 5] >> (a.t.i1 & 31)) & 1u) << 1;
  flags |= range & kRangeFlag;
  const float lse = LSE && !a.nonfinite ? a.m + __logf(a.s) : __builtin_nanf("");
  return ScanResult{a.t.i1, 0, a.t.v1, a.t.v2, lse, flags, seq, 0};
}

// FULL: d is a multiple of 64 * E, so every lane's chunks are in the row and the loads
// need no predicate.
template <typename T, int NC, bool FULL>
__global__ __launch_bounds__(256) void lmhead_kernel(Shape s, const float* __restrict__ x_row,
                                                     const T* __restrict__ gf,
                                                     const T* __restrict__ W,
                                                     const float* __restrict__ bias,
                                                     float* __restrict__ dist,
                                                     ScanPartial* parts) {
  __shared__ ScanPartial red[4];
  constexpr int E = Elem<T>::kPerFrag;
  const int d = s.d, V = s.vocab;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // z slice of this lane: chunk c covers elements [c*64E + lane*E, +E)
  float z[NC][E];
  bool ok[NC];
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int k0 = c * 64 * E + lane * E;
    ok[c] = FULL || k0 < d;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      z[c][e] = ok[c] ? x_row[k0 + e] : 0.f;
      ss += z[c][e] * z[c][e];
    }
  }
  const float inv = rsqrtf(wave_sum(ss) / d + s.eps);
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int e = 0; e < E; ++e)
      z[c][e] = ok[c] ? z[c][e] * inv * load_elem(gf, c * 64 * E + lane * E + e) : 0.f;

  Acc acc;
  acc_init(acc);
  // wave gw takes rows gw, gw + nw, gw + 2 nw, ... (two per trip): at any moment the
  // waves of the grid read one compact window of rows, not one stream per workgroup.
  // Two register sets alternate, so the next trip's rows (and their biases) are in flight
  // while this trip's are reduced.  Every load is unconditional (rows past V read the
  // last row again, never used; without a bias the biases read x_row and are discarded),
  // so the compiler's wait counts stay exact across the trips.
  const int nw = gridDim.x * 4, gw = blockIdx.x * 4 + wave;
  const float* bsrc = bias ? bias : x_row;
  auto issue = [&](int r, uint4 (&a)[NC], uint4 (&b)[NC], float& sa, float& sb) {
    const int ra = r < V ? r : V - 1, rb = r + nw < V ? r + nw : ra;
    const char* pa = reinterpret_cast<const char*>(W + (int64_t)ra * d);
    const char* pb = reinterpret_cast<const char*>(W + (int64_t)rb * d);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int off = (c * 64 * E + lane * E) * Elem<T>::kBytes;
      a[c] = ok[c] ? ld_stream(pa + off) : make_uint4(0, 0, 0, 0);
      b[c] = ok[c] ? ld_stream(pb + off) : make_uint4(0, 0, 0, 0);
    }
    sa = bsrc[bias ? ra : 0];
    sb = bsrc[bias ? rb : 0];
  };
  auto reduce = [&](int r, const uint4 (&a)[NC], const uint4 (&b)[NC], float sa, float sb) {
    const int r2 = r + nw;
    float da = 0.f, db = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      float fa[E], fb[E];
      frag_to_f32(a[c], fa);
      frag_to_f32(b[c], fb);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        da += z[c][e] * fa[e];
        db += z[c][e] * fb[e];
      }
    }
    da = wave_sum(da);
    db = wave_sum(db);
    const float la = da + (bias ? sa : 0.f);
    if (lane == 0) dist[r] = la;
    acc_push<true>(acc, la, r);
    if (r2 < V) {
      const float lb = db + (bias ? sb : 0.f);
      if (lane == 0) dist[r2] = lb;
      acc_push<true>(acc, lb, r2);
    }
  };
  // trips of this wave: rows gw + 2 nw k, k < trips
  const int trips = gw < V ? (V - gw + 2 * nw - 1) / (2 * nw) : 0;
  uint4 wa0[NC], wb0[NC], wa1[NC], wb1[NC];
  float ba0, bb0, ba1, bb1;
  issue(gw, wa0, wb0, ba0, bb0);
  int k = 0;
  for (; k + 2 < trips; k += 2) {
    issue(gw + (k + 1) * 2 * nw, wa1, wb1, ba1, bb1);
    reduce(gw + k * 2 * nw, wa0, wb0, ba0, bb0);
    issue(gw + (k + 2) * 2 * nw, wa0, wb0, ba0, bb0);
    reduce(gw + (k + 1) * 2 * nw, wa1, wb1, ba1, bb1);
  }
  if (k + 1 < trips) {
    issue(gw + (k + 1) * 2 * nw, wa1, wb1, ba1, bb1);
    reduce(gw + k * 2 * nw, wa0, wb0, ba0, bb0);
    reduce(gw + (k + 1) * 2 * nw, wa1, wb1, ba1, bb1);
  } else if (k < trips) {
    reduce(gw + k * 2 * nw, wa0, wb0, ba0, bb0);
  }
  // every lane holds the same wave accumulator; merge the 4 waves
  __syncthreads();
  if (lane == 0) red[wave] = to_partial(acc);
  __syncthreads();
  if (tid == 0) {
    Acc a = from_partial(red[0]);
    for (int w = 1; w < 4; ++w) acc_merge<true>(a, from_partial(red[w]));
    parts[blockIdx.x] = to_partial(a);
  }
}

// The LM head's second phase: merges the workgroups' partials in a fixed order and writes the
// session's summary.
__global__ __launch_bounds__(256) void lmhead_merge_kernel(const ScanPartial* parts, int nb,
                                                           ScanResult* result,
                                                           const uint32_t* bitmap,
                                                           const uint32_t* range) {
  __shared__ ScanPartial red[4];
  Acc a;
  acc_init(a);
  for (int b = threadIdx.x; b < nb; b += 256) acc_merge<true>(a, from_partial(parts[b]));
  a = block_acc<true>(a, red);
  if (threadIdx.x == 0) *result = make_result<true>(a, bitmap, range ? *range : 0u, 1u);
}

__global__ __launch_bounds__(256) void clear_counters_kernel(ScanPartial* bufs) {
  ScanPartial* b = bufs + blockIdx.x * (k::kScanBufBytes / sizeof(ScanPartial)) + k::kScanParts;
  for (int i = threadIdx.x; i < k::kScanCounters * 2; i += 256)
    reinterpret_cast<uint4*>(b)[i] = make_uint4(0, 0, 0, 0);
}

// What one distribution of a scan needs, from the batch's job or from a job of one (whose
// argument block is 25 times smaller: the workgroups read it from host memory).
struct ScanJob1 {
  float* dist1;
  const uint32_t* bitmap1;
  ScanResult* result1;
  const uint32_t* flag_src1;
  ScanPartial* parts;
  uint32_t* done;
  uint32_t seq;
  __device__ float* dist_of(int) const { return dist1; }
  __device__ const uint32_t* bitmap_of(int) const { return bitmap1; }
  __device__ ScanResult* result_of(int) const { return result1; }
  __device__ const uint32_t* flags_of(int) const { return flag_src1; }
  __device__ const float* src_of(int, int) const { return nullptr; }
  __device__ float4 load4(const float* dist, const float*, int64_t, int v) const {
    return *reinterpret_cast<const float4*>(dist + v);
  }
  __device__ float load1(const float* dist, const float*, int64_t, int v) const { return dist[v]; }
};
struct ScanJobN {
  k::ScanJob j;
  ScanPartial* parts;
  uint32_t* done;
  uint32_t seq;
  __device__ float* dist_of(int b) const { return j.dist[b]; }
  __device__ const uint32_t* bitmap_of(int b) const { return j.bitmap[b]; }
  __device__ ScanResult* result_of(int b) const { return j.result[b]; }
  __device__ const uint32_t* flags_of(int b) const { return j.flag_src[b]; }
  // With `src`, dist[b][v] = sum over splits of src[split][b][v] (+ bias[v]) is formed and
  // stored on the way.
  __device__ const float* src_of(int b, int V) const { return j.src ? j.src + (int64_t)b * V : nullptr; }
  __device__ float4 load4(const float* dist, const float* src, int64_t sstride, int v) const {
    if (!src) return *reinterpret_cast<const float4*>(dist + v);
    float4 q = *reinterpret_cast<const float4*>(src + v);
    for (int k = 1; k < j.src_splits; ++k) {
      const float4 p = *reinterpret_cast<const float4*>(src + k * sstride + v);
      q = make_float4(q.x + p.x, q.y + p.y, q.z + p.z, q.w + p.w);
    }
    if (j.bias) {
      const float4 bb = *reinterpret_cast<const float4*>(j.bias + v);
      q = make_float4(q.x + bb.x, q.y + bb.y, q.z + bb.z, q.w + bb.w);
    }
    return q;
  }
  __device__ float load1(const float* dist, const float* src, int64_t sstride, int v) const {
    if (!src) return dist[v];
    float y = src[v];
    for (int k = 1; k < j.src_splits; ++k) y += src[k * sstride + v];
    return j.bias ? y + j.bias[v] : y;
  }
};

// One launch: grid (blocks, distributions).  Block x of distribution b takes an equal share of
// the vocabulary's 16-byte units, 8 of a thread's loads in flight at once (which is all of them up
// to 131072 values in 64 distributions); a vocabulary that is no multiple of 4 is read value by
// value, one load per thread and trip.  The last workgroup of a distribution merges its partials
// (lane l partial l, nb <= 64) in a fixed order, and the last of the batch writes all results
// (lane b result b).  When they go to host memory (job.done), that one wave makes them visible
// to the host (one system-scope fence, which writes back its L2) and publishes the batch's
// sequence number: a fence per distribution, or per wave, would write the L2 back that many
// times.  With the merge as a second launch and branches in the push, a gate call through the
// Python binding took 28.0 us for one distribution of 128256 and 45.4 us for 64; now 22.6 and
// 36.4 (same box).
template <typename J, bool LSE>
__global__ __launch_bounds__(256) void scan_kernel(int V, J job) {
  constexpr int TPB = 256;
  __shared__ ScanPartial red[4];
  __shared__ int last;
  const int b = blockIdx.y, nb = gridDim.x, n = gridDim.y, tid = threadIdx.x;
  float* dist = job.dist_of(b);
  const float* src = job.src_of(b, V);
  const int64_t sstride = (int64_t)n * V;  // between partial splits of src
  Acc a;
  acc_init(a);
  if ((V & 3) == 0) {
    const int V4 = V >> 2;
    const int u0 = (int)((int64_t)blockIdx.x * V4 / nb), u1 = (int)((int64_t)(blockIdx.x + 1) * V4 / nb);
    constexpr int IN = 8;  // loads in flight per thread
    for (int u = u0 + tid; u < u1; u += IN * TPB) {
      float4 q[IN];
#pragma unroll
      for (int i = 0; i < IN; ++i) {
        const int ui = u + i * TPB;
        if (ui < u1) q[i] = job.load4(dist, src, sstride, 4 * ui);
      }
#pragma unroll
      for (int i = 0; i < IN; ++i) {
        const int ui = u + i * TPB;
        if (ui < u1) {
          if (src) *reinterpret_cast<float4*>(dist + 4 * ui) = q[i];
          acc_push<LSE>(a, q[i].x, 4 * ui);
          acc_push<LSE>(a, q[i].y, 4 * ui + 1);
          acc_push<LSE>(a, q[i].z, 4 * ui + 2);
          acc_push<LSE>(a, q[i].w, 4 * ui + 3);
        }
      }
    }
  } else {
    const int v0 = (int)((int64_t)blockIdx.x * V / nb), v1 = (int)((int64_t)(blockIdx.x + 1) * V / nb);
    for (int v = v0 + tid; v < v1; v += TPB) {
      const float y = job.load1(dist, src, sstride, v);
      if (src) dist[v] = y;
      acc_push<LSE>(a, y, v);
    }
  }
  a = block_acc<LSE>(a, red);
  if (tid == 0) {
    put_record(job.parts + (int64_t)b * nb + blockIdx.x, to_partial(a));
    last = last_arrival(scan_counter(job.parts, b), nb);
  }
  __syncthreads();
  if (!last || tid >= 64) return;
  // the distribution's last workgroup, one wave
  acc_init(a);
  const uint32_t* fs = job.flags_of(b);
  const uint32_t range = fs ? *fs : 0u;
  if (tid < nb) a = from_partial(get_record(job.parts + (int64_t)b * nb + tid));
  a = wave_acc<LSE>(a);
  ScanResult r{};
  bool final = true;
  if (tid == 0) {
    r = make_result<LSE>(a, job.bitmap_of(b), range, job.seq);
    if (n > 1) {
      put_record(scan_results(job.parts) + b, r);
      final = last_arrival(scan_counter(job.parts, k::kScanMax), n);
    }
  }
  if (!__shfl((int)final, 0, 64)) return;
  // the batch's last workgroup
  if (n > 1 && tid < n) r = get_record(scan_results(job.parts) + tid);
  if (tid < n) {  // two 16-byte stores per result (the record is 32-byte aligned)
    uint4 w[2];
    __builtin_memcpy(w, &r, 32);
    uint4* dst = reinterpret_cast<uint4*>(job.result_of(tid));
    dst[0] = w[0];
    dst[1] = w[1];
  }
  if (job.done) {
    __threadfence_system();  // every lane's results, before the number the host polls
    if (tid == 0) *reinterpret_cast<volatile uint32_t*>(job.done) = job.seq;
    __threadfence_system();
  }
}

template <typename T>
hipError_t launch_lmhead(const Shape& s, const float* x_row, const void* g_final, const void* w_lm,
                         const float* bias, float* dist, const uint32_t* bitmap,
                         ScanPartial* parts, ScanResult* result, const uint32_t* range,
                         hipStream_t st) {
  constexpr int E = Elem<T>::kPerFrag;
  const int nc = (s.d + 64 * E - 1) / (64 * E);
  const int nb = k::lmhead_blocks(s);
  const T* g = static_cast<const T*>(g_final);
  const T* W = static_cast<const T*>(w_lm);
  const bool full = s.d % (64 * E) == 0;
#define SPP_LMHEAD(NCV)                                                                        \
  if (full)                                                                                    \
    SPP_LAUNCH((lmhead_kernel<T, NCV, true>), dim3(nb), dim3(256), 0, st, s, x_row, g, W, bias, \
               dist, parts);                                                                   \
  else                                                                                         \
    SPP_LAUNCH((lmhead_kernel<T, NCV, false>), dim3(nb), dim3(256), 0, st, s, x_row, g, W, bias, \
               dist, parts)
  switch (nc) {
    case 1: SPP_LMHEAD(1); break;
    case 2: SPP_LMHEAD(2); break;
    case 4: SPP_LMHEAD(4); break;
    case 8: SPP_LMHEAD(8); break;
    case 10: SPP_LMHEAD(10); break;
    case 16: SPP_LMHEAD(16); break;
    default: return hipErrorInvalidValue;
  }
#undef SPP_LMHEAD
  SPP_LAUNCH(lmhead_merge_kernel, dim3(1), dim3(256), 0, st, parts, nb, result, bitmap, range);
  return hipGetLastError();
}

}  // namespace

namespace k {

// One 4-wave workgroup per CU of the MI355X (256 CUs): measured against 128 to 1024
// workgroups at the 8B and 70B vocabularies, more waves in flight streamed W_lm slower.
#ifndef SPP_LMHEAD_MAX_BLOCKS
#define SPP_LMHEAD_MAX_BLOCKS 256
#endif
int lmhead_blocks(const Shape& s) {
  int nb = (s.vocab + 31) / 32;  // at least 32 rows per block
  return nb < SPP_LMHEAD_MAX_BLOCKS ? (nb < 1 ? 1 : nb) : SPP_LMHEAD_MAX_BLOCKS;
}

hipError_t lmhead_gemv(const Shape& s, const float* x_row, const void* g_final, const void* w_lm,
                       const float* bias, float* dist, const uint32_t* bitmap,
                       ScanPartial* parts, ScanResult* result, const uint32_t* range,
                       hipStream_t st) {
  return s.bf16 ? launch_lmhead<bf16_t>(s, x_row, g_final, w_lm, bias, dist, bitmap, parts,
                                        result, range, st)
                : launch_lmhead<float>(s, x_row, g_final, w_lm, bias, dist, bitmap, parts,
                                       result, range, st);
}

// Launch shape of a scan of n distributions of `vocab` logits: 256-thread blocks, about
// 1024 of them over the batch (a batch of 64 fills the chip four times over; 1024-thread
// blocks, one per CU, measured slower), between 4 and 64 per distribution, and no block
// with fewer than one of the vocabulary's 16-byte units per thread.
void scan_launch(int vocab, int n, int* nb, int* tpb) {
  n = n < 1 ? 1 : n;
  *tpb = 256;
  *nb = 1024 / n;
  if (*nb < 4) *nb = 4;
  if (*nb > kScanMaxBlocks) *nb = kScanMaxBlocks;
  const int cap = (vocab + 4 * *tpb - 1) / (4 * *tpb);
  if (*nb > cap) *nb = cap;
  if (*nb < 1) *nb = 1;
}

hipError_t clear_scan_counters(ScanPartial* bufs, int n, hipStream_t st) {
  static_assert(kScanBufBytes % sizeof(ScanPartial) == 0 && sizeof(ScanPartial) == 32, "whole partials");
  SPP_LAUNCH(clear_counters_kernel, dim3(n), dim3(256), 0, st, bufs);
  return hipGetLastError();
}

hipError_t scan(const Shape& s, int n, const ScanJob& job, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (n > kScanMax) return hipErrorInvalidValue;
  int nb, tpb;
  scan_launch(s.vocab, n, &nb, &tpb);
  const dim3 grid(nb, n), block(tpb);
  if (n == 1 && !job.src && !job.with_lse) {
    const ScanJob1 j{job.dist[0], job.bitmap[0], job.result[0], job.flag_src[0], job.parts, job.done, job.seq};
    SPP_LAUNCH((scan_kernel<ScanJob1, false>), grid, block, 0, st, s.vocab, j);
  } else {
    const ScanJobN j{job, job.parts, job.done, job.seq};
    if (job.with_lse)
      SPP_LAUNCH((scan_kernel<ScanJobN, true>), grid, block, 0, st, s.vocab, j);
    else
      SPP_LAUNCH((scan_kernel<ScanJobN, false>), grid, block, 0, st, s.vocab, j);
  }
  return hipGetLastError();
}

}  // namespace k
}  // namespace spp

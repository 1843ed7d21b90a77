// Route: gate scoring and top-k selection (Sec. III-B-2: each token goes to
// its top-k activated experts; Alg. 2: the expert map is computed from the
// local hidden states).
//
// The selected ids must be those of exact arithmetic on the stored inputs,
// whatever the summation order.  Three stages make that cheap:
//   1. gate GEMM   bf16 MFMA 32x32x16, fp32 accumulation in short chains that
//                  are flushed into fp64 sums; also the squared row norms
//   2. select      one wavefront per token: keys, group limit, top-k by
//                  shuffle arg-max, and an interval test: every comparison
//                  the selection relied on must hold for ANY keys within the
//                  error bound of stage 1; tokens that fail are listed
//   3. re-score    one workgroup per listed token: the experts whose key
//                  interval reaches the selection get an fp64 dot product and
//                  the selection is redone in fp64
// Short batches (and fp32 rows) skip all three: every logit is computed in fp64, on the
// vector unit or the fp64 matrix instructions, and the selection works on fp64 keys.
// Error model of stage 1 for a chain of n bf16 products (exact in fp32) added
// in fp32: every addition is off by at most one ulp of the running sum, so
// |error| <= 2n * 2^-24 * sum|x_h w_h| <= 2n * 2^-24 * |x|_2 |w|_2.
#include <limits.h>

#include "moe_internal.h"

namespace moe {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr float kUlp = 5.9604645e-8f;   // 2^-24

// ------------------------------------------------------------------ helpers
// Pairwise lane exchange, step s pairs disjoint groups of 2^s lanes: steps 0..3
// are DPP moves inside a row of 16 lanes (quad permutes, then the half-row and
// row mirrors: after the quads are uniform a mirror pairs each lane with a lane
// of the other group), steps 4 and 5 cross rows through the LDS crossbar.
template <int CTRL>
__device__ __forceinline__ int dpp_mov(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}

template <int STEP>
__device__ __forceinline__ int lane_xchg32(int v) {
  if (STEP == 0) return dpp_mov<0xB1>(v);        // quad_perm [1,0,3,2]
  if (STEP == 1) return dpp_mov<0x4E>(v);        // quad_perm [2,3,0,1]
  if (STEP == 2) return dpp_mov<0x141>(v);       // row_half_mirror
  if (STEP == 3) return dpp_mov<0x140>(v);       // row_mirror
  return __shfl_xor(v, STEP == 4 ? 16 : 32);
}

template <int STEP>
__device__ __forceinline__ int lane_xchg(int v) { return lane_xchg32<STEP>(v); }
template <int STEP>
__device__ __forceinline__ float lane_xchg(float v) {
  return __builtin_bit_cast(float, lane_xchg32<STEP>(__builtin_bit_cast(int, v)));
}
template <int STEP>
__device__ __forceinline__ double lane_xchg(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)lane_xchg32<STEP>((int)(uint32_t)u);
  const uint32_t hi = (uint32_t)lane_xchg32<STEP>((int)(uint32_t)(u >> 32));
  return __builtin_bit_cast(double, (uint64_t(hi) << 32) | lo);
}

#define MOE_ALL_STEPS(F) F(0) F(1) F(2) F(3) F(4) F(5)

// Value of lane `l` (the same l in every lane) as a scalar broadcast: no LDS crossbar.
__device__ __forceinline__ int read_lane(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ float read_lane(float v, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
__device__ __forceinline__ double read_lane(double v, int l) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
  return __builtin_bit_cast(double, (uint64_t(hi) << 32) | lo);
}

// Sum over the wave in a fixed order, the same in every lane: a butterfly inside
// each row of 16 lanes, then (row0 + row1) + (row2 + row3) from the row results
// read as scalars.
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#define STEP_(S) v += lane_xchg<S>(v);
  STEP_(0) STEP_(1) STEP_(2) STEP_(3)
#undef STEP_
  const T r0 = read_lane(v, 0), r1 = read_lane(v, 16), r2 = read_lane(v, 32), r3 = read_lane(v, 48);
  return (r0 + r1) + (r2 + r3);
}

// Largest value over the wave, the same in every lane: the four DPP steps make
// each row of 16 lanes uniform, the four row results are then read as scalars.
template <typename T>
__device__ __forceinline__ T wave_max(T v) {
#define STEP_(S) { const T o = lane_xchg<S>(v); v = o > v ? o : v; }
  STEP_(0) STEP_(1) STEP_(2) STEP_(3)
#undef STEP_
  const T r0 = read_lane(v, 0), r1 = read_lane(v, 16), r2 = read_lane(v, 32), r3 = read_lane(v, 48);
  const T a = r1 > r0 ? r1 : r0, b = r3 > r2 ? r3 : r2;
  return b > a ? b : a;
}

// Largest value over the wave, ties to the lowest index, which must not fall from one
// lane to the next: the first lane that holds the maximum has it.  idx == INT_MAX marks
// "no candidate".  Result is the same in every lane.
template <typename T>
__device__ __forceinline__ void wave_argmax(T& v, int& idx) {
  const bool cand = idx != INT_MAX;
  const T vv = cand ? v : (T)-INFINITY;
  const T m = wave_max(vv);
  const uint64_t tie = __ballot(cand && vv == m);
  idx = tie != 0 ? read_lane(idx, __ffsll((unsigned long long)tie) - 1) : INT_MAX;
  v = tie != 0 ? m : (T)0;
}

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t hi16) {
  return __uint_as_float(hi16 << 16);
}

// Sum of squares of the eight bf16 values of a 16-byte piece, added to acc (fp32).
__device__ __forceinline__ float piece_sumsq(const uint4& a, float acc) {
  const uint32_t v[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float lo = bf16_bits_to_f32(v[q] & 0xffffu), hi = bf16_bits_to_f32(v[q] >> 16);
    acc = fmaf(lo, lo, acc);
    acc = fmaf(hi, hi, acc);
  }
  return acc;
}

// fp64 dot product (exact products) of two 16-byte pieces, 8 bf16 or 4 fp32, added to acc.
template <bool BF16>
__device__ __forceinline__ double piece_dot64(const uint4& a, const uint4& b, double acc) {
  const uint32_t av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (BF16) {
      acc = fma((double)bf16_bits_to_f32(av[i] & 0xffffu), (double)bf16_bits_to_f32(bv[i] & 0xffffu), acc);
      acc = fma((double)bf16_bits_to_f32(av[i] >> 16), (double)bf16_bits_to_f32(bv[i] >> 16), acc);
    } else {
      acc = fma((double)__uint_as_float(av[i]), (double)__uint_as_float(bv[i]), acc);
    }
  }
  return acc;
}

// Clears the re-score counter where no gate GEMM does (logits given by the caller): a
// kernel rather than a memset, so the call can be captured in a graph.
__global__ void clear_counters_kernel(int32_t* __restrict__ counters) { counters[threadIdx.x] = 0; }

// ------------------------------------------ stage 1 (bf16): MFMA gate GEMM
// Register-staged variant, used when H is not a multiple of 64 (it zero-fills
// the K tail); otherwise gate_dma_kernel below runs the same tile.
// Block tile 64 tokens x 128 experts, K step 64, 8 wavefronts as 2 (M) x 4 (N),
// each one 32x32 MFMA tile (16 fp32 accumulators flushed into 16 fp64 sums every
// K step): the flush is as much VALU work as the MFMAs are matrix work, so many
// light wavefronts per SIMD (three workgroups fit a CU) overlap the two and the
// register-staged loads better than four wavefronts with two tiles each did.
// LDS tiles are [row][8 pieces of 16 B] with the piece index XOR-ed by (row/2)&7
// so that the 16 lanes the LDS serves per cycle fall on 16 different 16-byte
// columns.
// K of the gate GEMM is split until about this many workgroups run (2 per CU)
constexpr int GBM = kGateTileM, GBN = kGateTileN, GBK = 64;

__device__ __forceinline__ int swz(int row, int piece) {
  return row * 8 + (piece ^ ((row >> 1) & 7));
}

template <int CHAIN_STEPS>
__global__ __launch_bounds__(512) void gate_mfma_kernel(const uint16_t* __restrict__ x,
                                                        const uint16_t* __restrict__ gate_w, int T,
                                                        int H, int E, float* __restrict__ logits,
                                                        float* __restrict__ xnorm2,
                                                        float* __restrict__ wnorm2,
                                                        int32_t* __restrict__ counters) {
  __shared__ uint4 As[2][GBM * 8];
  __shared__ uint4 Bs[2][GBN * 8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  const int m0 = blockIdx.x * GBM, n0 = blockIdx.y * GBN;
  const int all_steps = (H + GBK - 1) / GBK;
  const int per_split = (all_steps + gridDim.z - 1) / gridDim.z;
  const int ks0 = blockIdx.z * per_split;
  const int ksteps = (ks0 + per_split < all_steps ? ks0 + per_split : all_steps) - ks0;
  logits += size_t(blockIdx.z) * T * E;
  xnorm2 += size_t(blockIdx.z) * T;
  wnorm2 += size_t(blockIdx.z) * E;
  if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && tid < 64) counters[tid] = 0;

  // global -> register staging: A 1 piece / thread, B 2 pieces / thread
  const int lrow = tid >> 3, lpiece = tid & 7;        // lrow 0..63
  uint4 ra, rb[2];
  float xsq = 0.f, wsq[2] = {0.f, 0.f};
  auto gload = [&](int ks) {
    const int kcol = (ks0 + ks) * GBK + lpiece * 8;
    const bool kin = kcol < H;
    int r = m0 + lrow;
    r = r < T ? r : T - 1;
    ra = kin ? *reinterpret_cast<const uint4*>(x + size_t(r) * H + kcol) : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      int n = n0 + lrow + 64 * i;
      n = n < E ? n : E - 1;
      rb[i] = kin ? *reinterpret_cast<const uint4*>(gate_w + size_t(n) * H + kcol) : make_uint4(0, 0, 0, 0);
    }
  };
  auto lstore = [&](int buf) {
    As[buf][swz(lrow, lpiece)] = ra;
    const uint32_t v[4] = {ra.x, ra.y, ra.z, ra.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float lo = bf16_bits_to_f32(v[q] & 0xffffu), hi = bf16_bits_to_f32(v[q] >> 16);
      xsq = fmaf(lo, lo, xsq);
      xsq = fmaf(hi, hi, xsq);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) Bs[buf][swz(lrow + 64 * i, lpiece)] = rb[i];
    if (blockIdx.x == 0) {                            // the first token tile also sums the gate rows' squares
#pragma unroll
      for (int i = 0; i < 2; ++i) wsq[i] = piece_sumsq(rb[i], wsq[i]);
    }
  };

  f32x16 acc;
  double dsum[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) { acc[i] = 0.f; dsum[i] = 0.0; }

  gload(0);
  lstore(0);
  __syncthreads();
  for (int ks = 0; ks < ksteps; ++ks) {
    const int buf = ks & 1;
    if (ks + 1 < ksteps) gload(ks + 1);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int piece = kk * 2 + (lane >> 5);
      const uint4 av = As[buf][swz(wm * 32 + (lane & 31), piece)];
      const uint4 bv = Bs[buf][swz(wn * 32 + (lane & 31), piece)];
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av),
                                                    __builtin_bit_cast(bf16x8, bv), acc, 0, 0, 0);
    }
    if ((ks + 1) % CHAIN_STEPS == 0 || ks + 1 == ksteps) {
#pragma unroll
      for (int i = 0; i < 16; ++i) { dsum[i] += (double)acc[i]; acc[i] = 0.f; }
    }
    if (ks + 1 < ksteps) lstore(buf ^ 1);
    __syncthreads();
  }

  // D layout of the 32x32 MFMA: lane l, register i -> row (i/4)*8 + (l/32)*4 + i%4, col l%32
  const int col = n0 + wn * 32 + (lane & 31);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int row = m0 + wm * 32 + (i >> 2) * 8 + (lane >> 5) * 4 + (i & 3);
    if (row < T && col < E) logits[size_t(row) * E + col] = (float)dsum[i];
  }
  // squared row norms: the 8 threads with equal lrow hold one row's pieces
  if (blockIdx.y == 0) {
    float s = xsq;
    s += __shfl_xor(s, 1);
    s += __shfl_xor(s, 2);
    s += __shfl_xor(s, 4);
    const int r = m0 + lrow;
    if (lpiece == 0 && r < T) xnorm2[r] = s * 1.001f;
  }
  if (blockIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float s = wsq[i];
      s += __shfl_xor(s, 1);
      s += __shfl_xor(s, 2);
      s += __shfl_xor(s, 4);
      const int n = n0 + lrow + 64 * i;
      if (lpiece == 0 && n < E) wnorm2[n] = s * 1.001f;
    }
  }
}

// The gate GEMM with the operands brought global -> LDS directly
// (`global_load_lds_dwordx4`, no staging registers) into a ring of NS stages:
// one barrier per K step and an explicit vmcnt wait that leaves the younger
// stages in flight.  Tile BM tokens x 128 experts, eight wavefronts as BM/32 (M)
// x 256/BM (N), one or two 32x32 MFMA tiles each.  Needs H to be a multiple of 64
// (a DMA cannot zero-fill a K tail).  LDS slot s of a stage holds (row s/8, piece
// (s%8) ^ (row/2)&7): the lane that owns the slot fetches that piece, which is
// the swz() layout the fragment reads expect.
typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14));
}

template <int BM, int NS, int CHAIN_STEPS>
__device__ __forceinline__ void gate_dma_body(const uint16_t* __restrict__ x,
                                              const uint16_t* __restrict__ gate_w, int T, int H,
                                              int E, float* __restrict__ logits,
                                              float* __restrict__ xnorm2,
                                              float* __restrict__ wnorm2,
                                              int32_t* __restrict__ counters, uint4* smem) {
  constexpr int MW = BM / 32;                // wavefronts along M
  constexpr int NT = (GBN / 32) * MW / 8;    // MFMA tiles (32 experts each) per wavefront
  constexpr int NA = BM / 64;                // A load instructions per thread and step
  constexpr int NLOAD = NA + 2;              // load instructions per thread and step
  uint4* const As = smem;                    // [NS][BM * 8]
  uint4* const Bs = smem + NS * BM * 8;      // [NS][GBN * 8]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % MW, wn = wave / MW;
  const int m0 = blockIdx.x * BM, n0 = blockIdx.y * GBN;
  const int all_steps = H / GBK;
  const int per_split = (all_steps + gridDim.z - 1) / gridDim.z;
  const int ks0 = blockIdx.z * per_split;
  const int ksteps = (ks0 + per_split < all_steps ? ks0 + per_split : all_steps) - ks0;
  logits += size_t(blockIdx.z) * T * E;
  xnorm2 += size_t(blockIdx.z) * T;
  wnorm2 += size_t(blockIdx.z) * E;
  if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && tid < 64) counters[tid] = 0;

  // this thread's slots: tid + 512 i of the A stage (i < NA) and of the B stage (i < 2);
  // rows lrow + 64 i, and (lrow + 64 i) / 2 & 7 does not depend on i
  const int lrow = tid >> 3;
  const int gpiece = (tid & 7) ^ ((lrow >> 1) & 7);
  const uint16_t* asrc[NA];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int r = m0 + lrow + 64 * i;
    asrc[i] = x + size_t(r < T ? r : T - 1) * H + gpiece * 8;
  }
  const uint16_t* bsrc[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int n = n0 + lrow + 64 * i;
    bsrc[i] = gate_w + size_t(n < E ? n : E - 1) * H + gpiece * 8;
  }
  auto issue = [&](int ks) {
    const int kcol = (ks0 + ks) * GBK;
    const int st = ks % NS;
#pragma unroll
    for (int i = 0; i < NA; ++i)
      __builtin_amdgcn_global_load_lds((gptr_t)(asrc[i] + kcol),
                                       (lptr_t)(As + st * BM * 8 + (i * 8 + wave) * 64), 16, 0, 0);
#pragma unroll
    for (int i = 0; i < 2; ++i)
      __builtin_amdgcn_global_load_lds((gptr_t)(bsrc[i] + kcol),
                                       (lptr_t)(Bs + st * GBN * 8 + (i * 8 + wave) * 64), 16, 0, 0);
  };

  f32x16 acc[NT];
  double dsum[NT][16];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) { acc[j][i] = 0.f; dsum[j][i] = 0.0; }
  float xsq[NA], wsq[2] = {0.f, 0.f};
#pragma unroll
  for (int i = 0; i < NA; ++i) xsq[i] = 0.f;

#pragma unroll
  for (int d = 0; d < NS - 1; ++d)
    if (d < ksteps) issue(d);
  for (int ks = 0; ks < ksteps; ++ks) {
    // step ks must have landed; the NS-2 younger steps may stay in flight
    if (ks + NS - 2 < ksteps) wait_vmcnt<NLOAD * (NS - 2)>(); else wait_vmcnt<0>();
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    // every wavefront is done with step ks-1: refill its stage
    if (ks + NS - 1 < ksteps) issue(ks + NS - 1);
    const uint4* const Ast = As + (ks % NS) * BM * 8;
    const uint4* const Bst = Bs + (ks % NS) * GBN * 8;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int piece = kk * 2 + (lane >> 5);
      const uint4 av = Ast[swz(wm * 32 + (lane & 31), piece)];
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const uint4 bv = Bst[swz((wn * NT + j) * 32 + (lane & 31), piece)];
        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av),
                                                         __builtin_bit_cast(bf16x8, bv), acc[j], 0, 0, 0);
      }
    }
    if (blockIdx.y == 0) {                        // squared row norms from this thread's own pieces
#pragma unroll
      for (int i = 0; i < NA; ++i) xsq[i] = piece_sumsq(Ast[tid + 512 * i], xsq[i]);
    }
    if (blockIdx.x == 0) {                        // the first token tile also sums the gate rows' squares
#pragma unroll
      for (int i = 0; i < 2; ++i) wsq[i] = piece_sumsq(Bst[tid + 512 * i], wsq[i]);
    }
    if ((ks + 1) % CHAIN_STEPS == 0 || ks + 1 == ksteps) {
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) { dsum[j][i] += (double)acc[j][i]; acc[j][i] = 0.f; }
    }
  }

  // D layout of the 32x32 MFMA: lane l, register i -> row (i/4)*8 + (l/32)*4 + i%4, col l%32
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int col = n0 + (wn * NT + j) * 32 + (lane & 31);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int row = m0 + wm * 32 + (i >> 2) * 8 + (lane >> 5) * 4 + (i & 3);
      if (row < T && col < E) logits[size_t(row) * E + col] = (float)dsum[j][i];
    }
  }
  if (blockIdx.y == 0) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      float s = xsq[i];
      s += __shfl_xor(s, 1);
      s += __shfl_xor(s, 2);
      s += __shfl_xor(s, 4);
      const int r = m0 + lrow + 64 * i;
      if ((tid & 7) == 0 && r < T) xnorm2[r] = s * 1.001f;
    }
  }
  if (blockIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float s = wsq[i];
      s += __shfl_xor(s, 1);
      s += __shfl_xor(s, 2);
      s += __shfl_xor(s, 4);
      const int n = n0 + lrow + 64 * i;
      if ((tid & 7) == 0 && n < E) wnorm2[n] = s * 1.001f;
    }
  }
}

template <int BM, int NS, int CHAIN_STEPS>
__global__ __launch_bounds__(512) void gate_dma_kernel(const uint16_t* __restrict__ x,
                                                       const uint16_t* __restrict__ gate_w, int T,
                                                       int H, int E, float* __restrict__ logits,
                                                       float* __restrict__ xnorm2,
                                                       float* __restrict__ wnorm2,
                                                       int32_t* __restrict__ counters) {
  extern __shared__ uint4 gate_smem[];
  // The ring is handed on as a generic pointer: with the LDS array named in the
  // loop the compiler puts a vmcnt(0) in front of every LDS read that follows a
  // DMA in program order, which would drain the ring; the waits and the barrier
  // in the body order the DMA writes and the reads explicitly.
  gate_dma_body<BM, NS, CHAIN_STEPS>(x, gate_w, T, H, E, logits, xnorm2, wnorm2, counters, gate_smem);
}

// ----------------------------------------------------------- stage 2: select
struct SelCfg {
  int E, k, score_fn, renormalize, G, Kg, gn;
  float scale;
  float chain_err;   // 2n * 2^-24 of the gate accumulation (0 when logits are given)
  int have_norms;
  int nsplit;        // K splits of the gate GEMM: logits, token-row and gate-row norms are sums of this many slabs
  int T;             // tokens: slab strides are T*E (logits) and T (row norms)
};

// The gate's form, fixed at compile time for the two forms that layers are served with.
// The routing kernels are short: much of their time is fetching their own code, one
// cache line after the other on every CU, so a kernel holds what its gate executes.
enum GateForm {
  kGateSoftmax,    // softmax scores, no group limit
  kGateGrouped,    // sigmoid scores, group limit over aligned runs of whole lanes (aligned_groups)
  kGateAny         // everything else: decided at run time
};
template <int FORM> __device__ __forceinline__ bool is_softmax(const SelCfg& c) {
  return FORM == kGateSoftmax || (FORM == kGateAny && c.score_fn == MOE_SCORE_SOFTMAX);
}
template <int FORM> __device__ __forceinline__ bool has_groups(const SelCfg& c) {
  return FORM == kGateGrouped || (FORM == kGateAny && c.G > 1);
}
// Groups that are aligned runs of 1, 2, 4 .. 64 whole lanes, scored by one or two keys.
template <int EPL> __host__ __device__ __forceinline__ bool aligned_groups(const SelCfg& c) {
  const int gs = c.E / c.G;
  return gs % EPL == 0 && 64 % (gs / EPL) == 0 && c.gn <= 2;
}
// Group of the lane's expert i.
template <int EPL, int FORM> __device__ __forceinline__ int lane_group(const SelCfg& c, int lane, int i) {
  return (lane * EPL + (FORM == kGateGrouped ? 0 : i)) / (c.E / c.G);
}
template <int EPL> inline GateForm gate_form(const SelCfg& c) {
  if (c.G <= 1 && c.score_fn == MOE_SCORE_SOFTMAX) return kGateSoftmax;
  if (c.G > 1 && c.score_fn == MOE_SCORE_SIGMOID && aligned_groups<EPL>(c)) return kGateGrouped;
  return kGateAny;
}

// Sum of element p of `ns` (1, 2 or 4) slabs `stride` apart, in slab order.  The loads do not
// wait for one another: a slab loop that adds as it goes is one memory latency per slab.
__device__ __forceinline__ float slab_sum(const float* __restrict__ p, size_t stride, int ns) {
  if (ns == 1) return p[0];
  const float a = p[0], b = p[stride];
  if (ns == 2) return a + b;
  const float c = p[2 * stride], d = p[3 * stride];
  return ((a + b) + c) + d;
}

// The lane's EPL neighbouring elements of p[0, n), zeros past the end; whole 16-byte pieces
// where the rows keep their alignment (512 experts: two loads a lane and not eight, each of
// which would touch 16 times the lines it needs).
template <int EPL>
__device__ __forceinline__ void load_run(const float* __restrict__ p, int n, int lane, float (&v)[EPL]) {
  if (EPL % 4 == 0 && n % 4 == 0) {
#pragma unroll
    for (int i = 0; i < EPL; i += 4) {
      const int e = lane * EPL + i;
      const float4 q = e < n ? *reinterpret_cast<const float4*>(p + e) : make_float4(0.f, 0.f, 0.f, 0.f);
      v[i] = q.x;
      if (i + 1 < EPL) v[i + 1] = q.y;
      if (i + 2 < EPL) v[i + 2] = q.z;
      if (i + 3 < EPL) v[i + 3] = q.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < EPL; ++i) v[i] = lane * EPL + i < n ? p[lane * EPL + i] : 0.f;
  }
}
// The same of the slabs' sum, all loads first.
template <int EPL>
__device__ __forceinline__ void load_slabs(const float* __restrict__ p, int n, size_t stride, int ns, int lane,
                                           float (&v)[EPL]) {
  load_run<EPL>(p, n, lane, v);
  if (ns == 1) return;
  float b[EPL];
  load_run<EPL>(p + stride, n, lane, b);
  if (ns == 2) {
#pragma unroll
    for (int i = 0; i < EPL; ++i) v[i] += b[i];
    return;
  }
  float c[EPL], d[EPL];
  load_run<EPL>(p + 2 * stride, n, lane, c);
  load_run<EPL>(p + 3 * stride, n, lane, d);
#pragma unroll
  for (int i = 0; i < EPL; ++i) v[i] = ((v[i] + b[i]) + c[i]) + d[i];
}

// Norm of token t's row from the per-split sums of squares.
__device__ __forceinline__ float token_norm(const SelCfg& c, const float* __restrict__ xnorm2, int t) {
  if (!c.have_norms) return 0.f;
  return sqrtf(slab_sum(xnorm2 + t, c.T, c.nsplit));
}

// Fast key of one expert from its stage-1 logit z (the slabs already added up):
// key, the bound eps on |key - exact key|, and the value sc the weight is made of.
// wn = norm of the gate row (unused without norms).
template <int FORM>
__device__ __forceinline__ void fast_key_one(const SelCfg& c, float z, float xn, float wn,
                                             const float* __restrict__ logit_bias,
                                             const float* __restrict__ select_bias, int e,
                                             float& key, float& eps, float& sc) {
  float ez = 0.f;
  if (c.have_norms) ez = c.chain_err * xn * wn * 1.001f + 2.f * kUlp * fabsf(z);
  if (logit_bias) {
    z += logit_bias[e];
    ez += kUlp * fabsf(z);
  }
  if (is_softmax<FORM>(c)) {
    key = z; eps = ez; sc = z;
  } else {
    const float s = 1.0f / (1.0f + expf(-z));
    const float sb = select_bias ? select_bias[e] : 0.f;
    key = s + sb;
    sc = s;
    // |sigmoid(z+d)-sigmoid(z)| <= s(1-s)|d| + d^2/16 ; fp32 evaluation of
    // the sigmoid and of the bias add is good to a few ulp of 1+|sb|
    eps = ez * (s * (1.f - s) + ez + 16.f * kUlp) + 16.f * kUlp * (1.f + fabsf(sb));
  }
}

// Per-lane view of one token's experts: lane l holds experts l*EPL .. l*EPL + EPL-1, so that a
// group of experts is a run of lanes and what its lanes hold is first combined in registers.
template <typename FT, int EPL>
struct Keys {
  FT key[EPL];   // selection key
  FT eps[EPL];   // bound on |key - exact key|
  FT sc[EPL];    // value the weight is made of: logit (softmax) or sigmoid score
};

template <typename FT>
struct Groups {
  uint64_t kept;    // bit g: group g survives the group limit
  bool certain;     // the cut between kept and dropped groups holds for any keys within eps
  uint32_t need;    // bit per slot: the expert may be one of its group's group_score_n largest
  uint64_t open;    // bit g: whether group g is kept depends on exact scores
};

template <typename FT>
struct Picks {
  int id;        // lane j < k: j-th pick
  FT sc;         // its logit / score
  FT low;        // smallest lower bound of a picked key
  bool certain;  // every comparison held with the error intervals apart
};

// Fast keys of token t from the stage-1 logits.  All loads come first.
template <int EPL, int FORM>
__device__ __forceinline__ void fast_keys(const SelCfg& c, const float* __restrict__ logits_row,
                                          const float* __restrict__ logit_bias,
                                          const float* __restrict__ select_bias, float xn,
                                          const float* __restrict__ wnorm2, int lane,
                                          Keys<float, EPL>& K) {
  float z[EPL], wn2[EPL];
  load_slabs<EPL>(logits_row, c.E, size_t(c.T) * c.E, c.nsplit, lane, z);
  if (c.have_norms) {
    load_slabs<EPL>(wnorm2, c.E, c.E, c.nsplit, lane, wn2);
  } else {
#pragma unroll
    for (int i = 0; i < EPL; ++i) wn2[i] = 0.f;
  }
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const int e = lane * EPL + i;
    float key = -INFINITY, eps = 0.f, sc = 0.f;
    if (e < c.E)
      fast_key_one<FORM>(c, z[i], xn, c.have_norms ? sqrtf(wn2[i]) : 0.f, logit_bias, select_bias, e, key, eps, sc);
    K.key[i] = key; K.eps[i] = eps; K.sc[i] = sc;
  }
}

// Group limit: keep the Kg groups with the largest sum of their gn largest
// keys; ties go to the lowest group.  Lane g ends up holding group g's score.
template <typename FT, int EPL, int FORM>
__device__ __forceinline__ void group_stage(const SelCfg& c, const Keys<FT, EPL>& K, int lane,
                                            Groups<FT>& Gp) {
  const int gs = c.E / c.G;
  FT gsum = 0, gerr = 0;          // lane g: score of group g and the bound on its error
  uint32_t need = 0;
  if (FORM == kGateGrouped || aligned_groups<EPL>(c)) {
    // (max1, max2, max eps, two largest lower bounds) of the lane's own keys, then a
    // butterfly over the lanes of each group, all groups at once
    const int gl = gs / EPL;
    FT m1 = -INFINITY, m2 = -INFINITY, me = 0, l1 = -INFINITY, l2 = -INFINITY;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const FT k = K.key[i], l = k - K.eps[i];
      const FT klo = k < m1 ? k : m1, llo = l < l1 ? l : l1;
      m1 = k > m1 ? k : m1;
      m2 = klo > m2 ? klo : m2;
      l1 = l > l1 ? l : l1;
      l2 = llo > l2 ? llo : l2;
      me = K.eps[i] > me ? K.eps[i] : me;
    }
#define STEP_(S)                                                                   \
  if ((1 << S) < gl) {                                                             \
    const FT o1 = lane_xchg<S>(m1), o2 = lane_xchg<S>(m2), oe = lane_xchg<S>(me);  \
    const FT p1 = lane_xchg<S>(l1), p2 = lane_xchg<S>(l2);                         \
    const FT lo = m1 < o1 ? m1 : o1, hi2 = m2 > o2 ? m2 : o2;                      \
    m1 = m1 > o1 ? m1 : o1;                                                        \
    m2 = lo > hi2 ? lo : hi2;                                                      \
    me = me > oe ? me : oe;                                                        \
    const FT ql = l1 < p1 ? l1 : p1, qh = l2 > p2 ? l2 : p2;                       \
    l1 = l1 > p1 ? l1 : p1;                                                        \
    l2 = ql > qh ? ql : qh;                                                        \
  }
    MOE_ALL_STEPS(STEP_)
#undef STEP_
    const FT sum = c.gn == 2 ? m1 + m2 : m1;
    const FT nth_low = c.gn == 2 ? l2 : l1;              // <= the gn-th largest exact key
#pragma unroll
    for (int i = 0; i < EPL; ++i)
      if (K.key[i] + K.eps[i] >= nth_low) need |= 1u << i;
    // lane g fetches its group's values from the first lane of the run
    const int src = lane < c.G ? lane * gl : 0;
    gsum = __shfl(sum, src);
    gerr = __shfl(me, src) * (FT)c.gn;
  } else {
    for (int g = 0; g < c.G; ++g) {
      uint32_t taken = 0;
      FT sum = 0, me = 0, nth_low = INFINITY;
#pragma unroll
      for (int i = 0; i < EPL; ++i) {
        const int e = lane * EPL + i;
        if (e < c.E && e / gs == g) me = K.eps[i] > me ? K.eps[i] : me;
      }
      me = wave_max(me);
      for (int r = 0; r < c.gn; ++r) {
        FT v = 0; int idx = INT_MAX;
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
          const int e = lane * EPL + i;
          if (e < c.E && e / gs == g && !(taken >> i & 1) && (idx == INT_MAX || K.key[i] > v)) {
            v = K.key[i]; idx = e;
          }
        }
        wave_argmax(v, idx);
        sum += v;
        nth_low = v - me;       // keys come in descending order; me bounds every eps
        if (idx / EPL == lane) taken |= 1u << (idx % EPL);
      }
#pragma unroll
      for (int i = 0; i < EPL; ++i) {
        const int e = lane * EPL + i;
        if (e < c.E && e / gs == g && K.key[i] + K.eps[i] >= nth_low) need |= 1u << i;
      }
      if (lane == g) { gsum = sum; gerr = me * (FT)c.gn; }
    }
  }
  uint64_t kept = 0;
  FT low = INFINITY;
  for (int r = 0; r < c.Kg; ++r) {
    FT v = gsum; int idx = (lane < c.G && !(kept >> lane & 1)) ? lane : INT_MAX;
    wave_argmax(v, idx);
    kept |= uint64_t(1) << idx;
    const FT lo = read_lane(gsum - gerr, idx & 63);
    low = lo < low ? lo : low;
  }
  FT hi = (lane < c.G && !(kept >> lane & 1)) ? gsum + gerr : -INFINITY;
  hi = wave_max(hi);
  Gp.kept = kept;
  Gp.certain = (c.Kg >= c.G) || (low > hi);
  Gp.need = need;
  // A kept group whose lower bound clears every dropped group's upper bound stays
  // kept whatever the exact keys are (only kept groups can outrank it), and a
  // dropped group whose upper bound is below every kept group's lower bound stays
  // dropped; the cut is open only among the others.
  bool open = false;
  if (lane < c.G) open = (kept >> lane & 1) ? !(gsum - gerr > hi) : !(gsum + gerr < low);
  Gp.open = __ballot(open);
}

// Eligibility bits per slot: valid expert whose group is kept.
template <int EPL, int FORM>
__device__ __forceinline__ uint32_t eligible_mask(const SelCfg& c, uint64_t kept, int lane) {
  uint32_t elig = 0;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const int e = lane * EPL + i;
    if (e < c.E && (!has_groups<FORM>(c) || (kept >> lane_group<EPL, FORM>(c, lane, i) & 1))) elig |= 1u << i;
  }
  return elig;
}

// Top-k among the eligible experts, k successive arg-max reductions; ties go to
// the lowest expert index.
template <typename FT, int EPL>
__device__ __forceinline__ void topk_stage(const SelCfg& c, const Keys<FT, EPL>& K, uint32_t elig,
                                           int lane, Picks<FT>& P) {
  uint32_t taken = 0;
  FT prev_lo = INFINITY, low = INFINITY;
  P.id = -1; P.sc = 0; P.certain = true;
  for (int j = 0; j < c.k; ++j) {
    FT v = 0; int idx = INT_MAX;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      if ((elig >> i & 1) && !(taken >> i & 1) && (idx == INT_MAX || K.key[i] > v)) {
        v = K.key[i]; idx = lane * EPL + i;
      }
    }
    wave_argmax(v, idx);
    const int owner = (idx / EPL) & 63, slot = idx % EPL;
    FT oe = 0, os = 0;
#pragma unroll
    for (int i = 0; i < EPL; ++i)
      if (i == slot) { oe = K.eps[i]; os = K.sc[i]; }
    oe = read_lane(oe, owner);
    os = read_lane(os, owner);
    if (lane == owner) taken |= 1u << slot;
    if (lane == j) { P.id = idx; P.sc = os; }
    if (!(prev_lo > v + oe) && j > 0) P.certain = false;
    prev_lo = v - oe;
    low = prev_lo < low ? prev_lo : low;
  }
  FT hi = -INFINITY;
  bool any = false;
#pragma unroll
  for (int i = 0; i < EPL; ++i)
    if ((elig >> i & 1) && !(taken >> i & 1)) {
      const FT h = K.key[i] + K.eps[i];
      hi = (!any || h > hi) ? h : hi;
      any = true;
    }
  const bool some = __ballot(any) != 0;
  hi = wave_max(any ? hi : (FT)-INFINITY);
  if (some && !(prev_lo > hi)) P.certain = false;
  P.low = low;
}

// Weights of the picked experts; lane j < k returns w[t,j].
template <typename FT, int EPL, int FORM>
__device__ __forceinline__ FT pick_weight(const SelCfg& c, const Keys<FT, EPL>& K,
                                          const Picks<FT>& P, int lane) {
  const bool mine = lane < c.k;
  FT num, den;
  if (is_softmax<FORM>(c)) {
    if (c.renormalize) {
      const FT m = wave_max(mine ? P.sc : (FT)-INFINITY);
      num = mine ? (FT)exp((FT)(P.sc - m)) : (FT)0;
      den = wave_sum(num);
    } else {
      FT m = -INFINITY;
#pragma unroll
      for (int i = 0; i < EPL; ++i)
        if (lane * EPL + i < c.E) m = K.sc[i] > m ? K.sc[i] : m;
      m = wave_max(m);
      FT s = 0;
#pragma unroll
      for (int i = 0; i < EPL; ++i)
        if (lane * EPL + i < c.E) s += (FT)exp((FT)(K.sc[i] - m));
      den = wave_sum(s);
      num = mine ? (FT)exp((FT)(P.sc - m)) : (FT)0;
    }
  } else {
    num = mine ? P.sc : (FT)0;
    den = c.renormalize ? wave_sum(num) : (FT)1;
  }
  return num / den * (FT)c.scale;
}

template <int EPL, int FORM>
__global__ __launch_bounds__(256) void route_select_kernel(
    SelCfg c, int T, const float* __restrict__ logits, const float* __restrict__ logit_bias,
    const float* __restrict__ select_bias, const float* __restrict__ xnorm2,
    const float* __restrict__ wnorm2, int32_t* __restrict__ ids, float* __restrict__ w,
    int32_t* __restrict__ counters, int32_t* __restrict__ recheck,
    float* __restrict__ recheck_low) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  Keys<float, EPL> K;
  const float xn = token_norm(c, xnorm2, t);
  fast_keys<EPL, FORM>(c, logits + size_t(t) * c.E, logit_bias, select_bias, xn, wnorm2, lane, K);
  Groups<float> Gp;
  Gp.kept = 0; Gp.certain = true; Gp.need = 0; Gp.open = 0;
  if (has_groups<FORM>(c)) group_stage<float, EPL, FORM>(c, K, lane, Gp);
  Picks<float> P;
  topk_stage<float, EPL>(c, K, eligible_mask<EPL, FORM>(c, Gp.kept, lane), lane, P);
  if (P.certain && Gp.certain) {
    const float wt = pick_weight<float, EPL, FORM>(c, K, P, lane);
    if (lane < c.k) {
      ids[size_t(t) * c.k + lane] = P.id;
      w[size_t(t) * c.k + lane] = wt;
    }
  } else if (lane == 0) {
    // order of the list is irrelevant: every listed token is re-scored on its own
    const int slot = atomicAdd(&counters[0], 1);
    recheck[slot] = t;
    // with the groups settled, the re-scoring starts from the picks found here
    recheck_low[slot] = Gp.certain ? P.low : __builtin_nanf("");
  }
}

// --------------------------------------------------------- stage 3: re-score
// One workgroup per listed token, or one wavefront when the list is long (its length is
// known here only; the whole grid takes the same side).  Phase 0 (only when the group cut is in doubt): the
// experts that may be among their group's largest get exact keys and the groups
// are chosen in fp64.  Phase 1: with the groups fixed, the experts whose key
// interval reaches the picks get exact keys and the top-k is taken in fp64.
// Experts outside those sets keep their fast keys: by construction they cannot
// change either decision.  The four wavefronts of a shared token run the same selection
// steps on the same data (so their control flow is identical and the barriers are reached
// by all of them) and share out each exact dot product, a quarter of the token row each.  A
// wavefront's candidate list and exact logits live in its own slice of LDS; LDS
// operations of one wavefront execute in order.
// What bounds it is one token's chain: dependent loads, and the fetch of the code, which
// every CU does afresh.  Hence one form of the dot products (two experts at a time: the
// usual list is two picks whose order is in doubt), one copy of each step for both
// phases, and the gate's form fixed at compile time.
template <int EPL, int FORM>
__global__ __launch_bounds__(256, EPL <= 1 ? 3 : 2) void route_recheck_kernel(
    SelCfg c, int H, const void* __restrict__ x, const void* __restrict__ gate_w,
    const float* __restrict__ logits_in, const float* __restrict__ logits,
    const float* __restrict__ logit_bias, const float* __restrict__ select_bias,
    const float* __restrict__ xnorm2, const float* __restrict__ wnorm2, int32_t* __restrict__ ids,
    float* __restrict__ w, const int32_t* __restrict__ counters,
    const int32_t* __restrict__ recheck, const float* __restrict__ recheck_low) {
  constexpr int CB = 2;                          // experts per walk over the token row
  constexpr int U = 4;                           // pieces per thread and row in flight
  __shared__ int xlist_all[4][EPL * 64];
  __shared__ double zx_all[4][EPL * 64];
  __shared__ float2 rint_all[4][EPL * 64];       // key intervals of the listed experts
  __shared__ double part_all[4][CB];             // partial dot products of the wavefronts
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int* const xlist = xlist_all[wave];
  double* const zx = zx_all[wave];
  float2* const rint = rint_all[wave];
  const int n_list = counters[0];
  // a workgroup per token while all of them run at once, two per CU; past that a wavefront per
  // token.  Listed tokens, us with a wavefront / a workgroup each: 128 experts, hidden 2048, 430: 15.3 /
  // 13.8, 256 grouped experts, hidden 7168, 477: 41 / 32, but 128 grouped experts, 680: 21 / 28, 512
  // experts, 520: 26 / 35, 96 experts in six groups, 739: 34 / 50.
  const bool coop = n_list <= 512;
  const int team = coop ? 256 : 64, me = coop ? tid : lane;
  const int n16 = H / 8;                         // pieces of a bf16 row (fp32 rows have exact logits to begin with)

  // exact logits of the experts in xlist[0..n) -> zx[e]
  auto exact_logits = [&](int t, int n) {
    if (logits_in) {
      for (int q = lane; q < n; q += 64) {
        const int e = xlist[q];
        double z = (double)logits_in[size_t(t) * c.E + e];
        if (logit_bias) z += (double)logit_bias[e];
        zx[e] = z;
      }
      return;
    }
    const char* xrow = static_cast<const char*>(x) + size_t(t) * H * 2;
#pragma unroll 1
    for (int q0 = 0; q0 < n; q0 += CB) {
      double acc[CB];
      const char* wrow[CB];
      int ex[CB];
#pragma unroll
      for (int i = 0; i < CB; ++i) {
        acc[i] = 0.0;
        ex[i] = xlist[q0 + i < n ? q0 + i : n - 1];
        wrow[i] = static_cast<const char*>(gate_w) + size_t(ex[i]) * H * 2;
      }
#pragma unroll 1
      for (int p0 = me; p0 < n16; p0 += team * U) {
        uint4 a[U], b[CB][U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int p = min(p0 + u * team, n16 - 1);
          a[u] = *reinterpret_cast<const uint4*>(xrow + size_t(p) * 16);
#pragma unroll
          for (int i = 0; i < CB; ++i) b[i][u] = *reinterpret_cast<const uint4*>(wrow[i] + size_t(p) * 16);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (p0 + u * team < n16) {
#pragma unroll
            for (int i = 0; i < CB; ++i) acc[i] = piece_dot64<true>(a[u], b[i][u], acc[i]);
          }
      }
      double z[CB];
#pragma unroll
      for (int i = 0; i < CB; ++i) z[i] = wave_sum(acc[i]);
      if (coop) {
        // the four partial sums of each expert, added in wavefront order by everyone
#pragma unroll
        for (int i = 0; i < CB; ++i)
          if (lane == 0) part_all[wave][i] = z[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < CB; ++i) z[i] = ((part_all[0][i] + part_all[1][i]) + part_all[2][i]) + part_all[3][i];
        __syncthreads();                  // before the next batch overwrites the partial sums
      }
#pragma unroll
      for (int i = 0; i < CB; ++i)
        if (q0 + i < n && lane == 0) {
          if (logit_bias) z[i] += (double)logit_bias[ex[i]];
          zx[ex[i]] = z[i];
        }
    }
  };
  // list the experts flagged in `want`; returns how many
  auto make_list = [&](uint32_t want) {
    int n = 0;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const bool in = want >> i & 1;
      const uint64_t m = __ballot(in);
      if (in) xlist[n + __popcll(m & ((uint64_t(1) << lane) - 1))] = lane * EPL + i;
      n += __popcll(m);
    }
    return n;
  };

  for (int li = coop ? blockIdx.x : blockIdx.x * 4 + wave; li < n_list; li += coop ? gridDim.x : gridDim.x * 4) {
    const int t = recheck[li];
    Keys<float, EPL> K;
    Keys<double, EPL> D;
    Groups<float> Gf;
    Gf.kept = 0; Gf.certain = true; Gf.need = 0; Gf.open = 0;
    const float xn = token_norm(c, xnorm2, t);
    fast_keys<EPL, FORM>(c, logits + size_t(t) * c.E, logit_bias, select_bias, xn, wnorm2, lane, K);
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      D.key[i] = (double)K.key[i]; D.sc[i] = (double)K.sc[i]; D.eps[i] = 0.0;
    }
    if (has_groups<FORM>(c)) group_stage<float, EPL, FORM>(c, K, lane, Gf);
    uint64_t kept = Gf.kept;
    uint32_t exact = 0;          // slots of this lane that hold exact keys
#pragma unroll 1
    for (int phase = has_groups<FORM>(c) && !Gf.certain ? 0 : 1; phase < 2; ++phase) {
      uint32_t want = 0;
      if (has_groups<FORM>(c) && phase == 0) {
        // settle the groups in fp64: exact keys only where they can matter, the possible
        // largest members of the groups on whose scores the cut still depends.  The
        // other groups keep their fast scores, which the intervals already order
        // against every open group.
#pragma unroll
        for (int i = 0; i < EPL; ++i)
          if ((Gf.need >> i & 1) && (Gf.open >> lane_group<EPL, FORM>(c, lane, i) & 1)) want |= 1u << i;
      } else {
        // candidates of the top-k.  The smallest lower bound of the fast picks comes
        // from the selection pass unless the groups had to be settled here.
        const uint32_t elig = eligible_mask<EPL, FORM>(c, kept, lane);
        Picks<float> P;
        P.low = recheck_low[li];
        if (has_groups<FORM>(c) && !(P.low == P.low)) topk_stage<float, EPL>(c, K, elig, lane, P);
        // Only experts whose upper bound reaches the smallest lower bound of a pick can
        // be among the picks.  Of those, an expert whose interval is apart from every
        // other's is ordered against all of them by its fast key already; the ones whose
        // intervals meet another's get exact keys.
        uint32_t region = 0;
        float lo[EPL], hi[EPL];
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
          lo[i] = K.key[i] - K.eps[i];
          hi[i] = K.key[i] + K.eps[i];
          if ((elig >> i & 1) && hi[i] >= P.low) region |= 1u << i;
        }
        int nr = 0;
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
          const bool in = region >> i & 1;
          const uint64_t m = __ballot(in);
          if (in) {
            const int pos = nr + __popcll(m & ((uint64_t(1) << lane) - 1));
            xlist[pos] = lane * EPL + i;
            rint[pos] = make_float2(lo[i], hi[i]);
          }
          nr += __popcll(m);
        }
#pragma unroll 1
        for (int q = 0; q < nr; ++q) {
          const int m = xlist[q];
          const float2 iv = rint[q];
#pragma unroll
          for (int i = 0; i < EPL; ++i)
            if ((region >> i & 1) && lane * EPL + i != m && lo[i] <= iv.y && iv.x <= hi[i]) want |= 1u << i;
        }
        want &= ~exact;
      }
      const int n = make_list(want);
      exact_logits(t, n);
#pragma unroll
      for (int i = 0; i < EPL; ++i) {       // pull the exact logits into D
        if (!(want >> i & 1)) continue;
        const int e = lane * EPL + i;
        const double z = zx[e];
        if (is_softmax<FORM>(c)) {
          D.key[i] = z; D.sc[i] = z;
        } else {
          const double sg = 1.0 / (1.0 + exp(-z));
          D.sc[i] = sg;
          D.key[i] = sg + (select_bias ? (double)select_bias[e] : 0.0);
        }
      }
      exact |= want;
      if (has_groups<FORM>(c) && phase == 0) {
        Groups<double> Gd;
        group_stage<double, EPL, FORM>(c, D, lane, Gd);
        kept = Gd.kept;
      }
    }
    Picks<double> Q;
    topk_stage<double, EPL>(c, D, eligible_mask<EPL, FORM>(c, kept, lane), lane, Q);
    const double wt = pick_weight<double, EPL, FORM>(c, D, Q, lane);
    if (lane < c.k && (!coop || wave == 0)) {
      ids[size_t(t) * c.k + lane] = Q.id;
      w[size_t(t) * c.k + lane] = (float)wt;
    }
  }
}

// ------------- few tokens, small gate: gate, scores and top-k of a token in one pass
// One workgroup of sixteen wavefronts per token.  The wavefronts share out the experts and
// compute every logit exactly (fp64 sums of exact products, CB experts per walk
// over the token row); the first wavefront then builds fp64 keys for all experts
// and takes the group limit, the top-k and the weights in fp64.  One launch less than
// the forms below, which is what counts while there is at most one workgroup per CU and a
// wavefront walks few gate rows (the rule and what it measured: exact_form).
template <int EPL, int FORM, bool BF16>
__global__ __launch_bounds__(1024) void route_exact_kernel(
    SelCfg c, int H, const void* __restrict__ x, const void* __restrict__ gate_w,
    const float* __restrict__ logit_bias, const float* __restrict__ select_bias,
    int32_t* __restrict__ ids, float* __restrict__ w, int32_t* __restrict__ counters) {
  __shared__ double zx[EPL * 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t = blockIdx.x;
  if (t == 0 && threadIdx.x < 64) counters[threadIdx.x] = 0;   // nothing is re-scored
  const size_t row_bytes = size_t(H) * (BF16 ? 2 : 4);
  const char* xrow = static_cast<const char*>(x) + size_t(t) * row_bytes;
  const int n16 = int(row_bytes / 16);
  const int per = (c.E + 15) / 16;
  const int e_begin = min(c.E, wave * per), e_end = min(c.E, e_begin + per);
  constexpr int CB = 4, U = 4;   // experts per walk, pieces per lane and row in flight (8: spills)
  for (int e0 = e_begin; e0 < e_end; e0 += CB) {
    double acc[CB];
    const char* wrow[CB];
#pragma unroll
    for (int i = 0; i < CB; ++i) {
      acc[i] = 0.0;
      wrow[i] = static_cast<const char*>(gate_w) + size_t(min(e0 + i, e_end - 1)) * row_bytes;
    }
    for (int p0 = 0; p0 < n16; p0 += 64 * U) {
      uint4 a[U], b[CB][U];
      bool in[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        int p = p0 + u * 64 + lane;
        in[u] = p < n16;
        p = in[u] ? p : n16 - 1;
        a[u] = *reinterpret_cast<const uint4*>(xrow + size_t(p) * 16);
#pragma unroll
        for (int i = 0; i < CB; ++i) b[i][u] = *reinterpret_cast<const uint4*>(wrow[i] + size_t(p) * 16);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < CB; ++i) {
          const double d = piece_dot64<BF16>(a[u], b[i][u], 0.0);
          acc[i] += in[u] ? d : 0.0;
        }
    }
#pragma unroll
    for (int i = 0; i < CB; ++i) {
      double z = wave_sum(acc[i]);
      if (e0 + i < e_end && lane == 0) {
        if (logit_bias) z += (double)logit_bias[e0 + i];
        zx[e0 + i] = z;
      }
    }
  }
  __syncthreads();
  if (wave != 0) return;
  Keys<double, EPL> D;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const int e = lane * EPL + i;
    D.key[i] = -INFINITY; D.sc[i] = 0.0; D.eps[i] = 0.0;
    if (e < c.E) {
      const double z = zx[e];
      if (is_softmax<FORM>(c)) {
        D.key[i] = z; D.sc[i] = z;
      } else {
        const double sg = 1.0 / (1.0 + exp(-z));
        D.sc[i] = sg;
        D.key[i] = sg + (select_bias ? (double)select_bias[e] : 0.0);
      }
    }
  }
  uint64_t kept = 0;
  if (has_groups<FORM>(c)) {
    Groups<double> Gd;
    group_stage<double, EPL, FORM>(c, D, lane, Gd);
    kept = Gd.kept;
  }
  const uint32_t elig = eligible_mask<EPL, FORM>(c, kept, lane);
  Picks<double> Q;
  topk_stage<double, EPL>(c, D, elig, lane, Q);
  const double wt = pick_weight<double, EPL, FORM>(c, D, Q, lane);
  if (lane < c.k) {
    ids[size_t(t) * c.k + lane] = Q.id;
    w[size_t(t) * c.k + lane] = (float)wt;
  }
}

// ------------- few tokens, long gate rows: exact logits on the vector unit, then selection
// A workgroup of four wavefronts takes sixteen experts of one token (a wavefront: four gate
// rows, eight 16-byte pieces per lane and row in flight), so a token is shared out over
// E/16 workgroups and no wavefront walks more than four rows.  The 16 x 16 tile of the matrix
// form below does sixteen tokens' work for one, on one CU.
template <bool BF16>
__global__ __launch_bounds__(256) void gate_exact_rows_kernel(
    int H, int E, const void* __restrict__ x, const void* __restrict__ gate_w,
    const float* __restrict__ logit_bias, double* __restrict__ zx, int32_t* __restrict__ counters) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t = blockIdx.y;
  if (blockIdx.x == 0 && t == 0 && threadIdx.x < 64) counters[threadIdx.x] = 0;   // nothing is re-scored
  constexpr int CB = 4, U = 8;
  const int e0 = (blockIdx.x * 4 + wave) * CB;
  if (e0 >= E) return;
  const size_t row_bytes = size_t(H) * (BF16 ? 2 : 4);
  const char* xrow = static_cast<const char*>(x) + size_t(t) * row_bytes;
  const int n16 = int(row_bytes / 16);
  double acc[CB];
  const char* wrow[CB];
#pragma unroll
  for (int i = 0; i < CB; ++i) {
    acc[i] = 0.0;
    wrow[i] = static_cast<const char*>(gate_w) + size_t(min(e0 + i, E - 1)) * row_bytes;
  }
  for (int p0 = 0; p0 < n16; p0 += 64 * U) {
    uint4 a[U], b[CB][U];
    bool in[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int p = p0 + u * 64 + lane;
      in[u] = p < n16;
      p = in[u] ? p : n16 - 1;
      a[u] = *reinterpret_cast<const uint4*>(xrow + size_t(p) * 16);
#pragma unroll
      for (int i = 0; i < CB; ++i) b[i][u] = *reinterpret_cast<const uint4*>(wrow[i] + size_t(p) * 16);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < CB; ++i) {
        const double d = piece_dot64<BF16>(a[u], b[i][u], 0.0);
        acc[i] += in[u] ? d : 0.0;
      }
  }
#pragma unroll
  for (int i = 0; i < CB; ++i) {
    double z = wave_sum(acc[i]);
    if (e0 + i < E && lane == 0) {
      if (logit_bias) z += (double)logit_bias[e0 + i];
      zx[size_t(t) * E + e0 + i] = z;
    }
  }
}

// ------------- exact logits on fp64 matrix instructions, then selection
// A workgroup of sixteen wavefronts computes 16 tokens x 16 experts with
// v_mfma_f64_16x16x4_f64 (exact products, fp64 sums): the wavefronts share out K and
// their sums are added in a fixed order.  Per instruction (1024 multiply-adds) a lane
// widens one element of each operand, where the dot products of one token on the
// vector unit widen an element per multiply-add.  K runs in the order that makes a
// lane's load one 16-byte piece of its row, the same for both operands: piece 4g + q of
// the row for lanes 16q..16q+15, group g of four pieces going to wavefront g % 16.  The
// fp64 logits go to the workspace; a second kernel, one wavefront per token, selects.
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <bool BF16>
__global__ __launch_bounds__(1024) void gate_exact_kernel(
    int T, int H, int E, const void* __restrict__ x, const void* __restrict__ gate_w,
    const float* __restrict__ logit_bias, double* __restrict__ zx, int32_t* __restrict__ counters, int grid_row) {
  __shared__ double red[16][256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int block = grid_block(grid_row);
  if (block == 0 && tid < 64) counters[tid] = 0;        // nothing is re-scored
  const int n_etiles = (E + 15) / 16;
  const int ttile = block / n_etiles, e0 = (block - ttile * n_etiles) * 16, t0 = ttile * 16;
  if (t0 >= T) return;                                  // the whole workgroup
  const size_t row_bytes = size_t(H) * (BF16 ? 2 : 4);
  const int n16 = int(row_bytes / 16), groups = (n16 + 3) / 4;
  const char* const xrow = static_cast<const char*>(x) + size_t(min(t0 + (lane & 15), T - 1)) * row_bytes;
  const char* const wrow = static_cast<const char*>(gate_w) + size_t(min(e0 + (lane & 15), E - 1)) * row_bytes;
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  constexpr int U = 4;                       // groups in flight
  for (int g0 = wave; g0 < groups; g0 += 16 * U) {
    uint4 a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = (g0 + 16 * u) * 4 + (lane >> 4);
      a[u] = b[u] = make_uint4(0, 0, 0, 0);
      if (p < n16) {
        a[u] = *reinterpret_cast<const uint4*>(xrow + size_t(p) * 16);
        b[u] = *reinterpret_cast<const uint4*>(wrow + size_t(p) * 16);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (g0 + 16 * u >= groups) break;      // the same in every lane
      const uint32_t av[4] = {a[u].x, a[u].y, a[u].z, a[u].w}, bv[4] = {b[u].x, b[u].y, b[u].z, b[u].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (BF16) {
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)bf16_bits_to_f32(av[i] & 0xffffu),
                                                     (double)bf16_bits_to_f32(bv[i] & 0xffffu), acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)bf16_bits_to_f32(av[i] >> 16),
                                                     (double)bf16_bits_to_f32(bv[i] >> 16), acc, 0, 0, 0);
        } else {
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)__uint_as_float(av[i]),
                                                     (double)__uint_as_float(bv[i]), acc, 0, 0, 0);
        }
      }
    }
  }
  // D layout: lane l, element i -> token 4i + l/16, expert l%16
#pragma unroll
  for (int i = 0; i < 4; ++i) red[wave][(i * 4 + (lane >> 4)) * 16 + (lane & 15)] = acc[i];
  __syncthreads();
  const int t = t0 + (tid >> 4), e = e0 + (tid & 15);
  if (tid < 256 && t < T && e < E) {
    double z = red[0][tid];
#pragma unroll
    for (int w = 1; w < 16; ++w) z += red[w][tid];
    if (logit_bias) z += (double)logit_bias[e];
    zx[size_t(t) * E + e] = z;
  }
}

template <int EPL, int FORM>
__global__ __launch_bounds__(256) void select_exact_kernel(
    SelCfg c, int T, const double* __restrict__ zx, const float* __restrict__ select_bias,
    int32_t* __restrict__ ids, float* __restrict__ w) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  Keys<double, EPL> D;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const int e = lane * EPL + i;
    D.key[i] = -INFINITY; D.sc[i] = 0.0; D.eps[i] = 0.0;
    if (e < c.E) {
      const double z = zx[size_t(t) * c.E + e];
      if (is_softmax<FORM>(c)) {
        D.key[i] = z; D.sc[i] = z;
      } else {
        const double sg = 1.0 / (1.0 + exp(-z));
        D.sc[i] = sg;
        D.key[i] = sg + (select_bias ? (double)select_bias[e] : 0.0);
      }
    }
  }
  uint64_t kept = 0;
  if (has_groups<FORM>(c)) {
    Groups<double> Gd;
    group_stage<double, EPL, FORM>(c, D, lane, Gd);
    kept = Gd.kept;
  }
  const uint32_t elig = eligible_mask<EPL, FORM>(c, kept, lane);
  Picks<double> Q;
  topk_stage<double, EPL>(c, D, elig, lane, Q);
  const double wt = pick_weight<double, EPL, FORM>(c, D, Q, lane);
  if (lane < c.k) {
    ids[size_t(t) * c.k + lane] = Q.id;
    w[size_t(t) * c.k + lane] = (float)wt;
  }
}

// Which kernels compute exact logits.
enum ExactForm { kExactOneLaunch, kExactRows, kExactTiles };
// 16 x 16 tiles of the exact gate: workgroups of gate_exact_kernel
inline long exact_tiles(int T, int E) { return long((T + 15) / 16) * ((E + 15) / 16); }

// The form whose gate takes the least, from estimates in us that follow 1296 measured sizes (1 to
// 4096 tokens, 4 to 512 experts, hidden 256 to 7168, both types; the picked form is within 1 % of
// the best one in the mean, 16 % at worst).  Against the second launch that they save or pay:
//   one launch  a round of 256 pieces per wavefront that has experts, on a CU per token
//   rows        a round of 512 pieces per wavefront; past one workgroup per CU the workgroups'
//               starts and their wavefronts' rounds add up
//   tiles       one CU's fp64 matrix rate over the row, 256 tiles at a time
// e.g. bf16, one launch / rows / tiles: 8 experts, hidden 2048, 64 tokens 6.9 / 8.9 / 11.5; 128 experts,
// hidden 7168, 16 tokens 39 / 15 / 27; 64 experts, hidden 1024, 256 tokens 10.7 / 18.8 / 9.7.
ExactForm exact_form(bool bf16, int T, int E, int H) {
  const int pieces = H / (bf16 ? 8 : 4), per = (E + 15) / 16;
  const float wgs = float(T) * per / 256, tiles = exact_tiles(T, E) / 256.f;
  const int r256 = (pieces + 255) / 256, r512 = (pieces + 511) / 512;
  const float waves = float((E + 3) / 4) / (4 * per);      // of the rows form's workgroups, with experts
  const float one = (bf16 ? -1.f : -1.7f) + (bf16 ? .29f : .165f) * ((E + per - 1) / per) * r256;
  const float rows_one = bf16 ? 3.1f + (pieces > 256 ? .3f : 0.f) + 3.3f * (r512 - 1) : 1.f + 1.65f * (r512 - 1);
  const float rows_all = wgs * (bf16 ? .6f + 2.5f * waves * r512 : .3f + 1.6f * waves * r512);
  const float rows = rows_one > rows_all ? rows_one : rows_all;
  const float tile = (bf16 ? 2.75e-3f * H + .2f : 3.6e-3f * H + .4f) * (tiles > 1 ? tiles : 1.f);
  if (T <= 256 && E <= 64 && one <= rows && one <= tile) return kExactOneLaunch;
  return T <= 65535 && rows <= tile ? kExactRows : kExactTiles;      // rows: tokens along the grid's y
}

template <int EPL, int FORM, bool BF16>
void launch_route_exact(ExactForm form, const SelCfg& sc, const moe_config& c, int T, const void* x,
                        const void* gate_w, const float* logit_bias, const float* select_bias,
                        int32_t* ids, float* w, const RouteWs& ws, hipStream_t s) {
  const int E = c.n_experts;
  if constexpr (EPL == 1) {
    if (form == kExactOneLaunch) {
      // (bf16: the general instance; the soft-max one spills at sixteen wavefronts, 7.4 against 6.5 us)
      MOE_LAUNCH(MOE_K_GATE_GEMM, (route_exact_kernel<1, BF16 ? int(kGateAny) : FORM, BF16>), dim3(T), dim3(1024), 0,
                 s, sc, c.hidden, x, gate_w, logit_bias, select_bias, ids, w, ws.counters);
      return;
    }
  }
  // the logits area holds at least two floats per (token, expert): room for one double
  double* zx = reinterpret_cast<double*>(ws.logits);
  if (form == kExactRows) {
    MOE_LAUNCH(MOE_K_GATE_GEMM, gate_exact_rows_kernel<BF16>, dim3((E + 15) / 16, T), dim3(256), 0, s, c.hidden,
               E, x, gate_w, logit_bias, zx, ws.counters);
  } else {
    const dim3 grid = grid_of(size_t(exact_tiles(T, E)), 1024);
    MOE_LAUNCH(MOE_K_GATE_GEMM, gate_exact_kernel<BF16>, grid, dim3(1024), 0, s, T, c.hidden, E, x, gate_w,
               logit_bias, zx, ws.counters, int(grid.x));
  }
  MOE_LAUNCH(MOE_K_SELECT, (select_exact_kernel<EPL, FORM>), dim3((T + 3) / 4), dim3(256), 0, s, sc, T, zx,
             select_bias, ids, w);
}

template <int EPL, int FORM, typename... A>
void launch_route_exact_of(bool bf16, A&&... a) {
  if (bf16) launch_route_exact<EPL, FORM, true>(a...);
  else launch_route_exact<EPL, FORM, false>(a...);
}

template <int EPL, int FORM>
void launch_select_and_recheck(const SelCfg& sc, const moe_config& c, int T, const void* x,
                               const void* gate_w, const float* logit_bias,
                               const float* select_bias, const float* logits_in,
                               const float* logits, int32_t* ids, float* w, const RouteWs& ws,
                               hipStream_t s) {
  MOE_LAUNCH(MOE_K_SELECT, (route_select_kernel<EPL, FORM>), dim3((T + 3) / 4), dim3(256), 0, s, sc, T, logits,
             logit_bias, select_bias, ws.xnorm2, ws.wnorm2, ids, w, ws.counters, ws.recheck,
             ws.recheck_low);
  const int grid = T < 1024 ? T : 1024;
  MOE_LAUNCH(MOE_K_RESCORE, (route_recheck_kernel<EPL, FORM>), dim3(grid), dim3(256), 0, s, sc, c.hidden, x,
             gate_w, logits_in, logits, logit_bias, select_bias, ws.xnorm2, ws.wnorm2, ids, w, ws.counters,
             ws.recheck, ws.recheck_low);
}

}  // namespace

hipError_t launch_route(const moe_config& c, int T, const void* x, const void* gate_w,
                        const float* logit_bias, const float* select_bias,
                        const float* logits_in, int32_t* ids, float* w, const RouteWs& ws,
                        hipStream_t s) {
  const int E = c.n_experts, H = c.hidden;
  const bool bf16 = c.act_dtype == MOE_BF16;
  const float* logits = logits_in;
  SelCfg sc;
  sc.E = E; sc.k = c.top_k; sc.score_fn = c.score_fn; sc.renormalize = c.renormalize;
  sc.G = c.n_groups; sc.Kg = c.topk_groups; sc.gn = c.group_score_n; sc.scale = c.routed_scale;
  sc.chain_err = 0.f; sc.have_norms = 0; sc.nsplit = 1; sc.T = T;
  const int epl = (E + 63) / 64;
  // The exact gate against the bf16 pipeline of three launches, from what they take in whole
  // rounds of 256 tiles.  bf16, exact / pipeline in us: 128 experts, hidden 2048, 1024 tokens 21 / 26, 1536
  // tokens 29 / 27; hidden 4096, 512 tokens 21 / 30, 768 tokens 34 / 33; hidden 512, 4096 tokens 29 / 24 (the
  // selection on fp64 keys costs more per token: hence the limit on tiles).  A gate with groups
  // has the longer selection and re-scoring: 256 experts, hidden 7168, 288 and 400 tokens 53 / 54, 576
  // tokens (three rounds) 75 / 55; 128 experts, hidden 4096, 2048 tokens 60 / 39; 64 experts, hidden 2048, 4096
  // tokens 37 / 31.  fp32 rows have no other gate.
  const long tiles = exact_tiles(T, E), rounds = (tiles + 255) / 256;
  const bool few = tiles <= 1024 && (c.n_groups > 1 ? rounds * 256 * H < (E > 128 ? 1L << 22 : 1L << 21)
                                                    : tiles * H <= 1L << 20);
  // Up to 4096 tokens bf16 batches of T*E*H <= 5 * 2^25 (2^28 where a token's gate is long,
  // E*H > 2^19) have exact logits whatever that costs: their weights are fp64 arithmetic
  // rounded once, where the pipeline's are fp32 exponentials of fp32 logits.  This adds to the
  // tiles short rows (128 experts, hidden 512, 2304 tokens) and the batches that only rounding
  // up to whole tiles takes past the limit (33 tokens, 512 experts, hidden 14336).
  const size_t teh = size_t(T) * E * H;
  const bool fp64_band = T <= 4096 && (teh <= size_t(5) << 25 ||
                                       (size_t(E) * H > size_t(1) << 19 && teh <= size_t(1) << 28));
  const bool exact = !bf16 || fp64_band || few;
  // experts per lane and form of the gate -> one instance of the selection kernels
#define MOE_BY_FORM(F, EPL, ...)                                                      \
  switch (gate_form<EPL>(sc)) {                                                            \
    case kGateSoftmax: F<EPL, kGateSoftmax>(__VA_ARGS__); break;                      \
    case kGateGrouped: F<EPL, kGateGrouped>(__VA_ARGS__); break;                      \
    default: F<EPL, kGateAny>(__VA_ARGS__); break;                                    \
  }
#define MOE_BY_GATE(F, ...)                                                           \
  do {                                                                                \
    if (epl <= 1) { MOE_BY_FORM(F, 1, __VA_ARGS__) }                                  \
    else if (epl <= 2) { MOE_BY_FORM(F, 2, __VA_ARGS__) }                             \
    else if (epl <= 4) { MOE_BY_FORM(F, 4, __VA_ARGS__) }                             \
    else { MOE_BY_FORM(F, 8, __VA_ARGS__) }                                           \
  } while (0)
  if (!logits_in && exact) {
    const ExactForm form = exact_form(bf16, T, E, H);
    MOE_BY_GATE(launch_route_exact_of, bf16, form, sc, c, T, x, gate_w, logit_bias, select_bias, ids, w, ws, s);
    return hipGetLastError();
  }
  if (logits_in) {
    MOE_LAUNCH(MOE_K_GATE_NORMS, clear_counters_kernel, dim3(1), dim3(kRouteCounterBytes / 4), 0, s, ws.counters);
  } else {
    // the bf16 gate GEMM sums the gate rows' squares and clears the counter itself
    logits = ws.logits;
    sc.have_norms = 1;
    // few tiles: split K so that about two workgroups per CU run (one workgroup is
    // one wavefront per SIMD, which hides no latency); each split keeps at least 8
    // K steps
    const int blocks = ((T + GBM - 1) / GBM) * ((E + GBN - 1) / GBN);
    const int ksteps = (H + GBK - 1) / GBK;
    int nsplit = 1;
    const int cap = gate_split_cap(T, E);
    while (nsplit < cap && blocks * nsplit * 2 <= kGateWgTarget && ksteps / (nsplit * 2) >= 8) nsplit *= 2;
    const dim3 grid((T + GBM - 1) / GBM, (E + GBN - 1) / GBN, nsplit);
    if (H % GBK == 0) {
      // two stages (48 KB): three workgroups share a CU, which measured faster than
      // deeper rings with fewer workgroups, and than 128-token tiles
      constexpr int NS = 2;
      constexpr int lds = NS * (GBM + GBN) * 8 * 16;
      MOE_LAUNCH(MOE_K_GATE_GEMM, (gate_dma_kernel<GBM, NS, kGateChainSteps>), grid, dim3(512), lds, s,
                 static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(gate_w), T, H, E,
                 ws.logits, ws.xnorm2, ws.wnorm2, ws.counters);
    } else {
      MOE_LAUNCH(MOE_K_GATE_GEMM, gate_mfma_kernel<kGateChainSteps>, grid, dim3(512), 0, s,
                 static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(gate_w), T, H, E,
                 ws.logits, ws.xnorm2, ws.wnorm2, ws.counters);
    }
    sc.nsplit = nsplit;
    // chains of kGateChainSteps*64 products; +2 for the flush and the store.  The
    // partial dot products of the splits obey sum_s |x_s||w_s| <= |x||w|, so the
    // chain term is unchanged; summing the slabs in fp32 adds one ulp of that
    // product per addition and per slab store
    sc.chain_err = (2.f * kGateChainSteps * GBK + 2.f + 2.f * (nsplit - 1)) * kUlp;
  }
  MOE_BY_GATE(launch_select_and_recheck, sc, c, T, x, gate_w, logit_bias, select_bias, logits_in, logits, ids,
              w, ws, s);
#undef MOE_BY_GATE
#undef MOE_BY_FORM
  return hipGetLastError();
}

}  // namespace moe

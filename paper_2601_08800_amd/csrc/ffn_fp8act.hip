// Expert FFN with 8-bit activations: both GEMM operands are e4m3, the matrix
// cores run `v_mfma_f32_32x32x64_f8f6f4` (twice the rate of the bf16 MFMA).
//
//   quant   one wavefront per row, 16 lanes per block of 128 columns: amax -> scale =
//           amax / 448 (1 for an all-zero block), code = e4m3(x / scale) after a
//           clamp to +-448; codes [rows, K], scales [K/128][rows] (block-major, so
//           that a tile's scales of one K block are contiguous)
//   GEMM    C[rows, N] = sum over K blocks kb of sA[row, kb] * sB[n/128, kb] *
//           (Aq[rows, kb] . Bq[N, kb]^T): the products of a K block are summed by
//           the MFMA into a fresh fp32 accumulator and promoted into the running
//           sum with the two scales (fp32 FMA), block by block
// GEMM-1 applies SwiGLU and quantises the intermediate by the same rule: its tile spans the
// 128 columns of one block.
//
// GEMM tile: up to 192 rows x 256 weight rows (DUAL: 128 gate + the matching 128 up rows), K
// step 128 bytes = one scale block, eight wavefronts as 2 (row halves) x 4 (64 weight rows).
// An expert's rows are cut into tiles of equal height, in 32-row blocks (NB of them, a template
// argument).  Operands go global -> LDS by DMA into rings of their own (Ring8), rows of 128
// bytes with the piece index XOR-ed by (row/2)&7.  Inside a K step, MFMA sub-step s of lane
// half h takes bytes (2s+h)*32 .. +32 of the row for BOTH operands, so the pairing of A and B
// elements is right whatever order the instruction walks K in.  The weights are the first
// operand: a lane then holds columns of one activation row, so that a 32 x 32 block's sums
// have one scale per lane (one product and sixteen FMAs a block; with the rows in the
// registers it was sixteen products more, as much time as the MFMAs take).
//
// What bounds it: the matrix unit would need 0.75 us for a K step of 192 rows at the clock that
// it sustains; the step takes 1.5 us, because the LDS reads and the load instructions of a
// step (memory phase) take longer than its MFMAs and the two row halves take turns.  Against
// 128 x 128 tiles of four wavefronts, two workgroups per CU, all loads of a step waited for at
// once, and passes of their own for the intermediate's quantisation (one stream, us): 6007
// tokens of 7168, 32 of 256 experts, I 1024: routed GEMM-1 / -2 163 / 89 -> 161 / 82, one
// expert of 6007 rows 133 / 73 -> 92 / 67, quantisation 16 -> 0; whole layer 673 -> 605; 24 576
// tokens 2078 -> 1793, I 2048 3483 -> 2834; 256 tokens 233 -> 207.
// Also measured (one expert of 6144 rows, GEMM-1 97, with the weight block scales not yet in lanes): both halves in one phase with the next
// fragments read under the last block's MFMAs 103, the same with loads spread over the row
// blocks 111; 16 x 16 x 128 instructions 98-105; reads in front of the loads 101.

#include "device_util.h"
#include "moe_internal.h"

namespace moe {

namespace {

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kQBlock = 128;     // columns per activation scale, and K bytes per GEMM step
constexpr int kTileRec = 4;      // tile record: expert, first row, end row, the expert's first tile
constexpr int FBM = 192;          // rows of a tile at most

__device__ __forceinline__ int swz(int row, int piece) {
  return row * 8 + (piece ^ ((row >> 1) & 7));
}

// ------------------------------------------------------------------ quant
// x bf16 [rows, K] -> codes [rows, K], scales_t [K/128][rows_capacity].  One
// wavefront per row walks it in chunks of 512 columns: a lane owns 8
// neighbouring columns (one 16-byte load), 16 lanes share a block of 128.  Two
// chunks are in flight per trip.
__device__ __forceinline__ void quant_piece(const uint4 v, uint2& out, float& scale) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  float f[8];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = __uint_as_float(w[i] << 16);
    f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
  float amax = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf(f[i]));
#pragma unroll
  for (int s = 1; s < 16; s <<= 1) amax = fmaxf(amax, __shfl_xor(amax, s));
  scale = amax > 0.f ? amax / 448.0f : 1.0f;
#pragma unroll
  for (int i = 0; i < 8; ++i) f[i] = fminf(fmaxf(f[i] / scale, -448.0f), 448.0f);
  int lo = __builtin_amdgcn_cvt_pk_fp8_f32(f[0], f[1], 0, false);      // round to nearest even
  lo = __builtin_amdgcn_cvt_pk_fp8_f32(f[2], f[3], lo, true);
  int hi = __builtin_amdgcn_cvt_pk_fp8_f32(f[4], f[5], 0, false);
  hi = __builtin_amdgcn_cvt_pk_fp8_f32(f[6], f[7], hi, true);
  out = make_uint2((uint32_t)lo, (uint32_t)hi);
}

__global__ __launch_bounds__(256) void fp8act_quant_kernel(const uint16_t* __restrict__ x,
                                                          const int32_t* __restrict__ offsets,
                                                          int n_experts, int K, int rows_capacity,
                                                          uint8_t* __restrict__ codes,
                                                          float* __restrict__ scales_t) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  int rows = offsets ? offsets[n_experts] : rows_capacity;     // no offsets: every row
  rows = rows < rows_capacity ? rows : rows_capacity;
  if (row >= rows) return;
  const uint4* xr = reinterpret_cast<const uint4*>(x + size_t(row) * K);     // 8 columns per piece
  uint2* cr = reinterpret_cast<uint2*>(codes + size_t(row) * K);
  const int pieces = K / 8;                       // a multiple of 16
  const int g = lane >> 4, sub = lane & 15;
  for (int p0 = 0; p0 < pieces; p0 += 128) {      // the loop bounds are the same in every lane
    const int pa = p0 + lane, pb = p0 + 64 + lane;
    const bool ina = pa < pieces, inb = pb < pieces;
    const uint4 zero = make_uint4(0, 0, 0, 0);
    const uint4 va = ina ? xr[pa] : zero, vb = inb ? xr[pb] : zero;
    uint2 ca, cb;
    float sa, sb;
    quant_piece(va, ca, sa);
    quant_piece(vb, cb, sb);
    if (ina) {
      cr[pa] = ca;
      if (sub == 0) scales_t[size_t(p0 / 16 + g) * rows_capacity + row] = sa;
    }
    if (inb) {
      cr[pb] = cb;
      if (sub == 0) scales_t[size_t(p0 / 16 + 4 + g) * rows_capacity + row] = sb;
    }
  }
}

// ------------------------------------------------------------- tile table
// tiles[0] = number of M tiles, then (expert, first row, end row, the expert's first tile) per
// tile.  An expert's rows are cut into ceil(M / FBM) tiles of equal height (rounded up to 32
// rows).  One thread per expert; one wavefront scans the tile counts.
struct ExpertTiles { int lo, hi, step, count; };
__device__ __forceinline__ ExpertTiles tiles_of(const int32_t* __restrict__ offsets, int e, int rows_capacity) {
  ExpertTiles t;
  t.lo = min(max(offsets[e], 0), rows_capacity);
  t.hi = min(max(offsets[e + 1], t.lo), rows_capacity);
  const int m = t.hi - t.lo, full = (m + FBM - 1) / FBM;
  t.step = full ? ((m + full - 1) / full + 31) / 32 * 32 : FBM;
  t.count = (m + t.step - 1) / t.step;
  return t;
}

__global__ __launch_bounds__(512) void fp8act_tiles_kernel(const int32_t* __restrict__ offsets,
                                                          int n_experts, int rows_capacity,
                                                          int32_t* __restrict__ tiles, int max_tiles) {
  __shared__ int32_t start[512];
  const int e = threadIdx.x;
  ExpertTiles mine{0, 0, FBM, 0};
  if (e < n_experts) mine = tiles_of(offsets, e, rows_capacity);
  start[e] = mine.count;                        // experts past n_experts: no tiles
  __syncthreads();
  if (e < 64) {
    int n[8], sum = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) sum += n[i] = start[e * 8 + i];
    int incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o);
      if (e >= o) incl += v;
    }
    int run = incl - sum;
#pragma unroll
    for (int i = 0; i < 8; ++i) { start[e * 8 + i] = run; run += n[i]; }
    if (e == 63) tiles[0] = incl < max_tiles ? incl : max_tiles;
  }
  __syncthreads();
  if (e >= n_experts) return;
  int t = start[e];
  for (int r = mine.lo; r < mine.hi && t < max_tiles; r += mine.step, ++t) {
    tiles[1 + kTileRec * t] = e;
    tiles[2 + kTileRec * t] = r;
    tiles[3 + kTileRec * t] = min(r + mine.step, mine.hi);
    tiles[4 + kTileRec * t] = start[e];
  }
}

// ------------------------------------------------------------------- GEMM
// A codes [rows, K], sA_t [K/128][rows_capacity]; B codes [n_experts][N][K] (DUAL:
// B0 = gate, B1 = up), S [n_experts][N/128][K/128].  DUAL: hq codes [rows, N] and
// hs_t [N/128][rows_capacity] of the SwiGLU values; else C bf16 [rows, N].
typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// LDS of a tile of NB 32-row blocks: weight stages | activation stages | row scales.
template <int NB> struct Ring8 {
  static constexpr int kB = 256 * 8, kA = NB * 32 * 8;            // 16-byte slots of a stage
  static constexpr int kS = 256;                                          // row scales of a stage (a wavefront fetches 64)
  static constexpr int kSB = NB <= 2 ? 4 : 3;                             // weight stages
  static constexpr int kSA = NB == 1 ? 4 : (NB <= 5 ? 3 : 2);             // activation stages: kSB or one less
  static constexpr int kBytes = (kSB * kB + kSA * kA) * 16 + kSA * kS * 4;
  static_assert(kBytes <= 160 * 1024, "LDS of a CU");
};

template <bool DUAL, int NB, int WM>
__device__ __forceinline__ void fp8act_gemm_body(
    const uint8_t* __restrict__ A, const float* __restrict__ sA_t, int rows_capacity,
    const uint8_t* __restrict__ B0, const uint8_t* __restrict__ B1, const float* __restrict__ S0,
    const float* __restrict__ S1, uint16_t* __restrict__ C, uint8_t* __restrict__ hq, float* __restrict__ hs_t,
    int N, int K, int e, int row0, int row1, int n0, int wave, uint4* __restrict__ smem) {
  using R = Ring8<NB>;
  constexpr int SA = R::kSA, SB = R::kSB;
  constexpr int WB0 = WM == 0 ? 0 : (NB + 1) / 2;                 // first row block of this wavefront
  constexpr int NBW = WM == 0 ? (NB + 1) / 2 : NB / 2;            // ... and their number
  constexpr int NACC = NBW > 0 ? NBW : 1;
  constexpr int NLB = 4, NLA = WM == 0 ? (NB + 1) / 2 : NB / 2;   // load instructions per step
  constexpr int HALF = 128;
  uint4* const ringB = smem;
  uint4* const ringA = smem + SB * R::kB;
  float* const ringS = reinterpret_cast<float*>(ringA + SA * R::kA);
  const int lane = threadIdx.x & 63, wn = wave & 3;
  const int h = lane >> 5, l31 = lane & 31;
  const int nkb = K / kQBlock, nnb = N / 128;
  const int rows = row1 - row0;
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(A + size_t(row0) * K), 0, rows * K, 0x00020000);
  const int brows = N - n0 < HALF * (DUAL ? 1 : 2) ? N - n0 : HALF * (DUAL ? 1 : 2);
  const __amdgpu_buffer_rsrc_t rb0 = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(B0 + (size_t(e) * N + n0) * K), 0, brows * K, 0x00020000);
  const __amdgpu_buffer_rsrc_t rb1 = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>((DUAL ? B1 : B0) + (size_t(e) * N + n0) * K), 0, brows * K, 0x00020000);
  // load q of a stage fills its rows q*64 + wave*8 .. +8: lane l owns slot l%8 of row l/8 and
  // fetches the piece that belongs there
  const int lrow = wave * 8 + (lane >> 3), lpiece = (lane & 7) ^ ((wave * 4 + (lane >> 4)) & 7);
  int off[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) off[q] = (q * 64 + lrow) * K + lpiece * 16;
  // row scales of a stage: wavefronts w and w + 4 fetch the same 64
  const int srow = wn * 64 + lane;
  const float* const sp = sA_t + (row0 + srow < row1 ? row0 + srow : row1 - 1);
  auto issue_b = [&](int kb) {
    uint4* const st = ringB + (kb % SB) * R::kB + wave * 64;
#pragma unroll
    for (int q = 0; q < NLB; ++q) {
      if (DUAL && q >= 2)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rb1, (lptr_t)(st + q * 512), 16, off[q - 2], kb * kQBlock, 0, 0);
      else
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rb0, (lptr_t)(st + q * 512), 16, off[q], kb * kQBlock, 0, 0);
    }
  };
  auto issue_a = [&](int kb) {
    uint4* const st = ringA + (kb % SA) * R::kA + wave * 64;
#pragma unroll
    for (int q = 0; q < NLA; ++q)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lptr_t)(st + q * 512), 16, off[q], kb * kQBlock, 0, 0);
    __builtin_amdgcn_global_load_lds((gptr_t)(sp + size_t(kb) * rows_capacity),
                                     (lptr_t)(ringS + (kb % SA) * R::kS + wn * 64), 4, 0, 0);
  };
  constexpr int NLS = NLA + 1;

  f32x16 acc[NACC][2];
#pragma unroll
  for (int i = 0; i < NACC; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
  const int brow0 = DUAL ? wn * 32 : wn * 64;
  const int brow1 = DUAL ? HALF + wn * 32 : wn * 64 + 32;
  int nb0 = (n0 + (DUAL ? 0 : wn * 64)) / 128;
  nb0 = nb0 < nnb ? nb0 : nnb - 1;
  const float* const s0p = S0 + (size_t(e) * nnb + nb0) * nkb;
  const float* const s1p = DUAL ? S1 + (size_t(e) * nnb + nb0) * nkb : s0p;

  // Weight block scales: lane l holds those of K blocks l, l + 64, ..  (A scalar load in every step
  // misses its cache every sixteenth time, and the whole workgroup waits for memory.)
  float sv0, sv1;
  auto load_scales = [&](int kb) {
    sv0 = s0p[min(kb + lane, nkb - 1)];
    sv1 = s1p[min(kb + lane, nkb - 1)];
  };
  auto scale = [&](float v, int kb) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), kb & 63)); };
  load_scales(0);
  // The two wavefronts of a SIMD (w and w + 4, the two row halves) take turns: in one phase a
  // wavefront issues loads and reads all fragments of a step, in the next it multiplies them; row
  // half 1 runs one phase behind row half 0.
  //   phase   row half 0                                       row half 1
  //   2j      loads A(j+SA-1), B(j+SB-1), read step j          MFMAs of step j-1
  //   2j+1    MFMAs of step j                                  loads A(j+SA-1), B(j+SB-1), read step j
  // Step j+1 must have landed when phase 2j+1 ends: every wavefront waits for its own loads of it
  // before that barrier.  A stage is filled again two phases after row half 0 has read it and one
  // after row half 1 has, which therefore waits for its reads before the barrier.
#pragma unroll
  for (int g = 0; g < SB - 1; ++g) {
    if (g < SA - 1 && g < nkb) issue_a(g);
    if (g < nkb) issue_b(g);
  }
  // What was issued after step j+1's last load: SB-2 whole groups, or, with one activation stage
  // less, SA-2 and the weights of the group that held the step's activations.
  constexpr int kYounger = SA == SB ? (SB - 2) * (NLB + NLS) : NLB + (SA - 2) * (NLB + NLS);
  // Fragment (32 rows, sub-step s): lane l reads the 16-byte pieces (2s + l/32)*2, +1 of row l%32;
  // row blocks are multiples of 32 rows apart, which the swizzle does not see.
  int at[2][2];
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int t = 0; t < 2; ++t) at[s][t] = swz(l31, (2 * s + h) * 2 + t);
  auto frag = [&](const uint4* base, int s) {
    const uint4 lo = base[at[s][0]], hi = base[at[s][1]];
    return i32x8{(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
  };
  i32x8 fb[2][2], fa[NACC][2];                     // [sub-step][column block], [row block][sub-step]
  float sa[NACC];
  f32x16 part[2];                                  // sums of a K block, [column block]
  float f1 = 0.f;      // f1: scale of part[1], which is added up late
#pragma unroll
  for (int q = 0; q < 16; ++q) part[1][q] = 0.f;
  auto mma = [&](int i, int j) {
#pragma unroll
    for (int q = 0; q < 16; ++q) part[j][q] = 0.f;
    part[j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb[0][j], fa[i][0], part[j], 0, 0, 0, 0x7f7f7f7f, 0, 0x7f7f7f7f);
    part[j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb[1][j], fa[i][1], part[j], 0, 0, 0, 0x7f7f7f7f, 0, 0x7f7f7f7f);
  };
  auto add = [&](int i, int j, float f) {
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[i][j][q] = fmaf(part[j][q], f, acc[i][j][q]);
  };
  auto phase_end = [&](bool drain) {
    __builtin_amdgcn_sched_barrier(0);
    if (drain) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto landed = [&](int kb) {                      // step kb + 1
    if (kb + SB - 1 < nkb) wait_vmcnt<kYounger>(); else wait_vmcnt<0>();
  };
  landed(-1);
  phase_end(false);
  if (WM == 1) phase_end(false);                   // one phase behind row half 0
  for (int kb = 0; kb < nkb; ++kb) {
    if (kb + SA - 1 < nkb) issue_a(kb + SA - 1);
    if (kb + SB - 1 < nkb) issue_b(kb + SB - 1);
    if (kb > 0 && (kb & 63) == 0) {
      load_scales(kb);
      wait_vmcnt<0>();                             // here, so that no wait is needed where they are used
    }
    const float c0 = scale(sv0, kb), c1 = scale(sv1, kb);
    if constexpr (NBW > 0) {
      const uint4* const Bb = ringB + (kb % SB) * R::kB;
      const uint4* const Ab = ringA + (kb % SA) * R::kA + WB0 * 256;
      const float* const Sb = ringS + (kb % SA) * R::kS + WB0 * 32 + l31;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        fb[s][0] = frag(Bb + brow0 * 8, s);
        fa[0][s] = frag(Ab, s);
      }
#pragma unroll
      for (int s = 0; s < 2; ++s) fb[s][1] = frag(Bb + brow1 * 8, s);
#pragma unroll
      for (int i = 0; i < NBW; ++i) {
        if (i > 0) {
          fa[i][0] = frag(Ab + i * 256, 0);
          fa[i][1] = frag(Ab + i * 256, 1);
        }
        sa[i] = Sb[i * 32];
      }
      add(NBW - 1, 1, f1);
    }
    if (WM == 1) landed(kb);
    phase_end(WM == 1);
    if constexpr (NBW > 0) {
#pragma unroll
      for (int i = 0; i < NBW; ++i) {
        mma(i, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (i > 0) add(i - 1, 1, f1);
        __builtin_amdgcn_sched_barrier(0);
        mma(i, 1);
        __builtin_amdgcn_sched_barrier(0);
        add(i, 0, sa[i] * c0);
        f1 = sa[i] * c1;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (WM == 0) landed(kb);
    phase_end(false);
  }
  if (WM == 0) phase_end(false);
  if constexpr (NBW > 0) add(NBW - 1, 1, f1);

  // D layout: lane l, register q -> weight row (q/4)*8 + (l/32)*4 + q%4, activation row l%32: a
  // lane holds four neighbouring columns of one output row.
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the stages have been read by all
  if constexpr (DUAL) {
    // The tile's 128 columns are one block of the intermediate's quantisation: the largest
    // magnitude of a row over the four wavefronts of its half, then codes, turned around in LDS
    // so that a store writes whole 128-byte rows.
    float* const amax = reinterpret_cast<float*>(smem + FBM * 9);    // [4][FBM], behind the codes
#pragma unroll
    for (int i = 0; i < NBW; ++i) {
      float m = 0.f;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const float g = acc[i][0][q];
        const float v = g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * acc[i][1][q];
        acc[i][0][q] = v;
        m = fmaxf(m, fabsf(v));
      }
      m = fmaxf(m, __shfl_xor(m, 32));
      if (h == 0) amax[wn * FBM + (WB0 + i) * 32 + l31] = m;
    }
    __syncthreads();
    uint32_t* const codes = reinterpret_cast<uint32_t*>(smem);       // [FBM] rows of 9 pieces
#pragma unroll
    for (int i = 0; i < NBW; ++i) {
      const int r = (WB0 + i) * 32 + l31;
      const float m = fmaxf(fmaxf(amax[r], amax[FBM + r]), fmaxf(amax[2 * FBM + r], amax[3 * FBM + r]));
      const float scale = m > 0.f ? m / 448.0f : 1.0f;
      if (wn == 0 && h == 0 && row0 + r < row1) hs_t[size_t(n0 / kQBlock) * rows_capacity + row0 + r] = scale;
      // v / scale without the general division's scaling steps, for scales whose reciprocal is far
      // from the ends of the range (the general division took 3 us of a tile)
      const bool plain = __all(m == 0.f || (m > 0x1p-90f && m < 0x1p90f));
      const float rs = __builtin_amdgcn_rcpf(scale);
      auto quotient = [&](float v) {
        if (!plain) return v / scale;
        const float q = v * rs;
        return fmaf(fmaf(-scale, q, v), rs, q);
      };
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = fminf(fmaxf(quotient(acc[i][0][g * 4 + q]), -448.0f), 448.0f);
        int c = __builtin_amdgcn_cvt_pk_fp8_f32(v[0], v[1], 0, false);        // round to nearest even
        c = __builtin_amdgcn_cvt_pk_fp8_f32(v[2], v[3], c, true);
        codes[r * 36 + wn * 8 + g * 2 + h] = uint32_t(c);
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < (NB + 1) / 2; ++u) {
      const int r = u * 64 + wave * 8 + (lane >> 3);
      if (r < rows)
        *reinterpret_cast<uint4*>(hq + size_t(row0 + r) * N + n0 + (lane & 7) * 16) = smem[r * 9 + (lane & 7)];
    }
  } else {
    uint4* const turn = smem + wave * (2 * 32 * 9);
    uint16_t* const cw = C + size_t(row0) * N + n0 + wn * 64;
    const bool col_in = n0 + wn * 64 + (lane & 7) * 8 < N;
#pragma unroll
    for (int i = 0; i < NBW; ++i) {
      uint4* const t = turn + (i & 1) * 32 * 9;
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          reinterpret_cast<uint2*>(t + l31 * 9 + j * 4 + g)[h] =
              make_uint2(pack_bf16(acc[i][j][g * 4], acc[i][j][g * 4 + 1]),
                         pack_bf16(acc[i][j][g * 4 + 2], acc[i][j][g * 4 + 3]));
      asm volatile("" ::: "memory");               // the reads below see the writes above (same wavefront)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = u * 8 + (lane >> 3), row = (WB0 + i) * 32 + r;
        const uint4 v = t[r * 9 + (lane & 7)];
        if (row0 + row < row1 && col_in) *reinterpret_cast<uint4*>(cw + size_t(row) * N + (lane & 7) * 8) = v;
      }
      asm volatile("" ::: "memory");
    }
  }
}

template <bool DUAL>
__global__ __launch_bounds__(512) void fp8act_gemm_kernel(
    const uint8_t* __restrict__ A, const float* __restrict__ sA_t, int rows_capacity,
    const uint8_t* __restrict__ B0, const uint8_t* __restrict__ B1, const float* __restrict__ S0,
    const float* __restrict__ S1, uint16_t* __restrict__ C, uint8_t* __restrict__ hq, float* __restrict__ hs_t,
    int N, int K, const int32_t* __restrict__ offsets, const int32_t* __restrict__ tiles) {
  // handed on as a generic pointer: with the LDS array named in the loop the
  // compiler drains every DMA in flight before each LDS read
  extern __shared__ uint4 fsmem[];
  constexpr int BN = DUAL ? 128 : 256;
  const int n_ntiles = (N + BN - 1) / BN;
  const int total = tiles[0] * n_ntiles, per_xcd = (total + 7) >> 3;
  const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (int(blockIdx.x >> 3) >= per_xcd || logical >= total) return;
  const int at = logical / n_ntiles;
  const int ea = tiles[1 + kTileRec * at], first = tiles[4 + kTileRec * at];
  const int cnt = tiles_of(offsets, ea, rows_capacity).count;
  const int local = logical - first * n_ntiles;
  const int gsz = 4 * n_ntiles, grp = local / gsz, rem = local - grp * gsz;
  const int mc = min(cnt - grp * 4, 4);
  const int ntile = rem / mc, mtile = first + grp * 4 + (rem - ntile * mc);
  const int e = tiles[1 + kTileRec * mtile], row0 = tiles[2 + kTileRec * mtile],
            row1 = tiles[3 + kTileRec * mtile];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#define MOE_TILE8(NB)                                                                                   \
  case NB:                                                                                              \
    if (wave < 4) fp8act_gemm_body<DUAL, NB, 0>(A, sA_t, rows_capacity, B0, B1, S0, S1, C, hq, hs_t, N, K, e, row0, row1, ntile * BN, wave, fsmem); \
    else fp8act_gemm_body<DUAL, NB, 1>(A, sA_t, rows_capacity, B0, B1, S0, S1, C, hq, hs_t, N, K, e, row0, row1, ntile * BN, wave, fsmem);          \
    break
  switch ((row1 - row0 + 31) >> 5) {
    MOE_TILE8(1);
    MOE_TILE8(2);
    MOE_TILE8(3);
    MOE_TILE8(4);
    MOE_TILE8(5);
    MOE_TILE8(6);
  }
#undef MOE_TILE8
}

}  // namespace

// workspace: tiles | x codes | x scales | hmid codes | hmid scales
struct Fp8ActWs {
  int32_t* tiles;
  uint8_t* xq;
  float* xs_t;
  uint8_t* hq;
  float* hs_t;
  int max_tiles;
  size_t bytes;
};

static Fp8ActWs carve_fp8act(void* ws, int rows_capacity, int n_experts, int H, int I) {
  Fp8ActWs f;
  char* p = static_cast<char*>(ws);
  size_t off = 0;
  f.max_tiles = rows_capacity / 128 + n_experts + 1;
  f.tiles = reinterpret_cast<int32_t*>(p + off); off += align_up(size_t(1 + kTileRec * f.max_tiles) * 4);
  f.xq = reinterpret_cast<uint8_t*>(p + off);    off += align_up(size_t(rows_capacity) * H);
  f.xs_t = reinterpret_cast<float*>(p + off);    off += align_up(size_t(H / kQBlock) * rows_capacity * 4);
  f.hq = reinterpret_cast<uint8_t*>(p + off);    off += align_up(size_t(rows_capacity) * I);
  f.hs_t = reinterpret_cast<float*>(p + off);    off += align_up(size_t(I / kQBlock) * rows_capacity * 4);
  f.bytes = off;
  return f;
}

static bool fp8act_ok(const moe_config* c) {
  return c && c->act_dtype == MOE_BF16 && c->weight_dtype == MOE_FP8_E4M3_B128 && c->hidden > 0 &&
         c->inter_local > 0 && c->hidden % 128 == 0 && c->inter_local % 128 == 0;
}

}  // namespace moe

using namespace moe;

extern "C" {

size_t moe_fp8act_workspace_bytes(const moe_config* cfg, int32_t n_experts_here,
                                  int32_t rows_capacity) {
  if (!fp8act_ok(cfg) || n_experts_here < 1 || n_experts_here > 512 || rows_capacity < 0) return 0;
  return carve_fp8act(nullptr, rows_capacity, n_experts_here, cfg->hidden, cfg->inter_local).bytes;
}

// shared by the two FFN entry points: xs_q / xs_scales given -> no input quantisation
static moe_status fp8act_run(const moe_config* cfg, int32_t n_experts_here, const void* xs,
                             const void* xs_q, const float* xs_scales, const int32_t* offsets,
                             int32_t rows_capacity, const void* w_gate, const void* w_up,
                             const void* w_down, const float* s_gate, const float* s_up,
                             const float* s_down, void* ys, void* ws, size_t ws_bytes, void* stream) {
  if (!cfg) return MOE_ERR_INVALID_ARG;
  if (!fp8act_ok(cfg)) return MOE_ERR_UNSUPPORTED;
  if (n_experts_here < 1 || n_experts_here > 512 || rows_capacity < 0) return MOE_ERR_INVALID_ARG;
  if (rows_capacity == 0) return MOE_OK;
  const void* ptrs[] = {xs ? xs : xs_q, xs ? xs : static_cast<const void*>(xs_scales), offsets, w_gate,
                        w_up, w_down, s_gate, s_up, s_down, ys, ws};
  for (const void* p : ptrs)
    if (!p || (reinterpret_cast<uintptr_t>(p) & 15)) return MOE_ERR_INVALID_ARG;
  const int H = cfg->hidden, I = cfg->inter_local;
  Fp8ActWs f = carve_fp8act(ws, rows_capacity, n_experts_here, H, I);
  if (ws_bytes < f.bytes) return MOE_ERR_WORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  constexpr int lds = 160 * 1024;
  auto k1 = fp8act_gemm_kernel<true>;
  auto k2 = fp8act_gemm_kernel<false>;
  static uint64_t opted1 = 0, opted2 = 0;
  lds_opt_in(reinterpret_cast<const void*>(k1), lds, opted1);
  lds_opt_in(reinterpret_cast<const void*>(k2), lds, opted2);
  const dim3 qgrid((rows_capacity + 3) / 4);
  // as many tiles as the rows can come to, in eight equal runs.  (Lower tiles where 192 rows leave
  // CUs without one, a shared expert of 1500 to 4500 rows, were slower: 300 -> 323 us a layer at
  // 3000 tokens, I 512: they fetch the weights more often and take the CUs from the route beside.)
  const int max_mt = rows_capacity / FBM + (n_experts_here < rows_capacity ? n_experts_here : rows_capacity);
  auto grid = [&](int n_ntiles) { return dim3(unsigned((size_t(max_mt) * n_ntiles + 7) / 8 * 8)); };
  MOE_LAUNCH(MOE_K_FFN_TILES, fp8act_tiles_kernel, dim3(1), dim3(512), 0, s, offsets, n_experts_here,
             rows_capacity, f.tiles, f.max_tiles);
  const uint8_t* aq = static_cast<const uint8_t*>(xs_q);
  const float* as = xs_scales;
  if (xs) {
    MOE_LAUNCH(MOE_K_FFN_TILES, fp8act_quant_kernel, qgrid, dim3(256), 0, s,
               static_cast<const uint16_t*>(xs), offsets, n_experts_here, H, rows_capacity, f.xq, f.xs_t);
    aq = f.xq;
    as = f.xs_t;
  }
  MOE_LAUNCH(MOE_K_FFN_GEMM1, k1, grid(I / 128), dim3(512), lds, s, aq, as, rows_capacity,
             static_cast<const uint8_t*>(w_gate), static_cast<const uint8_t*>(w_up), s_gate, s_up,
             static_cast<uint16_t*>(nullptr), f.hq, f.hs_t, I, H, offsets, f.tiles);
  MOE_LAUNCH(MOE_K_FFN_GEMM2, k2, grid((H + 255) / 256), dim3(512), lds, s, f.hq, f.hs_t, rows_capacity,
             static_cast<const uint8_t*>(w_down), static_cast<const uint8_t*>(nullptr), s_down,
             static_cast<const float*>(nullptr), static_cast<uint16_t*>(ys), static_cast<uint8_t*>(nullptr),
             static_cast<float*>(nullptr), H, I, offsets, f.tiles);
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_DEVICE;
}

moe_status moe_quant_act(const moe_config* cfg, int32_t rows, const void* x, void* codes,
                         float* scales, void* stream) {
  if (!cfg) return MOE_ERR_INVALID_ARG;
  if (cfg->act_dtype != MOE_BF16 || cfg->hidden <= 0 || cfg->hidden % 128) return MOE_ERR_UNSUPPORTED;
  if (rows < 0) return MOE_ERR_INVALID_ARG;
  if (rows == 0) return MOE_OK;
  const void* ptrs[] = {x, codes, scales};
  for (const void* p : ptrs)
    if (!p || (reinterpret_cast<uintptr_t>(p) & 15)) return MOE_ERR_INVALID_ARG;
  hipStream_t s = static_cast<hipStream_t>(stream);
  MOE_LAUNCH(MOE_K_FFN_TILES, fp8act_quant_kernel, dim3((rows + 3) / 4), dim3(256), 0, s,
             static_cast<const uint16_t*>(x), static_cast<const int32_t*>(nullptr), 0, cfg->hidden, rows,
             static_cast<uint8_t*>(codes), scales);
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_DEVICE;
}

moe_status moe_expert_ffn_fp8act(const moe_config* cfg, int32_t n_experts_here, const void* xs,
                                 const int32_t* offsets, int32_t rows_capacity, const void* w_gate,
                                 const void* w_up, const void* w_down, const float* s_gate,
                                 const float* s_up, const float* s_down, void* ys, void* ws,
                                 size_t ws_bytes, void* stream) {
  if (!xs) return MOE_ERR_INVALID_ARG;
  return fp8act_run(cfg, n_experts_here, xs, nullptr, nullptr, offsets, rows_capacity, w_gate, w_up,
                    w_down, s_gate, s_up, s_down, ys, ws, ws_bytes, stream);
}

moe_status moe_expert_ffn_fp8q(const moe_config* cfg, int32_t n_experts_here, const void* xs_q,
                               const float* xs_scales, const int32_t* offsets,
                               int32_t rows_capacity, const void* w_gate, const void* w_up,
                               const void* w_down, const float* s_gate, const float* s_up,
                               const float* s_down, void* ys, void* ws, size_t ws_bytes,
                               void* stream) {
  if (!xs_q || !xs_scales) return MOE_ERR_INVALID_ARG;
  return fp8act_run(cfg, n_experts_here, nullptr, xs_q, xs_scales, offsets, rows_capacity, w_gate,
                    w_up, w_down, s_gate, s_up, s_down, ys, ws, ws_bytes, stream);
}

}  // extern "C"

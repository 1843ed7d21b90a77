// Grouped expert MLP (Sec. II: every expert is an independent MLP; under TP
// its projections are sliced and the partial results summed afterwards).
//
//   GEMM-1  hmid[r,:] = silu(xs[r,:] Wgate_e^T) .* (xs[r,:] Wup_e^T)   r in expert e's rows
//   GEMM-2  ys[r,:]   = hmid[r,:] Wdown_e^T
//
// Both are "TN" GEMMs (activations [rows,K] and weights [N,K], K contiguous)
// over ragged row groups whose bounds live on the device.  A one-block
// prologue turns `offsets` into a table of M tiles (expert, first row, end
// row); the GEMM grid is sized for the worst case and workgroups past the
// table's length exit at once, so there is no host round trip.
//
// bf16 path: v_mfma_f32_32x32x16_bf16, fp32 accumulation, K step 64.  GEMM-1
// loads a gate tile and the matching up tile so that one lane holds g and u of
// the same element and the SwiGLU is applied in registers.  Three kernels, by
// rows per expert: ffn_gemm8w_kernel (prefill: up to 256 rows x 256 weight rows
// per workgroup, operands global -> LDS directly, LDS rings; GEMM-2 of short groups
// of many experts: up to 128 rows x 512 weight rows), ffn_skinny_kernel
// (decode and fp8 weights: weight streaming, K split across wavefronts, no LDS
// staging) and ffn_shortk_kernel (GEMM-2 of narrow TP slices: K up to 128).  Which one
// runs: plan_ffn.  fp32 path: ffn_f32_kernel (matrix instructions), and for K up to 64 in
// large launches ffn_f32_valu_kernel.
// fp8 weights: the weight-streaming kernel widens the e4m3 codes to bf16 in
// registers (exact) and multiplies the fp32 partial sum of each 128-deep K block
// by the 128x128 block scale, and so do the short tiles of up to 64 rows that the tall-tile
// kernel has in the place of its own for a few dozen rows per expert (e4m3_body, chosen on the
// device: short_tile_rows); in higher ones and in the tall ones, which keep the codes
// in their LDS ring, code * scale is rounded to bf16 on the way to the matrix unit.
#include <type_traits>

#include "device_util.h"
#include "moe_internal.h"
#include "tile_rules.h"
#include "shortk_layout.h"

namespace moe {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) {
  return __builtin_bit_cast(uint16_t, (__bf16)f);   // round to nearest even
}

// silu(g) * u with the hardware exp2 and reciprocal (1 ulp each): the result is
// rounded to bf16 right after
__device__ __forceinline__ float silu_mul_fast(float g, float u) {
  const float t = __builtin_amdgcn_exp2f(g * -1.44269504088896341f);
  return g * u * __builtin_amdgcn_rcpf(1.0f + t);
}

__device__ __forceinline__ float silu_mul(float g, float u) {
  return g / (1.0f + __expf(-g)) * u;
}

// The same quotient without the general division's scaling steps, for finite g >= -kSiluPlain
// (the reciprocal is a normal number): the residual of g * rcp(d) is exact in an fma, so one
// correction leaves the rounding of the last step and the reciprocal's error squared.
constexpr float kSiluPlain = 87.f;
__device__ __forceinline__ float silu_mul_plain(float g, float u) {
  const float d = 1.0f + __expf(-g);
  const float r = __builtin_amdgcn_rcpf(d);
  const float q = g * r;
  return fmaf(fmaf(-d, q, g), r, q) * u;
}

// ------------------------------------------------------------- tile table
// tiles[0] = number of M tiles (| flags); then per tile a record (expert, first row, end
// row, index of the expert's first tile, number of tiles of the expert).
constexpr int kShortTiles = 1 << 30;          // the tiles are e4m3_body's
constexpr int kWholeTiles = 1 << 29;          // ... and stay whole
constexpr int kTileCount = kWholeTiles - 1;
constexpr int kTileRec = 5;
// K-split of leftover tiles (see ffn_gemm8w_kernel): at most this many tiles are
// split, into at most kSplitMax parts of at least kSplitMinSteps K steps, and all
// parts together are at most one workgroup per CU (split_parts).
constexpr int kSplitTickets = 256;
constexpr int kPartFloats = 512 * 128;        // fp32 accumulators of one workgroup
static_assert(kSplitTickets == kFfnSplitSlots && kCUs <= kFfnSplitSlots, "workspace holds one slot per part");
static_assert(size_t(kPartFloats) * 4 == kFfnPartBytes, "partial-sum slot size");
#ifndef MOE_SPREAD_SLOTS
#define MOE_SPREAD_SLOTS 2
#endif
#ifndef MOE_RING_EXTRA_A
#define MOE_RING_EXTRA_A 2
#endif
// An expert's rows are cut into ceil(M/bm) tiles of equal height (rounded up to 32
// rows) instead of full tiles plus a short tail.  One thread per expert (512 at most); the
// launch is one workgroup's latency chain in front of GEMM-1, so the scan runs in registers
// (DPP) and an expert's thread writes its tiles by itself when no expert has more than four;
// else one thread per tile looks its expert up.  Against a scan by one wavefront over shared
// memory and a look-up for every tile: one token (128 experts) 3.1 -> 2.2 us, 64 fp32 tokens (8
// experts) 2.5 -> 1.9, 65 536 tokens (2100 tiles) 10.1 -> 6.8; behind a dispatch of a few MB 4.6
// either way.  (No table, every workgroup scanning the offsets: 0.8 us a tile, 65 536 tokens
// 5356 -> 5452 us.)  Where the GEMM has a choice of tiles, their numbers at all heights come
// out of the same scan (0.5 us).
constexpr int kTileThreads = 512, kOwnTiles = 4;

// The table of one GEMM: tiles of bm rows, or short ones.
struct TileJob {
  int32_t* tiles;
  int bm;
  ShortTiles alt;
};

// CHOICE: one of the GEMMs may have short tiles.  (A branch at run time made the one-workgroup
// launch longer for all others: one bf16 token, 128 experts, 37.2 -> 38.1 us.)
template <bool CHOICE>
__global__ __launch_bounds__(kTileThreads) void ffn_tiles_kernel(const int32_t* __restrict__ offsets,
                                                       int n_experts, int rows_capacity, int max_tiles,
                                                       TileJob job, TileJob second,
                                                       int32_t* __restrict__ tickets) {
  __shared__ int32_t start[kTileThreads + 1];
  __shared__ int32_t off[kTileThreads + 1];
  __shared__ int4 wave_sum[kTileThreads / 64];
  __shared__ int32_t wave_many[kTileThreads / 64];
  const int e = threadIdx.x, lane = e & 63, wave = e >> 6;
  // a second workgroup, when launched, builds a second table
  if (blockIdx.x == 1) job = second;
  int32_t* const __restrict__ tiles = job.tiles;
  int bm = job.bm;
  int lo = 0, hi = 0;
  if (e < n_experts) {
    lo = min(max(offsets[e], 0), rows_capacity);
    hi = min(max(offsets[e + 1], 0), rows_capacity);
  }
  // arrival counters of the K-split tiles of the two GEMM launches that follow
  static_assert(kTileThreads == 2 * kSplitTickets, "one counter per thread");
  if (blockIdx.x == 0) tickets[e] = 0;
  // The expert's tiles at the height bm and, where the GEMM has the choice, at 64, 96 and 128 rows.
  const int rows = max(hi - lo, 0);
  int count[4] = {int(unsigned(rows + bm - 1) / unsigned(bm)), (rows + 63) >> 6, int(unsigned(rows + 95) / 96u),
                  (rows + 127) >> 7};
  int incl[4] = {wave_incl_sum(count[0]), 0, 0, 0}, many = __any(count[0] > kOwnTiles) ? 1 : 0;
  if (CHOICE && job.alt.nt) {
#pragma unroll
    for (int i = 1; i < 4; ++i) {
      incl[i] = wave_incl_sum(count[i]);
      many |= __any(count[i] > kOwnTiles) ? 1 << i : 0;
    }
    // the tallest tile in 32-row blocks: bit 3 + blocks, of the highest set
#pragma unroll
    for (int b = 4; b <= 8; ++b) many |= __any(rows > 32 * (b - 1) * count[0]) ? 8 << b : 0;
  }
  if (lane == 63) {
    wave_sum[wave] = make_int4(incl[0], incl[1], incl[2], CHOICE ? incl[3] : many);
    if (CHOICE) wave_many[wave] = many;
  }
  __syncthreads();
  int4 sum[kTileThreads / 64], all = make_int4(0, 0, 0, 0);
  many = 0;
#pragma unroll
  for (int w = 0; w < kTileThreads / 64; ++w) {
    sum[w] = wave_sum[w];
    all = make_int4(all.x + sum[w].x, all.y + sum[w].y, all.z + sum[w].z, all.w + sum[w].w);
    many |= CHOICE ? wave_many[w] : sum[w].w;
  }
  const int chosen = CHOICE && job.alt.nt ? short_tile_rows(job.alt, n_experts, RowTiles{all.x, all.y, all.z, all.w,
                                          many >> 7 ? (28 - __clz(many)) * 32 : 96}) : 0;
  const int at = chosen ? chosen / 32 - 1 : 0;
  auto pick = [&](int own, int c64, int c96, int c128) { return at == 0 ? own : (at == 1 ? c64 : (at == 2 ? c96 : c128)); };
  if (chosen) bm = chosen;
  const int mine = pick(count[0], count[1], count[2], count[3]);
  const int total = pick(all.x, all.y, all.z, all.w);
  const bool look_up = (many >> at) & 1;
  int before = 0;
#pragma unroll
  for (int w = 0; w < kTileThreads / 64; ++w)
    before += w < wave ? pick(sum[w].x, sum[w].y, sum[w].z, sum[w].w) : 0;
  const int first = before + pick(incl[0], incl[1], incl[2], incl[3]) - mine;     // experts past the last one: `total`
  const int n_tiles = total < max_tiles ? total : max_tiles;
  if (e == 0) tiles[0] = n_tiles | (chosen ? kShortTiles : 0) | (chosen && n_experts == 1 ? kWholeTiles : 0);
  auto write = [&](int t, int expert, int rlo, int rhi, int t0) {
    const int m = rhi - rlo, nt = int(unsigned(m + bm - 1) / unsigned(bm));
    const int step = (int(unsigned(m + nt - 1) / unsigned(nt)) + 31) / 32 * 32;
    const int r = rlo + (t - t0) * step;
    tiles[1 + kTileRec * t] = expert;
    tiles[2 + kTileRec * t] = r;
    tiles[3 + kTileRec * t] = (r + step < rhi) ? r + step : rhi;
    tiles[4 + kTileRec * t] = t0;
    tiles[5 + kTileRec * t] = int(unsigned(m + step - 1) / unsigned(step));
  };
  if (!look_up) {
#pragma unroll
    for (int i = 0; i < kOwnTiles; ++i)
      if (i < mine && first + i < n_tiles) write(first + i, e, lo, hi, first);
    return;
  }
  if (e < n_experts) {                               // (the next thread, of another wavefront, must not touch off[n_experts])
    start[e] = first;
    off[e] = lo;
    if (e == n_experts - 1) off[n_experts] = hi;
  }
  __syncthreads();
  // one thread per tile: its expert is the last one whose first tile is <= t
  for (int t = e; t < n_tiles; t += kTileThreads) {
    int x = 0, x_hi = n_experts;
    while (x_hi - x > 1) {
      const int mid = (x + x_hi) >> 1;
      if (start[mid] <= t) x = mid; else x_hi = mid;
    }
    write(t, x, off[x], off[x + 1], start[x]);
  }
}

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// ---------------------------------------- MFMA GEMM, 256x256 tile, 8 wavefronts
// Prefill-sized groups.  Block tile 256 rows x 256 weight rows (DUAL: 128 gate +
// the matching 128 up rows), 512 threads: wavefront (wm, wn) = (w/4, w%4) computes
// rows wm*128..+128 and the 64 weight rows of column block wn (DUAL: 32 gate + 32
// up), i.e. four 32-row blocks x two 32-column blocks = 128 accumulator registers.
// Operands go global -> LDS directly (`buffer_load_dwordx4 ... lds`, 16 B per
// lane, no register staging; a buffer descriptor per operand with the K step as
// scalar offset, which measured 1-4 % faster than 64-bit per-lane addresses and
// zero-fills rows past the tile's end); the
// per-lane offset is permuted so that the linear LDS write of a
// wavefront lands in the XOR-swizzled layout the MFMA operand reads expect
// (piece ^ (row/2)&7: the 16 lanes the LDS serves per cycle hit 16 different
// 16-byte columns).  Operand fragments are read one K sub-step ahead of the
// MFMAs that consume them.  Workgroup ids are remapped so that each XCD (own L2)
// walks a contiguous run of tiles, M tiles of one expert first: neighbours
// share the expert's weight panel and the activation panel.  Wavefronts w and
// w+4 (the two row halves) share a SIMD: while one of them waits (LDS latency, a
// load instruction being accepted, the barrier) the other keeps the matrix unit
// busy; on full tiles they do so in turns (see the two forms of the K loop).
// The operand pointers are __restrict__ on purpose: the compiler then knows that
// the LDS reads do not alias what the loads-to-LDS write (it cannot see their LDS
// side) and leaves the waiting for loads to the explicit vmcnt waits; without that
// it waits for every load in flight in front of each LDS read, which serialises
// the loop.  K step 64
// (128-byte rows: whole cache lines per row and load instruction); weights and
// activations have LDS rings of their own (see Ring).
// NBW = valid 32-row blocks of this wavefront's 128 rows (0..4).
// NB = valid 32-row blocks of the tile (1..8), WM = which half of the rows this
// wavefront computes; both compile-time so the K loop has no branches.  A weight
// stage holds 256 rows of 128 B, an activation stage NB*32 rows.  As many whole
// (activation + weight) stages as fit in the CU's 160 KB of LDS, at most four,
// give the depth of the weight ring; what is left takes up to two further
// activation stages (256-row tile: 2 weight + 3 activation stages = 160 KB;
// 160-row tile: 3 + 3; short tiles up to 4 + 6).  With the rotated K loop below
// the loads of a step must land three quarters of a step after the previous
// step's barrier, and the extra activation stage is worth 9 % on the 256-row
// tile.
// K step per stage: 64, i.e. 128-byte LDS rows, so that every load instruction
// moves whole cache lines.  (A K step of 32 would allow four stages for the tall
// tiles too, but its 64-byte row pieces halve the efficiency of the load path:
// measured 8 % slower on the 256-row tiles.)
// Eight e4m3 codes -> eight bf16 values of code * scale (exact widening to fp32,
// one fp32 multiply, round to nearest even).
__device__ __forceinline__ uint4 widen_scaled(uint2 c, float sc) {
  const f32x2 p0 = __builtin_amdgcn_cvt_pk_f32_fp8(c.x, false), p1 = __builtin_amdgcn_cvt_pk_f32_fp8(c.x, true);
  const f32x2 p2 = __builtin_amdgcn_cvt_pk_f32_fp8(c.y, false), p3 = __builtin_amdgcn_cvt_pk_f32_fp8(c.y, true);
  uint4 r;
  asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r.x) : "v"(p0[0] * sc), "v"(p0[1] * sc));
  asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r.y) : "v"(p1[0] * sc), "v"(p1[1] * sc));
  asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r.z) : "v"(p2[0] * sc), "v"(p2[1] * sc));
  asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r.w) : "v"(p3[0] * sc), "v"(p3[1] * sc));
  return r;
}

// Eight e4m3 codes -> eight bf16 values, exact.
__device__ __forceinline__ uint4 widen_codes(uint2 c) {
  return make_uint4(__builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c.x, 1.0f, false)),
                    __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c.x, 1.0f, true)),
                    __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c.y, 1.0f, false)),
                    __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c.y, 1.0f, true)));
}

// One part of a K-split tile: `parts` workgroups share the tile's K range, part
// `slot - slot0` of them is this one; parts == 1: the whole K range, no partial sums.
struct SplitJob {
  int parts, slot, slot0;
  float* partial;          // [kCUs][kPartFloats]
  int32_t* ticket;         // arrival counter of the tile
};

// F8: the weight tile holds e4m3 codes (64-byte rows: four pieces), widened to
// bf16 on the way from LDS to the matrix unit.
// BR: weight rows of a stage (256, or 512 for the wide tiles of short row groups).
template <int NB, bool F8 = false, int BR = 256> struct Ring {
  static constexpr int kBK = 64;
  static constexpr int kPPR = kBK / 8;                              // 16-byte pieces per activation row
  static constexpr int kPPRB = F8 ? kBK / 16 : kBK / 8;             // ... per weight row
  static constexpr int kARows = NB * 32;
  static constexpr int kASlots = kARows * kPPR;                     // 16-byte slots of an A stage
  static constexpr int kBSlots = BR * kPPRB;                        // ... of a B stage
  static constexpr int kLds = 160 * 1024;
  static constexpr int kFit = kLds / ((kASlots + kBSlots) * 16);
  static constexpr int kSB = kFit > 4 ? 4 : kFit;                   // weight stages
  // LDS left over after kSB whole stages takes further activation stages
  static constexpr int kMore = (kLds - kSB * (kASlots + kBSlots) * 16) / (kASlots * 16);
  static constexpr int kSA = kSB + (kMore > MOE_RING_EXTRA_A ? MOE_RING_EXTRA_A : kMore);
};

// F8: Be0 / Be1 point at e4m3 codes, Se0 / Se1 at the expert's block scales of
// the 128-row block this wavefront's weight rows lie in ([K/128] values).  The
// scaled weight code * scale is rounded to bf16 before the MFMA (the exact
// per-block scale would need a second set of accumulators).
// RAGGED: N or K is no multiple of 64.
template <bool DUAL, int NB, int WM, bool F8, bool RAGGED, int BR = 256>
__device__ __forceinline__ void gemm8w_body(const uint16_t* __restrict__ A,
                                            const char* __restrict__ Be0,
                                            const char* __restrict__ Be1,
                                            const float* __restrict__ Se0,
                                            const float* __restrict__ Se1,
                                            uint16_t* __restrict__ C, int N, int K, int row0,
                                            int row1, int n0, uint4* smem, int wave, int kbeg,
                                            int klen, const SplitJob& job) {
  static_assert(BR == 256 || (BR == 512 && WM == 0 && NB <= 4), "wide tiles: all wavefronts on one row half");
  constexpr int NBW = NB - WM * 4 < 0 ? 0 : (NB - WM * 4 > 4 ? 4 : NB - WM * 4);
  constexpr int HALF = BR / 2;                       // DUAL: gate rows | up rows of a stage
  constexpr int SA = Ring<NB, F8, BR>::kSA, SB = Ring<NB, F8, BR>::kSB;
  constexpr int KS = Ring<NB, F8, BR>::kBK;          // K step
  constexpr int PPR = Ring<NB, F8, BR>::kPPR;        // pieces per activation row in LDS
  constexpr int PPRB = Ring<NB, F8, BR>::kPPRB;      // pieces per weight row in LDS
  constexpr int RPI = 64 / PPR;                      // rows filled by one load instruction
  constexpr int RPIB = 64 / PPRB;
  constexpr int WB = F8 ? 1 : 2;                     // bytes per weight element
  constexpr int AS = Ring<NB, F8, BR>::kASlots;      // slots of an A stage
  constexpr int BS = Ring<NB, F8, BR>::kBSlots;      // slots of a B stage
  uint4* const ringA = smem;
  uint4* const ringB = smem + SA * AS;
  const int lane = threadIdx.x & 63;
  const int wn = BR == 512 ? wave : wave & 3;        // column block of this wavefront
  const int ksteps = (klen + KS - 1) / KS;           // this workgroup's K window starts at kbeg
  // A K that is not a multiple of the step ends in a short step: its pieces past K are
  // sent out of the descriptors' range and land as zeros.
  const int tail = RAGGED ? klen % KS : 0;
  constexpr int kOut = 0x7fffffff;

  // LDS row r keeps its piece p at slot p ^ f(r): f = (r/2)&7 for 128-byte rows,
  // (r/4)&3 for 64-byte rows; both keep the 16 lanes the LDS serves per cycle
  // on 16 different 16-byte columns.
  auto slot = [&](int row, int piece) {
    return row * PPR + (piece ^ (PPR == 8 ? (row >> 1) & 7 : (row >> 2) & 3));
  };
  auto slot_b = [&](int row, int piece) {
    return row * PPRB + (piece ^ (PPRB == 8 ? (row >> 1) & 7 : (row >> 2) & 3));
  };
  // loads: a wavefront instruction fills 64 consecutive slots = RPI rows.  Row
  // group rg = q*8 + wave; lane l -> row l/PPR, and it fetches the piece that
  // belongs in slot l%PPR of that row: (l%PPR) ^ ((rg*4 + l/16) & (PPR-1)).
  // A row groups exist for rg < NB*32/RPI.
  constexpr int AGROUPS = NB * 32 / RPI;
  constexpr int NAQ = AGROUPS / 8;                   // full rounds of 8 wavefronts
  constexpr int AREM = AGROUPS % 8;                  // wavefronts 0..AREM-1 load one more
  constexpr int NBQ = BR / RPIB / 8;                 // weight row groups per wavefront
  const int lrow = lane / PPR;
  // Operands through buffer descriptors: a wave-uniform base per operand (this
  // tile's first row / first weight row, at the K window's start), a 32-bit byte
  // offset per lane, and the K step as a scalar offset.  Rows past the tile's end
  // (or past the last weight row) are out of the descriptor's range and load zeros.
  const int arows = row1 - row0;
  const __amdgpu_buffer_rsrc_t rsrcA = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(A + size_t(row0) * K + kbeg), 0,
      int((size_t(arows - 1) * K + klen) * 2), 0x00020000);
  const int brows = (N - n0) < HALF * (DUAL ? 1 : 2) ? (N - n0) : HALF * (DUAL ? 1 : 2);
  const __amdgpu_buffer_rsrc_t rsrcB0 = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(Be0 + (size_t(n0) * K + kbeg) * WB), 0,
      int((size_t(brows - 1) * K + klen) * WB), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcB1 = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>((DUAL ? Be1 : Be0) + (size_t(n0) * K + kbeg) * WB), 0,
      int((size_t(brows - 1) * K + klen) * WB), 0x00020000);
  auto piece_a = [&](int q) { return (lane % PPR) ^ (((q * 8 + wave) * 4 + (lane >> 4)) & (PPR - 1)); };
  auto piece_b = [&](int q) { return (lane % PPRB) ^ (((q * 8 + wave) * 4 + (lane >> 4)) & (PPRB - 1)); };
  int aoff[NAQ + 1], boff[NBQ];
#pragma unroll
  for (int q = 0; q < NAQ + 1; ++q) aoff[q] = (((q * 8 + wave) * RPI + lrow) * K + piece_a(q) * 8) * 2;
#pragma unroll
  for (int q = 0; q < NBQ; ++q) {
    const int br = (q * 8 + wave) * RPIB + lane / PPRB;
    const int bl = (DUAL && br >= HALF) ? br - HALF : br;     // row inside its matrix' tile
    boff[q] = bl * K * WB + piece_b(q) * 16;
  }
  // weight row groups q: rows q*8*RPIB .. of the stage; the upper half is the up matrix
  auto b_is_up = [](int q) { return DUAL && q * 8 * RPIB >= HALF; };
#define MOE_LOAD_A_AT(off, kcol, dst) \
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcA, (lptr_t)(dst), 16, off, (kcol) * 2, 0, 0)
#define MOE_LOAD_B_AT(q, off, kcolb, dst)                                                        \
  do {                                                                                           \
    if (b_is_up(q)) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcB1, (lptr_t)(dst), 16, off, (kcolb), 0, 0); \
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcB0, (lptr_t)(dst), 16, off, (kcolb), 0, 0);            \
  } while (0)
#define MOE_LOAD_A(q, kcol, dst) MOE_LOAD_A_AT(aoff[q], kcol, dst)
#define MOE_LOAD_B(q, kcolb, dst) MOE_LOAD_B_AT(q, boff[q], kcolb, dst)
  const bool extra = AREM > 0 && wave < AREM;        // this wavefront loads one more A row group
  auto issue_a = [&](int ks) {
    const int kcol = ks * KS;
    uint4* st = ringA + (ks % SA) * AS;
    const int lim = tail != 0 && ks == ksteps - 1 ? tail : KS;
#pragma unroll
    for (int q = 0; q < NAQ; ++q)
      MOE_LOAD_A_AT(piece_a(q) * 8 < lim ? aoff[q] : kOut, kcol, st + (q * 8 + wave) * 64);
    if (extra) MOE_LOAD_A_AT(piece_a(NAQ) * 8 < lim ? aoff[NAQ] : kOut, kcol, st + (NAQ * 8 + wave) * 64);
  };
  auto issue_b = [&](int ks) {
    const int kcol = ks * KS * WB;
    uint4* st = ringB + (ks % SB) * BS;
    const int lim = tail != 0 && ks == ksteps - 1 ? tail : KS;
#pragma unroll
    for (int q = 0; q < NBQ; ++q)
      MOE_LOAD_B_AT(q, F8 || piece_b(q) * 8 < lim ? boff[q] : kOut, kcol, st + (q * 8 + wave) * 64);
  };
  // the same for a step that is known to be a whole one
  auto issue_a_whole = [&](int ks) {
    uint4* st = ringA + (ks % SA) * AS;
#pragma unroll
    for (int q = 0; q < NAQ; ++q) MOE_LOAD_A(q, ks * KS, st + (q * 8 + wave) * 64);
    if (extra) MOE_LOAD_A(NAQ, ks * KS, st + (NAQ * 8 + wave) * 64);
  };
  auto issue_b_whole = [&](int ks) {
    uint4* st = ringB + (ks % SB) * BS;
#pragma unroll
    for (int q = 0; q < NBQ; ++q) MOE_LOAD_B(q, ks * KS * WB, st + (q * 8 + wave) * 64);
  };
  // Issue group of step g (after its barrier): weights of step g+SB-1, then
  // activations of step g+SA-1 (SA >= SB).  Loads return in order, so at the
  // barrier of step ks everything younger than the weights of step ks may stay in
  // flight: the activation part of group ks-SB+1 (when SA > SB) and the SB-2 whole
  // groups after it.  Near the end of K, where groups shrink, wait for all.
  constexpr int YA = SA > SB ? 1 : 0;
  constexpr int YG = SB - 2;
  auto wait_step = [&](bool steady) {
    if (!steady) wait_vmcnt<0>();
    else if (extra) wait_vmcnt<YA * (NAQ + 1) + YG * (NAQ + 1 + NBQ)>();
    else wait_vmcnt<YA * NAQ + YG * (NAQ + NBQ)>();
  };

  constexpr int NA = NBW > 0 ? NBW : 1;
  f32x16 acc[NA][2];
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;

  const int arow = WM * 128;
  const int brow0 = DUAL ? wn * 32 : wn * 64;
  const int brow1 = DUAL ? HALF + wn * 32 : wn * 64 + 32;
  constexpr int NKK = KS / 16;                       // MFMA sub-steps per K step

#pragma unroll
  for (int g = 1 - SA; g < 0; ++g) {
    if (g + SB - 1 >= 0 && g + SB - 1 < ksteps) issue_b(g + SB - 1);
    if (g + SA - 1 < ksteps) issue_a(g + SA - 1);
  }
  // One load instruction of a step's issue group: ops 0..NBQ-1 are the weight row
  // groups, NBQ..NBQ+NAQ-1 the activation row groups (weights first: see above).
  constexpr int NOPS = NBQ + NAQ;
  auto issue_op = [&](int op, uint4* stb, uint4* sta, int kcb, int kca) {
    if (op < NBQ) MOE_LOAD_B(op, kcb * WB, stb + (op * 8 + wave) * 64);
    else if (op < NOPS) MOE_LOAD_A(op - NBQ, kca, sta + ((op - NBQ) * 8 + wave) * 64);
  };
  // Two forms of the K loop.  Full 256-row tiles of bf16 weights alternate the two
  // wavefronts of a SIMD between memory and MFMA phases (measured 4-6 % faster on
  // the long-K GEMM-1, 1 % on GEMM-2).  Shorter tiles, where row half 1 has fewer
  // MFMAs than row half 0 and the phases would not balance (160-row tiles: 5 %
  // slower), and e4m3 weights, whose widening makes the memory phase the longer one
  // (7-9 % slower), keep all wavefronts in one phase with loads, LDS reads and MFMAs
  // interleaved.
  constexpr bool kAlternate = !F8 && NB == 8;
  if constexpr (kAlternate) {
  // The two wavefronts of a SIMD (w and w+4, the two row halves) take turns: a
  // step has four phases, each closed by a barrier, and a wavefront alternates
  // between a memory phase (issue half of its loads, read the operand fragments of
  // two K sub-steps) and an MFMA phase (the 4 x NBW MFMAs on those fragments); row
  // half 1 runs one phase behind row half 0, so that at any time one wavefront of a
  // SIMD feeds the matrix unit while the other one's loads and LDS reads are
  // accepted:
  //   phase   row half 0                      row half 1
  //   4j      loads B(j+SB-1), read (j, 0-1)   MFMAs (j-1, 2-3)
  //   4j+1    MFMAs (j, 0-1)                   loads B(j+SB-1), read (j, 0-1)
  //   4j+2    loads A(j+SA-1), read (j, 2-3)   MFMAs (j, 0-1)
  //   4j+3    MFMAs (j, 2-3)                   loads A(j+SA-1), read (j, 2-3)
  // Step j+1 must have landed when phase 4j+3 ends: every wavefront waits for its
  // own loads of that step before that barrier.  A stage is refilled only after
  // the barrier that follows its last read (B(j-1)'s stage in phase 4j or later,
  // A(j-1)'s in phase 4j+2 or later).  That is why all fragments of a half step are
  // read in the memory phase: a read left for the MFMA phase of row half 1 (phase
  // 4j+4 for sub-step 3 of step j) would meet row half 0's refill of the same
  // weight stage; such a variant measured 1 % faster and gave outputs that changed
  // from run to run on the 16 384-token step.
  uint4 fa[2][NA], fb[2][2];
  auto read_half = [&](int ks, int h) {
    if constexpr (NBW > 0) {
      const uint4* Ab = ringA + (ks % SA) * AS;
      const uint4* Bb = ringB + (ks % SB) * BS;
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) {
        const int piece = (h * 2 + sub) * 2 + (lane >> 5);
        fb[sub][0] = Bb[slot_b(brow0 + (lane & 31), piece)];
        fb[sub][1] = Bb[slot_b(brow1 + (lane & 31), piece)];
#pragma unroll
        for (int i = 0; i < NBW; ++i) fa[sub][i] = Ab[slot(arow + i * 32 + (lane & 31), piece)];
      }
    }
  };
  auto mma_half = [&]() {
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      const bf16x8 b0 = __builtin_bit_cast(bf16x8, fb[sub][0]);
      const bf16x8 b1 = __builtin_bit_cast(bf16x8, fb[sub][1]);
#pragma unroll
      for (int i = 0; i < NBW; ++i) {
        const bf16x8 a = __builtin_bit_cast(bf16x8, fa[sub][i]);
        acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b0, acc[i][0], 0, 0, 0);
        acc[i][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b1, acc[i][1], 0, 0, 0);
      }
    }
  };
  // `drain`: this wavefront's LDS reads must have returned before the barrier
  // (the stage they read is refilled in the next phase).  Otherwise they may
  // still be in flight when the barrier is passed: the MFMAs that use them wait
  // for them one by one.
  auto phase_end = [&](auto drain_c) {
    __builtin_amdgcn_sched_barrier(0);               // nothing of the next phase moves in front of the barrier
    if constexpr (decltype(drain_c)::value) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr std::true_type drain{};
  constexpr std::false_type no_drain{};
  auto step = [&](int ks, auto steady_c) {
    constexpr bool ST = decltype(steady_c)::value;      // this step issues both of its load groups
    const int kb = ks + SB - 1, ka = ks + SA - 1;
    __builtin_amdgcn_sched_barrier(0);
    if (ST) issue_b_whole(kb);
    else if (kb < ksteps) issue_b(kb);
    read_half(ks, 0);
    __builtin_amdgcn_sched_barrier(0);
    phase_end(no_drain);
    mma_half();
    __builtin_amdgcn_sched_barrier(0);
    phase_end(no_drain);
    if (ST) issue_a_whole(ka);
    else if (ka < ksteps) issue_a(ka);
    read_half(ks, 1);
    __builtin_amdgcn_sched_barrier(0);
    if (WM == 1) wait_step(ST);
    // row half 1 reads the last fragments of this step's weight stage here, and
    // row half 0 refills that stage in the next phase
    if constexpr (WM == 1) phase_end(drain); else phase_end(no_drain);
    mma_half();
    __builtin_amdgcn_sched_barrier(0);
    if (WM == 0) wait_step(ST);
    phase_end(no_drain);
  };
  wait_step(SA - 2 < ksteps);                                 // step 0 has landed
  phase_end(no_drain);
  if (WM == 1) phase_end(no_drain);                          // one phase behind row half 0
  const int steady_steps = ksteps - (SA - 1) - (tail != 0);
  int ks = 0;
  for (; ks < steady_steps; ++ks) step(ks, std::true_type{});
  for (; ks < ksteps; ++ks) step(ks, std::false_type{});
  if (WM == 0) phase_end(no_drain);
  } else {
  // One turn of the K loop, rotated by a sub-step so that the synchronisation for
  // step j sits in front of the LAST sub-step of step j-1:
  //   wait for the loads of step j, barrier  (every wavefront holds its last
  //     fragments of step j-1 in registers, so that step's stages are free)
  //   slot 0: issue loads | read fragments (j, 0) | MFMAs (j-1, 3)
  //   slot 1: issue loads | read fragments (j, 1) | MFMAs (j, 0)
  //   slot 2:               read fragments (j, 2) | MFMAs (j, 1)
  //   slot 3:               read fragments (j, 3) | MFMAs (j, 2)
  // The first LDS reads after a barrier are covered by MFMAs that are already
  // fed, and the load instructions of the step's issue group (which stall a
  // wavefront until the load path accepts them) are handed out between MFMAs,
  // ahead of the slot's LDS reads.  SPREAD: the issue group is unconditional (all
  // but the last SA-1 turns); otherwise it is issued in one go behind a range check.
  constexpr int NA2 = NA;
  uint4 fa[2][NA2], fb[2][2];
#pragma unroll
  for (int i = 0; i < NA2; ++i) fa[1][i] = make_uint4(0, 0, 0, 0);
  fb[1][0] = fb[1][1] = make_uint4(0, 0, 0, 0);     // the first turn multiplies zeros
  auto mfmas = [&](int set) {
    const bf16x8 b0 = __builtin_bit_cast(bf16x8, fb[set][0]);
    const bf16x8 b1 = __builtin_bit_cast(bf16x8, fb[set][1]);
#pragma unroll
    for (int i = 0; i < NBW; ++i) {
      const bf16x8 a = __builtin_bit_cast(bf16x8, fa[set][i]);
      acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b0, acc[i][0], 0, 0, 0);
      acc[i][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b1, acc[i][1], 0, 0, 0);
    }
  };
  constexpr int NSLOT = MOE_SPREAD_SLOTS;                    // slots that issue loads
  constexpr int OPK = (NOPS + NSLOT - 1) / NSLOT;            // load instructions per slot
  auto turn = [&](int ks, auto spread_c) {
    constexpr bool SPREAD = decltype(spread_c)::value && NBW > 0;
    // step ks must have landed
    wait_step(ks + SA - 2 < ksteps);
    // a bare barrier (no fence): __syncthreads() would also drain the younger loads
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    // every wavefront has read all of step ks-1, so its stages can be refilled
    const int kb = ks + SB - 1, ka = ks + SA - 1;
    uint4* const stb = ringB + (kb % SB) * BS;
    uint4* const sta = ringA + (ka % SA) * AS;
    if constexpr (!SPREAD) {
      if (kb < ksteps) issue_b(kb);
      if (ka < ksteps) issue_a(ka);
    }
    if constexpr (NBW > 0) {
      const uint4* Ab = ringA + (ks % SA) * AS;
      const uint4* Bb = ringB + (ks % SB) * BS;
      float sc0 = 1.f, sc1 = 1.f;
      if constexpr (F8) { sc0 = Se0[ks >> 1]; sc1 = Se1[ks >> 1]; }   // one block = two K steps
      auto read_frags = [&](int kk, int set) {
        const int piece = kk * 2 + (lane >> 5);
        if constexpr (F8) {
          // sub-step kk: eight codes at bytes kk*16 + (lane/32)*8 of the row's 64
          const uint2 c0 = reinterpret_cast<const uint2*>(&Bb[slot_b(brow0 + (lane & 31), kk)])[lane >> 5];
          const uint2 c1 = reinterpret_cast<const uint2*>(&Bb[slot_b(brow1 + (lane & 31), kk)])[lane >> 5];
          fb[set][0] = widen_scaled(c0, sc0);
          fb[set][1] = widen_scaled(c1, sc1);
        } else {
          fb[set][0] = Bb[slot_b(brow0 + (lane & 31), piece)];
          fb[set][1] = Bb[slot_b(brow1 + (lane & 31), piece)];
        }
#pragma unroll
        for (int i = 0; i < NBW; ++i) fa[set][i] = Ab[slot(arow + i * 32 + (lane & 31), piece)];
      };
#pragma unroll
      for (int sl = 0; sl < NKK; ++sl) {
        const int set = sl & 1;                              // fragments read in this slot
        __builtin_amdgcn_sched_barrier(0);
        constexpr int NLD = OPK;
        const bool loads_here = sl < NSLOT;
        if constexpr (SPREAD) {
          if (sl < NSLOT) {
#pragma unroll
            for (int o = 0; o < OPK; ++o)
              if (sl * OPK + o < NOPS) issue_op(sl * OPK + o, stb, sta, kb * KS, ka * KS);
          }
        }
        read_frags(sl, set);
        mfmas(set ^ 1);
        if (NBW >= 2) {
          // one MFMA, then the loads while no LDS read of this wavefront is
          // outstanding, then MFMA / LDS read pairs
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          if (SPREAD && loads_here) __builtin_amdgcn_sched_group_barrier(0x020, NLD, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
#pragma unroll
          for (int i = 0; i < NBW + 1; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          }
          __builtin_amdgcn_sched_group_barrier(0x008, 2 * NBW - (NBW + 2), 0);
        }
      }
      if constexpr (SPREAD && AREM > 0) {
        if (extra)
          MOE_LOAD_A(NAQ, ka * KS, sta + (NAQ * 8 + wave) * 64);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  const int spread_steps = ksteps - (SA - 1) - (tail != 0);
  int ks = 0;
  for (; ks < spread_steps; ++ks) turn(ks, std::true_type{});
  for (; ks < ksteps; ++ks) turn(ks, std::false_type{});
  if constexpr (NBW > 0) mfmas(1);                           // sub-step 3 of the last step

  }
  // A K-split part leaves its fp32 accumulators in the workspace (register order:
  // 8-byte chunk c of thread t at index c*512 + t, so a wavefront's store is 512
  // contiguous bytes); the part that arrives last adds all parts in the
  // order of their K windows and carries on with the epilogue.  No workgroup waits
  // for another: every part counts itself in and all but the last one leave.
  if (job.parts > 1) {
    // The partial sums go past the XCD's own (non-coherent) L2 as device-scope
    // stores and are read back as device-scope loads, so no cache has to be
    // written back or invalidated as a whole; the wait below makes every store of
    // this part complete before the part counts itself in.
    uint64_t* const mine = reinterpret_cast<uint64_t*>(job.partial + size_t(job.slot) * kPartFloats) + threadIdx.x;
    if constexpr (NBW > 0) {
#pragma unroll
      for (int i = 0; i < NBW; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const uint64_t bits = uint64_t(__float_as_uint(acc[i][j][2 * q])) |
                                  (uint64_t(__float_as_uint(acc[i][j][2 * q + 1])) << 32);
            __hip_atomic_store(mine + ((i * 2 + j) * 8 + q) * 512, bits, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
          }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    int32_t* const flag = reinterpret_cast<int32_t*>(smem);   // the rings are idle from here on
    if (threadIdx.x == 0) *flag = atomicAdd(job.ticket, 1);
    __syncthreads();
    if (*flag != job.parts - 1) return;
    if constexpr (NBW > 0) {
      // one 32x32 block at a time: its chunks of all (at most four) parts are
      // fetched together, then added in the order of the parts
      const uint64_t* const all = reinterpret_cast<const uint64_t*>(job.partial + size_t(job.slot0) * kPartFloats) + threadIdx.x;
#pragma unroll
      for (int i = 0; i < NBW; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          uint64_t v[kSplitMax][8];
#pragma unroll
          for (int p = 0; p < kSplitMax; ++p)
            if (p < job.parts) {
#pragma unroll
              for (int q = 0; q < 8; ++q)
                v[p][q] = __hip_atomic_load(all + size_t(p) * (kPartFloats / 2) + ((i * 2 + j) * 8 + q) * 512,
                                            __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
          for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
#pragma unroll
          for (int p = 0; p < kSplitMax; ++p)
            if (p < job.parts) {
#pragma unroll
              for (int q = 0; q < 8; ++q) {
                acc[i][j][2 * q] += __uint_as_float(uint32_t(v[p][q]));
                acc[i][j][2 * q + 1] += __uint_as_float(uint32_t(v[p][q] >> 32));
              }
            }
        }
    }
  }

  // Epilogue.  Lane l holds column l%32 of each 32x32 block and rows
  // (q/4)*8 + (l/32)*4 + q%4: two rows are rounded to bf16 by one packed convert
  // and stored as the low / high half.  Only the last 32-row block of a tile can
  // hold rows of the next expert's segment; the others are stored unpredicated.
  if constexpr (NBW > 0) {
    const int lrow = arow + (lane >> 5) * 4;                    // first row of this lane, tile-relative
    const int valid = row1 - row0 - lrow;                        // rows r (tile-relative to lrow) < valid exist
    uint16_t* const cl = C + size_t(row0 + lrow) * N + n0 + (lane & 31);
    auto put2 = [&](uint16_t* p, float v0, float v1, bool ok0, bool ok1) {
      const uint32_t pk = pack_bf16(v0, v1);
      if (ok0) p[0] = uint16_t(pk);
      if (ok1) p[N] = uint16_t(pk >> 16);
    };
    // Sizes that are no multiple of 64 take the quotient: the reciprocal is one ulp
    // coarser, and g * u past the fp32 range times a reciprocal of zero (strongly
    // negative g) is no number where the quotient is zero.
    // The division costs 2.4 us of a 128-row tile's 14.5 (two wavefronts a SIMD, 64 values a
    // lane), its plain form 0.7.
    auto store_block = [&](int i, auto pred_c, auto swiglu) {
      constexpr bool PRED = decltype(pred_c)::value;
#pragma unroll
      for (int q = 0; q < 16; q += 2) {
        const int r = i * 32 + (q >> 2) * 8 + (q & 3);
        const bool ok0 = !PRED || r < valid, ok1 = !PRED || r + 1 < valid;
        uint16_t* const p = cl + size_t(r) * N;
        if (DUAL) {
          if (n0 + wn * 32 + (RAGGED ? lane & 31 : 0) < N)
            put2(p + wn * 32, swiglu(acc[i][0][q], acc[i][1][q]),
                 swiglu(acc[i][0][q + 1], acc[i][1][q + 1]), ok0, ok1);
        } else {
#pragma unroll
          for (int j = 0; j < 2; ++j)
            if (n0 + wn * 64 + j * 32 + (RAGGED ? lane & 31 : 0) < N)
              put2(p + wn * 64 + j * 32, acc[i][j][q], acc[i][j][q + 1], ok0, ok1);
        }
      }
    };
    const bool full = row1 - row0 == NB * 32;
#pragma unroll
    for (int i = 0; i < NBW; ++i) {
      auto store = [&](auto swiglu) {
        if (i == NBW - 1 && WM * 4 + NBW == NB && !full) store_block(i, std::true_type{}, swiglu);
        else store_block(i, std::false_type{}, swiglu);
      };
      if constexpr (DUAL && RAGGED) {
        float low = acc[i][0][0], high = low;
#pragma unroll
        for (int q = 1; q < 16; ++q) {
          low = fminf(low, acc[i][0][q]);
          high = fmaxf(high, acc[i][0][q]);
        }
        if (__any(!(low >= -kSiluPlain && high < INFINITY))) store([](float g, float u) { return silu_mul(g, u); });
        else store([](float g, float u) { return silu_mul_plain(g, u); });
      } else {
        store([](float g, float u) { return silu_mul_fast(g, u); });
      }
    }
  }
}

#undef MOE_LOAD_A
#undef MOE_LOAD_B
#undef MOE_LOAD_A_AT
#undef MOE_LOAD_B_AT

template <bool DUAL, int NB, bool F8, bool RAGGED, bool WIDE>
__device__ __forceinline__ void gemm8w_tile(const uint16_t* A, const char* Be0, const char* Be1,
                                            const float* Se0, const float* Se1, uint16_t* C, int N,
                                            int K, int row0, int row1, int n0, uint4* smem,
                                            int wave, int kbeg, int klen, const SplitJob& job) {
  if constexpr (WIDE) {
    // at most four row blocks: all eight wavefronts work on them, each on its own
    // 32 (DUAL) or 64 weight rows of a 512-row stage
    gemm8w_body<DUAL, NB, 0, F8, RAGGED, 512>(A, Be0, Be1, Se0, Se1, C, N, K, row0, row1, n0, smem, wave, kbeg, klen, job);
  } else {
    if (wave < 4) gemm8w_body<DUAL, NB, 0, F8, RAGGED>(A, Be0, Be1, Se0, Se1, C, N, K, row0, row1, n0, smem, wave, kbeg, klen, job);
    else gemm8w_body<DUAL, NB, 1, F8, RAGGED>(A, Be0, Be1, Se0, Se1, C, N, K, row0, row1, n0, smem, wave, kbeg, klen, job);
  }
}

// ---------------------------- MFMA GEMM, e4m3 weights, short tiles: up to 128 rows
// e4m3 weights with a few dozen rows per expert: the work is streaming the codes in, and a
// tile is short of rows, not of weights.  Tile: up to 128 rows (NB 32-row blocks) x 256
// weight rows (DUAL: 128 gate + the matching 128 up rows), K step 128 = one scale block = a
// whole cache line of every weight row.  All eight wavefronts work on all rows: wavefront
// (kh, wn) = (w/4, w%4) multiplies half kh of every K block with the 64 weight rows of
// column block wn, and the two halves are added at the end.  (The tall-tile kernel leaves the
// four wavefronts of its second row half without a row below 160 rows, and its K step of 64
// reads half lines.)  Codes are read as 16 bytes and widened to bf16 by one instruction a
// pair, exact; for up to 64 rows the block scale multiplies the fp32 sums of the K block,
// above (where a second set of sums would not fit the registers) code * scale is rounded
// to bf16 as in the tall-tile kernel.  The weights are the first operand, so a lane holds
// columns of one row; output rows are turned around in LDS and stored whole.
// Bound by nothing alone: 32 experts of 48 rows, hidden 7168, I 1024: GEMM-1 118, GEMM-2 62 us
// (4.0 / 3.8 TB/s of codes) against 125 / 70; a stream of the same loads alone runs at 6 TB/s, the
// same steps without loads take 90 us, and the two add up rather than overlap.  Where the tiles
// are taken: short_tile_rows.  Whole layer (us), on the tall tiles and with the choice: 64 tokens 188 -> 161, 700 292 ->
// 280; Zipf-routed 160 tokens 204 -> 158, 256 207 -> 193; hidden 4096, 16 of 128 experts, I
// 1536, 1000 tokens 178 -> 151; from 2500 tokens on unchanged.  The routed FFN of six batches of 1531 tokens (1119 to
// 1953 rows on 32 experts) 188-244 -> 167-226, on 128-row tiles alone 176-219.  Tried: weights loaded by one half of the
// wavefronts and activations by the other (deeper weight ring) 118 -> 125, all fragments a
// step ahead 118 -> 122, block scales in scalar registers loaded step by step (no difference),
// tiles of 128 rows at every load (an expert of that many rows then is the launch: Zipf-routed 128
// tokens, I 512, 111 -> 120).
template <int NB> struct RingE {
  static constexpr int kB = 256 * 8, kA = NB * 32 * 16;            // 16-byte slots of a stage
  static constexpr int kSB = NB == 1 ? 4 : 3;                      // weight stages
  static constexpr int kSA = NB <= 2 ? kSB : kSB - 1;              // activation stages
  static_assert((kSB * kB + kSA * kA) * 16 <= 160 * 1024, "LDS of a CU");
};

template <bool DUAL, int NB>
__device__ __forceinline__ void e4m3_body(const uint16_t* __restrict__ A, const char* __restrict__ B0,
                                          const char* __restrict__ B1, const float* __restrict__ s0p,
                                          const float* __restrict__ s1p, uint16_t* __restrict__ C, int N,
                                          int K, int row0, int row1, int n0, int wave, int kb0, int nkb,
                                          const SplitJob& job, uint4* __restrict__ smem) {
  using R = RingE<NB>;
  constexpr int SA = R::kSA, SB = R::kSB, NLA = NB, NLB = 4, HALF = 128;
  constexpr bool kExact = NB <= 2;
  uint4* const ringB = smem;
  uint4* const ringA = smem + SB * R::kB;
  const int lane = threadIdx.x & 63, wn = wave & 3, kh = wave >> 2;
  const int h = lane >> 5, l31 = lane & 31;
  const int rows = row1 - row0;
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(A + size_t(row0) * K + kb0 * 128), 0, ((rows - 1) * K + nkb * 128) * 2, 0x00020000);
  const int brows = N - n0 < HALF * (DUAL ? 1 : 2) ? N - n0 : HALF * (DUAL ? 1 : 2);
  const __amdgpu_buffer_rsrc_t rb0 = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(B0 + size_t(n0) * K + kb0 * 128), 0, (brows - 1) * K + nkb * 128, 0x00020000);
  const __amdgpu_buffer_rsrc_t rb1 = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>((DUAL ? B1 : B0) + size_t(n0) * K + kb0 * 128), 0, (brows - 1) * K + nkb * 128, 0x00020000);
  // weights: load q fills rows q*64 + wave*8 .. +8 of the stage, lane l slot l%8 of row l/8
  const int brow = wave * 8 + (lane >> 3), bpiece = (lane & 7) ^ ((wave * 4 + (lane >> 4)) & 7);
  // activations: load q fills rows q*32 + wave*4 .. +4, lane l slot l%16 of row l/16
  const int arow = wave * 4 + (lane >> 4), apiece = (lane & 15) ^ (arow & 15);
  int boff[4], aoff[NLA];
#pragma unroll
  for (int q = 0; q < 4; ++q) boff[q] = ((DUAL ? q & 1 : q) * 64 + brow) * K + bpiece * 16;
#pragma unroll
  for (int q = 0; q < NLA; ++q) aoff[q] = ((q * 32 + arow) * K + apiece * 8) * 2;
  auto issue_b = [&](int kb) {
    uint4* const st = ringB + (kb % SB) * R::kB + wave * 64;
#pragma unroll
    for (int q = 0; q < NLB; ++q) {
      if (DUAL && q >= 2) __builtin_amdgcn_raw_ptr_buffer_load_lds(rb1, (lptr_t)(st + q * 512), 16, boff[q], kb * 128, 0, 0);
      else __builtin_amdgcn_raw_ptr_buffer_load_lds(rb0, (lptr_t)(st + q * 512), 16, boff[q], kb * 128, 0, 0);
    }
  };
  auto issue_a = [&](int kb) {
    uint4* const st = ringA + (kb % SA) * R::kA + wave * 64;
#pragma unroll
    for (int q = 0; q < NLA; ++q)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lptr_t)(st + q * 512), 16, aoff[q], kb * 256, 0, 0);
  };
  f32x16 acc[NB][2];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
  const int brow0 = DUAL ? wn * 32 : wn * 64;
  const int brow1 = DUAL ? HALF + wn * 32 : wn * 64 + 32;
  // weight pieces kh*4 + t*2 + h of row l%32 (sixteen codes), activation pieces twice that, +1
  int bat[2], aat[2][2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int p = kh * 4 + t * 2 + h;
    bat[t] = l31 * 8 + (p ^ ((l31 >> 1) & 7));
#pragma unroll
    for (int u = 0; u < 2; ++u) aat[t][u] = l31 * 16 + ((p * 2 + u) ^ (l31 & 15));
  }
  // Block scales: lane l holds those of K blocks l, l + 64, ..  (A scalar load in every step misses
  // its cache every sixteenth time, and the whole workgroup waits for memory.)
  float sv0 = s0p[min(lane, nkb - 1)], sv1 = s1p[min(lane, nkb - 1)];
  auto scale = [&](float v, int kb) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), kb & 63)); };
  auto next_scales = [&](int kb) {
    if (kb > 0 && (kb & 63) == 0) {
      sv0 = s0p[min(kb + lane, nkb - 1)];
      sv1 = s1p[min(kb + lane, nkb - 1)];
      wait_vmcnt<0>();                               // here, so that no wait is needed where they are used
    }
  };
  auto read_codes = [&](int kb, uint4 (&code)[2][2]) {
    const uint4* const Bb = ringB + (kb % SB) * R::kB;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      code[0][t] = Bb[brow0 * 8 + bat[t]];
      code[1][t] = Bb[brow1 * 8 + bat[t]];
    }
  };
#pragma unroll
  for (int g = 0; g < SB - 1; ++g) {
    if (g < SA - 1 && g < nkb) issue_a(g);
    if (g < nkb) issue_b(g);
  }
  constexpr int kYounger = SA == SB ? (SB - 2) * (NLB + NLA) : NLB + (SA - 2) * (NLB + NLA);
  for (int kb = 0; kb < nkb; ++kb) {
    if (kb + SB - 2 < nkb) wait_vmcnt<kYounger>(); else wait_vmcnt<0>();
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    const uint4* const Ab = ringA + (kb % SA) * R::kA;
    uint4 code[2][2];
    read_codes(kb, code);
    if (kb + SA - 1 < nkb) issue_a(kb + SA - 1);
    if (kb + SB - 1 < nkb) issue_b(kb + SB - 1);
    next_scales(kb);
    const float c0 = scale(sv0, kb), c1 = scale(sv1, kb);
    uint4 fb[2][2][2];                               // [column block][t][u]: eight bf16 codes, exact
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const uint2 lo = make_uint2(code[j][t].x, code[j][t].y), hi = make_uint2(code[j][t].z, code[j][t].w);
        if constexpr (kExact) {
          fb[j][t][0] = widen_codes(lo);
          fb[j][t][1] = widen_codes(hi);
        } else {
          fb[j][t][0] = widen_scaled(lo, j == 0 ? c0 : c1);
          fb[j][t][1] = widen_scaled(hi, j == 0 ? c0 : c1);
        }
      }
    uint4 fa[2][2][2];                               // [set][t][u]: a row block ahead
    auto read_a = [&](int i) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u) fa[i & 1][t][u] = Ab[i * 512 + aat[t][u]];
    };
    read_a(0);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if (i + 1 < NB) read_a(i + 1);
      f32x16 part[2];
      if constexpr (kExact) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int q = 0; q < 16; ++q) part[j][q] = 0.f;
      }
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            f32x16& c = kExact ? part[j] : acc[i][j];
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fb[j][t][u]),
                                                        __builtin_bit_cast(bf16x8, fa[i & 1][t][u]), c, 0, 0, 0);
          }
      if constexpr (kExact) {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          acc[i][0][q] = fmaf(part[0][q], c0, acc[i][0][q]);
          acc[i][1][q] = fmaf(part[1][q], c1, acc[i][1][q]);
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  // The two wavefronts of a column block (one half of every K block each) add their sums:
  // half kh finishes registers 8*kh .. +8.  D layout (weights first): lane l holds activation row
  // l%32, register q weight row (q/4)*8 + (l/32)*4 + q%4.
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  // A K-split part leaves its sums in the workspace and the part that arrives last adds all
  // parts in the order of their K windows and carries on (as in the tall-tile kernel).
  if (job.parts > 1) {
    uint64_t* const mine = reinterpret_cast<uint64_t*>(job.partial + size_t(job.slot) * kPartFloats) + threadIdx.x;
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 8; ++q)
          __hip_atomic_store(mine + ((i * 2 + j) * 8 + q) * 512,
                             uint64_t(__float_as_uint(acc[i][j][2 * q])) |
                                 (uint64_t(__float_as_uint(acc[i][j][2 * q + 1])) << 32),
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    int32_t* const flag = reinterpret_cast<int32_t*>(smem);
    if (threadIdx.x == 0) *flag = atomicAdd(job.ticket, 1);
    __syncthreads();
    if (*flag != job.parts - 1) return;
    __syncthreads();                                   // the flag's place is used again below
    const uint64_t* const all = reinterpret_cast<const uint64_t*>(job.partial + size_t(job.slot0) * kPartFloats) + threadIdx.x;
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        uint64_t w[kSplitMax][8];
#pragma unroll
        for (int p = 0; p < kSplitMax; ++p)
          if (p < job.parts) {
#pragma unroll
            for (int q = 0; q < 8; ++q)
              w[p][q] = __hip_atomic_load(all + size_t(p) * (kPartFloats / 2) + ((i * 2 + j) * 8 + q) * 512,
                                          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
#pragma unroll
        for (int p = 0; p < kSplitMax; ++p)
          if (p < job.parts) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
              acc[i][j][2 * q] += __uint_as_float(uint32_t(w[p][q]));
              acc[i][j][2 * q + 1] += __uint_as_float(uint32_t(w[p][q] >> 32));
            }
          }
      }
  }
  float* const red = reinterpret_cast<float*>(smem);   // [wavefront][NB][2][8][64]
  float v[NB][2][8];
  // (two copies: a register index that depends on kh would be an indexed access per value)
  auto exchange = [&](auto kh_c) {
    constexpr int Q = decltype(kh_c)::value * 8;
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 8; ++q)
          red[(((wave ^ 4) * NB + i) * 2 + j) * 512 + q * 64 + lane] = acc[i][j][8 - Q + q];
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 8; ++q) v[i][j][q] = acc[i][j][Q + q] + red[((wave * NB + i) * 2 + j) * 512 + q * 64 + lane];
  };
  if (kh == 0) exchange(std::integral_constant<int, 0>{});
  else exchange(std::integral_constant<int, 1>{});
  __syncthreads();
  // the output tile, turned around in LDS: whole rows of it are stored
  constexpr int CP = DUAL ? 16 : 32, P = CP + 1;      // 16-byte pieces per row, and pitch
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < (DUAL ? 1 : 2); ++j)
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        float o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = DUAL ? silu_mul_fast(v[i][0][g * 4 + q], v[i][1][g * 4 + q]) : v[i][j][g * 4 + q];
        // columns wn*32|64 + j*32 + (2 kh + g)*8 + h*4 .. +4
        reinterpret_cast<uint2*>(smem + (i * 32 + l31) * P + wn * (CP / 4) + j * 4 + 2 * kh + g)[h] =
            make_uint2(pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3]));
      }
  __syncthreads();
  constexpr int RPT = 512 / CP;                        // rows per turn of the workgroup
#pragma unroll
  for (int u = 0; u < NB * 32 / RPT; ++u) {
    const int r = u * RPT + threadIdx.x / CP, piece = threadIdx.x % CP, col = n0 + piece * 8;
    if (r < rows && col < N) *reinterpret_cast<uint4*>(C + size_t(row0 + r) * N + col) = smem[r * P + piece];
  }
}

template <bool DUAL>
__device__ __forceinline__ void e4m3_tile(const uint16_t* A, const char* Be0, const char* Be1, const float* S0,
                                          const float* S1, uint16_t* C, int N, int K, int e, int row0, int row1,
                                          int n0, int wave, int part, const SplitJob& job, uint4* smem) {
  const int nkb = K / 128, nnb = N / 128;
  const int k0 = part * nkb / job.parts, k1 = (part + 1) * nkb / job.parts;
  int nb = (n0 + (DUAL ? 0 : (wave & 3) * 64)) / 128;
  nb = nb < nnb ? nb : nnb - 1;
  const float* const s0p = S0 + (size_t(e) * nnb + nb) * nkb + k0;
  const float* const s1p = DUAL ? S1 + (size_t(e) * nnb + nb) * nkb + k0 : s0p;
  switch ((row1 - row0 + 31) >> 5) {
    case 1: e4m3_body<DUAL, 1>(A, Be0, Be1, s0p, s1p, C, N, K, row0, row1, n0, wave, k0, k1 - k0, job, smem); break;
    case 2: e4m3_body<DUAL, 2>(A, Be0, Be1, s0p, s1p, C, N, K, row0, row1, n0, wave, k0, k1 - k0, job, smem); break;
    case 3: e4m3_body<DUAL, 3>(A, Be0, Be1, s0p, s1p, C, N, K, row0, row1, n0, wave, k0, k1 - k0, job, smem); break;
    default: e4m3_body<DUAL, 4>(A, Be0, Be1, s0p, s1p, C, N, K, row0, row1, n0, wave, k0, k1 - k0, job, smem); break;
  }
}

// Leftover tiles.  The hardware hands workgroups to CUs in the order of their
// ids, so when the number of tiles is not a multiple of the 256 CUs the last
// `left` tiles run on `left` CUs while the rest idle for a whole tile time.  When
// at most half of the CUs would be busy, those tiles are cut along K into `parts`
// workgroups each (parts * left <= 256), placed at the end of the grid; everything
// is derived from the tile count on the device, so there is no host round trip.
// The same rule spreads a launch of a few tiles (a shared expert at a decode
// batch) over the chip.
// WIDE: tiles of at most 128 rows (the table is built with that height) x 512
// weight rows, for GEMM-2 launches whose groups are short: twice the weight bytes
// per K step and barrier, half as many tiles.
// F8: or the short tiles of e4m3_body, if the table says so.  They are a branch of this kernel since
// only the device knows the rows; a launch of their own that has nothing to do takes 2-3 us.
template <bool DUAL, bool F8, bool RAGGED, bool WIDE>
__global__ __launch_bounds__(512) void ffn_gemm8w_kernel(
    const uint16_t* __restrict__ A, const void* __restrict__ B0, const void* __restrict__ B1,
    const float* __restrict__ S0, const float* __restrict__ S1, uint16_t* __restrict__ C, int N,
    int K, const int32_t* __restrict__ tiles, int m_fastest, float* __restrict__ partial,
    int32_t* __restrict__ tickets) {
  constexpr int kShortBN = DUAL ? 128 : 256;
  extern __shared__ uint4 smem[];
  const int n_mtiles = F8 ? tiles[0] & kTileCount : tiles[0];
  const bool short_tiles = F8 && (tiles[0] & kShortTiles);
  const int BN = WIDE && !short_tiles ? 2 * kShortBN : kShortBN;
  const int n_ntiles = (N + BN - 1) / BN;
  const int total = n_mtiles * n_ntiles;
  const int ksteps_all = (K + 63) / 64;
  const int pid = blockIdx.x;
  const int left = total % kCUs;
  const int parts = partial && !(F8 && (tiles[0] & kWholeTiles)) ? split_parts(left, ksteps_all / kSplitMinSteps) : 1;
  int logical, part = 0;
  SplitJob job{1, 0, 0, partial, tickets};
  if (parts >= 2) {
    // whole rounds first, every XCD walking a contiguous run of their tiles, then
    // the parts of the leftover tiles
    const int full = total - left;
    if (pid < full) {
      logical = (pid & 7) * (full >> 3) + (pid >> 3);
    } else {
      const int q = pid - full;
      if (q >= left * parts) return;
      const int j = q / parts;
      part = q - j * parts;
      logical = full + j;
      job.parts = parts;
      job.slot = q;
      job.slot0 = j * parts;
      job.ticket = tickets + j;
    }
  } else {
    const int per_xcd = (total + 7) >> 3;
    logical = (pid & 7) * per_xcd + (pid >> 3);
    if ((pid >> 3) >= per_xcd || logical >= total) return;
  }
  int mtile = logical / n_ntiles, ntile = logical - mtile * n_ntiles;
  if (m_fastest) {
    // Inside an expert's block of tiles: groups of up to four M tiles; per group
    // all N tiles, M tile fastest.  The ~32 workgroups an XCD runs at a time then
    // form a (4 M tiles) x (8 N tiles) patch: every weight panel is shared by
    // four of them, every activation panel by eight.
    const int first = tiles[4 + kTileRec * mtile], cnt = tiles[5 + kTileRec * mtile];
    const int local = logical - first * n_ntiles;
    const int gsz = 4 * n_ntiles;
    const int grp = local / gsz, rem = local - grp * gsz;
    const int left_m = cnt - grp * 4;
    const int mc = left_m < 4 ? left_m : 4;
    ntile = rem / mc;
    mtile = first + grp * 4 + (rem - ntile * mc);
  }
  const int e = tiles[1 + kTileRec * mtile], row0 = tiles[2 + kTileRec * mtile],
            row1 = tiles[3 + kTileRec * mtile];
  const int n0 = ntile * BN;
  // this workgroup's window of K steps (even bounds: a block scale spans two steps)
  int kb = 0, ke = ksteps_all;
  if (job.parts > 1) {
    kb = (part * ksteps_all / job.parts) & ~1;
    ke = part == job.parts - 1 ? ksteps_all : (((part + 1) * ksteps_all / job.parts) & ~1);
  }
  constexpr int WB = F8 ? 1 : 2;
  const char* Be0 = static_cast<const char*>(B0) + size_t(e) * N * K * WB;
  const char* Be1 = DUAL ? static_cast<const char*>(B1) + size_t(e) * N * K * WB : nullptr;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if constexpr (F8) {
    if (__builtin_expect(short_tiles, 0)) {
      e4m3_tile<DUAL>(A, Be0, Be1, S0, S1, C, N, K, e, row0, row1, n0, wave, part, job, smem);
      // The compiler lets this branch join the other one's entry.  With memory operations open
      // here it would drain the rings there in front of their loops (tall tiles 1-2 % slower).
      wait_vmcnt<0>();
      return;
    }
  }
  // F8: the scales of the 128-row block this wavefront's weight rows lie in
  const float* Se0 = nullptr;
  const float* Se1 = nullptr;
  if constexpr (F8) {
    const int nkb = K / 128, nnb = N / 128;
    int nb = (n0 + (WIDE ? wave : wave & 3) * (DUAL ? 32 : 64)) / 128;
    nb = nb < nnb ? nb : nnb - 1;
    Se0 = S0 + (size_t(e) * nnb + nb) * nkb + (kb >> 1);
    Se1 = DUAL ? S1 + (size_t(e) * nnb + nb) * nkb + (kb >> 1) : Se0;
  }
#define MOE_TILE_(NBV)                                                                        \
  gemm8w_tile<DUAL, NBV, F8, RAGGED, WIDE>(A, Be0, Be1, Se0, Se1, C, N, K, row0, row1, n0, smem, wave,   \
                                   kb * 64, (ke * 64 < K ? ke * 64 : K) - kb * 64, job)
  if constexpr (WIDE) {
    switch ((row1 - row0 + 31) >> 5) {   // valid 32-row blocks of the tile: at most four
      case 1: MOE_TILE_(1); break;
      case 2: MOE_TILE_(2); break;
      case 3: MOE_TILE_(3); break;
      default: MOE_TILE_(4); break;
    }
  } else {
    switch ((row1 - row0 + 31) >> 5) {   // valid 32-row blocks of the tile
      case 1: MOE_TILE_(1); break;
      case 2: MOE_TILE_(2); break;
      case 3: MOE_TILE_(3); break;
      case 4: MOE_TILE_(4); break;
      case 5: MOE_TILE_(5); break;
      case 6: MOE_TILE_(6); break;
      case 7: MOE_TILE_(7); break;
      default: MOE_TILE_(8); break;
    }
  }
#undef MOE_TILE_
}

// ----------------------------------------- MFMA GEMM, weight streaming (decode)
// Few rows per expert: the work is reading every weight once.  Tile = 32 rows x
// 64 weight rows (DUAL: 32 gate + the matching 32 up rows); the four wavefronts
// of a workgroup split K between them (wavefront w takes K slices w, w+4, ...,
// a slice being 128 bytes of every weight row: 64 bf16 or 128 e4m3 values), each
// with its own register-staged pipeline: no LDS, no barrier until the partial
// sums are added in a fixed order at the end.  Many small workgroups (n tiles of
// 32 / 64 columns) and two slices of loads in flight per wavefront keep all of
// HBM busy even when a single expert holds most rows; M tiles of one expert are
// neighbours in the grid, so its weights are read from HBM once.
// Inside a slice, MFMA sub-step kk of lane half h covers k = h*W/2 + kk*8 .. +8
// (W = slice width) for BOTH operands, so every lane reads one contiguous run.
template <bool DUAL, bool FP8>
__global__ __launch_bounds__(256) void ffn_skinny_kernel(
    const uint16_t* __restrict__ A, const void* __restrict__ B0, const void* __restrict__ B1,
    const float* __restrict__ S0, const float* __restrict__ S1, uint16_t* __restrict__ C, int N,
    int K, const int32_t* __restrict__ tiles) {
  constexpr int W = FP8 ? 128 : 64;          // K values per slice
  constexpr int NKK = W / 16;                // MFMA sub-steps per slice
  constexpr int BN = DUAL ? 32 : 64;         // output columns per workgroup
  constexpr int BL = FP8 ? NKK / 2 : NKK;    // 16-byte loads per lane, slice and weight block
  __shared__ float red[4][2][16][64];        // partial sums of the four wavefronts

  const int n_ntiles = (N + BN - 1) / BN;
  const int total = tiles[0] * n_ntiles;
  if (int(blockIdx.x) >= total) return;
  int mtile = blockIdx.x / n_ntiles;
  const int first = tiles[4 + kTileRec * mtile], cnt = tiles[5 + kTileRec * mtile];
  const int local = blockIdx.x - first * n_ntiles;      // inside the expert: M tile fastest
  const int ntile = local / cnt;
  mtile = first + (local - ntile * cnt);
  const int e = tiles[1 + kTileRec * mtile], row0 = tiles[2 + kTileRec * mtile],
            row1 = tiles[3 + kTileRec * mtile];
  const int n0 = ntile * BN;

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int h = lane >> 5;
  const size_t wb = FP8 ? 1 : 2;
  // this lane's rows: activation row, and the weight row of each of the two blocks.
  // Lanes past the tile's last row load nothing (their fragment stays zero and
  // their output rows are not stored): a short tile asks the memory pipeline for
  // its real rows only.
  int ar = row0 + (lane & 31);
  const bool a_valid = ar < row1;
  ar = a_valid ? ar : row1 - 1;
  const uint16_t* arow = A + size_t(ar) * K + h * (W / 2);
  const char* brow[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    int n = n0 + (DUAL ? 0 : j * 32) + (lane & 31);
    n = n < N ? n : N - 1;
    const char* base = static_cast<const char*>((DUAL && j == 1) ? B1 : B0) + size_t(e) * N * K * wb;
    brow[j] = base + (size_t(n) * K + h * (W / 2)) * wb;
  }

  f32x16 acc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[j][q] = 0.f;

  struct Slice { uint4 a[NKK]; uint4 b[2][BL]; };
  auto load = [&](int sl, Slice& r) {
    const int k0 = sl * W;
    if (!FP8 && k0 + W > K) {                // the last slice of a K that is no multiple of 64
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk) {
        const bool in = k0 + h * (W / 2) + kk * 8 < K;
        // (a value on the other side of the ?, not a variable: the choice of an address
        // would put that variable into scratch memory, and every load of the slice is flat)
        r.a[kk] = in && a_valid ? *reinterpret_cast<const uint4*>(arow + k0 + kk * 8) : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < 2; ++j)
          if (kk < BL)
            r.b[j][kk] = in ? *reinterpret_cast<const uint4*>(brow[j] + size_t(k0) * wb + kk * 16)
                            : make_uint4(0, 0, 0, 0);
      }
      return;
    }
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk)
      if (a_valid) r.a[kk] = *reinterpret_cast<const uint4*>(arow + k0 + kk * 8);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < BL; ++q)
        r.b[j][q] = *reinterpret_cast<const uint4*>(brow[j] + size_t(k0) * wb + q * 16);
  };
  auto compute = [&](int sl, const Slice& r) {
    if constexpr (FP8) {
      // one scale block along K per slice; the 32 columns lie inside one block
      const int nkb = (K + 127) / 128, nnb = (N + 127) / 128;
      f32x16 part[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
#pragma unroll
        for (int q = 0; q < 16; ++q) part[j][q] = 0.f;
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) {
          // eight codes of this sub-step -> eight bf16 (exact)
          const uint4 v = r.b[j][kk >> 1];
          const uint32_t c0 = (kk & 1) ? v.z : v.x, c1 = (kk & 1) ? v.w : v.y;
          const f32x2 p0 = __builtin_amdgcn_cvt_pk_f32_fp8(c0, false), p1 = __builtin_amdgcn_cvt_pk_f32_fp8(c0, true);
          const f32x2 p2 = __builtin_amdgcn_cvt_pk_f32_fp8(c1, false), p3 = __builtin_amdgcn_cvt_pk_f32_fp8(c1, true);
          // upper halves of the two floats side by side (the lower halves are zero:
          // an e4m3 value has three mantissa bits), one byte permute per pair
          auto pack = [](f32x2 p) {
            return __builtin_amdgcn_perm(__float_as_uint(p[1]), __float_as_uint(p[0]), 0x07060302u);
          };
          const uint4 w8 = make_uint4(pack(p0), pack(p1), pack(p2), pack(p3));
          part[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, r.a[kk]),
                                                            __builtin_bit_cast(bf16x8, w8), part[j], 0, 0, 0);
        }
        int n = n0 + (DUAL ? 0 : j * 32);
        n = n < N ? n : N - 1;
        const float* S = (DUAL && j == 1) ? S1 : S0;
        const float sc = S[(size_t(e) * nnb + n / 128) * nkb + sl];
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[j][q] = fmaf(sc, part[j][q], acc[j][q]);
      }
    } else {
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, r.a[kk]),
                                                           __builtin_bit_cast(bf16x8, r.b[j][kk]),
                                                           acc[j], 0, 0, 0);
    }
  };

  const int nslices = (K + W - 1) / W;
  Slice r0, r1;
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) r0.a[kk] = r1.a[kk] = make_uint4(0, 0, 0, 0);
  int sl = wave;
  if (sl < nslices) load(sl, r0);
  while (sl < nslices) {                     // two slices per trip: r0 and r1 alternate
    if (sl + 4 < nslices) load(sl + 4, r1);
    compute(sl, r0);
    sl += 4;
    if (sl >= nslices) break;
    if (sl + 4 < nslices) load(sl + 4, r0);
    compute(sl, r1);
    sl += 4;
  }

  // add the four partial sums in a fixed order: wavefront w finishes registers 4w..4w+3
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int q = 0; q < 16; ++q) red[wave][j][q][lane] = acc[j][q];
  __syncthreads();
#pragma unroll
  for (int qq = 0; qq < 4; ++qq) {
    const int q = wave * 4 + qq;
    float v[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
      v[j] = ((red[0][j][q][lane] + red[1][j][q][lane]) + red[2][j][q][lane]) + red[3][j][q][lane];
    // D layout: lane l, register q -> row (q/4)*8 + (l/32)*4 + q%4, col l%32
    const int row = row0 + (q >> 2) * 8 + (lane >> 5) * 4 + (q & 3);
    if (row >= row1) continue;
    if (DUAL) {
      const int col = n0 + (lane & 31);
      if (col < N) C[size_t(row) * N + col] = f32_to_bf16_bits(silu_mul(v[0], v[1]));
    } else {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int col = n0 + j * 32 + (lane & 31);
        if (col < N) C[size_t(row) * N + col] = f32_to_bf16_bits(v[j]);
      }
    }
  }
}

// -------------------------------------------------- MFMA GEMM-2, short K
// The down projection of a narrow TP slice (K = I_loc up to 128): a tile is a
// handful of K steps, so what counts is streaming w_down in and ys out without a
// gap, not the K loop.  A workgroup of four wavefronts takes 128 rows, keeps their
// activation fragments in registers (the whole K) and walks a run of 128-column
// blocks: the weights of the next block are in flight (global -> LDS, two stages)
// while the current block is multiplied and stored.  Small workgroups (52 KB of LDS
// at K = 96), so that three of them share a CU and fill each other's waits; the
// tall-tile kernel pays 6 us per tile beyond its K steps and has a CU to itself.
// The weights are the first MFMA operand, so a lane holds four neighbouring columns
// of one row, which go through LDS once more to be stored as whole 128-byte lines.
// LDS rows have an odd pitch in 16-byte pieces (the padding piece is loaded out of
// range: zeros), which keeps the operand reads free of bank conflicts.
// Bound by the output write and the weights at prefill sizes.  128 experts, hidden
// 2048, I_loc 96, against 128 x 128 tiles with register staging and 2-byte stores:
// 3001 tokens (24 008 rows: 98 MB out, 50 MB of weights, 30 us at the copy rate) 60 ->
// 34 us, 16 000 tokens (524 MB out) 254 -> 117 us; storing from the accumulators
// instead (16 bytes per lane, 32 contiguous bytes per row) took 39 / 187 us, two
// workgroups per CU instead of three 37 / 141 us.

template <int NKS>                                   // K sub-steps of 16: K <= 16 * NKS
__device__ __forceinline__ void shortk_body(const uint16_t* __restrict__ A,
                                            const uint16_t* __restrict__ Be,
                                            uint16_t* __restrict__ C, int N, int K, int row0,
                                            int row1, int nb0, int nb1, uint4* smem) {
  constexpr int P = ShortK<NKS>::kPieces;            // pieces per LDS row
  constexpr int kTurn = ShortK<NKS>::kTurn;          // slots in which a wavefront turns 32 x 64 outputs around
  constexpr int STAGE = ShortK<NKS>::kStage;         // 16-byte slots of a stage
  constexpr int NINST = ShortK<NKS>::kLoads, NLD = (NINST + 3) / 4;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = lane >> 5, l31 = lane & 31;
  const int wm = wave & 1, wn = wave >> 1;
  constexpr int kOut = kShortKOut;

  const int rows = row1 - row0;
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(A + size_t(row0) * K), 0, int(size_t(rows) * K * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
      C + size_t(row0) * N, 0, int(size_t(rows) * N * 2), 0x00020000);

  int boff[NLD];                                     // this lane's piece of load i, relative to the block
#pragma unroll
  for (int i = 0; i < NLD; ++i) boff[i] = shortk_slot_offset<NKS>((i * 4 + wave) * 64 + lane, K);
  // The block's place goes into the descriptor's base and its length is what the block
  // has of w_down, so that the lanes' own offsets decide what is read: a scalar offset
  // beside them need not count in the range check.
  auto issue = [&](int nb) {
    uint4* const st = smem + (nb & 1) * STAGE;
    const ShortKWindow win = shortk_window(nb, N, K);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(Be + win.first / 2), 0, win.bytes, 0x00020000);
#pragma unroll
    for (int i = 0; i < NLD; ++i)
      if (i * 4 + wave < NINST)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lptr_t)(st + (i * 4 + wave) * 64), 16, boff[i], 0, 0, 0);
  };
  issue(nb0);
  // activation fragments: rows wm*64 + i*32 + lane%32, k = kk*16 + h*8 .. +8
  bf16x8 af[2][NKS];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int kk = 0; kk < NKS; ++kk) {
      const int k = kk * 16 + h * 8;
      const int off = k < K ? ((wm * 64 + i * 32 + l31) * K + k) * 2 : kOut;
      af[i][kk] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(ra, off, 0, 0));
    }
  for (int nb = nb0; nb < nb1; ++nb) {
    // the weights of this block have landed; the eight stores of the block before
    // it are younger and may stay in flight
    if (nb == nb0) wait_vmcnt<0>(); else wait_vmcnt<8>();
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (nb + 1 < nb1) issue(nb + 1);                 // every wavefront is done with that stage
    const uint4* const st = smem + (nb & 1) * STAGE;
    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
#pragma unroll
    for (int kk = 0; kk < NKS; ++kk) {
      bf16x8 bf[2];
#pragma unroll
      for (int j = 0; j < 2; ++j)
        bf[j] = __builtin_bit_cast(bf16x8, st[(wn * 64 + j * 32 + l31) * P + kk * 2 + h]);
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[j], af[i][kk], acc[i][j], 0, 0, 0);
    }
    // Lane l holds row l%32 of block i, columns (q/4)*8 + (l/32)*4 + q%4 of block j.
    // The stage has served its purpose: each wavefront turns its 32-row halves
    // around in a slice of it, so that a store writes whole 128-byte lines.
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    uint4* const turn = smem + (nb & 1) * STAGE + wave * kTurn;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const uint2 v = make_uint2(pack_bf16(acc[i][j][g * 4], acc[i][j][g * 4 + 1]),
                                     pack_bf16(acc[i][j][g * 4 + 2], acc[i][j][g * 4 + 3]));
          reinterpret_cast<uint2*>(turn + l31 * 9 + j * 4 + g)[h] = v;
        }
      asm volatile("" ::: "memory");                 // the reads below see the writes above (same wavefront)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int row = t * 8 + (lane >> 3), piece = lane & 7;
        const u32x4 v = __builtin_bit_cast(u32x4, turn[row * 9 + piece]);
        const int col = nb * 128 + wn * 64 + piece * 8;
        const int off = col < N ? ((wm * 64 + i * 32 + row) * N + col) * 2 : kOut;
        __builtin_amdgcn_raw_buffer_store_b128(v, rc, off, 0, 0);
      }
      asm volatile("" ::: "memory");
    }
  }
}

// `split` workgroups share an M tile's column blocks.  Inside an expert the M
// tiles are neighbours (they stream the same weights), and every XCD walks a
// contiguous run of workgroups.
template <int NKS>
__global__ __launch_bounds__(256, NKS <= 6 ? 3 : 2) void ffn_shortk_kernel(const uint16_t* __restrict__ A,
                                                        const uint16_t* __restrict__ B,
                                                        uint16_t* __restrict__ C, int N, int K,
                                                        const int32_t* __restrict__ tiles, int split) {
  extern __shared__ uint4 smem[];
  const int total = tiles[0] * split, per_xcd = (total + 7) >> 3;
  const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (int(blockIdx.x >> 3) >= per_xcd || logical >= total) return;
  const int at = logical / split;                    // a tile of the same expert
  const int first = tiles[4 + kTileRec * at], cnt = tiles[5 + kTileRec * at];
  const int local = logical - first * split, part = local / cnt, mtile = first + local - part * cnt;
  const int e = tiles[1 + kTileRec * mtile], row0 = tiles[2 + kTileRec * mtile],
            row1 = tiles[3 + kTileRec * mtile];
  const int blocks = (N + 127) / 128;
  const int nb0 = part * blocks / split, nb1 = (part + 1) * blocks / split;
  if (nb0 >= nb1) return;
  shortk_body<NKS>(A, B + size_t(e) * N * K, C, N, K, row0, row1, nb0, nb1, smem);
}

void launch_shortk(const void* hmid, const void* w_down, void* ys, int N, int K, const int32_t* tiles,
                   int max_mt, hipStream_t s) {
  // about four rounds of three workgroups per CU, each with at least four column
  // blocks to overlap, unless that leaves CUs without a workgroup (decode sizes); with
  // one block each there is nothing to overlap, so not where the halves of a launch that
  // nearly fills the chip would come to a second round (8 experts, hidden 7168, I_loc 64, 144
  // rows each: 952 workgroups 12.1 us, 476 10.8)
  const int blocks = (N + 127) / 128;
  int most = (blocks + 3) / 4;
  while (most < blocks && long(max_mt) * most < 2 * kCUs) {
    const int twice = 2 * most < blocks ? 2 * most : blocks;
    if (2L * max_mt * twice > 7 * kCUs) break;
    most = twice;
  }
  int split = (12 * kCUs + max_mt - 1) / max_mt;
  split = split < most ? split : most;
  const int grid = (max_mt * split + 7) / 8 * 8;
#define MOE_SHORTK(NKS)                                                                            \
  do {                                                                                             \
    constexpr int lds = 2 * ShortK<NKS>::kStage * 16;                                              \
    static uint64_t opted = 0;                                                                     \
    auto k = ffn_shortk_kernel<NKS>;                                                               \
    lds_opt_in(reinterpret_cast<const void*>(k), lds, opted);                                      \
    MOE_LAUNCH(MOE_K_FFN_GEMM2, k, dim3(grid), dim3(256), lds, s, static_cast<const uint16_t*>(hmid), \
               static_cast<const uint16_t*>(w_down), static_cast<uint16_t*>(ys), N, K, tiles, split);   \
  } while (0)
  const int ks = (K + 15) / 16;
  if (ks <= 2) MOE_SHORTK(2);
  else if (ks <= 4) MOE_SHORTK(4);
  else if (ks <= 6) MOE_SHORTK(6);
  else MOE_SHORTK(8);
#undef MOE_SHORTK
}

// ------------------------------------------------------------ fp32 GEMM
// fp32 layers on v_mfma_f32_32x32x2_f32 (fp32 products and sums).  Tile 32 rows x
// 32 output columns (DUAL: with the matching up rows).  Operands go global -> LDS
// directly in chunks of 128 K values (512-byte rows: whole cache lines) into a
// ring of as many chunks as 144 KB hold (launches of more tiles than CUs: one chunk, see
// F32Ring::stages); the four wavefronts each multiply a quarter of every chunk and their
// sums are added in a fixed order at the end.
// These layers are small (64 tokens, hidden 256, 8 experts, I 512), so a launch is
// one workgroup's latency chain: small tiles put it on as many CUs as there are,
// the K split makes the arithmetic a quarter as long, and a short K is in flight
// as a whole before the first wait.  The fp32 matrix rate (128 multiply-adds per
// cycle and CU) needs 24 bytes per cycle even with this small tile, so long
// launches are not bound by the loads either.
// Measured against 64 x 64 tiles of VALU arithmetic (64-token layer, GEMM-1 / -2):
// 30.2 / 30.6 -> 7.0 / 5.9 us; 8 experts of 256 rows, hidden = I = 512: 72 / 43 -> 35 / 21 us;
// 8192 rows, hidden 2048, I 1024: 914 / 497 -> 629 / 339 us (109 TFLOP/s).  The same tile
// without LDS (lanes reading 16 bytes of 32 rows each) was slower: 13 / 15 us on the small
// layer, 2033 / 1447 us on the large one.
// LDS row r keeps its 16-byte piece p at slot p ^ (r & 15).
constexpr int kF32Chunk = 128;                        // K values per chunk
template <bool DUAL> struct F32Ring {
  static constexpr int kRows = DUAL ? 96 : 64;        // activation rows | weight rows
  static constexpr int kSlots = kRows * (kF32Chunk / 4);
  static constexpr int kStages = DUAL ? 3 : 4;        // 144 KB / 128 KB
  static constexpr int kStageBytes = kSlots * 16;
  static constexpr int kLds = kStages * kStageBytes;
  // Stages of a launch of at most `tiles` tiles: as many as K has chunks and the ring holds
  // while every tile has a CU to itself, else one, so that three (DUAL) or five workgroups
  // share a CU and load while others multiply.  8192 rows, hidden = I = 512, GEMM-1 / -2: 75 / 47 ->
  // 60 / 37 us; 1056 tiles, hidden = I = 256: 29 -> 22; below 256 tiles 7.8 against 8.5 us (K = 512).
  static int stages(int K, long tiles) {
    const int chunks = (K + kF32Chunk - 1) / kF32Chunk;
    const int most = tiles > kCUs ? 1 : kStages;
    return chunks < most ? chunks : most;
  }
};

template <bool DUAL>
__device__ __forceinline__ void ffn_f32_body(const float* __restrict__ A,
                                             const float* __restrict__ Be0,
                                             const float* __restrict__ Be1, float* __restrict__ C,
                                             int N, int K, int row0, int row1, int n0, int stages,
                                             uint4* smem) {
  constexpr int NB = DUAL ? 2 : 1, NS = F32Ring<DUAL>::kStages, SLOTS = F32Ring<DUAL>::kSlots;
  constexpr int NLD = F32Ring<DUAL>::kRows / 8;       // load instructions per wavefront and chunk
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = lane >> 5, l31 = lane & 31;
  const int brows = N - n0 < 32 ? N - n0 : 32;
  auto rsrc = [&](const float* p, int rows) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, int(size_t(rows) * K * 4), 0x00020000);
  };
  const __amdgpu_buffer_rsrc_t ra = rsrc(A + size_t(row0) * K, row1 - row0);
  const __amdgpu_buffer_rsrc_t rb0 = rsrc(Be0 + size_t(n0) * K, brows);
  const __amdgpu_buffer_rsrc_t rb1 = rsrc((DUAL ? Be1 : Be0) + size_t(n0) * K, brows);
  // One instruction fills two LDS rows; instruction i of wavefront w: rows
  // (i*4 + w)*2 + lane/32, the lane that owns slot s of row r fetches piece s ^ (r&15).
  // Rows past the tile (or past N) and pieces past K are out of range: zeros.
  auto issue = [&](int c, int stage) {
    uint4* const st = smem + stage * SLOTS;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int pair = i * 4 + wave, row = pair * 2 + h, local = row & 31;
      const int k = c * kF32Chunk + ((l31 ^ (row & 15)) * 4);
      const int off = k < K ? (local * K + k) * 4 : 0x7fffffff;
      lptr_t const dst = (lptr_t)(st + pair * 64);
      if (i < 4) __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, dst, 16, off, 0, 0, 0);
      else if (i < 8) __builtin_amdgcn_raw_ptr_buffer_load_lds(rb0, dst, 16, off, 0, 0, 0);
      else __builtin_amdgcn_raw_ptr_buffer_load_lds(rb1, dst, 16, off, 0, 0, 0);
    }
  };
  f32x16 acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[j][q] = 0.f;
  const int nch = (K + kF32Chunk - 1) / kF32Chunk;
#pragma unroll
  for (int c = 0; c < NS; ++c)
    if (c < stages) issue(c, c);                     // stages <= nch
  int stage = 0;                                     // of chunk c
  for (int c = 0; c < nch; ++c) {
    // chunk c must have landed; up to stages-1 younger ones stay in flight
    const int younger = nch - 1 - c < stages - 1 ? nch - 1 - c : stages - 1;
    if (NS > 3 && younger == 3) wait_vmcnt<3 * NLD>();
    else if (younger == 2) wait_vmcnt<2 * NLD>();
    else if (younger == 1) wait_vmcnt<NLD>();
    else wait_vmcnt<0>();
    asm volatile("s_barrier" ::: "memory");
    const uint4* const st = smem + stage * SLOTS;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      // MFMA i of lane half h multiplies element i of the same piece of both operands
      const int p = (wave * 8 + h * 4 + q) ^ (l31 & 15);
      const float4 a = __builtin_bit_cast(float4, st[l31 * 32 + p]);
      float4 b[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) b[j] = __builtin_bit_cast(float4, st[((j + 1) * 32 + l31) * 32 + p]);
      const float av[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          const float bv[4] = {b[j].x, b[j].y, b[j].z, b[j].w};
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], bv[i], acc[j], 0, 0, 0);
        }
    }
    if (c + stages < nch) {
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the stage has been read by all
      issue(c + stages, stage);
    }
    stage = stage + 1 < stages ? stage + 1 : 0;
  }
  // add the four partial sums in a fixed order: wavefront w finishes registers 4w..4w+3
  __syncthreads();
  float* const red = reinterpret_cast<float*>(smem);   // [4][NB][16][64]
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int q = 0; q < 16; ++q) red[((wave * NB + j) * 16 + q) * 64 + lane] = acc[j][q];
  __syncthreads();
#pragma unroll
  for (int qq = 0; qq < 4; ++qq) {
    const int q = wave * 4 + qq;
    float v[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      auto part = [&](int w) { return red[((w * NB + j) * 16 + q) * 64 + lane]; };
      v[j] = ((part(0) + part(1)) + part(2)) + part(3);
    }
    // D layout: lane l, register q -> row (q/4)*8 + (l/32)*4 + q%4, col l%32
    const int row = row0 + (q >> 2) * 8 + h * 4 + (q & 3), col = n0 + l31;
    if (row >= row1 || col >= N) continue;
    if constexpr (DUAL) v[0] = v[0] / (1.0f + expf(-v[0])) * v[NB - 1];
    C[size_t(row) * N + col] = v[0];
  }
}

template <bool DUAL>
__global__ __launch_bounds__(256) void ffn_f32_kernel(const float* __restrict__ A,
                                                     const float* __restrict__ B0,
                                                     const float* __restrict__ B1,
                                                     float* __restrict__ C, int N, int K,
                                                     const int32_t* __restrict__ tiles, int stages,
                                                     int grid_row) {
  extern __shared__ uint4 smem[];
  const int n_ntiles = (N + 31) / 32, block = grid_block(grid_row);
  const int mtile = block / n_ntiles, ntile = block - mtile * n_ntiles;
  if (mtile >= tiles[0]) return;
  const int e = tiles[1 + kTileRec * mtile], row0 = tiles[2 + kTileRec * mtile],
            row1 = tiles[3 + kTileRec * mtile];
  ffn_f32_body<DUAL>(A, B0 + size_t(e) * N * K, DUAL ? B1 + size_t(e) * N * K : nullptr, C, N, K,
                     row0, row1, ntile * 32, stages, smem);
}

// fp32, K up to 64 and many tiles: 64 x 64 tile of VALU arithmetic, 16x16 threads, 4x4 outputs per
// thread, K step 32; the next step's operands are fetched into registers while the
// current step is computed from LDS.  A tile of the kernel above is there a single chunk
// that is half empty, so its loads, barriers and sums cost more than its arithmetic.
template <bool DUAL>
__global__ __launch_bounds__(256) void ffn_f32_valu_kernel(const float* __restrict__ A,
                                                          const float* __restrict__ B0,
                                                          const float* __restrict__ B1,
                                                          float* __restrict__ C, int N, int K,
                                                          const int32_t* __restrict__ tiles) {
  constexpr int TB = 64, TK = 32, PER = TB * TK / 256;
  __shared__ __align__(16) float As[TK][TB + 4];
  __shared__ __align__(16) float Bg[TK][TB + 4];
  __shared__ __align__(16) float Bu[DUAL ? TK : 1][TB + 4];
  const int n_ntiles = (N + TB - 1) / TB;
  const int mtile = blockIdx.x / n_ntiles, ntile = blockIdx.x % n_ntiles;
  if (mtile >= tiles[0]) return;
  const int e = tiles[1 + kTileRec * mtile], row0 = tiles[2 + kTileRec * mtile],
            row1 = tiles[3 + kTileRec * mtile];
  const int n0 = ntile * TB;
  const float* Be0 = B0 + size_t(e) * N * K;
  const float* Be1 = DUAL ? B1 + size_t(e) * N * K : nullptr;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  float g[4][4] = {}, u[4][4] = {};
  float ra[PER], rg[PER], ru[PER];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int idx = threadIdx.x + i * 256;
      const int r = idx / TK, k = k0 + idx % TK;
      int ar = row0 + r; ar = ar < row1 ? ar : row1 - 1;
      int bn = n0 + r;   bn = bn < N ? bn : N - 1;
      ra[i] = k < K ? A[size_t(ar) * K + k] : 0.f;
      rg[i] = k < K ? Be0[size_t(bn) * K + k] : 0.f;
      if (DUAL) ru[i] = k < K ? Be1[size_t(bn) * K + k] : 0.f;
    }
  };
  fetch(0);
  for (int k0 = 0; k0 < K; k0 += TK) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int idx = threadIdx.x + i * 256;
      const int r = idx / TK, kk = idx % TK;
      As[kk][r] = ra[i];
      Bg[kk][r] = rg[i];
      if (DUAL) Bu[kk][r] = ru[i];
    }
    __syncthreads();
    if (k0 + TK < K) fetch(k0 + TK);
#pragma unroll
    for (int kk = 0; kk < TK; ++kk) {
      // rows of the LDS tiles are 68 floats, so groups of four stay 16-byte aligned
      const float4 a4 = *reinterpret_cast<const float4*>(&As[kk][ty * 4]);
      const float4 g4 = *reinterpret_cast<const float4*>(&Bg[kk][tx * 4]);
      const float4 u4 = DUAL ? *reinterpret_cast<const float4*>(&Bu[kk][tx * 4]) : make_float4(0.f, 0.f, 0.f, 0.f);
      const float a[4] = {a4.x, a4.y, a4.z, a4.w}, bg[4] = {g4.x, g4.y, g4.z, g4.w},
                  bu[4] = {u4.x, u4.y, u4.z, u4.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          g[i][j] = fmaf(a[i], bg[j], g[i][j]);
          if (DUAL) u[i][j] = fmaf(a[i], bu[j], u[i][j]);
        }
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = row0 + ty * 4 + i, col = n0 + tx * 4 + j;
      if (row < row1 && col < N) {
        float v = g[i][j];
        if (DUAL) v = v / (1.0f + expf(-v)) * u[i][j];
        C[size_t(row) * N + col] = v;
      }
    }
}

// Which kernel runs each GEMM of a call, and the height of its M tiles.
enum GemmKind { kGemmF32, kGemmF32Valu, kGemmStream, kGemmTall, kGemmWide, kGemmShortK };
struct FfnPlan {
  GemmKind g1, g2;
  int bm1, bm2;
};

// Rows per expert can only be bounded from above on the host; the kernels are
// picked by that bound (`avg`).  Tile counts are bounds too.
FfnPlan plan_ffn(const moe_config& c, int n_experts, int rows_capacity) {
  const int H = c.hidden, I = c.inter_local, avg = rows_capacity / n_experts;
  const bool fp8 = c.weight_dtype == MOE_FP8_E4M3_B128;
  const bool ragged = ((H | I) & 63) != 0;
  const int groups = n_experts < rows_capacity ? n_experts : rows_capacity;
  auto tiles_of = [&](int bm, int cols, int bn) {
    return long(rows_capacity / bm + groups) * ((cols + bn - 1) / bn);
  };
  FfnPlan p;
  if (c.act_dtype == MOE_F32) {
    // 32 x 32 tiles of fp32 matrix instructions, except a K up to 64 in launches of many of them.
    // hidden = I = 64: GEMM-1 of 32 768 rows (2112 tiles) 24 -> 21 us, 15 / 16 at 1056; hidden 1024, I 64:
    // GEMM-2 of 8192 rows (32 experts of 256, 9216 tiles) 39 -> 30, 2304 tiles 14.2 / 14.1.
    p = {kGemmF32, kGemmF32, 32, 32};
    if (H <= 64 && tiles_of(32, I, 32) > 6 * kCUs) { p.g1 = kGemmF32Valu; p.bm1 = 64; }
    if (I <= 64 && tiles_of(32, H, 32) >= 16 * kCUs) { p.g2 = kGemmF32Valu; p.bm2 = 64; }
    return p;
  }
  // GEMM-1 (K = H long): the weight-streaming kernel at decode sizes, then the LDS
  // rings of the tall-tile kernel, which stream the weights faster as soon as a tile
  // holds a few rows: measured on the 128-expert layer (hidden 2048, I 768) with the
  // switch at two rows per expert.  e4m3 weights switch at twelve: up to there the
  // block scale multiplies fp32 partial sums, above it code * scale is rounded to bf16.
  p.g1 = avg <= (fp8 ? 12 : 2) ? kGemmStream : kGemmTall;
  // Few rows per expert mean that the weights are streamed about once: tiles of at
  // most 160 rows there, which leaves room for a three-stage ring.
  p.bm1 = p.g1 == kGemmStream ? 32 : (avg <= 320 ? 160 : 256);
  // Sizes that are no multiple of 64 (I: a cut that is not even, 1408 / 8) differ in two things:
  //  - 160-row tiles also for long groups while they fit one round of the CUs, where a tall
  //    tile's length is the launch's: one group of 512 / 1024 rows, hidden 2048, I 200: 37 -> 28 /
  //    37 -> 33 us; 16 groups of 512: 39 -> 35; 320 tiles (128 experts, I 344): no gain.
  //  - the weight-streaming kernel up to 16 rows per expert where one tall tile per expert and
  //    128 columns would leave a second round of CUs less than half full: 64 experts, hidden 520,
  //    I 520 (320 tiles), 3 / 16 rows per expert: 22.4 -> 18.1 / 22.8 -> 20.9 us, 128 experts,
  //    hidden 2048, I 344 (384 tiles): 85 -> 68 / 91 -> 76; one whole round (128 experts, hidden 520,
  //    I 136) 12.6 against 13.7 us.
  const long tall = tiles_of(160, I, 128), first = long(groups) * ((I + 127) / 128);
  if (ragged && avg > 2 && avg <= 16 && first > kCUs && 2 * first <= 3 * kCUs) { p.g1 = kGemmStream; p.bm1 = 32; }
  if (ragged && p.bm1 == 256 && tall <= kCUs) p.bm1 = 160;
  // GEMM-2 (K = I_loc short, N = H wide):
  //  - K up to 128 (a layer cut over many TP ranks): the short-K kernel.
  //    128 experts, hidden 2048, I_loc 96: 13 / 14 us at 2 / 6 rows per expert, where the
  //    weight-streaming kernel (a K slice each for two of its wavefronts) takes 23 / 27 us; at K =
  //    192 the tall-tile kernel is the faster one (188 rows per expert: 49 against 54 us).
  //    At K = 128, where two of its workgroups share a CU and not three and the others have whole
  //    steps, only launches of many 128 x 128 blocks: 32 experts, hidden 2048, 112 rows each (960
  //    blocks) 16 against 13 us for the tall tiles, 8 experts, hidden 7168, 144 rows (952) 17
  //    against 12, 64 experts, hidden 2048, 16 rows (1152) 12.6 against 11.0 for the wide ones;
  //    32 experts, hidden 7168, 64 rows (2688) 20 against 24; against the weight-streaming
  //    kernel 16 experts, hidden 7168, one row (896) 10.5 / 9.7, 128 experts, hidden 2048, 4 rows
  //    (2112) 17 / 25 us.
  //  - up to twelve rows per expert: many small weight-streaming workgroups.
  //  - up to 96 rows per expert, when the experts give at least one such tile per CU:
  //    tiles of 128 rows x 512 weight rows.  128 experts, hidden 2048, I 768, bf16: 85 ->
  //    81, 94 -> 86, 102 -> 92 us at 32 / 64 / 96 rows per expert, 110 -> 115 us at 128;
  //    e4m3 weights at 64 rows per expert (32 experts, hidden 7168): 73 -> 61 us.
  //    (GEMM-1 keeps the narrow tiles: its wide form was slower at every size, the
  //    512-row bf16 stage leaves room for two ring stages only.)  For sizes that are no
  //    multiple of 64 from three rows per expert on if K is short, up to 384 (128 experts, hidden
  //    2048, I 200: 36 -> 31 us at twelve rows, I 344: 52 -> 50, 64 experts, I 1000: 55 against 58 at
  //    three), in the short-K kernel's place up to 16 rows if K is at most 48 (64 experts, I 40:
  //    8.5 -> 7.2 us), and not where most columns of the last tile are missing and the tiles are
  //    more than a round (hidden 1032, I 520, 128 experts: 53 against 45 us at 16 rows).
  //  - 128-row tiles for sizes that are no multiple of 64, long groups and no more tiles than CUs
  //    (one group of 256 / 1024 rows, hidden 2048, I 200: 13.5 -> 10.4 / 14 -> 10.8 us).
  //  - else 256-row tiles.
  const long blocks = tiles_of(128, H, 128);
  const bool short_k = ragged || I < kShortKMax || (avg <= 12 ? blocks > 1024 : blocks >= 2048);
  const long wide_tiles = long(n_experts) * ((H + 511) / 512);
  const bool wide = wide_tiles >= kCUs &&
                    (!ragged || wide_tiles <= kCUs || (H + 511) / 512 * 512 * 4L <= 5L * H);
  if (ragged && wide && (I <= 48 ? avg <= 16 : I > kShortKMax && I <= 384 && avg > 2 && avg <= 12)) {
    p.g2 = kGemmWide;
    p.bm2 = 128;
  } else if (!fp8 && I <= kShortKMax && short_k) { p.g2 = kGemmShortK; p.bm2 = 128; }
  else if (avg <= 12) { p.g2 = kGemmStream; p.bm2 = 32; }
  else if (avg <= 96 && wide) { p.g2 = kGemmWide; p.bm2 = 128; }
  else { p.g2 = kGemmTall; p.bm2 = ragged && avg >= 128 && tiles_of(128, H, 256) <= kCUs ? 128 : 256; }
  return p;
}

// The choice of tiles that the GEMM of `kind` has (e4m3 weights).
template <bool DUAL>
ShortTiles short_tiles_of(GemmKind kind, int bm, int N, int K, int n_experts, int rows_capacity) {
  if (kind != kGemmTall && kind != kGemmWide) return {};
  const bool wide = kind == kGemmWide;
  const int bn = DUAL ? 128 : 256, own = wide ? 512 : bn;
  const int nt_own = (N + own - 1) / own;
  return {(N + bn - 1) / bn, nt_own, (K + 63) / 64 / kSplitMinSteps,
          tall_grid(max_row_tiles(rows_capacity, n_experts, bm), nt_own, wide), DUAL, wide};
}

// One GEMM of the call: C[rows, N] = A[rows, K] B^T (DUAL: the gate|up pair with SwiGLU).
template <bool DUAL, bool F8>
void launch_gemm(GemmKind kind, int bm, const uint16_t* A, const void* B0, const void* B1,
                 const float* S0, const float* S1, uint16_t* C, int N, int K, int n_experts,
                 int rows_capacity, const int32_t* tiles, const FfnWs& ws, hipStream_t s) {
  constexpr int id = DUAL ? MOE_K_FFN_GEMM1 : MOE_K_FFN_GEMM2;
  const int max_mt = max_row_tiles(rows_capacity, n_experts, bm);
  if (kind == kGemmStream) {
    constexpr int BN = DUAL ? 32 : 64;
    MOE_LAUNCH(id, (ffn_skinny_kernel<DUAL, F8>), dim3(size_t(max_mt) * ((N + BN - 1) / BN)), dim3(256),
               0, s, A, B0, B1, S0, S1, C, N, K, tiles);
    return;
  }
  if (!DUAL && !F8 && kind == kGemmShortK) {
    launch_shortk(A, B0, C, N, K, tiles, max_mt, s);
    return;
  }
  constexpr int lds = 160 * 1024;         // all of a CU's LDS: the rings of the tallest tile fill it
  const bool wide = !DUAL && kind == kGemmWide;
  const int BN = DUAL ? 128 : (wide ? 512 : 256);
  const int grid = tall_grid(max_mt, (N + BN - 1) / BN, F8 && wide);
  auto k = ffn_gemm8w_kernel<DUAL, F8, false, false>;
  int form = 0;
  if constexpr (!F8) {
    if (((N | K) & 63) != 0) { k = ffn_gemm8w_kernel<DUAL, F8, true, false>; form = 1; }
  }
  if constexpr (!DUAL) {
    if (wide) { k = ffn_gemm8w_kernel<DUAL, F8, false, true>; form = 2; }
    if constexpr (!F8) {
      if (wide && ((N | K) & 63) != 0) { k = ffn_gemm8w_kernel<DUAL, F8, true, true>; form = 3; }
    }
  }
  static uint64_t opted[4] = {};
  lds_opt_in(reinterpret_cast<const void*>(k), lds, opted[form]);
  MOE_LAUNCH(id, k, dim3(grid), dim3(512), lds, s, A, B0, B1, S0, S1, C, N, K, tiles, 1, ws.partial,
             ws.tickets + (DUAL ? 0 : kSplitTickets));
}

template <bool DUAL>
void launch_f32(GemmKind kind, int bm, const float* A, const float* B0, const float* B1, float* C, int N,
                int K, int n_experts, int rows_capacity, const int32_t* tiles, hipStream_t s) {
  constexpr int id = DUAL ? MOE_K_FFN_GEMM1 : MOE_K_FFN_GEMM2;
  const int bn = kind == kGemmF32Valu ? 64 : 32;
  const int max_mt = rows_capacity / bm + (n_experts < rows_capacity ? n_experts : rows_capacity);
  const size_t blocks = size_t(max_mt) * ((N + bn - 1) / bn);
  if (kind == kGemmF32Valu) {
    MOE_LAUNCH(id, ffn_f32_valu_kernel<DUAL>, dim3(blocks), dim3(256), 0, s, A, B0, B1, C, N, K, tiles);
    return;
  }
  auto k = ffn_f32_kernel<DUAL>;
  static uint64_t opted = 0;
  lds_opt_in(reinterpret_cast<const void*>(k), F32Ring<DUAL>::kLds, opted);
  const int stages = F32Ring<DUAL>::stages(K, long(blocks));
  const dim3 grid = grid_of(blocks, 256);
  MOE_LAUNCH(id, k, grid, dim3(256), stages * F32Ring<DUAL>::kStageBytes, s, A, B0, B1, C, N, K, tiles, stages,
             int(grid.x));
}

template <bool F8>
void launch_pair(const FfnPlan& p, const moe_config& c, int n_experts, const void* xs,
                 int rows_capacity, const void* w_gate, const void* w_up, const void* w_down,
                 const float* s_gate, const float* s_up, const float* s_down, void* ys,
                 const int32_t* tiles2, const FfnWs& ws, hipStream_t s) {
  const int H = c.hidden, I = c.inter_local;
  uint16_t* const hmid = static_cast<uint16_t*>(ws.hmid);
  launch_gemm<true, F8>(p.g1, p.bm1, static_cast<const uint16_t*>(xs), w_gate, w_up, s_gate, s_up, hmid,
                        I, H, n_experts, rows_capacity, ws.tiles, ws, s);
  launch_gemm<false, F8>(p.g2, p.bm2, hmid, w_down, nullptr, s_down, nullptr,
                         static_cast<uint16_t*>(ys), H, I, n_experts, rows_capacity, tiles2, ws, s);
}

}  // namespace

hipError_t launch_expert_ffn(const moe_config& c, int n_experts, const void* xs,
                             const int32_t* offsets, int rows_capacity, const void* w_gate,
                             const void* w_up, const void* w_down, const float* s_gate,
                             const float* s_up, const float* s_down, void* ys, const FfnWs& ws,
                             hipStream_t s) {
  const int H = c.hidden, I = c.inter_local;
  const FfnPlan p = plan_ffn(c, n_experts, rows_capacity);
  // when the two GEMMs may cut the rows differently a second workgroup builds a second table
  TileJob t1{ws.tiles, p.bm1, {}}, t2{ws.tiles2, p.bm2, {}};
  if (c.weight_dtype == MOE_FP8_E4M3_B128) {
    t1.alt = short_tiles_of<true>(p.g1, p.bm1, I, H, n_experts, rows_capacity);
    if (n_experts > 1) t2.alt = short_tiles_of<false>(p.g2, p.bm2, H, I, n_experts, rows_capacity);
  }
  const bool one_table = p.bm1 == p.bm2 && !t1.alt.nt && !t2.alt.nt;
  int32_t* const tiles2 = one_table ? ws.tiles : ws.tiles2;
  MOE_LAUNCH(MOE_K_FFN_TILES, (t1.alt.nt || t2.alt.nt ? ffn_tiles_kernel<true> : ffn_tiles_kernel<false>),
             dim3(one_table ? 1 : 2), dim3(kTileThreads), 0, s, offsets, n_experts, rows_capacity, ws.max_tiles, t1, t2,
             ws.tickets);
  if (c.act_dtype == MOE_F32) {
    float* const hmid = static_cast<float*>(ws.hmid);
    launch_f32<true>(p.g1, p.bm1, static_cast<const float*>(xs), static_cast<const float*>(w_gate),
                     static_cast<const float*>(w_up), hmid, I, H, n_experts, rows_capacity, ws.tiles, s);
    launch_f32<false>(p.g2, p.bm2, hmid, static_cast<const float*>(w_down), nullptr,
                      static_cast<float*>(ys), H, I, n_experts, rows_capacity, tiles2, s);
  } else if (c.weight_dtype == MOE_FP8_E4M3_B128) {
    launch_pair<true>(p, c, n_experts, xs, rows_capacity, w_gate, w_up, w_down, s_gate, s_up, s_down, ys,
                      tiles2, ws, s);
  } else {
    launch_pair<false>(p, c, n_experts, xs, rows_capacity, w_gate, w_up, w_down, nullptr, nullptr, nullptr,
                       ys, tiles2, ws, s);
  }
  return hipGetLastError();
}

}  // namespace moe

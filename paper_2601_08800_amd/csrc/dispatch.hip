// Dispatch: build the expert-contiguous send buffer (Sec. II "EP"; Alg. 2).
//
// A stable counting sort of the local assignments by expert (the permutation is
// unique and repeatable):
//   1. count   per chunk of assignments the count of every local expert and every
//              assignment's rank among its expert's assignments of the chunk
//   2. place   counts, offsets = exclusive scan over experts (rebuilt by every
//              workgroup from the chunks' counts); position = offsets[e] + count in
//              the chunks before + rank
//   3. gather  one wavefront per token reads the row ONCE (16 B per lane,
//              coalesced) and writes it to each of its local positions
#include "moe_internal.h"

namespace moe {

namespace {

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
// streaming (non-temporal) 16-byte accesses: data that is touched once
__device__ __forceinline__ uint4 nt_load16(const void* p) {
  const u32x4_t v = __builtin_nontemporal_load(static_cast<const u32x4_t*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void nt_store16(void* p, uint4 v) {
  u32x4_t t = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(t, static_cast<u32x4_t*>(p));
}

constexpr int kSub = 64;   // assignments per count of the one-launch form: one wavefront

__device__ __forceinline__ uint64_t lanemask_lt() {
  return (uint64_t(1) << (threadIdx.x & 63)) - 1;
}

// Lanes of the wavefront that hold the same local expert as this lane: one
// ballot per bit of the expert index (at most 9), each narrowing the set to the
// lanes that agree with this lane on that bit.  Meaningful where e >= 0.
__device__ __forceinline__ uint64_t same_expert_lanes(int e, int E_loc) {
  uint64_t same = __ballot(e >= 0);
  const int nbits = E_loc > 1 ? 32 - __clz(E_loc - 1) : 0;
  for (int b = 0; b < nbits; ++b) {
    const bool bit = (e >> b) & 1;
    const uint64_t m = __ballot(bit);
    same &= bit ? m : ~m;
  }
  return same;
}

// The index, in two launches over chunks of whole runs of 1024 assignments (a
// workgroup of sixteen wavefronts, one per 64 assignments of the run).
//
// count: the lanes of a wavefront that go to the same local expert find each other with
// ballots; one thread per expert then orders the wavefronts, which yields, without
// atomics, the rank of every assignment among its expert's assignments of the chunk
// (parked in inv[]) and the chunk's count per expert (hist[chunk][E_loc]).
constexpr int kRun = 1024;
constexpr int kIndexWgs = 256;                 // chunks at most (longer ones instead)
inline int index_chunk(int A) { return ((A + kIndexWgs - 1) / kIndexWgs + kRun - 1) / kRun * kRun; }

__global__ __launch_bounds__(kRun) void dispatch_count_kernel(
    const int32_t* __restrict__ ids, int A, int e_lo, int E_loc, int chunk,
    int32_t* __restrict__ hist, int32_t* __restrict__ inv) {
  extern __shared__ int32_t cnt[];             // [16][E_loc]
  const int tid = threadIdx.x, wave = tid >> 6;
  const int a0 = blockIdx.x * chunk, a1 = min(A - a0, chunk) + a0;
  int at = 0;                                  // thread e: assignments of expert e so far
  for (int p = a0; p < a1; p += kRun) {
    for (int i = tid; i < 16 * E_loc; i += kRun) cnt[i] = 0;
    const int a = p + tid;
    int e = -1;
    if (a < a1) {
      e = ids[a] - e_lo;
      if (e < 0 || e >= E_loc) e = -1;
    }
    const uint64_t same = same_expert_lanes(e, E_loc);
    const int rank = __popcll(same & lanemask_lt());
    __syncthreads();
    if (e >= 0 && rank == 0) cnt[wave * E_loc + e] = __popcll(same);   // the lowest lane of each expert present
    __syncthreads();
    if (tid < E_loc) {                         // E_loc <= 512
#pragma unroll
      for (int w = 0; w < 16; ++w) {
        const int n = cnt[w * E_loc + tid];
        cnt[w * E_loc + tid] = at;
        at += n;
      }
    }
    __syncthreads();
    if (a < a1) inv[a] = e >= 0 ? cnt[wave * E_loc + e] + rank : -1;   // -1: expert not local
    __syncthreads();                           // before cnt[] is cleared again
  }
  if (tid < E_loc) hist[size_t(blockIdx.x) * E_loc + tid] = at;
}

// place: every workgroup adds up the chunks' counts per expert, those before its own
// chunk apart from the rest (up to 32 threads share an expert's chunks, their sums are
// added in LDS), and scans the totals into offsets;
// position = offsets[e] + count before the chunk + rank.  Workgroup 0 stores counts and
// offsets.
__global__ __launch_bounds__(kRun) void dispatch_place_kernel(
    const int32_t* __restrict__ ids, int A, int e_lo, int E_loc, int chunk, int n_chunks,
    const int32_t* __restrict__ hist, int32_t* __restrict__ counts, int32_t* __restrict__ offsets_out,
    int32_t* __restrict__ perm, int32_t* __restrict__ inv) {
  __shared__ int32_t before[512], total[512];  // before: becomes the chunk's first position of each expert
  __shared__ int32_t part_lo[kRun], part_all[kRun];
  const int tid = threadIdx.x, lane = tid & 63;
  const int mine = blockIdx.x;
  const int a0 = mine * chunk, a1 = min(A - a0, chunk) + a0;
  const int a_first = a0 + tid;
  int e = -1, rank = -1;                       // of this thread's first assignment: on their way meanwhile
  if (a_first < a1) {
    e = ids[a_first] - e_lo;
    rank = inv[a_first];
  }
  const int groups = min(kRun / E_loc, 32);    // threads per expert
  if (tid < groups * E_loc) {
    const int x = tid % E_loc, g = tid / E_loc;
    int lo = 0, all = 0;
#pragma unroll 4
    for (int ch = g; ch < n_chunks; ch += groups) {
      const int n = hist[size_t(ch) * E_loc + x];
      all += n;
      lo += ch < mine ? n : 0;
    }
    part_lo[tid] = lo;
    part_all[tid] = all;
  }
  __syncthreads();
  if (tid < E_loc) {
    int lo = 0, all = 0;
#pragma unroll 4
    for (int g = 0; g < groups; ++g) {
      lo += part_lo[g * E_loc + tid];
      all += part_all[g * E_loc + tid];
    }
    before[tid] = lo;
    total[tid] = all;
  }
  __syncthreads();
  if (tid < 64) {
    const int per = (E_loc + 63) / 64;
    const int x0 = min(E_loc, lane * per), x1 = min(E_loc, x0 + per);
    int sum = 0;
    for (int x = x0; x < x1; ++x) sum += total[x];
    int incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int o = __shfl_up(incl, off);
      if (lane >= off) incl += o;
    }
    int at = incl - sum;
    for (int x = x0; x < x1; ++x) {
      const int n = total[x];
      before[x] += at;
      if (mine == 0) {
        counts[x] = n;
        offsets_out[x] = at;
      }
      at += n;
    }
    if (lane == 63 && mine == 0) offsets_out[E_loc] = incl;
  }
  __syncthreads();
  for (int a = a_first; a < a1; a += kRun) {
    if (a != a_first) {
      e = ids[a] - e_lo;
      rank = inv[a];
    }
    if (rank < 0) continue;                    // inv[a] stays -1
    const int pos = before[e] + rank;
    perm[pos] = a;
    inv[a] = pos;
  }
}

// One wavefront per token: read the row once, write it to every local position.
// Lengths in 16-byte pieces: `src16` = pitch of a token row, `col16` = first
// piece of the copied column window, `row16` = width of the window = pitch of
// the destination rows (the whole row: col16 = 0, row16 = src16).
template <int PIECES>
__global__ __launch_bounds__(256) void dispatch_gather_kernel(const uint4* __restrict__ x,
                                                             const int32_t* __restrict__ inv,
                                                             uint4* __restrict__ xs, int T, int k,
                                                             int src16, int col16, int row16) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (t >= T) return;
  int pos = -1;
  if (lane < k) pos = inv[size_t(t) * k + lane];      // k <= 32
  const uint64_t have = __ballot(pos >= 0);
  if (!have) return;
  const uint4* src = x + size_t(t) * src16 + col16;
  for (int c0 = 0; c0 < row16; c0 += 64 * PIECES) {
    uint4 v[PIECES];
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
      const int c = c0 + i * 64 + lane;
      if (c < row16) v[i] = nt_load16(src + c);
    }
    uint64_t m = have;
    while (m) {
      const int j = __ffsll((unsigned long long)m) - 1;
      m &= m - 1;
      const int p = __shfl(pos, j);
      uint4* dst = xs + size_t(p) * row16;
#pragma unroll
      for (int i = 0; i < PIECES; ++i) {
        const int c = c0 + i * 64 + lane;
        if (c < row16) nt_store16(dst + c, v[i]);
      }
    }
  }
}

// Few assignments (A <= kSmallA, and T <= kSmallT: a workgroup per four tokens, two per CU
// at a time): the whole dispatch in one launch.  Every
// workgroup rebuilds the same index in its own LDS (count per sub-chunk, scan
// per expert, scan over experts, place: the steps and the order of the kernels
// above, so the permutation is the same), workgroup 0 stores it, and each
// workgroup then copies the rows of its four tokens, four wavefronts a row.  The
// redundant index work is a few microseconds on otherwise idle CUs and replaces two
// launches; it is a chain of LDS steps, so the workgroup has sixteen wavefronts and the
// scan over the sub-chunks keeps eight counts in flight.
// LDS: hist[n_sub][E_loc] | slot[n_sub*64] | cnt[E_loc] | offs[E_loc+1].
// Top-1, 4096 tokens (a second round of workgroups that rebuild the index), hidden 256 / 2048: 16.9 /
// 18.4 us against 9.3 / 12.2 in three launches; 2048 tokens 7.2 / 8.1, 2049 9.0 / 10.1.
constexpr int kSmallA = 4096, kSmallT = 2048;
constexpr size_t kSmallLds = 60 * 1024;
inline size_t small_lds_bytes(int E_loc, int n_sub) {
  return (size_t(n_sub) * E_loc + size_t(n_sub) * kSub + 2 * size_t(E_loc) + 1) * sizeof(int32_t);
}

template <int PIECES>
__global__ __launch_bounds__(1024) void dispatch_small_kernel(
    const int32_t* __restrict__ ids, int A, int e_lo, int E_loc, int n_sub,
    int32_t* __restrict__ counts, int32_t* __restrict__ offsets_out, int32_t* __restrict__ perm,
    int32_t* __restrict__ inv, const uint4* __restrict__ x, uint4* __restrict__ xs, int T, int k,
    int src16, int col16, int row16) {
  extern __shared__ int32_t lds[];
  int32_t* const hist = lds;                         // [n_sub][E_loc]
  int32_t* const slot = hist + n_sub * E_loc;        // [n_sub*64]: (e << 6 | rank), then position
  int32_t* const cnt = slot + n_sub * kSub;          // [E_loc]
  int32_t* const offs = cnt + E_loc;                 // [E_loc + 1]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool first = blockIdx.x == 0;
  for (int i = tid; i < n_sub * E_loc; i += 1024) hist[i] = 0;
  __syncthreads();
  // 1. count: ballots find the lanes of a sub-chunk that share an expert
  for (int sub = wave; sub < n_sub; sub += 16) {
    const int a = sub * kSub + lane;
    int e = -1;
    if (a < A) {
      e = ids[a] - e_lo;
      if (e < 0 || e >= E_loc) e = -1;
    }
    const uint64_t same = same_expert_lanes(e, E_loc);
    int rank = 0;
    if (e >= 0) {
      rank = __popcll(same & lanemask_lt());
      if (rank == 0) hist[sub * E_loc + e] = __popcll(same);
    }
    slot[a] = e >= 0 ? (e << 6 | rank) : -1;
  }
  __syncthreads();
  // 2. scan over the sub-chunks, one thread per expert
  for (int e = tid; e < E_loc; e += 1024) {
    int run = 0;
    for (int s0 = 0; s0 < n_sub; s0 += 8) {
      int c[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) c[i] = s0 + i < n_sub ? hist[(s0 + i) * E_loc + e] : 0;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (s0 + i < n_sub) hist[(s0 + i) * E_loc + e] = run;
        run += c[i];
      }
    }
    cnt[e] = run;
    if (first) counts[e] = run;
  }
  __syncthreads();
  // 3. offsets = exclusive scan of the counts (one wavefront)
  if (wave == 0) {
    const int per = (E_loc + 63) / 64;
    const int x0 = lane * per, x1 = (x0 + per < E_loc) ? x0 + per : E_loc;
    int sum = 0;
    for (int i = x0; i < x1; ++i) sum += cnt[i];
    int incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int o = __shfl_up(incl, off);
      if (lane >= off) incl += o;
    }
    int run = incl - sum;
    for (int i = x0; i < x1; ++i) {
      offs[i] = run;
      if (first) offsets_out[i] = run;
      run += cnt[i];
    }
    if (lane == 63) {
      offs[E_loc] = incl;
      if (first) offsets_out[E_loc] = incl;
    }
  }
  __syncthreads();
  // 4. place
  for (int a = tid; a < A; a += 1024) {
    const int sl = slot[a];
    int pos = -1;
    if (sl >= 0) {
      const int e = sl >> 6;
      pos = offs[e] + hist[(a / kSub) * E_loc + e] + (sl & 63);
      if (first) perm[pos] = a;
    }
    slot[a] = pos;
    if (first) inv[a] = pos;
  }
  __syncthreads();
  // 5. copy the rows of this workgroup's tokens: wavefront w takes runs w%4, w%4 + 4, .. of
  // 64 pieces of token w/4
  const int t = blockIdx.x * 4 + (wave >> 2);
  if (t >= T) return;
  int pos = -1;
  if (lane < k) pos = slot[t * k + lane];
  const uint64_t have = __ballot(pos >= 0);
  if (!have) return;
  const uint4* src = x + size_t(t) * src16 + col16;
  for (int c0 = (wave & 3) * 64; c0 < row16; c0 += 256 * PIECES) {
    uint4 v[PIECES];
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
      const int c = c0 + i * 256 + lane;
      if (c < row16) v[i] = nt_load16(src + c);
    }
    uint64_t m = have;
    while (m) {
      const int j = __ffsll((unsigned long long)m) - 1;
      m &= m - 1;
      const int p = __shfl(pos, j);
      uint4* dst = xs + size_t(p) * row16;
#pragma unroll
      for (int i = 0; i < PIECES; ++i) {
        const int c = c0 + i * 256 + lane;
        if (c < row16) nt_store16(dst + c, v[i]);
      }
    }
  }
}

// Per-row block scales follow their rows: out[kb][pos] = in[kb][token of pos] for
// the valid positions (both arrays are block-major: one row of the array per
// 128-column block).  blockIdx.y takes kScaleRun blocks: one thread walking all 56
// blocks of hidden 7168 was a chain of dependent loads on a quarter of the chip.
constexpr int kScaleRun = 8;
__global__ __launch_bounds__(256) void dispatch_scales_kernel(
    const float* __restrict__ in, int in_pitch, const int32_t* __restrict__ perm,
    const int32_t* __restrict__ offsets, int E_loc, int k, int n_blocks, float* __restrict__ out,
    int out_pitch) {
  const int pos = blockIdx.x * 256 + threadIdx.x;
  if (pos >= offsets[E_loc] || pos >= out_pitch) return;
  const int t = perm[pos] / k, kb0 = blockIdx.y * kScaleRun;
  float v[kScaleRun];
#pragma unroll
  for (int i = 0; i < kScaleRun; ++i) v[i] = in[size_t(min(kb0 + i, n_blocks - 1)) * in_pitch + t];
#pragma unroll
  for (int i = 0; i < kScaleRun; ++i)
    if (kb0 + i < n_blocks) out[size_t(kb0 + i) * out_pitch + pos] = v[i];
}

}  // namespace

hipError_t launch_dispatch_scales(const float* in, int in_pitch, const int32_t* perm,
                                  const int32_t* offsets, int E_loc, int k, int n_blocks, float* out,
                                  int out_pitch, hipStream_t s) {
  MOE_LAUNCH(MOE_K_DISPATCH_GATHER, dispatch_scales_kernel,
             dim3((out_pitch + 255) / 256, (n_blocks + kScaleRun - 1) / kScaleRun), dim3(256), 0, s,
             in, in_pitch, perm, offsets, E_loc, k, n_blocks, out, out_pitch);
  return hipGetLastError();
}

hipError_t launch_dispatch(const moe_config& c, int T, const void* x, const int32_t* ids,
                           int32_t* counts, int32_t* offsets, int32_t* perm, int32_t* inv,
                           void* xs, int tp_rank, int tp_size, const DispatchWs& ws,
                           hipStream_t s, int elem_bytes) {
  const int k = c.top_k;
  const int A = T * k;
  const int E_loc = c.expert_hi - c.expert_lo;
  const int n_sub = (A + kSub - 1) / kSub;
  // column window of TP rank tp_rank of tp_size (the whole row for 0 of 1);
  // elem_bytes overrides the element size of the rows (1: quantised codes)
  if (elem_bytes == 0) elem_bytes = c.act_dtype == MOE_F32 ? 4 : 2;
  const int src16 = c.hidden * elem_bytes / 16;
  const int row16 = src16 / tp_size;
  if (A <= kSmallA && T <= kSmallT && small_lds_bytes(E_loc, n_sub) <= kSmallLds) {
    MOE_LAUNCH(MOE_K_DISPATCH_GATHER, dispatch_small_kernel<4>, dim3((T + 3) / 4), dim3(1024),
               small_lds_bytes(E_loc, n_sub), s, ids, A, c.expert_lo, E_loc, n_sub, counts, offsets,
               perm, inv, static_cast<const uint4*>(x), static_cast<uint4*>(xs), T, k, src16,
               tp_rank * row16, row16);
    return hipGetLastError();
  }
  const int chunk = index_chunk(A), n_chunks = (A + chunk - 1) / chunk;
  MOE_LAUNCH(MOE_K_DISPATCH_HIST, dispatch_count_kernel, dim3(n_chunks), dim3(kRun),
             size_t(16) * E_loc * sizeof(int32_t), s, ids, A, c.expert_lo, E_loc, chunk, ws.block_hist, inv);
  MOE_LAUNCH(MOE_K_DISPATCH_SCATTER, dispatch_place_kernel, dim3(n_chunks), dim3(kRun), 0, s, ids, A,
             c.expert_lo, E_loc, chunk, n_chunks, ws.block_hist, counts, offsets, perm, inv);
  MOE_LAUNCH(MOE_K_DISPATCH_GATHER, dispatch_gather_kernel<8>, dim3((T + 3) / 4), dim3(256), 0, s,
             static_cast<const uint4*>(x), inv, static_cast<uint4*>(xs), T, k, src16,
             tp_rank * row16, row16);
  return hipGetLastError();
}

}  // namespace moe

// Sliced adjacency of the persistent plan: the kernels that lay a graph's rows
// and entries out for the step loops of k_tile_round.  They use no more of the
// device than threads, shared arrays, barriers and wavefront votes.
#pragma once

#include <climits>

namespace mqo {

// ---------------------------------------------------------------------------
// Sliced adjacency (unweighted graphs of at most ELL_MAX_ROWS rows).  The rows
// of a graph are sorted by descending degree (ord) and cut into slices of 64.
// A slice is a list of issue slots, 64 entries each, one per lane; eight slots
// form a block in which the 64 lanes' 8 entries lie side by side: one 16-byte
// load per lane and 1 KB per wavefront, fully coalesced.  An entry is a byte
// offset in an iterate tile of T columns (4 T x local row, 16 bits): the
// lane's next neighbour in ascending CSR order, or a row of zeros; adding a
// zero anywhere in a sum leaves every result bit-identical (a sum starts at
// +0 and never becomes -0).
//
// What bounds the step is the LDS: a 4- or 8-byte read runs as two passes of
// 32 lanes over 32 banks (of 4 or 8 bytes), each as long as the rows that
// meet on its fullest bank: 7.5 clocks for random rows, 2.8 conflict-free,
// 4.4 with at most two on a bank (measured).  So for T <= 2 a slot takes at
// most two different rows per bank and pass; the lanes with the fewest
// entries left wait with a zero row of a bank that is free (about 1.08 times
// the slots, 5 clocks per slot instead of 7.2).  A 16-byte read (T = 4) runs
// as four passes of 16 lanes and is left as it comes.
//
// Measured, one trajectory per workgroup, 64 of them: n = 1000, degree 100,
// 4.46 us per step (5.7 without the slots' rule, the general loop 14.5); with
// the entries of a wavefront's only slice kept in registers the whole
// 91-round solve went from 264.9 to 90.3 ms (112.3 as they come, 93.5 with
// the rule and the entries read again in every step); n = 3000, degree 100,
// 61 rounds with early exit, 247.9 (streaming plan) -> 47.5 ms (61.9 without
// the rule); n = 100, degree 10, 1000 steps 860 -> 593 us (711 with the
// entries read in every step).  The autotuner times it beside the other
// shapes for T <= 4 (a lane owns whole rows; wider tiles share a row between
// lanes, whose column loads then fall together anyway).
//
// Places in the workspace, without tables: graph g's slices (first block and
// block count) are at ell_slice_base, its blocks at ell_block_base, both
// rounded so that neighbouring graphs never overlap.  A slice as wide as w
// may take ell_slots(w) slots, and the widths of a sorted graph add up to at
// most its degrees / 64 plus its largest; one whose rows meet on few banks
// and would take more is stored as it comes, w slots.
// ---------------------------------------------------------------------------
constexpr int ELL_MAX_ROWS = 8192;

__host__ __device__ inline int32_t ell_slots(int32_t w) { return (w + w / 4 + 8 + 7) & ~7; }  // <= 1.25 w + 15
__host__ __device__ inline int64_t ell_slice_base(int64_t lo, int64_t g) { return (lo >> 6) + 2 * g; }
__host__ __device__ inline int64_t ell_block_base(int64_t lo, int64_t e0, int64_t g) {
  return (e0 >> 7) + (lo >> 2) + (lo >> 5) + 8 * g;
}
// the row order and the slices' first blocks; one workgroup per graph
__global__ __launch_bounds__(1024) void k_ell_order(const int32_t *__restrict__ row_ptr,
                                                    const int64_t *__restrict__ vtx_off, uint16_t *__restrict__ ord,
                                                    int2 *__restrict__ slices) {
  __shared__ uint32_t bins[ELL_MAX_ROWS];  // rows per degree (a degree is below the row count), then places
  __shared__ uint16_t so[ELL_MAX_ROWS];    // the order
  __shared__ uint32_t part[1024];
  const int32_t g = blockIdx.x, tid = threadIdx.x, nthr = blockDim.x;
  const int64_t lo = vtx_off[g];
  const int32_t n = (int32_t)(vtx_off[g + 1] - lo);
  const int32_t *rp = row_ptr + lo;
  for (int32_t d = tid; d < ELL_MAX_ROWS; d += nthr) bins[d] = 0u;
  __syncthreads();
  // bin 0 holds the largest possible degree, n - 1
  for (int32_t v = tid; v < n; v += nthr) atomicAdd(&bins[n - 1 - (rp[v + 1] - rp[v])], 1u);
  __syncthreads();
  constexpr int PER = ELL_MAX_ROWS / 1024;
  uint32_t own = 0;
  for (int i = 0; i < PER; ++i) own += bins[tid * PER + i];
  part[tid] = own;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const uint32_t t = tid >= off ? part[tid - off] : 0u;
    __syncthreads();
    part[tid] += t;
    __syncthreads();
  }
  uint32_t run = part[tid] - own;
  for (int i = 0; i < PER; ++i) {
    const uint32_t h = bins[tid * PER + i];
    bins[tid * PER + i] = run;
    run += h;
  }
  __syncthreads();
  for (int32_t v = tid; v < n; v += nthr) so[atomicAdd(&bins[n - 1 - (rp[v + 1] - rp[v])], 1u)] = (uint16_t)v;
  __syncthreads();
  for (int32_t i = tid; i < n; i += nthr) ord[lo + i] = so[i];
  if (tid == 0) {
    int2 *st = slices + ell_slice_base(lo, g);
    int32_t b = 0;
    for (int32_t s = 0; s * 64 < n; ++s) {
      const int32_t v = so[s * 64];  // the slice's longest row
      st[s] = make_int2(b, 0);
      b += ell_slots(rp[v + 1] - rp[v]) >> 3;
    }
  }
}

// the slots of a slice; one wavefront per (graph, slice)
__global__ __launch_bounds__(256) void k_ell_slots(const int32_t *__restrict__ row_ptr,
                                                   const int32_t *__restrict__ col_idx,
                                                   const int64_t *__restrict__ vtx_off, int32_t log2T, int32_t zrow,
                                                   const uint16_t *__restrict__ ord, int2 *__restrict__ slices,
                                                   uint4 *__restrict__ blocks) {
  // per wavefront, pass (32 lanes) and bank: the keys of the first and second row taken
  __shared__ uint32_t s_first[4][64], s_second[4][64];
  const int32_t g = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t lo = vtx_off[g];
  const int32_t n = (int32_t)(vtx_off[g + 1] - lo);
  const int32_t s = blockIdx.y * 4 + wave;
  if (s * 64 >= n) return;  // the whole wavefront
  const int32_t *rp = row_ptr + lo;
  int2 *sl = slices + ell_slice_base(lo, g) + s;
  const int32_t b0 = sl->x;
  uint4 *bl = blocks + (ell_block_base(lo, rp[0], g) + b0) * 64 + lane;
  const int32_t i = s * 64 + lane;
  const int32_t v = i < n ? ord[lo + i] : -1;
  const int32_t beg = v >= 0 ? rp[v] : 0, deg = v >= 0 ? rp[v + 1] - beg : 0;
  const int32_t w = __builtin_amdgcn_readfirstlane(deg);  // lane 0 holds the longest row
  const int32_t cap = ell_slots(w);
  const int32_t sh = 2 + log2T;
  auto column = [&](int32_t j) { return col_idx[beg + j] - (int32_t)lo; };
  volatile uint32_t *first = s_first[wave], *second = s_second[wave];
  bool fits = log2T <= 1;
  int32_t slots = 0;
  if (fits) {
    int32_t p = 0;
    int32_t u = p < deg ? column(p) : 0;
    while (__ballot(p < deg)) {
      if (slots == cap) {
        fits = false;
        break;
      }
      uint32_t q[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const bool act = p < deg;
        const int32_t bank = (lane & 32) | (u & 31);
        const uint32_t key = ((uint32_t)(deg - p) << 6) | (uint32_t)(63 - lane);  // most left first
        first[lane] = 0u;
        second[lane] = 0u;
        __builtin_amdgcn_wave_barrier();
        if (act) atomicMax(&s_first[wave][bank], key);
        __builtin_amdgcn_wave_barrier();
        bool win = act && first[bank] == key;
        if (act && !win) atomicMax(&s_second[wave][bank], key);
        __builtin_amdgcn_wave_barrier();
        win = win || (act && second[bank] == key);
        // a bank of this pass that no row, else at most one row, is read from
        const uint32_t none = (uint32_t)(__ballot(first[lane] == 0u) >> (lane & 32));
        const uint32_t one = (uint32_t)(__ballot(second[lane] == 0u) >> (lane & 32));
        const int32_t z = none ? __builtin_ctz(none) : one ? __builtin_ctz(one) : lane & 31;
        q[k] = (uint32_t)(win ? u : zrow + z) << sh;
        if (win) {
          ++p;
          u = p < deg ? column(p) : 0;
        }
        __builtin_amdgcn_wave_barrier();
      }
      bl[(int64_t)(slots >> 3) * 64] =
          make_uint4(q[0] | q[1] << 16, q[2] | q[3] << 16, q[4] | q[5] << 16, q[6] | q[7] << 16);
      slots += 8;
    }
  }
  if (!fits) {
    for (slots = 0; slots < w; slots += 8) {
      uint32_t q[8];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        q[k] = (uint32_t)(slots + k < deg ? column(slots + k) : zrow + (lane & 31)) << sh;
      bl[(int64_t)(slots >> 3) * 64] =
          make_uint4(q[0] | q[1] << 16, q[2] | q[3] << 16, q[4] | q[5] << 16, q[6] | q[7] << 16);
    }
  }
  if (lane == 0) sl->y = slots >> 3;
}

// ---------------------------------------------------------------------------
// Wide slices (the single-buffered step of T = 16, 32 or 64 trajectories,
// unweighted graphs): the R = 256 / T rows that a wavefront walks together
// (T / 4 lanes each) as one slice, blocks of 4 entries per row side by side:
// 32-bit byte offsets in the tile, one 16-byte load per lane for 4 gathers,
// a trip count that is the same for the whole wavefront, and one addition
// per gather for its address.  Padding as above (entries up to the slice's
// longest row, rounded up to 4).
//
// The gathers are bound by the LDS passes, two rows of 32 trajectories each:
// a pass takes two cycles when both rows lie in the same half of the banks
// (fewer instructions alone changed nothing: 5.2 VALU per 16-byte gather
// here, 6 in the general loop).  So rows are paired: the longest row left
// with the one of the next 64 whose neighbours most often lie in the other
// half at the same position of the row (39% of the reads then meet in one
// half instead of 50%; 128 or all rows to choose from would give 38%).
// Measured on the batch of 128 ER graphs of 700-800 vertices, p = 0.15, 512
// trajectories, 4 rounds: 224 -> 212 ms (222 without the pairing).
// ---------------------------------------------------------------------------
constexpr int WIDE_BITS = 8;           // 32-bit words of a row's parities that are compared
constexpr int WIDE_MAX_ELEMS = 32768;  // rows x trajectories of a tile: 8 lane items of 4 in 1024 threads
constexpr int WIDE_PAIR_LOG2T = 5;     // the width whose rows are paired
// the largest graph of a width; the arrays of k_wide_build and the step loop's
// slice table are sized by it, and the host offers no larger one
__host__ __device__ constexpr int32_t wide_max_rows(int32_t log2T) { return WIDE_MAX_ELEMS >> log2T; }
constexpr int WIDE_MAX_ROWS = wide_max_rows(4);
constexpr int WIDE_MAX_SLICES = WIDE_MAX_ELEMS / 256;

__host__ __device__ inline int32_t wide_rows(int32_t log2T) { return 256 >> log2T; }
__host__ __device__ inline int64_t wide_slice_base(int64_t lo, int64_t g) { return (lo >> 2) + 2 * g; }  // R >= 4

// pairs in `so` (rows by descending degree), by the first wavefront; bits:
// [n][WIDE_BITS] parities of the row's first neighbours; out: the new order
__device__ inline void wide_pair_rows(const uint16_t *so, const int32_t *rp, const uint32_t *bits, int32_t n,
                                      uint16_t *out) {
  const int lane = threadIdx.x & 63;
  int32_t at = lane < n ? lane : INT_MAX;  // place in so of the row this lane offers
  int32_t next = 64;
  uint32_t b[WIDE_BITS];
  int32_t deg = 0;
  auto fetch = [&]() {
    if (at == INT_MAX) return;
    const int32_t v = so[at];
    deg = rp[v + 1] - rp[v];
#pragma unroll
    for (int w = 0; w < WIDE_BITS; ++w) b[w] = bits[v * WIDE_BITS + w];
  };
#pragma unroll
  for (int w = 0; w < WIDE_BITS; ++w) b[w] = 0u;
  fetch();
  for (int32_t done = 0; done < n; done += 2) {
    // the longest row left: the smallest place
    int32_t first = at;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) first = min(first, __shfl_xor(first, d, 64));
    const int la = __builtin_ctzll(__ballot(at == first));
    const int32_t da = __shfl(deg, la, 64);
    int32_t meet = 0;
#pragma unroll
    for (int w = 0; w < WIDE_BITS; ++w) {
      const int32_t len = min(deg, da) - 32 * w;
      const uint32_t mask = len >= 32 ? ~0u : len > 0 ? (1u << len) - 1u : 0u;
      meet += __popc(~(b[w] ^ (uint32_t)__shfl((int)b[w], la, 64)) & mask);
    }
    // a much shorter partner would leave its slots empty
    int32_t cost = meet + (da - deg);
    cost = lane == la || at == INT_MAX ? INT_MAX : (cost << 6) | lane;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) cost = min(cost, __shfl_xor(cost, d, 64));
    const int lb = cost == INT_MAX ? -1 : cost & 63;
    if (lane == la) out[done] = so[at];
    if (lane == lb) out[done + 1] = so[at];
    if (lane == la || lane == lb) {
      const int32_t i = lane == la ? next : next + 1;
      at = i < n ? i : INT_MAX;
      fetch();
    }
    next += 2;
  }
}

// row order (paired), slices (first block, blocks) and entries; one
// workgroup per graph
__global__ __launch_bounds__(1024) void k_wide_build(const int32_t *__restrict__ row_ptr,
                                                     const int32_t *__restrict__ col_idx,
                                                     const int64_t *__restrict__ vtx_off, int32_t log2T, int32_t zrow,
                                                     uint16_t *__restrict__ ord, int2 *__restrict__ slices,
                                                     uint4 *__restrict__ blocks) {
  __shared__ uint32_t bits[wide_max_rows(WIDE_PAIR_LOG2T) * WIDE_BITS];  // used at that width alone
  __shared__ uint16_t so[WIDE_MAX_ROWS], sp[WIDE_MAX_ROWS];
  __shared__ int2 ss[WIDE_MAX_SLICES];
  const int32_t g = blockIdx.x, tid = threadIdx.x, nthr = blockDim.x;
  const int64_t lo = vtx_off[g];
  const int32_t n = (int32_t)(vtx_off[g + 1] - lo);
  const int32_t *rp = row_ptr + lo;
  const int32_t R = wide_rows(log2T), ns = (n + R - 1) / R;
  for (int32_t i = tid; i < n; i += nthr) {
    so[i] = ord[lo + i];
    sp[i] = so[i];
  }
  __syncthreads();
  if (log2T == WIDE_PAIR_LOG2T) {
    for (int32_t i = tid; i < n * WIDE_BITS; i += nthr) {
      const int32_t v = i / WIDE_BITS, w = i % WIDE_BITS;
      const int32_t j0 = rp[v] + 32 * w, j1 = min(rp[v + 1], j0 + 32);
      uint32_t x = 0;
      for (int32_t j = j0; j < j1; ++j) x |= (uint32_t)((col_idx[j] - (int32_t)lo) & 1) << (j - j0);
      bits[i] = x;
    }
    __syncthreads();
    if (tid < 64) wide_pair_rows(so, rp, bits, n, sp);
    __syncthreads();
  }
  for (int32_t i = tid; i < n; i += nthr) ord[lo + i] = sp[i];
  for (int32_t s = tid; s < ns; s += nthr) {
    int32_t w = 0;
    for (int32_t i = s * R; i < min(n, (s + 1) * R); ++i) w = max(w, rp[sp[i] + 1] - rp[sp[i]]);
    ss[s] = make_int2(0, (w + 3) >> 2);
  }
  __syncthreads();
  if (tid == 0) {
    int32_t b = 0;
    for (int32_t s = 0; s < ns; ++s) {
      ss[s].x = b;
      b += ss[s].y;
    }
  }
  __syncthreads();
  for (int32_t s = tid; s < ns; s += nthr) slices[wide_slice_base(lo, g) + s] = ss[s];
  if (n == 0) return;
  uint4 *bl = blocks + ell_block_base(lo, rp[0], g) * 64;
  const int sh = log2T + 2;
  for (int32_t s = 0; s < ns; ++s)
    for (int32_t k = tid; k < ss[s].y * R; k += nthr) {
      const int32_t r = k % R, b = k / R, i = s * R + r;
      const int32_t v = i < n ? sp[i] : -1;
      const int32_t beg = v >= 0 ? rp[v] : 0, deg = v >= 0 ? rp[v + 1] - beg : 0;
      uint32_t q[4];
#pragma unroll
      for (int t = 0; t < 4; ++t)
        q[t] = (uint32_t)(4 * b + t < deg ? col_idx[beg + 4 * b + t] - (int32_t)lo : zrow) << sh;
      bl[(int64_t)(ss[s].x + b) * R + r] = make_uint4(q[0], q[1], q[2], q[3]);
    }
}

}  // namespace mqo

// Device code of the FDA monitor for gfx950 (wave64): everything except the state kernel.
// Included by fda_api.hip only.
//
//   hash_table_kernel  once per context: the tabulated hash
//   finish_kernel    fixed-order fp64 sum of the per-workgroup partials -> state[K][S], or mean_state[S];
//                    on request with the estimate of Algorithm 1 lines 7-8 in the same launch
//   estimate_kernel  Algorithm 1 lines 7-8 on given states: mean state, M2, H (Thm 1, Thm 2), decision
//   sync_kernel      Algorithm 1 line 9: fused mean over workers + broadcast to all rows (+ the squared
//                    norm of the model change, for the refresh of xi)
//   sync_from_mean_kernel  the same from an average model that is already there, with xi
//   xi_norm_kernel / xi_scale_kernel   Section 3.2: the normalized model difference
#pragma once
#include "fda_kernels.hpp"

namespace fda {

// ---- the hash, tabulated once per context (Section 3.1 sketch; hash family: two cubics mod 2^31 - 1
// per row).  Per row group r and coordinate j one record of `words` 16-bit words; a record packs,
// lowest bits first, one field of `fb` bits per row slot of the group: bucket + m for sign -1, bucket
// for sign +1 (below 2 m, which fits: field_bits_for).  Slots past the group's last row (and whole
// records past d) hold a value below kDummyCells: the state kernels send those additions to a dummy
// region (whatever bucket and sign they decode from it, the bucket stays below kDummyCells).
// Layout [row group][block of 256 coordinates][dwords in load order]: the 2 * words dwords of the 4
// records that a lane of the state kernels loads together are placed where load_rec_block() reads
// them.  One thread writes one lane's share; a workgroup of kSmallThreads covers 4 blocks.
//
// grp >= 2: placed rows (see kPlacedFieldBits) for a state kernel of KC worker slots.  The rows of the
// group come in placement groups of grp; slot a of a placement group of n rows holds row (a + rot) % n of
// it, field = that row's number in the group times the buckets a row takes up (cells32_row_buckets) plus
// the plain field, and rot is chosen per coordinate so that the additions one instruction of the state
// kernel issues collide as little as the choice allows.  The model: the 16 lanes 16 g .. 16 g + 15 of a
// wave are served together, instruction (v, slot) takes coordinate 4 lane + v of the block from each, and
// two of them collide when the 8-byte words they address lie a multiple of 128 bytes apart: the word
// index of a field (cells32_bucket_word / 2) modulo 16 is its class.  Cost of an instruction = the largest number of lanes in one class; per (16 lanes, v,
// placement group) one thread places the 16 coordinates one after the other where the sum over the
// slots grows least, then revisits each twice.  The result depends only on the hash and the shape.
constexpr int kPlaceSweeps = 3;
__global__ void __launch_bounds__(kSmallThreads)
hash_table_kernel(const HashCoef hc, int l, int R, int slots, int m, int fb, int words, int grp, int KC,
                  long long d, long long dpad, uint16_t* __restrict__ table) {
  __shared__ uint16_t fld[kSmallThreads][4][kMaxLR];           // plain fields, by thread, coordinate, row
  __shared__ uint8_t rotsel[kSmallThreads][4][kMaxPlaceGroups];  // chosen rotation, by thread, coordinate, placement group
  __shared__ uint8_t hist[kSmallThreads / 64][16][kMaxLR][16];     // by wave, (16 lanes, v), slot, class
  const int r = blockIdx.y;
  const int tid = threadIdx.x;
  const long long j4 = ((long long)blockIdx.x * blockDim.x + tid) * 4;
  int rstart, rcnt;
  group_range(l, R, r, &rstart, &rcnt);
  const bool placed = grp >= 2;
  const uint32_t mrow = placed ? (uint32_t)cells32_row_buckets(2 * m, KC) : 0u;   // buckets per LDS row, as a field counts them
  for (int q = 0; q < 4; ++q) {
    const long long j = j4 + q;
    for (int i = 0; i < slots; ++i) {
      uint32_t f = (uint32_t)(j + 17 * i) & (uint32_t)(kDummyCells - 1);
      if (i < rcnt && j < d) {
        const uint32_t h = hash_entry(hc, rstart + i, (uint32_t)j, (uint32_t)m);
        f = (h & 0x7fffu) + (h >> 15) * (uint32_t)m;           // bucket + m * (sign is -1)
      }
      fld[tid][q][i] = (uint16_t)f;
    }
  }
  if (placed) {                                                // (uniform over the workgroup)
    const int ngroups = (rcnt + grp - 1) / grp;                // at most kMaxPlaceGroups: grp >= 2, at most kMaxLR rows
    for (int q = 0; q < 4; ++q)
      for (int g = 0; g < kMaxPlaceGroups; ++g) rotsel[tid][q][g] = 0;
    __syncthreads();
    const int wave = tid >> 6, lane = tid & 63;
    // problem (16 lanes gi, coordinate v) = lane & 15; placement groups lane >> 4, lane >> 4 + 4, ...
    const int prob = lane & 15, gi = prob >> 2, v = prob & 3;
    for (int g = lane >> 4; g < ngroups; g += 4) {
      const int g0 = g * grp, n = rcnt - g0 < grp ? rcnt - g0 : grp;
      if (n < 2) continue;
      uint8_t (*h)[16] = &hist[wave][prob][g0];                // n slots of 16 classes
      for (int a = 0; a < n; ++a)
        for (int c = 0; c < 16; ++c) h[a][c] = 0;
      const int member0 = wave * 64 + gi * 16;
      // class of member t's entry of row `row` (within the placement group)
      auto cls = [&](int t, int row) {
        const uint32_t field = (uint32_t)row * mrow + fld[member0 + t][v][g0 + row];
        return (int)((cells32_bucket_word(field, KC) >> 1) & 15u);
      };
      for (int sweep = 0; sweep < kPlaceSweeps; ++sweep) {
        for (int t = 0; t < 16; ++t) {
          if (sweep > 0) {
            const int cur = rotsel[member0 + t][v][g];
            for (int a = 0; a < n; ++a) { int row = a + cur; if (row >= n) row -= n; h[a][cls(t, row)] -= 1; }
          }
          int mx[kMaxLR];
          for (int a = 0; a < n; ++a) {
            int top = 0;
            for (int c = 0; c < 16; ++c) top = h[a][c] > top ? h[a][c] : top;
            mx[a] = top;
          }
          int best = 1 << 30, brot = 0;
          for (int rot = 0; rot < n; ++rot) {
            int cost = 0;
            for (int a = 0; a < n; ++a) {
              int row = a + rot; if (row >= n) row -= n;
              const int after = h[a][cls(t, row)] + 1;
              cost += after > mx[a] ? after : mx[a];
            }
            if (cost < best) { best = cost; brot = rot; }
          }
          rotsel[member0 + t][v][g] = (uint8_t)brot;
          for (int a = 0; a < n; ++a) { int row = a + brot; if (row >= n) row -= n; h[a][cls(t, row)] += 1; }
        }
      }
    }
    __syncthreads();
  }
  if (j4 >= dpad) return;
  uint32_t dw[2 * kMaxLR];                             // 4 records of at most kMaxLR words
  for (int t = 0; t < 2 * kMaxLR; ++t) dw[t] = 0u;
  for (int q = 0; q < 4; ++q) {
    unsigned long long bits[3] = {0ull, 0ull, 0ull};          // slots * fb <= 9 * 16 bits
    for (int i = 0; i < slots; ++i) {
      unsigned long long f = fld[tid][q][i];
      if (placed && i < rcnt) {
        const int g = i / grp, g0 = g * grp, n = rcnt - g0 < grp ? rcnt - g0 : grp;
        int row = i - g0 + rotsel[tid][q][g]; if (row >= n) row -= n;
        f = (unsigned long long)((uint32_t)row * mrow + fld[tid][q][g0 + row]);
      }
      const int pos = i * fb, idx = pos >> 6, sh = pos & 63;
      bits[idx] |= f << sh;
      if (sh + fb > 64) bits[idx + 1] |= f >> (64 - sh);
    }
    for (int t = 0; t < words; ++t) {
      const uint32_t w16 = (uint32_t)(bits[t >> 2] >> (16 * (t & 3))) & 0xffffu;
      const int w = q * words + t;                             // 16-bit word of the lane's share
      dw[w >> 1] |= w16 << (16 * (w & 1));
    }
  }
  const int N = 2 * words, n4 = N / 4, n2 = (N % 4) / 2;
  const int lane = (int)(j4 >> 2) & 63;
  uint32_t* blk = reinterpret_cast<uint32_t*>(table) +
                  ((size_t)r * (size_t)(dpad / kRecBlockCoords) + (size_t)(j4 / kRecBlockCoords)) * (size_t)(64 * N);
  for (int t = 0; t < N; ++t) {
    int off;
    if (t < 4 * n4) off = ((t >> 2) * 64 + lane) * 4 + (t & 3);
    else if (t < 4 * n4 + 2 * n2) off = n4 * 256 + lane * 2 + (t - 4 * n4);
    else off = n4 * 256 + n2 * 128 + lane;
    blk[off] = dw[t];
  }
}

__global__ void clear_u32_kernel(unsigned int* p, int n) {
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) p[t] = 0u;
}

// Index of the group of group_range(K, G) that holds item k.
__device__ inline int group_of(int K, int G, int k) {
  const int base = K / G, rem = K % G, big = rem * (base + 1);
  return k < big ? k / (base + 1) : rem + (k - big) / base;
}

// ----------------------------------------------------------------------------------------
// Algorithm 1 lines 7-8, all in fp64:
//   mean_k of the states;  row norms of the mean sketch;  M2 = their median (Section 3.1);
//   H_sketch = n - M2/(1+eps) (Thm 1);  H_linear = n - p^2 (Thm 2);  sync = H > theta.
// A row norm is added up in one fixed order, whichever kernel does it: the squares of 32 neighbouring
// cells as a tree, eight such sums (256 cells) in order, those in order.
// ----------------------------------------------------------------------------------------
constexpr int kEstCols = kSmallThreads;      // cells per workgroup of estimate_kernel
constexpr int kMaxEstBlocks = FDA_MAX_SKETCH_ROWS * ((FDA_STATIC_MAX_M + kEstCols - 1) / kEstCols);

struct EstimateArgs {
  int variants, l, m, K;
  double eps, theta, tie_tol;
  fda_estimate* out;
  fda_estimate* host;              // pinned host memory that receives the result too, or NULL
};
__device__ __forceinline__ double half_wave_sum(double v) {   // valid in lanes 0 and 32
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) v += __shfl_down(v, o, 32);
  return v;
}
// One thread: the result from the sums of the two scalar components and the l row norms.
__device__ inline void decide(const EstimateArgs& a, double nsum, double psum, const double* rows, int state_path) {
  fda_estimate e;
  e.mean_sqnorm = nsum / (double)a.K;
  e.mean_proj = 0.0; e.m2 = 0.0; e.h_linear = 0.0; e.h_sketch = 0.0;
  e.sync_linear = 0; e.sync_sketch = 0; e.near_tie_linear = 0; e.near_tie_sketch = 0;
  e.nonfinite = 0;
  e.state_path = state_path;
  const double band = a.tie_tol * fmax(e.mean_sqnorm, fabs(a.theta));
  if (a.variants & FDA_VARIANT_LINEAR) {
    e.mean_proj = psum / (double)a.K;
    e.h_linear = e.mean_sqnorm - e.mean_proj * e.mean_proj;
    if (isfinite(e.h_linear)) {
      e.sync_linear = e.h_linear > a.theta ? 1 : 0;
      e.near_tie_linear = fabs(e.h_linear - a.theta) <= band ? 1 : 0;
    } else {
      e.sync_linear = 1; e.nonfinite = 1;
    }
  }
  if (a.variants & FDA_VARIANT_SKETCH) {
    // median of l values: insertion sort, then middle (even l: mean of the two middle)
    double r[FDA_MAX_SKETCH_ROWS];
    for (int i = 0; i < a.l; ++i) {
      const double v = rows[i];
      int q = i;
      while (q > 0 && !(r[q - 1] <= v)) { r[q] = r[q - 1]; --q; }
      r[q] = v;
    }
    e.m2 = (a.l & 1) ? r[a.l / 2] : 0.5 * (r[a.l / 2 - 1] + r[a.l / 2]);
    e.h_sketch = e.mean_sqnorm - e.m2 / (1.0 + a.eps);
    if (isfinite(e.h_sketch)) {
      e.sync_sketch = e.h_sketch > a.theta ? 1 : 0;
      e.near_tie_sketch = fabs(e.h_sketch - a.theta) <= band ? 1 : 0;
    } else {
      e.sync_sketch = 1; e.nonfinite = 1;
    }
  }
  *a.out = e;
  if (a.host != nullptr) *a.host = e;
}
// What workgroups of one launch hand to each other goes through agent-scope accesses (which pass the L2 of the
// XCD) and counters: the writer waits until its stores have been acknowledged before it counts itself, the
// reader's loads cannot hit a stale line.  (__threadfence() would write back and invalidate the whole L2, once
// per workgroup: with 640 workgroups that was 20 of the 32 us of a launch.)
template <typename V>
__device__ __forceinline__ void agent_store(V* p, V x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename V>
__device__ __forceinline__ V agent_load(const V* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Every thread of a workgroup: is it the last of `count` to get here?
__device__ __forceinline__ bool finished_last(unsigned int* ticket, int count, int* flag) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0)
    *flag = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)count - 1u ? 1 : 0;
  __syncthreads();
  return *flag != 0;
}

// The workgroup that finished last: part[0], part[1] are the sums of the scalar components, then come the
// row norms' pieces, `per` to each 256 cells (their loads are independent: taken one after the other by one
// thread they cost a third of a microsecond each, cfg5 28 of them).
__device__ inline void finish_estimate(const EstimateArgs& a, const double* part, int per, int state_path) {
  __shared__ double blocks[kMaxEstBlocks];
  __shared__ double rows[FDA_MAX_SKETCH_ROWS];
  const int tid = threadIdx.x;
  const int bpr = (a.m + kEstCols - 1) / kEstCols;
  if (a.variants & FDA_VARIANT_SKETCH) {
    const int pieces = per == 1 ? bpr : (a.m + 31) / 32;     // of one row
    const int items = a.l * bpr * per;
    for (int t0 = 0; t0 < items; t0 += (int)blockDim.x) {    // one piece per thread, per (1 or 8) neighbours to a block
      const int t = t0 + tid, blk = t / per, i = blk / bpr, q = (blk - i * bpr) * per + (t - blk * per);
      const double x = t < items && q < pieces ? agent_load(part + 2 + i * pieces + q) : 0.0;
      double s = 0.0;
      for (int e = 0; e < per; ++e) s += __shfl(x, e, per);
      if (t < items && t == blk * per) blocks[blk] = s;
    }
    __syncthreads();
    if (tid < a.l) {
      double s = 0.0;
      for (int b = 0; b < bpr; ++b) s += blocks[tid * bpr + b];
      rows[tid] = s;
    }
    __syncthreads();
  }
  if (tid == 0) decide(a, agent_load(part), agent_load(part + 1), rows, state_path);
}
// sums of the two scalar components over the K states (of the first 256 threads of a workgroup)
__device__ inline void scalar_sums(const float* state, int K, int S, double* scratch, double* part) {
  double vn = 0.0, vp = 0.0;
  if (threadIdx.x < kSmallThreads)
    for (int k = threadIdx.x; k < K; k += kSmallThreads) {
      vn += (double)state[(size_t)k * S];
      vp += (double)state[(size_t)k * S + 1];
    }
  const double sn = block_sum(vn, scratch);
  const double sp = block_sum(vp, scratch);
  if (threadIdx.x == 0) { agent_store(part, sn); agent_store(part + 1, sp); }
}
// Workgroup b takes 256 consecutive cells of one sketch row (one cell per thread: mean over the
// K workers, squared, summed over the workgroup); workgroup 0 also takes the scalar components.
// The workgroup that finishes last takes the median and writes the result.  `ticket` counts finished
// workgroups and is left at 0.
__global__ void __launch_bounds__(kSmallThreads)
estimate_kernel(const float* __restrict__ state, EstimateArgs a, double* __restrict__ part,
                unsigned int* __restrict__ ticket, const PathRecord* __restrict__ path) {
  __shared__ double scratch[kSmallThreads / 32];
  __shared__ int last;
  const int cells = (a.variants & FDA_VARIANT_SKETCH) ? a.l * a.m : 0;
  const int S = 2 + cells;
  const int bpr = (a.m + kEstCols - 1) / kEstCols;   // workgroups per sketch row
  const int tid = threadIdx.x;
  // part[0], part[1]: sums of the two scalar components; part[2 + b]: workgroup b's row sum
  if (cells) {
    const int i = blockIdx.x / bpr, col = (blockIdx.x - i * bpr) * kEstCols + tid;
    double sq = 0.0;
    if (col < a.m) {
      double c = 0.0;
      for (int k0 = 0; k0 < a.K; k0 += 16) {       // the loads of 16 workers together, added in order
        float x[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) x[t] = state[(size_t)(k0 + t < a.K ? k0 + t : k0) * S + 2 + i * a.m + col];
#pragma unroll
        for (int t = 0; t < 16; ++t) c += k0 + t < a.K ? (double)x[t] : 0.0;
      }
      c /= (double)a.K;
      sq = c * c;
    }
    sq = half_wave_sum(sq);
    if ((tid & 31) == 0) scratch[tid >> 5] = sq;
    __syncthreads();
    if (tid == 0) {
      double r = 0.0;
      for (int q = 0; q < kSmallThreads / 32; ++q) r += scratch[q];
      agent_store(part + 2 + blockIdx.x, r);
    }
    __syncthreads();
  }
  if (blockIdx.x == 0) scalar_sums(state, a.K, S, scratch, part);
  if (!finished_last(ticket, (int)gridDim.x, &last)) return;
  // which kind of sketch cell the last state pass used
  finish_estimate(a, part, 1, cells && path != nullptr ? path->last : -1);
  if (tid == 0) *ticket = 0u;
}

// ----------------------------------------------------------------------------------------
// state[k][s] = sum over the partitions in fp64, of the partials of state_kernel (rows = K) or of
// mean_state_kernel (rows = 1; the result is divided by K, and one entry past the state, the summed squared
// norm of the model change, goes to *dnorm for fda_sync_from_mean).
// Workgroup 0 takes the scalar components.  The others take 32 neighbouring cells of one sketch row for `wl`
// workers each: 512 threads = 32 cells x wl workers x slices of the partitions.  A wave's loads are whole
// 128-byte runs, and the host splits the partitions so that a thread has about 16 of them: what bounds the
// kernel is their latency (the partials were just written by other XCDs; with all workers of 32 cells in one
// workgroup, up to 130 loads per thread, it took 52 us on cfg3 where it takes 9).  The slices are added in order:
// a fixed shape.
// With est.out != NULL the estimate follows in the same launch (7 us on cfg1, 13 on cfg3, 18 on cfg4, where
// the two kernels took 13, 18 and 23 and the gap between them).  The workgroup that is the last to finish
// among those of 32 cells averages them over the workers and leaves the sum of their squares; the last of
// all takes the median.
// ----------------------------------------------------------------------------------------
struct FinishParams {
  const double* part_np;           // [P][K][2], or [P][3]
  const unsigned char* part_sk;
  const CellUnit* units;           // [P][G][R]
  PathRecord* path;
  float* state;
  double* dnorm;                   // mean-state pass only (else NULL)
  unsigned int* ticket;            // [0]: all workgroups, then one per 32 cells; zero, left at zero
  double* est_part;
  int rows, K, l, m, P, G, R;      // l = m = 0: no sketch
  int wl;                          // 1, 2, 4, 8 or 16
  EstimateArgs est;                // est.out == NULL: no estimate
};
constexpr int kFinishThreads = 512;
constexpr int kFinishCols = 32;
constexpr int kFinishLanes = kFinishThreads / kFinishCols;
constexpr int kFinishStates = 64;  // workers averaged at a time
constexpr int kFinishLoads = 16;   // partials per thread the host aims at
// ... and loads at once: all of the 4-byte ones, 8 of the 8-byte ones of the average state, which has four or five to a
// thread where the vector is short (16 were repeats of the first for the most part: 11 x 123457 fp32 with its
// synchronization 25.2 us a step, now 23.9; 8 x 200000 30.2, now 28.8; 4 at once are no faster).
constexpr int kMeanLoads = 8;

// sum over the partitions slice, slice + slices, ... of value times unit.  The loads of a batch of N are issued
// together (those past the end repeat the first one).  For the 4-byte sums nothing may move across the end of the
// loads: beside the shorter batch of the 8-byte ones the compiler waited for the first partition before it issued
// the other fifteen, a second latency (5 x 61706 fp32 17.35 -> 17.5 us a step; as it is now 17.0, in 65 registers for
// 76; 16 x 2.6M 57.3, now 56.5).  The 8-byte loads are together without it, and with it 11 x 123457 takes 48.2 us for
// 47.9.
template <int N, typename V>
__device__ __forceinline__ double sum_partials(const V* q, size_t step, const CellUnit* un, int GR, int slice, int slices, int P) {
  double acc = 0.0;
  for (int p0 = slice; p0 < P; p0 += N * slices) {
    V x[N];
    double unit[N];
#pragma unroll
    for (int t = 0; t < N; ++t) {
      const int p = p0 + t * slices < P ? p0 + t * slices : p0;
      x[t] = q[p * step];
      unit[t] = un[(size_t)p * GR].unit;
    }
    if constexpr (sizeof(V) == 4) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < N; ++t) acc += p0 + t * slices < P ? unit[t] * (double)x[t] : 0.0;
  }
  return acc;
}

// The same where some workgroups redid their sketch: the kind of each partition says where its sum lies and how wide it
// is, so the units of a batch are loaded together and then its sums: two latencies for four partitions, where one after
// the other took two for each.  (One drift 2^14 times the others, us a call, state and average state: 16 x 2.6M fp32
// 217 and 62.8, now 212 and 57.8; 7 x 18M bf16 669 and 137.7, now 663 and 125.9; 8 x 3000001 bf16 147.7 and 53.7, now
// 143.0 and 42.7.  Batches of 16 are no faster, hold 129 registers and cost every call the second
// workgroup of a CU: 7 x 18M without such a drift 141.4 us a step for 138.0.)
constexpr int kKindLoads = 4;
__device__ __forceinline__ double sum_partials_by_kind(const unsigned char* base, size_t cell, size_t step, const CellUnit* un,
                                                       int GR, int slice, int slices, int P) {
  double acc = 0.0;
  for (int p0 = slice; p0 < P; p0 += kKindLoads * slices) {
    CellUnit u[kKindLoads];
    uint32_t lo[kKindLoads], hi[kKindLoads];
#pragma unroll
    for (int t = 0; t < kKindLoads; ++t) u[t] = un[(size_t)(p0 + t * slices < P ? p0 + t * slices : p0) * GR];
#pragma unroll
    for (int t = 0; t < kKindLoads; ++t) {
      const int p = p0 + t * slices < P ? p0 + t * slices : p0;
      const bool narrow = u[t].kind == kCellI32;
      const uint32_t* q = reinterpret_cast<const uint32_t*>(base + p * step) + (narrow ? cell : 2 * cell);
      lo[t] = q[0];
      hi[t] = q[narrow ? 0 : 1];
    }
#pragma unroll
    for (int t = 0; t < kKindLoads; ++t) {
      const long long wide = (long long)(((unsigned long long)hi[t] << 32) | lo[t]);
      const double x = u[t].kind == kCellI32   ? (double)(int)lo[t]
                       : u[t].kind == kCellI64 ? (double)wide
                                               : __longlong_as_double(wide);
      acc += p0 + t * slices < P ? u[t].unit * x : 0.0;
    }
  }
  return acc;
}

__global__ void __launch_bounds__(kFinishThreads)
finish_kernel(const FinishParams f) {
  __shared__ double sh[kFinishLanes][kFinishCols];
  __shared__ float st[kFinishStates][kFinishCols];
  __shared__ double scratch[kFinishThreads / 64];
  __shared__ int last;
  const int tid = threadIdx.x;
  const bool mean = f.dnorm != nullptr;
  const int cells = f.l * f.m, S = 2 + cells;
  // 0: every partial is of the kind the pass aims at (int32, mean-state pass int64)
  const int path = f.path->now;
  if (blockIdx.x == 0) {
    double (*s8)[64] = reinterpret_cast<double (*)[64]>(&sh[0][0]);        // [8][64]
    const int e0 = tid & 63, slice = tid >> 6;
    const int width = mean ? 3 : 2 * f.K;
    for (int eb = 0; eb < width; eb += 64) {
      const int e = eb + e0;
      double acc = 0.0;
      if (e < width) {
        for (int p0 = slice; p0 < f.P; p0 += 8 * kFinishLoads) {
          double x[kFinishLoads];
#pragma unroll
          for (int t = 0; t < kFinishLoads; ++t) x[t] = f.part_np[(size_t)(p0 + t * 8 < f.P ? p0 + t * 8 : p0) * width + e];
#pragma unroll
          for (int t = 0; t < kFinishLoads; ++t) acc += p0 + t * 8 < f.P ? x[t] : 0.0;
        }
      }
      s8[slice][e0] = acc;
      __syncthreads();
      if (slice == 0 && e < width) {
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) t += s8[q][e0];
        if (!mean) f.state[(size_t)(e >> 1) * S + (e & 1)] = (float)t;
        else if (e < 2) f.state[e] = (float)(t / (double)f.K);
        else *f.dnorm = t;
      }
      __syncthreads();
    }
    if (f.est.out != nullptr) scalar_sums(f.state, f.rows, S, scratch, f.est_part);
  } else {
    const int cb = (f.m + kFinishCols - 1) / kFinishCols;                  // runs of 32 cells per sketch row
    const int chunks = (f.rows + f.wl - 1) / f.wl;                         // workgroups per run
    const int b = ((int)blockIdx.x - 1) / chunks, k0 = ((int)blockIdx.x - 1 - b * chunks) * f.wl;
    const int i = b / cb;
    const int r = group_of(f.l, f.R, i);
    int rstart, rcnt;
    group_range(f.l, f.R, r, &rstart, &rcnt);
    const int col = tid & (kFinishCols - 1), y = tid / kFinishCols;
    const int c = (b - i * cb) * kFinishCols + col;
    const int slices = kFinishLanes / f.wl, kk = y & (f.wl - 1), slice = y / f.wl;
    const int GR = f.G * f.R;
    const size_t pstep = (size_t)f.rows * cells;                           // places of one partition
    const size_t in_group = (size_t)(i - rstart) * f.m + c;
    const int k = k0 + kk;
    const bool live = k < f.rows && c < f.m;
    double acc = 0.0;
    if (live) {
      const unsigned char* const base = f.part_sk + ((size_t)k * cells + (size_t)rstart * f.m) * 8;
      const CellUnit* const un = f.units + (f.rows > 1 ? group_of(f.rows, f.G, k) * f.R : 0) + r;
      if (path != 0) {
        acc = sum_partials_by_kind(base, in_group, pstep * 8, un, GR, slice, slices, f.P);
      } else if (mean) {
        acc = sum_partials<kMeanLoads>(reinterpret_cast<const long long*>(base) + in_group, pstep, un, GR, slice, slices, f.P);
      } else {
        acc = sum_partials<kFinishLoads>(reinterpret_cast<const int*>(base) + in_group, pstep * 2, un, GR, slice, slices, f.P);
      }
    }
    sh[y][col] = acc;
    __syncthreads();
    if (slice == 0) {
      double t = 0.0;
      for (int q = 0; q < slices; ++q) t += sh[q * f.wl + kk][col];
      const float v = (float)(mean ? t / (double)f.K : t);
      if (live) agent_store(f.state + (size_t)k * S + 2 + (size_t)i * f.m + c, v);
      st[kk][col] = v;
    }
    __syncthreads();
    // (only the last workgroup of a run goes on to the counter of the launch: hundreds of additions to one
    // address take microseconds)
    if (chunks > 1 && !finished_last(f.ticket + 1 + b, chunks, &last)) return;
    if (f.est.out != nullptr) {
      double avg = 0.0;
      if (chunks == 1) {
        if (y == 0)
          for (int q = 0; q < f.rows; ++q) avg += (double)st[q][col];
      } else {
        for (int kb = 0; kb < f.rows; kb += kFinishStates) {
          float x[kFinishStates / kFinishLanes];
#pragma unroll
          for (int q = 0; q < kFinishStates / kFinishLanes; ++q) {
            const int kq = kb + q * kFinishLanes + y;
            x[q] = kq < f.rows && c < f.m ? agent_load(f.state + (size_t)kq * S + 2 + (size_t)i * f.m + c) : 0.0f;
          }
#pragma unroll
          for (int q = 0; q < kFinishStates / kFinishLanes; ++q) st[q * kFinishLanes + y][col] = x[q];
          __syncthreads();
          if (y == 0)
            for (int q = 0; q < kFinishStates && kb + q < f.rows; ++q) avg += (double)st[q][col];
          __syncthreads();
        }
      }
      if (tid < 64) {
        avg /= (double)f.rows;
        const double s = half_wave_sum(y == 0 && c < f.m ? avg * avg : 0.0);
        if (tid == 0) agent_store(f.est_part + 2 + b, s);
      }
    }
    if (chunks > 1 && tid == 0) f.ticket[1 + b] = 0u;
  }
  const int runs = f.l * ((f.m + kFinishCols - 1) / kFinishCols);
  if (!finished_last(f.ticket, runs + 1, &last)) return;
  if (f.est.out != nullptr) finish_estimate(f.est, f.est_part, kEstCols / kFinishCols, cells ? path : -1);
  if (tid == 0) {
    f.path->last = path;
    f.path->now = 0;
    *f.ticket = 0u;
  }
}

// ----------------------------------------------------------------------------------------
// Algorithm 1 line 9: read the K rows once, average in fp32 in worker order, write the
// average to every row, to w_t0, and the old w_t0 to w_prev.  Or (sync_from_mean_kernel) the same when the
// average model is already there, with the xi of Section 3.2.
//
// Both are bound by HBM.  A workgroup takes one block of 4096 coordinates (two, and so on, where that would be
// more than 49152 workgroups): workgroups launched in address order work on neighbouring addresses of every
// row when they run together, which is what keeps the K + 2 interleaved read and write streams efficient in DRAM
// (2048 workgroups that take every 2048th block: 5.1 instead of 5.5 TB/s on 8 x 150 000 000 bf16; ranges of
// hundreds of KiB per workgroup: 3.5).  The limit is for launches whose predicate is zero, which cost 0.2 ns
// per workgroup (350M coordinates: 21 us, now 12).  A lane owns 4 consecutive coordinates of a wave's 256 (16 bytes
// of fp32, 8 bytes of bf16), so the fp32 vectors are moved in whole lines.  STREAM: every byte is read once
// and written once, so loads and stores carry the nontemporal hint -- chosen by the host for slabs
// too large to stay in the memory-side cache, where it gains 3-8 %; small slabs lose by it.
//
// The rows of a slab whose row length is no multiple of 128 bytes start anywhere in a line.  Storing to them
// with the lanes of the average would split one line of every four (bf16; eight for fp32) between two store
// instructions, and partly written lines cost DRAM a read: 8 x 150 000 001 bf16 ran at 4.0 TB/s where
// 8 x 150 000 000 ran at 5.1.  So the average goes through LDS, and every row is stored in 16-byte vectors
// counted from its own first line boundary; one line in 64 (fp32: 128) is split.
// ----------------------------------------------------------------------------------------
constexpr int kSyncV = 4;                    // coordinates per lane and vector
constexpr int kSyncVecs = 4;                 // vectors per thread and block: 4096 coordinates ...
constexpr int kSyncVecsSmall = 1;            // ... or 1024, where the larger blocks would not fill the chip
__host__ __device__ constexpr int sync_block(int vecs) { return vecs * kSyncV * kSmallThreads; }

template <typename VecT, bool NT>
__device__ __forceinline__ void store_vec_hint(void* p, VecT v) {
  if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<VecT*>(p));
  else *reinterpret_cast<VecT*>(p) = v;
}
// 4 slab elements at p as floats
template <bool NT>
__device__ __forceinline__ void load_slab4(const float* p, float (&x)[4]) {
  const f32x4 t = load_vec_hint<f32x4, NT>(p);
  x[0] = t.x; x[1] = t.y; x[2] = t.z; x[3] = t.w;
}
template <bool NT>
__device__ __forceinline__ void load_slab4(const bf16_t* p, float (&x)[4]) {
  const u32x2_h t = load_vec_hint<u32x2_h, NT>(p);
  x[0] = __uint_as_float(t.x << 16); x[1] = __uint_as_float(t.x & 0xffff0000u);
  x[2] = __uint_as_float(t.y << 16); x[3] = __uint_as_float(t.y & 0xffff0000u);
}
template <bool NT>
__device__ __forceinline__ void store_f32x4(float* p, const float (&x)[4]) {
  const f32x4 t = {x[0], x[1], x[2], x[3]};
  store_vec_hint<f32x4, NT>(p, t);
}
// what a slab row stores for 4 averaged values (the fp32 values, or their bf16 roundings), into the block's
// image in LDS
__device__ __forceinline__ void stage4(uint32_t* img, int e, const float (&x)[4], const float*) {
  const u32x4_a16 t = {__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3])};
  *reinterpret_cast<u32x4_a16*>(img + e) = t;
}
__device__ __forceinline__ void stage4(uint32_t* img, int e, const float (&x)[4], const bf16_t*) {
  const u32x2_a8 t = {f32_to_bf16_rne(x[0]) | (f32_to_bf16_rne(x[1]) << 16),
                      f32_to_bf16_rne(x[2]) | (f32_to_bf16_rne(x[3]) << 16)};
  *reinterpret_cast<u32x2_a8*>(img + e / 2) = t;
}
// The image's first n elements to the K rows, from element c0 of each.
template <typename T, bool NT>
__device__ __forceinline__ void store_rows(T* w, long long row_stride, int K, long long c0, int n, const uint32_t* img) {
  constexpr int kPer = 16 / (int)sizeof(T);          // elements of a 16-byte vector
  const int tid = threadIdx.x;
  const T* const elems = reinterpret_cast<const T*>(img);
  for (int k = 0; k < K; ++k) {
    T* const row = w + (long long)k * row_stride + c0;
    const int off = (int)(reinterpret_cast<uintptr_t>(row) & 127u);
    int head = off == 0 ? 0 : (128 - off) / (int)sizeof(T);      // elements in front of the row's first line boundary
    if (head > n) head = n;
    const int nvec = (n - head) / kPer;
    const int odd = sizeof(T) == 2 ? head & 1 : 0;
    for (int v = tid; v < nvec; v += kSmallThreads) {
      const int e = head + v * kPer;
      const uint32_t* src = img + (sizeof(T) == 2 ? e >> 1 : e);
      u32x4_a16 t = {src[0], src[1], src[2], src[3]};
      if (odd) {                                     // (the same for the whole row)
        const uint32_t next = src[4];
        t = u32x4_a16{__builtin_amdgcn_alignbit(t.y, t.x, 16), __builtin_amdgcn_alignbit(t.z, t.y, 16),
                      __builtin_amdgcn_alignbit(t.w, t.z, 16), __builtin_amdgcn_alignbit(next, t.w, 16)};
      }
      store_vec_hint<u32x4_a16, NT>(row + e, t);
    }
    // the elements in front (fewer than 64) and behind the vectors (fewer than 8)
    if (tid < head) row[tid] = elems[tid];
    const int done = head + nvec * kPer;
    if (tid >= 64 && tid - 64 < n - done) row[done + tid - 64] = elems[done + tid - 64];
  }
}

constexpr int kSyncGroup = 64;       // workgroups whose shares of the norm are added up in the launch
template <typename T, bool STREAM, int VECS>
__global__ void __launch_bounds__(kSmallThreads)
sync_kernel(T* __restrict__ w, float* __restrict__ w_t0, float* __restrict__ w_prev,
            const int32_t* __restrict__ pred, int K, long long d, long long row_stride, int per,
            double* __restrict__ norm_part, double* __restrict__ norm_group, unsigned int* __restrict__ ticket) {
  // norm_part != NULL: entry [workgroup] receives the workgroup's share of ||new w_t0 - old w_t0||^2
  // (fp32 squares of four coordinates, then fp64), which saves the refresh of xi its pass over both vectors.
  // The last of 64 neighbouring workgroups to finish adds their shares up, in order, into norm_group (a launch
  // of its own for that cost every step 4.7 us, also where nothing is synchronized).
  constexpr int V = kSyncV, kBlock = sync_block(VECS), H = VECS >= 2 ? 2 : 1;
  __shared__ double scratch[kSmallThreads / 64];
  __shared__ int last;
  __shared__ __align__(16) uint32_t img[kBlock * sizeof(T) / 4 + 4];
  if (pred != nullptr && *pred == 0) return;
  double nacc = 0.0;
  const float kf = (float)K;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const long long cbeg = (long long)blockIdx.x * per * kBlock;
  for (long long c0 = cbeg; c0 < cbeg + (long long)per * kBlock && c0 < d; c0 += kBlock) {
    const int n = d - c0 < kBlock ? (int)(d - c0) : kBlock;
#pragma unroll 1
    for (int q = 0; q < VECS; q += H) {
      // two vectors next to each other (a wave's 512 coordinates): the line they share is fetched once
      const int e0 = (wave * VECS + q) * 64 * V + lane * V;
      if (e0 + (H - 1) * 64 * V + V <= n) {
        float acc[H][V];
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
          for (int v = 0; v < V; ++v) acc[h][v] = 0.0f;
        const T* src = w + c0 + e0;
#pragma unroll 8
        for (int k = 0; k < K; ++k) {
#pragma unroll
          for (int h = 0; h < H; ++h) {
            float x[V];
            load_slab4<STREAM>(src + (long long)k * row_stride + h * 64 * V, x);
#pragma unroll
            for (int v = 0; v < V; ++v) acc[h][v] += x[v];
          }
        }
#pragma unroll
        for (int h = 0; h < H; ++h) {
          const long long j0 = c0 + e0 + h * 64 * V;
#pragma unroll
          for (int v = 0; v < V; ++v) acc[h][v] = acc[h][v] / kf;
          if (w_prev != nullptr || norm_part != nullptr) {
            float old[V];
            load_f32_vec<V, STREAM>(w_t0 + j0, old);
            if (w_prev != nullptr) store_f32x4<STREAM>(w_prev + j0, old);
            if (norm_part != nullptr) {
              const float dx = acc[h][0] - old[0], dy = acc[h][1] - old[1], dz = acc[h][2] - old[2], dw = acc[h][3] - old[3];
              nacc += (double)fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, dw * dw)));
            }
          }
          store_f32x4<STREAM>(w_t0 + j0, acc[h]);
          stage4(img, e0 + h * 64 * V, acc[h], static_cast<const T*>(nullptr));
        }
      } else {
        for (int h = 0; h < H; ++h)
          for (int v = 0; v < V; ++v) {
            const int e = e0 + h * 64 * V + v;
            if (e >= n) break;
            float a = 0.0f;
            for (int k = 0; k < K; ++k) a += Slab<T>::load_one(w + (long long)k * row_stride + c0 + e);
            a = a / kf;
            const float o = w_t0[c0 + e];
            if (w_prev != nullptr) w_prev[c0 + e] = o;
            if (norm_part != nullptr) nacc += (double)((a - o) * (a - o));
            w_t0[c0 + e] = a;
            Slab<T>::store_one(reinterpret_cast<T*>(img) + e, a);
          }
      }
    }
    __syncthreads();
    store_rows<T, STREAM>(w, row_stride, K, c0, n, img);
    __syncthreads();
  }
  if (norm_part != nullptr) {
    const double s = block_sum(nacc, scratch);
    if (threadIdx.x == 0) agent_store(norm_part + blockIdx.x, s);
    const int g = blockIdx.x / kSyncGroup, first = g * kSyncGroup;
    const int count = (int)gridDim.x - first < kSyncGroup ? (int)gridDim.x - first : kSyncGroup;
    if (!finished_last(ticket + g, count, &last)) return;
    if (threadIdx.x < 64) {
      const double t = wave_sum((int)threadIdx.x < count ? agent_load(norm_part + first + threadIdx.x) : 0.0);
      if (threadIdx.x == 0) { norm_group[g] = t; ticket[g] = 0u; }
    }
  }
}

// Algorithm 1 line 9 when the average model is already there (w_bar from mean_state_kernel):
// every row <- w_bar, w_prev <- w_t0, w_t0 <- w_bar, and (xi != NULL) the xi of Section 3.2,
// (w_bar - old w_t0) / ||w_bar - old w_t0||, with the squared norm taken from *dnorm.
// Workgroups (x, y) store `rows` rows of the same block, those of y = 0 the models: a small vector has too few blocks
// to fill the chip, and a workgroup stores its rows one after the other (all rows: 60 x 30000 fp32 12.6 us, 300 x 5000
// 50.4; split 5.4 and 5.1).
template <typename T, bool STREAM, int VECS>
__global__ void __launch_bounds__(kSmallThreads)
sync_from_mean_kernel(T* __restrict__ w, float* __restrict__ w_t0, float* __restrict__ w_prev,
                      float* __restrict__ xi, const float* __restrict__ w_bar,
                      const double* __restrict__ dnorm, const int32_t* __restrict__ pred, int K, int rows,
                      long long d, long long row_stride, int per) {
  constexpr int V = kSyncV, kBlock = sync_block(VECS);
  __shared__ __align__(16) uint32_t img[kBlock * sizeof(T) / 4 + 4];
  if (pred != nullptr && *pred == 0) return;
  const int k0 = (int)blockIdx.y * rows, krows = K - k0 < rows ? K - k0 : rows;
  const bool models = blockIdx.y == 0;
  float scale = 0.0f;
  if (xi != nullptr && models) {
    const double nrm = sqrt(*dnorm);
    scale = (nrm > 0.0 && isfinite(nrm)) ? (float)(1.0 / nrm) : 0.0f;
  }
  const long long cbeg = (long long)blockIdx.x * per * kBlock;
  for (long long c0 = cbeg; c0 < cbeg + (long long)per * kBlock && c0 < d; c0 += kBlock) {
    const int n = d - c0 < kBlock ? (int)(d - c0) : kBlock;
#pragma unroll
    for (int q = 0; q < VECS; ++q) {
      const int e0 = (q * kSmallThreads + (int)threadIdx.x) * V;
      const long long j0 = c0 + e0;
      if (e0 + V <= n) {
        float nb[V];
        load_f32_vec<V, STREAM>(w_bar + j0, nb);
        if (models) {
          float old[V];
          load_f32_vec<V, STREAM>(w_t0 + j0, old);
          if (w_prev != nullptr) store_f32x4<STREAM>(w_prev + j0, old);
          store_f32x4<STREAM>(w_t0 + j0, nb);
          if (xi != nullptr) {
            float x[V];
#pragma unroll
            for (int v = 0; v < V; ++v) x[v] = (scale == 0.0f) ? 0.0f : (nb[v] - old[v]) * scale;
            store_f32x4<STREAM>(xi + j0, x);
          }
        }
        stage4(img, e0, nb, static_cast<const T*>(nullptr));
      } else {
        for (int v = 0; v < V; ++v) {
          if (e0 + v >= n) break;
          const float a = w_bar[j0 + v];
          if (models) {
            const float o = w_t0[j0 + v];
            if (w_prev != nullptr) w_prev[j0 + v] = o;
            w_t0[j0 + v] = a;
            if (xi != nullptr) xi[j0 + v] = (scale == 0.0f) ? 0.0f : (a - o) * scale;
          }
          Slab<T>::store_one(reinterpret_cast<T*>(img) + e0 + v, a);
        }
      }
    }
    __syncthreads();
    store_rows<T, STREAM>(w + (long long)k0 * row_stride, row_stride, krows, c0, n, img);
    __syncthreads();
  }
}

// ----------------------------------------------------------------------------------------
// Section 3.2: xi = (w_t0 - w_prev) / ||w_t0 - w_prev||.  Pass 1: per-workgroup partial of
// the squared norm; pass 2: every workgroup re-sums the partials in the same fixed order
// and scales its share of the difference.
//
// Both are bound by HBM.  As in the synchronization a workgroup takes blocks of neighbouring coordinates, all
// loads of a block in flight together, with the nontemporal hint for vectors far beyond the memory-side cache;
// in pass 2 the first block's loads wait together with those of the partials.  (Strides of the whole grid, one
// vector in flight, no hints: both passes 632 us for 150M coordinates, now 488; 20M 67 and 60; 7M 28 and 23.)
// ----------------------------------------------------------------------------------------
template <bool STREAM>
__global__ void __launch_bounds__(kSmallThreads)
xi_norm_kernel(const float* __restrict__ w_t0, const float* __restrict__ w_prev,
               const int32_t* __restrict__ pred, long long d, double* __restrict__ partial) {
  constexpr int V = kSyncV, VECS = kSyncVecs, kBlock = sync_block(VECS);
  __shared__ double scratch[kSmallThreads / 64];
  if (pred != nullptr && *pred == 0) return;
  double acc = 0.0;
  for (long long c0 = (long long)blockIdx.x * kBlock; c0 < d; c0 += (long long)gridDim.x * kBlock) {
    float a[VECS][V], b[VECS][V];
#pragma unroll
    for (int q = 0; q < VECS; ++q) {
      const long long j0 = c0 + (q * kSmallThreads + (int)threadIdx.x) * V;
#pragma unroll
      for (int v = 0; v < V; ++v) a[q][v] = b[q][v] = 0.0f;
      if (j0 + V <= d) {
        load_f32_vec<V, STREAM>(w_t0 + j0, a[q]);
        load_f32_vec<V, STREAM>(w_prev + j0, b[q]);
      } else {
#pragma unroll
        for (int v = 0; v < V; ++v)
          if (j0 + v < d) { a[q][v] = w_t0[j0 + v]; b[q][v] = w_prev[j0 + v]; }
      }
    }
#pragma unroll
    for (int q = 0; q < VECS; ++q) {
      const float dx = a[q][0] - b[q][0], dy = a[q][1] - b[q][1], dz = a[q][2] - b[q][2], dw = a[q][3] - b[q][3];
      acc += (double)fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, dw * dw)));   // a short fp32 run, then fp64
    }
  }
  const double s = block_sum(acc, scratch);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// Workgroup b takes the `per` blocks from block b * per.
template <bool STREAM, int VECS>
__global__ void __launch_bounds__(kSmallThreads)
xi_scale_kernel(const float* __restrict__ w_t0, const float* __restrict__ w_prev,
                float* __restrict__ xi, const int32_t* __restrict__ pred, long long d, int per,
                const double* __restrict__ partial, int npartial) {
  constexpr int V = kSyncV, kBlock = sync_block(VECS);
  __shared__ double scratch[kSmallThreads / 64];
  __shared__ float scale_sh;
  if (pred != nullptr && *pred == 0) return;
  float a[VECS][V], b[VECS][V];
  auto load = [&](long long c0) {
#pragma unroll
    for (int q = 0; q < VECS; ++q) {
      const long long j0 = c0 + (q * kSmallThreads + (int)threadIdx.x) * V;
      if (j0 + V <= d) {
        load_f32_vec<V, STREAM>(w_t0 + j0, a[q]);
        load_f32_vec<V, STREAM>(w_prev + j0, b[q]);
      }
    }
  };
  const long long cbeg = (long long)blockIdx.x * per * kBlock, cend = cbeg + (long long)per * kBlock;
  load(cbeg);
  double acc = 0.0;
#pragma unroll 4
  for (int t = threadIdx.x; t < npartial; t += kSmallThreads) acc += partial[t];
  const double tot = block_sum(acc, scratch);
  if (threadIdx.x == 0) {
    const double nrm = sqrt(tot);
    scale_sh = (nrm > 0.0 && isfinite(nrm)) ? (float)(1.0 / nrm) : 0.0f;
  }
  __syncthreads();
  const float scale = scale_sh;
  for (long long c0 = cbeg; c0 < d;) {
#pragma unroll
    for (int q = 0; q < VECS; ++q) {
      const long long j0 = c0 + (q * kSmallThreads + (int)threadIdx.x) * V;
      if (j0 + V <= d) {
        float x[V];
#pragma unroll
        for (int v = 0; v < V; ++v) x[v] = (scale == 0.0f) ? 0.0f : (a[q][v] - b[q][v]) * scale;
        store_f32x4<STREAM>(xi + j0, x);
      } else {
        for (int v = 0; v < V && j0 + v < d; ++v)
          xi[j0 + v] = (scale == 0.0f) ? 0.0f : (w_t0[j0 + v] - w_prev[j0 + v]) * scale;
      }
    }
    c0 += kBlock;
    if (c0 >= cend) break;
    load(c0);
  }
}

}  // namespace fda

// Device code of the FDA monitor for gfx950 (wave64): the mean-state kernel.
//
// Algorithm 1 line 7 needs only the average state.  With all K workers in one address space the
// linearity of the AMS sketch (Section 3.1: sk(a u + b v) = a sk(u) + b sk(v)) gives it
// directly:  mean_k sk(u_k) = sk(mean_k u_k),  mean_k <xi,u_k> = <xi, mean_k u_k>,  so the
// sketch costs l LDS additions per coordinate instead of l*K and the pass is bound by the HBM
// stream again.  (The per-worker states of Algorithm 1 line 6 stay with state_kernel.)
//
// Workgroup (p, r) streams coordinates [p*chunk, (p+1)*chunk) of ALL K workers exactly once, in
// batches of KB slab rows, and owns the sketch rows of row group r (R > 1 only when l*m 8-byte
// cells do not fit in LDS; then every row group repeats the loads).  Per tile a lane owns V
// consecutive coordinates; for each it sums the K drifts, accumulates sum_k u^2 and <xi,u>
// (fp32 within the tile, fp64 across tiles; row group 0 only), and at the end of the tile adds
// sign * (sum of the K drifts) into the LDS sketch [row][bucket] once per sketch row.
// On request (w_bar != NULL) row group 0 also writes the average model w_t0 + mean_k u_k and
// accumulates the squared norm of what fda_sync_from_mean will see as the model change,
// (w_bar - w_t0) as rounded to fp32 -- Algorithm 1 line 9 and the xi of Section 3.2 then need
// no second pass over the slab.
//
// A drift enters as the integer round(u * Sm) (Sm: the workgroup's own unit, from a sample of its drifts,
// see fda_kernels.hpp; every scaled drift must stay below 2^30); the K integers of a coordinate are summed in
// 64 bits and added to 64-bit cells.  All of it is exact, so the result does not depend on the order of
// additions.  |sum of a cell| < K * chunk * 2^30, which the host keeps below 2^63.  A workgroup that met a
// drift too large for its terms does its sketch once more with fp64 sums and ds_add_f64 cells.
#pragma once
#include "fda_kernels.hpp"

namespace fda {

struct MeanParams {
  const void* w;
  const float* w_t0;
  const float* xi;
  long long row_stride;
  long long d;
  long long chunk;        // coordinates per partition (multiple of the tile)
  int K;
  int l;
  int m;
  int R;                  // sketch-row groups
  int P;                  // coordinate partitions, multiple of 8
  int do_lin;
  int do_sk;
  int vec_ok;             // all pointers / strides allow whole-vector loads
  float* w_bar;           // [d] or NULL: receives w_t0 + mean_k u_k
  double* part_np;        // [P][3]: sum_k ||u_k||^2, sum_k <xi,u_k>, ||w_bar - w_t0||^2 of the partition
  unsigned char* part_sk; // [P][l*m] 8-byte values: int64 or double (CellUnit::kind)
  CellUnit* units;        // [P][R]
  PathRecord* path;
  const uint16_t* table;  // [R][dpad] records of the tabulated hash, one field per row slot
  long long dpad;
};

template <typename T, int KB>
struct MeanBatch {
  static constexpr int kWords = kStateV * (int)sizeof(T) / 4;
  uint32_t w[KB][kWords];       // V elements of each of KB slab rows
};
template <int LR, int FB>
struct MeanHead {
  float w0[kStateV];
  float x[kStateV];
  uint32_t rec[RecGeom<LR, FB>::kDwords];      // the V records of the tabulated hash
};

constexpr int kMeanSampleRows = 8;            // workers a thread samples (all of them, or 8 in turn)

template <typename T, int KB, int LR, int FB>
__global__ void __launch_bounds__(kStateThreads)
mean_state_kernel(const MeanParams prm) {
  constexpr int V = kStateV;
  constexpr long long kTile = (long long)kStateThreads * V;
  using Batch = MeanBatch<T, KB>;
  using Geom = RecGeom<LR, FB>;
  using Head = MeanHead<LR, FB>;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  // consecutive workgroup ids go round-robin over the 8 XCDs: the R workgroups that read the
  // same coordinates get ids on one XCD and its L2
  const int b = blockIdx.x;
  const int xcd = b & 7, slot = b >> 3;
  const int r = slot % prm.R;
  const int p = (slot / prm.R) * 8 + xcd;
  int rstart = 0, rcnt = 0;
  if (prm.do_sk) group_range(prm.l, prm.R, r, &rstart, &rcnt);
  const bool scalars = r == 0;

  const int cells = rcnt * prm.m;
  const uint32_t dummy_base = (uint32_t)cells * 8u;
  const int lds_cells = prm.do_sk ? cells + kDummyCells : 0;
  double* red = reinterpret_cast<double*>(lds_raw + (size_t)lds_cells * 8);
  const int tid = threadIdx.x;
  {
    unsigned long long* c64 = reinterpret_cast<unsigned long long*>(lds_raw);
    for (int t = tid; t < lds_cells; t += kStateThreads) c64[t] = 0ull;
  }

  // spare row slots: their table fields hold buckets below kDummyCells, sent to the dummy region
  uint32_t rowbase[LR];
#pragma unroll
  for (int i = 0; i < LR; ++i) rowbase[i] = i < rcnt ? (uint32_t)(i * prm.m) * 8u : dummy_base;
  const uint32_t* const recs =
      reinterpret_cast<const uint32_t*>(prm.table + (size_t)r * prm.dpad * Geom::kWords);

  const long long cbeg = (long long)p * prm.chunk;
  long long cend = cbeg + prm.chunk;
  if (cend > prm.d) cend = prm.d;
  const long long dlim = prm.d;
  const bool lin = prm.do_lin && scalars;
  const float* const w0p = prm.w_t0;
  const float* const xip = lin ? prm.xi : prm.w_t0;     // without LinearFDA: any readable vector
  const T* const wbase = reinterpret_cast<const T*>(prm.w);
  const long long rs = prm.row_stride;
  const int K = prm.K;
  const int NB = (K + KB - 1) / KB;                     // batches of slab rows per tile
  const int tail = K - (NB - 1) * KB;                   // rows of the last batch, 1..KB
  // the unit of this workgroup's sketch terms
  float Sm = 1.0f;
  bool sketch = false;
  if (prm.do_sk) {
    double typical = 0.0;
    if (cend > cbeg) {
      const long long sbeg = sample_begin(cbeg, cend), len = cend - sbeg;
      auto row_of = [&](int i, int t) {
        const int k = K <= kMeanSampleRows ? (i < K ? i : K - 1) : (int)(((unsigned)(t >> 3) * kMeanSampleRows + i) % (unsigned)K);
        return wbase + (long long)k * rs;
      };
      const int rows = K < kMeanSampleRows ? K : kMeanSampleRows;
      float* const scratch = reinterpret_cast<float*>(red);
      typical = sample_mean(sample_drifts<kMeanSampleRows, T>(row_of, rows, w0p, sbeg, len, 1),
                            len < kStateThreads ? len : kStateThreads, rows, scratch);
      if (typical == 0.0)
        typical = sample_mean(sample_drifts<kMeanSampleRows, T>(row_of, rows, w0p, 0, dlim, kSampleRunsGlobal),
                              dlim < kSampleRunsGlobal * kStateThreads ? dlim : kSampleRunsGlobal * kStateThreads, rows, scratch);
    }
    const float unit = unit_for(typical, 0);
    sketch = unit != 0.0f;                    // otherwise the pass only notes whether there is any drift at all
    if (sketch) Sm = unit;
  }
  __syncthreads();                            // (the cells are clear)
  float* const wbp = scalars ? prm.w_bar : nullptr;
  const float kf = (float)K;

  double dn = 0.0, dp = 0.0, dd = 0.0;
  float amax = 0.0f;

  // SC: this workgroup also produces the scalar components; SK: it accumulates sketch rows.
  // MX: it notes the largest drift.  WIDE: the sketch in fp64, unscaled.
  auto run = [&](auto sc_tag, auto sk_tag, auto mx_tag, auto wide_tag) {
    constexpr bool SC = decltype(sc_tag)::value;
    constexpr bool SK = decltype(sk_tag)::value;
    constexpr bool MX = decltype(mx_tag)::value;
    constexpr bool WIDE = decltype(wide_tag)::value;
    using Acc = std::conditional_t<WIDE, double, long long>;
    Acc acc[V];               // sum over the workers of round(u * Sm), or of u
    float um[V];              // scalar workgroups: sum over the workers of u, for the average model
    float sn = 0.0f, sp = 0.0f;
#pragma unroll
    for (int v = 0; v < V; ++v) { acc[v] = Acc(0); um[v] = 0.0f; }

    // slab rows k0 .. k0+KB-1 (rows past the last worker repeat it; consume() drops them)
    auto load_batch_fast = [&](Batch& bt, long long j0, int k0) {
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        const int row = (k0 + k < K) ? k0 + k : K - 1;
        const T* src = wbase + (long long)row * rs + j0;
        if constexpr (sizeof(T) == 4) {
          const u32x4 q = load_vec_hint<u32x4, kNtSlab>(src);
          bt.w[k][0] = q.x; bt.w[k][1] = q.y; bt.w[k][2] = q.z; bt.w[k][3] = q.w;
        } else {
          const u32x2_h q = load_vec_hint<u32x2_h, kNtSlab>(src);
          bt.w[k][0] = q.x; bt.w[k][1] = q.y;
        }
      }
    };
    auto load_batch_slow = [&](Batch& bt, long long j0, int k0) {
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        const int row = (k0 + k < K) ? k0 + k : K - 1;
        const T* src = wbase + (long long)row * rs + j0;
        if constexpr (sizeof(T) == 4) {
#pragma unroll
          for (int v = 0; v < 4; ++v)
            bt.w[k][v] = (j0 + v < dlim) ? __float_as_uint(Slab<T>::load_one(src + v)) : 0u;
        } else {
          const uint16_t* h = reinterpret_cast<const uint16_t*>(src);
#pragma unroll
          for (int v = 0; v < 4; v += 2) {
            const uint32_t lo = (j0 + v < dlim) ? (uint32_t)h[v] : 0u;
            const uint32_t hi = (j0 + v + 1 < dlim) ? (uint32_t)h[v + 1] : 0u;
            bt.w[k][v >> 1] = lo | (hi << 16);
          }
        }
      }
    };
    auto load_table = [&](Head& h, long long j0) {
      // the table is padded to dpad (whole blocks of 256 coordinates): always whole records
      if constexpr (SK)
        load_rec_block<Geom::kDwords, kNtSlab>(recs + (j0 >> 8) * (64 * Geom::kDwords), (int)(j0 >> 2) & 63, h.rec);
    };
    auto load_head_fast = [&](Head& h, long long j0) {
      load_f32_vec<V, kNtShared>(w0p + j0, h.w0);
      if constexpr (SC) load_f32_vec<V, kNtShared>(xip + j0, h.x);
      load_table(h, j0);
    };
    auto load_head_slow = [&](Head& h, long long j0) {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const bool in = (j0 + v < dlim);
        h.w0[v] = in ? w0p[j0 + v] : 0.0f;
        if constexpr (SC) h.x[v] = in ? xip[j0 + v] : 0.0f;
      }
      load_table(h, j0);
    };

    // one batch of rows; `live` of its KB rows are workers (the others contribute nothing)
    auto consume = [&](const Batch& bt, const Head& h, auto tail_tag, int live) {
      constexpr bool TAIL = decltype(tail_tag)::value;
#pragma unroll
      for (int k = 0; k < KB; ++k) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
          float u = raw_elem(bt.w[k], v) - h.w0[v];
          if constexpr (TAIL) u = (k < live) ? u : 0.0f;
          if constexpr (SC) {
            sn = fmaf(u, u, sn);
            sp = fmaf(h.x[v], u, sp);
            um[v] += u;
          }
          if constexpr (MX) amax = fmaxf(amax, fabsf(u));
          if constexpr (SK && WIDE) acc[v] += (double)u;
          else if constexpr (SK) acc[v] += (long long)round_half_up(u * Sm);
        }
      }
    };

    // end of a tile: the scalar partials go to fp64, the V sums into the sketch rows
    auto finish = [&](const Head& h, long long j0, bool whole) {
      if constexpr (SC) {
        dn += (double)sn; dp += (double)sp;
        sn = 0.0f; sp = 0.0f;
        if (wbp != nullptr) {
          float wb[V], sd = 0.0f;
#pragma unroll
          for (int v = 0; v < V; ++v) {
            wb[v] = h.w0[v] + um[v] / kf;
            const float df = wb[v] - h.w0[v];        // the model change as fp32 storage keeps it
            sd = fmaf(df, df, sd);
          }
          if (whole) {
            store_f32_vec<V>(wbp + j0, wb);
            dd += (double)sd;
          } else {
            sd = 0.0f;
#pragma unroll
            for (int v = 0; v < V; ++v)
              if (j0 + v < dlim) {
                wbp[j0 + v] = wb[v];
                const float df = wb[v] - h.w0[v];
                sd = fmaf(df, df, sd);
              }
            dd += (double)sd;
          }
        }
#pragma unroll
        for (int v = 0; v < V; ++v) um[v] = 0.0f;
      }
      if constexpr (SK) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
#pragma unroll
          for (int i = 0; i < LR; ++i) {
            const uint32_t hw = rec_field<LR, FB>(h.rec, v, i);
            const uint32_t sb = hw & Geom::kFieldMask;                     // bucket + m * (sign is -1)
            const bool neg = sb >= (uint32_t)prm.m;
            const uint32_t off = ((neg ? sb - (uint32_t)prm.m : sb) << 3) + rowbase[i];
            if constexpr (WIDE) {
              atomicAdd(reinterpret_cast<double*>(lds_raw + off), neg ? -acc[v] : acc[v]);
            } else {
              const unsigned long long q = (unsigned long long)acc[v];
              atomicAdd(reinterpret_cast<unsigned long long*>(lds_raw + off), neg ? 0ull - q : q);
            }
          }
          acc[v] = Acc(0);
        }
      }
    };

    // tiles that lie wholly inside the chunk: software pipelined over (tile, batch), the next
    // batch's loads (and, before a tile's last batch, the next tile's w_t0 / xi / table) in
    // flight while the current batch is consumed
    const long long nfast = prm.vec_ok ? (cend > cbeg ? (cend - cbeg) / kTile : 0) : 0;
    long long j0 = cbeg + (long long)tid * V;
    if (nfast > 0) {
      Head hc;
      Batch bc;
      load_head_fast(hc, j0);
      load_batch_fast(bc, j0, 0);
      for (long long it = 0; it < nfast; ++it) {
        for (int bi = 1; bi < NB; ++bi) {
          Batch bn;
          load_batch_fast(bn, j0, bi * KB);
          consume(bc, hc, std::false_type{}, KB);
          bc = bn;
        }
        const long long jn = (it + 1 < nfast) ? j0 + kTile : j0;   // the last prefetch re-reads, unused
        Head hn;
        Batch bn;
        load_head_fast(hn, jn);
        load_batch_fast(bn, jn, 0);
        if (tail < KB) consume(bc, hc, std::true_type{}, tail);
        else consume(bc, hc, std::false_type{}, KB);
        finish(hc, j0, true);
        hc = hn;
        bc = bn;
        j0 += kTile;
      }
    }
    // what is left: at most one ragged tile, or everything when vectors are not possible
    for (; j0 < cend; j0 += kTile) {
      Head h;
      load_head_slow(h, j0);
      for (int bi = 0; bi < NB; ++bi) {
        Batch bt;
        load_batch_slow(bt, j0, bi * KB);
        if (bi == NB - 1 && tail < KB) consume(bt, h, std::true_type{}, tail);
        else consume(bt, h, std::false_type{}, KB);
      }
      finish(h, j0, false);
    }
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  if (scalars) {
    if (sketch) run(yes, yes, yes, no);
    else if (prm.do_sk) run(yes, no, yes, no);
    else run(yes, no, no, no);
  } else if (sketch) {
    run(no, yes, yes, no);
  } else if (prm.do_sk) {
    for (long long j = cbeg + tid; j < cend; j += kStateThreads)
      for (int k = 0; k < K; ++k) amax = fmaxf(amax, fabsf(Slab<T>::load_one(wbase + (long long)k * rs + j) - w0p[j]));
  }

  // the integer cells are void: a drift beyond their terms, or any drift at all where the sample saw none
  const bool bad = prm.do_sk && (sketch ? !(amax < kTermBound / Sm) : amax > 0.0f);

  // ---- workgroup reduction of the scalar components (fixed shape) ---------------------
  const int lane = tid & 63, wave = tid >> 6;
  constexpr int kWaves = kStateThreads / 64;
  if (scalars) {
    const double a = wave_sum(dn);
    const double c = wave_sum(dp);
    const double e = wave_sum(dd);
    if (lane == 0) { red[wave * 3] = a; red[wave * 3 + 1] = c; red[wave * 3 + 2] = e; }
  }
  __syncthreads();
  if (scalars && tid < 3) {
    double s = 0.0;
    for (int wv = 0; wv < kWaves; ++wv) s += red[wv * 3 + tid];
    if (tid == 1 && !lin) s = 0.0;               // no LinearFDA: the projection slot stays zero
    prm.part_np[(size_t)p * 3 + tid] = s;
  }
  if (!prm.do_sk) return;
  const bool again = block_all_max(bad ? 1.0f : 0.0f, red + kRedSums) != 0.0f;
  if (again) {
    // ---- redo: the sketch of this workgroup once more, in fp64, as in the pass --------------------------
    // (30 x 7M fp32: 284 us a call where every workgroup does this, 228 where one does, 149 where none does; element
    // by element 782 and 471.)
    double* const cd = reinterpret_cast<double*>(lds_raw);
    for (int t = tid; t < lds_cells; t += kStateThreads) cd[t] = 0.0;
    __syncthreads();
    // (the row bases are reloaded here: kept live from the pass they push eight and nine rows to 139..153 registers,
    // beyond what two workgroups per CU leave)
#pragma unroll
    for (int i = 0; i < LR; ++i) asm volatile("" : "+s"(rowbase[i]));
    run(no, yes, no, yes);
    __syncthreads();
  }
  // ---- flush the LDS sketch to this workgroup's slice of the partial buffer -----------
  {
    const int allcells = prm.l * prm.m;
    unsigned long long* out = reinterpret_cast<unsigned long long*>(prm.part_sk);
    const unsigned long long* c64 = reinterpret_cast<const unsigned long long*>(lds_raw);
    for (int t = tid; t < cells; t += kStateThreads)
      out[(size_t)p * allcells + (size_t)rstart * prm.m + t] = c64[t];
  }
  if (tid == 0) {
    prm.units[(size_t)p * prm.R + r] = CellUnit{again ? 1.0 : 1.0 / (double)Sm, again ? kCellF64 : kCellI64, 0};
    if (again) atomicMax(&prm.path->now, 1);
  }
}

}  // namespace fda

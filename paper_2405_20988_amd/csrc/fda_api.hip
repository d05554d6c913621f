// C ABI of the FDA monitor (include/fda.h): argument checks, launch planning, kernel
// launches.  Everything the path computes runs in the kernels of fda_kernels.hpp.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstddef>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>

#include "fda.h"
#include "fda_small_kernels.hpp"
#include "fda_state_launch.hpp"
#include "fda_mean_launch.hpp"

// Scratch of fda_estimate_variance_static: the per-workgroup partial sums of estimate_kernel
// (2 + FDA_MAX_SKETCH_ROWS * 128 doubles) and, 256-aligned behind them, its finished-workgroup
// counter.  Every GPU the library runs on holds its own copy until the process ends.  In host code
// this name is only a handle for hipGetSymbolAddress: the address kernels are given is the one
// static_scratch() looked up for the current device.
constexpr size_t kStaticPartDoubles = 2 + (size_t)FDA_MAX_SKETCH_ROWS * 128;
constexpr size_t kStaticTicketOffset = (kStaticPartDoubles * 8 + 255) / 256 * 256;
constexpr size_t kStaticScratchBytes = kStaticTicketOffset + 256;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

#define FDA_HIP(call)                                                                  \
  do {                                                                                 \
    hipError_t e_ = (call);                                                            \
    if (e_ != hipSuccess)                                                              \
      return fail(FDA_EHIP, "%s failed: %s", #call, hipGetErrorString(e_));            \
  } while (0)

// reduction scratch: the scalar sums (8 waves x 8 worker slots x 2 doubles), a double per wave behind them, and slack
constexpr int64_t kLdsReserve = 1536;
static_assert((fda::kRedSums + fda::kStateThreads / 64) * (int64_t)sizeof(double) <= kLdsReserve, "reduction scratch");
constexpr int kMaxRounds = 4;              // at most this many rounds of resident workgroups per launch
constexpr int64_t kMaxTermsPlanned = 12000;    // terms per 32-bit cell and workgroup the planner allows for
constexpr int64_t kMaxTermsPlannedSplit = 3500;   // ... per cell of a sign-split row
constexpr double kWorkgroupOverheadTiles = 6.0;   // what a state workgroup costs besides its tiles, in tiles
// the planner's cost model, in vector-ALU instructions per coordinate
constexpr double kElementCost = 6.5;       // load / unpack / drift / fixed point / scalar sums of one slab element
constexpr double kNegateCost = 2.0;        // ... its negated term, when the rows are not sign-split
constexpr double kDecodeCost = 2.5;        // one table field into an LDS address
constexpr double kSignCost = 3.0;          // ... and into a sign and a bucket, when the rows are not sign-split
constexpr double kSelectCost = 1.0;        // choosing the term or its negative for one 32-bit cell
constexpr double kAtomicCost = 7.5;        // one 32-bit LDS addition and the OR of what it returned
constexpr double kPairAddCost = 13.0;      // one 64-bit LDS addition (two cells) and the OR of what it returned
constexpr double kPlacedPairAddCost = 9.5; // ... when the table's row slots are placed against LDS collisions
// ... and its time model, for short launches
constexpr double kTileInstrUs = 0.0133, kWorkgroupUs = 8.3, kSlotUs = 0.9, kCellUs = 0.35e-3;
constexpr int64_t kQuickTiles = 24;
constexpr double kQuickGain = 0.85;        // a split is given up for one that the model puts below this share of its time
constexpr double kSharedByteCost = 0.25;   // per byte of w_t0 / xi / table read by one more workgroup
constexpr int kXiBlocks = 1024;           // workgroups of the norm pass of fda_update_xi at most: every workgroup of the scaling pass reads their sums
constexpr int kXiScaleBlocks = 24576;     // ... of the scaling pass (launches whose predicate is zero pay 0.2 ns for each)
constexpr int64_t kSyncSmall = 3ll << 19;  // coordinates below which the synchronization takes small blocks
constexpr int kSyncBlocks = 49152;         // workgroups of a synchronization kernel at most
constexpr int kRowWorkgroups = 512;        // ... that store rows: as many by splitting the rows, with at least ...
constexpr int kRowsAtLeast = 8;            // ... so many rows each
constexpr long long kStreamBytes = 512ll << 20;   // slabs beyond this are synchronized with streaming hints
constexpr int kPathWords = 64;        // the two path records, on lines of their own
constexpr int64_t kAlign = 256;

int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

// How the state pass is spread over the chip.
struct Split {
  int G, R, kcnt_max, rcnt_max, KC, LR, P;
  int split;        // sign-split LDS rows (2 m buckets per row)
  int shrink;       // StateParams::shrink
  int64_t chunk, lds_bytes;
};
// How one mean-state pass is spread over the chip.
struct MeanSplit {
  int R, rcnt_max, P, occ;
  int64_t chunk, lds_bytes;
};
struct Plan {
  Split narrow;     // fda_local_state
  MeanSplit mean;   // fda_mean_state
  int vec;          // elements per 16-byte slab load
  int fb;           // bits per field of the tabulated hash
  int narrow_fb;    // ... of the table the state pass streams (kPlacedFieldBits with placed rows)
  int grp;          // rows per placement group of that table (1: rows keep their slots)
  int words;        // 16-bit words per record of the table the state pass streams
  int mean_words;   // ... and of the mean-state pass's table
  bool shared_table;  // both passes split the rows alike and stream one table
  int64_t cells, S, dpad;
  int tickets;        // finished-workgroup counters: [0] estimate_kernel, then those of finish_kernel ...
  int sync_ticket;    // ... and, from here on, those of the synchronization kernel
  int64_t off_np, off_sk, off_units, off_xi, off_syncnorm, off_path, off_ticket, off_dnorm, off_est, off_table,
      off_mean_table, ws_bytes;
};

int validate(const fda_desc* d) {
  if (d == nullptr) return fail(FDA_EINVAL, "desc is NULL");
  if (d->K < 1) return fail(FDA_EINVAL, "K must be >= 1 (got %d)", d->K);
  if (d->d < 1) return fail(FDA_EINVAL, "d must be >= 1");
  if (d->d >= (int64_t)FDA_HASH_PRIME - 64)
    return fail(FDA_ERANGE, "d must be below 2^31 - 1 - 64: coordinates are hash keys modulo 2^31 - 1");
  if (d->row_stride < d->d) return fail(FDA_EINVAL, "row_stride must be >= d");
  if (d->dtype != FDA_F32 && d->dtype != FDA_BF16) return fail(FDA_EINVAL, "unknown dtype %d", d->dtype);
  if ((d->flags & ~FDA_DESC_PLAIN_TABLE) != 0) return fail(FDA_EINVAL, "unknown flags");
  if ((d->variants & ~(FDA_VARIANT_LINEAR | FDA_VARIANT_SKETCH)) != 0 || d->variants == 0)
    return fail(FDA_EINVAL, "variants must be a non-empty mask of FDA_VARIANT_LINEAR | FDA_VARIANT_SKETCH");
  if (d->variants & FDA_VARIANT_SKETCH) {
    if (d->l < 1 || d->l > FDA_MAX_SKETCH_ROWS)
      return fail(FDA_EINVAL, "l must be in 1..%d (got %d)", FDA_MAX_SKETCH_ROWS, d->l);
    if (d->m < 1) return fail(FDA_EINVAL, "m must be >= 1");
    if (d->m > 32767) return fail(FDA_ERANGE, "m must be below 32768 (bucket indices are tabulated in 15 bits)");
    if ((int64_t)d->l * d->m > (int64_t)1 << 24) return fail(FDA_ERANGE, "l*m too large");
    if (!(d->eps > -1.0)) return fail(FDA_EINVAL, "eps must be > -1");
    if (d->hash_coef == nullptr) return fail(FDA_EINVAL, "hash_coef is NULL");
    for (int t = 0; t < d->l * 8; ++t)
      if (d->hash_coef[t] >= FDA_HASH_PRIME)
        return fail(FDA_ERANGE, "hash_coef[%d] is not below 2^31 - 1", t);
  }
  return FDA_OK;
}

// Partitions: all workgroups do the same amount of work, so the launch should fill the resident
// slots a whole number of times; and a workgroup costs its set-up, reductions and flush on top of
// its tiles (measured: about six tiles' worth).  Among the first few feasible numbers of rounds of
// resident workgroups keep the cheapest: rounds x (tiles per workgroup + overhead).
// Feasible: a 32-bit cell should take about 12000 terms at most (16384 of typical size, one way, fill its
// band).  The cells of sign-split rows take the terms of one
// hash sign each, which do not cancel when the drifts themselves lean one way: they are kept at about
// 3500 expected terms (a term of mean magnitude is 2^18..2^19 units: the band of 2^30 then holds unless
// more than about half of a cell's mass leans one way -- such a call finishes on the 64-bit cells).
int64_t choose_partitions(const fda_desc* d, int64_t cells, int64_t tiles, int64_t slots, int64_t gr, int split) {
  int64_t pmin = 1;
  if (cells) {
    const int64_t per_row = (int64_t)d->m * (split ? 2 : 1);
    const int64_t terms = split ? kMaxTermsPlannedSplit : kMaxTermsPlanned;
    pmin = (d->d + per_row * terms - 1) / (per_row * terms);
    if (pmin > tiles) pmin = tiles;
  }
  int64_t P = 0;
  double best_time = -1.0;
  int tried = 0;
  for (int64_t rounds = 1; tried < kMaxRounds; ++rounds) {
    int64_t cand = slots * rounds / gr;                 // (whole groups of 8 partitions share an XCD each)
    if (cand < 1) cand = 1;
    if (cand > tiles) cand = tiles;
    if (cand < pmin) continue;                          // more rounds are needed: cand grows with them
    ++tried;
    const int64_t wgs = cand * gr;
    const double est = (double)((wgs + slots - 1) / slots) * ((double)((tiles + cand - 1) / cand) + kWorkgroupOverheadTiles);
    if (best_time < 0.0 || est < best_time * 0.98) { best_time = est; P = cand; }
    if (cand == tiles) break;                           // one tile per workgroup: nothing finer
  }
  return P;
}

int make_split(const fda_desc* d, int cus, int64_t lds_cu, Split* sp) {
  const bool sk = (d->variants & FDA_VARIANT_SKETCH) != 0;
  const int64_t cells = sk ? (int64_t)d->l * d->m : 0;
  const int64_t tile = (int64_t)fda::kStateThreads * fda::kStateV;
  const int64_t tiles = (d->d + tile - 1) / tile;
  // one workgroup per CU: the kernels hold more registers than two resident workgroups would allow
  const int64_t slots = cus;
  // Split the K workers into G groups and the l sketch rows into R groups so that one
  // workgroup's sketch (rows x m cells x worker slots) fits in LDS.  The kernel has KC worker
  // slots and LR row slots (compile-time); slots a group does not fill still execute.  Every
  // row group repeats the loads and the fixed-point conversion of its workers' elements; every
  // workgroup decodes its rows' table entries and re-reads w_t0 / xi / table (through L2).
  // Pick the split with the least estimated vector-ALU work per coordinate -- unless the launch is so short
  // that what a workgroup costs besides its tiles decides.
  const int l = sk ? d->l : 1;
  struct Cand { int G, R, KC, LR, split; double cost, us; int64_t P; };
  Cand best = {}, quick = {};
  for (int pass = 0; pass < 2; ++pass)        // first the cheapest, then the quickest that splits the rows like it
  for (int G = 1; G <= d->K; ++G) {
    const int kc = (d->K + G - 1) / G;
    int KC = 0;                                              // the smallest kernel that holds kc workers
    for (int c : fda::kKCSet)
      if (c >= kc) { KC = c; break; }
    if (KC == 0) continue;
    // sign-split rows (even slot counts): no negated terms, no select per addition, twice the LDS
    // (without a sketch either kind of kernel does the same)
    for (int split = KC % 2 == 0 ? 1 : 0; split >= 0; --split) {
      if (!fda::narrow_kernel_exists(KC, split != 0)) continue;
      for (int R = 1; R <= l; ++R) {
        const int rc = (l + R - 1) / R;
        int LR = 0;                                          // row slots of the kernel that would run
        if (rc <= fda::kMaxLR && KC * rc <= fda::max_slots(KC)) LR = rc;
        if (LR == 0) continue;
        const int64_t need = cells ? (int64_t)fda::cells32_words(rc, split ? 2 * d->m : d->m, KC) * 4 : 0;
        if (need + kLdsReserve > lds_cu) continue;
        // Estimated cost per coordinate, in vector-ALU instructions (an LDS addition counted as what it
        // keeps the compute unit from issuing): per element slot the load / drift / fixed-point work
        // (with the negated terms unless the rows are sign-split), per row slot the table field, per
        // addition the select (unless split), the overflow OR and the LDS instruction itself.
        const double wg = (double)G * R;
        const double pairs = KC % 2 == 0 ? KC / 2 : KC;                         // LDS instructions per row slot
        // (a table with placed rows avoids about a third of the LDS collisions)
        const bool can_place = split && cells && fda::placed_kernel_exists(KC) && fda::placed_group_rows(rc, d->m, KC) >= 2;
        auto cost_of = [&](bool placed) {
          const double per_add = KC % 2 != 0 ? kAtomicCost + kSelectCost
                                 : placed    ? kPlacedPairAddCost
                                 : split     ? kPairAddCost : kPairAddCost + 2.0 * kSelectCost;
          return wg * KC * (split ? kElementCost : kElementCost + kNegateCost) +
                 wg * LR * (split ? kDecodeCost : kDecodeCost + kSignCost) +
                 wg * LR * pairs * per_add +
                 wg * (8 + 2 * LR) * kSharedByteCost + 1e-3 * wg;
        };
        Cand c = {G, R, KC, LR, split, cost_of(can_place && !(d->flags & FDA_DESC_PLAIN_TABLE)), 0.0, 0};
        // (Without a sketch the pass is bound by its loads: the bytes every worker slot and every workgroup's
        // w_t0 and xi bring through the L2.  13 x 6.9M fp32: 7 groups of 2 slots 77 us, 2 of 8 69.)
        if (!cells) c.cost = wg * (KC * (d->dtype == FDA_F32 ? 4.1 : 2.05) + 8);
        c.P = choose_partitions(d, cells, tiles, slots, wg, split);
        // The time of the launch.  Measured on 5 x 250 and 7 x 1000 sketches, 61706 to 2.6M coordinates, 3 to 50
        // workers (within 10 %): a tile takes 32 clocks per instruction of the cost, a workgroup besides its
        // tiles 8.3 us, 0.9 us per worker slot (sample, sums) and 0.35 us per 1000 cells (flush).  (The same
        // for a plain table, which must not change the workgroups.)
        c.us = (double)((c.P * G * R + slots - 1) / slots) *
               ((double)((tiles + c.P - 1) / c.P) * (cost_of(can_place) / wg) * kTileInstrUs +
                kWorkgroupUs + kSlotUs * KC + kCellUs * rc * d->m * KC);
        if (pass == 0 && (best.G == 0 || c.cost < best.cost)) best = c;
        if (pass == 1 && KC % 2 == 0 && R == best.R && split == best.split && (quick.G == 0 || c.us < quick.us)) quick = c;
        break;   // a larger R only costs more for this G
      }
    }
  }
  if (best.G == 0)
    return fail(FDA_ERANGE, "one row of an m = %d sketch does not fit in %lld bytes of LDS", d->m,
                (long long)lds_cu);
  // Short launches: more groups of fewer workers where that is clearly faster (5 x 61706: 3 groups of 2 slots 9.9
  // us, 1 of 6 14.3; 30 x 100001: 15 of 2 14.0 us, 5 of 6 18.9).  Vectors below 24 tiles keep the cheapest split, which
  // measures slower there too (5 x 30000 fp32 24.3 us a step against 19.9, 60 x 30000 31.2 against 25.7): what speaks for
  // the line is only that small vectors exercise the kernels of six and eight slots.
  if (cells && tiles >= kQuickTiles && quick.G != 0 && quick.us < kQuickGain * best.us) best = quick;
  sp->G = best.G;
  sp->R = best.R;
  sp->split = best.split;
  sp->kcnt_max = (d->K + best.G - 1) / best.G;
  sp->rcnt_max = (l + best.R - 1) / best.R;
  sp->KC = best.KC;
  sp->LR = best.LR;
  const int64_t sk_bytes = cells ? (int64_t)fda::cells32_words(sp->rcnt_max, sp->split ? 2 * d->m : d->m, sp->KC) * 4 : 0;
  sp->lds_bytes = round_up(sk_bytes, 16) + kLdsReserve;
  sp->P = (int)best.P;
  sp->chunk = round_up((d->d + best.P - 1) / best.P, tile);
  // cells that may collect more than 4096 terms get a unit one bit coarser: the expected number of terms of a
  // cell and six standard deviations
  sp->shrink = 0;
  if (cells) {
    const double expect = (double)sp->chunk / ((double)d->m * (sp->split ? 2 : 1));
    if (expect + 6.0 * std::sqrt(expect) >= 4096.0) sp->shrink = 1;
  }
  return FDA_OK;
}

int make_mean_split(const fda_desc* d, int cus, int64_t lds_cu, MeanSplit* ms) {
  const bool sk = (d->variants & FDA_VARIANT_SKETCH) != 0;
  const int l = sk ? d->l : 1;
  // every workgroup reads all K workers; its sketch rows (8-byte cells) must fit in LDS, and the
  // fewer row groups the better, since each repeats all the loads
  int R = 0, rc = 0;
  int64_t bytes = 0;
  for (int cand = 1; cand <= l; ++cand) {
    rc = (l + cand - 1) / cand;
    if (rc > fda::kMeanMaxLR) continue;
    bytes = (sk ? ((int64_t)rc * d->m + fda::kDummyCells) * 8 : 0) + kLdsReserve;
    if (bytes <= lds_cu) { R = cand; break; }
  }
  if (R == 0)
    return fail(FDA_ERANGE, "one row of an m = %d sketch does not fit in %lld bytes of LDS", d->m,
                (long long)lds_cu);
  ms->R = R;
  ms->rcnt_max = rc;
  ms->lds_bytes = bytes;
  // Two workgroups per CU when the LDS allows and a workgroup alone does not keep enough loads in flight:
  // with 16-byte loads per lane and row (fp32 slabs) one workgroup per CU does, and half as many, longer
  // workgroups measured 3-6 % faster; with 8-byte loads (bf16) two per CU measured 3 % faster.
  ms->occ = (2 * bytes <= lds_cu && d->dtype == FDA_BF16) ? 2 : 1;
  const int64_t tile = (int64_t)fda::kStateThreads * fda::kStateV;
  const int64_t tiles = (d->d + tile - 1) / tile;
  int64_t P = (int64_t)cus * ms->occ / R / 8 * 8;  // one round of resident workgroups
  if (P < 8) P = 8;
  if (P > round_up(tiles, 8)) P = round_up(tiles, 8);
  ms->P = (int)P;
  ms->chunk = round_up((d->d + P - 1) / P, tile);
  return FDA_OK;
}

// Workgroups of a synchronization kernel, the blocks each of them takes, and the vectors per thread of a block:
// small ones where 4096 coordinates per workgroup would leave CUs without a workgroup or two.  (Measured: 1M coordinates 22.6 us small, 23.7 large; 2M x 8 bf16 16.6 and 15.7.)
struct SyncGrid { long long blocks; int per, vecs; };
SyncGrid sync_grid(int64_t d) {
  const int vecs = d < kSyncSmall ? fda::kSyncVecsSmall : fda::kSyncVecs;
  const long long n = (d + fda::sync_block(vecs) - 1) / fda::sync_block(vecs);
  const int per = (int)((n + kSyncBlocks - 1) / kSyncBlocks);
  return {(n + per - 1) / per, per, vecs};
}

int make_plan(const fda_desc* d, int cus, int64_t lds_cu, Plan* pl) {
  if (cus < 1 || lds_cu < 16384) return fail(FDA_EINVAL, "bad device description");
  const bool sk = (d->variants & FDA_VARIANT_SKETCH) != 0;
  pl->cells = sk ? (int64_t)d->l * d->m : 0;
  pl->S = 2 + pl->cells;
  pl->vec = d->dtype == FDA_F32 ? 4 : 8;
  int rc = make_mean_split(d, cus, lds_cu, &pl->mean);   // the stricter one first: its error message
  if (rc != FDA_OK) return rc;
  rc = make_split(d, cus, lds_cu, &pl->narrow);
  if (rc != FDA_OK) return rc;
  // the per-workgroup partials of fda_local_state and of fda_mean_state share one region
  int64_t np_bytes = (int64_t)pl->narrow.P * d->K * 2 * 8, sk_bytes = (int64_t)pl->narrow.P * d->K * pl->cells * 8;
  int64_t unit_count = (int64_t)pl->narrow.P * pl->narrow.G * pl->narrow.R;
  if (unit_count < (int64_t)pl->mean.P * pl->mean.R) unit_count = (int64_t)pl->mean.P * pl->mean.R;
  if (np_bytes < (int64_t)pl->mean.P * 3 * 8) np_bytes = (int64_t)pl->mean.P * 3 * 8;
  if (sk_bytes < (int64_t)pl->mean.P * pl->cells * 8) sk_bytes = (int64_t)pl->mean.P * pl->cells * 8;
  pl->off_np = 0;
  pl->off_sk = round_up(pl->off_np + np_bytes, kAlign);
  pl->off_units = round_up(pl->off_sk + sk_bytes, kAlign);
  pl->off_xi = round_up(pl->off_units + unit_count * (int64_t)sizeof(fda::CellUnit), kAlign);
  // one partial norm per workgroup of the synchronization kernel and one per group of them
  const int64_t sync_blocks = sync_grid(d->d).blocks, sync_groups = (sync_blocks + fda::kSyncGroup - 1) / fda::kSyncGroup;
  pl->off_syncnorm = round_up(pl->off_xi + kXiBlocks * 8, kAlign);
  pl->off_path = round_up(pl->off_syncnorm + (sync_blocks + sync_groups) * 8, kAlign);
  pl->off_ticket = pl->off_path + kPathWords * 4;
  const int64_t runs = sk ? (int64_t)d->l * ((d->m + fda::kFinishCols - 1) / fda::kFinishCols) : 0;   // of 32 cells
  pl->sync_ticket = 2 + (int)runs;
  pl->tickets = pl->sync_ticket + (int)sync_groups;
  pl->off_dnorm = round_up(pl->off_ticket + (int64_t)pl->tickets * 4, kAlign);
  pl->off_est = round_up(pl->off_dnorm + 8, kAlign);
  pl->off_table = round_up(pl->off_est + (2 + runs) * 8, kAlign);   // one piece of a row norm per run
  pl->dpad = round_up(d->d, fda::kRecBlockCoords);      // the table comes in whole blocks
  // the tabulated hash: per row group one record per coordinate with a field per row slot
  pl->fb = fda::field_bits_for(sk ? d->m : 1);
  // placed rows (slots chosen against LDS collisions): sign-split rows in an unskewed layout, when a
  // placement group of at least two rows fits the wider field
  pl->grp = 1;
  pl->narrow_fb = pl->fb;
  if (sk && pl->narrow.split && fda::placed_kernel_exists(pl->narrow.KC) &&
      !(d->flags & FDA_DESC_PLAIN_TABLE)) {
    const int g = fda::placed_group_rows(pl->narrow.rcnt_max, d->m, pl->narrow.KC);
    if (g >= 2) { pl->grp = g; pl->narrow_fb = fda::kPlacedFieldBits; }
  }
  pl->words = (pl->narrow.LR * pl->narrow_fb + 15) / 16;
  pl->mean_words = (pl->mean.rcnt_max * pl->fb + 15) / 16;
  pl->shared_table = pl->grp == 1 && pl->narrow.R == pl->mean.R && pl->narrow.LR == pl->mean.rcnt_max;
  const int64_t table_bytes = sk ? (int64_t)pl->narrow.R * pl->dpad * pl->words * 2 : 0;
  const int64_t mean_table_bytes =
      sk && !pl->shared_table ? (int64_t)pl->mean.R * pl->dpad * pl->mean_words * 2 : 0;
  pl->off_mean_table = pl->shared_table ? pl->off_table : round_up(pl->off_table + table_bytes, kAlign);
  pl->ws_bytes = round_up(pl->off_mean_table + mean_table_bytes + (pl->shared_table ? table_bytes : 0), kAlign);
  return FDA_OK;
}

void export_plan(const Plan& pl, fda_plan_info* out) {
  out->worker_groups = pl.narrow.G;
  out->row_groups = pl.narrow.R;
  out->rows_per_group = pl.narrow.rcnt_max;
  out->workers_per_group = pl.narrow.kcnt_max;
  out->partitions = pl.narrow.P;
  out->threads = fda::kStateThreads;
  out->chunk = pl.narrow.chunk;
  out->lds_bytes = pl.narrow.lds_bytes;
  out->workspace_bytes = pl.ws_bytes;
  out->state_floats = pl.S;
  out->mean_row_groups = pl.mean.R;
  out->mean_rows_per_group = pl.mean.rcnt_max;
  out->mean_partitions = pl.mean.P;
  out->mean_workgroups_per_cu = pl.mean.occ;
  out->mean_chunk = pl.mean.chunk;
  out->mean_lds_bytes = pl.mean.lds_bytes;
  out->sign_split_rows = pl.narrow.split;
  out->worker_slots = pl.narrow.KC;
  out->placed_row_group = pl.grp >= 2 ? pl.grp : 0;
  out->reserved = 0;
}

int device_shape(int* cus, int64_t* lds) {
  int dev = 0;
  FDA_HIP(hipGetDevice(&dev));
  int v = 0;
  FDA_HIP(hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev));
  *cus = v;
  FDA_HIP(hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
  *lds = v;
  return FDA_OK;
}

// Whole-vector loads and stores only need the alignment of the element type, which every entry point
// checks of its pointers: the vector path is always available (the element-wise path of the kernels
// serves the ragged end of a vector).
constexpr int kVecOk = 1;

// Route a launch (or, with prm == nullptr, the LDS-limit setup) to the translation unit that
// holds the kernel for this slab type and shape.
int dispatch_any(int dtype, const Split& sp, int FB, const fda::StateParams* prm, hipStream_t st) {
  const int KC = sp.KC, LR = sp.LR;
  const size_t lds = (size_t)sp.lds_bytes;
  hipError_t e = hipErrorInvalidValue;
#define FDA_CASE(t, kc) case kc: e = fda::launch_narrow_##t##_kc##kc(LR, FB, sp.split, prm, lds, st); break
  if (dtype == FDA_F32) {
    switch (KC) { FDA_CASE(f32, 1); FDA_CASE(f32, 2); FDA_CASE(f32, 4); FDA_CASE(f32, 6); FDA_CASE(f32, 8); }
  } else {
    switch (KC) { FDA_CASE(bf16, 1); FDA_CASE(bf16, 2); FDA_CASE(bf16, 4); FDA_CASE(bf16, 6); FDA_CASE(bf16, 8); }
  }
#undef FDA_CASE
  if (e == hipErrorInvalidValue)
    return fail(FDA_EINVAL, "internal: no state kernel for %d workers x %d rows per workgroup", KC, LR);
  if (e != hipSuccess) return fail(FDA_EHIP, "state kernel launch failed: %s", hipGetErrorString(e));
  return FDA_OK;
}

int dispatch_mean(int dtype, const MeanSplit& ms, int FB, const fda::MeanParams* prm, hipStream_t st) {
  const size_t lds = (size_t)ms.lds_bytes;
  const hipError_t e = dtype == FDA_F32 ? fda::launch_mean_f32(ms.rcnt_max, FB, prm, lds, st)
                                        : fda::launch_mean_bf16(ms.rcnt_max, FB, prm, lds, st);
  if (e == hipErrorInvalidValue)
    return fail(FDA_EINVAL, "internal: no mean-state kernel for %d rows per workgroup", ms.rcnt_max);
  if (e != hipSuccess) return fail(FDA_EHIP, "mean-state kernel launch failed: %s", hipGetErrorString(e));
  return FDA_OK;
}

// Pinned places for results that a program reads back: the estimate kernels write there themselves, which
// spares the call a copy (a pageable copy of 64 bytes behind a kernel: 9 us).  One page for all contexts of the
// process; a context takes a place on its first such call and gives it back when it is destroyed; the page goes
// with the last one.  No place free: the result is copied.
// Another stream of the program may be capturing a graph meanwhile: beside a capture in the global mode
// allocations, frees and waits are only allowed to threads in the relaxed mode (a wait in another mode is refused
// and voids the capture).
struct RelaxedCapture {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  RelaxedCapture() { if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) (void)hipGetLastError(); }
  ~RelaxedCapture() { if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) (void)hipGetLastError(); }
};
hipError_t wait_for(hipStream_t st) {
  const RelaxedCapture relaxed;
  return hipStreamSynchronize(st);
}
struct HostResults {
  static constexpr int kPlaces = 64;
  std::mutex mutex;
  fda_estimate* page = nullptr;
  uint64_t used = 0;
  fda_estimate* take() {
    std::lock_guard<std::mutex> lock(mutex);
    if (page == nullptr) {
      const RelaxedCapture relaxed;
      void* p = nullptr;
      if (hipHostMalloc(&p, kPlaces * sizeof(fda_estimate), hipHostMallocPortable) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
      }
      page = static_cast<fda_estimate*>(p);
    }
    for (int t = 0; t < kPlaces; ++t)
      if (!(used >> t & 1)) { used |= 1ull << t; return page + t; }
    return nullptr;
  }
  void give_back(fda_estimate* place) {
    if (place == nullptr) return;
    std::lock_guard<std::mutex> lock(mutex);
    used &= ~(1ull << (place - page));
    if (used != 0) return;
    const RelaxedCapture relaxed;
    if (hipHostFree(page) == hipSuccess) page = nullptr;
    else (void)hipGetLastError();                      // the page stays for the next context
  }
};
HostResults g_host_results;

constexpr int kProfSlots = 64;

// Device address of `scratch` on the current device, looked up once per device (with that device
// current) and kept: each GPU has its own copy of the array at its own address.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
unsigned char* g_scratch_ptr[kMaxDevices] = {};

int static_scratch(unsigned char** out) {
  int dev = -1;
  FDA_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(FDA_ERANGE, "device ordinal %d is beyond %d", dev, kMaxDevices - 1);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    FDA_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (p == nullptr) return fail(FDA_EHIP, "hipGetSymbolAddress returned a null address");
    g_scratch_ptr[dev] = static_cast<unsigned char*>(p);
  }
  *out = g_scratch_ptr[dev];
  return FDA_OK;
}

}  // namespace

// A launch that a context needs once in front of others.
struct Once {
  bool done = false, captured = false;   // enqueued to run; recorded into a graph
  unsigned long long capture = 0;        // ... by this capture
};
struct fda_ctx {
  fda_desc desc;
  fda::HashCoef coef;
  Plan plan;
  unsigned char* ws;
  int device;
  int cus;
  Once table;                     // the hash table of the state pass
  Once mean_table;                // ... of the mean-state pass (`table` when the plan shares it)
  Once tickets;                   // the counters' first clearing
  fda_estimate* host_place = nullptr;   // in HostResults, once a result has been read back
  // optional timing of the state kernel (fda_profile_enable)
  bool prof_on = false;
  hipEvent_t prof_start[kProfSlots] = {};
  hipEvent_t prof_stop[kProfSlots] = {};
  int prof_pending = 0;       // recorded pairs not yet read
  double prof_ms = 0.0;
  int64_t prof_launches = 0;
};

namespace {
// Whether the launch behind `once` is still to be enqueued on st.  One that is only being captured has done nothing
// yet: calls outside that capture, before its first replay, enqueue it for themselves.
int still_to_do(Once* once, hipStream_t st, bool* todo) {
  *todo = !once->done;
  if (once->done) return FDA_OK;
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  unsigned long long id = 0;
  FDA_HIP(hipStreamGetCaptureInfo(st, &status, &id));
  if (status == hipStreamCaptureStatusNone) {
    once->done = true;
  } else {
    *todo = !once->captured || once->capture != id;
    once->captured = true;
    once->capture = id;
  }
  return FDA_OK;
}

// The finished-workgroup counters of finish_kernel and estimate_kernel start at zero and are left
// at zero by every launch; the workspace arrives uninitialised, so they are cleared once.
int clear_tickets_once(fda_ctx* c, hipStream_t st) {
  bool todo;
  const int rc = still_to_do(&c->tickets, st, &todo);
  if (rc != FDA_OK || !todo) return rc;
  // (the path records, two pairs of ints, lie in front of the counters)
  hipLaunchKernelGGL(fda::clear_u32_kernel, dim3(64), dim3(fda::kSmallThreads), 0, st,
                     reinterpret_cast<unsigned int*>(c->ws + c->plan.off_path), kPathWords + c->plan.tickets);
  FDA_HIP(hipGetLastError());
  return FDA_OK;
}

// Fold the recorded event pairs into the running totals (waits for them).
int prof_drain(fda_ctx* c) {
  const RelaxedCapture relaxed;
  for (int t = 0; t < c->prof_pending; ++t) {
    FDA_HIP(hipEventSynchronize(c->prof_stop[t]));
    float ms = 0.0f;
    FDA_HIP(hipEventElapsedTime(&ms, c->prof_start[t], c->prof_stop[t]));
    c->prof_ms += ms;
    c->prof_launches += 1;
  }
  c->prof_pending = 0;
  return FDA_OK;
}

// Start / stop of one timed kernel (fda_profile_enable); slot < 0: timing is off.
int prof_begin(fda_ctx* c, hipStream_t st, int* slot) {
  *slot = -1;
  if (!c->prof_on) return FDA_OK;
  if (c->prof_pending == kProfSlots) {
    int rc = prof_drain(c);
    if (rc != FDA_OK) return rc;
  }
  *slot = c->prof_pending;
  FDA_HIP(hipEventRecord(c->prof_start[*slot], st));
  return FDA_OK;
}
int prof_end(fda_ctx* c, hipStream_t st, int slot) {
  if (slot < 0) return FDA_OK;
  FDA_HIP(hipEventRecord(c->prof_stop[slot], st));
  c->prof_pending = slot + 1;
  return FDA_OK;
}

int build_table(fda_ctx* ctx, int R, int slots, int fb, int words, int grp, int KC, int64_t off, hipStream_t st) {
  const fda_desc& d = ctx->desc;
  const Plan& pl = ctx->plan;
  const long long groups = pl.dpad / 4;
  // what the kernel's arrays assume: at most kMaxLR row slots, as many words of a record, placement groups of 2 rows
  // or more
  if (slots < 1 || slots > fda::kMaxLR || words < 1 || words > fda::kMaxLR || grp < 1 || grp > fda::kMaxLR ||
      slots * fb > words * 16)
    return fail(FDA_EINVAL, "table shape out of range: %d slots of %d bits in %d words, groups of %d", slots, fb, words, grp);
  hipLaunchKernelGGL(fda::hash_table_kernel,
                     dim3((unsigned)((groups + fda::kSmallThreads - 1) / fda::kSmallThreads), (unsigned)R),
                     dim3(fda::kSmallThreads), 0, st, ctx->coef, d.l, R, slots, d.m, fb, words, grp, KC,
                     (long long)d.d, (long long)pl.dpad, reinterpret_cast<uint16_t*>(ctx->ws + off));
  FDA_HIP(hipGetLastError());
  return FDA_OK;
}

// Before the first sketch of a context: the hash of every (row, coordinate), tabulated for the pass that is
// about to run (for_mean: fda_mean_state, else fda_local_state).
int prepare_sketch(fda_ctx* ctx, bool for_mean, hipStream_t st) {
  const Plan& pl = ctx->plan;
  Once* const once = for_mean && !pl.shared_table ? &ctx->mean_table : &ctx->table;
  bool todo;
  int rc = still_to_do(once, st, &todo);
  if (rc != FDA_OK || !todo) return rc;
  rc = for_mean
           ? build_table(ctx, pl.mean.R, pl.mean.rcnt_max, pl.fb, pl.mean_words, 1, 1, pl.off_mean_table, st)
           : build_table(ctx, pl.narrow.R, pl.narrow.LR, pl.narrow_fb, pl.words, pl.grp, pl.narrow.KC, pl.off_table, st);
  if (rc != FDA_OK) *once = Once{};
  return rc;
}

fda::PathRecord* path_record(const fda_ctx* ctx, bool for_mean) {
  return reinterpret_cast<fda::PathRecord*>(ctx->ws + ctx->plan.off_path) + (for_mean ? 1 : 0);
}

// The partials of a state pass -> state[rows][S] (rows = K), or mean_state[S] (rows = 1), with the estimate
// `est` on it (its rows are filled in here) unless est is NULL.
int launch_finish(fda_ctx* ctx, bool for_mean, float* state, const fda::EstimateArgs* est, hipStream_t st) {
  const fda_desc& d = ctx->desc;
  const Plan& pl = ctx->plan;
  const bool sk = (d.variants & FDA_VARIANT_SKETCH) != 0;
  fda::FinishParams f;
  f.part_np = reinterpret_cast<const double*>(ctx->ws + pl.off_np);
  f.part_sk = ctx->ws + pl.off_sk;
  f.units = reinterpret_cast<const fda::CellUnit*>(ctx->ws + pl.off_units);
  f.path = path_record(ctx, for_mean);
  f.state = state;
  f.dnorm = for_mean ? reinterpret_cast<double*>(ctx->ws + pl.off_dnorm) : nullptr;
  f.ticket = reinterpret_cast<unsigned int*>(ctx->ws + pl.off_ticket) + 1;
  f.est_part = reinterpret_cast<double*>(ctx->ws + pl.off_est);
  f.rows = for_mean ? 1 : d.K;
  f.K = d.K; f.l = sk ? d.l : 0; f.m = sk ? d.m : 0;
  f.P = for_mean ? pl.mean.P : pl.narrow.P;
  f.G = for_mean ? 1 : pl.narrow.G;
  f.R = for_mean ? pl.mean.R : pl.narrow.R;
  f.est = est != nullptr ? *est : fda::EstimateArgs{};
  f.wl = fda::kFinishLanes;
  while (f.wl > 1 && (f.wl / 2 >= f.rows || f.P * f.wl > fda::kFinishLanes * fda::kFinishLoads)) f.wl /= 2;
  const int blocks = 1 + f.l * ((f.m + fda::kFinishCols - 1) / fda::kFinishCols) * ((f.rows + f.wl - 1) / f.wl);
  hipLaunchKernelGGL(fda::finish_kernel, dim3(blocks), dim3(fda::kFinishThreads), 0, st, f);
  FDA_HIP(hipGetLastError());
  return FDA_OK;
}

// Launches go to the current device: it must be the one the context (and its workspace) lives on.
int check_device(const fda_ctx* ctx) {
  int dev = -1;
  FDA_HIP(hipGetDevice(&dev));
  if (dev != ctx->device)
    return fail(FDA_EINVAL, "the context was created on device %d but device %d is current", ctx->device, dev);
  return FDA_OK;
}

// The argument checks fda_local_state and fda_mean_state share.
int check_state_args(const fda_ctx* ctx, const void* w, const float* w_t0, const float* xi, const float* out) {
  if (ctx == nullptr || w == nullptr || w_t0 == nullptr || out == nullptr)
    return fail(FDA_EINVAL, "NULL argument");
  int rcd = check_device(ctx);
  if (rcd != FDA_OK) return rcd;
  const fda_desc& d = ctx->desc;
  if ((d.variants & FDA_VARIANT_LINEAR) && xi == nullptr)
    return fail(FDA_EINVAL, "xi is NULL but FDA_VARIANT_LINEAR is requested");
  const int esz = d.dtype == FDA_F32 ? 4 : 2;
  if (reinterpret_cast<uintptr_t>(w) % esz != 0 || reinterpret_cast<uintptr_t>(w_t0) % 4 != 0 ||
      reinterpret_cast<uintptr_t>(out) % 4 != 0 || (xi && reinterpret_cast<uintptr_t>(xi) % 4 != 0))
    return fail(FDA_EINVAL, "pointer not aligned to its element type");
  return FDA_OK;
}
}  // namespace

extern "C" {

const char* fda_strerror(int code) {
  switch (code) {
    case FDA_OK: return "success";
    case FDA_EINVAL: return "invalid argument";
    case FDA_ERANGE: return "value out of the supported range";
    case FDA_ENOMEM: return "workspace too small";
    case FDA_EHIP: return "HIP runtime error";
  }
  return "unknown error code";
}

const char* fda_last_error(void) { return g_err; }

int fda_plan(const fda_desc* desc, int32_t compute_units, int64_t lds_bytes_per_cu,
             fda_plan_info* out) {
  if (out == nullptr) return fail(FDA_EINVAL, "out is NULL");
  int rc = validate(desc);
  if (rc != FDA_OK) return rc;
  Plan pl;
  rc = make_plan(desc, compute_units, lds_bytes_per_cu, &pl);
  if (rc != FDA_OK) return rc;
  export_plan(pl, out);
  return FDA_OK;
}

int fda_workspace_bytes(const fda_desc* desc, size_t* bytes) {
  if (bytes == nullptr) return fail(FDA_EINVAL, "bytes is NULL");
  int rc = validate(desc);
  if (rc != FDA_OK) return rc;
  int cus = 0;
  int64_t lds = 0;
  rc = device_shape(&cus, &lds);
  if (rc != FDA_OK) return rc;
  Plan pl;
  rc = make_plan(desc, cus, lds, &pl);
  if (rc != FDA_OK) return rc;
  *bytes = (size_t)pl.ws_bytes;
  return FDA_OK;
}

int fda_create(fda_ctx** ctx, const fda_desc* desc, void* workspace, size_t workspace_bytes) {
  if (ctx == nullptr) return fail(FDA_EINVAL, "ctx is NULL");
  *ctx = nullptr;
  int rc = validate(desc);
  if (rc != FDA_OK) return rc;
  if (workspace == nullptr) return fail(FDA_EINVAL, "workspace is NULL");
  if (reinterpret_cast<uintptr_t>(workspace) % kAlign != 0)
    return fail(FDA_EINVAL, "workspace must be 256-byte aligned");
  int cus = 0;
  int64_t lds = 0;
  rc = device_shape(&cus, &lds);
  if (rc != FDA_OK) return rc;
  Plan pl;
  rc = make_plan(desc, cus, lds, &pl);
  if (rc != FDA_OK) return rc;
  if ((int64_t)workspace_bytes < pl.ws_bytes)
    return fail(FDA_ENOMEM, "workspace has %zu bytes, %lld needed", workspace_bytes, (long long)pl.ws_bytes);
  fda_ctx* c = new (std::nothrow) fda_ctx;
  if (c == nullptr) return fail(FDA_ENOMEM, "out of host memory");
  c->desc = *desc;
  c->desc.hash_coef = nullptr;
  std::memset(&c->coef, 0, sizeof(c->coef));
  if (desc->variants & FDA_VARIANT_SKETCH)
    std::memcpy(&c->coef, desc->hash_coef, sizeof(uint32_t) * 8 * desc->l);
  c->plan = pl;
  c->ws = static_cast<unsigned char*>(workspace);
  c->cus = cus;
  if (hipGetDevice(&c->device) != hipSuccess) {
    delete c;
    return fail(FDA_EHIP, "hipGetDevice failed");
  }
  // The dynamic-LDS limit of a kernel is one setting per process: raise it to everything the
  // device allows, so that a context created later with a smaller sketch cannot lower it under
  // what an earlier context's launches need.
  Split narrow_max = pl.narrow;
  MeanSplit mean_max = pl.mean;
  narrow_max.lds_bytes = mean_max.lds_bytes = lds;
  rc = dispatch_any(desc->dtype, narrow_max, pl.narrow_fb, nullptr, nullptr);
  if (rc == FDA_OK) rc = dispatch_mean(desc->dtype, mean_max, pl.fb, nullptr, nullptr);
  if (rc != FDA_OK) {
    delete c;
    return rc;
  }
  *ctx = c;
  return FDA_OK;
}

int fda_destroy(fda_ctx* ctx) {
  if (ctx == nullptr) return FDA_OK;
  for (int t = 0; t < kProfSlots; ++t) {
    if (ctx->prof_start[t]) (void)hipEventDestroy(ctx->prof_start[t]);
    if (ctx->prof_stop[t]) (void)hipEventDestroy(ctx->prof_stop[t]);
  }
  g_host_results.give_back(ctx->host_place);
  delete ctx;
  return FDA_OK;
}

int fda_last_state_path(fda_ctx* ctx, int32_t* path, void* stream) {
  if (ctx == nullptr || path == nullptr) return fail(FDA_EINVAL, "NULL argument");
  if (!(ctx->desc.variants & FDA_VARIANT_SKETCH)) { *path = -1; return FDA_OK; }
  hipStream_t st = static_cast<hipStream_t>(stream);
  fda::PathRecord rec;
  FDA_HIP(hipMemcpyAsync(&rec, path_record(ctx, false), sizeof(rec), hipMemcpyDeviceToHost, st));
  FDA_HIP(wait_for(st));
  *path = rec.last;
  return FDA_OK;
}

int fda_last_mean_state_path(fda_ctx* ctx, int32_t* path, void* stream) {
  if (ctx == nullptr || path == nullptr) return fail(FDA_EINVAL, "NULL argument");
  if (!(ctx->desc.variants & FDA_VARIANT_SKETCH)) { *path = -1; return FDA_OK; }
  hipStream_t st = static_cast<hipStream_t>(stream);
  fda::PathRecord rec;
  FDA_HIP(hipMemcpyAsync(&rec, path_record(ctx, true), sizeof(rec), hipMemcpyDeviceToHost, st));
  FDA_HIP(wait_for(st));
  *path = rec.last;
  return FDA_OK;
}

int fda_profile_enable(fda_ctx* ctx, int on) {
  if (ctx == nullptr) return fail(FDA_EINVAL, "ctx is NULL");
  if (on && ctx->prof_start[0] == nullptr) {
    for (int t = 0; t < kProfSlots; ++t) {
      FDA_HIP(hipEventCreate(&ctx->prof_start[t]));
      FDA_HIP(hipEventCreate(&ctx->prof_stop[t]));
    }
  }
  if (!on) {
    int rc = prof_drain(ctx);
    if (rc != FDA_OK) return rc;
  }
  ctx->prof_on = on != 0;
  return FDA_OK;
}

int fda_profile_read(fda_ctx* ctx, double* state_kernel_ms, int64_t* launches, int reset) {
  if (ctx == nullptr || state_kernel_ms == nullptr || launches == nullptr)
    return fail(FDA_EINVAL, "NULL argument");
  int rc = prof_drain(ctx);
  if (rc != FDA_OK) return rc;
  *state_kernel_ms = ctx->prof_ms;
  *launches = ctx->prof_launches;
  if (reset) { ctx->prof_ms = 0.0; ctx->prof_launches = 0; }
  return FDA_OK;
}

int fda_state_floats(const fda_ctx* ctx, int64_t* S) {
  if (ctx == nullptr || S == nullptr) return fail(FDA_EINVAL, "NULL argument");
  *S = ctx->plan.S;
  return FDA_OK;
}

int fda_get_plan(const fda_ctx* ctx, fda_plan_info* out) {
  if (ctx == nullptr || out == nullptr) return fail(FDA_EINVAL, "NULL argument");
  export_plan(ctx->plan, out);
  return FDA_OK;
}

static int local_state(fda_ctx* ctx, const void* w, const float* w_t0, const float* xi, float* state,
                       const fda::EstimateArgs* est, void* stream) {
  int rc = check_state_args(ctx, w, w_t0, xi, state);
  if (rc != FDA_OK) return rc;
  const fda_desc& d = ctx->desc;
  const Plan& pl = ctx->plan;
  const bool lin = (d.variants & FDA_VARIANT_LINEAR) != 0;
  const bool sk = (d.variants & FDA_VARIANT_SKETCH) != 0;
  hipStream_t st = static_cast<hipStream_t>(stream);

  const Split& sp = pl.narrow;
  fda::StateParams prm;
  prm.w = w; prm.w_t0 = w_t0; prm.xi = xi;
  prm.row_stride = d.row_stride; prm.d = d.d; prm.chunk = sp.chunk;
  prm.K = d.K; prm.l = sk ? d.l : 0; prm.m = sk ? d.m : 0;
  prm.G = sp.G; prm.R = sp.R; prm.P = sp.P; prm.shrink = sp.shrink;
  prm.do_lin = lin; prm.do_sk = sk;
  prm.vec_ok = kVecOk;
  prm.part_np = reinterpret_cast<double*>(ctx->ws + pl.off_np);
  prm.part_sk = ctx->ws + pl.off_sk;
  prm.units = reinterpret_cast<fda::CellUnit*>(ctx->ws + pl.off_units);
  prm.path = path_record(ctx, false);
  prm.table = reinterpret_cast<const uint16_t*>(ctx->ws + pl.off_table);
  prm.dpad = pl.dpad;
  prm.grp = pl.grp;

  rc = clear_tickets_once(ctx, st);
  if (rc == FDA_OK && sk) rc = prepare_sketch(ctx, false, st);
  if (rc != FDA_OK) return rc;
  int slot = -1;
  rc = prof_begin(ctx, st, &slot);
  if (rc != FDA_OK) return rc;
  rc = dispatch_any(d.dtype, sp, pl.narrow_fb, &prm, st);
  if (rc != FDA_OK) return rc;
  rc = prof_end(ctx, st, slot);
  if (rc != FDA_OK) return rc;
  return launch_finish(ctx, false, state, est, st);
}

int fda_local_state(fda_ctx* ctx, const void* w, const float* w_t0, const float* xi, float* state, void* stream) {
  return local_state(ctx, w, w_t0, xi, state, nullptr, stream);
}

static int mean_state_pass(fda_ctx* ctx, const void* w, const float* w_t0, const float* xi, float* mean_state,
                           float* w_bar, const fda::EstimateArgs* est, void* stream) {
  int rc = check_state_args(ctx, w, w_t0, xi, mean_state);
  if (rc != FDA_OK) return rc;
  const fda_desc& d = ctx->desc;
  const Plan& pl = ctx->plan;
  const MeanSplit& ms = pl.mean;
  const bool lin = (d.variants & FDA_VARIANT_LINEAR) != 0;
  const bool sk = (d.variants & FDA_VARIANT_SKETCH) != 0;
  // a cell's integer sum stays below K * chunk * 2^30 in magnitude
  if (sk && (double)d.K * (double)ms.chunk >= 8589934592.0)
    return fail(FDA_ERANGE, "K * coordinates per workgroup must stay below 2^33");
  if (w_bar != nullptr && reinterpret_cast<uintptr_t>(w_bar) % 4 != 0)
    return fail(FDA_EINVAL, "pointer not aligned to its element type");
  hipStream_t st = static_cast<hipStream_t>(stream);

  fda::MeanParams prm;
  prm.w = w; prm.w_t0 = w_t0; prm.xi = xi;
  prm.row_stride = d.row_stride; prm.d = d.d; prm.chunk = ms.chunk;
  prm.K = d.K; prm.l = sk ? d.l : 0; prm.m = sk ? d.m : 0;
  prm.R = ms.R; prm.P = ms.P;
  prm.do_lin = lin; prm.do_sk = sk;
  prm.vec_ok = kVecOk;
  prm.w_bar = w_bar;
  prm.part_np = reinterpret_cast<double*>(ctx->ws + pl.off_np);
  prm.part_sk = ctx->ws + pl.off_sk;
  prm.units = reinterpret_cast<fda::CellUnit*>(ctx->ws + pl.off_units);
  prm.path = path_record(ctx, true);
  prm.table = reinterpret_cast<const uint16_t*>(ctx->ws + pl.off_mean_table);
  prm.dpad = pl.dpad;

  rc = clear_tickets_once(ctx, st);
  if (rc == FDA_OK && sk) rc = prepare_sketch(ctx, true, st);
  if (rc != FDA_OK) return rc;
  int slot = -1;
  rc = prof_begin(ctx, st, &slot);
  if (rc != FDA_OK) return rc;
  rc = dispatch_mean(d.dtype, ms, pl.fb, &prm, st);
  if (rc != FDA_OK) return rc;
  rc = prof_end(ctx, st, slot);
  if (rc != FDA_OK) return rc;
  return launch_finish(ctx, true, mean_state, est, st);
}

int fda_mean_state(fda_ctx* ctx, const void* w, const float* w_t0, const float* xi, float* mean_state, float* w_bar,
                   void* stream) {
  return mean_state_pass(ctx, w, w_t0, xi, mean_state, w_bar, nullptr, stream);
}

// The argument checks of an estimate, and what its kernels take.
static int estimate_args(const fda_ctx* ctx, int rows, double theta, double tie_tol, fda_estimate* out_dev,
                         fda::EstimateArgs* args) {
  if (ctx == nullptr || out_dev == nullptr) return fail(FDA_EINVAL, "NULL argument");
  if (reinterpret_cast<uintptr_t>(out_dev) % 8 != 0) return fail(FDA_EINVAL, "out_dev must be 8-byte aligned");
  if (!(tie_tol >= 0.0)) return fail(FDA_EINVAL, "tie_tol must be >= 0");
  const fda_desc& d = ctx->desc;
  const bool sk = (d.variants & FDA_VARIANT_SKETCH) != 0;
  *args = {d.variants, sk ? d.l : 0, sk ? d.m : 1, rows, d.eps, theta, tie_tol, out_dev, nullptr};
  return FDA_OK;
}

// The result on its way to the host (args.host, if a place is free) and, behind the kernels, into out_host:
// waits for the stream.
static void want_result(fda_ctx* ctx, fda::EstimateArgs* args) {
  if (ctx->host_place == nullptr) ctx->host_place = g_host_results.take();
  args->host = ctx->host_place;
}
static int read_result(const fda::EstimateArgs& args, fda_estimate* out_host, hipStream_t st) {
  if (args.host == nullptr)
    FDA_HIP(hipMemcpyAsync(out_host, args.out, sizeof(fda_estimate), hipMemcpyDeviceToHost, st));
  FDA_HIP(wait_for(st));
  if (args.host != nullptr) std::memcpy(out_host, args.host, sizeof(fda_estimate));
  return FDA_OK;
}

static int estimate_rows(fda_ctx* ctx, const float* state, int rows, int mean_mode, double theta, double tie_tol,
                         fda_estimate* out_dev, fda_estimate* out_host, void* stream) {
  if (state == nullptr) return fail(FDA_EINVAL, "NULL argument");
  fda::EstimateArgs args;
  int rc = estimate_args(ctx, rows, theta, tie_tol, out_dev, &args);
  if (rc != FDA_OK) return rc;
  rc = check_device(ctx);
  if (rc != FDA_OK) return rc;
  const fda_desc& d = ctx->desc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int eblocks = args.l > 0 ? args.l * ((d.m + fda::kEstCols - 1) / fda::kEstCols) : 1;
  rc = clear_tickets_once(ctx, st);
  if (rc != FDA_OK) return rc;
  if (out_host != nullptr) want_result(ctx, &args);
  hipLaunchKernelGGL(fda::estimate_kernel, dim3(eblocks), dim3(fda::kSmallThreads), 0, st, state, args,
                     reinterpret_cast<double*>(ctx->ws + ctx->plan.off_est),
                     reinterpret_cast<unsigned int*>(ctx->ws + ctx->plan.off_ticket),
                     path_record(ctx, mean_mode != 0));
  FDA_HIP(hipGetLastError());
  return out_host != nullptr ? read_result(args, out_host, st) : FDA_OK;
}

int fda_estimate_variance(fda_ctx* ctx, const float* state, double theta, double tie_tol,
                          fda_estimate* out_dev, fda_estimate* out_host, void* stream) {
  return estimate_rows(ctx, state, ctx ? ctx->desc.K : 0, 0, theta, tie_tol, out_dev, out_host, stream);
}

int fda_estimate_variance_mean(fda_ctx* ctx, const float* mean_state, double theta, double tie_tol,
                               fda_estimate* out_dev, fda_estimate* out_host, void* stream) {
  return estimate_rows(ctx, mean_state, 1, 1, theta, tie_tol, out_dev, out_host, stream);
}

int fda_estimate_variance_static(const float* state, int32_t K, int32_t l, int32_t m, int32_t variants,
                                 double eps, double theta, double tie_tol, fda_estimate* out_dev,
                                 void* stream) {
  if (state == nullptr || out_dev == nullptr) return fail(FDA_EINVAL, "NULL argument");
  if (reinterpret_cast<uintptr_t>(state) % 4 != 0 || reinterpret_cast<uintptr_t>(out_dev) % 8 != 0)
    return fail(FDA_EINVAL, "state must be 4-byte and out_dev 8-byte aligned");
  if (K < 1) return fail(FDA_EINVAL, "K must be >= 1 (got %d)", K);
  if ((variants & ~(FDA_VARIANT_LINEAR | FDA_VARIANT_SKETCH)) != 0 || variants == 0)
    return fail(FDA_EINVAL, "variants must be a non-empty mask of FDA_VARIANT_LINEAR | FDA_VARIANT_SKETCH");
  if (!(tie_tol >= 0.0)) return fail(FDA_EINVAL, "tie_tol must be >= 0");
  const bool sk = (variants & FDA_VARIANT_SKETCH) != 0;
  if (sk) {
    if (l < 1 || l > FDA_MAX_SKETCH_ROWS)
      return fail(FDA_ERANGE, "l must be in 1..%d (got %d): the static scratch holds no more rows", FDA_MAX_SKETCH_ROWS, l);
    if (m < 1 || m > FDA_STATIC_MAX_M)
      return fail(FDA_ERANGE, "m must be in 1..%d (got %d): the static scratch holds no wider rows", FDA_STATIC_MAX_M, m);
    if (!(eps > -1.0)) return fail(FDA_EINVAL, "eps must be > -1");
  }
  const int bpr = sk ? (m + fda::kEstCols - 1) / fda::kEstCols : 1;
  const int eblocks = sk ? l * bpr : 1;
  if ((size_t)(2 + eblocks) > kStaticPartDoubles)
    return fail(FDA_ERANGE, "internal: %d partial sums do not fit the static scratch", 2 + eblocks);
  unsigned char* base = nullptr;
  int rc = static_scratch(&base);
  if (rc != FDA_OK) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  unsigned int* ticket = reinterpret_cast<unsigned int*>(base + kStaticTicketOffset);
  // the counter must start at zero whatever an earlier call left (a fill kernel, not a memset node)
  hipLaunchKernelGGL(fda::clear_u32_kernel, dim3(1), dim3(64), 0, st, ticket, 1);
  FDA_HIP(hipGetLastError());
  const fda::EstimateArgs args = {variants, sk ? l : 0, sk ? m : 1, K, eps, theta, tie_tol, out_dev, nullptr};
  hipLaunchKernelGGL(fda::estimate_kernel, dim3(eblocks), dim3(fda::kSmallThreads), 0, st, state, args,
                     reinterpret_cast<double*>(base), ticket, static_cast<const fda::PathRecord*>(nullptr));
  FDA_HIP(hipGetLastError());
  return FDA_OK;
}

namespace {
int sync_impl(fda_ctx* ctx, void* w, float* w_t0, float* w_prev, float* xi, const int32_t* pred_dev,
              void* stream);
}
int fda_sync(fda_ctx* ctx, void* w, float* w_t0, float* w_prev, const int32_t* pred_dev,
             void* stream) {
  return sync_impl(ctx, w, w_t0, w_prev, nullptr, pred_dev, stream);
}
int fda_sync_xi(fda_ctx* ctx, void* w, float* w_t0, float* w_prev, float* xi, const int32_t* pred_dev,
                void* stream) {
  if (w_prev == nullptr || xi == nullptr) return fail(FDA_EINVAL, "NULL argument");
  if (reinterpret_cast<uintptr_t>(xi) % 4 != 0) return fail(FDA_EINVAL, "pointer not aligned to its element type");
  return sync_impl(ctx, w, w_t0, w_prev, xi, pred_dev, stream);
}
// the instantiation for the slab type, the streaming hints and the block size.  (Small blocks of slabs beyond
// kStreamBytes, many workers of a small model: 150 x 1M fp32 272 us without the hints, 223 with them, 209 with large
// blocks; 90 x 1572863 291, 277 and 287; 200 x 1.2M 423, 381 and 470; 400 x 500K 337, 291 and 308.)
#define FDA_SYNC_PICK()                                                                                \
  do {                                                                                                 \
    const bool small = sg.vecs == fda::kSyncVecsSmall;                                                  \
    if (d.dtype == FDA_F32) {                                                                          \
      if (small && hinted) FDA_SYNC_LAUNCH(float, true, fda::kSyncVecsSmall);                           \
      else if (small) FDA_SYNC_LAUNCH(float, false, fda::kSyncVecsSmall);                               \
      else if (hinted) FDA_SYNC_LAUNCH(float, true, fda::kSyncVecs);                                    \
      else FDA_SYNC_LAUNCH(float, false, fda::kSyncVecs);                                               \
    } else {                                                                                           \
      if (small && hinted) FDA_SYNC_LAUNCH(fda::bf16_t, true, fda::kSyncVecsSmall);                     \
      else if (small) FDA_SYNC_LAUNCH(fda::bf16_t, false, fda::kSyncVecsSmall);                         \
      else if (hinted) FDA_SYNC_LAUNCH(fda::bf16_t, true, fda::kSyncVecs);                              \
      else FDA_SYNC_LAUNCH(fda::bf16_t, false, fda::kSyncVecs);                                         \
    }                                                                                                  \
  } while (0)
namespace {
// the two models and xi are too large to stay in the memory-side cache: streaming hints
bool xi_streams(int64_t d) { return 12 * d > kStreamBytes; }
// xi = (w_t0 - w_prev) / the norm whose square is spread over npartial sums
int launch_xi_scale(int64_t d, const float* w_t0, const float* w_prev, float* xi, const int32_t* pred_dev,
                    const double* partial, int npartial, hipStream_t st) {
  const SyncGrid sg = sync_grid(d);
  const int per = (int)((sg.blocks * sg.per + kXiScaleBlocks - 1) / kXiScaleBlocks);
  const dim3 grid((unsigned)((sg.blocks * sg.per + per - 1) / per)), block(fda::kSmallThreads);
#define FDA_XI_LAUNCH(S, N)                                                                                  \
  hipLaunchKernelGGL((fda::xi_scale_kernel<S, N>), grid, block, 0, st, w_t0, w_prev, xi, pred_dev, (long long)d, \
                     per, partial, npartial)
  if (sg.vecs == fda::kSyncVecsSmall) FDA_XI_LAUNCH(false, fda::kSyncVecsSmall);
  else if (xi_streams(d)) FDA_XI_LAUNCH(true, fda::kSyncVecs);
  else FDA_XI_LAUNCH(false, fda::kSyncVecs);
#undef FDA_XI_LAUNCH
  FDA_HIP(hipGetLastError());
  return FDA_OK;
}
// xi != NULL: the synchronization kernel also leaves the squared norm of the model change, and xi is
// written by the scaling pass of fda_update_xi alone
int sync_impl(fda_ctx* ctx, void* w, float* w_t0, float* w_prev, float* xi, const int32_t* pred_dev,
              void* stream) {
  if (ctx == nullptr || w == nullptr || w_t0 == nullptr) return fail(FDA_EINVAL, "NULL argument");
  int rcd = check_device(ctx);
  if (rcd != FDA_OK) return rcd;
  const fda_desc& d = ctx->desc;
  const uintptr_t esz = d.dtype == FDA_F32 ? 4 : 2;
  if (reinterpret_cast<uintptr_t>(w) % esz != 0 || reinterpret_cast<uintptr_t>(w_t0) % 4 != 0 ||
      (w_prev && reinterpret_cast<uintptr_t>(w_prev) % 4 != 0))
    return fail(FDA_EINVAL, "pointer not aligned to its element type");
  hipStream_t st = static_cast<hipStream_t>(stream);
  const SyncGrid sg = sync_grid(d.d);
  const bool hinted = (long long)d.K * d.d * (d.dtype == FDA_F32 ? 4 : 2) > kStreamBytes;
  const dim3 grid((unsigned)sg.blocks), block(fda::kSmallThreads);
  double* norm_part = xi != nullptr ? reinterpret_cast<double*>(ctx->ws + ctx->plan.off_syncnorm) : nullptr;
  double* norm_group = reinterpret_cast<double*>(ctx->ws + ctx->plan.off_syncnorm) + sg.blocks;
  unsigned int* ticket = reinterpret_cast<unsigned int*>(ctx->ws + ctx->plan.off_ticket) + ctx->plan.sync_ticket;
  if (xi != nullptr) {
    rcd = clear_tickets_once(ctx, st);
    if (rcd != FDA_OK) return rcd;
  }
#define FDA_SYNC_LAUNCH(T, S, N)                                                                       \
  hipLaunchKernelGGL((fda::sync_kernel<T, S, N>), grid, block, 0, st, static_cast<T*>(w), w_t0, w_prev, \
                     pred_dev, d.K, (long long)d.d, (long long)d.row_stride, sg.per, norm_part, norm_group, ticket)
  FDA_SYNC_PICK();
#undef FDA_SYNC_LAUNCH
  FDA_HIP(hipGetLastError());
  if (xi != nullptr) {
    return launch_xi_scale(d.d, w_t0, w_prev, xi, pred_dev, norm_group,
                           (int)((sg.blocks + fda::kSyncGroup - 1) / fda::kSyncGroup), st);
  }
  return FDA_OK;
}
}  // namespace

int fda_sync_from_mean(fda_ctx* ctx, void* w, float* w_t0, float* w_prev, float* xi,
                       const float* w_bar, const int32_t* pred_dev, void* stream) {
  if (ctx == nullptr || w == nullptr || w_t0 == nullptr || w_bar == nullptr)
    return fail(FDA_EINVAL, "NULL argument");
  int rcd = check_device(ctx);
  if (rcd != FDA_OK) return rcd;
  const fda_desc& d = ctx->desc;
  const uintptr_t esz = d.dtype == FDA_F32 ? 4 : 2;
  if (reinterpret_cast<uintptr_t>(w) % esz != 0 || reinterpret_cast<uintptr_t>(w_t0) % 4 != 0 ||
      reinterpret_cast<uintptr_t>(w_bar) % 4 != 0 || (w_prev && reinterpret_cast<uintptr_t>(w_prev) % 4 != 0) ||
      (xi && reinterpret_cast<uintptr_t>(xi) % 4 != 0))
    return fail(FDA_EINVAL, "pointer not aligned to its element type");
  hipStream_t st = static_cast<hipStream_t>(stream);
  const SyncGrid sg = sync_grid(d.d);
  const bool hinted = (long long)d.K * d.d * (d.dtype == FDA_F32 ? 4 : 2) > kStreamBytes;
  // The rows of a block are split over workgroups where the blocks are few, eight rows or more to each: 60 x 100000
  // fp32 in five parts 7.0 us, in one 14.0.  (From 512 blocks on one part: 60 x 500000, 489 blocks, 22.0.)
  long long splits = kRowWorkgroups / sg.blocks;
  if (splits > d.K / kRowsAtLeast) splits = d.K / kRowsAtLeast;
  if (splits < 1) splits = 1;
  const int rows = (int)((d.K + splits - 1) / splits);
  const dim3 grid((unsigned)sg.blocks, (unsigned)((d.K + rows - 1) / rows)), block(fda::kSmallThreads);
  const double* dnorm = reinterpret_cast<const double*>(ctx->ws + ctx->plan.off_dnorm);
#define FDA_SYNC_LAUNCH(T, S, N)                                                                       \
  hipLaunchKernelGGL((fda::sync_from_mean_kernel<T, S, N>), grid, block, 0, st, static_cast<T*>(w), w_t0, w_prev, \
                     xi, w_bar, dnorm, pred_dev, d.K, rows, (long long)d.d, (long long)d.row_stride, sg.per)
  FDA_SYNC_PICK();
#undef FDA_SYNC_LAUNCH
  FDA_HIP(hipGetLastError());
  return FDA_OK;
}

int fda_update_xi(fda_ctx* ctx, const float* w_t0, const float* w_prev, float* xi,
                  const int32_t* pred_dev, void* stream) {
  if (ctx == nullptr || w_t0 == nullptr || w_prev == nullptr || xi == nullptr)
    return fail(FDA_EINVAL, "NULL argument");
  int rcd = check_device(ctx);
  if (rcd != FDA_OK) return rcd;
  const fda_desc& d = ctx->desc;
  if (reinterpret_cast<uintptr_t>(w_t0) % 4 != 0 || reinterpret_cast<uintptr_t>(w_prev) % 4 != 0 ||
      reinterpret_cast<uintptr_t>(xi) % 4 != 0)
    return fail(FDA_EINVAL, "pointer not aligned to its element type");
  hipStream_t st = static_cast<hipStream_t>(stream);
  double* partial = reinterpret_cast<double*>(ctx->ws + ctx->plan.off_xi);
  long long blocks = (d.d + fda::sync_block(fda::kSyncVecs) - 1) / fda::sync_block(fda::kSyncVecs);
  if (blocks > kXiBlocks) blocks = kXiBlocks;
  if (xi_streams(d.d))
    hipLaunchKernelGGL(fda::xi_norm_kernel<true>, dim3((unsigned)blocks), dim3(fda::kSmallThreads), 0, st,
                       w_t0, w_prev, pred_dev, (long long)d.d, partial);
  else
    hipLaunchKernelGGL(fda::xi_norm_kernel<false>, dim3((unsigned)blocks), dim3(fda::kSmallThreads), 0, st,
                       w_t0, w_prev, pred_dev, (long long)d.d, partial);
  FDA_HIP(hipGetLastError());
  return launch_xi_scale(d.d, w_t0, w_prev, xi, pred_dev, partial, (int)blocks, st);
}

int fda_step(fda_ctx* ctx, void* w, float* w_t0, float* w_prev, float* xi, float* state, float* w_bar,
             double theta, double tie_tol, int32_t decide_by, int32_t flags, fda_estimate* out_dev,
             fda_estimate* out_host, void* stream) {
  if (ctx == nullptr || out_dev == nullptr) return fail(FDA_EINVAL, "NULL argument");
  if ((decide_by != FDA_VARIANT_LINEAR && decide_by != FDA_VARIANT_SKETCH) ||
      !(ctx->desc.variants & decide_by))
    return fail(FDA_EINVAL, "decide_by must be one of the context's variants");
  if ((flags & ~FDA_STEP_MEAN_STATE) != 0) return fail(FDA_EINVAL, "unknown flags");
  if (xi != nullptr && w_prev == nullptr) return fail(FDA_EINVAL, "w_prev is required when xi is given");
  const bool mean = (flags & FDA_STEP_MEAN_STATE) != 0;
  if (!mean && w_bar != nullptr) return fail(FDA_EINVAL, "w_bar needs FDA_STEP_MEAN_STATE");
  // (the synchronization checks this too, but a step that reads its decision back may end before it)
  if (reinterpret_cast<uintptr_t>(w_prev) % 4 != 0) return fail(FDA_EINVAL, "pointer not aligned to its element type");
  const int32_t* pred = reinterpret_cast<const int32_t*>(
      reinterpret_cast<const unsigned char*>(out_dev) +
      (decide_by == FDA_VARIANT_LINEAR ? offsetof(fda_estimate, sync_linear)
                                       : offsetof(fda_estimate, sync_sketch)));
  // the estimate is part of the launch that merges the partials of the state pass
  fda::EstimateArgs est;
  int rc = estimate_args(ctx, mean ? 1 : ctx->desc.K, theta, tie_tol, out_dev, &est);
  if (rc != FDA_OK) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (out_host != nullptr) want_result(ctx, &est);
  rc = mean ? mean_state_pass(ctx, w, w_t0, xi, state, w_bar, &est, stream) : local_state(ctx, w, w_t0, xi, state, &est, stream);
  if (rc != FDA_OK) return rc;
  if (out_host != nullptr) {
    // The program waits for the decision: what depends on it is enqueued when it is known, and most steps end
    // here -- two launches less in front of the wait (10 us).
    rc = read_result(est, out_host, st);
    if (rc != FDA_OK) return rc;
    if ((decide_by == FDA_VARIANT_LINEAR ? out_host->sync_linear : out_host->sync_sketch) == 0) return FDA_OK;
  }
  if (w_bar != nullptr) {
    rc = fda_sync_from_mean(ctx, w, w_t0, w_prev, xi, w_bar, pred, stream);
  } else {
    rc = xi != nullptr ? fda_sync_xi(ctx, w, w_t0, w_prev, xi, pred, stream)
                       : fda_sync(ctx, w, w_t0, w_prev, pred, stream);
  }
  if (rc != FDA_OK) return rc;
  if (out_host != nullptr) FDA_HIP(wait_for(st));
  return FDA_OK;
}

}  // extern "C"

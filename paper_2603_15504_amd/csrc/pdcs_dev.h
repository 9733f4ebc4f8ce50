// Device-side definitions shared by the PDCS kernels (gfx950, wave64).
//
// Data layout.  A launch covers a batch of B >= 1 LPs packed block-diagonally:
// instance b owns rows [row0, row0 + rows) and columns [col0, col0 + cols) of
// the concatenated matrix and of every m- and n-vector.  Work is handed out to
// workgroups through per-workgroup ranges that never straddle two instances,
// so every workgroup reads its instance's scalars once and writes one
// deterministic partial-sum record; a per-instance finalize kernel reduces the
// records of its instance in a fixed order (no floating-point atomics).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pdcs {

constexpr int kWave = 64;
constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kProbes = 16;        // t values per bisection pass
constexpr int kCheckCoarsen = 8;   // multisection passes: blocks this many times larger than the trial passes
constexpr int kMaxCand = 2;        // restart candidates: current PDHG output, average

enum Status : int32_t { kActive = 0, kDone = 1 };
enum Prec : int32_t { kFP64 = 0, kFP32 = 1 };

// Bisection phases for the normalized duality gap.
enum Phase : int32_t { kPhaseOff = 0, kPhaseExp = 1, kPhaseBisect = 2, kPhaseDone = 3 };

struct CandState {
  // reductions of the candidate pass
  double dxa2, dya2;        // ||x_c - x_a||^2, ||y_c - y_a||^2
  double r, scale;          // N-norm radius and sqrt(tau|b1|^2 + sigma|b2|^2)
  double errp, errd, gap, pobj, dobj, kkt;   // scaled L2 errors and KKT_omega
  double abs_p, abs_d, abs_gap, rel_p, rel_d, rel_gap;   // unscaled inf-norm errors
  // bisection state
  double t_lo, t_hi, t_base, val_lo, last_dist;
  int32_t phase, doublings, bracketed, pad;
  double rho;
};

// Per-instance scalar state.  Written only by the single-block finalize
// kernels (thread 0) and by the host at set-up.
struct Inst {
  // geometry
  int32_t row0, rows, col0, cols;
  int32_t m_zero, precision, status, exit_code;
  // step size, weight, reflection
  double omega, omega0, eta, eta_hat, eta_k, beta;
  double ca, cb;            // Halpern coefficients (k+1)/(k+2), 1/(k+2) of the pending commit
  double sum_eta;           // sum of accepted eta in the current restart interval
  // norms of the rescaled data (and inf-norms of the unscaled data)
  double h1, c1, h2, c2, gmax, h_inf, c_inf;
  // counters
  int64_t kbar, k, t, accepted, restarts, checks, fp64_iters, max_iter;
  int64_t check_every;
  int32_t pending, last_acc, check_due, method;
  int32_t use_avg, has_anchor, has_prev, switch_fp64;
  // line-search reductions kept for the reflection parameter
  double dx2, dy2, dydgdx, errp2, hy, cx;
  // restart bookkeeping
  double rho_anchor, kkt_anchor, rho_prev, kkt_prev;
  int32_t restart, chosen, optimal, use_kkt;
  int32_t force_kkt;  // option: restart decisions on KKT_omega instead of the normalized gap
  double best_rel, rel_tol, abs_tol, polish_tol, bisect_eps;
  int64_t stall, stall_checks;
  double best_any;    // lowest relative KKT error of the FP32 phase
  int64_t stall_any;  // checks since that record
  // termination errors of the last evaluated point
  double pobj, dobj, abs_p, abs_d, abs_gap, rel_p, rel_d, rel_gap;
  CandState cand[kMaxCand];
  double chk_rho[kMaxCand], chk_r[kMaxCand];  // values of the last restart check
  // infeasibility tests of the option list of Section 3 (exit codes 2-5)
  double eps_inf[4];        // tolerances: primal low, dual low, primal high, dual high
  double ratio_p, ratio_d;  // ratios of the last check (NaN: not evaluated)
  double prev_dobj, prev_negp;  // dual objective and -(primal objective) of z_hat at the previous check
  int32_t infeas_on, ray_due, trend_p, trend_d;
  int32_t has_prev_obj, stop_max_iter;
  int32_t soc_start;        // first second-order-cone row (row0 + rows when none)
  int32_t pad_inf1;
  double* trace;            // per-trial scalars of the first trace_cap trials (or null)
  int64_t trace_cap;
};
constexpr int kTrendChecks = 3;  // consecutive checks the low-accuracy infeasibility tests must pass
constexpr int kTraceStride = 16;  // kbar, eta, eta_bar, dx2, dy2, dy^T G dx, accepted, eta', beta, k,
                                  // then for accepted trials: c^T x_hat, h^T y_hat, sum l lam+, sum u lam-, err_p^2, err_d^2

// Row-block schedule of a CSR-like pass (one workgroup per block): either a
// single row of any length, or several consecutive rows holding at most
// kRowBlockCap nonzeros, which are staged as products in LDS.
constexpr int kRowBlockCap = 2048;
struct RowBlocks {
  const int32_t* blk_row0;     // first row of the block
  const int32_t* blk_row1;     // one past the last row
  const int32_t* blk_inst;     // instance (or panel) of the block
  const int32_t* inst_blk0;    // per instance: first block (B+1 entries)
  int32_t nblk;
};

// Band-tile layout of a sparse matrix for single large instances.  A band-tile
// holds the entries of one band of at most kBandRows consecutive rows whose
// gathered index falls in one window of at most 2^kBandColBits indices.  Its
// entries are sorted by gathered index and padded to whole iterations of
// kBandUnroll * kWave entries; entry e packs (index - window start) <<
// kBandSlotBits | slot, where slot < kBandSlots names the LDS accumulator it
// adds into: slots below the band's row count are the rows themselves, higher
// slots are extra accumulators of rows that repeat within one group of kWave
// consecutive entries (no two entries of such a group share a slot), and slot
// BandTiles::slots - 1 is the sink of the padding.  The extra slots of a row are
// consecutive.  A workgroup is one wave with one band-tile.  In a batch every instance has its
// own bands and windows; an instance with fewer windows than the batch's
// largest count has empty tiles (zero partial sums) for the missing ones.
constexpr int kBandRows = 8192;
constexpr int kBandSlots = 9216;
constexpr int kBandSlotBits = 14;
constexpr int kBandColBits = 32 - kBandSlotBits;
// (One wave, one band-tile per workgroup: tiles then spread evenly over the CUs,
// where pairs left some CUs two workgroups to do and others one.  m = 2.5e5,
// n = 5e5, power-law rows, nnz = 1.35e7, 540 tiles, G x and G^T y: FP32 110 us in
// pairs, 99 alone, FP64 153 and 130; m = 2e5, n = 5e5: 51 / 66 either way; a trial
// of 48 LPs in FP64: 108 and 99 us.)
constexpr int kBandUnroll = 16;
// All that a workgroup needs to know of its band-tile, in one read of its launch slot.
struct alignas(16) BandTile {
  int32_t tile;   // number of the band-tile, -1: an idle slot (all else 0)
  int32_t start;  // first entry
  int32_t nit;    // iterations of kBandUnroll * kWave entries
  int32_t row0;   // first row
  int32_t nrows;  // rows
  int32_t used;   // slots in use (rows + extra slots; the sink excluded)
  int32_t col0;   // window start
  int32_t panel;  // window index (partial-sum array)
  int64_t fold0;  // first entry in BandTiles::fold
  int32_t inst;   // instance (bands never cross instances)
  int32_t nfold;  // rows with extra slots
};
struct BandTiles {
  const BandTile* slot;      // launch slots; slot s runs on XCD s % 8
  const uint2* fold;         // per row with extra slots: row | extra slots << 16, first extra slot
  const uint32_t* pk;        // packed entries
  int32_t nslot;             // launch slots (workgroups)
  int32_t P;                 // windows
  int32_t slots;             // LDS accumulators: the most a tile uses, and the sink
};

// Schedule of an elementwise pass: contiguous element ranges per workgroup.
// Row ranges never split a cone block: the blocks inside range b are
// [blk_soc0[b], blk_soc1[b]) of the table (soc_r0: first row, soc_dim:
// dimension, soc_kind: 0 second-order cone, 1 exponential cone, 2 dual
// exponential cone; second-order cones first); all six are null when no instance has cone blocks.
struct Ranges {
  const int32_t* blk_start;
  const int32_t* blk_end;
  const int32_t* blk_inst;
  const int32_t* inst_blk0;    // per instance: first workgroup (B+1 entries)
  const int32_t* blk_soc0;
  const int32_t* blk_soc1;
  const int32_t* blk_exp0;     // first exponential cone of the range (blk_soc1 when none)
  const int32_t* soc_r0;
  const int32_t* soc_dim;
  const int8_t* soc_kind;
  int32_t nblk;
};

// ---------------------------------------------------------------------------
// Reductions
// ---------------------------------------------------------------------------
// One DPP lane move of a double (both 32-bit halves with the same control):
// lanes whose source is outside the pattern, or whose row is masked off,
// receive +0.0.
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ double dpp_move(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROW_MASK, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROW_MASK, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// Sum over the 64 lanes, returned to every lane: data-parallel-primitive lane
// moves inside the VALU instead of LDS-crossbar shuffles.  Pairs and quads
// (quad permutes), then rows of 16 (row shifts by 4 and 8: lane 15 of a row
// holds its row's sum), then rows 1 and 3 take lane 15 of the row before and
// rows 2 and 3 take lane 31, so lane 63 holds the total, which is read back
// as a uniform value.  Fixed order: deterministic.
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_move<0xB1>(v);        // quad_perm [1,0,3,2]
  v += dpp_move<0x4E>(v);        // quad_perm [2,3,0,1]
  v += dpp_move<0x114>(v);       // row_shr:4
  v += dpp_move<0x118>(v);       // row_shr:8
  v += dpp_move<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
  v += dpp_move<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, 63), hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, kWave));
  return v;
}

// Between an LDS access of one lane and another lane's of the same wave to the same
// place.  The hardware executes a wave's LDS instructions in order; the fence keeps the
// compiler from moving them past each other, and is no instruction itself.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Sum NV values over the workgroup; thread 0..NV-1 of the block write out[i].
// lds must hold WAVES * NV doubles.  Order is fixed: deterministic.
template <int NV, int WAVES = kWavesPerBlock>
__device__ __forceinline__ void block_sum_store(double (&v)[NV], double* lds, double* out) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    double s = wave_sum(v[i]);
    if (lane == 0) lds[wave * NV + i] = s;
  }
  __syncthreads();
  if (threadIdx.x < NV) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) s += lds[w * NV + threadIdx.x];
    out[threadIdx.x] = s;
  }
}

// Totals of 32 values over the wave: lane l gets that of value bitrev5(l % 32).
// Each step halves the values a lane carries (31 exchanges and additions for
// 32 separate sums' 192), and adds in wave_sum's tree: the same bits.
template <int N>
__device__ __forceinline__ void sum_step(double (&v)[32]) {
  constexpr int off = 16 / N;
  const bool up = (threadIdx.x & off) != 0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const double lo = v[i], hi = v[i + N];
    v[i] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, off, kWave);
  }
}

__device__ __forceinline__ double wave_sum32(double (&v)[32]) {
  sum_step<16>(v);
  sum_step<8>(v);
  sum_step<4>(v);
  sum_step<2>(v);
  sum_step<1>(v);
  return v[0] + __shfl_xor(v[0], 32, kWave);
}

// block_sum_store of 32 values by it.
__device__ __forceinline__ void block_sum32_store(double (&v)[32], double* lds, double* out) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const double s = wave_sum32(v);
  if (lane < 32) lds[wave * 32 + (int)(__brev((unsigned)lane) >> 27)] = s;
  __syncthreads();
  if (threadIdx.x < 32) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kWavesPerBlock; ++w) t += lds[w * 32 + threadIdx.x];
    out[threadIdx.x] = t;
  }
}

// As block_sum_store, but the first NS entries are sums and the rest maxima.
template <int NV, int NS>
__device__ __forceinline__ void block_summax_store(double (&v)[NV], double* lds, double* out) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    double s = (i < NS) ? wave_sum(v[i]) : wave_max(v[i]);
    if (lane == 0) lds[wave * NV + i] = s;
  }
  __syncthreads();
  if (threadIdx.x < NV) {
    const int i = threadIdx.x;
    double s = lds[i];
    for (int w = 1; w < kWavesPerBlock; ++w) s = (i < NS) ? s + lds[w * NV + i] : fmax(s, lds[w * NV + i]);
    out[i] = s;
  }
}

// Reduce the NV-wide records [b0, b1) of one instance inside one workgroup;
// the first NS fields are summed, the rest take the maximum.  Result is
// returned to every thread.  Fixed order: deterministic.
template <int NV, int NS>
__device__ __forceinline__ void reduce_records(const double* rec, int b0, int b1, double* lds,
                                               double (&res)[NV]) {
  if (b1 - b0 == 1) {  // a single record (uniform across the workgroup): every thread reads it
#pragma unroll
    for (int i = 0; i < NV; ++i) res[i] = rec[(size_t)b0 * NV + i];
    return;
  }
  double acc[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) acc[i] = 0.0;
  // four records per step: independent loads in flight before they are combined
  constexpr int U = NV <= 8 ? 4 : 1;
  int b = b0 + (int)threadIdx.x;
  for (; b + (U - 1) * kBlock < b1; b += U * kBlock) {
    double v[U][NV];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < NV; ++i) v[u][i] = rec[(size_t)(b + u * kBlock) * NV + i];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < NV; ++i) acc[i] = (i < NS) ? acc[i] + v[u][i] : fmax(acc[i], v[u][i]);
  }
  for (; b < b1; b += kBlock) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      double v = rec[(size_t)b * NV + i];
      acc[i] = (i < NS) ? acc[i] + v : fmax(acc[i], v);
    }
  }
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    double s = (i < NS) ? wave_sum(acc[i]) : wave_max(acc[i]);
    if (lane == 0) lds[wave * NV + i] = s;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    double s = lds[i];
    for (int w = 1; w < kWavesPerBlock; ++w) s = (i < NS) ? s + lds[w * NV + i] : fmax(s, lds[w * NV + i]);
    res[i] = s;
  }
  __syncthreads();
}

// reduce_records in two halves, for a workgroup that has other loads to issue in
// between, over at most kFoldRecords records of sums.  records_load: this thread's
// share.  records_store: the waves' sums into lds (kWavesPerBlock * NV doubles);
// after a barrier, records_total adds them (any thread).  The same order, and the
// same bits, as reduce_records.
constexpr int kFoldRecords = 2 * kBlock;
template <int NV>
__device__ __forceinline__ void records_load(const double* __restrict__ rec, int b0, int b1, double (&v)[NV]) {
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = 0.0;
  if (b1 <= b0) return;
  const int k0 = b0 + (int)threadIdx.x, k1 = k0 + kBlock;
  double a[NV], b[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) a[i] = rec[(size_t)min(k0, b1 - 1) * NV + i];
#pragma unroll
  for (int i = 0; i < NV; ++i) b[i] = rec[(size_t)min(k1, b1 - 1) * NV + i];
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = (k0 < b1 ? a[i] : 0.0) + (k1 < b1 ? b[i] : 0.0);
}
template <int NV>
__device__ __forceinline__ void records_store(const double (&v)[NV], double* lds) {
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const double s = wave_sum(v[i]);
    if ((threadIdx.x & (kWave - 1)) == 0) lds[threadIdx.x / kWave * NV + i] = s;
  }
}
template <int NV>
__device__ __forceinline__ void records_total(const double* lds, double (&v)[NV]) {
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    v[i] = lds[i];
    for (int w = 1; w < kWavesPerBlock; ++w) v[i] += lds[w * NV + i];
  }
}

// Products of entries [0, n) of a row block with NV vectors into LDS, n <= 256 U:
// every index and value is requested before the first gather, and every gather
// before the first product (entries past the end repeat the last one, whose LDS
// slots past n nobody reads).
// early() runs while the gathers are in flight.
template <int U, int NV, typename TM, typename TV, class Early>
__device__ __forceinline__ void stage_products(int n, const int32_t* __restrict__ idx, const TM* __restrict__ val,
                                               const TV* const (&xs)[NV], double* lds, Early&& early) {
  const int tid = threadIdx.x;
  int c[U];
  TM v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = min(u * kBlock + tid, n - 1);
    c[u] = __builtin_nontemporal_load(idx + i);
    v[u] = __builtin_nontemporal_load(val + i);
  }
  TV g[NV][U];
#pragma unroll
  for (int k = 0; k < NV; ++k)
#pragma unroll
    for (int u = 0; u < U; ++u) g[k][u] = xs[k][c[u]];
  early();
#pragma unroll
  for (int k = 0; k < NV; ++k)
#pragma unroll
    for (int u = 0; u < U; ++u) lds[k * kRowBlockCap + u * kBlock + tid] = (double)v[u] * (double)g[k][u];
}

// Products of one row block with NV gathered vectors, reduced per row; fn(r, s, d)
// is called exactly once per row r of the block, by one thread, with s[k] the
// row's dot product with xs[k] (FP64 accumulation) and d what pre(r) returned:
// pre loads what the row's epilogue needs, and is called before the products are
// formed, so that those loads are in flight with them.  early() is called once by
// every thread with the gathers in flight, mid() (which may synchronize) once they
// are done and before the first fn.  lds:
// NV * kRowBlockCap doubles plus kWavesPerBlock * NV doubles.  Every thread of
// the workgroup must call this (it synchronizes).
template <int NV, typename TM, typename TV, class Pre, class Early, class Mid, class Fn>
__device__ __forceinline__ void block_rows(int r0, int r1, const int32_t* __restrict__ ptr,
                                           const int32_t* __restrict__ idx, const TM* __restrict__ val,
                                           const TV* const (&xs)[NV], double* lds, Pre&& pre, Early&& early, Mid&& mid, Fn&& fn) {
  const int tid = threadIdx.x;
  const int R = r1 - r0;
  const int q0 = ptr[r0], q1 = ptr[r1];
  if (R == 1) {
    // one row of any length: register accumulation, unrolled streaming loads
    const auto d = pre(r0);
    early();
    double s[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) s[k] = 0.0;
    int q = q0 + tid;
    for (; q + 3 * kBlock < q1; q += 4 * kBlock) {
      int c[4];
      double v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        c[u] = __builtin_nontemporal_load(idx + q + u * kBlock);
        v[u] = (double)__builtin_nontemporal_load(val + q + u * kBlock);
      }
#pragma unroll
      for (int k = 0; k < NV; ++k)
#pragma unroll
        for (int u = 0; u < 4; ++u) s[k] += v[u] * (double)xs[k][c[u]];
    }
    for (; q < q1; q += kBlock) {
      const int c = __builtin_nontemporal_load(idx + q);
      const double v = (double)__builtin_nontemporal_load(val + q);
#pragma unroll
      for (int k = 0; k < NV; ++k) s[k] += v * (double)xs[k][c];
    }
    double* red = lds + NV * kRowBlockCap;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const double w = wave_sum(s[k]);
      if (lane == 0) red[wave * NV + k] = w;
    }
    mid();
    __syncthreads();
    if (tid == 0) {
      double t[NV];
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        t[k] = 0.0;
        for (int w = 0; w < kWavesPerBlock; ++w) t[k] += red[w * NV + k];
      }
      fn(r0, t, d);
    }
    return;
  }
  // several rows, at most kRowBlockCap nonzeros: stage the products in LDS
  const int n = q1 - q0;
  if (R <= kBlock) {
    int T = 64;
    while (T > 1 && T * R > kBlock) T >>= 1;
    const int g = min(tid / T, R - 1), li = tid & (T - 1);
    const int r = r0 + g;
    const int a = ptr[r] - q0, e = ptr[r + 1] - q0;
    const auto d = pre(r);
    if (n > 4 * kBlock) stage_products<8, NV>(n, idx + q0, val + q0, xs, lds, early);
    else if (n > 0) stage_products<4, NV>(n, idx + q0, val + q0, xs, lds, early);
    else early();
    mid();
    __syncthreads();
    double s[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) s[k] = 0.0;
    for (int i = a + li; i < e; i += T)
#pragma unroll
      for (int k = 0; k < NV; ++k) s[k] += lds[k * kRowBlockCap + i];
#pragma unroll
    for (int k = 0; k < NV; ++k)
      for (int off = T >> 1; off > 0; off >>= 1) s[k] += __shfl_xor(s[k], off, kWave);
    if (li == 0 && tid / T < R) fn(r, s, d);
  } else {
    if (n > 4 * kBlock) stage_products<8, NV>(n, idx + q0, val + q0, xs, lds, early);
    else if (n > 0) stage_products<4, NV>(n, idx + q0, val + q0, xs, lds, early);
    else early();
    mid();
    __syncthreads();
    for (int r = r0 + tid; r < r1; r += kBlock) {
      const int a = ptr[r] - q0, e = ptr[r + 1] - q0;
      const auto d = pre(r);
      double s[NV];
#pragma unroll
      for (int k = 0; k < NV; ++k) s[k] = 0.0;
      for (int i = a; i < e; ++i)
#pragma unroll
        for (int k = 0; k < NV; ++k) s[k] += lds[k * kRowBlockCap + i];
      fn(r, s, d);
    }
  }
}

template <int NV, typename TM, typename TV, class Pre, class Fn>
__device__ __forceinline__ void block_rows(int r0, int r1, const int32_t* __restrict__ ptr,
                                           const int32_t* __restrict__ idx, const TM* __restrict__ val,
                                           const TV* const (&xs)[NV], double* lds, Pre&& pre, Fn&& fn) {
  block_rows<NV>(r0, r1, ptr, idx, val, xs, lds, pre, [] {}, [] {}, fn);
}

// block_rows with no epilogue data: fn(r, s).
struct NoRow {};
template <int NV, typename TM, typename TV, class Fn>
__device__ __forceinline__ void block_rows(int r0, int r1, const int32_t* __restrict__ ptr,
                                           const int32_t* __restrict__ idx, const TM* __restrict__ val,
                                           const TV* const (&xs)[NV], double* lds, Fn&& fn) {
  block_rows<NV>(r0, r1, ptr, idx, val, xs, lds, [](int) { return NoRow{}; },
                 [&](int r, const double* s, const NoRow&) { fn(r, s); });
}

__device__ __forceinline__ double clampd(double v, double lo, double hi) {
  return fmin(fmax(v, lo), hi);
}

}  // namespace pdcs

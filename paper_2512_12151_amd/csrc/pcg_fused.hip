// One-kernel PCG iteration for systems of up to kFusedMaxSlices slices, the
// sizes at which the two-kernel iteration of pcg.hip spends its time in kernel
// boundaries and in chains of dependent loads, not in bytes.
//
// alpha_k and beta_k are both known once p^T q, r^T q and q^T q of iteration k
// are (|r - alpha q|^2 by its expansion, see pcg.hip), so an iteration needs
// one grid-wide reduction.  The launch at state k = (r_k, p_k, q_k and their
// sums) therefore does the whole of
//   r_{k+1} = r_k - alpha q_k,  p_{k+1} = r_{k+1} + beta p_k,
//   x += alpha p_k,  q_{k+1} = H_hat p_{k+1}
// and the partial sums of the next one.  Where the product needs p_{k+1} of
// another row it forms it from that row's r_k, q_k and p_k (the two FMAs the
// row's owner applies, so every copy has the same bits): three gathered
// vectors instead of one, which is cheap while the vectors sit in the caches
// and buys a kernel boundary (about 5 us of a 15 us iteration at 3k to 25k
// nodes).  r, p and q alternate between two buffers, because other workgroups
// still read the old ones.
//
// A slice (64 rows) belongs to kSliceWaves wavefronts.  They take its pairs of upper
// and lower slots in turn, up to kRoundPairs each per round, with every load
// of the round in flight at once, and leave the products B p_c and B^T p_r in
// LDS; then one thread per vector entry adds them in the slots' order, upper
// before lower, which is the order of the one-wavefront SpMV: the same sums,
// bit for bit, but two memory round trips deep instead of two per four slots.
//
// The residual replacement (pcg.hip) runs in the same kernel: the state's
// mode says what a launch does, and no host round trip is needed.
//   kNormal   test r_k, then the step above
//   kTested   the same, r_k was tested already
//   kFresh    r_k is given (the start, or just replaced): form p_k =
//             r_k + beta p_{k-1} and q_k
//   kReplace  r_k = b_hat - H_hat x in FP64 from the FP32 blocks
// The state is double-buffered by the parity of the launch, which the host
// toggles: a launch reads one copy and its workgroup 0 writes the other.
// Launches after the end copy the state on and return.
//
// Measured (us of kernel time per iteration, two kernels against this one):
// 250 nodes 9.1 -> 6.1, 2,880 nodes 14.7 -> 6.8, 24,565 nodes 15.8 -> 9.0.  A
// launch of 7 us spends about 2.9 us outside its own code (dispatch, the drain
// of its stores) and 1.7 us in loads that wait for loads: the state and the
// slot offsets, then the indices, then the gathers, behind which the sums hide.
#include <hip/hip_ext.h>

#include <type_traits>

#include "pcg_device.h"

namespace bfal {

namespace {

constexpr int kSliceWaves = 4;                                   // wavefronts per slice and workgroup
constexpr int kFusedBlock = kSliceWaves * kWave;
constexpr int kRoundPairs = 2;                                   // slot pairs per wavefront and round
constexpr int kRound = kSliceWaves * kRoundPairs;
constexpr int kRow3 = 3 * kSlice;                                // vector entries of a slice
constexpr int kRecPerLane = kFusedMaxSlices / kWave;             // partials per lane of a sum
static_assert(kFusedMaxSlices % kWave == 0 && kRow3 == 3 * kWave, "wavefronts 0-2 own the entries, 3 the norms");

// Loads at a 32-bit byte offset from a uniform base: one address register each
// instead of two (fused_groups admits a system only if they reach every array).
struct F3 { float v[3]; };
struct F9 { float v[9]; };
struct U5 { uint32_t v[5]; };

template <class T>
__device__ __forceinline__ T at32(const void* __restrict__ base, unsigned byte) {
  return *reinterpret_cast<const T*>(static_cast<const char*>(base) + byte);
}

template <class T>
__device__ __forceinline__ void put32(T* __restrict__ base, unsigned byte, T v) {
  *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + byte) = v;
}

__device__ __forceinline__ void load_block32(const float* __restrict__ base, unsigned slot, float b[9]) {
  const F9 w = at32<F9>(base, 36u * slot);
#pragma unroll
  for (int m = 0; m < 9; ++m) b[m] = w.v[m];
}

__device__ __forceinline__ void load_block32(const uint32_t* __restrict__ base, unsigned slot, float b[9]) {
  const U5 w = at32<U5>(base, 20u * slot);
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    b[2 * m] = __uint_as_float(w.v[m] << 16);
    b[2 * m + 1] = __uint_as_float(w.v[m] & 0xffff0000u);
  }
  b[8] = __uint_as_float(w.v[4] << 16);
}

// Partial sum m (r^T r, |L r|^2, p^T q, r^T q, q^T q) of state k, one per
// workgroup; and r^T r and |L r|^2 of a replaced residual, in a place of their
// own: the launch that reads them (kFresh) writes the sums of the same k, and
// its workgroups do not run in step.
__device__ __forceinline__ double* record(const PcgSystem& S, int k, int m) {
  return S.part + ((k & 1) * 5 + m) * kFusedMaxSlices;
}
__device__ __forceinline__ double* replaced_record(const PcgSystem& S, int m) {
  return S.part + (10 + m) * kFusedMaxSlices;
}

// Workgroups of the resident launch of this parity that have started, and
// kApart if one of them gave up waiting for the others.
constexpr unsigned kApart = 0x80000000u;
__device__ __forceinline__ unsigned* start_word(const PcgSystem& S, int par) {
  return resident_start(S) + par * (kStartWords / 2);
}

// The launch's report to the host (pinned memory): launches made and, once
// the solve has ended, the end's code and the iteration it ended at.
__device__ __forceinline__ void report(const PcgSystem& S, int launches, int done, int k) {
  if (!S.hstat || (!done && (launches & S.report_mask))) return;
  if (done) {
    __hip_atomic_store(&S.hstat[kWordIter], (unsigned long long)(unsigned)k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __threadfence_system();
  }
  __hip_atomic_store(&S.hstat[kWordState], ((unsigned long long)(unsigned)launches << 32) | (unsigned)done,
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The next launch's state; with an end code also the solver's scalars.
__device__ __forceinline__ void hand_on(const PcgSystem& S, PcgCtl next, int par) {
  ++next.launches;
  S.sc->ctl[par ^ 1] = next;
  *start_word(S, par ^ 1) = 0;
  S.sc->iter = S.sc->xbase = next.k;   // x holds every direction so far
  if (next.done == kEndBreakdown) {
    S.sc->flags |= FLAG_BREAKDOWN;
    S.sc->brk = 1;
  } else if (next.done) {
    S.sc->done = next.done;
  }
  report(S, next.launches, next.done, next.k);
}

// kReplace: r_k = b_hat - H_hat x in FP64 for the workgroup's slice (by one
// wavefront, in k_residual64's order), rounded to FP32, with r^T r and |L r|^2.
__device__ __forceinline__ void replace_residual(const PcgSystem& S, PcgCtl c, int sl, int par) {
  const int t = threadIdx.x;
  if (t >= kWave) return;
  double a0, a1, a2, rr = 0.0, rt = 0.0;
  row_product64(S, sl, t, S.x, a0, a1, a2);
  const int row = sl * kSlice + t;
  if (row < S.N) {
    double r0, r1, r2;
    rt = row_residual64(S, row, S.bhat, S.x, a0, a1, a2, r0, r1, r2);
    float* r = S.r + (c.k & 1) * S.pstride + 3LL * row;
    const float f0 = (float)r0, f1 = (float)r1, f2 = (float)r2;
    r[0] = f0;
    r[1] = f1;
    r[2] = f2;
    rr = (double)f0 * f0 + (double)f1 * f1 + (double)f2 * f2;
  }
  rr = wave_sum_all(rr);
  rt = wave_sum_all(rt);
  if (t == 0) {
    replaced_record(S, 0)[sl] = rr;
    replaced_record(S, 1)[sl] = rt;
    if (sl == 0) {
      c.mode = kFresh;
      hand_on(S, c, par);
    }
  }
}

template <class BT>
struct Slice {   // what a launch knows of its slice before the state
  int bu, bl, wu, wl, w;
  int uc[kRoundPairs], ub[kRoundPairs], lc[kRoundPairs];

  __device__ __forceinline__ void load_indices(const PcgSystem& S, int kk0, int lane) {
#pragma unroll
    for (int j = 0; j < kRoundPairs; ++j) {
      // past a width the last slot is read again (a slice without slots reads
      // the next slice's, or the arrays' padding) and its product is not added
      const int kk = kk0 + kSliceWaves * j;
      uc[j] = at32<int>(S.scol + bu, 4u * (unsigned)(max(min(kk, wu - 1), 0) * kSlice + lane));
      const int2 q = at32<int2>(S.sent + bl, 8u * (unsigned)(max(min(kk, wl - 1), 0) * kSlice + lane));
      ub[j] = q.x;
      lc[j] = q.y;
    }
  }
};

// One launch at a state to step from (kFreshState: to start or resume from).
template <class BT, bool kFreshState>
__device__ __forceinline__ void iterate(const PcgSystem& S, const PcgCtl& c, Slice<BT>& sl, int s, int par) {
  __shared__ float prod[2][kRound][2][kRow3];
  __shared__ float rsh[kRow3];
  __shared__ double sums[5], tail[kSliceWaves][5];
  const int t = threadIdx.x, lane = t % kWave, wv = __builtin_amdgcn_readfirstlane(t / kWave);
  const int k = c.k, ko = kFreshState ? k : k + 1;   // ko: iteration of the outputs
  // vectors: at a fresh state p_k = fma(beta, p_{k-1}, r_k), r_k stays; at k = 0 beta = 0 and r stands in for p
  const float* __restrict__ rin = S.r + (k & 1) * S.pstride;
  const float* __restrict__ qin = S.q + (k & 1) * S.pstride;
  const float* __restrict__ pin = kFreshState && k == 0 ? rin : S.P + ((ko + 1) & 1) * S.pstride;
  // partial sums of state k: wavefront 0 takes r^T r, 1 to 3 p^T q, r^T q and
  // q^T q; |L r|^2, on iterations that test it, also wavefront 0
  const bool test = kFreshState ? k > 0 : c.mode == kNormal && k > 0;
  const bool check = kFreshState ? test : test && c.phase == 0;   // |L r|^2 of state k is there
  const int nrec = S.fused_nwg;
  double rec[kRecPerLane], rec1[kRecPerLane];
  {
    const double* __restrict__ a = kFreshState ? replaced_record(S, 0) : record(S, k, wv == 0 ? 0 : wv + 1);
    // (unconditional: see Slice)
    const double* __restrict__ b = kFreshState ? replaced_record(S, 1) : wv == 0 ? record(S, k, 1) : a;
#pragma unroll
    for (int u = 0; u < kRecPerLane; ++u) rec[u] = a[min(lane + u * kWave, nrec - 1)];
#pragma unroll
    for (int u = 0; u < kRecPerLane; ++u) rec1[u] = b[min(lane + u * kWave, nrec - 1)];
  }
  // this thread's own entry (threads 0..191: entry t of the slice)
  const int n3 = 3 * S.N, el = kRow3 * s + t;
  const bool own = t < kRow3 && el < n3;
  const unsigned eo = 4u * min(el, n3 - 1);
  const float r_o = at32<float>(rin, eo), p_o = at32<float>(pin, eo);
  const float q_o = kFreshState ? 0.f : at32<float>(qin, eo);
  const double x_o = kFreshState ? 0.0 : at32<double>(S.x, 2u * eo);
  const int row = s * kSlice + lane;
  float lf[6];   // for wavefront 3, where |L r|^2 of the output is wanted (unconditional: see Slice)
  if (!kFreshState)
#pragma unroll
    for (int m = 0; m < 6; ++m) lf[m] = at32<float>(S.Lf, 4u * (m * S.N4 + min(row, S.N - 1)));
  // a round's blocks and gathers, all in flight together
  float bu_[kRoundPairs][9], bl_[kRoundPairs][9];
  F3 ru[kRoundPairs], qu[kRoundPairs], pu[kRoundPairs], rl[kRoundPairs], ql[kRoundPairs], pl[kRoundPairs];
  auto load_round = [&](int k0) {
#pragma unroll
    for (int j = 0; j < kRoundPairs; ++j) {
      const int kk = k0 + wv + kSliceWaves * j;
      load_block32(static_cast<const BT*>(S.blk), sl.bu + max(min(kk, sl.wu - 1), 0) * kSlice + lane, bu_[j]);
      const unsigned o = 12u * sl.uc[j], ol = 12u * sl.lc[j];
      ru[j] = at32<F3>(rin, o);
      if (!kFreshState) qu[j] = at32<F3>(qin, o);
      pu[j] = at32<F3>(pin, o);
      load_block32(static_cast<const BT*>(S.blk), sl.ub[j], bl_[j]);
      rl[j] = at32<F3>(rin, ol);
      if (!kFreshState) ql[j] = at32<F3>(qin, ol);
      pl[j] = at32<F3>(pin, ol);
    }
  };
  load_round(0);
  if (sl.w > kRound) sl.load_indices(S, kRound + wv, lane);
  // the sums of state k, and what to do with it, while the loads are in flight
  {
    double v = 0.0;
#pragma unroll
    for (int u = 0; u < kRecPerLane; ++u) v += lane + u * kWave < nrec ? rec[u] : 0.0;
    v = wave_sum_all(v);
    if (lane == 0) sums[wv == 0 ? 0 : wv + 1] = v;
    if (wv == 0 && check) {
      v = 0.0;
#pragma unroll
      for (int u = 0; u < kRecPerLane; ++u) v += lane + u * kWave < nrec ? rec1[u] : 0.0;
      v = wave_sum_all(v);
      if (lane == 0) sums[1] = v;
    }
  }
  __syncthreads();
  const bool leader = s == 0 && t == kRow3;   // in the wavefront with the least to do
  const double rho = sums[0], rt = check ? sums[1] : 0.0;
  PcgCtl next = c;
  float alpha = 0.f, beta = 0.f;
  if (kFreshState) {
    // a residual just replaced counts for convergence now
    const bool converged = test && ((c.phase == 0 && rt <= c.tol_bb) || rho == 0.0);
    if (k == 0 && S.aflags && *S.aflags) next.done = kEndAssembly;
    else if (converged) next.done = kEndConverged;
    else if (test && k >= c.max_iter) next.done = kEndMaxIter;
    if (leader && test) {
      S.sc->rho = rho;
      S.sc->rr_true = rt;
    }
    if (next.done) {
      if (leader) hand_on(S, next, par);
      return;
    }
    if (k > 0) {
      beta = c.rho_prev > 0.0 ? (float)(rho / c.rho_prev) : 0.f;
      next.rt_ref = rt;
      next.verified = k;
    }
    next.mode = kTested;
  } else {
    const double pq = sums[2], rq = sums[3], qq = sums[4];
    const bool converged = test && ((check && rt <= c.tol_bb) || rho == 0.0);
    const bool replace = test && c.replace_on && rho != 0.0 &&
                         (converged ? c.verified != k : check && rt <= 1e-2 * c.rt_ref);
    const bool capped = test && k >= c.max_iter;
    const bool broken = !(pq > 0.0);
    if (leader && test) {
      S.sc->rho = rho;
      if (check) S.sc->rr_true = rt;
    }
    if (__builtin_expect(replace | converged | capped | broken, 0)) {
      if (replace) next.mode = kReplace;
      else next.done = converged ? kEndConverged : capped ? kEndMaxIter : kEndBreakdown;
      if (leader) hand_on(S, next, par);
      return;
    }
    alpha = (float)(rho / pq);
    const double ad = alpha;
    const double rho_next = rho - 2.0 * ad * rq + ad * ad * qq;
    beta = rho_next > 0.0 ? (float)(rho_next / rho) : 0.f;
    next.k = k + 1;
    next.phase = c.phase + 1 == c.every ? 0 : c.phase + 1;
    next.mode = kNormal;
    next.rho_prev = rho;
  }
  const bool norm = !kFreshState && next.phase == 0;   // |L r|^2 of the output state is wanted
  const float r_n = kFreshState ? r_o : __fmaf_rn(-alpha, q_o, r_o);
  const float s_n = __fmaf_rn(beta, p_o, r_n);
  if (norm && t < kRow3) rsh[t] = r_n;
  float acc = 0.f;
  for (int k0 = 0, h = 0;; k0 += kRound, h ^= 1) {
#pragma unroll
    for (int j = 0; j < kRoundPairs; ++j) {
      float p[3];
#pragma unroll
      for (int m = 0; m < 3; ++m)
        p[m] = __fmaf_rn(beta, pu[j].v[m], kFreshState ? ru[j].v[m] : __fmaf_rn(-alpha, qu[j].v[m], ru[j].v[m]));
      float* o = &prod[h][wv + kSliceWaves * j][0][3 * lane];
#pragma unroll
      for (int m = 0; m < 3; ++m)
        o[m] = __fmaf_rn(bu_[j][3 * m + 2], p[2], __fmaf_rn(bu_[j][3 * m], p[0], __fmul_rn(bu_[j][3 * m + 1], p[1])));
#pragma unroll
      for (int m = 0; m < 3; ++m)
        p[m] = __fmaf_rn(beta, pl[j].v[m], kFreshState ? rl[j].v[m] : __fmaf_rn(-alpha, ql[j].v[m], rl[j].v[m]));
      o = &prod[h][wv + kSliceWaves * j][1][3 * lane];
#pragma unroll
      for (int m = 0; m < 3; ++m)
        o[m] = __fmaf_rn(bl_[j][6 + m], p[2], __fmaf_rn(bl_[j][m], p[0], __fmul_rn(bl_[j][3 + m], p[1])));
    }
    const bool more = k0 + kRound < sl.w;
    if (more) {   // the next round's loads pass behind the barrier and the sums
      load_round(k0 + kRound);
      if (k0 + 2 * kRound < sl.w) sl.load_indices(S, k0 + 2 * kRound + wv, lane);
    }
    __syncthreads();
    if (t < kRow3) {
      float y[kRound], z[kRound];
#pragma unroll
      for (int m = 0; m < kRound; ++m) {
        y[m] = prod[h][m][0][t];
        z[m] = prod[h][m][1][t];
      }
#pragma unroll
      for (int m = 0; m < kRound; ++m) {
        acc = k0 + m < sl.wu ? __fadd_rn(acc, y[m]) : acc;
        acc = k0 + m < sl.wl ? __fadd_rn(acc, z[m]) : acc;
      }
    }
    if (!more) break;
  }
  if (wv < 3) {
    const float q_n = __fadd_rn(s_n, acc);
    if (own) {
      put32(S.q + (ko & 1) * S.pstride, eo, q_n);
      put32(S.P + (ko & 1) * S.pstride, eo, s_n);
      if (!kFreshState) {
        put32(S.r + (ko & 1) * S.pstride, eo, r_n);
        put32(S.x, 2u * eo, fma((double)alpha, (double)p_o, x_o));
      }
    }
    const double rd = own ? (double)r_n : 0.0, sd = own ? (double)s_n : 0.0, qd = own ? (double)q_n : 0.0;
    const double o0 = wave_sum_all(rd * rd), o2 = wave_sum_all(sd * qd), o3 = wave_sum_all(rd * qd),
                 o4 = wave_sum_all(qd * qd);
    if (lane == 0) {
      tail[wv][0] = o0;
      tail[wv][2] = o2;
      tail[wv][3] = o3;
      tail[wv][4] = o4;
    }
  } else if (norm) {
    const float r0 = rsh[3 * lane], r1 = rsh[3 * lane + 1], r2 = rsh[3 * lane + 2];
    const double t0 = (double)lf[0] * r0;
    const double t1 = (double)lf[1] * r0 + (double)lf[2] * r1;
    const double t2 = (double)lf[3] * r0 + (double)lf[4] * r1 + (double)lf[5] * r2;
    const double o1 = wave_sum_all(row < S.N ? t0 * t0 + t1 * t1 + t2 * t2 : 0.0);
    if (lane == 0) tail[0][1] = o1;
  }
  __syncthreads();
  if (t < 5) record(S, ko, t)[s] = t == 1 ? (norm ? tail[0][1] : 0.0) : tail[0][t] + tail[1][t] + tail[2][t];
  if (leader) hand_on(S, next, par);
}

template <class BT>
__device__ __forceinline__ void fused_launch(const PcgSystem& S, int s, int par) {
  // everything that does not depend on the state is asked for beside it
  const PcgCtl c = uniform_load(&S.sc->ctl[par]);
  Slice<BT> sl;
  sl.bu = uniform_load(S.sbu + s);
  sl.bl = uniform_load(S.sbl + s);
  sl.wu = (uniform_load(S.sbu + s + 1) - sl.bu) / kSlice;
  sl.wl = (uniform_load(S.sbl + s + 1) - sl.bl) / kSlice;
  sl.w = max(sl.wu, sl.wl);
  sl.load_indices(S, __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), threadIdx.x % kWave);
  if (__builtin_expect((c.done != 0) | (c.mode > kTested), 0)) {
    if (c.done) {   // ended: hand the state on
      if (s == 0 && threadIdx.x == 0) {
        PcgCtl next = c;
        ++next.launches;
        S.sc->ctl[par ^ 1] = next;
        report(S, next.launches, c.done, c.k);
      }
    } else if (c.mode == kFresh) {
      iterate<BT, true>(S, c, sl, s, par);
    } else {
      if constexpr (std::is_same<BT, float>::value) replace_residual(S, c, s, par);   // BF16 solves run without it
    }
    // The compiler lays this branch out before the usual path and joins the
    // two: loads it left in flight here would be waited for there.
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_endpgm();
  }
  iterate<BT, false>(S, c, sl, s, par);
}

template <class BT>
__global__ void __launch_bounds__(kFusedBlock, 2) k_fused(PcgSystem S, int par) {
  fused_launch<BT>(S, xcd_block(blockIdx.x, S.fused_nwg), par);
}

template <class BT>
__global__ void __launch_bounds__(kFusedBlock, 2)
k_fused_batched(const PcgSystem* __restrict__ sys, const int* __restrict__ wg_sys, int par) {
  const int b = xcd_block(blockIdx.x, gridDim.x);
  const PcgSystem S = uniform_load(sys + uniform_load(wg_sys + b));
  fused_launch<BT>(S, b - S.fused_wg0, par);
}

// The resident kernel: the same iteration, with all workgroups of the system
// running at once and going from state to state without a launch between.
//
// What a launch costs per iteration (2.9 us outside its code, the loads that
// wait for loads, the blocks and indices read again) is paid once.  A slice has
// kResWaves wavefronts; its blocks and indices of the first kResWaves kP slots,
// its own entries of r, p and x and its copies of the r and p entries it
// gathers stay in registers (a copy goes through the FMAs its owner applies),
// so only q and the five sums cross between workgroups.
//
// Five more workgroups, the collectors, add one sum each.  A workgroup's sum is
// stored as 16 bytes, its two halves each beside the iteration it belongs to,
// after the workgroup's vector entries have been acknowledged; the collector
// reads them until all show that iteration, adds them in the order of the
// launches and stores the total the same way, which a wavefront of every
// workgroup reads until it has all five.  Data and signal arrive in one trip.
// (All workgroups reading all sums needs one trip less, but the reads queue:
// 27,000 cycles of a 31,000 cycle iteration at 384 slices; with one collector
// for all five 7,000 of 14,000.)  What crosses is stored and loaded with sc1
// (past the first-level cache, and from one die's L2 to another's).  Two
// buffers suffice: a workgroup writes state k + 2 after it has read the totals
// of k + 1, to which each workgroup contributes after its last read of state k.
//
// The kernel needs all its workgroups running.  A grid that the chip takes at
// once (pcg_resident) does run unless other kernels hold compute units, for
// instance two such grids that each got part of the chip, so the workgroups
// first count themselves: if they are not complete within kStartTicks, one
// marks the count, all leave without a step, and the solve goes on by
// launches.  Ordinary kernels of other streams are waited out (a copy of 256 MB
// takes 85 us; with 50 us instead of 100 a solve of 507 slices beside such
// copies went on by launches, 190 a second against 275), another resident grid
// is not worth waiting for: with 1 ms, solves of 416 slices and 41 iterations
// took 1.39 ms each on two threads and 1.26 on four, with 100 us 0.67 and 0.70
// (the two-kernel iteration 1.18 and 0.73; of 507 slices and 624 iterations, on
// four threads, 3.80 and 3.11 against 3.57).  Once complete, every later wait
// ends, as each workgroup waits only for running ones; kMaxPolls bounds it all
// the same.
//
// Measured (us per iteration, launches against this kernel): 250 nodes 6.1 ->
// 2.5, 2,880 nodes 6.8 -> 3.0, 24,565 nodes (slices of up to 18 slots) 9.0 ->
// 4.5.  An iteration of 7,200 cycles at 2,880 nodes is 3,500 from the last sum
// to the totals (two trips of about 1,000 and the addition), 800 for alpha and
// beta, behind which q is gathered, 1,500 for the products and their sum and
// 1,050 for the new entries and their acknowledgement; a 17th slot costs 2,000
// more.  Eight wavefronts of up to two held pairs use 125 registers: three
// pairs spill, as do the loads of two unheld slots at once, and a spill costs
// 3,000 cycles.
constexpr int kCollectors = 5;              // workgroups, one per sum
constexpr int kResWaves = 8;                // wavefronts per slice
constexpr int kResBlock = kResWaves * kWave;
constexpr long long kStartTicks = 10000;    // 100 us of the 100 MHz clock
constexpr int kMaxPolls = 1 << 21;          // over a second
constexpr int kSc1 = 16;                    // cache policy of the buffer accesses: sc1
static_assert(5 * 16 <= kTotalBytes, "a line holds the totals");

typedef int V3 __attribute__((ext_vector_type(3)));
typedef int V4 __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t Buffer;

__device__ __forceinline__ Buffer buffer_of(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00027000);
}
__device__ __forceinline__ Buffer exchange_of(const PcgSystem& S) {
  return buffer_of(S.part + kPartsPerSystem, 8 * kTaggedParts);
}

__device__ __forceinline__ F3 gather3(Buffer b, unsigned byte, unsigned base) {
  const V3 v = __builtin_amdgcn_raw_buffer_load_b96(b, (int)byte, (int)base, kSc1);
  F3 f;
  f.v[0] = __int_as_float(v.x);
  f.v[1] = __int_as_float(v.y);
  f.v[2] = __int_as_float(v.z);
  return f;
}

// Byte offsets of sum m of state k from workgroup 0, and of a copy of the line of its totals.
__device__ __forceinline__ int sum_at(int k, int m) { return 16 * (((k & 1) * 5 + m) * kFusedMaxSlices); }
__device__ __forceinline__ int totals_at(int k, int copy) {
  return 16 * 2 * 5 * kFusedMaxSlices + kTotalBytes * ((k & 1) * kTotalCopies + copy);
}

__device__ __forceinline__ void put_tagged(Buffer b, int byte, double v, int k) {
  const V4 w = {__double2loint(v), k, __double2hiint(v), k};
  __builtin_amdgcn_raw_buffer_store_b128(w, b, byte, 0, kSc1);
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Lane m < 5: total m of state k; false: it did not come.
__device__ __forceinline__ bool read_totals(Buffer b, int k, int copy, int lane, double& v) {
  V4 w;
  for (int i = 0;; ++i) {
    w = __builtin_amdgcn_raw_buffer_load_b128(b, totals_at(k, copy) + 16 * min(lane, 4), 0, kSc1);
    asm volatile("" ::: "memory");
    if (__all((w.y == k) & (w.w == k))) break;
    if (i == kMaxPolls) return false;
  }
  v = __hiloint2double(w.z, w.x);
  return true;
}

// (nobody waits for it: the launch's statistics)
__device__ __forceinline__ void count(int* n, int by) {
  (void)__hip_atomic_fetch_add(n, by, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A workgroup stops without having handed on a state: the host is told, and
// the launches queued behind find both copies of the state ended.
__device__ __forceinline__ void give_up(const PcgSystem& S) {
  if (S.hstat) __hip_atomic_store(&S.hstat[kWordStuck], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __threadfence_system();
  S.sc->ctl[0].done = S.sc->ctl[1].done = kEndStuck;
}

// What follows from the totals of state c.k: the step's alpha and beta and the
// next state, or false and in c how the solve or this stretch of it ended.
__device__ __forceinline__ bool advance(const PcgSystem& S, PcgCtl& c, double v, bool leader, float& alpha,
                                        float& beta) {
  const bool test = c.mode == kNormal && c.k > 0, check = test && c.phase == 0;
  const double rho = lane_value(v, 0), rt = check ? lane_value(v, 1) : 0.0;
  const double pq = lane_value(v, 2), rq = lane_value(v, 3), qq = lane_value(v, 4);
  const bool converged = test && ((check && rt <= c.tol_bb) || rho == 0.0);
  const bool replace = test && c.replace_on && rho != 0.0 &&
                       (converged ? c.verified != c.k : check && rt <= 1e-2 * c.rt_ref);
  const bool capped = test && c.k >= c.max_iter;
  const bool broken = !(pq > 0.0);
  if (leader && test) {
    S.sc->rho = rho;
    if (check) S.sc->rr_true = rt;
  }
  if (__builtin_expect(replace | converged | capped | broken, 0)) {
    if (replace) c.mode = kReplace;
    else c.done = converged ? kEndConverged : capped ? kEndMaxIter : kEndBreakdown;
    return false;
  }
  alpha = (float)(rho / pq);
  const double ad = alpha;
  const double rho_next = rho - 2.0 * ad * rq + ad * ad * qq;
  beta = rho_next > 0.0 ? (float)(rho_next / rho) : 0.f;
  ++c.k;
  c.phase = c.phase + 1 == c.every ? 0 : c.phase + 1;
  c.mode = kNormal;
  c.rho_prev = rho;
  return true;
}

// All workgroups of the launch have started (or none of them goes on).
__device__ __forceinline__ bool all_started(const PcgSystem& S, int par) {
  __shared__ int go;
  if (threadIdx.x == 0) {
    unsigned* w = start_word(S, par);
    const unsigned n = S.fused_nwg + kCollectors;
    unsigned v = __hip_atomic_fetch_add(w, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
    const long long t0 = wall_clock64();
    while (v < n) {   // (the mark makes it larger)
      if (wall_clock64() - t0 > kStartTicks &&
          __hip_atomic_compare_exchange_strong(w, &v, v | kApart, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT))
        v |= kApart;
      else
        v = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    go = v == n;
  }
  __syncthreads();
  return go != 0;
}

// The collector of sum m.
__device__ __forceinline__ void collect(const PcgSystem& S, PcgCtl c, int m, int par, int steps) {
  const int t = threadIdx.x, lane = t % kWave;
  const Buffer b = exchange_of(S);
  const int nrec = S.fused_nwg, k0 = c.k;
  if (t < 2 * kTotalCopies) put_tagged(b, totals_at(t & 1, t / 2) + 16 * m, 0.0, -1);
  __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
  __syncthreads();
  if (!all_started(S, par) || t >= kWave) return;
  for (int it = 0; it < steps; ++it) {
    const int k = c.k;
    double v = 0.0;
    if (it == 0) {
      const double* __restrict__ a = record(S, k, m);
      for (int u = 0; u < nrec; u += kWave) v += lane + u < nrec ? a[min(lane + u, nrec - 1)] : 0.0;
    } else {
      // (only the chunks that were not complete are read again)
      V4 w[kRecPerLane];
      unsigned open = (1u << div_up(nrec, kWave)) - 1;
      for (int n = 0; open; ++n) {
#pragma unroll
        for (int u = 0; u < kRecPerLane; ++u)
          if (open >> u & 1)
            w[u] = __builtin_amdgcn_raw_buffer_load_b128(b, 16 * min(lane + u * kWave, nrec - 1), sum_at(k, m), kSc1);
        asm volatile("" ::: "memory");
#pragma unroll
        for (int u = 0; u < kRecPerLane; ++u)
          if ((open >> u & 1) && __all((w[u].y == k) & (w[u].w == k))) open &= ~(1u << u);
        if (n == kMaxPolls) return;
      }
#pragma unroll
      for (int u = 0; u < kRecPerLane; ++u)
        if (u * kWave < nrec) v += lane + u * kWave < nrec ? __hiloint2double(w[u].z, w[u].x) : 0.0;
    }
    v = wave_sum_all(v);
    if (lane < kTotalCopies) put_tagged(b, totals_at(k, lane) + 16 * m, v, k);
    float alpha, beta;
    if (!read_totals(b, k, 0, lane, v) || !advance(S, c, v, false, alpha, beta)) return;
  }
}

struct Wide {   // a pair of slots that is not held: the blocks, and where to gather
  unsigned slot[2], at[2];
};
__device__ __forceinline__ Wide wide_slot(const PcgSystem& S, int bu, int bl, int wu, int wl, int kk, int lane) {
  Wide e;
  e.slot[0] = bu + max(min(kk, wu - 1), 0) * kSlice + lane;
  const int2 q = at32<int2>(S.sent + bl, 8u * (unsigned)(max(min(kk, wl - 1), 0) * kSlice + lane));
  e.slot[1] = q.x;
  e.at[0] = 12u * (unsigned)S.scol[e.slot[0]];
  e.at[1] = 12u * (unsigned)q.y;
  return e;
}

constexpr int kMaxP = 2;
typedef float Product[2][kRow3];
struct ResShared {
  Product prod[kResWaves * (kMaxP + 1)];
  float r[kRow3], lf[6][kSlice];
  Wide wide[kResBlock];
  double tail[4][5], total[5];
  int stuck;
};

// A slice.  kP: slot pairs per wavefront that stay in registers.
template <class BT, int kP>
__device__ __forceinline__ void resident(const PcgSystem& S, PcgCtl c, int s, int par, int steps, int bu, int bl,
                                         int wu, int wl, ResShared& sh) {
  constexpr int kHeld = kResWaves * kP;
  Product* const prod = sh.prod;
  Product* const prod2 = sh.prod + kHeld;
  const int t = threadIdx.x, lane = t % kWave, wv = __builtin_amdgcn_readfirstlane(t / kWave);
  const int w = max(wu, wl), copy = s % kTotalCopies;
  const unsigned stride = 4u * (unsigned)S.pstride;
  const Buffer rb = buffer_of(S.r, 2 * stride), qb = buffer_of(S.q, 2 * stride), pb = buffer_of(S.P, 2 * stride),
               tb = exchange_of(S);
  if (t == 0) sh.stuck = 0;
  if (t < 6 * kSlice) sh.lf[t / kSlice][t % kSlice] = at32<float>(S.Lf, 4u * (t / kSlice * S.N4 + min(s * kSlice + t % kSlice, S.N - 1)));
  // slots past a width are not written: a sum that starts at +0 is the same with their +0
  for (int e = t; e < kHeld * 2 * kRow3; e += kResBlock) (&prod[0][0][0])[e] = 0.f;
  if (t < 10) put_tagged(tb, sum_at(t / 5, t % 5) + 16 * s, 0.0, -1);   // no sum of this launch is there yet
  const int el = kRow3 * s + t, n3 = 3 * S.N;
  const bool own = t < kRow3 && el < n3;
  const unsigned eo = 4u * min(el, n3 - 1), cur0 = (c.k & 1) * stride;
  float r_o = at32<float>(S.r, eo + cur0), p_o = at32<float>(S.P, eo + cur0), q_o = at32<float>(S.q, eo + cur0);
  double x_o = at32<double>(S.x, 2u * eo);
  // the held slots
  float hu[kP][9], hl[kP][9];
  unsigned ou[kP], ol[kP];
  F3 ru[kP], pu[kP], rl[kP], pl[kP];
#pragma unroll
  for (int j = 0; j < kP; ++j) {
    const int kk = wv + kResWaves * j;
    const int eu = bu + max(min(kk, wu - 1), 0) * kSlice + lane;
    const int2 e = at32<int2>(S.sent + bl, 8u * (unsigned)(max(min(kk, wl - 1), 0) * kSlice + lane));
    ou[j] = 12u * (unsigned)S.scol[eu];
    ol[j] = 12u * (unsigned)e.y;
    load_block32(static_cast<const BT*>(S.blk), eu, hu[j]);
    load_block32(static_cast<const BT*>(S.blk), e.x, hl[j]);
    ru[j] = at32<F3>(S.r, ou[j] + cur0);
    pu[j] = at32<F3>(S.P, ou[j] + cur0);
    rl[j] = at32<F3>(S.r, ol[j] + cur0);
    pl[j] = at32<F3>(S.P, ol[j] + cur0);
  }
  sh.wide[t] = wide_slot(S, bu, bl, wu, wl, kHeld + wv, lane);
  __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): the tags are cleared
  const bool leader = s == 0 && t == kRow3;
  __syncthreads();
  if (!all_started(S, par)) {
    if (leader) {
      c.apart = 1;
      count(&S.sc->res_apart, 1);
      if (S.hstat) __hip_atomic_store(&S.hstat[kWordApart], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      hand_on(S, c, par);
    }
    return;
  }
  double mine = 0.0;   // threads 0 to 4: the workgroup's sums of the state
  int it = 0;
  for (; it < steps; ++it) {
    const unsigned cur = (c.k & 1) * stride;
    if (wv == kResWaves - 1) {   // (not one of those with the most to do)
      double v = 0.0;
      if (__builtin_expect(!read_totals(tb, c.k, copy, lane, v), 0)) sh.stuck = 1;
      if (lane < 5) sh.total[lane] = v;
    }
    __syncthreads();
    if (__builtin_expect(sh.stuck, 0)) {
      if (t == 0) give_up(S);
      return;
    }
    F3 qu[kP], ql[kP];
#pragma unroll
    for (int j = 0; j < kP; ++j) {
      qu[j] = gather3(qb, ou[j], cur);
      ql[j] = gather3(qb, ol[j], cur);
    }
    float alpha, beta;
    if (!advance(S, c, sh.total[min(lane, 4)], leader, alpha, beta)) break;
    const bool norm = c.phase == 0;
    const float r_n = __fmaf_rn(-alpha, q_o, r_o);
    const float s_n = __fmaf_rn(beta, p_o, r_n);
    if (norm && t < kRow3) sh.r[t] = r_n;
#pragma unroll
    for (int j = 0; j < kP; ++j) {
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        ru[j].v[m] = __fmaf_rn(-alpha, qu[j].v[m], ru[j].v[m]);
        pu[j].v[m] = __fmaf_rn(beta, pu[j].v[m], ru[j].v[m]);
        rl[j].v[m] = __fmaf_rn(-alpha, ql[j].v[m], rl[j].v[m]);
        pl[j].v[m] = __fmaf_rn(beta, pl[j].v[m], rl[j].v[m]);
      }
      if (wv + kResWaves * j < wu) {
        float* o = &prod[wv + kResWaves * j][0][3 * lane];
#pragma unroll
        for (int m = 0; m < 3; ++m)
          o[m] = __fmaf_rn(hu[j][3 * m + 2], pu[j].v[2],
                           __fmaf_rn(hu[j][3 * m], pu[j].v[0], __fmul_rn(hu[j][3 * m + 1], pu[j].v[1])));
      }
      if (wv + kResWaves * j < wl) {
        float* o = &prod[wv + kResWaves * j][1][3 * lane];
#pragma unroll
        for (int m = 0; m < 3; ++m)
          o[m] = __fmaf_rn(hl[j][6 + m], pl[j].v[2],
                           __fmaf_rn(hl[j][m], pl[j].v[0], __fmul_rn(hl[j][3 + m], pl[j].v[1])));
      }
    }
    // A load whose result a skipped slot does not use would be waited for where
    // its register is written next: behind the stores below, with their acknowledgement.
    __builtin_amdgcn_s_waitcnt(0x0f70);
    __syncthreads();
    float acc = 0.f;
    if (t < kRow3) {
#pragma unroll
      for (int j = 0; j < kP; ++j) {
        float y[kResWaves], z[kResWaves];
#pragma unroll
        for (int m = 0; m < kResWaves; ++m) {
          y[m] = prod[kResWaves * j + m][0][t];
          z[m] = prod[kResWaves * j + m][1][t];
        }
#pragma unroll
        for (int m = 0; m < kResWaves; ++m) {
          acc = __fadd_rn(acc, y[m]);
          acc = __fadd_rn(acc, z[m]);
        }
      }
    }
    // wider slices: the other slots, read again in every iteration
    for (int k0 = kHeld; k0 < w; k0 += kResWaves) {
      const int kk = k0 + wv;
      const Wide e = k0 == kHeld ? sh.wide[t] : wide_slot(S, bu, bl, wu, wl, kk, lane);
// (one after the other: the loads of both do not fit the registers)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float* o = &prod2[wv][h][3 * lane];
        if (kk < (h == 0 ? wu : wl)) {
          float b[9], p[3];
          load_block32(static_cast<const BT*>(S.blk), e.slot[h], b);
          const F3 r1 = gather3(rb, e.at[h], cur), q1 = gather3(qb, e.at[h], cur), p1 = gather3(pb, e.at[h], cur);
#pragma unroll
          for (int m = 0; m < 3; ++m) p[m] = __fmaf_rn(beta, p1.v[m], __fmaf_rn(-alpha, q1.v[m], r1.v[m]));
#pragma unroll
          for (int m = 0; m < 3; ++m)
            o[m] = h == 0 ? __fmaf_rn(b[3 * m + 2], p[2], __fmaf_rn(b[3 * m], p[0], __fmul_rn(b[3 * m + 1], p[1])))
                          : __fmaf_rn(b[6 + m], p[2], __fmaf_rn(b[m], p[0], __fmul_rn(b[3 + m], p[1])));
        } else {
          o[0] = o[1] = o[2] = 0.f;
        }
      }
      __builtin_amdgcn_s_waitcnt(0x0f70);
      __syncthreads();
      if (t < kRow3) {
#pragma unroll
        for (int m = 0; m < kResWaves; ++m) {
          acc = __fadd_rn(acc, prod2[m][0][t]);
          acc = __fadd_rn(acc, prod2[m][1][t]);
        }
      }
      __syncthreads();
    }
    if (wv < 3) {
      const float q_n = __fadd_rn(s_n, acc);
      if (own) {
        const int nxt = (int)((c.k & 1) * stride);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(q_n), qb, (int)eo, nxt, kSc1);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(r_n), rb, (int)eo, nxt, kSc1);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(s_n), pb, (int)eo, nxt, kSc1);
      }
      x_o = fma((double)alpha, (double)p_o, x_o);
      r_o = r_n;
      p_o = s_n;
      q_o = q_n;
      const double rd = own ? (double)r_n : 0.0, sd = own ? (double)s_n : 0.0, qd = own ? (double)q_n : 0.0;
      const double o0 = wave_sum_all(rd * rd), o2 = wave_sum_all(sd * qd), o3 = wave_sum_all(rd * qd),
                   o4 = wave_sum_all(qd * qd);
      if (lane == 0) {
        sh.tail[wv][0] = o0;
        sh.tail[wv][2] = o2;
        sh.tail[wv][3] = o3;
        sh.tail[wv][4] = o4;
      }
    } else if (wv == 3 && norm) {
      const float r0 = sh.r[3 * lane], r1 = sh.r[3 * lane + 1], r2 = sh.r[3 * lane + 2];
      float lf[6];
#pragma unroll
      for (int m = 0; m < 6; ++m) lf[m] = sh.lf[m][lane];
      const double t0 = (double)lf[0] * r0;
      const double t1 = (double)lf[1] * r0 + (double)lf[2] * r1;
      const double t2 = (double)lf[3] * r0 + (double)lf[4] * r1 + (double)lf[5] * r2;
      const double o1 = wave_sum_all(s * kSlice + lane < S.N ? t0 * t0 + t1 * t1 + t2 * t2 : 0.0);
      if (lane == 0) sh.tail[0][1] = o1;
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this wavefront's entries have arrived
    __syncthreads();
    if (t < 5) {
      mine = t == 1 ? (norm ? sh.tail[0][1] : 0.0) : sh.tail[0][t] + sh.tail[1][t] + sh.tail[2][t];
      put_tagged(tb, sum_at(c.k, t) + 16 * s, mine, c.k);
    }
  }
  if (it > 0) {   // (all have read the sums that the launch began with)
    if (own) put32(S.x, 2u * eo, x_o);
    if (t < 5) record(S, c.k, t)[s] = mine;
    if (leader) {
      count(&S.sc->res_iters, it);
      count(&S.sc->res_launches, 1);
    }
  }
  if (leader) hand_on(S, c, par);
}

template <class BT>
__device__ __forceinline__ void resident_launch(const PcgSystem& S, int s, int par, int steps) {
  const PcgCtl c = uniform_load(&S.sc->ctl[par]);
  if ((c.done != 0) | (c.mode > kTested) | c.apart) {   // nothing for this kernel to do
    if (s == 0 && threadIdx.x == 0) hand_on(S, c, par);
    return;
  }
  if (s >= S.fused_nwg) {
    collect(S, c, s - S.fused_nwg, par, steps);
    return;
  }
  const int bu = uniform_load(S.sbu + s), bl = uniform_load(S.sbl + s);
  const int wu = (uniform_load(S.sbu + s + 1) - bu) / kSlice, wl = (uniform_load(S.sbl + s + 1) - bl) / kSlice;
  const int w = max(wu, wl);
  __shared__ ResShared sh;
  if (w <= kResWaves)
    resident<BT, 1>(S, c, s, par, steps, bu, bl, wu, wl, sh);
  else
    resident<BT, kMaxP>(S, c, s, par, steps, bu, bl, wu, wl, sh);
}

template <class BT>
__global__ void __launch_bounds__(kResBlock) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_resident(PcgSystem S, int par, int steps) {
  resident_launch<BT>(S, blockIdx.x, par, steps);
}

}  // namespace

int pcg_fused_groups(int N) {
  const int nslices = div_up(N, kSlice);
  return nslices <= kFusedMaxSlices ? nslices : 0;
}

hipError_t launch_pcg_fused(const PcgSystem& S, bool bf16, int par, hipStream_t s, hipEvent_t t0, hipEvent_t t1) {
  const void* f =
      bf16 ? reinterpret_cast<const void*>(k_fused<uint32_t>) : reinterpret_cast<const void*>(k_fused<float>);
  PcgSystem Sx = S;
  void* args[] = {&Sx, &par};
  const dim3 grid(S.fused_nwg), block(kFusedBlock);
  return t0 && t1 ? hipExtLaunchKernel(f, grid, block, args, 0, s, t0, t1, 0)
                  : hipLaunchKernel(f, grid, block, args, 0, s);
}

// What the device takes at once, as the runtime works it out from the kernels'
// registers and LDS (two to a compute unit: 128 registers a thread, 47 KB); a
// grid beyond that would never run at once.  Systems that fit gain at every
// size (see above), so there is no other bound.
int pcg_resident_room(int num_cu) {
  int a = 0, b = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&a, reinterpret_cast<const void*>(k_resident<float>), kResBlock,
                                                   0) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, reinterpret_cast<const void*>(k_resident<uint32_t>), kResBlock,
                                                   0) != hipSuccess)
    return 0;   // (not known: by launches)
  return num_cu * (a < b ? a : b);
}

bool pcg_resident(const PcgSystem& S, int room) { return S.fused_nwg > 0 && S.fused_nwg + kCollectors <= room; }

hipError_t launch_pcg_resident(const PcgSystem& S, bool bf16, int par, int steps, hipStream_t s) {
  const void* f =
      bf16 ? reinterpret_cast<const void*>(k_resident<uint32_t>) : reinterpret_cast<const void*>(k_resident<float>);
  PcgSystem Sx = S;
  void* args[] = {&Sx, &par, &steps};
  return hipLaunchKernel(f, dim3(S.fused_nwg + kCollectors), dim3(kResBlock), args, 0, s);
}

hipError_t launch_pcg_fused_batched(const PcgSystem* sys, const int* wg_sys, int nwg, int par, hipStream_t s) {
  void* args[] = {&sys, &wg_sys, &par};
  return hipLaunchKernel(reinterpret_cast<const void*>(k_fused_batched<float>), dim3(nwg), dim3(kFusedBlock), args, 0,
                         s);
}

}  // namespace bfal

// HIP kernels (gfx950) of the search cascade's stages after MSV (hmm_msv.hip)
// and the cascade's launcher.
//
// One wavefront scores one target.  The model dimension (profile cells) is
// spread across the 64 lanes; database rows (residues) are processed in
// order.  Every wave-uniform quantity (target index, length, residue, the
// special states N/B/E/J/C) lives in scalar registers; branches on it are
// uniform.
//
//  Viterbi  packed saturating int16, two cells per VGPR; delete chain by
//           lazy propagation across slots; values past int16 re-based.
//  Rescore  the Viterbi recurrence in int32 with a -2^30 floor.
//  Forward  fp32 probabilities with exact power-of-two rescaling; the
//           delete chain crosses slots through a DPP prefix scan of affine
//           maps, E through a DPP sum.
//
// Cell layout (see hmm_host.cpp): packed kernels use slot 2*lane+half and
// cell slot*Q + q; 32-bit kernels use slot = lane and cell lane*Q + q.  The
// left neighbour of vector q is vector q-1 of the same slot, except q = 0,
// which takes vector Q-1 of the previous slot: one cross-lane shift per
// state per row.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "hmm_device.h"
#include "hmm_internal.h"

namespace hmmgpu {
namespace {


// ============================================================================ composition bias
//
// Composition-bias score of one target (nats; result in every lane): the
// forward probability ratio of a two-state null model (background, or the
// profile's mean match composition with odds r(a) = P.bias_r[a]; start
// 63/64 : 1/64, switch 1/64 per residue) against the background,
//   beta = ln (pi G_0 G_1 ... G_{L-1} 1),  G_0 = diag(1, r(x_0)),
//   G_i = [[63/64, r(x_i)/64], [1/64, 63/64 r(x_i)]].
// Each lane multiplies the 2x2 matrices of one contiguous segment of the
// target, then the segments are multiplied in order by a tree over the
// lanes; products are kept in [2^-20, 2^20] by exact power-of-two scaling
// with the exponents summed.
constexpr float kS8f = (float)(3.0 / M_LN2);

struct Mat2 {
  float a, b, c, d;   // [[a, b], [c, d]]
  int e;              // the product is this matrix times 2^e
};

__device__ __forceinline__ void mat2_mul(Mat2 &p, float ga, float gb, float gc, float gd, int ge) {
  const float a = fmaf(p.a, ga, p.b * gc), b = fmaf(p.a, gb, p.b * gd);
  const float c = fmaf(p.c, ga, p.d * gc), d = fmaf(p.c, gb, p.d * gd);
  p.a = a;
  p.b = b;
  p.c = c;
  p.d = d;
  p.e += ge;
  const float mx = fmaxf(fmaxf(a, b), fmaxf(c, d));
  if (mx > 0x1p20f || mx < 0x1p-20f) {
    int ex;
    (void)frexpf(mx, &ex);
    if (mx == 0.0f) ex = 0;
    const float s = ldexpf(1.0f, -ex);
    p.a *= s;
    p.b *= s;
    p.c *= s;
    p.d *= s;
    p.e += ex;
  }
}

__device__ float bias_score(const DevProfile &P, const uint8_t *x, int L, int lane) {
  constexpr float w = 1.0f / 64.0f, st = 63.0f / 64.0f;
  const int seg = (L + kWave - 1) / kWave;
  const int i0 = lane * seg, i1 = min(L, i0 + seg);
  Mat2 m{1.0f, 0.0f, 0.0f, 1.0f, 0};
  for (int i = i0; i < i1; i++) {   // lane-divergent, no cross-lane operation inside
    const float r = P.bias_r[x[i]];
    if (i == 0)
      mat2_mul(m, 1.0f, 0.0f, 0.0f, r, 0);
    else
      mat2_mul(m, st, w * r, w, st * r, 0);
  }
  for (int dd = 1; dd < kWave; dd <<= 1) {
    const float qa = __shfl_down(m.a, dd), qb = __shfl_down(m.b, dd), qc = __shfl_down(m.c, dd);
    const float qd = __shfl_down(m.d, dd);
    const int qe = __shfl_down(m.e, dd);
    if ((lane & (2 * dd - 1)) == 0 && lane + dd < kWave) mat2_mul(m, qa, qb, qc, qd, qe);
  }
  const float s0 = fmaf(st, m.a, w * m.c), s1 = fmaf(st, m.b, w * m.d);
  const float beta = logf(s0 + s1) + (float)m.e * (float)M_LN2;
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, beta), 0));
}

// Composition-bias filter on the MSV passes (list_ovf, count CNT_OVF): the
// bias score of each, and the ones whose MSV score less the bias still
// reaches the cutoff (or that overflowed MSV) go on to Viterbi's list.
__global__ void __launch_bounds__(256) bias_kernel(DevProfile P, DevDb db, DevOut out) {
  const int lane = threadIdx.x & 63;
  const int count = uni(__atomic_load_n(&db.counters[CNT_OVF], __ATOMIC_RELAXED));
  const WorkQueue<> queue(db, WORK_BIAS, count);
  for (int idx = queue.first(); idx < count;) {
    const int t = uni(db.list_ovf[idx]);
    const int L = uni(db.len[t]);
    const LenParams lp = db.lp[L];
    const float beta = bias_score(P, db.res + db.start[t], L, lane);
    uint8_t fl = (uint8_t)uni(db.flags_sorted[t]);
    const int raw = (int)uni((int)db.msv_sorted[t]);
    const bool go = (fl & HMM_MSV_OVF) || (float)raw - kS8f * fmaxf(beta, 0.0f) >= (float)lp.thr8;
    if (go) fl |= HMM_BIAS_PASS;
    db.flags_sorted[t] = fl;
    if (out.bias) out.bias[uni(db.perm[t])] = beta;
    if (go) db.list_vit[wave_fetch_add(&db.counters[CNT_VIT], 1)] = t;
    idx = queue.next();
  }
}

// The overflow list starts empty for Viterbi.
__global__ void reset_ovf(int32_t *c) {
  if (threadIdx.x == 0) c[CNT_OVF] = 0;
}

// ============================================================================ Viterbi int16
//
// Per row, with previous-row M, I, D and xB, every add saturating on its own:
//   M_k = sat(max(sat(xB+ENTRY16), sat(M_{k-1}+MM), sat(I_{k-1}+IM), sat(D_{k-1}+DM)) + msc_k(a))
//   I_k = sat(max(sat(M_k+MI), sat(I_k+II)) + isc_k(a))
//   D_k = max(sat(M_{k-1}+MD), sat(D_{k-1}+DD))          (current row)
//   xE = max_k M_k (delete transitions are <= 0, so D_k <= max M);
//   xJ = max(xJ, sat(xE+EJ16)); xB = max(sat(MOVE16), sat(xJ+MOVE16))
// overflow if some M or I reaches 32767.  xB depends on max(xJ, 0) only,
// so the wave-wide maximum is taken only when a cell reaches the value that
// would raise it.  The delete chain is computed inside each slot, then
// propagated across slots until no lane changes (exact: sat is monotone).
//
// Delete floor: D only feeds match cells (through D->M) and later deletes
// (through D->D <= 0), and every match cell of this and every later row
// includes the entry value xBe, which never decreases.  So a delete value
// d <= tau = xBe - max_k DM_k, and everything the chain derives from it, can
// never change a match cell: the kernel keeps D' = max(D, tau) instead of D
// (the floored recurrence's fixed point is exactly max(D, tau), since
// sat(tau + DD) <= tau), and sat(D' + DM) differs from sat(D + DM) only
// where both are <= xBe.  M, I, xE and the overflow test are unchanged, and
// the lazy propagation stops as soon as the chains that cross a slot
// boundary fall to the floor, instead of running every chain to its end.

// Overflow without a second pass: where the scores allow it the values are
// re-based instead of saturating.  Stored values are the true ones less `off`.
// When a match or insert value passes RL = 32766 - s_max (s_max: the largest
// emission score, so one row cannot take a value from RL to 32767), the largest
// is brought down to kRebaseTo and off grows by the difference; the result is
// then the exact int32 score, and the overflow flag says that some true value
// reached 32767.  Values that fall below the stored floor F = -32768 are clipped
// there, which changes nothing while
//   xBe - off >= F + W,  W = max(0, max isc) - min msc - min MI     (*)
// No match value is clipped: it is at least xBe + msc.  An insert value above
// its true one is at most F + max isc: the first row's is F + isc, from cells
// that start at F, and a later one is F itself, a clipped true value.  A row
// later it lies at or below M + MI, the insert maximum's other term, and at or
// below xBe where it enters a match maximum, so nothing more comes of it.  The
// delete floor lies above F.  xBe never decreases, so (*) is tested with the
// first row's (where it fails the target is not re-based) and, with the xBe that
// the latest row used, at every re-basing.  Where it fails at the first one, no
// value has reached 32767 yet: the target goes on without re-basing, and to the
// int32 rescore if one does.  Where it fails later, one has (two re-basings are
// at least RL + 1 + (RL + 1 - kRebaseTo) > 32767 up), and it goes there at once.
//
// Measured with every overflow left to the rescore, and re-based: M = 734 x 1M
// targets (1 % homologs), Viterbi 2.50 and 2.74 ms and the rescore 1.68 ms and
// none, 11.4 and 10.6 ms a search; M = 256 x 300,000, Viterbi 0.43 and 0.64 ms,
// 1,810 and 1,700 us a search.
constexpr int kRebaseTo = 8000;
// Instances that re-base: the profiles with a one-wave rescore (up to 768
// nodes; the others' rescore is cooperative).
template <int Q>
constexpr bool kRebase16 = Q <= 6;

// Threads per block of the Viterbi kernel.  Large instances run one wave per
// SIMD (4 waves per block): each wave may then use the whole register file,
// architectural and accumulation registers, and spills go to accumulation
// registers rather than to scratch memory.
template <int Q>
constexpr int kThreads16 = Q >= 16 ? 256 : 512;
// Instances whose transition planes, all but D->D, are read from LDS every
// row instead of being held in registers (D->D, which the lazy delete
// propagation also reads, stays in registers): 120 fewer registers at 20
// vectors per lane, so that two waves share a SIMD and hide each other's
// waits.
template <int Q>
constexpr bool kTrLds16 = Q == 16 || Q == 20;
template <int Q>
constexpr int kMinWaves16 = kTrLds16<Q> ? 2 : Q == 6 ? 4 : 1;
// Threads per block of the one-wave rescore and Forward kernels.
constexpr int kThreads32 = 512;

struct VitResult {
  int raw;
  bool ovf;    // a true match or insert value reached 32767
  bool redo;   // ... and raw is not the exact score
};


template <int Q, bool TRL = false>
__device__ __forceinline__ VitResult vit16_target(const uint32_t *__restrict__ emit, const uint32_t (&tr)[TR_N][Q],
                                                  const DevProfile &P, const uint8_t *x, int L,
                                                  const LenParams &lp, int lane, const uint32_t *ltr = nullptr) {
  uint32_t M[Q], I[Q], D[Q];
#pragma unroll
  for (int q = 0; q < Q; q++) M[q] = I[q] = D[q] = kNegNeg;
  uint32_t accM = kNegNeg, accI = kNegNeg;
  const int mv = lp.move16, ej = P.ej16, entry = P.entry16;
  int xJt = kNeg16;
  int xbt = mv + entry;   // the true xBe
  uint32_t xbe2 = splat16(sat16(xbt));
  auto floor_of = [&](int xbe) { return splat16(min(xbe - P.dm_max16, 32767)); };
  uint32_t tau2 = floor_of(sat16(mv + entry));
  const bool reb = kRebase16<Q> && mv + entry >= kNeg16 + P.rebase_w;
  int RL = reb ? 32766 - P.s_max : 32766;
  uint32_t rl2 = splat16(RL);
  int off = 0, top = 0;   // top: the largest true value at a re-basing
  // trigger: some accM > tm1, or some accI > RL, i.e. accI + iadj > tm1
  uint32_t tm1 = splat16(min(-ej, 32766));
  uint32_t iadj = reb ? splat16(min(-ej, 32766) - RL) : kNegNeg;
  // xJ, xB and the trigger from the largest (stored) match value m so far
  auto settle = [&](int m) {
    xJt = max(xJt, m + off + ej);
    xbt = max(mv, xJt + mv) + entry;
    xbe2 = splat16(sat16(xbt - off));
    tau2 = floor_of(sat16(xbt - off));
    const int t1 = max(min(max(xJt, 0) - ej - off, 32766), kNeg16);
    tm1 = splat16(t1);
    if (reb) iadj = splat16(max(t1 - RL, kNeg16));
  };
  auto load = [&](uint32_t(&e)[2 * Q], int a) {
    const uint32_t *er = emit + a * (2 * Q * kWave);
#pragma unroll
    for (int q = 0; q < 2 * Q; q++) e[q] = er[q * kWave];
  };
  auto row = [&](const uint32_t(&em)[2 * Q]) -> bool {
    // LDS planes: an offset the compiler cannot see through keeps their
    // reads inside the row (loop-invariant reads would be hoisted back
    // into registers)
    int lofs = 0;
    if (TRL) asm volatile("" : "+v"(lofs));
    auto trv = [&](int k, int q) -> uint32_t { return TRL ? ltr[lofs + (k * Q + q) * kWave] : tr[k][q]; };
    const uint32_t msh = slot_up16(M[Q - 1]);
    const uint32_t ish = slot_up16(I[Q - 1]);
    const uint32_t dsh = slot_up16(D[Q - 1]);
#pragma unroll
    for (int q = Q - 1; q >= 0; q--) {
      const uint32_t pm = q ? M[q - 1] : msh, pi = q ? I[q - 1] : ish, pd = q ? D[q - 1] : dsh;
      uint32_t m = i16_max(xbe2, i16_adds(pm, trv(TR_MMIN, q)));
      m = i16_max(m, i16_adds(pi, trv(TR_IMIN, q)));
      m = i16_max(m, i16_adds(pd, trv(TR_DMIN, q)));
      const uint32_t mn = i16_adds(m, em[q]);
      const uint32_t in =
          i16_adds(i16_max(i16_adds(M[q], trv(TR_MI, q)), i16_adds(I[q], trv(TR_II, q))), em[Q + q]);
      accM = i16_max(accM, mn);
      accI = i16_max(accI, in);
      M[q] = mn;
      I[q] = in;
    }
    uint32_t dc = kNegNeg;
    const uint32_t din = slot_up16(M[Q - 1]);
    // the floor joins the M->D term, which does not depend on the chain:
    // the chain itself is one add and one maximum per vector
#pragma unroll
    for (int q = 0; q < Q; q++) {
      const uint32_t md = i16_max(i16_adds(q ? M[q - 1] : din, trv(TR_MDIN, q)), tau2);
      D[q] = i16_max(md, i16_adds(dc, tr[TR_DDIN][q]));
      dc = D[q];
    }
    // A chain can cross into the next slot only from a slot whose last
    // delete value is above the floor (sat(tau + DD) <= tau <= D): when every
    // slot's last value is at the floor, nothing is left to propagate.
    // (A test of whether some slot's first cell would improve, in front of
    // the loop, measured slower: C3 Viterbi 2.90-2.94 against 2.85-2.87 ms.)
    if (any_lane(D[Q - 1] != tau2)) {
      for (int it = 0; it < 2 * kWave; it++) {
        dc = slot_up16(D[Q - 1]);
        bool moved = true;
#pragma unroll
        for (int q = 0; q < Q; q++) {
          if (moved) {
            const uint32_t nd = i16_max(D[q], i16_adds(dc, tr[TR_DDIN][q]));
            moved = any_lane(nd != D[q]);
            D[q] = nd;
            dc = nd;
          }
        }
        if (!moved) break;
      }
    }
    const uint32_t acc = kRebase16<Q> ? i16_max(accM, i16_adds(accI, iadj)) : accM;
    if (__builtin_expect(any_lane(i16_max(acc, tm1) != tm1), 0)) {
      const int m = wave_max_i32(hmax16(accM));
      if (m > RL || (kRebase16<Q> && any_lane(i16_max(accI, rl2) != rl2))) return true;
      settle(m);
    }
    return false;
  };
  uint32_t ea[2 * Q], eb[2 * Q];
  VitResult res;
  res.redo = false;
  for (int r = 0; r < L;) {
    int stop = 0;
    if (!drive_rows(x, L, r, stop, lane, ea, eb, load, row)) break;
    // a value above RL (32766 without re-basing: an overflow)
    if (!reb || RL == 32766) {
      res.redo = true;
      break;
    }
    const int m = wave_max_i32(hmax16(accM));
    const int hi = max(m, wave_max_i32(hmax16(accI)));
    int sh = hi - kRebaseTo;
    if (xbt - off - sh < kNeg16 + P.rebase_w) {
      if (off > 0) {
        res.redo = true;
        break;
      }
      RL = 32766;
      rl2 = splat16(RL);   // no value has reached 32767: on without re-basing
      sh = 0;
    }
    top = max(top, hi + off);
    off += sh;
    const uint32_t sh2 = splat16(sh);
#pragma unroll
    for (int q = 0; q < Q; q++) {
      M[q] = i16_subs(M[q], sh2);
      I[q] = i16_subs(I[q], sh2);
      D[q] = i16_subs(D[q], sh2);
    }
    accM = i16_subs(accM, sh2);
    accI = i16_subs(accI, sh2);
    settle(m - sh);
    r = stop + 1;
  }
  if (!res.redo && !reb) res.redo = any_lane(hmax16(accI) >= 32767);
  if (res.redo) {
    res.ovf = true;
    res.raw = 32767;
  } else {
    const int m = wave_max_i32(hmax16(accM)) + off;
    if (off > 0) top = max(top, max(m, wave_max_i32(hmax16(accI)) + off));
    res.ovf = top >= 32767;
    res.raw = res.ovf ? m + ej + mv : sat16(sat16(m + ej) + mv);
  }
  return res;
}

template <int Q, bool EMIT_LDS>
__global__ void __launch_bounds__(kThreads16<Q>, kMinWaves16<Q>) vit16_kernel(DevProfile P, DevDb db, DevOut out) {
  extern __shared__ uint32_t lds[];
  constexpr bool TRL = kTrLds16<Q>;
  static_assert(!(TRL && EMIT_LDS), "one LDS table per instance");
  const int lane = threadIdx.x & 63;
  // blocks without a target return before staging their table
  const int count = uni(__atomic_load_n(&db.counters[CNT_VIT], __ATOMIC_RELAXED));
  if ((int)blockIdx.x >= count) return;
  if (EMIT_LDS || TRL) {
    const uint4 *src = (const uint4 *)(EMIT_LDS ? P.vit_emit : P.vit_tr);
    const int n4 = (EMIT_LDS ? kAlpha * 2 : TR_N) * Q * kWave / 4;
    uint4 *dst = (uint4 *)lds;
    for (int i = threadIdx.x; i < n4; i += blockDim.x) dst[i] = src[i];
    __syncthreads();
  }
  const uint32_t *emit = (EMIT_LDS ? (const uint32_t *)lds : P.vit_emit) + lane;
  uint32_t tr[TR_N][Q];
#pragma unroll
  for (int k = 0; k < TR_N; k++)
#pragma unroll
    for (int q = 0; q < Q; q++)
      tr[k][q] = (!TRL || k == TR_DDIN) ? P.vit_tr[(k * Q + q) * kWave + lane] : 0u;
  const WorkQueue<> queue(db, WORK_VIT, count);
  for (int idx = queue.first(); idx < count;) {
    const int t = uni(db.list_vit[idx]);
    const int L = uni(db.len[t]);
    if (db.prio_by_len) length_priority(L, db.max_len);
    const LenParams lp = db.lp[L];
    const VitResult r = vit16_target<Q, TRL>(emit, tr, P, db.res + db.start[t], L, lp, lane, (const uint32_t *)lds + lane);
    const bool pass = r.ovf || r.raw >= lp.thr16;
    const uint8_t fl =
        (uint8_t)(uni(db.flags_sorted[t]) | HMM_VIT_RAN | (pass ? HMM_VIT_PASS : 0) | (r.ovf ? HMM_VIT_OVF : 0));
    db.flags_sorted[t] = fl;
    out.vit[uni(db.perm[t])] = r.raw;
    if (r.redo)
      db.list_ovf[wave_fetch_add(&db.counters[CNT_OVF], 1)] = t;
    else if (r.ovf)
      (void)wave_fetch_add(&db.counters[CNT_OVF_EXACT], 1);
    if (pass) db.list_fwd[wave_fetch_add(&db.counters[CNT_FWD], 1)] = t;
    idx = queue.next();
  }
}

// ============================================================================ Viterbi int32 rescore
//
// The int16 recurrence in int32 with every add floored at -2^30 and no upper
// clamp; run on the targets that overflowed int16.  One wave per target, for
// profiles up to 12 vectors per lane (longer ones: hmm_coop.hip): emission
// rows come from LDS, prefetched a row ahead; transitions stay in registers.

__device__ __forceinline__ int fl32(int v) { return max(v, kNeg32); }

// One target's int32 Viterbi score (raw, before the null model), emission
// rows from `emit` (lane's column of [20][2][Q][64]), transitions `tr`.
template <int Q>
__device__ __forceinline__ int vit32_target(const int *emit, const int (&tr)[TR_N][Q], const DevProfile &P,
                                            const uint8_t *x, int L, const LenParams &lp, int lane) {
  auto TR = [&](int k, int q) -> int { return tr[k][q]; };
  const int mv = lp.move16, ej = P.ej16, entry = P.entry16;
  int M[Q], I[Q], D[Q];
#pragma unroll
  for (int q = 0; q < Q; q++) M[q] = I[q] = D[q] = kNeg32;
  int accM = kNeg32;
  int xJt = kNeg32;
  int xB = fl32(mv);
  int xbe = fl32(xB + entry);
  int tau = xbe - P.dm_max32;   // delete floor (as in the int16 kernel); >= xbe >= -2^30
  int T = -ej + 1;
  auto load = [&](int(&e)[2 * Q], int a) {
    const int *er = emit + a * (2 * Q * kWave);
#pragma unroll
    for (int q = 0; q < 2 * Q; q++) e[q] = er[q * kWave];
  };
  auto row = [&](const int(&em)[2 * Q]) -> bool {
    const int msh = lane_up_i(M[Q - 1]);
    const int ish = lane_up_i(I[Q - 1]);
    const int dsh = lane_up_i(D[Q - 1]);
    // The oracle floors every add at -2^30.  Here every add saturates
    // (v_add_i32 clamp), so no sum wraps, and only two floors remain: the
    // insert maximum's -2^30 and the delete floor tau.  A value below
    // -2^30 (after an impossible emission or transition) reaches only
    // maxima that hold a term >= -2^30 -- the match maximum includes xBe,
    // the insert maximum -2^30, the delete maximum tau -- so it is dropped
    // there exactly as the oracle's floored -2^30 is, and every state
    // that is not below -2^30 equals the oracle's.
#pragma unroll
    for (int q = Q - 1; q >= 0; q--) {
      const int pm = q ? M[q - 1] : msh, pi = q ? I[q - 1] : ish, pd = q ? D[q - 1] : dsh;
      const int m = max(max(xbe, sadd32(pm, TR(TR_MMIN, q))),
                        max(sadd32(pi, TR(TR_IMIN, q)), sadd32(pd, TR(TR_DMIN, q))));
      const int mn = sadd32(m, em[q]);
      const int in = sadd32(max(max(sadd32(M[q], TR(TR_MI, q)), sadd32(I[q], TR(TR_II, q))), kNeg32), em[Q + q]);
      accM = max(accM, mn);
      M[q] = mn;
      I[q] = in;
    }
    int dc = kNeg32;
    const int din = lane_up_i(M[Q - 1]);
#pragma unroll
    for (int q = 0; q < Q; q++) {
      D[q] = max(max(sadd32(q ? M[q - 1] : din, TR(TR_MDIN, q)), sadd32(dc, TR(TR_DDIN, q))), tau);
      dc = D[q];
    }
    // Chains crossing into the next lane: nothing moves unless some lane's
    // first cell improves, which this one test rules out in the common case.
    if (any_lane(lane_up_i(D[Q - 1]) + TR(TR_DDIN, 0) > D[0])) {
      for (int it = 0; it < kWave; it++) {
        dc = lane_up_i(D[Q - 1]);
        bool moved = true;
#pragma unroll
        for (int q = 0; q < Q; q++) {
          if (moved) {
            const int nd = max(D[q], dc + TR(TR_DDIN, q));   // D[q] >= tau >= -2^30 already
            moved = any_lane(nd != D[q]);
            D[q] = nd;
            dc = nd;
          }
        }
        if (!moved) break;
      }
    }
    if (any_lane(accM >= T)) {
      const int m = wave_max_i32(accM);
      xJt = max(xJt, fl32(m + ej));
      xB = max(fl32(mv), fl32(xJt + mv));
      xbe = fl32(xB + entry);
      tau = xbe - P.dm_max32;
      T = max(xJt, 0) - ej + 1;
    }
    return false;
  };
  int ea[2 * Q], eb[2 * Q];
  int stop;
  (void)drive_rows(x, L, 0, stop, lane, ea, eb, load, row);
  const int m = wave_max_i32(accM);
  return fl32(fl32(m + ej) + mv);
}

template <int Q>
__device__ __forceinline__ void load_tr32(const DevProfile &P, int lane, int (&tr)[TR_N][Q]) {
#pragma unroll
  for (int k = 0; k < TR_N; k++)
#pragma unroll
    for (int q = 0; q < Q; q++) tr[k][q] = P.v32_tr[(k * Q + q) * kWave + lane];
}

template <int Q>
__global__ void __launch_bounds__(kThreads32) vit32_kernel(DevProfile P, DevDb db, DevOut out) {
  extern __shared__ int32_t lds32[];
  const int lane = threadIdx.x & 63;
  constexpr int kEmit = kAlpha * 2 * Q * kWave;   // dwords
  // blocks without a target return before staging their table
  const int count = uni(__atomic_load_n(&db.counters[CNT_OVF], __ATOMIC_RELAXED));
  if ((int)blockIdx.x >= count) return;
  for (int i = threadIdx.x; i < kEmit / 4; i += blockDim.x) ((int4 *)lds32)[i] = ((const int4 *)P.v32_emit)[i];
  __syncthreads();
  const int *emit = (const int *)lds32 + lane;
  int tr[TR_N][Q];
  load_tr32<Q>(P, lane, tr);
  const WorkQueue<> queue(db, WORK_OVF, count);
  for (int idx = queue.first(); idx < count;) {
    const int t = uni(db.list_ovf[idx]);
    const int L = uni(db.len[t]);
    if (db.prio_by_len) length_priority(L, db.max_len);
    const LenParams lp = db.lp[L];
    out.vit[uni(db.perm[t])] = vit32_target<Q>(emit, tr, P, db.res + db.start[t], L, lp, lane);
    idx = queue.next();
  }
}

// ============================================================================ Forward fp32
//
// Probability space, 1 = the start state.  Per row (residue a):
//   M_k = e_k(a)/f(a) * (M_{k-1} MM + I_{k-1} IM + D_{k-1} DM + B entry)    (previous row)
//   I_k = i_k(a)/f(a) * (M_k MI + I_k II)                                    (previous row)
//   D_k = M_{k-1} MD + D_{k-1} DD                                            (current row)
//   E = sum_k (M_k + D_k); J = J loop + E/2; C = C loop + E/2; N = N loop;
//   B = (N + J) move.
// The delete chain runs inside each slot with a zero entry value; the values
// entering the slots follow from an inclusive scan of the affine maps
// x -> D_out + P x across lanes (P = product of the slot's DD), whose P part
// is profile-constant and precomputed.  Values are rescaled by an exact power
// of two whenever the largest special value leaves [2^-40, 2^40]; the removed
// exponents are summed.  Result: ln(C move) + (sum of exponents) ln 2, nats.

// Per-profile register state of the one-wave Forward: transitions, exit
// weights and the P part of the delete-chain scan (the lane's P before each
// of the six steps).
template <int Q>
struct FwdRegs {
  float tr[TR_N + 1][Q], gx[Q], pstep[6];
};

template <int Q>
__device__ __forceinline__ void load_fwd_regs(const DevProfile &P, int lane, FwdRegs<Q> &R) {
  const float *trp = P.f_tr + lane;
#pragma unroll
  for (int k = 0; k <= TR_N; k++)
#pragma unroll
    for (int q = 0; q < Q; q++) R.tr[k][q] = trp[(k * Q + q) * kWave];
#pragma unroll
  for (int q = 0; q < Q; q++) R.gx[q] = trp[(TR_EXIT * Q + q) * kWave];   // exit weights: E = sum M g
  float p = P.f_tr[(TR_N * Q + Q - 1) * kWave + lane];
#define HMM_PSTEP(I, CTRL, MASK) \
  R.pstep[I] = p;                \
  p = p * dpp_f<CTRL, MASK>(p, 1.0f);
  HMM_PSTEP(0, kRowShr1, 0xf)
  HMM_PSTEP(1, kRowShr2, 0xf)
  HMM_PSTEP(2, kRowShr4, 0xf)
  HMM_PSTEP(3, kRowShr8, 0xf)
  HMM_PSTEP(4, kRowBcast15, 0xa)
  HMM_PSTEP(5, kRowBcast31, 0xc)
#undef HMM_PSTEP
}

// One target's Forward score in nats (before the null model), emission
// rows from `emit` (lane's column of [20][2][Q][64]).
template <int Q>
__device__ __forceinline__ float fwd_target(const float *emit, const FwdRegs<Q> &R, const DevProfile &P,
                                            const uint8_t *x, int L, const LenParams &lp, int lane) {
  auto TR = [&](int k, int q) -> float { return R.tr[k][q]; };
  const float(&gx)[Q] = R.gx;
  const float(&pstep)[6] = R.pstep;
  const float entry_p = P.entry_p;
  const float loop = lp.loop_p, move = lp.move_p;
  float M[Q], I[Q], D[Q];
#pragma unroll
  for (int q = 0; q < Q; q++) M[q] = I[q] = D[q] = 0.0f;
  float N = 1.0f, B = move, J = 0.0f, C = 0.0f;
  int shift = 0;
  auto load = [&](float(&e)[2 * Q], int a) {
    const float *er = emit + a * (2 * Q * kWave);
#pragma unroll
    for (int q = 0; q < 2 * Q; q++) e[q] = er[q * kWave];
  };
  auto row = [&](const float(&em)[2 * Q]) -> bool {
    const float bent = B * entry_p;
    // the first cell's predecessors are the previous lane's last cells
    // (none in lane 0), read through the lane shift of each multiply-add
    float sm0 = bent;
    fmac_up3(sm0, D[Q - 1], TR(TR_DMIN, 0), I[Q - 1], TR(TR_IMIN, 0), M[Q - 1], TR(TR_MMIN, 0));
    float part = 0.0f;   // this lane's part of E: sum of M g (deletes included through g)
#pragma unroll
    for (int q = Q - 1; q >= 0; q--) {
      const float sm =
          q ? fmaf(M[q - 1], TR(TR_MMIN, q), fmaf(I[q - 1], TR(TR_IMIN, q), fmaf(D[q - 1], TR(TR_DMIN, q), bent)))
            : sm0;
      const float si = fmaf(M[q], TR(TR_MI, q), I[q] * TR(TR_II, q));
      M[q] = em[q] * sm;
      I[q] = em[Q + q] * si;
      part = fmaf(M[q], gx[q], part);
    }
    // delete chain inside the lane from a zero entry (the first cell's M
    // predecessor is the previous lane's new last M)
    D[0] = mul_up(M[Q - 1], TR(TR_MDIN, 0));
#pragma unroll
    for (int q = 1; q < Q; q++) D[q] = fmaf(M[q - 1], TR(TR_MDIN, q), D[q - 1] * TR(TR_DDIN, q));
    float chain = D[Q - 1];
    scan_sum_affine(part, chain, pstep);
    const float carry = lane_up_f(chain);
#pragma unroll
    for (int q = 0; q < Q; q++) D[q] = fmaf(carry, TR(TR_N, q), D[q]);
    const float E = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, part), 63));
    J = fmaf(J, loop, 0.5f * E);
    C = fmaf(C, loop, 0.5f * E);
    N = N * loop;
    B = (N + J) * move;
    const float big = fmaxf(fmaxf(fmaxf(E, J), fmaxf(C, N)), B);
    if (big > 0x1p40f || big < 0x1p-40f) {
      int ex;
      (void)frexpf(big, &ex);
      ex = uni(ex);
      const float s = ldexpf(1.0f, -ex);
#pragma unroll
      for (int q = 0; q < Q; q++) {
        M[q] *= s;
        I[q] *= s;
        D[q] *= s;
      }
      J *= s;
      C *= s;
      N *= s;
      B *= s;
      shift += ex;
    }
    return false;
  };
  float ea[2 * Q], eb[2 * Q];
  int stop;
  (void)drive_rows(x, L, 0, stop, lane, ea, eb, load, row);
  return (float)(log((double)C * (double)move) + (double)shift * M_LN2);
}

template <int Q>
__global__ void __launch_bounds__(kThreads32) fwd_kernel(DevProfile P, DevDb db, DevOut out) {
  extern __shared__ float ldsf[];
  const int lane = threadIdx.x & 63;
  constexpr int kEmit = kAlpha * 2 * Q * kWave;
  // blocks without a target return before staging their table
  const int count = uni(__atomic_load_n(&db.counters[CNT_FWD], __ATOMIC_RELAXED));
  if ((int)blockIdx.x >= count) return;
  for (int i = threadIdx.x; i < kEmit / 4; i += blockDim.x) ((float4 *)ldsf)[i] = ((const float4 *)P.f_emit)[i];
  __syncthreads();
  const float *emit = (const float *)ldsf + lane;
  FwdRegs<Q> R;
  load_fwd_regs<Q>(P, lane, R);
  const WorkQueue<> queue(db, WORK_FWD, count);
  for (int idx = queue.first(); idx < count;) {
    const int t = uni(db.list_fwd[idx]);
    const int L = uni(db.len[t]);
    if (db.prio_by_len) length_priority(L, db.max_len);
    const LenParams lp = db.lp[L];
    const float f = fwd_target<Q>(emit, R, P, db.res + db.start[t], L, lp, lane);
    const bool pass = f > lp.fthr;
    const uint8_t fl = (uint8_t)(uni(db.flags_sorted[t]) | HMM_FWD_RAN | (pass ? HMM_FWD_PASS : 0));
    db.flags_sorted[t] = fl;
    out.fwd[uni(db.perm[t])] = f;
    if (pass) (void)wave_fetch_add(&db.counters[CNT_FWD_PASS], 1);
    idx = queue.next();
  }
}

// ============================================================================ fused tail
//
// For profiles of up to 384 nodes (3 int16 vectors per lane) the three
// stages after MSV run as one kernel: a wave takes an MSV survivor, scores
// it with the int16 Viterbi, rescores it in int32 at once if it overflowed,
// and runs Forward on it at once if it passed.  The staged kernels each wait
// for the longest target of the stage before them; here a target's stages
// follow each other without waiting for any other target, and a launch ends
// when its last wave's chain of stages does.  The three emission tables sit
// in LDS side by side (10 KB per vector of each: the int16 Viterbi's per
// int16 vector, the rescore's and Forward's per 32-bit vector);
// transitions are read per target and stage, so that no stage's
// registers stay live through the others.  Results, flags and counts are
// the staged kernels' (the survivor lists between the stages are not
// written).
template <int Q8>
constexpr int kThreadsTail = Q8 <= 2 ? 1024 : 512;

template <int Q8, int Q32>
__global__ void __launch_bounds__(kThreadsTail<Q8>) tail_kernel(DevProfile P, DevDb db, DevOut out) {
  extern __shared__ uint32_t ldst[];
  const int lane = threadIdx.x & 63;
  constexpr int n16 = kAlpha * 2 * Q8 * kWave, n32 = kAlpha * 2 * Q32 * kWave;   // dwords
  // blocks without a target return before staging their tables
  const int count = uni(__atomic_load_n(&db.counters[CNT_VIT], __ATOMIC_RELAXED));
  if ((int)blockIdx.x >= count) return;
  for (int i = threadIdx.x; i < n16 / 4; i += blockDim.x) ((uint4 *)ldst)[i] = ((const uint4 *)P.vit_emit)[i];
  for (int i = threadIdx.x; i < n32 / 4; i += blockDim.x) {
    ((uint4 *)(ldst + n16))[i] = ((const uint4 *)P.v32_emit)[i];
    ((uint4 *)(ldst + n16 + n32))[i] = ((const uint4 *)P.f_emit)[i];
  }
  __syncthreads();
  const uint32_t *e16 = ldst + lane;
  const int *e32 = (const int *)ldst + n16 + lane;
  const float *ef = (const float *)ldst + n16 + n32 + lane;
  const WorkQueue<> queue(db, WORK_VIT, count);
  for (int idx = queue.first(); idx < count;) {
    const int t = uni(db.list_vit[idx]);
    const int L = uni(db.len[t]);
    if (db.prio_by_len) length_priority(L, db.max_len);
    const LenParams lp = db.lp[L];
    const uint8_t *x = db.res + db.start[t];
    // the transition reads' lane offset, opaque to the compiler: otherwise
    // it keeps every read's address live through the loop
    int ln = lane;
    asm volatile("" : "+v"(ln));
    VitResult r;
    {
      uint32_t tr[TR_N][Q8];
#pragma unroll
      for (int k = 0; k < TR_N; k++)
#pragma unroll
        for (int q = 0; q < Q8; q++) tr[k][q] = P.vit_tr[(k * Q8 + q) * kWave + ln];
      r = vit16_target<Q8>(e16, tr, P, x, L, lp, lane);
    }
    const bool pass = r.ovf || r.raw >= lp.thr16;
    int vit = r.raw;
    if (r.ovf) (void)wave_fetch_add(&db.counters[CNT_OVF_EXACT], 1);
    if (r.redo) {
      int tr[TR_N][Q32];
      load_tr32<Q32>(P, ln, tr);
      vit = vit32_target<Q32>(e32, tr, P, x, L, lp, lane);
    }
    const int c = uni(db.perm[t]);
    out.vit[c] = vit;
    uint8_t fl = (uint8_t)(uni(db.flags_sorted[t]) | HMM_VIT_RAN | (pass ? HMM_VIT_PASS : 0) |
                           (r.ovf ? HMM_VIT_OVF : 0));
    if (pass) {
      (void)wave_fetch_add(&db.counters[CNT_FWD], 1);
      FwdRegs<Q32> R;
      load_fwd_regs<Q32>(P, ln, R);
      const float f = fwd_target<Q32>(ef, R, P, x, L, lp, lane);
      const bool fpass = f > lp.fthr;
      fl |= (uint8_t)(HMM_FWD_RAN | (fpass ? HMM_FWD_PASS : 0));
      out.fwd[c] = f;
      if (fpass) (void)wave_fetch_add(&db.counters[CNT_FWD_PASS], 1);
    }
    db.flags_sorted[t] = fl;
    idx = queue.next();
  }
}

// ============================================================================ small kernels

// One block per counter block: the list counters and the work counters.
__global__ void clear_counters(int32_t *counters) {
  int32_t *c = counters + (size_t)blockIdx.x * CNT_N;
  const int i = threadIdx.x;
  if (i < CNT_LISTS) c[i] = 0;
  if (i < WORK_STAGES * kWorkLanes) c[CNT_WORK + i * kWorkStride] = 0;
}

// Results in the caller's order, once every stage of a search is done: each
// thread takes one caller index c and its sorted index iperm[c]; the flags
// and MSV score come from the sorted arrays the stages wrote, and Viterbi
// and Forward scores, written in caller order by those stages for the
// targets they scored, get INT32_MIN and NaN where the stage did not run.
// Reads of iperm and writes of every output are contiguous.  The first block
// also exports the counts (the sum over the chunks' counter blocks).
__global__ void __launch_bounds__(256) results_kernel(DevDb db, DevOut out, int nblocks) {
  if (blockIdx.x == 0 && threadIdx.x == 0 && out.counts) {
    int64_t v[4] = {0, 0, 0, 0};
    for (int k = 0; k < nblocks; k++) {
      const int32_t *b = db.counters + k * CNT_N;
      v[0] += b[CNT_VIT];
      v[1] += b[CNT_OVF] + b[CNT_OVF_EXACT];
      v[2] += b[CNT_FWD];
      v[3] += b[CNT_FWD_PASS];
    }
    for (int i = 0; i < 4; i++) out.counts[i] = v[i];
  }
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= db.n) return;
  const int t = db.iperm[c];
  const uint8_t fl = db.flags_sorted[t];
  out.flags[c] = fl;
  out.msv[c] = db.msv_sorted[t];
  if (!(fl & HMM_VIT_RAN)) out.vit[c] = INT32_MIN;
  if (!(fl & HMM_FWD_RAN)) out.fwd[c] = __builtin_nanf("");
}

// ============================================================================ launcher

int g_num_cu = 0;

int num_cu() {
  if (!g_num_cu) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&g_num_cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (g_num_cu <= 0) g_num_cu = 256;
  }
  return g_num_cu;
}

template <typename K>
int blocks_per_cu(K kernel, int threads, size_t lds) {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, threads, lds) != hipSuccess || nb < 1) nb = 1;
  return nb;
}

template <int Q>
hipError_t launch_vit16(const DevProfile &P, const DevDb &db, const DevOut &o, hipStream_t s) {
  constexpr bool kLds = Q <= 8;
  const int threads = kThreads16<Q>;
  const size_t lds = kLds ? (size_t)kAlpha * 2 * Q * kWave * 4 : kTrLds16<Q> ? (size_t)TR_N * Q * kWave * 4 : 0;
  auto k = vit16_kernel<Q, kLds>;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  static int bpc = 0;
  if (!bpc) bpc = blocks_per_cu(k, threads, lds);
  const int64_t blocks = std::min((int64_t)bpc * num_cu(), db.n);
  hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(threads), lds, s, P, db, o);
  return hipGetLastError();
}

// Persistent launch of a list kernel: as many blocks as fit, at most one
// block per database target (few targets then spread over all CUs).
template <typename K>
hipError_t launch_list_kernel(K k, int threads, int &bpc, size_t lds, const DevProfile &P, const DevDb &db,
                              const DevOut &o, hipStream_t s) {
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  if (!bpc) bpc = blocks_per_cu(k, threads, lds);
  const int64_t blocks = std::min((int64_t)bpc * num_cu(), db.n);
  hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(threads), lds, s, P, db, o);
  return hipGetLastError();
}

// One-wave 32-bit kernels: the emission table in LDS (at most 120 KB, for
// 12 vectors per lane), transitions in registers.
template <int Q>
hipError_t launch_vit32(const DevProfile &P, const DevDb &db, const DevOut &o, hipStream_t s) {
  static_assert(Q <= 12, "longer profiles take the cooperative kernels");
  const size_t lds = (size_t)kAlpha * 2 * Q * kWave * 4;
  static int bpc = 0;
  return launch_list_kernel(vit32_kernel<Q>, kThreads32, bpc, lds, P, db, o, s);
}

template <int Q>
hipError_t launch_fwd(const DevProfile &P, const DevDb &db, const DevOut &o, hipStream_t s) {
  static_assert(Q <= 12, "longer profiles take the cooperative kernels");
  const size_t lds = (size_t)kAlpha * 2 * Q * kWave * 4;
  static int bpc = 0;
  return launch_list_kernel(fwd_kernel<Q>, kThreads32, bpc, lds, P, db, o, s);
}

// Fused tail (profiles of up to 3 int16 vectors per lane): the three
// emission tables in LDS, as many blocks as fit, at most one wave per target.
template <int Q8, int Q32>
hipError_t launch_tail_fused(const DevProfile &P, const DevDb &db, const DevOut &o, hipStream_t s) {
  const size_t lds = (size_t)kAlpha * 2 * kWave * 4 * (Q8 + 2 * Q32);
  static int bpc = 0;
  return launch_list_kernel(tail_kernel<Q8, Q32>, kThreadsTail<Q8>, bpc, lds, P, db, o, s);
}

// The int16 / 32-bit vector counts with a fused-tail instance.
bool tail_fused_instance(const DevProfile &P) {
  return (P.Q8 == 1 && P.Q32 <= 2) || (P.Q8 == 2 && (P.Q32 == 3 || P.Q32 == 4)) ||
         (P.Q8 == 3 && (P.Q32 == 5 || P.Q32 == 6));
}

hipError_t dispatch_tail_fused(const DevProfile &P, const DevDb &db, const DevOut &o, hipStream_t s) {
#define HMM_TAIL(a, b) \
  if (P.Q8 == a && P.Q32 == b) return launch_tail_fused<a, b>(P, db, o, s);
  HMM_TAIL(1, 1) HMM_TAIL(1, 2) HMM_TAIL(2, 3) HMM_TAIL(2, 4) HMM_TAIL(3, 5) HMM_TAIL(3, 6)
#undef HMM_TAIL
  return hipErrorInvalidValue;
}

#define HMM_Q8_CASES(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(10) X(12) X(14) X(16) X(20) X(24)
// One-wave instances of the 32-bit kernels; 14 and more vectors per lane
// (14, 16, 20, 24, 28, 32, 40, 48) run the cooperative ones.
#define HMM_Q32_CASES(X) X(1) X(2) X(3) X(4) X(5) X(6) X(8) X(10) X(12)

hipError_t launch_bias(const DevProfile &P, const DevDb &db, const DevOut &o, hipStream_t s) {
  static int bpc = 0;
  if (!bpc) bpc = blocks_per_cu(bias_kernel, 256, 0);
  const int64_t blocks = std::min((int64_t)bpc * num_cu(), db.n);
  hipLaunchKernelGGL(bias_kernel, dim3((unsigned)blocks), dim3(256), 0, s, P, db, o);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(reset_ovf, dim3(1), dim3(64), 0, s, db.counters);
  return hipGetLastError();
}

hipError_t dispatch_vit16(const DevProfile &P, const DevDb &db, const DevOut &o, hipStream_t s) {
  switch (P.Q8) {
#define HMM_CASE(q) \
  case q:           \
    return launch_vit16<q>(P, db, o, s);
    HMM_Q8_CASES(HMM_CASE)
#undef HMM_CASE
  }
  return hipErrorInvalidValue;
}

hipError_t dispatch_vit32(const DevProfile &P, const DevDb &db, const DevOut &o, hipStream_t s) {
  if (coop_instance(P.Q32)) return launch_vit32_coop(P, db, o, s);
  switch (P.Q32) {
#define HMM_CASE(q) \
  case q:           \
    return launch_vit32<q>(P, db, o, s);
    HMM_Q32_CASES(HMM_CASE)
#undef HMM_CASE
  }
  return hipErrorInvalidValue;
}

hipError_t dispatch_fwd(const DevProfile &P, const DevDb &db, const DevOut &o, hipStream_t s) {
  if (coop_instance(P.Q32)) return launch_fwd_coop(P, db, o, s);
  switch (P.Q32) {
#define HMM_CASE(q) \
  case q:           \
    return launch_fwd<q>(P, db, o, s);
    HMM_Q32_CASES(HMM_CASE)
#undef HMM_CASE
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_tail(const DevProfile &P, const DevDb *chunk, int K, const DevOut &o, hipStream_t s,
                       const SearchSync &y, hipEvent_t *ev, bool join = true, bool swap = false);

hipError_t launch_search(const DevProfile &P, const DevDb *chunk, int K, const DevOut &o, hipStream_t s,
                         const SearchSync &y, hipEvent_t *ev) {
  if (K < 1 || K > kMaxChunks) return hipErrorInvalidValue;
  hipError_t e = hipSuccess;
  auto ok = [&](hipError_t r) {
    if (e == hipSuccess) e = r;
    return e == hipSuccess;
  };
  auto mark = [&](int i, hipStream_t st) {
    if (ev) ok(hipEventRecord(ev[i], st));
  };
  mark(0, s);
  hipLaunchKernelGGL(clear_counters, dim3(K), dim3(64), 0, s, chunk[0].counters);
  ok(hipGetLastError());
  // MSV of every chunk, back to back on the search stream
  for (int k = 0; k < K && e == hipSuccess; k++) {
    if (chunk[k].n > 0) {
      ok(launch_msv(&P, &chunk[k], &o, 1, s));
      if (o.bias_filter) ok(launch_bias(P, chunk[k], o, s));
    }
    if (K > 1) ok(hipEventRecord(y.msv_done[k], s));
  }
  mark(1, s);
  if (e != hipSuccess) return e;
  return launch_tail(P, chunk, K, o, s, y, ev);
}

// The rest of each chunk's cascade as soon as its MSV is done, then the counts
// and the caller-order results.  A single search of one chunk runs it all on
// the search stream; chunks, and the searches of a group, on the handle's tail
// stream (event y.msv_done[k] on the search stream starts them, and the search
// stream waits for y.tail_done when `join` is set; a group joins all of its
// searches at its end).  With `o.fused_tail` and a profile that has a fused
// instance, one kernel takes all three stages.  Otherwise the rescore runs
// beside Forward (an overflow passes the Viterbi filter whatever its exact score,
// so Forward needs nothing from it), one of them on the handle's other stream.
// Only a search that keeps to the search stream and whose overflows are re-based
// (not o.rescore_apart) runs it before Forward: there it has nothing to do in
// ordinary searches, and an empty launch takes 4 us, a fork and join of streams
// 10 to 20.  (In a group of 12 the searches' streams overlap each other: 10.04 ms
// with the empty launches in line, 9.94 beside Forward.)  Which of the two keeps
// to the search stream starts first and ends without waiting for a join, and its
// blocks hold the CUs until it ends.  From 20 vectors per lane on that is the
// rescore, the longer one per target: 10,000 homologs at M = 1,500 26.4 ms,
// Forward first 28.0; 30,000 targets with 0.2 % homologs at M = 2,500 6.70 and
// 6.90, at M = 1,300 2.50 and 2.53; 1,000 open at M = 2,500 2.88 and 3.02.  Below, it
// is Forward: 30,000 with 1 % homologs at M = 800 1.42, rescore first 1.50, at M =
// 1,000 1.69 and 1.72; 300 open at M = 800 1.09 and 1.12.  `swap` exchanges the two
// streams.
hipError_t launch_tail(const DevProfile &P, const DevDb *chunk, int K, const DevOut &o, hipStream_t s,
                       const SearchSync &y, hipEvent_t *ev, bool join, bool swap) {
  hipError_t e = hipSuccess;
  auto ok = [&](hipError_t r) {
    if (e == hipSuccess) e = r;
    return e == hipSuccess;
  };
  auto mark = [&](int i, hipStream_t st) {
    if (ev) ok(hipEventRecord(ev[i], st));
  };
  const bool fused = o.fused_tail && tail_fused_instance(P);
  const bool own = K > 1 || !join;
  const bool apart = (o.rescore_apart || own) && !fused;
  const hipStream_t ts = !own ? s : swap ? y.aux : y.tail, as = swap ? y.tail : y.aux;
  const bool rescore_first = apart && !own && P.Q32 >= 20;
  const hipStream_t rs = apart && !rescore_first ? as : ts, fs = rescore_first ? as : ts;   // the rescore's and Forward's
  for (int k = 0; k < K && e == hipSuccess; k++) {
    const bool any = chunk[k].n > 0;
    const DevDb &ck = chunk[k];
    if (own && !ok(hipStreamWaitEvent(ts, y.msv_done[k], 0))) break;
    if (any && !ok(fused ? dispatch_tail_fused(P, ck, o, ts) : dispatch_vit16(P, ck, o, ts))) break;
    if (k == K - 1) mark(2, ts);
    if (apart && (!ok(hipEventRecord(y.vit_done[k], ts)) || !ok(hipStreamWaitEvent(as, y.vit_done[k], 0)))) break;
    if (any && !fused && !ok(dispatch_vit32(P, ck, o, rs))) break;
    if (k == K - 1) mark(3, fused ? ts : rs);
    if (any && !fused && !ok(dispatch_fwd(P, ck, o, fs))) break;
  }
  if (apart && ok(hipEventRecord(y.aux_done, as))) ok(hipStreamWaitEvent(ts, y.aux_done, 0));
  // chunk 0 starts at sorted index 0: its sorted arrays are the whole
  // database's
  DevDb all = chunk[0];
  all.n = 0;
  for (int k = 0; k < K; k++) all.n += chunk[k].n;
  if (e == hipSuccess && all.n > 0) {
    hipLaunchKernelGGL(results_kernel, dim3((unsigned)((all.n + 255) / 256)), dim3(256), 0, ts, all, o, K);
    ok(hipGetLastError());
  }
  if (own && ok(hipEventRecord(y.tail_done, ts)) && join) ok(hipStreamWaitEvent(s, y.tail_done, 0));
  if (join) mark(4, s);
  return e;
}

// Several searches of one database (one handle each) by different profiles,
// one chunk each: their counters are cleared, the MSV of profiles sharing a
// diagonal instance runs as group kernels (up to msv_group_max profiles per
// launch; the others alone), then each search's composition-bias filter
// (if on) and its cascade tail on its own handle's streams, all joined back
// into `s`.
hipError_t launch_search_group(const DevProfile *P, const DevDb *db, const DevOut *o, int n, hipStream_t s,
                               const SearchSync *const *y) {
  hipError_t e = hipSuccess;
  auto ok = [&](hipError_t r) {
    if (e == hipSuccess) e = r;
    return e == hipSuccess;
  };
  for (int i = 0; i < n && e == hipSuccess; i++) {
    hipLaunchKernelGGL(clear_counters, dim3(1), dim3(64), 0, s, db[i].counters);
    ok(hipGetLastError());
  }
  std::vector<int> done(n, 0);
  // a search's composition-bias filter (if on) and its cascade tail, on its
  // own handle's streams once its MSV (on `s`) is done.  Each handle's two
  // streams share the four hardware queues with the others' in the order in
  // which they were made: the first four tails have a queue each, the later ones
  // only two between them.  So from the fifth on every other pair exchanges its
  // streams.  What that gives depends on the streams that the process made
  // before.  Without and with the exchange, handles made one after another: 8
  // searches by profiles of 50 to 330 nodes 4.02 and 3.79 ms, 9 of 77 to 616 3.15
  // and 3.08, 12 of 50 to 400 9.99 and 9.83, 16 of 50 to 500 10.82 and 10.29; with
  // one to three other streams made and used before, between 6 % faster and 2 %
  // slower.  Exchanging every other one from the first on: 12 in 9.45, 16 in 9.9,
  // but 2 in 0.94 or 1.30, depending on those streams.
  auto tail = [&](int i) {
    if (o[i].bias_filter && db[i].n > 0) ok(launch_bias(P[i], db[i], o[i], s));
    ok(hipEventRecord(y[i]->msv_done[0], s));
    ok(launch_tail(P[i], &db[i], 1, o[i], s, *y[i], nullptr, false, i >= 4 && (i & 2)));
  };
  for (int i = 0; i < n && e == hipSuccess; i++) {
    if (done[i] || db[i].n == 0) continue;
    const int gmax = msv_group_max(P[i]);
    std::vector<int> grp{i};
    for (int j = i + 1; j < n && (int)grp.size() < gmax; j++)
      if (!done[j] && P[j].msv_diag == P[i].msv_diag && P[j].Qm == P[i].Qm) grp.push_back(j);
    for (int j : grp) done[j] = 1;
    DevProfile gp[kMaxMsvGroup];
    DevDb gd[kMaxMsvGroup];
    DevOut go[kMaxMsvGroup];
    for (size_t g = 0; g < grp.size(); g++) {
      gp[g] = P[grp[g]];
      gd[g] = db[grp[g]];
      go[g] = o[grp[g]];
    }
    ok(launch_msv(gp, gd, go, (int)grp.size(), s));
  }
  // The tails start after every MSV launch.  Started right after their own
  // group's launch, they share the CUs with the later MSV launches, which
  // absorb that (their waves take targets from work counters), but the
  // group still took longer (64 profiles of 50 to 400 nodes, with an MSV kernel
  // of three instructions per pair of cells: 350.7 against 345.0 ms).
  for (int i = 0; i < n && e == hipSuccess; i++) tail(i);
  // every search's tail joins the caller's stream
  for (int i = 0; i < n && e == hipSuccess; i++) ok(hipStreamWaitEvent(s, y[i]->tail_done, 0));
  return e;
}

}  // namespace hmmgpu

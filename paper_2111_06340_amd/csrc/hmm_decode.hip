// HIP kernels (gfx950) of posterior decoding: for every selected target,
// Forward with every row kept, Backward with the posterior probability of
// each state at each residue, the target's domain regions, and one
// optimal-accuracy alignment per region (the hit's row of the multiple
// sequence alignment).
//
// A team of W waves decodes one target at a time in a private scratch slot (one
// slot per resident team): W = 1 for short profiles, a workgroup of 2 or 4
// waves for longer ones.  Wave w holds the cells [64 QW w, 64 QW (w + 1)), QW of
// them per lane: a cell's neighbour lives in the same lane, in the next lane
// (one DPP shift), or, at a wave's edge, in the next wave.  A row takes one
// barrier: before it every wave does what needs nothing from the others and
// publishes a few values of its edge cell and its sums, after it every wave
// finishes its cells.  The delete chains are affine (max-plus in the
// alignment), so a wave's chain is scanned with nothing entering, and the value
// that does enter, x = sum over the waves before it of what they pass on times
// constant products, is added after the barrier with one multiply-add a cell.
//   1. Forward in fp32 probability space, keeping M_k(i) and I_k(i) of every
//      row and the row's special values (N, J-loop, C-loop and E parts).
//   2. Backward from row L down to row 1.  The backward delete chain runs
//      from cell k+1 to cell k, so this phase puts virtual lane v = 63 - l
//      on physical lane l: the chain then crosses lanes in the same
//      direction as the forward one (lane l-1 -> l) and reuses its DPP
//      prefix scan.  Each row's posteriors are normalised by that row's
//      total, sum over the states that can emit residue i
//         Z_i = sum_k (fM bM + fI bI) + fN bN + fJl bJ + fCl bC,
//      which is the same value P(x) in the row's scale, so no scale factor
//      has to be tracked.  Row i's total is published with row i - 1's values,
//      and the region rule and the optimal-accuracy recurrence (written from
//      the end of the region, max-plus form, a 4-bit traceback code per cell)
//      follow one row behind, so posteriors are never stored and a row still
//      takes one barrier.
//   3. Traceback of each region's alignment, from its start cell forwards.
// Values are kept inside [2^-32, 2^32] by exact power-of-two rescaling in
// both directions, so a product of a forward and a backward value stays far
// from the fp32 range limits.
//
// Lane-divergent branches appear only around stores (predicated writes of
// one lane's value); every cross-lane operation runs with all lanes active.
//
// Bound: each row's dependency chains and, for many targets, VALU issue (M =
// 734: about 930 instructions per target row, 16 bytes of HBM traffic a cell).
// One vmcnt counts loads and stores, in order, so what made rows wait for
// memory was any wait for the youngest of them: table loads pending at a loop's
// head, merges and copies of loaded registers, spills, a residue chunk's load.
// Measured against one wave per target for every profile, with the alignment's
// transitions tested in every cell: 2,000 targets at M = 734 5.71 -> 4.74 ms,
// 150 at M = 2,500 56.0 -> 8.2 ms, 2,000 at M = 256 in the static scratch 5.55
// -> 3.90 ms, 500 at M = 300 1.34 -> 1.0 ms.  Instances measured at M = 734: 2
// waves of 6 cells a lane 5.1 ms, 4 of 3 6.4 ms (before the joint scans); at M =
// 256: 1 wave of 4 cells 4.6 ms, 2 of 2 5.4 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <mutex>

#include "hmm_device.h"
#include "hmm_internal.h"

// Decode scratch of hmm_decode_static: one copy per device, never freed.
// Host code must not pass this name to a kernel (on the host it is only a
// stand-in for the symbol); kernels get the address static_decode_scratch
// looked up for the current device.
static __device__ __align__(256) float scratch[hmmgpu::kStaticDecodeBytes / sizeof(float)];

namespace hmmgpu {

hipError_t static_decode_scratch(float **ptr) {
  static std::mutex mu;
  static float *addr[256] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 256) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = (float *)p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

namespace {

constexpr float kNegInf = -__builtin_inff();
constexpr float kWinHi = 0x1p32f, kWinLo = 0x1p-32f;

// Lane l receives lane l-1's value; lane 0 receives `fill`.
__device__ __forceinline__ float lane_up_fill(float v, float fill) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, fill),
                                                               __builtin_bit_cast(int, v), 0x138, 0xf, 0xf, false));
}

__device__ __forceinline__ float wave_max_f(float v) {
  for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  return __builtin_bit_cast(float, uni(__builtin_bit_cast(int, v)));
}

__device__ __forceinline__ int wave_min_i32(int v) {
  for (int off = 32; off >= 1; off >>= 1) v = min(v, __shfl_xor(v, off));
  return uni(v);
}

__device__ __forceinline__ float readlane_f(float v, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}

// Memory written by other lanes of this wave becomes visible to its loads.
__device__ __forceinline__ void wave_fence() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup"); }

// The same with two sums and a maximum.
__device__ __forceinline__ void scan_sums_affine_max(float &s, float &t, float &a, const float (&ps)[6], float &m) {
#define HMM_STEP(P, CTRL)                                  \
  "v_add_f32_dpp %0, %0, %0 " CTRL "\n\t"                  \
  "v_fmac_f32_dpp %1, %1, %" #P " " CTRL "\n\t"            \
  "v_add_f32_dpp %2, %2, %2 " CTRL "\n\t"
#define HMM_MAX(CTRL) "v_max_f32_dpp %3, %3, %3 " CTRL "\n\t"
  asm volatile(
      "s_nop 1\n\t"
      HMM_STEP(4, "row_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1") HMM_MAX("row_shr:1 row_mask:0xf bank_mask:0xf")
      HMM_STEP(5, "row_shr:2 row_mask:0xf bank_mask:0xf bound_ctrl:1") HMM_MAX("row_shr:2 row_mask:0xf bank_mask:0xf")
      HMM_STEP(6, "row_shr:4 row_mask:0xf bank_mask:0xf bound_ctrl:1") HMM_MAX("row_shr:4 row_mask:0xf bank_mask:0xf")
      HMM_STEP(7, "row_shr:8 row_mask:0xf bank_mask:0xf bound_ctrl:1") HMM_MAX("row_shr:8 row_mask:0xf bank_mask:0xf")
      HMM_STEP(8, "row_bcast:15 row_mask:0xa bank_mask:0xf") HMM_MAX("row_bcast:15 row_mask:0xa bank_mask:0xf")
      HMM_STEP(9, "row_bcast:31 row_mask:0xc bank_mask:0xf") HMM_MAX("row_bcast:31 row_mask:0xc bank_mask:0xf")
      "s_nop 1"
      : "+v"(s), "+v"(a), "+v"(t), "+v"(m)
      : "v"(ps[0]), "v"(ps[1]), "v"(ps[2]), "v"(ps[3]), "v"(ps[4]), "v"(ps[5]));
#undef HMM_STEP
#undef HMM_MAX
}
// The P parts of affine_scan_fused for a lane's own P.
__device__ __forceinline__ void affine_steps(float p, float (&ps)[6]) {
  ps[0] = p;
  p = p * dpp_f<kRowShr1, 0xf>(p, 1.0f);
  ps[1] = p;
  p = p * dpp_f<kRowShr2, 0xf>(p, 1.0f);
  ps[2] = p;
  p = p * dpp_f<kRowShr4, 0xf>(p, 1.0f);
  ps[3] = p;
  p = p * dpp_f<kRowShr8, 0xf>(p, 1.0f);
  ps[4] = p;
  p = p * dpp_f<kRowBcast15, 0xa>(p, 1.0f);
  ps[5] = p;
}
// The same scan in max-plus form: maps x -> max(a, x + b), b in {0, -inf}.
__device__ __forceinline__ float maxplus_scan(float a, const float (&bs)[6]) {
  a = fmaxf(a, dpp_f<kRowShr1, 0xf>(a, kNegInf) + bs[0]);
  a = fmaxf(a, dpp_f<kRowShr2, 0xf>(a, kNegInf) + bs[1]);
  a = fmaxf(a, dpp_f<kRowShr4, 0xf>(a, kNegInf) + bs[2]);
  a = fmaxf(a, dpp_f<kRowShr8, 0xf>(a, kNegInf) + bs[3]);
  a = fmaxf(a, dpp_f<kRowBcast15, 0xa>(a, kNegInf) + bs[4]);
  a = fmaxf(a, dpp_f<kRowBcast31, 0xc>(a, kNegInf) + bs[5]);
  return a;
}
__device__ __forceinline__ void maxplus_steps(float b, float (&bs)[6]) {
  bs[0] = b;
  b = b + dpp_f<kRowShr1, 0xf>(b, 0.0f);
  bs[1] = b;
  b = b + dpp_f<kRowShr2, 0xf>(b, 0.0f);
  bs[2] = b;
  b = b + dpp_f<kRowShr4, 0xf>(b, 0.0f);
  bs[3] = b;
  b = b + dpp_f<kRowShr8, 0xf>(b, 0.0f);
  bs[4] = b;
  b = b + dpp_f<kRowBcast15, 0xa>(b, 0.0f);
  bs[5] = b;
}

// Gate of a transition in the alignment recurrence: 0 if allowed, -inf if
// its probability is zero.
__device__ __forceinline__ float gate(float p) { return p > 0.0f ? 0.0f : kNegInf; }

// What a wave publishes for a row, by row parity (no wave is two rows ahead of
// another, as every row has a barrier).
template <int W>
struct DecodeLds {
  float4 a[2][W], b[2][W];
  float v[W];
  int k[W];
  int slot;
};

// The barrier of a row: LDS writes before it are visible after it.  Global
// loads and stores stay in flight.
template <int W>
__device__ __forceinline__ void row_barrier() {
  if constexpr (W > 1) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  }
}

// Barrier after which the global writes of the team's waves are visible to it.
template <int W>
__device__ __forceinline__ void team_sync() {
  wave_fence();
  if constexpr (W > 1) __syncthreads();
}

constexpr int kDecThreads = 256;   // teams of one wave: threads per block

// Values computed from a table buffer are pinned before the buffer is loaded
// again: a use sunk below the load would need a copy of the loaded registers,
// and a copy waits for every load and store in flight.
template <int N>
__device__ __forceinline__ void pin(float (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; i++) asm volatile("" : "+v"(v[i]));
}

template <int QW, int W, bool GATED>
__global__ void __launch_bounds__(W == 1 ? kDecThreads : 64 * W)
    __attribute__((amdgpu_waves_per_eu(decode_waves_per_simd(QW, W, GATED), decode_waves_per_simd(QW, W, GATED))))
decode_kernel(DevProfile P, DevDb db, DevDecode d) {
  constexpr int Q = QW * W;
  constexpr int kRowF = 2 * Q * kWave;   // floats of one stored row
  constexpr int NB = (QW + 7) / 8;       // traceback dwords per lane per row
  constexpr int kCells = Q * kWave;
  __shared__ DecodeLds<W> sh;
  // Emissions: in LDS for teams of one wave (a block's four share the table);
  // from L2 for larger teams, of which LDS could hold the table of one or two.
  constexpr bool kEmitLds = W == 1;
  __shared__ float emit_lds[kEmitLds ? kAlpha * kRowF : 1];
  if constexpr (kEmitLds) {
    for (int i = threadIdx.x; i < kAlpha * kRowF / 4; i += blockDim.x)
      ((float4 *)emit_lds)[i] = ((const float4 *)P.d_emit)[i];
    __syncthreads();
  }
  const int lane = threadIdx.x & 63;
  const int vl = 63 - lane;
  const int w = W == 1 ? 0 : uni((int)(threadIdx.x >> 6));
  const int slot = W == 1 ? wave_id() : (int)blockIdx.x;
  if (slot >= d.nslots) return;
  const int maxL = db.max_len;
  float *post = d.scratch + (size_t)slot * d.slot_dw;
  float *spec = post + (size_t)maxL * kRowF;
  int32_t *regs = (int32_t *)(spec + (size_t)maxL * 8);
  uint32_t *tbv = (uint32_t *)(regs + (size_t)maxL * 4 + 8);
  const float entry_p = P.entry_p;
  // A phase's tables are read at its start, through lane and table offsets that
  // the compiler cannot see through: otherwise it keeps both phases' tables (or
  // their addresses) in registers across the targets.
  const float *trp = P.d_tr + w * (QW * kWave), *cst = P.d_const;
  unsigned fl = 0, bl = 0;   // this lane's column, forwards and backwards
  auto new_phase = [&]() {
    int sofs = 0;
    fl = (unsigned)lane;
    bl = (unsigned)vl;
    asm volatile("" : "+v"(fl), "+v"(bl), "+s"(sofs));
    trp = P.d_tr + w * (QW * kWave) + sofs;
    cst = P.d_const + sofs;
  };
  auto plane = [&](int k, int q, unsigned col) -> float { return (trp + (k * Q + q) * kWave)[col]; };
  // this wave's coefficient of what wave j publishes, in table t
  auto coef = [&](int t, int j) -> float { return cst[(t * kMaxDecWaves + w) * kMaxDecWaves + j]; };
  auto edge = [&](int k) -> float { return W > 1 ? cst[kDecEdge + w * 4 + k] : 0.0f; };

  const int count = uni(__atomic_load_n(&db.counters[CNT_DEC], __ATOMIC_RELAXED));
  const WorkQueue<W != 1> queue(db, WORK_DEC, count);
  auto next_item = [&]() -> int {
    if constexpr (W == 1)
      return queue.next();
    else
      return next_target(queue, &sh.slot);
  };
  for (int idx = queue.first(); idx < count; idx = next_item()) {
    const int t = uni(db.list_vit[idx]);
    const int L = uni(db.len[t]);
    const LenParams lp = db.lp[L];
    const float loop = lp.loop_p, move = lp.move_p;
    const uint8_t *x = db.res + db.start[t];
    const int c = uni(db.perm[t]);
    const int64_t co = db.coff[t];
    // residues 256 at a time (lane j holds dword j of block rblk)
    uint32_t rch = 0;
    int rblk = -1;
    auto res_at = [&](int r) -> int {
      const int blk = r >> 8;
      if (blk != rblk) {
        rblk = blk;
        rch = ((const uint32_t *)(x + (size_t)blk * 256))[lane];
        asm volatile("" : "+v"(rch));   // waited for here: at the use, every row would wait for all loads and stores
      }
      return (int)((((uint32_t)__builtin_amdgcn_readlane((int)rch, (r >> 2) & 63)) >> ((r & 3) * 8)) & 0xffu);
    };
    auto load_emit = [&](float(&e)[2 * QW], int a, unsigned col) {
      if constexpr (kEmitLds) {
        const float *er = emit_lds + a * kRowF + col;
#pragma unroll
        for (int q = 0; q < 2 * QW; q++) e[q] = er[q * kWave];
      } else {
        const float *er = P.d_emit + (size_t)a * kRowF + w * (QW * kWave);
#pragma unroll
        for (int q = 0; q < QW; q++) {
          e[q] = (er + q * kWave)[col];
          e[QW + q] = (er + (Q + q) * kWave)[col];
        }
      }
    };

    // ------------------------------------------------ 1. Forward, rows kept
    {
      new_phase();
      float ft[TR_N][QW], gx[QW], pre[QW], fc[QW], ps[6];
#pragma unroll
      for (int q = 0; q < QW; q++) {
#pragma unroll
        for (int k = 0; k < TR_N; k++) ft[k][q] = plane(k, q, fl);
        gx[q] = plane(DT_EXIT, q, fl);
        pre[q] = plane(DT_PRE, q, fl);
        if (W > 1) fc[q] = plane(DT_FC, q, fl);
      }
      // Waited for here: with these loads pending at the row loop's entry, its head
      // would wait for all loads and stores on every row.
#pragma unroll
      for (int k = 0; k < TR_N; k++) pin(ft[k]);
      pin(gx);
      pin(pre);
      if (W > 1) pin(fc);
      affine_steps(pre[QW - 1], ps);
      // transitions across the edges: out of the last cell (M->D, D->D; lane 63
      // publishes), into the first cell (lane 0 only)
      const float mdn = edge(0), ddn = edge(1);
      const float mm0 = lane == 0 ? ft[TR_MMIN][0] : 0.0f, im0 = lane == 0 ? ft[TR_IMIN][0] : 0.0f,
                  dm0 = lane == 0 ? ft[TR_DMIN][0] : 0.0f;
      float cF[W], cG[W];
#pragma unroll
      for (int j = 0; j < W; j++) {
        cF[j] = W > 1 ? coef(DC_F, j) : 0.0f;
        cG[j] = W > 1 ? coef(DC_FL, j) : 0.0f;
      }
      float M[QW], I[QW], D[QW];
#pragma unroll
      for (int q = 0; q < QW; q++) M[q] = I[q] = D[q] = 0.0f;
      float pM = 0.0f, pI = 0.0f, pD = 0.0f;   // left neighbour of the wave's first cell, previous row
      float N = 1.0f, B = move, J = 0.0f, C = 0.0f;
      int par = 0;
      auto row = [&](float(&em)[2 * QW], int r) {
        float sm0 = B * entry_p;
        const float bent = sm0;
        if constexpr (W > 1) sm0 = fmaf(pM, mm0, fmaf(pI, im0, fmaf(pD, dm0, sm0)));
        fmac_up3(sm0, D[QW - 1], ft[TR_DMIN][0], I[QW - 1], ft[TR_IMIN][0], M[QW - 1], ft[TR_MMIN][0]);
        float es = 0.0f;
#pragma unroll
        for (int q = QW - 1; q >= 0; q--) {
          const float sm =
              q ? fmaf(M[q - 1], ft[TR_MMIN][q], fmaf(I[q - 1], ft[TR_IMIN][q], fmaf(D[q - 1], ft[TR_DMIN][q], bent)))
                : sm0;
          const float si = fmaf(M[q], ft[TR_MI][q], I[q] * ft[TR_II][q]);
          M[q] = em[q] * sm;
          I[q] = em[QW + q] * si;
          es = fmaf(M[q], gx[q], es);
        }
        pin(M);
        pin(I);
        load_emit(em, res_at(min(r + 2, L - 1)), fl);   // unconditional: a merge of loaded values would wait for all loads
        // delete chain with nothing entering the wave
        D[0] = mul_up(M[QW - 1], ft[TR_MDIN][0]);
#pragma unroll
        for (int q = 1; q < QW; q++) D[q] = fmaf(M[q - 1], ft[TR_MDIN][q], D[q - 1] * ft[TR_DDIN][q]);
        float ca = D[QW - 1];
        scan_sum_affine(es, ca, ps);
        const float carry = lane_up_f(ca);
#pragma unroll
        for (int q = 0; q < QW; q++) D[q] = fmaf(carry, pre[q], D[q]);
        float E;
        if constexpr (W == 1) {
          E = readlane_f(es, 63);
        } else {
          if (lane == 63) {
            sh.a[par][w] = float4{es, fmaf(M[QW - 1], mdn, D[QW - 1] * ddn), M[QW - 1], I[QW - 1]};
            sh.b[par][w].x = D[QW - 1];
          }
          row_barrier<W>();
          const int nb = w > 0 ? w - 1 : 0;   // every transition into the first cell of wave 0 is 0
          float xw = 0.0f;
          E = 0.0f;
          pD = sh.b[par][nb].x;
#pragma unroll
          for (int j = 0; j < W; j++) {
            const float2 v = *(const float2 *)&sh.a[par][j];
            E += v.x;
            xw = fmaf(cF[j], v.y, xw);
            pD = fmaf(cG[j], v.y, pD);
          }
          pM = sh.a[par][nb].z;
          pI = sh.a[par][nb].w;
          par ^= 1;
#pragma unroll
          for (int q = 0; q < QW; q++) D[q] = fmaf(fc[q], xw, D[q]);
        }
        float Jl = J * loop, Cl = C * loop;
        J = fmaf(0.5f, E, Jl);
        C = fmaf(0.5f, E, Cl);
        N = N * loop;
        B = (N + J) * move;
        const float big = fmaxf(fmaxf(fmaxf(E, J), fmaxf(C, N)), B);
        if (any_lane(big > kWinHi || big < kWinLo)) {
          int ex;
          (void)frexpf(big, &ex);
          const float s = ldexpf(1.0f, -ex);
#pragma unroll
          for (int q = 0; q < QW; q++) {
            M[q] *= s;
            I[q] *= s;
            D[q] *= s;
          }
          pM *= s;
          pI *= s;
          pD *= s;
          J *= s;
          C *= s;
          N *= s;
          B *= s;
          E *= s;
          Jl *= s;
          Cl *= s;
        }
        float *pr = post + (size_t)r * kRowF + w * (QW * kWave);
#pragma unroll
        for (int q = 0; q < QW; q++) {
          (pr + q * kWave)[fl] = M[q];
          (pr + (Q + q) * kWave)[fl] = I[q];
        }
        if (w == 0 && lane == 0) *(float4 *)(spec + (size_t)r * 8) = float4{N, Jl, Cl, E};
      };
      float ea[2 * QW], eb[2 * QW];
      load_emit(ea, res_at(0), fl);
      load_emit(eb, res_at(min(1, L - 1)), fl);
      int r = 0;
      for (; r + 1 < L; r += 2) {
        row(ea, r);
        row(eb, r + 1);
      }
      if (r < L) row(ea, r);
    }
    team_sync<W>();

    // ------------------------------------------------ 2. Backward, posteriors, regions, alignments
    //
    // Iteration i computes Backward row i and its posteriors (up to their
    // normalisation), and the region rule and alignment of row r = i + 1.  A run
    // of rows with core >= rt2 is a candidate region, and inside it the
    // recurrence is the optimal-accuracy one written from the end of the
    // region (T(r) = sum_{j=r}^{e} (1 - core(j))):
    //   OM_k(r) = pM_k(r) + max{ T(r+1) [end], OM_{k+1}(r+1) [MM_k],
    //                            OI_k(r+1) [MI_k], OD_{k+1}(r) [MD_k] }
    //   OI_k(r) = pI_k(r) + max{ OM_{k+1}(r+1) [IM_k], OI_k(r+1) [II_k] }
    //   OD_k(r) = max{ OM_{k+1}(r+1) [DM_k], OD_{k+1}(r) [DD_k] }
    // (a transition of probability zero is not allowed; profiles without one,
    // past their last node, run the instance without these tests: GATED).  The
    // alignment starts at the match cell maximising OM_k(r) - T(r), and its
    // value is that maximum plus T(s).  When the run ends it is kept (it held
    // a residue with core >= rt1) or its residues get code 0.
    float sum_end = 0.0f;
    int nreg = 0;
    {
      new_phase();
      float mm[QW], im[QW], dm[QW], md[QW], dd[QW], mi[QW], ii[QW], gx[QW], suf[QW], bmd[QW], pad[QW], ps[6];
      float gsuf[QW], gc[QW], bs[6];
#pragma unroll
      for (int q = 0; q < QW; q++) {
        mm[q] = plane(DT_MMO, q, bl);
        im[q] = plane(DT_IMO, q, bl);
        dm[q] = plane(DT_DMO, q, bl);
        md[q] = plane(DT_MDO, q, bl);
        dd[q] = plane(DT_DDO, q, bl);
        mi[q] = plane(TR_MI, q, bl);
        ii[q] = plane(TR_II, q, bl);
        gx[q] = plane(DT_EXIT, q, bl);
        suf[q] = plane(DT_SUF, q, bl);
        bmd[q] = W > 1 ? plane(DT_BMD, q, bl) : 0.0f;
        pad[q] = plane(DT_PAD, q, bl);
        gsuf[q] = GATED ? plane(DT_GSUF, q, bl) : 0.0f;
        gc[q] = GATED && W > 1 ? plane(DT_GC, q, bl) : 0.0f;
      }
      pin(mm);
      pin(im);
      pin(dm);
      pin(md);
      pin(dd);
      pin(mi);
      pin(ii);
      pin(gx);
      pin(suf);
      if (W > 1) pin(bmd);
      pin(pad);
      if (GATED) pin(gsuf);
      if (GATED && W > 1) pin(gc);
      affine_steps(suf[0], ps);
      if constexpr (GATED) maxplus_steps(gsuf[0], bs);
      auto G = [&](float p) -> float { return GATED ? gate(p) : 0.0f; };
      // transitions across the edges: into this wave's first cell (M->., D->. of
      // the cell before; lane 63 publishes), out of its last cell (lane 0 only)
      const float edm = edge(2), edd = edge(3);
      const float mmB = lane == 0 ? mm[QW - 1] : 0.0f, imB = lane == 0 ? im[QW - 1] : 0.0f,
                  mdB = lane == 0 ? md[QW - 1] : 0.0f;
      float cB[W], cN[W], gB[W], gN[W];
#pragma unroll
      for (int j = 0; j < W; j++) {
        cB[j] = W > 1 ? coef(DC_B, j) : 0.0f;
        cN[j] = W > 1 ? coef(DC_BN, j) : 0.0f;
        gB[j] = W > 1 && GATED ? coef(DC_GB, j) : 0.0f;
        gN[j] = W > 1 && GATED ? coef(DC_GN, j) : 0.0f;
      }
      auto loadF = [&](float(&f)[2 * QW], float4 &sv, int i) {   // stored row i (1-based)
        const float *pr = post + (size_t)(i - 1) * kRowF + w * (QW * kWave);
#pragma unroll
        for (int q = 0; q < QW; q++) {
          f[q] = (pr + q * kWave)[bl];
          f[QW + q] = (pr + (Q + q) * kWave)[bl];
        }
        sv = *(const float4 *)(spec + (size_t)(i - 1) * 8);
      };
      float bM[QW], bI[QW];
      float bJ = 0.0f, bN = 0.0f, bC = 0.0f;
      float OM[QW], OI[QW];          // alignment row r + 1
      float pm[QW], pi[QW];          // posteriors of row r, not normalised
      float zrow = 0.0f, zcs = 0.0f, fe = 0.0f;   // row r: N, J, C part of Z; core part (lane 63: the wave's); E term
#pragma unroll
      for (int q = 0; q < QW; q++) {
        bM[q] = bI[q] = pm[q] = pi[q] = 0.0f;
        OM[q] = OI[q] = kNegInf;
      }
      int in_run = 0, run_e = 0, best_at = 0;
      float T = 0.0f, nexp = 0.0f, bestv = kNegInf, top = 0.0f;   // top: the run's largest core
      // core posterior and "no region" of the rows of a 64-row window (lane j: row
      // 64 k + j, 0-based), stored a window at a time
      float wcore = 0.0f;
      int wout = 0;
      auto flush = [&](int r0) {   // rows r0 .. of the window
        const int j = (r0 & ~63) + lane;
        if (j >= r0 && j < L) {
          if (d.pp) d.pp[co + j] = wcore;
          if (d.aln && wout) d.aln[co + j] = 0;
        }
      };
      int par = 0;
      // the run [s1, run_e] ends: a region, or residues of code 0
      auto close_run = [&](int s1) {
        const int e1 = run_e;
        if (any_lane(top >= d.rt1)) {
          float vmax = wave_max_f(bestv);
          auto key_of = [&]() {
            const int cell = (w * kWave + vl) * QW + (best_at & 63);
            return wave_min_i32(bestv == vmax ? ((best_at >> 6) - 1) * kCells + cell : INT_MAX);
          };
          int key;
          if constexpr (W == 1) {
            key = key_of();
          } else {
            __syncthreads();
            if (lane == 0) sh.v[w] = vmax;
            __syncthreads();
#pragma unroll
            for (int j = 0; j < W; j++) vmax = fmaxf(vmax, sh.v[j]);
            key = key_of();
            if (lane == 0) sh.k[w] = key;
            __syncthreads();
#pragma unroll
            for (int j = 0; j < W; j++) key = min(key, sh.k[j]);
            key = uni(key);
          }
          const int32_t score = __builtin_bit_cast(int32_t, vmax + T);
          const int32_t nx = __builtin_bit_cast(int32_t, nexp);
          if (w == 0 && lane < 6) {
            const int32_t v = lane == 0 ? s1 : lane == 1 ? e1 : lane == 2 ? key / kCells + 1
                            : lane == 3 ? key % kCells : lane == 4 ? score : nx;
            regs[nreg * 8 + lane] = v;
          }
          nreg++;
        } else if (d.aln && w == 0) {
          for (int j = s1 - 1 + lane; j <= e1 - 1; j += kWave) d.aln[co + j] = 0;
        }
        in_run = 0;
#pragma unroll
        for (int q = 0; q < QW; q++) OM[q] = OI[q] = kNegInf;
      };
      // iteration i; ec: emissions of residue i (0-based; x_{i+1}), fc, sv: kept row i
      auto step = [&](float(&ec)[2 * QW], float(&fc)[2 * QW], float4 &sv, int i) {
        const bool last = i == L;
        // ---- before the barrier: Backward row i
        float hl[QW], nI[QW], u[QW], wv[QW];
        float su = 0.0f, a0 = 0.0f;
#pragma unroll
        for (int q = 0; q < QW; q++) {
          u[q] = last ? 0.0f : ec[q] * bM[q];
          wv[q] = last ? 0.0f : ec[QW + q] * bI[q];
          su += u[q];
        }
        pin(u);
        pin(wv);
        load_emit(ec, res_at(max(i - 1, 0)), bl);   // for iteration i - 1 (unconditional, as in Forward)
        // delete chains with nothing entering the wave: Backward's of row i, and the
        // alignment's of row r = i + 1; with them the sums of su and of row r's
        // posteriors
        const float un0 = lane_up_f(u[0]);   // next cell of the lane's last cell (0 at the wave's edge)
        float dp[QW], od[QW];
#pragma unroll
        for (int q = QW - 1; q >= 0; q--) {
          const float un = q + 1 < QW ? u[q + 1] : un0;
          dp[q] = q + 1 < QW ? fmaf(dd[q], dp[q + 1], dm[q] * un) : dm[q] * un;
        }
        const float on_pre = lane_up_fill(OM[0], kNegInf);
#pragma unroll
        for (int q = QW - 1; q >= 0; q--) {
          const float fd = (q + 1 < QW ? OM[q + 1] : on_pre) + G(dm[q]);
          od[q] = q + 1 < QW ? fmaxf(fd, od[q + 1] + G(dd[q])) : fd;
        }
        float ca = dp[0], cm0 = od[0];
        scan_sums_affine_max(su, zcs, ca, ps, cm0);
        if constexpr (GATED) cm0 = maxplus_scan(od[0], bs);
        const float carry = lane_up_f(ca), dcar = lane_up_fill(cm0, kNegInf);
#pragma unroll
        for (int q = 0; q < QW; q++) dp[q] = fmaf(carry, suf[q], dp[q]);
        a0 = dp[0];
#pragma unroll
        for (int q = 0; q < QW; q++) {
          const float un = q + 1 < QW ? u[q + 1] : un0;
          const float dn = q + 1 < QW ? dp[q + 1] : carry;
          hl[q] = fmaf(mm[q], un, fmaf(mi[q], wv[q], md[q] * dn));
          nI[q] = fmaf(im[q], un, ii[q] * wv[q]);
        }
#pragma unroll
        for (int q = 0; q < QW; q++) od[q] = fmaxf(od[q], dcar + gsuf[q]);
        // ---- exchange
        float sall, zc, xw = 0.0f, uN = 0.0f, aN = 0.0f, xo = kNegInf, oN = kNegInf, odN = kNegInf;
        if constexpr (W == 1) {
          sall = readlane_f(su, 63);
          zc = readlane_f(zcs, 63);
        } else {
          if (lane == 63) {
            sh.a[par][w] = float4{su, fmaf(edm, u[0], edd * a0), zcs, fmaxf(OM[0] + G(edm), od[0] + G(edd))};
            sh.b[par][w] = float4{u[0], a0, OM[0], od[0]};
          }
          row_barrier<W>();
          const float4 nb = sh.b[par][w + 1 < W ? w + 1 : w];   // every transition out of the last wave's last cell is 0
          uN = nb.x;
          aN = nb.y;
          oN = w + 1 < W ? nb.z : kNegInf;
          odN = w + 1 < W ? nb.w : kNegInf;
          sall = zc = 0.0f;
#pragma unroll
          for (int j = 0; j < W; j++) {
            const float4 v = sh.a[par][j];
            sall += v.x;
            zc += v.z;
            xw = fmaf(cB[j], v.y, xw);
            aN = fmaf(cN[j], v.y, aN);
            xo = fmaxf(xo, GATED ? v.w + gB[j] : j > w ? v.w : kNegInf);
            odN = fmaxf(odN, GATED ? v.w + gN[j] : j > w + 1 ? v.w : kNegInf);
          }
          par ^= 1;
        }
        // ---- region rule and alignment of row r
        const int r = i + 1;
        bool inside = false;
        float core = 0.0f, inv = 0.0f;
        if (r <= L) {
          const float Z = zrow + zc;
          inv = __builtin_amdgcn_rcpf(Z);
          inv = fmaf(fmaf(-Z, inv, 1.0f), inv, inv);
          core = zc * inv;
          const float pend = fe * inv;
          sum_end += pend;
          inside = any_lane(core >= d.rt2);
          if (inside) {
            if (!in_run) {
              in_run = 1;
              run_e = r;
              top = 0.0f;
              T = 0.0f;
              nexp = 0.0f;
              bestv = kNegInf;
            }
            top = fmaxf(top, core);
            nexp += pend;
            const float Tn = T;
            T = Tn + (1.0f - core);
            if constexpr (W > 1) {
#pragma unroll
              for (int q = 0; q < QW; q++) od[q] = fmaxf(od[q], xo + gc[q]);
            }
            const float on0 = lane_up_fill(OM[0], oN), odn0 = lane_up_fill(od[0], odN);
            uint32_t tw[NB];
#pragma unroll
            for (int j = 0; j < NB; j++) tw[j] = 0;
            float rv = kNegInf;
            int rq = 0;
#pragma unroll
            for (int q = 0; q < QW; q++) {
              const float on = q + 1 < QW ? OM[q + 1] : on0;   // OM and OD of the next cell
              const float odn = q + 1 < QW ? od[q + 1] : odn0;
              const float cm = on + G(mm[q]), ci = OI[q] + G(mi[q]), cd = odn + G(md[q]);
              float best = Tn;
              uint32_t sel = 0;
              if (cm > best) { best = cm; sel = 1; }
              if (ci > best) { best = ci; sel = 2; }
              if (cd > best) { best = cd; sel = 3; }
              const float nm = fmaf(pm[q], inv, best) + pad[q];
              const float oi = OI[q] + G(ii[q]), oim = on + G(im[q]);
              const float ni = fmaf(pi[q], inv, fmaxf(oim, oi));
              const float odd = odn + G(dd[q]), odm = on + G(dm[q]);
              tw[q >> 3] |= (sel | (oi > oim ? 4u : 0u) | (odd > odm ? 8u : 0u)) << ((q & 7) * 4);
              OM[q] = nm;
              OI[q] = ni;
              if (nm > rv) { rv = nm; rq = q; }
            }
            if (rv - T > bestv) {
              bestv = rv - T;
              best_at = (r << 6) | rq;
            }
            uint32_t *tr = tbv + ((size_t)(r - 1) * W + w) * (NB * kWave);
#pragma unroll
            for (int j = 0; j < NB; j++) (tr + j * kWave)[63 - bl] = tw[j];
          }
        }
        if (!inside) {
          if (in_run) close_run(r + 1);
        }
        if (w == 0 && r <= L) {
          const bool mine = lane == ((r - 1) & 63);
          wcore = mine ? core : wcore;
          wout = mine ? !inside : wout;
          if (((r - 1) & 63) == 0) flush(r - 1);
        }
        // ---- Backward row i, finished (i = 0: values that nothing uses)
        const float bB = entry_p * sall;
        bJ = fmaf(loop, bJ, move * bB);
        bN = fmaf(loop, bN, move * bB);
        bC = last ? move : loop * bC;
        const float bE = 0.5f * (bC + bJ);
#pragma unroll
        for (int q = 0; q < QW; q++) {
          bM[q] = fmaf(bE, gx[q], W > 1 ? fmaf(xw, bmd[q], hl[q]) : hl[q]);
          bI[q] = nI[q];
        }
        if constexpr (W > 1) {
          bM[QW - 1] = fmaf(mmB, uN, fmaf(mdB, aN, bM[QW - 1]));
          bI[QW - 1] = fmaf(imB, uN, bI[QW - 1]);
        }
        // posteriors of row i, and the parts of its total
        float z = 0.0f;
#pragma unroll
        for (int q = 0; q < QW; q++) {
          pm[q] = fc[q] * bM[q];
          pi[q] = fc[QW + q] * bI[q];
          z += pm[q] + pi[q];
        }
        zcs = z;   // summed over the wave with the next row's scans
        zrow = fmaf(sv.x, bN, fmaf(sv.y, bJ, sv.z * bC));
        fe = sv.w * bE;
        pin(pm);
        pin(pi);
        asm volatile("" : "+v"(zrow), "+v"(fe), "+v"(zcs));
        loadF(fc, sv, max(i - 2, 1));   // for iteration i - 2
        // rescale the values carried to the next row
        const float big = fmaxf(fmaxf(fmaxf(bB, bJ), fmaxf(bN, bC)), bE);
        if (any_lane(big > kWinHi || big < kWinLo)) {
          int ex;
          (void)frexpf(big, &ex);
          const float sc = ldexpf(1.0f, -ex);
#pragma unroll
          for (int q = 0; q < QW; q++) {
            bM[q] *= sc;
            bI[q] *= sc;
          }
          bJ *= sc;
          bN *= sc;
          bC *= sc;
        }
      };
      // kept rows are read two rows ahead, emissions one
      float em[2 * QW], fa[2 * QW], fb[2 * QW];
      float4 sa, sb;
#pragma unroll
      for (int q = 0; q < 2 * QW; q++) em[q] = 0.0f;   // row L uses no emissions
      loadF(fa, sa, L);
      loadF(fb, sb, max(L - 1, 1));
      int i = L;
      for (; i >= 1; i -= 2) {
        step(em, fa, sa, i);
        step(em, fb, sb, i - 1);
      }
      if (i == 0) step(em, fa, sa, 0);
      if (in_run) close_run(1);
    }
    if (d.exp_dom && w == 0 && lane == 0) d.exp_dom[c] = sum_end;
    team_sync<W>();

    // ------------------------------------------------ 3. Tracebacks of the regions
    for (int rg = w; rg < nreg; rg += W) {
      const int32_t rv = regs[rg * 8 + (lane & 7)];
      const int s1 = __builtin_amdgcn_readlane(rv, 0), e1 = __builtin_amdgcn_readlane(rv, 1);
      const int si = __builtin_amdgcn_readlane(rv, 2), sc = __builtin_amdgcn_readlane(rv, 3);
      const int32_t score = __builtin_amdgcn_readlane(rv, 4), nx = __builtin_amdgcn_readlane(rv, 5);
      // traceback codes of one diagonal, 64 cells at a time: lane j holds the
      // code of (row i0 + j, cell c0 + j), and bit j of mrun says that a match
      // there goes on to the next match; a move off that diagonal reloads
      int i0 = -(1 << 30), c0 = 0;
      uint32_t codes = 0;
      uint64_t mrun = 0;
      auto seek = [&](int i, int cc) -> int {   // the place of (i, cc) on the diagonal held
        int j = i - i0;
        if (!(j >= 0 && j < kWave && cc - c0 == j)) {
          i0 = i;
          c0 = cc;
          j = 0;
          const int il = min(i + lane, maxL);
          const int cl = min(cc + lane, kCells - 1);
          const int pl = cl / QW, ql = cl - pl * QW;   // virtual lane across the waves, vector
          const uint32_t wd = tbv[(((size_t)(il - 1) * W + (pl >> 6)) * NB + (ql >> 3)) * kWave + (63 - (pl & 63))];
          codes = (wd >> ((ql & 7) * 4)) & 0xfu;
          mrun = __builtin_amdgcn_ballot_w64((codes & 3u) == 1u);
        }
        return j;
      };
      // codes collected 64 residues at a time, stored a window at a time
      int cw = (s1 - 1) >> 6;
      int code = 0;
      auto flush = [&](int wnd) {
        const int j = wnd * 64 + lane;
        if (d.aln && j >= s1 - 1 && j <= e1 - 1) d.aln[co + j] = (int16_t)code;
        code = 0;
      };
      // residues r0 .. r0 + n - 1 (0-based): codes v, v + 1, ...
      auto put = [&](int r0, int v, int n) {
        while (n > 0) {
          while (cw < (r0 >> 6)) {
            flush(cw);
            cw++;
          }
          const int take = min(n, kWave - (r0 & 63)), k = lane - (r0 & 63);
          if (k >= 0 && k < take) code = v + k;
          r0 += take;
          v += take;
          n -= take;
        }
      };
      int i = si, cc = sc, st = 0;   // st: 0 = M, 2 = I, 3 = D
      int b1 = si, k2 = sc + 1;
      for (int guard = 0; guard <= (e1 - s1 + 1) + kCells; guard++) {
        if (i > e1 || cc >= P.M) break;
        const int j = seek(i, cc);
        if (st == 0) {   // a run of matches at once
          const uint64_t rest = ~(mrun >> j);
          const int run = min(min(rest ? (int)__builtin_ctzll(rest) : kWave, kWave - j), min(e1 - i, P.M - 1 - cc));
          if (run > 0) {
            put(i - 1, cc + 1, run);
            i += run;
            cc += run;
            continue;
          }
        }
        const uint32_t nib = (uint32_t)__builtin_amdgcn_readlane((int)codes, j);
        if (st == 0) {
          put(i - 1, cc + 1, 1);
          const uint32_t f = nib & 3u;
          if (f == 0) {
            b1 = i;
            k2 = cc + 1;
            break;
          }
          if (f != 3) i++;
          if (f != 2) cc++;
          st = f == 1 ? 0 : (int)f;
        } else if (st == 2) {
          put(i - 1, -(cc + 1), 1);
          if ((nib >> 2) & 1u) {
            i++;
          } else {
            i++;
            cc++;
            st = 0;
          }
        } else {
          if ((nib >> 3) & 1u) {
            cc++;
          } else {
            i++;
            cc++;
            st = 0;
          }
        }
      }
      while (cw <= ((e1 - 1) >> 6)) {
        flush(cw);
        cw++;
      }
      const int di = wave_fetch_add(&db.counters[CNT_NDOM], 1);
      if (di < d.max_dom && lane < 9) {
        const int32_t v = lane == 0 ? c : lane == 1 ? s1 : lane == 2 ? e1 : lane == 3 ? si : lane == 4 ? b1
                        : lane == 5 ? sc + 1 : lane == 6 ? k2 : lane == 7 ? score : nx;
        ((int32_t *)(d.dom + di))[lane] = v;
      }
    }
    team_sync<W>();
  }
}

// Counts of the decoded alignments, one wave per domain record: every
// aligned residue for its state and residue, every step between consecutive
// states for its transition (a match-to-match step that skips nodes goes
// through their delete states).  Integer atomics, so the counts are exact.
// Records and codes are checked against the database and the profile, so
// a mismatched buffer cannot send a write out of the count table.
__global__ void __launch_bounds__(256) count_kernel(DevDb db, int M, const hmm_domain *dom, const int32_t *n_dom,
                                                    int32_t max_dom, const int16_t *aln, uint32_t *counts) {
  const int lane = threadIdx.x & 63;
  const int nw = uni((int)gridDim.x * (int)(blockDim.x >> 6));
  const int n = min(uni(*n_dom), max_dom);
  uint32_t *cm = counts, *ci = counts + (size_t)M * kAlpha, *ct = ci + (size_t)(M - 1) * kAlpha;
  enum { MM = 0, MI, MD, IM, II, DM, DD };
  for (int r = wave_id(); r < n; r += nw) {
    const int c = uni(dom[r].target);
    if (c < 0 || c >= db.n) continue;
    const int t = uni(db.iperm[c]);
    const int L = uni(db.len[t]);
    const int a1 = max(uni(dom[r].a), 1), b1 = min(uni(dom[r].b), L);
    const uint8_t *x = db.res + db.start[t];
    const int16_t *cod = aln + db.coff[t];
    for (int j = a1 - 1 + lane; j <= b1 - 1; j += kWave) {
      const int k = cod[j];
      if (k > M || k < -(M - 1) || k == 0) continue;
      const int a = x[j];
      atomicAdd(k > 0 ? &cm[(k - 1) * kAlpha + a] : &ci[(-k - 1) * kAlpha + a], 1u);
      if (j >= b1 - 1) continue;
      const int k2 = cod[j + 1];
      if (k2 > M || k2 < -(M - 1) || k2 == 0) continue;
      if (k > 0 && k2 > 0) {
        if (k2 == k + 1) {
          atomicAdd(&ct[(k - 1) * 7 + MM], 1u);
        } else if (k2 > k + 1) {
          atomicAdd(&ct[(k - 1) * 7 + MD], 1u);
          for (int kk = k + 1; kk < k2 - 1; kk++) atomicAdd(&ct[(kk - 1) * 7 + DD], 1u);
          atomicAdd(&ct[(k2 - 2) * 7 + DM], 1u);
        }
      } else if (k > 0) {
        if (-k2 == k) atomicAdd(&ct[(k - 1) * 7 + MI], 1u);
      } else if (k2 < 0) {
        if (k2 == k) atomicAdd(&ct[(-k - 1) * 7 + II], 1u);
      } else if (k2 == -k + 1) {
        atomicAdd(&ct[(-k - 1) * 7 + IM], 1u);
      }
    }
  }
}

// Targets to decode: those whose caller flags hold every bit of the mask.
__global__ void decode_select(DevDb db, const uint8_t *flags, int mask) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= db.n) return;
  const bool take = !flags || (flags[db.perm[t]] & mask) == mask;
  if (take) db.list_vit[atomicAdd(&db.counters[CNT_DEC], 1)] = (int32_t)t;
}

__global__ void decode_clear(int32_t *c) {
  if (threadIdx.x == 0) {
    c[CNT_DEC] = 0;
    c[CNT_NDOM] = 0;
  }
  if (threadIdx.x < kWorkLanes) c[CNT_WORK + (WORK_DEC * kWorkLanes + threadIdx.x) * kWorkStride] = 0;
}

__global__ void decode_export(const int32_t *c, int32_t *n_dom) {
  if (threadIdx.x == 0) *n_dom = c[CNT_NDOM];
}

template <int QW, int W, bool GATED>
int decode_teams_q() {
  auto k = decode_kernel<QW, W, GATED>;
  constexpr int threads = W == 1 ? kDecThreads : 64 * W;
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k, threads, 0) != hipSuccess || nb < 1) nb = 1;
  int dev = 0, ncu = 0;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
  if (ncu <= 0) ncu = 256;
  return nb * ncu * (W == 1 ? kDecThreads / kWave : 1);
}

template <int QW, int W, bool GATED>
hipError_t launch_decode_q(const DevDb &db, const DevProfile &P, const DevDecode &d, hipStream_t s) {
  constexpr int threads = W == 1 ? kDecThreads : 64 * W;
  constexpr int teams = W == 1 ? kDecThreads / kWave : 1;   // per block
  const int blocks = (d.nslots + teams - 1) / teams;
  hipLaunchKernelGGL((decode_kernel<QW, W, GATED>), dim3((unsigned)blocks), dim3(threads), 0, s, P, db, d);
  return hipGetLastError();
}

#define HMM_DEC_CASES(X) \
  X(1, 1) X(2, 1) X(3, 1) X(4, 1) X(5, 1) X(3, 2) X(4, 2) X(5, 2) X(6, 2) X(4, 4) X(5, 4) X(6, 4) X(7, 4) X(8, 4) \
  X(10, 4) X(12, 4)

}  // namespace

int decode_max_teams(const DevProfile &p) {
#define HMM_CASE(qw, w) \
  if (p.dec_qw == qw && p.dec_w == w) return p.dec_gated ? decode_teams_q<qw, w, true>() : decode_teams_q<qw, w, false>();
  HMM_DEC_CASES(HMM_CASE)
#undef HMM_CASE
  return 0;
}

hipError_t launch_count(const DevProfile &p, const DevDb &db, const hmm_domain *dom, const int32_t *n_dom,
                        int32_t max_dom, const int16_t *aln, uint32_t *counts, hipStream_t s) {
  const int blocks = (int)std::min<int64_t>(((int64_t)max_dom + 3) / 4, 2048);
  hipLaunchKernelGGL(count_kernel, dim3((unsigned)std::max(blocks, 1)), dim3(256), 0, s, db, p.M, dom, n_dom, max_dom,
                     aln, counts);
  return hipGetLastError();
}

hipError_t launch_decode(const DevProfile &p, const DevDb &db, const DevDecode &d, hipStream_t s) {
  hipLaunchKernelGGL(decode_clear, dim3(1), dim3(64), 0, s, db.counters);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || db.n <= 0) {
    if (e == hipSuccess) {
      hipLaunchKernelGGL(decode_export, dim3(1), dim3(64), 0, s, (const int32_t *)db.counters, d.n_dom);
      e = hipGetLastError();
    }
    return e;
  }
  const int threads = 256;
  hipLaunchKernelGGL(decode_select, dim3((unsigned)((db.n + threads - 1) / threads)), dim3(threads), 0, s, db,
                     d.sel_flags, d.sel_mask);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = hipErrorInvalidValue;
#define HMM_CASE(qw, w)                  \
  if (p.dec_qw == qw && p.dec_w == w)    \
    e = p.dec_gated ? launch_decode_q<qw, w, true>(db, p, d, s) : launch_decode_q<qw, w, false>(db, p, d, s);
  HMM_DEC_CASES(HMM_CASE)
#undef HMM_CASE
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(decode_export, dim3(1), dim3(64), 0, s, (const int32_t *)db.counters, d.n_dom);
  return hipGetLastError();
}

}  // namespace hmmgpu

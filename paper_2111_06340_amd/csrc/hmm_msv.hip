// MSV stage (gfx950): every target of the database against one profile, or
// against a group of profiles of one kernel instance.  One wavefront scores
// one target; every wave-uniform quantity (target, length, residue, table
// offset) lives in scalar registers.
#include <hip/hip_runtime.h>

#include <climits>
#include <type_traits>

#include "hmm_device.h"
#include "hmm_internal.h"

namespace hmmgpu {
namespace {

// ============================================================================ MSV
//
// Per row i (residue a), with previous-row values v and xB (uint8 semantics,
// (+)/(-) saturating):
//   xBe = xB (-) ENTRY8;  v_k = (max(v_{k-1}, xBe) (+) BIAS8) (-) COST8_k(a)
//   xE = max v; overflow if xE >= 255 - BIAS8; xJ = max(xJ, xE (-) EXIT8);
//   xB = max(BASE8 (-) MOVE8, xJ (-) MOVE8)
//
// Exact reformulation in fp16: every quantity is an integer of magnitude at
// most 2048, held as that integer times 2^-11, so fp16 adds and maxima are
// exact.  Rows are only computed while every cell is below the overflow line
// 255 - BIAS8, so v_{k-1} (+) BIAS8 never saturates and only xBe can reach
// the 255 ceiling.  With E = BIAS8 - COST8 and Bx = min(xBe, 255 - BIAS8):
//   v_k = max(v_{k-1} + E, Bx + E, 0), or, for w = v - Bx,
//   w_k = max(w_{k-1} + E, E, -Bx).
// While Bx does not change, u = max(w, 0) obeys
//   u_k = max(u_{k-1} + E, 0)
// (Bx >= 0, so the -Bx floor drops out), and in these units, where 1.0 is
// 2048, that is ONE packed add with the instruction's clamp to [0, 1]: a row
// costs one VALU instruction per two cells, plus half of one for the running
// maximum (a 3-way maximum takes two vectors' or two rows' cells).
//
// Two passes per target.  The fast pass runs every row on u with the first
// row's Bx and no test; at the end one test of the running maximum decides.
// If some cell is positive and none reached T, the smallest value that could
// change xB or overflow, then xB never changed and the maximum gives the
// score.  Background targets reach T with probability about 2^-19 (T lies
// some 19 bits above the score distribution's location); homologs and other
// high scorers do, and run the exact pass on w from the first row, as do
// targets without a positive cell (their score lies below Bx: a few residues
// against a few nodes) and the degenerate Bx = 255 - BIAS8 (u cannot tell
// v = Bx, an overflow, from less).  Past T, u may lose fp16 exactness or
// saturate at 1.0, but rounding is monotone and T is far below 1.0, so the
// maximum still compares at or above T.
//
// Two layouts of the cells over the 64 lanes x 2 halves x Q vectors:
//  diagonal (M + 1 <= 128 Q, Q <= kMaxQDiag): MSV cells depend only on their
//    diagonal predecessor, so each of the P = 128 Q positions follows one
//    diagonal of the DP matrix: at row r position p holds cell (p + r) mod P,
//    and its predecessor is the same position's previous value.  No
//    cross-lane operation is needed.  State dword k holds the diagonals k and
//    k + P/2 and reads D[k + r mod P/2], D[c] = (E_c, E_{(c + P/2) mod P});
//    every P/2 rows the two halves of each state dword swap roles.  The
//    padding cell between cell M-1 and cell 0 (P >= M + 1) keeps diagonals
//    apart.
//    LDS reads: one dword per lane is read at 116 bytes per clock and CU,
//    two or four at 220 (measured; below 8-byte alignment 8 to 16), so
//    from kMinQWide vectors on, where the one-dword reads would take longer
//    than the row's arithmetic, a lane holds the state dwords 2 lane and
//    2 lane + 1 of each pair of vectors and reads both at once.  For odd r
//    their address is odd: a second copy of the table, one dword ahead,
//    keeps it aligned.
//  striped (larger M): slot 2*lane + half holds cells slot*Q + q; vector 0
//    takes vector Q-1 of the previous slot through one DPP lane shift and
//    one v_alignbit per row.  Tables are read four vectors at a time.
//
// Bound: VALU issue (an independent packed instruction takes 4.1 to 4.3 clocks
// of a SIMD).  Measured, a launch over the whole database, against the kernels
// before (three-way maximum with -Bx in every cell, dword reads, one work
// counter): M = 734 x 1,000,000 targets 10.4 -> 7.0 ms; M = 2,500 x 300,000 10.0
// -> 6.4 ms; M = 256 x 200,000 1.39 -> 0.92 ms; M = 300 x 50,000 0.74 -> 0.32 ms;
// groups x 200,000: two profiles of 300 nodes 2.3 -> 1.4 ms, four of 200 nodes
// 3.1 -> 1.8 ms, four of 100 nodes 2.0 -> 1.05 ms.
typedef _Float16 h16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ h16x2 as_h2(uint32_t v) { return __builtin_bit_cast(h16x2, v); }
__device__ __forceinline__ uint32_t as_u(h16x2 v) { return __builtin_bit_cast(uint32_t, v); }
// the score v in both halves
__device__ __forceinline__ h16x2 h2_splat(int v) {
  const _Float16 h = (_Float16)((float)v * 0x1p-11f);
  return h16x2{h, h};
}
__device__ __forceinline__ h16x2 h2_max(h16x2 a, h16x2 b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ h16x2 h2_max3(h16x2 a, h16x2 b, h16x2 c) { return h2_max(h2_max(a, b), c); }
// the larger half's score
__device__ __forceinline__ int h2_hmax(h16x2 v) { return (int)((float)__builtin_elementwise_maximum(v.x, v.y) * 2048.0f); }
// max(u + e, 0)
__device__ __forceinline__ h16x2 h2_step(h16x2 u, uint32_t e) {
  h16x2 r;
  asm("v_pk_add_f16 %0, %1, %2 clamp" : "=v"(r) : "v"(u), "v"(e));
  return r;
}

// ---------------------------------------------------------------- table reads
//
// The LDS tables of G profiles of one instance and a lane's reads of them.
// Dwords per residue, and how the entries of a row (diagonal offset r) are read:
//   diagonal, one profile, Q < kMinQWide: D, a dword at a time;
//   diagonal, one profile, Q >= kMinQWide: D, then D one dword ahead; pairs of
//     vectors together (an odd last vector alone);
//   diagonal, G = 2 or 4 profiles: the G profiles' D interleaved by dword, a
//     vector of all G profiles together (always aligned);
//   striped: quads of vectors together, then a pair, then one.
template <int Q, bool DIAG, int G>
struct MsvTab {
  static constexpr bool kWide = DIAG && G == 1 && msv_wide(Q);
  static constexpr int kRow = msv_row_dwords(Q, DIAG) * G;
  static constexpr int kBytes = kAlpha * kRow * 4;
  static constexpr int kHalf = Q * kWave;   // diagonal: rows of a phase (P/2)
  const char *lds;
  int lane;

  // Vector v = g Q + q (profile g) of residue a, K rows after diagonal
  // offset ofs (in bytes, ofs a multiple of 4 rows; 0 in the striped layout).
  template <int K>
  __device__ __forceinline__ void load(uint32_t (&c)[G * Q], int a, int ofs) const {
    const char *row = lds + (a * (kRow * 4) + ofs);
    if constexpr (!DIAG) {
      constexpr int q4 = Q / 4 * 4;
      const char *p4 = row + lane * 16;
#pragma unroll
      for (int q = 0; q < q4; q += 4) {
        const uint4 v = *(const uint4 *)(p4 + q * kWave * 4);
        c[q] = v.x;
        c[q + 1] = v.y;
        c[q + 2] = v.z;
        c[q + 3] = v.w;
      }
      if constexpr (Q - q4 >= 2) {
        const uint2 v = *(const uint2 *)(row + q4 * kWave * 4 + lane * 8);
        c[q4] = v.x;
        c[q4 + 1] = v.y;
      }
      if constexpr (Q % 2 == 1) c[Q - 1] = *(const uint32_t *)(row + (Q - 1) * kWave * 4 + lane * 4);
    } else if constexpr (G == 4) {
#pragma unroll
      for (int q = 0; q < Q; q++) {
        const uint4 v = *(const uint4 *)(row + lane * 16 + (q * kWave + K) * 16);
        c[q] = v.x;
        c[Q + q] = v.y;
        c[2 * Q + q] = v.z;
        c[3 * Q + q] = v.w;
      }
    } else if constexpr (G == 2) {
#pragma unroll
      for (int q = 0; q < Q; q++) {
        const uint2 v = *(const uint2 *)(row + lane * 8 + (q * kWave + K) * 8);
        c[q] = v.x;
        c[Q + q] = v.y;
      }
    } else if constexpr (kWide) {
      constexpr int kOdd = (K & 1) * 2 * kHalf * 4 + (K & ~1) * 4;   // the copy one dword ahead for odd rows
#pragma unroll
      for (int q = 0; q + 2 <= Q; q += 2) {
        const uint2 v = *(const uint2 *)(row + lane * 8 + q * kWave * 4 + kOdd);
        c[q] = v.x;
        c[q + 1] = v.y;
      }
      if constexpr (Q % 2 == 1) c[Q - 1] = *(const uint32_t *)(row + lane * 4 + ((Q - 1) * kWave + K) * 4);
    } else {
#pragma unroll
      for (int q = 0; q < Q; q++) c[q] = *(const uint32_t *)(row + lane * 4 + (q * kWave + K) * 4);
    }
  }

  // Diagonal: profile g's vectors alone, at any offset r in [0, P/2].
  __device__ __forceinline__ void load_one(uint32_t (&c)[Q], int a, int r, int g) const {
    const uint32_t *row = (const uint32_t *)lds + a * kRow;
#pragma unroll
    for (int q = 0; q < Q; q++) {
      const bool pair = kWide && (q < Q / 2 * 2);
      const int k = pair ? (q / 2) * 2 * kWave + 2 * lane + (q & 1) : q * kWave + lane;
      c[q] = row[(k + r) * G + g];
    }
  }
};

// ---------------------------------------------------------------- fast pass

// The maximum of v[0..N) in 3-way maxima ((N - 1) / 2 of them for odd N), as a
// tree, so that few of them wait on the one before.
template <int N>
__device__ __forceinline__ h16x2 h2_max_tree(const h16x2 (&v)[N]) {
  if constexpr (N == 1) {
    return v[0];
  } else if constexpr (N == 2) {
    return h2_max(v[0], v[1]);
  } else {
    constexpr int T = N / 3, C = N - 3 * T;
    h16x2 t[T + C];
#pragma unroll
    for (int i = 0; i < C; i++) t[T + i] = v[3 * T + i];
#pragma unroll
    for (int i = 0; i < T; i++) t[i] = h2_max3(v[3 * i], v[3 * i + 1], v[3 * i + 2]);
    return h2_max_tree<T + C>(t);
  }
}

// Every row of one target on u, against G profiles; acc[g] is the running
// maximum of profile g (in u).  Table entries are read R rows ahead, into two
// buffers in alternation; residues arrive 256 at a time (lane j holds dword j
// of the chunk) and are read a dword (four rows) ahead of the arithmetic.  A
// chunk that holds none of the target's rows is not fetched (its load re-reads
// the chunk before; residue codes past the target's end only select table rows
// that no row uses), so reads run at most 256 bytes past a target, inside the
// database's 1 KB zero tail.  The loops over dwords stop before the ones that
// start a chunk or a phase (state swap), so that their bodies are straight
// lines without register copies.
template <int Q, bool DIAG, int G, int R>
__device__ __forceinline__ void msv_fast(const MsvTab<Q, DIAG, G> &tab, const uint8_t *x, int L, int lane,
                                         h16x2 (&acc)[G]) {
  constexpr int V = G * Q;
  constexpr int kPhase = Q * kWave / 4;   // diagonal: dwords of residues per phase
  h16x2 u[V];
#pragma unroll
  for (int v = 0; v < V; v++) u[v] = h16x2{0, 0};
#pragma unroll
  for (int g = 0; g < G; g++) acc[g] = h16x2{0, 0};
  const uint32_t *p = (const uint32_t *)x;
  auto chunk = [&](int k, int own) { return p[(size_t)(256 * k < L ? k : own) * kWave + lane]; };
  uint32_t cur = chunk(0, 0), nxt = chunk(1, 0);
  auto code = [](uint32_t w, int r) { return (int)((w >> (8 * r)) & 0xffu); };
  auto advance = [&](const uint32_t(&c)[V]) {
    if constexpr (!DIAG) {
      const uint32_t sh = slot_up16(as_u(u[Q - 1]));
#pragma unroll
      for (int q = Q - 1; q >= 0; q--) u[q] = h2_step(q ? u[q - 1] : as_h2(sh), c[q]);
    } else {
#pragma unroll
      for (int v = 0; v < V; v++) u[v] = h2_step(u[v], c[v]);
    }
  };
  // one row, and two rows (whose cells enter the maximum together)
  auto row = [&](const uint32_t(&c)[V]) {
    advance(c);
#pragma unroll
    for (int g = 0; g < G; g++) {
      h16x2 m[Q + 1];
#pragma unroll
      for (int q = 0; q < Q; q++) m[q] = u[g * Q + q];
      m[Q] = acc[g];
      acc[g] = h2_max_tree(m);
    }
  };
  auto row2 = [&](const uint32_t(&c0)[V], const uint32_t(&c1)[V]) {
    advance(c0);
    h16x2 f[V];
#pragma unroll
    for (int v = 0; v < V; v++) f[v] = u[v];
    advance(c1);
#pragma unroll
    for (int g = 0; g < G; g++) {
      h16x2 m[2 * Q + 1];
#pragma unroll
      for (int q = 0; q < Q; q++) {
        m[q] = f[g * Q + q];
        m[Q + q] = u[g * Q + q];
      }
      m[2 * Q] = acc[g];
      acc[g] = h2_max_tree(m);
    }
  };
  int ofs = 0;                             // diagonal: table offset of the dword being read
  int wrap_at = DIAG ? kPhase : INT_MAX;   // dword that starts the next phase
  const int nd = L >> 2, rem = L & 3;
  uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)cur, 0);
  uint32_t ba[R][V], bb[R][V];
  // the first R rows of dword w, into `b`
  auto prime = [&](uint32_t(&b)[R][V]) {
    tab.template load<0>(b[0], code(w, 0), ofs);
    if constexpr (R >= 2) tab.template load<1>(b[1], code(w, 1), ofs);
    if constexpr (R == 4) {
      tab.template load<2>(b[2], code(w, 2), ofs);
      tab.template load<3>(b[3], code(w, 3), ofs);
    }
  };
  // w and ofs of dword i; EVENT: one that may start a chunk or a phase
  auto fetch = [&](int i, auto event) {
    constexpr bool EVENT = decltype(event)::value;
    if (EVENT && (i & 63) == 0) {
      cur = nxt;
      nxt = chunk((i >> 6) + 1, i >> 6);
    }
    w = (uint32_t)__builtin_amdgcn_readlane((int)cur, i & 63);
    if (DIAG) ofs = EVENT && i == wrap_at ? 0 : ofs + 16 * G;
  };
  // the rows of dword i, while entries further on are read
  auto dword = [&](uint32_t(&now)[R][V], uint32_t(&ahead)[R][V], int i, auto event) {
    if constexpr (R == 4) {
      fetch(i + 1, event);
      prime(ahead);
      __builtin_amdgcn_sched_barrier(0);
      row2(now[0], now[1]);
      row2(now[2], now[3]);
    } else if constexpr (R == 2) {
      tab.template load<2>(ahead[0], code(w, 2), ofs);
      tab.template load<3>(ahead[1], code(w, 3), ofs);
      __builtin_amdgcn_sched_barrier(0);
      row2(now[0], now[1]);
      fetch(i + 1, event);
      prime(now);
      __builtin_amdgcn_sched_barrier(0);
      row2(ahead[0], ahead[1]);
    } else {
      tab.template load<1>(ahead[0], code(w, 1), ofs);
      __builtin_amdgcn_sched_barrier(0);
      row(now[0]);
      tab.template load<2>(now[0], code(w, 2), ofs);
      __builtin_amdgcn_sched_barrier(0);
      row(ahead[0]);
      tab.template load<3>(ahead[0], code(w, 3), ofs);
      __builtin_amdgcn_sched_barrier(0);
      row(now[0]);
      fetch(i + 1, event);
      prime(now);
      __builtin_amdgcn_sched_barrier(0);
      row(ahead[0]);
    }
    if (decltype(event)::value && i + 1 == wrap_at) {   // the halves of each state dword swap diagonals
#pragma unroll
      for (int v = 0; v < V; v++) u[v] = as_h2(__builtin_amdgcn_alignbit(as_u(u[v]), as_u(u[v]), 16));
      wrap_at += kPhase;
    }
  };
  const auto plain = std::false_type{};
  const auto event = std::true_type{};
  // with four rows per buffer the buffers change places after every dword
  auto settle = [&]() {
    if constexpr (R == 4) {
#pragma unroll
      for (int r = 0; r < R; r++)
#pragma unroll
        for (int v = 0; v < V; v++) ba[r][v] = bb[r][v];
    }
  };
  prime(ba);
  for (int i = 0; i < nd;) {
    const int e = min(nd, min((i | 63) + 1, wrap_at) - 1);   // first dword whose successor may be an event
    if constexpr (R == 4) {
      for (; i + 1 < e; i += 2) {
        dword(ba, bb, i, plain);
        dword(bb, ba, i + 1, plain);
      }
      if (i < e) {
        dword(ba, bb, i++, plain);
        settle();
      }
    } else {
      for (; i < e; i++) dword(ba, bb, i, plain);
    }
    if (i < nd) {
      dword(ba, bb, i++, event);
      settle();
    }
  }
  // the last 0..3 rows
  if (rem > 0) row(ba[0]);
  if (rem > 1) {
    if constexpr (R == 1) tab.template load<1>(ba[0], code(w, 1), ofs);
    row(ba[R == 1 ? 0 : 1]);
  }
  if (rem > 2) {
    if constexpr (R < 4) tab.template load<2>(ba[0], code(w, 2), ofs);
    row(ba[R < 4 ? 0 : 2]);
  }
}

// ---------------------------------------------------------------- exact pass

struct MsvResult {
  int raw;
  bool ovf;
};

// One target against profile g of the tables, on w.  The rows test whether some
// cell has reached the trigger value T (the smallest that changes xB or
// overflows); the row that fired updates xJ and xB and re-bases w to the new Bx.
//  up to 12 vectors: rows run in batches of B, with one test after each; if it
//    finds such a cell the batch is run again from its first row, with a test
//    after every row.
//  above: a test after every row; no state is kept to run one again.  A long
//    profile's hits stay in this pass while the other targets' waves are done:
//    M = 1,900 x 50,000 targets, 0.4 % of them homologs, 1.61 ms (with a copy of
//    the state and dword reads 1.94; without homologs 1.04), M = 3,072 2.76 (3.25).
//    (At 9 vectors batches are faster: 30,000 targets of up to 5,000 residues by
//    1,025 nodes, a search 6.42 with them before, 6.37 now, row by row 6.5 ms.)
template <int Q, bool DIAG, int G>
__device__ __forceinline__ MsvResult msv_exact(const MsvTab<Q, DIAG, G> &tab, int g, const DevProfile &P,
                                               const uint8_t *x, int L, int mv, int lane) {
  auto splat = [](int v) -> uint32_t { return (uint32_t)uni((int)as_u(h2_splat(v))); };
  const int entry8 = P.entry8, exit8 = P.exit8;
  const int ovf_line = 255 - P.bias8;
  const int base = max(kBase8 - mv, 0);
  if (ovf_line <= 0) return MsvResult{255, true};
  int xJt = 0;
  int Bx = min(max(base - entry8, 0), ovf_line);
  uint32_t nbx = splat(-Bx);
  h16x2 acc = as_h2(nbx);
  h16x2 w[Q];
#pragma unroll
  for (int q = 0; q < Q; q++) w[q] = acc;
  // in w units: some cell has w > T - Bx - 1
  auto trigger_thr = [&]() { return splat(min(ovf_line, max(xJt, kBase8) + 4) - Bx - 1); };
  uint32_t thr = trigger_thr();
  auto fired = [&]() { return any_lane(as_u(h2_max(acc, as_h2(thr))) != thr); };
  auto row = [&](const uint32_t(&c)[Q]) {
    const uint32_t sh = DIAG ? 0u : slot_up16(as_u(w[Q - 1]));
#pragma unroll
    for (int q = Q - 1; q >= 0; q--)
      w[q] = h2_max3((DIAG ? w[q] : q ? w[q - 1] : as_h2(sh)) + as_h2(c[q]), as_h2(c[q]), as_h2(nbx));
    h16x2 m[Q + 1];
#pragma unroll
    for (int q = 0; q < Q; q++) m[q] = w[q];
    m[Q] = acc;
    acc = h2_max_tree(m);
  };
  // after a row that fired: false if it overflowed
  auto settle = [&]() -> bool {
    const int m = wave_max_i32(h2_hmax(acc)) + Bx;   // largest cell so far
    if (m >= ovf_line) return false;
    xJt = max(xJt, max(m - exit8, 0));
    const int nBx = min(max(max(base, max(xJt - mv, 0)) - entry8, 0), ovf_line);
    if (nBx != Bx) {   // re-base w and the running maximum to the new Bx
      const h16x2 d = as_h2(splat(Bx - nBx));
#pragma unroll
      for (int q = 0; q < Q; q++) w[q] += d;
      acc += d;
      Bx = nBx;
      nbx = splat(-Bx);
    }
    thr = trigger_thr();
    return true;
  };
  const uint32_t *p = (const uint32_t *)x;
  uint32_t cur = 0, wd = 0;
  constexpr int kHalf = Q * kWave;
  constexpr int B = Q <= 6 ? 4 : Q <= 12 ? 2 : 1;
  int dr = 0;   // row modulo P/2 (diagonal)
  for (int r = 0; r < L; r += B) {
    if ((r & 255) == 0) cur = p[(r >> 2) + lane];
    if ((r & 3) == 0) wd = (uint32_t)__builtin_amdgcn_readlane((int)cur, (r >> 2) & 63);
    uint32_t c[B][Q];
#pragma unroll
    for (int k = 0; k < B; k++) {
      if constexpr (DIAG)
        tab.load_one(c[k], (int)(wd & 0xffu), dr + k, g);
      else
        tab.template load<0>(c[k], (int)(wd & 0xffu), 0);
      wd >>= 8;
    }
    if constexpr (B == 1) {
      row(c[0]);
      if (__builtin_expect(fired(), 0) && !settle()) return MsvResult{255, true};
    } else {
      const h16x2 acc0 = acc;
      h16x2 w0[Q];
#pragma unroll
      for (int q = 0; q < Q; q++) w0[q] = w[q];
      const int rows = min(B, L - r);
      if (rows == B) {
#pragma unroll
        for (int k = 0; k < B; k++) row(c[k]);
      }
      if (rows < B || __builtin_expect(fired(), 0)) {
#pragma unroll
        for (int q = 0; q < Q; q++) w[q] = w0[q];
        acc = acc0;
#pragma unroll
        for (int k = 0; k < B; k++) {
          if (k < rows) {
            row(c[k]);
            if (fired() && !settle()) return MsvResult{255, true};
          }
        }
      }
    }
    if constexpr (DIAG) {
      dr += B;
      if (dr == kHalf) {   // the halves of each state dword swap diagonals
        dr = 0;
#pragma unroll
        for (int q = 0; q < Q; q++) w[q] = as_h2(__builtin_amdgcn_alignbit(as_u(w[q]), as_u(w[q]), 16));
      }
    }
  }
  const int m = wave_max_i32(h2_hmax(acc)) + Bx;
  return MsvResult{max(max(m - exit8, 0) - mv, 0), false};
}

// ---------------------------------------------------------------- kernel

// Runs of consecutive (sorted) targets for the MSV waves (WorkQueue), so that
// waves slowed by other kernels on their CU, or by longer targets, take fewer.
// A run is 8 targets, or fewer where the waves would otherwise get fewer than
// 4 runs each.
constexpr int kMsvRun = 8;

template <int G>
struct MsvGroup {
  DevProfile P[G];
  DevDb db[G];
  DevOut out[G];
};

// Waves per SIMD: two blocks per CU where two tables fit in LDS and 64
// registers hold a lane's state.
template <int Q, bool DIAG, int G>
constexpr int kMsvWaves = MsvTab<Q, DIAG, G>::kBytes <= 80 * 1024 && G * Q <= 12 ? 8 : 4;
// Rows per table buffer.
template <int Q, bool DIAG, int G>
constexpr int kMsvRows = G * Q <= 3 ? 4 : G * Q <= (kMsvWaves<Q, DIAG, G> == 8 ? 6 : 12) ? 2 : 1;

// Searches of one database by ng <= G profiles of one instance (G = 1: a
// single search): a wave scores a target against all of them, so that the
// residue stream, its scalar handling and the reads' addresses are shared.
// Each profile keeps its own state, outputs and survivor list; tables of
// absent profiles (g >= ng) hold padding cells only.
template <int Q, bool DIAG, int G>
__global__ void __launch_bounds__(1024)
    __attribute__((amdgpu_waves_per_eu(kMsvWaves<Q, DIAG, G>, kMsvWaves<Q, DIAG, G>)))
msv_kernel(MsvGroup<G> A, int ng) {
  using Tab = MsvTab<Q, DIAG, G>;
  extern __shared__ uint32_t lds[];
  if constexpr (G == 1) {
    const uint4 *src = (const uint4 *)A.P[0].msv;
    for (int i = threadIdx.x; i < kAlpha * Tab::kRow / 4; i += blockDim.x) ((uint4 *)lds)[i] = src[i];
  } else {
    for (int g = 0; g < G; g++) {
      const uint32_t *src = A.P[g < ng ? g : 0].msv;
      for (int i = threadIdx.x; i < kAlpha * Tab::kRow / G; i += blockDim.x)
        lds[i * G + g] = g < ng ? src[i] : kMsvPad2;
    }
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const Tab tab{(const char *)lds, lane};
  const DevDb &D0 = A.db[0];
  const int n = (int)D0.n;
  // The next target's length and start are read during the current target's
  // epilogue, so a target starts with one round trip (its length parameters
  // and first residue chunks, in parallel) instead of three.  The work
  // counters are the first profile's.
  const int nw = num_waves();
  const int run = max(1, min(kMsvRun, n / (4 * nw)));
  const WorkQueue<> runs(D0, WORK_MSV, (n + run - 1) / run);
  int t = runs.first() * run;
  int tend = min(t + run, n);
  int Lnext = 0;
  int64_t snext = 0;
  if (t < n) {
    Lnext = uni(D0.len[t]);
    snext = D0.start[t];
  }
  while (t < n) {
    const int L = Lnext;
    const uint8_t *x = D0.res + snext;
    if (D0.prio_by_len) length_priority(L, D0.max_len);
    const bool run_ends = t + 1 >= tend;
    const int asked = run_ends ? runs.ask() : 0;
    h16x2 acc[G];
    msv_fast<Q, DIAG, G, kMsvRows<Q, DIAG, G>>(tab, x, L, lane, acc);
    int raw[G];
    unsigned redo = 0;   // profiles that need the exact pass
#pragma unroll
    for (int g = 0; g < G; g++) {
      const DevProfile &P = A.P[g];
      const int mv = A.db[g].lp[L].move8;
      const int ovf_line = 255 - P.bias8;
      const int Bx = min(max(max(kBase8 - mv, 0) - P.entry8, 0), max(ovf_line, 0));
      const int m = wave_max_i32(h2_hmax(acc[g]));   // u units
      if ((m <= 0 || m + Bx >= min(ovf_line, kBase8 + 4)) && g < ng) redo |= 1u << g;
      raw[g] = max(max(m + Bx - P.exit8, 0) - mv, 0);
    }
    int tn = t + 1;
    if (run_ends) {
      tn = runs.item(asked) * run;
      tend = min(tn + run, n);
    }
    if (tn < n) {
      Lnext = uni(D0.len[tn]);
      snext = D0.start[tn];
    }
    // sorted order: neighbouring waves score neighbouring targets, so these
    // stores fill whole cache lines; results_kernel writes the caller's order
    auto emit = [&](int g, int r, bool ovf) {
      const DevDb &db = A.db[g];
      const bool pass = ovf || r >= db.lp[L].thr8;
      db.flags_sorted[t] = (uint8_t)((pass ? HMM_MSV_PASS : 0) | (ovf ? HMM_MSV_OVF : 0));
      db.msv_sorted[t] = (int16_t)r;
      // with the composition-bias filter on, MSV passes go to the filter's
      // list (the overflow list, unused until Viterbi) instead of Viterbi's
      if (pass) {
        const bool bf = A.out[g].bias_filter != 0;
        (bf ? db.list_ovf : db.list_vit)[wave_fetch_add(&db.counters[bf ? CNT_OVF : CNT_VIT], 1)] = t;
      }
    };
#pragma unroll
    for (int g = 0; g < G; g++)
      if (g < ng && !((redo >> g) & 1u)) emit(g, raw[g], false);
    while (__builtin_expect(redo != 0, 0)) {
      const int g = G == 1 ? 0 : __builtin_ctz(redo);
      redo &= redo - 1;
      const MsvResult r = msv_exact<Q, DIAG, G>(tab, g, A.P[g], x, L, A.db[g].lp[L].move8, lane);
      emit(g, r.raw, r.ovf);
    }
    t = tn;
  }
}

// ---------------------------------------------------------------- launchers

int num_cu() {
  static int ncu = 0;
  if (!ncu) {
    int dev = 0, v = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev);
    ncu = v > 0 ? v : 256;
  }
  return ncu;
}

template <int Q, bool DIAG, int G>
hipError_t launch(const DevProfile *P, const DevDb *db, const DevOut *o, int ng, hipStream_t s) {
  MsvGroup<G> A;
  for (int g = 0; g < G; g++) {
    A.P[g] = P[g < ng ? g : 0];
    A.db[g] = db[g < ng ? g : 0];
    A.out[g] = o[g < ng ? g : 0];
  }
  constexpr int threads = 1024;
  constexpr size_t lds = MsvTab<Q, DIAG, G>::kBytes;
  auto k = msv_kernel<Q, DIAG, G>;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  static int bpc = 0;
  if (!bpc) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k, threads, lds) != hipSuccess || nb < 1) nb = 1;
    bpc = nb;
  }
  int64_t blocks = (int64_t)bpc * num_cu();
  const int64_t cap = (db[0].n + threads / 64 - 1) / (threads / 64);
  if (blocks > cap) blocks = cap;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(threads), lds, s, A, ng);
  return hipGetLastError();
}

#define HMM_MSV_DIAG_CASES(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8)
#define HMM_MSV_STRIPED_CASES(X) X(8) X(9) X(10) X(11) X(12) X(14) X(16) X(18) X(20) X(22) X(24)

}  // namespace

int msv_group_max(const DevProfile &P) {
  if (!P.msv_diag) return 1;
  return P.Qm <= 2 ? 4 : P.Qm <= 4 ? 2 : 1;
}

hipError_t launch_msv(const DevProfile *P, const DevDb *db, const DevOut *o, int ng, hipStream_t s) {
  const int Q = P[0].Qm;
  if (ng > 1) {
#define HMM_GROUP(q, g) \
  if (P[0].msv_diag && Q == q && ng <= g) return launch<q, true, g>(P, db, o, ng, s);
    HMM_GROUP(1, 2) HMM_GROUP(1, 4) HMM_GROUP(2, 2) HMM_GROUP(2, 4) HMM_GROUP(3, 2) HMM_GROUP(4, 2)
#undef HMM_GROUP
    return hipErrorInvalidValue;
  }
  if (P[0].msv_diag) {
    switch (Q) {
#define HMM_CASE(q) \
  case q:           \
    return launch<q, true, 1>(P, db, o, 1, s);
      HMM_MSV_DIAG_CASES(HMM_CASE)
#undef HMM_CASE
    }
  } else {
    switch (Q) {
#define HMM_CASE(q) \
  case q:           \
    return launch<q, false, 1>(P, db, o, 1, s);
      HMM_MSV_STRIPED_CASES(HMM_CASE)
#undef HMM_CASE
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace hmmgpu

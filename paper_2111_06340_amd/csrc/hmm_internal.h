// Internal declarations shared by the host side (hmm_host.cpp) and the
// kernels (the .hip files) of the GPU library.  Not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hmmgpu.h"

namespace hmmgpu {

constexpr int kWave = 64;           // CDNA wavefront
constexpr int kAlpha = 20;          // residue alphabet
constexpr int kBase8 = 190;         // MSV offset of the N/J start
constexpr int kNeg16 = -32768;      // int16 "minus infinity"
constexpr int32_t kNeg32 = -(1 << 30);  // int32 rescore floor
constexpr int kMaxQ8 = 24;          // 128 cells per packed vector -> M <= 3072
constexpr int kMaxQDiag = 8;        // largest MSV diagonal-layout instance (LDS 20 KB per vector)
constexpr int kMaxMsvGroup = 4;     // most profiles of one MSV launch
constexpr int kMaxQ32 = 48;         // 64 cells per 32-bit vector -> M <= 3072

// Transition planes of the per-cell "into" layout (cell k = node k+1).
//   MMIN/IMIN/DMIN: M_k, I_k, D_k (node k) -> M_{k+1};  MDIN/DDIN: M_k, D_k
//   -> D_{k+1};  MI/II: M_{k+1}/I_{k+1} -> I_{k+1}.  Structural and padding
//   cells hold the type's minus infinity (probability 0 in Forward).
enum { TR_MMIN = 0, TR_IMIN, TR_DMIN, TR_MDIN, TR_DDIN, TR_MI, TR_II, TR_N };

// Per-target-length parameters, one entry per L = 0..max_len.
struct LenParams {
  int32_t move8;    // MSV cost of N->B / J->B / C->T
  int32_t thr8;     // MSV pass: msv_raw >= thr8 (0..256)
  int32_t move16;   // Viterbi score of the moves (<= 0)
  int32_t thr16;    // Viterbi pass: vit >= thr16
  float loop_p;     // Forward N/C/J self-loop probability L/(L+3)
  float move_p;     // Forward move probability 3/(L+3)
  float fthr;       // Forward pass: fwd > fthr (nats); -inf when F3 >= 1
  float pad;
};

// Device-side profile, passed to kernels by value.
struct DevProfile {
  int32_t M, Q8, Q32;
  int32_t Qm;                   // vectors per lane of the MSV kernel
  int32_t msv_diag;             // MSV layout: 1 diagonal, 0 striped (see msv below)
  int32_t bias8, entry8, exit8;
  int32_t entry16, ej16;
  // Largest D->M transition score over the nodes (int16 and int32 scales;
  // minus infinity when M = 1): a delete value d with d + dm_max <= the
  // B->M entry value can no longer change any match cell.
  int32_t dm_max16, dm_max32;
  // Re-basing of the int16 Viterbi: the largest emission score, and W (the least
  // distance of xBe from the int16 floor; so large that no target qualifies
  // where the emission scores leave no room).
  int32_t s_max, rebase_w;
  float entry_p;                // 2/(M(M+1))
  float bias_r[kAlpha];         // composition-bias filter: mean match emission / background
  // MSV table, packed fp16 scores E = BIAS8 - COST8 times 2^-11 (padding
  // cells -1), msv_row_dwords per residue.
  // msv_diag = 1: [20][P], P = 128 Qm, dword c = (E_c, E_{(c + P/2) mod P});
  // from kMinQWide vectors on [20][2][P], the second row one dword ahead;
  // msv_diag = 0: the striped packed layout at msv_stripe_dword.
  const uint32_t *msv;
  const uint32_t *vit_emit;     // [20][2][Q8][64] packed i16: msc plane, isc plane
  const uint32_t *vit_tr;       // [TR_N][Q8][64] packed i16
  const int32_t *v32_emit;      // [20][2][Q32][64]
  const int32_t *v32_tr;        // [TR_N][Q32][64]
  const float *f_emit;          // [20][2][Q32][64] odds e/f, i/f
  // [TR_N + 3][Q32][64]: probabilities; plane TR_PRE: D-chain products
  // prod_{j<=q} DDIN(lane*Q + j); plane TR_SUF: prod_{j=q+1}^{Q} DDIN(lane*Q + j)
  // (the last factor belongs to the next lane's first cell; 0 past the end);
  // plane TR_EXIT: exit weight g_c of cell c (see hmm_profile_upload), so
  // that a row's E = sum_c M_c g_c
  const float *f_tr;
  // Decoding: teams of dec_w waves, dec_qw cells per lane and wave; cell of plane
  // p (= wave * dec_qw + vector) and lane l: ((p / dec_qw) * 64 + l) * dec_qw + p % dec_qw.
  int32_t dec_qw, dec_w;
  int32_t dec_gated;            // 1: some transition inside the profile has probability 0
  const float *d_emit;          // [20][2][dec_w dec_qw][64] odds, as f_emit
  const float *d_tr;            // [DT_N][dec_w dec_qw][64]
  const float *d_const;         // [kDecConst]
};
enum { TR_PRE = TR_N, TR_SUF = TR_N + 1, TR_EXIT = TR_N + 2 };

// Planes of the decoding's transitions: 0 .. TR_N-1 as in TR_* ("into" form),
// then
//   DT_EXIT: exit weights; DT_PRE: prod_{j<=q} DDIN over the lane's cells;
//   DT_FC: the factor from the value entering the wave's first delete cell to
//     this delete cell;
//   DT_MMO .. DT_DDO: the transitions out of the cell's node into the next one;
//   DT_SUF: the factor from the next lane's first delete cell to this one in the
//     Backward direction; DT_BMD: M->D times the factor from the value entering
//     the wave's last delete cell to the next cell;
//   DT_GSUF, DT_GC: 0 where the factor of DT_SUF, resp. of the value entering the
//     wave's last delete cell, has no zero transition, else -inf;
//   DT_PAD: 0 for the profile's cells, -inf past them.
enum {
  DT_EXIT = TR_N, DT_PRE, DT_FC, DT_MMO, DT_IMO, DT_DMO, DT_MDO, DT_DDO, DT_SUF, DT_BMD, DT_GSUF, DT_GC, DT_PAD, DT_N
};
// Constant tables [DC_N][wave][published by wave j]: coefficients of what wave j
// passes on in wave w's entering value (DC_F, DC_B; max-plus DC_GB), in the last
// delete cell of wave w - 1 (DC_FL) and in the first of wave w + 1 (DC_BN, DC_GN).
// Then, per wave: M->D and D->D out of its last cell, D->M and D->D into its first.
constexpr int kMaxDecWaves = 4;
enum { DC_F = 0, DC_FL, DC_B, DC_BN, DC_GB, DC_GN, DC_N };
constexpr int kDecEdge = DC_N * kMaxDecWaves * kMaxDecWaves;
constexpr int kDecConst = kDecEdge + kMaxDecWaves * 4;
// Waves per SIMD of a decoding instance: as many as its registers allow.
constexpr int decode_waves_per_simd(int qw, int w, bool gated) {
  return qw == 1 ? 4 : qw == 2 ? 3 : qw <= (gated ? 4 : 6) ? 2 : 1;
}
// The decoding instance of a profile of q vectors per lane: the smallest that
// holds it.
inline bool decode_split(int q, int *qw, int *w) {
  static const int list[][2] = {{1, 1}, {2, 1}, {3, 1}, {4, 1}, {5, 1}, {3, 2}, {4, 2}, {5, 2}, {6, 2}, {4, 4},
                                {5, 4}, {6, 4}, {7, 4}, {8, 4}, {10, 4}, {12, 4}};
  for (const auto &e : list)
    if (e[0] * e[1] >= q) {
      *qw = e[0];
      *w = e[1];
      return true;
    }
  return false;
}

// Counters in the database scratch (device int32).
enum {
  CNT_VIT = 0, CNT_OVF, CNT_FWD, CNT_FWD_PASS,
  CNT_DEC, CNT_NDOM,   // posterior decoding: list size, domains found
  CNT_OVF_EXACT,       // int16 overflows scored exactly by re-basing (not in CNT_OVF)
  CNT_LISTS = 8,       // the counters above
  // work counters of the stages, kWorkLanes of them each, kWorkStride apart
  CNT_WORK = 32
};
// Stages that hand their targets out through work counters (WorkQueue).
enum { WORK_MSV = 0, WORK_BIAS, WORK_VIT, WORK_OVF, WORK_FWD, WORK_DEC, WORK_STAGES };
// One counter that every wave of the chip bumps is served at about 15 ns a bump
// (measured: 50,000 targets of 300 nodes taken one by one 0.74 ms, the work
// itself 0.2 ms), so each stage has one per XCD (blocks go round the 8 XCDs),
// in a cache line of its own.
constexpr int kWorkLanes = 8, kWorkStride = 32;
constexpr int CNT_N = CNT_WORK + WORK_STAGES * kWorkLanes * kWorkStride;

struct DevDb {
  int64_t n;
  int32_t max_len;
  const uint8_t *res;           // packed residues, each target 16-byte aligned
  const int64_t *start;         // [n] byte offset of each target (sorted order)
  const int32_t *len;           // [n]
  const int32_t *perm;          // [n] sorted index -> caller index
  uint8_t *flags_sorted;        // [n] scratch: every stage's flags, sorted order
  int16_t *msv_sorted;          // [n] scratch: MSV scores, sorted order
  int32_t *list_vit;            // [n] MSV survivors (sorted indices)
  int32_t *list_ovf;            // [n] int16 Viterbi overflows
  int32_t *list_fwd;            // [n] Viterbi survivors
  int32_t *counters;            // [CNT_N]
  const LenParams *lp;          // [max_len + 1]
  const int64_t *coff;          // [n] offset of each target in the caller's residue array
  const int32_t *iperm;         // [n] caller index -> sorted index
  int32_t prio_by_len;          // 1: the search stages' waves take issue priority by target length
};

struct DevOut {
  int16_t *msv;
  int32_t *vit;
  float *fwd;
  uint8_t *flags;
  int64_t *counts;
  float *bias;                  // optional bias scores
  int32_t bias_filter;          // 1: composition-bias filter between MSV and Viterbi
  int32_t fused_tail;           // 1: the stages after MSV as one kernel where an instance exists
  int32_t rescore_apart;        // 1: the int32 rescore and Forward beside each other
};

// Posterior decoding (hmm_decode): outputs and per-wave scratch.
struct DevDecode {
  hmm_domain *dom;              // [max_dom] domain records
  int32_t max_dom;
  int32_t *n_dom;               // device int32: domains found (may exceed max_dom)
  float *exp_dom;               // [n] caller order, or null
  float *pp;                    // [n_residues] caller layout, or null
  int16_t *aln;                 // [n_residues] caller layout, or null
  const uint8_t *sel_flags;     // [n] caller order; null = decode every target
  int32_t sel_mask;             // decode targets with (flags & mask) == mask
  float rt1, rt2;               // region thresholds on the core posterior
  float *scratch;               // nslots * slot_dw floats
  int64_t slot_dw;              // dwords per team slot
  int32_t nslots;               // teams of the decode launch (one slot each)
};

// Dwords of one decode slot for teams of w waves of qw cells per lane and
// targets up to max_len: kept Forward rows [max_len][2][w qw][64], their
// specials [max_len][8], regions [max_len / 2 + 1][8], traceback codes
// [max_len][w][ceil(qw/8)][64].
inline int64_t decode_slot_dw(int qw, int w, int max_len) {
  const int64_t nb = (qw + 7) / 8;
  const int64_t dw = (int64_t)max_len * (2 * qw * w * 64 + 8 + 4 + w * nb * 64) + 8;
  return (dw + 63) / 64 * 64;
}

// Largest number of teams of the decode kernel of profile p resident at once.
int decode_max_teams(const DevProfile &p);

// Enqueue the decode of the selected targets on `stream` (d.nslots teams).
hipError_t launch_decode(const DevProfile &p, const DevDb &db, const DevDecode &d, hipStream_t stream);

// Bytes of the decode scratch held in a file-scope device array, for the
// entry point that allocates nothing (hmm_decode_static).
constexpr size_t kStaticDecodeBytes = (size_t)512 << 20;

// Device address of that array on the current device: looked up once per
// device (hipGetSymbolAddress) and kept for the life of the process.
hipError_t static_decode_scratch(float **ptr);

// Forward and int32 rescore of long profiles with one workgroup of several
// waves per target (hmm_coop.hip): coop_instance(Q) tells whether vectors
// per lane Q have such an instance.
bool coop_instance(int Q);
hipError_t launch_fwd_coop(const DevProfile &p, const DevDb &db, const DevOut &o, hipStream_t stream);
hipError_t launch_vit32_coop(const DevProfile &p, const DevDb &db, const DevOut &o, hipStream_t stream);

// A search runs in up to kMaxChunks chunks of the length-sorted database
// (contiguous ranges of about equal residue counts), pipelined: the MSV
// kernels of the chunks run back to back on the search stream, and the rest
// of each chunk's cascade (Viterbi, the int32 rescore, Forward) on a second
// stream as soon as the chunk's MSV is done, so it overlaps the next chunk's
// MSV.  A search of one chunk needs no second stream.  Each chunk has its own
// counter block and keeps its survivor lists inside its own index range.
constexpr int kMaxChunks = 8;

// Streams and events that order one database handle's searches.
struct SearchSync {
  hipStream_t tail = nullptr;           // Viterbi and Forward of the chunks
  hipStream_t aux = nullptr;            // the int32 rescore beside Forward (rescore_apart), or
                                        // Forward beside the rescore (see launch_tail)
  hipEvent_t msv_done[kMaxChunks] = {}; // recorded on the search stream
  hipEvent_t vit_done[kMaxChunks] = {}; // recorded on tail
  hipEvent_t aux_done = nullptr, tail_done = nullptr;
};

// The sorted targets [a, b) as a database of their own, with counter block k.
inline DevDb chunk_of(const DevDb &d, int64_t a, int64_t b, int k) {
  DevDb c = d;
  c.n = b - a;
  c.start += a;
  c.len += a;
  c.perm += a;
  c.coff += a;
  c.flags_sorted += a;
  c.msv_sorted += a;
  c.list_vit += a;
  c.list_ovf += a;
  c.list_fwd += a;
  c.counters += (size_t)k * CNT_N;
  return c;
}

// Enqueue the whole cascade of the chunks chunk[0..nchunks) on `stream`;
// all of its work is joined back into `stream`.  The last kernel writes the
// results in caller order and the counts (the sum over the chunks' counter
// blocks, which start at chunk[0].counters).  When `ev` is non-null, ev[0..4]
// are recorded at the start, after the last MSV, after the last Viterbi, after
// the last rescore and at the end, each on the stream that ran it.
hipError_t launch_search(const DevProfile &p, const DevDb *chunk, int nchunks, const DevOut &out,
                         hipStream_t stream, const SearchSync &sync, hipEvent_t *ev);

// Enqueue a group of n one-chunk searches of one database (one handle each):
// MSV of profiles sharing a diagonal instance as group kernels, then each
// search's tail on its own streams y[i], joined back into `stream`.
hipError_t launch_search_group(const DevProfile *P, const DevDb *db, const DevOut *o, int n, hipStream_t stream,
                               const SearchSync *const *y);

// Enqueue the emission and transition counts of the alignments of
// dom[0 .. min(*n_dom, max_dom)) (codes in aln, caller residue layout) into
// counts: uint32 [M][20] match, [M-1][20] insert, [M-1][7] transitions.
hipError_t launch_count(const DevProfile &p, const DevDb &db, const hmm_domain *dom, const int32_t *n_dom,
                        int32_t max_dom, const int16_t *aln, uint32_t *counts, hipStream_t stream);

// The packed 16-bit VALU rate the device sustains (element-ops per second),
// measured by a timed kernel of independent add/maximum chains; scratch
// holds one word per thread of the launch (2 x CUs x 1024).
hipError_t probe_pk16(uint32_t *scratch, int64_t scratch_words, hipStream_t stream, double *ops_per_s,
                      float *ms);

// MSV tables.  Diagonal instances from kMinQWide vectors per lane on keep two
// copies of each residue's row.
constexpr int kMinQWide = 6;
constexpr bool msv_wide(int Q) { return Q >= kMinQWide; }
constexpr int msv_row_dwords(int Q, bool diag) { return Q * kWave * (diag ? (msv_wide(Q) ? 4 : 2) : 1); }
// Striped row: dword of vector q of a lane (vectors by fours, then two, then one).
constexpr int msv_stripe_dword(int Q, int q, int lane) {
  const int q4 = Q / 4 * 4, q2 = Q / 2 * 2;
  return q < q4 ? (q & ~3) * kWave + lane * 4 + (q & 3)
                : q < q2 ? q4 * kWave + lane * 2 + (q - q4) : q2 * kWave + lane;
}
constexpr uint32_t kMsvPad2 = 0xbc00bc00u;   // two padding cells

// Enqueue the MSV stage of ng searches of one database by profiles of one
// instance (ng at most msv_group_max of the profile).
int msv_group_max(const DevProfile &P);
hipError_t launch_msv(const DevProfile *P, const DevDb *db, const DevOut *o, int ng, hipStream_t s);

// Number of packed vectors per lane.
inline int q8_of(int M) { return (M + 2 * kWave - 1) / (2 * kWave); }
inline int q32_of(int M) { return (M + kWave - 1) / kWave; }

}  // namespace hmmgpu

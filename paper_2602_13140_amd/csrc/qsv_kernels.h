// Internal launch interface between the C-ABI layer and the HIP kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "qsv_plan.h"

#ifdef __HIPCC__
#define QSV_HD __host__ __device__
#else
#define QSV_HD
#endif

namespace qsv {

// Circuit fields the device-side matrix builders need.
struct CircDev {
    int n, n_layers, reupload, n_rot, rot[3];
    int slots() const { return reupload + n_rot; }
};

// How state rows map to samples.  Plain calls: row = sample.  Gradient launches: row r of the
// chunk is circuit gid = row0 + r; sample = gid / per, variant v = gid % per; v < two_p replaces
// the matrix of parameter v/2 of the circuit being run by its +pi/2 (v even) or -pi/2 (v odd)
// shifted version.  Whole-circuit gradients use per = 2P+1 (variant 2P is the unshifted circuit);
// the layer-by-layer gradient runs the circuit's last layers only and shifts parameters of their
// first layer: per = two_p = 2 * slots * n, or (PassArgs::turns) per = two_p = slots * n: R(t + pi) is what the two shifted
// rotations are made of, R(t +- pi/2) = (R(t) +- R(t + pi)) / sqrt 2.
struct RowMap {
    int grad;        // 0 plain, 1 gradient
    int two_p;       // variants that replace a matrix: v < two_p (also the row stride of the shifted table)
    int per;         // circuits per sample (two_p + 1 when the unshifted circuit is among them)
    int64_t row0;
    int slots_n;     // (reupload + n_rot) * n
    int n;
};

struct PassArgs {
    float2* state;       // the buffer the tiles are written to
    const float2* in;    // the buffer the tiles are read from: state itself, or (a pass with an index map
                         // must not write what it reads) another buffer of the same shape
    const unsigned* imap;  // not NULL: n entries; an amplitude whose position (tile bits plus its place in
                         // the tile at the end of the pass) has bit j set is written to the index with the
                         // bits imap[j] flipped: deferred CNOTs (needs n > tile and n <= 28)
    const float2* src;   // not NULL: tiles are read from src[sample of the row] instead of in (needs n >= tile)
    const void* ops;     // Op list of the pass (direct: DirectOp)
    double* zout;        // not NULL: the pass also writes <Z_zq> partials [tile][wavefront] (needs n >= tile)
    const float2* unturned;  // not NULL (direct, with zout): states a [samples][2^n], and the partials are of three sums each: z |b|^2,
                         // and the real and imaginary part of z conj(a) b, z = +-1 by bit zq, b the row's state
    int turns;           // direct: variant v turns parameter v's angle by pi (rm.two_p of them a sample): see RowMap
    int zq;
    int nostore;         // with zout: the state is not written back
    int nt_store;        // nontemporal tile stores (states much larger than the last-level cache)
    int rev;             // workgroups take the tiles in descending order (see run_circuit and reversed_tile)
    int prio;            // wavefronts raise their issue priority while they compute addresses and issue the
                         // tile's loads, and again for its stores (the gates run at the base priority)
    const float* mats;   // [samples if rowdep][n_mats][8], unitaries in execution order: factored in groups,
                         // or plain matrices when several rows share a tile (n < tile) and differ in them
    const int* exec_of;  // [n_mats]: (layer * n + qubit) -> execution-order index
    const float* ovr;    // gradient: [samples if rowdep][2P][8] shifted matrices
    uint64_t total;      // valid extended indices = rows * 2^n
    int n, c, w;
    int n_mats;
    int rowdep;          // matrices differ per sample
    RowMap rm;
    // direct = 1: ops is a list of DirectOp (see qsv_lower.h) and the fields below are set
    int direct;
    int gather;          // the amplitudes are read through imap (position p from the index it maps to) and written
                         // where they sit
    unsigned mate;       // gather: the tile of a row that has the other halves of tile t's lines is t ^ mate (0: t itself)
    int s_in, s_out;     // register layouts in which the tile is loaded and stored
    int first_mat;       // index of the pass's first unitary
    int warm_ops, warm_mats;   // bytes of the operation list and of the table to fetch ahead (0: none)
    unsigned g_sample0, g_rem0;   // gradient rows: rm.row0 / rm.per and rm.row0 % rm.per
};

// The tile that workgroup b of `tiles` takes in a pass that goes downwards.  Workgroups go to the eight XCDs in turn; with
// rev = 2 eights of tiles change places and keep their order inside, so that a tile stays on its XCD.
QSV_HD inline unsigned reversed_tile(unsigned b, unsigned tiles, int rev) {
    return rev == 2 && (tiles & 7u) == 0 ? tiles - 8u - (b & ~7u) + (b & 7u) : tiles - 1u - b;
}

// The tile of a row that workgroup b of the row takes: t and t ^ mate are eight apart (mate = 0: tile b).  b without bit
// 3 numbers the pairs: it fills the tile's bits other than the lowest bit of mate.  Needs 16 tiles in a row.
QSV_HD inline unsigned mate_order(unsigned b, unsigned mate) {
    if (mate == 0) return b;
    const unsigned pair = (b & 7u) | (b >> 4 << 3), below = (mate & (0u - mate)) - 1u;
    return ((pair & below) | (pair & ~below) << 1) ^ ((b >> 3) & 1u ? mate : 0u);
}

// k_pass_direct takes states of n >= tile qubits (a tile lies in one row), at most this many (a row is at most
// 2^31 bytes), through one LDS plane; k_pass takes the rest: several rows in a tile, 29 and 30 qubits, two planes.
constexpr int kDirectMaxQubits = 28;
hipError_t launch_pass(int tile, int planes, const PassArgs& a, uint64_t n_tiles, hipStream_t st);

// A mirrored pass on the states psi and lambda = O psi at once, with the transition sums of its unitaries: reverse mode.
struct PairArgs {
    const float2* psi;     // the circuit's states after the pass, [rows][2^n]; only read
    const float2* lam_in;  // lambda after the pass; NULL: O psi, for the observable below (the circuit's last pass)
    float2* lam_out;       // lambda before the pass; another buffer than lam_in if imap; NULL: not wanted
    const unsigned* imap;  // as PassArgs::imap, read through
    const void* ops;       // DirectOp list of the paired interpreter
    const float* mats;     // [samples if rowdep][n_mats][8], paired
    float* sums;           // [unitaries][rows][2^(n - 10)][4]: a record per unitary (execution order) and wavefront
    int64_t sample0;       // row r belongs to sample sample0 + r
    int64_t rows;
    int n, c, w, n_mats, rowdep, s_in, s_out, first_mat, first_u, warm_ops, warm_mats;
    unsigned mate;
    int rev, nt_store;
    int kind, q;           // observable, as launch_adj_init's
    uint64_t mask;
    const double* coef;
};
constexpr int kPairMaxTile = 13;
hipError_t launch_pair_pass(int tile, const PairArgs& a, hipStream_t st);
inline size_t pair_sums_bytes(int n, int64_t n_mats) { return (size_t)n_mats * ((size_t)16 << (n - 10)); }   // of a row
// From the records of all unitaries, the derivatives with respect to the angles of the rows' samples, written into
// f[sample][2p], f[sample][2p+1] as (g, -g).  order: (layer * n + qubit) by position; entry_of: its entry in the inverse
// circuit's paired table back of n_mats entries; corr: the scale table.
hipError_t launch_pair_finish(const float* sums, int64_t rows, const CircDev& c, const float* params, int64_t sample0,
                              int64_t P, const int* order, const int* entry_of, const float* back, int n_mats,
                              const double* corr, double* f, hipStream_t st);

// Address, on the current device (which must be `device`), of the library's fixed scratch array of
// kStaticScratchBytes bytes (256-byte aligned).  Looked up once per device; allocates nothing.
constexpr size_t kStaticScratchBytes = (size_t)4 << 20;
hipError_t static_scratch(int device, void** ptr);
hipError_t set_pass_attributes(int device);   // the current device, which must be `device`

// one-gate-per-launch kernels (fallback for n < 4 and cross-check path)
hipError_t launch_naive_u(float2* state, int64_t rows, int n, int q, const float* mats,
                          const float* ovr, int mat_id, int n_mats, int rowdep, const RowMap& rm,
                          hipStream_t st);
hipError_t launch_naive_cnot(float2* state, int64_t rows, int n, int ctrl, int tgt, hipStream_t st);
hipError_t launch_naive_cz_ladder(float2* state, int64_t rows, int n, hipStream_t st);

// fused per-(layer, qubit) unitaries; out: [samples if reupload][n_layers*n][8] floats.  order
// (device, [n_layers*n], NULL = natural order) gives the (layer*n + qubit) id stored at each position of
// a sample's table.  period = n: the order table has n entries, describes a one-layer circuit and
// repeats for every layer (the table of the whole circuit as the tables of its layers, run one by one,
// back to back).  plain: every entry is the matrix; else factored in groups (see kMatGroup), as the
// interpreters of the fused pass read them.  scale (NULL: not wanted): [tables][n_layers*n] complex doubles.
enum class MatForm { plain, factored, direct, paired, phaseless };   // direct, paired: factored, for those interpreters;
                                                             // phaseless: matrices up to a phase, which a group's last one has
// groups (device, NULL: every kMatGroup entries): the n_groups groups of a table (of a layer, if period = n) with their
// scalars as entries of their own (see Plan::groups; form = direct or paired): n_groups entries more a table or layer.
// form = direct with groups: scale (may be NULL) receives what the rounded scalars lack, float / exact, [tables][groups of all
// layers][2].  form = paired: scale (then [tables][n_layers*n][2] doubles by position) receives what sums of products of two states that
// have come through the unitaries up to this one are to be multiplied by, and the same without this one.
hipError_t launch_build_mats(const CircDev& c, const float* params, const float* feats, int64_t samples, int inverse,
                             const int* order, int period, const int* groups, int n_groups, MatForm form, float* out,
                             double* scale, hipStream_t st);
// bytes of the scale table
inline size_t mat_scale_bytes(const CircDev& c, int64_t samples) {
    return (size_t)(c.reupload ? samples : 1) * (size_t)c.n_layers * (size_t)c.n * 16;
}
// shifted matrices for the parameter-shift rule; out: [samples if reupload][2P][8].  They replace entries of a
// table of `per` entries per sample with that scale table (NULL: a plain one); exec_of: position in
// it of (layer*n + qubit)
hipError_t launch_build_shifted(const CircDev& c, const float* params, const float* feats, int64_t samples,
                                const int* exec_of, const double* scale, int per, float* out, hipStream_t st);
// What a one-layer circuit's unitary is to be multiplied by for one of its angles to be turned by pi, from the right (behind =
// 0) or from the left; [samples if reupload][P][8].
hipError_t launch_build_turns(const CircDev& c, const float* params, const float* feats, int64_t samples, int behind,
                              float* out, hipStream_t st);

// encoding
hipError_t launch_norms(const float* x, int64_t samples, int64_t dim, double* partial, int nblk,
                        double* inv_norm, float* norm_out, hipStream_t st);
// Norms and state rows: inv_norm receives 1/||x_b||, norm_out (may be NULL) ||x_b||; partial: samples * nblk doubles.
// k_norm_finish goes where a state has at most so many amplitudes (k_encode_write has both sides)
constexpr uint64_t kEncodeFolded = 1ull << 20;
hipError_t launch_encode(const float* x, int64_t samples, int64_t dim, int n, double* partial, int nblk, double* inv_norm,
                         float* norm_out, float2* state, hipStream_t st);
// A whole small workload in one launch: encoding, circuit (decode = 1: followed by its inverse), final
// state, and the measurement `kind` (QSV_M_PROBS or QSV_M_EXPZ_ALL).  A thread keeps 2^regs amplitudes
// (regs = 2, 3 or 4), the other index bits are bits of the thread number (at most 8: 256 threads); with
// fewer than 6 of them a wavefront holds 2^(6 - bits) samples.  A workgroup keeps the matrices of its
// samples in LDS (at most kSmallMats).
constexpr int kSmallMaxQubits = 10;
// batch * 2^n up to which one launch beats the fused passes.  With 10 qubits the pass kernel has a tile per row
// and takes the lead earlier (1024 rows, 6 layers: 32 against 36 us; 2048 rows: 49 against 41, 20 layers 186
// against 91).
constexpr int64_t small_apply_amplitudes(int n) { return (int64_t)1 << (n == 10 ? 20 : 21); }
constexpr int kSmallMats = 512;   // matrices a workgroup keeps in LDS (16 KiB)
inline int small_rows_per_group(int n, int regs) {
    const int tb = n > regs ? n - regs : 0;
    return tb < 6 ? 64 >> tb : 1;
}
// Whether the circuit has any unitary: if so its angles and features are staged in LDS and its matrices built there.
QSV_HD inline bool small_has_unitaries(const CircDev& c) { return c.n_layers > 0 && c.reupload + c.n_rot > 0; }
QSV_HD inline int small_staged_angles(const CircDev& c) { return c.n_layers * (c.reupload + c.n_rot) * c.n; }
QSV_HD inline int small_staged_features(const CircDev& c, int rows) { return c.reupload ? rows * c.n : 0; }
inline int64_t small_mats_per_group(const CircDev& c, int regs) {
    if (!small_has_unitaries(c)) return 0;
    return (int64_t)(c.reupload ? small_rows_per_group(c.n, regs) : 1) * c.n_layers * c.n;
}
// Amplitudes per thread: the most that still gives the chip about four wavefronts per SIMD (4096), else the
// fewest; among those only what fits the matrix limit.  0: nothing fits.
inline int small_choose_regs(const CircDev& c, int64_t batch) {
    int fallback = 0;
    for (int r = 4; r >= 2; --r) {
        if (c.n - r > 8 || small_mats_per_group(c, r) > kSmallMats) continue;
        const int rows_g = small_rows_per_group(c.n, r);
        const int tb = c.n > r ? c.n - r : 0;
        const int64_t waves = ((batch + rows_g - 1) / rows_g) * (tb > 6 ? 1 << (tb - 6) : 1);
        if (waves >= 4096) return r;
        fallback = r;             // the smallest that fits so far
    }
    return fallback;
}
// What a launch of k_forward_small is made of.
struct SmallShape {
    int rows;            // samples per workgroup
    unsigned threads;
    int mat_floats;      // LDS floats of the workgroup's matrices (a multiple of 8)
    size_t lds;          // dynamic LDS in bytes
};
inline SmallShape small_shape(const CircDev& c, int regs, int64_t batch) {
    SmallShape s;
    const int tb = c.n > regs ? c.n - regs : 0;
    s.threads = tb > 6 ? 64u << (tb - 6) : 64u;
    // Per-sample matrices are most of such a launch's work (a wavefront of 16 samples builds them for 18 us, 4 qubits,
    // 6 layers), so while the chip has wavefronts to spare (eight per CU) the samples spread over them.
    s.rows = small_rows_per_group(c.n, regs);
    if (c.reupload && s.rows > 1) {
        const int64_t spread = (batch + 2047) / 2048;
        if (spread < s.rows) s.rows = (int)spread;
    }
    // sums across wavefronts, the matrices (only as many as this circuit has: LDS per workgroup decides how
    // many workgroups a CU holds), and two exchange buffers (several wavefronts per sample only) that share
    // their place with the staged angles and features
    const bool has = small_has_unitaries(c);
    s.mat_floats = has ? (c.reupload ? s.rows : 1) * c.n_layers * c.n * 8 : 0;
    const size_t stage = has ? (size_t)(small_staged_angles(c) + small_staged_features(c, s.rows)) * sizeof(float) : 0;
    const size_t exchange = s.threads > 64 ? 2 * (size_t)(2 << regs) * s.threads * sizeof(float) : 0;
    s.lds = 64 * sizeof(double) + (size_t)s.mat_floats * sizeof(float) + (stage > exchange ? stage : exchange);
    return s;
}
// x = NULL: start from the amplitudes in `state`; passes pass_first..pass_last (0 = the circuit, 1 = its inverse);
// kind = 0: no measurement (the final state is always written)
hipError_t launch_forward_small(int regs, const float* x, int64_t dim, int64_t batch, const CircDev& c, int entangler,
                                const float* params, const float* feats, int pass_first, int pass_last, int kind,
                                float2* state, float* out, float* norm_out, hipStream_t st);
// Reverse-mode gradient of a whole small batch (see k_sweep_small) into f[batch][2P+1]; back: the phaseless table of the
// inverse circuit in natural order; kept (NULL: do without): n_layers * batch * 2^n amplitudes; sums: batch * n_layers *
// sweep_record_bytes(n) bytes.  At most kSmallMats unitaries.
hipError_t launch_sweep_small(const float* x, int64_t dim, int64_t batch, const CircDev& c, int entangler,
                              const float* params, const float* back, int kind, int q, uint64_t mask, const float* targets,
                              float2* kept, double* sums, double* f, hipStream_t st);
inline size_t sweep_record_bytes(int n) { return (size_t)(n > 8 ? 1 << (n - 8) : 1) * 32 * 8; }
hipError_t launch_encode_write(const float* x, int64_t dim, int n, int64_t rows, const double* inv_norm,
                               const RowMap& rm, float2* state, hipStream_t st);

// measurement
hipError_t launch_probs(const float2* state, uint64_t total, float* out, hipStream_t st);
// partial: rows * max(1, 2^n / 4096) * 13 doubles or fewer; the finishing kernels take the same rows and n
hipError_t launch_expz_block(const float2* state, int64_t rows, int n, double* partial, hipStream_t st);
// <Z_q> of every qubit (q_only < 0) or of q_only in one launch, where a row is a block's work
bool expz_in_one_launch(int n, int64_t rows);
hipError_t launch_expz_small(const float2* state, int64_t rows, int n, int q_only, float* out_f, hipStream_t st);
// What the scalars of a table's groups lack of the exact ones, as launch_build_mats writes it: the product of the entries
// first .. first + count - 1 of a sample's `stride`.
struct Residues { const double* table; int first, count, stride; };
// res (NULL: none): of the tables that the rows, which are samples then, have come through; rowdep: a table per sample
hipError_t launch_expz_finish(const double* partial, int64_t rows, int n, int q_only, float* out_f,
                              double* out_d, hipStream_t st, const Residues* res = nullptr, int rowdep = 0);
// Where one-qubit results of gradient rows go: circuit gid = row0 + r lands at
// out[(gid / per) * stride + offset + gid % per].
struct Scatter { int64_t row0, per, stride, offset; };
hipError_t launch_expz_finish_scatter(const double* partial, int64_t rows, int n, int q, double* out,
                                      const Scatter& sc, hipStream_t st, const Residues* res = nullptr, int rowdep = 0);
// out[scatter(row)] = sum of the row's per_row partials written by a pass with zout
hipError_t launch_zsum_finish(const double* partial, int64_t rows, int64_t per_row, double* out,
                              const Scatter& sc, hipStream_t st);
// The two results of a turned row b from its three sums (PassArgs::unturned), <Z> of (a + b) / sqrt 2 and of (a - b) / sqrt 2, at
// out[(gid / per) * stride + offset + 2 (gid % per)] and behind it; <Z> of a is out[(gid / per) * stride + unturned_at].
// Without their scalars' rounding: what a has come through since the two parted is in ra, b's in rb1 and rb2; a phase of
// a few 1e-8 between them would show in the results in full.  rowdep: a table per sample.
hipError_t launch_turned_finish(const double* partial, int64_t rows, int64_t per_row, double* out, const Scatter& sc,
                                int64_t unturned_at, const Residues& ra, const Residues& rb1, const Residues& rb2, int rowdep,
                                hipStream_t st);
// states[r] = src[sample of row r] for the rows of a gradient chunk (src: [samples][2^n])
hipError_t launch_gather_rows(const float2* src, int n, int64_t rows, const RowMap& rm, float2* states,
                              hipStream_t st);
// partial: [rows][n_v][nblk] doubles with nblk = max(1, 2^(n-m) / 4096)
hipError_t launch_marginal_block(const float2* state, int64_t rows, int n, uint64_t mask, int64_t n_v,
                                 double* partial, hipStream_t st);
hipError_t launch_marginal_finish(const double* partial, int64_t rows_times_v, int64_t nblk, float* out,
                                  int renorm_mode, double* scale, hipStream_t st);
hipError_t launch_project(float2* state, int64_t rows, int n, uint64_t mask, const double* scale,
                          hipStream_t st);
hipError_t launch_fidelity_block(const float2* state, int64_t rows, int n, const float* x, int64_t dim,
                                 double* partial, int nblk, const RowMap& rm, hipStream_t st);
hipError_t launch_fidelity_finish(const double* partial, int nblk, int64_t rows, float* out, double* out_d,
                                  hipStream_t st);
// trash reset: rows (sample, outcome) of a chunk from the state; sum of the rows' fidelities per sample
hipError_t launch_reset_rows(const float2* state, int n, uint64_t mask, int64_t rows, const RowMap& rm,
                             float2* work, hipStream_t st);
hipError_t launch_reset_sum(const double* Frow, int64_t per, int64_t B, float* out, hipStream_t st);
// finite-shot <Z_q> from samples [rows][shots] -> out [rows][n]
hipError_t launch_shot_expz(const long long* samples, int64_t shots, int64_t rows, int n, float* out,
                            hipStream_t st);
// sampling: bsum/cum are uint64 [rows][nblk], nblk = max(1, 2^n / 4096); sub (NULL: do without, same samples)
// uint64 [rows][nblk][16]
hipError_t launch_sample(const float2* state, int64_t rows, int n, const double* uniforms, int64_t shots,
                         unsigned long long* cum, unsigned long long* sub, long long* out, hipStream_t st);

// <P> of a Pauli string (X on xmask, Y on ymask, Z on zmask) per row; partial: rows * blocks * 2 doubles
hipError_t launch_pauli(const float2* state, int64_t rows, int n, uint64_t xmask, uint64_t ymask,
                        uint64_t zmask, double* partial, float* out, hipStream_t st);

// Reverse-mode gradient.  launch_adj_init: S[2r] = A[r], S[2r+1] = O A[r] (rows of A) for the
// diagonal observable O: kind 0 Z_q; kind 1 -P0(mask); kind 2 sum_q coef[r][q] Z_q.
// launch_trash_loss: f[sample0+r][2P] = 1 - P0(mask) of row r (partial: rows * blocks doubles, blocks
// as for the <Z> reductions).  launch_mse_coef: from z[rows][n] and targets y[samples][n], the loss
// 1/n sum (z-y)^2 into f[.][2P] and coef = 2/n (z-y).
// launch_adj_init: lambda = O psi for the rows of A; paired = 1 writes (psi, lambda) into rows 2r, 2r+1
// of S, paired = 0 writes lambda alone into row r.
// back: the inverse circuit's table, every layer's unitaries in the order of a one-layer plan (exec_of: position
// of a qubit's; NULL: natural order).
// launch_trans: the transition sums of the row pairs (psi0 + rstride r 2^n, lam0 + rstride r 2^n), both taken back to
// the start of a layer: adj_trans_count(n, row_pairs) partials for each pair and qubit, 8 doubles each.
// launch_adj_layers: from the partials of the layers layer0 .. layer0 + n_layers - 1, one layer's after the other's, the
// derivatives with respect to their angles, written into f[sample][2p], f[sample][2p+1] as (g, -g).  partial has room
// for n_layers * row_pairs * n * (adj_trans_blocks(n) + 1) * 8 doubles (the sums go behind the partials).
hipError_t launch_adj_init(const float2* A, int n, int kind, int q, uint64_t mask, const double* coef,
                           int64_t rows, float2* S, int paired, hipStream_t st);
hipError_t launch_trash_loss(const float2* A, int n, uint64_t mask, int64_t rows, int64_t sample0, int64_t P,
                             double* partial, double* f, hipStream_t st, const Residues* res = nullptr, int rowdep = 0);
hipError_t launch_mse_coef(const double* z, const float* y, int n, int64_t rows, int64_t sample0, int64_t P,
                           double* coef, double* f, hipStream_t st);
// optimiser steps in double on float storage; t is the 1-based step count of Adam
hipError_t launch_sgd(float* p, const float* g, int64_t count, double lr, hipStream_t st);
hipError_t launch_adam(float* p, const float* g, float* m, float* v, int64_t count, int64_t t, double lr,
                       double b1, double b2, double eps, hipStream_t st);
int adj_trans_blocks(int n);
int adj_trans_count(int n, int64_t row_pairs);
hipError_t launch_trans(const float2* psi0, const float2* lam0, int rstride, int n, int64_t row_pairs, double* partial,
                        hipStream_t st);
hipError_t launch_adj_layers(double* partial, int64_t row_pairs, const CircDev& c, int layer0, int n_layers,
                             const float* params, int64_t sample0, int64_t P, const float* back, const int* exec_of,
                             MatForm form, double* f, hipStream_t st);

// gradient assembly from f[B][2P+1] (double)
hipError_t launch_grad_finish(const double* f, int64_t B, int64_t P, const CircDev& c, const float* feats,
                              float* loss, float* grad, float* mean_loss, float* mean_grad,
                              hipStream_t st);

}  // namespace qsv

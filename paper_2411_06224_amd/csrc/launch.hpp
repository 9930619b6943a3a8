// Host launchers of the HIP kernels and their argument blocks.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstdint>

#include "common.hpp"

namespace maspcg {

constexpr int kMaxLv = 16;

// Kernel timing: when set, the next launch reports its own start and end to
// these events (the runtime stamps them from the dispatch itself, so the
// elapsed time excludes the gaps between launches); the launch consumes them.
struct DispatchEvents {
    hipEvent_t start = nullptr, stop = nullptr;
};
inline DispatchEvents& dispatch_events() {
    static thread_local DispatchEvents e;
    return e;
}

template <typename F, typename... Args>
void launch_kernel(F kernel, dim3 grid, dim3 block, uint32_t shmem, hipStream_t s, Args... args) {
    DispatchEvents& e = dispatch_events();
    hipExtLaunchKernelGGL(kernel, grid, block, shmem, s, e.start, e.stop, 0u, args...);
    e = DispatchEvents{};
}

// Device views of the solver's data in the caller's workspace.
struct SolverView {
    int V, N, M, NS, L, nnzb;
    int D0, RG, G;  // work groups: D0 level-0 domains = RG slots; G groups
    int sym;        // 1: H64 holds the group-symmetric storage (nsb blocks), 0: the full slot-ordered H;
                    // H32 (mixed) always holds the full storage (nnzb blocks)
    int nsb;        // blocks of the stored slot-ordered H (H64 / H32 planes)
    int maxT;       // most transposed entries of one group (symmetric storage)
    const int* gorder;  // [G] SpMV group of each workgroup, or null: xcd_group
    int units[kMaxLv];
    int ndom[kMaxLv];
    // plans
    const int* remap;     // [NS]
    const int* map;       // [V]
    const int* perm_src;  // [nsb] caller block of each stored block (H64)
    const int* perm_full; // [nnzb] caller block of each full slot-ordered block (H32: full storage)
    const int* srp;       // symmetric storage: [NS+1] stored rows
    const int* sci;       // [nsb] column slot of each stored block
    const uint8_t* srow;  // [nsb] local row (slot - group start) of each stored block
    const int* tptr;      // [NS+1] transposed entries of each row
    const int* tidx;      // stored block of each transposed entry
    const int* rp0;       // [NS+1]
    const int* ci0;       // [nnzb]
    const int* lead1;     // [NS]
    const int* anc;       // [(L-1)*NS]
    const int* g_u1;      // [G+1]
    int W1;                       // restriction: most level-1 units in a group
    // levels l >= 2, [G][L-2][W1] (entry (g, l - 2, i) for level-1 unit i of group g, -1 / 0 pad):
    const int* ganc;              // its level-l unit
    const int* gpos;              // its partial position, -1 if it writes none
    const uint64_t* gmask;        // writers: group-local level-1 units below it
    const uint64_t* lmask;        // [NS] leader slots: lanes of the domain in the slot's level-1 unit
    // the restriction by output, padded per group: level-1 unit i of group g
    // at [g * W1 + i] (lowest slot, -1 pad; lane mask), writer e of levels
    // >= 2 at [g * GW + e] (partial position, -1 pad; entry (l - 2) W1 + i of
    // the group's ganc row; member mask over the group's level-1 units)
    const int* gu1_slot;
    const uint64_t* gu1_mask;
    int GW;
    int rpass;  // restrict_passes of the SpMV's threads
    const int* gw_pos;
    const int* gw_li;
    const uint64_t* gw_mask;
    const int* cp_ptr[kMaxLv];    // l >= 2: [S_l + 1]
    // two-launch iteration (Plan::hptr): the level-1 units whose coarse
    // correction group g reads, [hptr[g], hptr[g + 1]) (its own first), and
    // the group's local index of each one's level-2 unit; those level-2
    // entries, [h2ptr[g], h2ptr[g + 1]), with their corrections' positions in
    // yall at every level >= 2; the local unit of every block of the SpMV's
    // storage with a column outside the group
    const int *hptr, *hu, *h2ptr, *hy;
    const uint16_t *hpar, *hidx;
    int maxH, maxH2;  // most units / level-2 entries of one group
    int ncb;   // coarse workgroups of the apply (all_coarse_blocks)
    int GA;    // level-0 workgroups of the apply (apply_blocks): its rho (and, by recurrence, ||r||^2) partials
    // stored slot-ordered matrix (9 planes: H64 of nsb, H32 of nnzb values)
    double* H64;
    float* H32;
    // inverses per level: packed pairs (N = 16) or column-major (3N)^2 per domain
    double* inv64[kMaxLv];
    float* inv32[kMaxLv];
    // vectors in slot order (3*NS doubles)
    double *b, *x, *r, *z, *q;
    double* p[2];  // search direction p_k lives in p[k & 1]
    // coarse vectors: r1 [3*units[1]], y_l [3*ndom[l]*N] for l >= 1, coarse partials [3*n_cpart]
    double* r1;
    double* y[kMaxLv];  // laid end to end from yall
    double* yall;
    double* cpart;
    // the same restrictions of q = H p (q1, qpart), and the restricted
    // residual C_l r of levels l >= 2 ([3*ndom[l]*N]) that the coarse apply
    // keeps between iterations: C_l r_k = C_l r_{k-1} - alpha_k C_l q_k
    double* q1;
    double* qpart;
    double* rc[kMaxLv];
    // partial sums: one per group [G] (P_rr: one per level-0 workgroup of the
    // apply [GA] after an iteration by recurrence), P_rho [GA + ncb]: the
    // level-0 workgroups' r^T z, then (by recurrence) the coarse workgroups'
    // r_l^T y_l
    double2* P_sp;  // one per group [G]: p_k^T q_k and r_{k-1}^T p_k
    double *P_rr, *P_bb, *P_rho[2];
    DevState* st;
    int* flag;  // inversion status
};

// Inverses of domain size 16 (FP64 and FP32, every level) are stored
// symmetric-packed for a wave that multiplies a pair of domains (2p, 2p + 1)
// straight out of its registers (mas.hip, pair_product): 2352 entries per
// pair, those of two lower triangles.  Of each domain's 48 x 48 inverse the
// three 16 x 16 tiles (1,0), (2,0), (2,1) below the diagonal are kept whole;
// the diagonal tiles of the two domains share tiles, the first domain's lower
// triangle (diagonal halved, so that using an entry for its row and for its
// column counts the diagonal once) and the second's strictly upper one, whose
// diagonal follows the nine tiles.  Entry (r, c) of a tile sits in lane
// r + 16 (c / 4) as its entry c % 4, 16 bytes of a lane side by side.  Other
// domain sizes keep full column-major (3N)^2 blocks.
constexpr int kPairEntries = 2352;
constexpr int kTile = 256;
constexpr int kPairDiag = 9 * kTile;  // the second domain's diagonal

// Place of entry (r, c) in its tile.
template <typename TI>
__host__ __device__ constexpr int tile_at(int r, int c) {
    const int lane = r + 16 * (c >> 2), v = c & 3;
    return sizeof(TI) == 8 ? (v >> 1) * 128 + 2 * lane + (v & 1) : 4 * lane + v;
}

// Tile below the diagonal, block row I > J, of the pair's first (half = 0) or
// second domain.
__host__ __device__ constexpr int tile_below(int I, int J, int half) { return 3 * half + (I == 1 ? 0 : 1 + J); }

// Place of entry (i, j), i >= j, of a domain's inverse in its pair.
template <typename TI>
__host__ __device__ constexpr int pair_at(int half, int i, int j) {
    const int I = i / 16, J = j / 16, r = i % 16, c = j % 16;
    return I > J                ? kTile * tile_below(I, J, half) + tile_at<TI>(r, c)
           : half == 0          ? kTile * (6 + I) + tile_at<TI>(r, c)
           : r == c             ? kPairDiag + i
                                : kTile * (6 + I) + tile_at<TI>(c, r);
}

// Stored inverse entries of nd domains of size N.
inline size_t inverse_entries(int N, int nd) {
    return N == 16 ? static_cast<size_t>((nd + 1) / 2) * kPairEntries : static_cast<size_t>(nd) * 9 * N * N;
}

// Workgroups of the apply.  N = 16: kApplyDomains consecutive level-0 (or
// level-1) domains per workgroup, a pair per wave, and one pair of domains of
// the levels above per workgroup; other sizes: one group of
// level-0 domains (apply_blocks = G) and one coarse domain each.
constexpr int kApplyDomains = 8;
inline int apply_blocks(int N, int M, int G) { return N == 16 ? (M + kApplyDomains - 1) / kApplyDomains : G; }
inline int coarse_blocks(int N, int l, int nd) {
    return N == 16 ? (l == 1 ? (nd + kApplyDomains - 1) / kApplyDomains : (nd + 1) / 2) : nd;
}
inline int all_coarse_blocks(int L, int N, const int* ndom) {
    int n = 0;
    for (int l = 1; l < L; ++l) n += coarse_blocks(N, l, ndom[l]);
    return n;
}

// Build-phase views.
struct BuildView {
    int L, N, nnzb;
    int units[kMaxLv];
    int ndom[kMaxLv];
    int nnzA[kMaxLv];
    const int* red_ptr[kMaxLv];  // level l >= 1
    const int* red_src[kMaxLv];  // level 1: caller block indices
    const int* dom_ptr[kMaxLv];
    const int* dom_blk[kMaxLv];  // level 0: caller block indices
    const int* dom_ab[kMaxLv];
    const int* remap;
    double* A[kMaxLv];  // level l >= 1: 9 planes of nnzA[l]
    double* inv64[kMaxLv];
    float* inv32[kMaxLv];
    int* flag;
};

// Residual kernel modes.
enum ResidMode {
    kResidInit = 0,     // r = b - H x0 with ||r||^2, ||b||^2 and the restriction
    kResidReplace = 1,  // r = b - H x with ||r||^2 and the restriction (skipped after a stop)
    kResidConfirm = 2,  // as kResidReplace, run after the host cleared a stop
    kResidFinal = 3     // scratch = b - H x with ||.||^2 only
};
// MAS apply modes of the separate coarse and level-0 launches.
//  kApplyPlain: z = M^-1 r outside PCG (no decision, no partials).
//  kApplyInit:  the first apply of a solve; decision on r_0 with ||b||.
//  kApplyIter:  iteration k after the x/r update kernel restricted r_k:
//               coarse residuals straight from that restriction (kept for
//               the recurrence), decision on r_k.
// An iteration by recurrence applies in one launch (launch_apply_rec): alpha_k,
// C_l r_k = C_l r_{k-1} - alpha_k C_l q_k from the restriction of q_k the SpMV
// left and the coarse corrections y_l beside x += alpha p, r -= alpha q and
// z = Inv_0 r; the next SpMV adds the corrections to z where it reads it and
// takes the decision on r_k.  Where some group reads more units than the SpMV
// can stage (Plan::hptr), a third launch does both (launch_prolong).
enum ApplyMode { kApplyPlain = 0, kApplyInit = 1, kApplyIter = 2 };

// spmv.hip
hipError_t launch_spmv_user(int n_rows, const int* rp, const int* ci, const void* val, bool f32, const double* x,
                            double* y, hipStream_t s);
// iteration k: p_k = z_{k-1} + beta p_{k-1} (p_1 = z_0) into p[k & 1], q = H
// p_k, the partials of p_k^T q_k and r_{k-1}^T p_k.
// restrict_q: also the restriction of q to the coarse levels (q1, qpart);
// rec: the previous iteration ran launch_apply_rec; split: and no
// launch_prolong, so that z_{k-1} is v.z plus the coarse corrections in yall,
// and one workgroup more takes the decision on r_{k-1}
hipError_t launch_spmv_pq(const SolverView& v, bool f32, int k, bool restrict_q, bool rec, bool split,
                          hipStream_t s);
// Shared memory of the SpMV kernels besides a group's staged corrections
// (24 bytes for each of maxH units and maxH2 level-2 entries).
size_t spmv_shared_bytes(int RG, int maxT, bool sym);
// Bytes of shared memory the SpMV kernels can lend to the restriction of q
// after their stream (their product planes).
size_t spmv_restrict_capacity();
// Threads per workgroup of the SpMV kernels.
int spmv_threads();
hipError_t launch_residual(const SolverView& v, int mode, double* out, hipStream_t s);

// vectors.hip
hipError_t launch_state_reset(const SolverView& v, hipStream_t s);
hipError_t launch_clear_stop(const SolverView& v, hipStream_t s);
hipError_t launch_finalize(const SolverView& v, hipStream_t s);
hipError_t launch_permute_H(const SolverView& v, const double* Hu, bool f32, hipStream_t s);
hipError_t launch_perm_in(const SolverView& v, const double* src, double* dst, hipStream_t s);
hipError_t launch_perm_out(const SolverView& v, const double* src, double* dst, hipStream_t s);
hipError_t launch_init_rhs(const SolverView& v, hipStream_t s);
hipError_t launch_update(const SolverView& v, int k, hipStream_t s);
// The restriction of a vector r in the caller's node order.
hipError_t launch_restrict(const SolverView& v, const double* r, hipStream_t s);
hipError_t launch_adjoint_scatter(int n_rows, const int* rp, const int* ci, const double* lam, const double* x,
                                  void* out, bool f32, hipStream_t s);

// mas.hip
hipError_t launch_coarse_sums(const BuildView& b, const double* Hu, hipStream_t s);
hipError_t launch_invert(const BuildView& b, const double* Hu, bool want32, hipStream_t s);
// Coarse levels plus the convergence decision (mode as ApplyMode; k = 0:
// the initial apply); rr_true: the residual partials hold b - H x rather
// than the recurrence (residual replacement, FP64 confirmation).
hipError_t launch_apply_coarse(const SolverView& v, bool f32, int mode, int k, double tol, bool x0_given, bool mixed,
                               bool rr_true, hipStream_t s);
// The decision on r_k alone, after an iteration k by recurrence.
hipError_t launch_decision(const SolverView& v, int k, bool mixed, hipStream_t s);
hipError_t launch_apply_level0(const SolverView& v, bool f32, int mode, int k, hipStream_t s);
// z = M^-1 r outside PCG after launch_restrict(v, r): the coarse levels, then
// level 0 with the prolongation (r, z: the caller's node order).
hipError_t launch_apply_plain(const SolverView& v, bool f32, const double* r, double* z, hipStream_t s);
// Iteration k by recurrence: x/r update, level 0 and the coarse levels in
// one launch (see ApplyMode).
hipError_t launch_apply_rec(const SolverView& v, bool f32, int k, hipStream_t s);
// After launch_apply_rec: the coarse corrections added to z, and the decision
// on r_k.
hipError_t launch_prolong(const SolverView& v, int k, bool mixed, hipStream_t s);

// assemble.hip: block-list assembly (scratch in the caller's workspace).
struct AsmLayout {
    int cb;                      // index bits: n_rows < 2^cb
    uint64_t *key, *key_sorted;  // (row << cb) | col per listed block
    int *pos, *pos_sorted;       // list position of each listed block
    int *head, *seg;             // segment heads of the sorted list and their exclusive scan
    int *seg_start;              // first sorted entry of each distinct (row, col)
    int* flag;                   // [0]: bit 0 index out of range; [1]: distinct blocks
    void* tmp;                   // radix sort / scan scratch of tmp_bytes
    size_t tmp_bytes;
};
// Layout of the assembly scratch from ws (ws = nullptr: sizes only; *total
// receives the bytes needed).
AsmLayout assemble_layout(char* ws, int n_rows, long long n_in, size_t* total);
// Exclusive scan of n ints into out[0..n] (out[n] = total); n + 1 <= 2^20.
hipError_t launch_scan(const int* in, int n, int* out, int* totals, hipStream_t s);
// Keys, stable sort by (row, col) and segment heads of the listed blocks;
// row_ptr of the result; flag[0] bit 0: index out of range, flag[1]: the
// number of distinct blocks.
hipError_t launch_assemble_sort(const AsmLayout& L, int n_rows, long long n_in, const int* rows, const int* cols,
                                int* row_ptr, hipStream_t s);
// Sums every (row, col) segment in list order into col_idx / val.
hipError_t launch_assemble_reduce(const AsmLayout& L, long long n_in, const double* blocks, int* col_idx, double* val,
                                  int nnzb, hipStream_t s);
// Both steps at once for lists of short rows (*taken: the list is one), with
// no host round trip between them: row_ptr, and, if every index was in range,
// no row too long and row_ptr[n_rows] <= capacity, col_idx and val.  flag[0]
// bit 0: index out of range; bit 1: a row too long for this path; flag[1]:
// row_ptr[n_rows].
hipError_t launch_assemble_rows(const AsmLayout& L, int n_rows, long long n_in, const int* rows, const int* cols,
                                const double* blocks, int* row_ptr, int* col_idx, double* val, long long capacity,
                                hipStream_t s, bool* taken);

// hierarchy.hip: supernode hierarchy on the device, every level queued at
// once; the level state on the device ends it (no host round trip).
struct HierState {
    int n_units;          // units of the current level
    int occupied;         // occupied units of the current level
    int levels;           // levels built so far
    int done;             // 1: no further level
    int bad;              // 1: the node-order pattern had an entry out of range
    int units[kMaxLv];
};
struct HierLayout {
    unsigned long long* mask;
    int *sn, *rep, *up, *cnt, *off, *totals;
    HierState* st;
};
// The pattern the hierarchy is built from: slot-ordered (map = null; rows
// and columns are slots), or in the caller's node order with the node ->
// slot map (nnzb blocks; checked against V).
struct HierPattern {
    const int *rp, *ci, *map;
    long long nnzb;
};
HierLayout hierarchy_layout(char* ws, int NS, int L_max, size_t* total);
// Levels 0 .. L_cap - 1 at most; H.sn + l NS receives the unit of every slot
// at level l, H.st the level count and units.
hipError_t launch_hierarchy(const HierLayout& H, int NS, int V, int N, int L_cap, const int* remap,
                            const HierPattern& pat, hipStream_t s);
// out_units[0] = levels (-1: invalid pattern), out_units[1 + l] = units of
// level l (kMaxLv + 1 entries); out_sn[l V + i] = unit of node i at level l,
// -1 past the last level (kMaxLv V entries).
hipError_t launch_hier_export(const HierLayout& H, int V, int NS, const int* map, int* out_units, int* out_sn,
                              hipStream_t s);

}  // namespace maspcg

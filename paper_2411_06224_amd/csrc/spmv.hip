// 3x3-block CSR sparse matrix-vector products (Supp. Eq. 2: T_spmv of a PCG
// iteration).
//
// A workgroup owns a group of consecutive block rows and streams the
// group's blocks, which are contiguous in memory, in chunks: thread t takes
// blocks t, t + 256, ... of the chunk (consecutive threads read consecutive
// values of each plane), multiplies each 3x3 block by its x entry and parks
// the three products in LDS.  Every (row, component) pair of the group has
// one owner thread that then adds its row's products in column order.  The
// load is balanced by blocks, not rows, so rows of 7 and 19 blocks (the two
// node classes of the tet cube) or long contact / affine rows cost the same
// per block.  Products and sums are FP64; FP32-stored values are widened on
// load.
#include "decision.hpp"
#include "launch.hpp"
#include "planner.hpp"
#include "restrict.hpp"

namespace maspcg {
namespace {

constexpr int kThreads = 256;
constexpr int kChunk = 1024;       // blocks staged in LDS per pass
// LDS planes of products are kPad doubles longer than a chunk, so that the
// three components of one row, read by neighbouring lanes at the same
// offset of consecutive planes, fall in different banks
constexpr int kPad = 1;
constexpr int kPlane = kChunk + kPad;

// acc + p[lo] + p[lo + 1] + ... + p[hi - 1], added in this order; eight
// entries are loaded at a time so that their LDS latencies overlap (a body's
// row of 1,500 blocks: 102 us of the product with four, 84 with eight)
__device__ __forceinline__ double sum_run(double acc, const double* p, int lo, int hi) {
    int k = lo;
    for (; k + 8 <= hi; k += 8) {
        double a[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) a[j] = p[k + j];
#pragma unroll
        for (int j = 0; j < 8; ++j) acc += a[j];
    }
    for (; k + 4 <= hi; k += 4) {
        const double a0 = p[k], a1 = p[k + 1], a2 = p[k + 2], a3 = p[k + 3];
        acc = (((acc + a0) + a1) + a2) + a3;
    }
    for (; k < hi; ++k) acc += p[k];
    return acc;
}

// acc plus p[tl[tp] - cs], p[tl[tp + 1] - cs], ... in list order for the
// entries of tl[tp, te) below ce (the lists ascend); tp advances past them.
__device__ __forceinline__ double sum_listed(double acc, const double* p, const int* tl, int& tp, int te, int cs,
                                             int ce) {
    while (tp < te) {
        int kk[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) kk[j] = tp + j < te ? tl[tp + j] : ce;
        double v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = kk[j] < ce ? p[kk[j] - cs] : 0.0;
        int n = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (kk[j] < ce) {
                acc += v[j];
                ++n;
            }
        tp += n;
        if (n < 4) break;
    }
    return acc;
}

// Block values: caller layout (9 consecutive values per block) or the
// solver's planar layout (value c of block k at c * stride + k).
template <typename T, bool kPlanar>
struct Blocks {
    const T* __restrict__ v;
    long long stride;
    __device__ __forceinline__ double at(int k, int c) const {
        return kPlanar ? static_cast<double>(v[c * stride + k]) : static_cast<double>(v[9LL * k + c]);
    }
};

// The vector H multiplies: x itself, or the new search direction z + beta p
// formed on the fly from the previous one (kSplit: z with its coarse correction
// still to be added, staged in LDS at the group's local unit h / 3 of the
// column).
struct XVec {
    static constexpr bool kUnits = false;
    const double* __restrict__ x;
    __device__ __forceinline__ double at(int i, int) const { return x[i]; }
};
template <bool kSplit>
struct XDir {
    static constexpr bool kUnits = kSplit;
    const double* __restrict__ z;
    const double* __restrict__ p;
    double beta;
    const double* ycor;
    __device__ __forceinline__ double at(int i, int h) const {
        return __fma_rn(beta, p[i], kSplit ? z[i] + ycor[h] : z[i]);
    }
};

// Column indices of this thread's blocks t, t + 256, ... of the chunk
// starting at cs, loaded one chunk ahead of their use so that a chunk's
// gathers need not wait for them.  The loads are unconditional, at indices
// clamped to the range's last block (none for an empty range).
constexpr int kRowPer = kChunk / kThreads;

struct ChunkCols {
    int j[kRowPer];
    int h[kRowPer];  // local unit of each column (kUnits)
};

template <bool kUnits = false>
__device__ __forceinline__ ChunkCols chunk_cols(const int* __restrict__ ci, int cs, int ke,
                                                const uint16_t* __restrict__ hidx = nullptr) {
    ChunkCols c;
#pragma unroll
    for (int kk = 0; kk < kRowPer; ++kk) c.j[kk] = c.h[kk] = 0;
    if (cs < ke) {
#pragma unroll
        for (int kk = 0; kk < kRowPer; ++kk) {
            const int k = min(cs + static_cast<int>(threadIdx.x) + kk * kThreads, ke - 1);
            c.j[kk] = ci[k];
            if constexpr (kUnits) c.h[kk] = hidx[k];
        }
    }
    return c;
}

// The group a workgroup of the matrix-streaming kernels takes: the
// planner's order when the groups' stored blocks are uneven, else the
// contiguous per-XCD mapping of every group kernel.
__device__ __forceinline__ int spmv_group(const SolverView& v) {
    return v.gorder ? uniform_load(v.gorder + blockIdx.x) : xcd_group(blockIdx.x, v.G);
}

// Row sums of rows [r0, r1) of H x.  Owner o = 3 (row - r0) + c is thread
// o (acc[0]) or o - 256 (acc[1]); 3 (r1 - r0) <= 512.  prod: 3 * kPlane LDS.
// kLds: x of the columns r0 .. r1 - 1 is read from xs (LDS), the others
// through X.  first: chunk_cols(ci, rp[r0], rp[r1]), which the caller may
// load early.
template <typename T, bool kPlanar, typename X, bool kLds = false>
__device__ __forceinline__ void stream_rows(const int* __restrict__ rp, const int* __restrict__ ci,
                                            Blocks<T, kPlanar> H, X x, int r0, int r1, double* prod,
                                            double (&acc)[2], const ChunkCols& first, const double* xs = nullptr,
                                            const uint16_t* __restrict__ hidx = nullptr) {
    const int t = threadIdx.x;
    const int nown = 3 * (r1 - r0);
    int rb[2], re[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int o = t + q * kThreads;
        acc[q] = 0.0;
        rb[q] = re[q] = 0;
        if (o < nown) {
            const int row = r0 + o / 3;
            rb[q] = rp[row];
            re[q] = rp[row + 1];
        }
    }
    const int kb = uniform_load(rp + r0), ke = uniform_load(rp + r1);
    ChunkCols nc = first;
    for (int cs = kb; cs < ke; cs += kChunk) {
        const int ce = min(cs + kChunk, ke);
        const ChunkCols cc = nc;
#pragma unroll
        for (int kk = 0; kk < kRowPer; ++kk) {
            const int k = cs + t + kk * kThreads;
            if (k >= ce) break;
            const int j = cc.j[kk];
            double x0, x1, x2;
            const int jl = j - r0;
            if (kLds && jl >= 0 && jl < r1 - r0) {
                x0 = xs[3 * jl];
                x1 = xs[3 * jl + 1];
                x2 = xs[3 * jl + 2];
            } else {
                const int h = 3 * cc.h[kk];
                x0 = x.at(3 * j, h);
                x1 = x.at(3 * j + 1, h + 1);
                x2 = x.at(3 * j + 2, h + 2);
            }
            const int e = k - cs;
            prod[e] = H.at(k, 0) * x0 + H.at(k, 1) * x1 + H.at(k, 2) * x2;
            prod[kPlane + e] = H.at(k, 3) * x0 + H.at(k, 4) * x1 + H.at(k, 5) * x2;
            prod[2 * kPlane + e] = H.at(k, 6) * x0 + H.at(k, 7) * x1 + H.at(k, 8) * x2;
        }
        nc = chunk_cols<X::kUnits>(ci, cs + kChunk, ke, hidx);  // the next chunk's columns, in flight through the sums
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int o = t + q * kThreads;
            if (o < nown) {
                const int c = o % 3;
                const int lo = max(rb[q], cs), hi = min(re[q], ce);
                acc[q] = sum_run(acc[q], prod + c * kPlane, lo - cs, hi - cs);
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------- symmetric storage
// Group-symmetric storage: a group keeps one copy of each internal block
// pair (the block with column >= row), used for both H_ij and H_ji = H_ij^T,
// and its blocks with a column outside the group.  Per chunk of stored blocks
// thread t multiplies block t, t + 256, ... by x of its column (to its row,
// prod planes 0..2) and, for an internal off-diagonal block, its transpose by
// x of its row (to its column, planes 3..5).  Owner o = 3 (row - r0) + c then
// adds its row's direct products in column order and its transposed entries
// in stored order.  xs: x on the group's own slots (LDS); external columns
// are gathered through X; tl: the group's transposed entries (LDS).
constexpr int kSymChunk = 512;
constexpr int kSymPlane = kSymChunk + kPad;
constexpr int kTlRegs = 4;  // transposed-list entries a thread loads ahead (a longer list's rest is loaded late)
constexpr int kSymPer = kSymChunk / kThreads;

// Column slot and local row of this thread's stored blocks t, t + 256, ...
// of the chunk starting at cs, loaded one chunk ahead (as chunk_cols).
struct SymCols {
    int j[kSymPer];
    int r[kSymPer];
    int h[kSymPer];  // local unit of each column (kUnits)
};

template <bool kUnits = false>
__device__ __forceinline__ SymCols sym_cols(const SolverView& v, int cs, int ke) {
    SymCols c;
#pragma unroll
    for (int kk = 0; kk < kSymPer; ++kk) c.j[kk] = c.r[kk] = c.h[kk] = 0;
    if (cs < ke) {
#pragma unroll
        for (int kk = 0; kk < kSymPer; ++kk) {
            const int k = min(cs + static_cast<int>(threadIdx.x) + kk * kThreads, ke - 1);
            c.j[kk] = v.sci[k];
            c.r[kk] = v.srow[k];
            if constexpr (kUnits) c.h[kk] = v.hidx[k];
        }
    }
    return c;
}

template <typename T, typename X>
__device__ __forceinline__ void stream_sym(const SolverView& v, const T* __restrict__ H, X xg, const double* xs,
                                           const int* tl, int tb0, int r0, int r1, double* prod, double (&acc)[2],
                                           const SymCols& first) {
    const int t = threadIdx.x;
    const int nown = 3 * (r1 - r0), rows = r1 - r0;
    const long long st = v.nsb;
    int rb[2], re[2], tp[2], te[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int o = t + q * kThreads;
        acc[q] = 0.0;
        rb[q] = re[q] = tp[q] = te[q] = 0;
        if (o < nown) {
            const int row = r0 + o / 3;
            rb[q] = v.srp[row];
            re[q] = v.srp[row + 1];
            tp[q] = v.tptr[row] - tb0;
            te[q] = v.tptr[row + 1] - tb0;
        }
    }
    const int kb = uniform_load(v.srp + r0), ke = uniform_load(v.srp + r1);
    SymCols nc = first;
    for (int cs = kb; cs < ke; cs += kSymChunk) {
        const int ce = min(cs + kSymChunk, ke);
        const SymCols cc = nc;
#pragma unroll
        for (int kk = 0; kk < kSymPer; ++kk) {
            const int k = cs + t + kk * kThreads;
            if (k >= ce) break;
            const int j = cc.j[kk];
            const int r = cc.r[kk];
            const int jl = j - r0;
            const bool internal = jl >= 0 && jl < rows;
            double x0, x1, x2;
            if (internal) {
                x0 = xs[3 * jl];
                x1 = xs[3 * jl + 1];
                x2 = xs[3 * jl + 2];
            } else {
                const int h = 3 * cc.h[kk];
                x0 = xg.at(3 * j, h);
                x1 = xg.at(3 * j + 1, h + 1);
                x2 = xg.at(3 * j + 2, h + 2);
            }
            const double h0 = static_cast<double>(H[k]), h1 = static_cast<double>(H[st + k]),
                         h2 = static_cast<double>(H[2 * st + k]), h3 = static_cast<double>(H[3 * st + k]),
                         h4 = static_cast<double>(H[4 * st + k]), h5 = static_cast<double>(H[5 * st + k]),
                         h6 = static_cast<double>(H[6 * st + k]), h7 = static_cast<double>(H[7 * st + k]),
                         h8 = static_cast<double>(H[8 * st + k]);
            const int e = k - cs;
            prod[e] = h0 * x0 + h1 * x1 + h2 * x2;
            prod[kSymPlane + e] = h3 * x0 + h4 * x1 + h5 * x2;
            prod[2 * kSymPlane + e] = h6 * x0 + h7 * x1 + h8 * x2;
            if (internal && jl != r) {
                const double y0 = xs[3 * r], y1 = xs[3 * r + 1], y2 = xs[3 * r + 2];
                prod[3 * kSymPlane + e] = h0 * y0 + h3 * y1 + h6 * y2;
                prod[4 * kSymPlane + e] = h1 * y0 + h4 * y1 + h7 * y2;
                prod[5 * kSymPlane + e] = h2 * y0 + h5 * y1 + h8 * y2;
            }
        }
        nc = sym_cols<X::kUnits>(v, cs + kSymChunk, ke);  // the next chunk's columns, in flight through the sums
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int o = t + q * kThreads;
            if (o < nown) {
                const int c = o % 3;
                const int lo = max(rb[q], cs), hi = min(re[q], ce);
                acc[q] = sum_run(acc[q], prod + c * kSymPlane, lo - cs, hi - cs);
                acc[q] = sum_listed(acc[q], prod + (3 + c) * kSymPlane, tl, tp[q], te[q], cs, ce);
            }
        }
        __syncthreads();
    }
}

// y = H x for a caller's matrix, nine consecutive values per block.  A wave
// takes a few rows, whose blocks are contiguous, 64 blocks at a time: it
// loads the 576 values as they lie (512 bytes per load; with a thread reading
// the nine values of its own block, 72 bytes apart, the L1 had 64 lines to
// look up per load, and that set the time), turns them in LDS, multiplies one
// block per lane and parks the products in LDS, where one lane per (row,
// component) adds them in column order.  Waves share nothing, so no barrier
// holds them in step.  A workgroup whose rows hold more than kLongRows blocks
// (long contact or body rows), or one of whose waves would have more than half
// of them and a chain of many batches, streams them with all its waves
// instead (20,000 rows of 13 blocks with a few of 300 / 700 / 1,500, FP64: 11.4
// / 19.6 / 36.1 -> 9.8 / 16.1 / 28.8 us, FP32 10.6 / 18.9 / 35.5 -> 10.9 / 16.1 /
// 28.5; the look at the waves costs 48^3 3 %, so it starts where one can have
// such a chain at all).
// 48^3, back to back on cached data: FP64 22.7 -> 19.1 us (6.4 TB/s), FP32 15.4
// -> 14.0.  Four rows a wave and one batch between two sums for FP64, eight
// and two for FP32 (FP64 with eight and two 4 % slower, FP32 with four and one
// 6 %).
template <typename T>
struct UserShape {
    static constexpr int rows = sizeof(T) == 8 ? 4 : 8;     // of a wave
    static constexpr int batches = sizeof(T) == 8 ? 1 : 2;  // of 64 blocks between two sums
    static constexpr int plane = 64 * batches + kPad;
    static constexpr int group = rows * (kThreads / 64);    // rows of a workgroup
    static constexpr int uneven = 64 * rows;                // blocks of a wave that may exceed those of the others together
};
constexpr int kLongRows = 2048;

template <typename T>
__device__ __forceinline__ void wave_rows(const int* __restrict__ rp, const int* __restrict__ ci,
                                          const T* __restrict__ val, const double* __restrict__ x,
                                          double* __restrict__ y, int r0, int r1, T* stage, double* prod) {
    constexpr int kBatches = UserShape<T>::batches, kWavePlane = UserShape<T>::plane;
    const int lane = threadIdx.x & 63;
    const int nown = 3 * (r1 - r0);
    const int row = r0 + min(lane, nown - 1) / 3, c = lane % 3;
    const int rb = rp[row], re = rp[row + 1];
    const int kb = uniform_load(rp + r0), ke = uniform_load(rp + r1);
    double acc = 0.0;
    for (int cs = kb; cs < ke; cs += 64 * kBatches) {
        T h[kBatches][9];
        int j[kBatches];
#pragma unroll
        for (int b = 0; b < kBatches; ++b) {
            const int k0 = min(cs + 64 * b, ke - 1);
            const long long last = 9LL * ke - 1;
            j[b] = ci[min(k0 + lane, ke - 1)];
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const long long e = 9LL * k0 + 64 * i + lane;
                h[b][i] = val[e < last ? e : last];
            }
        }
        double xv[kBatches][3];
#pragma unroll
        for (int b = 0; b < kBatches; ++b)
#pragma unroll
            for (int i = 0; i < 3; ++i) xv[b][i] = x[3LL * j[b] + i];
#pragma unroll
        for (int b = 0; b < kBatches; ++b) {
            if (cs + 64 * b >= ke) break;
#pragma unroll
            for (int i = 0; i < 9; ++i) stage[64 * i + lane] = h[b][i];
            wave_lds_sync();
            double v[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) v[i] = static_cast<double>(stage[9 * lane + i]);
            wave_lds_sync();
            const int e = 64 * b + lane;
#pragma unroll
            for (int i = 0; i < 3; ++i)
                prod[i * kWavePlane + e] = v[3 * i] * xv[b][0] + v[3 * i + 1] * xv[b][1] + v[3 * i + 2] * xv[b][2];
        }
        wave_lds_sync();
        const int ce = min(cs + 64 * kBatches, ke);
        if (lane < nown) acc = sum_run(acc, prod + c * kWavePlane, max(rb, cs) - cs, min(re, ce) - cs);
        wave_lds_sync();
    }
    if (lane < nown) y[3LL * r0 + lane] = acc;
}

template <typename T>
__global__ void __launch_bounds__(kThreads) k_spmv_user(int n_rows, const int* __restrict__ rp,
                                                         const int* __restrict__ ci, const T* __restrict__ val,
                                                         const double* __restrict__ x, double* __restrict__ y) {
    constexpr int kWaves = kThreads / 64;
    constexpr int kStage = 576 * sizeof(T) / sizeof(double);
    constexpr int kPerWave = kStage + 3 * UserShape<T>::plane;
    constexpr int kWaveRows = UserShape<T>::rows, kUserRows = UserShape<T>::group;
    __shared__ double sm[kWaves * kPerWave > 3 * kPlane ? kWaves * kPerWave : 3 * kPlane];
    const int g = xcd_group(blockIdx.x, gridDim.x);  // neighbouring rows, which share entries of x, on one XCD
    const int r0 = g * kUserRows, r1 = min(r0 + kUserRows, n_rows);
    const int kb = uniform_load(rp + r0), ke = uniform_load(rp + r1);
    bool waves = ke - kb <= kLongRows;
    if (waves && ke - kb > UserShape<T>::uneven) {
        int longest = 0;
#pragma unroll
        for (int w = 0, k0 = kb; w < kWaves; ++w) {
            const int k1 = uniform_load(rp + min(r0 + (w + 1) * kWaveRows, r1));
            longest = max(longest, k1 - k0);
            k0 = k1;
        }
        waves = longest <= UserShape<T>::uneven || 2 * longest <= ke - kb;
    }
    if (waves) {
        const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int w0 = r0 + w * kWaveRows, w1 = min(w0 + kWaveRows, r1);
        if (w0 < w1)
            wave_rows<T>(rp, ci, val, x, y, w0, w1, reinterpret_cast<T*>(sm + w * kPerWave), sm + w * kPerWave + kStage);
        return;
    }
    double acc[2];
    stream_rows<T, false>(rp, ci, Blocks<T, false>{val, 0}, XVec{x}, r0, r1, sm, acc, chunk_cols(ci, kb, ke));
    const int t = threadIdx.x;
    if (t < 3 * (r1 - r0)) y[3LL * r0 + t] = acc[0];
}

// Products per launch after the stream: q of the group's rows, the partials
// of p_k^T q and r^T p_k (rp) and, with kRQ > 0 (writer passes), the
// restriction of q to the coarse levels (q1 and qpart, as restrict_group computes C_l r) from
// the plan pl loaded at the kernel's start, staged in the product planes
// (free once the stream's last barrier has passed; the host checks that
// they hold it, spmv_restrict_capacity).
template <int kRQ>
__device__ __forceinline__ void finish_pq(const SolverView& v, int g, int nown, int r0, double* __restrict__ qk,
                                          const double (&acc)[2],
                                          const double (&pv)[2], double rp, double* prod, double* buf,
                                          const RestrictLoads<kRQ ? kRQ : 1>& pl) {
    const int t = threadIdx.x;
    if constexpr (kRQ) restrict_ready(pl);
    double part = 0.0;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int o = t + q * kThreads;
        if (o < nown) {
            qk[3LL * r0 + o] = acc[q];
            part += pv[q] * acc[q];
        }
    }
    if constexpr (kRQ) {
        double* rs = prod;
        double* rsm = prod + 3 * v.RG;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int o = t + q * kThreads;
            if (o < 3 * v.RG) rs[o] = o < nown ? acc[q] : 0.0;
        }
        double sigma, srp;
        block_sum2(part, rp, buf, sigma, srp);  // its barriers also publish rs
        if (t == 0) v.P_sp[g] = {sigma, srp};
        restrict_group<true>(v, g, pl, rs, rsm, v.q1, v.qpart);  // the host checked restrict_passes
    } else {
        double sigma, srp;
        block_sum2(part, rp, buf, sigma, srp);
        if (t == 0) v.P_sp[g] = {sigma, srp};
    }
}

// The coarse corrections of a group's level-1 units (kSplit), in LDS: y_1 at
// the unit plus the sum over the levels >= 2 of y_l at its ancestors, the same
// sum in every group that reads the unit.  The levels >= 2 are summed once per
// distinct level-2 unit (at 48^3 a group reads about 76 units under 23 of
// them).  unit_load issues a thread's table loads (level-2 entry t / 3,
// component t % 3; units t and t + 256), unit_gather the corrections they
// name; unit_stage adds up, takes what is left over, and leaves the sums in
// ycor.  The two round trips overlap the rho sum.  Every load of the two is
// unconditional, at clamped indices: a branch around one would wait for it.
constexpr int kUnitLevels = 7;     // levels >= 2 whose corrections a thread loads ahead
constexpr int kUnitTables = 14;    // levels >= 2 whose positions it loads ahead (all of them)
constexpr int kUnits = 2;          // units whose corrections it loads ahead
static_assert(kUnitTables >= kMaxLv - 2 && kUnits * kThreads >= kMaxHalo,
              "only level-2 entries can be left over");

struct UnitLoads {
    int n, n2, nl;   // units and level-2 entries of the group, levels >= 2
    const int* pos;  // position of entry i at level 2 + l: pos[l n2 + i]
    int at[kUnitTables], u[kUnits], par[kUnits];
    double y[kUnitLevels], y1[kUnits][3];
};

__device__ __forceinline__ UnitLoads unit_load(const SolverView& v, int g) {
    UnitLoads U;
    const int t = threadIdx.x;
    const int h0 = uniform_load(v.hptr + g), q0 = uniform_load(v.h2ptr + g);
    U.n = uniform_load(v.hptr + g + 1) - h0;
    U.n2 = uniform_load(v.h2ptr + g + 1) - q0;
    U.nl = max(v.L - 2, 0);
    // (no level >= 2, no unit: stand-ins with entries)
    U.pos = U.n2 > 0 ? v.hy + static_cast<long long>(U.nl) * q0 : v.hptr;
    const int* hu = U.n > 0 ? v.hu + h0 : v.hptr;
    const uint16_t* hpar = U.n > 0 ? v.hpar + h0 : reinterpret_cast<const uint16_t*>(v.hptr);
    const int i2 = max(min(t / 3, U.n2 - 1), 0), last = max(U.nl - 1, 0);
#pragma unroll
    for (int l = 0; l < kUnitTables; ++l) U.at[l] = U.pos[min(l, last) * U.n2 + i2];
#pragma unroll
    for (int q = 0; q < kUnits; ++q) {
        const int i = max(min(t + q * kThreads, U.n - 1), 0);
        U.u[q] = hu[i];
        U.par[q] = hpar[i];
    }
    return U;
}

__device__ __forceinline__ void unit_gather(const SolverView& v, UnitLoads& U) {
    const int c = threadIdx.x % 3;
    const double* y = U.n > 0 ? v.yall : v.z;
    const int keep = U.n > 0 ? -1 : 0, keep2 = U.n2 > 0 ? -1 : 0;  // (stand-ins name no position)
#pragma unroll
    for (int l = 0; l < kUnitLevels; ++l) U.y[l] = y[3LL * (U.at[l] & keep2) + c];
#pragma unroll
    for (int q = 0; q < kUnits; ++q)
#pragma unroll
        for (int e = 0; e < 3; ++e) U.y1[q][e] = y[3LL * (U.u[q] & keep) + e];
}

// ycor: 3 maxH doubles, then 3 maxH2 for the level-2 sums.  Ends with a
// barrier.  buf: the rho buckets the caller has written, folded on the way
// into buf[0] (by the last wave, which has the least to stage).
__device__ __forceinline__ void unit_stage(const SolverView& v, const UnitLoads& U, double* ycor, double* buf) {
    const int t = threadIdx.x;
    double* up = ycor + 3 * v.maxH;
    // sum of y_l over kUnitLevels levels from 2 + l0 on, positions at
    auto levels = [&](double s, const int* at, int l0, int c) {
        double y[kUnitLevels];
#pragma unroll
        for (int l = 0; l < kUnitLevels; ++l) y[l] = v.yall[3LL * at[l] + c];
#pragma unroll
        for (int l = 0; l < kUnitLevels; ++l)
            if (l0 + l < U.nl) s += y[l];
        return s;
    };
    if (U.n == 0 && t < 3) ycor[t] = 0.0;  // no coarse levels: every block names unit 0
    if (t < 3 * U.n2) {
        double s = 0.0;
#pragma unroll
        for (int l = 0; l < kUnitLevels; ++l)
            if (l < U.nl) s += U.y[l];
        if (U.nl > kUnitLevels) s = levels(s, U.at + kUnitLevels, kUnitLevels, t % 3);
        up[t] = s;
    }
    for (int e = t + kThreads; e < 3 * U.n2; e += kThreads) {
        const int i = e / 3, c = e - 3 * i;
        int at[kUnitTables];
#pragma unroll
        for (int l = 0; l < kUnitTables; ++l) at[l] = U.pos[min(l, U.nl - 1) * U.n2 + i];
        double s = levels(0.0, at, 0, c);
        if (U.nl > kUnitLevels) s = levels(s, at + kUnitLevels, kUnitLevels, c);
        up[e] = s;
    }
    __syncthreads();
    if (t >= kThreads - 64) partials_fold(buf);
#pragma unroll
    for (int q = 0; q < kUnits; ++q) {
        const int i = t + q * kThreads;
        if (i < U.n) {
#pragma unroll
            for (int e = 0; e < 3; ++e) ycor[3 * i + e] = U.nl > 0 ? U.y1[q][e] + up[3 * U.par[q] + e] : U.y1[q][e];
        }
    }
    __syncthreads();
}

// The group's own units are the first of its list: local unit of slot s,
// negative for an empty slot or without coarse levels (remap: a stand-in).
__device__ __forceinline__ int own_unit(const SolverView& v, int g, int slot) {
    const int u = (v.L > 1 ? v.anc : v.remap)[slot] - uniform_load(v.g_u1 + g);
    return v.L > 1 ? u : -1;
}

constexpr int kRhoPer = 8;  // rho partials a thread loads ahead: up to 2048 in all

// PCG iteration k over the solver's group of slots: the new direction
// p_k = z_{k-1} + beta_{k-1} p_{k-1} (beta = rho_{k-1} / rho_{k-2} summed from
// the partials; p_1 = z_0) on the group's own slots, q_k = H p_k and the
// partials of p_k^T q_k and r_{k-1}^T p_k.
//
// The direction is staged in LDS on the group's own slots and formed wherever H
// gathers it, with the same beta and the same fused multiply-add, so the same
// bits, in every workgroup.  (Formed by the recurrence q_k = H z_{k-1} + beta
// q_{k-1}, which gathers z alone, the product takes 1.4 us less at 48^3, but
// what it carries on costs the solution of a sheet with bodies up to 20 times
// its accuracy, even with q formed afresh every 50 iterations.)
//
// kSplit: z_{k-1} = v.z + the coarse corrections, which the level-0 apply left
// out so that it need not wait for the coarse levels.  A group reads few
// distinct level-1 units, so it sums each unit's levels once into LDS
// (unit_stage); an outside column then costs one 16-bit index and three LDS
// reads more.
struct DirLoads {
    double z[2], p[2], r[2];
    int unit[2];
};

template <bool kSplit>
__device__ __forceinline__ DirLoads dir_load(const SolverView& v, int g, int r0, int nown, const double* pold) {
    DirLoads D;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int o = min(static_cast<int>(threadIdx.x) + q * kThreads, nown - 1);
        const long long e = 3LL * r0 + o;
        D.z[q] = v.z[e];
        D.p[q] = pold[e];
        D.r[q] = v.r[e];
        D.unit[q] = kSplit ? own_unit(v, g, r0 + o / 3) : -1;
    }
    return D;
}

// rho_{k-1} and beta, the own part of p_k in xs and stored; pv: p_k at the
// thread's rows; rp: its part of r_{k-1}^T p_k.  Ends with a barrier.
template <bool kSplit>
__device__ __forceinline__ double dir_stage(const SolverView& v, int k, int g, int r0, int nown, DirLoads& D,
                                            const PartialLoads<kSplit ? kRhoPer : 4>& rl, int nrho, double rk2,
                                            const UnitLoads& U, double* ycor, double* xs, double* buf,
                                            double (&pv)[2], double& rp) {
    const int t = threadIdx.x;
    rp = 0.0;
    const double* Prho = v.P_rho[(k - 1) & 1];
    partials_bucket<kSplit ? kRhoPer : 4>(rl, Prho, nrho, buf);
    if constexpr (kSplit) {
        unit_stage(v, U, ycor, buf);
    } else {
        __syncthreads();
        if (t < 64) partials_fold(buf);
        __syncthreads();
    }
    const double rk1 = buf[0];  // buf is next written after later barriers
    if (g == 0 && t == 0) v.st->rho[(k - 1) & 1] = rk1;
    const double beta = k > 1 && rk2 != 0.0 ? rk1 / rk2 : 0.0;  // (r^T z underflows before r does)
    double* pk = v.p[k & 1];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int o = t + q * kThreads;
        pv[q] = 0.0;
        if (o < nown) {
            double z = D.z[q];
            if (kSplit && D.unit[q] >= 0) z += ycor[3 * D.unit[q] + o % 3];
            pv[q] = __fma_rn(beta, D.p[q], z);
            pk[3LL * r0 + o] = pv[q];
            rp += D.r[q] * pv[q];
        }
        if (o < 3 * v.RG) xs[o] = pv[q];
    }
    __syncthreads();
    return beta;
}

template <typename T, int kRQ, bool kSplit>
__global__ void __launch_bounds__(kThreads) k_spmv_pq(SolverView v, const T* __restrict__ H, int k, int nrho,
                                                      int flags) {
    __shared__ double prod[3 * kPlane];
    __shared__ double buf[256];
    extern __shared__ double dyn[];  // xs[3 RG] (+ ycor[3 (maxH + maxH2)])
    if (kSplit && static_cast<int>(blockIdx.x) >= v.G) {  // one workgroup more takes the decision on r_{k-1}
        convergence_decision(v, false, k - 1, 0.0, flags, v.GA, spmv_mark(k), buf);
        return;
    }
    const int g = spmv_group(v);
    const int r0 = g * v.RG, r1 = min(r0 + v.RG, v.NS);
    const int nown = 3 * (r1 - r0);
    double* xs = dyn;
    double* ycor = dyn + 3 * v.RG;
    // every independent load before the first wait, unconditionally at
    // clamped indices (see partials_load); k = 1 has no p_0 (beta = 0)
    const double* pold = k > 1 ? v.p[(k - 1) & 1] : v.z;
    UnitLoads U{};
    if constexpr (kSplit) U = unit_load(v, g);
    const auto rl = partials_load<kSplit ? kRhoPer : 4>(v.P_rho[(k - 1) & 1], nrho);
    DirLoads D = dir_load<kSplit>(v, g, r0, nown, pold);
    const ChunkCols c0 = chunk_cols<kSplit>(v.ci0, uniform_load(v.rp0 + r0), uniform_load(v.rp0 + r1), v.hidx);
    RestrictLoads<kRQ ? kRQ : 1> pl{};
    if constexpr (kRQ) pl = restrict_load<kRQ>(v, g);
    const int stop = uniform_load(&v.st->done);
    keep_loads_issued();
    if (stopped_before<kSplit>(stop, k)) return;  // after a stop nothing is written
    const double rk2 = uniform_load(&v.st->rho[k & 1]);  // rho_{k-2} as the previous SpMV recorded it
    if constexpr (kSplit) unit_gather(v, U);
    double pv[2], acc[2], rp;
    const double beta = dir_stage<kSplit>(v, k, g, r0, nown, D, rl, nrho, rk2, U, ycor, xs, buf, pv, rp);
    const Blocks<T, true> Hb{H, v.nnzb};
    stream_rows<T, true, XDir<kSplit>, true>(v.rp0, v.ci0, Hb, XDir<kSplit>{v.z, pold, beta, ycor}, r0, r1, prod, acc,
                                             c0, xs, v.hidx);
    finish_pq<kRQ>(v, g, nown, r0, v.q, acc, pv, rp, prod, buf, pl);
}

// k_spmv_pq on the group-symmetric storage.
template <typename T, int kRQ, bool kSplit>
__global__ void __launch_bounds__(kThreads) k_spmv_pq_sym(SolverView v, const T* __restrict__ H, int k, int nrho,
                                                          int flags) {
    __shared__ double prod[6 * kSymPlane];
    __shared__ double buf[256];
    extern __shared__ double dyn[];  // xs[3 RG] doubles (+ ycor[3 (maxH + maxH2)]) + tl[maxT] ints
    if (kSplit && static_cast<int>(blockIdx.x) >= v.G) {  // one workgroup more takes the decision on r_{k-1}
        convergence_decision(v, false, k - 1, 0.0, flags, v.GA, spmv_mark(k), buf);
        return;
    }
    const int t = threadIdx.x;
    const int g = spmv_group(v);
    const int r0 = g * v.RG, r1 = min(r0 + v.RG, v.NS);
    const int nown = 3 * (r1 - r0);
    double* xs = dyn;
    double* ycor = dyn + 3 * v.RG;
    int* tl = reinterpret_cast<int*>(ycor + (kSplit ? 3 * (v.maxH + v.maxH2) : 0));
    // loads as in k_spmv_pq, and the group's transposed-entry list, which
    // goes to LDS with the own part
    const double* pold = k > 1 ? v.p[(k - 1) & 1] : v.z;
    UnitLoads U{};
    if constexpr (kSplit) U = unit_load(v, g);
    const auto rl = partials_load<kSplit ? kRhoPer : 4>(v.P_rho[(k - 1) & 1], nrho);
    DirLoads D = dir_load<kSplit>(v, g, r0, nown, pold);
    const int tb0 = uniform_load(v.tptr + r0), tn = uniform_load(v.tptr + r1) - tb0;
    const int* tsrc = tn > 0 ? v.tidx + tb0 : v.srp;  // srp: a stand-in with entries when the list is empty
    int tlr[kTlRegs];
#pragma unroll
    for (int j = 0; j < kTlRegs; ++j) tlr[j] = tsrc[min(t + j * kThreads, max(tn - 1, 0))];
    const SymCols c0 = sym_cols<kSplit>(v, uniform_load(v.srp + r0), uniform_load(v.srp + r1));
    RestrictLoads<kRQ ? kRQ : 1> pl{};
    if constexpr (kRQ) pl = restrict_load<kRQ>(v, g);
    const int stop = uniform_load(&v.st->done);
    keep_loads_issued();
    if (stopped_before<kSplit>(stop, k)) return;  // after a stop nothing is written
    const double rk2 = uniform_load(&v.st->rho[k & 1]);  // rho_{k-2} as the previous SpMV recorded it
    if constexpr (kSplit) unit_gather(v, U);
#pragma unroll
    for (int j = 0; j < kTlRegs; ++j)
        if (t + j * kThreads < tn) tl[t + j * kThreads] = tlr[j];
    for (int e = t + kTlRegs * kThreads; e < tn; e += kThreads) tl[e] = v.tidx[tb0 + e];
    double pv[2], acc[2], rp;
    const double beta = dir_stage<kSplit>(v, k, g, r0, nown, D, rl, nrho, rk2, U, ycor, xs, buf, pv, rp);
    stream_sym<T>(v, H, XDir<kSplit>{v.z, pold, beta, ycor}, xs, tl, tb0, r0, r1, prod, acc, c0);
    finish_pq<kRQ>(v, g, nown, r0, v.q, acc, pv, rp, prod, buf, pl);
}

// out = b - H x in FP64 over a group, with the partials of ||out||^2 (and
// ||b||^2 for the initial residual) and, except for the final check, the
// restriction of the new residual to the coarse levels.
template <int kMode, bool kSym>
__global__ void __launch_bounds__(kThreads) k_residual(SolverView v, double* __restrict__ out) {
    __shared__ double prod[(kSym ? 6 * kSymPlane : 3 * kPlane)];
    __shared__ double scratch[kThreads / 64];
    extern __shared__ double dyn[];  // rs[3*RG] + restriction scratch (+ xs[3*RG] + tl[maxT] ints)
    if (kMode == kResidReplace && v.st->done) return;
    const int g = spmv_group(v);
    const int r0 = g * v.RG, r1 = min(r0 + v.RG, v.NS);
    double acc[2];
    const RestrictLoads<> pl = restrict_load(v, g);
    if constexpr (kSym) {
        double* xs = dyn + 3 * v.RG + restrict_smem_doubles(v.RG, v.W1, v.L);
        int* tl = reinterpret_cast<int*>(xs + 3 * v.RG);
        const int nown = 3 * (r1 - r0);
        for (int o = threadIdx.x; o < 3 * v.RG; o += kThreads) xs[o] = o < nown ? v.x[3LL * r0 + o] : 0.0;
        const int tb0 = v.tptr[r0], tn = v.tptr[r1] - tb0;
        for (int e = threadIdx.x; e < tn; e += kThreads) tl[e] = v.tidx[tb0 + e];
        __syncthreads();
        stream_sym<double>(v, v.H64, XVec{v.x}, xs, tl, tb0, r0, r1, prod, acc, sym_cols(v, v.srp[r0], v.srp[r1]));
    } else {
        stream_rows<double, true>(v.rp0, v.ci0, Blocks<double, true>{v.H64, v.nnzb}, XVec{v.x}, r0, r1, prod, acc,
                                  chunk_cols(v.ci0, v.rp0[r0], v.rp0[r1]));
    }
    restrict_ready(pl);
    double rr = 0.0, bb = 0.0;
    double* rs = dyn;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int o = threadIdx.x + q * kThreads;
        if (o < 3 * v.RG) {
            double e = 0.0;
            if (o < 3 * (r1 - r0)) {
                const long long i = 3LL * r0 + o;
                const double bv = v.b[i];
                e = bv - acc[q];
                out[i] = e;
                rr += e * e;
                bb += bv * bv;
            }
            rs[o] = e;
        }
    }
    rr = block_sum(rr, scratch);  // its barriers also publish rs
    if (kMode == kResidInit) bb = block_sum(bb, scratch);
    if (threadIdx.x == 0) {
        v.P_rr[g] = rr;
        if (kMode == kResidInit) v.P_bb[g] = bb;
    }
    if (kMode != kResidFinal) restrict_group_any(v, g, pl, rs, dyn + 3 * v.RG, v.r1, v.cpart);
}

}  // namespace

hipError_t launch_spmv_user(int n_rows, const int* rp, const int* ci, const void* val, bool f32, const double* x,
                            double* y, hipStream_t s) {
    if (n_rows <= 0) return hipSuccess;
    const dim3 b(kThreads);
    if (f32)
        launch_kernel(k_spmv_user<float>, dim3(ceil_div(n_rows, UserShape<float>::group)), b, 0, s, n_rows, rp, ci,
                      static_cast<const float*>(val), x, y);
    else
        launch_kernel(k_spmv_user<double>, dim3(ceil_div(n_rows, UserShape<double>::group)), b, 0, s, n_rows, rp, ci,
                      static_cast<const double*>(val), x, y);
    return hipGetLastError();
}

template <int kRQ, bool kSplit>
void launch_spmv_pq_t(const SolverView& v, bool f32, int k, bool rec, hipStream_t s) {
    dim3 g(v.G + (kSplit ? 1 : 0)), b(kThreads);
    const int flags = f32 ? kFlagMixed : 0, nrho = rec ? v.GA + v.ncb : v.GA;
    const size_t vec = sizeof(double) * 3 * (static_cast<size_t>(v.RG) + (kSplit ? v.maxH + v.maxH2 : 0));
    if (v.sym && !f32) {
        launch_kernel(k_spmv_pq_sym<double, kRQ, kSplit>, g, b, vec + sizeof(int) * v.maxT, s, v,
                      static_cast<const double*>(v.H64), k, nrho, flags);
    } else if (f32) {
        launch_kernel(k_spmv_pq<float, kRQ, kSplit>, g, b, vec, s, v, static_cast<const float*>(v.H32), k,
                      nrho, flags);
    } else {
        launch_kernel(k_spmv_pq<double, kRQ, kSplit>, g, b, vec, s, v, static_cast<const double*>(v.H64), k,
                      nrho, flags);
    }
}

hipError_t launch_spmv_pq(const SolverView& v, bool f32, int k, bool restrict_q, bool rec, bool split,
                          hipStream_t s) {
    static_assert(kMaxRestrictPasses == 2, "one instance per pass count");
    const int rq = restrict_q ? v.rpass : 0;
    if ((restrict_q && rq == 0) || (split && !rec)) return hipErrorInvalidValue;
    if (rq == 1) {
        split ? launch_spmv_pq_t<1, true>(v, f32, k, rec, s) : launch_spmv_pq_t<1, false>(v, f32, k, rec, s);
    } else if (rq == 2) {
        split ? launch_spmv_pq_t<2, true>(v, f32, k, rec, s) : launch_spmv_pq_t<2, false>(v, f32, k, rec, s);
    } else {
        split ? launch_spmv_pq_t<0, true>(v, f32, k, rec, s) : launch_spmv_pq_t<0, false>(v, f32, k, rec, s);
    }
    return hipGetLastError();
}

size_t spmv_shared_bytes(int RG, int maxT, bool sym) {
    return sizeof(double) * (max(3 * kPlane, 6 * kSymPlane) + 256 + 3 * static_cast<size_t>(RG)) +
           (sym ? sizeof(int) * static_cast<size_t>(maxT) : 0);
}

int spmv_threads() { return kThreads; }

size_t spmv_restrict_capacity() { return sizeof(double) * static_cast<size_t>(min(3 * kPlane, 6 * kSymPlane)); }

template <bool kSym>
void launch_residual_t(const SolverView& v, int mode, double* out, hipStream_t s) {
    dim3 g(v.G), b(kThreads);
    size_t shmem = sizeof(double) * (3 * v.RG + restrict_smem_doubles(v.RG, v.W1, v.L));
    if (kSym) shmem += sizeof(double) * 3 * v.RG + sizeof(int) * v.maxT;
    switch (mode) {
        case kResidInit: launch_kernel(k_residual<kResidInit, kSym>, g, b, shmem, s, v, out); break;
        case kResidReplace: launch_kernel(k_residual<kResidReplace, kSym>, g, b, shmem, s, v, out); break;
        case kResidConfirm: launch_kernel(k_residual<kResidConfirm, kSym>, g, b, shmem, s, v, out); break;
        default: launch_kernel(k_residual<kResidFinal, kSym>, g, b, shmem, s, v, out); break;
    }
}

hipError_t launch_residual(const SolverView& v, int mode, double* out, hipStream_t s) {
    if (v.sym)
        launch_residual_t<true>(v, mode, out, s);
    else
        launch_residual_t<false>(v, mode, out, s);
    return hipGetLastError();
}

}  // namespace maspcg

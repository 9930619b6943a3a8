// MAS preconditioner on the device: coarse matrices, batched domain
// inversion and the apply (Supp. Eq. 4-6; algorithm "Compute MAS
// preconditioner" in Sec. 4.3).
#include <algorithm>

#include "decision.hpp"
#include "launch.hpp"

namespace maspcg {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

// Inverse entries in the apply.  Full-layout level-0 FP64 inverses (136 MB
// at the 48^3 cube) do not fit the 256 MB MALL next to H, so they are
// streamed with non-temporal loads that leave the caches to H, the vectors
// and the coarse inverses (kStream); the symmetric-packed FP64 set (69 MB),
// the FP32 set of the mixed solve and the coarse levels (16 MB) fit and are
// read through the caches.
template <typename TI, bool kStream = true>
__device__ __forceinline__ double inv_load(const TI* p) {
    if constexpr (sizeof(TI) == 8 && kStream)
        return __builtin_nontemporal_load(p);
    else
        return static_cast<double>(*p);
}

// ------------------------------------------------------------ coarse sums
// A_l = C H C^T by levels (Supp. Eq. 5: A_(l) = C A C^T with unit 3x3
// weights).  Each coarse block owns a list of fine blocks and sums it in a
// fixed order: no atomics, bitwise reproducible.  Nine consecutive threads
// take one coarse block, thread c summing entry c over the list in order,
// four list entries loaded at a time (their indices, then their values), so
// that the list's loads overlap instead of following one another.
constexpr int kSumRound = 4;

__global__ void __launch_bounds__(256) k_coarse_sum_first(int nnzA, const int* __restrict__ ptr,
                                                           const int* __restrict__ src, const double* __restrict__ Hu,
                                                           double* __restrict__ A) {
    const long long gt = static_cast<long long>(blockIdx.x) * 256 + threadIdx.x;
    if (gt >= 9LL * nnzA) return;
    const int t = static_cast<int>(gt / 9), c = static_cast<int>(gt % 9);
    const int qe = ptr[t + 1];
    int q = ptr[t];
    double s = 0.0;
    for (; q + kSumRound <= qe; q += kSumRound) {
        int i[kSumRound];
#pragma unroll
        for (int j = 0; j < kSumRound; ++j) i[j] = src[q + j];
        double a[kSumRound];
#pragma unroll
        for (int j = 0; j < kSumRound; ++j) a[j] = Hu[9LL * i[j] + c];
#pragma unroll
        for (int j = 0; j < kSumRound; ++j) s += a[j];
    }
    for (; q < qe; ++q) s += Hu[9LL * src[q] + c];
    A[static_cast<long long>(c) * nnzA + t] = s;
}

__global__ void __launch_bounds__(256) k_coarse_sum_next(int nnzA, int nnzPrev, const int* __restrict__ ptr,
                                                          const int* __restrict__ src, const double* __restrict__ Ap,
                                                          double* __restrict__ A) {
    const long long gt = static_cast<long long>(blockIdx.x) * 256 + threadIdx.x;
    if (gt >= 9LL * nnzA) return;
    const int t = static_cast<int>(gt / 9), c = static_cast<int>(gt % 9);
    const double* Apc = Ap + static_cast<long long>(c) * nnzPrev;
    const int qe = ptr[t + 1];
    int q = ptr[t];
    double s = 0.0;
    for (; q + kSumRound <= qe; q += kSumRound) {
        int i[kSumRound];
#pragma unroll
        for (int j = 0; j < kSumRound; ++j) i[j] = src[q + j];
        double a[kSumRound];
#pragma unroll
        for (int j = 0; j < kSumRound; ++j) a[j] = Apc[i[j]];
#pragma unroll
        for (int j = 0; j < kSumRound; ++j) s += a[j];
    }
    for (; q < qe; ++q) s += Apc[src[q]];
    A[static_cast<long long>(c) * nnzA + t] = s;
}

// ------------------------------------------------------- domain inversion
// One workgroup of four waves per domain (all levels in one launch).  The
// domain matrix (3N x 3N, padded to 16T with identity rows on empty lanes so
// that the inverse of the occupied part comes out directly) sits in LDS and
// is inverted in place by block Gauss-Jordan over 16x16 tiles:
//   P = inv(A_kk) (register-resident scalar Gauss-Jordan, 16 pivots, wave 0),
//   A_kj <- P A_kj, A_ij <- A_ij - A_ik A_kj, A_ik <- -A_ik P, A_kk <- P,
// with the tile products on v_mfma_f64_16x16x4f64, the tiles of each phase
// dealt round-robin to the four waves.  Pivots are Schur complement
// diagonals of an SPD matrix; a pivot <= 0 flags NOT_SPD.
//
// MFMA f64 16x16x4 lane layout on gfx950: lane l supplies A[l % 16][l / 16]
// and B[l / 16][l % 16]; result register v of lane l is D[l / 16 + 4 v][l % 16].

struct DomTable {
    int off[kMaxLv + 1];  // first workgroup of each level
};

__device__ __forceinline__ int level_of(const DomTable& tab, int L, int g) {
    int l = 0;
    while (l + 1 < L && g >= tab.off[l + 1]) ++l;
    return l;
}

constexpr int kInvWaves = 4;
constexpr int kInvThreads = 64 * kInvWaves;

template <int T>
__global__ void __launch_bounds__(kInvThreads) k_invert(BuildView B, const double* __restrict__ Hu, int want32,
                                                        DomTable tab) {
    constexpr int NP = 16 * T;
    constexpr int LD = NP + 1;  // odd stride: a 16-row column read hits 16 distinct bank pairs
    __shared__ double A[NP * LD];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index, uniform in the wave
    const int l = level_of(tab, B.L, blockIdx.x);
    const int d = blockIdx.x - tab.off[l];
    const int N = B.N, n = 3 * N;

    for (int e = tid; e < NP * LD; e += kInvThreads) A[e] = 0.0;
    __syncthreads();

    // gather the upper in-domain blocks and mirror them
    const int* dptr = B.dom_ptr[l];
    for (int q = dptr[d] + tid; q < dptr[d + 1]; q += kInvThreads) {
        const int k = B.dom_blk[l][q];
        const int ab = B.dom_ab[l][q];
        const int a = ab & 255, b = ab >> 8;
        double v[9];
        if (l == 0) {
#pragma unroll
            for (int c = 0; c < 9; ++c) v[c] = Hu[9LL * k + c];
        } else {
#pragma unroll
            for (int c = 0; c < 9; ++c) v[c] = B.A[l][(long long)c * B.nnzA[l] + k];
        }
        if (a == b) {
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int c = r; c < 3; ++c) {
                    A[(3 * a + r) * LD + 3 * a + c] = v[3 * r + c];
                    A[(3 * a + c) * LD + 3 * a + r] = v[3 * r + c];
                }
        } else {
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    A[(3 * a + r) * LD + 3 * b + c] = v[3 * r + c];
                    A[(3 * b + c) * LD + 3 * a + r] = v[3 * r + c];
                }
        }
    }
    // occupied lanes of this domain as a bit mask (every wave forms the same)
    bool occ_lane = false;
    if (lane < N) {
        const int u = d * N + lane;
        occ_lane = (l == 0) ? (B.remap[u] >= 0) : (u < B.units[l]);
    }
    const unsigned long long occ = __ballot(occ_lane);
    __syncthreads();
    for (int p = tid; p < NP; p += kInvThreads) {
        const bool live = p < n && ((occ >> (p / 3)) & 1ull);
        if (!live) A[p * LD + p] = 1.0;
    }
    __syncthreads();

    const int c16 = lane & 15, g4 = lane >> 4;
    bool ok = true;
#pragma unroll
    for (int k = 0; k < T; ++k) {
        const int base = 16 * k;
        // ---- P = inv(A_kk) by wave 0: lane holds column c16, rows 4 g4 + v
        if (w == 0) {
            double a[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) a[v] = A[(base + 4 * g4 + v) * LD + base + c16];
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int jg = j >> 2, jv = j & 3;
                const double aj = a[jv];
                const double piv = __shfl(aj, jg * 16 + j);
                const double rowj = __shfl(aj, jg * 16 + c16);
                double colj[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) colj[v] = __shfl(a[v], g4 * 16 + j);
                ok = ok && (piv > 0.0) && finite(piv);
                const double inv = 1.0 / piv;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 4 * g4 + v;
                    if (i == j)
                        a[v] = (c16 == j) ? inv : a[v] * inv;
                    else
                        a[v] = (c16 == j) ? -colj[v] * inv : a[v] - colj[v] * rowj * inv;
                }
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) A[(base + 4 * g4 + v) * LD + base + c16] = a[v];
        }
        __syncthreads();
        // ---- row panel: A_kj <- P A_kj, tile j (j != k) to wave (its rank) % 4
#pragma unroll
        for (int j = 0; j < T; ++j) {
            if (j == k || (j - (j > k)) % kInvWaves != w) continue;
            v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const double av = A[(base + c16) * LD + base + 4 * kk + g4];
                const double bv = A[(base + 4 * kk + g4) * LD + 16 * j + c16];
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) A[(base + g4 + 4 * v) * LD + 16 * j + c16] = acc[v];
        }
        __syncthreads();
        // ---- trailing update: A_ij <- A_ij - A_ik A_kj, tile (i, j) to wave (its rank) % 4
#pragma unroll
        for (int i = 0; i < T; ++i) {
            if (i == k) continue;
#pragma unroll
            for (int j = 0; j < T; ++j) {
                if (j == k || ((i - (i > k)) * (T - 1) + (j - (j > k))) % kInvWaves != w) continue;
                v4d acc;
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[v] = A[(16 * i + g4 + 4 * v) * LD + 16 * j + c16];
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    const double av = -A[(16 * i + c16) * LD + base + 4 * kk + g4];
                    const double bv = A[(base + 4 * kk + g4) * LD + 16 * j + c16];
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) A[(16 * i + g4 + 4 * v) * LD + 16 * j + c16] = acc[v];
            }
        }
        __syncthreads();
        // ---- column panel: A_ik <- -A_ik P, tile i (i != k) to wave (its rank) % 4;
        // a tile's wave reads it whole before writing it (one wave, in order)
#pragma unroll
        for (int i = 0; i < T; ++i) {
            if (i == k || (i - (i > k)) % kInvWaves != w) continue;
            v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const double av = -A[(16 * i + c16) * LD + base + 4 * kk + g4];
                const double bv = A[(base + 4 * kk + g4) * LD + base + c16];
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) A[(16 * i + g4 + 4 * v) * LD + base + c16] = acc[v];
        }
        __syncthreads();
    }
    if (w == 0 && !ok && lane == 0) atomicOr(B.flag, 1);

    const bool packed = l == 0 && B.packed0;
    if (packed) {
        // FP64: symmetric-packed lower triangle (the mean of the two
        // triangles of the computed inverse), zero on empty lanes
        double* o64 = B.inv64[0] + (long long)d * kPacked;
        for (int j = w; j < kPackedN; j += kInvWaves)  // column j (rows j..47) by wave j % 4
            for (int i = j + lane; i < kPackedN; i += 64) {
                const bool live = ((occ >> (i / 3)) & 1ull) && ((occ >> (j / 3)) & 1ull);
                o64[packed_col(j) + i - j] = live ? 0.5 * (A[i * LD + j] + A[j * LD + i]) : 0.0;
            }
    }
    // column-major n x n, zero rows/columns on empty lanes
    const long long off = (long long)d * n * n;
    double* o64 = packed ? nullptr : B.inv64[l] + off;
    float* o32 = want32 ? B.inv32[l] + off : nullptr;
    if (o64 || o32)
        for (int e = tid; e < n * n; e += kInvThreads) {
            const int col = e / n, row = e - col * n;
            const bool live = ((occ >> (row / 3)) & 1ull) && ((occ >> (col / 3)) & 1ull);
            const double val = live ? A[row * LD + col] : 0.0;
            if (o64) o64[e] = val;
            if (o32) o32[e] = static_cast<float>(val);
        }
}

// ------------------------------------------------------------------ apply
constexpr int kRound = 8;  // coarse partials loaded per round by one lane

// Sum of a unit's partials part[m0 .. m1) (three components each) over 16
// lanes, lane sub taking m0 + sub, + 16, + 32, ... in this order, then folded
// within the lanes' DPP row.  kR are loaded per round (at clamped indices, the
// ones past the range not added) so that their latencies overlap: a unit of
// the top levels has partials from about a hundred groups.
template <int kR>
__device__ __forceinline__ void gather_unit16(const double* __restrict__ part, int m0, int m1, int sub, double& s0,
                                              double& s1, double& s2) {
    s0 = s1 = s2 = 0.0;
    for (int m = m0 + sub; m < m1; m += 16 * kR) {
        double a0[kR], a1[kR], a2[kR];
#pragma unroll
        for (int j = 0; j < kR; ++j) {
            const int mj = min(m + 16 * j, m1 - 1);
            a0[j] = part[3 * mj];
            a1[j] = part[3 * mj + 1];
            a2[j] = part[3 * mj + 2];
        }
#pragma unroll
        for (int j = 0; j < kR; ++j)
            if (m + 16 * j < m1) {
                s0 += a0[j];
                s1 += a1[j];
                s2 += a2[j];
            }
    }
    s0 = row16_sum(s0);
    s1 = row16_sum(s1);
    s2 = row16_sum(s2);
}

// The same over a whole wave (other domain sizes): two loads in flight per
// lane.
__device__ __forceinline__ void gather_unit64(const double* __restrict__ part, int m0, int m1, int lane, double& s0,
                                              double& s1, double& s2) {
    s0 = s1 = s2 = 0.0;
    for (int m = m0 + lane; m < m1; m += 128) {
        const int mb = m + 64;
        s0 += part[3 * m];
        s1 += part[3 * m + 1];
        s2 += part[3 * m + 2];
        if (mb < m1) {
            s0 += part[3 * mb];
            s1 += part[3 * mb + 1];
            s2 += part[3 * mb + 2];
        }
    }
    s0 = wave_sum(s0);
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
}

// Coarse levels l >= 1 (workgroups 1.. of the launch, one per domain, all
// levels at once): r_l for the domain's N units straight from the residual's
// restriction -- level 1 from r_1, higher levels as sums of the per-group
// partials the restriction left for each unit (a contiguous range per unit;
// for N = 16 sixteen lanes per unit, all units at once, else one wave per
// unit), kept in rc_l inside PCG -- then y_l = Inv_{l,d} r_l.
template <typename TI, int kN>
__global__ void __launch_bounds__(256) k_apply_coarse(SolverView v, DomTable tab, int mode, int k, double tol,
                                                      int flags) {
    __shared__ double rl[128];
    __shared__ double buf[256];
    if (blockIdx.x == 0) {
        if (mode != kApplyPlain) convergence_decision(v, mode == kApplyInit, k, tol, flags, buf);
        return;
    }
    const int gb = blockIdx.x - 1;
    int l = 1;
    while (l + 1 < v.L && gb >= tab.off[l + 1]) ++l;
    const int d = gb - tab.off[l];
    const int N = kN > 0 ? kN : v.N, n = 3 * N;
    const int u0 = d * N;
    const int nu = min(N, v.units[l] - u0);
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    const TI* inv;
    if constexpr (sizeof(TI) == 8)
        inv = v.inv64[l];
    else
        inv = v.inv32[l];
    inv += static_cast<long long>(d) * n * n;
    // N = 16: four threads per row, each holding a quarter of the row's
    // inverse entries, loaded before the gather so that both are in flight
    constexpr int kParts = 4;
    constexpr int kCols = kN > 0 ? (3 * kN + kParts - 1) / kParts : 1;
    double pre[kCols];
    const int prow = t % n, ppart = t / n;
    if constexpr (kN > 0) {
        if (t < kParts * n) {
#pragma unroll
            for (int j = 0; j < kCols; ++j) {
                const int kk = ppart * kCols + j;
                pre[j] = kk < n ? inv_load<TI, false>(inv + static_cast<long long>(kk) * n + prow) : 0.0;
            }
        }
    }
    // the stop flag is read once these loads are in flight; after a stop
    // nothing is written
    const int stop = v.st->done;
    keep_loads_issued();
    if (mode == kApplyIter && stop) return;
    const bool keep = mode != kApplyPlain;  // r_l of levels >= 2 kept for the recurrence
    if (l == 1) {
        if (t < n) rl[t] = t < 3 * nu ? v.r1[3 * u0 + t] : 0.0;
    } else if constexpr (kN == 16) {
        const int* cp = v.cp_ptr[l];
        const int a = t >> 4, sub = t & 15;
        const bool own = a < nu;
        double s0, s1, s2;
        gather_unit16<kRound>(v.cpart, own ? cp[u0 + a] : 0, own ? cp[u0 + a + 1] : 0, sub, s0, s1, s2);
        if (sub == 0) {
            if (keep && own) {
                double* rc = v.rc[l] + 3 * (u0 + a);
                rc[0] = s0;
                rc[1] = s1;
                rc[2] = s2;
            }
            rl[3 * a] = s0;
            rl[3 * a + 1] = s1;
            rl[3 * a + 2] = s2;
        }
    } else {
        const int* cp = v.cp_ptr[l];
        for (int a = w; a < N; a += 4) {
            const bool own = a < nu;
            double s0, s1, s2;
            gather_unit64(v.cpart, own ? cp[u0 + a] : 0, own ? cp[u0 + a + 1] : 0, lane, s0, s1, s2);
            if (lane == 0) {
                if (keep && own) {
                    double* rc = v.rc[l] + 3 * (u0 + a);
                    rc[0] = s0;
                    rc[1] = s1;
                    rc[2] = s2;
                }
                rl[3 * a] = s0;
                rl[3 * a + 1] = s1;
                rl[3 * a + 2] = s2;
            }
        }
    }
    __syncthreads();
    if constexpr (kN > 0) {
        __shared__ double quarter[kParts][3 * kN];
        if (t < kParts * n) {
            double a = 0.0;
#pragma unroll
            for (int j = 0; j < kCols; ++j) {
                const int kk = ppart * kCols + j;
                if (kk < n) a += pre[j] * rl[kk];
            }
            quarter[ppart][prow] = a;
        }
        __syncthreads();
        if (t < n) v.y[l][3 * u0 + t] = ((quarter[0][t] + quarter[1][t]) + quarter[2][t]) + quarter[3][t];
    } else if (t < n) {
        double acc = 0.0;
#pragma unroll 8
        for (int kk = 0; kk < n; ++kk) acc += inv_load<TI, false>(inv + static_cast<long long>(kk) * n + t) * rl[kk];
        v.y[l][3 * u0 + t] = acc;
    }
}

constexpr int kPreLevels = 8;  // coarse levels whose corrections are prefetched
constexpr int kGroupThreads = 384;

// Row i of the inverse of level-0 domain d times its residual rd (LDS),
// full column-major layout.
template <typename TI, int kN>
__device__ __forceinline__ double full_row(const TI* __restrict__ inv0, int n, int d, int row, const double* rd) {
    const TI* inv = inv0 + (long long)d * n * n + row;
    double acc = 0.0;
    if constexpr (kN > 0) {
#pragma unroll
        for (int kk = 0; kk < 3 * kN; ++kk) acc += inv_load(inv + kk * 3 * kN) * rd[kk];
    } else {
#pragma unroll 8
        for (int kk = 0; kk < n; ++kk) acc += inv_load(inv + kk * n) * rd[kk];
    }
    return acc;
}

template <typename TI>
__device__ __forceinline__ const TI* level0_inverses(const SolverView& v) {
    if constexpr (sizeof(TI) == 8)
        return v.inv64[0];
    else
        return v.inv32[0];
}

// Level 0 over a group of D0 domains, one thread per DOF:
//   z = Inv_{0,d} r_d + sum_{l >= 1} y_l[unit of the slot at level l]
// (prolongation of every coarse level, Supp. Eq. 6) and the partial of
// rho = r^T z.  Returns at once after a stop.
template <typename TI, int kN, int kMode>
__global__ void __launch_bounds__(kGroupThreads) k_apply_level0(SolverView v, int k) {
    __shared__ double rs[kGroupThreads];
    __shared__ double red[16];
    const int N = kN > 0 ? kN : v.N;
    const int n = 3 * N;
    const int g = xcd_group(blockIdx.x, v.G), t = threadIdx.x;
    const int nd = min(v.D0, v.M - g * v.D0);  // domains of this group
    const bool live = t < nd * n;
    const long long base = 3LL * g * v.RG;
    const int slot = g * v.RG + t / 3, c = t % 3;
    // coarse corrections of the slot (prolongation), loaded with r so that
    // their latency ends before the inverse stream starts
    int u[kPreLevels];
#pragma unroll
    for (int j = 0; j < kPreLevels; ++j)
        u[j] = (live && j + 1 < v.L) ? v.anc[static_cast<long long>(j) * v.NS + slot] : -1;
    const double rv = live ? v.r[base + t] : 0.0;
    // the stop flag is read once these loads are in flight; after a stop
    // nothing is written
    const int stop = v.st->done;
    keep_loads_issued();
    if (kMode != kApplyPlain && stop) return;
    double ycor[kPreLevels];
#pragma unroll
    for (int j = 0; j < kPreLevels; ++j) ycor[j] = u[j] >= 0 ? v.y[j + 1][3 * u[j] + c] : 0.0;
    rs[t] = rv;
    __syncthreads();
    double zv = 0.0;
    if (live) {
        const int dl = t / n, row = t - dl * n;
        double acc = full_row<TI, kN>(level0_inverses<TI>(v), n, g * v.D0 + dl, row, rs + dl * n);
#pragma unroll
        for (int j = 0; j < kPreLevels; ++j)
            if (u[j] >= 0) acc += ycor[j];
        if (v.L > kPreLevels + 1) {
            // deeper hierarchies: the remaining levels' unit ids at once, then
            // their corrections at once
            constexpr int kRest = kMaxLv - 1 - kPreLevels;
            int ur[kRest];
#pragma unroll
            for (int j = 0; j < kRest; ++j)
                ur[j] = kPreLevels + 1 + j < v.L ? v.anc[static_cast<long long>(kPreLevels + j) * v.NS + slot] : -1;
            double yr[kRest];
#pragma unroll
            for (int j = 0; j < kRest; ++j) yr[j] = ur[j] >= 0 ? v.y[kPreLevels + 1 + j][3 * ur[j] + c] : 0.0;
#pragma unroll
            for (int j = 0; j < kRest; ++j)
                if (ur[j] >= 0) acc += yr[j];
        }
        zv = acc;
        v.z[base + t] = zv;
    }
    if (kMode == kApplyPlain) return;
    const double part = block_sum_last(rv * zv, red);
    if (t == 0) v.P_rho[k & 1][g] = part;
}

// The symmetric-packed FP64 inverses (domain size 16) of a group's domains
// times their residuals: the packed inverses of two domains at a time
// (18.8 KB, contiguous) are staged in LDS with coalesced loads, the next
// pair's loads in flight (in registers) while the current pair is
// multiplied.  (With FP32 inverses the full layout streams faster: the
// staging rounds, not the bytes, then bound the kernel.)  Four threads per
// row each take twelve columns: entry (i, kk) of the inverse is (kk, i) of
// the stored lower triangle when kk > i.
constexpr int kPairs = 2;                                // domains staged per round
constexpr int kStageLoads = (kPairs * kPacked + kGroupThreads - 1) / kGroupThreads;  // entries per thread and round

struct PackedPair {
    double nxt[kStageLoads];
};

__device__ __forceinline__ void fetch_pair(PackedPair& P, const double* __restrict__ inv, int p, int nd) {
    const int cnt = min(kPairs, nd - kPairs * p) * kPacked;
    const double* src = inv + static_cast<long long>(kPairs * p) * kPacked;
#pragma unroll
    for (int j = 0; j < kStageLoads; ++j) {
        const int e = threadIdx.x + kGroupThreads * j;
        P.nxt[j] = e < cnt ? inv_load<double, false>(src + e) : 0.0;
    }
}

// zs[48 d + i] = (Inv_{0,d} r_d)_i for the nd domains of the group, whose
// first pair is already fetched into P; rs: their residuals (visible after
// the first barrier here).  Ends with a barrier.
__device__ __forceinline__ void packed_rounds(PackedPair& P, const double* __restrict__ inv, int nd, const double* rs,
                                              double* zs, double* stage) {
    const int t = threadIdx.x;
    const int rounds = (nd + kPairs - 1) / kPairs;
    const int row = t >> 2, q = t & 3;  // 96 rows of a pair, four quarters each
    const int dl = row / 48, i = row - 48 * dl;
    for (int p = 0; p < rounds; ++p) {
        const int cnt = min(kPairs, nd - kPairs * p) * kPacked;
#pragma unroll
        for (int j = 0; j < kStageLoads; ++j) {
            const int e = t + kGroupThreads * j;
            if (e < cnt) stage[e] = P.nxt[j];
        }
        __syncthreads();  // the pair (and, the first time, r) are visible
        if (p + 1 < rounds) fetch_pair(P, inv, p + 1, nd);
        const int d = kPairs * p + dl;
        double s = 0.0;
        if (d < nd) {
            const double* Ad = stage + dl * kPacked;
            const double* rd = rs + 48 * d;
#pragma unroll
            for (int m = 0; m < 12; ++m) {
                const int kk = 12 * q + m;
                const int idx = kk <= i ? packed_col(kk) + i - kk : packed_col(i) + kk - i;
                s += Ad[idx] * rd[kk];
            }
        }
        // the row's four quarters, added as (q0 + q1) + (q2 + q3)
        s = dpp_add<0xb1>(s);  // quad_perm [1, 0, 3, 2]
        s = dpp_add<0x4e>(s);  // quad_perm [2, 3, 0, 1]
        if (q == 0 && d < nd) zs[48 * d + i] = s;
        __syncthreads();  // stage free for the next pair
    }
}

// k_apply_level0 with the symmetric-packed inverses (packed_rounds).
template <int kMode>
__global__ void __launch_bounds__(kGroupThreads) k_apply_level0_packed(SolverView v, int k) {
    __shared__ double rs[kGroupThreads];
    __shared__ double zs[kGroupThreads];
    __shared__ double stage[kPairs * kPacked];
    __shared__ double red[16];
    const int g = xcd_group(blockIdx.x, v.G), t = threadIdx.x;
    const int nd = min(v.D0, v.M - g * v.D0);  // domains of this group
    const bool live = t < nd * 48;
    const long long base = 3LL * g * v.RG;
    const int slot = g * v.RG + t / 3, c = t % 3;
    const double* inv = v.inv64[0] + static_cast<long long>(g) * v.D0 * kPacked;
    PackedPair P;
    fetch_pair(P, inv, 0, nd);
    const double rv = live ? v.r[base + t] : 0.0;
    // the stop flag is read once these loads are in flight; after a stop
    // nothing is written
    const int stop = v.st->done;
    keep_loads_issued();
    if (kMode != kApplyPlain && stop) return;
    rs[t] = rv;
    packed_rounds(P, inv, nd, rs, zs, stage);
    // the corrections of the slot (prolongation) at every coarse level,
    // loaded after the rounds (registers held through them would cost a
    // workgroup per CU): all unit ids at once, then all corrections at once
    int u[kMaxLv - 1];
#pragma unroll
    for (int j = 0; j < kMaxLv - 1; ++j)
        u[j] = (live && j + 1 < v.L) ? v.anc[static_cast<long long>(j) * v.NS + slot] : -1;
    double ycor[kMaxLv - 1];
#pragma unroll
    for (int j = 0; j < kMaxLv - 1; ++j) ycor[j] = u[j] >= 0 ? v.y[j + 1][3 * u[j] + c] : 0.0;
    double zv = 0.0;
    if (live) {
        double acc = zs[t];
#pragma unroll
        for (int j = 0; j < kMaxLv - 1; ++j)
            if (u[j] >= 0) acc += ycor[j];
        zv = acc;
        v.z[base + t] = zv;
    }
    if (kMode == kApplyPlain) return;
    const double part = block_sum_last(rv * zv, red);
    if (t == 0) v.P_rho[k & 1][g] = part;
}

// ---------------------------------------------- apply of a two-launch iteration
// Iteration k by recurrence, in one launch after the SpMV.  Every workgroup
// forms alpha_k = rho_{k-1} / sigma_k from the sigma partials; then
//  - a group workgroup performs x += alpha p_k and r -= alpha q_k on its DOF
//    and z = Inv_{0,d} r_d, with the partials of r^T z and ||r_k||^2;
//  - a coarse workgroup updates the restricted residual of its units,
//    C_l r_k = C_l r_{k-1} - alpha_k C_l q_k (level 1 in r_1, levels >= 2 in
//    rc_l, C_l q_k gathered from the restriction of q_k the SpMV left; each
//    unit has one writer), and computes y_l = Inv_{l,d} C_l r_k and the
//    partial of (C_l r_k)^T y_l.
// rho_k = r^T z + sum_l (C_l r)^T y_l is the sum of both kinds of partials.
// The two do not depend on each other: the prolongation, which would make
// level 0 wait for the coarse levels, is left to the next SpMV.  So the
// coarse levels, a chain of round trips to memory that leaves most of the
// machine idle (7-9 us as a launch of its own at 48^3), run beside the
// streaming of the level-0 inverses.  Four level-1 domains share a workgroup
// (two threads per row); a domain of a higher level, whose units gather up to
// a hundred partials each, has one to itself (eight threads per row).
struct RecTable {
    int off[kMaxLv + 1];  // first coarse workgroup of each level >= 1
    int pad;              // coarse workgroups rounded up to whole rounds of XCDs
};

// alpha_k, or false (after flagging NOT_SPD or NOT_FINITE from group 0) when
// sigma <= 0 or a value is not finite: every workgroup sees the same sigma
// and returns without writing.
__device__ __forceinline__ bool rec_alpha(const SolverView& v, int k, bool report, const PartialLoads<>& sig,
                                          double rho, double* buf, double& alpha) {
    const double sigma = partials_sum(sig, v.P_sigma, v.G, buf);
    if (!(sigma > 0.0) || !finite(sigma) || !finite(rho)) {
        if (report && threadIdx.x == 0) {
            v.st->status = (finite(sigma) && finite(rho)) ? -2 : -6;
            v.st->done = 1;
            v.st->iter = k - 1;
        }
        return false;
    }
    alpha = rho / sigma;
    return true;
}

constexpr int kRecRound = 4;  // partials per lane and round in the coarse workgroups of this launch

// rl[384], buf[256], sum[384], red[16]: shared memory.
template <typename TI, int kN>
__device__ __forceinline__ void rec_coarse(const SolverView& v, const RecTable& tab, int k, int b, double* rl,
                                           double* buf, double* sum, double* red) {
    const int t = threadIdx.x;
    int l = 1;
    while (l + 1 < v.L && b >= tab.off[l + 1]) ++l;
    const int N = kN > 0 ? kN : v.N, n = 3 * N;
    const TI* invl;
    if constexpr (sizeof(TI) == 8)
        invl = v.inv64[l];
    else
        invl = v.inv32[l];
    PartialLoads<> sig = partials_load(v.P_sigma, v.G);
    const double rho = v.st->rho[(k - 1) & 1];
    double part = 0.0;
    if (kN == 16 && l == 1) {
        constexpr int kCols = 24;
        const int dl = t / 96, half = t % 96 / 48, row = t % 48;
        const int d = kRecLevel1 * (b - tab.off[1]) + dl;
        const bool dom = d < v.ndom[1];
        const int e = 48 * d + row;
        const bool own = dom && half == 0 && e < 3 * v.units[1];
        const int ec = own ? e : 0;
        const double prev = v.r1[ec], qv = v.q1[ec];
        double pre[kCols];
        const TI* inv = invl + (dom ? static_cast<long long>(d) * 2304 : 0) + 48 * kCols * half + row;
#pragma unroll
        for (int j = 0; j < kCols; ++j) pre[j] = inv_load<TI, false>(inv + 48 * j);
        const int stop = v.st->done;
        keep_loads_issued();
        if (stop) return;
        double alpha;
        if (!rec_alpha(v, k, false, sig, rho, buf, alpha)) return;
        double r = 0.0;
        if (own) {
            r = prev - alpha * qv;
            v.r1[e] = r;
        }
        if (half == 0) rl[48 * dl + row] = r;
        __syncthreads();
        double a = 0.0;
#pragma unroll
        for (int j = 0; j < kCols; ++j) a += pre[j] * rl[48 * dl + kCols * half + j];
        if (half == 1) sum[48 * dl + row] = a;
        __syncthreads();
        if (half == 0 && dom) {
            a += sum[48 * dl + row];
            v.y[1][e] = a;
            part = r * a;
        }
    } else {
        const int d = b - tab.off[l];
        const int u0 = d * N, nu = min(N, v.units[l] - u0);
        constexpr int kParts = 8, kCols = 6;  // N = 16
        const int row = t % 48, seg = t / 48;
        const TI* inv = invl + static_cast<long long>(d) * n * n;
        double pre[kCols];
        double p0 = 0.0, p1 = 0.0, p2 = 0.0, q1v = 0.0;
        int m0 = 0, m1 = 0;
        if constexpr (kN == 16) {
#pragma unroll
            for (int j = 0; j < kCols; ++j) pre[j] = inv_load<TI, false>(inv + 48 * (kCols * seg + j) + row);
            const int u = u0 + min(t >> 4, nu - 1);
            p0 = v.rc[l][3 * u];
            p1 = v.rc[l][3 * u + 1];
            p2 = v.rc[l][3 * u + 2];
            m0 = v.cp_ptr[l][u];
            m1 = v.cp_ptr[l][u + 1];
        } else if (l == 1) {
            const int e = 3 * u0 + min(t, 3 * nu - 1);
            p0 = v.r1[e];
            q1v = v.q1[e];
        }
        const int stop = v.st->done;
        keep_loads_issued();
        if (stop) return;
        double alpha;
        if (!rec_alpha(v, k, false, sig, rho, buf, alpha)) return;
        double r = 0.0;
        if (kN != 16 && l == 1) {
            if (t < 3 * nu) {
                r = p0 - alpha * q1v;
                v.r1[3 * u0 + t] = r;
            }
            if (t < n) rl[t] = r;
        } else {
            auto put = [&](int a, bool own, double c0, double c1, double c2, double s0, double s1, double s2) {
                if (own) {
                    s0 = c0 - alpha * s0;
                    s1 = c1 - alpha * s1;
                    s2 = c2 - alpha * s2;
                    double* rc = v.rc[l] + 3 * (u0 + a);
                    rc[0] = s0;
                    rc[1] = s1;
                    rc[2] = s2;
                }
                rl[3 * a] = own ? s0 : 0.0;
                rl[3 * a + 1] = own ? s1 : 0.0;
                rl[3 * a + 2] = own ? s2 : 0.0;
            };
            double s0, s1, s2;
            if constexpr (kN == 16) {
                const int a = t >> 4, sub = t & 15;
                if (t < 256) {  // whole waves
                    gather_unit16<kRecRound>(v.qpart, m0, m1, sub, s0, s1, s2);
                    if (sub == 0) put(a, a < nu, p0, p1, p2, s0, s1, s2);
                }
            } else {
                const int lane = t & 63;
                for (int a = t >> 6; a < N; a += kGroupThreads / 64) {
                    const bool own = a < nu;
                    gather_unit64(v.qpart, own ? v.cp_ptr[l][u0 + a] : 0, own ? v.cp_ptr[l][u0 + a + 1] : 0, lane, s0,
                                  s1, s2);
                    if (lane == 0) {
                        const double* rc = v.rc[l] + 3 * (u0 + min(a, nu - 1));
                        put(a, own, rc[0], rc[1], rc[2], s0, s1, s2);
                    }
                }
            }
        }
        __syncthreads();
        if constexpr (kN == 16) {
            double a = 0.0;
#pragma unroll
            for (int j = 0; j < kCols; ++j) a += pre[j] * rl[kCols * seg + j];
            sum[t] = a;  // [part][row]
            __syncthreads();
            if (t < 48) {
#pragma unroll
                for (int j = 1; j < kParts; ++j) a += sum[48 * j + t];
                v.y[l][3 * u0 + t] = a;
                part = rl[t] * a;
            }
        } else if (t < n) {
            double a = 0.0;
#pragma unroll 8
            for (int kk = 0; kk < n; ++kk) a += inv_load<TI, false>(inv + static_cast<long long>(kk) * n + t) * rl[kk];
            v.y[l][3 * u0 + t] = a;
            part = rl[t] * a;
        }
    }
    part = block_sum_last(part, red);
    if (t == 0) v.P_rho[k & 1][v.G + b] = part;
}

template <typename TI, int kN>
__global__ void __launch_bounds__(kGroupThreads) k_apply_rec(SolverView v, RecTable tab, int k) {
    constexpr bool kPackedInv = kN == 16 && sizeof(TI) == 8;
    __shared__ double rs[kGroupThreads];
    __shared__ double zs[kGroupThreads];
    __shared__ double stage[kPackedInv ? kPairs * kPacked : kGroupThreads];
    __shared__ double red[16];
    const int t = threadIdx.x;
    if (static_cast<int>(blockIdx.x) < tab.pad) {
        if (static_cast<int>(blockIdx.x) < v.ncb) rec_coarse<TI, kN>(v, tab, k, blockIdx.x, rs, zs, stage, red);
        return;
    }
    const int N = kN > 0 ? kN : v.N;
    const int n = 3 * N;
    const int g = xcd_group(blockIdx.x - tab.pad, v.G);
    const int nd = min(v.D0, v.M - g * v.D0);  // domains of this group
    const bool live = t < nd * n;
    const long long i = 3LL * g * v.RG + (live ? t : 0);
    PackedPair P;
    const double* inv = v.inv64[0] + static_cast<long long>(g) * v.D0 * kPacked;
    if constexpr (kPackedInv) fetch_pair(P, inv, 0, nd);
    const PartialLoads<> sig = partials_load(v.P_sigma, v.G);
    const double rho = v.st->rho[(k - 1) & 1];
    const double xv = v.x[i], pv = v.p[k & 1][i], ro = v.r[i], qv = v.q[i];
    // the stop flag is read once these loads are in flight; after a stop
    // nothing is written
    const int stop = v.st->done;
    keep_loads_issued();
    if (stop) return;
    double alpha;
    if (!rec_alpha(v, k, g == 0, sig, rho, zs, alpha)) return;  // zs is first written after a later barrier
    double rv = 0.0;
    if (live) {
        v.x[i] = xv + alpha * pv;
        rv = ro - alpha * qv;
        v.r[i] = rv;
    }
    rs[t] = rv;
    double zv = 0.0;
    if constexpr (kPackedInv) {
        packed_rounds(P, inv, nd, rs, zs, stage);
        if (live) zv = zs[t];
    } else {
        __syncthreads();
        if (live) zv = full_row<TI, kN>(level0_inverses<TI>(v), n, g * v.D0 + t / n, t % n, rs + t / n * n);
    }
    if (live) v.z[i] = zv;
    double prho, prr;
    block_sum2_last(rv * zv, rv * rv, red, prho, prr);
    if (t == 0) {
        v.P_rho[k & 1][g] = prho;
        v.P_rr[g] = prr;
    }
}

DomTable make_table(const int* ndom, int first, int L) {
    DomTable t{};
    int acc = 0;
    for (int l = 0; l <= kMaxLv; ++l) t.off[l] = 0;
    for (int l = first; l < L; ++l) {
        t.off[l] = acc;
        acc += ndom[l];
    }
    for (int l = L; l <= kMaxLv; ++l) t.off[l] = acc;
    return t;
}

template <int T>
void launch_invert_t(const BuildView& b, const double* Hu, bool want32, int total, const DomTable& tab, hipStream_t s) {
    launch_kernel(k_invert<T>, dim3(total), dim3(kInvThreads), 0, s, b, Hu, want32 ? 1 : 0, tab);
}

}  // namespace

hipError_t launch_coarse_sums(const BuildView& b, const double* Hu, hipStream_t s) {
    for (int l = 1; l < b.L; ++l) {
        const int g = ceil_div(9LL * b.nnzA[l], 256);  // nine threads per coarse block
        if (g == 0) continue;
        if (l == 1)
            launch_kernel(k_coarse_sum_first, dim3(g), dim3(256), 0, s, b.nnzA[1], b.red_ptr[1], b.red_src[1], Hu,
                               b.A[1]);
        else
            launch_kernel(k_coarse_sum_next, dim3(g), dim3(256), 0, s, b.nnzA[l], b.nnzA[l - 1], b.red_ptr[l],
                               b.red_src[l], b.A[l - 1], b.A[l]);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_invert(const BuildView& b, const double* Hu, bool want32, hipStream_t s) {
    const DomTable tab = make_table(b.ndom, 0, b.L);
    const int total = tab.off[kMaxLv];
    const int T = ceil_div(3 * b.N, 16);
    switch (T) {
        case 1: launch_invert_t<1>(b, Hu, want32, total, tab, s); break;
        case 2: launch_invert_t<2>(b, Hu, want32, total, tab, s); break;
        case 3: launch_invert_t<3>(b, Hu, want32, total, tab, s); break;
        case 4: launch_invert_t<4>(b, Hu, want32, total, tab, s); break;
        case 5: launch_invert_t<5>(b, Hu, want32, total, tab, s); break;
        case 6: launch_invert_t<6>(b, Hu, want32, total, tab, s); break;
        case 7: launch_invert_t<7>(b, Hu, want32, total, tab, s); break;
        case 8: launch_invert_t<8>(b, Hu, want32, total, tab, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_apply_coarse(const SolverView& v, bool f32, int mode, int k, double tol, bool x0_given, bool mixed,
                               bool rr_true, hipStream_t s, bool decision_only) {
    const DomTable tab = make_table(v.ndom, 1, v.L);
    const int total = decision_only ? 1 : 1 + tab.off[kMaxLv];  // workgroup 0 decides convergence
    const int flags = (x0_given ? kFlagX0 : 0) | (mixed ? kFlagMixed : 0) | (rr_true ? kFlagRrTrue : 0);
    if (v.N == 16) {
        if (f32) launch_kernel((k_apply_coarse<float, 16>), dim3(total), dim3(256), 0, s, v, tab, mode, k, tol, flags);
        else launch_kernel((k_apply_coarse<double, 16>), dim3(total), dim3(256), 0, s, v, tab, mode, k, tol, flags);
    } else {
        if (f32) launch_kernel((k_apply_coarse<float, 0>), dim3(total), dim3(256), 0, s, v, tab, mode, k, tol, flags);
        else launch_kernel((k_apply_coarse<double, 0>), dim3(total), dim3(256), 0, s, v, tab, mode, k, tol, flags);
    }
    return hipGetLastError();
}

template <typename TI, int kN>
void launch_level0_t(const SolverView& v, int mode, int k, hipStream_t s) {
    dim3 g(v.G), b(round_waves(3 * v.RG));
    if constexpr (kN == 16 && sizeof(TI) == 8) {
        b = dim3(kGroupThreads);
        if (mode == kApplyPlain)
            launch_kernel(k_apply_level0_packed<kApplyPlain>, g, b, 0, s, v, k);
        else if (mode == kApplyInit)
            launch_kernel(k_apply_level0_packed<kApplyInit>, g, b, 0, s, v, k);
        else
            launch_kernel(k_apply_level0_packed<kApplyIter>, g, b, 0, s, v, k);
    } else {
        if (mode == kApplyPlain)
            launch_kernel((k_apply_level0<TI, kN, kApplyPlain>), g, b, 0, s, v, k);
        else if (mode == kApplyInit)
            launch_kernel((k_apply_level0<TI, kN, kApplyInit>), g, b, 0, s, v, k);
        else
            launch_kernel((k_apply_level0<TI, kN, kApplyIter>), g, b, 0, s, v, k);
    }
}

hipError_t launch_apply_level0(const SolverView& v, bool f32, int mode, int k, hipStream_t s) {
    if (v.N == 16) {
        if (f32) launch_level0_t<float, 16>(v, mode, k, s);
        else launch_level0_t<double, 16>(v, mode, k, s);
    } else {
        if (f32) launch_level0_t<float, 0>(v, mode, k, s);
        else launch_level0_t<double, 0>(v, mode, k, s);
    }
    return hipGetLastError();
}

hipError_t launch_apply_rec(const SolverView& v, bool f32, int k, hipStream_t s) {
    RecTable tab{};
    int acc = 0;
    for (int l = 1; l < v.L; ++l) {
        tab.off[l] = acc;
        acc += l == 1 && v.N == 16 ? ceil_div(v.ndom[1], kRecLevel1) : v.ndom[l];
    }
    for (int l = v.L; l <= kMaxLv; ++l) tab.off[l] = acc;
    if (acc != v.ncb) return hipErrorInvalidValue;  // the P_rho arrays hold G + ncb partials
    tab.pad = ceil_div(acc, kXcds) * kXcds;
    dim3 g(tab.pad + v.G), b(kGroupThreads);
    if (v.N == 16) {
        if (f32) launch_kernel((k_apply_rec<float, 16>), g, b, 0, s, v, tab, k);
        else launch_kernel((k_apply_rec<double, 16>), g, b, 0, s, v, tab, k);
    } else {
        if (f32) launch_kernel((k_apply_rec<float, 0>), g, b, 0, s, v, tab, k);
        else launch_kernel((k_apply_rec<double, 0>), g, b, 0, s, v, tab, k);
    }
    return hipGetLastError();
}

}  // namespace maspcg

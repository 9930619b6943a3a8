// MAS preconditioner on the device: coarse matrices, batched domain
// inversion and the apply (Supp. Eq. 4-6; algorithm "Compute MAS
// preconditioner" in Sec. 4.3).
#include <algorithm>
#include <type_traits>

#include "decision.hpp"
#include "launch.hpp"

namespace maspcg {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

// Inverse entries in the apply of domain sizes other than 16 (full layout):
// FP64 level-0 inverses are streamed with non-temporal loads that leave the
// caches to H, the vectors and the coarse inverses (kStream); the others are
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
// kRound list entries loaded at a time (their indices, then their values;
// past the end the last one again), so that the list's loads overlap instead
// of following one another.
template <int kRound, typename F>
__device__ __forceinline__ double list_sum(const int* __restrict__ src, int q, int qe, F&& value) {
    double s = 0.0;
    for (; q < qe; q += kRound) {
        int i[kRound];
#pragma unroll
        for (int j = 0; j < kRound; ++j) i[j] = src[min(q + j, qe - 1)];
        double a[kRound];
#pragma unroll
        for (int j = 0; j < kRound; ++j) a[j] = value(i[j]);
#pragma unroll
        for (int j = 0; j < kRound; ++j)
            if (q + j < qe) s += a[j];
    }
    return s;
}

constexpr int kRoundFirst = 4, kRoundNext = 8;

__global__ void __launch_bounds__(256) k_coarse_sum_first(int nnzA, const int* __restrict__ ptr,
                                                           const int* __restrict__ src, const double* __restrict__ Hu,
                                                           double* __restrict__ A) {
    const long long gt = static_cast<long long>(blockIdx.x) * 256 + threadIdx.x;
    if (gt >= 9LL * nnzA) return;
    const int t = static_cast<int>(gt / 9), c = static_cast<int>(gt % 9);
    A[static_cast<long long>(c) * nnzA + t] =
        list_sum<kRoundFirst>(src, ptr[t], ptr[t + 1], [&](int i) { return Hu[9LL * i + c]; });
}

__global__ void __launch_bounds__(256) k_coarse_sum_next(int nnzA, int nnzPrev, const int* __restrict__ ptr,
                                                          const int* __restrict__ src, const double* __restrict__ Ap,
                                                          double* __restrict__ A) {
    const long long gt = static_cast<long long>(blockIdx.x) * 256 + threadIdx.x;
    if (gt >= 9LL * nnzA) return;
    const int t = static_cast<int>(gt / 9), c = static_cast<int>(gt % 9);
    const double* Apc = Ap + static_cast<long long>(c) * nnzPrev;
    A[static_cast<long long>(c) * nnzA + t] =
        list_sum<kRoundNext>(src, ptr[t], ptr[t + 1], [&](int i) { return Apc[i]; });
}

// ------------------------------------------------------- domain inversion
// Domain sizes other than 16 (those: below), one workgroup of four waves per
// domain (all levels in one launch).  The
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

template <int n, int i = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (i < n) {
        f(std::integral_constant<int, i>{});
        static_for<n, i + 1>(f);
    }
}

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
            // step j: the pivot by readlane, column j by DPP (lane j of each row
            // of 16), row j, which no DPP form moves across the rows of 16, by
            // one shuffle beside the division
            static_for<16>([&](auto jc) {
                constexpr int j = jc.value, jg = j >> 2, jv = j & 3;
                const double rowj = __shfl(a[jv], jg * 16 + c16);
                const double piv = lane_value(a[jv], jg * 16 + j);
                double colj[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) colj[v] = dpp_row_lane<j>(a[v]);
                ok = ok && (piv > 0.0) && finite(piv);
                const double inv = 1.0 / piv;
                // with 1 in place of the pivot column's entry of row j, and 0 in
                // place of the column's other entries, all entries take one form
                const double sc = c16 == j ? inv : rowj * inv;
#pragma unroll
                for (int v = 0; v < 4; ++v) a[v] = __fma_rn(-colj[v], sc, c16 == j ? 0.0 : a[v]);
                if (g4 == jg) a[jv] = sc;
            });
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

    // column-major n x n, zero rows/columns on empty lanes
    const long long off = (long long)d * n * n;
    double* o64 = B.inv64[l] + off;
    float* o32 = want32 ? B.inv32[l] + off : nullptr;
    for (int e = tid; e < n * n; e += kInvThreads) {
        const int col = e / n, row = e - col * n;
        const bool live = ((occ >> (row / 3)) & 1ull) && ((occ >> (col / 3)) & 1ull);
        const double val = live ? A[row * LD + col] : 0.0;
        o64[e] = val;
        if (o32) o32[e] = static_cast<float>(val);
    }
}

// ---- domain size 16: a wave per domain, in registers
// The 48 x 48 matrix as 16 x 16 tiles in the result layout of the MFMA (lane
// l, register v: row l / 16 + 4 v, column l % 16).  In this layout a tile is
// the B operand as it is, and the A operand of its transpose.  Sweeping the
// tiles of a symmetric matrix,
//   P = inv(A_kk), A_kj <- P A_kj, A_ij <- A_ij - A_ik P A_kj,
//   A_ik <- A_ik P, A_kk <- -P      (the inverse is minus the swept matrix),
// needs A_ik = A_ki^T as an A operand only, so no tile passes through LDS, no
// barrier separates the steps, and of the symmetric pairs of tiles only the
// one that a later step reads is formed: 18 tile products instead of 24.
// The tiles are swept last to first, which leaves those above the diagonal:
// as transposes of the packed ones (launch.hpp) they are stored 256
// contiguous bytes at a time.
//
// Through LDS, four waves per domain, 70 of 97 us at 48^3 went to the tile
// products' operands (18.8 KB of LDS per domain also kept the workgroups to 8
// per CU); now 75 us (45 -> 33 at 33^3; 8^3, a single wave's chain, 15 -> 17).
// More waves per SIMD, or workgroups of one or two domains, take as long.
using Tile = v4d;

// acc + X^T Y
__device__ __forceinline__ Tile tile_product(Tile x, Tile y, Tile acc) {
#pragma unroll
    for (int k = 0; k < 4; ++k) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[k], y[k], acc, 0, 0, 0);
    return acc;
}

// Scalar Gauss-Jordan in place, 16 pivots: the pivot by readlane and column j
// by DPP (lane j of each row of 16), row j, which no DPP form moves across
// the rows of 16, by one shuffle beside the division (with six 64-bit shuffles
// a step instead, and the four-wave kernel, 127 us at 48^3 for its 97).
__device__ __forceinline__ Tile tile_inverse(Tile a, bool& ok) {
    const int lane = threadIdx.x & 63, c16 = lane & 15, g4 = lane >> 4;
    static_for<16>([&](auto jc) {
        constexpr int j = jc.value, jv = j >> 2, jg = j & 3;
        const double rowj = __shfl(a[jv], jg * 16 + c16);
        const double piv = lane_value(a[jv], jg * 16 + j);
        double colj[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) colj[v] = dpp_row_lane<j>(a[v]);
        ok = ok && (piv > 0.0) && finite(piv);
        const double inv = 1.0 / piv;
        // with 1 in place of the pivot column's entry of row j, and 0 in
        // place of the column's other entries, all entries take one form
        const double sc = c16 == j ? inv : rowj * inv;
#pragma unroll
        for (int v = 0; v < 4; ++v) a[v] = __fma_rn(-colj[v], sc, c16 == j ? 0.0 : a[v]);
        if (g4 == jg) a[jv] = sc;
    });
    return a;
}

// Store of the tile above the diagonal whose transpose is tile (I, J), I >= J,
// of the packed inverse: this lane's entries are row c16, columns g4 + 4 v.
template <typename TO>
__device__ __forceinline__ void store_tile(TO* __restrict__ out, Tile a, int I, int J, int half,
                                           unsigned long long occ) {
    const int lane = threadIdx.x & 63, r = lane & 15, g4 = lane >> 4;
    const bool row_live = (occ >> ((16 * I + r) / 3)) & 1ull;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int c = g4 + 4 * v;
        const double x = row_live && ((occ >> ((16 * J + c) / 3)) & 1ull) ? a[v] : 0.0;
        if (I > J) {
            out[kTile * tile_below(I, J, half) + tile_at<TO>(r, c)] = static_cast<TO>(x);
        } else {
            if (half == 0 ? r >= c : r < c)
                out[kTile * (6 + I) + tile_at<TO>(r, c)] = static_cast<TO>(half == 0 && r == c ? 0.5 * x : x);
            if (half == 1 && r == c) out[kPairDiag + 16 * I + r] = static_cast<TO>(x);
        }
    }
}

constexpr int kWaveDomains = 4;  // waves, and domains, per workgroup

__global__ void __launch_bounds__(64 * kWaveDomains, 4) k_invert_waves(BuildView B, const double* __restrict__ Hu,
                                                                       int want32, DomTable tab) {
    __shared__ int maps[kWaveDomains][256];
    const int lane = threadIdx.x & 63, c16 = lane & 15, g4 = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l = level_of(tab, B.L, blockIdx.x);
    const int d = kWaveDomains * (blockIdx.x - tab.off[l]) + w;
    if (d >= B.ndom[l]) return;
    const int q0 = uniform_load(B.dom_ptr[l] + d), q1 = uniform_load(B.dom_ptr[l] + d + 1);
    const int u = 16 * d + c16;
    const unsigned long long occ =
        __ballot(lane < 16 && (l == 0 ? B.remap[u] >= 0 : u < B.units[l]));

    // block of each pair of nodes a <= b, or -1
    int* map = maps[w];
#pragma unroll
    for (int i = 0; i < 4; ++i) map[lane + 64 * i] = -1;
    wave_lds_sync();
    for (int q = q0 + lane; q < q1; q += 64) {
        const int ab = B.dom_ab[l][q];
        map[16 * (ab & 255) + (ab >> 8)] = B.dom_blk[l][q];
    }
    wave_lds_sync();
    // entry (i, j), i <= j, of the matrix; what is read where there is no
    // block is any entry of the level (of the inverses, where it has none)
    const double* base = q0 == q1 ? B.inv64[l] : l == 0 ? Hu : B.A[l];
    const int other = q0 == q1 ? 0 : B.dom_blk[l][q0];
    const long long by_block = l == 0 ? 9 : 1, by_entry = l == 0 ? 1 : B.nnzA[l];
    auto entry = [&](int i, int j) {
        const int a = i / 3, b = j / 3;
        const int k = map[16 * a + b];
        const double x = base[by_block * (k < 0 ? other : k) + by_entry * (3 * (i - 3 * a) + j - 3 * b)];
        return k >= 0 ? x : i == j && !((occ >> a) & 1ull) ? 1.0 : 0.0;
    };
    // tile of block rows and columns I >= J; swept in the order 2, 1, 0, so
    // Xst, Yst: s, t = the places 2 - I, 2 - J in that order
    auto tile = [&](int I, int J) {
        Tile t;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = 16 * I + g4 + 4 * v, c = 16 * J + c16;
            t[v] = I == J ? entry(min(r, c), max(r, c)) : entry(c, r);
        }
        return t;
    };
    Tile d0 = tile(2, 2), x01 = tile(2, 1), x02 = tile(2, 0), d1 = tile(1, 1), x12 = tile(1, 0), d2 = tile(0, 0);
    const Tile zero = {0.0, 0.0, 0.0, 0.0};
    bool ok = true;

    Tile p = tile_inverse(d0, ok), n = -p;
    Tile r1 = tile_product(n, x01, zero), r2 = tile_product(n, x02, zero);
    d1 = tile_product(x01, r1, d1);
    x12 = tile_product(x01, r2, x12);
    d2 = tile_product(x02, r2, d2);
    Tile y10 = tile_product(x01, p, zero), y20 = tile_product(x02, p, zero);
    d0 = n;

    p = tile_inverse(d1, ok), n = -p;
    Tile r0 = tile_product(n, y10, zero);
    r2 = tile_product(n, x12, zero);
    d0 = tile_product(y10, r0, d0);
    d2 = tile_product(x12, r2, d2);
    y20 = tile_product(x12, r0, y20);
    Tile y21 = tile_product(x12, p, zero);
    y10 = -r0;
    d1 = n;

    p = tile_inverse(d2, ok), n = -p;
    r0 = tile_product(n, y20, zero);
    r1 = tile_product(n, y21, zero);
    d0 = tile_product(y20, r0, d0);
    d1 = tile_product(y21, r1, d1);
    y10 = tile_product(y21, r0, y10);
    if (!ok && lane == 0) atomicOr(B.flag, 1);

    auto store = [&](auto* out) {
        out += static_cast<long long>(d >> 1) * kPairEntries;
        const int half = d & 1;
        store_tile(out, -d0, 2, 2, half, occ);
        store_tile(out, -d1, 1, 1, half, occ);
        store_tile(out, p, 0, 0, half, occ);
        store_tile(out, -y10, 2, 1, half, occ);
        store_tile(out, r0, 2, 0, half, occ);
        store_tile(out, r1, 1, 0, half, occ);
    };
    store(B.inv64[l]);
    if (want32) store(B.inv32[l]);
}

// ------------------------------------------------------------------ apply
// First coarse workgroup of each level >= 1 (coarse_blocks per level).
struct CoarseTable {
    int off[kMaxLv + 1];
};

__device__ __forceinline__ int coarse_level(const CoarseTable& tab, int L, int b) {
    int l = 1;
    while (l + 1 < L && b >= tab.off[l + 1]) ++l;
    return l;
}

template <typename TI>
__device__ __forceinline__ const TI* inverses(const SolverView& v, int l) {
    if constexpr (sizeof(TI) == 8)
        return v.inv64[l];
    else
        return v.inv32[l];
}

// ---- domain size 16: a wave multiplies a pair of domains out of registers
// The pair's packed inverses (launch.hpp; 18.8 KB in FP64) are 36 entries
// per lane and one diagonal entry of the second domain per row, loaded as
// 16-byte loads, 1 KB contiguous per wave and load, all in flight at once:
// the launch then streams while its scalars (alpha) are still being formed,
// nothing is staged in LDS and no barrier separates the loads.  Lane
// (c16, g4) = (lane % 16, lane / 16) holds row c16, columns 4 g4 .. 4 g4 + 3
// of every tile.
template <typename TI>
struct PairRegs {
    TI a[9][4];
    TI diag[2];  // the second domain's diagonal at the lane's rows (see pair_rows)
};

// Rows of the pair a lane owns in the vectors: e = lane and, for lanes below
// 32, lane + 64 (0..47: the first domain, 48..95: the second).
__device__ __forceinline__ int pair_row(int lane, int q) { return lane + 64 * q; }
__device__ __forceinline__ bool pair_owns(int lane, int q) { return q == 0 || lane < 32; }

template <typename TI>
__device__ __forceinline__ void pair_load(PairRegs<TI>& P, const TI* __restrict__ pair, int lane) {
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        if constexpr (sizeof(TI) == 8) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const double2 x = *reinterpret_cast<const double2*>(pair + kTile * j + 128 * h + 2 * lane);
                P.a[j][2 * h] = x.x;
                P.a[j][2 * h + 1] = x.y;
            }
        } else {
            const float4 x = *reinterpret_cast<const float4*>(pair + kTile * j + 4 * lane);
            P.a[j][0] = x.x;
            P.a[j][1] = x.y;
            P.a[j][2] = x.z;
            P.a[j][3] = x.w;
        }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int i = pair_row(lane, q) - 48;
        P.diag[q] = pair[kPairDiag + min(max(i, 0), 47)];
    }
}

// Sums of col[0..3] over the 16 lanes of a row: lane l of the row ends with
// the sum of col[l % 4].
__device__ __forceinline__ double row16_sum4(const double (&col)[4], int lane) {
    const bool b0 = lane & 1, b1 = lane & 2;
    const double k0 = (b0 ? col[1] : col[0]) + dpp_get<0xb1>(b0 ? col[0] : col[1]);  // quad_perm [1, 0, 3, 2]
    const double k1 = (b0 ? col[3] : col[2]) + dpp_get<0xb1>(b0 ? col[2] : col[3]);
    double k = (b1 ? k1 : k0) + dpp_get<0x4e>(b1 ? k0 : k1);  // quad_perm [2, 3, 0, 1]
    k = dpp_add<0x128>(k);                                    // row_ror 8
    return dpp_add<0x124>(k);                                 // row_ror 4
}

constexpr int kPairLds = 96 + 5 * 96;  // doubles of LDS per wave: the vector, four row parts and the column part

// out[q] = the pair's product at the lane's rows, x[q] the vector there
// (zero on rows that hold nothing).  sm: kPairLds doubles of the wave's own;
// no barrier: the wave's LDS accesses stay in order.  An entry below the
// diagonal is used for its row and for its column; a tile's row sums are
// folded over the four lane groups through LDS, its column sums over the 16
// lanes of a row by DPP, the four columns at once.
template <typename TI>
__device__ __forceinline__ void pair_product(const PairRegs<TI>& P, const double (&x)[2], double* sm, int lane,
                                             double (&out)[2]) {
    double* xs = sm;
    double* part = sm + 96;
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (pair_owns(lane, q)) xs[pair_row(lane, q)] = x[q];
    wave_lds_sync();
    const int c16 = lane & 15, g4 = lane >> 4;
    double row[2][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
#pragma unroll
    for (int J = 0; J < 3; ++J)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            // one block column of one domain at a time: with more operands
            // read ahead the entries would no longer fit in 128 registers
            __builtin_amdgcn_sched_barrier(0);
            double xc[4], col[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                xc[v] = xs[48 * h + 16 * J + 4 * g4 + v];
                col[v] = 0.0;
            }
#pragma unroll
            for (int I = J; I < 3; ++I) {
                const double xr = xs[48 * h + 16 * I + c16];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    double a = static_cast<double>(P.a[I > J ? tile_below(I, J, h) : 6 + J][v]);
                    if (I == J) a = (c16 >= 4 * g4 + v) == (h == 0) ? a : 0.0;  // the domain's triangle
                    row[h][I] += a * xc[v];
                    col[v] += a * xr;
                }
            }
            // the row sums are formed here, not once their entries have all
            // been kept for the end
#pragma unroll
            for (int I = J; I < 3; ++I) asm volatile("" : "+v"(row[h][I]));
            const double k = row16_sum4(col, lane);
            if (c16 < 4) part[4 * 96 + 48 * h + 16 * J + 4 * g4 + c16] = k;
        }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int I = 0; I < 3; ++I) part[96 * g4 + 48 * h + 16 * I + c16] = row[h][I];
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int e = pair_row(lane, q);
        out[q] = 0.0;
        if (pair_owns(lane, q)) {
            double s = ((part[e] + part[96 + e]) + (part[192 + e] + part[288 + e])) + part[384 + e];
            if (e >= 48) s += static_cast<double>(P.diag[q]) * x[q];
            out[q] = s;
        }
    }
}

constexpr int kPairThreads = 256;  // four waves
constexpr int kPairWaves = 4;      // waves per SIMD: 128 registers, 72 of them the FP64 pair's entries

// ---- other domain sizes
constexpr int kGroupThreads = 384;

// Sum of a unit's partials part[m0 .. m1) (three components each) over a
// wave: two loads in flight per lane.
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

// Row `row` of a domain's inverse (full column-major layout) times rd (LDS).
template <typename TI, bool kStream>
__device__ __forceinline__ double full_row(const TI* __restrict__ inv, int n, int row, const double* rd) {
    double acc = 0.0;
#pragma unroll 8
    for (int kk = 0; kk < n; ++kk) acc += inv_load<TI, kStream>(inv + static_cast<long long>(kk) * n + row) * rd[kk];
    return acc;
}

// ---- the scalars of an iteration by recurrence
struct RecLoads {
    PartialLoads<4, double2> sp;
    double rho;
};

__device__ __forceinline__ RecLoads rec_load(const SolverView& v, int k) {
    RecLoads R;
    R.sp = partials_load(v.P_sp, v.G);
    R.rho = uniform_load(&v.st->rho[(k - 1) & 1]);
    return R;
}

// alpha_k = rho_{k-1} / sigma_k (see line_step), or false (after flagging NOT_SPD or
// NOT_FINITE where report is set) when sigma <= 0 or a value is not finite:
// every workgroup sees the same sums and returns without writing.  buf: 512
// doubles of shared memory, not written again before another barrier.
__device__ __forceinline__ bool rec_alpha(const SolverView& v, int k, bool report, const RecLoads& R, double* buf,
                                          double& alpha) {
    const double2 s = partials_sum(R.sp, v.P_sp, v.G, buf);
    alpha = line_step(s.x, s.y, R.rho);
    if (!(alpha == alpha)) {
        if (report && threadIdx.x == 0) {
            v.st->status = (finite(s.x) && finite(s.y)) ? -2 : -6;
            v.st->done = 1;
            v.st->iter = k - 1;
        }
        return false;
    }
    return true;
}

// ---- coarse levels
// Workgroup b of the coarse levels: r_l of its domains' units, then y_l =
// Inv_{l,d} r_l.  kRec (iteration k by recurrence): r_l <- r_l - alpha_k
// (C_l q_k) from the restriction of q_k the SpMV left (q_1, qpart), in place
// (r_1, rc_l; each unit has one writer), and the partial of r_l^T y_l.
// Otherwise straight from the residual's restriction (r_1, cpart), kept in
// rc_l for the recurrence unless mode is kApplyPlain.  Level 1 has its values
// in r_1; a unit of a higher level sums the contiguous range of per-group
// partials the restriction left for it (up to about a hundred at the top).

// Domain size 16: eight level-1 domains, a pair per wave, or one pair of a
// higher level (three waves gather, one multiplies).  sm: 4 kPairLds doubles,
// buf: 512 (256 without kRec), red: 16.
constexpr int kItem = 8;     // partials of an item
constexpr int kItems = 192;  // items at a time: one per thread of the gathering waves

template <typename TI, bool kRec>
__device__ __forceinline__ void coarse_pairs(const SolverView& v, const CoarseTable& tab, int mode, int k, int b,
                                             double* sm, double* buf, double* red) {
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int l = coarse_level(tab, v.L, b);
    const int pairs = (v.ndom[l] + 1) / 2, nrow = 3 * v.units[l];
    RecLoads R{};
    if constexpr (kRec) R = rec_load(v, k);
    PairRegs<TI> P;
    double x[2] = {0.0, 0.0}, out[2] = {0.0, 0.0}, part = 0.0;
    if (l == 1) {
        const int p = 4 * (b - tab.off[1]) + w;
        int e[2];
        bool own[2];
        double prev[2], qv[2] = {0.0, 0.0};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            e[q] = 96 * p + pair_row(lane, q);
            own[q] = pair_owns(lane, q) && e[q] < nrow;
            prev[q] = v.r1[own[q] ? e[q] : 0];
            if constexpr (kRec) qv[q] = v.q1[own[q] ? e[q] : 0];
        }
        pair_load(P, inverses<TI>(v, 1) + static_cast<long long>(min(p, pairs - 1)) * kPairEntries, lane);
        const int stop = v.st->done;
        keep_loads_issued();
        if (mode != kApplyPlain && stop) return;
        double alpha = 0.0;
        if (kRec && !rec_alpha(v, k, false, R, buf, alpha)) return;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (!own[q]) continue;
            x[q] = kRec ? prev[q] - alpha * qv[q] : prev[q];
            if (kRec) v.r1[e[q]] = x[q];
        }
        if (p < pairs) {
            pair_product(P, x, sm + w * kPairLds, lane, out);
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (own[q]) {
                    v.y[1][e[q]] = out[q];
                    part += x[q] * out[q];
                }
        }
    } else {
        // waves 0 to 2 gather, wave 3 holds the inverses.  A unit of the top
        // levels can have hundreds of partials beside units that have a few,
        // so the pair's partials are dealt as items of up to kItem of one
        // unit, one per thread: two round trips (the ranges, the partials)
        // whatever their spread.  Items are summed in order per (unit,
        // component).
        const int p = b - tab.off[l];
        const int u0 = 32 * p, nu = min(32, v.units[l] - u0);
        int* first = reinterpret_cast<int*>(sm + 3 * kPairLds);  // [33] first item of each unit
        int* from = first + 34;                                  // [32] its first partial
        int* to = from + 32;                                     // [32] end of its partials
        double* isum = sm + kPairLds;                            // [3 kItems] sums of the items at hand
        const int* cp = v.cp_ptr[l] + u0;
        const double* src = kRec ? v.qpart : v.cpart;
        const bool entry = t < 96 && t < 3 * nu;
        double prev = 0.0;
        if (kRec && entry) prev = v.rc[l][3 * u0 + t];
        int m0 = 0, m1 = 0;
        if (t < nu) {
            m0 = cp[t];
            m1 = cp[t + 1];
        }
        const int stop = v.st->done;
        keep_loads_issued();
        if (mode != kApplyPlain && stop) return;
        if (w == 0) {
            int n = (m1 - m0 + kItem - 1) / kItem;
#pragma unroll
            for (int o = 1; o < 32; o <<= 1) {
                const int below = __shfl_up(n, o);
                if (lane >= o) n += below;
            }
            if (lane < 32) {
                if (lane == 0) first[0] = 0;
                first[lane + 1] = n;
                from[lane] = m0;
                to[lane] = m1;
            }
        }
        __syncthreads();
        const int items = first[32];
        // item it into isum[it % kItems]; many: with all its loads in flight
        auto gather = [&](int it, auto many) {
            int a = 0;
#pragma unroll
            for (int step = 16; step > 0; step >>= 1)
                if (first[a + step] <= it) a += step;
            const int f = from[a] + kItem * (it - first[a]), e = min(f + kItem, to[a]);
            double s0 = 0.0, s1 = 0.0, s2 = 0.0;
            if constexpr (many.value) {
                double c0[kItem], c1[kItem], c2[kItem];
#pragma unroll
                for (int j = 0; j < kItem; ++j) {
                    const int mj = min(f + j, e - 1);
                    c0[j] = src[3 * mj];
                    c1[j] = src[3 * mj + 1];
                    c2[j] = src[3 * mj + 2];
                }
#pragma unroll
                for (int j = 0; j < kItem; ++j)
                    if (f + j < e) {
                        s0 += c0[j];
                        s1 += c1[j];
                        s2 += c2[j];
                    }
            } else {
#pragma unroll 1
                for (int m = f; m < e; ++m) {
                    s0 += src[3 * m];
                    s1 += src[3 * m + 1];
                    s2 += src[3 * m + 2];
                }
            }
            isum[3 * t] = s0;
            isum[3 * t + 1] = s1;
            isum[3 * t + 2] = s2;
        };
        if (t < kItems && t < items) gather(t, std::true_type{});
        // (after the gather in the text, so that its registers are not counted
        // on top of these)
        if (w == 3) pair_load(P, inverses<TI>(v, l) + static_cast<long long>(p) * kPairEntries, lane);
        double s = 0.0;
        for (int i0 = 0;;) {
            __syncthreads();
            if (entry) {
                const int a = t / 3, c = t - 3 * a;
                const int hi = min(first[a + 1] - i0, kItems);
#pragma unroll 4
                for (int i = max(first[a] - i0, 0); i < hi; ++i) s += isum[3 * i + c];
            }
            i0 += kItems;
            if (i0 >= items) break;
            __syncthreads();
            if (t < kItems && i0 + t < items) gather(i0 + t, std::false_type{});  // (rare; few registers)
        }
        double alpha = 0.0;
        if (kRec && !rec_alpha(v, k, false, R, buf, alpha)) return;
        if (t < 96) {
            const double r = entry ? (kRec ? prev - alpha * s : s) : 0.0;
            if (entry && mode != kApplyPlain) v.rc[l][3 * u0 + t] = r;
            sm[t] = r;
        }
        __syncthreads();
        if (w == 3) {
#pragma unroll
            for (int q = 0; q < 2; ++q) x[q] = pair_owns(lane, q) ? sm[pair_row(lane, q)] : 0.0;
            pair_product(P, x, sm + kPairLds, lane, out);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int e = pair_row(lane, q);
                if (pair_owns(lane, q) && e < 3 * nu) {
                    v.y[l][3 * u0 + e] = out[q];
                    part += x[q] * out[q];
                }
            }
        }
    }
    if constexpr (kRec) {
        part = block_sum_last(part, red);
        if (t == 0) v.P_rho[k & 1][v.GA + b] = part;
    }
}

// Other domain sizes: one domain per workgroup, a wave per unit for the
// gather, a thread per row.  rl: 128 doubles, buf: 512 (256 without kRec), red: 16.
template <typename TI, bool kRec>
__device__ __forceinline__ void coarse_domain(const SolverView& v, const CoarseTable& tab, int mode, int k, int b,
                                              double* rl, double* buf, double* red) {
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    const int l = coarse_level(tab, v.L, b);
    const int d = b - tab.off[l], N = v.N, n = 3 * N;
    const int u0 = d * N, nu = min(N, v.units[l] - u0);
    RecLoads R{};
    if constexpr (kRec) R = rec_load(v, k);
    const int stop = v.st->done;
    keep_loads_issued();
    if (mode != kApplyPlain && stop) return;
    double alpha = 0.0;
    if (kRec && !rec_alpha(v, k, false, R, buf, alpha)) return;
    if (l == 1) {
        double r = 0.0;
        if (t < 3 * nu) {
            r = v.r1[3 * u0 + t];
            if constexpr (kRec) {
                r -= alpha * v.q1[3 * u0 + t];
                v.r1[3 * u0 + t] = r;
            }
        }
        if (t < n) rl[t] = r;
    } else {
        const int* cp = v.cp_ptr[l];
        for (int a = w; a < N; a += static_cast<int>(blockDim.x >> 6)) {
            const bool own = a < nu;
            double s[3];
            gather_unit64(kRec ? v.qpart : v.cpart, own ? cp[u0 + a] : 0, own ? cp[u0 + a + 1] : 0, lane, s[0], s[1],
                          s[2]);
            if (lane == 0) {
                double* rc = v.rc[l] + 3 * (u0 + a);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const double r = own ? (kRec ? rc[c] - alpha * s[c] : s[c]) : 0.0;
                    if (own && mode != kApplyPlain) rc[c] = r;
                    rl[3 * a + c] = r;
                }
            }
        }
    }
    __syncthreads();
    double part = 0.0;
    if (t < n) {
        const double y = full_row<TI, false>(inverses<TI>(v, l) + static_cast<long long>(d) * n * n, n, t, rl);
        v.y[l][3 * u0 + t] = y;
        part = rl[t] * y;
    }
    if constexpr (kRec) {
        part = block_sum_last(part, red);
        if (t == 0) v.P_rho[k & 1][v.GA + b] = part;
    }
}

// The coarse levels as a launch of their own (outside the recurrence), with
// the convergence decision on the n_rr partials of ||r||^2 in workgroup 0.
template <typename TI, int kN>
__global__ void __launch_bounds__(kPairThreads, kPairWaves) k_apply_coarse(SolverView v, CoarseTable tab, int mode, int k,
                                                               double tol, int flags, int n_rr) {
    __shared__ double sm[kN == 16 ? 4 * kPairLds : 128];
    __shared__ double buf[256];
    if (blockIdx.x == 0) {
        if (mode != kApplyPlain) convergence_decision(v, mode == kApplyInit, k, tol, flags, n_rr, 1, buf);
        return;
    }
    if constexpr (kN == 16)
        coarse_pairs<TI, false>(v, tab, mode, k, blockIdx.x - 1, sm, buf, nullptr);
    else
        coarse_domain<TI, false>(v, tab, mode, k, blockIdx.x - 1, sm, buf, nullptr);
}

// ---- level 0
// Sum over l >= 1 of y_l at the slot's unit (prolongation of every coarse
// level, Supp. Eq. 6): kProlong levels' unit ids at once, then their
// corrections at once, unconditional loads at clamped levels.  The pair kernel
// loads the first round's ids ahead of the inverses (ahead of them the
// corrections too, registers spill: 16 -> 31 us at 48^3).
constexpr int kProlong = 8;

struct Prolong {
    int u[kProlong];
};

__device__ __forceinline__ void prolong_ids(const SolverView& v, Prolong& R, int slot, int l0 = 0) {
    const int* anc = v.L > 1 ? v.anc : v.remap;  // (no coarse level: a stand-in)
#pragma unroll
    for (int j = 0; j < kProlong; ++j) R.u[j] = anc[static_cast<long long>(max(min(l0 + j, v.L - 2), 0)) * v.NS + slot];
}

__device__ __forceinline__ double prolong_sum(const SolverView& v, const Prolong& R, int c, int l0 = 0) {
    double y[kProlong];
#pragma unroll
    for (int j = 0; j < kProlong; ++j) {
        const double* yl = v.L > 1 ? v.y[min(l0 + j + 1, v.L - 1)] : v.z;
        y[j] = yl[3LL * (v.L > 1 ? max(R.u[j], 0) : 0) + c];
    }
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < kProlong; ++j)
        if (l0 + j + 1 < v.L && R.u[j] >= 0) s += y[j];
    return s;
}

__device__ __forceinline__ double prolong_rest(const SolverView& v, double s, int slot, int c) {
    for (int l0 = kProlong; l0 + 1 < v.L; l0 += kProlong) {
        Prolong R;
        prolong_ids(v, R, slot, l0);
        s += prolong_sum(v, R, c, l0);
    }
    return s;
}

// z = Inv_{0,d} r_d + the prolongation of the coarse corrections and, inside
// PCG, the partial of rho = r^T z.  kApplyPlain: r from src and z to dst, both
// in the caller's node order.  Domain size 16: eight domains per
// workgroup, a pair per wave.
template <typename TI, int kMode>
__global__ void __launch_bounds__(kPairThreads, kPairWaves) k_apply_level0_pairs(SolverView v, int k,
                                                                                 const double* __restrict__ src,
                                                                                 double* __restrict__ dst) {
    __shared__ double sm[4 * kPairLds];
    __shared__ double red[4];
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int b = xcd_group(blockIdx.x, v.GA);
    const int p = 4 * b + w;
    const bool live = 2 * p < v.M;
    int e[2];
    bool own[2];
    double x[2], out[2] = {0.0, 0.0}, cor[2];
    long long at[2];
    Prolong R[2];
    int slot[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        e[q] = 96 * p + pair_row(lane, q);
        own[q] = pair_owns(lane, q) && e[q] < 3 * v.NS;
        slot[q] = own[q] ? e[q] / 3 : 0;
        at[q] = e[q];
        prolong_ids(v, R[q], slot[q]);
        if (kMode == kApplyPlain) {
            const int node = v.remap[slot[q]];
            own[q] = own[q] && node >= 0;
            at[q] = 3LL * node + e[q] % 3;
        }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const double xv = (kMode == kApplyPlain ? src : v.r)[own[q] ? at[q] : 0];
        x[q] = own[q] ? xv : 0.0;
    }
    PairRegs<TI> P;
    pair_load(P, inverses<TI>(v, 0) + static_cast<long long>(live ? p : 0) * kPairEntries, lane);
    const int stop = v.st->done;
    keep_loads_issued();
    if (kMode != kApplyPlain && stop) return;
#pragma unroll
    for (int q = 0; q < 2; ++q) cor[q] = own[q] ? prolong_sum(v, R[q], e[q] % 3) : 0.0;
    if (live) pair_product(P, x, sm + w * kPairLds, lane, out);
    double part = 0.0;
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (own[q]) {
            const double z = out[q] + prolong_rest(v, cor[q], slot[q], e[q] % 3);
            (kMode == kApplyPlain ? dst : v.z)[at[q]] = z;
            part += x[q] * z;
        }
    if (kMode == kApplyPlain) return;
    part = block_sum_last(part, red);
    if (t == 0) v.P_rho[k & 1][b] = part;
}

// The same for other domain sizes: a group of D0 domains per workgroup, one
// thread per DOF.
template <typename TI, int kMode>
__global__ void __launch_bounds__(kGroupThreads) k_apply_level0(SolverView v, int k, const double* __restrict__ src,
                                                                double* __restrict__ dst) {
    __shared__ double rs[kGroupThreads];
    __shared__ double red[16];
    const int n = 3 * v.N;
    const int g = xcd_group(blockIdx.x, v.G), t = threadIdx.x;
    const int nd = min(v.D0, v.M - g * v.D0);  // domains of this group
    const bool live = t < nd * n;
    long long at = 3LL * g * v.RG + t;
    bool own = live;
    if (kMode == kApplyPlain) {
        const int node = live ? v.remap[g * v.RG + t / 3] : -1;
        own = node >= 0;
        at = 3LL * node + t % 3;
    }
    const double rv = own ? (kMode == kApplyPlain ? src : v.r)[at] : 0.0;
    const int stop = v.st->done;
    keep_loads_issued();
    if (kMode != kApplyPlain && stop) return;
    const int slot = live ? g * v.RG + t / 3 : 0;
    Prolong R;
    prolong_ids(v, R, slot);
    const double cor = live ? prolong_rest(v, prolong_sum(v, R, t % 3), slot, t % 3) : 0.0;
    rs[t] = rv;
    __syncthreads();
    double zv = 0.0;
    if (live) {
        const int dl = t / n;
        zv = full_row<TI, true>(inverses<TI>(v, 0) + static_cast<long long>(g * v.D0 + dl) * n * n, n, t - dl * n,
                                rs + dl * n) +
             cor;
        if (own) (kMode == kApplyPlain ? dst : v.z)[at] = zv;
    }
    if (kMode == kApplyPlain) return;
    const double part = block_sum_last(rv * zv, red);
    if (t == 0) v.P_rho[k & 1][g] = part;
}

// ---- apply of a two-launch iteration
// Iteration k by recurrence, in one launch after the SpMV.  Every workgroup
// forms alpha_k from the partials of p^T q and r^T p; the first workgroups take the coarse
// levels (coarse_pairs / coarse_domain), the others perform x += alpha p_k and
// r -= alpha q_k on their level-0 domains and z = Inv_{0,d} r_d, with the
// partials of r^T z and ||r_k||^2.  rho_k = r^T z + sum_l (C_l r)^T y_l is the
// sum of both kinds of partials.  The two do not depend on each other: the
// prolongation, which would make level 0 wait for the coarse levels, is left
// to the next SpMV.  So the coarse levels, a chain of round trips to memory
// that leaves most of the machine idle (7-9 us as a launch of its own at
// 48^3), run beside the streaming of the level-0 inverses.
// pad: coarse workgroups rounded up to whole rounds of XCDs.
template <typename TI>
__global__ void __launch_bounds__(kPairThreads, kPairWaves) k_apply_rec_pairs(SolverView v, CoarseTable tab, int pad, int k) {
    __shared__ double sm[4 * kPairLds];
    __shared__ double buf[512];
    __shared__ double red[16];
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    if (static_cast<int>(blockIdx.x) < pad) {
        if (static_cast<int>(blockIdx.x) < v.ncb) coarse_pairs<TI, true>(v, tab, kApplyIter, k, blockIdx.x, sm, buf, red);
        return;
    }
    const int b = xcd_group(blockIdx.x - pad, v.GA);
    const int p = 4 * b + w;
    const bool live = 2 * p < v.M;
    const RecLoads R = rec_load(v, k);
    int e[2];
    bool own[2];
    double xv[2], pv[2], ro[2], qv[2];
    const double *pk = v.p[k & 1], *qk = v.q;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        e[q] = 96 * p + pair_row(lane, q);
        own[q] = pair_owns(lane, q) && e[q] < 3 * v.NS;
        const int i = own[q] ? e[q] : 0;
        xv[q] = v.x[i];
        pv[q] = pk[i];
        ro[q] = v.r[i];
        qv[q] = qk[i];
    }
    PairRegs<TI> P;
    pair_load(P, inverses<TI>(v, 0) + static_cast<long long>(live ? p : 0) * kPairEntries, lane);
    // the stop flag is read once these loads are in flight; after a stop
    // nothing is written
    const int stop = v.st->done;
    keep_loads_issued();
    if (stop) return;
    double alpha;
    if (!rec_alpha(v, k, b == 0, R, buf, alpha)) return;
    double x[2], out[2] = {0.0, 0.0}, prho = 0.0, prr = 0.0;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        x[q] = 0.0;
        if (!own[q]) continue;
        v.x[e[q]] = xv[q] + alpha * pv[q];
        x[q] = ro[q] - alpha * qv[q];
        v.r[e[q]] = x[q];
    }
    if (live) pair_product(P, x, sm + w * kPairLds, lane, out);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (!own[q]) continue;
        v.z[e[q]] = out[q];
        prho += x[q] * out[q];
        prr += x[q] * x[q];
    }
    double srho, srr;
    block_sum2_last(prho, prr, red, srho, srr);
    if (t == 0) {
        v.P_rho[k & 1][b] = srho;
        v.P_rr[b] = srr;
    }
}

template <typename TI>
__global__ void __launch_bounds__(kGroupThreads) k_apply_rec(SolverView v, CoarseTable tab, int pad, int k) {
    __shared__ double rs[kGroupThreads];
    __shared__ double buf[512];
    __shared__ double red[16];
    const int t = threadIdx.x;
    if (static_cast<int>(blockIdx.x) < pad) {
        if (static_cast<int>(blockIdx.x) < v.ncb) coarse_domain<TI, true>(v, tab, kApplyIter, k, blockIdx.x, rs, buf, red);
        return;
    }
    const int n = 3 * v.N;
    const int g = xcd_group(blockIdx.x - pad, v.G);
    const int nd = min(v.D0, v.M - g * v.D0);  // domains of this group
    const bool live = t < nd * n;
    const long long i = 3LL * g * v.RG + (live ? t : 0);
    const RecLoads R = rec_load(v, k);
    const double xv = v.x[i], pv = v.p[k & 1][i], ro = v.r[i], qv = v.q[i];
    const int stop = v.st->done;
    keep_loads_issued();
    if (stop) return;
    double alpha;
    if (!rec_alpha(v, k, g == 0, R, buf, alpha)) return;
    double rv = 0.0;
    if (live) {
        v.x[i] = xv + alpha * pv;
        rv = ro - alpha * qv;
        v.r[i] = rv;
    }
    rs[t] = rv;
    __syncthreads();
    double zv = 0.0;
    if (live) {
        const int dl = t / n;
        zv = full_row<TI, true>(inverses<TI>(v, 0) + static_cast<long long>(g * v.D0 + dl) * n * n, n, t - dl * n,
                                rs + dl * n);
        v.z[i] = zv;
    }
    double prho, prr;
    block_sum2_last(rv * zv, rv * rv, red, prho, prr);
    if (t == 0) {
        v.P_rho[k & 1][g] = prho;
        v.P_rr[g] = prr;
    }
}

// z += the prolongation of every coarse level, a thread per DOF, and the
// decision on r_k in workgroup 0: the rest of the iteration where the SpMV
// cannot stage the corrections (launch_prolong).
__global__ void __launch_bounds__(256) k_prolong(SolverView v, int k, int flags) {
    __shared__ double buf[256];
    if (blockIdx.x == 0) {
        convergence_decision(v, false, k, 0.0, flags, v.GA, 1, buf);
        return;
    }
    const long long e = static_cast<long long>(blockIdx.x - 1) * 256 + threadIdx.x;
    if (e >= 3LL * v.NS) return;
    const int slot = static_cast<int>(e / 3), c = static_cast<int>(e - 3LL * slot);
    Prolong R;
    prolong_ids(v, R, slot);
    const double z = v.z[e];
    v.z[e] = z + prolong_rest(v, prolong_sum(v, R, c), slot, c);  // (unused after a stop)
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
    if (b.N == 16) {
        int groups[kMaxLv];
        for (int l = 0; l < b.L; ++l) groups[l] = ceil_div(b.ndom[l], kWaveDomains);
        const DomTable tab = make_table(groups, 0, b.L);
        launch_kernel(k_invert_waves, dim3(tab.off[kMaxLv]), dim3(64 * kWaveDomains), 0, s, b, Hu, want32 ? 1 : 0, tab);
        return hipGetLastError();
    }
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

namespace {

CoarseTable coarse_table(const SolverView& v) {
    CoarseTable t{};
    int acc = 0;
    for (int l = 1; l < v.L; ++l) {
        t.off[l] = acc;
        acc += coarse_blocks(v.N, l, v.ndom[l]);
    }
    for (int l = v.L; l <= kMaxLv; ++l) t.off[l] = acc;
    return t;
}

template <typename TI, int kMode>
void launch_level0_t(const SolverView& v, int k, const double* src, double* dst, hipStream_t s) {
    if (v.N == 16)
        launch_kernel((k_apply_level0_pairs<TI, kMode>), dim3(v.GA), dim3(kPairThreads), 0, s, v, k, src, dst);
    else
        launch_kernel((k_apply_level0<TI, kMode>), dim3(v.G), dim3(round_waves(3 * v.RG)), 0, s, v, k, src, dst);
}

template <typename TI>
void launch_rec_t(const SolverView& v, int k, hipStream_t s) {
    const CoarseTable tab = coarse_table(v);
    const int pad = ceil_div(v.ncb, kXcds) * kXcds;
    dim3 g(pad + v.GA);
    if (v.N == 16)
        launch_kernel(k_apply_rec_pairs<TI>, g, dim3(kPairThreads), 0, s, v, tab, pad, k);
    else
        launch_kernel(k_apply_rec<TI>, g, dim3(kGroupThreads), 0, s, v, tab, pad, k);
}

}  // namespace

hipError_t launch_apply_coarse(const SolverView& v, bool f32, int mode, int k, double tol, bool x0_given, bool mixed,
                               bool rr_true, hipStream_t s) {
    const CoarseTable tab = coarse_table(v);
    const dim3 g(1 + v.ncb), b(kPairThreads);  // workgroup 0 decides convergence
    const int flags = (x0_given ? kFlagX0 : 0) | (mixed ? kFlagMixed : 0) | (rr_true ? kFlagRrTrue : 0);
    if (v.N == 16) {
        if (f32) launch_kernel((k_apply_coarse<float, 16>), g, b, 0, s, v, tab, mode, k, tol, flags, v.G);
        else launch_kernel((k_apply_coarse<double, 16>), g, b, 0, s, v, tab, mode, k, tol, flags, v.G);
    } else {
        if (f32) launch_kernel((k_apply_coarse<float, 0>), g, b, 0, s, v, tab, mode, k, tol, flags, v.G);
        else launch_kernel((k_apply_coarse<double, 0>), g, b, 0, s, v, tab, mode, k, tol, flags, v.G);
    }
    return hipGetLastError();
}

hipError_t launch_decision(const SolverView& v, int k, bool mixed, hipStream_t s) {
    launch_kernel((k_apply_coarse<double, 0>), dim3(1), dim3(kPairThreads), 0, s, v, CoarseTable{},
                  static_cast<int>(kApplyIter), k, 0.0, mixed ? kFlagMixed : 0, v.GA);
    return hipGetLastError();
}

hipError_t launch_apply_level0(const SolverView& v, bool f32, int mode, int k, hipStream_t s) {
    if (mode == kApplyInit)
        f32 ? launch_level0_t<float, kApplyInit>(v, k, nullptr, nullptr, s)
            : launch_level0_t<double, kApplyInit>(v, k, nullptr, nullptr, s);
    else
        f32 ? launch_level0_t<float, kApplyIter>(v, k, nullptr, nullptr, s)
            : launch_level0_t<double, kApplyIter>(v, k, nullptr, nullptr, s);
    return hipGetLastError();
}

hipError_t launch_apply_plain(const SolverView& v, bool f32, const double* r, double* z, hipStream_t s) {
    hipError_t e;
    if (v.ncb > 0 && (e = launch_apply_coarse(v, f32, kApplyPlain, 0, 0.0, false, f32, false, s)) != hipSuccess)
        return e;
    f32 ? launch_level0_t<float, kApplyPlain>(v, 0, r, z, s) : launch_level0_t<double, kApplyPlain>(v, 0, r, z, s);
    return hipGetLastError();
}

hipError_t launch_prolong(const SolverView& v, int k, bool mixed, hipStream_t s) {
    launch_kernel(k_prolong, dim3(1 + ceil_div(3LL * v.NS, 256)), dim3(256), 0, s, v, k, mixed ? kFlagMixed : 0);
    return hipGetLastError();
}

hipError_t launch_apply_rec(const SolverView& v, bool f32, int k, hipStream_t s) {
    if (f32)
        launch_rec_t<float>(v, k, s);
    else
        launch_rec_t<double>(v, k, s);
    return hipGetLastError();
}

}  // namespace maspcg

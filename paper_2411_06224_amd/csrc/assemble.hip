// Assembly of a list of 3x3 blocks into 3x3-block CSR (what the hash-based
// reduction of Sec. 6.2 computes: the blocks of equal (row, col) key meet
// contiguously after sorting by key and are reduced segment by segment).
//
// Each listed block gets the key (row << cb) | col, cb the bit width of the
// largest index (n_rows < 2^cb); a stable radix sort of
// (key, list position) pairs (rocPRIM) places equal keys together in list
// order; segment heads and their exclusive scan number the distinct blocks;
// each distinct block is summed over its segment in list order, nine
// threads per block.  The sums are those of a sequential pass over the
// list, and no row length is limited.
//
// That path sorts 12 bytes per listed block in five passes.  Where the rows
// are short (rows_path) the list is grouped by row alone, with one atomic
// per run of equal rows, and each row is sorted by (column, list position)
// on its own, in registers and LDS: the same order, the same sums.
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include <algorithm>

#include "launch.hpp"
#include "replan.hpp"

namespace maspcg {
namespace {

constexpr int kAsmThreads = 256;
constexpr int kWave = 64;
constexpr int kAsmBatch = 4;  // listed blocks loaded together by the segment sums
constexpr int kScanItems = 1024;  // elements per block of the scan

__global__ void k_fill_int(int* __restrict__ p, long long n, int value) {
    const long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) p[i] = value;
}

// Exclusive scan of n ints: per-block scans with block totals (pass 1), a
// scan of the totals (pass 2, one block, at most kScanItems totals), offsets
// added back (pass 3).  out[n] = the grand total.
__device__ inline int block_exclusive_scan(int v, int* sh, int& total) {
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int o = 1; o < kAsmThreads; o <<= 1) {
        const int a = t >= o ? sh[t - o] : 0;
        __syncthreads();
        sh[t] += a;
        __syncthreads();
    }
    total = sh[kAsmThreads - 1];
    const int excl = sh[t] - v;
    __syncthreads();
    return excl;
}

__global__ void __launch_bounds__(kAsmThreads) k_scan_blocks(const int* __restrict__ in, int n, int* __restrict__ out,
                                                             int* __restrict__ totals) {
    __shared__ int sh[kAsmThreads];
    const int base = blockIdx.x * kScanItems + threadIdx.x * 4;
    int v[4], s = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        v[j] = base + j < n ? in[base + j] : 0;
        s += v[j];
    }
    int total;
    int run = block_exclusive_scan(s, sh, total);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (base + j < n) out[base + j] = run;
        run += v[j];
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = total;
}

__global__ void __launch_bounds__(kAsmThreads) k_scan_totals(int* __restrict__ totals, int nb, int* __restrict__ grand) {
    __shared__ int sh[kAsmThreads];
    const int base = threadIdx.x * 4;
    int v[4], s = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        v[j] = base + j < nb ? totals[base + j] : 0;
        s += v[j];
    }
    int total;
    int run = block_exclusive_scan(s, sh, total);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (base + j < nb) totals[base + j] = run;
        run += v[j];
    }
    if (threadIdx.x == 0) *grand = total;
}

__global__ void k_scan_add(int* __restrict__ out, int n, const int* __restrict__ totals) {
    const int i = blockIdx.x * kScanItems + threadIdx.x;
    const int add = totals[blockIdx.x];
    for (int j = i; j < min(n, static_cast<int>(blockIdx.x + 1) * kScanItems); j += blockDim.x) out[j] += add;
}

// Key and list position of every listed block; an index out of range
// raises flag bit 0 (its key sorts last and is never reduced).
__device__ __forceinline__ uint64_t key_sentinel(int cb) { return (1ull << (2 * cb)) - 1; }  // above every valid key

__global__ void __launch_bounds__(kAsmThreads) k_asm_keys(long long n_in, int n_rows, int cb,
                                                          const int* __restrict__ rows, const int* __restrict__ cols,
                                                          uint64_t* __restrict__ key, int* __restrict__ pos,
                                                          int* __restrict__ flag) {
    const long long k = static_cast<long long>(blockIdx.x) * kAsmThreads + threadIdx.x;
    if (k >= n_in) return;
    const int r = rows[k], c = cols[k];
    const bool bad = r < 0 || r >= n_rows || c < 0 || c >= n_rows;
    if (bad) atomicOr(flag, 1);
    key[k] = bad ? key_sentinel(cb) : (static_cast<uint64_t>(r) << cb) | static_cast<uint64_t>(c);
    pos[k] = static_cast<int>(k);
}

__global__ void __launch_bounds__(kAsmThreads) k_asm_heads(long long n_in, const uint64_t* __restrict__ key,
                                                           int* __restrict__ head) {
    const long long k = static_cast<long long>(blockIdx.x) * kAsmThreads + threadIdx.x;
    if (k < n_in) head[k] = (k == 0 || key[k] != key[k - 1]) ? 1 : 0;
}

// Segment starts, row pointers and the number of distinct blocks.  Row r
// begins at the segment of its first sorted entry; rows without blocks take
// the next row's start (every row_ptr entry has one writer).
__global__ void __launch_bounds__(kAsmThreads) k_asm_rows(long long n_in, int n_rows, int cb,
                                                          const uint64_t* __restrict__ key,
                                                          const int* __restrict__ head, const int* __restrict__ seg,
                                                          int* __restrict__ seg_start, int* __restrict__ row_ptr,
                                                          int* __restrict__ flag) {
    const long long k = static_cast<long long>(blockIdx.x) * kAsmThreads + threadIdx.x;
    if (n_in == 0) {
        for (long long r = k; r <= n_rows; r += static_cast<long long>(gridDim.x) * kAsmThreads) row_ptr[r] = 0;
        if (k == 0) flag[1] = 0;
        return;
    }
    if (k >= n_in) return;
    const uint64_t kk = key[k];
    const bool valid = kk < key_sentinel(cb);
    const int r = static_cast<int>(kk >> cb);
    if (head[k] && valid) {
        seg_start[seg[k]] = static_cast<int>(k);
        const int pr = k == 0 ? -1 : static_cast<int>(key[k - 1] >> cb);
        for (int rr = pr + 1; rr <= r; ++rr) row_ptr[rr] = seg[k];
    }
    // the last valid entry closes the remaining rows and counts the blocks
    const bool last = valid && (k + 1 == n_in || key[k + 1] >= key_sentinel(cb));
    if (last) {
        const int total = seg[k] + head[k];
        for (int rr = r + 1; rr <= n_rows; ++rr) row_ptr[rr] = total;
        seg_start[total] = static_cast<int>(k + 1);
        flag[1] = total;
    }
    if (k == 0 && !valid) {  // every index out of range: nothing to assemble
        for (int rr = 0; rr <= n_rows; ++rr) row_ptr[rr] = 0;
        flag[1] = 0;
    }
}

// Distinct block b = t / 9, entry t % 9: the sum over its segment in list
// order (nine consecutive threads read one listed block).  The segment is
// read kAsmBatch entries at a time: their positions, then their values, all
// in flight together, then added in order.
__global__ void __launch_bounds__(kAsmThreads) k_asm_reduce(int nnzb, int cb, const uint64_t* __restrict__ key,
                                                            const int* __restrict__ pos,
                                                            const int* __restrict__ seg_start,
                                                            const double* __restrict__ blocks,
                                                            int* __restrict__ col_idx, double* __restrict__ val) {
    const long long t = static_cast<long long>(blockIdx.x) * kAsmThreads + threadIdx.x;
    if (t >= 9LL * nnzb) return;
    const int b = static_cast<int>(t / 9), c = static_cast<int>(t - 9LL * b);
    const int e0 = seg_start[b], e1 = seg_start[b + 1];
    double acc = 0.0;
    for (int e = e0; e < e1; e += kAsmBatch) {
        int p[kAsmBatch];
#pragma unroll
        for (int j = 0; j < kAsmBatch; ++j) p[j] = pos[min(e + j, e1 - 1)];
        double x[kAsmBatch];
#pragma unroll
        for (int j = 0; j < kAsmBatch; ++j) x[j] = blocks[9LL * p[j] + c];
#pragma unroll
        for (int j = 0; j < kAsmBatch; ++j)
            if (e + j < e1) acc += x[j];
    }
    val[9LL * b + c] = acc;
    if (c == 0) col_idx[b] = static_cast<int>(key[e0] & ((1ull << cb) - 1));
}

// ------------------------------------------------- lists of short rows
//
// cnt[r] blocks of row r are counted, and each learns its slot within the
// row; a scan places the rows; (column, list position) pairs are scattered
// to their slots; a workgroup per few consecutive rows ranks their pairs; a
// second scan makes row_ptr of the distinct columns; a workgroup per few
// rows adds them up.  The slots depend on the order of the atomics, the
// ranks do not: no two pairs are equal.
//
// 9.0 million blocks in 110,592 rows (a 48^3 cube's elements): sort, heads,
// scan and rows take 690 us, the kernels before the sums here 260; 62 thousand
// blocks in 729 rows: 121 -> 76 us for the whole call.  Uneven rows (3.8
// million blocks on the 33 thousand of 279 thousand nodes that touch): 769 ->
// 640 us for the contact reduction around it.

constexpr int kPool = 448;       // blocks of a workgroup's rows sorted and summed together, rows rounded up to 4
constexpr int kPoolAim = 336;    // ... aimed at on average
constexpr int kPoolRows = 63;    // rows of a workgroup, at most
constexpr int kRowGroup = 2048;  // blocks of a longer row that a workgroup sorts in LDS
constexpr int kSliceRows = 8;    // a workgroup per so many rows shares the batches of rows beyond the pool
constexpr int kAsmWaves = kAsmThreads / kWave;

// The arrays of the short-row path in the scratch of the sorting path: each
// of those below holds one int per listed block, or one per row, of which
// there are fewer (rows_path).
struct RowArrays {
    int* cnt;          // blocks per row; [n_rows] = 0
    int* start;        // first pair of each row; [n_rows] = their number
    int* slot;         // of each listed block within its row
    uint64_t* pair;    // (column << 32) | list position, in slot order
    // by workgroup, from start[its first row] (by row, where the rows exceed the pool): the sorted blocks (as slots,
    // or list positions), the first sorted block of each distinct (row, column) and that column
    int *order, *seg_first, *seg_col;
    int* distinct;     // columns per row; [n_rows] = 0
};

RowArrays row_arrays(const AsmLayout& L, long long n_in) {
    return {L.head, L.seg, L.pos, L.key, L.pos_sorted, L.seg_start, reinterpret_cast<int*>(L.key_sorted),
            reinterpret_cast<int*>(L.key_sorted) + n_in};
}

__global__ void __launch_bounds__(kAsmThreads) k_asm_clear(int n_rows, int* __restrict__ cnt,
                                                           int* __restrict__ flag) {
    const long long i = static_cast<long long>(blockIdx.x) * kAsmThreads + threadIdx.x;
    if (i <= n_rows) cnt[i] = 0;
    if (i < 2) flag[i] = 0;
}

// Counting is bound by the atomics (about 25 per ns): one per distinct row of
// a wave, found a row at a time.  An element lists its blocks row by row,
// four to a run, and its neighbours in the list share its nodes: 50 us for
// 9.0 million blocks; 88 with an atomic per run, 565 with one per block.
__global__ void __launch_bounds__(kAsmThreads) k_asm_count(int n_in, int n_rows, const int* __restrict__ rows,
                                                           int* __restrict__ cnt, int* __restrict__ slot,
                                                           int* flag) {
    if (flag[0] & 2) return;
    const int k = blockIdx.x * kAsmThreads + threadIdx.x, lane = threadIdx.x % kWave;
    const int r = k < n_in ? rows[k] : -1;
    const bool valid = r >= 0 && r < n_rows;
    if (k < n_in && !valid) atomicOr(flag, 1);
    unsigned long long left = __ballot(valid);
    int first = lane, same = 0, before = 0;
    while (left) {
        const int l = __ffsll(left) - 1;
        const unsigned long long match = __ballot(r == __builtin_amdgcn_readlane(r, l));
        if (match >> lane & 1) {
            first = l;
            same = __popcll(match);
            before = __popcll(match & ((1ull << lane) - 1ull));
        }
        left &= ~match;
    }
    int base = 0;
    if (valid && lane == first) {
        base = atomicAdd(cnt + r, same);
        if (base + same > kRowGroup) atomicOr(flag, 2);  // the sorting path takes the list: nothing below runs
    }
    base = __shfl(base, first);
    if (k < n_in) slot[k] = base + before;
}

__global__ void __launch_bounds__(kAsmThreads) k_asm_scatter(int n_in, int n_rows, const int* __restrict__ rows,
                                                             const int* __restrict__ cols,
                                                             const int* __restrict__ start,
                                                             const int* __restrict__ slot,
                                                             uint64_t* __restrict__ pair, int* flag) {
    const int k = blockIdx.x * kAsmThreads + threadIdx.x;
    if (k >= n_in || flag[0] & 2) return;
    const int r = rows[k], c = cols[k];
    if (r < 0 || r >= n_rows) return;  // flagged and not counted
    if (c < 0 || c >= n_rows) atomicOr(flag, 1);
    pair[start[r] + slot[k]] = static_cast<uint64_t>(static_cast<uint32_t>(c)) << 32 | static_cast<uint32_t>(k);
}

// Exclusive scan of n <= kScanOne ints by one workgroup: a launch instead of
// the three of the general scan.
constexpr int kScanOne = 16 * kAsmThreads;
__global__ void __launch_bounds__(kAsmThreads) k_scan_one(const int* __restrict__ in, int n, int* __restrict__ out) {
    __shared__ int sh[kAsmThreads];
    const int base = threadIdx.x * 16;
    int v[16], s = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        v[j] = base + j < n ? in[base + j] : 0;
        s += v[j];
    }
    int total;
    int run = block_exclusive_scan(s, sh, total);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        if (base + j < n) out[base + j] = run;
        run += v[j];
    }
}

// The rows of a workgroup: where each begins among its blocks, and in the
// pool, with every row rounded up to four.
struct PoolRows {
    int st[kPoolRows + 1], base[kPoolRows + 1];
};

__device__ __forceinline__ void pool_rows(PoolRows& P, int r0, int nr, const int* __restrict__ start) {
    if (threadIdx.x < kWave) {
        const int lane = threadIdx.x;
        const int s = start[r0 + min(lane, nr)], len = start[r0 + min(lane + 1, nr)] - s;
        int end = (len + 3) & ~3;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int y = __shfl_up(end, o);
            if (lane >= o) end += y;
        }
        if (lane <= nr) {
            P.st[lane] = s - __shfl(s, 0);
            P.base[lane] = end - ((len + 3) & ~3);
        }
    }
    __syncthreads();
}

// The row of place e: at[row] <= e < at[row + 1] (at: st or base).
__device__ __forceinline__ int pool_row(const int* at, int nr, int e) {
    int lo = 0, hi = nr;
    while (hi - lo > 1) {
        const int mid = (lo + hi) / 2;
        if (at[mid] <= e) lo = mid;
        else hi = mid;
    }
    return lo;
}

// A workgroup's rows go through the pool in batches: the rows from w0 that
// fit it together, or one row.
__device__ __forceinline__ int batch_end(const PoolRows& P, int nr, int w0) {
    const int end = P.base[w0] + kPool;
    return P.base[nr] <= end ? nr : max(w0 + 1, pool_row(P.base, nr, end));
}

// Sorts the rows.  A pair's place is the number of smaller pairs of its row,
// counted against the whole row read from LDS four pairs at a time, for two
// pairs per lane (the LDS reads bound the loop): no exchange steps and no
// waits between them, and rows of any mix of lengths share the lanes.  The
// pairs are compared as doubles (rows_path), not as 64-bit integers.  A row
// beyond the pool is sorted by the whole workgroup (bitonic, in LDS).  9.0 million blocks: 131 us (214 with a pair
// per lane, 448 with a wave per row).
__global__ void __launch_bounds__(kAsmThreads) k_asm_row_sort(int n_rows, int group_rows, int slices,
                                                              const int* __restrict__ start,
                                                              const uint64_t* __restrict__ pair,
                                                              int* __restrict__ order, int* __restrict__ seg_first,
                                                              int* __restrict__ seg_col, int* __restrict__ distinct,
                                                              const int* __restrict__ flag) {
    __shared__ __align__(16) uint64_t sh[kRowGroup];
    __shared__ PoolRows P;
    __shared__ int heads_of[kPoolRows], wave_heads[2][kAsmWaves];
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int groups = gridDim.x / slices, slice = blockIdx.x / groups;
    const int r0 = (blockIdx.x - slice * groups) * group_rows, nr = min(group_rows, n_rows - r0);
    if (blockIdx.x == 0 && threadIdx.x == 0) distinct[n_rows] = 0;
    if (uniform_load(flag) & 2) return;
    const int g0 = uniform_load(start + r0);
    if (slice > 0 && uniform_load(start + r0 + nr) - g0 + 3 * nr <= kPool) return;  // within the pool
    pool_rows(P, r0, nr, start);
    for (int i = 0, w0 = 0, w1; w0 < nr; ++i, w0 = w1) {
        w1 = batch_end(P, nr, w0);
        if (i % slices != slice) continue;
        const int t0 = P.st[w0], p0 = P.base[w0], s0 = g0 + t0, total = P.st[w1] - t0;
        __syncthreads();
        if (P.base[w1] - p0 <= kPool) {
            double* pool = reinterpret_cast<double*>(sh);
            int* col = reinterpret_cast<int*>(pool + kPool);
            int row[2];
            double a[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int e = threadIdx.x + q * kAsmThreads;
                if (e < kPool) sh[e] = ~0ull;  // not less than any pair
                row[q] = pool_row(P.st, nr, t0 + max(min(e, total - 1), 0));
                if (e < total) a[q] = __longlong_as_double(static_cast<long long>(pair[s0 + e]));
            }
            if (threadIdx.x < kPoolRows) heads_of[threadIdx.x] = 0;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int e = threadIdx.x + q * kAsmThreads;
                if (e < total) pool[P.base[row[q]] - p0 + e - (P.st[row[q]] - t0)] = a[q];
            }
            __syncthreads();
            const int p = 2 * threadIdx.x;  // two neighbours of the pool, of one row
            if (p < P.base[w1] - p0) {
                const int w = pool_row(P.base, nr, p0 + p), a0 = P.base[w] - p0, a1 = P.base[w + 1] - p0;
                const double2 a = *reinterpret_cast<const double2*>(pool + p);
                int rank[2] = {0, 0};
                for (int j = a0; j < a1; j += 4) {
                    const double2 b = *reinterpret_cast<const double2*>(pool + j);
                    const double2 d = *reinterpret_cast<const double2*>(pool + j + 2);
                    rank[0] += (b.x < a.x) + (b.y < a.x) + (d.x < a.x) + (d.y < a.x);
                    rank[1] += (b.x < a.y) + (b.y < a.y) + (d.x < a.y) + (d.y < a.y);
                }
                const int s1 = P.st[w] - t0, len = P.st[w + 1] - P.st[w];
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    if (p + q - a0 < len) {
                        order[s0 + s1 + rank[q]] = s1 + p + q - a0;
                        col[s1 + rank[q]] = __double2hiint(q ? a.y : a.x);
                    }
            }
            __syncthreads();
            unsigned long long heads[2];
            bool head[2];
            int c[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int e = threadIdx.x + q * kAsmThreads;
                c[q] = e < total ? col[e] : 0;
                head[q] = e < total && (e == (P.st[row[q]] - t0) || col[e - 1] != c[q]);
                heads[q] = __ballot(head[q]);
                if (lane == 0) wave_heads[q][wave] = __popcll(heads[q]);
                if (head[q]) atomicAdd(&heads_of[row[q]], 1);
            }
            __syncthreads();
            int found = 0;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                int j = found;
                for (int v = 0; v < kAsmWaves; ++v) {
                    if (v < wave) j += wave_heads[q][v];
                    found += wave_heads[q][v];
                }
                if (head[q]) {
                    j += s0 + __popcll(heads[q] & ((1ull << lane) - 1ull));
                    seg_first[j] = threadIdx.x + q * kAsmThreads;
                    seg_col[j] = c[q];
                }
            }
            if (w0 + static_cast<int>(threadIdx.x) < w1)
                distinct[r0 + w0 + threadIdx.x] = heads_of[w0 + threadIdx.x];
            continue;
        }
        const int n = total;  // one row beyond the pool
        int width = 2;
        while (width < n) width *= 2;
        for (int i = threadIdx.x; i < width; i += kAsmThreads) sh[i] = i < n ? pair[s0 + i] : ~0ull;
        for (int k = 2; k <= width; k *= 2)
            for (int j = k / 2; j > 0; j /= 2) {
                __syncthreads();
                for (int t = threadIdx.x; t < width / 2; t += kAsmThreads) {
                    const int i = 2 * (t & ~(j - 1)) + (t & (j - 1));
                    const uint64_t x = sh[i], y = sh[i + j];
                    if ((x > y) == ((i & k) == 0)) sh[i] = y, sh[i + j] = x;
                }
            }
        __syncthreads();
        int found = 0;
        for (int i0 = 0; i0 < n; i0 += kAsmThreads) {
            const int i = i0 + threadIdx.x;
            const uint64_t x = i < n ? sh[i] : 0;
            const bool head = i < n && (i == 0 || sh[i - 1] >> 32 != x >> 32);
            const unsigned long long heads = __ballot(head);
            if (lane == 0) wave_heads[0][wave] = __popcll(heads);
            __syncthreads();
            int at = s0 + found;
            for (int v = 0; v < kAsmWaves; ++v) {
                if (v < wave) at += wave_heads[0][v];
                found += wave_heads[0][v];
            }
            if (i < n) order[s0 + i] = static_cast<int>(x & 0xffffffffu);
            if (head) {
                at += __popcll(heads & ((1ull << lane) - 1ull));
                seg_first[at] = i;
                seg_col[at] = static_cast<int>(x >> 32);
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) distinct[r0 + w0] = found;
    }
}

// Sums the rows, in list order within a distinct column.  The values of a
// workgroup's rows are loaded flat, in slot order -- an element's run of
// blocks is one piece of memory -- all in flight at once, turned in LDS and
// added from there, nine lanes to a column; those of rows that exceed the
// pool are gathered, kAsmBatch at a time.  Does nothing where an index was
// out of range, a row too long, or the result larger than capacity.
//
// Bound by the reading of the values, 9.0 million x 72 bytes: 270 us with
// nine threads per column reading straight from memory, now 254 us (2.7
// TB/s).  Smaller pools of two rows (224, 256, 320 blocks) take 3 to 11 %
// longer over the whole call, and so do three rows in this one.
__global__ void __launch_bounds__(kAsmThreads) k_asm_row_sum(int n_rows, int group_rows, int slices,
                                                             long long capacity,
                                                             const int* __restrict__ start,
                                                             const uint64_t* __restrict__ pair,
                                                             const int* __restrict__ order,
                                                             const int* __restrict__ seg_first,
                                                             const int* __restrict__ seg_col,
                                                             int* __restrict__ flag,
                                                             const int* __restrict__ row_ptr,
                                                             const double* __restrict__ blocks,
                                                             int* __restrict__ col_idx, double* __restrict__ val) {
    __shared__ double x[9 * kPool];
    __shared__ int pos[kPool], ord[kPool], first[kPool + 1];
    __shared__ PoolRows P;
    constexpr int kLoads = 4, kBatches = (9 * kPool + kLoads * kAsmThreads - 1) / (kLoads * kAsmThreads);
    const int nnzb = uniform_load(row_ptr + n_rows);
    if (blockIdx.x == 0 && threadIdx.x == 0) flag[1] = nnzb;
    if (uniform_load(static_cast<const int*>(flag)) != 0 || nnzb > capacity) return;
    const int groups = gridDim.x / slices, slice = blockIdx.x / groups;
    const int r0 = (blockIdx.x - slice * groups) * group_rows, nr = min(group_rows, n_rows - r0);
    const int g0 = uniform_load(start + r0);
    if (slice > 0 && uniform_load(start + r0 + nr) - g0 + 3 * nr <= kPool) return;  // within the pool
    pool_rows(P, r0, nr, start);
    for (int i = 0, w0 = 0, w1; w0 < nr; ++i, w0 = w1) {
        w1 = batch_end(P, nr, w0);
        if (i % slices != slice) continue;
        const int s0 = g0 + P.st[w0], total = __builtin_amdgcn_readfirstlane(P.st[w1] - P.st[w0]);
        const int o0 = row_ptr[r0 + w0], n = row_ptr[r0 + w1] - o0;
        if (P.base[w1] - P.base[w0] <= kPool) {
            __syncthreads();
            for (int i = threadIdx.x; i < total; i += kAsmThreads) {
                pos[i] = static_cast<int>(pair[s0 + i] & 0xffffffffu);
                ord[i] = 9 * order[s0 + i];
                first[i] = i < n ? seg_first[s0 + i] : total;
            }
            if (threadIdx.x == 0) first[total] = total;
            __syncthreads();
            double v[kBatches][kLoads];
#pragma unroll
            for (int b = 0; b < kBatches; ++b)
                if (b * kLoads * kAsmThreads < 9 * total)
#pragma unroll
                    for (int q = 0; q < kLoads; ++q) {
                        const int t = threadIdx.x, e = min((b * kLoads + q) * kAsmThreads + t, 9 * total - 1);
                        const int i = e / 9;
                        v[b][q] = blocks[9LL * pos[i] + (e - 9 * i)];
                    }
#pragma unroll
            for (int b = 0; b < kBatches; ++b)
                if (b * kLoads * kAsmThreads < 9 * total)
#pragma unroll
                    for (int q = 0; q < kLoads; ++q) {
                        const int e = (b * kLoads + q) * kAsmThreads + threadIdx.x;
                        if (e < 9 * total) x[e] = v[b][q];
                    }
            __syncthreads();
            const int c = threadIdx.x % 9;
            for (int j = threadIdx.x / 9; j < n && threadIdx.x < kAsmThreads / 9 * 9; j += kAsmThreads / 9) {
                const int e0 = first[j], e1 = first[j + 1];
                double acc = 0.0;
                for (int e = e0; e < e1; e += kAsmBatch) {
                    double y[kAsmBatch];
#pragma unroll
                    for (int q = 0; q < kAsmBatch; ++q) y[q] = x[ord[min(e + q, e1 - 1)] + c];
#pragma unroll
                    for (int q = 0; q < kAsmBatch; ++q)
                        if (e + q < e1) acc += y[q];
                }
                val[9LL * (o0 + j) + c] = acc;
                if (c == 0) col_idx[o0 + j] = seg_col[s0 + j];
            }
            continue;
        }
        for (int t = threadIdx.x; t < 9 * n; t += kAsmThreads) {
            const int j = t / 9, c = t - 9 * j;
            const int e0 = seg_first[s0 + j], e1 = j + 1 < n ? seg_first[s0 + j + 1] : total;
            double acc = 0.0;
            for (int e = e0; e < e1; e += kAsmBatch) {
                double y[kAsmBatch];
#pragma unroll
                for (int q = 0; q < kAsmBatch; ++q) y[q] = blocks[9LL * order[s0 + min(e + q, e1 - 1)] + c];
#pragma unroll
                for (int q = 0; q < kAsmBatch; ++q)
                    if (e + q < e1) acc += y[q];
            }
            val[9LL * (o0 + j) + c] = acc;
            if (c == 0) col_idx[o0 + j] = seg_col[s0 + j];
        }
    }
}

// Lists from 2 million blocks are sampled first (6 us): the pairs of equal
// rows among kSamples blocks of the list are kSamples^2 / (2 n) times the mean
// length of a block's row.  Beyond 1,000 (bodies in many contacts) the atomics
// meet on few addresses (20.0 million blocks, most in 8,000 rows: 275 us of
// counting against 1,770 for the whole by sorting) and some row is beyond
// kRowGroup.  The launches below then return at once, 135 us in all for that
// list, so from 16 million blocks the host reads the answer first (20 us).
constexpr int kSamples = 1024, kSampleSlots = 2 * kSamples, kSampleThreads = kSamples;
constexpr long long kSampleFrom = 1 << 21, kSampleRead = 1 << 24;
constexpr int kSampleLength = 1000;

__global__ void __launch_bounds__(kSampleThreads) k_asm_sample(int n_in, const int* __restrict__ rows,
                                                               int* __restrict__ flag) {
    __shared__ int key[kSampleSlots], cnt[kSampleSlots];
    __shared__ int total;
    for (int i = threadIdx.x; i < kSampleSlots; i += kSampleThreads) key[i] = -1, cnt[i] = 0;
    if (threadIdx.x == 0) total = 0;
    __syncthreads();
    const int step = n_in / kSamples;
    for (int i = threadIdx.x; i < kSamples; i += kSampleThreads) {
        const unsigned mix = static_cast<unsigned>(i) * 2654435761u;
        const int r = rows[static_cast<long long>(i) * step + (mix >> 8) % step];
        if (r < 0) continue;
        unsigned at = (static_cast<unsigned>(r) * 2654435761u) >> 21;  // 11 bits
        while (true) {  // at most half of the slots are ever taken
            const int old = atomicCAS(&key[at], -1, r);
            if (old == -1 || old == r) break;
            at = (at + 1) % kSampleSlots;
        }
        const int before = atomicAdd(&cnt[at], 1);
        if (before) atomicAdd(&total, before);
    }
    __syncthreads();
    if (threadIdx.x == 0 && 2.0 * n_in * total > static_cast<double>(kSampleLength) * kSamples * kSamples)
        flag[0] = 2;  // the sorting path takes the list: nothing below runs
}

// At most 512 blocks per row on average, and more blocks than rows, so that
// the arrays by row fit the scratch (of a size by the list): below, most
// waves would find an empty row; above, the rows are long for one wave and
// the atomics meet on few addresses.
// The pairs are compared as the doubles of the same bits, which order alike
// while a column's stay below those of infinity.
bool rows_path(int n_rows, long long n_in) {
    return n_in > n_rows && n_in <= 512LL * n_rows && n_rows < 0x7ff00000;
}

size_t tmp_bytes(long long n_in, int key_bits) {
    const int n = static_cast<int>(std::max<long long>(n_in, 1));
    size_t sb = 0, scb = 0;
    rocprim::radix_sort_pairs(nullptr, sb, static_cast<uint64_t*>(nullptr), static_cast<uint64_t*>(nullptr),
                              static_cast<int*>(nullptr), static_cast<int*>(nullptr), n, 0, key_bits);
    rocprim::exclusive_scan(nullptr, scb, static_cast<int*>(nullptr), static_cast<int*>(nullptr), 0, n,
                            rocprim::plus<int>());
    return std::max(sb, scb);
}

// Bit width of the indices of an n_rows system: the smallest cb with
// n_rows < 2^cb, so that every valid key stays below the sentinel.
int index_bits(int n_rows) {
    int cb = 1;
    while (cb < 31 && (1LL << cb) <= n_rows) ++cb;
    return cb;
}

}  // namespace

AsmLayout assemble_layout(char* ws, int n_rows, long long n_in, size_t* total) {
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char* p = ws ? ws + off : nullptr;
        off += (std::max<size_t>(bytes, 1) + 255) / 256 * 256;
        return p;
    };
    const size_t m = n_in > 0 ? static_cast<size_t>(n_in) : 1;
    AsmLayout L{};
    L.key = reinterpret_cast<uint64_t*>(take(sizeof(uint64_t) * m));
    L.key_sorted = reinterpret_cast<uint64_t*>(take(sizeof(uint64_t) * m));
    L.pos = reinterpret_cast<int*>(take(sizeof(int) * m));
    L.pos_sorted = reinterpret_cast<int*>(take(sizeof(int) * m));
    L.head = reinterpret_cast<int*>(take(sizeof(int) * m));
    L.seg = reinterpret_cast<int*>(take(sizeof(int) * m));
    L.seg_start = reinterpret_cast<int*>(take(sizeof(int) * (m + 1)));
    L.flag = reinterpret_cast<int*>(take(sizeof(int) * 2));
    L.cb = index_bits(n_rows);
    L.tmp_bytes = tmp_bytes(n_in, 2 * L.cb);
    L.tmp = take(L.tmp_bytes);
    if (total) *total = off;
    return L;
}

hipError_t launch_scan(const int* in, int n, int* out, int* totals, hipStream_t s) {
    const int nb = (n + kScanItems - 1) / kScanItems;
    if (nb > 4 * kAsmThreads) return hipErrorInvalidValue;
    launch_kernel(k_scan_blocks, dim3(nb), dim3(kAsmThreads), 0, s, in, n, out, totals);
    launch_kernel(k_scan_totals, dim3(1), dim3(kAsmThreads), 0, s, totals, nb, out + n);
    launch_kernel(k_scan_add, dim3(nb), dim3(kAsmThreads), 0, s, out, n, static_cast<const int*>(totals));
    return hipGetLastError();
}

hipError_t launch_assemble_sort(const AsmLayout& L, int n_rows, long long n_in, const int* rows, const int* cols,
                                int* row_ptr, hipStream_t s) {
    launch_kernel(k_fill_int, dim3(1), dim3(64), 0, s, L.flag, 2LL, 0);
    if (n_in > 0)
        launch_kernel(k_asm_keys, dim3(ceil_div(n_in, kAsmThreads)), dim3(kAsmThreads), 0, s, n_in, n_rows, L.cb, rows,
                      cols, L.key, L.pos, L.flag);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_assemble_sort_keys(L, n_rows, n_in, row_ptr, s, false);
}

hipError_t launch_assemble_sort_keys(const AsmLayout& L, int n_rows, long long n_in, int* row_ptr, hipStream_t s,
                                     bool clear_flag) {
    if (clear_flag) launch_kernel(k_fill_int, dim3(1), dim3(64), 0, s, L.flag, 2LL, 0);
    hipError_t e;
    if (n_in > 0) {
        const int g = ceil_div(n_in, kAsmThreads);
        size_t bytes = L.tmp_bytes;
        if ((e = rocprim::radix_sort_pairs(L.tmp, bytes, L.key, L.key_sorted, L.pos, L.pos_sorted,
                                           static_cast<int>(n_in), 0, 2 * L.cb, s)) != hipSuccess)
            return e;
        launch_kernel(k_asm_heads, dim3(g), dim3(kAsmThreads), 0, s, n_in, static_cast<const uint64_t*>(L.key_sorted),
                      L.head);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        bytes = L.tmp_bytes;
        if ((e = rocprim::exclusive_scan(L.tmp, bytes, L.head, L.seg, 0, static_cast<int>(n_in),
                                         rocprim::plus<int>(), s)) != hipSuccess)
            return e;
        launch_kernel(k_asm_rows, dim3(g), dim3(kAsmThreads), 0, s, n_in, n_rows, L.cb,
                      static_cast<const uint64_t*>(L.key_sorted), static_cast<const int*>(L.head),
                      static_cast<const int*>(L.seg), L.seg_start, row_ptr, L.flag);
    } else {
        launch_kernel(k_asm_rows, dim3(ceil_div(n_rows + 1, kAsmThreads)), dim3(kAsmThreads), 0, s, 0LL, n_rows,
                      L.cb, static_cast<const uint64_t*>(L.key_sorted), static_cast<const int*>(L.head),
                      static_cast<const int*>(L.seg), L.seg_start, row_ptr, L.flag);
    }
    return hipGetLastError();
}

hipError_t launch_assemble_reduce(const AsmLayout& L, long long n_in, const double* blocks, int* col_idx, double* val,
                                  int nnzb, hipStream_t s) {
    (void)n_in;
    if (nnzb <= 0) return hipSuccess;
    launch_kernel(k_asm_reduce, dim3(ceil_div(9LL * nnzb, kAsmThreads)), dim3(kAsmThreads), 0, s, nnzb, L.cb,
                  static_cast<const uint64_t*>(L.key_sorted), static_cast<const int*>(L.pos_sorted),
                  static_cast<const int*>(L.seg_start), blocks, col_idx, val);
    return hipGetLastError();
}

hipError_t launch_assemble_rows(const AsmLayout& L, int n_rows, long long n_in, const int* rows, const int* cols,
                                const double* blocks, int* row_ptr, int* col_idx, double* val, long long capacity,
                                hipStream_t s, bool* taken) {
    *taken = false;
    if (!rows_path(n_rows, n_in)) return hipSuccess;
    const int n = static_cast<int>(n_in);
    const RowArrays A = row_arrays(L, n_in);
    hipError_t e;
    auto scan = [&](const int* in, int* out) -> hipError_t {
        if (n_rows < kScanOne) {
            launch_kernel(k_scan_one, dim3(1), dim3(kAsmThreads), 0, s, in, n_rows + 1, out);
            return hipGetLastError();
        }
        size_t bytes = L.tmp_bytes;
        return rocprim::exclusive_scan(L.tmp, bytes, in, out, 0, n_rows + 1, rocprim::plus<int>(), s);
    };
    launch_kernel(k_asm_clear, dim3(ceil_div(n_rows + 1LL, kAsmThreads)), dim3(kAsmThreads), 0, s, n_rows, A.cnt,
                  L.flag);
    if (n_in >= kSampleFrom) {
        launch_kernel(k_asm_sample, dim3(1), dim3(kSampleThreads), 0, s, n, rows, L.flag);
        if (n_in >= kSampleRead) {
            int flag = 0;
            if ((e = hipGetLastError()) != hipSuccess ||
                (e = hipMemcpyAsync(&flag, L.flag, sizeof(int), hipMemcpyDeviceToHost, s)) != hipSuccess ||
                (e = hipStreamSynchronize(s)) != hipSuccess)
                return e;
            if (flag & 2) return hipSuccess;
        }
    }
    launch_kernel(k_asm_count, dim3(ceil_div(n_in, kAsmThreads)), dim3(kAsmThreads), 0, s, n, n_rows, rows, A.cnt,
                  A.slot, L.flag);
    if ((e = hipGetLastError()) != hipSuccess || (e = scan(A.cnt, A.start)) != hipSuccess) return e;
    launch_kernel(k_asm_scatter, dim3(ceil_div(n_in, kAsmThreads)), dim3(kAsmThreads), 0, s, n, n_rows, rows, cols,
                  static_cast<const int*>(A.start), static_cast<const int*>(A.slot), A.pair, L.flag);
    const int group_rows = static_cast<int>(std::clamp<long long>(kPoolAim * static_cast<long long>(n_rows) / n_in, 1,
                                                                  kPoolRows));
    const int slices = ceil_div(group_rows, kSliceRows);
    const dim3 grid(ceil_div(n_rows, group_rows) * slices);
    launch_kernel(k_asm_row_sort, grid, dim3(kAsmThreads), 0, s, n_rows, group_rows, slices,
                  static_cast<const int*>(A.start),
                  static_cast<const uint64_t*>(A.pair), A.order, A.seg_first, A.seg_col, A.distinct,
                  static_cast<const int*>(L.flag));
    if ((e = hipGetLastError()) != hipSuccess || (e = scan(A.distinct, row_ptr)) != hipSuccess) return e;
    launch_kernel(k_asm_row_sum, grid, dim3(kAsmThreads), 0, s, n_rows, group_rows, slices, capacity,
                  static_cast<const int*>(A.start),
                  static_cast<const uint64_t*>(A.pair), static_cast<const int*>(A.order),
                  static_cast<const int*>(A.seg_first), static_cast<const int*>(A.seg_col), L.flag,
                  static_cast<const int*>(row_ptr), blocks, col_idx, val);
    *taken = true;
    return hipGetLastError();
}

}  // namespace maspcg

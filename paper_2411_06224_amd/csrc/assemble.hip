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
// are short on average (rows_path) the list is grouped by row alone, with one
// atomic per distinct row of a wave, and each row is sorted by (column, list
// position) on its own, in registers and LDS: the same order, the same sums.
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include <algorithm>
#include <type_traits>

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
// rows adds them up.  What does not fit a workgroup's pool is dealt to all of
// them (group_items).  The slots depend on the order of the atomics, the
// ranks do not: no two pairs are equal.
//
// 9.0 million blocks in 110,592 rows (a 48^3 cube's elements): sort, heads,
// scan and rows take 690 us, the kernels before the sums here 260; 62 thousand
// blocks in 729 rows: 121 -> 76 us for the whole call.  Bodies in contact
// beside elements, the whole call by sorting and here: 0.23 million blocks (a
// sheet of 64^2 cells with 31 bodies) 201 -> 115 us; 3.7 million (256^2, 500
// bodies, rows of up to 735) 504 -> 340; rows of 1,200 in lists of 0.03, 0.3
// and 9 million 149 -> 127, 254 -> 145 and 1,091 -> 920 us.  Slower than by
// sorting are small lists with a single long row (3,000 of 30,000 blocks: 129
// -> 175 us, of which its pieces take 55) and lists in mixed order whose rows
// are hit from everywhere (1.5 million blocks, half of them on 250 rows: 339 ->
// 600 us; see k_asm_sample for longer ones).

constexpr int kPool = 448;       // blocks of a workgroup's rows sorted and summed together, rows rounded up to 4
constexpr int kPoolAim = 336;    // ... aimed at on average
constexpr int kPoolRows = 24;    // rows of a workgroup, at most (with 12, 3.0 million blocks, 3 a row, take 829 us for 630)
constexpr int kPiece = 1024;     // blocks of a longer row that a workgroup places
constexpr int kChunk = 2048;     // ... among so many at a time
constexpr int kRowLimit = 8192;  // blocks of a row, at most
constexpr int kSumTile = kAsmThreads;  // sorted blocks of a longer row that a workgroup sums
constexpr int kAsmWaves = kAsmThreads / kWave;

// The arrays of the short-row path in the scratch of the sorting path: each
// of those below holds one int per listed block, or one per row, of which
// there are fewer (rows_path).
struct RowArrays {
    int* cnt;          // blocks per row; [n_rows] = 0
    int* start;        // first pair of each row; [n_rows] = their number
    int* slot;         // of each listed block within its row
    uint64_t* pair;    // (column << 32) | list position, in slot order
    // by batch, from start[its first row]: the sorted blocks (as slots of the batch), the first sorted block of each
    // distinct (row, column) and that column; of a row beyond the pool the sorted list positions and their columns
    int *order, *seg_first, *seg_col;
    int* distinct;     // columns per row; [n_rows] = 0
    int* item;         // flag[2] pairs of ints: (row, piece) of a row beyond the pool, (row, -rows) of a batch
};

RowArrays row_arrays(const AsmLayout& L, int n_rows, long long n_in) {
    return {L.head, L.seg, L.pos, L.key, L.pos_sorted, L.seg_start, reinterpret_cast<int*>(L.key_sorted),
            reinterpret_cast<int*>(L.key_sorted) + n_in, L.head + n_rows + 1};
}

__global__ void __launch_bounds__(kAsmThreads) k_asm_clear(int n_rows, int* __restrict__ cnt,
                                                           int* __restrict__ flag) {
    const long long i = static_cast<long long>(blockIdx.x) * kAsmThreads + threadIdx.x;
    if (i <= n_rows) cnt[i] = 0;
    if (i < 3) flag[i] = 0;
}

// Counting is bound by the atomics (about 25 per ns): one per distinct row of
// a wave, found a row at a time.  An element lists its blocks row by row,
// four to a run, and its neighbours in the list share its nodes: 50 us for
// 9.0 million blocks; 88 with an atomic per run, 565 with one per block.  In
// mixed order there is little to find: the search ends after kCountRounds rows.
constexpr int kCountRounds = 16;  // rows of a wave found so; the rest take an atomic each
__global__ void __launch_bounds__(kAsmThreads) k_asm_count(int n_in, int n_rows,
                                                           const int* __restrict__ rows, int* __restrict__ cnt,
                                                           int* __restrict__ slot, int* flag) {
    if (flag[0] & 2) return;
    const int k = blockIdx.x * kAsmThreads + threadIdx.x, lane = threadIdx.x % kWave;
    const int r = k < n_in ? rows[k] : -1;
    const bool valid = r >= 0 && r < n_rows;
    if (k < n_in && !valid) atomicOr(flag, 1);
    unsigned long long left = __ballot(valid);
    int first = lane, same = 0, before = 0;
    for (int round = 0; left && round < kCountRounds; ++round) {
        const int l = __ffsll(left) - 1;
        const unsigned long long match = __ballot(r == __builtin_amdgcn_readlane(r, l));
        if (match >> lane & 1) {
            first = l;
            same = __popcll(match);
            before = __popcll(match & ((1ull << lane) - 1ull));
        }
        left &= ~match;
    }
    if (left >> lane & 1) same = 1;
    int base = 0;
    if (valid && lane == first) {
        base = atomicAdd(cnt + r, same);
        if (base + same > kRowLimit) atomicOr(flag, 2);  // the sorting path takes the list: nothing below runs
    }
    base = __shfl(base, first);
    if (k < n_in) slot[k] = base + before;
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

// Rows that follow one another: where each begins among their blocks, and in
// the pool, with every row rounded up to four.  A row beyond the pool counts
// as more than the pool, so that it stands alone.
__host__ __device__ __forceinline__ int pool_place(int len) { return len > kPool ? kPool + 4 : (len + 3) & ~3; }

struct PoolRows {
    int st[kPoolRows + 1], base[kPoolRows + 1];
};

__device__ __forceinline__ void pool_rows(PoolRows& P, int r0, int nr, const int* __restrict__ start) {
    if (threadIdx.x < kWave) {
        const int lane = threadIdx.x;
        const int s = start[r0 + min(lane, nr)], len = start[r0 + min(lane + 1, nr)] - s;
        const int place = pool_place(len);
        int end = place;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int y = __shfl_up(end, o);
            if (lane >= o) end += y;
        }
        if (lane <= nr) {
            P.st[lane] = s - __shfl(s, 0);
            P.base[lane] = end - place;
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

// The rows from the first that fit the pool together, or one row.
__device__ __forceinline__ int batch_end(const PoolRows& P, int nr) {
    return P.base[nr] <= kPool ? nr : max(1, pool_row(P.base, nr, kPool));
}

// A group's rows are cut into batches by that rule.  Its workgroup takes the
// first; those after it, and the pieces of rows beyond the pool, are items,
// dealt to all workgroups: rows of any mix of lengths may lie side by side.
// visit(i, k): pieces k = 0, 1, ... of row r0 + i, or a batch of -k rows from
// there (k < 0).
template <typename F>
__device__ __forceinline__ void group_items(int r0, int nr, const int* __restrict__ start, F&& visit) {
    constexpr int kLoads = 8;
    int from = 0, base = 0, s = start[r0];
    auto batch = [&](int to) {
        if (from > 0 && base <= kPool) visit(from, from - to);
        from = to;
        base = 0;
    };
    for (int i0 = 0; i0 < nr; i0 += kLoads) {
        int e[kLoads];  // (their loads in flight together)
#pragma unroll
        for (int j = 0; j < kLoads; ++j) e[j] = start[r0 + min(i0 + j + 1, nr)];
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            const int i = i0 + j, len = e[j] - s;
            if (i >= nr) break;
            s = e[j];
            if (i > from && base + pool_place(len) > kPool) batch(i);
            base += pool_place(len);
            if (len > kPool)
                for (int k = 0; k * kPiece < len; ++k) visit(i, k);
        }
    }
    batch(nr);
}

__global__ void __launch_bounds__(kAsmThreads) k_asm_scatter(int n_in, int n_rows, const int* __restrict__ rows,
                                                             const int* __restrict__ cols,
                                                             const int* __restrict__ start,
                                                             const int* __restrict__ slot, int group_rows,
                                                             uint64_t* __restrict__ pair, int* __restrict__ distinct,
                                                             int* __restrict__ item, int* flag) {
    if (flag[0] & 2) return;
    const int k = blockIdx.x * kAsmThreads + threadIdx.x, lane = threadIdx.x % kWave;
    const int r = k < n_in ? rows[k] : -1;
    const bool valid = r >= 0 && r < n_rows;  // (else flagged and not counted)
    int items = 0, r0 = 0, nr = 0;
    if (valid) {
        const int c = cols[k], at = slot[k], s0 = start[r];
        const bool bad = c < 0 || c >= n_rows;
        if (bad) atomicOr(flag, 1);
        // (a bad column as 0, so that the pairs always have an order)
        pair[s0 + at] = static_cast<uint64_t>(static_cast<uint32_t>(bad ? 0 : c)) << 32 | static_cast<uint32_t>(k);
        if (at == 0) {  // one block of each row; of a group's first row that has any, the group's items
            r0 = r / group_rows * group_rows;
            nr = min(group_rows, n_rows - r0);
            const int g0 = start[r0];
            if (s0 == g0 && start[r0 + nr] - g0 + 3 * nr > kPool)
                group_items(r0, nr, start, [&](int, int) { ++items; });
        }
    }
    if (__ballot(items > 0)) {
        int end = items;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int y = __shfl_up(end, o);
            if (lane >= o) end += y;
        }
        int q = 0;
        if (lane == kWave - 1) q = atomicAdd(flag + 2, end);
        q = __shfl(q, kWave - 1) + end - items;
        if (items)
            group_items(r0, nr, start, [&](int i, int piece) {
                item[2 * q] = r0 + i;
                item[2 * q + 1] = piece;
                ++q;
                if (piece == 0) distinct[r0 + i] = 0;
            });
    }
}

// Places the pairs of one piece of a row beyond the pool in the sorted row.
// The row passes through LDS kPiece pairs at a time, sorted there in tiles of
// one pair per thread (by rank, as below); a pair's place is the sum of its
// places in all tiles, found by binary search, and it is the first of its
// column if its predecessor in no tile has that column.  Bound by the LDS
// reads of the ranks and searches: 27 us for each kChunk pairs of the row.  With
// pieces of 2,048 a row of 3,000 takes 68 us instead of 55, rows of 1,200 in
// their thousands 198 us instead of 302; sorted by one workgroup each (bitonic)
// and summed by it, they took 100 us apiece, one after another.
constexpr int kPieceTiles = kPiece / kAsmThreads;

__device__ __forceinline__ void sort_piece(double* sh, int row, int s0, int len, int first,
                                           const uint64_t* __restrict__ pair, int* __restrict__ order,
                                           int* __restrict__ sorted_col, int* __restrict__ distinct) {
    const int t = threadIdx.x;
    // (past the end: not less than any pair)
    auto at = [&](int e) { return __longlong_as_double(e < len ? static_cast<long long>(pair[s0 + e]) : ~0ll); };
    const int own = min(kPiece, len - first);
    double a[kPieceTiles];
    int place[kPieceTiles];
    unsigned heads = 0;
#pragma unroll
    for (int q = 0; q < kPieceTiles; ++q) {
        a[q] = at(first + t + q * kAsmThreads);
        place[q] = 0;
        if (t + q * kAsmThreads < own) heads |= 1u << q;
    }
    for (int c0 = 0; c0 < len; c0 += kChunk) {
        const int n = min(kChunk, len - c0);
        __syncthreads();
        for (int e = t; e < ((n + kAsmThreads - 1) & -kAsmThreads); e += kAsmThreads) sh[e] = at(c0 + e);
        __syncthreads();
#pragma unroll 1
        for (int p = 0; p < n; p += kAsmThreads) {
            double* tile = sh + p;
            const double x = tile[t];
            const int m = min(kAsmThreads, n - p);
            int rank = 0;
#pragma unroll 4
            for (int j = 0; j < m; j += 4) {
                const double2 b = *reinterpret_cast<const double2*>(tile + j);
                const double2 d = *reinterpret_cast<const double2*>(tile + j + 2);
                rank += (b.x < x) + (b.y < x) + (d.x < x) + (d.y < x);
            }
            __syncthreads();
            if (t < m) tile[rank] = x;
        }
        __syncthreads();
        // the places of K of the thread's pairs, their searches side by side
        auto search = [&](auto K) {
#pragma unroll 1
            for (int p = 0; p < n; p += kAsmThreads) {
                const double* tile = sh + p;
                int k[K.value] = {};  // pairs of the tile below each: the pads are not
#pragma unroll
                for (int step = kAsmThreads / 2; step > 0; step /= 2)
#pragma unroll
                    for (int q = 0; q < K.value; ++q)
                        if (tile[k[q] + step - 1] < a[q]) k[q] += step;
#pragma unroll
                for (int q = 0; q < K.value; ++q) {
                    if (tile[k[q]] < a[q]) ++k[q];
                    if (k[q] > 0 && __double2hiint(tile[k[q] - 1]) == __double2hiint(a[q])) heads &= ~(1u << q);
                    place[q] += k[q];
                }
            }
        };
        if (own <= 2 * kAsmThreads)
            search(std::integral_constant<int, 2>{});
        else
            search(std::integral_constant<int, kPieceTiles>{});
    }
#pragma unroll
    for (int q = 0; q < kPieceTiles; ++q)
        if (t + q * kAsmThreads < own) {
            order[s0 + place[q]] = __double2loint(a[q]);
            sorted_col[s0 + place[q]] = __double2hiint(a[q]);
        }
    int n = __popc(heads);
#pragma unroll
    for (int o = kWave / 2; o > 0; o /= 2) n += __shfl_xor(n, o);
    if (t % kWave == 0 && n) atomicAdd(distinct + row, n);
}

// Sorts the rows.  A pair's place is the number of smaller pairs of its row,
// counted against the whole row read from LDS four pairs at a time, for two
// pairs per lane (the LDS reads bound the loop): no exchange steps and no
// waits between them, and rows of any mix of lengths share the lanes.  The
// pairs are compared as doubles (rows_path), not as 64-bit integers.  The
// items follow.  9.0 million blocks: 140 us (214 with a pair per lane, 448 with
// a wave per row).
__global__ void __launch_bounds__(kAsmThreads) k_asm_row_sort(int n_rows, int group_rows,
                                                              const int* __restrict__ start,
                                                              const uint64_t* __restrict__ pair,
                                                              const int* __restrict__ item,
                                                              int* __restrict__ order, int* __restrict__ seg_first,
                                                              int* __restrict__ seg_col, int* __restrict__ distinct,
                                                              const int* __restrict__ flag) {
    __shared__ __align__(16) uint64_t sh[kChunk];
    __shared__ PoolRows P;
    __shared__ int heads_of[kPoolRows], wave_heads[2][kAsmWaves];
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    if (blockIdx.x == 0 && threadIdx.x == 0) distinct[n_rows] = 0;
    if (uniform_load(flag) & 2) return;
    const int items = uniform_load(flag + 2), groups = gridDim.x;
    // the group's first batch, then items
    for (int i = static_cast<int>(blockIdx.x) - groups; i < items; i += groups) {
        int r0 = blockIdx.x * group_rows, nr = min(group_rows, n_rows - r0);
        if (i >= 0) {
            r0 = uniform_load(item + 2 * i);
            nr = -uniform_load(item + 2 * i + 1);
        }
        const int s0 = uniform_load(start + r0);
        if (i >= 0) __syncthreads();
        if (nr <= 0) {
            sort_piece(reinterpret_cast<double*>(sh), r0, s0, uniform_load(start + r0 + 1) - s0, -nr * kPiece, pair,
                       order, seg_col, distinct);
            continue;
        }
        pool_rows(P, r0, nr, start);
        const int rows = batch_end(P, nr), total = P.st[rows], places = P.base[rows];
        if (places <= kPool) {
            double* pool = reinterpret_cast<double*>(sh);
            int* col = reinterpret_cast<int*>(pool + kPool);
            int row[2];
            double a[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int e = threadIdx.x + q * kAsmThreads;
                if (e < kPool) sh[e] = ~0ull;  // not less than any pair
                row[q] = pool_row(P.st, rows, max(min(e, total - 1), 0));
                if (e < total) a[q] = __longlong_as_double(static_cast<long long>(pair[s0 + e]));
            }
            if (threadIdx.x < kPoolRows) heads_of[threadIdx.x] = 0;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int e = threadIdx.x + q * kAsmThreads;
                if (e < total) pool[P.base[row[q]] + e - P.st[row[q]]] = a[q];
            }
            __syncthreads();
            const int p = 2 * threadIdx.x;  // two neighbours of the pool, of one row
            if (p < places) {
                const int w = pool_row(P.base, rows, p), a0 = P.base[w], a1 = P.base[w + 1];
                const double2 a = *reinterpret_cast<const double2*>(pool + p);
                int rank[2] = {0, 0};
                for (int j = a0; j < a1; j += 4) {
                    const double2 b = *reinterpret_cast<const double2*>(pool + j);
                    const double2 d = *reinterpret_cast<const double2*>(pool + j + 2);
                    rank[0] += (b.x < a.x) + (b.y < a.x) + (d.x < a.x) + (d.y < a.x);
                    rank[1] += (b.x < a.y) + (b.y < a.y) + (d.x < a.y) + (d.y < a.y);
                }
                const int s1 = P.st[w], len = P.st[w + 1] - P.st[w];
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
                head[q] = e < total && (e == P.st[row[q]] || col[e - 1] != c[q]);
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
            if (static_cast<int>(threadIdx.x) < rows)
                distinct[r0 + threadIdx.x] = heads_of[threadIdx.x];
        }
    }
}

// Sums the columns that begin among kSumTile sorted blocks of a row beyond
// the pool: their values through LDS, kPool blocks at a time (the last column
// may go on past the tile).  The columns before them are counted from the
// sorted column indices.
__device__ __forceinline__ void sum_tile(double* x, int* pos, int* first, int* wave_heads, int s0, int len, int from,
                                         int o0, const int* __restrict__ order, const int* __restrict__ sorted_col,
                                         const double* __restrict__ blocks, int* __restrict__ col_idx,
                                         double* __restrict__ val) {
    const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
    const int* col = sorted_col + s0;
    const int to = min(from + kSumTile, len);
    int before = 0;  // columns that begin below the thread's block of the tile, of its wave's
    for (int e = t; e < from; e += kAsmThreads) before += e == 0 || col[e] != col[e - 1];
    const int c_last = col[to - 1];
    int end = to;  // of the last column, the same in every wave
    while (end < len) {
        const unsigned long long same = __ballot(end + lane < len && col[end + lane] == c_last);
        end += ~same ? __ffsll(~same) - 1 : kWave;
        if (~same) break;
    }
    const int e = from + t;
    const bool head = e < to && (e == 0 || col[e] != col[e - 1]);
    const unsigned long long heads = __ballot(head);
#pragma unroll
    for (int o = kWave / 2; o > 0; o /= 2) before += __shfl_xor(before, o);
    __syncthreads();
    if (lane == 0) {
        wave_heads[wave] = before;
        wave_heads[kAsmWaves + wave] = __popcll(heads);
    }
    __syncthreads();
    int o = o0, n = 0, j0 = 0;
    for (int w = 0; w < kAsmWaves; ++w) {
        o += wave_heads[w];
        if (w == wave) j0 = n;
        n += wave_heads[kAsmWaves + w];
    }
    if (n == 0) return;  // within a column
    if (head) {
        const int j = j0 + __popcll(heads & ((1ull << lane) - 1ull));
        first[j] = e;
        col_idx[o + j] = col[e];
    }
    if (t == 0) first[n] = end;
    __syncthreads();
    const int c = t % 9;
    double last = 0.0;  // of the last column, threads 0 to 8
    for (int b0 = first[0], b1; b0 < end; b0 = b1) {
        b1 = min(b0 + kPool, end);
        for (int i = t; i < b1 - b0; i += kAsmThreads) pos[i] = order[s0 + b0 + i];
        __syncthreads();
        const int values = 9 * (b1 - b0);
        constexpr int kLoads = 9;  // in flight together
#pragma unroll 1
        for (int i0 = 0; i0 < values; i0 += kLoads * kAsmThreads) {
            double v[kLoads];
#pragma unroll
            for (int q = 0; q < kLoads; ++q) {
                const int i = min(i0 + t + q * kAsmThreads, values - 1);
                v[q] = blocks[9LL * pos[i / 9] + i % 9];
            }
#pragma unroll
            for (int q = 0; q < kLoads; ++q) {
                const int i = i0 + t + q * kAsmThreads;
                if (i < values) x[i] = v[q];
            }
        }
        __syncthreads();
        auto add = [&](double s, int e0, int e1) {
#pragma unroll 4
            for (int i = e0; i < e1; ++i) s += x[9 * (i - b0) + c];
            return s;
        };
        if (b0 == first[0] && t < kAsmThreads / 9 * 9)  // the pool holds the others whole
            for (int j = t / 9; j < n - 1; j += kAsmThreads / 9)
                val[9LL * (o + j) + c] = add(0.0, first[j], first[j + 1]);
        if (t < 9) last = add(last, max(b0, first[n - 1]), b1);
        __syncthreads();
    }
    if (t < 9) val[9LL * (o + n - 1) + c] = last;
}
static_assert(kSumTile <= kAsmThreads && kSumTile <= kPool, "a thread per block, and all but the last column at once");

// Sums the rows, in list order within a distinct column.  The values of a
// workgroup's rows are loaded flat, in slot order -- an element's run of
// blocks is one piece of memory -- all in flight at once, turned in LDS and
// added from there, nine lanes to a column; the items follow, pieces tile by
// tile.  Does nothing where an index was
// out of range, a row too long, or the result larger than capacity.
//
// Bound by the reading of the values, 9.0 million x 72 bytes: 270 us with
// nine threads per column reading straight from memory, now 254 to 265 us (2.5
// TB/s).  Smaller pools of two rows (224, 256, 320 blocks) take 3 to 11 %
// longer over the whole call, and so do three rows in this one.
__global__ void __launch_bounds__(kAsmThreads, 4) k_asm_row_sum(int n_rows, int group_rows,
                                                             long long capacity,
                                                             const int* __restrict__ start,
                                                             const uint64_t* __restrict__ pair,
                                                             const int* __restrict__ item,
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
    const int items = uniform_load(static_cast<const int*>(flag) + 2), groups = gridDim.x;
    constexpr int kTiles = kPiece / kSumTile;  // of a piece; a batch is the first
    for (int i = static_cast<int>(blockIdx.x) - groups; i < kTiles * items; i += groups) {
        int r0 = blockIdx.x * group_rows, nr = min(group_rows, n_rows - r0);
        if (i >= 0) {
            r0 = uniform_load(item + 2 * (i / kTiles));
            nr = -uniform_load(item + 2 * (i / kTiles) + 1);
            if (nr > 0 && i % kTiles) continue;
        }
        const int s0 = uniform_load(start + r0), o0 = uniform_load(row_ptr + r0);
        if (nr <= 0) {
            const int len = uniform_load(start + r0 + 1) - s0, from = -nr * kPiece + i % kTiles * kSumTile;
            if (from < len) sum_tile(x, pos, first, ord, s0, len, from, o0, order, seg_col, blocks, col_idx, val);
            continue;
        }
        if (i >= 0) __syncthreads();
        pool_rows(P, r0, nr, start);
        const int rows = batch_end(P, nr), total = __builtin_amdgcn_readfirstlane(P.st[rows]);
        const int n = row_ptr[r0 + rows] - o0;
        if (P.base[rows] <= kPool) {
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
        }
    }
}

// Lists from 2 million blocks are sampled first (4 to 7 us): the pairs of equal
// rows among kSamples blocks of the list are kSamples^2 / (2 n) times the mean
// length of a block's row.  Beyond kSampleLength the rows' pieces and the
// atomics, which meet on few addresses, take longer than the sort (9 million
// blocks, 5 in 8 on rows of 7,000: 1,330 us by sorting), and rows beyond
// kRowLimit are likely.  The longer the list, the less the sort's fixed costs
// count: kSampleProduct divided by its blocks is the limit then (contacts of
// bodies, by sorting and here: 7 million of a mean of 1,650 947 and 924 us, 10
// million 1,145 and 1,239, 18 million 1,683 and 2,126; 10 million of 834 1,013
// and 992, 20 million 1,818 and 1,933, of 1,106 1,820 and 2,168).  In mixed order
// (neighbours in the list differ) every block takes an atomic and its values
// are read alone: from kMixedLength on sorting is faster (9 million blocks,
// rows of 128: 1,366 and 1,428 us; of 200: 1,275 and 1,490; of 400: 1,273 and
// 1,570).  The launches below then return at once, 90 us in all for such a list,
// 135 for 20 million blocks, so from 16 million the host reads the answer
// first (20 us).
constexpr int kSamples = 1024, kSampleSlots = 2 * kSamples, kSampleThreads = kSamples;
constexpr long long kSampleFrom = 1 << 21, kSampleRead = 1 << 24;
constexpr int kSampleLength = 3000, kMixedLength = 180;
constexpr double kSampleProduct = 1.2e10;

__global__ void __launch_bounds__(kSampleThreads) k_asm_sample(int n_in, const int* __restrict__ rows,
                                                               int* __restrict__ flag) {
    __shared__ int key[kSampleSlots], cnt[kSampleSlots];
    __shared__ int total, ends;
    for (int i = threadIdx.x; i < kSampleSlots; i += kSampleThreads) key[i] = -1, cnt[i] = 0;
    if (threadIdx.x == 0) total = ends = 0;
    __syncthreads();
    const int step = n_in / kSamples;
    for (int i = threadIdx.x; i < kSamples; i += kSampleThreads) {
        const unsigned mix = static_cast<unsigned>(i) * 2654435761u;
        const int* p = rows + static_cast<long long>(i) * step + (mix >> 8) % (step - 1);
        const int r = p[0];
        const unsigned long long differ = __ballot(r != p[1]);
        if (threadIdx.x % kWave == 0) atomicAdd(&ends, __popcll(differ));
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
    // (8 of 8 neighbours differ in mixed order; where elements list runs of four, 2 of 8)
    const double limit = 8 * ends > 7 * kSamples ? kMixedLength : kSampleLength;
    const double longest = fmin(limit, kSampleProduct / n_in);
    if (threadIdx.x == 0 && 2.0 * n_in * total > longest * kSamples * kSamples)
        flag[0] = 2;  // the sorting path takes the list: nothing below runs
}

// Few blocks per row leave the workgroups little to sort and sum, and the
// longer the list the less its fixed costs count for the sort: by sorting and
// here, in mixed order / in runs of two, 1.5 blocks a row in 0.3 million 234 and
// 152 / 213 and 133 us, in 1.5 million 372 and 420 / 374 and 340; 2 a row in 1.5
// million 367 and 374 / 363 and 285, in 3 million 618 and 739 / 579 and 544; 3 a
// row in 3 million 574 and 630 / 526 and 423, in 9 million 1,464 and 1,751 /
// 1,305 and 1,136; 4 in 9 million 1,467 and 1,612 / 1,282 and 952.  Rows of more
// than the pool on average are mostly pieces (500 a row, 0.3 million blocks in
// runs of four: 209 and 157 us, in 1.5 million 268 and 323; 400 a row 266 and
// 211).  The items take the tail of the counts: there is at most one, two ints,
// per 180 blocks, and the list exceeds the rows by a sixteenth.
// The pairs are compared as the doubles of the same bits, which order alike
// while a column's stay below those of infinity.
bool rows_path(int n_rows, long long n_in) {
    const int least = n_in < (1 << 20) ? 1 : n_in < (1 << 21) ? 2 : n_in < (1 << 22) ? 3 : 4;
    return n_in - n_rows > n_rows / 16 && n_in >= static_cast<long long>(least) * n_rows && n_in <= 400LL * n_rows &&
           n_rows < 0x7ff00000;
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
    L.flag = reinterpret_cast<int*>(take(sizeof(int) * 3));
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
    const RowArrays A = row_arrays(L, n_rows, n_in);
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
    launch_kernel(k_asm_count, dim3(ceil_div(n_in, kAsmThreads)), dim3(kAsmThreads), 0, s, n, n_rows, rows, A.cnt, A.slot, L.flag);
    if ((e = hipGetLastError()) != hipSuccess || (e = scan(A.cnt, A.start)) != hipSuccess) return e;
    const int group_rows = static_cast<int>(std::clamp<long long>(kPoolAim * static_cast<long long>(n_rows) / n_in, 1,
                                                                  kPoolRows));
    const dim3 grid(ceil_div(n_rows, group_rows));
    launch_kernel(k_asm_scatter, dim3(ceil_div(n_in, kAsmThreads)), dim3(kAsmThreads), 0, s, n, n_rows, rows, cols,
                  static_cast<const int*>(A.start), static_cast<const int*>(A.slot), group_rows, A.pair, A.distinct, A.item,
                  L.flag);
    launch_kernel(k_asm_row_sort, grid, dim3(kAsmThreads), 0, s, n_rows, group_rows,
                  static_cast<const int*>(A.start),
                  static_cast<const uint64_t*>(A.pair), static_cast<const int*>(A.item), A.order, A.seg_first,
                  A.seg_col, A.distinct, static_cast<const int*>(L.flag));
    if ((e = hipGetLastError()) != hipSuccess || (e = scan(A.distinct, row_ptr)) != hipSuccess) return e;
    launch_kernel(k_asm_row_sum, grid, dim3(kAsmThreads), 0, s, n_rows, group_rows, capacity,
                  static_cast<const int*>(A.start),
                  static_cast<const uint64_t*>(A.pair), static_cast<const int*>(A.item),
                  static_cast<const int*>(A.order), static_cast<const int*>(A.seg_first), static_cast<const int*>(A.seg_col), L.flag,
                  static_cast<const int*>(row_ptr), blocks, col_idx, val);
    *taken = true;
    return hipGetLastError();
}

}  // namespace maspcg

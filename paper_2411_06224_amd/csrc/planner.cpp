// Host-side symbolic analysis (see planner.hpp).
//
// Ordering (Sec. 4.2): the node graph is partitioned into
// M = ceil(V / (N - N_o)) parts of at most N nodes, the slack N_o searched
// upward from 0 (Eq. num_subdomains).  The paper uses METIS; here the
// partitioner is a recursive BFS bisection with fully specified tie-breaks
// so that an independent implementation reproduces it bit for bit:
//   split(S, k): k == 1 -> S is the next part; otherwise kL = k/2,
//   nL = floor(|S| kL / k) and S is cut after its first nL nodes in
//   pseudo-peripheral BFS order (start at the smallest id, twice jump to the
//   smallest id on the deepest BFS level, then the BFS visit order with
//   ascending neighbours, restarting at the smallest unvisited id).
// Part p occupies slots [pN, pN + N) in ascending node order; the rest of
// its slots are padding (-1), one part per MAS domain (Fig. mapping).
//
// Hierarchy (Sec. 4.1, Supp. Alg. 2-5): at each level the units of a domain
// that are coupled by stored blocks form connected components; each
// component is a supernode of the next level, numbered inside its domain by
// its lowest lane and globally by domain order.  N consecutive supernodes
// form a domain of the next level.  Construction stops at a single domain,
// at max_levels, or when no component merges two units.
#include "planner.hpp"

#include <algorithm>
#include <array>
#include <cstring>
#include <numeric>
#include <thread>

namespace maspcg {
namespace {

struct Graph {
    std::vector<int> off, nbr;
};

// f(first, end, t) on ranges t of n independent items, one per thread: as many
// as the blocks that the items hold are worth starting (62 thousand blocks, the
// plan of a given partition: 2.3 ms with one thread, 1.7 with four, 2.0 with
// eight).
int range_threads(int n, long long blocks) {
    const int hw = static_cast<int>(std::thread::hardware_concurrency());
    return std::max(1, std::min({hw, n, blocks >= (1 << 16) ? 8 : blocks >= (1 << 15) ? 4 : 1}));
}

template <typename F>
void on_ranges(int n, int threads, F&& f) {
    auto begin = [&](int t) { return static_cast<int>(static_cast<long long>(n) * t / threads); };
    std::vector<std::thread> th;
    for (int t = 1; t < threads; ++t) th.emplace_back([&, t] { f(begin(t), begin(t + 1), t); });
    f(0, begin(1), 0);
    for (auto& x : th) x.join();
}

// Both directions of every edge (self loops and out-of-range ends
// dropped), each node's neighbours ascending and distinct: the edge list
// bucketed by node, then each bucket sorted.
Graph symmetrize(int V, const int32_t* ptr, const int32_t* adj) {
    std::vector<int> start(V + 1, 0);
    for (int i = 0; i < V; ++i)
        for (int p = ptr[i]; p < ptr[i + 1]; ++p) {
            const int j = adj[p];
            if (j < 0 || j >= V || j == i) continue;
            start[i + 1]++;
            start[j + 1]++;
        }
    for (int i = 0; i < V; ++i) start[i + 1] += start[i];
    std::vector<int> fill(start.begin(), start.end() - 1), nb(start[V]);
    for (int i = 0; i < V; ++i)
        for (int p = ptr[i]; p < ptr[i + 1]; ++p) {
            const int j = adj[p];
            if (j < 0 || j >= V || j == i) continue;
            nb[fill[i]++] = j;
            nb[fill[j]++] = i;
        }
    Graph g;
    g.off.assign(V + 1, 0);
    g.nbr.reserve(nb.size());
    for (int i = 0; i < V; ++i) {
        std::sort(nb.begin() + start[i], nb.begin() + start[i + 1]);
        for (int q = start[i]; q < start[i + 1]; ++q)
            if (q == start[i] || nb[q] != nb[q - 1]) g.nbr.push_back(nb[q]);
        g.off[i + 1] = static_cast<int>(g.nbr.size());
    }
    return g;
}

// A set of the recursion: nodes[lo, hi) (in the parent's BFS order), to be
// cut into k parts numbered from p0.
struct BisectTask {
    int lo, hi, k, p0;
};

// One worker of the recursive bisection.  nodes[] and asc[] are shared by
// all workers, each task owning its range: asc[lo, hi) holds the task's set
// ascending (split from the parent's ascending list, not sorted again).
// Each worker has its own membership tags, so workers on disjoint tasks do
// not interact, and a task's split depends on its set alone: the parts do
// not depend on how the tasks are spread over workers.
class Bisection {
  public:
    Bisection(const Graph& g, int* nodes, int* asc)
        : g_(g), nodes_(nodes), asc_(asc), in_(g.off.size() - 1, -1), seen_(g.off.size() - 1, -1),
          depth_(g.off.size() - 1, 0), tmp_(g.off.size() - 1) {}

    // Splits t (k >= 2) into its left and right tasks.
    void split(const BisectTask& t, BisectTask& left, BisectTask& right) {
        const int kl = t.k / 2;
        const int n = t.hi - t.lo;
        const int nl = static_cast<int>(static_cast<long long>(n) * kl / t.k);
        if (n > 0) {
            reorder(nodes_ + t.lo, asc_ + t.lo, n);
            split_ascending(nodes_ + t.lo, asc_ + t.lo, n, nl);
        }
        left = {t.lo, t.lo + nl, kl, t.p0};
        right = {t.lo + nl, t.hi, t.k - kl, t.p0 + kl};
    }

    // The whole subtree of t: part[node] for its nodes.
    void finish(const BisectTask& root, int* part) {
        std::vector<BisectTask> stack{root};
        while (!stack.empty()) {
            const BisectTask t = stack.back();
            stack.pop_back();
            if (t.k == 1) {
                for (int q = t.lo; q < t.hi; ++q) part[nodes_[q]] = t.p0;
                continue;
            }
            BisectTask left, right;
            split(t, left, right);
            stack.push_back(right);
            stack.push_back(left);
        }
    }

  private:
    // BFS inside the current set from root; appends visit order to out and
    // records depths.  Returns the deepest level reached.
    int bfs(int root, std::vector<int>& out) {
        size_t head = out.size();
        out.push_back(root);
        seen_[root] = mark_;
        depth_[root] = 0;
        int deepest = 0;
        while (head < out.size()) {
            const int u = out[head++];
            for (int p = g_.off[u]; p < g_.off[u + 1]; ++p) {
                const int v = g_.nbr[p];
                if (in_[v] != set_ || seen_[v] == mark_) continue;
                seen_[v] = mark_;
                depth_[v] = depth_[u] + 1;
                deepest = std::max(deepest, depth_[v]);
                out.push_back(v);
            }
        }
        return deepest;
    }

    // asc: the set ascending.
    void reorder(int* S, const int* asc, int n) {
        set_ = ++tag_;
        for (int q = 0; q < n; ++q) in_[S[q]] = set_;
        int root = asc[0];
        std::vector<int> visit;
        visit.reserve(n);
        for (int rep = 0; rep < 2; ++rep) {
            mark_ = ++tag_;
            visit.clear();
            const int deepest = bfs(root, visit);
            int best = -1;
            for (int v : visit)
                if (depth_[v] == deepest && (best < 0 || v < best)) best = v;
            root = best;
        }
        mark_ = ++tag_;
        visit.clear();
        bfs(root, visit);
        size_t scan = 0;
        while (static_cast<int>(visit.size()) < n) {
            while (seen_[asc[scan]] == mark_) ++scan;
            bfs(asc[scan], visit);
        }
        std::copy(visit.begin(), visit.end(), S);
    }

    // asc (the set ascending) reordered into the ascending lists of the
    // first nl nodes of S and of the rest.
    void split_ascending(const int* S, int* asc, int n, int nl) {
        const int left = ++tag_;
        for (int q = 0; q < nl; ++q) in_[S[q]] = left;
        int a = 0, b = nl;
        for (int q = 0; q < n; ++q) {
            const int v = asc[q];
            tmp_[in_[v] == left ? a++ : b++] = v;
        }
        std::copy(tmp_.begin(), tmp_.begin() + n, asc);
    }

    const Graph& g_;
    int *nodes_, *asc_;
    std::vector<int> in_, seen_, depth_, tmp_;
    int tag_ = 0, set_ = -1, mark_ = -1;
};

// Recursive bisection of all V nodes into k parts (see the file comment):
// the top of the recursion is split level by level, the tasks of a level
// on threads of their own, until there are enough subtrees for the
// threads; each subtree is then finished on a thread.
void bisect(const Graph& g, int k, std::vector<int>& part) {
    const int V = static_cast<int>(g.off.size()) - 1;
    std::vector<int> nodes(V), asc(V);
    std::iota(nodes.begin(), nodes.end(), 0);
    std::iota(asc.begin(), asc.end(), 0);
    const int hw = static_cast<int>(std::thread::hardware_concurrency());
    const int T = std::max(1, std::min(hw, 8));
    auto run_all = [&](int n_tasks, const auto& work) {
        if (n_tasks == 1 || T == 1) {
            for (int i = 0; i < n_tasks; ++i) work(i);
            return;
        }
        std::vector<std::thread> th;
        th.reserve(n_tasks);
        for (int i = 0; i < n_tasks; ++i) th.emplace_back(work, i);
        for (auto& x : th) x.join();
    };
    std::vector<BisectTask> level{{0, V, k, 0}};
    while (static_cast<int>(level.size()) < T) {
        std::vector<BisectTask> next(2 * level.size());
        bool any = false;
        for (const BisectTask& t : level) any |= t.k > 1;
        if (!any) break;
        run_all(static_cast<int>(level.size()), [&](int i) {
            const BisectTask& t = level[i];
            if (t.k <= 1) {  // a finished part (k = 1) or a placeholder (k = 0) moves down as it is
                next[2 * i] = t;
                next[2 * i + 1] = {t.hi, t.hi, 0, t.p0};  // placeholder: nothing to do
                return;
            }
            Bisection b(g, nodes.data(), asc.data());
            b.split(t, next[2 * i], next[2 * i + 1]);
        });
        level.swap(next);
    }
    run_all(static_cast<int>(level.size()), [&](int i) {
        if (level[i].k < 1) return;
        Bisection b(g, nodes.data(), asc.data());
        b.finish(level[i], part.data());
    });
}

// Components of the units of each domain under the block pattern (rp, ci)
// over units.  Returns the next-level id of every unit (-1 if empty) and the
// number of components.
int components(int units, int N, const std::vector<int>& rp, const std::vector<int>& ci,
               const std::vector<char>& occupied, std::vector<int>& comp) {
    comp.assign(units, -1);
    int next = 0;
    std::vector<int> stack;
    for (int d = 0; d * N < units; ++d) {
        const int lo = d * N, hi = std::min(units, lo + N);
        for (int u = lo; u < hi; ++u) {
            if (!occupied[u] || comp[u] >= 0) continue;
            const int id = next++;
            comp[u] = id;
            stack.assign(1, u);
            while (!stack.empty()) {
                const int s = stack.back();
                stack.pop_back();
                for (int p = rp[s]; p < rp[s + 1]; ++p) {
                    const int t = ci[p];
                    if (t < lo || t >= hi || comp[t] >= 0) continue;
                    comp[t] = id;
                    stack.push_back(t);
                }
            }
        }
    }
    return next;
}

// Galerkin pattern and reduction plan: block (s, t) of the fine matrix goes
// to block (up[s], up[t]) of the coarse one.  The fine blocks are ordered
// by (up[s], up[t]), equal pairs in block order: a stable counting sort by
// up[t], then one by up[s].
void coarsen(const std::vector<int>& rp, const std::vector<int>& ci, const std::vector<int>& up, int coarse_units,
             std::vector<int>& rpC, std::vector<int>& ciC, std::vector<int>& red_ptr, std::vector<int>& red_src) {
    const int fine_units = static_cast<int>(rp.size()) - 1;
    const int nnz = rp.back();
    std::vector<long long> key(nnz);
    std::vector<int> row(nnz);
    for (int s = 0; s < fine_units; ++s)
        for (int p = rp[s]; p < rp[s + 1]; ++p) {
            key[p] = static_cast<long long>(up[s]) * coarse_units + up[ci[p]];
            row[p] = up[s];
        }
    std::vector<int> by_col(nnz), cnt(coarse_units + 1);
    for (int p = 0; p < nnz; ++p) cnt[up[ci[p]] + 1]++;
    for (int c = 0; c < coarse_units; ++c) cnt[c + 1] += cnt[c];
    for (int p = 0; p < nnz; ++p) by_col[cnt[up[ci[p]]]++] = p;
    std::fill(cnt.begin(), cnt.end(), 0);
    for (int p = 0; p < nnz; ++p) cnt[row[p] + 1]++;
    for (int c = 0; c < coarse_units; ++c) cnt[c + 1] += cnt[c];
    red_src.resize(nnz);
    for (int q = 0; q < nnz; ++q) red_src[cnt[row[by_col[q]]]++] = by_col[q];
    rpC.assign(coarse_units + 1, 0);
    ciC.clear();
    red_ptr.assign(1, 0);
    for (int q = 0; q < nnz; ++q) {
        const long long k = key[red_src[q]];
        if (q == 0 || k != key[red_src[q - 1]]) {
            if (q) red_ptr.push_back(q);
            ciC.push_back(static_cast<int>(k % coarse_units));
            rpC[k / coarse_units + 1]++;
        }
    }
    red_ptr.push_back(nnz);
    for (int s = 0; s < coarse_units; ++s) rpC[s + 1] += rpC[s];
}

void domain_plan(const std::vector<int>& rp, const std::vector<int>& ci, int units, int N, std::vector<int>& ptr,
                 std::vector<int>& blk, std::vector<int>& ab) {
    const int nd = (units + N - 1) / N;
    ptr.assign(1, 0);
    blk.clear();
    ab.clear();
    for (int d = 0; d < nd; ++d) {
        const int lo = d * N, hi = std::min(units, lo + N);
        for (int s = lo; s < hi; ++s)
            for (int p = rp[s]; p < rp[s + 1]; ++p) {
                const int t = ci[p];
                if (t < s || t >= lo + N) continue;
                blk.push_back(p);
                ab.push_back((s - lo) | ((t - lo) << 8));
            }
        ptr.push_back(static_cast<int>(blk.size()));
    }
}

// Group-symmetric storage (see Plan::srp).  Storage windows, of whole groups,
// are independent.
void symmetric_storage(Plan& P) {
    const int NS = P.NS, RG = P.RG, W = storage_window(P.N), n_win = (NS + W - 1) / W;
    const int T = range_threads(n_win, P.nnzb);
    P.srp.assign(NS + 1, 0);
    P.tptr.assign(NS + 1, 0);
    std::vector<int> trans(n_win, 0);  // transposed entries of the window: blocks left of the diagonal in it
    on_ranges(n_win, T, [&](int w0, int w1, int) {
        for (int w = w0; w < w1; ++w)
            for (int s = w * W; s < std::min((w + 1) * W, NS); ++s) {
                const int r0 = s / RG * RG, r1 = std::min(r0 + RG, NS);
                int stored = 0;
                for (int k = P.rp0[s]; k < P.rp0[s + 1]; ++k) {
                    const int j = P.ci0[k];
                    trans[w] += j >= w * W && j < s;
                    if (j >= r0 && j < r1 && j != s) {
                        if (j < s) continue;
                        P.tptr[j + 1]++;
                    }
                    ++stored;
                }
                P.srp[s + 1] = stored;
            }
    });
    for (int s = 0; s < NS; ++s) {
        P.srp[s + 1] += P.srp[s];
        P.tptr[s + 1] += P.tptr[s];
    }
    P.sci.resize(P.srp[NS]);
    P.sperm.resize(P.srp[NS]);
    P.srow.resize(P.srp[NS]);
    P.tidx.resize(P.tptr[NS]);
    std::vector<int> fill(P.tptr.begin(), P.tptr.end() - 1);
    on_ranges(n_win, T, [&](int w0, int w1, int) {
        for (int s = w0 * W; s < std::min(w1 * W, NS); ++s) {
            const int r0 = s / RG * RG, r1 = std::min(r0 + RG, NS);
            int o = P.srp[s];
            for (int k = P.rp0[s]; k < P.rp0[s + 1]; ++k) {
                const int j = P.ci0[k];
                if (j >= r0 && j < r1 && j != s) {
                    if (j < s) continue;
                    P.tidx[fill[j]++] = o;  // ascending within row j
                }
                P.sci[o] = j;
                P.sperm[o] = P.perm_src[k];
                P.srow[o++] = static_cast<uint8_t>(s - r0);
            }
        }
    });
    P.maxT = 0;
    for (int g = 0; g < P.G; ++g) {
        const int r0 = g * RG, r1 = std::min(r0 + RG, NS);
        P.maxT = std::max(P.maxT, P.tptr[r1] - P.tptr[r0]);
    }
    P.sym = *std::max_element(trans.begin(), trans.end()) <= kMaxTransposed;
}

// The level-1 units each group's SpMV reads (see Plan::hptr).  Groups are
// independent.  full: the SpMV streams the full storage.
void halo_units(Plan& P, bool full) {
    const int NS = P.NS, RG = P.RG, G = P.G, L = P.L;
    P.halo = true;
    P.maxH = P.maxH2 = 0;
    P.hptr.assign(static_cast<size_t>(G) + 1, 0);
    P.h2ptr.assign(static_cast<size_t>(G) + 1, 0);
    P.hidx.assign(full ? P.ci0.size() : P.sci.size(), 0);
    if (L < 2) return;
    const std::vector<int>& rp = full ? P.rp0 : P.srp;
    const std::vector<int>& ci = full ? P.ci0 : P.sci;  // (both hold every block with a column outside the group)
    const int T = range_threads(G, P.nnzb);
    struct Part {
        std::vector<int> hu, h2slot;
        std::vector<uint16_t> hpar;
        int maxH = 0, maxH2 = 0;
        bool fits = true;
    };
    std::vector<Part> parts(T);
    std::vector<int> lead(P.units[1]);  // first slot of each level-1 unit
    for (int s = 0; s < NS; ++s)
        if (P.lead1[s] >= 0) lead[P.lead1[s]] = s;
    // units and level-2 entries of each group, and the blocks' local units
    on_ranges(G, T, [&](int g0, int g1, int t) {
        Part& R = parts[t];
        std::vector<std::pair<int, int>> ext;      // outside units, in the order found
        std::vector<std::pair<int, uint16_t>> at;  // blocks with a column outside, and the unit's place in that order
        std::vector<std::pair<int, int>> two;  // level-2 units, and a slot below each
        std::vector<uint16_t> local(kMaxHalo + 1);
        std::vector<int> seen(P.units[1], -1), seen2(L > 2 ? P.units[2] : 0, -1);
        std::vector<uint16_t> place(P.units[1]), place2(L > 2 ? P.units[2] : 0);
        for (int g = g0; g < g1; ++g) {
            const int r0 = g * RG, r1 = std::min(r0 + RG, NS);
            const int own = P.g_u1[g + 1] - P.g_u1[g];
            ext.clear();
            at.clear();
            for (int k = rp[r0]; k < rp[r1]; ++k) {
                const int j = ci[k];
                if (j >= r0 && j < r1) continue;
                const int u = P.anc[j];
                if (seen[u] != g) {
                    seen[u] = g;
                    place[u] = static_cast<uint16_t>(ext.size());
                    if (own + static_cast<int>(ext.size()) == kMaxHalo) {
                        R.fits = false;
                        return;
                    }
                    ext.emplace_back(u, static_cast<int>(ext.size()));
                }
                at.emplace_back(k, place[u]);
            }
            const int n = own + static_cast<int>(ext.size());
            if (n > kMaxHalo) {
                R.fits = false;
                return;
            }
            R.maxH = std::max(R.maxH, n);
            std::sort(ext.begin(), ext.end());
            const size_t h0 = R.hu.size();
            for (int i = 0; i < own; ++i) R.hu.push_back(P.g_u1[g] + i);
            for (size_t i = 0; i < ext.size(); ++i) {
                R.hu.push_back(ext[i].first);
                local[ext[i].second] = static_cast<uint16_t>(own + i);
            }
            for (const auto& [k, i] : at) P.hidx[k] = local[i];
            two.clear();
            if (L > 2)
                for (int i = 0; i < n; ++i) {
                    const int a = P.up[1][R.hu[h0 + i]];
                    if (seen2[a] != g) {
                        seen2[a] = g;
                        two.emplace_back(a, lead[R.hu[h0 + i]]);
                    }
                }
            std::sort(two.begin(), two.end());
            for (size_t i = 0; i < two.size(); ++i) {
                place2[two[i].first] = static_cast<uint16_t>(i);
                R.h2slot.push_back(two[i].second);
            }
            for (int i = 0; i < n; ++i) R.hpar.push_back(L > 2 ? place2[P.up[1][R.hu[h0 + i]]] : 0);
            R.maxH2 = std::max(R.maxH2, static_cast<int>(two.size()));
            P.hptr[g + 1] = n;
            P.h2ptr[g + 1] = static_cast<int>(two.size());
        }
    });
    for (Part& R : parts) {
        if (!R.fits) {
            P.halo = false;
            P.maxH = P.maxH2 = 0;
            for (auto* x : {&P.hptr, &P.hu, &P.h2ptr, &P.h2slot}) x->clear();
            for (auto* x : {&P.hpar, &P.hidx}) x->clear();
            return;
        }
        P.maxH = std::max(P.maxH, R.maxH);
        P.maxH2 = std::max(P.maxH2, R.maxH2);
        P.hu.insert(P.hu.end(), R.hu.begin(), R.hu.end());
        P.hpar.insert(P.hpar.end(), R.hpar.begin(), R.hpar.end());
        P.h2slot.insert(P.h2slot.end(), R.h2slot.begin(), R.h2slot.end());
    }
    for (int g = 0; g < G; ++g) {
        P.hptr[g + 1] += P.hptr[g];
        P.h2ptr[g + 1] += P.h2ptr[g];
    }
}

// Workgroup order of the SpMV.  The group kernels give each XCD a
// contiguous range of groups, dispatched in order.  Groups with far more
// stored blocks than the mean (rows coupled to many distant columns, such as
// the rows of bodies attached to a sheet) tend to sit together at one end of
// the numbering, so one XCD gets all of them and starts them last.  When a
// group holds more than 1.5x the mean, the heavy groups are dealt
// round-robin over the XCDs, heaviest first, at the head of each XCD's
// order, and each XCD is then filled with a contiguous run of the other
// groups (keeping neighbouring groups, which share halo entries, on one
// XCD).  Otherwise gorder stays empty.
void spmv_order(Plan& P) {
    const int G = P.G, NS = P.NS, RG = P.RG;
    const std::vector<int>& rp = P.sym ? P.srp : P.rp0;
    std::vector<long long> cnt(std::max(G, 0));
    for (int g = 0; g < G; ++g) {
        const int r0 = g * RG, r1 = std::min(r0 + RG, NS);
        cnt[g] = rp[r1] - rp[r0];
    }
    P.gorder = spmv_group_order(cnt);
}

}  // namespace

// A group is one workgroup of the SpMV: its chunks of blocks follow one
// another, so where the machine is not full of groups the iteration takes as
// long as one group's chain, and smaller groups, of 1, 2 or 4 domains instead of
// 8, shorten it.  Each workgroup has its prologue, its partial sums and its
// writers, though, and stores fewer pairs once; and past the number that runs at
// once (kGroupsPerCu per CU: four of 33 KB of LDS) a second round begins.
// Iteration in us with 1 / 2 / 4 / 8 domains per group, FP64 and mixed, on both
// sides of each limit (cubes, * plain grids):
//   308 domains   18.8 / 19.0 / 21.1 / 25.3,  17.4 / 17.3 / 18.3 / 21.3
//   400 *         18.4 / 18.0 / 18.1 / 20.8,  17.4 / 16.8 / 16.9 / 18.4
//   1,372         29.4 / 22.5 / 23.9 / 27.8,  25.5 / 20.0 / 20.3 / 23.0
//   1,600 *       29.9 / 21.3 / 20.1 / 22.0,  27.8 / 20.0 / 18.0 / 18.7
//   4,000         60.0 / 44.3 / 33.7 / 35.2,  54.1 / 38.6 / 28.4 / 28.7
//   4,308         63.6 / 46.1 / 43.0 / 37.2,  56.7 / 40.2 / 30.9 / 29.6
// Where one window of 128 rows holds more than three times the mean (rows of
// bodies with many contacts), its chain alone is the iteration: such groups
// are halved down to 1,024 blocks while that leaves no more than kHeavyGroups per
// CU (sheets with bodies in contact):
//   822 domains   23.5 / 24.7 / 30.4 / 44.2,  21.7 / 21.4 / 24.9 / 34.2
//   1,072         25.9 / 27.0 / 32.5 / 45.8,  24.3 / 23.5 / 26.3 / 34.6
//   5,835         82.3 / 58.6 / 59.4 / 72.0,  74.0 / 52.9 / 52.0 / 59.2
//   6,636         92.0 / 64.3 / 63.8 / 76.0,  82.6 / 59.1 / 56.0 / 63.2
//   12,984        209 / 141 / 118.6 / 120.4,  166 / 112 / 88.8 / 88.7
// Other domain sizes keep groups of about 128 rows.
int group_domains(int M, int N, long long nnzb, long long window_blocks) {
    constexpr int kCus = 256;
    constexpr double kGroupsPerCu[3] = {1.5, 3, 4}, kHeavyGroups[3] = {3.5, 12, 12};  // of 1, 2 and 4 domains
    const int most = std::max(1, kWindowSlots / N);
    if (N != 16) return most;
    auto fits = [&](int i, const double (&per_cu)[3]) { return M <= (1 << i) * kCus * per_cu[i]; };
    int i = 0;
    while (i < 3 && !fits(i, kGroupsPerCu)) ++i;
    const int windows = (M + most - 1) / most;
    if (window_blocks * windows > 3 * nnzb)
        while (i > 0 && (window_blocks << i) > 1024LL * most && fits(i - 1, kHeavyGroups)) --i;
    return 1 << i;
}

std::vector<int> spmv_group_order(const std::vector<long long>& cnt) {
    const int G = static_cast<int>(cnt.size());
    std::vector<int> gorder;
    if (G <= 0) return gorder;
    double mean = 0.0;
    for (int g = 0; g < G; ++g) mean += static_cast<double>(cnt[g]);
    mean /= G;
    std::vector<int> heavy, light;
    for (int g = 0; g < G; ++g) (static_cast<double>(cnt[g]) > 1.5 * mean ? heavy : light).push_back(g);
    if (heavy.empty()) return gorder;
    std::stable_sort(heavy.begin(), heavy.end(), [&](int a, int b) { return cnt[a] > cnt[b]; });
    const int q = G / kXcdCount, rem = G % kXcdCount;
    std::array<std::vector<int>, kXcdCount> lists;
    auto cap = [&](int x) { return static_cast<size_t>(q + (x < rem ? 1 : 0)); };
    int x = 0;
    for (const int g : heavy) {
        while (lists[x].size() == cap(x)) x = (x + 1) % kXcdCount;
        lists[x].push_back(g);
        x = (x + 1) % kXcdCount;
    }
    size_t li = 0;
    for (x = 0; x < kXcdCount; ++x)
        while (lists[x].size() < cap(x)) lists[x].push_back(light[li++]);
    // workgroup b = i kXcdCount + x runs the i-th group of XCD x's list
    gorder.assign(G, -1);
    for (x = 0; x < kXcdCount; ++x)
        for (size_t i = 0; i < lists[x].size(); ++i) gorder[i * kXcdCount + x] = lists[x][i];
    return gorder;
}

std::string analyze(int V, int nnzb, const int32_t* row_ptr, const int32_t* col_idx, const int32_t* g_ptr,
                    const int32_t* g_adj, int N, int max_levels, Plan& P, const int32_t* part, int n_parts,
                    bool f32_values) {
    if (V <= 0 || nnzb < V || !row_ptr || !col_idx) return "empty matrix or null pattern";
    if (N < 1 || N > 40) return "domain_size must be in [1, 40]";
    if ((g_ptr == nullptr) != (g_adj == nullptr)) return "graph needs both g_ptr and g_adj";
    if (row_ptr[0] != 0 || row_ptr[V] != nnzb) return "row_ptr must start at 0 and end at nnzb";
    for (int i = 0; i < V; ++i) {
        if (row_ptr[i + 1] < row_ptr[i]) return "row_ptr not monotone";
        bool diag = false;
        for (int p = row_ptr[i]; p < row_ptr[i + 1]; ++p) {
            const int j = col_idx[p];
            if (j < 0 || j >= V) return "column index out of range";
            if (p > row_ptr[i] && j <= col_idx[p - 1]) return "columns must be strictly ascending in a row";
            diag |= (j == i);
        }
        if (!diag) return "every row needs its diagonal block";
    }
    for (int i = 0; i < V; ++i)
        for (int p = row_ptr[i]; p < row_ptr[i + 1]; ++p) {
            const int j = col_idx[p];
            if (!std::binary_search(col_idx + row_ptr[j], col_idx + row_ptr[j + 1], i)) return "pattern is not symmetric";
        }
    if (g_ptr) {
        if (g_ptr[0] != 0) return "g_ptr must start at 0";
        for (int i = 0; i < V; ++i)
            if (g_ptr[i + 1] < g_ptr[i]) return "g_ptr not monotone";
    }

    P = Plan();
    P.V = V;
    P.N = N;
    P.nnzb = nnzb;

    // ---- partition with the slack search of Eq. num_subdomains, or the
    // caller's (every part 1..N nodes)
    if (part) {
        if (n_parts < 1 || n_parts > V) return "n_parts must be in [1, n_rows]";
        std::vector<int> size(n_parts, 0);
        for (int i = 0; i < V; ++i) {
            if (part[i] < 0 || part[i] >= n_parts) return "part id out of range";
            if (++size[part[i]] > N) return "a part holds more than domain_size nodes";
        }
        for (int q = 0; q < n_parts; ++q)
            if (size[q] == 0) return "empty part";
    }
    const Graph g = part ? Graph() : (g_ptr ? symmetrize(V, g_ptr, g_adj) : symmetrize(V, row_ptr, col_idx));
    P.part.assign(V, 0);
    bool found = false;
    if (part) {
        P.part.assign(part, part + V);
        P.M = n_parts;
        P.No = 0;
        found = true;
    }
    for (int No = 0; No < N && !found; ++No) {
        const int M = (V + (N - No) - 1) / (N - No);
        bisect(g, M, P.part);
        std::vector<int> size(M, 0);
        bool fits = true;
        for (int i = 0; i < V; ++i) fits &= (++size[P.part[i]] <= N);
        if (fits) {
            P.M = M;
            P.No = No;
            found = true;
        }
    }
    if (!found) return "partition failed";

    // ---- slots (one part per domain, ascending node ids, -1 padding)
    P.NS = P.M * N;
    P.map.assign(V, -1);
    P.remap.assign(P.NS, -1);
    {
        std::vector<int> fill(P.M, 0);
        for (int i = 0; i < V; ++i) {
            const int s = P.part[i] * N + fill[P.part[i]]++;
            P.map[i] = s;
            P.remap[s] = i;
        }
    }

    // ---- H in slot order
    P.rp0.assign(P.NS + 1, 0);
    P.ci0.resize(nnzb);
    P.perm_src.resize(nnzb);
    for (int s = 0; s < P.NS; ++s) {
        const int i = P.remap[s];
        P.rp0[s + 1] = P.rp0[s] + (i >= 0 ? row_ptr[i + 1] - row_ptr[i] : 0);
    }
    {
        auto rows = [&](int s0, int s1, int) {
            std::vector<std::pair<int, int>> row;
            for (int s = s0; s < s1; ++s) {
                const int i = P.remap[s];
                if (i < 0) continue;
                row.clear();
                for (int p = row_ptr[i]; p < row_ptr[i + 1]; ++p) row.emplace_back(P.map[col_idx[p]], p);
                std::sort(row.begin(), row.end());
                for (size_t q = 0; q < row.size(); ++q) {
                    P.ci0[P.rp0[s] + q] = row[q].first;
                    P.perm_src[P.rp0[s] + q] = row[q].second;
                }
            }
        };
        on_ranges(P.NS, range_threads(P.NS, nnzb), rows);
    }

    // ---- hierarchy
    P.units.push_back(P.NS);
    P.ndom.push_back(P.M);
    // room for every level up front: the loop holds references into rpA /
    // ciA while it appends the next level
    P.rpA.reserve(kMaxLevels);
    P.ciA.reserve(kMaxLevels);
    P.red_ptr.reserve(kMaxLevels);
    P.red_src.reserve(kMaxLevels);
    P.rpA.emplace_back();  // level 0 uses rp0 / ci0
    P.ciA.emplace_back();
    P.red_ptr.emplace_back();
    P.red_src.emplace_back();
    int occupied_count = V;
    for (int l = 0;; ++l) {
        if (P.ndom[l] == 1) break;
        if (max_levels > 0 && l + 1 >= max_levels) break;
        if (l + 1 >= kMaxLevels) break;
        const std::vector<int>& rp = l == 0 ? P.rp0 : P.rpA[l];
        const std::vector<int>& ci = l == 0 ? P.ci0 : P.ciA[l];
        std::vector<char> occ(P.units[l], 1);
        if (l == 0)
            for (int s = 0; s < P.NS; ++s) occ[s] = P.remap[s] >= 0;
        std::vector<int> comp;
        const int S = components(P.units[l], N, rp, ci, occ, comp);
        if (S == occupied_count) break;  // nothing merged
        P.up.push_back(comp);
        P.units.push_back(S);
        P.ndom.push_back((S + N - 1) / N);
        P.rpA.emplace_back();
        P.ciA.emplace_back();
        P.red_ptr.emplace_back();
        P.red_src.emplace_back();
        coarsen(rp, ci, comp, S, P.rpA[l + 1], P.ciA[l + 1], P.red_ptr[l + 1], P.red_src[l + 1]);
        occupied_count = S;
    }
    P.L = static_cast<int>(P.units.size());

    // ---- inversion plans
    P.dom_ptr.resize(P.L);
    P.dom_blk.resize(P.L);
    P.dom_ab.resize(P.L);
    for (int l = 0; l < P.L; ++l)
        domain_plan(l == 0 ? P.rp0 : P.rpA[l], l == 0 ? P.ci0 : P.ciA[l], P.units[l], N, P.dom_ptr[l], P.dom_blk[l],
                    P.dom_ab[l]);

    // ---- restriction / prolongation plans
    P.lead1.assign(P.NS, -1);
    if (P.L > 1) {
        for (int d = 0; d < P.M; ++d) {
            int last = -1;  // ids inside a domain appear in increasing order of lowest lane
            for (int a = 0; a < N; ++a) {
                const int u = P.up[0][d * N + a];
                if (u > last) {
                    P.lead1[d * N + a] = u;
                    last = u;
                }
            }
        }
    }
    P.lmask.assign(P.NS, 0);
    if (P.L > 1)
        for (int d = 0; d < P.M; ++d)
            for (int a = 0; a < N; ++a) {
                const int u = P.lead1[d * N + a];
                if (u < 0) continue;
                uint64_t m = 0;
                for (int b = 0; b < N; ++b)
                    if (P.up[0][d * N + b] == u) m |= uint64_t(1) << b;
                P.lmask[d * N + a] = m;
            }
    P.anc.assign(static_cast<size_t>(std::max(P.L - 1, 0)) * P.NS, -1);
    for (int l = 1; l < P.L; ++l)
        for (int s = 0; s < P.NS; ++s) {
            const int below = l == 1 ? s : P.anc[static_cast<size_t>(l - 2) * P.NS + s];
            P.anc[static_cast<size_t>(l - 1) * P.NS + s] = below < 0 ? -1 : P.up[l - 1][below];
        }
    // ---- work groups and per-group coarse partials
    long long window_blocks = 0;
    for (int s = 0, W = storage_window(N); s < P.NS; s += W)
        window_blocks = std::max<long long>(window_blocks, P.rp0[std::min(s + W, P.NS)] - P.rp0[s]);
    P.D0 = group_domains(P.M, N, nnzb, window_blocks);
    P.RG = P.D0 * N;
    P.G = (P.M + P.D0 - 1) / P.D0;
    P.g_u1.assign(P.G + 1, 0);
    if (P.L > 1) {
        // level-1 ids follow domain order: count the units of each group
        for (int s = 0; s < P.NS; ++s)
            if (P.lead1[s] >= 0) P.g_u1[s / P.RG + 1]++;
        for (int g = 0; g < P.G; ++g) P.g_u1[g + 1] += P.g_u1[g];
    }
    P.anc1.assign(P.L, {});
    P.lead_pos.assign(P.L, {});
    P.cp_ptr.assign(P.L, {});
    P.n_cpart = 0;
    if (P.L > 2) {
        const int S1 = P.units[1];
        std::vector<int> a(S1);
        std::iota(a.begin(), a.end(), 0);
        for (int l = 2; l < P.L; ++l) {
            for (int& v : a) v = P.up[l - 1][v];
            P.anc1[l] = a;
            // (unit, writer) of every distinct (group, unit) pair, by group;
            // their positions by (unit, group)
            std::vector<std::pair<int, int>> pairs;
            std::vector<int> seen(P.units[l], -1);
            for (int g = 0; g < P.G; ++g)
                for (int t = P.g_u1[g]; t < P.g_u1[g + 1]; ++t)
                    if (seen[a[t]] != g) {
                        seen[a[t]] = g;
                        pairs.emplace_back(a[t], t);
                    }
            P.lead_pos[l].assign(S1, -1);
            P.cp_ptr[l].assign(P.units[l] + 1, 0);
            for (const auto& [u, t] : pairs) P.cp_ptr[l][u + 1]++;
            P.cp_ptr[l][0] = P.n_cpart;
            for (int u = 0; u < P.units[l]; ++u) P.cp_ptr[l][u + 1] += P.cp_ptr[l][u];
            std::vector<int> next(P.cp_ptr[l].begin(), P.cp_ptr[l].end() - 1);
            for (const auto& [u, t] : pairs) P.lead_pos[l][t] = next[u]++;
            P.n_cpart += static_cast<int>(pairs.size());
        }
    }

    P.W1 = 1;
    for (int g = 0; g < P.G; ++g) P.W1 = std::max(P.W1, P.g_u1[g + 1] - P.g_u1[g]);
    P.ganc.assign(P.L, {});
    P.gpos.assign(P.L, {});
    P.gmask.assign(P.L, {});
    for (int l = 2; l < P.L; ++l) {
        P.ganc[l].assign(static_cast<size_t>(P.G) * P.W1, -1);
        P.gpos[l].assign(static_cast<size_t>(P.G) * P.W1, -1);
        for (int g = 0; g < P.G; ++g)
            for (int t = P.g_u1[g]; t < P.g_u1[g + 1]; ++t) {
                const size_t o = static_cast<size_t>(g) * P.W1 + (t - P.g_u1[g]);
                P.ganc[l][o] = P.anc1[l][t];
                P.gpos[l][o] = P.lead_pos[l][t];
            }
        P.gmask[l].assign(static_cast<size_t>(P.G) * P.W1, 0);
        if (P.W1 <= 64)
            for (int g = 0; g < P.G; ++g) {
                const int lo = P.g_u1[g], n1 = P.g_u1[g + 1] - lo;
                for (int i = 0; i < n1; ++i) {
                    if (P.lead_pos[l][lo + i] < 0) continue;
                    uint64_t m = 0;
                    for (int j = 0; j < n1; ++j)
                        if (P.anc1[l][lo + j] == P.anc1[l][lo + i]) m |= uint64_t(1) << j;
                    P.gmask[l][static_cast<size_t>(g) * P.W1 + i] = m;
                }
            }
    }

    // the restriction tables by output (see Plan)
    P.gu1_slot.assign(static_cast<size_t>(P.G) * P.W1, -1);
    P.gu1_mask.assign(static_cast<size_t>(P.G) * P.W1, 0);
    if (P.L > 1)
        for (int s = 0; s < P.NS; ++s) {
            const int u = P.lead1[s];
            if (u < 0) continue;
            const int g = s / P.RG;
            const size_t o = static_cast<size_t>(g) * P.W1 + (u - P.g_u1[g]);
            P.gu1_slot[o] = s;
            P.gu1_mask[o] = P.lmask[s];
        }
    std::vector<int> writers(P.G, 0);
    for (int l = 2; l < P.L; ++l)
        for (size_t o = 0; o < P.gpos[l].size(); ++o) writers[o / P.W1] += P.gpos[l][o] >= 0;
    P.GW = std::max(1, *std::max_element(writers.begin(), writers.end()));
    P.gw_pos.assign(static_cast<size_t>(P.G) * P.GW, -1);
    P.gw_li.assign(static_cast<size_t>(P.G) * P.GW, 0);
    P.gw_mask.assign(static_cast<size_t>(P.G) * P.GW, 0);
    for (int g = 0; g < P.G; ++g) {
        size_t e = static_cast<size_t>(g) * P.GW;
        for (int l = 2; l < P.L; ++l)
            for (int i = 0; i < P.W1; ++i) {
                const size_t o = static_cast<size_t>(g) * P.W1 + i;
                if (P.gpos[l][o] < 0) continue;
                P.gw_pos[e] = P.gpos[l][o];
                P.gw_li[e] = (l - 2) * P.W1 + i;
                P.gw_mask[e++] = P.gmask[l][o];
            }
    }

    symmetric_storage(P);
    halo_units(P, f32_values || !P.sym);
    spmv_order(P);

    // ---- per-node units for reports
    P.sn.assign(static_cast<size_t>(P.L) * V, -1);
    for (int i = 0; i < V; ++i) {
        P.sn[i] = P.map[i];
        for (int l = 1; l < P.L; ++l) P.sn[static_cast<size_t>(l) * V + i] = P.anc[static_cast<size_t>(l - 1) * P.NS + P.map[i]];
    }
    return "";
}

}  // namespace maspcg

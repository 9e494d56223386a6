// Graph checks and random-walk generation (Sample of Algorithm 1).
//
// Uniform walks follow the DeepWalk sampler of Section 2 ("Sampling
// process"): each transition picks a neighbour of the current node
// uniformly.  node2vec walks (named in Sections 3 and 5.4) bias the choice by
// the previous node with return parameter p and in-out parameter q; they are
// drawn by rejection so no per-edge alias tables are needed.
//
// Layout: walks are stored step-major, walk[t][col] at t * W + col, so the W
// lanes of a launch write each step as one coalesced row.  One lane owns one
// walk: the step loop is a chain of dependent loads (row bounds, then the
// neighbour), and thousands of walks in flight per CU hide that latency.
#include "common.h"
#include "scan.h"

namespace felog {

// --------------------------------------------------------------------------
// Graph validation: one thread per CSR entry.  Records the smallest offending
// row and the kind of fault as (row << 3 | code) with an atomic minimum.
// --------------------------------------------------------------------------
__device__ __forceinline__ int64_t row_of_entry(const int64_t* indptr, int32_t n, int64_t e)
{
    int32_t lo = 0, hi = n - 1;   // last row r with indptr[r] <= e
    while (lo < hi) {
        int32_t mid = lo + (hi - lo + 1) / 2;
        if (indptr[mid] <= e) lo = mid; else hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ int64_t find_in_row(const int64_t* indptr, const int32_t* indices,
                                               int32_t row, int32_t x)
{
    int64_t lo = indptr[row], hi = indptr[row + 1];
    while (lo < hi) {
        int64_t mid = lo + ((hi - lo) >> 1);
        if (indices[mid] < x) lo = mid + 1; else hi = mid;
    }
    return (lo < indptr[row + 1] && indices[lo] == x) ? lo : -1;
}

__global__ void validate_graph_kernel(const int64_t* indptr, const int32_t* indices,
                                      const float* weights, int32_t n, int64_t nnz,
                                      unsigned long long* bad)
{
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nnz) return;
    int32_t u = (int32_t)row_of_entry(indptr, n, e);
    int32_t v = indices[e];
    int code = 0;
    if (v < 0 || v >= n) code = 1;
    else if (v == u) code = 2;
    else if (e > indptr[u] && indices[e - 1] >= v) code = 3;
    else {
        int64_t r = find_in_row(indptr, indices, v, u);
        if (r < 0) code = 4;
        else if (weights) {
            float w = weights[e];
            if (!(w > 0.0f) || !isfinite(w)) code = 5;
            else if (weights[r] != w) code = 6;
        }
    }
    if (code) atomicMin(bad, ((unsigned long long)u << 3) | (unsigned long long)code);
}

void launch_validate_graph(Graph& g, unsigned long long* d_bad)
{
    Ctx& c = *g.ctx;
    FELOG_HIP(hipMemsetAsync(d_bad, 0xFF, sizeof(unsigned long long), c.stream));
    if (g.nnz == 0) return;
    int64_t blocks = (g.nnz + 255) / 256;
    hipLaunchKernelGGL(validate_graph_kernel, dim3(blocks), dim3(256), 0, c.stream,
                       g.indptr.as<int64_t>(), g.indices.as<int32_t>(),
                       g.weighted ? g.weights.as<float>() : nullptr, g.n, g.nnz, d_bad);
    FELOG_HIP(hipGetLastError());
}

// Largest edge weight of each row (1 for unweighted graphs): the rejection bound.
__global__ void row_wmax_kernel(const int64_t* indptr, const float* weights, int32_t n,
                                float* wmax)
{
    int32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    float m = 0.0f;
    if (weights) {
        for (int64_t e = indptr[v]; e < indptr[v + 1]; ++e) m = fmaxf(m, weights[e]);
    } else {
        m = indptr[v + 1] > indptr[v] ? 1.0f : 0.0f;
    }
    wmax[v] = m;
}

void launch_row_wmax(Graph& g)
{
    Ctx& c = *g.ctx;
    g.wmax.alloc(&c, sizeof(float) * g.n);
    hipLaunchKernelGGL(row_wmax_kernel, dim3((g.n + 255) / 256), dim3(256), 0, c.stream,
                       g.indptr.as<int64_t>(), g.weighted ? g.weights.as<float>() : nullptr, g.n,
                       g.wmax.as<float>());
    FELOG_HIP(hipGetLastError());
}

// (index, weight) records of a weighted graph's entries.  A node2vec attempt
// reads the proposal's index and weight; from two arrays that is two random
// cache lines, from one record one.  The walk kernel is bound by such random
// line fetches: with p = 0.5, q = 2 and weights in (0, 1] most proposals are
// rejected, so a step takes several attempts.
__global__ void edge_records_kernel(const int32_t* __restrict__ indices,
                                    const float* __restrict__ weights, int64_t nnz,
                                    int2* __restrict__ edges)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < nnz) edges[e] = make_int2(indices[e], __float_as_int(weights[e]));
}

void build_edge_records(Graph& g)
{
    Ctx& c = *g.ctx;
    if (!g.weighted) return;
    g.edges.alloc(&c, sizeof(int2) * std::max<int64_t>(g.nnz, 1));
    if (g.nnz)
        hipLaunchKernelGGL(edge_records_kernel, dim3((g.nnz + 255) / 256), dim3(256), 0,
                           c.stream, g.indices.as<int32_t>(), g.weights.as<float>(), g.nnz,
                           g.edges.as<int2>());
    FELOG_HIP(hipGetLastError());
    c.sync();
    g.weights.release();
}

// --------------------------------------------------------------------------
// Uniform walks.  Transition t of walk `wid` moves from v to its neighbour
// number floor(x0 * deg(v) / 2^32), x0 = word 0 of Philox(wid, t, WALK).
// --------------------------------------------------------------------------
__global__ __launch_bounds__(256) void walk_uniform_kernel(
    const int64_t* __restrict__ indptr, const int32_t* __restrict__ indices,
    const int32_t* __restrict__ starts, int64_t n_starts, int64_t W, int64_t col0,
    int64_t col_end, int32_t L, uint64_t seed, int64_t id_base, int32_t* __restrict__ walks)
{
    int64_t col = col0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (col >= col_end) return;
    int64_t si = col % n_starts;
    int32_t v = starts ? starts[si] : (int32_t)si;
    int64_t wid = id_base + col;
    walks[col] = v;
    int32_t t = 0;
    for (; t + 1 < L; ++t) {
        int64_t lo = indptr[v];
        int64_t deg = indptr[v + 1] - lo;
        if (deg == 0) break;
        Rand4 r = philox4x32((uint32_t)wid, (uint32_t)(wid >> 32), (uint32_t)t, kTagWalk, seed);
        v = indices[lo + scale32(r.v[0], (uint32_t)deg)];
        walks[(int64_t)(t + 1) * W + col] = v;
    }
    for (int32_t s = t + 1; s < L; ++s) walks[(int64_t)s * W + col] = -1;
}

// --------------------------------------------------------------------------
// node2vec walks by rejection.  From v (previous node `prev`), attempt a of
// transition t uses Philox(wid, t, N2V | a): propose the neighbour
// floor(x0 * deg / 2^32), draw u = (x1 >> 8) * 2^-24, and accept when
//   u * (wmax(v) * alpha_max) < w(v, x) * alpha(prev, x)
// in FP32, alpha = 1/p (x == prev), 1 (x adjacent to prev), 1/q (otherwise).
// The first transition uses alpha = 1 and the bound wmax(v).  The adjacency
// test is a binary search in the shorter of the sorted rows of prev and x
// (the graph is symmetric), and it is skipped when the proposal is decided
// by the extreme alpha values alone (same result).
//
// The transition takes the first accepted attempt in attempt order, or after
// max_attempts rejections the last proposal.
//
// Bound by chains of dependent random reads of very different lengths: one to
// tens of attempts per transition, each with none to 20 rounds of search.  A
// lane therefore goes its own way through its walk: every pass of the loop
// gives the searching lanes ROUNDS rounds and, once kN2vProposers lanes are
// between attempts (or none is searching), those their next attempt (a Philox
// block, most of a pass's instructions).  A wave then takes as many passes as
// the longest of its 64 walks' sums needs; with all lanes at the same
// transition, two attempts at a time, it was the sum of the longest, and idle
// searches read along.  Against that, 40 steps from every node, ms:
//   deg 29, weighted, p = 0.5, q = 2: R-MAT 2^18 2.70 -> 1.73, 300,007 nodes of
//   equal degree 2.46 -> 2.42 (their long stretches of the same length leave
//   lockstep little to lose); p = 0.25, q = 4: 8.1 -> 4.9 and 6.1 -> 5.5;
//   R-MAT 2^20, deg 16, unweighted, p = 1, q = 2 4.0 -> 3.6.
// Rounds: five beyond the caches (300,007 nodes of equal degree 2.42 ms, two 2.68;
// R-MAT 2^20, deg 16, p = 1, q = 2 7 % faster than two); two where the indices are
// small, as the lanes' searches then end together less often than a round trip is
// long: R-MAT of 59,716 nodes, weighted, p = 0.25 five rounds 18 % (q = 0.5) and 20 %
// (q = 2) slower, 150,000 nodes of equal degree, 17 MB of indices, up to 20 %.
// --------------------------------------------------------------------------
constexpr int kN2vProposers = 16;  // 8 to 32 are within 7 %

template <int ROUNDS>
__global__ __launch_bounds__(256) void walk_node2vec_kernel(
    const int64_t* __restrict__ indptr, const int32_t* __restrict__ indices,
    const int2* __restrict__ edges, const float* __restrict__ wmax,
    const int32_t* __restrict__ starts, int64_t n_starts, int64_t W, int64_t col0,
    int64_t col_end, int32_t L, float inv_p, float inv_q, float amax, uint32_t max_attempts,
    uint64_t seed, int64_t id_base, int32_t* __restrict__ walks,
    unsigned long long* __restrict__ capped)
{
    const int64_t col = col0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (col >= col_end) return;
    const int64_t si = col % n_starts;
    int32_t v = starts ? starts[si] : (int32_t)si;
    const int64_t wid = id_base + col;
    walks[col] = v;
    uint32_t my_capped = 0;
    const float a_hi = fmaxf(1.0f, inv_q), a_lo = fminf(1.0f, inv_q);
    // the transition from v (row lo, deg; previous node's row plo, pdeg), and its
    // attempt
    int32_t t = 0, prev = -1;
    int64_t lo = indptr[v], plo = 0;
    uint32_t deg = (uint32_t)(indptr[v + 1] - lo), pdeg = 0;
    float bound = wmax[v];
    uint32_t attempt = 0;
    // the proposal, its row and largest weight
    int32_t x = -1;
    int64_t xlo = 0;
    uint32_t xdeg = 0;
    float wx = 0.0f, w = 0.0f, lhs = 0.0f;
    // the search: target in indices[base + l, base + h)
    int64_t base = 0;
    uint32_t l = 0, h = 0;
    int32_t target = 0;
    enum { kPropose, kSearch, kDone };
    int mode = L > 1 && deg > 0 ? kPropose : kDone;

    // the attempt's end: the next transition, or the next attempt
    auto settle = [&](bool accept) {
        if (!accept && ++attempt < max_attempts) {
            mode = kPropose;
            return;
        }
        if (!accept) ++my_capped;
        walks[(int64_t)(t + 1) * W + col] = x;
        prev = v;
        plo = lo;
        pdeg = deg;
        v = x;
        lo = xlo;
        deg = xdeg;
        bound = __fmul_rn(wx, amax);
        attempt = 0;
        ++t;
        mode = t + 1 < L && deg > 0 ? kPropose : kDone;
    };

    for (;;) {
        const int searching = __popcll(__ballot(mode == kSearch));
        const int proposing = __popcll(__ballot(mode == kPropose));
        if (searching + proposing == 0) break;
        if (mode == kPropose && (proposing >= kN2vProposers || searching == 0)) {
            const Rand4 r = philox4x32((uint32_t)wid, (uint32_t)(wid >> 32), (uint32_t)t,
                                       kTagN2V | attempt, seed);
            const int64_t e = lo + scale32(r.v[0], deg);
            if (edges) {
                const int2 rec = edges[e];
                x = rec.x;
                w = __int_as_float(rec.y);
            } else {
                x = indices[e];
                w = 1.0f;
            }
            lhs = __fmul_rn((float)(r.v[1] >> 8) * (1.0f / 16777216.0f), bound);
            bool accept = false, undecided = false;
            if (t == 0) accept = lhs < w;
            else if (x == prev) accept = lhs < __fmul_rn(w, inv_p);
            else if (lhs < __fmul_rn(w, a_hi)) {
                accept = lhs < __fmul_rn(w, a_lo);
                undecided = !accept;
            }
            if (accept || undecided || attempt + 1 == max_attempts) {
                xlo = indptr[x];
                xdeg = (uint32_t)(indptr[x + 1] - xlo);
                wx = wmax[x];
            }
            if (undecided) {
                const bool in_x = xdeg < pdeg;
                base = in_x ? xlo : plo;
                h = in_x ? xdeg : pdeg;
                l = 0;
                target = in_x ? prev : x;
                mode = kSearch;
            } else {
                settle(accept);
            }
        }
#pragma unroll
        for (int k = 0; k < ROUNDS; ++k)
            if (mode == kSearch) {
                const uint32_t mid = l + ((h - l) >> 1);
                const int32_t val = indices[base + mid];
                if (val < target) l = mid + 1;
                else h = mid;
                const bool adj = val == target;
                if (adj || l >= h) settle(lhs < __fmul_rn(w, adj ? 1.0f : inv_q));
            }
    }
    for (int32_t s = t + 1; s < L; ++s) walks[(int64_t)s * W + col] = -1;
    if (my_capped) atomicAdd(capped, (unsigned long long)my_capped);
}

// The same walks with the lanes of a wave at the same transition, so that a step's
// walks are written as one row (lanes at transitions of their own write a line
// each), with A attempts in flight.  Without SEARCH, for q = 1: alpha is 1/p at the
// previous node and 1 elsewhere, and no attempt is undecided.  With SEARCH, for rows
// of like length far beyond the caches, where few searches outlast the others and
// the lines that are written in parts cost the most.  40 steps from every node, ms,
// with the kernel above and this one: q = 1, 300,007 nodes of degree 29, weighted,
// p = 1 0.74 and 0.48, p = 0.25 1.80 and 0.96; R-MAT 2^20, deg 16, p = 0.25 2.49 and
// 1.83.  10^6 nodes of equal degree 16, p = 1, q = 4 11.0 and 6.5, weighted 11.5 and
// 7.7.
template <int A, bool SEARCH>
__global__ __launch_bounds__(256) void walk_node2vec_rows_kernel(
    const int64_t* __restrict__ indptr, const int32_t* __restrict__ indices,
    const int2* __restrict__ edges, const float* __restrict__ wmax,
    const int32_t* __restrict__ starts, int64_t n_starts, int64_t W, int64_t col0,
    int64_t col_end, int32_t L, float inv_p, float inv_q, float amax, uint32_t max_attempts,
    uint64_t seed, int64_t id_base, int32_t* __restrict__ walks,
    unsigned long long* __restrict__ capped)
{
    const int64_t col = col0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (col >= col_end) return;
    const int64_t si = col % n_starts;
    int32_t v = starts ? starts[si] : (int32_t)si;
    const int64_t wid = id_base + col;
    walks[col] = v;
    uint32_t my_capped = 0;
    const float a_hi = fmaxf(1.0f, inv_q), a_lo = fminf(1.0f, inv_q);
    int32_t t = 0, prev = -1;
    int64_t plo = 0;                  // the previous node's row
    uint32_t pdeg = 0;
    for (; t + 1 < L; ++t) {
        const int64_t lo = indptr[v];
        const uint32_t deg = (uint32_t)(indptr[v + 1] - lo);
        if (deg == 0) break;
        const float bound = t == 0 ? wmax[v] : __fmul_rn(wmax[v], amax);
        int32_t x = -1;
        for (uint32_t attempt = 0;; attempt += A) {   // max_attempts is a multiple of A
            int32_t xs[A];
            float ws[A], lhs[A];
#pragma unroll
            for (int k = 0; k < A; ++k) {
                const Rand4 r = philox4x32((uint32_t)wid, (uint32_t)(wid >> 32), (uint32_t)t,
                                           kTagN2V | (attempt + k), seed);
                const int64_t e = lo + scale32(r.v[0], deg);
                if (edges) {
                    const int2 rec = edges[e];
                    xs[k] = rec.x;
                    ws[k] = __int_as_float(rec.y);
                } else {
                    xs[k] = indices[e];
                    ws[k] = 1.0f;
                }
                lhs[k] = __fmul_rn((float)(r.v[1] >> 8) * (1.0f / 16777216.0f), bound);
            }
            bool undecided = false, found = false;   // an undecided attempt, and its end
            if constexpr (SEARCH) {
                static_assert(A == 1, "one search at a time");
                undecided = t > 0 && xs[0] != prev && lhs[0] < __fmul_rn(ws[0], a_hi) &&
                            !(lhs[0] < __fmul_rn(ws[0], a_lo));
                if (undecided) {
                    const int64_t xlo = indptr[xs[0]];
                    const uint32_t xdeg = (uint32_t)(indptr[xs[0] + 1] - xlo);
                    const bool in_x = xdeg < pdeg;
                    const int64_t base = in_x ? xlo : plo;
                    const int32_t target = in_x ? prev : xs[0];
                    uint32_t l = 0, h = in_x ? xdeg : pdeg;
                    bool adj = false;
                    while (l < h) {
                        const uint32_t mid = l + ((h - l) >> 1);
                        const int32_t val = indices[base + mid];
                        if (val < target) l = mid + 1;
                        else h = mid;
                        adj = val == target;
                        if (adj) break;
                    }
                    found = lhs[0] < __fmul_rn(ws[0], adj ? 1.0f : inv_q);
                }
            }
            bool accept = false;
#pragma unroll
            for (int k = 0; k < A; ++k)
                if (!accept) {
                    x = xs[k];
                    const float alpha = t > 0 && x == prev ? inv_p : t > 0 && SEARCH ? a_lo : 1.0f;
                    accept = undecided ? found : lhs[k] < __fmul_rn(ws[k], alpha);
                }
            if (accept) break;
            if (attempt + A >= max_attempts) {
                ++my_capped;
                break;
            }
        }
        walks[(int64_t)(t + 1) * W + col] = x;
        if constexpr (SEARCH) {
            plo = lo;
            pdeg = deg;
        }
        prev = v;
        v = x;
    }
    for (int32_t s = t + 1; s < L; ++s) walks[(int64_t)s * W + col] = -1;
    if (my_capped) atomicAdd(capped, (unsigned long long)my_capped);
}

// Which kernel, by the indices' (the searches') and the entries' (the proposals')
// bytes; times relative to the other choice, 40 steps from every node, five p by
// five q.
// q = 1: one attempt at a time beyond 16 MB of entries, where wasted reads cost the
// most (15 to 128 MB, R-MAT and equal degrees: two 0.93 to 1.22 times the time of
// one).  Below, a round trip is most of the time: four where a weight or p < 0.5
// rejects many (12 MB, weighted: two 1.21 to 1.48 times the time of four), else two
// (6 MB, p >= 0.5: four 1.05 to 1.84 times the time of two).
// Else lanes at their own transitions, except on rows of like length (none longer
// than eight times the mean) of more than 48 MB of indices, or 24 MB where neither
// weights nor p < 1 reject: 61 to 66 MB five rounds 0.91 to 1.66 times the time of
// rows; 33 MB 1.04 to 1.29 there, q > 1 and weights or p < 1 0.82 to 1.00; R-MAT 2^20
// (rows of every length), q > 1 and weights or p < 1 0.72 to 0.99.
// Rounds above: 24 MB lies between 17 MB, where five lose, and 33 MB, where two do.
constexpr int64_t kN2vEntryBytes = (int64_t)16 << 20, kN2vIndexBytes = (int64_t)24 << 20;
constexpr int64_t kN2vRowsBytes = (int64_t)48 << 20;

void launch_walk_columns(Walks& w, const felog_walk_params& p, const Active* starts,
                         int64_t n_starts, int64_t col0, int64_t ncols, hipStream_t s,
                         unsigned long long* d_capped)
{
    Graph& g = *w.g;
    FELOG_REQUIRE(col0 >= 0 && ncols >= 0 && col0 + ncols <= w.W, "walk columns out of range");
    if (ncols == 0) return;
    const int32_t* st = starts ? starts->nodes.as<int32_t>() : nullptr;
    const int64_t blocks = (ncols + 255) / 256;
    if (p.kind == FELOG_WALK_UNIFORM) {
        hipLaunchKernelGGL(walk_uniform_kernel, dim3(blocks), dim3(256), 0, s,
                           g.indptr.as<int64_t>(), g.indices.as<int32_t>(), st, n_starts, w.W,
                           col0, col0 + ncols, w.L, p.seed, w.id_base, w.data.as<int32_t>());
    } else {
        FELOG_REQUIRE(d_capped, "node2vec walks need a device counter for capped proposals");
        float inv_p = 1.0f / p.p, inv_q = 1.0f / p.q;
        float amax = fmaxf(1.0f, fmaxf(inv_p, inv_q));
        constexpr uint32_t max_attempts = 1u << 16;
        const int64_t index_bytes = g.nnz * 4, entry_bytes = g.nnz * (g.weighted ? 8 : 4);
        const bool like_rows = g.max_degree > 0 && g.max_degree <= 8 * (g.nnz / g.n + 1);
        const bool few_rejected = !g.weighted && p.p >= 1.0f;
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(blocks), dim3(256), 0, s, g.indptr.as<int64_t>(),
                               g.indices.as<int32_t>(), g.weighted ? g.edges.as<int2>() : nullptr,
                               g.wmax.as<float>(), st, n_starts, w.W, col0, col0 + ncols, w.L,
                               inv_p, inv_q, amax, max_attempts, p.seed, w.id_base,
                               w.data.as<int32_t>(), d_capped);
        };
        if (inv_q == 1.0f) {
            if (entry_bytes > kN2vEntryBytes)
                launch(walk_node2vec_rows_kernel<1, false>);
            else if (g.weighted || amax > 2.0f)
                launch(walk_node2vec_rows_kernel<4, false>);
            else launch(walk_node2vec_rows_kernel<2, false>);
        } else if (index_bytes <= kN2vIndexBytes) {
            launch(walk_node2vec_kernel<2>);
        } else if (like_rows && (index_bytes > kN2vRowsBytes || few_rejected)) {
            launch(walk_node2vec_rows_kernel<1, true>);
        } else {
            launch(walk_node2vec_kernel<5>);
        }
    }
    FELOG_HIP(hipGetLastError());
}

void launch_walks(Walks& w, const felog_walk_params& p, const Active* starts, int64_t n_starts)
{
    Ctx& c = *w.g->ctx;
    w.have_valid = false;
    w.capped = 0;
    if (p.kind == FELOG_WALK_UNIFORM) {
        launch_walk_columns(w, p, starts, n_starts, 0, w.W, c.stream, nullptr);
        return;
    }
    DevBuf cap;
    cap.alloc(&c, sizeof(unsigned long long));
    FELOG_HIP(hipMemsetAsync(cap.ptr, 0, sizeof(unsigned long long), c.stream));
    launch_walk_columns(w, p, starts, n_starts, 0, w.W, c.stream, cap.as<unsigned long long>());
    unsigned long long h = 0;
    FELOG_HIP(hipMemcpyAsync(&h, cap.ptr, sizeof h, hipMemcpyDeviceToHost, c.stream));
    c.sync();
    w.capped = (int64_t)h;
}

// --------------------------------------------------------------------------
// Columns [col0, col0 + ncols) of a step-major corpus as walk-major rows of L.
// A block turns a tile of 64 walks by 64 steps through LDS, so that both the
// reads (64 walks of a step) and the writes (64 steps of a walk) are runs of
// 256 bytes; rows of 65 words keep the column reads off each other's banks.
// It costs microseconds beside the copy to the host that follows; turning the
// rows on the host instead took 40 ms for 300,007 walks of 80 (generated and
// read: 54.4 -> 15.5 ms).
// --------------------------------------------------------------------------
constexpr int kTurn = 64;

__global__ __launch_bounds__(256) void walk_rows_kernel(const int32_t* __restrict__ walks,
                                                        int64_t W, int32_t L, int64_t col0,
                                                        int64_t ncols, int32_t* __restrict__ rows)
{
    __shared__ int32_t tile[kTurn][kTurn + 1];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t c0 = (int64_t)blockIdx.x * kTurn;
    const int32_t t0 = (int32_t)blockIdx.y * kTurn;
    for (int t = wv; t < kTurn; t += 4)
        if (t0 + t < L && c0 + lane < ncols)
            tile[t][lane] = walks[(int64_t)(t0 + t) * W + col0 + c0 + lane];
    __syncthreads();
    for (int c = wv; c < kTurn; c += 4)
        if (c0 + c < ncols && t0 + lane < L)
            rows[(c0 + c) * L + t0 + lane] = tile[lane][c];
}

void launch_walk_rows(const Walks& w, int64_t col0, int64_t ncols, int32_t* rows, hipStream_t s)
{
    const dim3 grid((uint32_t)((ncols + kTurn - 1) / kTurn), (uint32_t)((w.L + kTurn - 1) / kTurn));
    hipLaunchKernelGGL(walk_rows_kernel, grid, dim3(256), 0, s, w.data.as<int32_t>(), w.W, w.L,
                       col0, ncols, rows);
    FELOG_HIP(hipGetLastError());
}

// --------------------------------------------------------------------------
// Columns whose walk yields pairs (two or more nodes), and their count per
// chunk of `chunk` consecutive walks.
// --------------------------------------------------------------------------
struct LongWalk {
    const int32_t* second_step;   // walk[1][*]
    __device__ bool operator()(int64_t col) const { return second_step[col] >= 0; }
};
struct ColumnId {
    __device__ int32_t operator()(int64_t col) const { return (int32_t)col; }
};

// Walks per chunk that yield pairs: valid_cols is sorted, so the count of chunk
// c is the number of entries in [c * chunk, (c + 1) * chunk), by binary search.
__global__ void chunk_count_kernel(const int32_t* valid_cols, int64_t n_valid, int64_t n_chunks,
                                   int64_t chunk, unsigned long long* counts)
{
    int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n_chunks) return;
    auto lower = [&](int64_t x) {
        int64_t lo = 0, hi = n_valid;
        while (lo < hi) {
            int64_t mid = lo + ((hi - lo) >> 1);
            if (valid_cols[mid] < x) lo = mid + 1; else hi = mid;
        }
        return lo;
    };
    counts[c] = (unsigned long long)(lower((c + 1) * chunk) - lower(c * chunk));
}

// valid_cols of the columns with pred(col), and their counts per chunk
template <class Pred>
static void set_valid_columns(Walks& w, int64_t chunk, Pred pred)
{
    Ctx& c = *w.g->ctx;
    int64_t n_chunks = (w.W + chunk - 1) / chunk;
    w.chunk_valid.assign(n_chunks, 0);
    if (w.L < 2 || w.W == 0) {
        w.n_valid = 0;
        w.valid_cols.alloc(&c, sizeof(int32_t));
    } else {
        w.n_valid = compact(c, pred, ColumnId{}, w.W, w.valid_cols);
        DevBuf cnt;
        cnt.alloc(&c, sizeof(unsigned long long) * n_chunks);
        hipLaunchKernelGGL(chunk_count_kernel, dim3((n_chunks + 255) / 256), dim3(256), 0,
                           c.stream, w.valid_cols.as<int32_t>(), w.n_valid, n_chunks, chunk,
                           cnt.as<unsigned long long>());
        FELOG_HIP(hipGetLastError());
        std::vector<unsigned long long> h(n_chunks);
        FELOG_HIP(hipMemcpyAsync(h.data(), cnt.ptr, sizeof(unsigned long long) * n_chunks,
                                 hipMemcpyDeviceToHost, c.stream));
        c.sync();
        for (int64_t i = 0; i < n_chunks; ++i) w.chunk_valid[i] = (int64_t)h[i];
    }
    w.have_valid = true;
    w.chunk_for_valid = chunk;
}

void launch_valid_columns(Walks& w, int64_t chunk)
{
    if (w.have_valid && w.chunk_for_valid == chunk) return;
    set_valid_columns(w, chunk, LongWalk{w.data.as<int32_t>() + w.W});
}

// A walk has a second node exactly when its start node has a neighbour: both
// samplers stop only at a node without neighbours, and node2vec takes its last
// proposal when every attempt is rejected.  So the columns that yield pairs are
// known from the start list alone, before any walk is written.
struct StartHasNeighbour {
    const int64_t* indptr;
    const int32_t* starts;    // null: start of column col is col mod n_starts
    int64_t n_starts;
    __device__ bool operator()(int64_t col) const
    {
        const int64_t si = col % n_starts;
        const int32_t v = starts ? starts[si] : (int32_t)si;
        return indptr[v + 1] > indptr[v];
    }
};

void plan_valid_columns(Walks& w, const Active* starts, int64_t n_starts, int64_t chunk)
{
    const Graph& g = *w.g;
    set_valid_columns(w, chunk, StartHasNeighbour{g.indptr.as<int64_t>(),
                                                  starts ? starts->nodes.as<int32_t>() : nullptr,
                                                  n_starts});
}

}  // namespace felog

// Skip-gram with negative sampling (Train of Algorithm 1; Eq. (1)-(2)).
//
// One minibatch = P consecutive pairs of a chunk's pair order (centre
// position j, then offset slot, then walk).  The pair order is implicit:
// pair g of a chunk is walk valid_cols[g mod Wv] at slice g / Wv, where the
// slice table lists the (j, slot) combinations with both positions inside a
// walk.  Every walk in a chunk has either L nodes or one (an isolated start),
// and the one-node walks are left out of valid_cols, so this closed form is
// exactly the order "next P pairs whose positions both hold a node".
//
// Every pair reads the tables as they stand at the minibatch's start; each
// row's deltas are summed and added once.  A pair touches K + 2 rows: its
// context (in-table) and its centre and K negatives (out-table).  FP32
// atomics on table rows are slow on this part (an L2 atomic unit handles a
// few dwords per clock and hot rows serialise), so the deltas are sorted by
// destination row instead.  Per minibatch:
//   prep     one thread per touch: node ids (walk reads, noise draws) and an
//            integer atomic per touched row whose old value is the touch's
//            rank within the row (rank 0 marks the row's first touch).
//   scan     two passes over the touches: segment offsets of the touched
//            rows, their list, one work item per row of at most kChunk
//            touches and one per kChunk touches of the rows with more.  No
//            atomics: same-address device atomics serialise at about one per
//            12 ns on this part.
//   forward  one wave per pair, two pairs at d = 64 (sgns_forward.h): gather
//            in[ctx], out[ctr], out[neg_1..K]; K+1 dots, sigma and the
//            coefficients g in FP64 over the FP32 entries; writes (g_k, ctx)
//            and the touch's pair-order key at the out-row's segment
//            position, sum_k g_k out[t_k] (rounded to FP32 once) and the pair
//            at the in-row's; out rows touched once are updated in place.
//   split    chunks of the rows with more than kChunk touches: exact sums
//            (below), stored per chunk.
//   reduce   rows of at most kChunk touches, out rows first (they read the
//            in-table as of the minibatch start), then in rows: the touches
//            are sorted by key inside a 16-lane group and their terms summed
//            in FP64 in pair order, added to the row with one rounding.
//   merge    each split row adds its chunks' sums in chunk order.
// prep and scan read only the walks and the noise table, so with two sets
// of their buffers the next minibatch's run on a second stream while this
// one trains.  Every sum is independent of the order the atomics produced,
// so a minibatch's update is bit-identical from run to run.  The split rows'
// sums are exact: each term (an exact FP64 product g * x, or an FP32 per-pair
// delta) is bounded by lr 2^15 in magnitude and rounded once to a multiple
// of 2^(e - 35), e = floor(log2 lr); in FP64, sums of such multiples below
// lr 2^17 carry no rounding error in any order.
// In the apply, lanes own elements 4 (gl + 16 i) .. +3 of a row, so each row
// access is a coalesced 256-byte transaction per i.
#include <algorithm>
#include <cmath>
#include <optional>

#include "common.h"
#include "noise.h"
#include "sgns_device.h"
#include "sgns_forward.h"

namespace felog {

// A launch group: the ids and sorts of up to kIdGroupMax minibatches in one
// launch of each pass (minibatch i in the blocks with blockIdx.y = i, in id
// set set0 + i).  One minibatch's passes are a few dependent loads per thread
// over a few thousand blocks at most, and its launches and the events between
// the two streams cost as much again.
constexpr int kIdGroupMax = 8;
struct GroupMb {
    int64_t vcol_base;     // offset of the minibatch's chunk in valid_cols
    uint32_t Wv;           // valid columns of the chunk
    uint32_t first_pair;   // first pair of the minibatch in its chunk
    uint32_t npairs;
};
// Elements per id set of each array of MinibatchBufs.
struct SetStrides {
    int64_t n, touches, in, out, split_in, split_out, mrows_in, mrows_out, scan_blocks;
};

// ------------------------------------------------------------------- prep
struct PrepArgs {
    const int32_t* __restrict__ walks;   // step-major [L][W]
    int64_t W;
    const int32_t* __restrict__ vcols;
    const int32_t* __restrict__ slices;  // (j << 8) | slot
    GroupMb g[kIdGroupMax];
    int32_t set0;
    SetStrides st;
    int64_t id_base;
    int32_t window;
    uint64_t seed;
    NoiseTable noise;
    uint32_t* cnt_in;        // (these four by id set)
    uint32_t* cnt_out;
    int32_t* touch_row;      // [P][K+2]: context, centre, negatives (-1: negative == centre)
    uint32_t* touch_pos;     // [P][K+2]: rank of the touch within its row
};

// Grid-stride over the touches: the launch is capped at a few blocks per CU,
// which leaves room for the training launches it runs beside.
template <int K>
__global__ __launch_bounds__(256) void sgns_prep_kernel(PrepArgs a)
{
    const GroupMb mb = a.g[blockIdx.y];
    const int64_t set = a.set0 + (int32_t)blockIdx.y;
    const int32_t* vcols = a.vcols + mb.vcol_base;
    uint32_t* const cnt_in = a.cnt_in + set * a.st.n;
    uint32_t* const cnt_out = a.cnt_out + set * a.st.n;
    int32_t* const touch_row = a.touch_row + set * a.st.touches;
    uint32_t* const touch_pos = a.touch_pos + set * a.st.touches;
    const uint32_t nt = mb.npairs * (K + 2);
    for (uint32_t t = blockIdx.x * 256 + threadIdx.x; t < nt; t += gridDim.x * 256) {
        int32_t row = -1;
        bool out = false;
        const uint32_t p = t / (K + 2), r = t - p * (K + 2);
        const uint32_t gq = mb.first_pair + p;
        const uint32_t sidx = gq / mb.Wv;
        const uint32_t rank = gq - sidx * mb.Wv;
        const int32_t js = a.slices[sidx];
        const int32_t col = vcols[rank];
        const int32_t j = js >> 8, s = js & 255;
        const int32_t ctr = a.walks[(int64_t)j * a.W + col];
        if (r == 0) {
            const int32_t off = s < a.window ? s - a.window : s - a.window + 1;
            row = a.walks[(int64_t)(j + off) * a.W + col];
        } else if (r == 1) {
            row = ctr;
            out = true;
        } else {
            // negative k = r - 2: Philox(walk id, (j << 8) | slot, NEG | k / 2), words
            // 2 (k mod 2) and 2 (k mod 2) + 1
            const uint32_t k = r - 2;
            const int64_t wid = a.id_base + col;
            const Rand4 x = philox4x32((uint32_t)wid, (uint32_t)(wid >> 32), (uint32_t)js,
                                       kTagNeg | (k >> 1), a.seed);
            const uint32_t lo = (k & 1) ? x.v[2] : x.v[0];
            const uint32_t hi = (k & 1) ? x.v[3] : x.v[1];
            const int32_t neg = noise_draw(a.noise, ((uint64_t)hi << 32) | lo);
            row = neg != ctr ? neg : -1;   // a negative equal to the centre is skipped
            out = true;
        }
        touch_row[t] = row;
        touch_pos[t] = row >= 0 ? atomicAdd((out ? cnt_out : cnt_in) + row, 1u) : 0u;
    }
}

// ------------------------------------------------------------------- scan
// Items: the in-touches i (touch i (K+2)) and, in further blocks, the
// out-touches e (touch (e / (K+1)) (K+2) + 1 + e mod (K+1)).  A first touch
// (rank 0) lists its row; the scanned values are (entries | chunks << 32),
// the rows listed, the rows split over chunks, their chunks and the out rows
// touched once (which the forward updates itself).  A thread takes I items:
// 2 up to 65,536 pairs per minibatch (shorter chains of dependent loads per
// thread and more blocks than with 8; on R-MAT 2^20, d = 128, K = 5:
// 39.5 -> 34.0 us per minibatch at P = 1,024, 73.2 -> 64.7 at 16,384,
// 146.3 -> 142.7 at 65,536), 8 above, where every block's sum over the
// partials of the blocks before it (quadratic in their number) would grow.
constexpr int kScanT = 256;
constexpr int kScanISmall = 2, kScanILarge = 8;
constexpr int64_t kScanSmallPairs = 65536;
static_assert(kScanT * kScanISmall == kScanSpanMin, "fewest items per scan block");

struct ScanArgs {
    uint32_t npairs[kIdGroupMax];
    int32_t set0;
    SetStrides st;
    // by id set
    const int32_t* touch_row;
    const uint32_t* touch_pos;
    const uint32_t* cnt_in;
    uint32_t* cnt_out;
    unsigned long long* part_ec;   // per block
    uint4* part_rm;                // per block: rows, split rows, chunks of split rows,
                                   // single-touch out rows
    int32_t* list_in;
    int32_t* list_out;
    int32_t* off_in;
    int32_t* off_out;
    int4* chunks_in;
    int4* chunks_out;
    int4* split_in;                // chunks of split rows: row, first entry, length, partial row
    int4* split_out;
    int4* mrows_in;                // split rows: row, first chunk, chunks, list slot
    int4* mrows_out;
    uint32_t* meta;
    int32_t reset;                 // zero the counters of the rows done here (else the
                                   // whole counter arrays are zeroed before the ids)
};

// The arguments of this block's minibatch, and its items and blocks: in-touches
// in blocks [0, nb_in), out-touches in [nb_in, nb).
struct ScanMb : ScanArgs {
    uint32_t n_in, n_out, nb_in, nb;
};
template <int K>
__device__ __forceinline__ ScanMb scan_mb(const ScanArgs& g, uint32_t span)
{
    ScanMb a;
    static_cast<ScanArgs&>(a) = g;
    const int64_t set = g.set0 + (int32_t)blockIdx.y;
    a.n_in = g.npairs[blockIdx.y];
    a.n_out = a.n_in * (K + 1);
    a.nb_in = (a.n_in + span - 1) / span;
    a.nb = a.nb_in + (a.n_out + span - 1) / span;
    a.touch_row += set * g.st.touches;
    a.touch_pos += set * g.st.touches;
    a.cnt_in += set * g.st.n;
    a.cnt_out += set * g.st.n;
    a.part_ec += set * g.st.scan_blocks;
    a.part_rm += set * g.st.scan_blocks;
    a.list_in += set * g.st.in;
    a.list_out += set * g.st.out;
    a.off_in += set * g.st.n;
    a.off_out += set * g.st.n;
    a.chunks_in += set * g.st.in;
    a.chunks_out += set * g.st.out;
    a.split_in += set * g.st.split_in;
    a.split_out += set * g.st.split_out;
    a.mrows_in += set * g.st.mrows_in;
    a.mrows_out += set * g.st.mrows_out;
    a.meta += set * kMetaWords;
    return a;
}

// Items base .. base + I - 1 of a table (n items): the row each one
// lists (-1 if none) and the row's touch count.  BATCH issues the loads of
// all the items before it uses any (indices past the end clamped, their
// values dropped): two round trips to memory instead of 2 I, for when
// the scan is on the minibatch's critical path.  Otherwise each item's loads
// wait for the previous item, which leaves more bandwidth to the launches
// that run beside the scan.
template <int K, bool BATCH, int I>
__device__ __forceinline__ void scan_items(const ScanMb& a, bool out, uint32_t base, uint32_t n,
                                           int32_t (&rows)[I], uint32_t (&cs)[I])
{
    const uint32_t* cnt = out ? a.cnt_out : a.cnt_in;
    if (BATCH) {
        const uint32_t last = n > 0 ? n - 1 : 0;
        uint32_t pos[I];
#pragma unroll
        for (int k = 0; k < I; ++k) {
            const uint32_t i = min(base + k, last);
            const uint32_t t = out ? (i / (K + 1)) * (K + 2) + 1 + i % (K + 1) : i * (K + 2);
            rows[k] = a.touch_row[t];
            pos[k] = a.touch_pos[t];
        }
#pragma unroll
        for (int k = 0; k < I; ++k) {
            const bool first = base + k < n && rows[k] >= 0 && pos[k] == 0u;
            rows[k] = first ? rows[k] : -1;
            cs[k] = cnt[first ? rows[k] : 0];
        }
#pragma unroll
        for (int k = 0; k < I; ++k) cs[k] = rows[k] >= 0 ? cs[k] : 0u;
    } else {
#pragma unroll
        for (int k = 0; k < I; ++k) {
            rows[k] = -1;
            cs[k] = 0u;
            if (base + k < n) {
                const uint32_t i = base + k;
                const uint32_t t = out ? (i / (K + 1)) * (K + 2) + 1 + i % (K + 1) : i * (K + 2);
                const int32_t r = a.touch_row[t];
                if (r >= 0 && a.touch_pos[t] == 0u) {
                    rows[k] = r;
                    cs[k] = cnt[r];
                }
            }
        }
    }
}

__device__ __forceinline__ uint4 add4(uint4 a, uint4 b)
{
    return make_uint4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}

// An out row with a single touch in the minibatch is read and written by that
// touch's pair only, so the forward adds its delta in place: it gets no
// segment entry and no work item.
__device__ __forceinline__ bool single_out(uint32_t c, bool out) { return out && c == 1u; }

__device__ __forceinline__ uint4 split_counts(uint32_t c, bool out)
{
    const uint32_t nch = (c + kChunk - 1) / kChunk;
    return make_uint4(1u, nch > 1 ? 1u : 0u, nch > 1 ? nch : 0u, single_out(c, out) ? 1u : 0u);
}

__device__ __forceinline__ unsigned long long pack_ec(uint32_t c, bool out)
{
    const uint32_t e = single_out(c, out) ? 0u : c;
    return (unsigned long long)e | ((unsigned long long)((e + kChunk - 1) / kChunk) << 32);
}

template <int K, bool BATCH, int I>
__global__ __launch_bounds__(256) void sgns_scan_partials(ScanArgs g)
{
    __shared__ unsigned long long s_ec[kScanT];
    __shared__ uint4 s_rm[kScanT];
    const ScanMb a = scan_mb<K>(g, kScanT * I);
    if (blockIdx.x >= a.nb) return;
    const bool out = blockIdx.x >= a.nb_in;
    const uint32_t nb = out ? blockIdx.x - a.nb_in : blockIdx.x;
    const uint32_t n = out ? a.n_out : a.n_in;
    const uint32_t base = nb * (kScanT * I) + threadIdx.x * I;
    unsigned long long ec = 0;
    uint4 rm = make_uint4(0u, 0u, 0u, 0u);
    int32_t rows[I];
    uint32_t cs[I];
    scan_items<K, BATCH, I>(a, out, base, n, rows, cs);
#pragma unroll
    for (int k = 0; k < I; ++k) {
        if (rows[k] >= 0) {
            ec += pack_ec(cs[k], out);
            rm = add4(rm, split_counts(cs[k], out));
        }
    }
    s_ec[threadIdx.x] = ec;
    s_rm[threadIdx.x] = rm;
    __syncthreads();
    for (int s = kScanT / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            s_ec[threadIdx.x] += s_ec[threadIdx.x + s];
            s_rm[threadIdx.x] = add4(s_rm[threadIdx.x], s_rm[threadIdx.x + s]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        a.part_ec[blockIdx.x] = s_ec[0];
        a.part_rm[blockIdx.x] = s_rm[0];
    }
}

template <int K, bool BATCH, int I>
__global__ __launch_bounds__(256) void sgns_scan_write(ScanArgs g)
{
    __shared__ unsigned long long s_ec[kScanT];
    __shared__ uint4 s_rm[kScanT];
    const ScanMb a = scan_mb<K>(g, kScanT * I);
    if (blockIdx.x >= a.nb) return;
    const bool out = blockIdx.x >= a.nb_in;
    const uint32_t b0 = out ? a.nb_in : 0u;   // first block of this table
    const uint32_t n = out ? a.n_out : a.n_in;
    const uint32_t nb = blockIdx.x - b0;
    // offset of this block: partials of the earlier blocks of the same table
    unsigned long long pre = 0;
    uint4 pre_rm = make_uint4(0u, 0u, 0u, 0u);
    for (uint32_t b = b0 + threadIdx.x; b < blockIdx.x; b += kScanT) {
        pre += a.part_ec[b];
        pre_rm = add4(pre_rm, a.part_rm[b]);
    }
    s_ec[threadIdx.x] = pre;
    s_rm[threadIdx.x] = pre_rm;
    __syncthreads();
    for (int s = kScanT / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            s_ec[threadIdx.x] += s_ec[threadIdx.x + s];
            s_rm[threadIdx.x] = add4(s_rm[threadIdx.x], s_rm[threadIdx.x + s]);
        }
        __syncthreads();
    }
    const unsigned long long blk_ec = s_ec[0];
    const uint4 blk_rm = s_rm[0];
    __syncthreads();

    const uint32_t base = nb * (kScanT * I) + threadIdx.x * I;
    // (entries scanned in the low word; the chunk count in the high word is unused here)
    int32_t rows[I];
    uint32_t cs[I];
    unsigned long long mine = 0;
    uint4 mine_rm = make_uint4(0u, 0u, 0u, 0u);
    scan_items<K, BATCH, I>(a, out, base, n, rows, cs);
#pragma unroll
    for (int k = 0; k < I; ++k) {
        if (rows[k] >= 0) {
            mine += pack_ec(cs[k], out);
            mine_rm = add4(mine_rm, split_counts(cs[k], out));
        }
    }
    // block exclusive scans
    s_ec[threadIdx.x] = mine;
    s_rm[threadIdx.x] = mine_rm;
    __syncthreads();
    for (int off = 1; off < kScanT; off <<= 1) {
        const unsigned long long add = threadIdx.x >= off ? s_ec[threadIdx.x - off] : 0ull;
        const uint4 add_rm = threadIdx.x >= off ? s_rm[threadIdx.x - off] : make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
        s_ec[threadIdx.x] += add;
        s_rm[threadIdx.x] = add4(s_rm[threadIdx.x], add_rm);
        __syncthreads();
    }
    const unsigned long long run = blk_ec + s_ec[threadIdx.x] - mine;
    const uint4 at = s_rm[threadIdx.x];
    uint32_t slot = blk_rm.x + at.x - mine_rm.x;    // list slot
    uint32_t mrow = blk_rm.y + at.y - mine_rm.y;    // split-row index
    uint32_t mchunk = blk_rm.z + at.z - mine_rm.z;  // first chunk of the next split row
    uint32_t sgl = blk_rm.w + at.w - mine_rm.w;     // single-touch out rows before
    uint32_t entry = (uint32_t)run;
    int32_t* list = out ? a.list_out : a.list_in;
    int32_t* off = out ? a.off_out : a.off_in;
    int4* chunks = out ? a.chunks_out : a.chunks_in;   // one per row of at most kChunk touches
    int4* split = out ? a.split_out : a.split_in;      // chunks of the split rows
    int4* mrows = out ? a.mrows_out : a.mrows_in;
#pragma unroll
    for (int k = 0; k < I; ++k) {
        if (rows[k] >= 0) {
            const uint32_t c = cs[k];
            list[slot] = rows[k];
            if (single_out(c, out)) {
                // the forward adds this row's delta; -1 - slot marks it and
                // carries its list slot
                off[rows[k]] = -1 - (int32_t)slot;
                if (a.reset) a.cnt_out[rows[k]] = 0u;
                ++sgl;
            } else {
                const uint32_t nch = (c + kChunk - 1) / kChunk;
                off[rows[k]] = (int32_t)entry;
                if (nch == 1) {
                    chunks[slot - mrow - sgl] =
                        make_int4(rows[k], (int32_t)entry, (int32_t)c, (int32_t)slot);
                } else {
                    mrows[mrow] = make_int4(rows[k], (int32_t)mchunk, (int32_t)nch, (int32_t)slot);
                    for (uint32_t j = 0; j < nch; ++j)
                        split[mchunk + j] = make_int4(rows[k], (int32_t)(entry + j * kChunk),
                                                      (int32_t)min((uint32_t)kChunk, c - j * kChunk),
                                                      (int32_t)(mchunk + j));
                    ++mrow;
                    mchunk += nch;
                }
                entry += c;
            }
            ++slot;
        }
        if (base + k + 1 == n) {   // the table's last item: totals
            a.meta[out ? 1 : 0] = slot;
            a.meta[out ? 3 : 2] = slot - mrow - sgl;   // rows of one chunk
            a.meta[out ? 5 : 4] = mrow;          // split rows
            a.meta[out ? 7 : 6] = mchunk;        // their chunks
        }
    }
}

// ---------------------------------------------------------------- forward
struct FwdArgs {
    const float* __restrict__ tin;
    float* __restrict__ tout;      // single-touch out rows are updated here
    const int32_t* __restrict__ touch_row;
    const uint32_t* __restrict__ touch_pos;
    const int32_t* __restrict__ off_in;
    const int32_t* __restrict__ off_out;
    uint32_t npairs;
    int32_t ppw;             // pairs per wave, ppw (K + 2) <= 64
    float lr;
    int4* ent_out;           // (FP64 g, ctx, pair-order key p (K+1) + k) by out-row
                             // segment position
    float* dinp;             // [P][d] sum_k g_k out[t_k] (FP64 sum, rounded once) by
                             // in-row segment position
    uint32_t* key_in;        // the pair p, same position
    double* loss_part;       // one slot per wave
    float* cap_out;          // capture != NULL: single-touch out-row deltas to cap_out[slot][d]
};

// A wave takes its ppw pairs one step (sgns_forward.h) at a time.  CAP: the
// deltas of the out rows touched once are captured, not applied.  Bound by the
// random row reads and the rows, deltas and entries written: 65,536 pairs on
// R-MAT 2^20 (d = 128, K = 5) 87 -> 62 us, about 330 MB at 5.3 TB/s.  Before, a
// half wave per pair needed 164 registers (three waves per SIMD) and each dot
// five ds_bpermute steps.  One step holds 74 registers (six waves); two steps
// per batch share more arithmetic and were no faster (62 - 65 us).
template <int D, int K, bool CAP>
__global__ __launch_bounds__(256) void sgns_forward_kernel(FwdArgs a)
{
    constexpr int S = 1;
    using Batch = FwdBatch<D, K, S, kStream>;
    constexpr int T = K + 2, H = Batch::H, L = Batch::L, V = Batch::V;
    const int lane = threadIdx.x & 63;
    const uint32_t gl = lane & (L - 1);
    const uint32_t gwave = blockIdx.x * (blockDim.x >> 6) +
                           (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t q0 = gwave * (uint32_t)a.ppw;
    if (q0 >= a.npairs) return;
    const int np = (int)min((uint32_t)a.ppw, a.npairs - q0);

    // ---- touch metadata: lane l < np T holds touch l of the wave's pairs and
    //      its position in its row's segment, or, for an out row touched once
    //      in the minibatch, the row's list slot (and a bit in `single`)
    int32_t m_row = -1;
    int32_t m_pos = 0;
    bool m_single = false;
    if (lane < np * T) {
        const uint32_t t = q0 * T + lane;
        m_row = a.touch_row[t];
        const uint32_t rk = a.touch_pos[t];
        const bool in = (lane % T) == 0;
        if (m_row >= 0) {
            const int32_t off = (in ? a.off_in : a.off_out)[m_row];
            m_single = off < 0;
            m_pos = m_single ? -1 - off : off + (int32_t)rk;
        }
    }
    const unsigned long long single = __ballot(m_single);

    const double lr = (double)a.lr;
    double lacc = 0.0;
    for (int base = 0; base < np; base += S * H) {
        Batch bt;
        bt.load(a.tin, a.tout, m_row, base, np);
        bt.coefficients(m_row, base, np, lr, lacc);
        // the lane that evaluated a touch writes its entry
        {
            const int32_t pos = __shfl(m_pos, bt.touch);
            const int pr = bt.touch / T;
            const int32_t ctx = __shfl(m_row, pr * T);
            if (bt.mine && !((single >> bt.touch) & 1ull))
                store_nt(&a.ent_out[pos],
                         pack_entry(bt.g, ctx, (q0 + (uint32_t)pr) * (K + 1) +
                                                   (uint32_t)(bt.touch - pr * T - 1)));
        }
#pragma unroll
        for (int b = 0; b < S; ++b) {
            const int p = base + b * H + (H == 2 ? lane >> 5 : 0);
            const bool live = p < np;
            const int src = (live ? p : 0) * T;
            double gk[K + 1];
#pragma unroll
            for (int k = 0; k <= K; ++k) gk[k] = bt.coef(b, k);
            // out rows touched once: row + g in[ctx] in FP64, rounded once (or
            // the delta alone, when capturing)
#pragma unroll
            for (int k = 0; k <= K; ++k) {
                int32_t slot = 0;
                if constexpr (CAP) slot = __shfl(m_pos, src + 1 + k);
                if (live && bt.row[b][k] >= 0 && ((single >> (src + 1 + k)) & 1ull)) {
                    f2* dst = reinterpret_cast<f2*>(CAP ? a.cap_out + (int64_t)slot * D
                                                        : a.tout + (int64_t)bt.row[b][k] * D);
#pragma unroll
                    for (int i = 0; i < V; ++i)
                        store_row2<kStream>(row_at(dst, i * L + gl),
                                            bt.out_row(b, i, gk[k],
                                                       CAP ? f2{0.0f, 0.0f} : bt.vo[b][k][i]));
                }
            }
            const int32_t pos_in = __shfl(m_pos, src);
            if (live) {
                if (gl == 0) store_nt(&a.key_in[pos_in], q0 + (uint32_t)p);
                f2* dp = reinterpret_cast<f2*>(a.dinp + (int64_t)pos_in * D);
                f2 o[V];
                bt.in_delta(b, gk, o);
#pragma unroll
                for (int i = 0; i < V; ++i) store_row2<kStream>(row_at(dp, i * L + gl), o[i]);
            }
        }
    }
    lacc = wave_total(lacc);
    if (lane == 0) a.loss_part[gwave] += lacc;
}

// ---------------------------------------------------------------- reduce
// Out rows: delta out[t] = sum over touches of g * in[ctx].
// In rows:  delta in[c]  = sum over touches of the pair's in-row delta.
// Rows of at most kChunk touches: one 16-lane group per row sorts the
// touches by their pair-order key (a bitonic network over the group) and
// sums their FP64 terms in that order, so the result is the sequential sum
// in pair order whatever the atomics did.  Chunks of the rows with more
// touches (their membership follows the atomics' order) get exact sums
// instead, which a merge adds in chunk order.
// Sort (key, a, b) ascending over the 16 lanes of a group, of which the first
// `most` hold keys (the others the largest key): the bitonic network's stages
// up to that many lanes.  The keys carry their lane; the values move once, at
// the end.
__device__ __forceinline__ void sort16(uint32_t key, double& va, int32_t& vb, int gl, int most)
{
    uint32_t from = (uint32_t)gl;
    auto stage = [&](uint32_t pk, uint32_t pf, int k, int j) {
        const bool up = (gl & k) == 0;        // this pair of lanes sorts ascending
        const bool low = (gl & j) == 0;       // this lane keeps the smaller key
        const bool take = (low == up) ? pk < key : pk > key;
        key = take ? pk : key;
        from = take ? pf : from;
    };
    stage(from_xor<1>(key), from_xor<1>(from), 2, 1);
    if (most > 2) {
        stage(from_xor<2>(key), from_xor<2>(from), 4, 2);
        stage(from_xor<1>(key), from_xor<1>(from), 4, 1);
    }
    if (most > 4) {
        stage(from_xor<4>(key), from_xor<4>(from), 8, 4);
        stage(from_xor<2>(key), from_xor<2>(from), 8, 2);
        stage(from_xor<1>(key), from_xor<1>(from), 8, 1);
    }
    if (most > 8) {
        stage(from_xor<8>(key), from_xor<8>(from), 16, 8);
        stage(from_xor<4>(key), from_xor<4>(from), 16, 4);
        stage(from_xor<2>(key), from_xor<2>(from), 16, 2);
        stage(from_xor<1>(key), from_xor<1>(from), 16, 1);
    }
    const int lane = (int)((threadIdx.x & 48u) | from);
    va = __shfl(va, lane);
    vb = __shfl(vb, lane);
}

// Two launches per minibatch, each over a list of work items of three kinds:
//   first:  chunks of split out rows, chunks of split in rows (exact sums,
//           stored), out rows of at most kChunk touches (sorted FP32 sums);
//   second: in rows of at most kChunk touches, then the merge of the split
//           out rows and split in rows (their chunks' sums in chunk order).
// Out rows need the in-table as of the minibatch start, so every in row is
// written in the second launch.
struct ApplyArgs {
    float* tin;
    float* tout;
    const int4* ent_out;          // (FP64 g, ctx, pair-order key) by out segment position
    const float* dinp;            // in-row delta of each pair, by in segment position
    const uint32_t* key_in;       // pair by in segment position
    const int4* chunks_in;        // rows of at most kChunk touches
    const int4* chunks_out;
    const int4* split_in;         // chunks of split rows
    const int4* split_out;
    const int4* mrows_in;         // split rows
    const int4* mrows_out;
    double* partial_in;           // exact sums of the split rows' chunks
    double* partial_out;
    uint32_t* cnt_in;
    uint32_t* cnt_out;
    const uint32_t* meta;         // this minibatch's counters
    float* cap_in;                // capture != NULL: deltas to capture[list slot][d]
    float* cap_out;
    unsigned long long* row_totals;
    double grid_c;                // 1.5 * 2^(floor(log2 lr) + 17)
    int32_t reset;                // zero the counters of the rows done here
};

template <int D, int PHASE>
__global__ __launch_bounds__(256) void sgns_apply_kernel(ApplyArgs a)
{
    constexpr int V4 = D / 64;
    // rows in flight per group.  No load is issued for slots past the item's
    // end: pointed at row 0, they all read one line, which queued in one memory
    // channel (with 2 rows, us per minibatch before and after: 5,000 pairs,
    // d = 256, K = 7 72.5 and 56, 65,536 pairs 162 and 157; Algorithm 1 at
    // 16,384 pairs on 20,000 nodes 66.7 and 59.5 ms).  One row is slower there
    // (58.5, 158.5, 62.7), four hold too many registers (58.6, 165.5, 62.2).
    constexpr int kRows = 2;
    const int lane = threadIdx.x & 63;
    const int grp = lane >> 4, gl = lane & 15;
    const int g0 = grp << 4;
    // item ranges [0, e1) [e1, e2) [e2, e3)
    const uint32_t e1 = PHASE == 0 ? a.meta[7] : a.meta[2];
    const uint32_t e2 = e1 + (PHASE == 0 ? a.meta[6] : a.meta[5]);
    const uint32_t e3 = e2 + (PHASE == 0 ? a.meta[3] : a.meta[4]);
    const uint32_t nw = gridDim.x * (blockDim.x >> 6);
    // the descriptor of item c: a chunk of a split row, a row of one chunk, or
    // a split row to merge
    auto desc_of = [&](uint32_t c) -> int4 {
        const int kind = c < e1 ? 0 : (c < e2 ? 1 : 2);
        const uint32_t ci = kind == 0 ? c : (kind == 1 ? c - e1 : c - e2);
        const int4* arr = PHASE == 0
            ? (kind == 0 ? a.split_out : (kind == 1 ? a.split_in : a.chunks_out))
            : (kind == 0 ? a.chunks_in : (kind == 1 ? a.mrows_out : a.mrows_in));
        return arr[ci];
    };
    const uint32_t stride = nw * 4u;
    const uint32_t first = (blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 4u;
    int4 next = first + grp < e3 ? desc_of(first + grp) : make_int4(0, 0, 0, 0);
    for (uint32_t base = first; base < e3; base += stride) {
        const uint32_t c = base + grp;
        const int4 d = next;
        // the next item's descriptor is in flight while this one is done
        if (c + stride < e3) next = desc_of(c + stride);
        if (c >= e3) continue;
        const int kind = c < e1 ? 0 : (c < e2 ? 1 : 2);
        if (PHASE == 1 && kind > 0) {
            // merge of a split row: its chunks' exact sums in chunk order
            const bool out = kind == 1;
            const int4 m = d;
            float4 cur[V4];
            get_row<D>(out ? a.tout : a.tin, out ? a.cap_out : a.cap_in, m.x, cur, gl);
            const double* partial = out ? a.partial_out : a.partial_in;
            double acc[D / 16];
#pragma unroll
            for (int e = 0; e < D / 16; ++e) acc[e] = 0.0;
            for (int32_t j = 0; j < m.z; ++j) {
                const double* pr = partial + (int64_t)(m.y + j) * D;
#pragma unroll
                for (int i = 0; i < V4; ++i) {
                    const double2* q = reinterpret_cast<const double2*>(pr + (i * 16 + gl) * 4);
                    const double2 u = q[0], v = q[1];
                    acc[4 * i + 0] += u.x;
                    acc[4 * i + 1] += u.y;
                    acc[4 * i + 2] += v.x;
                    acc[4 * i + 3] += v.y;
                }
            }
            put_row<D>(out ? a.tout : a.tin, out ? a.cap_out : a.cap_in, m.x, m.w, cur, acc, gl);
            if (a.reset && gl == 0) (out ? a.cnt_out : a.cnt_in)[m.x] = 0;
            continue;
        }
        // out rows draw on in[ctx] with coefficient g, in rows on the per-pair deltas
        const bool split = PHASE == 0 && kind < 2;
        const bool out = PHASE == 0 ? kind != 1 : false;
        const int32_t row = d.x, start = d.y, len = d.z, slot = d.w;
        const float* src = out ? a.tin : a.dinp;
        double my_g = 1.0;
        int32_t my_src = start + gl;
        uint32_t my_key = 0xffffffffu;
        if (gl < len) {
            if (out) {
                const int4 e = a.ent_out[start + gl];
                my_g = entry_g(e);
                my_src = e.z;
                my_key = (uint32_t)e.w;
            } else {
                my_key = a.key_in[start + gl];
            }
        }
        if (split) {
            // exact sums, stored for the merge
            double acc[D / 16];
#pragma unroll
            for (int e = 0; e < D / 16; ++e) acc[e] = 0.0;
            const double gc = a.grid_c;
            for (int32_t i0 = 0; i0 < len; i0 += kRows) {
                double gg[kRows];
                float4 x[kRows][V4];
#pragma unroll
                for (int u = 0; u < kRows; ++u) {
                    const int32_t idx = min(i0 + u, kChunk - 1);
                    const bool ok = i0 + u < len;
                    gg[u] = ok ? __shfl(my_g, g0 + idx) : 0.0;
                    const int32_t rr = __shfl(my_src, g0 + idx);
                    const float4* rp = row4<D>(src, rr);
#pragma unroll
                    for (int i = 0; i < V4; ++i) x[u][i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    if (ok)
#pragma unroll
                        for (int i = 0; i < V4; ++i) x[u][i] = rp[i * 16 + gl];
                }
#pragma unroll
                for (int u = 0; u < kRows; ++u) {
                    // each FP64 term g * x is rounded once more, onto the grid
                    const double gd = gg[u];
#pragma unroll
                    for (int i = 0; i < V4; ++i) {
                        acc[4 * i + 0] += on_grid(gd * (double)x[u][i].x, gc);
                        acc[4 * i + 1] += on_grid(gd * (double)x[u][i].y, gc);
                        acc[4 * i + 2] += on_grid(gd * (double)x[u][i].z, gc);
                        acc[4 * i + 3] += on_grid(gd * (double)x[u][i].w, gc);
                    }
                }
            }
            double* pr = (out ? a.partial_out : a.partial_in) + (int64_t)slot * D;
#pragma unroll
            for (int i = 0; i < V4; ++i) {
                double2* q = reinterpret_cast<double2*>(pr + (i * 16 + gl) * 4);
                q[0] = make_double2(acc[4 * i + 0], acc[4 * i + 1]);
                q[1] = make_double2(acc[4 * i + 2], acc[4 * i + 3]);
            }
            continue;
        }
        // a row of at most kChunk touches: FP64 sum in pair order
        float4 cur[V4];
        get_row<D>(out ? a.tout : a.tin, out ? a.cap_out : a.cap_in, row, cur, gl);
        sort16(my_key, my_g, my_src, gl, len);
        double acc[D / 16];
#pragma unroll
        for (int e = 0; e < D / 16; ++e) acc[e] = 0.0;
        for (int32_t i0 = 0; i0 < len; i0 += kRows) {
            double gg[kRows];
            float4 x[kRows][V4];
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                const int32_t idx = min(i0 + u, kChunk - 1);
                const bool ok = i0 + u < len;
                gg[u] = __shfl(my_g, g0 + idx);
                const int32_t rr = __shfl(my_src, g0 + idx);
                const float4* rp = row4<D>(src, rr);
#pragma unroll
                for (int i = 0; i < V4; ++i) x[u][i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (ok)
#pragma unroll
                    for (int i = 0; i < V4; ++i) x[u][i] = rp[i * 16 + gl];
            }
#pragma unroll
            for (int u = 0; u < kRows; ++u)
#pragma unroll
                for (int i = 0; i < V4; ++i) {
                    // in rows: g = 1, and 1 * x + acc is exactly x + acc
                    acc[4 * i + 0] = fma(gg[u], (double)x[u][i].x, acc[4 * i + 0]);
                    acc[4 * i + 1] = fma(gg[u], (double)x[u][i].y, acc[4 * i + 1]);
                    acc[4 * i + 2] = fma(gg[u], (double)x[u][i].z, acc[4 * i + 2]);
                    acc[4 * i + 3] = fma(gg[u], (double)x[u][i].w, acc[4 * i + 3]);
                }
        }
        put_row<D>(out ? a.tout : a.tin, out ? a.cap_out : a.cap_in, row, slot, cur, acc, gl);
        if (a.reset && gl == 0) (out ? a.cnt_out : a.cnt_in)[row] = 0;
    }
    // the second launch counts the minibatch's touched rows
    if (PHASE == 1 && blockIdx.x == 0 && threadIdx.x == 0) {
        a.row_totals[0] += a.meta[0];
        a.row_totals[1] += a.meta[1];
        a.row_totals[2] += a.meta[1] - a.meta[3] - a.meta[5];   // out rows touched once
    }
}

// Fixed-order FP64 sum of the per-wave loss partials (one block).
__global__ __launch_bounds__(256) void loss_reduce_kernel(const double* part, int64_t n,
                                                          double* out)
{
    __shared__ double lds[256];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) acc += part[i];
    lds[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) lds[threadIdx.x] += lds[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = lds[0];
}

void launch_loss_reduce(const double* part, int64_t n, double* out, hipStream_t s)
{
    hipLaunchKernelGGL(loss_reduce_kernel, dim3(1), dim3(256), 0, s, part, n, out);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
// (j, slot) slices with both positions inside a walk of length L, in pair order.
static std::vector<int32_t> make_slices(int32_t L, int32_t w)
{
    std::vector<int32_t> out;
    for (int32_t j = 0; j < L; ++j)
        for (int32_t s = 0; s < 2 * w; ++s) {
            int32_t off = s < w ? s - w : s - w + 1;
            if (j + off >= 0 && j + off < L) out.push_back((j << 8) | s);
        }
    return out;
}

static TrainSchedule make_schedule(Walks& w, const felog_train_params& p)
{
    const int64_t chunk = chunk_walks_of(p);
    FELOG_REQUIRE(w.chunk_ready.empty() || w.chunk_for_valid == chunk,
                  "the corpus is being written in chunks of %lld walks, not %lld",
                  (long long)w.chunk_for_valid, (long long)chunk);
    launch_valid_columns(w, chunk);
    TrainSchedule s;
    s.nslices = (int64_t)make_slices(w.L, p.window).size();
    int64_t base = 0;
    for (size_t c = 0; c < w.chunk_valid.size(); ++c) {
        int64_t pairs = w.chunk_valid[c] * s.nslices;
        FELOG_REQUIRE(pairs < ((int64_t)1 << 32),
                      "a chunk yields %lld pairs; at most 2^32 - 1 are supported (use a "
                      "smaller chunk_walks)", (long long)pairs);
        s.chunk_first_mb.push_back(s.B);
        s.chunk_pairs.push_back(pairs);
        s.chunk_valid_base.push_back(base);
        base += w.chunk_valid[c];
        s.B += (pairs + p.minibatch_pairs - 1) / p.minibatch_pairs;
        s.total_pairs += pairs;
    }
    return s;
}

TrainSchedule train_schedule(Walks& w, const felog_train_params& p) { return make_schedule(w, p); }

std::vector<int32_t> train_slices(int32_t L, int32_t window) { return make_slices(L, window); }

int64_t count_minibatches(Walks& w, const felog_train_params& p, int64_t* total_pairs)
{
    TrainSchedule s = make_schedule(w, p);
    if (total_pairs) *total_pairs = s.total_pairs;
    return s.B;
}

// (Re)allocates the counters and offsets of `sets` id sets.
static void alloc_id_counters(Model& m, int sets)
{
    Ctx& c = *m.ctx;
    const bool spare = sets > kIdSets;
    const int64_t n = m.g->n;
    MinibatchBufs& b = m.mb;
    m.id_sets = 0;
    for (DevBuf* x : {&b.cnt_in, &b.cnt_out, &b.off_in, &b.off_out, &m.meta}) x->release();
    for (DevBuf* x : {&b.cnt_in, &b.cnt_out, &b.off_in, &b.off_out})
        x->alloc(&c, sizeof(uint32_t) * n * sets, spare);
    m.meta.alloc(&c, sizeof(uint32_t) * sets * kMetaWords, spare);
    m.id_sets = sets;
    m.counters_dirty = true;
}

void model_alloc_update_state(Model& m)
{
    Ctx& c = *m.ctx;
    alloc_id_counters(m, kIdSets);
    m.row_totals.alloc(&c, sizeof(uint64_t) * 3);
    m.loss_out.alloc(&c, sizeof(double));
}

// Rows split over chunks have more than kChunk touches, so at most
// touches / (kChunk + 1) of them, with ceil(c / kChunk) <= 2 c / (kChunk + 1)
// chunks each: at most touches / 8 + 1 chunks in all.
static int64_t max_split_rows(int64_t touches) { return touches / (kChunk + 1) + 1; }

// Largest minibatch whose launches all go to the training stream.
constexpr int64_t kOneStreamPairs = 2048;
// Touches of a launch group of ids.
constexpr int64_t kIdGroupTouches = (int64_t)1 << 21;
// Zero the row counters whole when n <= this many times the minibatch's touches.
constexpr int64_t kZeroWholeRatio = 8;
static int64_t max_split_chunks(int64_t touches) { return touches / 8 + 1; }

// Launch geometry and per-minibatch values of one minibatch.
struct MinibatchLaunch {
    uint32_t npairs;
    int dim, K;
    int set;              // id set
    SetStrides st;
    uint32_t fwd_blocks, reduce_blocks;
    int64_t split_in;     // partial-sum rows reserved for the in-table (the out-table's follow)
    double grid_c;        // exact-sum grid constant of this minibatch's learning rate
    bool zero_whole;      // the row counters are zeroed whole before the ids (else reset rows)
};

// Launch values of a group's ids.
struct IdGroup {
    int K, set0, count;
    uint32_t npairs[kIdGroupMax];
    uint32_t prep_blocks, scan_blocks;   // of the largest minibatch
    int scan_i;           // scan items per thread (kScanISmall or kScanILarge)
    bool one_stream;      // ids on the training stream (on the critical path)
    bool zero_whole;
    SetStrides st;
};

// Zeroes a[0, n) and b[0, n) from element `off`: 16-byte stores, then the tails.
__global__ __launch_bounds__(256) void zero_counters_kernel(uint32_t* a, uint32_t* b, int64_t n)
{
    const int64_t head = min(n, (int64_t)((16 - (reinterpret_cast<uintptr_t>(a) & 15)) & 15) / 4);
    const int64_t n4 = (n - head) / 4, tail = n - head - 4 * n4;
    const int64_t stride = (int64_t)gridDim.x * 256;
    const uint4 z = make_uint4(0u, 0u, 0u, 0u);
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < 2 * n4; i += stride) {
        uint4* p = reinterpret_cast<uint4*>((i < n4 ? a : b) + head);
        p[i < n4 ? i : i - n4] = z;
    }
    if (blockIdx.x == 0 && threadIdx.x < 8) {
        const int t = threadIdx.x & 3;
        uint32_t* p = threadIdx.x < 4 ? a : b;
        if (t < head) p[t] = 0u;
        if (t < tail) p[head + 4 * n4 + t] = 0u;
    }
}

// Zeroes the counters of id sets [set0, set0 + count).
static void zero_counters(Model& m, int set0, int count, hipStream_t s)
{
    const int64_t n = m.g->n, total = n * count;
    const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>((total / 2 + 255) / 256, 512));
    // both arrays come from an allocator and have the same offset from 16 bytes
    hipLaunchKernelGGL(zero_counters_kernel, dim3(blocks), dim3(256), 0, s,
                       m.mb.cnt_in.as<uint32_t>() + set0 * n, m.mb.cnt_out.as<uint32_t>() + set0 * n,
                       total);
}

// When the ids run on a second stream and the table is not much larger than
// the minibatch's touches, the row counters are zeroed whole before each
// minibatch's ids (two streaming writes of n words beside the training
// launches) instead of with one scattered write per touched row on the
// training stream; otherwise the rows are reset as they are done.
// Ids, ranks and the destination sort of a group (reads only the walks and
// the noise table, so it may run ahead of the training of earlier ones).
template <int K>
static void launch_ids_t(Model& m, PrepArgs pa, const IdGroup& ig, hipStream_t s)
{
    MinibatchBufs& mb = m.mb;
    if (ig.zero_whole) zero_counters(m, ig.set0, ig.count, s);
    pa.set0 = ig.set0;
    pa.st = ig.st;
    pa.cnt_in = mb.cnt_in.as<uint32_t>();
    pa.cnt_out = mb.cnt_out.as<uint32_t>();
    pa.touch_row = mb.touch_row.as<int32_t>();
    pa.touch_pos = mb.touch_pos.as<uint32_t>();
    hipLaunchKernelGGL((sgns_prep_kernel<K>), dim3(ig.prep_blocks, ig.count), dim3(256), 0, s, pa);
    ScanArgs sa{};
    for (int i = 0; i < ig.count; ++i) sa.npairs[i] = ig.npairs[i];
    sa.set0 = ig.set0;
    sa.st = ig.st;
    sa.touch_row = pa.touch_row;
    sa.touch_pos = pa.touch_pos;
    sa.cnt_in = pa.cnt_in;
    sa.cnt_out = pa.cnt_out;
    sa.part_rm = mb.partials.as<uint4>();
    sa.part_ec = reinterpret_cast<unsigned long long*>(sa.part_rm + m.id_sets_cap * ig.st.scan_blocks);
    sa.list_in = mb.list_in.as<int32_t>();
    sa.list_out = mb.list_out.as<int32_t>();
    sa.off_in = mb.off_in.as<int32_t>();
    sa.off_out = mb.off_out.as<int32_t>();
    sa.chunks_in = mb.chunks_in.as<int4>();
    sa.chunks_out = mb.chunks_out.as<int4>();
    sa.split_in = mb.split_in.as<int4>();
    sa.split_out = mb.split_out.as<int4>();
    sa.mrows_in = mb.mrows_in.as<int4>();
    sa.mrows_out = mb.mrows_out.as<int4>();
    sa.meta = m.meta.as<uint32_t>();
    sa.reset = ig.zero_whole ? 0 : 1;
    const bool small = ig.scan_i == kScanISmall;
    const dim3 grid(ig.scan_blocks, ig.count), block(256);
    if (ig.one_stream && small) {
        hipLaunchKernelGGL((sgns_scan_partials<K, true, kScanISmall>), grid, block, 0, s, sa);
        hipLaunchKernelGGL((sgns_scan_write<K, true, kScanISmall>), grid, block, 0, s, sa);
    } else if (ig.one_stream) {
        hipLaunchKernelGGL((sgns_scan_partials<K, true, kScanILarge>), grid, block, 0, s, sa);
        hipLaunchKernelGGL((sgns_scan_write<K, true, kScanILarge>), grid, block, 0, s, sa);
    } else if (small) {
        hipLaunchKernelGGL((sgns_scan_partials<K, false, kScanISmall>), grid, block, 0, s, sa);
        hipLaunchKernelGGL((sgns_scan_write<K, false, kScanISmall>), grid, block, 0, s, sa);
    } else {
        hipLaunchKernelGGL((sgns_scan_partials<K, false, kScanILarge>), grid, block, 0, s, sa);
        hipLaunchKernelGGL((sgns_scan_write<K, false, kScanILarge>), grid, block, 0, s, sa);
    }
    FELOG_HIP(hipGetLastError());
}

// Forward and the two apply launches of one minibatch whose ids are ready.
// ev (optional): [0] recorded before the forward, [1] after it, [2] after the
// first apply launch, [3] at the end.
template <int D, int K>
static void launch_train_t(Model& m, FwdArgs fa, const MinibatchLaunch& ml, float* cap_in,
                           float* cap_out, hipStream_t s, hipEvent_t* ev)
{
    const MinibatchBufs& mb = m.mb;
    const SetStrides& st = ml.st;
    const int64_t set = ml.set;
    fa.touch_row = mb.touch_row.as<int32_t>() + set * st.touches;
    fa.touch_pos = mb.touch_pos.as<uint32_t>() + set * st.touches;
    fa.off_in = mb.off_in.as<int32_t>() + set * st.n;
    fa.off_out = mb.off_out.as<int32_t>() + set * st.n;
    fa.cap_out = cap_out;
    if (ev) FELOG_HIP(hipEventRecord(ev[0], s));
    if (cap_out)
        hipLaunchKernelGGL((sgns_forward_kernel<D, K, true>), dim3(ml.fwd_blocks), dim3(256), 0, s, fa);
    else
        hipLaunchKernelGGL((sgns_forward_kernel<D, K, false>), dim3(ml.fwd_blocks), dim3(256), 0, s, fa);
    if (ev) FELOG_HIP(hipEventRecord(ev[1], s));
    double* part_in = m.partial.as<double>();
    double* part_out = part_in + ml.split_in * D;
    ApplyArgs aa{};
    aa.tin = m.tin.as<float>();
    aa.tout = m.tout.as<float>();
    aa.ent_out = fa.ent_out;
    aa.dinp = fa.dinp;
    aa.key_in = fa.key_in;
    aa.chunks_in = mb.chunks_in.as<int4>() + set * st.in;
    aa.chunks_out = mb.chunks_out.as<int4>() + set * st.out;
    aa.split_in = mb.split_in.as<int4>() + set * st.split_in;
    aa.split_out = mb.split_out.as<int4>() + set * st.split_out;
    aa.mrows_in = mb.mrows_in.as<int4>() + set * st.mrows_in;
    aa.mrows_out = mb.mrows_out.as<int4>() + set * st.mrows_out;
    aa.partial_in = part_in;
    aa.partial_out = part_out;
    aa.cnt_in = mb.cnt_in.as<uint32_t>() + set * st.n;
    aa.cnt_out = mb.cnt_out.as<uint32_t>() + set * st.n;
    aa.meta = m.meta.as<uint32_t>() + set * kMetaWords;
    aa.cap_in = cap_in;
    aa.cap_out = cap_out;
    aa.row_totals = m.row_totals.as<unsigned long long>();
    aa.grid_c = ml.grid_c;
    aa.reset = ml.zero_whole ? 0 : 1;
    hipLaunchKernelGGL((sgns_apply_kernel<D, 0>), dim3(ml.reduce_blocks), dim3(256), 0, s, aa);
    if (ev) FELOG_HIP(hipEventRecord(ev[2], s));
    hipLaunchKernelGGL((sgns_apply_kernel<D, 1>), dim3(ml.reduce_blocks), dim3(256), 0, s, aa);
    if (ev) FELOG_HIP(hipEventRecord(ev[3], s));
    FELOG_HIP(hipGetLastError());
}

#define FELOG_FOR_K(X)                                                               \
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) \
    X(16) X(17) X(18) X(19) X(20)

static void launch_ids(Model& m, const PrepArgs& pa, const IdGroup& ig, hipStream_t s)
{
    switch (ig.K) {
#define FELOG_CASE(k)                   \
    case k:                             \
        launch_ids_t<k>(m, pa, ig, s);  \
        break;
        FELOG_FOR_K(FELOG_CASE)
#undef FELOG_CASE
        default: fail(FELOG_EUNSUPPORTED, "negatives = %d not supported", ig.K);
    }
}

template <int D>
static void launch_train_d(Model& m, const FwdArgs& fa, const MinibatchLaunch& ml, float* ci,
                           float* co, hipStream_t s, hipEvent_t* ev)
{
    switch (ml.K) {
#define FELOG_CASE(k)                                    \
    case k:                                              \
        launch_train_t<D, k>(m, fa, ml, ci, co, s, ev);  \
        break;
        FELOG_FOR_K(FELOG_CASE)
#undef FELOG_CASE
        default: fail(FELOG_EUNSUPPORTED, "negatives = %d not supported", ml.K);
    }
}

static void launch_train(Model& m, const FwdArgs& fa, const MinibatchLaunch& ml, float* ci,
                         float* co, hipStream_t s, hipEvent_t* ev)
{
    if (ml.dim == 64) launch_train_d<64>(m, fa, ml, ci, co, s, ev);
    else if (ml.dim == 128) launch_train_d<128>(m, fa, ml, ci, co, s, ev);
    else launch_train_d<256>(m, fa, ml, ci, co, s, ev);
}

// Elements per id set for minibatches of up to P pairs and K negatives.
static SetStrides set_strides(int64_t n, int64_t P, int64_t K)
{
    const int64_t touches_out = P * (K + 1);
    SetStrides st{};
    st.n = n;
    st.touches = P * (K + 2);
    st.in = P;
    st.out = touches_out;
    st.split_in = max_split_chunks(P);
    st.split_out = max_split_chunks(touches_out);
    st.mrows_in = max_split_rows(P);
    st.mrows_out = max_split_rows(touches_out);
    st.scan_blocks = (P + kScanSpanMin - 1) / kScanSpanMin +
                     (touches_out + kScanSpanMin - 1) / kScanSpanMin;
    return st;
}

// Bytes of one id set, without its counters and offsets, and of those.
static uint64_t id_set_bytes(const SetStrides& st)
{
    return 8 * (uint64_t)st.touches + (4 + 16) * (uint64_t)(st.in + st.out) +
           16 * (uint64_t)(st.split_in + st.split_out + st.mrows_in + st.mrows_out) +
           24 * (uint64_t)st.scan_blocks;
}
static uint64_t id_counter_bytes(int64_t n) { return 16 * (uint64_t)n + 4 * kMetaWords; }

// Id sets beyond kIdSets are optional, and each holds 16 bytes per node: all of
// a model's take at most an eighth of its two tables or 256 MiB, whichever is
// more (at 65,536 pairs on 2^20 nodes eight sets take 0.15 GB beside 1.07 GB of
// tables at d = 128; sixteen on 2^27 nodes would take 28 GB at any d).
static int id_sets_wanted(const Model& m, const SetStrides& st, int want)
{
    const int64_t tables = 2 * (int64_t)sizeof(float) * m.g->n * m.dim;
    const int64_t room = std::max<int64_t>(tables / 8, (int64_t)256 << 20);
    const int64_t cost = (int64_t)(id_set_bytes(st) + id_counter_bytes(m.g->n));
    return (int)std::max<int64_t>(kIdSets, std::min<int64_t>(want, kIdSets + room / cost));
}

// (Re)allocates the arrays of `sets` id sets other than the counters.
static void alloc_id_sets(Model& m, int sets, const SetStrides& st)
{
    Ctx& c = *m.ctx;
    MinibatchBufs& b = m.mb;
    const bool spare = sets > kIdSets;
    struct {
        DevBuf& buf;
        size_t bytes;
    } const arrays[] = {
        {b.touch_row, sizeof(int32_t) * st.touches},
        {b.touch_pos, sizeof(uint32_t) * st.touches},
        {b.list_in, sizeof(int32_t) * st.in},
        {b.list_out, sizeof(int32_t) * st.out},
        {b.chunks_in, sizeof(int4) * st.in},
        {b.chunks_out, sizeof(int4) * st.out},
        {b.split_in, sizeof(int4) * st.split_in},
        {b.split_out, sizeof(int4) * st.split_out},
        {b.mrows_in, sizeof(int4) * st.mrows_in},
        {b.mrows_out, sizeof(int4) * st.mrows_out},
        {b.partials, (sizeof(uint4) + sizeof(unsigned long long)) * st.scan_blocks}};
    m.id_sets_cap = 0;
    for (const auto& x : arrays) x.buf.release();
    for (const auto& x : arrays) x.buf.alloc(&c, sets * x.bytes, spare);
    m.id_sets_cap = sets;
}

// Frees the id sets, but for their counters, and the buffers of one minibatch.
static void drop_id_buffers(Model& m)
{
    MinibatchBufs& b = m.mb;
    m.cap_pairs = 0;
    m.cap_K = 0;
    m.id_sets_cap = 0;
    for (DevBuf* x : {&b.touch_row, &b.touch_pos, &b.list_in, &b.list_out, &b.chunks_in,
                      &b.chunks_out, &b.split_in, &b.split_out, &b.mrows_in, &b.mrows_out,
                      &b.partials, &m.ent_out, &m.dinp, &m.key_in, &m.partial})
        x->release();
}

// Leaves the model kIdSets id sets if it has more; it takes no more from then on.
void shrink_id_sets(Model& m)
{
    if (std::max(m.id_sets, m.id_sets_cap) <= kIdSets) return;
    m.few_id_sets = true;
    try {
        if (m.id_sets > kIdSets) alloc_id_counters(m, kIdSets);
        if (m.id_sets_cap > kIdSets)
            alloc_id_sets(m, kIdSets, set_strides(m.g->n, m.cap_pairs, m.cap_K));
    } catch (const Error& e) {
        if (e.code != FELOG_ENOMEM) throw;   // (they are taken on the next use)
        (void)hipGetLastError();
        clear_error();
    }
}

// The model's scratch for minibatches of P pairs and K negatives with at least
// kIdSets id sets, and up to `want` (id_sets_wanted) where the budget and the
// card have room; returns the id sets there are.
static int ensure_id_buffers(Model& m, int64_t P, int K, int want)
{
    Ctx& c = *m.ctx;
    const int64_t n = m.g->n;
    const bool grows = m.cap_pairs < P || m.cap_K < K;
    const int64_t cp = std::max<int64_t>(m.cap_pairs, P);
    const int ck = std::max(m.cap_K, K);
    const SetStrides st = set_strides(n, cp, ck);
    MinibatchBufs& b = m.mb;
    DevBuf* const sets_bufs[] = {&b.cnt_in, &b.cnt_out, &b.off_in, &b.off_out, &m.meta,
                                 &b.touch_row, &b.touch_pos, &b.list_in, &b.list_out,
                                 &b.chunks_in, &b.chunks_out, &b.split_in, &b.split_out,
                                 &b.mrows_in, &b.mrows_out, &b.partials};
    want = m.few_id_sets ? kIdSets : id_sets_wanted(m, st, want);
    const int have = std::min(m.id_sets, m.id_sets_cap);
    if (!grows && have >= want) return have;
    if (grows) drop_id_buffers(m);   // an allocation that fails leaves no stale capacity
    auto alloc_all = [&](int sets) {
        // (sets of a smaller minibatch beyond those wanted now are given back)
        if (m.id_sets < sets || (grows && m.id_sets > sets)) alloc_id_counters(m, sets);
        if (m.cap_pairs < cp || m.cap_K < ck) {
            m.ent_out.alloc(&c, sizeof(int4) * cp * (ck + 1));
            m.dinp.alloc(&c, sizeof(float) * cp * m.dim);
            m.key_in.alloc(&c, sizeof(uint32_t) * cp);
            m.split_rows_in = st.split_in;
            m.partial.alloc(&c, sizeof(double) * (st.split_in + st.split_out) * m.dim);
            m.cap_pairs = cp;
            m.cap_K = ck;
        }
        if (m.id_sets_cap < sets) alloc_id_sets(m, sets, st);
    };
    int sets = want;
    if (c.budget && sets > kIdSets) {
        // more than fit the budget are not tried
        uint64_t held = 0, need = (id_set_bytes(st) + id_counter_bytes(n)) * (uint64_t)sets;
        for (DevBuf* x : sets_bufs) held += x->bytes;
        if (grows)
            need += 16 * (uint64_t)cp * (ck + 1) + 4 * (uint64_t)cp * (m.dim + 1) +
                    8 * (uint64_t)(st.split_in + st.split_out) * m.dim;
        const uint64_t room = c.budget + held - std::min(c.budget + held, c.in_use);
        if (need > room) sets = std::max(kIdSets, m.id_sets_cap);
    }
    // where memory is short: with kIdSets, then without the plans of smaller
    // minibatches too
    for (int attempt = 0;; ++attempt) {
        try {
            alloc_all(sets);
            break;
        } catch (const Error& e) {
            if (e.code != FELOG_ENOMEM || attempt == 2) throw;
            (void)hipGetLastError();
            clear_error();
            if (attempt == 0) {
                if (std::max(sets, m.id_sets) > kIdSets) m.few_id_sets = true;   // not tried again
                for (DevBuf* x : sets_bufs) x->release();
                m.id_sets = m.id_sets_cap = 0;
                sets = kIdSets;
            } else {
                drop_plans(m);
            }
        }
    }
    return std::min(m.id_sets, m.id_sets_cap);
}

// Fewest minibatches of a call that planned launches serve.  They start with the
// plans of the first ones, a workgroup each, which take 30 us and more however
// few there are; the launches of ids and scans are 28 us per minibatch.  us of
// a call (ids / planned), 100,000 nodes, d = 128, K = 5: 1,024 pairs 124 / 134 for one
// minibatch, 152 / 166 two, 178 / 176 three; 2,048 pairs 123 / 170, 157 / 212, 192 /
// 231, 224 / 240 and 265 / 251 for one to five (on 1,000 nodes 133 / 149, 169 / 171,
// 203 / 184, 241 / 197); 256 pairs 118 / 118, 144 / 145.
static int64_t planned_fewest(int64_t touches)
{
    return touches <= kSmallMaxTouches / 4 ? 1 : touches <= kSmallMaxTouches ? 3 : 4;
}

void train_minibatches(Model& m, const Walks& wc, const felog_train_params& p, int64_t first_mb,
                       int64_t n_mb, bool apply, felog_train_stats* stats, int32_t* rows_in,
                       float* d_in_host, int64_t cap_in, int64_t* n_in, int32_t* rows_out,
                       float* d_out_host, int64_t cap_out, int64_t* n_out)
{
    Walks& w = const_cast<Walks&>(wc);
    Ctx& c = *m.ctx;
    c.make_current();
    TrainSchedule sch = make_schedule(w, p);
    const int K = p.negatives;
    const int64_t P = p.minibatch_pairs;
    int64_t end = n_mb < 0 ? sch.B : std::min<int64_t>(sch.B, first_mb + n_mb);
    if (first_mb > sch.B) first_mb = sch.B;
    if (!apply) FELOG_REQUIRE(first_mb < sch.B, "minibatch %lld out of range (%lld minibatches)",
                              (long long)first_mb, (long long)sch.B);

    if (m.precision == FELOG_PREC_BF16) {
        std::vector<int32_t> sl = make_slices(w.L, p.window);
        DevBuf slices;
        slices.alloc(&c, sizeof(int32_t) * std::max<size_t>(sl.size(), 1));
        if (!sl.empty())
            FELOG_HIP(hipMemcpyAsync(slices.ptr, sl.data(), sizeof(int32_t) * sl.size(),
                                     hipMemcpyHostToDevice, c.stream));
        if (apply) {
            train_minibatches_bf16(m, w, p, sch, slices.as<int32_t>(), first_mb, end, nullptr,
                                   nullptr, stats);
            return;
        }
        // capture: deltas into dense zeroed tables, then the touched rows
        const int64_t cnt = (int64_t)m.g->n * m.dim;
        FELOG_REQUIRE(cnt <= ((int64_t)1 << 31), "delta capture of a BF16 model is limited to "
                      "n * d <= 2^31");
        DevBuf din, dout;
        din.alloc(&c, sizeof(float) * cnt);
        dout.alloc(&c, sizeof(float) * cnt);
        FELOG_HIP(hipMemsetAsync(din.ptr, 0, din.bytes, c.stream));
        FELOG_HIP(hipMemsetAsync(dout.ptr, 0, dout.bytes, c.stream));
        felog_train_stats st{};
        train_minibatches_bf16(m, w, p, sch, slices.as<int32_t>(), first_mb, first_mb + 1,
                               din.as<float>(), dout.as<float>(), &st);
        std::vector<int32_t> ids(2 * (size_t)p.minibatch_pairs + p.shared_negatives);
        FELOG_HIP(hipMemcpyAsync(ids.data(), m.bf_ids.ptr, sizeof(int32_t) * ids.size(),
                                 hipMemcpyDeviceToHost, c.stream));
        std::vector<float> hin(cnt), hout(cnt);
        FELOG_HIP(hipMemcpyAsync(hin.data(), din.ptr, sizeof(float) * cnt, hipMemcpyDeviceToHost,
                                 c.stream));
        FELOG_HIP(hipMemcpyAsync(hout.data(), dout.ptr, sizeof(float) * cnt,
                                 hipMemcpyDeviceToHost, c.stream));
        c.sync();
        std::vector<char> seen_in(m.g->n, 0), seen_out(m.g->n, 0);
        int64_t ui = 0, uo = 0;
        const int64_t Pn = p.minibatch_pairs;
        auto put = [&](int32_t row, bool out) {
            std::vector<char>& seen = out ? seen_out : seen_in;
            if (row < 0 || seen[row]) return;
            seen[row] = 1;
            int64_t& u = out ? uo : ui;
            FELOG_REQUIRE(u < (out ? cap_out : cap_in), "capture buffers too small");
            (out ? rows_out : rows_in)[u] = row;
            std::copy_n((out ? hout : hin).data() + (int64_t)row * m.dim, m.dim,
                        (out ? d_out_host : d_in_host) + u * m.dim);
            ++u;
        };
        for (int64_t q = 0; q < Pn; ++q) put(ids[q], false);
        for (int64_t q = 0; q < Pn; ++q) if (ids[q] >= 0) put(ids[Pn + q], true);
        for (int64_t q = 0; q < p.shared_negatives; ++q) put(ids[2 * Pn + q], true);
        if (n_in) *n_in = ui;
        if (n_out) *n_out = uo;
        if (stats) *stats = st;
        return;
    }

    const std::vector<int32_t> sl = make_slices(w.L, p.window);
    DevBuf slices;
    slices.alloc(&c, sizeof(int32_t) * std::max<size_t>(sl.size(), 1));
    if (!sl.empty())
        FELOG_HIP(hipMemcpyAsync(slices.ptr, sl.data(), sizeof(int32_t) * sl.size(),
                                 hipMemcpyHostToDevice, c.stream));
    const int64_t touches = P * (K + 2);
    if (apply && touches <= kSmallMaxTouches && small_path_applies(m, p)) {
        train_minibatches_small(m, w, p, sch, slices.as<int32_t>(), first_mb, end, stats);
        return;
    }
    // planned launches where they apply, for calls of a few minibatches only
    // where the ids' buffers find no room
    const bool few = end - first_mb < planned_fewest(touches);
    auto planned = [&] {
        return apply && touches <= 2 * kSmallMaxTouches &&
               train_minibatches_planned(m, w, p, sch, slices.as<int32_t>(), first_mb, end, stats);
    };
    if (!few && planned()) return;

    // Launch groups: the ids of up to eight minibatches together, about 2^21
    // touches, in two rings of id sets; without the memory for them (or for a
    // single minibatch) one by one in a ring of kIdSets.
    const bool one_stream = P <= kOneStreamPairs;
    int G = 1;
    if (apply && !one_stream)
        G = (int)std::max<int64_t>(1, std::min<int64_t>({(int64_t)kIdGroupMax, end - first_mb,
                                                         kIdGroupTouches / (P * (K + 2))}));
    // pairs per forward wave: two steps (at 65,536 pairs, d = 128, K = 5 one
    // step ran 71 us, two to four 63; at 5,000 pairs, d = 256, K = 7 one step
    // 18.1, two 17.4, four 20.2), one where two would leave fewer than eight
    // waves per compute unit
    const int side = m.dim == 64 ? 2 : 1;
    const int ppw = P >= (int64_t)2 * side * c.num_cus * 8 ? std::min(64 / (K + 2), 2 * side) : side;
    const int64_t waves = (P + ppw - 1) / ppw;
    const int64_t blocks = (waves + 3) / 4;
    // the call's own buffers come before the id sets, which take what is left
    DevBuf loss_part, vin, vout;
    std::optional<HoldScratch> hold;
    int id_sets = 0;
    try {
        loss_part.alloc(&c, sizeof(double) * blocks * 4);
        if (!apply) {
            vin.alloc(&c, sizeof(float) * (size_t)P * m.dim);
            vout.alloc(&c, sizeof(float) * (size_t)P * (K + 1) * m.dim);
        }
        hold.emplace(m);
        id_sets = ensure_id_buffers(m, P, K, G > 1 ? 2 * G : kIdSets);
    } catch (const Error& e) {
        if (e.code != FELOG_ENOMEM || !few) throw;
        const std::string what = felog_last_error();
        loss_part.release();
        if (apply) drop_id_buffers(m);
        if (planned()) return;
        set_error("%s", what.c_str());
        throw;
    }
    if (G > 1 && id_sets < 2 * G) G = std::max(1, id_sets / 2);
    const int rings = G > 1 ? 2 : kIdSets;
    const SetStrides st = set_strides(m.g->n, m.cap_pairs, m.cap_K);
    FELOG_HIP(hipMemsetAsync(loss_part.ptr, 0, sizeof(double) * blocks * 4, c.stream));
    FELOG_HIP(hipMemsetAsync(m.row_totals.ptr, 0, sizeof(uint64_t) * 3, c.stream));

    PrepArgs pa{};
    pa.walks = w.data.as<int32_t>();
    pa.W = w.W;
    pa.vcols = w.valid_cols.as<int32_t>();
    pa.slices = slices.as<int32_t>();
    pa.id_base = w.id_base;
    pa.window = p.window;
    pa.seed = p.seed;
    pa.noise = NoiseTable{m.cdf.as<uint64_t>(), m.guide.as<int32_t>(), m.total_weight,
                          m.guide_bits};

    FwdArgs fa{};
    fa.tin = m.tin.as<float>();
    fa.tout = m.tout.as<float>();
    fa.ppw = ppw;
    fa.ent_out = m.ent_out.as<int4>();
    fa.dinp = m.dinp.as<float>();
    fa.key_in = m.key_in.as<uint32_t>();
    fa.loss_part = loss_part.as<double>();

    const double lr0 = (double)p.lr_start, lr1 = (double)p.lr_end;
    // Small minibatches run everything on one stream: their launches are
    // chains of a few dependent loads each, and waiting on another stream's
    // events costs more than the overlap gains.
    const bool zero_whole = !one_stream && (int64_t)m.g->n <= kZeroWholeRatio * P * (K + 2);
    // minibatches that reset their rows expect zero counters and leave them
    // zero; the others zero them first and leave them dirty
    if (!zero_whole && m.counters_dirty) {
        zero_counters(m, 0, m.id_sets, c.stream);
        m.counters_dirty = false;
    }
    if (zero_whole) m.counters_dirty = true;
    // the launch values of minibatch b
    size_t chunk = 0;
    size_t gated = 0;   // walk chunks [0, gated) are known to be written
    auto frame = [&](int64_t b, int set, MinibatchLaunch& ml, GroupMb& mb) {
        while (chunk + 1 < sch.chunk_first_mb.size() && sch.chunk_first_mb[chunk + 1] <= b) ++chunk;
        const int64_t first = (b - sch.chunk_first_mb[chunk]) * P;
        const int64_t np = std::min<int64_t>(P, sch.chunk_pairs[chunk] - first);
        mb.vcol_base = sch.chunk_valid_base[chunk];
        mb.Wv = (uint32_t)w.chunk_valid[chunk];
        mb.first_pair = (uint32_t)first;
        mb.npairs = (uint32_t)np;
        ml = MinibatchLaunch{};
        ml.dim = m.dim;
        ml.K = K;
        ml.set = set;
        ml.st = st;
        ml.npairs = (uint32_t)np;
        ml.fwd_blocks = (uint32_t)(((np + ppw - 1) / ppw + 3) / 4);
        // 16 blocks per CU (faster than 6, 8 or 32 at 65,536 pairs on 2^20 rows),
        // but no more than the items can use: at most one row per touch and per
        // table row, plus the chunks of split rows, 16 items per block at a time
        const int64_t touches = np * (K + 2);
        const int64_t items = std::min<int64_t>(touches, 2 * (int64_t)m.g->n) + touches / kChunk + 16;
        ml.reduce_blocks = (uint32_t)std::max<int64_t>(
            1, std::min<int64_t>((int64_t)c.num_cus * 16, (items + 15) / 16));
        ml.split_in = m.split_rows_in;
        ml.zero_whole = zero_whole;
        const double lr = lr0 - (lr0 - lr1) * (double)b / (double)std::max<int64_t>(1, sch.B - 1);
        const float lr32 = (float)lr;
        ml.grid_c = lr32 > 0.0f ? std::ldexp(1.5, std::ilogb(lr32) + 17) : 1.5;
        return lr32;
    };
    // the launch values of a group's ids from its minibatches'
    auto finish_group = [&](IdGroup& ig, const PrepArgs& a, int set0, int count) {
        ig.K = K;
        ig.set0 = set0;
        ig.count = count;
        ig.one_stream = one_stream;
        ig.zero_whole = zero_whole;
        ig.st = st;
        ig.scan_i = P <= kScanSmallPairs ? kScanISmall : kScanILarge;
        const int64_t span = (int64_t)kScanT * ig.scan_i;
        for (int i = 0; i < count; ++i) {
            const int64_t np = a.g[i].npairs;
            ig.npairs[i] = a.g[i].npairs;
            ig.prep_blocks = std::max(ig.prep_blocks, (uint32_t)std::min<int64_t>(
                (int64_t)c.num_cus * 4, (np * (K + 2) + 255) / 256));
            ig.scan_blocks = std::max(ig.scan_blocks, (uint32_t)((np + span - 1) / span +
                                                                 (np * (K + 1) + span - 1) / span));
        }
    };
    // stream s reads the walks of chunk ch next: wait until they are written
    auto gate = [&](hipStream_t s, size_t ch) {
        while (gated <= ch && gated < w.chunk_ready.size())
            FELOG_HIP(hipStreamWaitEvent(s, w.chunk_ready[gated++], 0));
    };

    // sampled timing: [0] before the group's ids (on the id stream) and [1] after
    // them for the first timed minibatch of a group (each timed one counts its
    // share), [2] before the forward, [3] after it, [4] after the first apply launch,
    // [5] after the second
    const int every = apply ? c.timing_every : 0;
    const size_t pool = c.timing_pool.size() / kTimingEvents;
    size_t next_slot = 0, used_slots = 0;
    int64_t timed = 0;
    double ms_prep = 0.0, ms_fwd = 0.0, ms_apply = 0.0, ms_apply_first = 0.0;
    std::vector<double> ids_share(pool, 0.0);   // by slot: timed minibatches of its group per
                                                // minibatch of it, 0 without id events
    auto harvest = [&](size_t slot) {
        hipEvent_t* e = &c.timing_pool[kTimingEvents * slot];
        FELOG_HIP(hipEventSynchronize(e[5]));
        float a0 = 0.0f, f = 0.0f, ap = 0.0f, ap0 = 0.0f;
        if (ids_share[slot] > 0.0) FELOG_HIP(hipEventElapsedTime(&a0, e[0], e[1]));
        FELOG_HIP(hipEventElapsedTime(&f, e[2], e[3]));
        FELOG_HIP(hipEventElapsedTime(&ap, e[3], e[5]));
        FELOG_HIP(hipEventElapsedTime(&ap0, e[3], e[4]));
        ms_prep += a0 * ids_share[slot];
        ms_fwd += f;
        ms_apply += ap;
        ms_apply_first += ap0;
        ++timed;
    };
    auto take_slot = [&](int64_t b) -> int {
        if (!(every > 0 && pool > 0 && (b - first_mb) % every == 0)) return -1;
        if (used_slots == pool) harvest(next_slot);   // reuse the oldest slot
        else ++used_slots;
        const int slot = (int)next_slot;
        ids_share[slot] = 0.0;
        next_slot = (next_slot + 1) % pool;
        return slot;
    };

    int64_t pairs_done = 0;
    FELOG_HIP(hipEventRecord(c.ev0, c.stream));
    if (apply && end > first_mb) {
        // ids of the next groups on the second stream while a group trains on the
        // first (or all in order on the first, for small minibatches)
        hipStream_t ids_s = c.stream;
        if (!one_stream) {
            c.ensure_aux();
            ids_s = c.aux;
            FELOG_HIP(hipEventRecord(c.pipe_ev[0], c.stream));
            FELOG_HIP(hipStreamWaitEvent(ids_s, c.pipe_ev[0], 0));
        }
        struct Mb {
            MinibatchLaunch ml;
            float lr;
            int slot;
        };
        Mb mbs[kIdSets][kIdGroupMax];
        hipEvent_t* ready = c.pipe_ev + 1;               // [ring] ids ready
        hipEvent_t* freed = c.pipe_ev + 1 + kIdSets;     // [ring] buffers free
        const int64_t ngroups = (end - first_mb + G - 1) / G;
        auto issue_ids = [&](int64_t gi) {
            const int ring = (int)(gi % rings);
            const int64_t b0 = first_mb + gi * G;
            const int count = (int)(std::min<int64_t>(end, b0 + G) - b0);
            PrepArgs a = pa;
            int timed_here = 0, first_slot = -1;
            for (int i = 0; i < count; ++i) {
                Mb& x = mbs[ring][i];
                x.lr = frame(b0 + i, ring * G + i, x.ml, a.g[i]);
                gate(ids_s, chunk);
                x.slot = take_slot(b0 + i);
                if (x.slot >= 0 && timed_here++ == 0) first_slot = x.slot;
            }
            IdGroup ig{};
            finish_group(ig, a, ring * G, count);
            // the ring's previous group must be done with its sets
            if (!one_stream && gi >= rings) FELOG_HIP(hipStreamWaitEvent(ids_s, freed[ring], 0));
            hipEvent_t* e = first_slot >= 0 ? &c.timing_pool[kTimingEvents * first_slot] : nullptr;
            if (e) {
                ids_share[first_slot] = (double)timed_here / count;
                FELOG_HIP(hipEventRecord(e[0], ids_s));
            }
            launch_ids(m, a, ig, ids_s);
            if (e) FELOG_HIP(hipEventRecord(e[1], ids_s));
            if (!one_stream) FELOG_HIP(hipEventRecord(ready[ring], ids_s));
        };
        for (int64_t gi = 0; gi < rings - 1 && gi < ngroups; ++gi) issue_ids(gi);
        for (int64_t gi = 0; gi < ngroups; ++gi) {
            const int ring = (int)(gi % rings);
            const int64_t b0 = first_mb + gi * G;
            const int count = (int)(std::min<int64_t>(end, b0 + G) - b0);
            // (into the sets of the group before this one)
            if (gi + rings - 1 < ngroups) issue_ids(gi + rings - 1);
            if (!one_stream) FELOG_HIP(hipStreamWaitEvent(c.stream, ready[ring], 0));
            for (int i = 0; i < count; ++i) {
                const Mb& x = mbs[ring][i];
                hipEvent_t* e = x.slot >= 0 ? &c.timing_pool[kTimingEvents * x.slot] : nullptr;
                FwdArgs f = fa;
                f.lr = x.lr;
                f.npairs = x.ml.npairs;
                launch_train(m, f, x.ml, nullptr, nullptr, c.stream, e ? e + 2 : nullptr);
                pairs_done += x.ml.npairs;
            }
            if (!one_stream) FELOG_HIP(hipEventRecord(freed[ring], c.stream));
        }
    } else if (!apply) {
        // capture: the deltas of one minibatch, by touched-list position, not applied
        const int64_t b = first_mb;
        MinibatchLaunch ml;
        PrepArgs a = pa;
        const float lr = frame(b, 0, ml, a.g[0]);
        IdGroup ig{};
        finish_group(ig, a, 0, 1);
        gate(c.stream, chunk);
        FELOG_HIP(hipMemsetAsync(vin.ptr, 0, vin.bytes, c.stream));
        FELOG_HIP(hipMemsetAsync(vout.ptr, 0, vout.bytes, c.stream));
        launch_ids(m, a, ig, c.stream);
        FwdArgs f = fa;
        f.lr = lr;
        f.npairs = ml.npairs;
        launch_train(m, f, ml, vin.as<float>(), vout.as<float>(), c.stream, nullptr);
        unsigned long long tot[2];
        FELOG_HIP(hipMemcpyAsync(tot, m.row_totals.ptr, sizeof tot, hipMemcpyDeviceToHost,
                                 c.stream));
        c.sync();
        const int64_t ui = (int64_t)tot[0], uo = (int64_t)tot[1];
        FELOG_REQUIRE(rows_in && d_in_host && rows_out && d_out_host,
                      "capture buffers must not be NULL");
        FELOG_REQUIRE(ui <= cap_in && uo <= cap_out,
                      "capture buffers hold %lld / %lld rows, need %lld / %lld",
                      (long long)cap_in, (long long)cap_out, (long long)ui, (long long)uo);
        FELOG_HIP(hipMemcpyAsync(rows_in, m.mb.list_in.ptr, sizeof(int32_t) * ui,
                                 hipMemcpyDeviceToHost, c.stream));
        FELOG_HIP(hipMemcpyAsync(rows_out, m.mb.list_out.ptr, sizeof(int32_t) * uo,
                                 hipMemcpyDeviceToHost, c.stream));
        FELOG_HIP(hipMemcpyAsync(d_in_host, vin.ptr, sizeof(float) * ui * m.dim,
                                 hipMemcpyDeviceToHost, c.stream));
        FELOG_HIP(hipMemcpyAsync(d_out_host, vout.ptr, sizeof(float) * uo * m.dim,
                                 hipMemcpyDeviceToHost, c.stream));
        FELOG_HIP(hipMemsetAsync(m.row_totals.ptr, 0, sizeof(uint64_t) * 3, c.stream));
        c.sync();
        if (n_in) *n_in = ui;
        if (n_out) *n_out = uo;
        pairs_done += ml.npairs;
    }
    hipLaunchKernelGGL(loss_reduce_kernel, dim3(1), dim3(256), 0, c.stream,
                       loss_part.as<double>(), blocks * 4, m.loss_out.as<double>());
    FELOG_HIP(hipGetLastError());
    FELOG_HIP(hipEventRecord(c.ev1, c.stream));
    double loss = 0.0;
    unsigned long long rows[3] = {0, 0, 0};
    FELOG_HIP(hipMemcpyAsync(&loss, m.loss_out.ptr, sizeof loss, hipMemcpyDeviceToHost, c.stream));
    FELOG_HIP(hipMemcpyAsync(rows, m.row_totals.ptr, sizeof rows, hipMemcpyDeviceToHost,
                             c.stream));
    c.sync();
    if (c.aux) FELOG_HIP(hipStreamSynchronize(c.aux));
    // harvest the slots still pending, oldest first
    for (size_t k = 0; k < used_slots; ++k)
        harvest((next_slot + pool - used_slots + k) % pool);
    float ms = 0.0f;
    FELOG_HIP(hipEventElapsedTime(&ms, c.ev0, c.ev1));
    if (stats) {
        stats->minibatches = end - first_mb;
        stats->pairs = pairs_done;
        stats->minibatches_total = sch.B;
        stats->loss = loss;
        stats->ms = ms;
        stats->rows_in = (int64_t)rows[0];
        stats->rows_out = (int64_t)rows[1];
        stats->rows_out_single = (int64_t)rows[2];
        stats->timed_launches = timed;
        stats->ms_forward = ms_fwd;
        stats->ms_apply = ms_apply;
        stats->ms_apply_first = ms_apply_first;
        stats->ms_prep = ms_prep;
        stats->path = 0;
        stats->update_blocks = 0;
        stats->timed_minibatches = timed;
        stats->ms_update = 0.0;
    }
}

}  // namespace felog

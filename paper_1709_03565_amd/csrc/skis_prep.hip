// skis_prep.hip -- preprocessing for the root draw and the first live in-edge:
// validation, per-row prefix products P and q (Eq. gamma_v / Eq. probn), integer root
// weights W, the weight total C, Gamma (exactly rounded) and the alias table (Eq. probu).
// Under the linear threshold model (Sec. 6) the same kernels form per-row running sums of w
// in place of the products (gamma_v is the sum of v's in-weights).
#include <algorithm>

#include "skis_internal.h"

namespace skis {

enum : int { ERR_ROWPTR = 1, ERR_COL = 2, ERR_SELFLOOP = 4, ERR_WEIGHT = 8, ERR_LTSUM = 16 };

// Linear threshold model: a row's weights may sum to at most 1 (Sec. 6); rounding may take the
// sum past 1 by this much, no more.
constexpr double LT_SUM_SLACK = 0x1p-20;

constexpr int32_t SHORT_ROW = 128; // rows up to this length are one lane's, up to LONG_ROW one wave's
constexpr int32_t LONG_ROW = 1024; // rows above this length are taken by a whole workgroup

// An edge's faults but for the self-loop
__device__ __forceinline__ int check_range(int32_t u, float wf, int32_t n)
{
    int bad = 0;
    if (u < 0 || u >= n) bad |= ERR_COL;
    if (!(wf >= 0.0f && wf <= 1.0f)) bad |= ERR_WEIGHT;
    return bad;
}

__device__ __forceinline__ int check_edge(int32_t u, float wf, int64_t v, int32_t n)
{
    return check_range(u, wf, n) | (u == (int32_t)v ? (int)ERR_SELFLOOP : 0);
}

// The products of a row (Eq. gamma_v / Eq. probn) are formed left to right:
// P[e] = P[e-1] * (1 - w[e]) with 1 before the row's first edge, one rounding per product
// (the build disables contraction; __dmul_rn / __dsub_rn pin the operations), and
// q[v] = the row's last P (1 for an empty row).  A row's products are one dependent chain
// of multiplies, so a long row is bound by the latency of that chain, not by bandwidth.

// Rows longer than LONG_ROW (with bounds inside [0, m]), listed first so that k_prep_long can
// run beside k_prep_rows.  Rows above HUGE_ROW (a few dozen on the largest power-law graphs) are
// listed apart, from the list's far end (long_rows[n - 1 - k]), so that k_prep_long takes them
// first: the longest chain then starts with the kernel instead of wherever the list put it.
// Each workgroup takes a contiguous slice of rows, counts its long rows (LDS atomics), reserves
// their places with one global atomic and lists them in a second pass over the slice: one
// atomic per wave on a single address had cost milliseconds at 40M rows.
constexpr int32_t HUGE_ROW = 1 << 18;
// k_prep_long takes the rows above HUGE_ROW longest first while there are at most this many
// (about 75 on the 1.4B-edge power-law graphs), in list order beyond.
constexpr int HUGE_ORDER_MAX = 1024;

__global__ __launch_bounds__(256) void k_find_long(int32_t n, int64_t m, const int32_t *__restrict__ row_ptr,
                                                   int32_t *__restrict__ long_rows, unsigned int *__restrict__ n_long,
                                                   unsigned int *__restrict__ n_huge)
{
    __shared__ unsigned int s_cnt, s_base, s_cur;
    const int t = threadIdx.x, lane = t & 63;
    const int64_t per = (((int64_t)n + gridDim.x - 1) / gridDim.x + 255) / 256 * 256;
    const int64_t v0 = (int64_t)blockIdx.x * per, v1 = v0 + per < (int64_t)n ? v0 + per : (int64_t)n;
    // 0: neither, 1: long, 2: huge
    auto kind = [&](int64_t v) -> int {
        if (v >= v1) return 0;
        const int32_t a = row_ptr[v], b = row_ptr[v + 1];
        if (!(a >= 0 && b >= a && (int64_t)b <= m && b - a > LONG_ROW)) return 0; // (b - a may wrap for b < 0)
        return b - a > HUGE_ROW ? 2 : 1;
    };
    if (t == 0) {
        s_cnt = 0;
        s_cur = 0;
    }
    __syncthreads();
    unsigned int mine = 0;
    for (int64_t v = v0 + t; v < v1; v += 256) mine += kind(v) == 1 ? 1u : 0u;
    if (mine) atomicAdd(&s_cnt, mine);
    __syncthreads();
    if (t == 0) s_base = s_cnt ? atomicAdd(n_long, s_cnt) : 0u;
    __syncthreads();
    const unsigned int base = s_base;
    // every lane of a wave runs the same trip count, so the whole wave takes part in each ballot
    for (int64_t v00 = v0; v00 < v1; v00 += 256) {
        const int64_t v = v00 + t;
        const int k = kind(v);
        if (k == 2) long_rows[(int64_t)n - 1 - atomicAdd(n_huge, 1u)] = (int32_t)v;
        const unsigned long long mask = __ballot(k == 1);
        if (mask) {
            unsigned int off = 0;
            if (lane == 0) off = atomicAdd(&s_cur, (unsigned int)__popcll(mask));
            off = (unsigned int)__builtin_amdgcn_readfirstlane((int)off);
            if (k == 1) long_rows[base + off + (unsigned int)__popcll(mask & ((1ull << lane) - 1ull))] = (int32_t)v;
        }
    }
}

// The coin threshold of an edge from its weight.
__device__ __forceinline__ uint32_t edge_threshold(float w)
{
    return coin_threshold_hi(weight_bits(w));
}

// One 256-thread workgroup per long row (the next row of the list taken with one atomic, so
// that the workgroup holding the longest row takes no other; the rows above HUGE_ROW come
// first), LONG_EDGES in-edges at a time.  A row's products are one dependent chain; on the
// longest row that chain bounds the whole preprocessing, so lane 0 of wave 0 does nothing but
// run it: it reads two fp64 factors per LDS read, the reads of the next LONG_TRIP factors in
// flight while the current ones are multiplied (at most nine LDS operations outstanding, so
// the wait for the current factors never waits on the newer reads: with 32 reads in flight
// the 4-bit LDS counter forced a wait for the newest ones), and keeps, every LONG_BLK
// products, the running product before the block (a checkpoint).  The other three waves, at
// the same time, load chunk c + 1 (coalesced, every load of a thread issued before the first
// is used), validate it, write its coin thresholds and put its factors 1 - w into LDS
// (1 past the row's end: a multiply by 1 leaves the chain as it is), and rebuild the products
// of chunk c - 1: each thread takes a block, starts from its checkpoint and multiplies the
// same factors in the same order, so every product is the chain's own, and writes them out.
// Lane 0 thus issues no store and one LDS read per two factors: a single lane's LDS and global
// stores had made the chain up to four times slower than its multiplies.  Three factor buffers
// rotate (chained, fed, rebuilt).  LT: the terms are w (0 past the row's end) and the chain
// adds.
constexpr int LONG_EDGES = 3072;               // 77 KB of LDS: nine waves of k_prep_rows beside it
constexpr int LONG_TRIP = 16;                  // factors per batch of the chain's LDS reads
constexpr int LONG_PAD = 64;                   // read-ahead past a chunk
constexpr int LONG_BLK = 64;                   // products per checkpoint
constexpr int LONG_FEED = 192;                 // threads of waves 1-3
constexpr int LONG_PER = (LONG_EDGES + LONG_FEED - 1) / LONG_FEED; // edges a feeding thread loads
static_assert(LONG_EDGES % LONG_BLK == 0 && LONG_BLK == 4 * LONG_TRIP, "checkpoints fall on batch quads");
static_assert(LONG_PAD >= LONG_TRIP, "the chain reads one batch past a block");
static_assert(LONG_EDGES / LONG_BLK <= LONG_FEED, "one rebuilt block per feeding thread");

static_assert(LONG_EDGES >= HUGE_ORDER_MAX, "the huge rows' order shares the factors' LDS");

template <bool LT> __device__ __forceinline__ double chain_op(double x, double f)
{
    return LT ? __dadd_rn(x, f) : __dmul_rn(x, f);
}

// Lane 0's chain over one chunk of len factors F (identity terms past len up to the next
// multiple of LONG_BLK plus LONG_TRIP): the checkpoints into CK, the running value returned.
template <bool LT> __device__ __forceinline__ double chain_chunk(const double *F, double *CK, int len, double run)
{
    const double2 *F2 = reinterpret_cast<const double2 *>(F);
    double2 xa[LONG_TRIP / 2], xb[LONG_TRIP / 2];
#pragma unroll
    for (int k = 0; k < LONG_TRIP / 2; ++k) xa[k] = F2[k];
    // The empty asm statements pin the order reads -> multiplies -> reads: each takes the
    // running value as an operand (so the multiplies before it stay before it) and orders the
    // LDS reads around it; without them the reads of a batch drift in among the other batch's
    // multiplies and the count of LDS operations in flight passes 15 again.
    for (int i0 = 0; i0 < len; i0 += LONG_BLK) {
        CK[i0 / LONG_BLK] = run; // the product before element i0
        const double2 *B = F2 + i0 / 2;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int k = 0; k < LONG_TRIP / 2; ++k) xb[k] = B[(2 * h + 1) * (LONG_TRIP / 2) + k];
            asm volatile("" : "+v"(run)::"memory");
#pragma unroll
            for (int k = 0; k < LONG_TRIP / 2; ++k) run = chain_op<LT>(chain_op<LT>(run, xa[k].x), xa[k].y);
            asm volatile("" : "+v"(run)::"memory");
#pragma unroll
            for (int k = 0; k < LONG_TRIP / 2; ++k) xa[k] = B[(2 * h + 2) * (LONG_TRIP / 2) + k];
            asm volatile("" : "+v"(run)::"memory");
#pragma unroll
            for (int k = 0; k < LONG_TRIP / 2; ++k) run = chain_op<LT>(chain_op<LT>(run, xb[k].x), xb[k].y);
            asm volatile("" : "+v"(run)::"memory");
        }
    }
    return run;
}

// Lane 0's chain over a chunk of len equal terms w (LT).  While the sum stays between two powers of
// two, adding w moves it by the same multiple of its last place each time (w rounded to it, unless w
// lies halfway between two): a block of 64 then takes one addition and a check.  1M nodes, 20M edges of
// equal row weights: k_prep_long 1.17 -> 0.70 ms.
__device__ __forceinline__ double equal_chunk(double *CK, int len, double run, double w)
{
    for (int i0 = 0; i0 < len; i0 += LONG_BLK) {
        CK[i0 / LONG_BLK] = run;
        const int cnt = min(LONG_BLK, len - i0);
        const double inc = __dsub_rn(__dadd_rn(run, w), run);
        const double end = __dadd_rn(run, __dmul_rn((double)cnt, inc));
        const long long ex = __double_as_longlong(run) >> 52, half = ex - 53; // half a last place is 2^(half - 1023)
        const bool tie = half <= 0 || fabs(__dsub_rn(w, inc)) == __longlong_as_double(half << 52);
        if (!tie && ex == __double_as_longlong(end) >> 52) {
            run = end;
        } else {
            for (int k = 0; k < cnt; ++k) run = __dadd_rn(run, w);
        }
    }
    return run;
}

// A feeding thread's rebuild of block blk of a chunk (len factors F, cnt = min(LONG_BLK,
// len - blk * LONG_BLK) > 0 of them in the block) from its checkpoint x into dst.
template <bool LT>
__device__ __forceinline__ void rebuild_block(const double *F, int blk, int cnt, double x, double *__restrict__ dst)
{
    // two halves of 32 factors (fewer registers: k_prep_rows's waves share the SIMDs)
    const double2 *F2 = reinterpret_cast<const double2 *>(F + blk * LONG_BLK);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        double2 f[LONG_BLK / 4];
#pragma unroll
        for (int k = 0; k < LONG_BLK / 4; ++k) f[k] = F2[h * (LONG_BLK / 4) + k];
        double *d = dst + h * (LONG_BLK / 2);
        const int c = cnt - h * (LONG_BLK / 2);
        if (c >= LONG_BLK / 2) {
#pragma unroll
            for (int k = 0; k < LONG_BLK / 4; ++k) {
                x = chain_op<LT>(x, f[k].x);
                d[2 * k] = x;
                x = chain_op<LT>(x, f[k].y);
                d[2 * k + 1] = x;
            }
        } else {
#pragma unroll
            for (int k = 0; k < LONG_BLK / 4; ++k) {
                if (2 * k >= c) break;
                x = chain_op<LT>(x, f[k].x);
                d[2 * k] = x;
                if (2 * k + 1 >= c) break;
                x = chain_op<LT>(x, f[k].y);
                d[2 * k + 1] = x;
            }
        }
    }
}

// Tails.  Where coins are frequent the product underflows within some ten thousand edges and stays at
// a denormal of a few units (fl(x f) = x for every later factor f) or at zero, while the row may
// have millions more.  Once a whole chunk has left such a value as it was, k_prep_long gives the
// rest of the row to k_prep_tails, pieces of which all CUs take: each edge's factor is checked to
// leave the value as it is, and if one does not (a larger weight further on) the host has the long
// rows done again without tails.  4M nodes and 70M edges of trivalency weights: the long rows took
// 5.0 ms, the longest chain's time; now 0.33 ms and 0.06 ms for the tails.
struct TailPiece {
    int32_t e0, e1; // edges
    int32_t v;      // row
    int32_t units;  // the product in units of 2^-1074
};
// Values taken for a tail: weights of 2^-20 and more bring a long product below.
constexpr int TAIL_UNITS = 1 << 20;
constexpr int TAIL_PIECE = 16384;
// A row with pieces has more than 2 LONG_EDGES edges, and the rows of a valid graph are disjoint.
static inline int64_t tail_pieces_max(int64_t m) { return m / TAIL_PIECE + m / (2 * LONG_EDGES) + 1; }

__global__ __launch_bounds__(256) void k_prep_tails(int32_t n, const int32_t *__restrict__ row_ptr,
                                                    const int32_t *__restrict__ col, const float *__restrict__ w,
                                                    uint32_t *__restrict__ th, double *__restrict__ P, int *err,
                                                    int *mixed, const TailPiece *__restrict__ pieces,
                                                    const unsigned int *__restrict__ n_pieces, unsigned int max_pieces,
                                                    int64_t m, int *__restrict__ redo)
{
    const unsigned int np = *n_pieces;
    if (np > max_pieces) return; // only where rows overlap, which k_prep_rows reports
    int bad = 0;
    bool same = true, moved = false;
    for (unsigned int i = blockIdx.x; i < np; i += gridDim.x) {
        const TailPiece p = pieces[i];
        if (p.e0 < 0 || (int64_t)p.e1 > m || p.v < 0 || p.v >= n) continue; // likewise
        const double x = __longlong_as_double((long long)p.units);
        const uint32_t th0 = th ? edge_threshold(w[row_ptr[p.v]]) : 0u;
        for (int32_t e0 = p.e0 + (int32_t)threadIdx.x; e0 < p.e1; e0 += 1024) { // below 2^31 - 1024: see the host
            int32_t u[4];
            float wf[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int32_t e = min(e0 + k * 256, p.e1 - 1);
                u[k] = col[e];
                wf[k] = w[e];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int32_t e = e0 + k * 256;
                if (e >= p.e1) break;
                bad |= check_edge(u[k], wf[k], p.v, n);
                moved = moved || __dmul_rn(x, __dsub_rn(1.0, (double)wf[k])) != x;
                if (th) {
                    const uint32_t tx = edge_threshold(wf[k]);
                    same = same && tx == th0;
                    th[e] = tx;
                }
                P[e] = x;
            }
        }
    }
    if (bad) atomicOr(err, bad);
    if (!same && !*mixed) *mixed = 1;
    if (moved && !*redo) *redo = 1;
}

// Edge: uint32_t where the last chunk of a row may end past 2^31 (see the host), else int32_t, with which
// the longest chains are some 3 % faster (8.5M edges, 436 thousand nodes: 785 us for 818).
template <bool LT, typename Edge>
__global__ __launch_bounds__(256) void k_prep_long(int32_t n, const int32_t *__restrict__ row_ptr,
                                                   const int32_t *__restrict__ col, const float *__restrict__ w,
                                                   uint32_t *__restrict__ th,
                                                   double *__restrict__ P, double *__restrict__ q, int *err,
                                                   int *mixed, const int32_t *__restrict__ long_rows,
                                                   const unsigned int *__restrict__ n_long,
                                                   const unsigned int *__restrict__ n_huge,
                                                   unsigned int *__restrict__ next_row, TailPiece *__restrict__ pieces,
                                                   unsigned int *__restrict__ n_pieces, unsigned int max_pieces)
{
    __shared__ __align__(16) double s_f[3][LONG_EDGES + LONG_PAD]; // factors of three chunks (+ read-ahead pad)
    __shared__ double s_ck[2][LONG_EDGES / LONG_BLK];               // checkpoints of two chunks
    int32_t *const s_hrow = reinterpret_cast<int32_t *>(s_f[0]), *const s_hlen = s_hrow + HUGE_ORDER_MAX; // before the row
    __shared__ unsigned int s_r, s_piece;
    __shared__ int32_t s_pick;
    __shared__ double s_run[2]; // the chain after each of the last two chunks
    __shared__ unsigned int s_diff[3]; // LT: the last chunk of each buffer whose terms are not all the row's first
    [[maybe_unused]] unsigned int gen = 1; // number of the row's first chunk
    if (threadIdx.x < 3) s_diff[threadIdx.x] = 0u;
    const int t = threadIdx.x;
    const unsigned int nh = *n_huge, cnt = nh + *n_long;
    const double ident = LT ? 0.0 : 1.0;
    for (int i = t; i < LONG_PAD; i += 256) s_f[0][LONG_EDGES + i] = s_f[1][LONG_EDGES + i] = s_f[2][LONG_EDGES + i] = ident;
    // waves 1-3 put chunk c0 of row v (edges [c0, b)) into buffer `buf`; returns their flags.
    // Every load and store is unconditional, at the edge clamped to the row's last one (a
    // clamped store writes the value that edge's own thread writes), so the compiler's wait
    // counts stay exact: with loads and stores under branches it waited for every store.
    uint32_t th0 = 0u; // the row's first threshold
    bool same = true;
    [[maybe_unused]] float w0 = 0.0f; // the row's first weight
    auto feed = [&](int32_t v, int32_t c0, int32_t b, int buf, unsigned int num) -> int {
        [[maybe_unused]] bool diff = false;
        int32_t u[LONG_PER];
        float wf[LONG_PER];
#pragma unroll
        for (int k = 0; k < LONG_PER; ++k) {
            const Edge ec = min((Edge)c0 + t - 64 + k * LONG_FEED, (Edge)b - 1);
            u[k] = col[ec];
            wf[k] = w[ec];
        }
        int bad = 0;
#pragma unroll
        for (int k = 0; k < LONG_PER; ++k) {
            const int i = t - 64 + k * LONG_FEED;
            const Edge e = (Edge)c0 + i, ec = min(e, (Edge)b - 1);
            const float x = wf[k];
            bad |= check_edge(u[k], x, v, n);
            if (LT) diff = diff || x != w0; // a clamped one repeats the row's last
            if (th) {
                const uint32_t tx = edge_threshold(x);
                same = same && tx == th0;
                th[ec] = tx;
            }
            const double f = e < (Edge)b ? (LT ? (double)x : __dsub_rn(1.0, (double)x)) : ident;
            if (k + 1 < LONG_PER || i < LONG_EDGES) s_f[buf][i] = f;
        }
        if (LT && diff) s_diff[buf] = num;
        return bad;
    };
    for (;;) {
        if (t == 0) s_r = atomicAdd(next_row, 1u);
        __syncthreads();
        const unsigned int r = s_r;
        if (r >= cnt) break;
        int32_t v;
        if (r >= nh) {
            v = long_rows[r - nh];
        } else if (nh > (unsigned int)HUGE_ORDER_MAX) {
            v = long_rows[(int64_t)n - 1 - r];
        } else {
            // place r of the huge rows by length, longest first (equal lengths by row id): the
            // row that exactly r rows go before
            for (unsigned int j = t; j < nh; j += 256) {
                const int32_t x = long_rows[(int64_t)n - 1 - j];
                s_hrow[j] = x;
                s_hlen[j] = row_ptr[x + 1] - row_ptr[x];
            }
            __syncthreads();
            for (unsigned int j = t; j < nh; j += 256) {
                const int32_t lj = s_hlen[j], vj = s_hrow[j];
                unsigned int rank = 0;
                for (unsigned int i = 0; i < nh; ++i)
                    rank += (s_hlen[i] > lj || (s_hlen[i] == lj && s_hrow[i] < vj)) ? 1u : 0u;
                if (rank == r) s_pick = vj;
            }
            __syncthreads();
            v = s_pick;
        }
        const int32_t a = row_ptr[v], b = row_ptr[v + 1];
        int nchunks = (int)(((Edge)(b - a) + LONG_EDGES - 1) / LONG_EDGES);
        int bad = 0;
        if (th) th0 = edge_threshold(w[a]);
        if (LT) w0 = w[a];
        if (t >= 64) bad |= feed(v, a, b, 0, gen);
        __syncthreads();
        double run = ident; // lane 0's chain
        [[maybe_unused]] long long before = 0; // the product before the chunk just done
        for (int c = 0; c <= nchunks; ++c) {
            if (t == 0) {
                if (c < nchunks) {
                    const int len = min(b - (a + c * LONG_EDGES), LONG_EDGES);
                    if (LT && s_diff[c % 3] != gen + (unsigned int)c)
                        run = equal_chunk(s_ck[c & 1], len, run, (double)w0);
                    else
                        run = chain_chunk<LT>(s_f[c % 3], s_ck[c & 1], len, run);
                    if (!LT) s_run[c & 1] = run;
                }
            } else if (t >= 64) {
                if (c + 1 < nchunks) bad |= feed(v, a + (c + 1) * LONG_EDGES, b, (c + 1) % 3, gen + (unsigned int)c + 1u);
                if (c >= 1) { // rebuild chunk c - 1 from its checkpoints, one block per thread
                    const int32_t cp0 = a + (c - 1) * LONG_EDGES;
                    const int lenp = min(b - cp0, LONG_EDGES);
                    const int blk = t - 64;
                    if (blk * LONG_BLK < lenp)
                        rebuild_block<LT>(s_f[(c - 1) % 3], blk, min(LONG_BLK, lenp - blk * LONG_BLK),
                                          s_ck[(c - 1) & 1][blk], P + cp0 + blk * LONG_BLK);
                }
            }
            __syncthreads();
            if constexpr (!LT) {
                // the same decision in every thread: lane 0 writes this place again after the next barrier
                if (!pieces || c + 2 >= nchunks) continue;
                const long long units = __double_as_longlong(s_run[c & 1]);
                if (units < TAIL_UNITS && c > 0 && units == before) {
                    const int32_t e0 = a + (c + 1) * LONG_EDGES;
                    const int np = (b - e0 + TAIL_PIECE - 1) / TAIL_PIECE;
                    if (t == 0) s_piece = atomicAdd(n_pieces, (unsigned int)np);
                    __syncthreads();
                    const unsigned int p0 = s_piece;
                    if ((uint64_t)p0 + (unsigned int)np <= max_pieces) {
                        for (int i = t; i < np; i += 256) {
                            const int32_t x = e0 + i * TAIL_PIECE;
                            pieces[p0 + i] = {x, b - x > TAIL_PIECE ? x + TAIL_PIECE : b, v, (int32_t)units};
                        }
                        nchunks = c + 1; // what is left here: this chunk's products
                    }
                }
                before = units;
            }
        }
        if (t == 0) {
            if (LT) {
                if (run > 1.0 + LT_SUM_SLACK) bad |= ERR_LTSUM;
                q[v] = lt_q(run);
            } else {
                q[v] = run;
            }
        }
        if (LT) gen += (unsigned int)nchunks;
        if (bad) atomicOr(err, bad);
        if (!same && !*mixed) *mixed = 1;
        same = true;
        __syncthreads();
    }
}

// The rows up to LONG_ROW edges: validation, coin thresholds, P and q; the row records of all rows,
// the long ones too.  A wave takes 64 rows at a time (`per` such units an atomic).  The edges of the
// rows up to SHORT_ROW go into LDS, as many rows as fit, coalesced; each lane forms its row's
// products there in place, left to right, and they go out coalesced.  The rows between SHORT_ROW
// and LONG_ROW follow one by one, by the whole wave as in k_prep_long.  A thread that read its own
// row from memory had kept a wave's loads on 64 lines and waited a memory latency for every eight
// edges, and a 256-thread workgroup a row left most of the device idle on rows of some hundred
// edges: 4M nodes and 70M edges of trivalency weights took 1.36 ms (and the rows of 257 to 1024
// edges another 0.5 ms in k_prep_long), now 0.56 ms; the bytes alone take 0.25 ms.
// The units are taken as the waves get to them, since waves that find no room beside the long rows
// start late.  LT: running sums S in P (S[e] = S[e-1] + w[e], 0 before the row's first edge) and
// q = 1 - the row's sum.  th and rows are null when no coin will be drawn (LT, the preprocessing
// alone).  *mixed: set when some row's edges differ in their threshold.
constexpr int ROWS_CAP = LONG_ROW; // edges in LDS: 8.6 KB with the pad and the checkpoints
constexpr int ROWS_FLIGHT = 6;     // edges a lane loads at a time

template <bool LT>
__global__ __launch_bounds__(64) void k_prep_rows(int32_t n, int64_t m, const int32_t *__restrict__ row_ptr,
                                                  const int32_t *__restrict__ col, const float *__restrict__ w,
                                                  int32_t *__restrict__ rp_copy, uint2 *__restrict__ rows,
                                                  uint32_t *__restrict__ th, double *__restrict__ P,
                                                  double *__restrict__ q, int *err, int *mixed,
                                                  unsigned int *__restrict__ next_unit, unsigned int per)
{
    __shared__ __align__(16) double s_f[ROWS_CAP + LONG_PAD]; // a short edge's (col, w), then its product; factors
    __shared__ double s_ck[ROWS_CAP / LONG_BLK];
    const int lane = threadIdx.x;
    const double ident = LT ? 0.0 : 1.0;
    const unsigned int units = (unsigned int)(((int64_t)n + 63) / 64);
    int bad = 0;
    bool same = true;
    for (unsigned int g1 = 0, g = 0;; ++g) {
        if (g == g1) {
            unsigned int x = 0;
            if (lane == 0) x = atomicAdd(next_unit, per);
            g = (unsigned int)__builtin_amdgcn_readfirstlane((int)x);
            if (g >= units) break;
            g1 = min(g + per, units);
        }
        const int64_t v = (int64_t)g * 64 + lane;
        int32_t a = 0, b = 0;
        bool ok = false;
        uint32_t th0 = 0u;
        if (v < n) {
            a = row_ptr[v];
            b = row_ptr[v + 1];
            rp_copy[v] = a;
            if (v == n - 1) {
                rp_copy[n] = b;
                if (rows) rows[n] = make_uint2((uint32_t)b, 0u);
                if ((int64_t)b != m) bad |= ERR_ROWPTR;
            }
            if (v == 0 && a != 0) bad |= ERR_ROWPTR;
            ok = a >= 0 && (int64_t)b <= m && a <= b;
            if (!ok) {
                bad |= ERR_ROWPTR;
                q[v] = 1.0;
            } else if (rows && b - a > SHORT_ROW) {
                th0 = edge_threshold(w[a]);
            }
        }
        const int32_t len = b - a;
        const bool is_short = ok && len <= SHORT_ROW;
        double run = ident;
        // the short rows, by as many lanes as fit at a time
        for (unsigned long long todo = __ballot(is_short && len > 0); todo;) {
            const bool cand = (todo >> lane) & 1ull;
            int32_t off = cand ? len : 0; // inclusive sums of the candidates' lengths
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int32_t y = __shfl_up(off, d, 64);
                if (lane >= d) off += y;
            }
            const bool in = cand && off <= ROWS_CAP; // the first ones: the sums ascend
            off -= cand ? len : 0;
            const unsigned long long now = __ballot(in);
            todo &= ~now;
            // their edges, in runs of neighbouring rows (empty ones between them do not count)
            const unsigned long long gap = __ballot(!(in || (is_short && len == 0)));
            auto runs = [&](auto &&body) {
                for (unsigned long long left = now; left;) {
                    const int l0 = __ffsll(left) - 1;
                    const unsigned long long after = gap & ~((1ull << l0) - 1ull);
                    const unsigned long long mine = after ? left & ((1ull << (__ffsll(after) - 1)) - 1ull) : left;
                    const int l1 = 63 - __clzll(mine);
                    left &= ~mine;
                    const int32_t e0 = __builtin_amdgcn_readlane(a, l0);
                    body(e0, __builtin_amdgcn_readlane(b, l1) - e0, __builtin_amdgcn_readlane(off, l0));
                }
            };
            runs([&](int32_t e0, int32_t cnt, int32_t o) {
                for (int i0 = lane; i0 - lane < cnt; i0 += 64 * ROWS_FLIGHT) {
                    int32_t u[ROWS_FLIGHT];
                    float wf[ROWS_FLIGHT];
#pragma unroll
                    for (int k = 0; k < ROWS_FLIGHT; ++k) { // clamped, so unconditional
                        const int i = min(i0 + k * 64, cnt - 1);
                        u[k] = col[e0 + i];
                        wf[k] = w[e0 + i];
                    }
#pragma unroll
                    for (int k = 0; k < ROWS_FLIGHT; ++k) {
                        const int i = min(i0 + k * 64, cnt - 1);
                        s_f[o + i] = __longlong_as_double((long long)((uint64_t)(uint32_t)u[k] << 32 | __float_as_uint(wf[k])));
                        if (th) th[e0 + i] = edge_threshold(wf[k]);
                        bad |= check_range(u[k], wf[k], n); // the self-loops are seen below
                    }
                }
            });
            __syncthreads();
            if (in) {
                const uint32_t w0 = (uint32_t)__double_as_longlong(s_f[off]);
                if (th) th0 = edge_threshold(__uint_as_float(w0));
                for (int i0 = 0; i0 < len; i0 += 4) {
                    uint64_t x[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) x[k] = (uint64_t)__double_as_longlong(s_f[off + min(i0 + k, len - 1)]);
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        if (i0 + k >= len) break;
                        const uint32_t wb = (uint32_t)x[k];
                        const float wf = __uint_as_float(wb);
                        if ((int32_t)(x[k] >> 32) == (int32_t)v) bad |= ERR_SELFLOOP;
                        if (th && same && wb != w0) same = edge_threshold(wf) == th0;
                        run = chain_op<LT>(run, LT ? (double)wf : __dsub_rn(1.0, (double)wf));
                        s_f[off + i0 + k] = run;
                    }
                }
            }
            __syncthreads();
            runs([&](int32_t e0, int32_t cnt, int32_t o) {
                for (int i = lane; i < cnt; i += 64) P[e0 + i] = s_f[o + i];
            });
            __syncthreads();
        }
        // the rows of one wave
        for (unsigned long long todo = __ballot(ok && !is_short && len <= LONG_ROW); todo; todo &= todo - 1ull) {
            const int l = __ffsll(todo) - 1;
            const int32_t e0 = __builtin_amdgcn_readlane(a, l), cnt = __builtin_amdgcn_readlane(len, l);
            const uint32_t t0 = (uint32_t)__builtin_amdgcn_readlane((int)th0, l);
            const int32_t row = (int32_t)((int64_t)g * 64 + l);
            const int end = (cnt + LONG_BLK - 1) / LONG_BLK * LONG_BLK + LONG_TRIP;
            for (int i0 = lane; i0 - lane < end; i0 += 64 * ROWS_FLIGHT) {
                int32_t u[ROWS_FLIGHT];
                float wf[ROWS_FLIGHT];
#pragma unroll
                for (int k = 0; k < ROWS_FLIGHT; ++k) {
                    const int i = min(i0 + k * 64, cnt - 1);
                    u[k] = col[e0 + i];
                    wf[k] = w[e0 + i];
                }
#pragma unroll
                for (int k = 0; k < ROWS_FLIGHT; ++k) {
                    const int i = i0 + k * 64, ic = min(i, cnt - 1);
                    bad |= check_edge(u[k], wf[k], row, n);
                    if (th) {
                        const uint32_t x = edge_threshold(wf[k]);
                        same = same && x == t0;
                        th[e0 + ic] = x;
                    }
                    const double f = i < cnt ? (LT ? (double)wf[k] : __dsub_rn(1.0, (double)wf[k])) : ident;
                    if (i < end) s_f[i] = f;
                }
            }
            __syncthreads();
            double r = ident;
            if (lane == 0) r = chain_chunk<LT>(s_f, s_ck, cnt, r);
            __syncthreads();
            if (lane * LONG_BLK < cnt)
                rebuild_block<LT>(s_f, lane, min(LONG_BLK, cnt - lane * LONG_BLK), s_ck[lane], P + e0 + lane * LONG_BLK);
            r = __longlong_as_double((long long)readlane64((unsigned long long)__double_as_longlong(r), 0));
            if (lane == l) run = r;
            __syncthreads();
        }
        if (ok) {
            if (len <= LONG_ROW) {
                if (LT) {
                    if (run > 1.0 + LT_SUM_SLACK) bad |= ERR_LTSUM;
                    q[v] = lt_q(run);
                } else {
                    q[v] = run;
                }
            }
            if (rows) rows[v] = make_uint2((uint32_t)a, th0);
        }
    }
    if (bad) atomicOr(err, bad);
    if (!same && !*mixed) *mixed = 1; // every writer writes 1
}

// Sum of hi:lo over the wave, two 64-bit halves with carry (every lane gets it).
__device__ __forceinline__ void wave_sum128(uint64_t &lo, uint64_t &hi)
{
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        const uint64_t olo = __shfl_xor(lo, d, 64), ohi = __shfl_xor(hi, d, 64);
        const uint64_t nlo = lo + olo;
        hi = hi + ohi + (nlo < lo ? 1ull : 0ull);
        lo = nlo;
    }
}

// W_v = ceil(gamma_v * 2^s) and k_v = gamma_v * 2^53 (an integer: gamma_v = 1 - q_v lies on
// the grid 2^-53 Z because q_v is in [0,1]).  Per-block partial sums of W (u64) and k (u128).
__global__ __launch_bounds__(256) void k_weights(int32_t n, int s_shift, const double *__restrict__ q,
                                                 uint64_t *__restrict__ W, uint64_t *__restrict__ partW,
                                                 u128 *__restrict__ partK)
{
    __shared__ uint64_t shW[4];
    __shared__ uint64_t shKlo[4], shKhi[4];
    uint64_t accW = 0;
    u128 accK = 0;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const double g = __dsub_rn(1.0, q[v]);
        const uint64_t k = (uint64_t)ldexp(g, 53);
        uint64_t Wv;
        if (k == 0) {
            Wv = 0;
        } else if (s_shift >= 53) {
            Wv = k << (s_shift - 53);
        } else {
            const int d = 53 - s_shift;
            Wv = (k + ((1ull << d) - 1)) >> d; // ceil(k / 2^d)
        }
        W[v] = Wv;
        accW += Wv;
        accK += (u128)k;
    }
    // block reduction (4 waves)
    accW = wave_sum(accW);
    uint64_t lo = (uint64_t)accK, hi = (uint64_t)(accK >> 64);
    wave_sum128(lo, hi);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) {
        shW[wid] = accW;
        shKlo[wid] = lo;
        shKhi[wid] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t sw = 0;
        u128 sk = 0;
        for (int i = 0; i < (int)(blockDim.x / 64); ++i) {
            sw += shW[i];
            sk += ((u128)shKhi[i] << 64) | shKlo[i];
        }
        partW[blockIdx.x] = sw;
        partK[blockIdx.x] = sk;
    }
}

struct PrepScalars {
    uint64_t C;
    double Gamma;
};

// One wave adds the partial sums (integers: the order does not matter).  A single lane's loop over
// the 4096 partials of a large graph, one memory latency each, had taken 0.4 ms.
__global__ __launch_bounds__(64) void k_weights_final(int nb, const uint64_t *__restrict__ partW,
                                                      const u128 *__restrict__ partK, PrepScalars *out)
{
    uint64_t C = 0;
    u128 K = 0;
    for (int i = threadIdx.x; i < nb; i += 64) {
        C += partW[i];
        K += partK[i];
    }
    C = wave_sum(C);
    uint64_t lo = (uint64_t)K, hi = (uint64_t)(K >> 64);
    wave_sum128(lo, hi);
    if (threadIdx.x == 0) {
        out->C = C;
        out->Gamma = ldexp(u128_to_double(((u128)hi << 64) | lo), -53);
    }
}

// ---- alias table: the sequential sweep expressed by prefix sums -------------------------
// Light nodes (a = n*W <= C) in id order have deficits d = C - a, heavy nodes surpluses
// s = a - C.  With inclusive prefix sums D (over lights) and S (over heavies):
//   light i:  thr = a, alias = heavy j with j = min{ j : S_j > D_{i-1} } (itself if none);
//   heavy j:  thr = C + S_j - D_k with k = min{ k : D_k >= S_j }, alias = heavy j+1 (itself
//             for the last heavy, whose thr is then C).
// This reproduces the sweep exactly: the current heavy's remainder after light k is
// C + S_j - D_k, and heavy j turns into a bucket at the first light that brings it to <= C.
__global__ __launch_bounds__(256) void k_alias_flags(int32_t n, const uint64_t *__restrict__ W, uint64_t C,
                                                     uint32_t *__restrict__ light)
{
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
        light[v] = ((uint64_t)n * W[v] <= C) ? 1u : 0u;
}

__global__ __launch_bounds__(256) void k_alias_split(int32_t n, const uint64_t *__restrict__ W, uint64_t C,
                                                     const uint32_t *__restrict__ light,
                                                     const uint32_t *__restrict__ lrank, int32_t *__restrict__ lid,
                                                     int32_t *__restrict__ hid, u128 *__restrict__ dval,
                                                     u128 *__restrict__ sval)
{
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t a = (uint64_t)n * W[v];
        const uint32_t lr = lrank[v];
        if (light[v]) {
            lid[lr] = (int32_t)v;
            dval[lr] = (u128)(C - a);
        } else {
            const uint32_t hr = (uint32_t)v - lr;
            hid[hr] = (int32_t)v;
            sval[hr] = (u128)(a - C);
        }
    }
}

__global__ __launch_bounds__(256) void k_add_inplace(int64_t len, u128 *__restrict__ excl, const u128 *__restrict__ val)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < len; i += (int64_t)gridDim.x * blockDim.x)
        excl[i] += val[i];
}

__global__ __launch_bounds__(256) void k_alias_light(int32_t n, int64_t L, int64_t H, const uint64_t *__restrict__ W,
                                                     const int32_t *__restrict__ lid, const int32_t *__restrict__ hid,
                                                     const u128 *__restrict__ dval, const u128 *__restrict__ Dinc,
                                                     const u128 *__restrict__ Sinc, AliasEntry *__restrict__ table)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < L; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = lid[i];
        const u128 dex = Dinc[i] - dval[i];
        int64_t lo = 0, hi = H; // first j with Sinc[j] > dex
        while (lo < hi) {
            int64_t mid = (lo + hi) >> 1;
            if (Sinc[mid] > dex) hi = mid; else lo = mid + 1;
        }
        AliasEntry e;
        e.thr = (uint64_t)n * W[v];
        e.alias = lo < H ? hid[lo] : v;
        e.pad = 0;
        table[v] = e;
    }
}

__global__ __launch_bounds__(256) void k_alias_heavy(int64_t L, int64_t H, uint64_t C, const int32_t *__restrict__ hid,
                                                     const u128 *__restrict__ Dinc, const u128 *__restrict__ Sinc,
                                                     AliasEntry *__restrict__ table)
{
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < H; j += (int64_t)gridDim.x * blockDim.x) {
        const u128 Sj = Sinc[j];
        int64_t lo = 0, hi = L; // first k with Dinc[k] >= Sj (exists: Sinc[H-1] == Dinc[L-1])
        while (lo < hi) {
            int64_t mid = (lo + hi) >> 1;
            if (Dinc[mid] >= Sj) hi = mid; else lo = mid + 1;
        }
        const int64_t k = lo < L ? lo : L - 1;
        AliasEntry e;
        e.thr = (uint64_t)((u128)C + Sj - Dinc[k]);
        e.alias = j + 1 < H ? hid[j + 1] : hid[j];
        e.pad = 0;
        table[hid[j]] = e;
    }
}

static unsigned grid_for(int64_t items, int block = 256)
{
    int64_t g = (items + block - 1) / block;
    int64_t cap = (int64_t)device_cu_count() * 16;
    if (g > cap) g = cap;
    return (unsigned)(g > 0 ? g : 1);
}

// Workgroups a CU: one of the long rows' (77 KB of LDS) and at most this many of the other rows'
// (9 KB), few enough that both find room whichever kernel the device starts first (filling every
// CU, k_prep_rows had held the longest chain back by about 19 ms at 40M rows).  Measured against two
// with chunks of 2048 edges beside ten, and one of 4096 beside seven: 4M rows alone 1.09, 1.06 and
// 1.14 ms, 1M rows in a build 1.40-1.46, 1.47-1.64 and 1.41 ms, 40M rows 31.4, 32.6 and 32.5 ms.
constexpr int LONG_PER_CU = 1, ROWS_PER_CU = 9;

static int root_shift(int32_t n)
{
    int L = 0;
    while ((1ll << L) < (int64_t)(n < 2 ? 2 : n)) ++L;
    return 62 - L;
}

// The alias table's columns into the caller's arrays (either may be null): the strided copies had
// taken 234 us for 4M nodes.
__global__ __launch_bounds__(256) void k_alias_columns(int32_t n, const AliasEntry *__restrict__ table,
                                                       uint64_t *__restrict__ thr, int32_t *__restrict__ alias)
{
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < n; v += (int64_t)gridDim.x * 256) {
        const AliasEntry e = table[v];
        if (thr) thr[v] = e.thr;
        if (alias) alias[v] = e.alias;
    }
}

void alias_columns(int32_t n, const AliasEntry *table, uint64_t *thr, int32_t *alias, hipStream_t s)
{
    if (!thr && !alias) return;
    hipLaunchKernelGGL(k_alias_columns, dim3(grid_for(n)), dim3(256), 0, s, n, table, thr, alias);
    SKIS_HIP_TRY(hipGetLastError());
}

void preprocess(Arena &arena, int32_t n, int64_t m, const int32_t *row_ptr, const int32_t *col, const float *w,
                bool build_alias, Prep &out, hipStream_t s, int model, bool coins, double *P_out)
{
    if (model != MODEL_IC && model != MODEL_LT) throw Error{SKIS_EINVAL, "model must be 0 (IC) or 1 (LT)"};
    out.model = model;
    const int lt = model == MODEL_LT ? 1 : 0;
    out.row_ptr.alloc(arena, (size_t)n + 1);
    out.col = col;
    out.w = w;
    if (lt) coins = false;
    const size_t m_quad = (size_t)((m + 3) & ~(int64_t)3);
    if (coins) {
        out.th.alloc(arena, m_quad > 0 ? m_quad : 4);
        out.rows.alloc(arena, (size_t)n + 1);
    }
    // the products go straight into the caller's buffer where the paired stores allow it
    double *P = P_out && (reinterpret_cast<uintptr_t>(P_out) & 15) == 0 ? P_out : nullptr;
    if (!P) {
        out.P.alloc(arena, (size_t)(m > 0 ? m : 1));
        P = out.P.ptr;
    }
    out.q.alloc(arena, (size_t)n);
    out.W.alloc(arena, (size_t)n);
    // every threshold below m is written by the row kernels; the quad padding past m is clear
    if (out.th.count > (size_t)m)
        SKIS_HIP_TRY(hipMemsetAsync(out.th.ptr + m, 0, (out.th.count - (size_t)m) * sizeof(uint32_t), s));
    DevBuf<int> err;
    constexpr int FLAGS = 8;
    err.alloc(arena, FLAGS);
    SKIS_HIP_TRY(hipMemsetAsync(err.ptr, 0, FLAGS * sizeof(int), s));
    int *const mixed = err.ptr + 1, *const redo = err.ptr + 2; // read with the flags
    DevBuf<int32_t> long_rows;
    long_rows.alloc(arena, (size_t)n);
    unsigned int *n_long = reinterpret_cast<unsigned int *>(err.ptr + 3);
    unsigned int *next_long = reinterpret_cast<unsigned int *>(err.ptr + 4);
    unsigned int *n_huge = reinterpret_cast<unsigned int *>(err.ptr + 5);
    unsigned int *n_pieces = reinterpret_cast<unsigned int *>(err.ptr + 6);
    unsigned int *next_unit = reinterpret_cast<unsigned int *>(err.ptr + 7);
    DevBuf<TailPiece> pieces;
    // (a piece's last strides stay below 2^31; graphs within 2^14 edges of the limit go without tails)
    if (!lt && m < (int64_t)INT32_MAX - TAIL_PIECE) pieces.alloc(arena, (size_t)tail_pieces_max(m));
    const unsigned int max_pieces = (unsigned int)tail_pieces_max(m);
    if (reinterpret_cast<uintptr_t>(P) & 15) throw Error{SKIS_EHIP, "internal error: P is not 16-byte aligned"};
    // The long rows' chains (bound by their length) run beside the short rows.  k_prep_long
    // follows k_find_long on the caller's stream and k_prep_rows goes to a second stream, which
    // first waits for the listing: the device then starts the chains first (when k_prep_rows
    // was dispatched first, the other stream's kernels started milliseconds late, and the
    // longest chain with them).
    hipLaunchKernelGGL(k_find_long, dim3(grid_for(n)), dim3(256), 0, s, n, m, row_ptr, long_rows.ptr, n_long, n_huge);
    SKIS_HIP_TRY(hipGetLastError());
    hipStream_t s2 = side_stream();
    hipEvent_t fork = nullptr, join = nullptr;
    SKIS_HIP_TRY(hipEventCreateWithFlags(&fork, hipEventDisableTiming));
    struct EvGuard {
        hipEvent_t *a, *b;
        ~EvGuard()
        {
            if (*a) (void)hipEventDestroy(*a);
            if (*b) (void)hipEventDestroy(*b);
        }
    } evg{&fork, &join};
    SKIS_HIP_TRY(hipEventCreateWithFlags(&join, hipEventDisableTiming));
    SKIS_HIP_TRY(hipEventRecord(fork, s));
    auto launch_long = [&](TailPiece *tails) {
        const bool far = m > (int64_t)INT32_MAX - LONG_EDGES;
        auto *const kernel = lt ? far ? k_prep_long<true, uint32_t> : k_prep_long<true, int32_t>
                                : far ? k_prep_long<false, uint32_t> : k_prep_long<false, int32_t>;
        hipLaunchKernelGGL(kernel, dim3((unsigned)device_cu_count() * LONG_PER_CU), dim3(256), 0, s, n, row_ptr, col,
                           w, out.th.ptr, P, out.q.ptr, err.ptr, mixed, long_rows.ptr, n_long, n_huge, next_long, tails,
                           n_pieces, max_pieces);
    };
    launch_long(pieces.ptr);
    if (pieces.ptr)
        hipLaunchKernelGGL(k_prep_tails, dim3((unsigned)device_cu_count() * 4), dim3(256), 0, s, n, row_ptr, col, w,
                           out.th.ptr, P, err.ptr, mixed, pieces.ptr, n_pieces, max_pieces, m, redo);
    const hipError_t long_err = hipGetLastError();
    // from here on, s waits for s2 before anything else, whatever fails
    hipError_t side_err = hipStreamWaitEvent(s2, fork, 0);
    if (side_err == hipSuccess) {
        // some eight turns a wave; at most 8 units at a time, so that the last ones end together
        const int64_t units = ((int64_t)n + 63) / 64, waves = (int64_t)device_cu_count() * ROWS_PER_CU;
        const unsigned per = (unsigned)std::min<int64_t>(std::max<int64_t>(units / (waves * 8), 1), 8);
        hipLaunchKernelGGL(lt ? k_prep_rows<true> : k_prep_rows<false>, dim3((unsigned)std::min(units, waves)), dim3(64), 0,
                           s2, n, m, row_ptr, col, w, out.row_ptr.ptr, out.rows.ptr, out.th.ptr, P, out.q.ptr, err.ptr,
                           mixed, next_unit, per);
        side_err = hipGetLastError();
    }
    const hipError_t rec_err = hipEventRecord(join, s2);
    if (rec_err != hipSuccess) (void)hipStreamSynchronize(s2); // no event to wait on: drain it here
    SKIS_HIP_TRY(rec_err);
    SKIS_HIP_TRY(hipStreamWaitEvent(s, join, 0));
    SKIS_HIP_TRY(long_err);
    SKIS_HIP_TRY(side_err);
    int hflags[3] = {0, 0, 0};
    SKIS_HIP_TRY(hipMemcpyAsync(hflags, err.ptr, sizeof(hflags), hipMemcpyDeviceToHost, s));
    SKIS_HIP_TRY(hipStreamSynchronize(s));
    if (hflags[2] && !hflags[0]) { // a factor moved a product that had been taken for constant
        SKIS_HIP_TRY(hipMemsetAsync(next_long, 0, sizeof(int), s));
        launch_long(nullptr);
        SKIS_HIP_TRY(hipGetLastError());
        SKIS_HIP_TRY(hipMemcpyAsync(hflags, err.ptr, sizeof(hflags), hipMemcpyDeviceToHost, s));
        SKIS_HIP_TRY(hipStreamSynchronize(s));
    }
    out.uniform = coins && !hflags[1];
    const int herr = hflags[0];
    if (herr) {
        std::string msg = "invalid graph:";
        if (herr & ERR_ROWPTR) msg += " row_ptr must start at 0, end at m and be nondecreasing;";
        if (herr & ERR_COL) msg += " col entries must lie in [0, n);";
        if (herr & ERR_SELFLOOP) msg += " self-loops are not allowed;";
        if (herr & ERR_WEIGHT) msg += " w must be in [0, 1] (no NaN);";
        if (herr & ERR_LTSUM) msg += " linear threshold model: a node's in-weights must sum to at most 1;";
        throw Error{SKIS_EINVAL, msg};
    }
    const unsigned gw = grid_for(n);
    DevBuf<uint64_t> partW;
    DevBuf<u128> partK;
    DevBuf<PrepScalars> sc;
    partW.alloc(arena, gw);
    partK.alloc(arena, gw);
    sc.alloc(arena, 1);
    hipLaunchKernelGGL(k_weights, dim3(gw), dim3(256), 0, s, n, root_shift(n), out.q.ptr, out.W.ptr, partW.ptr,
                       partK.ptr);
    SKIS_HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_weights_final, dim3(1), dim3(64), 0, s, (int)gw, partW.ptr, partK.ptr, sc.ptr);
    SKIS_HIP_TRY(hipGetLastError());
    PrepScalars hs;
    SKIS_HIP_TRY(hipMemcpyAsync(&hs, sc.ptr, sizeof(hs), hipMemcpyDeviceToHost, s));
    SKIS_HIP_TRY(hipStreamSynchronize(s));
    out.C = hs.C;
    out.Gamma = hs.Gamma;
    if (!build_alias || out.C == 0) return;

    out.alias.alloc(arena, (size_t)n);
    DevBuf<uint32_t> light, lrank, Ltot;
    DevBuf<int32_t> lid, hid;
    DevBuf<u128> dval, sval, Dinc, Sinc;
    light.alloc(arena, n);
    lrank.alloc(arena, n);
    Ltot.alloc(arena, 1);
    hipLaunchKernelGGL(k_alias_flags, dim3(grid_for(n)), dim3(256), 0, s, n, out.W.ptr, out.C, light.ptr);
    SKIS_HIP_TRY(hipGetLastError());
    excl_scan<uint32_t>(arena, light.ptr, lrank.ptr, n, Ltot.ptr, s);
    uint32_t hL = 0;
    SKIS_HIP_TRY(hipMemcpyAsync(&hL, Ltot.ptr, sizeof(hL), hipMemcpyDeviceToHost, s));
    SKIS_HIP_TRY(hipStreamSynchronize(s));
    const int64_t L = hL, H = (int64_t)n - hL;
    lid.alloc(arena, L);
    hid.alloc(arena, H);
    dval.alloc(arena, L);
    sval.alloc(arena, H);
    Dinc.alloc(arena, L);
    Sinc.alloc(arena, H);
    hipLaunchKernelGGL(k_alias_split, dim3(grid_for(n)), dim3(256), 0, s, n, out.W.ptr, out.C, light.ptr, lrank.ptr,
                       lid.ptr, hid.ptr, dval.ptr, sval.ptr);
    SKIS_HIP_TRY(hipGetLastError());
    excl_scan<u128>(arena, dval.ptr, Dinc.ptr, L, nullptr, s);
    excl_scan<u128>(arena, sval.ptr, Sinc.ptr, H, nullptr, s);
    hipLaunchKernelGGL(k_add_inplace, dim3(grid_for(L)), dim3(256), 0, s, L, Dinc.ptr, dval.ptr);
    hipLaunchKernelGGL(k_add_inplace, dim3(grid_for(H)), dim3(256), 0, s, H, Sinc.ptr, sval.ptr);
    SKIS_HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_alias_light, dim3(grid_for(L)), dim3(256), 0, s, n, L, H, out.W.ptr, lid.ptr, hid.ptr,
                       dval.ptr, Dinc.ptr, Sinc.ptr, out.alias.ptr);
    SKIS_HIP_TRY(hipGetLastError());
    if (H > 0) {
        hipLaunchKernelGGL(k_alias_heavy, dim3(grid_for(H)), dim3(256), 0, s, L, H, out.C, hid.ptr, Dinc.ptr,
                           Sinc.ptr, out.alias.ptr);
        SKIS_HIP_TRY(hipGetLastError());
    }
    SKIS_HIP_TRY(hipStreamSynchronize(s));
}

} // namespace skis

// skis_transpose.hip -- node -> samples transpose of the sketch by a stable LSD radix sort of
// the (node, sample) pairs on the node id: two passes of half the bits each for 9 to 22 bits and
// entries enough (k_tr_*, below), else 8 bits per pass (k_rs_*).
//
// A direct scatter from the sketch writes one 4-byte id per entry to a random place in HBM
// (each write a partial-line update).  The sort instead writes every pass in runs: each
// tile of RS_TILE entries sends its entries of one digit to one contiguous range.  Per pass:
//   k_rs_hist     digit counts per tile, one contiguous row per tile; per-chunk digit sums,
//                 one exclusive scan of those (digit-major) and a walk over each chunk's rows
//                 give every (tile, digit) its output offset, again one row per tile;
//   k_rs_scatter  each wave ranks its entries among equal digits with one ballot per digit
//                 bit (lanes in order) in one pass that also counts the wave's digits, the
//                 waves of a tile are ordered by a prefix of their counts, the tile is sorted
//                 by digit in LDS (stable) and written out in order, so each digit's run of
//                 the tile goes to its offset with consecutive lanes.
// The input is in sample order, so every list H(v) comes out sorted by sample id.
// The last pass writes only the sample ids and counts each node's entries; node_ptr is the
// exclusive scan of those counts.
#include <algorithm>
#include <type_traits>

#include "skis_internal.h"

namespace skis {

constexpr int RS_BLOCK = 1024;
constexpr int RS_WAVES = RS_BLOCK / 64;
constexpr int RS_TILE = 16384;                // entries per tile (digit runs of ~64 entries)
constexpr int RS_SPAN = RS_TILE / RS_WAVES;   // entries per wave, in rounds of 64

// vals[p] = j for every entry p of sample j (one wave per sample)
__global__ __launch_bounds__(256) void k_rs_vals(uint64_t T, const int64_t *__restrict__ sptr,
                                                 int32_t *__restrict__ vals)
{
    const int lane = threadIdx.x & 63;
    const uint64_t wid = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const uint64_t nw = ((uint64_t)gridDim.x * blockDim.x) >> 6;
    for (uint64_t j = wid; j < T; j += nw) {
        const int64_t a = sptr[j], b = sptr[j + 1];
        for (int64_t p = a + lane; p < b; p += 64) vals[p] = (int32_t)j;
    }
}

__global__ __launch_bounds__(RS_BLOCK) void k_rs_hist(uint64_t N, const int32_t *__restrict__ keys, int shift,
                                                      uint64_t ntiles, uint32_t *__restrict__ H)
{
    __shared__ uint32_t h[256];
    for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        if (threadIdx.x < 256) h[threadIdx.x] = 0u;
        __syncthreads();
        const uint64_t e0 = tile * RS_TILE;
        constexpr int R = RS_TILE / RS_BLOCK;
        int32_t kr[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint64_t e = e0 + (uint64_t)r * RS_BLOCK + threadIdx.x;
            kr[r] = e < N ? keys[e] : -1;
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (kr[r] >= 0) atomicAdd(&h[((uint32_t)kr[r] >> shift) & 255u], 1u);
        __syncthreads();
        if (threadIdx.x < 256) H[tile * 256 + threadIdx.x] = h[threadIdx.x]; // one contiguous row per tile
        __syncthreads();
    }
}

// Output offsets of every (tile, digit) from the tile-major histogram H[tile][digit]: the
// entries of digit d go after those of every smaller digit and, within d, tile by tile.
// k_rs_chunk_sums adds the rows of each chunk of RS_CHUNK tiles per digit into C[d][chunk]
// (digit-major, so one exclusive scan of C gives every (digit, chunk) its base), and
// k_rs_offsets walks the chunk's rows from that base, writing OFF[tile][digit].  Every access
// to H and OFF is a contiguous row of 256 values.
constexpr int RS_CHUNK = 64;

__global__ __launch_bounds__(256) void k_rs_chunk_sums(uint64_t ntiles, const uint32_t *__restrict__ H,
                                                       uint64_t nchunks, uint32_t *__restrict__ C)
{
    for (uint64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const uint64_t t0 = c * RS_CHUNK, t1 = min(t0 + RS_CHUNK, ntiles);
        uint32_t acc = 0;
        for (uint64_t t = t0; t < t1; ++t) acc += H[t * 256 + threadIdx.x];
        C[(uint64_t)threadIdx.x * nchunks + c] = acc;
    }
}

__global__ __launch_bounds__(256) void k_rs_offsets(uint64_t ntiles, const uint32_t *__restrict__ H,
                                                    uint64_t nchunks, const int64_t *__restrict__ CB,
                                                    int64_t *__restrict__ OFF)
{
    for (uint64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const uint64_t t0 = c * RS_CHUNK, t1 = min(t0 + RS_CHUNK, ntiles);
        int64_t acc = CB[(uint64_t)threadIdx.x * nchunks + c];
        for (uint64_t t = t0; t < t1; ++t) {
            OFF[t * 256 + threadIdx.x] = acc;
            acc += H[t * 256 + threadIdx.x];
        }
    }
}

// Lanes of the wave holding the same digit d as this lane (among the valid ones); digits
// have `bits` significant bits (uniform), the others are zero.
__device__ __forceinline__ unsigned long long same_digit_mask(bool valid, uint32_t d, int bits)
{
    unsigned long long m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        if (b >= bits) break;
        const bool bit = (d >> b) & 1u;
        const unsigned long long bb = __ballot(bit);
        m &= bit ? bb : ~bb;
    }
    return m;
}

__global__ __launch_bounds__(RS_BLOCK) __attribute__((amdgpu_waves_per_eu(4))) void k_rs_scatter(uint64_t N, const int32_t *__restrict__ kin,
                                                         const int32_t *__restrict__ vin, int32_t *__restrict__ kout,
                                                         int32_t *__restrict__ vout, int shift, int bits,
                                                         uint64_t ntiles, const int64_t *__restrict__ OFF,
                                                         uint32_t *__restrict__ deg)
{
    __shared__ long long base[256];        // output offset of each digit for this tile
    __shared__ uint32_t tstart[256 + 1];   // first tile-local position of each digit
    __shared__ uint32_t cnt[RS_WAVES][256]; // per-wave digit counts, then each wave's running index
    __shared__ int32_t sk[RS_TILE], sv[RS_TILE]; // the tile, then the tile sorted by digit
    __shared__ uint32_t s_scan[RS_WAVES + 1];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const unsigned long long lt = (1ull << lane) - 1ull;
    constexpr int R = RS_SPAN / 64;
    constexpr int PER = RS_TILE / RS_BLOCK;
    // the next tile's entries and digit offsets are loaded while this one is sorted and
    // written (unconditional loads: an index past the end reads the last entry, unused)
    int32_t kr[R], vr[R];
    long long bnext = 0;
    uint64_t tile = blockIdx.x;
    if (tile < ntiles) {
        const uint64_t s0 = tile * RS_TILE + (uint64_t)w * RS_SPAN;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint64_t e = min(s0 + (uint64_t)r * 64 + lane, N - 1);
            kr[r] = kin[e];
            vr[r] = vin[e];
        }
        if (threadIdx.x < 256) bnext = OFF[tile * 256 + threadIdx.x];
    }
    for (; tile < ntiles; tile += gridDim.x) {
        const uint64_t t0 = tile * RS_TILE;
        const uint64_t s0 = t0 + (uint64_t)w * RS_SPAN;
        const int nvalid = (int)min((uint64_t)RS_TILE, N - t0);
        if (threadIdx.x < 256) base[threadIdx.x] = bnext;
        for (int i = threadIdx.x; i < RS_WAVES * 256; i += RS_BLOCK) (&cnt[0][0])[i] = 0u;
        const uint64_t tn = tile + gridDim.x;
        if (tn < ntiles && threadIdx.x < 256) bnext = OFF[tn * 256 + threadIdx.x];
        __syncthreads();
        // one ranking pass over the wave's span (in registers, in order): the rank of each
        // entry among the equal digits before it in the wave, while the leader of each digit
        // and round advances the wave's count of that digit
        uint32_t lp[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool valid = s0 + (uint64_t)r * 64 + lane < N;
            const uint32_t d = valid ? (((uint32_t)kr[r] >> shift) & 255u) : 0u;
            const unsigned long long m = same_digit_mask(valid, d, bits);
            lp[r] = valid ? cnt[w][d] + (uint32_t)__popcll(m & lt) : 0xFFFFFFFFu;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (valid && !(m & lt)) cnt[w][d] += (uint32_t)__popcll(m);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        __syncthreads();
        // digit d of the tile: its waves in order, after the digits below d
        {
            const int d = threadIdx.x; // digits 0..255; the other threads add nothing
            uint32_t acc = 0;
            if (d < 256)
                for (int k = 0; k < RS_WAVES; ++k) {
                    const uint32_t x = cnt[k][d];
                    cnt[k][d] = acc;
                    acc += x;
                }
            uint32_t tot;
            const uint32_t ex = block_excl_scan<RS_BLOCK, uint32_t>(acc, s_scan, &tot);
            if (d < 256) {
                tstart[d] = ex;
                if (d == 255) tstart[256] = tot;
                for (int k = 0; k < RS_WAVES; ++k) cnt[k][d] += ex;
            }
        }
        __syncthreads();
        // the tile sorted by digit (stably) in LDS
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (lp[r] != 0xFFFFFFFFu) {
                const uint32_t d = ((uint32_t)kr[r] >> shift) & 255u;
                const uint32_t pos = cnt[w][d] + lp[r];
                sk[pos] = kr[r];
                sv[pos] = vr[r];
            }
        __syncthreads();
        // the next tile's loads go out before this one is written
        if (tn < ntiles) {
            const uint64_t n0 = tn * RS_TILE + (uint64_t)w * RS_SPAN;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint64_t e = min(n0 + (uint64_t)r * 64 + lane, N - 1);
                kr[r] = kin[e];
                vr[r] = vin[e];
            }
        }
        // phase 3: the sorted tile goes out in order, each digit's run to its offset.  In the
        // last pass (deg set) the keys are not written: each run of equal keys within a
        // digit's run adds its length to deg[key], as -first at its first element and
        // last + 1 at its last one (the pass's keys are sorted within a digit's run).
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int i = k * RS_BLOCK + threadIdx.x;
            if (i < nvalid) {
                const int32_t key = sk[i];
                const uint32_t d = ((uint32_t)key >> shift) & 255u;
                const long long pos = base[d] + (long long)(i - (int)tstart[d]);
                vout[pos] = sv[i];
                if (!deg) {
                    kout[pos] = key;
                } else {
                    const bool first = i == (int)tstart[d] || sk[i - 1] != key;
                    const bool last = i + 1 == (int)tstart[d + 1] || sk[i + 1] != key;
                    if (first) atomicAdd(&deg[key], (uint32_t)(-i));
                    if (last) atomicAdd(&deg[key], (uint32_t)(i + 1));
                }
            }
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_rs_fill_u32(uint64_t count, uint32_t *__restrict__ p, uint32_t v)
{
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

static unsigned grid_rs(uint64_t items, int block, int per_cu = 8)
{
    uint64_t g = (items + block - 1) / block;
    const uint64_t cap = (uint64_t)device_cu_count() * per_cu;
    if (g > cap) g = cap;
    return (unsigned)(g > 0 ? g : 1);
}

// Two passes where the node ids have 9 to 22 bits: low half, high half.  A pass costs its traffic, so
// digits as wide as LDS takes beat three passes of 8 bits.
//  - The first pass writes, beside the sample ids, the high halves alone (2 B): the second pass's
//    chunks are pieces of the entries of one low half, which their place thus tells.
//  - A tile's run of one digit is short of a line (14 entries), so the workgroups of an XCD take
//    neighbouring tiles of the first pass, so that its L2 may put lines together.
//  - In the second pass a workgroup takes whole chunks and keeps each digit's next place in a register
//    from tile to tile, so counts are kept per chunk and not per tile.
//  - Every low half has a chunk, if an empty one: the place of digit h in the first chunk of low half l
//    is node_ptr of node (h, l), so no degrees are counted.
// 401M entries of 1M nodes: 8.6 -> 5.0 ms; 153M of 4M nodes: 3.45 -> 2.75 ms.  What is left is the partial
// lines of the first pass: tiles of half the size, two workgroups a CU, took 1.5 ms for 1.1 there.
struct TrChunk {
    uint32_t e0, e1; // entries
};
constexpr int TR_TILES = 16; // tiles of a chunk of the second pass, at most: tables small, ends even
constexpr int TR_XCD = 8;
constexpr int TR_GROUP = 32; // tiles of the first pass a column of the scan

// Threads and rounds of a wave a tile: LDS holds the tile and its waves' digit counts.  In the
// second pass two workgroups share a CU (one's ranking beside the other's writing).
constexpr int tr_block(bool last) { return last ? 512 : 1024; }
constexpr int tr_rounds(int dbits, bool last) { return dbits <= 10 ? 14 : last ? 11 : 10; }
constexpr int tr_tile(int dbits, bool last) { return tr_rounds(dbits, last) * tr_block(last); }
// the widths that kernels are built for: the next one takes a digit of fewer bits
constexpr int tr_width(int dbits) { return dbits <= 7 ? 7 : dbits <= 10 ? 10 : 11; }

// Lanes of the wave (among `valid` ones) whose digit of BITS bits is this lane's.
template <int BITS> __device__ __forceinline__ unsigned long long equal_digits(unsigned long long valid, uint32_t d)
{
    uint32_t lo = (uint32_t)valid, hi = (uint32_t)(valid >> 32);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const uint32_t mine = (uint32_t)((int32_t)(d << (31 - b)) >> 31); // all ones where the bit is set
        const unsigned long long bb = __ballot((int32_t)mine < 0);
        lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)bb, mine, 0x90); // lo & ~(bb ^ mine)
        hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(bb >> 32), mine, 0x90);
    }
    return (unsigned long long)hi << 32 | lo;
}

// First pass: digit counts of each tile, a row of D values; their sums over each group of TR_GROUP
// tiles, digit-major (S[d * groups + g]); and, once those are scanned, each tile's places, a row again.
__global__ __launch_bounds__(512) void k_tr_tiles(const int32_t *__restrict__ keys, uint32_t N, uint32_t tile, int D,
                                                  uint16_t *__restrict__ H)
{
    __shared__ uint32_t h[2048];
    for (int d = threadIdx.x; d < D; d += 512) h[d] = 0u;
    __syncthreads();
    const uint32_t e0 = blockIdx.x * tile, e1 = (uint32_t)min((uint64_t)N, (uint64_t)e0 + tile);
    constexpr int U = 14;
    for (uint32_t i0 = e0 + threadIdx.x; i0 < e1; i0 += 512 * U) {
        uint32_t k[U];
#pragma unroll
        for (int u = 0; u < U; ++u) k[u] = (uint32_t)keys[min(i0 + u * 512, e1 - 1)] & (uint32_t)(D - 1);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * 512 < e1) atomicAdd(&h[k[u]], 1u);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < D; d += 512) H[(uint64_t)blockIdx.x * D + d] = (uint16_t)h[d];
}

__global__ __launch_bounds__(128) void k_tr_sums(uint32_t ntiles, int D, const uint16_t *__restrict__ H, uint32_t groups,
                                                 uint32_t *__restrict__ S)
{
    const uint32_t t0 = blockIdx.x * TR_GROUP, t1 = min(t0 + TR_GROUP, ntiles);
    for (int d = threadIdx.x; d < D; d += 128) {
        uint32_t acc = 0;
#pragma unroll 8
        for (uint32_t t = t0; t < t1; ++t) acc += H[(uint64_t)t * D + d];
        S[(uint64_t)d * groups + blockIdx.x] = acc;
    }
}

__global__ __launch_bounds__(128) void k_tr_places(uint32_t ntiles, int D, const uint16_t *__restrict__ H,
                                                   uint32_t groups, const int64_t *__restrict__ SB,
                                                   uint32_t *__restrict__ places)
{
    const uint32_t t0 = blockIdx.x * TR_GROUP, t1 = min(t0 + TR_GROUP, ntiles);
    for (int d = threadIdx.x; d < D; d += 128) {
        uint32_t acc = (uint32_t)SB[(uint64_t)d * groups + blockIdx.x];
#pragma unroll 8
        for (uint32_t t = t0; t < t1; ++t) {
            places[(uint64_t)t * D + d] = acc;
            acc += H[(uint64_t)t * D + d];
        }
    }
}

// The second pass's chunks from the starts of the D low halves (CB[l * stride], CB[D * stride] = N):
// pieces of at most `piece` entries, at least one a low half; first[l] is its first chunk.
__global__ __launch_bounds__(1024) void k_tr_chunks(int D, int64_t stride, const int64_t *__restrict__ CB, uint32_t piece,
                                                    TrChunk *__restrict__ chunks, uint32_t *__restrict__ first,
                                                    uint32_t *__restrict__ n_out, uint32_t *__restrict__ next)
{
    __shared__ uint32_t s_scan[1024 / 64 + 1];
    uint32_t c0 = 0;
    for (int l0 = 0; l0 < D; l0 += 1024) {
        const int l = l0 + (int)threadIdx.x;
        uint32_t a = 0, b = 0, np = 0;
        if (l < D) {
            a = (uint32_t)CB[(int64_t)l * stride];
            b = (uint32_t)CB[(int64_t)(l + 1) * stride];
            np = max(1u, (b - a + piece - 1) / piece);
        }
        uint32_t tot;
        const uint32_t ex = c0 + block_excl_scan<1024, uint32_t>(np, s_scan, &tot);
        if (l < D) {
            first[l] = ex;
            for (uint32_t k = 0; k < np; ++k) chunks[ex + k] = {a + k * piece, k + 1 < np ? a + (k + 1) * piece : b};
        }
        c0 += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        *n_out = c0;
        *next = 0;
    }
}

// Digit counts of each chunk: C[d * stride + c] (zero past the last chunk).  A node in most samples
// fills its chunks with one digit: four counters a digit, by lane, where the atomics of a wave on one
// counter had taken a cycle each.
__global__ __launch_bounds__(512) void k_tr_hist(const TrChunk *__restrict__ chunks, const uint32_t *__restrict__ n_chunks,
                                                 uint32_t stride, const uint16_t *__restrict__ keys, int D,
                                                 uint32_t *__restrict__ C)
{
    __shared__ uint32_t h[2048 * 4];
    const uint64_t *const quads = reinterpret_cast<const uint64_t *>(keys); // the keys are padded to whole quads
    const uint32_t nc = *n_chunks, copy = threadIdx.x & 3;
    for (uint32_t c = blockIdx.x; c < stride; c += gridDim.x) {
        for (int d = threadIdx.x; d < D * 4; d += 512) h[d] = 0u;
        __syncthreads();
        if (c < nc) {
            const TrChunk ch = chunks[c];
            constexpr int U = 4;
            const uint32_t q1 = ch.e1 > ch.e0 ? (ch.e1 + 3) / 4 : 0;
            for (uint32_t q0 = ch.e0 / 4 + threadIdx.x; q0 < q1; q0 += 512 * U) {
                uint64_t k[U];
#pragma unroll
                for (int u = 0; u < U; ++u) k[u] = quads[min(q0 + u * 512, q1 - 1)];
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const uint32_t e = (q0 + u * 512) * 4 + x;
                        if (e >= ch.e0 && e < ch.e1) atomicAdd(&h[(uint32_t)(k[u] >> (16 * x) & 0xFFFFu) * 4 + copy], 1u);
                    }
            }
        }
        __syncthreads();
        for (int d = threadIdx.x; d < D; d += 512) {
            const uint4 x = reinterpret_cast<const uint4 *>(h)[d];
            C[(uint64_t)d * stride + c] = x.x + x.y + x.z + x.w;
        }
        __syncthreads();
    }
}

// As k_rs_scatter.  LAST: the keys are the digits and are not written, and a workgroup goes chunk by
// chunk (the next chunk is taken when one is begun, so that the next tile's loads are always out
// before this one is written); else it takes every (gridDim / TR_XCD)-th tile of its XCD's part, at
// the places of `places`.
template <int BITS, bool LAST>
__global__ __launch_bounds__(tr_block(LAST)) __attribute__((amdgpu_waves_per_eu(4))) void
k_tr_scatter(uint32_t N, const TrChunk *__restrict__ chunks, const uint32_t *__restrict__ n_chunks, uint32_t stride,
             uint32_t *__restrict__ next, const int64_t *__restrict__ CB, const uint32_t *__restrict__ places,
             const std::conditional_t<LAST, uint16_t, int32_t> *__restrict__ kin, const int32_t *__restrict__ vin,
             uint16_t *__restrict__ kout, int32_t *__restrict__ vout, int dbits)
{
    constexpr int BLOCK = tr_block(LAST), WAVES = BLOCK / 64, R = tr_rounds(BITS, LAST), TILE = R * BLOCK, SPAN = R * 64;
    constexpr int DMAX = 1 << BITS, OWN = (DMAX + BLOCK - 1) / BLOCK; // digits a thread keeps
    __shared__ std::conditional_t<LAST, uint16_t, uint32_t> sk[TILE]; // the tile sorted by digit
    __shared__ int32_t sv[TILE];
    __shared__ uint16_t cnt[WAVES][DMAX]; // per-wave digit counts, then each wave's running index
    __shared__ uint32_t gb[DMAX];         // a digit's place for the tile's element 0
    __shared__ uint32_t s_scan[WAVES + 1];
    __shared__ uint32_t s_next;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int D = 1 << dbits;
    const unsigned long long lt = (1ull << lane) - 1ull;
    uint32_t c = blockIdx.x, e0, e1;
    [[maybe_unused]] uint32_t nc = 0, step = 0;
    if constexpr (LAST) {
        nc = *n_chunks;
        if (c >= nc) return;
        e0 = chunks[c].e0;
        e1 = chunks[c].e1;
    } else {
        const uint32_t ntiles = (N + (TILE - 1)) / TILE;
        const uint32_t parts = gridDim.x % TR_XCD == 0 ? TR_XCD : 1, part = (ntiles + parts - 1) / parts;
        step = gridDim.x / parts;
        c = blockIdx.x % parts * part + blockIdx.x / parts;
        nc = min(ntiles, (blockIdx.x % parts + 1) * part); // the part's end
        if (c >= nc) return;
        e0 = c * TILE;
        e1 = (uint32_t)min((uint64_t)N, (uint64_t)e0 + TILE);
    }
    uint32_t kr[R];
    int32_t vr[R];
    auto load = [&](uint32_t at) { // an index past the end reads the last entry, unused
        const uint32_t s0 = at + (uint32_t)(w * SPAN + lane);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t e = min(s0 + (uint32_t)r * 64u, N - 1u);
            kr[r] = (uint32_t)kin[e];
            vr[r] = vin[e];
        }
    };
    load(e0);
    bool fresh = true;     // the first tile at these places
    uint32_t place[OWN]{}; // next output place of this thread's digits
    for (;;) {
        if (fresh) {
#pragma unroll
            for (int o = 0; o < OWN; ++o)
                if (t * OWN + o < D)
                    place[o] = LAST ? (uint32_t)CB[(uint64_t)(t * OWN + o) * stride + c] : places[(uint64_t)c * D + t * OWN + o];
            if (LAST && t == 0) s_next = gridDim.x + atomicAdd(next, 1u);
        }
        const int nvalid = (int)min((uint32_t)TILE, e1 - e0);
        for (int i = t; i < WAVES * DMAX / 2; i += BLOCK) reinterpret_cast<uint32_t *>(&cnt[0][0])[i] = 0u;
        __syncthreads();
        // the rank of each entry among the equal digits before it in the wave
        uint32_t lp[(R + 1) / 2]{}; // two a register
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool valid = w * SPAN + r * 64 + lane < nvalid;
            const uint32_t d = valid ? kr[r] & (uint32_t)(D - 1) : 0u;
            const unsigned long long m = equal_digits<BITS>(__ballot(valid), d);
            const uint32_t before = cnt[w][d];
            lp[r / 2] |= (before + (uint32_t)__popcll(m & lt)) << (r % 2 * 16);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (valid && !(m & lt)) cnt[w][d] = (uint16_t)(before + __popcll(m));
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        __syncthreads();
        // the digits of the tile in order, a digit's waves in order
        {
            uint32_t tot[OWN]{}, sum = 0, all;
#pragma unroll
            for (int o = 0; o < OWN; ++o) {
                if (t * OWN + o < D)
#pragma unroll
                    for (int k = 0; k < WAVES; ++k) tot[o] += cnt[k][t * OWN + o];
                sum += tot[o];
            }
            uint32_t ex = block_excl_scan<BLOCK, uint32_t>(sum, s_scan, &all);
#pragma unroll
            for (int o = 0; o < OWN; ++o) {
                const int d = t * OWN + o;
                if (d >= D) break;
                gb[d] = place[o] - ex;
                place[o] += tot[o];
                uint32_t run = ex;
#pragma unroll
                for (int k = 0; k < WAVES; ++k) {
                    const uint32_t x = cnt[k][d];
                    cnt[k][d] = (uint16_t)run;
                    run += x;
                }
                ex += tot[o];
            }
        }
        __syncthreads();
        [[maybe_unused]] const uint32_t after = LAST ? s_next : 0u; // written before this tile's first barrier at the latest
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (w * SPAN + r * 64 + lane < nvalid) {
                const uint32_t pos = (uint32_t)cnt[w][kr[r] & (uint32_t)(D - 1)] + (lp[r / 2] >> (r % 2 * 16) & 0xFFFFu);
                sk[pos] = kr[r];
                sv[pos] = vr[r];
            }
        __syncthreads();
        // the next tile's loads go out before this one is written
        bool more = true;
        if constexpr (LAST) {
            fresh = e1 - e0 <= (uint32_t)TILE;
            if (fresh) {
                c = after;
                more = c < nc;
                if (more) {
                    e0 = chunks[c].e0;
                    e1 = chunks[c].e1;
                }
            } else {
                e0 += TILE;
            }
        } else {
            c += step;
            more = c < nc;
            e0 = more ? c * TILE : e0;
            e1 = (uint32_t)min((uint64_t)N, (uint64_t)e0 + TILE);
        }
        if (more) load(e0);
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int i = k * BLOCK + t;
            if (i < nvalid) {
                const uint32_t key = sk[i];
                const uint32_t pos = gb[LAST ? key : key & (uint32_t)(D - 1)] + (uint32_t)i;
                vout[pos] = sv[i];
                if (!LAST) kout[pos] = (uint16_t)(key >> dbits);
            }
        }
        if (!more) break;
        __syncthreads();
    }
}

// node_ptr (and the degrees) of node v = (h << lbits) + l from the places of the digits h.
__global__ __launch_bounds__(256) void k_tr_ptr(int32_t n, int lbits, uint32_t stride, const int64_t *__restrict__ CB,
                                                const uint32_t *__restrict__ first, uint32_t N,
                                                int64_t *__restrict__ node_ptr, uint32_t *__restrict__ deg)
{
    const uint32_t lmask = (1u << lbits) - 1u;
    auto at = [&](int64_t v) -> int64_t {
        if (v >= n) return N;
        return CB[(uint64_t)(v >> lbits) * stride + first[(uint32_t)v & lmask]];
    };
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v <= n; v += (int64_t)gridDim.x * 256) {
        const int64_t p = at(v);
        node_ptr[v] = p;
        if (v < n) deg[v] = (uint32_t)(at(v + 1) - p);
    }
}

template <bool LAST, typename... Args>
static void tr_scatter(int dbits, unsigned grid, hipStream_t s, Args... args)
{
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(grid), dim3(tr_block(LAST)), 0, s, args..., dbits); };
    switch (tr_width(dbits)) {
    case 7: go(k_tr_scatter<7, LAST>); break;
    case 10: go(k_tr_scatter<10, LAST>); break;
    default: go(k_tr_scatter<11, LAST>);
    }
    SKIS_HIP_TRY(hipGetLastError());
}

static void two_pass_transpose(Arena &arena, const int32_t *nodes, const int32_t *vals, uint32_t N, int32_t n, int bits,
                               int64_t *node_ptr, int32_t *node_samples, uint32_t *deg, hipStream_t s)
{
    const int lbits = (bits + 1) / 2, hbits = bits - lbits;
    const uint32_t L = 1u << lbits, Hd = 1u << hbits;
    const uint32_t cus = (uint32_t)device_cu_count();
    const uint32_t tile1 = (uint32_t)tr_tile(lbits, false), ntiles = (uint32_t)(((uint64_t)N + tile1 - 1) / tile1);
    const uint32_t groups = (ntiles + TR_GROUP - 1) / TR_GROUP;
    const uint32_t piece = (uint32_t)(TR_TILES * tr_tile(hbits, true)), nc = L + N / piece; // at most so many chunks
    DevBuf<uint16_t> key, H;
    DevBuf<int32_t> val;
    DevBuf<TrChunk> chunks;
    DevBuf<uint32_t> places, C, first, misc;
    DevBuf<int64_t> CB;
    key.alloc(arena, ((uint64_t)N + 3) / 4 * 4);
    val.alloc(arena, N);
    H.alloc(arena, (uint64_t)ntiles * L);
    places.alloc(arena, (uint64_t)ntiles * L);
    chunks.alloc(arena, nc);
    first.alloc(arena, L);
    misc.alloc(arena, 2);
    const uint64_t cells1 = (uint64_t)L * groups, cells2 = (uint64_t)Hd * nc;
    C.alloc(arena, std::max(cells1, cells2));
    CB.alloc(arena, std::max(cells1, cells2) + 1);
    uint32_t *const n_chunks = misc.ptr, *const next = misc.ptr + 1;
    hipLaunchKernelGGL(k_tr_tiles, dim3(ntiles), dim3(512), 0, s, nodes, N, tile1, (int)L, H.ptr);
    hipLaunchKernelGGL(k_tr_sums, dim3(groups), dim3(128), 0, s, ntiles, (int)L, H.ptr, groups, C.ptr);
    SKIS_HIP_TRY(hipGetLastError());
    excl_scan_u32_to_i64(arena, C.ptr, CB.ptr, (int64_t)cells1, CB.ptr + cells1, s);
    hipLaunchKernelGGL(k_tr_places, dim3(groups), dim3(128), 0, s, ntiles, (int)L, H.ptr, groups, CB.ptr, places.ptr);
    hipLaunchKernelGGL(k_tr_chunks, dim3(1), dim3(1024), 0, s, (int)L, (int64_t)groups, CB.ptr, piece, chunks.ptr, first.ptr,
                       n_chunks, next);
    SKIS_HIP_TRY(hipGetLastError());
    tr_scatter<false>(lbits, std::min((ntiles + TR_XCD - 1) / TR_XCD * TR_XCD, cus), s, N, (const TrChunk *)nullptr,
                      (const uint32_t *)nullptr, 0u, (uint32_t *)nullptr, (const int64_t *)nullptr,
                      (const uint32_t *)places.ptr, nodes, vals, key.ptr, val.ptr);
    hipLaunchKernelGGL(k_tr_hist, dim3(std::min(nc, cus * 4)), dim3(512), 0, s, chunks.ptr, n_chunks, nc, key.ptr, (int)Hd,
                       C.ptr);
    SKIS_HIP_TRY(hipGetLastError());
    excl_scan_u32_to_i64(arena, C.ptr, CB.ptr, (int64_t)cells2, CB.ptr + cells2, s);
    tr_scatter<true>(hbits, std::min(nc, cus * 2), s, N, (const TrChunk *)chunks.ptr, (const uint32_t *)n_chunks, nc, next,
                     (const int64_t *)CB.ptr, (const uint32_t *)nullptr, (const uint16_t *)key.ptr,
                     (const int32_t *)val.ptr, (uint16_t *)nullptr, node_samples);
    hipLaunchKernelGGL(k_tr_ptr, dim3(grid_rs((uint64_t)n + 1, 256)), dim3(256), 0, s, n, lbits, nc, CB.ptr, first.ptr, N,
                       node_ptr, deg);
    SKIS_HIP_TRY(hipGetLastError());
    SKIS_HIP_TRY(hipStreamSynchronize(s)); // the temporaries are released on return
}

void radix_transpose(Arena &arena, const int64_t *sample_ptr, const int32_t *nodes, int32_t *owner, uint64_t T,
                     uint64_t N, int32_t n, int64_t *node_ptr, int32_t *node_samples, uint32_t *deg, hipStream_t s)
{
    if (N == 0 || T == 0) throw Error{SKIS_EHIP, "internal error: empty transpose"};
    int bits = 1;
    while (bits < 31 && ((uint64_t)(n - 1) >> bits) != 0) ++bits;
    // Half the bits a pass needs entries enough: below some 512 a low half its chunks are mostly empty.
    // 16.8M samples: 8.6 (8 bits a pass) and 5.0 ms for 20 bits, 3.45 and 2.75 for 22, 1.36 and 1.07
    // for 20 bits of few entries; from 23 bits on, a digit's counts leave no room in LDS.
    if (bits > 8 && bits <= 22 && N >= ((uint64_t)512 << ((bits + 1) / 2)) && N <= 0xFFFF0000ull) {
        DevBuf<int32_t> v;
        if (!owner) {
            v.alloc(arena, N);
            owner = v.ptr;
            hipLaunchKernelGGL(k_rs_vals, dim3(grid_rs(T * 64, 256, 16)), dim3(256), 0, s, T, sample_ptr, owner);
            SKIS_HIP_TRY(hipGetLastError());
        }
        two_pass_transpose(arena, nodes, owner, (uint32_t)N, n, bits, node_ptr, node_samples, deg, s);
        return;
    }
    const int passes = (bits + 7) / 8;
    const uint64_t ntiles = (N + RS_TILE - 1) / RS_TILE;
    DevBuf<int32_t> ka, kb, va, vb;
    DevBuf<uint32_t> H;
    DevBuf<int64_t> OFF;
    ka.alloc(arena, N);
    int32_t *vals = owner; // the sample id of every entry, scratch after the first pass
    if (!vals) {
        va.alloc(arena, N);
        vals = va.ptr;
    }
    if (passes > 1) vb.alloc(arena, N);
    kb.alloc(arena, N);
    const uint64_t nchunks = (ntiles + RS_CHUNK - 1) / RS_CHUNK;
    H.alloc(arena, 256 * ntiles);
    OFF.alloc(arena, 256 * ntiles);
    DevBuf<uint32_t> C;
    DevBuf<int64_t> CB;
    C.alloc(arena, 256 * nchunks);
    CB.alloc(arena, 256 * nchunks + 1);
    if (!owner) {
        hipLaunchKernelGGL(k_rs_vals, dim3(grid_rs(T * 64, 256, 16)), dim3(256), 0, s, T, sample_ptr, vals);
        SKIS_HIP_TRY(hipGetLastError());
    }
    const unsigned gt = (unsigned)std::min<uint64_t>(ntiles, (uint64_t)device_cu_count() * 8);
    // pass p reads (kin, vin) and writes (kout, vout); the sketch's nodes are the first keys,
    // the last pass writes the values straight into node_samples
    const int32_t *kin = nodes;
    const int32_t *vin = vals;
    // the last pass counts each node's entries instead of writing the sorted keys
    hipLaunchKernelGGL(k_rs_fill_u32, dim3(grid_rs(n, 256, 4)), dim3(256), 0, s, (uint64_t)n, deg, 0u);
    for (int p = 0; p < passes; ++p) {
        const bool lastp = p == passes - 1;
        int32_t *kout = lastp ? nullptr : ((p & 1) ? ka.ptr : kb.ptr);
        int32_t *vout = lastp ? node_samples : ((p & 1) ? vals : vb.ptr);
        hipLaunchKernelGGL(k_rs_hist, dim3(gt), dim3(RS_BLOCK), 0, s, N, kin, 8 * p, ntiles, H.ptr);
        SKIS_HIP_TRY(hipGetLastError());
        hipLaunchKernelGGL(k_rs_chunk_sums, dim3(grid_rs(nchunks * 256, 256, 8)), dim3(256), 0, s, ntiles, H.ptr,
                           nchunks, C.ptr);
        excl_scan_u32_to_i64(arena, C.ptr, CB.ptr, (int64_t)(256 * nchunks), CB.ptr + 256 * nchunks, s);
        hipLaunchKernelGGL(k_rs_offsets, dim3(grid_rs(nchunks * 256, 256, 8)), dim3(256), 0, s, ntiles, H.ptr,
                           nchunks, CB.ptr, OFF.ptr);
        SKIS_HIP_TRY(hipGetLastError());
        hipLaunchKernelGGL(k_rs_scatter, dim3(gt), dim3(RS_BLOCK), 0, s, N, kin, vin, kout, vout, 8 * p,
                           std::min(8, bits - 8 * p), ntiles, OFF.ptr, lastp ? deg : nullptr);
        SKIS_HIP_TRY(hipGetLastError());
        kin = kout;
        vin = vout;
    }
    excl_scan_u32_to_i64(arena, deg, node_ptr, n, node_ptr + n, s);
    SKIS_HIP_TRY(hipStreamSynchronize(s)); // the temporaries are released on return
}

} // namespace skis

// skis_query.h -- declarations of the query kernels' host launchers.
#pragma once
#include <mutex>

#include "skis_internal.h"

namespace skis {

constexpr int EST_BLOCK = 1024;   // threads per query in k_estimate
constexpr int EST_MAX_SET = 4096; // largest seed set one estimate workgroup holds in LDS
constexpr int EST_WALK = 4;       // sample-list entries a thread walks per round, loads issued together

constexpr int EST_HASH_SLOTS = 16384; // LDS hash of a light set's sample ids in k_est_set
constexpr int EST_HASH_MAX = 10922;   // list entries a light set's members hold at most (1.5 slots each)
constexpr int32_t EST_ROUND = 1 << 16; // sets of one round of skis_estimate
constexpr uint64_t EST_WALK_MAX = 0xFFFF0000ull; // entries that k_est_set's walk counts in 32 bits
constexpr unsigned long long EST_PARKED = ~0ull; // cov of a set that k_est_set left to the next kernel

// What k_est_set reports (each word is only ever set to 1).
struct EstFlags {
    int ptr;    // set_ptr does not rise from 0
    int node;   // a node id outside [0, n)
    int large;  // a set above EST_MAX_SET entries was left out
    int parked; // a set above EST_HASH_MAX list entries was parked
};

constexpr int GREEDY_HOT = 2048;  // hot nodes decremented in LDS

struct GreedyState {
    int32_t vstar;              // this round's pick (-1: none left)
    unsigned shrunk;            // a heavy round has cut the lists down (they are in the work copy)
    int32_t cur;                // which of the two delta buffers holds the current counts
    unsigned long long dstar;   // delta of this round's pick: the samples it newly covers
    unsigned long long cov;     // coverage of the picks so far
    double est;
    unsigned flipped;           // the round's argmax has switched buffers: the spare one is to be cleared
    int32_t rounds;             // rounds whose pick k_greedy_argmax has taken
    unsigned light;             // the others are k_greedy_small's
    unsigned before;            // small sketches: entries left before the last round
};

// A tile of GREEDY_TILE nodes keeps its best node as of its last scan and the second gain.  Delta
// only falls, so g2 bounds the gains of all its other nodes from above ever after.
constexpr int GREEDY_TILE = 2048;
struct __align__(8) GreedyTile {
    double g;   // its gain
    double g2;  // the largest gain of the others, -1: none
    int32_t v;  // the node, -1: every node of the tile is chosen
    int32_t d;  // its delta
};
constexpr int GREEDY_BLOCK = 1024; // the pick is one workgroup's
constexpr int GREEDY_BIG = 512;    // in the one-workgroup form, a sample above this is uncovered by all threads
// Sketches whose greedy runs in one workgroup, with no launches inside its rounds, but for the first ones.
constexpr int GREEDY_SMALL_TILES = 2048;
constexpr uint64_t GREEDY_SMALL_ENTRIES = 1ull << 19;
constexpr uint64_t GREEDY_SMALL_ROUND = 1ull << 15;
// entries left, and lowered by the last round, up to which one workgroup does the rest (over graphs of
// 2000 to 4M nodes and 8 to 500 thousand entries 32768 to 98304 and 8192 to 49152 are within 4 %)
constexpr uint32_t GREEDY_FEW_LEFT = 65536, GREEDY_FEW_LOWERED = 8192;
// the entries left after a round, in parts a line apart (one counter for 2048 workgroups takes 19 us)
constexpr int GREEDY_LEFT_PARTS = 32, GREEDY_LEFT_STEP = 16;

// A newly covered sample in a queue of k_greedy_cover: its first entry (a sketch may hold 2^33 entries
// and more) and its entries; 12 bytes.
struct CoverItem {
    uint32_t lo, hi;
    int32_t size;
    __host__ __device__ void set(int64_t a, int64_t b)
    {
        lo = (uint32_t)a;
        hi = (uint32_t)(a >> 32);
        size = (int32_t)(b - a);
    }
    __host__ __device__ int64_t first() const { return (int64_t)((uint64_t)hi << 32 | lo); }
    __host__ __device__ int32_t len() const { return size; }
};

// One recount work item: entries [p0, p0 + len) of node v's list.
struct RecountItem {
    int64_t p0;
    int32_t len;
    int32_t v;
};

// Per-sketch scratch for estimate.
struct QueryScratch {
    DevBuf<uint32_t> bitmaps; // sets above EST_MAX_SET entries: one bitmap of T bits each in flight
    DevBuf<int> err;
    DevBuf<uint32_t> split;   // the parked sets' list and tickets, flags
};

// The service's host copy of the lists' lengths: two bytes a node, LONG_LIST where node_ptr tells.
constexpr uint16_t LONG_LIST = 0xFFFF;

// Entries of the lists of nodes[0 .. count), repeated nodes counted again.
inline uint64_t list_entries(const uint16_t *list_len, const int64_t *node_ptr, const int32_t *nodes, int32_t count)
{
    uint64_t entries = 0;
    bool exact = true;
    for (int32_t i = 0; i < count; ++i) {
        const uint16_t len = list_len[nodes[i]];
        exact = exact && len != LONG_LIST;
        entries += len;
    }
    if (!exact)
        for (int32_t i = 0; i < count; ++i)
            if (list_len[nodes[i]] == LONG_LIST)
                entries += (uint64_t)(node_ptr[nodes[i] + 1] - node_ptr[nodes[i]]) - LONG_LIST;
    return entries;
}

void estimate_batch(const Sketch &sk, QueryScratch &qs, int32_t Q, const int64_t *set_ptr, const int32_t *set_nodes,
                    uint64_t *cov, double *est, hipStream_t s);
// nq sets in CSR form on the device: sets of at most EST_MAX_SET entries whose members' lists hold
// at most EST_HASH_MAX entries are answered, heavier ones parked (cov = EST_PARKED, est = their sum
// of q, ticket 0 where ticket is not null), sets above EST_MAX_SET entries left out.  check:
// set_ptr is checked first (at most EST_BLOCK sets); else it has been.  Waits, and returns what was
// met; spare (device) takes the flags when no place in host memory is free.
EstFlags estimate_light(const Sketch &sk, int32_t nq, bool check, const int64_t *set_ptr, const int32_t *set_nodes,
                        unsigned long long *cov, double *est, uint32_t *ticket, EstFlags *spare, hipStream_t s);
// Makes the page of host memory that the flags go to, once a process (estimates themselves allocate none).
void make_flags_page();
// The sets that estimate_light parked, split over the device by windows of sample ids.  heavy
// (nq + 1 words) and ticket (nq words) are scratch.
void estimate_split(const Sketch &sk, int32_t nq, const int64_t *set_ptr, const int32_t *set_nodes,
                    unsigned long long *cov, double *est, uint32_t *heavy, uint32_t *ticket, hipStream_t s);
// A batch of the service, nq checked sets in one workgroup each, with a bitmap of T bits where the
// set's lists hold more than EST_HASH_MAX entries; the nlarge sets listed in large[] (indexes into the
// CSR: every set above EST_MAX_SET entries or EST_WALK_MAX list entries is) by the chunked path with
// one node bitmap of n bits each in nodebits.  bitmaps holds a zeroed bitmap of bitmap_words words
// for every workgroup (max(nq, nlarge) of them) and is left zeroed.  The CSR, large, cov and est may
// be pinned host memory; cov of a set that met an error is not written.  Stream-ordered; no host
// synchronisation.
void estimate_launch(const Sketch &sk, int32_t nq, const int64_t *set_ptr, const int32_t *set_nodes,
                     const int64_t *large, int32_t nlarge, uint32_t *bitmaps, uint64_t bitmap_words,
                     uint32_t *nodebits, unsigned long long *cov, double *est, int *err, EstFlags *flags, hipStream_t s);
// The ng large sets listed in qlist[g0 .. g0+ng) (set qlist[g0+b] uses bitmap b and node bitmap b).
void estimate_launch_large(const Sketch &sk, const int64_t *qlist, int64_t g0, int32_t ng, const int64_t *set_ptr,
                           const int32_t *set_nodes, uint32_t *bitmaps, uint64_t bitmap_words, uint32_t *nodebits,
                           unsigned long long *cov, double *est, int *err, hipStream_t s);
// Zero-fills count words with a kernel (capturable, unlike a memset node).
void fill_u32(uint32_t *p, uint64_t count, hipStream_t s);
void greedy(const Sketch &sk, QueryScratch &qs, int32_t k, int32_t *seeds, uint64_t *marg, uint64_t *cov_out,
            double *est_out, hipStream_t s);

} // namespace skis

// The opaque handle of the C ABI: the sketch, its estimate scratch, and a lock that
// serialises the calls that use that scratch.
struct skis_sketch {
    skis::Sketch core;
    skis::QueryScratch qs;
    std::mutex mu;
};

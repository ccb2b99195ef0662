// The sampling phase on per-minibatch bitmaps (bitmap.hip): the plan (which
// hyperbatches take it, and its sizes) and the launches.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "../../include/agnes.h"

namespace agnes {

struct Store;
struct Ctl;

constexpr int kBmThreads = 1024;              // workgroup of the first kernel
constexpr int kBmStage = 4096;                // neighbours that a sampling chunk holds in LDS
constexpr int kBmListNodes = 512;             // nodes of one list block at most
constexpr int kBmMaxH = 128;                  // minibatches
constexpr int kBmMaxB = 4096;                 // targets per minibatch (all in LDS, to be placed)
constexpr int kBmMaxK = 256;                  // node ranges
constexpr int kBmListMax = 4096;              // workgroups of the list kernel, each a row of partial statistics
constexpr int kRangeTables = 6;               // tables of about 1, 2, 4, .. 32 ranges of equal weight

struct BitmapPlan {
    bool use;
    int K, range_max;     // node ranges, and the nodes of the longest one
    const int32_t *bounds, *first_block;   // device: [K+1] first node and first list block of every range
    const int32_t* blocks;                 // device: [nb+1] first node of every list block
    int64_t nb;           // list blocks
    const int32_t* spans;    // device: first list block and the one after the last of
    int n_spans;             // every feature block that lies in several list blocks
    int rb, list_groups;     // list blocks per run, workgroups of the list kernel
    int jw;               // 32-bit words of a node's minibatch mask
    int64_t capR;         // requests of one minibatch in any hop, at most
    int64_t capE;         // sampled edges of one minibatch in any hop, at most
    int64_t capC;         // sampling chunks of one minibatch in any hop, at most
    // the block of device memory that is cleared at the start of every
    // hyperbatch: byte offsets of its parts
    size_t st1, st2, ticket, tmark, bytes;
    int64_t tmarks;       // bytes of one hop's topology-block marks
};

// Per-call values: an argument of the first kernel, or, for a captured launch
// sequence, in pinned host memory that it reads.
struct BmParams {
    const int32_t* targets;   // [H][B], device or pinned host memory
    uint64_t seed;
    int64_t mb_base;
};

// Everything the launches need; pointers are device addresses (host_*: pinned
// host memory written by the kernels).
struct BitmapArgs {
    const Store* s;
    BitmapPlan p;
    int H, B, L;
    const int32_t* fanouts;
    const int64_t* cap;       // [L+1] frontier capacities
    int64_t capN;
    int sample_groups;        // most workgroups of a looping kernel (0: its own choice)
    const BmParams* params_host;   // of a captured launch sequence; null: `given`
    BmParams given;
    BmParams* params;
    char* zero;               // the cleared block
    Ctl* ctl;
    int32_t *lsz, *host_lsz;  // [H][L+1]
    int64_t *ecount, *host_ecount;   // [H][L]
    uint32_t* host_err;       // [H]
    int32_t* nodes;           // [H][capN] local-id order
    int32_t* deg;             // [H][capR] degrees, local-id order
    uint32_t* rp;             // [H][capR] first edge of a row within its minibatch
    int32_t* cg;              // [H][capE] sampled neighbours, a chunk's grouped by range
    uint16_t* ce;             // [H][capE] their places in the chunk
    uint16_t* tab;            // [H][capC][K+1] first neighbour of every range in a chunk
    uint32_t* cbase;          // [H][capC] first edge of a chunk
    uint64_t* se[2];          // [H][capN] (node, local id), ascending by node
    int32_t* os[2];           // [H][K+1] entries of se before every range
    int32_t* rt;              // [H][nb+1] final entries of se before every list block
    int32_t *row_ptr[AGNES_MAX_LAYERS], *col[AGNES_MAX_LAYERS];
    uint64_t* list_key;       // the final list (not se[L & 1])
    int32_t* list_val;
    int64_t* node_off;        // [H+1]
    int32_t* nodes_out;
    uint32_t* part;           // pinned: [list_groups][2 + AGNES_MAX_LAYERS] distinct rows, feature blocks, topology blocks
};

// The store's degree classes, and the edges that a minibatch of B uniform targets
// is expected to sample in all hops by them.
void build_degree_classes(Store& s, const std::vector<uint32_t>& indeg, const agnes_csr& csr);
double expected_edges(const Store& s, int B, const int32_t* fanouts, int L);
BitmapPlan bitmap_plan(const Store& s, int H, int B, const int32_t* fanouts, int L, const int64_t* cap);
// What captured launches of the plan depend on, appended to `key`: two stores of
// one size, one after the other at the same addresses, differ in their node ranges.
void bitmap_key(const BitmapPlan& p, std::vector<uint64_t>& key);
// The sampling kernels up to the last hop's union: when they are done the
// layer sizes, edge counts and errors are in the pinned block.
void bitmap_hops(const BitmapArgs& a, hipStream_t st);
// The final list in (node, minibatch) order, the packed node lists and the
// statistics' partial sums.
void bitmap_list(const BitmapArgs& a, hipStream_t st);

}  // namespace agnes

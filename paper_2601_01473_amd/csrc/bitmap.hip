// The sampling phase on per-minibatch bitmaps.
//
// A minibatch's union and relabelling touch no other minibatch: its node list
// grows by the sampled neighbours it does not hold yet, in ascending node id.
// So no sort is needed.  The node range is cut into K ranges (of about equal
// in-degree weight, at most 2^17 nodes while K stays small), and one workgroup
// per (minibatch, range) keeps a bitmap of its range in LDS:
//   k_bm_sample  a workgroup takes a chunk of consecutive rows of a minibatch,
//                samples their neighbours into LDS and writes them grouped by
//                range, each with its place in the chunk (tab: where every
//                range's run begins)
//   k_bm_union   marks its range's runs of the minibatch's chunks, clears the
//                nodes already held, and what is left are the new nodes: a new
//                node's local id is the minibatch's size, plus the new nodes of
//                the lower ranges, plus its rank among the set bits.  Emits the
//                new nodes, the merged (node, local id) list, the row starts of
//                the next hop, and every edge's column.
// Two launches per hop instead of 10 to 16, and a sampled neighbour is written
// once and read twice, where the radix sort moves it three times.
//
// The gather (and the statistics) want the pairs of all minibatches in (node,
// minibatch) order.  k_bm_list builds that list from the minibatches' sorted
// lists: the union of the last hop records, per minibatch and list block (a run
// of at most 512 nodes), how many of its entries lie before the block (rt), so
// the position of a block in the list is the sum of rt over the minibatches,
// and inside the block a mask of minibatches per node gives every entry its
// place.
//
// Waits between workgroups: those of one minibatch take their range from a
// counter of that minibatch, so whoever waits for lower ranges waits for
// workgroups that already run, and these publish before they wait.  A status
// word carries its value and its flag, so no fence is needed.
#include <algorithm>
#include <cmath>

#include "bitmap.hpp"
#include "device.hpp"
#include "runtime.hpp"

namespace agnes {

// ----------------------------------------------------------------- plan

constexpr int kTicketStride = 32;                  // tickets lie on lines of their own: atomics on one line serialize
constexpr int kRunBlocks = 4;                      // list blocks of a run at most

static int xcd_grid(int64_t items, int most) {
    const int64_t g = std::max<int64_t>(1, std::min<int64_t>(items, most));
    return (int)((g + kXcds - 1) / kXcds * kXcds);
}

// Rows of one sampling chunk at fanout f: their neighbours fit the LDS stage.
// Above 32 draws a wave takes a row at a time, so a chunk has 16 rows, four per
// wave.  A whole prepare with 8 / 16 / 32 / 64 rows, in us: 97 / 96 / 102 / 116
// (2^15 nodes of degree 200, 8 x 1024, fanout 33), 105 / 110 / 121 / 138 (fanout
// 64), 232 / 203 / 200 / 199 (2^19 nodes of degree 60, 64 x 1024, fanout 40),
// 306 / 280 / 269 / 269 (16 x 1024, [7, 40]).  Alone off that line: fanout 256 of
// 2^15 nodes of degree 200, where 8 rows take 281 and 16, with twice the LDS, 429.
static int chunk_rows(int f) {
    int r = f <= 32 ? kBlock : 16;
    while (r > 1 && (int64_t)r * f > kBmStage) r >>= 1;
    return r;
}

// Class of a count: 0, 1, 2 to 3, 4 to 7, ...
static int log2_class(uint64_t x) { return x ? 64 - __builtin_clzll(x) : 0; }

void build_degree_classes(Store& s, const std::vector<uint32_t>& indeg, const agnes_csr& csr) {
    constexpr int C = 33;
    std::vector<double> count(C * C, 0.0), sum(C * C, 0.0), in(C, 0.0);
    for (int64_t v = 0; v < csr.num_nodes; v++) {
        const int64_t d = csr.offsets_dtype == AGNES_INT64
                              ? ((const int64_t*)csr.offsets)[v + 1] - ((const int64_t*)csr.offsets)[v]
                              : ((const int32_t*)csr.offsets)[v + 1] - ((const int32_t*)csr.offsets)[v];
        const int c = log2_class(indeg[(size_t)v]), x = c * C + log2_class((uint64_t)d);
        count[x] += 1.0;
        sum[x] += (double)d;
        in[c] += (double)indeg[(size_t)v];
    }
    s.degrees.clear();
    for (int c = 0; c < C; c++) {
        Store::DegreeClass k{0.0, in[c] / std::max(1.0, (double)csr.num_edges), {}};
        for (int x = c * C; x < (c + 1) * C; x++) {
            if (count[x] == 0.0) continue;
            k.cells.push_back(Store::DegreeCell{count[x], sum[x] / count[x]});
            k.nodes += count[x];
        }
        if (k.nodes > 0.0) s.degrees.push_back(k);
    }
}

// Targets are any nodes alike, a sampled neighbour is a node in proportion to
// its in-degree, and nodes that several edges reach count once.  (Within 10 % of
// what is sampled on R-MAT graphs of degree 16, 20 and 60 and on a regular one,
// 1024 and 4096 targets, 2 and 3 hops.)
double expected_edges(const Store& s, int B, const int32_t* fanouts, int L) {
    std::vector<double> held(s.degrees.size());
    for (size_t c = 0; c < held.size(); c++) held[c] = B * s.degrees[c].nodes / (double)s.num_nodes;
    double all = 0.0;
    for (int l = 0; l < L; l++) {
        double e = 0.0;
        for (size_t c = 0; c < held.size(); c++) {
            double k = 0.0;                            // sampled by all nodes of the class
            for (const auto& x : s.degrees[c].cells) k += x.nodes * std::min(x.degree, (double)fanouts[l]);
            e += held[c] * k / s.degrees[c].nodes;
        }
        all += e;
        for (size_t c = 0; c < held.size() && l + 1 < L; c++) {
            const auto& k = s.degrees[c];
            held[c] += (k.nodes - held[c]) * (1.0 - std::exp(-e * k.share / k.nodes));
        }
    }
    return all;
}

// Whether the unions' workgroups are long enough to lose against the radix sort,
// which spreads any minibatch over the whole card.  Few minibatches make few
// workgroups (H K), each of which walks its share of a minibatch's edges alone.
// In us, fitted to both sides of 160 shapes of 1 to 8 minibatches (within 5 and
// 7 %): the bitmaps 30 + 36 per hop + 16 per 1024 targets + 11.8 per 1000 edges
// of a workgroup + 21 per million edges, the radix path 35 + 100 per hop + 5 per
// 1024 targets + 62 per million edges, and above 32 draws, where its sampler
// keeps a row's draws in memory, 0.08 times their square and more.  Left to the
// radix path, bitmaps / radix: 1646 / 520 (regular graph, degree 40, 2^18 nodes,
// 1 x 4096, [20, 15, 10]), 690 / 430 (R-MAT 2^20, degree 60, the same), 479 / 390
// (regular, 1 x 1024, [15, 10, 5]); bitmaps: 309 / 386 (R-MAT 2^20, degree 20,
// 1 x 1024, [20, 15, 10]), 756 / 1213 (degree 60, 1 x 4096, [50, 50]), 317 / 398
// (regular, 8 x 4096, [10, 5]).
static bool union_is_serial(const Store& s, const BitmapPlan& p, int H, int B, const int32_t* fanouts, int L,
                            const int64_t* cap) {
    const double serial = 11.8e-3 / p.K, radix = 41e-6 * H;
    if (serial <= radix) return false;                 // (the targets alone never decide: 11 us per 1024, at most 4096)
    double less = 64.0 * L - 0.011 * B, most = 0.0;
    for (int l = 0; l < L; l++) {
        if (fanouts[l] > 32 && s.max_degree > fanouts[l]) less += 0.08 * fanouts[l] * fanouts[l];
        most += (double)cap[l] * (double)std::min<int64_t>(fanouts[l], s.max_degree);
    }
    if ((serial - radix) * most <= less) return false;  // (small ones need no closer look: 1 to 2 us of the call)
    return (serial - radix) * expected_edges(s, B, fanouts, L) > less;
}

BitmapPlan bitmap_plan(const Store& s, int H, int B, const int32_t* fanouts, int L, const int64_t* cap) {
    BitmapPlan p{};
    p.jw = H <= 32 ? 1 : H <= 64 ? 2 : 4;
    // What a minibatch samples, as a graph of this average degree suggests (half
    // the fanout or half the degree: measured between 0.4 and 1.0 of it on R-MAT
    // graphs)
    const double degree = std::max(1.0, (double)s.num_edges / (double)s.num_nodes);
    double rows = B, edges = 0.0, most_edges = 0.0;
    for (int l = 0; l < L; l++) {
        const double e = 0.5 * rows * std::min((double)fanouts[l], degree);
        edges += e;
        most_edges = std::max(most_edges, e);
        rows = std::min(rows + e, (double)s.num_nodes);
    }
    // Ranges: for about 2048 workgroups, and for about 1500 sampled neighbours
    // each, but no fewer than 64; at most 32 (and more where their length is
    // limited).
    const double want = std::min(std::max(2048.0 / H, most_edges / 1500.0), most_edges / 64.0);
    int q = 0;
    while (q + 1 < kRangeTables && (double)(1 << q) < want) q++;
    p.K = s.range_tab[q].count;
    p.range_max = s.range_tab[q].longest;
    p.bounds = s.ranges.as<int32_t>() + s.range_tab[q].at;
    p.first_block = p.bounds + p.K + 1;
    p.blocks = s.list_blocks.as<int32_t>();
    p.nb = s.n_list_blocks;
    p.capR = 0;
    p.capE = 0;
    p.capC = 0;
    for (int l = 0; l < L; l++) {
        const int rows = chunk_rows(fanouts[l]);
        p.capR = std::max<int64_t>(p.capR, cap[l]);
        p.capE = std::max<int64_t>(p.capE, cap[l] * fanouts[l]);
        p.capC = std::max<int64_t>(p.capC, (cap[l] + rows - 1) / rows);
    }
    p.spans = s.list_spans.as<int32_t>();
    p.n_spans = s.n_list_spans;
    // runs of list blocks: shorter where there are few, since a wave's blocks follow each other
    p.rb = (int)std::max<int64_t>(1, std::min<int64_t>(kRunBlocks, p.nb / 4096));
    const int64_t per_wg = (int64_t)p.rb * kWavesPerBlock;
    p.list_groups = xcd_grid((p.nb + per_wg - 1) / per_wg, s.sample_groups > 0 ? s.sample_groups : 1024);
    p.tmarks = (s.nblk + 15) / 16 * 16;
    size_t at = 0;
    auto take = [&](size_t bytes) {
        const size_t x = at;
        at = (at + bytes + 255) / 256 * 256;
        return x;
    };
    p.st1 = take((size_t)L * H * p.K * 8);
    p.st2 = take((size_t)L * H * (p.K + 1) * 8);
    p.ticket = take((size_t)L * H * kTicketStride * 4);
    p.tmark = take((size_t)L * p.tmarks);
    p.bytes = at;
    // Against the radix sort and merge-path join, in us: a workgroup of the union
    // costs what is left of its latency with as many of them in flight as LDS
    // allows (0.01 with 16 KiB of bits, 0.02 with 32, 0.06 with 64); the radix
    // path about 75 more per hop for its launches, and 0.06 per thousand edges.
    // Measured per prepare, bitmaps / radix, 32-byte rows, average degree 6 at
    // 2^25 nodes and 4 at 2^26: taken by the rule 126 / 206 (2^25 nodes, 1 x 64,
    // [5, 5]), 158 / 258 (2^25, 8 x 256, [10, 5]), 187 / 266 (2^23, 64 x 64,
    // [5, 5]), 920 / 1031 (2^23, 128 x 1024, [25, 10]), 173 / 204 (2^26, 1 x 64);
    // left to the radix path 1333 / 1103 (2^25, 64 x 1024, [15, 10, 5]),
    // 412 / 289 (2^26, 16 x 1024, [10, 5]), 4627 / 1581 (2^26, 128 x 1024,
    // [15, 10, 5]).
    // Two limits are of the kernels' layout, not of their speed.  kBmMaxH: the list
    // kernel's masks have up to four words per node.  With eight (256 minibatches of
    // 64 to 1024 targets) bitmaps took 0.57 to 0.84 of the radix path's time at 2^14
    // to 2^20 nodes, 0.97 to 1.13 at 2^22 and 2034 / 1798 at 2^23.  kBmMaxB: all of
    // a minibatch's targets are compared with each other in LDS.  With 8192 of them
    // 1.53 (2^14 nodes, 64 x 8192, [10]) to 0.87 (2^22, 16 x 8192, [10, 5]), with
    // 6000 0.67 to 0.79 (32 x 6000, [15, 10]).
    const double wg = p.range_max <= (1 << 17) ? 0.01 : p.range_max <= (1 << 18) ? 0.02 : 0.06;
    p.use = s.join_path == 0 && s.bitmaps && H <= kBmMaxH && B <= kBmMaxB && p.K <= kBmMaxK && p.capE < ((int64_t)1 << 31) &&
            (int64_t)L * s.nblk <= ((int64_t)1 << 26) && (double)H * p.K * L * wg <= 75.0 * L + 6e-5 * H * edges &&
            !union_is_serial(s, p, H, B, fanouts, L, cap);
    return p;
}

void bitmap_key(const BitmapPlan& p, std::vector<uint64_t>& key) {
    const auto a = [](const void* x) { return (uint64_t)(uintptr_t)x; };
    const uint64_t v[] = {(uint64_t)p.use, (uint64_t)p.K, (uint64_t)p.range_max, (uint64_t)p.nb, a(p.bounds),
                          a(p.blocks), (uint64_t)p.capR, (uint64_t)p.capE, (uint64_t)p.capC, (uint64_t)p.tmarks};
    key.insert(key.end(), v, v + sizeof(v) / sizeof(v[0]));
}

// ----------------------------------------------------------------- device helpers

__device__ __forceinline__ uint64_t status_load(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void status_store(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
constexpr uint64_t kReady = 1ull << 63;

// Sum of the values of status words p[0 .. n), once all of them are there.
// Called by one whole wave; every word belongs to a workgroup that runs.
__device__ __forceinline__ int64_t status_sum(const uint64_t* p, int n) {
    int64_t sum = 0;
    for (int i = lane_id(); i < n; i += kWave) {
        uint64_t v;
        while (!((v = status_load(p + i)) & kReady)) __builtin_amdgcn_s_sleep(1);
        sum += (int64_t)(v & ~kReady);
    }
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) sum += (int64_t)shfl64((uint64_t)sum, lane_id() ^ d);
    return sum;
}

// Inclusive sums and maxima over a wave by data-parallel moves between lanes
// (row shifts by 1, 2, 4 and 8, then lane 15 of a row and lane 31 to the rows
// after it): six vector instructions, where a shuffle goes through LDS six times.
// The moves are arguments, evaluated by the whole wave: inside a conditional
// they would read lanes that are switched off.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t lane_move(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
template <typename F>
__device__ __forceinline__ uint32_t wave_scan(uint32_t v, F combine) {
    v = combine(v, lane_move<0x111, 0xf>(v));
    v = combine(v, lane_move<0x112, 0xf>(v));
    v = combine(v, lane_move<0x114, 0xf>(v));
    v = combine(v, lane_move<0x118, 0xf>(v));
    v = combine(v, lane_move<0x142, 0xa>(v));
    v = combine(v, lane_move<0x143, 0xc>(v));
    return v;
}
__device__ __forceinline__ uint32_t wave_sums(uint32_t v) {
    return wave_scan(v, [](uint32_t a, uint32_t b) { return a + b; });
}
__device__ __forceinline__ uint32_t wave_maxima(uint32_t v) {
    return wave_scan(v, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
}
__device__ __forceinline__ uint32_t last_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1);
}

// Exclusive prefix sum over a workgroup of T threads; lds: T / 64 entries.
template <int T>
__device__ __forceinline__ uint32_t wg_exclusive_scan(uint32_t v, uint32_t* lds, uint32_t& total) {
    const uint32_t inc = wave_sums(v);
    if (lane_id() == kWave - 1) lds[threadIdx.x / kWave] = inc;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < T / kWave; w++) {
        const uint32_t x = lds[w];
        if (w < (int)(threadIdx.x / kWave)) base += x;
        tot += x;
    }
    __syncthreads();
    total = tot;
    return base + inc - v;
}

// Sum of v over a workgroup of T threads.
template <int T>
__device__ __forceinline__ int64_t wg_sum(int64_t v, int64_t* lds) {
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) v += (int64_t)shfl64((uint64_t)v, lane_id() ^ d);
    if (lane_id() == 0) lds[threadIdx.x / kWave] = v;
    __syncthreads();
    int64_t t = 0;
    for (int w = 0; w < T / kWave; w++) t += lds[w];
    __syncthreads();
    return t;
}

// Orders a wave's LDS accesses before the ones after it (LDS serves a wave in
// order; this keeps the compiler to it).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ----------------------------------------------------------------- targets

// Workgroup j < H: minibatch j's targets become its first B nodes, with their
// degrees and the row starts of hop 0.  A target out of range or given twice
// (found by a hash table in LDS) leaves the minibatch empty and is reported.
// Every workgroup clears a share of the block that the later kernels count in.
template <typename OffT>
__global__ __launch_bounds__(kBmThreads) void k_bm_init(BmParams given, const BmParams* prm_host, BmParams* prm, int H, int B, int L,
                                                        int64_t num_nodes, int64_t capN, int64_t capR, int32_t f,
                                                        int slots, const OffT* off, int32_t* nodes, int32_t* deg, uint32_t* rp,
                                                        int32_t* lsz, int32_t* host_lsz, int64_t* ecount,
                                                        int64_t* host_ecount, uint32_t* host_err, uint4* zero,
                                                        int64_t zero_pieces, Ctl* ctl) {
    constexpr int T = kBmThreads, M = kBmMaxB / T;
    static_assert(kBmMaxB % T == 0);
    extern __shared__ __align__(16) uint32_t seen[];   // [slots], a power of two, at least 2 B
    __shared__ uint32_t lds[T / kWave];
    __shared__ uint32_t bad;
    const int t = threadIdx.x, j = blockIdx.x;
    for (int64_t i = (int64_t)blockIdx.x * T + t; i < zero_pieces; i += (int64_t)gridDim.x * T)
        zero[i] = uint4{0u, 0u, 0u, 0u};
    if (j >= H) return;
    if (t == 0) bad = 0;
    for (int i = t; i < slots; i += T) seen[i] = ~0u;
    if (j == 0) {
        int64_t* c = (int64_t*)ctl;
        for (int i = t; i < (int)(sizeof(Ctl) / 8); i += T) c[i] = 0;
        if (t == 0) *prm = prm_host ? *prm_host : given;
    }
    const int32_t* targets = (prm_host ? prm_host->targets : given.targets) + (int64_t)j * B;
    __syncthreads();
    int32_t d[M];
#pragma unroll
    for (int m = 0; m < M; m++) {
        const int i = m * T + t;
        d[m] = 0;
        if (i >= B) continue;
        int32_t v = targets[i];
        if (v < 0 || v >= num_nodes) {
            atomicOr(&bad, 1u);
            v = 0;
        }
        nodes[(int64_t)j * capN + i] = v;
        d[m] = (int32_t)(off[v + 1] - off[v]);
        // (at least half of the slots stay free, so the search ends)
        uint32_t at = ((uint32_t)v * 2654435761u) >> 16 & (slots - 1), was;
        while ((was = atomicCAS(&seen[at], ~0u, (uint32_t)v)) != ~0u && was != (uint32_t)v) at = (at + 1) & (slots - 1);
        if (was != ~0u) atomicOr(&bad, 2u);
    }
    uint32_t run = 0;
#pragma unroll
    for (int m = 0; m < M; m++) {
        if (m * T >= B) break;
        const int i = m * T + t;
        uint32_t tot;
        const uint32_t ex = wg_exclusive_scan<T>((uint32_t)(d[m] < f ? d[m] : f), lds, tot);
        if (i < B) {
            deg[(int64_t)j * capR + i] = d[m];
            rp[(int64_t)j * capR + i] = run + ex;
        }
        run += tot;
    }
    if (t == 0) {
        const bool ok = bad == 0;                      // (the scan's barriers lie between)
        const int64_t e = ok ? (int64_t)run : 0;
        lsz[(int64_t)j * (L + 1)] = host_lsz[(int64_t)j * (L + 1)] = ok ? B : 0;
        ecount[(int64_t)j * L] = host_ecount[(int64_t)j * L] = e;
        host_err[j] = bad;
    }
}

// Minibatch j's sorted (target, index) list and how many of its targets lie below
// every range, by counting: part x of j's workgroups takes the x-th 256 of the
// B + K + 1 questions "how many targets lie below this", each against all targets
// in LDS (four per read).  The first union needs the answers, the sampling of hop
// 0 does not, so these workgroups run beside that hop's sampling.  As a bitonic
// sort in the kernel before it: 16.6 + 17.5 us for the two kernels at 32 x 1024
// targets of 2^20 nodes, fanout 15, now 7.7 + 18.6; 22.6 + 27.9 at 64 x 1024 of
// 2^23, fanout 25, now 12.8 + 31.5.  (The same sort by one workgroup of the
// sampling launch outlasts the sampling: 27 us.)
// (Targets given twice would share a place, but then the minibatch is empty.)
// sm: ceil(B / 4) uint4.
__device__ __forceinline__ void place_targets(uint4* sm, int j, int part, int B, int L, int K, const int32_t* bounds,
                                              const int32_t* lsz, const int32_t* nodes, int64_t capN, uint64_t* se,
                                              int32_t* os) {
    uint32_t* tg = (uint32_t*)sm;
    const int pieces = (B + 3) / 4;
    const bool ok = lsz[(int64_t)j * (L + 1)] > 0;
    nodes += (int64_t)j * capN;
    for (int i = threadIdx.x; i < 4 * pieces; i += kBlock) tg[i] = i < B ? (uint32_t)nodes[i] : ~0u;
    const int q = part * kBlock + (int)threadIdx.x, k = q - B;
    const uint32_t own = q >= B && k <= K ? (uint32_t)bounds[k] : 0u;
    __syncthreads();
    const uint32_t v = q < B ? tg[q] : own;
    uint32_t below = 0;
#pragma unroll 4
    for (int i = 0; i < pieces; i++) {
        const uint4 x = sm[i];
        below += (uint32_t)(x.x < v) + (uint32_t)(x.y < v) + (uint32_t)(x.z < v) + (uint32_t)(x.w < v);
    }
    if (q < B) se[(int64_t)j * capN + below] = ((uint64_t)v << 32) | (uint32_t)q;
    else if (k <= K) os[(int64_t)j * (K + 1) + k] = ok ? (int32_t)below : 0;
}

// ----------------------------------------------------------------- sampling

// Every request of the hop, in chunks of CR consecutive rows of a minibatch,
// chunk-major, so that the workgroups in flight serve about the same nodes for
// every minibatch (the new nodes of a hop are ascending), and XCD x takes the
// x-th eighth of the chunks: the adjacency lines that the minibatches share
// come into one L2.  A chunk's draws are spread over the threads:
//   1. a thread per Philox block (four draws of one row) draws the positions;
//   2. a thread per row (a wave per row for fanouts above 32) resolves Floyd's
//      collisions draw by draw (a draw that meets an earlier position takes its
//      own last one) and ranks the positions;
//   3. a thread per edge loads its neighbour and finds its node range;
//   4. the neighbours leave grouped by range, each with its place in the chunk
//      (the order inside a run is free: the union works on bits).
// A thread per row instead (all draws in registers, unrolled for the fanout)
// took 32 us for 65 thousand rows at fanout 25, most of it instruction fetch
// and one wave's own arithmetic.
// Also writes the row pointers and marks the topology blocks that the hop
// touches (plain stores of a byte each: counting them here, with an atomic per
// request, ran at the rate of a few cache lines, 100 instead of 27 us for 138
// thousand requests).
// The first `sorts` workgroups of hop 0 place the targets.
// Dynamic LDS: first row pointers [H+1], row offsets [CR], neighbours [CR f],
// sizes [H], range bounds [K+1], run ends [K], row nodes, degrees and first
// edges [CR each], places [CR f] and rows, then ranges [CR f] (16-bit).
template <typename OffT, int MAXK>
__global__ __launch_bounds__(kBlock) void k_bm_sample(int l, int L, int H, int32_t f, int CR, const BmParams* prm,
                                                      const OffT* off, const int32_t* adj, int e_blk_log2,
                                                      int64_t nblk, const int32_t* nodes, int64_t capN, int64_t capR,
                                                      int64_t capE, int64_t capC, int K, const int32_t* bounds,
                                                      const int32_t* lsz, const int64_t* ecount, const uint32_t* rp,
                                                      int32_t* cg, uint16_t* ce, uint16_t* tab, uint32_t* cbase,
                                                      int32_t* row_ptr, uint8_t* tmark, int sorts, int B,
                                                      uint64_t* se, int32_t* os) {
    extern __shared__ __align__(16) int64_t rpo[];
    if ((int)blockIdx.x < sorts) {
        const int parts = (B + K + kBlock) / kBlock, j = (int)blockIdx.x / parts;
        if (j < H) place_targets((uint4*)rpo, j, (int)blockIdx.x % parts, B, L, K, bounds, lsz, nodes, capN, se, os);
        return;
    }
    const int bid = (int)blockIdx.x - sorts, bids = (int)gridDim.x - sorts;   // (sorts: a multiple of kXcds)
    OffT* soff = (OffT*)(rpo + H + 1);
    int32_t* su = (int32_t*)(soff + CR);
    int32_t* size = su + CR * f;
    int32_t* bnd = size + H;
    uint32_t* fill = (uint32_t*)(bnd + K + 1);
    int32_t* sv = (int32_t*)(fill + K);
    int32_t* sd = sv + CR;
    uint32_t* sfirst = (uint32_t*)(sd + CR);
    uint16_t* sp = (uint16_t*)(sfirst + CR);
    uint16_t* sr = sp + CR * f;
    __shared__ int64_t lds[kWavesPerBlock];
    __shared__ uint32_t lds32[kWavesPerBlock];
    __shared__ int smax;
    __shared__ uint32_t e_first, sh_n;
    const int t = threadIdx.x;
    if (t == 0) smax = 0;
    for (int i = t; i <= K; i += kBlock) bnd[i] = bounds[i];
    __syncthreads();
    int64_t carry = 0;
    for (int b = 0; b < H; b += kBlock) {
        const int j = b + t;
        const int n = j < H ? lsz[(int64_t)j * (L + 1) + l] : 0;
        int64_t tot;
        const int64_t ex = block_exclusive_scan((int64_t)(j < H ? n + 1 : 0), lds, tot);
        if (j < H) {
            rpo[j] = carry + ex;
            size[j] = n;
            atomicMax(&smax, n);
        }
        carry += tot;
    }
    __syncthreads();
    const uint64_t seed = prm->seed;
    const int64_t mb_base = prm->mb_base;
    const int64_t items = (int64_t)((smax + CR - 1) / CR) * H;
    const int64_t per = (items + kXcds - 1) / kXcds;
    const int64_t lo = std::min<int64_t>(items, (int64_t)(bid % kXcds) * per);
    const int64_t hi = std::min<int64_t>(items, lo + per);
    const int64_t step = bids / kXcds;
    // the next request's node and row start are loaded while this one is sampled
    auto request = [&](int64_t x, int& j, int& r, int32_t& v, uint32_t& e) {
        const int c = (int)(x / H);
        j = (int)(x - (int64_t)c * H);
        const int64_t p = (int64_t)c * CR + t;
        r = t < CR && p < size[j] ? (int)p : -1;
        if (r >= 0) {
            v = nodes[(int64_t)j * capN + r];
            e = rp[(int64_t)j * capR + r];
        }
    };
    int64_t x = lo + bid / kXcds;
    int jn = 0, rn = -1;
    int32_t vn = 0;
    uint32_t en = 0;
    if (x < hi) request(x, jn, rn, vn, en);
    const int blocks4 = (f + 3) / 4;
    for (; x < hi; x += step) {
        const int j = jn, r = rn;
        const int32_t v = vn;
        const uint32_t e = en;
        if (x + step < hi) request(x + step, jn, rn, vn, en);
        const int c = (int)(x / H);
        if (c == 0 && t == 0) row_ptr[rpo[j] + size[j]] = (int32_t)ecount[(int64_t)j * L + l];
        const int rows = std::min(CR, size[j] - c * CR);
        if (rows <= 0) continue;                         // (the whole workgroup)
        if (t == 0) e_first = e;
        for (int i = t; i < K; i += kBlock) fill[i] = 0;
        int64_t o0 = 0, deg = 0;
        if (r >= 0) {
            o0 = (int64_t)off[v];
            deg = (int64_t)off[v + 1] - o0;
        }
        __syncthreads();
        const uint32_t e0 = e_first;
        if (r >= 0) {
            const int64_t blk = o0 >> e_blk_log2;
            tmark[blk < nblk ? blk : nblk - 1] = 1;
            row_ptr[rpo[j] + r] = (int32_t)e;
            soff[t] = (OffT)o0;
            sv[t] = v;
            sd[t] = (int32_t)deg;
            sfirst[t] = e - e0;
            if (t == rows - 1) sh_n = e - e0 + (uint32_t)(deg < f ? deg : f);
        }
        __syncthreads();
        const uint32_t n = sh_n;                         // the chunk's neighbours
        // 1. positions, four draws per item
        for (int i = t; i < rows * blocks4; i += kBlock) {
            const int row = i / blocks4, b = i - row * blocks4;
            const int32_t dg = sd[row];
            if (dg <= f || 4 * b >= f) continue;
            const Words4 w = philox4x64_10((uint64_t)b, (uint64_t)sv[row], (uint64_t)(mb_base + j), (uint64_t)l, seed, 0);
            int32_t* out = su + sfirst[row] + 4 * b;
            const uint64_t t1 = (uint64_t)(dg - f + 4 * b + 1);   // draw 4 b is below this
#pragma unroll
            for (int q = 0; q < 4; q++)
                if (4 * b + q < f) out[q] = (int32_t)draw_below(w.w[q], t1 + (uint64_t)q);
        }
        __syncthreads();
        // 2. collisions and ranks
        if (MAXK > 0) {
            if (r >= 0) {
                constexpr int MK = MAXK > 0 ? MAXK : 1;
                const uint32_t at = e - e0;
                const int32_t dg = (int32_t)deg;
                if (dg <= f) {                           // every neighbour: positions 0 .. k-1
                    for (int i = 0; i < dg; i++) {
                        su[at + i] = i;
                        sp[at + i] = (uint16_t)(at + i);
                        sr[at + i] = (uint16_t)t;
                    }
                } else {
                    int32_t pos[MK];
#pragma unroll
                    for (int i = 0; i < MK; i++) {
                        pos[i] = i < f ? su[at + i] : 0x7FFFFFFF;
                        bool seen = false;
#pragma unroll
                        for (int q = 0; q < i; q++) seen |= pos[q] == pos[i];
                        if (seen && i < f) pos[i] = dg - f + i;
                    }
#pragma unroll
                    for (int i = 0; i < MK; i++) {
                        if (i >= f) break;
                        int rank = 0;
#pragma unroll
                        for (int q = 0; q < MK; q++) rank += pos[q] < pos[i] ? 1 : 0;
                        su[at + i] = pos[i];
                        sp[at + i] = (uint16_t)(at + rank);
                        sr[at + i] = (uint16_t)t;
                    }
                }
            }
        } else {
            const int lane = lane_id();
            for (int row = t / kWave; row < rows; row += kWavesPerBlock) {
                const int32_t dg = sd[row];
                const uint32_t at = sfirst[row];
                if (dg <= f) {
                    for (int i = lane; i < dg; i += kWave) {
                        su[at + i] = i;
                        sp[at + i] = (uint16_t)(at + i);
                        sr[at + i] = (uint16_t)row;
                    }
                    continue;
                }
                for (int i0 = 0; i0 < f; i0 += kWave) {
                    const int m = std::min(kWave, f - i0);
                    const bool mine = lane < m;
                    int32_t pos = mine ? su[at + i0 + lane] : -1 - lane;
                    for (int i = 0; i < i0; i++)
                        if (mine && su[at + i] == pos) pos = dg - f + i0 + lane;
                    for (int i = 0; i + 1 < m; i++) {
                        const int32_t p = __builtin_amdgcn_readlane(pos, i);
                        if (lane > i && p == pos) pos = dg - f + i0 + lane;
                    }
                    if (f <= kWave) {
                        int rank = 0;
                        for (int i = 0; i < m; i++) rank += __builtin_amdgcn_readlane(pos, i) < pos ? 1 : 0;
                        if (mine) sp[at + lane] = (uint16_t)(at + rank);
                    }
                    if (mine) {
                        su[at + i0 + lane] = pos;
                        sr[at + i0 + lane] = (uint16_t)row;
                    }
                    wave_lds_fence();
                }
                if (f <= kWave) continue;
                for (int i0 = lane; i0 < f; i0 += kWave) {
                    const int32_t pos = su[at + i0];
                    int rank = 0;
                    for (int i = 0; i < f; i++) rank += su[at + i] < pos ? 1 : 0;
                    sp[at + i0] = (uint16_t)(at + rank);
                }
            }
        }
        __syncthreads();
        // 3. neighbours and their ranges, four per thread in flight
        for (uint32_t i0 = t; i0 < n; i0 += 4 * kBlock) {
            int32_t u[4];
            int g[4];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const uint32_t i = i0 + q * kBlock;
                u[q] = i < n ? adj[(int64_t)soff[sr[i]] + su[i]] : 0;
            }
            upper_segments<4>(bnd, K, u, g);
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const uint32_t i = i0 + q * kBlock;
                if (i < n) {
                    su[i] = u[q];
                    sr[i] = (uint16_t)g[q];
                    atomicAdd(&fill[g[q]], 1u);
                }
            }
        }
        __syncthreads();
        // 4. the runs
        uint32_t run = 0;
        uint16_t* tb = tab + ((int64_t)j * capC + c) * (K + 1);
        for (int g0 = 0; g0 < K; g0 += kBlock) {
            const int g = g0 + t;
            const uint32_t m = g < K ? fill[g] : 0u;
            uint32_t tot;
            const uint32_t ex = wg_exclusive_scan<kBlock>(m, lds32, tot);
            if (g < K) {
                fill[g] = run + ex;
                tb[g] = (uint16_t)(run + ex);
            }
            run += tot;
        }
        if (t == 0) {
            tb[K] = (uint16_t)n;
            cbase[(int64_t)j * capC + c] = e0;
        }
        __syncthreads();
        const int64_t base = (int64_t)j * capE + e0;
        for (uint32_t i = t; i < n; i += kBlock) {
            const uint32_t to = atomicAdd(&fill[sr[i]], 1u);
            cg[base + to] = su[i];
            ce[base + to] = sp[i];
        }
        __syncthreads();
    }
}

// ----------------------------------------------------------------- union

constexpr int kOldCap = 512;                       // held nodes of a range kept in LDS (every s-th of more)
constexpr int kNewCap = 2048;                      // new nodes listed in LDS at a time
constexpr int kUnRuns = 256;                       // runs located at a time

struct RangeMap {
    const uint64_t* bm;      // bits of the new nodes
    const uint32_t* pref;    // set bits before every four words
    // New nodes before bit x of the range.
    __device__ __forceinline__ uint32_t rank(uint32_t x) const {
        const uint32_t w = x >> 6;
        const uint64_t* q = bm + (w & ~3u);
        uint32_t r = pref[w >> 2];
#pragma unroll
        for (uint32_t i = 0; i < 4; i++) {
            const uint64_t m = i < (w & 3u) ? ~0ull : (i == (w & 3u) ? (1ull << (x & 63)) - 1ull : 0ull);
            r += (uint32_t)__popcll(q[i] & m);
        }
        return r;
    }
    __device__ __forceinline__ bool has(uint32_t x) const { return (bm[x >> 6] >> (x & 63)) & 1ull; }
};

// The held nodes of the range: se[0 .. n), of which LDS keeps every stride-th.
struct OldNodes {
    const uint64_t* se;
    const uint32_t* lds;
    int n, m, stride;
    // Entries with a node below u[q]: Q searches in lockstep.
    template <int Q>
    __device__ __forceinline__ void lower_bounds(const uint32_t (&u)[Q], int (&out)[Q]) const {
#pragma unroll
        for (int q = 0; q < Q; q++) out[q] = 0;
        int len = m;
        while (len > 1) {
            const int half = len >> 1;
#pragma unroll
            for (int q = 0; q < Q; q++) out[q] = lds[out[q] + half - 1] < u[q] ? out[q] + half : out[q];
            len -= half;
        }
#pragma unroll
        for (int q = 0; q < Q; q++) {
            if (len == 1 && lds[out[q]] < u[q]) out[q]++;
            if (stride == 1) continue;
            int b = out[q] > 0 ? (out[q] - 1) * stride + 1 : 0;
            int e = std::min(n, out[q] * stride);
            while (b < e) {
                const int mid = (b + e) >> 1;
                if ((uint32_t)(se[mid] >> 32) < u[q]) b = mid + 1; else e = mid;
            }
            out[q] = b;
        }
    }
};

// Workgroup (j, k): the union and relabelling of minibatch j in range k (see
// the top).  A chain of dependent loads (ticket, runs, neighbours, status of the
// lower ranges, offsets) around a little LDS work, so what counts is how many
// workgroups are in flight: 256 threads and 16 KiB of bits for 2^17 nodes.  The
// workgroups of a minibatch are dealt to one XCD, whose L2 collects the columns
// they store alone.
// f_next: the next hop's fanout, or -1 after the last hop, which writes rt.
// Dynamic LDS: bits, prefix counts, bounds, list entries before every range.
template <typename OffT, int T>
__global__ __launch_bounds__(T, 6) void k_bm_union(
    int l, int L, int H, int K, const int32_t* bounds, const int32_t* first_block, const int32_t* blocks,
    int range_max, int64_t capN, int64_t capR, int64_t capE, int64_t capC, int CR, int32_t f_next, const OffT* off,
    const int32_t* cg, const uint16_t* ce, const uint16_t* tab, const uint32_t* cbase, const uint64_t* se_in, uint64_t* se_out,
    const int32_t* os_in, int32_t* os_out, int32_t* lsz, int32_t* host_lsz, int64_t* ecount, int64_t* host_ecount,
    uint64_t* st1, uint64_t* st2, uint32_t* ticket, int32_t* nodes, int32_t* deg, uint32_t* rp, int32_t* col,
    int32_t* rt, int64_t nb) {
    constexpr int W = T / kWave;
    extern __shared__ __align__(16) uint64_t bm[];
    uint32_t* pref = (uint32_t*)(bm + range_max / 64);   // (range_max: a multiple of 256)
    __shared__ uint32_t oldn[kOldCap], newx[kNewCap];
    __shared__ uint32_t run_at[kUnRuns], run_e[kUnRuns];
    __shared__ uint16_t run_len[kUnRuns];
    __shared__ uint32_t lds[W];
    __shared__ int64_t lds64[W];
    __shared__ int64_t sh_before, sh_edges;              // (two words: no barrier need lie between the first's readers
    __shared__ int sh_k;                                 // and the second's writer where a range has no new nodes)
    const int t = threadIdx.x, w = t / kWave, lane = lane_id();
    const int parts = f_next >= 0 ? K + 1 : K;            // with the held nodes' row starts
    const int j = (int)((blockIdx.x / kXcds) / parts) * kXcds + (int)(blockIdx.x % kXcds);
    if (j >= H) return;
    if (t == 0) sh_k = (int)atomicAdd(&ticket[j * kTicketStride], 1u) + K - parts;
    const int size = lsz[(int64_t)j * (L + 1) + l];
    int64_t before = 0;
    for (int x = t; x < j; x += T) before += ecount[(int64_t)x * L + l];
    const int64_t col0 = wg_sum<T>(before, lds64);       // (its barriers publish sh_k)
    const int k = sh_k;
    // the first ticket: row starts of the held nodes under the next fanout
    if (k < 0) {
        uint32_t run = 0;
        for (int i0 = 0; i0 < size; i0 += 8 * T) {
            const int i = i0 + 8 * t;
            uint32_t c[8], sum = 0;
#pragma unroll
            for (int q = 0; q < 8; q++) {
                const int32_t d = i + q < size ? deg[(int64_t)j * capR + i + q] : 0;
                c[q] = (uint32_t)(d < f_next ? d : f_next);
                sum += c[q];
            }
            uint32_t tot;
            uint32_t ex = run + wg_exclusive_scan<T>(sum, lds, tot);
#pragma unroll
            for (int q = 0; q < 8; q++) {
                if (i + q < size) rp[(int64_t)j * capR + i + q] = ex;
                ex += c[q];
            }
            run += tot;
        }
        if (t == 0) status_store(&st2[(int64_t)j * (K + 1)], kReady | run);
        return;
    }
    const uint32_t r0 = (uint32_t)bounds[k], range = (uint32_t)bounds[k + 1] - r0;
    const int ob = os_in[(int64_t)j * (K + 1) + k], oe = os_in[(int64_t)j * (K + 1) + k + 1];
    const int words = (int)((range + 255) >> 8) * 4;      // whole groups of four
    for (int i = t; i < words; i += T) bm[i] = 0;
    const int chunks = (size + CR - 1) / CR;
    const int64_t edges = (int64_t)j * capE;
    // the runs of chunks c0 .. of this range
    auto locate = [&](int c0) {
        const int c = c0 + t;
        if (t >= kUnRuns) {
        } else if (c < chunks) {
            const uint16_t* tb = tab + ((int64_t)j * capC + c) * (K + 1) + k;
            const uint32_t e0 = cbase[(int64_t)j * capC + c];
            const uint32_t a = tb[0];
            run_e[t] = e0;
            run_at[t] = e0 + a;
            run_len[t] = (uint16_t)(tb[1] - a);
        } else {
            run_e[t] = run_at[t] = 0;
            run_len[t] = 0;
        }
        __syncthreads();
    };
    // calls fn(i, at, len, e0) with the i-th entries of four runs: a group of 16,
    // 32 or 64 lanes per run, by the runs' average length
    const int64_t E = ecount[(int64_t)j * L + l], avg = E / std::max<int64_t>(1, (int64_t)chunks * K);
    const int lanes = avg <= 12 ? 16 : (avg <= 24 ? 32 : 64), per = kWave / lanes;
    auto walk = [&](int c0, auto&& fn) {
        const int n = std::min(kUnRuns, chunks - c0), sub = lane / lanes;
        for (int g = w * 4 * per; g < n; g += W * 4 * per) {
            uint32_t at[4], len[4], e0[4], most = 0;
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int r = g + q * per + sub;              // (below kUnRuns: runs past the last are empty)
                at[q] = run_at[r];
                e0[q] = run_e[r];
                len[q] = run_len[r];
                most = std::max(most, len[q]);
            }
            for (uint32_t i = lane % lanes; i < most; i += lanes) fn(i, at, len, e0);
        }
    };
    OldNodes old;
    old.se = se_in + (int64_t)j * capN + ob;
    old.n = oe - ob;
    old.stride = std::max(1, (old.n + kOldCap - 1) / kOldCap);
    old.m = (old.n + old.stride - 1) / old.stride;
    old.lds = oldn;
    for (int i = t; i < old.m; i += T) oldn[i] = (uint32_t)(old.se[(int64_t)i * old.stride] >> 32);
    for (int c0 = 0; c0 < chunks; c0 += kUnRuns) {
        if (c0 > 0) __syncthreads();
        locate(c0);                                       // (its barrier also publishes the cleared bits)
        walk(c0, [&](uint32_t i, const uint32_t* at, const uint32_t* len, const uint32_t*) {
            uint32_t x[4];
#pragma unroll
            for (int q = 0; q < 4; q++)
                x[q] = i < len[q] ? (uint32_t)cg[edges + at[q] + i] - r0 : 0xFFFFFFFFu;
#pragma unroll
            for (int q = 0; q < 4; q++)
                if (i < len[q]) atomicOr((uint32_t*)bm + (x[q] >> 5), 1u << (x[q] & 31));
        });
    }
    __syncthreads();
    if (old.stride == 1) {
        for (int i = t; i < old.n; i += T) {
            const uint32_t x = oldn[i] - r0;
            atomicAnd((uint32_t*)bm + (x >> 5), ~(1u << (x & 31)));
        }
    } else {
        for (int i = t; i < old.n; i += T) {
            const uint32_t x = (uint32_t)(old.se[i] >> 32) - r0;
            atomicAnd((uint32_t*)bm + (x >> 5), ~(1u << (x & 31)));
        }
    }
    __syncthreads();
    uint32_t nn = 0;                                      // new nodes of the range
    for (int g0 = 0; g0 < words; g0 += 4 * T) {           // four consecutive words per thread
        const int g = g0 + 4 * t;
        uint32_t sum = 0;
        if (g < words) {
#pragma unroll
            for (int q = 0; q < 4; q++) sum += (uint32_t)__popcll(bm[g + q]);
        }
        uint32_t tot;
        const uint32_t ex = nn + wg_exclusive_scan<T>(sum, lds, tot);
        if (g < words) pref[g >> 2] = ex;
        nn += tot;
    }
    if (t == 0) status_store(&st1[(int64_t)j * K + k], kReady | nn);
    if (w == 0) {
        const int64_t v = status_sum(st1 + (int64_t)j * K, k);
        if (lane == 0) sh_before = v;
    }
    __syncthreads();                                      // (prefix counts complete, too)
    const int pre = (int)sh_before;
    const int first = size + pre;                         // local id of the range's first new node
    const RangeMap map{bm, pref};
    if (t == 0) {
        os_out[(int64_t)j * (K + 1) + k] = ob + pre;
        if (k == K - 1) {
            const int n = first + (int)nn;
            os_out[(int64_t)j * (K + 1) + K] = n;
            lsz[(int64_t)j * (L + 1) + l + 1] = host_lsz[(int64_t)j * (L + 1) + l + 1] = n;
            if (rt) rt[(int64_t)j * (nb + 1) + nb] = n;
        }
    }
    // new nodes in ascending order, kNewCap at a time: listed in LDS by the
    // threads that hold their words, then written by consecutive threads
    uint32_t run = 0;
    uint64_t* out = se_out + (int64_t)j * capN + ob + pre;
    for (uint32_t b0 = 0; b0 < nn; b0 += kNewCap) {
        if (b0 > 0) __syncthreads();
        for (int i = t; i < words; i += T) {
            uint64_t bits = bm[i];
            if (!bits) continue;
            uint32_t r = pref[i >> 2];
            for (int q = i & ~3; q < i; q++) r += (uint32_t)__popcll(bm[q]);
            r -= b0;                                          // (a word before the window wraps to a large value)
            if ((int32_t)r >= kNewCap || (int32_t)r <= -kWave) continue;
            while (bits) {
                if (r < (uint32_t)kNewCap) newx[r] = (uint32_t)i * 64 + (uint32_t)__ffsll((unsigned long long)bits) - 1;
                bits &= bits - 1;
                r++;
            }
        }
        __syncthreads();
        const uint32_t bn = std::min<uint32_t>(kNewCap, nn - b0);
        constexpr int Q = 2;                                  // nodes of a thread in flight
        for (uint32_t i0 = 0; i0 < bn; i0 += Q * T) {
            uint32_t u[Q];
            int lb[Q];
#pragma unroll
            for (int q = 0; q < Q; q++) {
                const uint32_t i = i0 + q * T + t;
                u[q] = r0 + (i < bn ? newx[i] : 0u);
            }
            int32_t d[Q] = {};
            if (f_next >= 0) {
#pragma unroll
                for (int q = 0; q < Q; q++)
                    if (i0 + q * T + t < bn) d[q] = (int32_t)(off[u[q] + 1] - off[u[q]]);
            }
            old.lower_bounds<Q>(u, lb);
#pragma unroll
            for (int q = 0; q < Q; q++) {
                const uint32_t i = i0 + q * T + t;
                if (i >= bn) continue;
                const int loc = first + (int)(b0 + i);
                nodes[(int64_t)j * capN + loc] = (int32_t)u[q];
                out[lb[q] + b0 + i] = ((uint64_t)u[q] << 32) | (uint32_t)loc;
            }
            if (f_next >= 0) {
#pragma unroll
                for (int q = 0; q < Q; q++) {
                    const uint32_t i = i0 + q * T + t;
                    if (i0 + q * T >= bn) break;
                    const uint32_t c = i < bn ? (uint32_t)(d[q] < f_next ? d[q] : f_next) : 0u;
                    uint32_t tot;
                    const uint32_t ex = wg_exclusive_scan<T>(c, lds, tot);
                    if (i < bn) {
                        deg[(int64_t)j * capR + first + b0 + i] = d[q];
                        rp[(int64_t)j * capR + first + b0 + i] = run + ex;   // the lower ranges' edges are added below
                    }
                    run += tot;
                }
            }
        }
    }
    if (f_next >= 0 && t == 0) status_store(&st2[(int64_t)j * (K + 1) + k + 1], kReady | run);
    // the held nodes move up by the new nodes below them
    for (int i = t; i < old.n; i += T) {
        const uint64_t e = old.se[i];
        out[i + map.rank((uint32_t)(e >> 32) - r0)] = e;
    }
    if (rt) {
        const int b0 = first_block[k], b1 = first_block[k + 1];
        for (int i0 = b0; i0 < b1; i0 += 4 * T) {
            uint32_t u[4];
            int lb[4];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int i = i0 + q * T + t;
                u[q] = i < b1 ? (uint32_t)blocks[i] : r0;
            }
            old.lower_bounds<4>(u, lb);
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int i = i0 + q * T + t;
                if (i < b1) rt[(int64_t)j * (nb + 1) + i] = ob + pre + lb[q] + (int)map.rank(u[q] - r0);
            }
        }
    }
    // every edge's column
    for (int c0 = 0; c0 < chunks; c0 += kUnRuns) {
        if (chunks > kUnRuns) {
            __syncthreads();
            locate(c0);
        }
        walk(c0, [&](uint32_t i, const uint32_t* at, const uint32_t* len, const uint32_t* e0) {
            uint32_t u[4], x[4], e[4];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const bool on = i < len[q];
                u[q] = on ? (uint32_t)cg[edges + at[q] + i] : r0;
                e[q] = on ? e0[q] + ce[edges + at[q] + i] : 0u;
            }
            bool held = false;
            int32_t loc[4];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                x[q] = u[q] - r0;
                const bool is_new = map.has(x[q]);
                loc[q] = is_new ? first + (int)map.rank(x[q]) : -1;
                held |= i < len[q] && !is_new;
            }
            if (held) {
                int lb[4];
                old.lower_bounds<4>(u, lb);
#pragma unroll
                for (int q = 0; q < 4; q++)
                    if (i < len[q] && loc[q] < 0) loc[q] = (int32_t)(uint32_t)old.se[lb[q]];
            }
#pragma unroll
            for (int q = 0; q < 4; q++)
                if (i < len[q]) col[col0 + e[q]] = loc[q];
        });
    }
    // row starts: the edges of the held nodes and of the lower ranges' new nodes
    if (f_next >= 0) {
        if (w == 0) {
            const int64_t v = status_sum(st2 + (int64_t)j * (K + 1), k + 1);
            if (lane == 0) sh_edges = v;
        }
        __syncthreads();
        const uint32_t base = (uint32_t)sh_edges;        // (this workgroup's row starts are written: barriers between)
        for (uint32_t i = t; i < nn; i += T) rp[(int64_t)j * capR + first + i] += base;
        if (k == K - 1 && t == 0) {
            const int64_t e = (int64_t)base + run;
            ecount[(int64_t)j * L + l + 1] = host_ecount[(int64_t)j * L + l + 1] = e;
        }
    }
}

// ----------------------------------------------------------------- list

// The final list in (node, minibatch) order: value = local id.  A wave takes
// runs of kRunBlocks consecutive list blocks: one load per lane and block
// boundary brings the run's rt words, then each block's entries (consecutive in
// every minibatch's sorted list) are loaded while the block before is placed.
// List blocks have about equal in-degree weight (with blocks of equal length a
// skewed graph's dense blocks, whose ids are alike in their low bits, fell to a
// few workgroups: 466 us at 2^23 nodes), and the runs go to the XCDs in turn.
// Also packs the node lists into the output, and counts the distinct rows, the
// topology blocks that were marked and the feature blocks: a list block holds
// whole feature blocks or a piece of one; those of the second kind (spans: their
// first list block and the one after their last) hold rows if rt grows over them.
constexpr int kLightRounds = 4;
constexpr int kLightEntries = kLightRounds * kWave;   // entries of a block kept in registers
constexpr int kListItems = 8;                         // entries per thread per round of the packing

// 32-bit words of one wave's LDS: masks, entries before every node, heads of the
// minibatches' entries, entries of the minibatches before, the run's rt words.
static constexpr int list_wave_words(int H, int jw) {
    return (kBmListNodes * jw + kBmListNodes + 4 + kLightEntries + (H + 1) + (kRunBlocks + 1) * H + 3) / 4 * 4;
}

template <int JW>
__global__ __launch_bounds__(kBlock) void k_bm_list(int H, int L, int64_t num_nodes, int64_t nb, const int32_t* blocks, int rb,
                                                    int64_t capN, const uint64_t* se, const int32_t* rt,
                                                    const int32_t* lsz, const int32_t* nodes_ws, uint32_t rpb,
                                                    const int32_t* spans, int n_spans, const uint8_t* tmark,
                                                    int64_t tmarks, uint64_t* list_key, int32_t* list_val,
                                                    int64_t* node_off_g, int32_t* nodes_out, uint32_t* part,
                                                    Ctl* ctl) {
    extern __shared__ __align__(16) int64_t list_sm[];
    int64_t* node_off = list_sm;                       // [H+1]
    uint32_t* wave_sm = (uint32_t*)(list_sm + (H + 2) / 2 * 2);   // (16-byte aligned)
    __shared__ int64_t lds[kWavesPerBlock];
    __shared__ uint32_t cnt[2 + AGNES_MAX_LAYERS];
    const int t = threadIdx.x, w = wave_id(), lane = lane_id();
    uint32_t* mask = wave_sm + w * list_wave_words(H, JW);   // [kBmListNodes][JW]
    uint32_t* pref = mask + kBmListNodes * JW;         // [kBmListNodes+4]
    uint32_t* heads = pref + kBmListNodes + 4;         // [kLightEntries]
    uint32_t* jpre = heads + kLightEntries;            // [H+1]
    uint32_t* rtl = jpre + H + 1;                      // [kRunBlocks+1][H]
    if (t < 2 + AGNES_MAX_LAYERS) cnt[t] = 0;
    uint32_t nd = 0, nf = 0;
    // Opens block i of the run and loads its first entries: minibatch jj and
    // (node, local id) ent of entries lane, 64 + lane, ...  Returns the entries.
    uint64_t ent[kLightRounds];
    int jj[kLightRounds];
    auto open = [&](int i) -> uint32_t {
        uint32_t n = 0;
#pragma unroll
        for (int r = 0; r < kLightRounds; r++) heads[r * kWave + lane] = 0;
        wave_lds_fence();
        for (int j0 = 0; j0 < H; j0 += kWave) {
            const int j = j0 + lane;
            const uint32_t c = j < H ? rtl[(i + 1) * H + j] - rtl[i * H + j] : 0u;
            const uint32_t inc = wave_sums(c);
            if (j < H) jpre[j] = n + inc - c;
            if (c > 0 && n + inc - c < (uint32_t)kLightEntries) heads[n + inc - c] = (uint32_t)j + 1;
            n += last_lane(inc);
        }
        if (lane == 0) jpre[H] = n;
        wave_lds_fence();
        uint32_t carry = 0;
#pragma unroll
        for (int r = 0; r < kLightRounds; r++) {
            const uint32_t x = r * kWave + lane;
            jj[r] = 0;
            ent[r] = 0;
            if ((uint32_t)(r * kWave) >= n) continue;
            const uint32_t h = wave_maxima(std::max(heads[x], lane == 0 ? carry : 0u));
            carry = last_lane(h);
            if (x < n) {
                const int j = (int)h - 1;
                jj[r] = j;
                ent[r] = se[(int64_t)j * capN + rtl[i * H + j] + (x - jpre[j])];
            }
        }
        return n;
    };
    const int64_t runs = (nb + rb - 1) / rb;           // (rb <= kRunBlocks)
    const int64_t turns = (runs + kWavesPerBlock * kXcds - 1) / (kWavesPerBlock * kXcds);
    for (int64_t y = blockIdx.x / kXcds; y < turns; y += gridDim.x / kXcds) {
        const int64_t b0 = ((y * kXcds + blockIdx.x % kXcds) * kWavesPerBlock + w) * rb;
        if (b0 >= nb) continue;
        const int m = (int)std::min<int64_t>(rb, nb - b0);
        int64_t base = 0;
        for (int j0 = 0; j0 < H; j0 += kWave) {
            const int j = j0 + lane;
            int64_t s = 0;
            if (j < H) {
                const int32_t* p = rt + (int64_t)j * (nb + 1) + b0;
                uint32_t v[kRunBlocks + 1];
#pragma unroll
                for (int i = 0; i <= kRunBlocks; i++) v[i] = i <= m ? (uint32_t)p[i] : 0u;
#pragma unroll
                for (int i = 0; i <= kRunBlocks; i++) rtl[i * H + j] = v[i];
                s = v[0];
            }
#pragma unroll
            for (int d = kWave / 2; d > 0; d >>= 1) s += (int64_t)shfl64((uint64_t)s, lane ^ d);
            base += s;
        }
        const int32_t edge = lane <= m ? blocks[b0 + lane] : 0;
        wave_lds_fence();
        uint32_t n = open(0);
        for (int i = 0; i < m; i++) {
            const uint32_t n0 = (uint32_t)__shfl(edge, i, kWave);
            const int bn = __shfl(edge, i + 1, kWave) - (int)n0;
            uint64_t e[kLightRounds];
            int ej[kLightRounds];
#pragma unroll
            for (int r = 0; r < kLightRounds; r++) {
                e[r] = ent[r];
                ej[r] = jj[r];
            }
            const uint32_t next = i + 1 < m ? (n > (uint32_t)kLightEntries ? 0u : open(i + 1)) : 0u;
            if (n > 0) {
                for (int x = lane; x < (bn * JW + 3) / 4; x += kWave) ((uint4*)mask)[x] = uint4{0u, 0u, 0u, 0u};
                wave_lds_fence();
                auto mark = [&](const uint64_t* en, const int* mj, uint32_t x0) {
#pragma unroll
                    for (int r = 0; r < kLightRounds; r++)
                        if (x0 + r * kWave + lane < n)
                            atomicOr(&mask[((uint32_t)(en[r] >> 32) - n0) * JW + (JW > 1 ? mj[r] >> 5 : 0)], 1u << (mj[r] & 31));
                };
                auto place = [&](const uint64_t* en, const int* mj, uint32_t x0) {
#pragma unroll
                    for (int r = 0; r < kLightRounds; r++)
                        if (x0 + r * kWave + lane < n) {
                            const uint32_t at = (uint32_t)(en[r] >> 32) - n0;
                            const uint32_t* q = mask + at * JW;
                            uint32_t to = pref[at];
#pragma unroll
                            for (int x = 0; x < JW; x++) {
                                const uint32_t below = (1u << (mj[r] & 31)) - 1u;
                                to += __popc(q[x] & (x < (mj[r] >> 5) ? ~0u : x == (mj[r] >> 5) ? below : 0u));
                            }
                            list_key[base + to] = (en[r] & 0xFFFFFFFF00000000ull) | (uint32_t)mj[r];
                            list_val[base + to] = (int32_t)(uint32_t)en[r];
                        }
                };
                mark(e, ej, 0);
                // a block of more entries than registers hold (rare): the
                // others are loaded where they are used
                for (uint32_t x0 = kLightEntries; x0 < n; x0 += kLightEntries) {
                    uint64_t en[kLightRounds];
                    int mj[kLightRounds];
#pragma unroll
                    for (int r = 0; r < kLightRounds; r++) {
                        const uint32_t x = x0 + r * kWave + lane;
                        mj[r] = x < n ? upper_segment(jpre, H, x) : 0;
                        en[r] = x < n ? se[(int64_t)mj[r] * capN + rtl[i * H + mj[r]] + (x - jpre[mj[r]])] : 0;
                    }
                    mark(en, mj, x0);
                }
                wave_lds_fence();
                uint32_t run = 0;                      // four consecutive nodes per lane
                for (int x0 = 0; x0 < bn; x0 += 4 * kWave) {
                    const int x = x0 + 4 * lane;
                    uint32_t c[4], sum = 0;
                    uint4 v[JW];                       // 4 JW consecutive words
#pragma unroll
                    for (int q = 0; q < JW; q++)
                        v[q] = 4 * q < (bn - x) * JW ? ((const uint4*)mask)[(x * JW) / 4 + q] : uint4{0u, 0u, 0u, 0u};
                    const uint32_t* words = (const uint32_t*)v;
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        c[q] = 0;
#pragma unroll
                        for (int y1 = 0; y1 < JW; y1++) c[q] += __popc(words[q * JW + y1]);
                        nd += c[q] > 0;
                        sum += c[q];
                    }
                    const uint32_t inc = wave_sums(sum);
                    uint32_t ex = run + inc - sum;
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        if (x + q < bn) pref[x + q] = ex;
                        ex += c[q];
                    }
                    run += last_lane(inc);
                }
                if (lane == 0) pref[bn] = run;
                wave_lds_fence();
                place(e, ej, 0);
                for (uint32_t x0 = kLightEntries; x0 < n; x0 += kLightEntries) {
                    uint64_t en[kLightRounds];
                    int mj[kLightRounds];
#pragma unroll
                    for (int r = 0; r < kLightRounds; r++) {
                        const uint32_t x = x0 + r * kWave + lane;
                        mj[r] = x < n ? upper_segment(jpre, H, x) : 0;
                        en[r] = x < n ? se[(int64_t)mj[r] * capN + rtl[i * H + mj[r]] + (x - jpre[mj[r]])] : 0;
                    }
                    place(en, mj, x0);
                }
                // whole feature blocks
                if (n0 % rpb == 0 && ((uint32_t)bn % rpb == 0 || n0 + bn == (uint32_t)num_nodes))
                    for (uint32_t x = lane * rpb; x < (uint32_t)bn; x += kWave * rpb)
                        nf += pref[std::min<uint32_t>(x + rpb, (uint32_t)bn)] > pref[x];
                wave_lds_fence();
            }
            base += n;
            n = n > (uint32_t)kLightEntries && i + 1 < m ? open(i + 1) : next;
        }
    }
    // feature blocks in several list blocks
    for (int64_t i = (int64_t)blockIdx.x * kWavesPerBlock + w; i < n_spans; i += (int64_t)gridDim.x * kWavesPerBlock) {
        const int32_t s0 = spans[2 * i], s1 = spans[2 * i + 1];
        bool any = false;
        for (int j = lane; j < H; j += kWave) any |= rt[(int64_t)j * (nb + 1) + s1] > rt[(int64_t)j * (nb + 1) + s0];
        if (__any(any) && lane == 0) nf++;
    }
    __syncthreads();                                   // cnt is cleared
    // topology blocks: byte marks set
    for (int l = 0; l < L; l++) {
        const uint32_t* m = (const uint32_t*)(tmark + (int64_t)l * tmarks);
        uint32_t c = 0;
        for (int64_t i = (int64_t)blockIdx.x * kBlock + t; i < tmarks / 4; i += (int64_t)gridDim.x * kBlock)
            c += __popc(m[i]);
        c = wave_sums(c);
        if (lane == kWave - 1 && c) atomicAdd(&cnt[2 + l], c);
    }
    // the output node lists: read and written in consecutive order, all of a
    // round's entries loaded before any is stored
    int64_t rows = 0;
    for (int b = 0; b < H; b += kBlock) {
        const int j = b + t;
        int64_t tot;
        const int64_t ex = block_exclusive_scan((int64_t)(j < H ? lsz[(int64_t)j * (L + 1) + L] : 0), lds, tot);
        if (j < H) node_off[j] = rows + ex;
        rows += tot;
    }
    if (t == 0) node_off[H] = rows;
    __syncthreads();
    if (blockIdx.x == 0) {
        for (int j = t; j <= H; j += kBlock) node_off_g[j] = node_off[j];
        if (t == 0) ctl->rows = rows;
    }
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t b = (int64_t)blockIdx.x * kBlock + t; b < rows; b += stride * kListItems) {
        int64_t x[kListItems];
        int j[kListItems];
        int32_t v[kListItems];
#pragma unroll
        for (int i = 0; i < kListItems; i++) x[i] = std::min<int64_t>(b + i * stride, rows - 1);
        upper_segments<kListItems>(node_off, H, x, j);
#pragma unroll
        for (int i = 0; i < kListItems; i++) v[i] = nodes_ws[(int64_t)j[i] * capN + (x[i] - node_off[j[i]])];
#pragma unroll
        for (int i = 0; i < kListItems; i++)
            if (b + i * stride < rows) nodes_out[b + i * stride] = v[i];
    }
    nd = wave_sums(nd);
    nf = wave_sums(nf);
    if (lane == kWave - 1) {
        if (nd) atomicAdd(&cnt[0], nd);
        if (nf) atomicAdd(&cnt[1], nf);
    }
    __syncthreads();
    // (a row per workgroup, added up on the host: atomics on a few lines would serialize)
    if (t < 2 + L) part[(int64_t)blockIdx.x * (2 + AGNES_MAX_LAYERS) + t] = cnt[t];
}

// ----------------------------------------------------------------- launches

template <typename Fn>
static void allow_lds(Fn* kernel, size_t bytes) {
    if (bytes > 65536)
        AGNES_CHECK_HIP(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
}

template <typename OffT>
static void hops(const BitmapArgs& a, hipStream_t st) {
    const Store& s = *a.s;
    const BitmapPlan& p = a.p;
    const OffT* off = s.offsets.as<OffT>();
    const int H = a.H, L = a.L;
    const int extra = (int)std::min<int64_t>(64, (int64_t)(p.bytes >> 16));
    int slots = 64;                                    // (8192 at most, 32 KiB)
    while (slots < 2 * a.B) slots <<= 1;
    AGNES_LAUNCH((k_bm_init<OffT>), dim3(H + extra), dim3(kBmThreads), (size_t)slots * 4, st, a.given, a.params_host, a.params, H, a.B, L,
                 s.num_nodes, a.capN, p.capR, a.fanouts[0], slots, off, a.nodes, a.deg, a.rp, a.lsz, a.host_lsz, a.ecount,
                 a.host_ecount, a.host_err, (uint4*)a.zero, (int64_t)(p.bytes / 16), a.ctl);
    const size_t union_lds = (size_t)p.range_max / 256 * 36;
    for (int l = 0; l < L; l++) {
        const int32_t f = a.fanouts[l];
        const int cur = l & 1, CR = chunk_rows(f);
        const int most = a.sample_groups > 0 ? a.sample_groups : 2048;
        const int g = xcd_grid((int64_t)H * ((a.cap[l] + CR - 1) / CR), most);
        const int sorts = l == 0 ? (H * ((a.B + p.K + kBlock) / kBlock) + kXcds - 1) / kXcds * kXcds : 0;
        const size_t sample_lds = std::max((size_t)(H + 1) * 8 + (size_t)CR * (sizeof(OffT) + 12) + (size_t)CR * f * 8 +
                                               (size_t)(H + 2 * p.K + 1) * 4,
                                           sorts > 0 ? (size_t)(a.B + 3) / 4 * 16 : (size_t)0);
        uint8_t* tm = (uint8_t*)(a.zero + p.tmark) + (int64_t)l * p.tmarks;
#define AGNES_BM_SAMPLE(MK)                                                                                    \
    AGNES_LAUNCH((k_bm_sample<OffT, MK>), dim3(sorts + g), dim3(kBlock), sample_lds, st, l, L, H, f, CR, a.params,      \
                 off, s.indices.as<int32_t>(), s.e_blk_log2, s.nblk, a.nodes, a.capN, p.capR, p.capE, p.capC,  \
                 p.K, p.bounds, a.lsz, a.ecount, a.rp, a.cg, a.ce, a.tab, a.cbase, a.row_ptr[l], tm, sorts, a.B,    \
                 a.se[0], a.os[0])
        // (the pairs compared grow with the square of the bound: common fanouts get their own)
        if (f <= 5) AGNES_BM_SAMPLE(5);
        else if (f <= 10) AGNES_BM_SAMPLE(10);
        else if (f <= 15) AGNES_BM_SAMPLE(15);
        else if (f <= 20) AGNES_BM_SAMPLE(20);
        else if (f <= 25) AGNES_BM_SAMPLE(25);
        else if (f <= 32) AGNES_BM_SAMPLE(32);
        else AGNES_BM_SAMPLE(0);
#undef AGNES_BM_SAMPLE
        const bool last = l + 1 == L;
        const int gu = (H + kXcds - 1) / kXcds * kXcds * (p.K + (last ? 0 : 1));
#define AGNES_BM_UNION(T)                                                                                         \
    AGNES_LAUNCH((k_bm_union<OffT, T>), dim3(gu), dim3(T), union_lds, st, l, L, H, p.K, p.bounds, p.first_block,  \
                 p.blocks, p.range_max, a.capN, p.capR, p.capE, p.capC, CR, last ? -1 : a.fanouts[l + 1], off,    \
                 a.cg, a.ce, a.tab, a.cbase, a.se[cur], a.se[cur ^ 1], a.os[cur], a.os[cur ^ 1], a.lsz,           \
                 a.host_lsz, a.ecount, a.host_ecount, (uint64_t*)(a.zero + p.st1) + (int64_t)l * H * p.K,         \
                 (uint64_t*)(a.zero + p.st2) + (int64_t)l * H * (p.K + 1),                                        \
                 (uint32_t*)(a.zero + p.ticket) + (int64_t)l * H * kTicketStride, a.nodes, a.deg, a.rp, a.col[l], \
                 last ? a.rt : nullptr, p.nb)
        // (longer ranges take more LDS: as many waves in flight with more threads each)
        if (p.range_max <= (1 << 17)) AGNES_BM_UNION(256);
        else {
            allow_lds(&k_bm_union<OffT, 512>, union_lds);
            AGNES_BM_UNION(512);
        }
#undef AGNES_BM_UNION
    }
    AGNES_CHECK_HIP(hipGetLastError());
}

void bitmap_hops(const BitmapArgs& a, hipStream_t st) {
    if (a.s->offsets64) hops<int64_t>(a, st);
    else hops<int32_t>(a, st);
}

void bitmap_list(const BitmapArgs& a, hipStream_t st) {
    const Store& s = *a.s;
    const BitmapPlan& p = a.p;
    const size_t lds = ((size_t)(a.H + 1) * 8 + 15) / 16 * 16 + (size_t)kWavesPerBlock * list_wave_words(a.H, p.jw) * 4;
#define AGNES_BM_LIST(JW)                                                                                          \
    do {                                                                                                           \
        allow_lds(&k_bm_list<JW>, lds);                                                                            \
        AGNES_LAUNCH((k_bm_list<JW>), dim3(p.list_groups), dim3(kBlock), lds, st, a.H, a.L, s.num_nodes, p.nb,     \
                     p.blocks, p.rb, a.capN, a.se[a.L & 1], a.rt, a.lsz, a.nodes, (uint32_t)s.rpb, p.spans,        \
                     p.n_spans, (const uint8_t*)(a.zero + p.tmark), p.tmarks, a.list_key, a.list_val, a.node_off,  \
                     a.nodes_out, a.part, a.ctl);                                                                  \
    } while (0)
    if (p.jw == 1) AGNES_BM_LIST(1);
    else if (p.jw == 2) AGNES_BM_LIST(2);
    else AGNES_BM_LIST(4);
#undef AGNES_BM_LIST
    AGNES_CHECK_HIP(hipGetLastError());
}

}  // namespace agnes

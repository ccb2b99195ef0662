// bitmap.hip on the CPU.  A workgroup's threads are coroutines: a lane runs to its
// next exchange with the wave or to a barrier, and a wave runs on until all its
// lanes wait at a barrier before another wave gets its turn.  Between two barriers
// the waves may run in any order on the device; here they run lowest first or
// highest first, which shows accesses that no barrier orders.  Workgroups run one
// after the other, so a wait for a later one ends the program.
//
// waves keys: exit status 0 if plans that launch differently have different keys.
// waves plan IN: prints the edges that a minibatch is expected to sample, and 1 if the
// hyperbatch is sampled on bitmaps.
// waves IN OUT: reads sizes, graph, targets, node ranges and list blocks, runs one
// hyperbatch and writes its sizes, lists, CSR blocks and statistics.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>
#include <ucontext.h>

#include <string>

#include BITMAP_SOURCE

dim3 threadIdx, blockIdx, gridDim;

namespace agnes {

alignas(16) uint64_t bm[20480];                        // dynamic LDS, under each kernel's name
alignas(16) int64_t rpo[20480], list_sm[20480];
alignas(16) uint32_t seen[40960];

void check_launch(hipStream_t, const char*) {}
DeviceAllocator& device_allocator() {
    static DeviceAllocator a;
    return a;
}

}  // namespace agnes

static void die(const char* what) {
    fprintf(stderr, "workgroup %u, thread %u: %s\n", blockIdx.x, threadIdx.x, what);
    exit(3);
}

// ------------------------------------------------------------ waves

enum State { kRuns, kExchange, kBarrier, kDone };
struct Lane {
    ucontext_t at;
    State state;
    uint64_t value;
    char* stack;
};
static Lane lanes[1024];
static uint64_t values[1024];
static ucontext_t scheduler;
static const std::function<void()>* body;
static bool highest_first;

static void lane_main() {
    (*body)();
    lanes[threadIdx.x].state = kDone;
}
static void yield(State s) {
    Lane& me = lanes[threadIdx.x];
    me.state = s;
    swapcontext(&me.at, &scheduler);
}
void workgroup_barrier() { yield(kBarrier); }
void wait_forever() { die("waits for a workgroup that has not run"); }
const uint64_t* exchange(uint64_t v) {
    lanes[threadIdx.x].value = v;
    yield(kExchange);
    return values + threadIdx.x / 64 * 64;
}

static void run_wave(int w) {
    for (;;) {
        int waiting = 0, done = 0;
        for (int t = 64 * w; t < 64 * w + 64; t++) {
            if (lanes[t].state == kRuns) {
                threadIdx.x = t;
                swapcontext(&scheduler, &lanes[t].at);
            }
            waiting += lanes[t].state == kExchange;
            done += lanes[t].state == kDone;
        }
        if (waiting == 0) {
            if (done != 0 && done != 64) die("a barrier that part of a wave does not reach");
            return;
        }
        if (waiting != 64) die("an exchange that part of the wave does not reach");
        for (int t = 64 * w; t < 64 * w + 64; t++) {
            values[t] = lanes[t].value;
            lanes[t].state = kRuns;
        }
    }
}

void launch(dim3 grid, dim3 block, size_t lds, const std::function<void()>& kernel) {
    const int T = (int)block.x, W = T / 64;
    if (lds > sizeof(agnes::bm)) die("too much LDS");
    gridDim = grid;
    body = &kernel;
    for (blockIdx.x = 0; blockIdx.x < grid.x; blockIdx.x++) {
        for (int t = 0; t < T; t++) {
            Lane& l = lanes[t];
            if (!l.stack) l.stack = (char*)malloc(1 << 16);
            getcontext(&l.at);
            l.at.uc_stack.ss_sp = l.stack;
            l.at.uc_stack.ss_size = 1 << 16;
            l.at.uc_link = &scheduler;
            makecontext(&l.at, lane_main, 0);
            l.state = kRuns;
        }
        for (int done = 0; done < T;) {
            for (int w = 0; w < W; w++) run_wave(highest_first ? W - 1 - w : w);
            done = 0;
            for (int t = 0; t < T; t++) {
                if (lanes[t].state == kDone) done++;
                else lanes[t].state = kRuns;
            }
        }
    }
}

// ------------------------------------------------------------ one hyperbatch

// Memory that ends at a page that cannot be accessed.
template <typename T>
static T* room(size_t items) {
    const size_t bytes = (items * sizeof(T) + 15) / 16 * 16, page = 4096, full = (bytes + page - 1) / page * page;
    char* p = (char*)mmap(nullptr, full + page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (p == MAP_FAILED || mprotect(p + full, page, PROT_NONE)) die("no memory");
    memset(p, 0xA5, full);
    return (T*)(p + full - bytes);
}
template <typename T>
static T* read_array(FILE* f, size_t n) {
    T* p = room<T>(n);
    if (fread(p, sizeof(T), n, f) != n) die("short input");
    return p;
}
template <typename T>
static void write_array(FILE* f, const T* p, size_t n) {
    fwrite(p, sizeof(T), n, f);
}

// Two stores of one size, the second where the first one was, cut differently.
static bool keys_differ() {
    using namespace agnes;
    const int32_t fanouts[] = {10, 5};
    const int64_t cap[] = {256, 2816, 16384};
    auto key = [&](int ranges, int longest, int64_t blocks, char* bounds) {
        static Store s;
        s.num_nodes = 16384;
        s.num_edges = 16384 * 8;
        s.nblk = 128;
        for (auto& t : s.range_tab) t = Store::RangeTable{0, ranges, longest};
        s.n_list_blocks = blocks;
        s.ranges.ptr = bounds;
        std::vector<uint64_t> k;
        bitmap_key(bitmap_plan(s, 8, 256, fanouts, 2, cap), k);
        s.ranges.ptr = nullptr;
        return k;
    };
    char at[8];
    const auto k = key(8, 4096, 1024, at);
    return k == key(8, 4096, 1024, at) && k != key(9, 4096, 1024, at) && k != key(8, 4352, 1024, at) &&
           k != key(8, 4096, 1025, at) && k != key(8, 4096, 1024, at + 4);
}

// Reads sizes and graph; K node ranges of equal length.
static int print_plan(const char* path) {
    using namespace agnes;
    FILE* in = fopen(path, "rb");
    if (!in) die("no input");
    const int64_t* h = read_array<int64_t>(in, 6);
    const int64_t n = h[0], E = h[1], K = h[5];
    const int H = (int)h[2], B = (int)h[3], L = (int)h[4];
    const int32_t* fanouts = read_array<int32_t>(in, L);
    const int64_t* off = read_array<int64_t>(in, n + 1);
    const int32_t* adj = read_array<int32_t>(in, E);
    std::vector<uint32_t> indeg(n, 0u);
    for (int64_t i = 0; i < E; i++) indeg[adj[i]]++;
    static Store s;
    s.num_nodes = n;
    s.num_edges = E;
    s.nblk = 1;
    for (int64_t v = 0; v < n; v++) s.max_degree = std::max(s.max_degree, off[v + 1] - off[v]);
    for (auto& t : s.range_tab) t = Store::RangeTable{0, (int)K, (int)((n / K + 255) / 256 * 256)};
    s.n_list_blocks = n / 16 + 1;
    agnes_csr csr{n, E, AGNES_INT64, off, adj};
    build_degree_classes(s, indeg, csr);
    int64_t cap[AGNES_MAX_LAYERS + 1] = {B};
    for (int l = 0; l < L; l++) cap[l + 1] = std::min<int64_t>(cap[l] * (1 + fanouts[l]), std::max<int64_t>(n, B));
    printf("%.1f %d\n", expected_edges(s, B, fanouts, L), (int)bitmap_plan(s, H, B, fanouts, L, cap).use);
    return 0;
}

int main(int argc, char** argv) {
    using namespace agnes;
    if (argc == 2) return keys_differ() ? 0 : 1;
    if (argv[1] == std::string("plan")) return print_plan(argv[2]);
    FILE* in = fopen(argv[1], "rb");
    if (!in) die("no input");
    const int64_t* h = read_array<int64_t>(in, 12);
    const int64_t n = h[0], E = h[1], K = h[5], nb = h[6];
    const int H = (int)h[2], B = (int)h[3], L = (int)h[4];
    highest_first = h[11] != 0;
    const int32_t* fanouts = read_array<int32_t>(in, L);
    int64_t* off = read_array<int64_t>(in, n + 1);
    int32_t* adj = read_array<int32_t>(in, E);
    const int32_t* targets = read_array<int32_t>(in, (size_t)H * B);
    int32_t* ranges = read_array<int32_t>(in, 2 * (K + 1));
    int32_t* blocks = read_array<int32_t>(in, nb + 1);

    Store& s = *new Store();
    s.num_nodes = n;
    s.num_edges = E;
    s.offsets64 = 1;
    s.rpb = h[7];
    s.e_blk_log2 = (int)h[8];
    s.nblk = E > 0 ? ((E - 1) >> s.e_blk_log2) + 1 : 1;
    s.offsets.ptr = off;
    s.indices.ptr = adj;
    s.ranges.ptr = ranges;
    s.list_blocks.ptr = blocks;
    s.n_list_blocks = nb;
    int longest = 0;
    for (int k = 0; k < K; k++) longest = std::max(longest, ranges[k + 1] - ranges[k]);
    for (auto& t : s.range_tab) t = Store::RangeTable{0, (int)K, (longest + 255) / 256 * 256};

    int64_t cap[AGNES_MAX_LAYERS + 1] = {B};
    for (int l = 0; l < L; l++) cap[l + 1] = std::min<int64_t>(cap[l] * (1 + fanouts[l]), std::max<int64_t>(n, B));
    BitmapArgs a{};
    a.s = &s;
    a.p = bitmap_plan(s, H, B, fanouts, L, cap);
    const BitmapPlan& p = a.p;
    a.H = H; a.B = B; a.L = L;
    a.fanouts = fanouts;
    a.cap = cap;
    a.capN = cap[L];
    a.given = BmParams{targets, (uint64_t)h[9], h[10]};
    a.params = room<BmParams>(1);
    a.zero = room<char>(p.bytes);
    a.ctl = room<Ctl>(1);
    a.lsz = room<int32_t>((size_t)H * (L + 1));
    a.host_lsz = room<int32_t>((size_t)H * (L + 1));
    a.ecount = room<int64_t>((size_t)H * L);
    a.host_ecount = room<int64_t>((size_t)H * L);
    a.host_err = room<uint32_t>(H);
    a.nodes = room<int32_t>(H * a.capN);
    a.deg = room<int32_t>(H * p.capR);
    a.rp = room<uint32_t>(H * p.capR);
    a.cg = room<int32_t>(H * p.capE);
    a.ce = room<uint16_t>(H * p.capE);
    a.tab = room<uint16_t>(H * p.capC * (p.K + 1));
    a.cbase = room<uint32_t>(H * p.capC);
    for (int i = 0; i < 2; i++) {
        a.se[i] = room<uint64_t>(H * a.capN);
        a.os[i] = room<int32_t>((size_t)H * (p.K + 1));
    }
    a.rt = room<int32_t>(H * (p.nb + 1));
    for (int l = 0; l < L; l++) {
        a.row_ptr[l] = room<int32_t>(H * cap[l] + H);
        a.col[l] = room<int32_t>(std::max<int64_t>(1, H * cap[l] * fanouts[l]));
    }
    a.list_key = a.se[(L & 1) ^ 1];
    a.list_val = room<int32_t>(H * a.capN);
    a.node_off = room<int64_t>(H + 1);
    a.nodes_out = room<int32_t>(H * a.capN);
    a.part = room<uint32_t>((size_t)p.list_groups * (2 + AGNES_MAX_LAYERS));
    bitmap_hops(a, nullptr);
    bitmap_list(a, nullptr);

    FILE* out = fopen(argv[2], "wb");
    if (!out) die("no output");
    write_array(out, a.host_err, H);
    write_array(out, a.host_lsz, (size_t)H * (L + 1));
    write_array(out, a.host_ecount, (size_t)H * L);
    int64_t rows = 0;
    for (int j = 0; j < H; j++) rows += a.host_lsz[j * (L + 1) + L];
    write_array(out, a.nodes_out, rows);
    write_array(out, a.list_key, rows);
    write_array(out, a.list_val, rows);
    int64_t sum[2 + AGNES_MAX_LAYERS] = {};
    for (int g = 0; g < p.list_groups; g++)
        for (int i = 0; i < 2 + L; i++) sum[i] += a.part[g * (2 + AGNES_MAX_LAYERS) + i];
    write_array(out, sum, 2 + L);
    for (int l = 0; l < L; l++) {
        int64_t rp = H, e = 0;
        for (int j = 0; j < H; j++) {
            rp += a.host_lsz[j * (L + 1) + l];
            e += a.host_ecount[j * L + l];
        }
        write_array(out, a.row_ptr[l], rp);
        write_array(out, a.col[l], e);
    }
    return fclose(out) ? 3 : 0;
}

// Host-side check of the kernel launches (paper_2409_00918_amd/csrc/
// disdp_kernels.hip, its host code only) without a GPU: the runtime calls it
// makes are the stubs below, which record every launch.
//
//   launch_check            checks, over random calls:
//     * the single-tensor and conversion launches: grids within what a
//       dispatch counts, and every element of head, groups and tail dealt out
//       exactly once, piece after piece, from the right addresses (arrays of
//       more elements than one grid holds included);
//     * the two-tile order is a permutation of the tiles;
//     * the many-tensor tables: a block finds its tensor, and the tensor's
//       rows or offsets are its addresses; how many tensors a launch holds.
//   launch_check order DTYPE MODE ADAM N P0 P1 ...
//                           prints 1 when a call over contributions at those
//                           addresses would take two tiles together per XCD.
//
// Prints "launch_check: ok" and exits 0; a failed check prints the case and
// exits 1.
#include "../../paper_2409_00918_amd/csrc/disdp_kernels.hip"

#include <cinttypes>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

// ---- stubs for the runtime -------------------------------------------------
namespace {
struct Launch {
    const void *fn;
    int64_t blocks;
    int lanes;
    std::vector<unsigned char> args;
};
std::vector<Launch> g_launches;
// what to keep of a launch's arguments: of the many-tensor kernel g_multi_fn its
// whole struct, of any other kernel this much
size_t g_arg_bytes = 0;
const void *g_multi_fn = nullptr;
constexpr int kCus = 256;
}  // namespace

extern "C" hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t,
                                      hipStream_t)
{
    const unsigned char *a = static_cast<const unsigned char *>(args[0]);
    const size_t bytes = fn == g_multi_fn ? sizeof(disdp::MultiLaunch) : g_arg_bytes;
    g_launches.push_back({fn, int64_t(grid.x), int(block.x),
                          std::vector<unsigned char>(a, a + bytes)});
    return hipSuccess;
}
extern "C" hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
extern "C" hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t at, int)
{
    *v = at == hipDeviceAttributeMultiprocessorCount ? kCus : 160 << 10;
    return hipSuccess;
}
extern "C" hipError_t hipExtStreamGetCUMask(hipStream_t, uint32_t words, uint32_t *mask)
{
    for (uint32_t i = 0; i < words; ++i)
        mask[i] = ~0u;
    return hipSuccess;
}
extern "C" hipError_t hipPeekAtLastError(void) { return hipSuccess; }
extern "C" hipError_t hipGetLastError(void) { return hipSuccess; }
// what the compiler's kernel stubs and registration refer to: no kernel is
// registered or run
extern "C" void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
extern "C" void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *,
                                      void *, void *, void *, int *) {}
extern "C" void __hipUnregisterFatBinary(void **) {}
extern "C" const char __hip_fatbin[8] = {};
extern "C" hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
extern "C" hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }

namespace disdp {
namespace {

uint64_t rng_state = 0x243F6A8885A308D3ull;
uint64_t next()
{
    uint64_t x = (rng_state += 0x9E3779B97F4A7C15ull);
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}
int64_t below(int64_t k) { return static_cast<int64_t>(next() % static_cast<uint64_t>(k)); }

int failures = 0;
#define CHECK(cond, ...)                                                   \
    do {                                                                   \
        if (!(cond)) {                                                     \
            std::printf("FAIL %s:%d: %s: ", __FILE__, __LINE__, #cond);    \
            std::printf(__VA_ARGS__);                                      \
            std::printf("\n");                                             \
            if (++failures > 20)                                           \
                std::exit(1);                                              \
        }                                                                  \
    } while (0)

constexpr int64_t kGrid = 0xffffffffLL;   // work-items of one dispatch

// The tile that block `block` of a piece takes, as deal() computes it.
int64_t tile_of(const Split &sp, int64_t block, int lanes_log2)
{
    int64_t tile = block - sp.lead;
    const int64_t last = tile | ((8 << sp.together) - 1);
    if (sp.together && tile >= 0 && (last + 1) << lanes_log2 <= sp.n_groups)
        tile = last - (8 << sp.together) + 1 + ((tile & 7) << sp.together) +
               ((tile >> 3) & ((1 << sp.together) - 1));
    return tile;
}

// A piece's blocks: the single elements first, the head's groups, then every
// tile once.
void check_split(const Split &sp, int64_t blocks, int lanes, const char *what)
{
    const int log2 = lanes == 64 ? 6 : 8;
    const int64_t tiles = (sp.n_groups + lanes - 1) / lanes;
    CHECK(blocks == sp.lead + tiles && blocks >= 1, "%s: %" PRId64 " blocks", what, blocks);
    CHECK(sp.singles == ((sp.head & 3) || sp.tail), "%s: block of single elements", what);
    CHECK(sp.lead == sp.singles + (sp.head >= 4), "%s: blocks in front", what);
    CHECK(sp.head >= 0 && sp.head < 256 && (sp.head >> 2) <= lanes && sp.tail >= 0 && sp.tail < 4,
          "%s: head %d tail %d", what, sp.head, sp.tail);
    if (sp.together && tiles < 1 << 18) {
        std::vector<char> seen(static_cast<size_t>(tiles));
        for (int64_t b = sp.lead; b < blocks; ++b) {
            const int64_t t = tile_of(sp, b, log2);
            CHECK(t >= 0 && t < tiles && !seen[t], "%s: tile %" PRId64, what, t);
            if (t >= 0 && t < tiles)
                seen[t] = 1;
        }
    }
}

// ---- one tensor ----------------------------------------------------------------
struct Call {
    LaunchArgs a;
    Kind kind;
    int gb;
};

template <int W>
void check_vector_w(const Call &c)
{
    using Args = VectorArgs<W>;
    int64_t done = 0, groups = 0;
    for (size_t i = 0; i < g_launches.size(); ++i) {
        const Launch &l = g_launches[i];
        Args k;
        std::memcpy(&k, l.args.data(), sizeof k);
        CHECK(l.blocks * l.lanes <= kGrid, "grid of %" PRId64 " blocks", l.blocks);
        CHECK(k.lanes_log2 == (l.lanes == 64 ? 6 : 8), "lanes");
        check_split(k.split, l.blocks, l.lanes, "vector");
        CHECK(k.split.head == (i == 0 ? c.a.head : 0), "head of piece %zu", i);
        CHECK(k.split.tail == (i + 1 == g_launches.size() ? c.a.n & 3 : 0), "tail of piece %zu", i);
        for (int w = 0; w < c.a.W; ++w)
            CHECK(k.g[w] == reinterpret_cast<Base>(c.a.g[w]) + done * c.gb, "piece %zu g%d", i, w);
        const struct { Base got; const void *p; int esz; } outs[] = {
            {k.p, c.a.p, 4}, {k.m, c.a.m, 4}, {k.v, c.a.v, 4}, {k.p16, c.a.p16, 2},
            {k.agg_f32, c.a.agg_f32, 4}, {k.agg_i32, c.a.agg_i32, 4}};
        for (const auto &o : outs)
            CHECK(o.got == (o.p ? reinterpret_cast<Base>(o.p) + done * o.esz : 0),
                  "piece %zu output", i);
        done += 4 * k.split.n_groups;
        groups += k.split.n_groups;
    }
    CHECK(groups == c.a.n >> 2, "%" PRId64 " groups of %" PRId64, groups, c.a.n >> 2);
}

char *fake(int i) { return reinterpret_cast<char *>((uintptr_t(1) << 50) + (uintptr_t(i) << 43)); }

Call random_call()
{
    Call c{};
    const int ws[] = {1, 2, 3, 4, 5, 6, 7, 8, 12, 16, 9, 13, 24, 64};
    c.a.W = ws[below(14)];
    c.a.mode = static_cast<int>(below(2));
    c.a.gdtype = static_cast<int>(below(c.a.mode == kAggFixed ? 3 : 2));
    c.gb = c.a.gdtype == kGradBF16 ? 2 : 4;
    c.kind = below(2) ? kAggregateAdam : kAggregateOnly;
    const int64_t most = int64_t(1) << (1 + below(37));    // up to eight grids
    c.a.n = below(most);
    c.a.head = below(2) ? 0 : static_cast<int>(below(256));
    if (c.a.n + c.a.head == 0)
        c.a.n = 1;
    for (int w = 0; w < c.a.W; ++w)
        c.a.g[w] = fake(w);
    if (c.kind == kAggregateAdam) {
        c.a.p = reinterpret_cast<float *>(fake(70));
        c.a.m = reinterpret_cast<float *>(fake(71));
        c.a.v = reinterpret_cast<float *>(fake(72));
        c.a.p16 = below(2) ? reinterpret_cast<uint16_t *>(fake(73)) : nullptr;
    }
    if (c.kind == kAggregateOnly || below(3) == 0)
        c.a.agg_f32 = reinterpret_cast<float *>(fake(74));
    return c;
}

template <int W>
bool check_if(const Call &c)
{
    if (c.a.W != W)
        return false;
    g_arg_bytes = sizeof(VectorArgs<W>);
    CHECK(launch(c.a, c.kind, true, nullptr) == hipSuccess, "launch");
    check_vector_w<W>(c);
    return true;
}

void check_vector(int iters)
{
    for (int it = 0; it < iters; ++it) {
        const Call c = random_call();
        setenv("DISDP_LAUNCH_SHAPE", below(3) ? "" : "shared", 1);
        g_launches.clear();
        if (!(check_if<1>(c) || check_if<2>(c) || check_if<3>(c) || check_if<4>(c) ||
              check_if<5>(c) || check_if<6>(c) || check_if<7>(c) || check_if<8>(c) ||
              check_if<12>(c) || check_if<16>(c))) {
            g_arg_bytes = sizeof(VectorArgs<0>);
            CHECK(launch(c.a, c.kind, true, nullptr) == hipSuccess, "launch");
            check_vector_w<0>(c);
        }
    }
    unsetenv("DISDP_LAUNCH_SHAPE");
}

void check_quantize(int iters)
{
    g_arg_bytes = sizeof(QuantizeVectorArgs);
    for (int it = 0; it < iters; ++it) {
        QuantizeArgs q{};
        q.gdtype = static_cast<int>(below(2));
        const int gb = q.gdtype == kGradBF16 ? 2 : 4;
        q.n = below(int64_t(1) << (1 + below(37)));
        q.head = below(2) ? 0 : static_cast<int>(below(256));
        if (q.n + q.head == 0)
            q.n = 1;
        q.g = fake(0);
        q.out = reinterpret_cast<int32_t *>(fake(1));
        g_launches.clear();
        CHECK(launch_quantize(q, true, nullptr) == hipSuccess, "launch");
        int64_t done = 0;
        for (size_t i = 0; i < g_launches.size(); ++i) {
            const Launch &l = g_launches[i];
            QuantizeVectorArgs k;
            std::memcpy(&k, l.args.data(), sizeof k);
            CHECK(l.lanes == 64 && l.blocks * 64 <= kGrid, "grid");
            CHECK(k.lead == k.edges.lead && l.blocks == k.lead + (k.n_groups + 63) / 64, "blocks");
            if (k.lead)
                check_split(k.edges, k.lead, 64, "edges");
            CHECK(k.edges.n_groups == 0 && k.edges.head == (i == 0 ? q.head : 0) &&
                      k.edges.tail == (i + 1 == g_launches.size() ? q.n & 3 : 0),
                  "edges of piece %zu", i);
            CHECK(k.g == reinterpret_cast<Base>(q.g) + done * gb &&
                      k.out == reinterpret_cast<Base>(q.out) + done * 4,
                  "addresses of piece %zu", i);
            done += 4 * k.n_groups;
        }
        CHECK(done == (q.n & ~int64_t(3)), "groups");
    }
}

// ---- several tensors -----------------------------------------------------------
MultiArgs g_multi;   // (38 KB)

// The blocks of a recorded many-tensor launch, found as the kernel finds them.
// Returns the tensors it holds; `at`: the first of them in g_multi.
int check_multi_launch(const Launch &l, int at)
{
    MultiLaunch k;
    std::memcpy(&k, l.args.data(), sizeof k);
    const int W = g_multi.W, gb = g_multi.gdtype == kGradBF16 ? 2 : 4;
    const uint32_t *first = reinterpret_cast<const uint32_t *>(k.table);
    const int slots = (k.count + 16) & ~15;
    CHECK(k.count >= 2 && k.count <= kMultiMost && k.W == W, "count %d", k.count);
    CHECK(k.rows_at % 8 == 0 && k.rows_at >= 4 * (slots + k.count) &&
              k.rows_at + (k.flat ? 8 * k.count + 8 * (W + 4) : 8 * (W + 4) * k.count) <= kMultiTable,
          "table of %d tensors", k.count);
    const int64_t *offsets = reinterpret_cast<const int64_t *>(k.table + k.rows_at);
    for (int j = 0; j < k.count; ++j) {
        const int c = at + j;
        // as the kernel reads them
        const Base *row = reinterpret_cast<const Base *>(offsets) + (k.flat ? k.count : j * (W + 4));
        const int64_t off = k.flat ? offsets[j] : k.zero;
        for (int i = 0; i < W + 4; ++i) {
            const int esz = i < W ? gb : i == W + 3 ? 2 : 4;
            const void *want = g_multi.ptr[c * (W + 4) + i];
            const Base got = row[i] ? row[i] + off * esz : 0;
            CHECK(got == reinterpret_cast<Base>(want), "tensor %d array %d", c, i);
        }
        const uint32_t shape = first[slots + j];
        const int last = shape >> 10;
        Split sp = make_split(0, shape & 255, (shape >> 8) & 3, 0);
        const int64_t blocks = int64_t(first[j + 1]) - first[j];
        if (last)
            sp.n_groups = (blocks - sp.lead - 1) * 64 + last;
        CHECK(sp.n_groups == g_multi.n[c] >> 2 && sp.head == g_multi.head[c] &&
                  sp.tail == (g_multi.n[c] & 3),
              "tensor %d: shape", c);
        check_split(sp, blocks, 64, "tensor");
        for (int64_t b : {int64_t(first[j]), int64_t(first[j + 1]) - 1}) {
            int j16 = 0, found = 0;
            for (int i = 0; i < 16; ++i)
                j16 += k.coarse[i] <= static_cast<uint64_t>(b);
            j16 = 16 * (j16 - 1);
            CHECK(j16 >= 0 && j16 + 16 <= slots, "coarse list");
            for (int i = 0; i < 16; ++i)
                found += first[j16 + i] <= static_cast<uint64_t>(b);
            CHECK(j16 + found - 1 == j, "block %" PRId64 " finds tensor %d of %d", b,
                  j16 + found - 1, j);
        }
    }
    CHECK(first[k.count] == l.blocks && l.blocks * 64 <= kGrid, "blocks");
    return k.count;
}

template <int W>
const void *multi_fn()
{
    return reinterpret_cast<const void *>(&multi_kernel<W, kGradF32, kAggFP32>);
}

// T tensors of random sizes, in buffers of their own or slices of flat ones.
int run_multi(int T, int W, int gdtype, int mode, bool flat, int64_t largest)
{
    const int per = W + 4, gb = gdtype == kGradBF16 ? 2 : 4;
    g_multi = MultiArgs{};
    g_multi.count = T;
    g_multi.W = W;
    g_multi.gdtype = gdtype;
    g_multi.mode = mode;
    int64_t at = 4 * below(1000);
    for (int c = 0; c < T; ++c) {
        const int64_t n = 1 + below(largest);
        g_multi.head[c] = static_cast<int>(below(256 < n ? 256 : n));
        g_multi.n[c] = n - g_multi.head[c];
        for (int i = 0; i < per; ++i) {
            const int esz = i < W ? gb : i == W + 3 ? 2 : 4;
            g_multi.ptr[c * per + i] =
                fake(i) + (at + (flat ? 0 : 4 * below(1 << 10))) * esz;
        }
        at += n + 4 * (1 + below(64));
    }
    g_launches.clear();
    g_arg_bytes = sizeof(Split);
    g_multi_fn = W == 8 ? multi_fn<8>() : W == 1 ? multi_fn<1>() : multi_fn<0>();
    CHECK(launch_multi(g_multi, nullptr) == hipSuccess, "launch");
    return static_cast<int>(g_launches.size());
}

void check_multi(int iters)
{
    for (int it = 0; it < iters; ++it) {
        // fp32 kernels of W = 8 and of a run-time W, told apart by the kernel
        const int W = below(2) ? 8 : 9;
        run_multi(1 + static_cast<int>(below(240)), W, kGradF32, kAggFP32, below(2), 1 + below(100000));
        int at = 0;
        for (const Launch &l : g_launches)
            at += l.fn == g_multi_fn ? check_multi_launch(l, at) : 1;   // alone: the vector kernel
        CHECK(at == g_multi.count, "%d tensors of %d", at, g_multi.count);
    }
    // what the public header states for W = 8
    CHECK(run_multi(36, 8, kGradF32, kAggFP32, false, 1000) == 1, "36 tensors");
    CHECK(run_multi(37, 8, kGradF32, kAggFP32, false, 1000) == 2, "37 tensors");
    CHECK(run_multi(232, 8, kGradF32, kAggFP32, true, 1000) == 1, "232 slices");
    CHECK(run_multi(233, 8, kGradF32, kAggFP32, true, 1000) == 2, "233 slices");
    CHECK(run_multi(236, 1, kGradF32, kAggFP32, true, 1000) == 1, "236 slices");
}

// ---- the two-tile order ------------------------------------------------------
int order_of(const LaunchArgs &a, Kind kind)
{
    g_launches.clear();
    g_arg_bytes = sizeof(Split);
    CHECK(launch(a, kind, true, nullptr) == hipSuccess, "launch");
    Split sp;   // the first member of every VectorArgs
    std::memcpy(&sp, g_launches.front().args.data(), sizeof sp);
    return sp.together;
}

// `W` contributions `apart` bytes from each other.
int order(int gdtype, int mode, bool adam, int W, int64_t n, int64_t apart)
{
    LaunchArgs a{};
    a.gdtype = gdtype;
    a.mode = mode;
    a.W = W;
    a.n = n;
    for (int w = 0; w < W; ++w)
        a.g[w] = fake(0) + apart * w;
    a.p = a.m = a.v = reinterpret_cast<float *>(fake(70));
    a.agg_f32 = adam ? nullptr : reinterpret_cast<float *>(fake(71));
    return order_of(a, adam ? kAggregateAdam : kAggregateOnly);
}

void check_order()
{
    constexpr int64_t MiB = int64_t(1) << 20;
    const struct { int gt, mode; bool adam; int W; int64_t n, apart; int want; } cases[] = {
        {kGradBF16, kAggFP32, true, 16, 25000000, 50 * MiB, 1},
        {kGradBF16, kAggFP32, true, 12, 25000000, 50 * MiB, 1},
        {kGradBF16, kAggFixed, true, 20, 25000000, 50 * MiB, 1},
        {kGradBF16, kAggFP32, false, 16, 25000000, 50 * MiB, 1},
        {kGradBF16, kAggFixed, false, 24, 25000000, 50 * MiB, 1},
        // few contributions, another type
        {kGradBF16, kAggFP32, true, 8, 25000000, 50 * MiB, 0},
        {kGradBF16, kAggFP32, false, 12, 25000000, 50 * MiB, 0},
        {kGradF32, kAggFP32, true, 16, 25000000, 100 * MiB, 0},
        // few rounds; many elements
        {kGradBF16, kAggFP32, false, 16, 10000000, 20 * MiB, 0},
        {kGradBF16, kAggFP32, false, 16, 13000000, 26 * MiB, 1},
        {kGradBF16, kAggFP32, true, 16, 700000000, 1400 * MiB, 1},
        {kGradBF16, kAggFP32, true, 16, 700000001, 1400 * MiB, 0},
        // a multiple of 64 MiB apart, and 5 MiB beside it
        {kGradBF16, kAggFP32, true, 16, 25000000, 64 * MiB, 0},
        {kGradBF16, kAggFP32, true, 16, 25000000, 128 * MiB + 4 * MiB, 0},
        {kGradBF16, kAggFP32, true, 16, 25000000, 128 * MiB - 4 * MiB, 0},
        {kGradBF16, kAggFP32, true, 16, 25000000, 128 * MiB + 5 * MiB, 1},
        {kGradBF16, kAggFP32, true, 16, 25000000, 128 * MiB - 5 * MiB, 1},
        {kGradBF16, kAggFP32, true, 16, 25000000, 0, 0},
    };
    for (const auto &c : cases)
        CHECK(order(c.gt, c.mode, c.adam, c.W, c.n, c.apart) == c.want,
              "dtype %d mode %d adam %d W %d n %" PRId64 " apart %" PRId64 ": want %d", c.gt, c.mode,
              c.adam, c.W, c.n, c.apart, c.want);
    // contributions in falling order are as far apart
    LaunchArgs a{};
    a.gdtype = kGradBF16;
    a.W = 16;
    a.n = 25000000;
    for (int w = 0; w < 16; ++w)
        a.g[w] = fake(1) - 64 * MiB * w;
    a.p = a.m = a.v = reinterpret_cast<float *>(fake(70));
    CHECK(order_of(a, kAggregateAdam) == 0, "falling order");
}

}  // namespace
}  // namespace disdp

int main(int argc, char **argv)
{
    using namespace disdp;
    if (argc > 1 && std::strcmp(argv[1], "order") == 0) {
        if (argc < 7 || argc - 6 > kMaxW)
            return 2;
        LaunchArgs a{};
        a.gdtype = std::atoi(argv[2]);
        a.mode = std::atoi(argv[3]);
        const bool adam = std::atoi(argv[4]) != 0;
        a.n = std::atoll(argv[5]);
        a.W = argc - 6;
        for (int w = 0; w < a.W; ++w)
            a.g[w] = reinterpret_cast<const void *>(std::strtoull(argv[6 + w], nullptr, 10));
        a.p = a.m = a.v = reinterpret_cast<float *>(fake(70));
        a.agg_f32 = reinterpret_cast<float *>(fake(71));
        std::printf("%d\n", order_of(a, adam ? kAggregateAdam : kAggregateOnly));
        return 0;
    }
    check_vector(20000);
    check_quantize(5000);
    check_multi(500);
    check_order();
    if (failures) {
        std::printf("launch_check: %d failures\n", failures);
        return 1;
    }
    std::printf("launch_check: ok\n");
    return 0;
}

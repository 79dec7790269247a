// CPU test of how the hot-column layout's row blocks are chosen (hot_plan.h):
// blocks cut as the device does, on relabelled graphs (rows with entries first)
// most of whose vertices have none, and on graphs that fill their blocks.
#include <cstdio>
#include <cstdlib>

#include "hot_plan.h"

using namespace lilac;

#define CHECK(c)                                                            \
    do {                                                                    \
        if (!(c)) {                                                         \
            std::fprintf(stderr, "FAIL %s:%d: %s\n", __FILE__, __LINE__, #c); \
            std::exit(1);                                                   \
        }                                                                   \
    } while (0)

constexpr int32_t kKeys = 1536, kSpan = 24576, kPart = 8 * kSpan, kCu = 256;

struct Graph {
    std::vector<int32_t> rp, filled;   // filled: non-empty rows before each row
    int32_t rows() const { return (int32_t)rp.size() - 1; }
};

// `full` rows of `len` entries (the first of them `first` times as many), each
// followed by `gap` empty ones, then empty ones up to `rows`.
static Graph graph(int32_t rows, int32_t full, int32_t len, int32_t gap = 0, int32_t first = 1)
{
    Graph g;
    g.rp.assign((size_t)rows + 1, 0);
    g.filled.assign((size_t)rows + 1, 0);
    for (int32_t r = 0; r < rows; ++r) {
        const bool on = r % (gap + 1) == 0 && r / (gap + 1) < full;
        g.rp[r + 1] = g.rp[r] + (on ? (r == 0 ? len * first : len) : 0);
        g.filled[r + 1] = g.filled[r] + (on ? 1 : 0);
    }
    return g;
}

// The device's rule, row by row.
static HotCut cut(const Graph &g, int64_t target)
{
    HotCut k;
    for (int32_t r0 = 0; r0 < g.rows(); r0 += kPart) {
        const int32_t end = std::min(r0 + kPart, g.rows());
        int32_t start = r0;
        k.brow.push_back(start);
        k.bent.push_back(g.rp[start]);
        for (int32_t r = r0 + 1; r < end; ++r)
            if (r - start >= kSpan || g.filled[r + 1] - g.filled[start] > kKeys ||
                g.rp[r] - g.rp[start] >= target) {
                start = r;
                k.brow.push_back(start);
                k.bent.push_back(g.rp[start]);
            }
    }
    k.brow.push_back(g.rows());
    k.bent.push_back(g.rp.back());
    return k;
}

static int tries;

static HotCut choose(const Graph &g, int32_t *per = nullptr, double *heaviest = nullptr)
{
    tries = 0;
    const int64_t nnz = g.rp.back();
    const std::vector<int64_t> ts = hot_few_targets(std::max<int64_t>(4096, nnz / kCu));
    CHECK(ts.back() <= INT32_MAX);
    HotCut c = hot_cut_few(ts.size(), kCu, [&](size_t i) {
        ++tries;
        return cut(g, ts[i]);
    });
    std::vector<int32_t> owner;
    const int32_t grid = std::min(c.blocks(), kCu);
    hot_assign(c, grid, owner);
    std::vector<int64_t> entries((size_t)grid, 0);
    std::vector<int32_t> blocks((size_t)grid, 0);
    for (int32_t b = 0; b < c.blocks(); ++b) {
        CHECK(owner[b] >= 0 && owner[b] < grid);
        entries[owner[b]] += c.bent[b + 1] - c.bent[b];
        blocks[owner[b]] += c.bent[b + 1] > c.bent[b];
    }
    if (per)
        *per = *std::max_element(blocks.begin(), blocks.end());
    if (heaviest)
        *heaviest = (double)*std::max_element(entries.begin(), entries.end()) * grid / (double)nnz;
    return c;
}

int main()
{
    int32_t per;
    double load;
    // mostly empty: blocks of empty rows alone never get fewer; every workgroup
    // keeps about its share of the entries, in a few tries
    const int32_t empty[][3] = {{8000000, 100000, 1000}, {5000000, 100000, 600},
                                {4000000, 150000, 400}, {4000000, 60000, 833}};
    for (const auto &e : empty) {
        choose(graph(e[0], e[1], e[2]), &per, &load);
        std::printf("%d rows, %d of %d entries: heaviest %.2f, %d tries\n", e[0], e[1], e[2], load,
                    tries);
        CHECK(load <= 1.3);
        CHECK(tries <= 24);
    }
    // the same with the rows apart, and with a heavy first row
    choose(graph(6000000, 100000, 300, 50), &per, &load);
    CHECK(load <= 1.3 && tries <= 24);
    choose(graph(3000000, 100000, 300, 0, 300), &per, &load);
    CHECK(load <= 1.3 && tries <= 24);
    // a graph that fills most of its rows: no workgroup has two blocks
    HotCut c = choose(graph(262144, 150000, 29), &per, &load);
    std::printf("%d blocks, heaviest %.2f\n", c.blocks(), load);
    CHECK(c.blocks() <= kCu && per == 1);
    // few entries: one try
    c = choose(graph(70000, 30000, 4), &per, &load);
    CHECK(tries == 1 && per == 1);
    std::printf("hot plan ok\n");
    return 0;
}

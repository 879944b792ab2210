// Host run of the depth order of several views straight from the preprocess's
// output (k_bucket.hip, depth_order_views): culled entries, padded chunks, an
// empty view, views of uneven size, ties (one bucket larger than an LDS sort,
// so the merge path runs), and one view with a device count.  Checks the order
// by (view, float64 depth, position), the tile offsets and the totals.
#include "hip/hip_runtime.h"
#include "k_bucket_host.inc"
#include <cstdio>
#include <random>
using namespace fdgs;

int main() {
    std::mt19937_64 rng(11);
    const std::vector<std::vector<int64_t>> cases = {{700}, {3000}, {1, 0, 1024, 2500}, {4000, 300}, {0, 0}};
    for (size_t trial = 0; trial < cases.size(); ++trial) {
        const auto &sizes = cases[trial];
        const int V = (int)sizes.size();
        std::vector<ViewDesc> table(V);
        std::vector<uint32_t> chunk_view;
        int64_t n_total = 0, max_n = 0;
        for (int v = 0; v < V; ++v) {
            table[v].p_off = n_total;
            table[v].n_proc = sizes[v];
            const int64_t chunks = std::max<int64_t>((sizes[v] + kViewChunk - 1) / kViewChunk, 1);
            for (int64_t c = 0; c < chunks; ++c) chunk_view.push_back((uint32_t)v);
            n_total += chunks * kViewChunk;
            max_n = std::max(max_n, sizes[v]);
        }
        const bool one = V == 1;
        int64_t n_dev = sizes[0];
        if (one) { n_total = sizes[0] + 333; max_n = n_total; }   // the bound is larger than the device count
        const int64_t blocks = (n_total + kPreprocessBlock - 1) / kPreprocessBlock;
        std::vector<uint8_t> vis(n_total, 1);                      // garbage outside the views' entries
        std::vector<uint64_t> dk(n_total, 0x7ff8000000000000ull), offsets(n_total, 77);
        std::vector<uint32_t> tiles(n_total, 1000000u), range(2 * blocks, 0u);
        for (int64_t b = 0; b < blocks; ++b) range[2 * b] = ~0u;
        std::vector<uint32_t> ref;
        for (int v = 0; v < V; ++v)
            for (int64_t i = 0; i < sizes[v]; ++i) {
                const int64_t j = table[v].p_off + i;
                double z = 2.0 + 4.0 * std::uniform_real_distribution<double>(0, 1)(rng);
                if (trial == 3 && i % 2) z = 3.25;                 // ties: 2000 in one bucket
                std::memcpy(&dk[j], &z, 8);
                vis[j] = rng() % 4 != 0;
                tiles[j] = (uint32_t)(rng() % 40);
                if (!vis[j]) continue;
                ref.push_back((uint32_t)j);
                const uint32_t key = __float_as_uint((float)z);
                uint32_t *r = &range[2 * (j / kPreprocessBlock)];
                r[0] = std::min(r[0], key);
                r[1] = std::max(r[1], key);
            }
        std::sort(ref.begin(), ref.end(), [&](uint32_t a, uint32_t b) {
            const uint32_t va = one ? 0 : chunk_view[a / kViewChunk], vb = one ? 0 : chunk_view[b / kViewChunk];
            return std::tie(va, dk[a], a) < std::tie(vb, dk[b], b);
        });
        size_t words = 0, clear = 0;
        bucket_work(nullptr, max_n, V, &words, &clear);
        std::vector<uint32_t> work(words, 0xdeadbeefu), alt(n_total, 5u), bucketed(n_total, 5u), out(n_total, 5u);
        std::fill(work.begin(), work.begin() + clear, 0u);
        int64_t counts[2] = {-1, -1};
        depth_order_views(vis.data(), dk.data(), tiles.data(), range.data(), one ? &n_dev : nullptr, n_total,
                          one ? nullptr : table.data(), one ? nullptr : chunk_view.data(), V, max_n, work.data(),
                          alt.data(), bucketed.data(), out.data(), offsets.data(), counts, nullptr);
        uint64_t run = 0;
        int64_t bad = 0;
        for (size_t k = 0; k < ref.size(); ++k) {
            bad += out[k] != ref[k] || offsets[k] != run;
            run += tiles[ref[k]];
        }
        std::printf("trial %zu: %zu visible, %lld misplaced, counts %lld %lld\n", trial, ref.size(), (long long)bad,
                    (long long)counts[0], (long long)counts[1]);
        if (bad || counts[0] != (int64_t)ref.size() || counts[1] != (int64_t)run) return 1;
    }
    return 0;
}

// Host run of the depth order (k_bucket.hip, depth_order_views) over storage
// orders and depth laws: random, ascending and clustered storage, a dense slab
// with a sparse rest, far outliers, and all depths equal (one bucket of many
// LDS pieces, so every merge pass runs).  Checks the order by (float64 depth,
// position) and, but for equal depths, that no bucket outgrows a small multiple
// of the mean, however the entries are stored.
#include "hip/hip_runtime.h"
#include "k_bucket_host.inc"
#include <cstdio>
#include <random>
using namespace fdgs;

int main() {
    std::mt19937_64 rng(5);
    auto uni = [&]() { return std::uniform_real_distribution<double>(0, 1)(rng); };
    struct Case { const char *name; int64_t n; int law, store; };
    const Case cases[] = {{"even, random", 20000, 0, 0},    {"even, ascending", 20000, 0, 1},
                          {"even, clustered", 20000, 0, 2}, {"slab, random", 20000, 1, 0},
                          {"slab, ascending", 20000, 1, 1}, {"outliers, random", 20000, 2, 0},
                          {"few, ascending", 700, 0, 1},    {"equal", 2500, 3, 0}};
    for (const Case &c : cases) {
        const int64_t n = c.n, blocks = (n + kPreprocessBlock - 1) / kPreprocessBlock;
        std::vector<double> z(n);
        for (int64_t i = 0; i < n; ++i) {
            z[i] = 3.0 + 2.0 * uni();
            if (c.law == 1) z[i] = uni() < 0.9 ? 4.0 * (1.0 + 0.01 * uni()) : std::exp(4.0 * uni());
            if (c.law == 2 && i % 4000 == 7) z[i] = i % 8000 == 7 ? 0.02 : 5e4;
            if (c.law == 3) z[i] = 4.0;
        }
        if (c.store) std::sort(z.begin(), z.end());
        if (c.store == 2) {                                    // pieces of 700 neighbours in depth, in any order
            std::vector<int64_t> piece((n + 699) / 700);
            for (size_t k = 0; k < piece.size(); ++k) piece[k] = (int64_t)k;
            std::shuffle(piece.begin(), piece.end(), rng);
            std::vector<double> s;
            for (int64_t p : piece) s.insert(s.end(), z.begin() + p * 700, z.begin() + std::min(n, (p + 1) * 700));
            z = s;
        }
        std::vector<uint8_t> vis(n);
        std::vector<uint64_t> dk(n), offsets(n, 77);
        std::vector<uint32_t> tiles(n), range(2 * blocks, 0u), samples(4 * kSampleBlocks, ~0u), ref;
        for (int64_t b = 0; b < blocks; ++b) range[2 * b] = ~0u;
        for (int64_t j = 0; j < n; ++j) {
            std::memcpy(&dk[j], &z[j], 8);
            vis[j] = rng() % 5 != 0;
            tiles[j] = (uint32_t)(rng() % 9);
            if (!vis[j]) continue;
            ref.push_back((uint32_t)j);
            const uint32_t key = __float_as_uint((float)z[j]);
            uint32_t *r = &range[2 * (j / kPreprocessBlock)];
            r[0] = std::min(r[0], key);
            r[1] = std::max(r[1], key);
            uint32_t &s = samples[j / 64];                     // some visible entry of the wavefront (every
            if (s == ~0u || rng() % 8 == 0) s = key;           // workgroup is sampled: fewer than kSampleBlocks)
        }
        std::sort(ref.begin(), ref.end(), [&](uint32_t a, uint32_t b) { return std::tie(dk[a], a) < std::tie(dk[b], b); });
        size_t words = 0, clear = 0;
        bucket_work(nullptr, n, 1, &words, &clear);
        std::vector<uint32_t> work(words, 0xdeadbeefu), alt(n, 5u), bucketed(n, 5u), out(n, 5u);
        std::fill(work.begin(), work.begin() + clear, 0u);
        int64_t counts[2] = {-1, -1};
        depth_order_views(vis.data(), dk.data(), tiles.data(), range.data(), nullptr, n, nullptr, nullptr, 1, n, work.data(),
                          alt.data(), bucketed.data(), out.data(), offsets.data(), counts, nullptr, samples.data());
        const BucketWork w = bucket_work(work.data(), n, 1, &words, &clear);
        const uint32_t nb = 1u << bucket_log2_for(n);
        uint32_t largest = 0;
        for (uint32_t b = 0; b < nb; ++b) largest = std::max(largest, w.start[b + 1] - w.start[b]);
        uint64_t run = 0;
        int64_t bad = 0;
        for (size_t k = 0; k < ref.size(); ++k) {
            bad += out[k] != ref[k] || offsets[k] != run;
            run += tiles[ref[k]];
        }
        // A bin's share of the sample is within a factor of two, three quarters of the buckets go by it,
        // and a float32 exponent inside a bin halves the density once more: 6 times the mean, and the
        // scatter of a bucket's own count.  The slab's ends lie somewhere inside a part of their bin, whose
        // buckets they share with nothing: there what counts is that no bucket needs merging.
        const double mean = (double)ref.size() / nb;
        const double most = c.law == 3 ? 1e9 : c.law == 1 ? kCap : 6.0 * mean + 5.0 * std::sqrt(6.0 * mean);
        std::printf("%-18s %zu visible, %lld misplaced, largest bucket %u (mean %.1f, at most %.0f)\n", c.name, ref.size(),
                    (long long)bad, largest, mean, most);
        if (bad || counts[0] != (int64_t)ref.size() || counts[1] != (int64_t)run || largest > most) return 1;
    }
    return 0;
}

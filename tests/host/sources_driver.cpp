// Who adds the sources: the tiles (each reads the list) up to 4096 sources and
// 4 Mi pairs of a tile and a source, a launch of their own past either, in the
// one-launch step and, summed over the entries, in a batch.
#include <cstdio>
#include <vector>

#include "fw2.h"
#include "fake_runtime.hpp"

static int g_fail = 0;

struct Sources {
    std::vector<int64_t> idx;
    std::vector<int32_t> sig;
    std::vector<float> w, signals;
    explicit Sources(int n) : idx(n), sig(n, 0), w(n, 1.0f), signals(100, 0.0f)
    {
        for (int q = 0; q < n; ++q) idx[q] = q;
    }
    fw2_status add(fw2_domain *d) const
    {
        return fw2_add_source(d, (int32_t)idx.size(), idx.data(), sig.data(), w.data(), 1, 100, signals.data());
    }
};

static fw2_domain *create(const Uniform &u)
{
    uint64_t bytes = 0;
    fw2_domain *dom = nullptr;
    CHECK(fw2_workspace_bytes_full(&u.d, &bytes) == FW2_OK);
    CHECK(fw2_create_domain(&u.d, fake::alloc(bytes, 0), bytes, &dom) == FW2_OK);
    CHECK(dom && fw2_set_graph_chunk(dom, 0) == FW2_OK);
    return dom;
}

int main()
{
    {
        // 24 x 94 tiles of 64 x 16: 1859 sources are 4 Mi pairs less 400
        Uniform u(1500, 1500, 1, 2);
        fw2_domain *dom = create(u);
        for (int n : {0, 1, 1859, 1860, 4096}) {
            CHECK(Sources(n).add(dom) == FW2_OK);
            CHECK(fw2_step(dom, 2) == FW2_OK);
            CHECK((fake::pressure_variant == 4) == (n <= 1859));
        }
        fw2_destroy_domain(dom);
    }
    {
        // 2 x 16 tiles of 64 x 8: the count limits, not the pairs
        Uniform u(128, 128, 1, 1);
        fw2_domain *dom = create(u);
        for (int n : {4096, 4097}) {
            CHECK(Sources(n).add(dom) == FW2_OK);
            CHECK(fw2_step(dom, 2) == FW2_OK);
            CHECK((fake::pressure_variant == 4) == (n <= 4096));
        }
        fw2_destroy_domain(dom);
    }
    uint64_t bytes = 0;
    CHECK(fw2_batch_workspace_bytes(4, &bytes) == FW2_OK);
    fw2::BatchTable *table = (fw2::BatchTable *)fake::alloc(bytes, 0);
    fw2_batch *b = nullptr;
    CHECK(fw2_batch_create(4, table, bytes, nullptr, &b) == FW2_OK);
    Uniform ua(1024, 512, 1, 4), ub(100, 90, 1, 2);      // 16 x 64 = 1024 tiles of 64 x 8, and 2 x 12
    fw2_domain *one = create(ua), *two = create(ua), *few = create(ub);
    fw2_domain *all[3] = {one, few, two};
    const int64_t steps[3] = {1000, 1000, 1000};
    const struct {
        int n1, nf, n2;
        bool own;                                // a launch of their own
    } cases[] = {{0, 0, 0, false}, {4000, 3, 0, false}, {4096, 0, 0, false}, {4097, 0, 0, true}, {4096, 1, 0, true},
                 {2048, 0, 2048, false}, {2048, 5, 2048, true}, {2049, 0, 2048, true}, {0, 4097, 0, true}};
    for (auto &c : cases) {
        CHECK(Sources(c.n1).add(one) == FW2_OK && Sources(c.nf).add(few) == FW2_OK && Sources(c.n2).add(two) == FW2_OK);
        CHECK(fw2_batch_set_domains(b, 3, all, steps) == FW2_OK);
        CHECK(fw2_batch_step(b, 2) == FW2_OK);
        CHECK(((fake::batch_tile & fw2::kBatchSources) != 0) == c.own);
        int tiles = 0, own = 0;
        for (int k = 0; k < 3; ++k) {
            tiles += table->e[k].a.src.n;
            own += table->e[k].src.n;
        }
        const int total = c.n1 + c.nf + c.n2;
        CHECK(tiles == (c.own ? 0 : total) && (!c.own || own == total));
    }
    fw2_batch_destroy(b);
    for (fw2_domain *d : all) fw2_destroy_domain(d);
    std::printf("sources: %d failed\n", g_fail);
    return g_fail ? 1 : 0;
}

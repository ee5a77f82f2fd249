// Which 2D kernels a grid's size selects: the last grid on one side of each
// limit and the first on the other.
#include <cstdio>

#include "fw2.h"
#include "fake_runtime.hpp"

static int g_fail = 0;

int main()
{
    const struct {
        int64_t nx, ny;
        int L, variant, stream;
    } cases[] = {
        {1500, 1853, 4, 5, 0}, {1500, 1854, 4, 5, 1},          // 22 arrays of 1536 x 1861 or 1862: 240 MiB
        {1500, 1630, 2, 4, 0}, {1500, 1631, 2, 5, 0},          // 25 arrays of 1536 x 1638 or 1639: 240 MiB
        {1024, 256, 4, 4, 0}, {1024, 257, 4, 5, 0},            // 256 or 272 tiles of 64 x 16
        {500, 400, 5, 5, 0},
    };
    for (auto &c : cases) {
        Uniform u(c.nx, c.ny, 1, c.L);
        uint64_t bytes = 0;
        fw2_domain *dom = nullptr;
        CHECK(fw2_workspace_bytes_full(&u.d, &bytes) == FW2_OK);
        CHECK(fw2_create_domain(&u.d, fake::alloc(bytes, 0), bytes, &dom) == FW2_OK);
        CHECK(fw2_set_graph_chunk(dom, 0) == FW2_OK && fw2_step(dom, 2) == FW2_OK);
        CHECK(fake::pressure_variant == c.variant);
        CHECK(fake::pressure_args.stream == c.stream);
        fw2_destroy_domain(dom);
    }
    std::printf("limits: %d failed\n", g_fail);
    return g_fail ? 1 : 0;
}

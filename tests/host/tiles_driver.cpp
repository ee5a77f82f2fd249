// The tile of the batched kernels that each requested tile selects.
#include <cstdio>

#include "fw2.h"
#include "fake_runtime.hpp"

static int g_fail = 0;

int main()
{
    uint64_t bytes = 0, ws = 0;
    CHECK(fw2_batch_workspace_bytes(2, &bytes) == FW2_OK);
    fw2_batch *b = nullptr;
    CHECK(fw2_batch_create(2, fake::alloc(bytes, 0), bytes, nullptr, &b) == FW2_OK);
    Uniform u(100, 90, 1, 2);
    CHECK(fw2_workspace_bytes(&u.d, &ws) == FW2_OK);
    fw2_domain *dom = nullptr;
    CHECK(fw2_create_domain(&u.d, fake::alloc(ws, 0), ws, &dom) == FW2_OK);
    const int64_t steps = 1000;
    const struct {
        int cols, rows, kernel_rows;
    } tiles[] = {{256, 4, 8}, {64, 16, 16}, {64, 8, 8}, {256, 8, 16}, {64, 15, 8}, {64, 1, 8}, {256, 2, 8}, {256, 5, 16},
                 {64, 1024, 16}, {64, 4, 8}};
    CHECK(fw2_batch_set_domains(b, 1, &dom, &steps) == FW2_OK);
    CHECK(fw2_batch_step(b, 1) == FW2_OK && fake::batch_tile == 8);       // the default
    CHECK(fw2_batch_set_tile(b, 64, 16) == FW2_E_STATE);                  // only while it is empty
    for (auto &t : tiles) {
        CHECK(fw2_batch_set_domains(b, 0, nullptr, nullptr) == FW2_OK);
        CHECK(fw2_batch_set_tile(b, t.cols, t.rows) == FW2_OK);
        CHECK(fw2_batch_set_domains(b, 1, &dom, &steps) == FW2_OK);
        CHECK(fw2_batch_step(b, 1) == FW2_OK && fake::batch_tile == t.kernel_rows);
    }
    CHECK(fw2_batch_set_domains(b, 0, nullptr, nullptr) == FW2_OK);
    CHECK(fw2_batch_set_tile(b, 128, 8) == FW2_E_INVALID && fw2_batch_set_tile(b, 64, 0) == FW2_E_INVALID);
    fw2_batch_destroy(b);
    fw2_destroy_domain(dom);
    std::printf("tiles: %d failed\n", g_fail);
    return g_fail ? 1 : 0;
}

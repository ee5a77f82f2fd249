// The workspace a domain needs holds its state and medium once; the second
// state block of the one-launch step is used where the caller's workspace has
// room for it, and lies past everything else.
#include <cstdio>

#include "fw2.h"
#include "fake_runtime.hpp"

static int g_fail = 0;

static fw2_domain *create(const Uniform &u, char *ws, uint64_t bytes, fw2_status want)
{
    fw2_domain *dom = nullptr;
    CHECK(fw2_create_domain(&u.d, ws, bytes, &dom) == want);
    if (dom) CHECK(fw2_set_graph_chunk(dom, 0) == FW2_OK);
    return dom;
}

int main()
{
    const struct {
        int64_t nx, ny, nz;
        int L;
        bool small;                              // a grid of one-launch steps
    } cases[] = {{64, 48, 1, 1, true}, {97, 131, 1, 2, true}, {480, 480, 1, 2, true}, {65, 33, 1, 4, true},
                 {97, 131, 1, 5, false}, {1030, 1000, 1, 4, false}, {20, 16, 12, 2, false}};
    for (auto &c : cases) {
        Uniform u(c.nx, c.ny, c.nz, c.L);
        const int nd = u.d.ndim, n_state = 1 + nd + 2 * nd * c.L;
        const uint64_t stride = (uint64_t)((c.nx + 8 + 63) / 64 * 64) * (c.ny + 8) * (nd == 3 ? c.nz + 8 : 1) * 4;
        uint64_t base = 0, full = 0;
        CHECK(fw2_workspace_bytes(&u.d, &base) == FW2_OK);
        CHECK(fw2_workspace_bytes_full(&u.d, &full) == FW2_OK);
        CHECK(base >= (n_state + 3) * stride && base < (n_state + 3) * stride + 65536);
        CHECK(c.small ? full >= base + n_state * stride && full < base + n_state * stride + 1024 : full == base);
        char *ws = (char *)fake::alloc(full, 0);
        CHECK(create(u, ws, base - 1, FW2_E_NOMEM) == nullptr);
        for (uint64_t bytes : {base, full - 1, full}) {
            if (bytes < base) continue;          // no second block: full - 1 is too small
            const bool one = c.small && bytes == full;
            std::memset(ws, 0xff, full);
            fw2_domain *dom = create(u, ws, bytes, FW2_OK);
            if (!dom) return 1;
            for (uint64_t q = bytes == full ? full : base; q < full; ++q)
                if (ws[q] != (char)0xff) {
                    CHECK(!"nothing past the room in use is written");
                    break;
                }
            const int before = fake::pressure_launches;
            CHECK(fw2_step(dom, 2) == FW2_OK && fake::pressure_launches == before + 2);
            CHECK((fake::pressure_variant == 4) == one);
            if (one) {                           // the second step, back from the shadow block
                const char *shadow = (const char *)fake::pressure_args.p;
                CHECK(fake::pressure_args.out < 0);
                CHECK(shadow >= ws + base && shadow + n_state * stride <= ws + full);
                CHECK(((uintptr_t)shadow - (uintptr_t)(fake::pressure_args.p + fake::pressure_args.out)) % 256 == 0);
            } else {
                CHECK(fake::pressure_args.out == 0);
            }
            CHECK(fw2_step(dom, 1) == FW2_OK && fake::pressure_variant != 4 && fake::pressure_args.out == 0);
            CHECK(fw2_current_step(dom) == 3);
            // out of place the caller's blocks serve: one launch with either workspace
            char *blocks = (char *)fake::alloc(3 * n_state * stride, 0);
            CHECK(fw2_step_into(dom, 2, blocks, blocks + n_state * stride) == FW2_OK);
            CHECK((fake::pressure_variant == 4) == c.small);
            fw2_destroy_domain(dom);
        }
    }
    uint64_t b = 0;
    CHECK(fw2_workspace_bytes_full(nullptr, &b) == FW2_E_INVALID);
    std::printf("workspaces: %d failed\n", g_fail);
    return g_fail ? 1 : 0;
}

// Which field transfers and state copies go by a kernel: only those whose
// buffer lies, whole, on the domain's own device, and only where the launch
// goes there too.  Everything else takes the copy calls, which cross devices.
#include <cstdio>
#include <vector>

#include "fw2.h"
#include "fake_runtime.hpp"

static int g_fail = 0;

int main()
{
    Uniform u(40, 24, 1, 2);
    hipStream_t stream1 = (hipStream_t)(uintptr_t)0x100;     // a stream of device 1
    for (int with_stream = 0; with_stream < 2; ++with_stream) {
        u.d.stream = with_stream ? (void *)stream1 : nullptr;
        uint64_t bytes = 0, state = 0;
        CHECK(fw2_workspace_bytes(&u.d, &bytes) == FW2_OK);
        fake::current_device = 1;
        fw2_domain *dom = nullptr;
        CHECK(fw2_create_domain(&u.d, fake::alloc(bytes, 1), bytes, &dom) == FW2_OK);
        if (!dom) return 1;
        CHECK(fw2_state_bytes(dom, &state) == FW2_OK);
        const uint64_t p_bytes = 40 * 24 * 4;
        for (int cur = 0; cur < 2; ++cur)
            for (int dev = 0; dev < 2; ++dev) {
                fake::current_device = cur;
                const bool kernel = dev == 1 && (with_stream || cur == 1);
                void *field = fake::alloc(p_bytes, dev), *block = fake::alloc(state, dev);
                fake::copies = fake::packs = fake::unpacks = 0;
                CHECK(fw2_read_fields(dom, FW2_FIELD_P, field, FW2_DEVICE) == FW2_OK);
                CHECK(fw2_write_fields(dom, FW2_FIELD_P, field, FW2_DEVICE) == FW2_OK);
                CHECK(fw2_save_state(dom, block) == FW2_OK);
                CHECK(fw2_load_state(dom, block, 0) == FW2_OK);
                CHECK(fake::packs == (kernel ? 2 : 0) && fake::unpacks == (kernel ? 2 : 0));
                CHECK(fake::copies == (kernel ? 0 : 4));
            }
        // a block that ends one element past its allocation
        fake::current_device = 1;
        fake::packs = fake::copies = 0;
        std::vector<float> spare(p_bytes / 4 + 64);
        fake::memory[(uintptr_t)spare.data()] = fake::Allocation{p_bytes - 4, 1};
        CHECK(fw2_read_fields(dom, FW2_FIELD_P, spare.data(), FW2_DEVICE) == FW2_OK);
        CHECK(fake::packs == 0 && fake::copies == 1);
        fake::memory.erase((uintptr_t)spare.data());
        fw2_destroy_domain(dom);
    }
    std::printf("transfer routes: %d failed\n", g_fail);
    return g_fail ? 1 : 0;
}

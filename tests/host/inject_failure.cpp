// A failed injection from host arrays leaves no copy out of the context's pinned
// memory under way: the next injection overwrites that memory.
#include "fake_hip.hpp"

#include "crp.h"

static int check(bool ok, const char* what)
{
    std::printf("%s: %s\n", ok ? "ok" : "FAILED", what);
    return ok ? 0 : 1;
}

int main(int argc, char** argv)
{
    crp_config c;
    std::memset(&c, 0, sizeof c);
    c.precision = CRP_FP64;
    c.field_mode = CRP_FIELD_GRID;
    c.renormalize = 1;
    c.tol = 1e-4;
    c.hmin = 1e20;
    c.hmax = 1e22;
    c.eps_loss = 0.1;
    c.seed = 1;
    c.queue_capacity = 4096;
    c.neutral_capacity = 16;
    c.inject_order = CRP_ORDER_LONGEST_FIRST;
    crp_ctx* ctx = nullptr;
    int bad = check(crp_create(&c, nullptr, &ctx) == CRP_OK, "create");
    if (bad)
        return bad;
    std::vector<double> grid(4 * 4 * 4 * 3, 1e-13);
    const double origin[3] = {0, 0, 0};
    bad += check(crp_set_field_grid(ctx, grid.data(), CRP_F64, 0, 4, 4, 4, 1e21, origin) == CRP_OK,
                 "grid");
    const int n = 1000;
    std::vector<uint32_t> id(n);
    std::vector<int32_t> A(n, 1), Z(n, 1);
    std::vector<double> E(n, 1e19), pos(3 * n, 0.0), dir(3 * n, 0.0), lmax(n, 1e22);
    for (int i = 0; i < n; ++i) {
        id[i] = (uint32_t)i;
        dir[3 * i] = 1.0;
    }
    auto inject = [&] {
        return crp_inject(ctx, n, id.data(), A.data(), Z.data(), E.data(), pos.data(), dir.data(),
                          lmax.data(), 0);
    };
    // (the first injection waits anyway, to allocate the sort's buffers)
    bad += check(inject() == CRP_OK, "first injection");
    for (int i = 1; i < argc; ++i) {
        fake::fail_kernel = argv[i];
        bad += check(inject() == CRP_EDEVICE, (std::string("refused: ") + argv[i]).c_str());
        bad += check(fake::pending.empty(), "no copy under way after the failure");
        fake::fail_kernel.clear();
        bad += check(inject() == CRP_OK, "the same injection goes through afterwards");
        bad += check(fake::pending.empty(), "and waits for its copy");
    }
    crp_destroy(ctx);
    return bad;
}

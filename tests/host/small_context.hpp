// A context on a 4^3 FP64 grid and batches for it, for the drivers of this folder.
#pragma once

#include "fake_hip.hpp"

#include "crp.h"

inline int check(bool ok, const std::string& what)
{
    std::printf("%s: %s\n", ok ? "ok" : "FAILED", what.c_str());
    return ok ? 0 : 1;
}

inline crp_ctx* make_context(int64_t capacity)
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
    c.queue_capacity = capacity;
    c.neutral_capacity = 16;
    c.inject_order = CRP_ORDER_LONGEST_FIRST;
    crp_ctx* ctx = nullptr;
    if (check(crp_create(&c, nullptr, &ctx) == CRP_OK, "create"))
        return nullptr;
    std::vector<double> grid(4 * 4 * 4 * 3, 1e-13);
    const double origin[3] = {0, 0, 0};
    if (check(crp_set_field_grid(ctx, grid.data(), CRP_F64, 0, 4, 4, 4, 1e21, origin) == CRP_OK,
              "grid"))
        return nullptr;
    return ctx;
}

// Two nodes; with channels, both rates are 1e-25 per metre.
inline crp_status set_tables(crp_ctx* ctx, bool channels)
{
    const double e[2] = {1e17, 1e21}, zero[2] = {0, 0}, open[2] = {1e-25, 1e-25};
    return crp_set_tables(ctx, 2, e, channels ? open : zero, channels ? open : zero, zero);
}

// n protons from the origin.
inline crp_status inject(crp_ctx* ctx, int n)
{
    std::vector<uint32_t> id(n);
    std::vector<int32_t> A(n, 1), Z(n, 1);
    std::vector<double> E(n, 1e19), pos(3 * (size_t)n, 0.0), dir(3 * (size_t)n, 0.0),
        lmax(n, 1e22);
    for (int i = 0; i < n; ++i) {
        id[i] = (uint32_t)i;
        dir[3 * (size_t)i] = 1.0;
    }
    return crp_inject(ctx, n, id.data(), A.data(), Z.data(), E.data(), pos.data(), dir.data(),
                      lmax.data(), 0);
}

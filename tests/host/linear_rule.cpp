// Which kernel runs on the linear layout: prints, for each batch size given, the
// layout of the propagation kernel launched and its blocks.
#include "small_context.hpp"

#include "crp_internal.hpp"

int main(int argc, char** argv)
{
    fake::on_launch = [](const std::string& name, dim3 grid, dim3, void** args) {
        const size_t at = name.find("k_propagate");
        if (at == std::string::npos)
            return;
        // k_propagate<int, T, int, ...>: ...ILi0EdLi7ELi128ELb0EE...
        const char layout = name[name.find("dLi", at) + 3];
        const auto* P = *(const crp::PropParams**)args[0];
        std::printf("layout %c lanes %d blocks %d\n", layout, P->lane_cap, (int)grid.x);
    };
    int bad = 0;
    for (int i = 1; i < argc; ++i) {
        const int n = std::atoi(argv[i]);
        crp_ctx* ctx = make_context(n);
        if (!ctx)
            return 1;
        bad += check(set_tables(ctx, true) == CRP_OK, "tables");
        bad += check(inject(ctx, n) == CRP_OK, "inject " + std::to_string(n));
        crp_propagate(ctx, 0);
        crp_destroy(ctx);
    }
    return bad;
}

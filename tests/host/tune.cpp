// What the autotuner launches and what it keeps.  The kernel is a hook that sets the
// run's counters; its duration follows from the launch shape.
//   tune shapes N      prints the trials on N candidates and the shape that is kept
//   tune keep P3 P16   with three blocks per unit P3 percent and refill 16 P16 percent
//                      faster than the filled unit with refill 4: prints the shape kept
//   tune cache FILE    a shape tuned on a small batch is not taken for a large one
#include "small_context.hpp"

#include "crp_internal.hpp"

static int trials = 0;
static bool show = false;
static double three_faster = 0.0, sixteen_faster = 0.0;      // percent

static void kernel(const std::string& name, dim3 grid, dim3 block, void** args)
{
    const size_t at = name.find("k_propagate");
    if (at == std::string::npos)
        return;
    const auto* P = *(const crp::PropParams**)args[0];
    ++trials;
    if (show)
        std::printf("trial layout %c block %d lanes %d refill %d\n", name[name.find("dLi", at) + 3],
                    (int)block.x, P->lane_cap, P->refill);
    P->cnt->steps = 1000000;
    const int waves = (int)grid.x / fake::cus * (int)block.x / 64;
    double ms = waves == 4 ? 20.0 : 10.0;
    if (waves == 6)
        ms /= 1.0 + 0.01 * three_faster;
    if (P->refill == 16)
        ms /= 1.0 + 0.01 * sixteen_faster;
    fake::elapsed_ms = (float)ms;
}

int main(int argc, char** argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    fake::on_launch = kernel;
    crp_ctx* ctx = make_context(1 << 17);
    if (!ctx)
        return 1;
    int bad = check(set_tables(ctx, true) == CRP_OK, "tables");
    crp_launch best;
    double rate = 0.0;
    auto tune = [&](const char* cache) { return crp_tune(ctx, 0, cache, &best, &rate); };
    if (what == "shapes") {
        bad += check(inject(ctx, std::atoi(argv[2])) == CRP_OK, "inject");
        show = true;
        bad += check(tune(nullptr) == CRP_OK, "tune");
    } else if (what == "keep") {
        three_faster = std::atof(argv[2]);
        sixteen_faster = std::atof(argv[3]);
        bad += check(inject(ctx, 70000) == CRP_OK, "inject");
        bad += check(tune(nullptr) == CRP_OK, "tune");
    } else {
        const char* file = argv[2];
        bad += check(inject(ctx, 3000) == CRP_OK && tune(file) == CRP_OK && trials > 0, "small");
        trials = 0;
        bad += check(tune(file) == CRP_OK && trials == 0, "small again: from the cache");
        crp_propagate(ctx, 0);
        trials = 0;
        bad += check(tune(file) == CRP_OK && trials == 0, "nothing pending: from the cache");
        bad += check(inject(ctx, 70000) == CRP_OK && tune(file) == CRP_OK && trials > 0,
                     "large: trials of its own");
        trials = 0;
        bad += check(tune(file) == CRP_OK && trials == 0, "large again: from the cache");
    }
    std::printf("kept block %d blocks %d refill %d\n", best.block, best.blocks_per_cu, best.refill);
    crp_destroy(ctx);
    return bad;
}

// What the autotuner launches and what it keeps.  The kernel is a hook that sets the
// run's counters; its duration follows from the launch shape.
//   tune trials        every trial is launched as a large batch is
//   tune keep PCT      with three blocks per unit PCT percent faster than the filled
//                      unit on the calibration batch: prints the shape that is kept
#include "small_context.hpp"

#include "crp_internal.hpp"

struct Launch {
    int blocks, threads, lane_cap, refill, no_append;
};
static std::vector<Launch> launches;
static double three_faster = 0.0;      // percent

static void kernel(const std::string& name, dim3 grid, dim3 block, void** args)
{
    if (name.find("k_propagate") == std::string::npos)
        return;
    const auto* P = *(const crp::PropParams**)args[0];
    launches.push_back({(int)grid.x, (int)block.x, P->lane_cap, P->refill, P->no_append});
    P->cnt->steps = 1000000;
    const int waves = (int)grid.x / fake::cus * (int)block.x / 64;
    fake::elapsed_ms = waves == 8   ? 10.0f
                       : waves == 6 ? (float)(10.0 / (1.0 + 0.01 * three_faster))
                                    : 20.0f;
}

int main(int argc, char** argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    fake::on_launch = kernel;
    const int n = 300;
    crp_ctx* ctx = make_context(4096);
    if (!ctx)
        return 1;
    int bad = check(set_tables(ctx, what == "keep") == CRP_OK, "tables");
    bad += check(inject(ctx, n) == CRP_OK, "inject");
    if (what == "keep")
        three_faster = std::atof(argv[2]);
    crp_launch best;
    double rate = 0.0;
    launches.clear();
    bad += check(crp_tune(ctx, 0, nullptr, &best, &rate) == CRP_OK && !launches.empty(), "tune");
    if (what == "trials") {
        int refills = 0;
        for (const Launch& l : launches) {
            const bool full = l.blocks == fake::cus * (512 / l.threads);
            const bool few = l.blocks == fake::cus * 3 || l.blocks == fake::cus * 2;
            bad += check(l.lane_cap == 64 && (full || few),
                         "trial of " + std::to_string(l.blocks) + " x " +
                             std::to_string(l.threads) + ", lanes " + std::to_string(l.lane_cap));
            refills |= l.refill == 64 ? 2 : l.refill == 4 ? 1 : 0;
        }
        bad += check(refills == 3, "the refill thresholds are told apart");
        // the run itself is spread: one candidate per wave, no blocks without one
        launches.clear();
        crp_propagate(ctx, 0);
        bad += check(launches.size() == 1 && launches[0].lane_cap == 1 &&
                         launches[0].blocks == (n + launches[0].threads / 64 - 1) /
                                                   (launches[0].threads / 64),
                     "the run is spread");
    } else {
        std::printf("kept %d %d\n", best.block, best.blocks_per_cu);
    }
    crp_destroy(ctx);
    return bad;
}

// A failed injection from host arrays leaves no copy out of the context's pinned
// memory under way: the next injection overwrites that memory.
#include "small_context.hpp"

int main(int argc, char** argv)
{
    const int n = 1000;
    crp_ctx* ctx = make_context(8 * n);
    if (!ctx)
        return 1;
    // (the first injection waits anyway, to allocate the sort's buffers)
    int bad = check(inject(ctx, n) == CRP_OK, "first injection");
    for (int i = 1; i < argc; ++i) {
        fake::fail_kernel = argv[i];
        bad += check(inject(ctx, n) == CRP_EDEVICE, std::string("refused: ") + argv[i]);
        bad += check(fake::pending.empty(), "no copy under way after the failure");
        fake::fail_kernel.clear();
        bad += check(inject(ctx, n) == CRP_OK, "the same injection goes through afterwards");
        bad += check(fake::pending.empty(), "and waits for its copy");
    }
    crp_destroy(ctx);
    return bad;
}

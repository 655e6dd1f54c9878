// Prints the launch plan the library chooses for each grid read from stdin
// ("D Q nx ny nz precision streaming hold", hold planes at either end), one line of name=value pairs per grid.
// The plans are host arithmetic: the kernel launchers are the stubs of
// tests/sanitize/launcher_stubs.cpp.
#include "lbm_api.cpp"

#include <cinttypes>
#include <cstdio>

int main() {
    int D, Q, precision, streaming, hold;
    int64_t ext[3];
    while (std::scanf("%d %d %" SCNd64 " %" SCNd64 " %" SCNd64 " %d %d %d", &D, &Q, &ext[0], &ext[1],
                      &ext[2], &precision, &streaming, &hold) == 8) {
        std::vector<int32_t> e(static_cast<size_t>(Q) * D);
        std::vector<double> w(Q);
        double c = 0;
        const double end[] = {1.0, 0.0, 0.0, 0.5, 0.5};   // (rho, U, T), T > 0 in 2D and 3D
        lbm_ctx* ctx = nullptr;
        if (lbm_velocity_set(D, Q, e.data(), w.data(), &c) != LBM_OK ||
            lbm_create(&ctx, D, Q, e.data(), w.data(), c, ext, 1.3, precision, 1.0, nullptr) !=
                LBM_OK ||
            lbm_set_streaming(ctx, streaming) != LBM_OK ||
            lbm_set_fixed_planes(ctx, hold, hold, end, end) != LBM_OK) {
            std::printf("error=%s\n", lbm_last_error(ctx));
            continue;
        }
        const KParams& k = ctx->kp;
        const long long blocks = lbm::step_blocks(ctx->model, ctx->prec, k);
        const int chunk = cyclic_chunk(k, D);
        std::printf("flat=%d nt=%d rg=%d rs=%d ps=%d gpp=%d chunks=%d rpb=%d bx=%d resident=%d local=%d lds=%d "
                    "split=%d blocks=%lld order=%d strip_steps=%d strip_w=%d strip_threads=%d "
                    "bytes=%zu\n",
                    k.flat, k.nt, k.rg, k.rs, k.ps, k.gpp, k.chunks, k.rpb, k.bx, k.resident, k.resident_local,
                    lbm::held_lds_bytes(k.resident), k.split, blocks, blocks % (8LL * chunk) == 0, k.strip.steps, k.strip.w,
                    k.strip.threads, pop_bytes(ctx));
        lbm_destroy(ctx);
    }
    return 0;
}

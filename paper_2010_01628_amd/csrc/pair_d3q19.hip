// Two-steps-per-pass kernels of the D3Q19 central-moment lattice.
#include "two_step.hpp"

namespace lbm {

void launch_pair_q19(int precision, bool walls, bool general, const void* src, void* dst, const Geom& g, const Phys& ph,
                     const PairShape& sh, uint32_t key2, hipStream_t st)
{
    switch (precision) {
    case PREC_FP64: LaunchPair<LatD3Q19, double>::step(walls, general, src, dst, g, ph, sh, key2, st); break;
    case PREC_FP32: LaunchPair<LatD3Q19, float>::step(walls, general, src, dst, g, ph, sh, key2, st); break;
    case PREC_FP16: LaunchPair<LatD3Q19, _Float16>::step(walls, general, src, dst, g, ph, sh, key2, st); break;
    case PREC_BF16SR: LaunchPair<LatD3Q19, bf16sr_t>::step(walls, general, src, dst, g, ph, sh, key2, st); break;
    default: LaunchPair<LatD3Q19, bf16_t>::step(walls, general, src, dst, g, ph, sh, key2, st); break;
    }
}

int pair_threads_q19(int precision)
{
    return precision == PREC_FP64 ? pair_threads<LatD3Q19, double>() : pair_threads<LatD3Q19, float>();
}

PairShape pair_shape(int nx, int ny, int nz, int q, int eb, int threads, int cus, double* us)
{
    PairShape best{};
    double best_us = 1e300;
    const bool aligned_rows = (int64_t)nx * eb % 128 == 0;
    auto try_shape = [&](int w, int h) {
        const int hx = w < nx, hy = h < ny, W = w + 2 * hx, H = h + 2 * hy;
        const int waves = (W * H + 63) / 64;
        const int tx = (nx + w - 1) / w, ty = (ny + h - 1) / h;
        // 128-byte lines of one array that a plane's loads and stores touch;
        // a tile row that starts or ends inside a line shares that line's
        // store with its neighbour
        const bool aligned = aligned_rows && (int64_t)w * eb % 128 == 0;
        const double row = (double)w * eb / 128;
        const double lines = H * (row + (aligned ? 2 * hx : 1 + hx)) + h * (row + (aligned ? 0 : 2));
        const double plane_us = 0.8 + (eb == 8 ? 2 : 1) * 0.14 * waves * q / 19 + 0.047 * lines * q / 19;
        for (int len = nz, tz = 1;; len = (nz + tz - 1) / tz) { // each length once
            const int64_t groups = (int64_t)tx * ty * tz;
            if (groups > (1 << 20)) break;
            const double t = 2.0 + (double)((groups + cus - 1) / cus) * (len + 2) * plane_us;
            if (t < best_us) {
                best_us = t;
                best = PairShape{w, h, len, tx, ty, tz};
            }
            if (len == 1) break;
            tz = (nz + len - 2) / (len - 1);
        }
    };
    auto rows_for = [&](int w) {
        const int W = w + (w < nx ? 2 : 0);
        if (W > threads) return;
        const int rows = threads / W;
        if (rows >= ny) try_shape(w, ny);
        else if (rows >= 3) {
            const int ty = (ny + rows - 3) / (rows - 2);
            try_shape(w, (ny + ty - 1) / ty);
            if ((ny + rows - 3) / (rows - 2) * (rows - 2) != ny) try_shape(w, rows - 2);
        }
    };
    for (int w = 128 / eb; w < nx; w += 128 / eb) rows_for(w); // whole lines
    for (int w = nx, k = 1;; w = (nx + k - 1) / k) {           // equal tiles
        if (w < 8 && k > 1) break;
        rows_for(w);
        if (w == 1) break;
        k = (nx + w - 2) / (w - 1);
    }
    *us = best_us;
    return best;
}

} // namespace lbm

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

namespace {

// Estimated time of one plane of a w x h tile (PairShape's comment).
double plane_us(int nx, int ny, int q, int eb, bool cached, int w, int h)
{
    const int hx = w < nx, hy = h < ny, W = w + 2 * hx, H = h + 2 * hy;
    const int waves = (W * H + 63) / 64;
    // 128-byte lines of one array that a plane's loads and stores touch; a
    // tile row that starts or ends inside a line shares that line's store
    // with its neighbour, which costs nothing where the last-level cache holds
    // the lattice (100^3 FP32, a pair: 57 us with that share, measured 44)
    const bool aligned = (int64_t)nx * eb % 128 == 0 && (int64_t)w * eb % 128 == 0;
    const double row = (double)w * eb / 128;
    const double lines = H * (row + (aligned ? 2 * hx : (cached ? hx : 1 + hx))) + h * (row + (aligned || cached ? 0 : 2));
    const double us = 0.8 + (eb == 8 ? 2 : 1) * 0.14 * waves * q / 19 + 0.047 * lines * q / 19;
    // three wavefronts per SIMD (D3Q27, 4 bytes) issue less well than two or
    // four: 200^3 505 us without this factor, measured 637, 96^3 50 / 61
    return q == 27 && eb <= 4 ? 1.2 * us : us;
}

// The tile sizes worth trying: widths of whole lines and equal shares of the
// row, each as high as the threads allow, or in equal shares of the columns.
template <class F> void for_tiles(int nx, int ny, int eb, int threads, F&& f)
{
    auto rows_for = [&](int w) {
        const int W = w + (w < nx ? 2 : 0);
        if (W > threads) return;
        const int rows = threads / W;
        if (rows >= ny) f(w, ny);
        else if (rows >= 3) {
            const int ty = (ny + rows - 3) / (rows - 2);
            f(w, (ny + ty - 1) / ty);
            if (ty * (rows - 2) != ny) f(w, rows - 2);
        }
    };
    for (int w = 128 / eb; w < nx; w += 128 / eb) rows_for(w);
    for (int w = nx, k = 1;; w = (nx + k - 1) / k) {
        if (w < 8 && k > 1) break;
        rows_for(w);
        if (w == 1) break;
        k = (nx + w - 2) / (w - 1);
    }
}

} // namespace

PairShape pair_shape(int nx, int ny, int nz, int q, int eb, bool cached, int threads, int cus, double* us)
{
    PairShape best{};
    *us = 1e300;
    for_tiles(nx, ny, eb, threads, [&](int w, int h) {
        const int tx = (nx + w - 1) / w, ty = (ny + h - 1) / h;
        const double plane = plane_us(nx, ny, q, eb, cached, w, h);
        for (int len = nz, tz = 1;; len = (nz + tz - 1) / tz) { // each length once
            const int64_t groups = (int64_t)tx * ty * tz;
            if (groups > (1 << 20)) break;
            const double t = 2.0 + (double)((groups + cus - 1) / cus) * (len + 2) * plane;
            if (t < *us) {
                *us = t;
                best = PairShape{w, h, len, tx, ty, tz, 0, 1};
            }
            if (len == 1) break;
            tz = (nz + len - 2) / (len - 1);
        }
    });
    return best;
}

PairShape pair_block_shape(int nx, int ny, int nz, int threads, int cus)
{
    PairShape best{};
    int least = threads + 1;
    for (int h = 1; h <= ny; ++h) {
        const int H = h + 2 * (h < ny);
        if ((int64_t)nx * H > threads) break;
        for (int d = 1; d <= nz; ++d) {
            const int nodes = nx * H * (d + 2 * (d < nz));
            if (nodes > threads) break;
            const int ty = (ny + h - 1) / h, tz = (nz + d - 1) / d;
            if ((int64_t)ty * tz <= cus && nodes < least) {
                least = nodes;
                best = PairShape{nx, h, d, 1, ty, tz, 1, 0};
            }
        }
    }
    return best;
}
int pair_block_threads_of(int eb)
{
    return eb == 8 ? pair_block_threads<LatD3Q19, double>() : pair_block_threads<LatD3Q19, float>();
}

PairShape pair_tile(int nx, int ny, int q, int eb, bool cached, int threads, double* us)
{
    PairShape best{};
    double best_us = 1e300;
    for_tiles(nx, ny, eb, threads, [&](int w, int h) {
        const int tx = (nx + w - 1) / w, ty = (ny + h - 1) / h;
        const double plane = plane_us(nx, ny, q, eb, cached, w, h);
        if (tx * ty * plane < best_us) {
            best_us = tx * ty * plane;
            *us = plane;
            best = PairShape{w, h, 0, tx, ty, 0, 0, 1};
        }
    });
    return best;
}

} // namespace lbm

// Internal interface between the host API (lbm_api.cpp) and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstdlib>

namespace lbm {

// kernel storage types; PREC_BF16SR: BF16 with stochastic rounding (plain
// D3Q19 central-moment steps only)
enum { PREC_FP64 = 0, PREC_FP32 = 1, PREC_FP16 = 2, PREC_BF16 = 3, PREC_BF16SR = 4 };
enum { FORCE_NONE = 0, FORCE_UNIFORM = 1, FORCE_FIELD = 2, FORCE_ROW_TABLE = 3 };

struct Geom {
    int nx, ny, nz, nxy;
    int N;          // nodes
    int rev = 0;    // single steps: planes last to first; the results do not depend on it
    int64_t stride; // elements between consecutive population arrays (>= N)
    int xcd_chunk = 1; // 1-D step grids: rows per XCD run (1 = launch order)
    int row_stage = 0; // periodic A-B / AA odd step with whole-row work-groups: x-moving populations via LDS
    int flat = 0;      // kernels that use thread_node(): 1-D grid over all nodes in index order
    int off32 = 0;     // every population array is below 4 GiB (32-bit element byte offsets)
    int even_cached = 0; // AA even step with 16-bit storage: population loads without the streaming hint
    int occ_waves = 0;   // step kernels: cap on resident wavefronts per SIMD (0: none), by LDS allocation
    int lds_per_cu = 163840; // bytes of LDS per compute unit
};

// x width of a 256-thread work-group over rows longer than 256 nodes that no
// single work-group spans: the widest of 256, 128, 64 and 32 that divides the
// row (no lane idles at the row's end), else 256
inline int row_width(int nx)
{
    return nx % 256 == 0 ? 256 : nx % 128 == 0 ? 128 : nx % 64 == 0 ? 64 : nx % 32 == 0 ? 32 : 256;
}

struct Phys {
    double omega, omega_bulk, omega_hi[9];
    double rho0;
    int force_mode;
    double force[3];
    const double* force_field; // device, double[3N]
    const double* row_table;   // device, double[ny]: F_x per y row
    uint32_t sr_key;           // stochastic rounding: key of the current step
};

#define LBM_DECLARE_LAUNCHERS(SUFFIX)                                                                              \
    void launch_step_##SUFFIX(int precision, int pattern, bool walls, bool general, bool nt, const void* src,        \
                              void* dst, const Geom& g, const Phys& ph, dim3 grid, dim3 block, hipStream_t st);     \
    void launch_init_##SUFFIX(int precision, int pattern, bool walls, void* buf, const Geom& g, double rho0,         \
                              const double* rho, const double* u, dim3 grid, dim3 block, hipStream_t st);           \
    void launch_set_pops_##SUFFIX(int precision, int pattern, bool walls, void* buf, const Geom& g, double rho0,     \
                                  const double* f, dim3 grid, dim3 block, hipStream_t st);                          \
    void launch_get_pops_##SUFFIX(int precision, int pattern, bool walls, const void* buf, const Geom& g,           \
                                  double rho0, double* f, dim3 grid, dim3 block, hipStream_t st);                   \
    void launch_moments_##SUFFIX(int precision, int pattern, bool walls, const void* buf, const Geom& g,            \
                                 const Phys& ph, double* rho, double* u, double* partials, dim3 grid, dim3 block,   \
                                 hipStream_t st);
LBM_DECLARE_LAUNCHERS(q19)
LBM_DECLARE_LAUNCHERS(q27)
#undef LBM_DECLARE_LAUNCHERS

void launch_step_q19rm(int precision, int pattern, bool walls, bool general, bool nt, const void* src, void* dst,
                       const Geom& g, const Phys& ph, dim3 grid, dim3 block, hipStream_t st);

void launch_step_q27rm(int precision, int pattern, bool walls, bool nt, const void* src, void* dst, const Geom& g,
                       const Phys& ph, dim3 grid, dim3 block, hipStream_t st);

// Dispatch on the lattice (q = 19 or 27) and the moment space.
inline void launch_step(int q, bool raw, int precision, int pattern, bool walls, bool general, bool nt,
                        const void* src, void* dst, const Geom& g, const Phys& ph, dim3 grid, dim3 block,
                        hipStream_t st)
{
    if (q == 27 && raw) launch_step_q27rm(precision, pattern, walls, nt, src, dst, g, ph, grid, block, st);
    else if (q == 27) launch_step_q27(precision, pattern, walls, general, nt, src, dst, g, ph, grid, block, st);
    else if (raw) launch_step_q19rm(precision, pattern, walls, general, nt, src, dst, g, ph, grid, block, st);
    else launch_step_q19(precision, pattern, walls, general, nt, src, dst, g, ph, grid, block, st);
}
inline void launch_init(int q, int precision, int pattern, bool walls, void* buf, const Geom& g, double rho0,
                        const double* rho, const double* u, dim3 grid, dim3 block, hipStream_t st)
{
    if (q == 27) launch_init_q27(precision, pattern, walls, buf, g, rho0, rho, u, grid, block, st);
    else launch_init_q19(precision, pattern, walls, buf, g, rho0, rho, u, grid, block, st);
}
inline void launch_set_pops(int q, int precision, int pattern, bool walls, void* buf, const Geom& g, double rho0,
                            const double* f, dim3 grid, dim3 block, hipStream_t st)
{
    if (q == 27) launch_set_pops_q27(precision, pattern, walls, buf, g, rho0, f, grid, block, st);
    else launch_set_pops_q19(precision, pattern, walls, buf, g, rho0, f, grid, block, st);
}
inline void launch_get_pops(int q, int precision, int pattern, bool walls, const void* buf, const Geom& g, double rho0,
                            double* f, dim3 grid, dim3 block, hipStream_t st)
{
    if (q == 27) launch_get_pops_q27(precision, pattern, walls, buf, g, rho0, f, grid, block, st);
    else launch_get_pops_q19(precision, pattern, walls, buf, g, rho0, f, grid, block, st);
}
inline void launch_moments(int q, int precision, int pattern, bool walls, const void* buf, const Geom& g,
                           const Phys& ph, double* rho, double* u, double* partials, dim3 grid, dim3 block,
                           hipStream_t st)
{
    if (q == 27) launch_moments_q27(precision, pattern, walls, buf, g, ph, rho, u, partials, grid, block, st);
    else launch_moments_q19(precision, pattern, walls, buf, g, ph, rho, u, partials, grid, block, st);
}
// Two steps per pass (two_step.hpp): tiles of w x h columns (tx x ty of them),
// tz runs of len planes; `block`: a thread per node of a w x h x len block.
struct PairShape {
    int w, h, len;
    int tx, ty, tz;
    int block;
    int nt = 1; // streaming hint on the sweeps' stores
};
// Whether passes of two steps, and ensembles, take ordinary accesses instead of
// streaming ones, for a state of this many bytes (all buffers) in x rows of
// row_bytes: where the 256 MiB last-level cache keeps it from one launch to the
// next, or rows that are not whole 128-byte lines share lines, which it merges
// (two steps, streaming / ordinary, us: 200^3 FP32 320 / 265, 330x150x200 FP32 282 /
// 219, FP64 516 / 389).
inline bool ordinary_accesses(int64_t bytes, int buffers, int64_t row_bytes)
{
    return bytes >= (int64_t)24000000 * buffers && (bytes <= ((int64_t)256 << 20) || row_bytes % 128 != 0);
}
// Whether single steps go through the planes upwards and downwards in turn,
// with ordinary accesses: each starts with the planes that the step before
// took last, which the last-level cache still holds.  That pays up to about
// three times its size in place (AA) and twice with two buffers.  Always
// upwards, streaming / in turn, us per step: AA FP32 160^3 (311 MB) 115 / 89,
// 192^3 196 / 160, FP16 256^3 (637 MB) 204 / 191, FP32 256^3 (1.3 GB) 419 / 433;
// A-B FP32 144^3 (454 MB) 101 / 89, FP16 192^3 (538 MB) 96 / 97, FP64 96^3 (269
// MB) 53 / 37; magnetic 96x128x96 (377 MB) 90 / 72, 128x160x128 (839 MB) 156 /
// 158.  Two buffers that fit the cache gain nothing (FP16 144^3 35.7 / 36.1),
// nor do they with 2-byte storage (160^3, 311 MB, 75 / 76).
inline bool alternate_planes(int64_t bytes, int buffers, int elem_bytes)
{
    if (buffers == 1) return bytes >= 24000000 && bytes <= 800000000;
    return elem_bytes >= 4 && bytes > ((int64_t)256 << 20) && bytes <= 480000000;
}
// LBM_TWO_STEP: 0 keeps single steps, 1 takes passes of two wherever they are
// possible; -1: by the estimates.  Without it, a variable that picks a launch
// or an addressing of the single step keeps single steps, which it is about.
inline int two_step_choice()
{
    if (const char* env = std::getenv("LBM_TWO_STEP")) return env[0] == '0' ? 0 : (env[0] == '1' ? 1 : -1);
    const char* off32 = std::getenv("LBM_OFF32");
    const bool single = (off32 && off32[0] == '0') || std::getenv("LBM_ROW_STAGING") || std::getenv("LBM_XCD_CHUNK") ||
                        std::getenv("LBM_WAVES_PER_SIMD");
    return single ? 0 : -1;
}
// Passes of two steps that `nsteps` steps may take on this stream.  A pass
// changes buffers once for its two steps, so a call that is recorded into a
// graph takes an even number of them: it then leaves the populations in the
// buffer that single steps leave them in, and a graph of an even number of
// steps can be replayed.
inline int64_t pairs_in(int64_t nsteps, hipStream_t st)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    // (the null stream cannot be recorded)
    if (nsteps >= 2 && st && hipStreamIsCapturing(st, &status) != hipSuccess) (void)hipGetLastError();
    return status == hipStreamCaptureStatusActive ? nsteps / 4 * 2 : nsteps / 2;
}
// threads of the pair kernel's work-groups (columns of a tile, halo included)
int pair_threads_q19(int precision);
int pair_threads_q27(int precision);
void launch_pair_q19(int precision, bool walls, bool general, const void* src, void* dst, const Geom& g,
                     const Phys& ph, const PairShape& sh, uint32_t key2, hipStream_t st);
void launch_pair_q19rm(int precision, bool walls, bool general, const void* src, void* dst, const Geom& g,
                       const Phys& ph, const PairShape& sh, uint32_t key2, hipStream_t st);
void launch_pair_q27(int precision, bool raw, bool walls, const void* src, void* dst, const Geom& g,
                     const Phys& ph, const PairShape& sh, hipStream_t st);
inline void launch_pair(int q, bool raw, int precision, bool walls, bool general, const void* src, void* dst,
                        const Geom& g, const Phys& ph, const PairShape& sh, uint32_t key2, hipStream_t st)
{
    if (q == 27) launch_pair_q27(precision, raw, walls, src, dst, g, ph, sh, st);
    else if (raw) launch_pair_q19rm(precision, walls, general, src, dst, g, ph, sh, key2, st);
    else launch_pair_q19(precision, walls, general, src, dst, g, ph, sh, key2, st);
}
// Tiles of a pair launch, at most `threads` columns each, one work-group per
// compute unit at a time, and the time estimated for it (microseconds).  The
// estimate, fitted to 64x13, 32x28 and 128x5 tiles on 256^3 with 2- and 4-byte
// storage: a plane takes 0.8 us, 0.14 us per wavefront (its two collisions;
// twice that in FP64) and 0.047 us per 128-byte line of one array that it
// loads or stores (all scaled by q / 19).  `cached`: the last-level cache
// holds the lattice.
PairShape pair_shape(int nx, int ny, int nz, int q, int eb, bool cached, int threads, int cus, double* us);
// The smallest block of whole x rows, at most `threads` nodes with its halo,
// that leaves at most one work-group per compute unit (w = 0: none).  Two
// single steps against blocks, us: 32^3 FP64 10.5 / 7.7, FP32 9.9 / 6.2, FP16
// 9.2 / 5.5, D3Q27 FP32 11.3 / 7.8; 16^3 FP64 10.0 / 5.3; 24^3 FP32 8.5 / 6.1.
// With more than one round of work-groups the halo's steps cost more than the
// launch saved: 48^3 FP32 12.5 / 14.6.
PairShape pair_block_shape(int nx, int ny, int nz, int threads, int cus);
int pair_block_threads_of(int eb);
// The tile with the lowest estimated time for a whole plane of a lattice that
// shares the GPU with others (no run length), and one of its planes' time.
PairShape pair_tile(int nx, int ny, int q, int eb, bool cached, int threads, double* us);

// nout: totals written to out (at most NDIAG_OUT)
void launch_reduce(const double* partials, int nblocks, double* out, hipStream_t st, int nout = 8);

// learned rates (mlp.hip)
constexpr int MLP_PARAMS = 1737;
void launch_step_mlp(int precision, int pattern, bool walls, bool nt, const void* src, void* dst, const Geom& g,
                     const Phys& ph, const void* net, uint32_t* fb_partials, dim3 grid, dim3 block, hipStream_t st);
// FP64 loss partials of launch_train_loss; gradient and loss partials of
// launch_train_backward
int train_loss_parts(const Geom& g);
int train_rows(const Geom& g);
int train_groups(const Geom& g);
// energy (device, [E, E_target]) or nullptr: adds the energy term ew ((E - E_t) / E_t)^2
void launch_train_loss(const float* post, const Geom& g, float rho0, const float* target, const float* inv_sigma,
                       float* gbuf, double* loss_partials, const double* energy, float ew, hipStream_t st);
// per-block partial kinetic energies after each of `steps` steps (posts,
// step_stride floats apart; pulled) and of its target moments:
// partials[2 k train_loss_parts + b] and partials[(2 k + 1) train_loss_parts + b]
void launch_train_energy(const float* posts, int64_t step_stride, int steps, const Geom& g, float rho0, const float* targets,
                         double* partials, hipStream_t st);
// gout != nullptr: also write dL/df(t) (rollout back-propagation), with the
// loss on f(t) against `target` (or nullptr) added to it, by way of `rates`
// (9 N floats) and `xbar` (11 N, dL/dfeatures), both scratch; accumulate: add to
// grad_partials instead of overwriting them
void launch_train_backward(const float* state, const float* gbuf, const Geom& g, const Phys& ph, const void* net,
                           float* grad_partials, float* rates, float* xbar, float* gout, bool accumulate, const float* target,
                           const float* inv_sigma, double* loss_partials, const double* energy, float ew, hipStream_t st);
// tmp: reduce_grad_tmp_bytes() of device scratch
size_t reduce_grad_tmp_bytes();
void launch_reduce_grad(const float* partials, int nparts, double* grad, double* tmp, hipStream_t st);
// out[b] = sum of n partials at partials + b * row, b < rows (the last row: n_last)
void launch_sum_partials(const double* partials, int rows, int64_t row, int n, int n_last, double* out, hipStream_t st);
void launch_adam(float* theta, float* m1, float* m2, const double* grad, float lr, float b1, float b2, float eps,
                 float c1, float c2, hipStream_t st);
void launch_mlp_pack(const float* theta, const float* inv_scale, void* packed, hipStream_t st);
void launch_project_q27(const double* f27, int64_t N, double* f19, float* mom, hipStream_t st);
size_t mlp_packed_bytes();
void launch_feature_sumsq(int precision, int pattern, bool walls, const void* buf, const Geom& g, const Phys& ph,
                          double* partials, double* out, int nblocks, dim3 grid, dim3 block, hipStream_t st);

constexpr int NDIAG_OUT = 8;

} // namespace lbm

// Sets the message returned by lbm_last_error() on this thread.
void lbm_internal_set_error(const char* msg);

// The learned-rate network object behind the opaque lbm_mlp of lbm.h.
struct lbm_mlp {
    hipStream_t stream = nullptr;
    float* theta = nullptr;     // FP32 master parameters (device)
    float* m1 = nullptr;        // Adam moments
    float* m2 = nullptr;
    double* grad = nullptr;     // accumulated gradient (FP64)
    float* inv_scale = nullptr; // 16 floats
    void* packed = nullptr;     // bf16 network for the kernels
    float* inv_sigma = nullptr; // 10 floats
    int64_t adam_t = 0;
    // training scratch, grown on demand
    float* gbuf = nullptr; // two adjoint buffers of 19 N floats (rollouts alternate them)
    int64_t gbuf_elems = 0;
    float* traj = nullptr; // rollout states after steps 1..s (19 x stride floats each)
    int64_t traj_elems = 0;
    float* grad_parts = nullptr;
    int64_t grad_parts_n = 0;
    double* loss_parts = nullptr;
    int64_t loss_parts_n = 0;
    double* loss_dev = nullptr;
    double* loss_host = nullptr;
    double* red_tmp = nullptr; // gradient reduction slices
    float* isig_steps = nullptr; // rollouts: 10 inverse moment scales per step
    int64_t isig_steps_n = 0;
    double* loss_steps = nullptr; // rollouts: loss of each step (device, and its host copy)
    int64_t loss_steps_n = 0;
    double* loss_steps_host = nullptr;
    double energy_weight = 0.0; // rollouts: weight of the kinetic-energy term
    double* energies = nullptr; // rollouts: [E, E_target] per step (device)
    int64_t energies_n = 0;
    double* energy_parts = nullptr; // per-block partial energies of every step
    int64_t energy_parts_n = 0;
};


// ensemble (ensemble.hip)
namespace lbm {
// off32: every box's population arrays are below 4 GiB (32-bit element
// offsets); nt: streaming loads and stores in the plain step
void launch_ens_step(int q, int precision, bool mlp, bool off32, bool nt, const void* src, void* dst, const void* boxes,
                     const int* tile_box, int ntiles, float rho0, const void* net, uint32_t* fb, int grid, int block,
                     int occ_waves, int lds_per_cu, hipStream_t st);
void launch_ens_energy(int q, int precision, const void* buf, const void* boxes, const int* tile_box, int ntiles,
                       int nboxes, const int* tile_count, double rho0, double* tile_out, double* box_out, int grid,
                       hipStream_t st);
size_t ens_box_desc_bytes();
// two plain steps in one pass: one work-group per item of the list, which
// holds the XCDs' items in turn (item k belongs to XCD k % 8); len = 0: none
struct EnsPairItem {
    int box, x0, y0, z0;
    int w, h, len, W;
};
void launch_ens_pair(int q, int precision, const void* src, void* dst, const void* boxes, const EnsPairItem* items,
                     int nitems, float rho0, bool nt, hipStream_t st);
void ens_fill_box_desc(void* out, int L, int tile0, int64_t off, int64_t stride, double omega);
} // namespace lbm

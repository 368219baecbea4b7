// The lattice handle behind the opaque lbm_handle of include/lbm.h, shared by
// the host-side sources of the library.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm.h"
#include "lbm_internal.hpp"
#include "coupled.hpp"

namespace lbm {

// What a lattice's single steps go through, for the choice of their accesses.
struct StepState {
    int64_t bytes;     // all buffers of all lattices
    int buffers;       // of each lattice: 2 (A-B), 1 (AA)
    int elem_bytes, q;
    int coupled;       // lbm_coupling
    bool whole_lines;  // rows, or a staged work-group's rows together, are whole 128-byte lines
};
// Whether single steps take ordinary accesses: where the 256 MiB last-level
// cache keeps the state from one step to the next, with a lower end for small
// states, which streaming accesses serve as well.  us per step, streaming /
// ordinary:
//   plain, 24 MB a buffer for q = 19: FP32 A-B 64^3 (2 x 20 MB) 7.7 / 8.4,
//   64x64x80 11.0 / 10.2, 96^3 27.5 / 22.4, 128x128x100 46.1 / 38.3, FP64 64^3 17.5 /
//   13.6, FP16 128^3 30.8 / 27.0, FP32 AA 128^3 54.6 / 48.8; D3Q27 FP32 64^3 (2 x 28
//   MB) 9.6 / 10.7, 64x64x80 14.9 / 13.0
//   magnetic FP32 64^3 16.5 / 13.6, two-phase FP32 64x64x80 17.4 / 15.4
//   Shan-Chen and two colours, which read a lattice twice: Shan-Chen FP32 64x80x80
//   (62 MB) 16.8 / 18.6, FP64 64^3 (80 MB) 18.5 / 20.4, 64x64x80 (100 MB) 23.6 / 24.3,
//   FP32 128x80x64 (100 MB) 27.5 / 25.0, FP64 80x80x64 (125 MB) 39.1 / 31.6; two colours
//   FP32 64x64x80 (100 MB) 24.5 / 25.6, 128x80x64 (199 MB) 57.0 / 47.0;
//   on rows that share lines Shan-Chen FP32 72x72x64 (50 MB) 15.7 / 16.4, 75^3 (64 MB)
//   23.1 / 21.2
// Beyond the cache only rows that share lines gain: plain FP32 201x199x150 (912
// MB) 265 / 210, D3Q27 437 / 306, FP64 170x150x141 273 / 233, magnetic FP32
// 170x150x141 349 / 304, two-phase FP32 201x199x150 356 / 329, FP64 97x90x80 (290 MB)
// 87.1 / 80.2, 201x199x100 445 / 429, though 100^3 (416 MB) 97.3 / 102.7; Shan-Chen
// FP32 150x140x130 (415 MB) 131 / 125, 201x199x150 (912 MB) 271 / 276; two colours
// FP32 150x130x110 (652 MB) 192 / 201.  Whole lines: FP32 A-B 256x96x100 65.7 / 70.0,
// FP16 AA 192^3 83 / 94 (both upwards; in turn 60 and 72).
inline bool single_ordinary(const StepState& s)
{
    const bool twice = s.coupled == LBM_COUPLED_SHAN_CHEN || s.coupled == LBM_COUPLED_COLOUR;
    const double whole = s.coupled == LBM_COUPLED_COLOUR ? 62.5e6 : 45e6;
    const double least = twice ? (s.whole_lines ? whole : 30e6) : s.coupled ? 24e6 : 24e6 * s.q / 19;
    if ((double)s.bytes < least * s.buffers) return false;
    if (s.bytes <= ((int64_t)256 << 20)) return true;
    if (s.whole_lines || s.coupled == LBM_COUPLED_COLOUR) return false;
    return s.coupled != LBM_COUPLED_SHAN_CHEN || s.bytes <= 480000000;
}

} // namespace lbm

// State of a coupled lattice (lbm_params.coupled != LBM_COUPLED_NONE).
struct lbm_coupled {
    void* buf[2] = {nullptr, nullptr}; // its populations (A-B), same stride as the flow lattice
    int q = 0;                         // populations per node (7 phase, 21 magnetic, 0 Shan-Chen)
    void* scratch = nullptr;           // phase field phi or pseudo-potential psi (collision arithmetic type)
    double sc_G = 0.0;                 // Shan-Chen interaction strength
    lbm::CgConst cc{};                 // colour-gradient constants (buf: blue colour)
    lbm::PhaseConst pc{};
    lbm::MhdConst mc{};
};

struct lbm_handle {
    lbm_params p;
    int kprec = 0;                     // kernel storage type (lbm::PREC_*; BF16SR for stochastic rounding)
    int device = 0;
    hipStream_t stream = nullptr;
    lbm::Geom g{};
    lbm::Phys ph{};
    void* buf[2] = {nullptr, nullptr};
    int cur = 0;
    int64_t steps = 0;
    double* row_table = nullptr;
    double* partials = nullptr;
    double* diag_dev = nullptr;
    double* diag_host = nullptr;
    dim3 grid, block;
    dim3 step_grid, step_block;        // launch shape of the plain step kernel (tunable)
    int row_stage_pref = -1;           // -1: default (staged wherever possible), 0/1: tuner's choice
    lbm::PairShape pair{};             // tiles of the two-steps-per-pass launch
    bool pair_ok = false;              // lbm_step takes two steps per pass where it can
    bool cached = false;               // passes of two steps without the streaming hint (ordinary_accesses)
    bool alternate = false;            // single steps take the planes upwards and downwards in turn
    bool walls = false, general = false, nt = true;
    int64_t bytes = 0;
    int nblocks = 0;
    const lbm_mlp* mlp = nullptr;
    uint32_t* fb_partials = nullptr; // per-block fallback counts of the learned step
    lbm_coupled* cp = nullptr;         // coupled lattice, if any
};

// Grid of the field and diagnostics kernels, which loop over z planes: about
// 4096 work-groups (at least one per x-y block), and their number.
inline dim3 diag_grid(const lbm_handle* h)
{
    const int64_t per_plane = (int64_t)h->grid.x * h->grid.y;
    int64_t gz = 4096 / per_plane;
    gz = gz < 1 ? 1 : (gz > (int64_t)h->grid.z ? (int64_t)h->grid.z : gz);
    return dim3(h->grid.x, h->grid.y, (unsigned)gz);
}
inline int blocks_of(dim3 g) { return (int)(g.x * g.y * g.z); }

// Coupled-lattice parts of the entry points (coupled_api.cpp).
int coupled_validate(const lbm_params* p);
int coupled_create(lbm_handle* h);
void coupled_destroy(lbm_handle* h);
int coupled_step(lbm_handle* h);
int coupled_moments(lbm_handle* h, double* rho, double* u, double* diag, int on_device);
// error reporting of lbm_api.cpp (message for lbm_last_error)
int lbm_fail(int code, const char* fmt, ...);

// Learned-rate D3Q19 step, its training kernels, and the D3Q27 -> D3Q19
// projection that produces training data.
#include "dual.hpp"
#include "lattice_kernels.hpp"
#include "mlp_device.hpp"

namespace lbm {

// Raw features of reading L1 from the pre-collision state (the kernels scale
// them by MlpInfer::inv_scale).
template <class R> __device__ inline void mlp_features(const CMState<R>& st, R x[MLP_NIN])
{
    const R ir = R(1) / st.rho;
    const RawMoments<R>& n = st.n;
    x[0] = st.rho - R(1);
    x[1] = st.k4 * ir;
    x[2] = n.m210 * ir;
    x[3] = n.m120 * ir;
    x[4] = n.m201 * ir;
    x[5] = n.m102 * ir;
    x[6] = n.m021 * ir;
    x[7] = n.m012 * ir;
    x[8] = n.m220 * ir;
    x[9] = n.m202 * ir;
    x[10] = n.m022 * ir;
}

// Collision with learned rates of this lane's node, populations s in place;
// returns whether the node fell back.  All 64 lanes take part.
template <class S, bool SERIAL>
__device__ __attribute__((always_inline)) inline bool learned_collide(const MlpInfer& net, const Phys& ph, const ForceRaw& fr, float s[19])
{
    float Fx, Fy, Fz;
    force_value(ph, fr, Fx, Fy, Fz);
    float xin[MLP_NIN], zout[MLP_NOUT];
    CMState<float> st;
    pre_collide<float, true>(s, (float)ph.rho0, Fx, Fy, Fz, st);
    mlp_features(st, xin);
    mlp_forward_regs<SERIAL>(net, xin, zout);
    const bool fb = mlp_fallback(zout);
    const Rates<float> rt = rates_of<float>(ph);
    RawMoments<float> p;
    if (fb && ph.omega_bulk == 1.0)
        relax<float, false>(st, rt, p); // the paper's rates: the plain step's arithmetic, bit for bit
    else
        relax_learned(st, rt, zout, p);
    if constexpr (Codec<S>::increment)
        post_collide_increment(st, p, s);
    else
        post_collide(st, p, s);
    return fb;
}

// ---------------------------------------------------------------------------
// Step with learned rates (FP32 collision; FP32/FP16/BF16 storage).  Every
// lane of every wavefront takes part in the network (lanes past the lattice
// edge work on a clamped node and store nothing).  The number of nodes that
// fell back is added to fb_partials[block].
// ---------------------------------------------------------------------------
// ROWS (A-B, periodic, work-groups of whole x rows, blockDim.x == nx <= 256):
// the populations that move along x are staged through LDS as in
// k_step_ab_rows (each source row read aligned, once); the network copy's
// barrier serves both.  Same values as the direct reads, bit for bit.
template <class S, Pattern P, bool WALLS, bool NT, bool O32 = false, bool ROWS = false>
__device__ inline void step_mlp_body(const S* src, S* dst, const Geom& g, const Phys& ph,
                                     const MlpPacked* __restrict__ net, uint32_t* __restrict__ fb_partials)
{
    static_assert(!ROWS || (P == AB && !WALLS), "row staging: periodic A-B only");
    // the inference part of the network, once per work-group in LDS: each
    // wavefront reads its MFMA weight operands and bias accumulators from
    // there instead of from memory (~17 KB per wavefront).  Its loads are
    // issued first, the populations' next, so both are in flight together.
    __shared__ __align__(16) uint32_t net_lds[MLP_INFER_WORDS];
    const NetCopy netcopy = net_copy_begin(&net->infer, MLP_INFER_WORDS);
    const MlpInfer* snet = reinterpret_cast<const MlpInfer*>(net_lds);
    const int xr = blockIdx.x * blockDim.x + threadIdx.x;
    const int yr = blockIdx.y * blockDim.y + threadIdx.y;
    const bool valid = xr < g.nx && yr < g.ny;
    const int x = xr < g.nx ? xr : g.nx - 1;
    const int y = yr < g.ny ? yr : g.ny - 1;
    const int z = plane_z(g);
    NodeIdx d;
    node_idx(g, x, y, z, d);
    // the force's loads next, then the populations' (ahead of them for every
    // storage type here: learned FP16 +2-3 %, FP32 within noise)
    const ForceRaw fr = force_load(ph, g, nb(d, 0, 0, 0), y);
    float s[19];
    if constexpr (ROWS) {
        using L = LatD3Q19;
        __shared__ S rows[moving_x_count<L>()][256];
        const int row0 = threadIdx.y * blockDim.x;
        S direct[L::Q];
        {
            int k = 0;
#pragma unroll
            for (int i = 0; i < L::Q; ++i) {
                const S v = ld<S, NT>(pop_at<S, O32, true>(src, g.stride, i, nb(d, 0, -L::cy(i), -L::cz(i))));
                if (L::cx(i) != 0) {
                    rows[k][row0 + x] = v;
                    ++k;
                } else {
                    direct[i] = v;
                }
            }
        }
        net_copy_finish(netcopy, &net->infer, MLP_INFER_WORDS, net_lds);
        int k = 0;
#pragma unroll
        for (int i = 0; i < L::Q; ++i) {
            if (L::cx(i) != 0) {
                int xs = x - L::cx(i);
                xs = xs < 0 ? xs + g.nx : (xs >= g.nx ? xs - g.nx : xs);
                s[i] = Codec<S>::dec(rows[k][row0 + xs]);
                ++k;
            } else {
                s[i] = Codec<S>::dec(direct[i]);
            }
        }
    } else {
        gather<LatD3Q19, S, P, WALLS, NT, O32>(src, g.stride, d, s);
        net_copy_finish(netcopy, &net->infer, MLP_INFER_WORDS, net_lds);
    }
    // SERIAL (mlp_block_regs): the AA steps and streamed 2-byte A-B
    const bool fb = learned_collide<S, P != AB || (NT && sizeof(S) == 2)>(*snet, ph, fr, s);
    if (valid) scatter<LatD3Q19, S, P, WALLS, NT, O32>(dst, g.stride, d, s);
    // fallback count: one atomic add per wavefront that has fallen-back
    // nodes (none in normal operation), so a wavefront neither waits for the
    // others of its block nor for a read before it retires
    const uint64_t ballot = __ballot(valid && fb);
    if (ballot != 0 && ((threadIdx.x + blockDim.x * threadIdx.y) & 63) == 0) {
        const int bid = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
        atomicAdd(&fb_partials[bid], (uint32_t)__popcll(ballot));
    }
}

// Four waves per SIMD or more without spills, three for the AA odd step with
// walls.
template <class S, bool WALLS, bool NT, bool O32, bool ROWS = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_step_mlp_ab(
    const S* src, S* dst, Geom g, Phys ph, const MlpPacked* __restrict__ net, uint32_t* __restrict__ fb_partials)
{
    step_mlp_body<S, AB, WALLS, NT, O32, ROWS>(src, dst, g, ph, net, fb_partials);
}

template <class S, Pattern P, bool WALLS, bool NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((P == AA_ODD && WALLS ? 3 : 4)))) void k_step_mlp(const S* src, S* dst, Geom g, Phys ph,
                                                  const MlpPacked* __restrict__ net, uint32_t* __restrict__ fb_partials)
{
    step_mlp_body<S, P, WALLS, NT>(src, dst, g, ph, net, fb_partials);
}

// ---------------------------------------------------------------------------
// Training, reading L5: loss on the 10 raw moments of f(t+1) after one A-B
// step from f(t) (periodic, no force).
//
// Energy term (rollouts, `energy` != nullptr): the gradient of
// ew ((E - E_t) / E_t)^2, with the kinetic energies E = 1/2 sum |j|^2 / rho of
// the populations and E_t of the target moments (energy[0] = E, energy[1] =
// E_t, from k_train_energy), is added per node: 2 ew (E - E_t) / E_t^2
// (c_i . u - |u|^2 / 2).  The term's value is formed by the host.
// ---------------------------------------------------------------------------
// Loss of one node with populations s (deviations): its sum of squares, and
// dL/df_i to put(i, value) for every i that want(i).
template <class W, class P>
__device__ __attribute__((always_inline)) inline double train_loss_node(const float s[19], int n, int N, float rho0, const float* __restrict__ target,
                                         const float* __restrict__ inv_sigma, const double* __restrict__ energy, float ew,
                                         W want, P put)
{
    // moments of f = w rho0 + s: rest part (1, 0,0,0, 1/3 x3, 0 x3) rho0
    float m[10] = {rho0, 0, 0, 0, rho0 / 3.0f, rho0 / 3.0f, rho0 / 3.0f, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 19; ++i) {
        const float cx = LatD3Q19::cx(i), cy = LatD3Q19::cy(i), cz = LatD3Q19::cz(i);
        m[0] += s[i];
        m[1] += cx * s[i];
        m[2] += cy * s[i];
        m[3] += cz * s[i];
        m[4] += cx * cx * s[i];
        m[5] += cy * cy * s[i];
        m[6] += cz * cz * s[i];
        m[7] += cx * cy * s[i];
        m[8] += cx * cz * s[i];
        m[9] += cy * cz * s[i];
    }
    double l2 = 0.0;
    float dm[10];
    const float two_over_n = 2.0f / (float)N;
#pragma unroll
    for (int k = 0; k < 10; ++k) {
        const float r = (m[k] - target[(int64_t)k * N + n]) * inv_sigma[k];
        l2 += (double)r * (double)r;
        dm[k] = two_over_n * r * inv_sigma[k];
    }
    float ce = 0.0f, ux = 0.0f, uy = 0.0f, uz = 0.0f, u2 = 0.0f;
    if (energy) {
        ce = (float)(2.0 * ew * (energy[0] - energy[1]) / (energy[1] * energy[1]));
        const float ir = 1.0f / m[0];
        ux = m[1] * ir;
        uy = m[2] * ir;
        uz = m[3] * ir;
        u2 = 0.5f * (ux * ux + uy * uy + uz * uz);
    }
#pragma unroll
    for (int i = 0; i < 19; ++i) {
        if (!want(i)) continue;
        const float cx = LatD3Q19::cx(i), cy = LatD3Q19::cy(i), cz = LatD3Q19::cz(i);
        float gi = dm[0] + cx * dm[1] + cy * dm[2] + cz * dm[3] + cx * cx * dm[4] + cy * cy * dm[5] + cz * cz * dm[6] +
                   cx * cy * dm[7] + cx * cz * dm[8] + cy * cz * dm[9];
        if (energy) gi += ce * (cx * ux + cy * uy + cz * uz - u2);
        put(i, gi);
    }
    return l2;
}

// node n of the lattice
__device__ inline void node_of(const Geom& g, int n, NodeIdx& d)
{
    const int r = n / g.nx;
    node_idx(g, n - r * g.nx, r % g.ny, r / g.ny, d);
}

// Loss after the last step of a rollout (or the only one) and dL/df_i(y, t+1),
// written to gbuf (SoA floats, stride N); post: post-collision buffer written
// by the learned step (A-B).  256 consecutive nodes per block, one FP64 loss
// partial each.
__global__ __launch_bounds__(256) void k_train_loss(const float* __restrict__ post, Geom g, float rho0,
                                                    const float* __restrict__ target, const float* __restrict__ inv_sigma,
                                                    float* __restrict__ gbuf, double* __restrict__ loss_partials,
                                                    const double* __restrict__ energy, float ew)
{
    __shared__ double red[4];
    const int n = blockIdx.x * 256 + threadIdx.x;
    double v = 0.0;
    if (n < g.N) {
        NodeIdx d;
        node_of(g, n, d);
        float s[19];
        gather<LatD3Q19, float, AB, false>(post, g.stride, d, s);
        v = train_loss_node(s, n, g.N, rho0, target, inv_sigma, energy, ew, [](int) { return true; },
                            [&](int i, float gi) { gbuf[(int64_t)i * g.N + n] = gi; });
    }
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) loss_partials[blockIdx.x] = ((red[0] + red[1]) + (red[2] + red[3])) / (double)g.N;
}

// Per-block FP64 partial kinetic energies 1/2 |j|^2 / rho of the populations
// pulled after each step (no force; blockIdx.y = step, states `stride` floats
// apart) and of its target moments (rho, j), 256 consecutive nodes per block:
// out[(2 step) gridDim.x + b] and out[(2 step + 1) gridDim.x + b].
__global__ __launch_bounds__(256) void k_train_energy(const float* __restrict__ posts, int64_t step_stride, Geom g, float rho0,
                                                      const float* __restrict__ targets, double* __restrict__ out)
{
    __shared__ double red[2][4];
    const float* post = posts + (int64_t)blockIdx.y * step_stride;
    const float* target = targets + (int64_t)blockIdx.y * 10 * g.N;
    const int n = blockIdx.x * 256 + threadIdx.x;
    double e = 0.0, et = 0.0;
    if (n < g.N) {
        NodeIdx d;
        node_of(g, n, d);
        float s[19];
        gather<LatD3Q19, float, AB, false>(post, g.stride, d, s);
        double r = rho0, jx = 0.0, jy = 0.0, jz = 0.0;
#pragma unroll
        for (int i = 0; i < 19; ++i) {
            r += s[i];
            jx += LatD3Q19::cx(i) * (double)s[i];
            jy += LatD3Q19::cy(i) * (double)s[i];
            jz += LatD3Q19::cz(i) * (double)s[i];
        }
        e = 0.5 * (jx * jx + jy * jy + jz * jz) / r;
        const double rt = target[n], tx = target[(int64_t)g.N + n], ty = target[2 * (int64_t)g.N + n],
                     tz = target[3 * (int64_t)g.N + n];
        et = 0.5 * (tx * tx + ty * ty + tz * tz) / rt;
    }
    e = wave_sum(e);
    et = wave_sum(et);
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = e;
        red[1][threadIdx.x >> 6] = et;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const double* r = red[threadIdx.x];
        out[(int64_t)(2 * blockIdx.y + threadIdx.x) * gridDim.x + blockIdx.x] = (r[0] + r[1]) + (r[2] + r[3]);
    }
}

// Backward pass, a wavefront per x row (per 64 nodes of a longer one):
// recompute the forward state from f(t), pull dL/df*_i(x) = dL/df_i(x + c_i,
// t+1), form dL/domega_j = kbar_{10+j} (-(k_{10+j} - k_eq) - R_{10+j}/2) with
// kbar = S(+u)^T M^-T gbar, then back-propagate through the network.  Writes
// the row's 1737 gradient entries to grad_partials[row].
//
// PROP (rollouts): also the rates (1 of nodes that fall back), rates_out[j N +
// x], and dL/dx of the features (ReLU masks, W1^T, the input scales),
// xbar_out[i N + x], for k_train_dstate.
//
// What bounds both: latency and, in k_train_dstate, issue; a 32^3 step is 1024
// rows.  32^3, us per step, both together: 47 with all derivatives in the row's
// own wavefront, 44 with one wavefront per derivative of 64 nodes, 35 with
// three derivatives to a wavefront.  The loss on f(t) and the energies were
// three more launches per step (15 us).
struct TrainLoss {
    const float* target;    // NULL: no loss on f(t)
    const float* inv_sigma;
    const double* energy;   // or NULL
    float ew;
    double* partials;
};
template <bool PROP>
__global__ __launch_bounds__(64) void k_train_backward(const float* __restrict__ state, const float* __restrict__ gbuf,
                                                       Geom g, Phys ph, const MlpPacked* __restrict__ net,
                                                       float* __restrict__ grad_partials, float* __restrict__ rates_out,
                                                       float* __restrict__ xbar_out, int accumulate)
{
    const float rho0 = (float)ph.rho0;
    __shared__ MlpTrain snet;
    __shared__ uint16_t tx[MLP_TILE], th1[MLP_TILE], th2[MLP_TILE], tdz[MLP_TILE], tdh[MLP_TILE];
    __shared__ float tz[64 * MLP_NOUT];
    const int l = threadIdx.x;
    const int xr = blockIdx.x * 64 + l;
    const bool valid = xr < g.nx;
    NodeIdx d;
    node_idx(g, valid ? xr : g.nx - 1, blockIdx.y, blockIdx.z, d);
    float s[19], gbar[19];
    gather<LatD3Q19, float, AB, false>(state, g.stride, d, s);
    // adjoint of the streaming
#pragma unroll
    for (int i = 0; i < 19; ++i)
        gbar[i] = gbuf[(int64_t)i * g.N + nb(d, LatD3Q19::cx(i), LatD3Q19::cy(i), LatD3Q19::cz(i))];
    // the network, and with `accumulate` the partials of the later steps, which
    // this step's are added to: everything the wavefront reads is in flight at once
    constexpr int NCHUNK = (int)sizeof(MlpTrain) / 16;
    uint4 nc[(NCHUNK + 63) / 64];
#pragma unroll
    for (int c = 0; c < (NCHUNK + 63) / 64; ++c) nc[c] = reinterpret_cast<const uint4*>(&net->train)[min(c * 64 + l, NCHUNK - 1)];
    float* gp = grad_partials + (int64_t)(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z)) * MLP_NPARAM;
    const int col = l & 31, row4 = 4 * (l >> 5); // accumulator register r: row 8 (r / 4) + row4 + r % 4, column col
    float g1[16], g2[16], g3[5], gb[3];
    {
        const float* q = gp;
        auto old = [&](bool on, int at) { return accumulate && on ? q[at] : 0.0f; };
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = 8 * (r >> 2) + row4 + (r & 3);
            g1[r] = old(col < MLP_NIN, MLP_OFF_W1 + row * MLP_NIN + col);
            g2[r] = old(true, MLP_OFF_W2 + row * 32 + col);
            if (r < 5) g3[r] = old(row < MLP_NOUT, MLP_OFF_W3 + row * 32 + col);
        }
        gb[0] = old(l < 32, MLP_OFF_B1 + l);
        gb[1] = old(l < 32, MLP_OFF_B2 + l);
        gb[2] = old(l < MLP_NOUT, MLP_OFF_B3 + l);
    }
#pragma unroll
    for (int c = 0; c < (NCHUNK + 63) / 64; ++c) reinterpret_cast<uint4*>(&snet)[min(c * 64 + l, NCHUNK - 1)] = nc[c];
    __syncthreads();
    CMState<float> st;
    pre_collide<float, true>(s, rho0, 0.0f, 0.0f, 0.0f, st);
    float xin[MLP_NIN], zout[MLP_NOUT], rates[MLP_NOUT];
    mlp_features(st, xin);
    mlp_forward_wave(snet, tx, th1, th2, tz, xin, zout);
    const bool fb = mlp_rates(zout, rates);
    RawMoments<float> kb;
    pops_from_raw_T(gbar, kb);
    shift_all_T(kb, st.ux, st.uy, st.uz);
    const RawMoments<float>& n = st.n;
    // no force in training: R = 0 on rows 10..18
    float dz[MLP_NOUT] = {-kb.m210 * n.m210, -kb.m120 * n.m120, -kb.m201 * n.m201, -kb.m102 * n.m102, -kb.m021 * n.m021,
                          -kb.m012 * n.m012, -kb.m220 * n.m220, -kb.m202 * n.m202, -kb.m022 * n.m022};
    const bool active = valid && !fb;
#pragma unroll
    for (int k = 0; k < 32; ++k) tdz[l * MLP_LDS_STRIDE + k] = (k < MLP_NOUT && active) ? f32_to_bf16(dz[k]) : 0;
    __syncthreads();
    // column sums of a tile: each half-wave its 32 rows, then together
    auto column_sum = [&](const uint16_t* t) {
        float sb = 0.0f;
#pragma unroll
        for (int q = 0; q < 32; ++q) sb += bf16_to_f32(t[((l & 32) + q) * MLP_LDS_STRIDE + (l & 31)]);
        return sb + __shfl_xor(sb, 32, 64);
    };
    // dW3[o][h] = sum_n dz[n][o] h2[n][h]
    {
        const f32x16_t acc = mfma_AtB(tdz, th2);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int o = 8 * (r >> 2) + row4 + (r & 3);
            if (r < 5 && o < MLP_NOUT) gp[MLP_OFF_W3 + o * 32 + col] = g3[r < 5 ? r : 0] + acc[r];
        }
    }
    // db3, and dh2 = (dz W3) * relu'(h2)
    {
        const float sb = column_sum(tdz);
        if (l < MLP_NOUT) gp[MLP_OFF_B3 + l] = gb[2] + sb;
    }
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
        const f32x16_t acc = mfma_xwT<32>(tdz, rb, snet.w3t, 32);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = acc_row(rb, r), h = l & 31;
            const float a2 = bf16_to_f32(th2[row * MLP_LDS_STRIDE + h]);
            tdh[row * MLP_LDS_STRIDE + h] = f32_to_bf16(a2 > 0.0f ? acc[r] : 0.0f);
        }
    }
    __syncthreads();
    // dW2, db2, dh1 = (dh2 W2) * relu'(h1) written over tdz
    {
        const f32x16_t acc = mfma_AtB(tdh, th1);
#pragma unroll
        for (int r = 0; r < 16; ++r) gp[MLP_OFF_W2 + (8 * (r >> 2) + row4 + (r & 3)) * 32 + col] = g2[r] + acc[r];
    }
    {
        const float sb = column_sum(tdh);
        if (l < 32) gp[MLP_OFF_B2 + l] = gb[1] + sb;
    }
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
        const f32x16_t acc = mfma_xwT<32>(tdh, rb, snet.w2t, 32);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = acc_row(rb, r), h = l & 31;
            const float a1 = bf16_to_f32(th1[row * MLP_LDS_STRIDE + h]);
            tdz[row * MLP_LDS_STRIDE + h] = f32_to_bf16(a1 > 0.0f ? acc[r] : 0.0f);
        }
    }
    __syncthreads();
    // dW1[o][i] = sum_n dh1[n][o] x[n][i], db1
    {
        const f32x16_t acc = mfma_AtB(tdz, tx);
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (col < MLP_NIN) gp[MLP_OFF_W1 + (8 * (r >> 2) + row4 + (r & 3)) * MLP_NIN + col] = g1[r] + acc[r];
    }
    {
        const float sb = column_sum(tdz);
        if (l < 32) gp[MLP_OFF_B1 + l] = gb[0] + sb;
    }
    if constexpr (PROP) {
        if (!valid) return;
        const int n0 = nb(d, 0, 0, 0);
        // xbar = (W1^T dh1) * inv_scale: dh1 of this lane's node is row l of tdz
        float xbar[MLP_NIN];
#pragma unroll
        for (int i = 0; i < MLP_NIN; ++i) xbar[i] = 0.0f;
#pragma unroll 8
        for (int o = 0; o < 32; ++o) {
            const float dh = bf16_to_f32(tdz[l * MLP_LDS_STRIDE + o]);
            const uint4 *wr = reinterpret_cast<const uint4*>(snet.w1 + o * 16), w0 = wr[0], w1 = wr[1];
            const uint32_t ww[6] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y};
#pragma unroll
            for (int i = 0; i < MLP_NIN; ++i) xbar[i] += dh * bf16_to_f32((uint16_t)(ww[i / 2] >> (16 * (i & 1))));
        }
#pragma unroll
        for (int j = 0; j < MLP_NOUT; ++j) rates_out[(int64_t)j * g.N + n0] = rates[j];
#pragma unroll
        for (int i = 0; i < MLP_NIN; ++i) xbar_out[(int64_t)i * g.N + n0] = xbar[i] * snet.inv_scale[i];
    }
}

// dL/df_j(x, t), written to gout[j N + x]: forward derivatives of the collision
// along TRAIN_K populations j from TRAIN_K blockIdx.y (dual.hpp), at fixed rates and
// through the features, with the rates and dL/dfeatures of k_train_backward.
// With `target` (every step but the first) the loss on f(t) itself is added,
// and its sum of squares goes to loss_partials[64-node block].
// Three populations to a wavefront share the collision's values (2783 VALU
// instructions per wavefront); 32^3, 32 steps of a rollout, us: one 1748, two
// 1527, three 1447, four 1630 (spills).
constexpr int TRAIN_K = 3;
__global__ __launch_bounds__(64) void k_train_dstate(
    const float* __restrict__ state, const float* __restrict__ gbuf, Geom g, Phys ph, const float* __restrict__ rates,
    const float* __restrict__ xbar_in, float* __restrict__ gout, TrainLoss tl)
{
    const float rho0 = (float)ph.rho0;
    const int nr = blockIdx.x * 64 + threadIdx.x, j0 = TRAIN_K * blockIdx.y;
    typedef Dual<TRAIN_K> D;
    const bool valid = nr < g.N;
    const int n0 = valid ? nr : g.N - 1;
    NodeIdx d;
    node_of(g, n0, d);
    float s[19], gbar[19];
    gather<LatD3Q19, float, AB, false>(state, g.stride, d, s);
#pragma unroll
    for (int i = 0; i < 19; ++i)
        gbar[i] = gbuf[(int64_t)i * g.N + nb(d, LatD3Q19::cx(i), LatD3Q19::cy(i), LatD3Q19::cz(i))];
    auto constant = [](float c) {
        D r(0.0);
        r.v = c;
        return r;
    };
    Rates<D> rt = rates_of<D>(ph);
    float xbar[MLP_NIN];
#pragma unroll
    for (int k = 0; k < MLP_NOUT; ++k) rt.omega_hi[k] = constant(rates[(int64_t)k * g.N + n0]);
#pragma unroll
    for (int k = 0; k < MLP_NIN; ++k) xbar[k] = xbar_in[(int64_t)k * g.N + n0];
    float loss[TRAIN_K] = {};
    if (tl.target) {
        double l2 = train_loss_node(s, n0, g.N, rho0, tl.target, tl.inv_sigma, tl.energy, tl.ew,
                                    [&](int i) { return i >= j0 && i < j0 + TRAIN_K; }, [&](int i, float gi) {
#pragma unroll
                                        for (int k = 0; k < TRAIN_K; ++k)
                                            if (i == j0 + k) loss[k] = gi;
                                    });
        if (j0 == 0) {
            l2 = wave_sum(valid ? l2 : 0.0);
            if (threadIdx.x == 0) tl.partials[blockIdx.x] = l2 / (double)g.N;
        }
    }
    D sd[19];
#pragma unroll
    for (int i = 0; i < 19; ++i) {
        sd[i].v = s[i];
#pragma unroll
        for (int k = 0; k < TRAIN_K; ++k) sd[i].d[k] = i == j0 + k ? 1.0f : 0.0f;
    }
    CMState<D> sdt;
    pre_collide<D, true>(sd, constant(rho0), D(0.0), D(0.0), D(0.0), sdt);
    D xd[MLP_NIN];
    mlp_features(sdt, xd);
    RawMoments<D> pd;
    relax<D, true>(sdt, rt, pd);
    post_collide_increment(sdt, pd, sd);
#pragma unroll
    for (int k = 0; k < TRAIN_K; ++k) {
        if (j0 + k >= 19) break;
        float acc = 0.0f;
#pragma unroll
        for (int i = 0; i < 19; ++i) acc += gbar[i] * sd[i].d[k];
#pragma unroll
        for (int i = 0; i < MLP_NIN; ++i) acc += xbar[i] * xd[i].d[k];
        if (tl.target) acc = acc + loss[k];
        if (valid) gout[(int64_t)(j0 + k) * g.N + n0] = acc;
    }
}

// grad[p] += sum over the per-wavefront partials, in FP64 and a fixed order
// (repeatable bit for bit).  Stage 1: block (x, y) sums slice y of the
// partials for 64 parameters, four lanes per parameter over interleaved
// partials (each wavefront reads 64 consecutive floats per partial), into
// tmp[y][p]; stage 2 adds the slices.
constexpr int MLP_RED_SLICES = 32;
__global__ __launch_bounds__(256) void k_reduce_grad_slices(const float* __restrict__ partials, int nparts,
                                                            double* __restrict__ tmp)
{
    __shared__ double red[4][64];
    const int l = threadIdx.x & 63, sub = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + l;
    const int chunk = (nparts + MLP_RED_SLICES - 1) / MLP_RED_SLICES;
    const int w0 = blockIdx.y * chunk, w1 = min(nparts, w0 + chunk);
    double s = 0.0;
    if (p < MLP_NPARAM)
        for (int w = w0 + sub; w < w1; w += 4) s += (double)partials[(int64_t)w * MLP_NPARAM + p];
    red[sub][l] = s;
    __syncthreads();
    if (sub == 0 && p < MLP_NPARAM) tmp[(int64_t)blockIdx.y * MLP_NPARAM + p] = (red[0][l] + red[1][l]) + (red[2][l] + red[3][l]);
}
__global__ __launch_bounds__(256) void k_reduce_grad(const double* __restrict__ tmp, double* __restrict__ grad)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= MLP_NPARAM) return;
    double s = 0.0;
    for (int y = 0; y < MLP_RED_SLICES; ++y) s += tmp[(int64_t)y * MLP_NPARAM + p];
    grad[p] += s;
}

// out[b] = sum of the n partials at partials + b * row (the last row: n_last of them), fixed order
__global__ __launch_bounds__(256) void k_sum_partials(const double* __restrict__ partials, int64_t row, int n, int n_last,
                                                      double* __restrict__ out)
{
    __shared__ double red[256];
    const double* p = partials + (int64_t)blockIdx.x * row;
    const int count = blockIdx.x == gridDim.x - 1 ? n_last : n;
    double s = 0.0;
    for (int i = threadIdx.x; i < count; i += 256) s += p[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

// Adam on the FP32 master parameters (FP64 gradient).
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ theta, float* __restrict__ m1, float* __restrict__ m2,
                                              const double* __restrict__ grad, float lr, float b1, float b2, float eps,
                                              float c1, float c2)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= MLP_NPARAM) return;
    const float gr = (float)grad[p];
    const float a = b1 * m1[p] + (1.0f - b1) * gr;
    const float b = b2 * m2[p] + (1.0f - b2) * gr * gr;
    m1[p] = a;
    m2[p] = b;
    theta[p] -= lr * (a / c1) / (sqrtf(b / c2) + eps);
}

// FP32 master parameters + inverse feature scales -> packed bf16 network.
__global__ __launch_bounds__(256) void k_mlp_pack(const float* __restrict__ theta, const float* __restrict__ inv_scale,
                                                  MlpPacked* __restrict__ out)
{
    const int t = threadIdx.x;
    MlpInfer& in = out->infer;
    MlpTrain& tr = out->train;
    for (int i = t; i < 5 * 512; i += 256) {
        const int p = i / 512, l = i % 512 / 8, k = mlp_op_unit(p, l, i % 8), o = l & 31;
        float w = 0.0f;
        if (p == 0) w = k < MLP_NIN ? theta[MLP_OFF_W1 + o * MLP_NIN + k] : 0.0f;
        else if (p < 3) w = theta[MLP_OFF_W2 + o * 32 + k];
        else w = o < MLP_NOUT ? theta[MLP_OFF_W3 + o * 32 + k] : 0.0f;
        in.op[p][i % 512] = f32_to_bf16(w);
    }
    for (int i = t; i < 32 * 16; i += 256) {
        const int o = i / 16, k = i % 16;
        tr.w1[i] = k < MLP_NIN ? f32_to_bf16(theta[MLP_OFF_W1 + o * MLP_NIN + k]) : 0;
    }
    for (int i = t; i < 32 * 32; i += 256) {
        const int o = i / 32, k = i % 32;
        const uint16_t v2 = f32_to_bf16(theta[MLP_OFF_W2 + o * 32 + k]);
        tr.w2[i] = v2;
        tr.w2t[k * 32 + o] = v2;
        const uint16_t v3 = o < MLP_NOUT ? f32_to_bf16(theta[MLP_OFF_W3 + o * 32 + k]) : 0;
        tr.w3[i] = v3;
        tr.w3t[k * 32 + o] = v3;
    }
    if (t < 32) {
        in.b1[t] = tr.b1[t] = theta[MLP_OFF_B1 + t];
        in.b2[t] = tr.b2[t] = theta[MLP_OFF_B2 + t];
        in.b3[t] = tr.b3[t] = t < MLP_NOUT ? theta[MLP_OFF_B3 + t] : 0.0f;
    }
    if (t < 16) in.inv_scale[t] = tr.inv_scale[t] = t < MLP_NIN ? inv_scale[t] : 0.0f;
}

// D3Q27 populations (canonical, double) -> D3Q19 populations with the same 19
// raw moments, and the 10 moments (rho, j, Pi) of the D3Q27 state.
__global__ __launch_bounds__(256) void k_project_q27(const double* __restrict__ f27, int64_t N, double* __restrict__ f19,
                                                     float* __restrict__ mom)
{
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    RawMoments<double> m = {};
#pragma unroll
    for (int i = 0; i < 27; ++i) {
        const double v = f27[(int64_t)i * N + n];
        const int a = cx27(i), b = cy27(i), c = cz27(i);
        const int a2 = a * a, b2 = b * b, c2 = c * c;
        m.m000 += v;
        m.m100 += a * v;
        m.m010 += b * v;
        m.m001 += c * v;
        m.m200 += a2 * v;
        m.m020 += b2 * v;
        m.m002 += c2 * v;
        m.m110 += a * b * v;
        m.m101 += a * c * v;
        m.m011 += b * c * v;
        m.m210 += a2 * b * v;
        m.m120 += a * b2 * v;
        m.m201 += a2 * c * v;
        m.m102 += a * c2 * v;
        m.m021 += b2 * c * v;
        m.m012 += b * c2 * v;
        m.m220 += a2 * b2 * v;
        m.m202 += a2 * c2 * v;
        m.m022 += b2 * c2 * v;
    }
    if (f19) {
        double s[19];
        pops_from_raw(m, s);
#pragma unroll
        for (int i = 0; i < 19; ++i) f19[(int64_t)i * N + n] = s[i];
    }
    if (mom) {
        const double v[10] = {m.m000, m.m100, m.m010, m.m001, m.m200, m.m020, m.m002, m.m110, m.m101, m.m011};
#pragma unroll
        for (int k = 0; k < 10; ++k) mom[(int64_t)k * N + n] = (float)v[k];
    }
}

// Per-block FP64 sums of squares of the 11 raw network inputs of the current
// state (to fit the input scales); partials[block][11].
template <class S, Pattern P, bool WALLS>
__global__ __launch_bounds__(256) void k_feature_sumsq(const S* __restrict__ buf, Geom g, Phys ph, double* __restrict__ partials)
{
    __shared__ double red[4][MLP_NIN];
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y * blockDim.y + threadIdx.y;
    const int z = blockIdx.z;
    double v[MLP_NIN] = {};
    if (x < g.nx && y < g.ny) {
        NodeIdx d;
        node_idx(g, x, y, z, d);
        float s[19];
        gather<LatD3Q19, S, P, WALLS>(buf, g.stride, d, s);
        float Fx, Fy, Fz;
        node_force(ph, g, nb(d, 0, 0, 0), y, Fx, Fy, Fz);
        CMState<float> st;
        pre_collide<float, true>(s, (float)ph.rho0, Fx, Fy, Fz, st);
        float xin[MLP_NIN];
        mlp_features(st, xin);
#pragma unroll
        for (int k = 0; k < MLP_NIN; ++k) v[k] = (double)xin[k] * (double)xin[k];
    }
    const int tid = threadIdx.x + blockDim.x * threadIdx.y;
#pragma unroll
    for (int k = 0; k < MLP_NIN; ++k) {
        double a = v[k];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
        if ((tid & 63) == 0) red[tid >> 6][k] = a;
    }
    __syncthreads();
    if (tid < MLP_NIN) {
        double t = 0.0;
        for (int i = 0; i < (int)((blockDim.x * blockDim.y + 63) / 64); ++i) t += red[i][tid];
        partials[(int64_t)(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z)) * MLP_NIN + tid] = t;
    }
}

// out[k] = sum over blocks of partials[block][k], k < 11 (FP64, fixed order)
__global__ void k_sum_features(const double* __restrict__ partials, int nblocks, double* __restrict__ out)
{
    const int k = threadIdx.x;
    if (k >= MLP_NIN) return;
    double t = 0.0;
    for (int b = 0; b < nblocks; ++b) t += partials[(int64_t)b * MLP_NIN + k];
    out[k] = t;
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
void launch_feature_sumsq(int precision, int pattern, bool walls, const void* buf, const Geom& g, const Phys& ph,
                          double* partials, double* out, int nblocks, dim3 grid, dim3 block, hipStream_t st)
{
#define LBM_FEAT(S_)                                                                                              \
    switch (pattern) {                                                                                            \
    case AB:                                                                                                      \
        if (walls) hipLaunchKernelGGL((k_feature_sumsq<S_, AB, true>), grid, block, 0, st, (const S_*)buf, g, ph, partials); \
        else hipLaunchKernelGGL((k_feature_sumsq<S_, AB, false>), grid, block, 0, st, (const S_*)buf, g, ph, partials); \
        break;                                                                                                    \
    case AA_EVEN:                                                                                                 \
        if (walls) hipLaunchKernelGGL((k_feature_sumsq<S_, AA_EVEN, true>), grid, block, 0, st, (const S_*)buf, g, ph, partials); \
        else hipLaunchKernelGGL((k_feature_sumsq<S_, AA_EVEN, false>), grid, block, 0, st, (const S_*)buf, g, ph, partials); \
        break;                                                                                                    \
    default:                                                                                                      \
        if (walls) hipLaunchKernelGGL((k_feature_sumsq<S_, AA_ODD, true>), grid, block, 0, st, (const S_*)buf, g, ph, partials); \
        else hipLaunchKernelGGL((k_feature_sumsq<S_, AA_ODD, false>), grid, block, 0, st, (const S_*)buf, g, ph, partials); \
    }
    switch (precision) {
    case PREC_FP32: LBM_FEAT(float); break;
    case PREC_FP16: LBM_FEAT(_Float16); break;
    default: LBM_FEAT(bf16_t); break;
    }
#undef LBM_FEAT
    hipLaunchKernelGGL(k_sum_features, dim3(1), dim3(64), 0, st, partials, nblocks, out);
}

template <class S>
static void step_mlp_s(int pattern, bool walls, bool nt, const void* src, void* dst, const Geom& g, const Phys& ph,
                       const void* net, uint32_t* fb, dim3 grid, dim3 block, hipStream_t st)
{
    const S* a = (const S*)src;
    S* b = (S*)dst;
    const MlpPacked* w = (const MlpPacked*)net;
    // row staging: a periodic A-B lattice whose work-groups span whole rows,
    // FP32 storage (at 256^3 staged 0.683 -> 0.702 of 8 TB/s; FP16 storage
    // read directly 0.474, staged 0.462)
    const bool rows = sizeof(S) >= 4 && g.row_stage && (int)block.x == g.nx && grid.x == 1 && block.x * block.y <= 256;
#define LBM_MLP_STEP(P, W, NT_)                                                                       \
    do {                                                                                              \
        if constexpr (P == AB && !W && sizeof(S) >= 4) {                                              \
            if (rows && g.off32) hipLaunchKernelGGL((k_step_mlp_ab<S, W, NT_, true, true>), grid, block, 0, st, a, b, g, ph, w, fb); \
            else if (rows) hipLaunchKernelGGL((k_step_mlp_ab<S, W, NT_, false, true>), grid, block, 0, st, a, b, g, ph, w, fb); \
            else if (g.off32) hipLaunchKernelGGL((k_step_mlp_ab<S, W, NT_, true>), grid, block, 0, st, a, b, g, ph, w, fb); \
            else hipLaunchKernelGGL((k_step_mlp_ab<S, W, NT_, false>), grid, block, 0, st, a, b, g, ph, w, fb); \
        }                                                                                             \
        else if constexpr (P == AB) {                                                                 \
            if (g.off32) hipLaunchKernelGGL((k_step_mlp_ab<S, W, NT_, true>), grid, block, 0, st, a, b, g, ph, w, fb); \
            else hipLaunchKernelGGL((k_step_mlp_ab<S, W, NT_, false>), grid, block, 0, st, a, b, g, ph, w, fb); \
        }                                                                                             \
        else hipLaunchKernelGGL((k_step_mlp<S, P, W, NT_>), grid, block, 0, st, a, b, g, ph, w, fb);    \
    } while (0)
#define LBM_MLP_NT(P, W) \
    if (nt) LBM_MLP_STEP(P, W, true); else LBM_MLP_STEP(P, W, false)
#define LBM_MLP_W(P) \
    if (walls) { LBM_MLP_NT(P, true); } else { LBM_MLP_NT(P, false); }
    switch (pattern) {
    case AB: LBM_MLP_W(AB); break;
    case AA_EVEN: LBM_MLP_W(AA_EVEN); break;
    default: LBM_MLP_W(AA_ODD); break;
    }
#undef LBM_MLP_W
#undef LBM_MLP_NT
#undef LBM_MLP_STEP
}

void launch_step_mlp(int precision, int pattern, bool walls, bool nt, const void* src, void* dst, const Geom& g,
                     const Phys& ph, const void* net, uint32_t* fb_partials, dim3 grid, dim3 block, hipStream_t st)
{
    switch (precision) {
    case PREC_FP32: step_mlp_s<float>(pattern, walls, nt, src, dst, g, ph, net, fb_partials, grid, block, st); break;
    case PREC_FP16: step_mlp_s<_Float16>(pattern, walls, nt, src, dst, g, ph, net, fb_partials, grid, block, st); break;
    default: step_mlp_s<bf16_t>(pattern, walls, nt, src, dst, g, ph, net, fb_partials, grid, block, st); break;
    }
}

int train_loss_parts(const Geom& g) { return (g.N + 255) / 256; }
// gradient partials (wavefronts of k_train_backward), loss partials (64-node blocks of k_train_dstate)
int train_rows(const Geom& g) { return (g.nx + 63) / 64 * g.ny * g.nz; }
int train_groups(const Geom& g) { return (g.N + 63) / 64; }

void launch_train_loss(const float* post, const Geom& g, float rho0, const float* target, const float* inv_sigma,
                       float* gbuf, double* loss_partials, const double* energy, float ew, hipStream_t st)
{
    hipLaunchKernelGGL(k_train_loss, dim3(train_loss_parts(g)), dim3(256), 0, st, post, g, rho0, target, inv_sigma, gbuf,
                       loss_partials, energy, ew);
}

void launch_train_energy(const float* posts, int64_t step_stride, int steps, const Geom& g, float rho0, const float* targets,
                         double* partials, hipStream_t st)
{
    hipLaunchKernelGGL(k_train_energy, dim3(train_loss_parts(g), steps), dim3(256), 0, st, posts, step_stride, g, rho0,
                       targets, partials);
}

void launch_train_backward(const float* state, const float* gbuf, const Geom& g, const Phys& ph, const void* net,
                           float* grad_partials, float* rates, float* xbar, float* gout, bool accumulate, const float* target,
                           const float* inv_sigma, double* loss_partials, const double* energy, float ew, hipStream_t st)
{
    const dim3 grid((g.nx + 63) / 64, g.ny, g.nz);
    if (!gout) {
        hipLaunchKernelGGL(k_train_backward<false>, grid, dim3(64), 0, st, state, gbuf, g, ph, (const MlpPacked*)net,
                           grad_partials, nullptr, nullptr, (int)accumulate);
        return;
    }
    hipLaunchKernelGGL(k_train_backward<true>, grid, dim3(64), 0, st, state, gbuf, g, ph, (const MlpPacked*)net,
                       grad_partials, rates, xbar, (int)accumulate);
    hipLaunchKernelGGL(k_train_dstate, dim3(train_groups(g), (19 + TRAIN_K - 1) / TRAIN_K), dim3(64), 0, st, state, gbuf, g, ph, rates, xbar, gout,
                       TrainLoss{target, inv_sigma, energy, ew, loss_partials});
}

size_t reduce_grad_tmp_bytes() { return sizeof(double) * MLP_RED_SLICES * MLP_NPARAM; }

void launch_reduce_grad(const float* partials, int nparts, double* grad, double* tmp, hipStream_t st)
{
    hipLaunchKernelGGL(k_reduce_grad_slices, dim3((MLP_NPARAM + 63) / 64, MLP_RED_SLICES), dim3(256), 0, st, partials,
                       nparts, tmp);
    hipLaunchKernelGGL(k_reduce_grad, dim3((MLP_NPARAM + 255) / 256), dim3(256), 0, st, tmp, grad);
}

void launch_sum_partials(const double* partials, int rows, int64_t row, int n, int n_last, double* out, hipStream_t st)
{
    hipLaunchKernelGGL(k_sum_partials, dim3(rows), dim3(256), 0, st, partials, row, n, n_last, out);
}

void launch_adam(float* theta, float* m1, float* m2, const double* grad, float lr, float b1, float b2, float eps,
                 float c1, float c2, hipStream_t st)
{
    hipLaunchKernelGGL(k_adam, dim3((MLP_NPARAM + 255) / 256), dim3(256), 0, st, theta, m1, m2, grad, lr, b1, b2, eps, c1,
                       c2);
}

void launch_mlp_pack(const float* theta, const float* inv_scale, void* packed, hipStream_t st)
{
    hipLaunchKernelGGL(k_mlp_pack, dim3(1), dim3(256), 0, st, theta, inv_scale, (MlpPacked*)packed);
}

void launch_project_q27(const double* f27, int64_t N, double* f19, float* mom, hipStream_t st)
{
    hipLaunchKernelGGL(k_project_q27, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, st, f27, N, f19, mom);
}

size_t mlp_packed_bytes() { return sizeof(MlpPacked); }

} // namespace lbm

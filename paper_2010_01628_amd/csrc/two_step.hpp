// Two A-B steps in one pass over memory, for the single lattice and the
// ensemble.
//
// A work-group owns a tile of x-y columns and sweeps a run of z planes.  At
// plane p it pulls f(t), collides (first step) and puts the result in LDS;
// plane p - 1 then has every neighbour's first-step result, is pulled from
// LDS, collides again (second step) and is stored.  The state between the two
// steps never reaches memory.  Tiles carry one halo column on each side whose
// first step is computed again by the neighbouring tile (none along an axis
// that the tile spans whole: its neighbours wrap inside the tile); a run of
// planes repeats the plane before and after it.
//
// Same arithmetic as two single steps, in the same order at every node, with
// the state between them rounded to the storage type: bitwise the same
// populations.
//
// What bounds it: a single step moves 2 Q values per node and runs at the rate
// of a copy of its own traffic; a pair moves Q in (the halo columns again: HBM
// reads 1.11 times the lattice with 64x13 tiles) and Q out.  256^3 FP32, 64x13
// tiles in three runs of planes: 834 us for two single steps, 620 for a pair;
// its loads and stores alone take 540, its collisions alone 360.
//
// LDS: a first-step population is needed one plane after the one it was
// computed on where c_z = 0, two planes where c_z = +1, and at once where
// c_z = -1, so they take 2, 3 and 1 slots; those that do not move in x or y
// stay in their thread's registers.  One column takes 4 + 8 x 2 + 4 x 3 = 32
// values on D3Q19, 48 on D3Q27.
#pragma once

#include "lattice_kernels.hpp"

namespace lbm {

// Constant tables of one lattice's exchange through LDS.
template <class L> struct Pair {
    static constexpr bool own(int i) { return L::cx(i) == 0 && L::cy(i) == 0; }
    // populations before i with the same c_z that move in x or y
    static constexpr int rank(int i)
    {
        int k = 0;
        for (int j = 0; j < i; ++j) k += L::cz(j) == L::cz(i) && !own(j);
        return k;
    }
    static constexpr int count(int cz)
    {
        int k = 0;
        for (int j = 0; j < L::Q; ++j) k += L::cz(j) == cz && !own(j);
        return k;
    }
    static constexpr int QM = count(-1), QZ = count(0), QP = count(1);
    static constexpr int SLOTS = QM + 2 * QZ + 3 * QP;
    // population that only moves by cz along z
    static constexpr int axis(int cz)
    {
        for (int j = 0; j < L::Q; ++j)
            if (own(j) && L::cz(j) == cz) return j;
        return -1;
    }
};

// Threads per work-group, one work-group per compute unit: as many columns as
// its LDS holds.  Wide tiles pay: a tile's halo columns are single elements of
// lines of their own.  256^3 FP32, a pair: 1024 threads on 64x13 tiles 620 us,
// on 32x28 750, two work-groups of 512 on 32x13 657, on 64x5 680; tiles of 30
// columns, whose rows share 128-byte lines with the neighbour's, 1400.
template <class L, class S> constexpr int pair_threads()
{
    constexpr int col = Pair<L>::SLOTS * (int)sizeof(S);
    if constexpr (col <= 128) return 1024;
    else if constexpr (col <= 192) return 768;
    else if constexpr (col <= 256) return 512;
    else return 384;
}
// wavefronts per SIMD that this makes (the registers are kept within it)
template <class L, class S> constexpr int pair_waves() { return pair_threads<L, S>() / 256; }

// One work-group's share.
struct PairTile {
    int nx, ny, nz;     // lattice
    int64_t stride;     // elements between population arrays
    int x0, y0, z0;     // first node stored
    int w, h, len;      // nodes stored along x, y and z
    int hx, hy;         // halo columns on each side (1, or 0 where the tile spans the axis)
    int W;              // columns per tile row (the same for every tile of a launch: w + 2 hx of the widest)
    int nt;             // streaming hint on the stores
};

// Element at a wavefront-uniform base and a 32-bit per-lane byte offset.
template <class S> __device__ inline const S* lane_at(const S* base, uint32_t off)
{
    typedef __attribute__((address_space(1))) const char gchar;
    gchar* gb = (gchar*)base;
    asm("" : "+s"(gb));
    return reinterpret_cast<const S*>((const char*)(gb + off));
}
template <class S> __device__ inline S* lane_at(S* base, uint32_t off)
{
    return const_cast<S*>(lane_at(static_cast<const S*>(base), off));
}

// Store of one element at byte offset `off` from a wavefront-uniform base;
// nothing is written where off lies beyond `range` bytes.
template <class S, bool STREAM> __device__ inline void st_range(S* base, uint32_t range, uint32_t off, S v)
{
    constexpr int NT = STREAM ? 2 : 0; // the non-temporal bit of the instruction
    auto rsrc = __builtin_amdgcn_make_buffer_rsrc(base, 0, range, 0x00027000);
    if constexpr (sizeof(S) == 8) {
        typedef int v2i __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2i, v), rsrc, (int)off, 0, NT);
    } else if constexpr (sizeof(S) == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), rsrc, (int)off, 0, NT);
    } else {
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(short, v), rsrc, (int)off, 0, NT);
    }
}

// the bits of a stored value, for an asm operand
__device__ inline double& reg(double& v) { return v; }
__device__ inline float& reg(float& v) { return v; }
__device__ inline _Float16& reg(_Float16& v) { return v; }
__device__ inline uint16_t& reg(bf16_t& v) { return v.bits; }
__device__ inline uint16_t& reg(bf16sr_t& v) { return v.bits; }

template <class L, class S, bool WALLS, bool GENERAL, bool FIELD, int T>
__device__ inline void pair_sweep(const S* __restrict__ src, S* __restrict__ dst, const PairTile& t, const Phys& ph,
                                  uint32_t key2, int64_t N, S* lds)
{
    using R = typename Codec<S>::R;
    using E = Pair<L>;
    constexpr int Q = L::Q;
    const int tid = threadIdx.x;
    const int W = t.W, nxy = t.nx * t.ny;
    // The stored columns come first, w to a row, so that wavefronts store
    // whole rows of the tile; then the halo rows below and above, then the
    // halo columns left and right.
    int cx = 0, cy = 0;
    bool column = true;
    const bool stored = tid < t.w * t.h;
    if (stored) {
        cy = tid / t.w;
        cx = tid - cy * t.w + t.hx;
        cy += t.hy;
    } else {
        const int We = t.w + 2 * t.hx; // columns of this tile's rows
        int r = tid - t.w * t.h;
        if (r < 2 * t.hy * We) {
            const int up = r >= We;
            cx = r - up * We;
            cy = up * (t.h + 1);
        } else {
            r -= 2 * t.hy * We;
            column = r < 2 * t.hx * t.h;
            const int right = r >= t.h;
            cy = column ? r - right * t.h + t.hy : 0;
            cx = column ? right * (t.w + 1) : 0;
        }
    }
    const int col = column ? cy * W + cx : T - 1; // place in LDS
    // this thread's column; lanes without one take the tile's first
    int gx = column ? t.x0 - t.hx + cx : t.x0, gy = column ? t.y0 - t.hy + cy : t.y0;
    gx = gx < 0 ? gx + t.nx : (gx >= t.nx ? gx - t.nx : gx);
    // (beyond a wall the halo row is never read by a stored node)
    gy = gy < 0 ? gy + t.ny : (gy >= t.ny ? gy - t.ny : gy);
    const bool ylo = WALLS && gy == 0, yhi = WALLS && gy == t.ny - 1;
    auto blocked = [&](int dy) { return WALLS && ((dy < 0 && ylo) || (dy > 0 && yhi)); };
    // wavefronts with a row at a wall: only these take the bounce-back's
    // second load over the first (200x101x75 FP32, a pair: with an address
    // selected per lane in every wavefront 89 us, so 70, without walls 63)
    const bool at_wall = WALLS && __builtin_amdgcn_ballot_w64(ylo || yhi) != 0;
    // byte offsets of the column and its neighbours within a plane
    uint32_t off[3][3]; // [1 + dx][1 + dy]
    {
        const int ox[3] = {gx == 0 ? t.nx - 1 : gx - 1, gx, gx == t.nx - 1 ? 0 : gx + 1};
        const int oy[3] = {(gy == 0 ? t.ny - 1 : gy - 1) * t.nx, gy * t.nx, (gy == t.ny - 1 ? 0 : gy + 1) * t.nx};
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) off[a][b] = (uint32_t)(ox[a] + oy[b]) * (uint32_t)sizeof(S);
    }
    const uint32_t self = off[1][1];
    // LDS columns of the neighbours (wrapping where the tile spans the axis);
    // only stored lanes need theirs, the others read their own
    int lcol[3][3];
    {
        const int spanx = t.w - 1, spany = (t.h - 1) * W;
        const int lx[3] = {t.hx == 0 && cx == 0 ? spanx : -1, 0, t.hx == 0 && cx == spanx ? -spanx : 1};
        const int ly[3] = {t.hy == 0 && cy == 0 ? spany : -W, 0, t.hy == 0 && cy == t.h - 1 ? -spany : W};
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) lcol[a][b] = stored ? col + lx[a] + ly[b] : col;
    }
    S* const ldsM = lds;
    S* const ldsZ = lds + E::QM * T;
    S* const ldsP = ldsZ + 2 * E::QZ * T;

    // the force at this plane and, for the second step, at the plane before
    R Fx = R(0), Fy = R(0), Fz = R(0);
    if (ph.force_mode == FORCE_UNIFORM) {
        Fx = (R)ph.force[0];
        Fy = (R)ph.force[1];
        Fz = (R)ph.force[2];
    } else if (ph.force_mode == FORCE_ROW_TABLE) {
        Fx = (R)ph.row_table[gy];
    }
    R Fx1 = Fx, Fy1 = Fy, Fz1 = Fz;

    S in[Q];
    ForceRaw fin{0.0, 0.0, 0.0};
    // f(t) at plane p.  The array distance and the offsets pass through an asm
    // each time, so that the bases are formed by scalar instructions beside
    // the loads (kept for the whole sweep, they do not fit the scalar
    // registers) and the offsets stay 32 bits wide
    auto load = [&](int p) {
        int64_t stride = t.stride;
        asm volatile("" : "+s"(stride));
#pragma unroll
        for (int a = 0; a < 9; ++a) asm volatile("" : "+v"(off[a / 3][a % 3]));
        const S* pl[3];
        pl[0] = src + (int64_t)(p == 0 ? t.nz - 1 : p - 1) * nxy;
        pl[1] = src + (int64_t)p * nxy;
        pl[2] = src + (int64_t)(p == t.nz - 1 ? 0 : p + 1) * nxy;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const S* base = pl[1 - L::cz(i)] + i * stride;
            in[i] = *lane_at(base, off[1 - L::cx(i)][1 - L::cy(i)]);
        }
        if (at_wall) {
#pragma unroll
            for (int i = 0; i < Q; ++i)
                if (L::cy(i) != 0 && blocked(-L::cy(i))) in[i] = *lane_at(pl[1] + L::opp(i) * stride, off[1][1]);
        }
        if constexpr (FIELD) {
            const double* f = ph.force_field + (int64_t)p * nxy;
            const uint32_t o = self / (uint32_t)sizeof(S) * 8u;
            fin.x = *lane_at(f, o);
            fin.y = *lane_at(f + N, o);
            fin.z = *lane_at(f + 2 * N, o);
        }
    };

    constexpr int A0 = E::axis(0), AP = E::axis(1), AM = E::axis(-1);
    S rest = S(), up1 = S(), up2 = S(); // rest at p - 1; c_z = +1 at p - 1 and p - 2
    S low[Q];                           // WALLS: c_z = -1, c_y != 0 populations at p - 1
    int zpar = 0, p3 = 0;               // slots of plane p
    const int sweep = t.len + 2;        // planes
    int pz = t.z0 == 0 ? t.nz - 1 : t.z0 - 1, pp = 0, ps = 0;
    auto arrived = [&]() { // waits for the loads
#pragma unroll
        for (int i = 0; i < Q; ++i) asm volatile("" : "+v"(reg(in[i])));
        if constexpr (FIELD) asm volatile("" : "+v"(fin.x), "+v"(fin.y), "+v"(fin.z));
    };
    // second-step populations v of plane z
    R v[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) v[i] = R(0);
    // Lanes that store nothing pass an offset beyond the buffer's range, which
    // the hardware drops, instead of taking a branch: with every plane's 19
    // stores unconditional, the wait for the next plane's loads counts past
    // them and does not wait for the stores.
    auto store = [&](int z, bool on) {
        int64_t stride = t.stride;
        uint32_t o = stored && on ? self : 0x80000000u;
        asm volatile("" : "+s"(stride), "+v"(o));
        S* const base = dst + (int64_t)z * nxy;
        const uint32_t range = (uint32_t)nxy * (uint32_t)sizeof(S);
        if (t.nt) {
#pragma unroll
            for (int i = 0; i < Q; ++i) st_range<S, true>(base + i * stride, range, o, Codec<S>::enc(v[i]));
        } else {
#pragma unroll
            for (int i = 0; i < Q; ++i) st_range<S, false>(base + i * stride, range, o, Codec<S>::enc(v[i]));
        }
    };
    load(pz);
    arrived();
    for (int k = 0; k < sweep; ++k) {
        R s[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) s[i] = Codec<S>::dec(in[i]);
        if constexpr (FIELD) {
            Fx = (R)fin.x;
            Fy = (R)fin.y;
            Fz = (R)fin.z;
        }
        const int pn = pz == t.nz - 1 ? 0 : pz + 1;
        load(pn); // in flight during both collisions (one plane too many at the end)
        // the plane before's stores, behind the loads that the next plane waits for
        store(ps, k >= 3);
        NodeMacro<R> mac;
        L::template collide<R, GENERAL, Codec<S>::increment>(s, (R)ph.rho0, Fx, Fy, Fz, ph, mac);
        if constexpr (Codec<S>::stochastic) dither_bf16(s, ph.sr_key, (uint32_t)(pz * nxy) + self / (uint32_t)sizeof(S));
        S q[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) q[i] = Codec<S>::enc(s[i]);
        {
            S* const wz = ldsZ + zpar * (E::QZ * T) + col;
            S* const wp = ldsP + p3 * (E::QP * T) + col;
#pragma unroll
            for (int i = 0; i < Q; ++i)
                if (!E::own(i)) {
                    if (L::cz(i) < 0) ldsM[E::rank(i) * T + col] = q[i];
                    else if (L::cz(i) == 0) wz[E::rank(i) * T] = q[i];
                    else wp[E::rank(i) * T] = q[i];
                }
        }
        __syncthreads();
        {
            const int p3m1 = p3 == 0 ? 2 : p3 - 1, p3m2 = p3 == 2 ? 0 : p3 + 1;
            const S* const rz = ldsZ + (1 - zpar) * (E::QZ * T);
            const S* const rp = ldsP + p3m2 * (E::QP * T);
            const S* const rpb = ldsP + p3m1 * (E::QP * T); // plane p - 1 (bounce-back)
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                const int c = lcol[1 - L::cx(i)][1 - L::cy(i)];
                S a;
                if (E::own(i)) a = L::cz(i) < 0 ? q[AM] : (L::cz(i) == 0 ? rest : up2);
                else if (L::cz(i) < 0) a = ldsM[E::rank(i) * T + c];
                else if (L::cz(i) == 0) a = rz[E::rank(i) * T + c];
                else a = rp[E::rank(i) * T + c];
                v[i] = Codec<S>::dec(a);
            }
            if (at_wall) {
#pragma unroll
                for (int i = 0; i < Q; ++i)
                    if (L::cy(i) != 0 && blocked(-L::cy(i))) {
                        const int o = L::opp(i);
                        S a;
                        if (L::cz(o) < 0) a = low[o];
                        else if (L::cz(o) == 0) a = rz[E::rank(o) * T + col];
                        else a = rpb[E::rank(o) * T + col];
                        v[i] = Codec<S>::dec(a);
                    }
            }
        }
        __syncthreads(); // every value of this plane's exchange has been taken
        if (k >= 2) {
            L::template collide<R, GENERAL, Codec<S>::increment>(v, (R)ph.rho0, Fx1, Fy1, Fz1, ph, mac);
            if constexpr (Codec<S>::stochastic) dither_bf16(v, key2, (uint32_t)(pp * nxy) + self / (uint32_t)sizeof(S));
        }
        arrived();
        rest = q[A0];
        up2 = up1;
        up1 = q[AP];
        if constexpr (WALLS) {
#pragma unroll
            for (int i = 0; i < Q; ++i)
                if (L::cz(i) < 0 && L::cy(i) != 0) low[i] = q[i];
        }
        if constexpr (FIELD) {
            Fx1 = Fx;
            Fy1 = Fy;
            Fz1 = Fz;
        }
        zpar ^= 1;
        p3 = p3 == 2 ? 0 : p3 + 1;
        ps = pp;
        pp = pz;
        pz = pn;
    }
    store(ps, true);
}

template <class L, class S, bool WALLS, bool GENERAL, bool FIELD>
__global__ __launch_bounds__((pair_threads<L, S>())) __attribute__((amdgpu_waves_per_eu((pair_waves<L, S>())))) void k_step_pair(const S* __restrict__ src, S* __restrict__ dst,
                                                                      Geom g, Phys ph, PairShape sh, uint32_t key2)
{
    constexpr int T = pair_threads<L, S>();
    __shared__ S lds[Pair<L>::SLOTS * T];
    // work-groups go to the eight XCDs in turn: each XCD takes one contiguous
    // run of the tiles (x fastest, then y, then z), whose halos its L2 shares
    const int run = gridDim.x / 8;
    int k = (blockIdx.x % 8) * run + blockIdx.x / 8;
    if (k >= sh.tx * sh.ty * sh.tz) return;
    PairTile t;
    t.nx = g.nx;
    t.ny = g.ny;
    t.nz = g.nz;
    t.stride = g.stride;
    const int ix = k % sh.tx;
    k /= sh.tx;
    const int iy = k % sh.ty, iz = k / sh.ty;
    t.x0 = ix * sh.w;
    t.y0 = iy * sh.h;
    t.z0 = iz * sh.len;
    t.w = min(sh.w, g.nx - t.x0);
    t.h = min(sh.h, g.ny - t.y0);
    t.len = min(sh.len, g.nz - t.z0);
    t.hx = sh.w < g.nx;
    t.hy = sh.h < g.ny;
    t.W = sh.w + 2 * t.hx;
    t.nt = sh.nt;
    pair_sweep<L, S, WALLS, GENERAL, FIELD, T>(src, dst, t, ph, key2, g.N, lds);
}

// ---------------------------------------------------------------------------
// The same for lattices too small to fill the GPU with sweeps: a work-group
// takes a w x h x d block of nodes with one halo node on each side (none along
// an axis that the block spans), one thread per node, both steps at once, the
// whole state between them in LDS.  The halo repeats most of the first step
// (32x2x2 blocks: 512 first steps for 128 stored nodes), but a launch takes
// one trip to memory and two collisions where two single steps take two
// launches and two trips.
// ---------------------------------------------------------------------------
template <class L, class S> constexpr int pair_block_threads() { return sizeof(S) == 8 ? 512 : 1024; }

template <class L, class S, bool WALLS, bool GENERAL>
__global__ __launch_bounds__((pair_block_threads<L, S>())) void k_step_pair_block(const S* __restrict__ src,
                                                                                 S* __restrict__ dst, Geom g, Phys ph,
                                                                                 PairShape sh, uint32_t key2)
{
    using R = typename Codec<S>::R;
    constexpr int Q = L::Q, T = pair_block_threads<L, S>();
    __shared__ S lds[(Q - 1) * T]; // population i > 0 of the node in place p: lds[(i - 1) T + p]
    int k = blockIdx.x;
    const int bx = k % sh.tx;
    k /= sh.tx;
    const int x0 = bx * sh.w, y0 = k % sh.ty * sh.h, z0 = k / sh.ty * sh.len;
    const int w = min(sh.w, g.nx - x0), h = min(sh.h, g.ny - y0), d = min(sh.len, g.nz - z0);
    const int hx = sh.w < g.nx, hy = sh.h < g.ny, hz = sh.len < g.nz;
    const int W = w + 2 * hx, H = h + 2 * hy, D = d + 2 * hz;
    // stored nodes first, then the halo: z faces, y faces, x faces
    int r = threadIdx.x, cx, cy, cz;
    const bool stored = r < w * h * d;
    bool node = true;
    if (stored) {
        cz = r / (w * h);
        r -= cz * w * h;
        cy = r / w;
        cx = r - cy * w + hx;
        cy += hy;
        cz += hz;
    } else if ((r -= w * h * d) < 2 * hz * W * H) {
        const int up = r >= W * H;
        r -= up * W * H;
        cz = up * (D - 1);
        cy = r / W;
        cx = r - cy * W;
    } else if ((r -= 2 * hz * W * H) < 2 * hy * W * d) {
        const int up = r >= W * d;
        r -= up * W * d;
        cy = up * (H - 1);
        cz = r / W;
        cx = r - cz * W;
        cz += hz;
    } else {
        r -= 2 * hy * W * d;
        node = r < 2 * hx * h * d;
        const int up = node && r >= h * d;
        r = node ? r - up * h * d : 0;
        cx = up * (W - 1);
        cz = r / h;
        cy = r - cz * h + hy;
        cz += hz;
    }
    const int place = node ? (cz * H + cy) * W + cx : T - 1;
    // its lattice node (wrapped; beyond a wall a halo node is never read)
    auto wrap = [](int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); };
    const int x = wrap(x0 - hx + cx, g.nx), y = wrap(y0 - hy + cy, g.ny), z = wrap(z0 - hz + cz, g.nz);
    NodeIdx n;
    node_idx(g, x, y, z, n);
    R s[Q], F[3];
    gather<L, S, AB, WALLS>(src, g.stride, n, s);
    node_force(ph, g, nb(n, 0, 0, 0), y, F[0], F[1], F[2]);
    NodeMacro<R> mac;
    L::template collide<R, GENERAL, Codec<S>::increment>(s, (R)ph.rho0, F[0], F[1], F[2], ph, mac);
    if constexpr (Codec<S>::stochastic) dither_bf16(s, ph.sr_key, (uint32_t)nb(n, 0, 0, 0));
    const S rest = Codec<S>::enc(s[0]);
#pragma unroll
    for (int i = 1; i < Q; ++i) lds[(i - 1) * T + place] = Codec<S>::enc(s[i]);
    __syncthreads();
    if (!stored) return;
    // places of the neighbours, wrapping where the block spans the axis
    const int px[3] = {hx == 0 && cx == 0 ? w - 1 : -1, 0, hx == 0 && cx == w - 1 ? 1 - w : 1};
    const int py[3] = {(hy == 0 && cy == 0 ? h - 1 : -1) * W, 0, (hy == 0 && cy == h - 1 ? 1 - h : 1) * W};
    const int pz[3] = {(hz == 0 && cz == 0 ? d - 1 : -1) * H * W, 0, (hz == 0 && cz == d - 1 ? 1 - d : 1) * H * W};
    s[0] = Codec<S>::dec(rest);
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        int at = (i - 1) * T + place + px[1 - L::cx(i)] + py[1 - L::cy(i)] + pz[1 - L::cz(i)];
        if (beyond<WALLS>(n, -L::cy(i))) at = (L::opp(i) - 1) * T + place;
        s[i] = Codec<S>::dec(lds[at]);
    }
    L::template collide<R, GENERAL, Codec<S>::increment>(s, (R)ph.rho0, F[0], F[1], F[2], ph, mac);
    if constexpr (Codec<S>::stochastic) dither_bf16(s, key2, (uint32_t)nb(n, 0, 0, 0));
    scatter<L, S, AB, WALLS, false>(dst, g.stride, n, s);
}

// Shape of a pair launch on this lattice.
template <class L, class S> struct LaunchPair {
    static void step(bool walls, bool general, const void* src, void* dst, const Geom& g, const Phys& ph,
                     const PairShape& sh, uint32_t key2, hipStream_t st)
    {
        if (walls) by_rates<true>(general, src, dst, g, ph, sh, key2, st);
        else by_rates<false>(general, src, dst, g, ph, sh, key2, st);
    }
    template <bool WALLS>
    static void by_rates(bool general, const void* src, void* dst, const Geom& g, const Phys& ph, const PairShape& sh,
                         uint32_t key2, hipStream_t st)
    {
        if constexpr (L::Q == 19) { // D3Q27 has fixed rates
            if (general) return by_force<WALLS, true>(src, dst, g, ph, sh, key2, st);
        }
        by_force<WALLS, false>(src, dst, g, ph, sh, key2, st);
    }
    template <bool WALLS, bool GENERAL>
    static void by_force(const void* src, void* dst, const Geom& g, const Phys& ph, const PairShape& sh, uint32_t key2,
                         hipStream_t st)
    {
        if (sh.block) {
            const int hx = sh.w < g.nx, hy = sh.h < g.ny, hz = sh.len < g.nz;
            const int nodes = (sh.w + 2 * hx) * (sh.h + 2 * hy) * (sh.len + 2 * hz);
            hipLaunchKernelGGL((k_step_pair_block<L, S, WALLS, GENERAL>), dim3(sh.tx * sh.ty * sh.tz),
                               dim3((nodes + 63) / 64 * 64), 0, st, (const S*)src, (S*)dst, g, ph, sh, key2);
            return;
        }
        const dim3 grid((unsigned)((sh.tx * sh.ty * sh.tz + 7) / 8 * 8)), block(pair_threads<L, S>());
        const S* a = (const S*)src;
        S* b = (S*)dst;
        if (ph.force_mode == FORCE_FIELD)
            hipLaunchKernelGGL((k_step_pair<L, S, WALLS, GENERAL, true>), grid, block, 0, st, a, b, g, ph, sh, key2);
        else
            hipLaunchKernelGGL((k_step_pair<L, S, WALLS, GENERAL, false>), grid, block, 0, st, a, b, g, ph, sh, key2);
    }
};

} // namespace lbm

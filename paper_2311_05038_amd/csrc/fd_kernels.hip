// Step kernels and set-up kernels for gfx950 (MI355X).
//
// 2D (z, x):  a block of 4 waves loads a tile of 128 columns x 8, 16 or 32 rows
//   with its halo at once, exchanges it through LDS and updates it (the
//   largest 16-bit grids: one wave per block streams a 128-column strip down z
//   with the 9 rows z-4..z+4 in registers).  One read of cur/prev/c and one
//   write per cell and step (16 B/cell in FP32, 10 B with 16-bit fields).
//   Several FP32 steps per launch: fd_multi2d.hip.
// 3D (z, y, x): NW waves per block.  A block owns a tile of the x-y plane
//   (256x8 cells for FP32 fields, 128x8 for 16-bit) and a chunk of `zc`
//   planes; lanes stream along z (the slow axis) with a 9-deep register queue
//   per cell, and x/y neighbours come from a double-buffered LDS copy of the
//   current plane with a 4-cell halo.  Most grids whose fields stay in the
//   Infinity Cache, and most adjoint steps, take 2 or 4 planes per block
//   instead, all loads in flight at once (k_step3d_short; fd_plan.hpp says
//   where).
// Both follow the fused step of arXiv 2311.05038, Section 7 (Listing 3's
// add_source, fd_pzz, fd_pxx, fd_time and swap in one pass).
#include <algorithm>

#include <type_traits>

#include "fd_device.hpp"
#include "fd_launch.hpp"
#include "fd_plan.hpp"

// The 16-bit steps order their memory operations so that the next plane's
// loads overlap the compute: the z sponge factor travels with the
// prefetched data, the prefetch is unconditional (planes past the chunk are
// in bounds or read as zero), and each new plane is stored one plane late,
// right before the next prefetch.  Vector loads and stores share one
// completion counter, and the compiler waits for a load by waiting until
// every older memory operation has completed once both kinds are
// outstanding: a load issued after the prefetch and used at once, a
// skipped prefetch (the previous registers are then copied, which waits),
// or a store issued right after the compute would each make a plane wait
// for its own prefetch.  Measured at 768x768x512: BF16 649 -> 566 us.  The
// FP32 steps keep the plain order (stores right after the compute, the
// sponge factor loaded after the barrier), which measured faster for them
// (512^3 366 against 387 us): their loop is bandwidth-bound with more bytes
// in flight per wave already.
namespace fdk {

// --------------------------------------------------------------------------
// Epilogue shared by 2D and 3D: receivers, source, padding, store.
// --------------------------------------------------------------------------
// A row's outgoing values.  The 16-bit steps store them one plane (row)
// later, right before the next prefetch (see the ordering note above); the
// FP32 steps store them at once.
template <typename T, int VX>
struct Outgoing {
    Pack<T, VX> o;
    Pack<float, VX> L;  // history value (L cur or cur), history modes only
    T *dst;
    float *ldst;
    bool ok;
};

template <typename T, int VX, int MODE, bool STREAM>
__device__ __forceinline__ void flush(Outgoing<T, VX> &out)
{
    if (out.ok) {
        if constexpr (STREAM)
            stp_stream<T, VX>(out.dst, out.o);
        else
            stp<T, VX>(out.dst, out.o);
        if constexpr (stores_history(MODE)) stp<float, VX>(out.ldst, out.L);
    }
    out.ok = false;
}

// nw holds the new values (FP32 fields) or the new values in storage units
// (16-bit fields: value = h.sn * nw).  FULL: every cell of the lane lies
// inside the grid (x < nx), so no padding mask is needed.  The adjoint
// step (which reads lap and g here) stores at once; the forward steps leave
// their stores in `out`.  lp: the history value to store (history modes), or
// in the adjoint step the centre value of cur (the previous step's new
// value, for a deferred gradient term); pv: the centre value of prev (the
// new value of two steps back, for a second deferred term).
template <int ST, int VX, int MODE, bool STREAM, bool FULL>
__device__ __forceinline__ void finish_cells(const StepArgs &a, const HalfCtx &h, int z, int y,
                                             int x0, bool store_ok, size_t row, uint32_t eo,
                                             float (&nw)[VX],
                                             const float (&lp)[VX], const float (&pv)[VX],
                                             const float (&cc)[VX],
                                             const float (&G)[VX], float inj, float &bmax,
                                             Outgoing<typename Stor<ST>::T, VX> &out)
{
    using T = typename Stor<ST>::T;
    // Receiver box membership of this row (z, y).
    int rrow = -1;
    {
        const int zr = z - a.rec.z0, yr = y - a.rec.y0;
        if (zr >= 0 && yr >= 0 && zr % a.rec.dz == 0 && yr % a.rec.dy == 0 &&
            zr / a.rec.dz < a.rec.nz && yr / a.rec.dy < a.rec.ny)
            rrow = (zr / a.rec.dz) * a.rec.ny + yr / a.rec.dy;
    }
    if constexpr (MODE == kAdj) {
        if (a.resid_row != nullptr && rrow >= 0) {
#pragma unroll
            for (int v = 0; v < VX; ++v) {
                const int xr = x0 + v - a.rec.x0;
                if (x0 + v < a.nx && xr >= 0 && xr % a.rec.dx == 0 && xr / a.rec.dx < a.rec.nx)
                    nw[v] = fmaf(cc[v] * G[v], a.resid_row[(size_t)rrow * a.rec.nx + xr / a.rec.dx], nw[v]);
            }
        }
    } else {
        if (a.trace_row != nullptr && rrow >= 0) {
#pragma unroll
            for (int v = 0; v < VX; ++v) {
                const int xr = x0 + v - a.rec.x0;
                if (x0 + v < a.nx && xr >= 0 && xr % a.rec.dx == 0 && xr / a.rec.dx < a.rec.nx) {
                    if constexpr (ST == kF32)
                        a.trace_row[(size_t)rrow * a.rec.nx + xr / a.rec.dx] = nw[v];
                    else
                        a.trace_row[(size_t)rrow * a.rec.nx + xr / a.rec.dx] = nw[v] * h.sn;
                }
            }
        }
        if (z == a.sz && y == a.sy) {
            const float inj_s = ST == kF32 ? inj : inj * h.sn_inv;
#pragma unroll
            for (int v = 0; v < VX; ++v)
                if (x0 + v == a.sx) nw[v] += inj_s;
        }
    }
#pragma unroll
    for (int v = 0; v < VX; ++v) {
        if (!FULL && x0 + v >= a.nx) nw[v] = 0.0f;
        if constexpr (ST != kF32) bmax = fmaxf(bmax, fabsf(nw[v]));
    }
    T *dst = (T *)(a.out != nullptr ? a.out : a.prev);
    if constexpr (ST == kF32) {
#pragma unroll
        for (int v = 0; v < VX; ++v) out.o.v[v] = nw[v];
    } else {
        encode_pairs<ST, VX>(nw, out.o.v);
    }
    out.dst = at(dst + row, eo);
    out.ok = store_ok;
    if constexpr (stores_history(MODE)) {
#pragma unroll
        for (int v = 0; v < VX; ++v) out.L.v[v] = (FULL || x0 + v < a.nx) ? lp[v] : 0.0f;
        out.ldst = at(a.lap + row, eo);
    }
    if constexpr (MODE == kAdj) {
        flush<T, VX, MODE, STREAM>(out);
        // the time sum in FP64, one term per level in descending level order
        // however many terms share a pass over g
        if (store_ok && a.gmode != 1) {
            const Pack<float, VX> lw = ldp<float, VX>(at(a.lap + row, eo));
            Pack<double, VX> gg = ldp<double, VX>(at(a.g + row, eo));
            if (a.gmode == 3) {
                const Pack<float, VX> lw3 = ldp<float, VX>(at(a.lap3 + row, eo));
#pragma unroll
                for (int v = 0; v < VX; ++v) gg.v[v] = fma((double)pv[v], (double)lw3.v[v], gg.v[v]);
            }
            if (a.gmode >= 2) {
                const Pack<float, VX> lw2 = ldp<float, VX>(at(a.lap2 + row, eo));
#pragma unroll
                for (int v = 0; v < VX; ++v) gg.v[v] = fma((double)lp[v], (double)lw2.v[v], gg.v[v]);
            }
#pragma unroll
            for (int v = 0; v < VX; ++v) gg.v[v] = fma((double)nw[v], (double)lw.v[v], gg.v[v]);
            stp<double, VX>(at(a.g + row, eo), gg);
        }
    }
}


// The same update on 16-bit fields read as raw codes q (P = 2^ec q, Pold =
// 2^ep qp, and L q computed from the raw q), producing the new field in its
// storage units 2^-en: (G sc)(2 q + c L q) - (G^2 sp) qp with sc = 2^(ec-en)
// and sp = 2^(ep-en).  This is the scaled arithmetic exactly, since
// multiplying by 2^k does not round.
template <int ST>
__device__ __forceinline__ float update(float G, float ctr, float c, float lap, float prev,
                                        const HalfCtx &h)
{
    if constexpr (ST == kF32)
        return leapfrog(G, ctr, c, lap, prev);
    else
        return fmaf(G * h.sc, fmaf(c, lap, 2.0f * ctr), -((G * G) * h.sp) * prev);
}

// --------------------------------------------------------------------------
// 2D
// --------------------------------------------------------------------------
// The streaming 2D step (16-bit fields on the largest grids, forward): one
// wave takes 128 columns and `zc` rows.  CQ: c is read as 16-bit fixed-point
// codes.
constexpr int k2dVX = 2;
template <int ST, bool CQ>
__device__ __forceinline__ void step2d_tile(const StepArgs &a, int tx, int tz,
                                            float (*row)[64 * k2dVX + 8], const HalfCtx &h,
                                            float inj, float &bmax)
{
    static_assert(ST != kF32, "16-bit fields");
    using T = typename Stor<ST>::T;
    using CT = std::conditional_t<CQ, uint16_t, float>;
    constexpr int VX = k2dVX, TX = 64 * VX;
    const int lane = threadIdx.x & 63;
    const int xb = tx * TX;
    const int x0 = xb + lane * VX;
    const int zb = tz * a.zc;
    const int ze = min(zb + a.zc, a.nz);
    const T *__restrict__ cur = (const T *)a.cur;
    const T *__restrict__ prv = (const T *)a.prev;
    const size_t px = (size_t)a.px;
    const bool lane_in = x0 < a.px;
    const int nx = a.nx, nz = a.nz;

    float gxv[VX];
#pragma unroll
    for (int v = 0; v < VX; ++v) gxv[v] = (x0 + v < nx) ? a.gx[x0 + v] : 0.0f;

    int hx = -1, hslot = 0;
    if (lane < 4) {
        hx = xb - 4 + lane;
        hslot = lane;
    } else if (lane >= 60) {
        hx = xb + TX + (lane - 60);
        hslot = TX + 4 + (lane - 60);
    }
    const bool hlane = (lane < 4) || (lane >= 60);
    const bool hvalid = hx >= 0 && hx < nx;

    // Loads return raw packs (zero outside the grid); values are decoded
    // where they are consumed, so a prefetch never waits for its own load.
    using PT = Pack<T, VX>;
    using PC = Pack<CT, VX>;
    const CT *cbase;
    if constexpr (CQ)
        cbase = a.c16;
    else
        cbase = a.c;
    auto ld_cur = [&](int z) -> PT {
        PT p{};
        if (z >= 0 && z < nz && lane_in) p = ldp<T, VX>(cur + (size_t)z * px + x0);
        return p;
    };
    auto ld_prev = [&](int z) -> PT {
        PT p{};
        if (z < nz && lane_in) p = ldp<T, VX>(prv + (size_t)z * px + x0);
        return p;
    };
    auto ld_c = [&](int z) -> PC {
        PC p{};
        if (z < nz && lane_in) p = ldp<CT, VX>(cbase + (size_t)z * px + x0);
        return p;
    };
    auto ld_halo = [&](int z) -> T { return (hvalid && z < nz) ? cur[(size_t)z * px + hx] : (T)0; };

    float q[9][VX];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const PT p = ld_cur(zb - 4 + k);
#pragma unroll
        for (int v = 0; v < VX; ++v) q[k][v] = decode_raw<ST>(p.v[v]);
    }
    PT la = ld_cur(zb + 4), pv = ld_prev(zb);
    PC cv = ld_c(zb);
    T hv = ld_halo(zb);
    // the row's sponge factor travels with the prefetch: a load issued after
    // it and waited for in the same row would also wait for the prefetch
    float gn = a.gz[zb];
    Outgoing<T, VX> out;
    out.ok = false;

    for (int z = zb; z < ze; ++z) {
        float pc[VX], cc[VX];
#pragma unroll
        for (int v = 0; v < VX; ++v) {
            q[8][v] = decode_raw<ST>(la.v[v]);
            pc[v] = decode_raw<ST>(pv.v[v]);
            if constexpr (CQ)
                cc[v] = (float)cv.v[v] * a.c16_scale;   // exact: a power-of-two scale
            else
                cc[v] = cv.v[v];
        }
        const float hc = decode_raw<ST>(hv);
        const float gzp = gn;
        // the previous row's stores go out after the wait for this row's
        // data and just before the next prefetch
        __builtin_amdgcn_sched_barrier(0);
        flush<T, VX, kFwd, false>(out);
        la = ld_cur(z + 5);
        pv = ld_prev(z + 1);
        cv = ld_c(z + 1);
        hv = ld_halo(z + 1);
        gn = z + 1 < nz ? a.gz[z + 1] : 0.0f;
        float *rw = row[z & 1];
#pragma unroll
        for (int v = 0; v < VX; ++v) rw[4 + lane * VX + v] = q[4][v];
        if (hlane) rw[hslot] = hc;
        __syncthreads();
        float nw[VX], G[VX];
#pragma unroll
        for (int v = 0; v < VX; ++v) {
            const int li = 4 + lane * VX + v;
            const float lx = stencil_taps(rw[li - 4], rw[li - 3], rw[li - 2], rw[li - 1],
                                          rw[li + 1], rw[li + 2], rw[li + 3], rw[li + 4]);
            const float lz = stencil_taps(q[0][v], q[1][v], q[2][v], q[3][v], q[5][v], q[6][v],
                                          q[7][v], q[8][v]);
            const float lap = fmaf(2.0f * kA0, q[4][v], lz + lx);
            G[v] = gzp * gxv[v];
            nw[v] = update<ST>(G[v], q[4][v], cc[v], lap, pc[v], h);
        }
        // (the forward step stores no history value: q[4] stands in for it)
        finish_cells<ST, VX, kFwd, false, false>(a, h, z, 0, x0, lane_in, (size_t)z * px, (uint32_t)x0, nw,
                                                 q[4], pc, cc, G, inj, bmax, out);
#pragma unroll
        for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int v = 0; v < VX; ++v) q[k][v] = q[k + 1][v];
    }
    flush<T, VX, kFwd, false>(out);
}

template <int ST, bool CQ>
__global__ __launch_bounds__(64) void k_step2d(StepArgs a)
{
    __shared__ float row[2][64 * k2dVX + 8];
    const int nb = a.tiles_x * a.tiles_z;
    const int t = xcd_tile(blockIdx.x, nb);
    const int tx = t % a.tiles_x, tz = t / a.tiles_x;
    float inj = 0.0f;
    if (a.n + 1 < a.nt) inj = a.amp * a.wavelet[a.n + 1];
    const HalfCtx h = half_prologue<ST>(a, inj, blockIdx.x == 0);
    float bmax = 0.0f;
    step2d_tile<ST, CQ>(a, tx, tz, row, h, inj, bmax);
    block_max_to<64>(max_slot(a.meta, (int)((a.n + 1) & 3)), bmax * h.sn, nullptr);
}

// One 2D step with every load of a block's tile in flight at once.  A block
// owns 128 columns x 8 RZ rows (a thread 4 columns x RZ rows); P with its halo
// of 4 cells goes to LDS, one barrier, and the update follows.  (A wave that
// streams down a strip row by row, as in the kernel above, waits about 0.5 us
// of memory latency per row on grids too small for many waves.  Per step:
// FP32 256^2 4.5 -> 3.4 us, 1024^2 7.8 -> 5.4, 1201 x 1747 10.5 -> 8.6, 2048 x
// 4096 23.9 -> 22.7; BF16 256^2 7.6 -> 5.2, 1024^2 12.5 -> 7.3, 1201 x 1747
// 12.8 -> 9.4.)
template <int ST, int RZ, int MODE, bool CQ>
__device__ __forceinline__ void step2d_block(const StepArgs &a, int tx, int tz, float *pl, bool block0, int32_t *red)
{
    static_assert(ST == kF32 || MODE == kFwd, "16-bit fields: forward steps");
    using T = typename Stor<ST>::T;
    using CT = std::conditional_t<CQ, uint16_t, float>;
    using PT = Pack<T, 4>;
    constexpr int TX = 128, TZ = 8 * RZ, LW = TX + 8;
    const int lx = threadIdx.x & 31, lg = threadIdx.x >> 5;
    const int xb = tx * TX, zb = tz * TZ, x0 = xb + 4 * lx, z0 = zb + RZ * lg;
    const int nx = a.nx, nz = a.nz, pxi = a.px;
    const size_t px = (size_t)pxi;
    const T *__restrict__ cur = (const T *)a.cur;
    const T *__restrict__ prv = (const T *)a.prev;
    const CT *cb;
    if constexpr (CQ)
        cb = a.c16;
    else
        cb = a.c;
    const bool xin = x0 < pxi;
    PT own[RZ], pv[RZ], zh{}, xh{};
    Pack<CT, 4> cv[RZ];
#pragma unroll
    for (int r = 0; r < RZ; ++r) {
        own[r] = PT{};
        if (xin && z0 + r < nz) own[r] = ldp<T, 4>(cur + (size_t)(z0 + r) * px + x0);
    }
    // halo rows: one 4-cell unit a thread; halo columns: one for 2 TZ threads
    const int hrow = lg < 4 ? lg - 4 : TZ + lg - 4, hz = zb + hrow;
    if (xin && hz >= 0 && hz < nz) zh = ldp<T, 4>(cur + (size_t)hz * px + x0);
    const int crow = threadIdx.x >> 1, cx = threadIdx.x & 1 ? xb + TX : xb - 4;
    const bool cl = threadIdx.x < 2 * TZ;
    if (cl && zb + crow < nz && cx >= 0 && cx < pxi) xh = ldp<T, 4>(cur + (size_t)(zb + crow) * px + cx);
#pragma unroll
    for (int r = 0; r < RZ; ++r) {
        pv[r] = PT{};
        cv[r] = Pack<CT, 4>{};
        if (xin && z0 + r < nz) {
            pv[r] = ldp<T, 4>(prv + (size_t)(z0 + r) * px + x0);
            cv[r] = ldp<CT, 4>(cb + (size_t)(z0 + r) * px + x0);
        }
    }
    float gx[4], gz[RZ];
#pragma unroll
    for (int v = 0; v < 4; ++v) gx[v] = x0 + v < nx ? a.gx[x0 + v] : 0.0f;
#pragma unroll
    for (int r = 0; r < RZ; ++r) gz[r] = z0 + r < nz ? a.gz[z0 + r] : 0.0f;
    float inj = 0.0f;
    if constexpr (MODE != kAdj)
        if (a.n + 1 < a.nt) inj = a.amp * a.wavelet[a.n + 1];
    const HalfCtx h = half_prologue<ST>(a, inj, block0);

    auto put = [&](int at_l, const PT &p) {
        Pack<float, 4> o;
#pragma unroll
        for (int v = 0; v < 4; ++v) o.v[v] = decode_raw<ST>(p.v[v]);
        stp<float, 4>(pl + at_l, o);
    };
    const int li = (RZ * lg + 4) * LW + 4 + 4 * lx;
#pragma unroll
    for (int r = 0; r < RZ; ++r) put(li + r * LW, own[r]);
    put((hrow + 4) * LW + 4 + 4 * lx, zh);
    if (cl) put((crow + 4) * LW + (threadIdx.x & 1 ? 4 + TX : 0), xh);
    __syncthreads();

    float col[RZ + 8][4];
#pragma unroll
    for (int k = 0; k < RZ + 8; ++k) {
        const Pack<float, 4> p = ldp<float, 4>(pl + li + (k - 4) * LW);
#pragma unroll
        for (int v = 0; v < 4; ++v) col[k][v] = p.v[v];
    }
    float lzz[RZ][4];
    if constexpr (ST == kF32) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float in[RZ + 8], out[RZ];
#pragma unroll
            for (int k = 0; k < RZ + 8; ++k) in[k] = col[k][v];
            axis_d2_run<RZ>(in, out);
#pragma unroll
            for (int r = 0; r < RZ; ++r) lzz[r][v] = out[r];
        }
    }
    float bmax = 0.0f;
#pragma unroll
    for (int r = 0; r < RZ; ++r) {
        const Pack<float, 4> pl4 = ldp<float, 4>(pl + li + r * LW - 4), pr4 = ldp<float, 4>(pl + li + r * LW + 4);
        float row[12], nw[4], lp[4], G[4], pc[4], cc[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            row[v] = pl4.v[v];
            row[4 + v] = col[4 + r][v];
            row[8 + v] = pr4.v[v];
            pc[v] = decode_raw<ST>(pv[r].v[v]);
            if constexpr (CQ)
                cc[v] = (float)cv[r].v[v] * a.c16_scale;   // exact: a power-of-two scale
            else
                cc[v] = cv[r].v[v];
            G[v] = gz[r] * gx[v];
        }
        float lxx[4];
        if constexpr (ST == kF32) axis_d2_run<4>(row, lxx);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float u = col[4 + r][v];
            float lap;
            if constexpr (ST == kF32) {
                lap = lzz[r][v] + lxx[v];
            } else {
                const float lx8 = stencil_taps(row[v], row[v + 1], row[v + 2], row[v + 3], row[v + 5], row[v + 6],
                                               row[v + 7], row[v + 8]);
                const float lz8 = stencil_taps(col[r][v], col[r + 1][v], col[r + 2][v], col[r + 3][v], col[r + 5][v],
                                               col[r + 6][v], col[r + 7][v], col[r + 8][v]);
                lap = fmaf(2.0f * kA0, u, lz8 + lx8);
            }
            nw[v] = update<ST>(G[v], u, cc[v], lap, pc[v], h);
            lp[v] = MODE == kAdj ? u : lap;
        }
        Outgoing<T, 4> out;
        finish_cells<ST, 4, MODE, false, false>(a, h, z0 + r, 0, x0, xin && z0 + r < nz, (size_t)(z0 + r) * px,
                                                (uint32_t)x0, nw, lp, pc, cc, G, inj, bmax, out);
        flush<T, 4, MODE, false>(out);
    }
    if constexpr (ST != kF32)
        block_max_to<256>(max_slot(a.meta, (int)((a.n + 1) & 3)), bmax * h.sn, (float *)red);
}

template <int ST, int RZ, int MODE, bool CQ>
__global__ __launch_bounds__(256) void k_step2d_block(StepArgs a)
{
    __shared__ __attribute__((aligned(16))) float pl[(8 * RZ + 8) * 136];
    __shared__ int32_t red[4];
    const int t = xcd_tile(blockIdx.x, a.tiles_x * a.tiles_z);
    step2d_block<ST, RZ, MODE, CQ>(a, t % a.tiles_x, t / a.tiles_x, pl, blockIdx.x == 0, red);
}

// Batched 2D FP32 step: block b belongs to the item whose tile range holds
// b; every item keeps its own grid, fields and step index.
template <int MODE>
__global__ __launch_bounds__(256) void k_step2d_batch(Batch2D b)
{
    __shared__ __attribute__((aligned(16))) float pl[(8 + 8) * 136];
    const int t = blockIdx.x;
    int i = 0;
    while (i + 1 < b.count && t >= b.begin[i + 1]) ++i;
    const StepArgs &a = b.it[i];
    const int lt = t - b.begin[i];
    step2d_block<kF32, 1, MODE, false>(a, lt % a.tiles_x, lt / a.tiles_x, pl, false, nullptr);
}

// --------------------------------------------------------------------------
// 3D
// --------------------------------------------------------------------------
// A wave covers RPW rows of the tile at once (64/RPW lanes per row, VX
// cells per lane), so a lane's VX cells are contiguous in x; the block's NW
// waves stack NW*RPW rows, and each thread handles RY such row groups.
// CQ: c is read as 16-bit fixed-point codes q (16-bit fields, forward step):
// 2 P + c L P = s (2 P / s + q L P) with s = 2^(e-16), and s joins the
// other power-of-two factors of the update (exact; the Laplacian keeps the
// scale of the stored codes).
template <int ST, int VX, int RY, int NW, int RPW, int MODE, bool CQ>
__global__ __launch_bounds__(64 * NW) void k_step3d(StepArgs a)
{
    static_assert(!CQ || (ST != kF32 && MODE == kFwd), "16-bit c: 16-bit fields, forward step");
    using T = typename Stor<ST>::T;
    using CT = std::conditional_t<CQ, uint16_t, float>;
    static_assert(NW == 2 || NW == 4 || NW == 8, "waves per block");
    static_assert(RPW == 1 || RPW == 2, "rows per wave");
    static_assert(8 % (NW * RPW) == 0, "y-halo rows per wave");
    constexpr int LPR = 64 / RPW;   // lanes per row
    constexpr int TX = LPR * VX, TY = NW * RPW * RY, LW = TX + 8, LH = TY + 8, HH = 8 / (NW * RPW);
    __shared__ float pl[2][LH * LW];
    __shared__ float red[NW];
    const int lane = threadIdx.x & 63, wy = threadIdx.x >> 6;
    const int col = lane % LPR, trow = wy * RPW + lane / LPR;   // thread's column and row
    const int nb = a.tiles_x * a.tiles_y * a.tiles_z;
    const int t = xcd_tile3d(blockIdx.x, nb, a.resident);
    const int tx = t % a.tiles_x;
    const int t2 = t / a.tiles_x;
    const int ty = t2 % a.tiles_y, tz = t2 / a.tiles_y;
    const int xb = tx * TX, yb = ty * TY, x0 = xb + col * VX;
    const int zb = tz * a.zc, ze = min(zb + a.zc, a.nz);
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const size_t px = (size_t)a.px, pp = (size_t)ny * px;
    const int zlo = ST == kF32 ? -a.zghost : 0, zhi = ST == kF32 ? nz + a.zghost : nz;
    const bool lane_in = x0 < a.px;
    const T *__restrict__ cur = (const T *)a.cur;
    const T *__restrict__ prv = (const T *)a.prev;

    float inj = 0.0f;
    if constexpr (MODE != kAdj)
        if (a.n + 1 < a.nt) inj = a.amp * a.wavelet[a.n + 1];
    const HalfCtx h = half_prologue<ST>(a, inj, blockIdx.x == 0);

    // FULL: every lane's cells, every row and every y-halo row of the tile
    // lie inside the grid, so loads need no per-lane or per-row tests (the z
    // tests are uniform); other tiles take the checked path.
    auto tile = [&](auto full_c) -> float {
        constexpr bool FULL = decltype(full_c)::value;
        int yj[RY];
        bool yin[RY];
        float gyv[RY];
    #pragma unroll
        for (int j = 0; j < RY; ++j) {
            yj[j] = yb + trow + NW * RPW * j;
            yin[j] = FULL || yj[j] < ny;
            gyv[j] = yin[j] ? a.gy[yj[j]] : 0.0f;
        }
        float gxv[VX], gxv2[VX];
    #pragma unroll
        for (int v = 0; v < VX; ++v) {
            gxv[v] = (FULL || x0 + v < nx) ? a.gx[x0 + v] : 0.0f;
            gxv2[v] = gxv[v] * gxv[v];
        }

        // y-halo rows handled by this thread: k = (wy + NW hh) RPW + its row
        // within the wave, hh < 8 / (NW RPW).
        int hy[HH], hyslot[HH];
        bool hyv[HH];
    #pragma unroll
        for (int hh = 0; hh < HH; ++hh) {
            const int k = (wy + NW * hh) * RPW + lane / LPR;
            const int ly = k < 4 ? k - 4 : TY + k - 4;
            hy[hh] = yb + ly;
            hyv[hh] = FULL || (hy[hh] >= 0 && hy[hh] < ny && lane_in);
            hyslot[hh] = (ly + 4) * LW + 4 + col * VX;
        }
        // x-halo cell handled by this thread (threads < 8 TY).
        const bool hxl = threadIdx.x < 8 * TY;
        int hxx = 0, hxy = 0, hxslot = 0;
        if (hxl) {
            const int lr = threadIdx.x >> 3, ci = threadIdx.x & 7;
            hxx = ci < 4 ? xb - 4 + ci : xb + TX + ci - 4;
            hxy = yb + lr;
            hxslot = (lr + 4) * LW + (ci < 4 ? ci : TX + ci);
        }
        const bool hxv = hxl && hxx >= 0 && hxx < nx && hxy < ny;

        // Element offsets within a plane (32-bit: a plane holds < 2^29
        // cells): each access is a wave-uniform plane pointer plus a lane
        // offset, which keeps the address arithmetic scalar.  (FP32 fields,
        // bandwidth-bound, measured faster with plain 64-bit addresses.)
        constexpr bool OFF32 = ST != kF32;
        constexpr bool LATE = ST != kF32;   // the 16-bit memory-op order (see top)
        auto addr = [&](auto *base, int z, uint32_t e, int y, int x) {
            if constexpr (OFF32)
                return at(base + (size_t)z * pp, e);
            else
                return base + (size_t)z * pp + (size_t)y * px + x;
        };
        uint32_t eo[RY], eohy[HH];
    #pragma unroll
        for (int j = 0; j < RY; ++j) eo[j] = (uint32_t)(yj[j] * a.px + x0);
    #pragma unroll
        for (int hh = 0; hh < HH; ++hh) eohy[hh] = (FULL || hyv[hh]) ? (uint32_t)(hy[hh] * a.px + x0) : 0u;
        const uint32_t eohx = hxv ? (uint32_t)(hxy * a.px + hxx) : 0u;

        // Loads return raw packs (zero outside the grid); values are decoded
        // where they are consumed, so a prefetch never waits for its own load.
        using PT = Pack<T, VX>;
        using PC = Pack<CT, VX>;
        const CT *cbase;
        if constexpr (CQ)
            cbase = a.c16;
        else
            cbase = a.c;
        // cur (the only field read off its own planes) is readable over
        // [-zghost, nz + zghost): a z-slab's ghost planes, or zero edges
        auto ld3 = [&](const T *base, int z, int j) -> PT {
            PT p{};
            if (z >= zlo && z < zhi && (FULL || (yin[j] && lane_in)))
                p = ldp<T, VX>(addr(base, z, eo[j], yj[j], x0));
            return p;
        };
        auto ld3nt = [&](const T *base, int z, int j) -> PT {
            PT p{};
            if (z < nz && (FULL || (yin[j] && lane_in)))
                p = ldp_stream<T, VX>(addr(base, z, eo[j], yj[j], x0));
            return p;
        };
        auto ldc3 = [&](int z, int j) -> PC {
            PC p{};
            if (z < nz && (FULL || (yin[j] && lane_in)))
                p = ldp_stream<CT, VX>(addr(cbase, z, eo[j], yj[j], x0));
            return p;
        };
        auto ldhy = [&](int z, int hh) -> PT {
            PT p{};
            if ((FULL || hyv[hh]) && z < nz) p = ldp<T, VX>(addr(cur, z, eohy[hh], hy[hh], x0));
            return p;
        };
        auto ldhx = [&](int z) -> T {
            return (hxv && z < nz) ? *addr(cur, z, eohx, hxy, hxx) : (T)0;
        };

        float q[RY][9][VX];
    #pragma unroll
        for (int j = 0; j < RY; ++j)
    #pragma unroll
            for (int k = 0; k < 8; ++k) {
                const PT p = ld3(cur, zb - 4 + k, j);
    #pragma unroll
                for (int v = 0; v < VX; ++v) q[j][k][v] = decode_raw<ST>(p.v[v]);
            }
        // Prefetched raw data of one plane zz: cur at zz + 4 (the queue's
        // next entry), prev and c at zz, and the halo cells of cur at zz.
        struct Ahead {
            PT la[RY], pv[RY], yh[HH];
            PC cv[RY];
            T xh;
            float gz;   // sponge factor of plane zz (16-bit steps)
        };
        auto fetch = [&](int zz, Ahead &r) {
    #pragma unroll
            for (int j = 0; j < RY; ++j) {
                r.la[j] = ld3(cur, zz + 4, j);
                r.pv[j] = ld3nt(prv, zz, j);
                r.cv[j] = ldc3(zz, j);
            }
    #pragma unroll
            for (int hh = 0; hh < HH; ++hh) r.yh[hh] = ldhy(zz, hh);
            r.xh = ldhx(zz);
            if constexpr (LATE) r.gz = zz < nz ? a.gz[zz] : 0.0f;
        };
        Ahead ah;
        fetch(zb, ah);
        float bmax = 0.0f;
        Outgoing<T, VX> out[RY];
    #pragma unroll
        for (int j = 0; j < RY; ++j) out[j].ok = false;

        // One plane: slot k of the register queue holds plane z - 4 + k; the
        // values shift down one slot per plane.
        auto plane_step = [&](int z) {
            float pc[RY][VX], cc[RY][VX], yhc[HH][VX];
    #pragma unroll
            for (int j = 0; j < RY; ++j)
    #pragma unroll
                for (int v = 0; v < VX; ++v) {
                    q[j][8][v] = decode_raw<ST>(ah.la[j].v[v]);
                    pc[j][v] = decode_raw<ST>(ah.pv[j].v[v]);
                    cc[j][v] = (float)ah.cv[j].v[v];
                }
    #pragma unroll
            for (int hh = 0; hh < HH; ++hh)
    #pragma unroll
                for (int v = 0; v < VX; ++v) yhc[hh][v] = decode_raw<ST>(ah.yh[hh].v[v]);
            const float xhc = decode_raw<ST>(ah.xh);
            const float gzp = ah.gz;
            // 16-bit: the previous plane's stores go out after the wait for
            // this plane's data and just before the next prefetch
            if constexpr (LATE) {
                __builtin_amdgcn_sched_barrier(0);
    #pragma unroll
                for (int j = 0; j < RY; ++j) flush<T, VX, MODE, true>(out[j]);
            }
            if (LATE || z + 1 < ze) fetch(z + 1, ah);
            float *P = pl[z & 1];
    #pragma unroll
            for (int j = 0; j < RY; ++j)
    #pragma unroll
                for (int v = 0; v < VX; ++v) P[(trow + NW * RPW * j + 4) * LW + 4 + col * VX + v] = q[j][4][v];
    #pragma unroll
            for (int hh = 0; hh < HH; ++hh)
    #pragma unroll
                for (int v = 0; v < VX; ++v) P[hyslot[hh] + v] = yhc[hh][v];
            if (hxl) P[hxslot] = xhc;
            __syncthreads();
            const float gzz = LATE ? gzp : a.gz[z];
    #pragma unroll
            for (int j = 0; j < RY; ++j) {
                float nw[VX], lp[VX], G[VX];
                if constexpr (ST != kF32) {
                    // 16-bit fields (VALU-bound): taps summed over the three
                    // axes before weighting, and the sponge factor's square
                    // taken per lane and per row, which saves instructions at
                    // a different FP32 rounding order.
                    const float gr = gzz * gyv[j];
                    const float sc = CQ ? h.sc * a.c16_scale : h.sc;
                    const float two = CQ ? 2.0f * a.c16_inv : 2.0f;
                    const float r1 = gr * sc, r2 = (gr * gr) * h.sp;
    #pragma unroll
                    for (int v = 0; v < VX; ++v) {
                        const int li = (trow + NW * RPW * j + 4) * LW + 4 + col * VX + v;
                        const float(&qq)[9][VX] = q[j];
                        float sk[4];
    #pragma unroll
                        for (int k = 1; k <= 4; ++k)
                            sk[k - 1] = ((P[li - k] + P[li + k]) + (P[li - k * LW] + P[li + k * LW])) +
                                        (qq[4 - k][v] + qq[4 + k][v]);
                        const float ctr = qq[4][v];
                        const float lap = fmaf(3.0f * kA0, ctr,
                                               fmaf(kA4, sk[3], fmaf(kA3, sk[2], fmaf(kA2, sk[1], kA1 * sk[0]))));
                        G[v] = 0.0f;
                        nw[v] = fmaf(gxv[v] * r1, fmaf(cc[j][v], lap, two * ctr), -(gxv2[v] * r2) * pc[j][v]);
                        lp[v] = lap;
                    }
                } else {
    #pragma unroll
                for (int v = 0; v < VX; ++v) {
                    const int li = (trow + NW * RPW * j + 4) * LW + 4 + col * VX + v;
                    const float u = q[j][4][v];
                    const float lx = axis_d2(P[li - 4], P[li - 3], P[li - 2], P[li - 1], u, P[li + 1],
                                             P[li + 2], P[li + 3], P[li + 4]);
                    const float lyv = axis_d2(P[li - 4 * LW], P[li - 3 * LW], P[li - 2 * LW], P[li - LW], u,
                                              P[li + LW], P[li + 2 * LW], P[li + 3 * LW], P[li + 4 * LW]);
                    const float lz = axis_d2(q[j][0][v], q[j][1][v], q[j][2][v], q[j][3][v], u,
                                             q[j][5][v], q[j][6][v], q[j][7][v], q[j][8][v]);
                    const float lap = lz + (lyv + lx);
                    G[v] = (gzz * gyv[j]) * gxv[v];
                    nw[v] = update<ST>(G[v], q[j][4][v], cc[j][v], lap, pc[j][v], h);
                    lp[v] = MODE == kAdj ? q[j][4][v] : lap;
                }
                }
                if constexpr (OFF32)
                    finish_cells<ST, VX, MODE, true, FULL>(a, h, z, yj[j], x0, lane_in && yin[j],
                                                           (size_t)z * pp, eo[j], nw, lp, pc[j], cc[j], G, inj,
                                                           bmax, out[j]);
                else
                    finish_cells<ST, VX, MODE, true, FULL>(a, h, z, yj[j], x0, lane_in && yin[j],
                                                           (size_t)z * pp + (size_t)yj[j] * px, (uint32_t)x0, nw,
                                                           lp, pc[j], cc[j], G, inj, bmax, out[j]);
                if constexpr (!LATE) flush<T, VX, MODE, true>(out[j]);
            }
        };
        using std::integral_constant;
        for (int z = zb; z < ze; ++z) {
            plane_step(z);
    #pragma unroll
            for (int j = 0; j < RY; ++j)
    #pragma unroll
                for (int k = 0; k < 8; ++k)
    #pragma unroll
                    for (int v = 0; v < VX; ++v) q[j][k][v] = q[j][k + 1][v];
        }
    #pragma unroll
        for (int j = 0; j < RY; ++j) flush<T, VX, MODE, true>(out[j]);
        return bmax;
    };
    // (measured: a small gain with 16-bit fields, a small loss with FP32)
    const bool full = ST != kF32 && xb + TX <= nx && yb >= 4 && yb + TY + 4 <= ny;
    const float bmax = full ? tile(std::true_type{}) : tile(std::false_type{});
    if constexpr (ST != kF32)
        block_max_to<64 * NW>(max_slot(a.meta, (int)((a.n + 1) & 3)), bmax * h.sn, red);
}

// --------------------------------------------------------------------------
// 3D, grids too small to fill the device with long chunks
// --------------------------------------------------------------------------
// The streaming kernel above keeps one plane of loads in flight per wave: on a
// grid whose chunks are a few planes long it spends a memory latency on every
// plane and eight on priming its queue (96 x 120 x 152: 12.5 us for 28 MB).
// Here a block owns 64 x 16 cells of ZC planes and issues every load of them
// at once: 8 + ZC planes of P, ZC of Pold and c and the x and y halos, 16
// bytes a lane; the ZC planes then go to LDS, one barrier, and the update
// follows.  P is read (8 + ZC) / ZC + 1/2 + 1/8 times, so blocks are dealt x
// first, then z: the z neighbours that read the same planes run at the same
// time on one XCD and find them in its L2 (y before z: 201 x 333 x 289 72
// against 58 us).  Per step, streaming / this: 64^3 8.2 / 5.0 us, 96 x 120 x
// 152 12.5 / 11.2, 78 x 259 x 333 30.0 / 26.5, 201 x 333 x 289 66 / 58;
// adjoint 96 x 120 x 152 14.6 / 12.7, 201 x 333 x 289 108 / 92.  Arithmetic and
// results are those of k_step3d.  NTS: Pold, c and the new level bypass the
// caches (grids beyond the Infinity Cache).
template <int ST, int ZC, int MODE, bool CQ, bool NTS>
__global__ __launch_bounds__(256) void k_step3d_short(StepArgs a)
{
    static_assert(ST == kF32 ? !CQ : MODE == kFwd, "16-bit fields: forward steps; 16-bit c with them only");
    using T = typename Stor<ST>::T;
    using CT = std::conditional_t<CQ, uint16_t, float>;
    using PT = Pack<T, 4>;
    using PC = Pack<CT, 4>;
    constexpr int TX = kShortTX, TY = kShortTY, LW = TX + 8, LH = TY + 8, NT = 16 * TY;
    // 4-cell loads of the y halo (8 rows a plane) and of the x halo (2 a row)
    constexpr int YT = 8 * ZC * 16, XT = TY * ZC * 2;
    constexpr int YH = (YT + NT - 1) / NT, XH = (XT + NT - 1) / NT;
    __shared__ __attribute__((aligned(16))) float pl[ZC][LH * LW];
    __shared__ float red[4];
    const int lx = threadIdx.x & 15, ly = threadIdx.x >> 4;
    const int t = xcd_tile(blockIdx.x, a.tiles_x * a.tiles_y * a.tiles_z);
    const int tx = t % a.tiles_x, t2 = t / a.tiles_x, tz = t2 % a.tiles_z, ty = t2 / a.tiles_z;
    const int xb = tx * TX, yb = ty * TY, zb = tz * ZC, x0 = xb + 4 * lx, y = yb + ly;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int zlo = ST == kF32 ? -a.zghost : 0, zhi = ST == kF32 ? nz + a.zghost : nz;
    const size_t px = (size_t)a.px, pp = (size_t)ny * px;
    const bool in = x0 < a.px && y < ny;
    const T *cur = (const T *)a.cur, *prv = (const T *)a.prev;
    const CT *cb;
    if constexpr (CQ)
        cb = a.c16;
    else
        cb = a.c;
    auto load = [&](int z, int yy, int xx, bool ok) -> PT {
        PT p{};
        if (ok) p = ldp<T, 4>(cur + (ptrdiff_t)z * (ptrdiff_t)pp + (size_t)yy * px + xx);
        return p;
    };
    PT q[ZC + 8], pv[ZC], yh[YH], xh[XH];
    PC cv[ZC];
    int ys[YH], xs[XH];
#pragma unroll
    for (int k = 0; k < ZC + 8; ++k) {
        const int z = zb - 4 + k;
        q[k] = load(z, y, x0, in && z >= zlo && z < zhi);
    }
#pragma unroll
    for (int k = 0; k < YH; ++k) {
        const int u = k * NT + (int)threadIdx.x, zz = u / 128, r = (u >> 4) & 7, xx = xb + 4 * (u & 15);
        const int row = r < 4 ? r : TY + r, yy = yb + row - 4;   // row of the LDS plane
        yh[k] = load(zb + zz, yy, xx, u < YT && xx < a.px && yy >= 0 && yy < ny && zb + zz < nz);
        ys[k] = u < YT ? zz * LH * LW + row * LW + 4 + 4 * (u & 15) : -1;
    }
#pragma unroll
    for (int k = 0; k < XH; ++k) {
        const int u = k * NT + (int)threadIdx.x, zz = u / (2 * TY), r = (u >> 1) % TY, side = u & 1;
        const int xx = side ? xb + TX : xb - 4, yy = yb + r;
        xh[k] = load(zb + zz, yy, xx, u < XT && xx >= 0 && xx < a.px && yy < ny && zb + zz < nz);
        xs[k] = u < XT ? zz * LH * LW + (r + 4) * LW + (side ? 4 + TX : 0) : -1;
    }
#pragma unroll
    for (int k = 0; k < ZC; ++k) {
        pv[k] = PT{};
        cv[k] = PC{};
        if (in && zb + k < nz) {
            const size_t e = (size_t)(zb + k) * pp + (size_t)y * px + x0;
            pv[k] = NTS ? ldp_stream<T, 4>(prv + e) : ldp<T, 4>(prv + e);
            cv[k] = NTS ? ldp_stream<CT, 4>(cb + e) : ldp<CT, 4>(cb + e);
        }
    }
    float gx[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) gx[v] = x0 + v < nx ? a.gx[x0 + v] : 0.0f;
    const float gy = y < ny ? a.gy[y] : 0.0f;
    float gz[ZC];
#pragma unroll
    for (int k = 0; k < ZC; ++k) gz[k] = zb + k < nz ? a.gz[zb + k] : 0.0f;
    float inj = 0.0f;
    if constexpr (MODE != kAdj)
        if (a.n + 1 < a.nt) inj = a.amp * a.wavelet[a.n + 1];
    const HalfCtx h = half_prologue<ST>(a, inj, blockIdx.x == 0);

    float *base = &pl[0][0];
    auto put = [&](float *at_l, const PT &p) {
        Pack<float, 4> o;
#pragma unroll
        for (int v = 0; v < 4; ++v) o.v[v] = decode_raw<ST>(p.v[v]);
        stp<float, 4>(at_l, o);
    };
    const int li = (ly + 4) * LW + 4 + 4 * lx;
#pragma unroll
    for (int k = 0; k < ZC; ++k) put(pl[k] + li, q[k + 4]);
#pragma unroll
    for (int k = 0; k < YH; ++k)
        if (ys[k] >= 0) put(base + ys[k], yh[k]);
#pragma unroll
    for (int k = 0; k < XH; ++k)
        if (xs[k] >= 0) put(base + xs[k], xh[k]);
    __syncthreads();

    float lz[ZC][4];
    if constexpr (ST == kF32) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float col[ZC + 8], out[ZC];
#pragma unroll
            for (int k = 0; k < ZC + 8; ++k) col[k] = q[k].v[v];
            axis_d2_run<ZC>(col, out);
#pragma unroll
            for (int k = 0; k < ZC; ++k) lz[k][v] = out[k];
        }
    }
    float bmax = 0.0f;
#pragma unroll
    for (int k = 0; k < ZC; ++k) {
        const int z = zb + k;
        if (z >= nz) break;
        const float *P = pl[k] + li;
        const Pack<float, 4> xl = ldp<float, 4>(P - 4), xr = ldp<float, 4>(P + 4);
        Pack<float, 4> r[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            r[e] = ldp<float, 4>(P + (e - 4) * LW);
            r[4 + e] = ldp<float, 4>(P + (e + 1) * LW);
        }
        float row[12];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            row[v] = xl.v[v];
            row[4 + v] = decode_raw<ST>(q[k + 4].v[v]);
            row[8 + v] = xr.v[v];
        }
        float nw[4], lp[4], G[4], pc[4], cc[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            pc[v] = decode_raw<ST>(pv[k].v[v]);
            cc[v] = (float)cv[k].v[v];
        }
        if constexpr (ST == kF32) {
            float lxx[4];
            axis_d2_run<4>(row, lxx);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float u = row[4 + v];
                const float lyy = axis_d2(r[0].v[v], r[1].v[v], r[2].v[v], r[3].v[v], u, r[4].v[v], r[5].v[v],
                                          r[6].v[v], r[7].v[v]);
                const float lap = lz[k][v] + (lyy + lxx[v]);
                G[v] = (gz[k] * gy) * gx[v];
                nw[v] = leapfrog(G[v], u, cc[v], lap, pc[v]);
                lp[v] = MODE == kAdj ? u : lap;
            }
        } else {
            // the operations of the streaming kernel's 16-bit step, in its order
            const float gr = gz[k] * gy;
            const float sc = CQ ? h.sc * a.c16_scale : h.sc, two = CQ ? 2.0f * a.c16_inv : 2.0f;
            const float r1 = gr * sc, r2 = (gr * gr) * h.sp;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float sk[4];
#pragma unroll
                for (int e = 1; e <= 4; ++e)
                    sk[e - 1] = ((row[4 + v - e] + row[4 + v + e]) + (r[4 - e].v[v] + r[3 + e].v[v])) +
                                (decode_raw<ST>(q[k + 4 - e].v[v]) + decode_raw<ST>(q[k + 4 + e].v[v]));
                const float ctr = row[4 + v];
                const float lap = fmaf(3.0f * kA0, ctr, fmaf(kA4, sk[3], fmaf(kA3, sk[2], fmaf(kA2, sk[1], kA1 * sk[0]))));
                G[v] = 0.0f;
                nw[v] = fmaf(gx[v] * r1, fmaf(cc[v], lap, two * ctr), -((gx[v] * gx[v]) * r2) * pc[v]);
                lp[v] = lap;
            }
        }
        Outgoing<T, 4> out;
        finish_cells<ST, 4, MODE, NTS, false>(a, h, z, y, x0, in, (size_t)z * pp + (size_t)y * px, (uint32_t)x0,
                                              nw, lp, pc, cc, G, inj, bmax, out);
        flush<T, 4, MODE, NTS>(out);
    }
    if constexpr (ST != kF32) block_max_to<NT>(max_slot(a.meta, (int)((a.n + 1) & 3)), bmax * h.sn, red);
}

// --------------------------------------------------------------------------
// Set-up and utility kernels
// --------------------------------------------------------------------------
__global__ void k_fill_u32(uint32_t *p, size_t n, uint32_t val)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = val;
}

// f(i, row, x) for every element i = row n + x of nrows rows of n.  A grid
// holds fewer than 2^32 - 2^23 elements, so the division that finds the row is
// a 32-bit one (a 64-bit one per element cost these kernels as much as their
// memory traffic: k_get_field at 512^3 252 us for 1.07 GB).
template <typename F>
__device__ __forceinline__ void for_elements(int64_t nrows, int32_t n, F f)
{
    const uint32_t total = (uint32_t)nrows * (uint32_t)n, stride = gridDim.x * blockDim.x;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
        const uint32_t row = i / (uint32_t)n;
        f((size_t)i, (size_t)row, (size_t)(i - row * (uint32_t)n));
    }
}

// c = (v dt/h)^2 rounded from FP64 to FP32.
__device__ __forceinline__ float model_c(float v, double r)
{
    const double qq = (double)v * r;
    return (float)(qq * qq);
}

// c padded (skipped when c is null); also the velocity range (max as float
// bits) and a flag for non-positive or non-finite values.  A block folds its
// maximum in once, and only if it exceeds what is there: with one atomic per
// wave the kernel was bound by those on one word (1024^2 190 us, 512^3 514).
__global__ __launch_bounds__(256) void k_model_c(const float *__restrict__ v, float *__restrict__ c, int64_t nrows,
                                                 int32_t nx, int32_t px, double r, uint32_t *scratch)
{
    __shared__ uint32_t red[2][4];
    uint32_t vmax = 0, bad = 0;
    for_elements(nrows, nx, [&](size_t i, size_t rw, size_t x) {
        const float vi = v[i];
        if (!(vi > 0.0f) || !(vi < 3.0e38f)) bad = 1;
        vmax = max(vmax, __float_as_uint(fabsf(vi)));
        if (c != nullptr) c[rw * (size_t)px + x] = model_c(vi, r);
    });
    for (int off = 32; off >= 1; off >>= 1) {
        vmax = max(vmax, (uint32_t)__shfl_xor((int)vmax, off, 64));
        bad |= (uint32_t)__shfl_xor((int)bad, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = vmax;
        red[1][threadIdx.x >> 6] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < 4; ++k) {
            vmax = max(vmax, red[0][k]);
            bad |= red[1][k];
        }
        if (vmax > __atomic_load_n(&scratch[0], __ATOMIC_RELAXED)) atomicMax(&scratch[0], vmax);
        if (bad) atomicOr(&scratch[1], 1u);
    }
}

// c in 16-bit unsigned fixed point: q = min(RNE(c 2^(16-e)), 65535), where
// inv_scale = 2^(16-e) and c < 2^e for every cell (the product is exact).
__global__ void k_model_c16(const float *__restrict__ v, uint16_t *__restrict__ c16, int64_t nrows,
                            int32_t nx, int32_t px, double r, float inv_scale)
{
    for_elements(nrows, nx, [&](size_t i, size_t rw, size_t x) {
        const float q = fminf(rintf(model_c(v[i], r) * inv_scale), 65535.0f);
        c16[rw * (size_t)px + x] = (uint16_t)q;
    });
}

// First source addition of a shot into the zeroed level-0 field (+ the
// storage exponent and magnitude of levels 0 and -1).  The wave also scans
// the shot's nt injected values amp * s[n] and records a non-finite one in
// the shot's health flags.
template <int ST>
__global__ void k_begin(void *cur, int64_t src_off, float amp, const float *wavelet, int64_t nt,
                        int32_t *meta)
{
    bool bad = false;
    for (int64_t i = threadIdx.x; i < nt; i += blockDim.x) bad |= !(fabsf(amp * wavelet[i]) <= 3.4028235e38f);
    if (__ballot(bad) != 0 && threadIdx.x == 0) atomicOr((uint32_t *)&meta[kHealth], kNonfiniteInput);
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    using T = typename Stor<ST>::T;
    const float x0 = amp * wavelet[0];
    if constexpr (ST == kF32) {
        ((T *)cur)[src_off] = x0;
    } else {
        // the state was cleared: every exponent and magnitude slot is zero
        const int e0 = storage_exponent(fabsf(x0));
        ((T *)cur)[src_off] = encode<ST>(x0, pow2i(-e0));
        meta[0] = e0;
        meta[slot_word(0, 0)] = (int32_t)__float_as_uint(fabsf(x0));
    }
}

template <int ST>
__global__ void k_get_field(const void *buf, float *__restrict__ out, int64_t nrows, int32_t nx,
                            int32_t px, const int32_t *meta, int32_t level_slot)
{
    using T = typename Stor<ST>::T;
    float s = 1.0f;
    if constexpr (ST != kF32) s = pow2i(meta[level_slot]);
    for_elements(nrows, nx, [&](size_t i, size_t rw, size_t x) {
        out[i] = decode<ST>(((const T *)buf)[rw * (size_t)px + x], s);
    });
}

// Clears a level's magnitude slots.
__global__ void k_clear_level(int32_t *meta, int32_t level) { meta[slot_word(level, threadIdx.x)] = 0; }

// max |x| over a dense array, folded into a level's magnitude slots.
__global__ void k_absmax(const float *__restrict__ x, size_t n, int32_t *meta, int32_t level)
{
    float m = 0.0f;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) m = fmaxf(m, fabsf(x[i]));
    for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    if ((threadIdx.x & 63) == 0) fold_max(max_slot(meta, level), m);
}

// Dense FP32 -> padded stored field; 16-bit storage takes its exponent from
// the magnitude in meta[4 + slot] and records it in meta[slot].
template <int ST>
__global__ void k_set_field(const float *__restrict__ in, void *buf, int64_t nrows, int32_t nx,
                            int32_t px, int32_t *meta, int32_t slot)
{
    using T = typename Stor<ST>::T;
    float inv = 1.0f;
    if constexpr (ST != kF32) {
        const int e = storage_exponent(level_max(meta, slot, slot));
        inv = pow2i(-e);
        if (blockIdx.x == 0 && threadIdx.x == 0) meta[slot] = e;
    }
    bool bad = false;
    for_elements(nrows, px, [&](size_t i, size_t rw, size_t x) {
        const float v = x < (size_t)nx ? in[rw * (size_t)nx + x] : 0.0f;
        bad |= !(fabsf(v) <= 3.4028235e38f);
        ((T *)buf)[i] = encode<ST>(v, inv);
    });
    // a non-finite value set into the shot is recorded in its health flags
    if (__ballot(bad) != 0 && (threadIdx.x & 63) == 0) atomicOr((uint32_t *)&meta[kHealth], kNonfiniteInput);
}

// The two copies of a ghost exchange in one launch: n16 16-byte words from
// u_own to d_ghost and from d_own to u_ghost.  (Two device-to-device copies
// cost 13 us a step of three small slabs; this kernel about 4 an exchange.)
__global__ __launch_bounds__(256) void k_exchange(const uint4 *__restrict__ u_own, uint4 *__restrict__ d_ghost,
                                                  const uint4 *__restrict__ d_own, uint4 *__restrict__ u_ghost,
                                                  size_t n16)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n16; i += stride) {
        const uint4 a = u_own[i], b = d_own[i];
        d_ghost[i] = a;
        u_ghost[i] = b;
    }
}

// Sets `bit` in *flags when a stored level holds a non-finite value (NaN or
// infinity), and (health non-null) the shot's sticky non-finite-input flag: the exponent field of a code all ones (FP32 0x7F800000,
// binary16 0x7C00, bfloat16 0x7F80), tested on the raw codes 16 bytes at a
// time without decoding; one atomic per wave that found one.
template <int ST>
__global__ void k_nonfinite(const uint4 *__restrict__ p, size_t n16, uint32_t *flags, uint32_t bit,
                            const int32_t *health)
{
    if (health != nullptr && blockIdx.x == 0 && threadIdx.x == 0) {
        const uint32_t hf = (uint32_t)*health & kNonfiniteInput;
        if (hf) atomicOr(flags, hf);
    }
    bool bad = false;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n16; i += stride) {
        const uint4 q = p[i];
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if constexpr (ST == kF32)
                bad |= (w[k] & 0x7F800000u) == 0x7F800000u;
            else if constexpr (ST == kF16)
                bad |= ((w[k] & 0x7C00u) == 0x7C00u) | ((w[k] & 0x7C000000u) == 0x7C000000u);
            else
                bad |= ((w[k] & 0x7F80u) == 0x7F80u) | ((w[k] & 0x7F800000u) == 0x7F800000u);
        }
    }
    if (__ballot(bad) != 0 && (threadIdx.x & 63) == 0) atomicOr(flags, bit);
}

// grad_v += dJ/dc * 2c/v with v = (h/dt) sqrt(c): 2 g dt / (h sqrt(c)).
__global__ void k_grad_finish(const double *__restrict__ g, const float *__restrict__ c,
                              double *__restrict__ grad_v, int64_t nrows, int32_t nx, int32_t px,
                              double two_dt_over_h)
{
    for_elements(nrows, nx, [&](size_t i, size_t rw, size_t x) {
        const size_t p = rw * (size_t)px + x;
        grad_v[i] += g[p] * two_dt_over_h / sqrt((double)c[p]);
    });
}

// image += the accumulated zero-lag correlation (padded -> dense).
__global__ void k_image_finish(const double *__restrict__ g, double *__restrict__ image,
                               int64_t nrows, int32_t nx, int32_t px)
{
    for_elements(nrows, nx, [&](size_t i, size_t rw, size_t x) { image[i] += g[rw * (size_t)px + x]; });
}

// --------------------------------------------------------------------------
// Host launchers
// --------------------------------------------------------------------------
static int grid_blocks(size_t n, int threads)
{
    size_t b = (n + threads - 1) / threads;
    if (b > 8192) b = 8192;
    if (b < 1) b = 1;
    return (int)b;
}

hipError_t launch_fill_u32(void *p, size_t nwords, uint32_t val, hipStream_t s)
{
    if (nwords == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_blocks(nwords, 256)), dim3(256), 0, s,
                       (uint32_t *)p, nwords, val);
    return hipGetLastError();
}

hipError_t launch_model_c(const float *v, float *c, int64_t nrows, int32_t nx, int32_t px,
                          double r, uint32_t *scratch, hipStream_t s)
{
    hipLaunchKernelGGL(k_model_c, dim3(std::min(2048, (grid_blocks((size_t)nrows * nx, 256) + 3) / 4)), dim3(256), 0, s,
                       v, c, nrows, nx, px, r, scratch);
    return hipGetLastError();
}

hipError_t launch_model_c16(const float *v, uint16_t *c16, int64_t nrows, int32_t nx, int32_t px,
                            double r, float inv_scale, hipStream_t s)
{
    hipLaunchKernelGGL(k_model_c16, dim3(grid_blocks((size_t)nrows * nx, 256)), dim3(256), 0, s,
                       v, c16, nrows, nx, px, r, inv_scale);
    return hipGetLastError();
}

hipError_t launch_begin(int storage, void *cur, int64_t src_off, float amp,
                        const float *wavelet, int64_t nt, int32_t *meta, hipStream_t s)
{
    switch (storage) {
    case kF32: hipLaunchKernelGGL(k_begin<kF32>, dim3(1), dim3(64), 0, s, cur, src_off, amp, wavelet, nt, meta); break;
    case kF16: hipLaunchKernelGGL(k_begin<kF16>, dim3(1), dim3(64), 0, s, cur, src_off, amp, wavelet, nt, meta); break;
    default: hipLaunchKernelGGL(k_begin<kBF16>, dim3(1), dim3(64), 0, s, cur, src_off, amp, wavelet, nt, meta); break;
    }
    return hipGetLastError();
}

hipError_t launch_get_field(int storage, const void *buf, float *out, int64_t nrows, int32_t nx,
                            int32_t px, const int32_t *meta, int32_t level_slot, hipStream_t s)
{
    const dim3 g(grid_blocks((size_t)nrows * nx, 256)), b(256);
    switch (storage) {
    case kF32: hipLaunchKernelGGL(k_get_field<kF32>, g, b, 0, s, buf, out, nrows, nx, px, meta, level_slot); break;
    case kF16: hipLaunchKernelGGL(k_get_field<kF16>, g, b, 0, s, buf, out, nrows, nx, px, meta, level_slot); break;
    default: hipLaunchKernelGGL(k_get_field<kBF16>, g, b, 0, s, buf, out, nrows, nx, px, meta, level_slot); break;
    }
    return hipGetLastError();
}

hipError_t launch_set_field(int storage, const float *in, void *buf, int64_t nrows, int32_t nx,
                            int32_t px, int32_t *meta, int32_t slot, hipStream_t s)
{
    if (storage != kF32) {
        hipLaunchKernelGGL(k_clear_level, dim3(1), dim3(kMaxSlots), 0, s, meta, slot);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_absmax, dim3(grid_blocks((size_t)nrows * nx, 256)), dim3(256), 0, s,
                           in, (size_t)nrows * nx, meta, slot);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const dim3 g(grid_blocks((size_t)nrows * px, 256)), b(256);
    switch (storage) {
    case kF32: hipLaunchKernelGGL(k_set_field<kF32>, g, b, 0, s, in, buf, nrows, nx, px, meta, slot); break;
    case kF16: hipLaunchKernelGGL(k_set_field<kF16>, g, b, 0, s, in, buf, nrows, nx, px, meta, slot); break;
    default: hipLaunchKernelGGL(k_set_field<kBF16>, g, b, 0, s, in, buf, nrows, nx, px, meta, slot); break;
    }
    return hipGetLastError();
}

hipError_t launch_exchange(const void *u_own, void *d_ghost, const void *d_own, void *u_ghost, size_t bytes,
                           hipStream_t s)
{
    if (bytes % 16 != 0) return hipErrorInvalidValue;
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    hipLaunchKernelGGL(k_exchange, dim3(grid_blocks(n16, 256)), dim3(256), 0, s, (const uint4 *)u_own,
                       (uint4 *)d_ghost, (const uint4 *)d_own, (uint4 *)u_ghost, n16);
    return hipGetLastError();
}

hipError_t launch_nonfinite(int storage, const void *level, size_t bytes, uint32_t *flags, uint32_t bit,
                            const int32_t *health, hipStream_t s)
{
    if (bytes % 16 != 0) return hipErrorInvalidValue;
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    const dim3 g(grid_blocks(n16, 256)), b(256);
    const uint4 *p = (const uint4 *)level;
    switch (storage) {
    case kF32: hipLaunchKernelGGL(k_nonfinite<kF32>, g, b, 0, s, p, n16, flags, bit, health); break;
    case kF16: hipLaunchKernelGGL(k_nonfinite<kF16>, g, b, 0, s, p, n16, flags, bit, health); break;
    default: hipLaunchKernelGGL(k_nonfinite<kBF16>, g, b, 0, s, p, n16, flags, bit, health); break;
    }
    return hipGetLastError();
}

hipError_t launch_image_finish(const double *g, double *image, int64_t nrows, int32_t nx,
                               int32_t px, hipStream_t s)
{
    hipLaunchKernelGGL(k_image_finish, dim3(grid_blocks((size_t)nrows * nx, 256)), dim3(256), 0, s,
                       g, image, nrows, nx, px);
    return hipGetLastError();
}

hipError_t launch_grad_finish(const double *g, const float *c, double *grad_v, int64_t nrows,
                              int32_t nx, int32_t px, double two_dt_over_h, hipStream_t s)
{
    hipLaunchKernelGGL(k_grad_finish, dim3(grid_blocks((size_t)nrows * nx, 256)), dim3(256), 0,
                       s, g, c, grad_v, nrows, nx, px, two_dt_over_h);
    return hipGetLastError();
}

// Tile shapes.  2D: one wave, 64*VX columns by zc rows.  3D: NW waves of
// RPW rows each, (64/RPW*VX) x (NW*RPW*RY) cells by zc planes: FP32 fields
// 256x8 (4 cells x 2 rows per lane) or, chosen per grid, 128x8 (below),
// 16-bit fields 128x8 (4 cells x 1 row per lane, two rows per wave: half the
// y-halo loads of a 256x4 tile, measured 568 -> 554 us at 768x768x512 BF16).
// (Overridable at build time for tuning.)
#ifndef FD_3D_VX32
#define FD_3D_VX32 4
#endif
#ifndef FD_3D_RY32
#define FD_3D_RY32 2
#endif
#ifndef FD_3D_VX16
#define FD_3D_VX16 4
#endif
#ifndef FD_3D_RY16
#define FD_3D_RY16 1
#endif
#ifndef FD_3D_NW32
#define FD_3D_NW32 4
#endif
#ifndef FD_3D_NW16
#define FD_3D_NW16 4
#endif
#ifndef FD_3D_RPW32
#define FD_3D_RPW32 1
#endif
#ifndef FD_3D_RPW16
#define FD_3D_RPW16 2
#endif
constexpr int k3dVX32 = FD_3D_VX32, k3dRY32 = FD_3D_RY32;   // FP32 fields
constexpr int k3dVX16 = FD_3D_VX16, k3dRY16 = FD_3D_RY16;   // 16-bit fields

// FP32 fields have two tile shapes: 256x8 (4 cells x 2 rows per lane, 2
// waves per SIMD) and 128x8 (4 cells x 1 row per lane, two rows per wave, 3
// waves per SIMD).  The wide tile is faster on large grids that it fits
// (512^3 369 against 390 us, 768x768x512 860 against 925: about 5.5% per
// column), the narrow one where the x size leaves much of the last 256-wide
// tile empty (384^3 210 -> 155 us, 640x640x256 358 -> 310, 896x448x256 331 ->
// 305) and below 2^26 cells, where short z-chunks fill the device and twice
// the columns help (768x256x256 140 -> 135); same bits either way.
constexpr int k3dRYN32 = 1, k3dRPWN32 = 2;
constexpr int k3dTXW32 = 64 / FD_3D_RPW32 * k3dVX32, k3dTXN32 = 64 / k3dRPWN32 * k3dVX32;

// Whether an FP32 3D step takes the narrow tile: when its padded width, at
// 1.055 times the cost per column, is smaller, or when the grid (at the
// wide tile's padded width) holds fewer than 2^26 cells.
static bool narrow_tile_f32(int nx, int ny, int nz)
{
    const int64_t wide = ((int64_t)nx + k3dTXW32 - 1) / k3dTXW32 * k3dTXW32;
    const int64_t narrow = ((int64_t)nx + k3dTXN32 - 1) / k3dTXN32 * k3dTXN32;
    return 1000 * wide > 1055 * narrow || wide * ny * nz < ((int64_t)1 << 26);
}

// The 3D forward kernel of a storage kind (16-bit c or not; FP32: the
// narrow tile or not).
template <int ST, bool CQ, bool NARROW = false>
static const void *step3d_fwd_kernel()
{
    if constexpr (ST == kF32 && NARROW)
        return reinterpret_cast<const void *>(&k_step3d<kF32, k3dVX32, k3dRYN32, FD_3D_NW32, k3dRPWN32, kFwd, false>);
    else if constexpr (ST == kF32)
        return reinterpret_cast<const void *>(&k_step3d<kF32, k3dVX32, k3dRY32, FD_3D_NW32, FD_3D_RPW32, kFwd, false>);
    else
        return reinterpret_cast<const void *>(&k_step3d<ST, k3dVX16, k3dRY16, FD_3D_NW16, FD_3D_RPW16, kFwd, CQ>);
}

// Blocks of the 3D forward kernel that fit on the device at once (queried
// once per kernel; the CU count times the occupancy per CU).
static int64_t resident_blocks_3d(int storage, bool cq, bool narrow)
{
    static int64_t cache[6] = {0, 0, 0, 0, 0, 0};
    const int k = storage == kF32 ? (narrow ? 5 : 0) : (storage == kF16 ? 1 : 2) + (cq ? 2 : 0);
    if (cache[k] == 0) {
        int dev = 0, cus = 0, per_cu = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e == hipSuccess) {
            const void *f = storage == kF32 ? (narrow ? step3d_fwd_kernel<kF32, false, true>()
                                                      : step3d_fwd_kernel<kF32, false>())
                            : storage == kF16 ? (cq ? step3d_fwd_kernel<kF16, true>() : step3d_fwd_kernel<kF16, false>())
                                              : (cq ? step3d_fwd_kernel<kBF16, true>() : step3d_fwd_kernel<kBF16, false>());
            const int threads = 64 * (storage == kF32 ? FD_3D_NW32 : FD_3D_NW16);
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, threads, 0);
        }
        (void)hipGetLastError();
        cache[k] = (e == hipSuccess && cus > 0 && per_cu > 0) ? (int64_t)cus * per_cu : 512;
    }
    return cache[k];
}

// Tile shapes.  3D: NW waves of RPW rows, (64/RPW VX) x (NW RPW RY) cells by
// zc planes (the defaults come from a sweep of shapes on the 512^3 and
// 768x768x512 grids; FP32 grids pick the wide or the narrow tile with
// narrow_tile_f32).
// 2D: blocks of 128 columns by 8 RZ rows.  FP32 fields take RZ = 1 everywhere
// (RZ = 2 and 4 within 3% where they are faster: 1024^2 5.6 / 5.4 / 5.8 us,
// 2048 x 4096 22.7 / 23.3 / 25.1).  16-bit blocks each read the 128 magnitude
// words and fold a maximum, so larger blocks pay earlier (BF16, RZ = 1 / 2 / 4:
// 512^2 5.4 / 5.8 / 7.1 us, 1024^2 8.2 / 7.2 / 7.7, 1201 x 1747 13.0 / 9.3 /
// 9.6, 2048^2 19.6 / 14.6 / 11.8), and above 1536 blocks of RZ = 4 the
// streaming kernel with chunks of 16 rows is kept (2048 x 4096 binary16 23.1
// us against 26.2, with 16-bit c 22.1 against 24.8).
//
// 3D also has the short kernel (k_step3d_short): short_plan says where.
void plan_tiles(StepArgs &a, int ndim, int storage, int mode)
{
    if (ndim == 2) {
        // a.vx records RZ (0: the streaming kernel)
        a.tiles_x = (a.px + 127) / 128;
        a.tiles_y = 1;
        auto blocks = [&](int rz) { return (int64_t)a.tiles_x * ((a.nz + 8 * rz - 1) / (8 * rz)); };
        a.vx = storage == kF32 || blocks(1) <= 320 ? 1 : blocks(2) <= 1100 ? 2 : blocks(4) <= 1536 ? 4 : 0;
        a.zc = a.vx ? 8 * a.vx : 16;
        a.tiles_z = (a.nz + a.zc - 1) / a.zc;
    } else {
        // 3D: a.vx records the tile width in units of 64 cells, which picks
        // the FP32 kernel (4: 256 wide, 2: 128 wide; the short kernel: 1, or 0
        // with accesses that bypass the caches)
        const bool narrow = storage == kF32 && narrow_tile_f32(a.nx, a.ny, a.nz);
        const int VX = storage == kF32 ? k3dVX32 : k3dVX16;
        const int RY = storage == kF32 ? (narrow ? k3dRYN32 : k3dRY32) : k3dRY16;
        const int NW = storage == kF32 ? FD_3D_NW32 : FD_3D_NW16;
        const int RPW = storage == kF32 ? (narrow ? k3dRPWN32 : FD_3D_RPW32) : FD_3D_RPW16;
        const int TX = 64 / RPW * VX, TY = NW * RPW * RY;
        const ShortPlan sp = short_plan(a.nz, a.ny, a.nx, a.px, storage == kF32, mode == kAdj, TX, TY);
        if (sp.zc > 0) {
            a.vx = sp.stream ? 0 : 1;
            a.zc = sp.zc;
            a.tiles_x = (a.px + kShortTX - 1) / kShortTX;
            a.tiles_y = (a.ny + kShortTY - 1) / kShortTY;
            a.tiles_z = (a.nz + a.zc - 1) / a.zc;
            return;
        }
        a.vx = (int16_t)(TX / 64);
        a.tiles_x = (a.nx + TX - 1) / TX;
        a.tiles_y = (a.ny + TY - 1) / TY;
        // Planes per block: a block streams zc planes after priming 8 halo
        // planes, and blocks run in R = ceil(blocks / resident) rounds, so
        // the time goes as (R + 3/16) * (zc + 8), the fraction standing for
        // filling and draining the device, which a later round overlaps with
        // the blocks still running (512^3 FP32: two rounds of 64 planes 364
        // us against one round of 128 planes 371 us; 16-bit fields: one
        // round of 171 planes and two of 86 within 1%).  The column is cut
        // into k equal chunks (zc = ceil(nz / k) >= 4: short columns, such
        // as a z-slab's, need short chunks to fill the device: 32 planes of
        // 512^2 in chunks of 8 take 31 us against 40 in chunks of 16); ties
        // go to the longer chunk (less halo traffic).
        const int64_t cols = (int64_t)a.tiles_x * a.tiles_y;
        const int64_t resident = resident_blocks_3d(storage, a.c16 != nullptr, narrow);
        a.resident = (int32_t)std::min<int64_t>(resident, 1 << 30);
        int64_t best = -1;
        for (int k = 1; k <= std::max(1, a.nz / 4); ++k) {
            const int zc = (a.nz + k - 1) / k;
            const int64_t nb = cols * ((a.nz + zc - 1) / zc);
            const int64_t cost = (16 * ((nb + resident - 1) / resident) + 3) * (int64_t)(zc + 8);
            if (best < 0 || cost < best) {
                best = cost;
                a.zc = zc;
            }
        }
        a.tiles_z = (a.nz + a.zc - 1) / a.zc;
    }
}

template <int ST, int MODE, bool CQ = false>
static void launch3d(const StepArgs &a, int nb, hipStream_t s)
{
    if constexpr (ST == kF32) {
        if (a.vx == 1 && a.zc == 2)
            hipLaunchKernelGGL((k_step3d_short<kF32, 2, MODE, false, false>), dim3(nb), dim3(256), 0, s, a);
        else if (a.vx == 1)
            hipLaunchKernelGGL((k_step3d_short<kF32, 4, MODE, false, false>), dim3(nb), dim3(256), 0, s, a);
        else if (a.vx == 0)
            hipLaunchKernelGGL((k_step3d_short<kF32, 4, MODE, false, true>), dim3(nb), dim3(256), 0, s, a);
        else if (a.vx * 64 == k3dTXN32)
            hipLaunchKernelGGL((k_step3d<ST, k3dVX32, k3dRYN32, FD_3D_NW32, k3dRPWN32, MODE, false>), dim3(nb),
                               dim3(64 * FD_3D_NW32), 0, s, a);
        else
            hipLaunchKernelGGL((k_step3d<ST, k3dVX32, k3dRY32, FD_3D_NW32, FD_3D_RPW32, MODE, false>), dim3(nb),
                               dim3(64 * FD_3D_NW32), 0, s, a);
    }
    else if (a.vx == 1 && a.zc == 2)
        hipLaunchKernelGGL((k_step3d_short<ST, 2, MODE, CQ, false>), dim3(nb), dim3(256), 0, s, a);
    else if (a.vx == 1)
        hipLaunchKernelGGL((k_step3d_short<ST, 4, MODE, CQ, false>), dim3(nb), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((k_step3d<ST, k3dVX16, k3dRY16, FD_3D_NW16, FD_3D_RPW16, MODE, CQ>), dim3(nb),
                           dim3(64 * FD_3D_NW16), 0, s, a);
}

template <int ST, int MODE = kFwd, bool CQ = false>
static void launch2d(const StepArgs &a, int nb, hipStream_t s)
{
    if constexpr (ST == kF32) {
        hipLaunchKernelGGL((k_step2d_block<ST, 1, MODE, CQ>), dim3(nb), dim3(256), 0, s, a);
    } else {
        if (a.vx == 1) hipLaunchKernelGGL((k_step2d_block<ST, 1, MODE, CQ>), dim3(nb), dim3(256), 0, s, a);
        else if (a.vx == 2) hipLaunchKernelGGL((k_step2d_block<ST, 2, MODE, CQ>), dim3(nb), dim3(256), 0, s, a);
        else if (a.vx == 4) hipLaunchKernelGGL((k_step2d_block<ST, 4, MODE, CQ>), dim3(nb), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((k_step2d<ST, CQ>), dim3(nb), dim3(64), 0, s, a);
    }
}

hipError_t launch_step(StepArgs a, int ndim, int storage, int mode, hipStream_t s)
{
    // 16-bit c is built for the forward step on 16-bit fields only
    if (a.c16 != nullptr && (storage == kF32 || mode != kFwd)) return hipErrorInvalidValue;
    // a recompute that keeps L(cur) is launch_multi2d's in 2D
    if (ndim == 2 && (mode == kFwdLap || (storage != kF32 && mode != kFwd))) return hipErrorInvalidValue;
    plan_tiles(a, ndim, storage, mode);
    const int nb = a.tiles_x * a.tiles_y * a.tiles_z;
    if (ndim == 2) {
        const bool cq = a.c16 != nullptr;
        if (storage == kF32 && mode == kAdj) launch2d<kF32, kAdj>(a, nb, s);
        else if (storage == kF32) launch2d<kF32>(a, nb, s);
        else if (storage == kF16 && cq) launch2d<kF16, kFwd, true>(a, nb, s);
        else if (storage == kF16) launch2d<kF16>(a, nb, s);
        else if (cq) launch2d<kBF16, kFwd, true>(a, nb, s);
        else launch2d<kBF16>(a, nb, s);
    } else {
        if (storage == kF32) {
            if (mode == kFwd) launch3d<kF32, kFwd>(a, nb, s);
            else if (mode == kFwdLap) launch3d<kF32, kFwdLap>(a, nb, s);
            else launch3d<kF32, kAdj>(a, nb, s);
        } else if (storage == kF16) {
            if (a.c16 != nullptr) launch3d<kF16, kFwd, true>(a, nb, s);
            else launch3d<kF16, kFwd>(a, nb, s);
        } else {
            if (a.c16 != nullptr) launch3d<kBF16, kFwd, true>(a, nb, s);
            else launch3d<kBF16, kFwd>(a, nb, s);
        }
    }
    return hipGetLastError();
}

hipError_t launch_step_batch2d(Batch2D &b, int mode, hipStream_t s)
{
    if (mode != kFwd && mode != kAdj) return hipErrorInvalidValue;
    int total = 0;
    for (int i = 0; i < b.count; ++i) {
        plan_tiles(b.it[i], 2, kF32, mode);
        b.begin[i] = total;
        total += b.it[i].tiles_x * b.it[i].tiles_z;
    }
    b.begin[b.count] = total;
    if (total == 0) return hipSuccess;
    if (mode == kAdj) hipLaunchKernelGGL(k_step2d_batch<kAdj>, dim3(total), dim3(256), 0, s, b);
    else hipLaunchKernelGGL(k_step2d_batch<kFwd>, dim3(total), dim3(256), 0, s, b);
    return hipGetLastError();
}

}  // namespace fdk

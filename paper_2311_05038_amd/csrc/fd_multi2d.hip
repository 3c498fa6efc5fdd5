// Several 2D FP32 time steps per launch (temporal blocking) for gfx950.
//
// A 2D grid of a survey is small: on 256 x 256 cells a step moves 1 MB, less
// than a kernel launch takes, and up to 2048 x 4096 the fields stay in the
// 256 MB Infinity Cache, whose bandwidth (8 TB/s for a copy) then bounds a
// kernel that reads three fields and writes one every step.  Here a block
// loads a tile of P, Pold and c once, takes S steps on it and stores the last
// two levels: launches and traffic fall by S, against redundant work in a
// halo of 4 S cells around the tile.
//
// Layout.  A block of TXL * NZ threads owns an ext tile of (4 TXL) x (RZ NZ)
// cells; a thread keeps 4 columns x RZ rows of P, Pold and c in registers for
// all S steps.  P is also written to LDS after every step (two buffers, one
// barrier per step): the rows above and below a thread's run and the 4
// columns on each side are read from there, 16 bytes at a time.  The valid
// region shrinks by 4 cells a side and step, and waves whose rows have left
// it skip the step; cells outside it hold unused values.  Tiles overlap by
// 8 S cells, so S steps cost (ext tile minus the skipped rows) / (inner tile)
// of the work: 1.56 for S = 4 on 128 x 128.
//
// The forward step is VALU-bound (by the counters 34 vector instructions per
// computed cell and step, which take 82% of a launch's time on 2048 x 4096 and
// 66% on 1024^2; the adjoint's 43%, its history and FP64 sum move at 4.5 TB/s):
// the differences of neighbouring cells that the second difference needs
// twice, u[i+1] - u[i] and u[i+2] - u[i], are formed once per run of cells and
// subtracted, 1.25 instructions less per axis and cell than in axis_d2.
//
// A block walks over its tiles: the next tile's P is copied straight into the
// LDS buffer that the last step of the present one no longer writes, and
// Pold and c arrive while the first step's differences are computed, so only
// a block's first tile waits for its loads.
//
// Per cell the operations and their order are those of the single step
// kernels in 2D: the results are the same bits.
#include <algorithm>

#include "fd_device.hpp"
#include "fd_launch.hpp"

namespace fdk {

// 16 bytes per lane from global memory straight into LDS: lane l of the wave
// writes at lds + 16 l (lds is the wave's address, the same in every lane).
__device__ __forceinline__ void load_to_lds16(const float *g, float *lds)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)g,
                                     (__attribute__((address_space(3))) void *)lds, 16, 0, 0);
}

// An item's arguments, in scalar registers from here on: read where they are
// used, the compiler loads them again in every step (600 scalar loads in the
// batched kernel, each a wait shared with the LDS reads: 3.2 us a step on a
// 128 x 128 tile against 2.3 with a lone item).
template <int N>
__device__ __forceinline__ MultiArgs item_args(const MultiBatch<N> &b, int i)
{
    MultiArgs a = b.it[N > 1 ? i : 0];
    if constexpr (N > 1) {
        static_assert(sizeof(MultiArgs) % 4 == 0, "words");
        uint32_t w[sizeof(MultiArgs) / 4];
        __builtin_memcpy(w, &a, sizeof(a));
#pragma unroll
        for (size_t k = 0; k < sizeof(MultiArgs) / 4; ++k) asm volatile("" : "+s"(w[k]));
        __builtin_memcpy(&a, w, sizeof(a));
    }
    return a;
}

template <int TXL, int RZ, int NZ, int MODE, int WPS, int N>
__global__ __launch_bounds__(TXL *NZ, WPS) void k_multi2d(const MultiBatch<N> b)
{
    constexpr int NT = TXL * NZ, EX = 4 * TXL, EZ = RZ * NZ;
    static_assert(NT % 64 == 0, "whole waves");
    // two objects, so that a copy into one is known not to touch the other;
    // 4 rows before and after hold whatever reads past the tile find
    __shared__ __attribute__((aligned(16))) float buf0[(EZ + 8) * EX];
    __shared__ __attribute__((aligned(16))) float buf1[(EZ + 8) * EX];
    const int lx = threadIdx.x % TXL, lz = threadIdx.x / TXL;
    const int lbase = (RZ * lz + 4) * EX + 4 * lx;
    const int total = b.total;
    // XCD k (blocks are dealt round-robin) walks the k-th eighth of the tiles
    const int per = (total + 7) >> 3, xcd = blockIdx.x & 7, stride = (int)(gridDim.x >> 3);
    const int tend = min(total, (xcd + 1) * per);

    // The item whose tiles hold t: lane i holds item i's first tile.  (A walk
    // over them by scalar loads, each waiting for the one before, cost 1 us a
    // tile.)  A lone item's arguments are at fixed places instead.
    int first_tile = INT32_MAX;
    if constexpr (N > 1)
        if ((int)(threadIdx.x & 63) < b.count) first_tile = b.begin[threadIdx.x & 63];
    auto item_of = [&](int t) -> int {
        if constexpr (N > 1)
            return __popcll(__ballot(first_tile <= t)) - 1;
        else
            return 0;
    };

    // P of tile t into `buf` (rows and columns clamped into the field)
    auto fetch = [&](int t, int i, float *buf) {
        const MultiArgs &a = b.it[i];
        const int lt = t - b.begin[i], tz = lt / a.tiles_x, tx = lt - tz * a.tiles_x;
        const int zb = tz * (EZ - 8 * a.steps) - 4 * a.steps, xb = tx * (EX - 8 * a.steps) - 4 * a.steps;
#pragma unroll
        for (int r = 0; r < RZ; ++r) {
            const int u = r * NT + (int)threadIdx.x;
            const int z = min(max(zb + u / TXL, 0), a.nz - 1);
            const int x = min(max(xb + 4 * (u % TXL), 0), a.px - 4);
            const int u0 = __builtin_amdgcn_readfirstlane(r * NT + ((int)threadIdx.x & ~63));
            load_to_lds16(a.cur + (size_t)z * a.px + x, buf + 4 * EX + 4 * u0);
        }
    };

    int t = xcd * per + (int)(blockIdx.x >> 3);
    if (t >= tend) return;
    int it = item_of(t);
    fetch(t, it, buf0);
    for (bool first = true;; first = false) {
        const MultiArgs a = item_args(b, it);
        const int S = a.steps, H = 4 * S;
        const int lt = t - b.begin[it], tz = lt / a.tiles_x, tx = lt - tz * a.tiles_x;
        const int xb = tx * (EX - 2 * H) - H, zb = tz * (EZ - 2 * H) - H;
        const int x0 = xb + 4 * lx, z0 = zb + RZ * lz;
        const bool edge = xb < 0 || zb < 0 || xb + EX > a.nx || zb + EZ > a.nz;
        const bool xin = x0 >= 0 && x0 < a.px;
        // the thread's columns belong to this tile (not to its halo)
        const bool own_x = 4 * lx >= H && 4 * lx < EX - H && xin;
        const int xc = min(max(x0, 0), a.px - 4);

        float A[RZ][4], B[RZ][4], C[RZ][4], gx[4], gz[RZ];
        auto field = [&](const float *f, float (&o)[RZ][4]) {
#pragma unroll
            for (int r = 0; r < RZ; ++r) {
                const int z = min(max(z0 + r, 0), a.nz - 1);
                const Pack<float, 4> p = ldp<float, 4>(f + (size_t)z * a.px + xc);
#pragma unroll
                for (int v = 0; v < 4; ++v) o[r][v] = p.v[v];
            }
        };
        asm volatile("" ::: "memory");   // the loads below stay behind the copy of P
        field(a.prev, B);
        field(a.c, C);
        {
            const Pack<float, 4> p = ldp<float, 4>(a.gx + xc);
#pragma unroll
            for (int v = 0; v < 4; ++v) gx[v] = p.v[v];
#pragma unroll
            for (int r = 0; r < RZ; ++r) gz[r] = a.gz[min(max(z0 + r, 0), a.nz - 1)];
        }
        // a block's first tile waits for its P here (all but the 2 RZ loads of
        // Pold and c, at least, that were issued after it); later ones waited
        // before the stores of the tile before
        if (first) {
            static_assert(RZ <= 8, "the count of a wait on memory");
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * RZ) : "memory");
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RZ; ++r) {
            const Pack<float, 4> p = ldp<float, 4>(buf0 + lbase + r * EX);
#pragma unroll
            for (int v = 0; v < 4; ++v) A[r][v] = p.v[v];
        }
        // zero outside the grid
        auto mask = [&](float (&o)[RZ][4]) {
            int zo = z0, xo = x0;
            asm volatile("" : "+v"(zo), "+v"(xo));   // keep no derived mask in registers
#pragma unroll
            for (int r = 0; r < RZ; ++r) {
                const bool zi = (unsigned)(zo + r) < (unsigned)a.nz;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (!(zi && (unsigned)(xo + v) < (unsigned)a.nx)) o[r][v] = 0.0f;
            }
        };
        auto put = [&](float *buf, const float (&u)[RZ][4]) {
#pragma unroll
            for (int r = 0; r < RZ; ++r) {
                Pack<float, 4> p;
#pragma unroll
                for (int v = 0; v < 4; ++v) p.v[v] = u[r][v];
                stp<float, 4>(buf + lbase + r * EX, p);
            }
        };
        if (edge) {
            // only the cells outside the grid change, and no step has begun
            mask(A);
            put(buf0, A);
        }
        // whole rows of the tile's inner region (clipped to the field) to dst
        auto store = [&](float *dst, const float (&u)[RZ][4], bool stream = false) {
            if (dst != nullptr && own_x) {
                int zo = z0, xo = x0;
                asm volatile("" : "+v"(zo), "+v"(xo));   // keep no derived address in registers
#pragma unroll
                for (int r = 0; r < RZ; ++r) {
                    const int row = zo - zb + r, z = zo + r;
                    if (row >= H && row < EZ - H && z < a.nz) {
                        Pack<float, 4> p;
#pragma unroll
                        for (int v = 0; v < 4; ++v) p.v[v] = u[r][v];
                        if (stream)
                            stp_stream<float, 4>(dst + (size_t)z * a.px + xo, p);
                        else
                            stp<float, 4>(dst + (size_t)z * a.px + xo, p);
                    }
                }
            }
        };
        if (a.keep1 != nullptr) store(a.keep1, A);
        if (a.keep0 != nullptr) store(a.keep0, B);

        // receiver rows of this thread (owned ones; in the adjoint, where the
        // residual enters, those of the halo too) and the source cell
        int rowbits = 0, srccell = -1;
        const bool rec_x = MODE == kAdj ? xin : own_x;
        if ((MODE == kAdj ? a.resid != nullptr : a.trace != nullptr) && rec_x) {
#pragma unroll
            for (int r = 0; r < RZ; ++r) {
                const int zr = z0 + r - a.rz0, row = RZ * lz + r;
                const bool mine = MODE == kAdj ? z0 + r < a.nz : row >= H && row < EZ - H;
                if (mine && zr >= 0 && zr % a.rdz == 0 && zr / a.rdz < a.rnz) rowbits |= 1 << r;
            }
        }
        if (MODE != kAdj && a.sx >= x0 && a.sx < x0 + 4 && a.sz >= z0 && a.sz < z0 + RZ)
            srccell = 4 * (a.sz - z0) + a.sx - x0;

        // step s (0 <= s < S) from u in `src` and o (two levels back); the new
        // level replaces o and goes to `dst`
        auto step = [&](int s, const float *src, float *dst, const float (&u)[RZ][4], float (&o)[RZ][4], bool pair, bool sync = true) {
            if (sync) __syncthreads();
            const int lo = 4 * (s + 1);
            if (!(RZ * lz + RZ > lo && RZ * lz < EZ - lo)) return;
            float lzz[RZ][4];
            {
                float q[RZ + 8][4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const Pack<float, 4> p = ldp<float, 4>(src + lbase + (k - 4) * EX);
                    const Pack<float, 4> w = ldp<float, 4>(src + lbase + (RZ + k) * EX);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        q[k][v] = p.v[v];
                        q[RZ + 4 + k][v] = w.v[v];
                    }
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    float in[RZ + 8], out[RZ];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        in[r] = q[r][v];
                        in[RZ + 4 + r] = q[RZ + 4 + r][v];
                    }
#pragma unroll
                    for (int r = 0; r < RZ; ++r) in[r + 4] = u[r][v];
                    axis_d2_run<RZ>(in, out);
#pragma unroll
                    for (int r = 0; r < RZ; ++r) lzz[r][v] = out[r];
                }
            }
#pragma unroll
            for (int r = 0; r < RZ; ++r) {
                const Pack<float, 4> pl = ldp<float, 4>(src + lbase + r * EX - 4);
                const Pack<float, 4> pr = ldp<float, 4>(src + lbase + r * EX + 4);
                float in[12], lxx[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    in[v] = pl.v[v];
                    in[4 + v] = u[r][v];
                    in[8 + v] = pr.v[v];
                }
                axis_d2_run<4>(in, lxx);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    lzz[r][v] = lzz[r][v] + lxx[v];
                    o[r][v] = leapfrog(gz[r] * gx[v], u[r][v], C[r][v], lzz[r][v], o[r][v]);
                }
            }
            int zo = z0, xo = x0;
            asm volatile("" : "+v"(zo), "+v"(xo));   // keep no derived index in registers
            if (rowbits != 0) {
#pragma unroll
                for (int r = 0; r < RZ; ++r) {
                    if ((rowbits >> r) & 1) {
                        const int rrow = (zo + r - a.rz0) / a.rdz;
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int xr = xo + v - a.rx0;
                            if (xo + v < a.nx && xr >= 0 && xr % a.rdx == 0 && xr / a.rdx < a.rnx) {
                                const size_t at_r = (size_t)rrow * a.rnx + xr / a.rdx;
                                if constexpr (MODE == kAdj)
                                    o[r][v] = fmaf(C[r][v] * (gz[r] * gx[v]), a.resid[s * a.rec_stride + at_r], o[r][v]);
                                else
                                    a.trace[s * a.rec_stride + at_r] = o[r][v];
                            }
                        }
                    }
                }
            }
            if (MODE != kAdj && srccell >= 0) {
                const float inj = a.n + s + 1 < a.nt ? a.amp * a.wavelet[a.n + s + 1] : 0.0f;
                int sc = srccell;
                asm volatile("" : "+v"(sc));
#pragma unroll
                for (int r = 0; r < RZ; ++r)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (sc == 4 * r + v) o[r][v] += inj;
            }
            if (edge) mask(o);
            if (s + 1 < S) put(dst, o);
            if constexpr (MODE == kFwdLap) {
                if (edge) mask(lzz);
                store(a.hist + s * a.hist_stride, lzz, true);
            }
            if constexpr (MODE == kFwdKeep) store(a.hist + s * a.hist_stride, o);
            if constexpr (MODE == kAdj) {
                // the gradient's FP64 sum: one pass over it for two steps (or
                // the last one alone), each cell's terms in the order of the
                // steps.  (Held in registers for all S steps, which 3 rows a
                // thread leave room for, it measured slower: 37 us a step
                // for 8 x 1024^2 against 33.)
                if ((pair || s + 1 == S) && own_x) {
#pragma unroll
                    for (int r = 0; r < RZ; ++r) {
                        const int row = zo - zb + r, z = zo + r;
                        if (row >= H && row < EZ - H && z < a.nz) {
                            const size_t e = (size_t)z * a.px + xo;
                            const float *h = a.hist + s * a.hist_stride + e;
                            Pack<double, 4> g = ldp<double, 4>(a.g + e);
                            const Pack<float, 4> h1 = ldp_stream<float, 4>(h);
                            if (pair) {
                                const Pack<float, 4> h2 = ldp_stream<float, 4>(h - a.hist_stride);
#pragma unroll
                                for (int v = 0; v < 4; ++v) g.v[v] = fma((double)u[r][v], (double)h2.v[v], g.v[v]);
                            }
#pragma unroll
                            for (int v = 0; v < 4; ++v) g.v[v] = fma((double)o[r][v], (double)h1.v[v], g.v[v]);
                            stp<double, 4>(a.g + e, g);
                        }
                    }
                }
            }
        };

        const int tn = t + stride, in = tn < tend ? item_of(tn) : 0;
        int s = 0;
        for (; s + 2 < S; s += 2) {
            step(s, buf0, buf1, A, B, false);
            step(s + 1, buf1, buf0, B, A, true);
        }
        if (s + 1 < S) {
            step(s, buf0, buf1, A, B, false);
            // the last step reads buf1 and writes no buffer: the next tile's P
            // goes to buf0 meanwhile (every wave is past reading it)
            __syncthreads();
            if (tn < tend) fetch(tn, in, buf0);
            step(s + 1, buf1, buf0, B, A, true, false);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the copy of P, before the stores below
            store(a.out1, A);
            store(a.out0, B);
        } else {
            if (s < S) step(s, buf0, buf1, A, B, false);
            __syncthreads();
            if (tn < tend) {
                fetch(tn, in, buf0);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            if (s < S) {
                store(a.out1, B);
                store(a.out0, A);
            } else {   // no step: the levels pass through
                store(a.out1, A);
                store(a.out0, B);
            }
        }
        if (tn >= tend) return;
        t = tn;
        it = in;
    }
}

// --------------------------------------------------------------------------
// Host: tile shapes, their choice and the launch
// --------------------------------------------------------------------------
namespace {

// The tile shapes, with what a launch of them costs in us (least squares of the
// relative error over 1 to 10 steps on 17 grids and surveys of 200 x 170 to 12 x
// 700 x 1500, 8% rms, 14% for the 128 x 128 recompute and adjoint; the timed
// launches are in profiles/multi_step_costs.csv):
// per round of blocks and tile `tile` + `step` for every step, in proportion
// to the rows that still take part, + `odd` from the second round on when an
// odd number of steps leaves no buffer to copy the next tile into.  Rows:
// kFwd; kFwdLap and kFwdKeep; kAdj.
struct Cost {
    double tile, step, odd;
};
struct Shape {
    int ex, ez;        // ext tile
    int slack;         // rows a wave covers: it takes part while one is valid
    Cost cost[3];
};
constexpr int kShapes = 4;
constexpr Shape kShape[kShapes] = {
    {64, 64, 4, {{1.55, 0.93, 0.5}, {1.95, 1.16, 0.3}, {3.1, 1.24, 0.5}}},
    {96, 96, 8, {{3.4, 1.79, 0.7}, {4.6, 1.98, 1.5}, {8.7, 2.31, 1.8}}},
    {128, 96, 6, {{4.3, 1.91, 1.0}, {6.2, 2.29, 2.2}, {11.8, 2.44, 4.3}}},
    {128, 128, 8, {{6.2, 2.34, 1.8}, {8.8, 2.79, 3.1}, {18.1, 3.17, 7.1}}},
};
constexpr double kLaunchUs = 2.5;

int device_cus()
{
    static const int cus = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            n = 256;
        (void)hipGetLastError();
        return n >= 8 ? n : 8;
    }();
    return cus;
}

int64_t tiles_of(const Shape &sh, int nz, int px, int steps, int *tiles_x)
{
    const int ix = sh.ex - 8 * steps, iz = sh.ez - 8 * steps;
    const int tx = (px + ix - 1) / ix;
    if (tiles_x) *tiles_x = tx;
    return (int64_t)tx * ((nz + iz - 1) / iz);
}

template <int MODE, int N>
void launch_shape(const MultiBatch<N> &b, int shape, hipStream_t s)
{
    // whole eighths of the device (see the walk over the tiles in the kernel)
    const int per = (b.total + 7) / 8, cus8 = device_cus() / 8;
    auto go = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(8 * std::min(per, cus8)), dim3(threads), 0, s, b);
    };
    switch (shape) {
    case 0: go(k_multi2d<16, 1, 64, MODE, 4, N>, 1024); break;
    case 1: go(k_multi2d<24, 3, 32, MODE, 3, N>, 768); break;
    case 2: go(k_multi2d<32, 3, 32, MODE, 4, N>, 1024); break;
    default: go(k_multi2d<32, 4, 32, MODE, 4, N>, 1024); break;
    }
}

template <int N>
hipError_t launch_items(const MultiArgs *items, int count, int mode, int shape, hipStream_t s)
{
    MultiBatch<N> b;
    int64_t total = 0;
    for (int i = 0; i < count; ++i) {
        b.it[i] = items[i];
        b.begin[i] = (int32_t)total;
        total += tiles_of(kShape[shape], items[i].nz, items[i].px, items[i].steps, &b.it[i].tiles_x);
    }
    if (total == 0) return hipSuccess;
    if (total > INT32_MAX) return hipErrorInvalidValue;
    b.begin[count] = (int32_t)total;
    b.total = (int32_t)total;
    b.count = count;
    switch (mode) {
    case kFwd: launch_shape<kFwd>(b, shape, s); break;
    case kFwdLap: launch_shape<kFwdLap>(b, shape, s); break;
    case kFwdKeep: launch_shape<kFwdKeep>(b, shape, s); break;
    default: launch_shape<kAdj>(b, shape, s); break;
    }
    return hipGetLastError();
}

}  // namespace

int multi2d_shape(const MultiGrid *grids, int count, int steps, int mode, double *us)
{
    int best = -1;
    double best_us = 0.0;
    for (int k = 0; k < kShapes; ++k) {
        const Shape &sh = kShape[k];
        const Cost &c = sh.cost[mode == kAdj ? 2 : mode == kFwd ? 0 : 1];
        if (sh.ez - 8 * steps < 16) continue;   // an inner tile of at least 16 rows
        int64_t tiles = 0;
        for (int i = 0; i < count; ++i) tiles += tiles_of(sh, grids[i].nz, grids[i].px, steps, nullptr);
        const int64_t blocks = device_cus() / 8 * 8, rounds = (tiles + blocks - 1) / blocks;
        double t = c.tile + ((steps & 1) && rounds > 1 ? c.odd : 0.0);
        for (int s = 1; s <= steps; ++s) t += c.step * std::min(1.0, (double)(sh.ez - 8 * s + sh.slack) / sh.ez);
        t = kLaunchUs + (double)rounds * t;
        if (best < 0 || t < best_us) {
            best = k;
            best_us = t;
        }
    }
    if (us) *us = best_us;
    return best;
}

hipError_t launch_multi2d(const MultiArgs *items, int count, int mode, hipStream_t s)
{
    if (count < 1 || count > kBatchMax) return hipErrorInvalidValue;
    MultiGrid g[kBatchMax];
    int steps = 0;
    for (int i = 0; i < count; ++i) {
        g[i] = MultiGrid{items[i].nz, items[i].px};
        steps = std::max(steps, items[i].steps);
    }
    const int shape = multi2d_shape(g, count, steps, mode, nullptr);
    if (shape < 0) return hipErrorInvalidValue;
    return count == 1 ? launch_items<1>(items, count, mode, shape, s)
                      : launch_items<kBatchMax>(items, count, mode, shape, s);
}

}  // namespace fdk

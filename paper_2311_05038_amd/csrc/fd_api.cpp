// C ABI of the finite-difference engine: validation, buffer layouts, handle
// management and kernel dispatch.  Declarations and semantics: include/fd.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../include/fd.h"
#include "fd_host.hpp"
#include "fd_launch.hpp"

using fdk::StepArgs;
using namespace fdh;

namespace {

fd_status hip_fail(hipError_t e, const char *what)
{
    return fail(FD_ERR_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

fd_status do_begin(const fd_model *m, fd_state *st, const fd_shot *s, hipStream_t stream)
{
    const Layout &L = m->L;
    hipError_t e = fdk::launch_fill_u32(st->base, L.state_least / 4, 0u, stream);
    if (e != hipSuccess) return hip_fail(e, "fd_begin_shot fill");
    // a z-slab adds the source only on its own planes
    if (s->src_z >= L.z0 && s->src_z < L.z0 + L.nz) {
        fd_shot local = *s;
        local.src_z -= L.z0;
        e = fdk::launch_begin(L.storage, st->buf[0], (int64_t)src_offset(L, &local), m->amp,
                              s->wavelet, s->nt, st->meta, stream);
        if (e != hipSuccess) return hip_fail(e, "fd_begin_shot");
    }
    st->next = 0;
    return FD_OK;
}

fd_status do_step(const fd_model *m, fd_state *st, const fd_shot *s, int64_t n, float *trace_row,
                  hipStream_t stream)
{
    int64_t skip = 0;
    StepArgs a = base_args(m, s, &skip);
    a.cur = st->buf[n & 1];
    a.prev = st->buf[(n + 1) & 1];
    a.n = n;
    a.trace_row = (nrec_of(s) > 0 && trace_row && skip >= 0) ? trace_row + skip : nullptr;
    a.meta = st->meta;
    a.zghost = is_slab(m->L) ? (int16_t)kGhost : (int16_t)0;
    hipError_t e = fdk::launch_step(a, m->L.ndim, m->L.storage, fdk::kFwd, stream);
    if (e != hipSuccess) return hip_fail(e, "step kernel launch");
    st->next = n + 1;
    return FD_OK;
}

// ---- several 2D FP32 steps per launch --------------------------------------

// How a run of steps is cut into launches of several steps each: `steps` at
// most per launch, for the least modelled time over the run.
struct MultiPlan {
    int steps;   // 0: no shape fits, or single steps are not slower
    double us;   // the run's modelled time
    bool lone;   // (adjoint) one step of the run as a launch of its own
};

// A single step's time on `cells` padded cells, us (256^2 3.4, 1024^2 5.5,
// 2048 x 4096 22.7): the launch, or the fields' 16 bytes per cell.
double single_us(double cells) { return 3.2 + cells * 2.35e-6; }
// The same of an adjoint step, which also reads the history and reads and
// writes the FP64 sum, over cells covered by its 128-wide tiles: 256^2 4.0,
// 1024^2 7.5, 2000^2 20.0, 8 x 1024^2 38.5 with one history field, and more
// once many of them pass through the cache (28 bytes a cell besides).
double single_adjoint_us(double cells) { return 4.6 + cells * (cells <= 9.0e6 ? 5.5e-6 : 6.6e-6); }

// Cells whose two pairs of levels and c, 20 bytes a cell, stay in the 256 MB
// Infinity Cache from one launch to the next.  A launch on more reads HBM and
// takes 1.00 (16 shots of 1024^2) to 1.14 (2 of 2048 x 4096) of its modelled
// time; kOutOfCache is the value that chose best over both and the mixes below.
constexpr double kGroupCells = 13.0e6;
constexpr double kOutOfCache = 1.08;

// pairs: launches come in pairs that start and end on the same buffers, so a
// run is cut into whole pairs of `steps` and a rest of one pair (or of one or
// two single steps).  Otherwise launches follow one another freely, as equal
// as they can be; in the adjoint, where a lone step is the single step
// kernel's, one may be split off if that is clearly less (5 steps of 2000^2:
// 4 + 1 87 us, 2 + 3 115).
MultiPlan plan_multi(const fdk::MultiGrid *grids, int count, int64_t run, int mode, bool pairs)
{
    double cells = 0.0, covered = 0.0;
    for (int i = 0; i < count; ++i) {
        cells += (double)grids[i].nz * grids[i].px;
        covered += (double)grids[i].nz * ((grids[i].px + 127) / 128 * 128);
    }
    double us[fdk::kMultiSteps + 1] = {0.0};
    for (int k = 1; k <= fdk::kMultiSteps; ++k) {
        if (fdk::multi2d_shape(grids, count, k, mode, &us[k]) < 0) us[k] = 1e300;
        // beyond the cache a launch of few steps is bound by its 24 bytes a
        // cell (a shot of three steps on 3000 x 5000: 162 us as 2 + 1, 145 as
        // single steps)
        if (cells > kGroupCells) us[k] = std::max(us[k], 2.5 + cells * 3.8e-6);
    }
    if (mode == fdk::kAdj) us[1] = single_adjoint_us(covered);
    auto equal = [&](int64_t m, int k) {
        const int64_t n = (m + k - 1) / k;
        return m == 0 ? 0.0 : (double)n * us[(m + n - 1) / n];
    };
    MultiPlan best{0, pairs ? (double)run * single_us(cells) : 1e300, false};
    for (int k = 1; k <= fdk::kMultiSteps && k <= run; ++k) {
        double t;
        if (pairs) {
            const int64_t rest = run % (2 * k);
            t = (double)(run / (2 * k)) * 2.0 * us[k];
            t += rest <= 2 ? (double)rest * single_us(cells) : us[(rest + 1) / 2] + us[rest / 2];
        } else {
            t = equal(run, k);
        }
        if (t < best.us) best = MultiPlan{k, t, false};
    }
    if (mode == fdk::kAdj)
        for (int k = 2; k <= fdk::kMultiSteps && k < run; ++k) {
            const double t = equal(run - 1, k) + us[1];
            if (t < (best.lone ? 1.0 : 0.9) * best.us) best = MultiPlan{k, t, true};
        }
    return best;
}

fdk::MultiArgs multi_args(const fd_model *m, const fd_shot *s, int64_t n, int steps)
{
    const StepArgs a = base_args(m, s);
    fdk::MultiArgs o{};
    o.c = a.c;
    o.gz = a.gz;
    o.gx = a.gx;
    o.wavelet = a.wavelet;
    o.nz = a.nz;
    o.nx = a.nx;
    o.px = a.px;
    o.sz = a.sz;
    o.sx = a.sx;
    o.amp = a.amp;
    o.n = n;
    o.nt = a.nt;
    o.rz0 = a.rec.z0;
    o.rx0 = a.rec.x0;
    o.rnz = a.rec.nz;
    o.rnx = a.rec.nx;
    o.rdz = a.rec.dz;
    o.rdx = a.rec.dx;
    o.rec_stride = nrec_of(s);
    o.steps = steps;
    return o;
}

// A shot in flight: up to FD_BATCH_MAX of them advance together.
struct Flight {
    const fd_model *m;
    fd_state *st;
    const fd_shot *shot;
    int64_t n, end;   // next step, step to stop at
    float *traces;    // [nt][nrec] or null
    float *keep;      // where the levels at step n go (a checkpoint slot), or null
};

fd_status keep_levels(const Flight &f, hipStream_t s)
{
    const size_t bytes = f.m->L.field;
    hipError_t e = hipMemcpyAsync(f.keep, f.st->buf[f.n & 1], bytes, hipMemcpyDeviceToDevice, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync((char *)f.keep + bytes, f.st->buf[(f.n + 1) & 1], bytes, hipMemcpyDeviceToDevice, s);
    return e == hipSuccess ? FD_OK : hip_fail(e, "checkpoint copy");
}

// Steps every flight to its end.  Launches of several steps come in pairs:
// the first writes the state's second pair of levels, the next one writes
// back, so that after a pair (and so after every call) level n is in
// buf[n & 1] again, as single steps leave it.  Same bits either way.
fd_status advance_group(Flight *f, int count, hipStream_t s)
{
    int64_t run = 0;
    bool paired = true;
    for (int i = 0; i < count; ++i) {
        run = std::max(run, f[i].end - f[i].n);
        paired = paired && f[i].st->pair[0] != nullptr;
    }
    int running = 0, steps = 0;
    while (run > 0) {
        // planned anew when shots have ended, for those that still run
        fdk::MultiGrid grids[FD_BATCH_MAX];
        int now = 0;
        for (int i = 0; i < count; ++i)
            if (f[i].n < f[i].end) grids[now++] = fdk::MultiGrid{(int)f[i].m->L.nz, f[i].m->L.px};
        if (now != running) {
            running = now;
            steps = paired && run > 2 ? plan_multi(grids, now, run, fdk::kFwd, true).steps : 0;
        }
        if (steps > 0 && run > 2) {
            for (int half = 0; half < 2; ++half) {
                fdk::MultiArgs it[FD_BATCH_MAX];
                int k = 0;
                for (int i = 0; i < count; ++i) {
                    const int64_t r = std::min<int64_t>(f[i].end - f[i].n, 2 * steps);
                    if (r <= 0) continue;
                    // the second half takes the smaller part of what is left
                    const int64_t first = (r + 1) / 2, nf = half == 0 ? f[i].n : f[i].n + first;
                    fdk::MultiArgs a = multi_args(f[i].m, f[i].shot, nf, (int)(half == 0 ? first : r - first));
                    float *b[2] = {(float *)f[i].st->buf[0], (float *)f[i].st->buf[1]};
                    if (half == 0) {
                        a.cur = b[nf & 1];
                        a.prev = b[(nf + 1) & 1];
                        a.out1 = f[i].st->pair[0];
                        a.out0 = f[i].st->pair[1];
                        if (f[i].keep) {
                            a.keep1 = f[i].keep;
                            a.keep0 = (float *)((char *)f[i].keep + f[i].m->L.field);
                        }
                    } else {
                        a.cur = f[i].st->pair[0];
                        a.prev = f[i].st->pair[1];
                        a.out1 = b[(f[i].n + r) & 1];
                        a.out0 = b[(f[i].n + r + 1) & 1];
                    }
                    if (f[i].traces && nrec_of(f[i].shot) > 0)
                        a.trace = f[i].traces + (size_t)nf * (size_t)nrec_of(f[i].shot);
                    it[k++] = a;
                }
                const hipError_t e = fdk::launch_multi2d(it, k, fdk::kFwd, s);
                if (e != hipSuccess) return hip_fail(e, "multi-step launch");
            }
            for (int i = 0; i < count; ++i) {
                const int64_t r = std::min<int64_t>(f[i].end - f[i].n, 2 * steps);
                if (r <= 0) continue;
                f[i].n += r;
                f[i].keep = nullptr;
                f[i].st->next = f[i].n;
            }
            run -= 2 * steps;
        } else {
            fdk::Batch2D b;
            b.count = 0;
            for (int i = 0; i < count; ++i) {
                if (f[i].n >= f[i].end) continue;
                if (f[i].keep) {
                    const fd_status st = keep_levels(f[i], s);
                    if (st != FD_OK) return st;
                    f[i].keep = nullptr;
                }
                if (count == 1) {
                    const int64_t nrec = nrec_of(f[i].shot);
                    const fd_status st = do_step(f[i].m, f[i].st, f[i].shot, f[i].n,
                                                 f[i].traces ? f[i].traces + (size_t)f[i].n * (size_t)nrec : nullptr, s);
                    if (st != FD_OK) return st;
                } else {
                    StepArgs a = base_args(f[i].m, f[i].shot);
                    a.cur = f[i].st->buf[f[i].n & 1];
                    a.prev = f[i].st->buf[(f[i].n + 1) & 1];
                    a.n = f[i].n;
                    const int64_t nrec = nrec_of(f[i].shot);
                    a.trace_row = (f[i].traces && nrec > 0) ? f[i].traces + (size_t)f[i].n * (size_t)nrec : nullptr;
                    a.meta = f[i].st->meta;
                    b.it[b.count++] = a;
                }
            }
            if (count > 1) {
                const hipError_t e = fdk::launch_step_batch2d(b, fdk::kFwd, s);
                if (e != hipSuccess) return hip_fail(e, "batched step launch");
            }
            for (int i = 0; i < count; ++i)
                if (f[i].n < f[i].end) f[i].st->next = ++f[i].n;
            run -= 1;
        }
    }
    return FD_OK;
}

// advance_group on all flights together or on consecutive groups of about
// equal shares within kGroupCells, whichever is modelled faster: groups stay
// in the cache, one launch leaves fewer blocks idle in its last round of
// tiles.  Together and in groups, ms: 12 mixed shots of 0.3 to 8 M cells
// 7.94, 8.31; 12 of 1448^2 6.22, 5.80; 2 of 2048 x 4096 4.12, 3.68; 12 of
// them 11.0, 11.2.
fd_status advance_alike(Flight *f, int count, hipStream_t s)
{
    fdk::MultiGrid grids[FD_BATCH_MAX];
    double total = 0.0;
    int64_t run = 0;
    for (int i = 0; i < count; ++i) {
        const Layout &L = f[i].m->L;
        grids[i] = fdk::MultiGrid{(int)L.nz, L.px};
        total += (double)L.npad;
        run = std::max(run, f[i].end - f[i].n);
    }
    int first[FD_BATCH_MAX + 1] = {0}, groups = 0;
    if (total > kGroupCells && count > 1 && run > 2) {
        const double share = total / std::ceil(total / kGroupCells);
        double grouped = 0.0;
        for (int i = 0; i < count; first[++groups] = i) {
            const int i0 = i;
            double sum = (double)f[i++].m->L.npad;
            while (i < count && sum + 0.5 * (double)f[i].m->L.npad <= share && sum + (double)f[i].m->L.npad <= kGroupCells)
                sum += (double)f[i++].m->L.npad;
            const MultiPlan part = plan_multi(grids + i0, i - i0, run, fdk::kFwd, true);
            grouped += part.us * (part.steps > 0 && sum > kGroupCells ? kOutOfCache : 1.0);
        }
        const MultiPlan whole = plan_multi(grids, count, run, fdk::kFwd, true);
        if (whole.us * (whole.steps > 0 ? kOutOfCache : 1.0) <= grouped) groups = 0;
    }
    if (groups == 0) first[groups = 1] = count;
    for (int g = 0; g < groups; ++g) {
        const fd_status st = advance_group(f + first[g], first[g + 1] - first[g], s);
        if (st != FD_OK) return st;
    }
    return FD_OK;
}

// The shots that still run: those with a second pair of levels, then those
// without, since one that has none must not make the others of a call take
// single steps.  (Where all take single steps, they share the launches.)
fd_status advance(Flight *f, int count, hipStream_t s)
{
    int64_t run = 0;
    for (int i = 0; i < count; ++i) run = std::max(run, f[i].end - f[i].n);
    for (const bool with : {true, false}) {
        Flight g[FD_BATCH_MAX];
        int at[FD_BATCH_MAX], k = 0;
        for (int i = 0; i < count; ++i)
            if (f[i].n < f[i].end && (run <= 2 || (f[i].st->pair[0] != nullptr) == with)) {
                at[k] = i;
                g[k++] = f[i];
            }
        if (k == 0) continue;
        const fd_status st = advance_alike(g, k, s);
        for (int j = 0; j < k; ++j) f[at[j]] = g[j];
        if (st != FD_OK) return st;
    }
    return FD_OK;
}

// Shots of one 2D FP32 model after do_begin: steps 0 .. nt-1 with the
// checkpoints before steps 0, K, 2K, ... (ckpt may be null) and the traces.
fd_status run_steps(const fd_model *m, fd_state *const *states, const fd_shot *const *shots, int32_t count,
                    float *const *traces, void *const *ckpt, int32_t every, hipStream_t s)
{
    const int64_t nt = shots[0]->nt;
    bool any = false;
    for (int32_t i = 0; ckpt && i < count; ++i) any = any || ckpt[i];
    const int64_t stride = any ? every : nt;
    for (int64_t n = 0; n < nt; n += stride) {
        for (int32_t i0 = 0; i0 < count; i0 += FD_BATCH_MAX) {
            Flight f[FD_BATCH_MAX];
            int k = 0;
            for (int32_t i = i0; i < std::min<int32_t>(count, i0 + FD_BATCH_MAX); ++i) {
                char *slot = ckpt ? (char *)ckpt[i] : nullptr;
                if (slot) slot += (size_t)(n / stride) * ckpt_slot_bytes(m->L);
                f[k++] = Flight{m, states[i], shots[i], n, std::min(nt, n + stride), traces ? traces[i] : nullptr,
                                (float *)slot};
            }
            const fd_status st = advance(f, k, s);
            if (st != FD_OK) return st;
        }
    }
    return FD_OK;
}

// The same for one shot of any model.
fd_status shot_steps(const fd_model *m, fd_state *st, const fd_shot *shot, float *traces, void *ckpt,
                     int32_t every, hipStream_t s)
{
    const Layout &L = m->L;
    if (L.ndim == 2 && L.storage == FD_F32) return run_steps(m, &st, &shot, 1, &traces, &ckpt, every, s);
    const int64_t nrec = nrec_of(shot);
    for (int64_t n = 0; n < shot->nt; ++n) {
        if (ckpt && n % every == 0) {
            char *slot = (char *)ckpt + (size_t)(n / every) * ckpt_slot_bytes(L);
            const fd_status e = keep_levels(Flight{m, st, shot, n, shot->nt, nullptr, (float *)slot}, s);
            if (e != FD_OK) return e;
        }
        const fd_status e = do_step(m, st, shot, n, traces ? traces + (size_t)n * (size_t)nrec : nullptr, s);
        if (e != FD_OK) return e;
    }
    return FD_OK;
}

}  // namespace

extern "C" {

const char *fd_last_error(void) { return last_error(); }

const char *fd_version(void) { return "fd-mi355x 0.1 (gfx950, radius 4)"; }

fd_status fd_query_bytes(const fd_grid *grid, int64_t nt, int32_t ckpt_every, fd_sizes *out)
{
    fd_status st = check_grid(grid);
    if (st != FD_OK) return st;
    if (!out) return fail(FD_ERR_INVALID_ARG, "out is NULL");
    if (nt < 0 || ckpt_every < 0) return fail(FD_ERR_INVALID_ARG, "nt and ckpt_every must be >= 0");
    const Layout L = make_layout(*grid);
    out->model = L.model_bytes;
    out->state = L.state_bytes;
    const bool whole = !is_slab(L);  // slabs step one call at a time only
    out->checkpoints = (whole && nt > 0 && ckpt_every > 0) ? (size_t)n_ckpt(nt, ckpt_every) * ckpt_slot_bytes(L) : 0;
    out->adjoint_work = (whole && ckpt_every > 0) ? adjoint_work_bytes(L, ckpt_every) : 0;
    out->routines_work = whole ? (size_t)L.ndim * L.f32field : 0;
    return ok();
}

fd_status fd_create_model(const fd_grid *grid, const float *velocity, void *model_buf,
                          size_t model_bytes, void *stream, fd_model **out)
{
    fd_status st = check_grid(grid);
    if (st != FD_OK) return st;
    if (!velocity || !model_buf || !out) return fail(FD_ERR_INVALID_ARG, "NULL velocity, buffer or out");
    const Layout L = make_layout(*grid);
    if (model_bytes < L.model_bytes)
        return fail(FD_ERR_INVALID_ARG, "model buffer too small (%zu < %zu bytes)", model_bytes, L.model_bytes);
    if ((uintptr_t)model_buf % kAlign) return fail(FD_ERR_INVALID_ARG, "model buffer must be 256-byte aligned");

    fd_model *m = new (std::nothrow) fd_model;
    if (!m) return fail(FD_ERR_OUT_OF_MEMORY, "host allocation failed");
    m->grid = *grid;
    if (m->grid.sponge_width > 0 && !(m->grid.sponge_alpha > 0.0))
        m->grid.sponge_alpha = 0.3 / m->grid.sponge_width;
    m->L = L;
    char *base = (char *)model_buf;
    const bool fixed16 = L.c_storage == FD_C_FIXED16;
    m->c = fixed16 ? nullptr : (float *)(base + L.c_off);
    m->c16 = fixed16 ? (uint16_t *)(base + L.c_off) : nullptr;
    m->c16_scale = 1.0f;
    m->c16_inv = 1.0f;
    m->gz = (float *)(base + L.gz_off);
    m->gy = (float *)(base + L.gy_off);
    m->gx = (float *)(base + L.gx_off);
    m->scratch = (uint32_t *)(base + L.scratch_off);
    m->amp = source_amp(*grid);

    // Damping profiles, FP64 on the host, stored FP32; a z-slab takes its
    // planes' factors from the whole grid's profile.
    const double alpha = m->grid.sponge_alpha;
    const int32_t W = m->grid.sponge_width;
    const uint32_t f = m->grid.sponge_faces;
    const std::vector<float> gzg = damping_profile(L.nzg, W, alpha, f & FD_FACE_ZLO, f & FD_FACE_ZHI);
    const std::vector<float> gz(gzg.begin() + L.z0, gzg.begin() + L.z0 + L.nz);
    const std::vector<float> gy = grid->ndim == 3 ? damping_profile(L.ny, W, alpha, f & FD_FACE_YLO, f & FD_FACE_YHI)
                                                  : std::vector<float>(1, 1.0f);
    const std::vector<float> gx = damping_profile(L.nx, W, alpha, f & FD_FACE_XLO, f & FD_FACE_XHI);

    hipStream_t s = (hipStream_t)stream;
    uint32_t host_scratch[2] = {0, 0};
    hipError_t e = hipMemcpyAsync(m->gz, gz.data(), gz.size() * 4, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(m->gy, gy.data(), gy.size() * 4, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(m->gx, gx.data(), gx.size() * 4, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = fdk::launch_fill_u32((uint32_t *)(base + L.c_off), L.cfield / 4, 0u, s);
    if (e == hipSuccess) e = fdk::launch_fill_u32(m->scratch, 2, 0u, s);
    // FP32 c, or (16-bit c) only the velocity range: the fixed-point scale
    // depends on the largest c
    if (e == hipSuccess)
        e = fdk::launch_model_c(velocity, m->c, L.nz * L.ny, (int32_t)L.nx, L.px,
                                grid->dt / grid->dh, m->scratch, s);
    if (e == hipSuccess) e = hipMemcpyAsync(host_scratch, m->scratch, 8, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        delete m;
        return hip_fail(e, "fd_create_model");
    }
    if (host_scratch[1]) {
        delete m;
        return fail(FD_ERR_INVALID_ARG, "velocity must be positive and finite everywhere");
    }
    float vmax;
    std::memcpy(&vmax, &host_scratch[0], 4);
    st = check_stability(*grid, vmax);
    if (st != FD_OK) {
        delete m;
        return st;
    }
    if (fixed16) {
        const int ex = c16_exponent(vmax, grid->dt / grid->dh);
        m->c16_scale = std::ldexp(1.0f, ex - 16);
        m->c16_inv = std::ldexp(1.0f, 16 - ex);
        e = fdk::launch_model_c16(velocity, m->c16, L.nz * L.ny, (int32_t)L.nx, L.px,
                                  grid->dt / grid->dh, std::ldexp(1.0f, 16 - ex), s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) {
            delete m;
            return hip_fail(e, "fd_create_model");
        }
    }
    // Settle, outside any stream capture, what later launches on this device
    // look up once and cache: the device address of the static routine work
    // area of fd_step_routines_noalloc, and the 3D launch plan's occupancy.
    // A failure here is left to the calls that need them, which report it.
    {
        void *area = nullptr;
        (void)fdk::routines_scratch(s, &area);
        StepArgs a = base_args(m, nullptr, nullptr);
        fdk::plan_tiles(a, L.ndim, L.storage, fdk::kFwd);
        const fdk::MultiGrid mg{(int)L.nz, L.px};
        if (L.ndim == 2) (void)fdk::multi2d_shape(&mg, 1, 1, fdk::kFwd, nullptr);   // the CU count
        (void)hipGetLastError();
    }
    *out = m;
    return ok();
}

fd_status fd_destroy_model(fd_model *model)
{
    delete model;
    return ok();
}

fd_status fd_create_state(const fd_model *model, void *state_buf, size_t state_bytes, fd_state **out)
{
    if (!model || !state_buf || !out) return fail(FD_ERR_INVALID_ARG, "NULL model, buffer or out");
    if (state_bytes < model->L.state_least)
        return fail(FD_ERR_INVALID_ARG, "state buffer too small (%zu < %zu bytes)", state_bytes,
                    model->L.state_least);
    if ((uintptr_t)state_buf % kAlign) return fail(FD_ERR_INVALID_ARG, "state buffer must be 256-byte aligned");
    fd_state *st = new (std::nothrow) fd_state;
    if (!st) return fail(FD_ERR_OUT_OF_MEMORY, "host allocation failed");
    st->m = model;
    st->base = state_buf;
    st->buf[0] = (char *)state_buf + model->L.ghost;
    st->buf[1] = (char *)state_buf + model->L.field + model->L.ghost;
    const bool paired = model->L.pair_off != 0 && state_bytes >= model->L.state_bytes;
    for (int k = 0; k < 2; ++k)
        st->pair[k] = paired ? (float *)((char *)state_buf + model->L.pair_off + k * model->L.field) : nullptr;
    st->meta = (int32_t *)((char *)state_buf + model->L.meta_off);
    st->next = -1;
    *out = st;
    return ok();
}

fd_status fd_destroy_state(fd_state *state)
{
    delete state;
    return ok();
}

fd_status fd_begin_shot(const fd_model *model, fd_state *state, const fd_shot *shot, void *stream)
{
    if (!model || !state) return fail(FD_ERR_INVALID_ARG, "NULL model or state");
    if (state->m != model) return fail(FD_ERR_INVALID_ARG, "state was created for another model");
    fd_status st = check_shot(model, shot);
    if (st != FD_OK) return st;
    st = do_begin(model, state, shot, (hipStream_t)stream);
    return st == FD_OK ? ok() : st;
}

fd_status fd_step(const fd_model *model, fd_state *state, const fd_shot *shot, int64_t n,
                  float *trace_row, void *stream)
{
    if (!model || !state) return fail(FD_ERR_INVALID_ARG, "NULL model or state");
    if (state->m != model) return fail(FD_ERR_INVALID_ARG, "state was created for another model");
    fd_status st = check_shot(model, shot);
    if (st != FD_OK) return st;
    if (state->next < 0) return fail(FD_ERR_INVALID_ARG, "fd_begin_shot has not been called");
    if (n != state->next) return fail(FD_ERR_INVALID_ARG, "step %lld requested, next step is %lld",
                                      (long long)n, (long long)state->next);
    if (n >= shot->nt) return fail(FD_ERR_INVALID_ARG, "step %lld beyond the shot's %lld steps",
                                   (long long)n, (long long)shot->nt);
    st = do_step(model, state, shot, n, trace_row, (hipStream_t)stream);
    return st == FD_OK ? ok() : st;
}

fd_status fd_run_shot(const fd_model *model, fd_state *state, const fd_shot *shot, float *traces,
                      void *ckpt, size_t ckpt_bytes, int32_t ckpt_every, void *stream)
{
    if (!model || !state) return fail(FD_ERR_INVALID_ARG, "NULL model or state");
    if (state->m != model) return fail(FD_ERR_INVALID_ARG, "state was created for another model");
    fd_status st = check_shot(model, shot);
    if (st != FD_OK) return st;
    const Layout &L = model->L;
    if (is_slab(L)) return fail(FD_ERR_UNSUPPORTED, "a z-slab steps with fd_step and fd_slab_exchange");
    if (ckpt) {
        if (ckpt_every < 1) return fail(FD_ERR_INVALID_ARG, "ckpt_every must be >= 1");
        const size_t need = (size_t)n_ckpt(shot->nt, ckpt_every) * ckpt_slot_bytes(L);
        if (ckpt_bytes < need)
            return fail(FD_ERR_INVALID_ARG, "checkpoint buffer too small (%zu < %zu bytes)", ckpt_bytes, need);
        if ((uintptr_t)ckpt % kAlign) return fail(FD_ERR_INVALID_ARG, "checkpoint buffer must be 256-byte aligned");
    }
    hipStream_t s = (hipStream_t)stream;
    st = do_begin(model, state, shot, s);
    if (st != FD_OK) return st;
    st = shot_steps(model, state, shot, traces, ckpt, ckpt_every, s);
    return st == FD_OK ? ok() : st;
}

struct fd_shot_graph {
    hipGraphExec_t exec;
    fd_state *state;
    int64_t nt;
};

fd_status fd_shot_graph_create(const fd_model *model, fd_state *state, const fd_shot *shot, float *traces,
                               fd_shot_graph **out)
{
    if (!model || !state || !out) return fail(FD_ERR_INVALID_ARG, "NULL model, state or output handle");
    *out = nullptr;
    if (state->m != model) return fail(FD_ERR_INVALID_ARG, "state was created for another model");
    fd_status st = check_shot(model, shot);
    if (st != FD_OK) return st;
    if (is_slab(model->L)) return fail(FD_ERR_UNSUPPORTED, "a z-slab steps with fd_step and fd_slab_exchange");
    fd_shot_graph *h = new (std::nothrow) fd_shot_graph{};
    if (!h) return fail(FD_ERR_OUT_OF_MEMORY, "cannot allocate the graph handle");
    const int64_t next_before = state->next;  // recording advances the host counter only
    {
        // the tile plan of a 3D step asks the runtime for the kernel's
        // occupancy once per storage kind; ask before the capture starts
        int64_t skip = 0;
        StepArgs a = base_args(model, shot, &skip);
        fdk::plan_tiles(a, model->L.ndim, model->L.storage, fdk::kFwd);
    }
    // The launches are recorded on a private stream (default priority) and
    // replayed on the caller's: the capture itself runs nothing.
    hipStream_t cs = nullptr;
    hipError_t e = hipStreamCreateWithFlags(&cs, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) {
        if (cs) (void)hipStreamDestroy(cs);
        delete h;
        return hip_fail(e, "graph capture start");
    }
    st = do_begin(model, state, shot, cs);
    if (st == FD_OK) st = shot_steps(model, state, shot, traces, nullptr, 0, cs);
    hipGraph_t g = nullptr;
    e = hipStreamEndCapture(cs, &g);  // ends the capture whether or not recording succeeded
    if (st == FD_OK && e == hipSuccess) e = hipGraphInstantiate(&h->exec, g, nullptr, nullptr, 0);
    if (g) (void)hipGraphDestroy(g);
    (void)hipStreamDestroy(cs);
    if (st == FD_OK && e != hipSuccess) st = hip_fail(e, "graph capture");
    state->next = next_before;  // nothing ran on the device
    if (st != FD_OK) {
        delete h;
        return st;
    }
    h->state = state;
    h->nt = shot->nt;
    *out = h;
    return ok();
}

fd_status fd_shot_graph_launch(fd_shot_graph *g, void *stream)
{
    if (!g) return fail(FD_ERR_INVALID_ARG, "NULL graph");
    const hipError_t e = hipGraphLaunch(g->exec, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "graph launch");
    g->state->next = g->nt;
    return ok();
}

fd_status fd_shot_graph_destroy(fd_shot_graph *g)
{
    if (g) (void)hipGraphExecDestroy(g->exec);
    delete g;
    return ok();
}

fd_status fd_run_shots(const fd_model *model, fd_state *const *states, const fd_shot *const *shots,
                       int32_t count, float *const *traces, void *const *ckpt, size_t ckpt_bytes,
                       int32_t ckpt_every, void *stream)
{
    if (!model) return fail(FD_ERR_INVALID_ARG, "NULL model");
    if (count < 1 || count > 4096) return fail(FD_ERR_INVALID_ARG, "count must be in [1, 4096]");
    if (!states || !shots) return fail(FD_ERR_INVALID_ARG, "NULL states or shots array");
    const Layout &L = model->L;
    if (is_slab(L)) return fail(FD_ERR_UNSUPPORTED, "a z-slab steps with fd_step and fd_slab_exchange");
    for (int32_t i = 0; i < count; ++i) {
        if (!states[i] || states[i]->m != model) return fail(FD_ERR_INVALID_ARG, "shot %d: state missing or of another model", i);
        fd_status st = check_shot(model, shots[i]);
        if (st != FD_OK) return st;
        if (shots[i]->nt != shots[0]->nt) return fail(FD_ERR_INVALID_ARG, "shot %d: all shots must share nt", i);
        for (int32_t j = 0; j < i; ++j)
            if (states[j] == states[i]) return fail(FD_ERR_INVALID_ARG, "shot %d repeats a state", i);
        if (ckpt && ckpt[i]) {
            if (ckpt_every < 1) return fail(FD_ERR_INVALID_ARG, "ckpt_every must be >= 1");
            const size_t need = (size_t)n_ckpt(shots[i]->nt, ckpt_every) * ckpt_slot_bytes(L);
            if (ckpt_bytes < need)
                return fail(FD_ERR_INVALID_ARG, "checkpoint buffer too small (%zu < %zu bytes)", ckpt_bytes, need);
            if ((uintptr_t)ckpt[i] % kAlign) return fail(FD_ERR_INVALID_ARG, "checkpoint buffer must be 256-byte aligned");
        }
    }
    hipStream_t s = (hipStream_t)stream;
    const bool batched = L.ndim == 2 && L.storage == FD_F32 && count > 1;
    if (!batched) {
        for (int32_t i = 0; i < count; ++i) {
            fd_status st = fd_run_shot(model, states[i], shots[i], traces ? traces[i] : nullptr,
                                       ckpt ? ckpt[i] : nullptr, ckpt_bytes, ckpt_every, stream);
            if (st != FD_OK) return st;
        }
        return ok();
    }
    for (int32_t i = 0; i < count; ++i) {
        fd_status st = do_begin(model, states[i], shots[i], s);
        if (st != FD_OK) return st;
    }
    const fd_status st = run_steps(model, states, shots, count, traces, ckpt, ckpt_every, s);
    return st == FD_OK ? ok() : st;
}

}  // extern "C"

namespace {

// Checkpointed backward pass shared by the gradient and the image, for
// `count` shots on one model: each segment is recomputed storing the
// history field of every step (L w^n for the gradient, w^n for the image),
// then the z-form adjoint field is stepped back through the segment
// accumulating sum_k z^k * hist^{k-1} in FP64, one sum per shot (acc[i],
// padded, inside work[i]).  In 2D a launch takes several steps of a group of
// shots; in 3D the shots' steps are launched one by one.
// Per shot and cell the arithmetic is the same either way.
struct ShotIO {
    const fd_shot *shot;
    const float *adj;
    const void *ckpt;
    void *work;
};

// The cut of `m` steps into `n` launches for the backward pass: at most `cap`
// steps each, the larger ones last; `even`: an even number of launches, or one.
struct Cut {
    int64_t m, n;
    Cut(int64_t steps, int cap, bool even) : m(steps), n((steps + cap - 1) / cap)
    {
        if (even && n > 1 && (n & 1)) ++n;
    }
    int steps(int64_t i) const { return (int)(m / n + (i >= n - m % n ? 1 : 0)); }
};

// Whether a first launch of the image's recompute, of k < 2 steps on `count`
// shots, is better done as copies of the checkpoints' P to the history (3.3 us
// each and 8 bytes a cell at 7 TB/s) and a single step: per step of a lone
// 2000^2 shot with a checkpoint at every step 51 -> 30 us.
bool copies_first(const fdk::MultiGrid *grids, int count, int k)
{
    const double cells = (double)grids[0].nz * grids[0].px, all = count * cells;
    double us = 0.0;
    (void)fdk::multi2d_shape(grids, count, k, fdk::kFwdKeep, &us);
    us = std::max(us, 2.5 + all * 2.6e-6);
    return count * (3.3 + cells * 1.15e-6) + (k > 0 ? single_us(all) : 0.0) < us;
}

const char *ckpt_slot(const Layout &L, const void *ckpt, int64_t seg)
{
    return (const char *)ckpt + (size_t)seg * ckpt_slot_bytes(L);
}

// Whether the step kernels may read levels at `p`: they load 16 bytes at a
// time (a slot and its levels are multiples of 256 bytes, so the buffer's
// address decides).
bool vector_aligned(const void *p) { return (uintptr_t)p % 16 == 0; }

// backward_pass on 2D grids, up to FD_BATCH_MAX shots: several steps per
// launch.  Two pairs of levels, the recompute state's and the adjoint state's
// places in the work buffers, serve the adjoint recursion in turn; while a
// segment is recomputed, the one that does not hold the adjoint state serves
// the recompute, which reads the checkpoint where it lies.  The gradient's
// recompute needs a second pair of its own (the image's does not: its levels
// go to the history) and takes the segment's last two history fields, which
// only its last launch writes: that one reads the first pair, since the
// launches are even in number, and it stores no levels.
//
// A lone step of the adjoint or of the image's recompute is the single step
// kernel's, which has no halo to compute and loads each field once (2000 x
// 2000: adjoint 18 us against 36, recompute 13 against 25).
fd_status backward_2d(const fd_model *model, const ShotIO *io, int32_t count, int32_t every, bool image,
                      hipStream_t s)
{
    const Layout &L = model->L;
    const ptrdiff_t fl = (ptrdiff_t)(L.f32field / 4);
    auto level = [&](int32_t i, int p, int which) -> float * {   // pair 0: recompute state, 1: adjoint state
        return (float *)io[i].work + (p == 0 ? which : 2 + every + which) * fl;
    };
    auto hist = [&](int32_t i, int64_t slot) -> float * { return (float *)io[i].work + (2 + slot) * fl; };
    const int64_t nt = io[0].shot->nt, nseg = n_ckpt(nt, every);
    fdk::MultiGrid grids[FD_BATCH_MAX];
    std::fill(grids, grids + count, fdk::MultiGrid{(int)L.nz, L.px});
    auto most = [&](int64_t run, int mode) { return std::max(1, plan_multi(grids, count, run, mode, false).steps); };
    const int64_t seg0 = std::min<int64_t>(nt, every);
    // (the gradient's at least 2, so that its last launch writes both fields
    // of the tail)
    const int cap = std::max(2, most(seg0, image ? fdk::kFwdKeep : fdk::kFwdLap));
    auto launch = [&](auto make_args, int mode) -> hipError_t {
        fdk::MultiArgs it[FD_BATCH_MAX];
        for (int32_t i = 0; i < count; ++i) it[i] = make_args(i);
        return fdk::launch_multi2d(it, count, mode, s);
    };
    auto launch_single = [&](auto make_args, int mode) -> hipError_t {
        if (count == 1) return fdk::launch_step(make_args(0), 2, L.storage, mode, s);
        fdk::Batch2D b;
        b.count = count;
        for (int32_t i = 0; i < count; ++i) b.it[i] = make_args(i);
        return fdk::launch_step_batch2d(b, mode, s);
    };
    // the pair that holds the adjoint state, and which of its levels is
    // z^(k+1) (the other is z^(k+2))
    int zp = 1, zi = 0;
    for (int64_t seg = nseg - 1; seg >= 0; --seg) {
        const int64_t n0 = seg * every, n1 = std::min<int64_t>(nt, n0 + every), m = n1 - n0;
        const Cut cut = image ? Cut(m - 1, cap, false) : Cut(m, cap, true);
        // The kernels read 16 bytes at a time: a checkpoint at an address that
        // does not allow it is copied first, to levels that the launch reading
        // it does not write (the gradient's launch 0 of several writes the
        // free pair, and not the history's last two fields).
        auto restored = [&](int32_t i, int which) -> float * {
            return image || cut.n == 1 ? level(i, 1 - zp, which) : hist(i, m - 2 + which);
        };
        auto saved = [&](int32_t i, int which) -> float * {
            if (!vector_aligned(io[i].ckpt)) return restored(i, which);
            return (float *)(ckpt_slot(L, io[i].ckpt, seg) + which * L.field);
        };
        auto copy = [&](float *to, int32_t i, int which) {
            return hipMemcpyAsync(to, ckpt_slot(L, io[i].ckpt, seg) + which * L.field, L.field,
                                  hipMemcpyDeviceToDevice, s);
        };
        for (int32_t i = 0; i < count; ++i) {
            if (vector_aligned(io[i].ckpt)) continue;
            for (int which = 0; which < 2; ++which) {
                const hipError_t e = copy(restored(i, which), i, which);
                if (e != hipSuccess) return hip_fail(e, "checkpoint restore");
            }
        }
        int64_t p = 0;
        if (image) {
            // slot p holds w^(n0+p); slot 0 is the checkpoint's P, copied or
            // stored by the first launch
            const int k0 = cut.n == 0 ? 0 : cut.steps(0);
            const bool copied = k0 < 2 && copies_first(grids, count, k0);
            if (copied)
                for (int32_t i = 0; i < count; ++i) {
                    const hipError_t e = copy(hist(i, 0), i, 0);
                    if (e != hipSuccess) return hip_fail(e, "checkpoint restore");
                }
            for (int64_t l = 0; l < cut.n || (l == 0 && !copied); ++l) {
                const int k = l == 0 ? k0 : cut.steps(l);
                auto cur = [&](int32_t i) { return p == 0 ? saved(i, 0) : hist(i, p); };
                auto prev = [&](int32_t i) { return p == 0 ? saved(i, 1) : hist(i, p - 1); };
                const hipError_t e =
                    k == 1 && (l > 0 || copied)
                        ? launch_single(
                              [&](int32_t i) {
                                  StepArgs a = base_args(model, io[i].shot);
                                  a.cur = cur(i);
                                  a.prev = prev(i);
                                  a.out = hist(i, p + 1);
                                  a.n = n0 + p;
                                  return a;
                              },
                              fdk::kFwd)
                        : launch(
                              [&](int32_t i) {
                                  fdk::MultiArgs a = multi_args(model, io[i].shot, n0 + p, k);
                                  a.cur = cur(i);
                                  a.prev = prev(i);
                                  if (p == 0) a.keep1 = hist(i, 0);
                                  a.hist = k > 0 ? hist(i, p + 1) : nullptr;
                                  a.hist_stride = fl;
                                  return a;
                              },
                              fdk::kFwdKeep);
                if (e != hipSuccess) return hip_fail(e, "recompute steps");
                p += k;
            }
        } else {
            for (int64_t l = 0; l < cut.n; ++l) {
                const int k = cut.steps(l);
                const bool last = l + 1 == cut.n;
                // launch 0 reads the checkpoint; odd launches read the free
                // pair, even ones the history's last two fields
                auto place = [&](int32_t i, int64_t after, int which) -> float * {
                    return (after & 1) == 0 ? level(i, 1 - zp, which) : hist(i, m - 2 + which);
                };
                const hipError_t e = launch(
                    [&](int32_t i) {
                        fdk::MultiArgs a = multi_args(model, io[i].shot, n0 + p, k);
                        a.cur = l == 0 ? saved(i, 0) : place(i, l - 1, 0);
                        a.prev = l == 0 ? saved(i, 1) : place(i, l - 1, 1);
                        if (!last) {
                            a.out1 = place(i, l, 0);
                            a.out0 = place(i, l, 1);
                        }
                        a.hist = hist(i, p);
                        a.hist_stride = fl;
                        return a;
                    },
                    fdk::kFwdLap);
                if (e != hipSuccess) return hip_fail(e, "recompute steps");
                p += k;
            }
        }
        int64_t k = n1;   // adjoint steps k = n1 .. n0+1
        const MultiPlan plan = plan_multi(grids, count, m, fdk::kAdj, false);
        const Cut back(plan.lone ? m - 1 : m, std::max(1, plan.steps), false);
        for (int64_t l = 0; k > n0; ++l) {
            const int c = l < back.n ? back.steps(l) : 1;
            // (nt = 0: no source in the adjoint recursion)
            auto resid = [&](int32_t i) -> const float * {
                const int64_t nrec = nrec_of(io[i].shot);
                return nrec > 0 ? io[i].adj + (size_t)(k - 1) * (size_t)nrec : nullptr;
            };
            auto sum = [&](int32_t i) { return (double *)((float *)io[i].work + (4 + every) * fl); };
            if (c == 1) {   // z^k takes the place of z^(k+2)
                const hipError_t e = launch_single(
                    [&](int32_t i) {
                        StepArgs a = base_args(model, io[i].shot);
                        a.cur = level(i, zp, zi);
                        a.prev = level(i, zp, 1 - zi);
                        a.n = k;
                        a.nt = 0;
                        a.lap = hist(i, k - 1 - n0);
                        a.resid_row = resid(i);
                        a.g = sum(i);
                        return a;
                    },
                    fdk::kAdj);
                if (e != hipSuccess) return hip_fail(e, "adjoint steps");
                zi = 1 - zi;
            } else {
                const hipError_t e = launch(
                    [&](int32_t i) {
                        fdk::MultiArgs a = multi_args(model, io[i].shot, 0, c);
                        a.nt = 0;
                        a.cur = level(i, zp, zi);
                        a.prev = level(i, zp, 1 - zi);
                        a.out1 = level(i, 1 - zp, 0);
                        a.out0 = level(i, 1 - zp, 1);
                        a.resid = resid(i);
                        a.rec_stride = -nrec_of(io[i].shot);
                        a.hist = hist(i, k - 1 - n0);
                        a.hist_stride = -fl;
                        a.g = sum(i);
                        return a;
                    },
                    fdk::kAdj);
                if (e != hipSuccess) return hip_fail(e, "adjoint steps");
                zp = 1 - zp;
                zi = 0;
            }
            k -= c;
        }
    }
    return FD_OK;
}

fd_status backward_pass(const fd_model *model, const ShotIO *io, int32_t count, size_t ckpt_bytes,
                        int32_t ckpt_every, size_t work_bytes, bool image, hipStream_t s,
                        double **acc)
{
    const Layout &L = model->L;
    if (L.storage != FD_F32) return fail(FD_ERR_UNSUPPORTED, "the adjoint needs FP32 storage");
    if (ckpt_every < 1) return fail(FD_ERR_INVALID_ARG, "ckpt_every must be >= 1");
    if (count < 1) return fail(FD_ERR_INVALID_ARG, "count must be >= 1");
    for (int32_t i = 0; i < count; ++i) {
        fd_status st = check_shot(model, io[i].shot);
        if (st != FD_OK) return st;
        if (!io[i].adj || !io[i].ckpt || !io[i].work) return fail(FD_ERR_INVALID_ARG, "shot %d: NULL adj, ckpt or work", i);
        if (io[i].shot->nt != io[0].shot->nt) return fail(FD_ERR_INVALID_ARG, "shot %d: all shots must share nt", i);
        if ((uintptr_t)io[i].work % kAlign) return fail(FD_ERR_INVALID_ARG, "work buffer must be 256-byte aligned");
        for (int32_t j = 0; j < i; ++j)
            if (io[j].work == io[i].work) return fail(FD_ERR_INVALID_ARG, "shot %d repeats a work buffer", i);
    }
    const int64_t nt = io[0].shot->nt;
    const int64_t nseg = n_ckpt(nt, ckpt_every);
    if (ckpt_bytes < (size_t)nseg * ckpt_slot_bytes(L))
        return fail(FD_ERR_INVALID_ARG, "checkpoint buffer too small");
    if (work_bytes < adjoint_work_bytes(L, ckpt_every))
        return fail(FD_ERR_INVALID_ARG, "adjoint work buffer too small (%zu < %zu bytes)", work_bytes,
                    adjoint_work_bytes(L, ckpt_every));
    // work layout: recompute state (2), history (K), adjoint state (2), FP64 sum
    auto fw = [&](int32_t i, int64_t n) -> void * { return (char *)io[i].work + (size_t)(n & 1) * L.f32field; };
    auto hist = [&](int32_t i, int64_t slot) -> float * {
        return (float *)((char *)io[i].work + (2 + (size_t)slot) * L.f32field);
    };
    auto zf = [&](int32_t i, int64_t k) -> void * {
        return (char *)io[i].work + (2 + (size_t)ckpt_every + (size_t)(k & 1)) * L.f32field;
    };
    auto gsum = [&](int32_t i) -> double * {
        return (double *)((char *)io[i].work + (4 + (size_t)ckpt_every) * L.f32field);
    };
    auto launch_all = [&](auto make_args, int mode) -> hipError_t {
        for (int32_t i = 0; i < count; ++i) {
            hipError_t e = fdk::launch_step(make_args(i), L.ndim, L.storage, mode, s);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    };

    for (int32_t i = 0; i < count; ++i) {
        hipError_t e = fdk::launch_fill_u32(zf(i, 0), (2 * L.f32field + align_up(L.npad * 8)) / 4, 0u, s);
        if (e != hipSuccess) return hip_fail(e, "adjoint clear");
        acc[i] = gsum(i);
    }
    if (L.ndim == 2) {
        // in groups of at most kGroupCells cells.  (A group's levels, c and
        // sum are 28 bytes a cell and its history streams through besides,
        // so at the limit not all of them stay in the Infinity Cache; the
        // gradient of 8 shots of 1024^2 in groups of at most 5, 9, 13, 18 M
        // cells or together: 15.3, 14.3, 14.07, 14.05, 14.2 ms.)
        const int32_t most = (int32_t)std::clamp(kGroupCells / (double)L.npad, 1.0, (double)FD_BATCH_MAX);
        const int32_t groups = (count + most - 1) / most;
        for (int32_t g = 0; g < groups; ++g) {
            const int32_t i0 = (int32_t)((int64_t)count * g / groups), i1 = (int32_t)((int64_t)count * (g + 1) / groups);
            const fd_status st = backward_2d(model, io + i0, i1 - i0, ckpt_every, image, s);
            if (st != FD_OK) return st;
        }
        return FD_OK;
    }
    for (int64_t seg = nseg - 1; seg >= 0; --seg) {
        const int64_t n0 = seg * ckpt_every;
        const int64_t n1 = std::min<int64_t>(nt, n0 + ckpt_every);
        if (image) {
            // The image's history is the field itself: slot s holds w^(n0+s).
            // Slot 0 is the checkpoint's P; each recompute step reads its
            // Pold from the checkpoint (or, where its address does not allow
            // vector loads, a copy in the recompute state's place) or the
            // slot before and writes the next level into the next slot (out
            // of place), a plain forward step.
            auto pold = [&](int32_t i) -> void * {
                return vector_aligned(io[i].ckpt) ? (void *)(ckpt_slot(L, io[i].ckpt, seg) + L.field) : fw(i, 0);
            };
            for (int32_t i = 0; i < count; ++i) {
                const char *slot = ckpt_slot(L, io[i].ckpt, seg);
                hipError_t e = hipMemcpyAsync(hist(i, 0), slot, L.field, hipMemcpyDeviceToDevice, s);
                if (e == hipSuccess && !vector_aligned(io[i].ckpt))
                    e = hipMemcpyAsync(fw(i, 0), slot + L.field, L.field, hipMemcpyDeviceToDevice, s);
                if (e != hipSuccess) return hip_fail(e, "checkpoint restore");
            }
            for (int64_t n = n0; n + 1 < n1; ++n) {
                hipError_t e = launch_all(
                    [&](int32_t i) {
                        StepArgs a = base_args(model, io[i].shot);
                        a.cur = hist(i, n - n0);
                        a.prev = n == n0 ? pold(i) : (void *)hist(i, n - 1 - n0);
                        a.out = hist(i, n + 1 - n0);
                        a.n = n;
                        a.trace_row = nullptr;
                        return a;
                    },
                    fdk::kFwd);
                if (e != hipSuccess) return hip_fail(e, "recompute step");
            }
        } else {
            for (int32_t i = 0; i < count; ++i) {
                const char *slot = ckpt_slot(L, io[i].ckpt, seg);
                hipError_t e = hipMemcpyAsync(fw(i, n0), slot, L.field, hipMemcpyDeviceToDevice, s);
                if (e == hipSuccess) e = hipMemcpyAsync(fw(i, n0 + 1), slot + L.field, L.field, hipMemcpyDeviceToDevice, s);
                if (e != hipSuccess) return hip_fail(e, "checkpoint restore");
            }
            for (int64_t n = n0; n < n1; ++n) {
                hipError_t e = launch_all(
                    [&](int32_t i) {
                        StepArgs a = base_args(model, io[i].shot);
                        a.cur = fw(i, n);
                        a.prev = fw(i, n + 1);
                        a.n = n;
                        a.trace_row = nullptr;
                        a.lap = hist(i, n - n0);
                        return a;
                    },
                    fdk::kFwdLap);
                if (e != hipSuccess) return hip_fail(e, "recompute step");
            }
        }
        // Adjoint steps k = n1 .. n0+1 in groups of three from the top of the
        // segment: the first two of a group leave their gradient terms to the
        // last, which adds all three (z^(k+2) is its prev and z^(k+1) its cur,
        // both read anyway), so g is read and written once per three steps.
        // A shorter last group (two or one steps) works the same way.  The
        // history of the segment is rebuilt by the next recompute, so groups
        // stay inside it.
        const int64_t m = n1 - n0;
        for (int64_t k = n1; k >= n0 + 1; --k) {
            const int64_t j = n1 - k;
            const int64_t size = std::min<int64_t>(3, m - j / 3 * 3);
            const int32_t gmode = j % 3 < size - 1 ? 1 : (size == 1 ? 0 : (int32_t)size);
            hipError_t e = launch_all(
                [&](int32_t i) {
                    StepArgs a = base_args(model, io[i].shot);
                    const int64_t nrec = nrec_of(io[i].shot);
                    a.cur = zf(i, k + 1);
                    a.prev = zf(i, k);
                    a.n = k;
                    a.nt = 0;  // no source in the adjoint recursion
                    a.lap = hist(i, k - 1 - n0);
                    a.lap2 = gmode >= 2 ? hist(i, k - n0) : nullptr;
                    a.lap3 = gmode == 3 ? hist(i, k + 1 - n0) : nullptr;
                    a.gmode = gmode;
                    a.resid_row = nrec > 0 ? io[i].adj + (size_t)(k - 1) * (size_t)nrec : nullptr;
                    a.g = gsum(i);
                    return a;
                },
                fdk::kAdj);
            if (e != hipSuccess) return hip_fail(e, "adjoint step");
        }
    }
    return FD_OK;
}

}  // namespace

extern "C" {

fd_status fd_adjoint_gradient(const fd_model *model, const fd_shot *shot, const float *adj,
                              const void *ckpt, size_t ckpt_bytes, int32_t ckpt_every, void *work,
                              size_t work_bytes, double *grad_v, void *stream)
{
    return fd_adjoint_gradient_shots(model, &shot, 1, &adj, &ckpt, ckpt_bytes, ckpt_every, &work,
                                     work_bytes, grad_v, stream);
}

fd_status fd_rtm_image(const fd_model *model, const fd_shot *shot, const float *data,
                       const void *ckpt, size_t ckpt_bytes, int32_t ckpt_every, void *work,
                       size_t work_bytes, double *image, void *stream)
{
    return fd_rtm_image_shots(model, &shot, 1, &data, &ckpt, ckpt_bytes, ckpt_every, &work,
                              work_bytes, image, stream);
}

namespace {

fd_status backward_shots(const fd_model *model, const fd_shot *const *shots, int32_t count,
                         const float *const *adj, const void *const *ckpt, size_t ckpt_bytes,
                         int32_t ckpt_every, void *const *work, size_t work_bytes, double *out,
                         bool image, void *stream)
{
    if (!model) return fail(FD_ERR_INVALID_ARG, "NULL model");
    if (!out) return fail(FD_ERR_INVALID_ARG, image ? "NULL image" : "NULL grad_v");
    if (count < 1 || count > 4096) return fail(FD_ERR_INVALID_ARG, "count must be in [1, 4096]");
    if (!shots || !adj || !ckpt || !work) return fail(FD_ERR_INVALID_ARG, "NULL shots, adj, ckpt or work array");
    if (is_slab(model->L)) return fail(FD_ERR_UNSUPPORTED, "the adjoint and the image are not built for z-slabs");
    std::vector<ShotIO> io((size_t)count);
    for (int32_t i = 0; i < count; ++i) io[i] = ShotIO{shots[i], adj[i], ckpt[i], work[i]};
    hipStream_t s = (hipStream_t)stream;
    std::vector<double *> acc((size_t)count, nullptr);
    fd_status st = backward_pass(model, io.data(), count, ckpt_bytes, ckpt_every, work_bytes,
                                 image, s, acc.data());
    if (st != FD_OK) return st;
    const Layout &L = model->L;
    // shot after shot, so the FP64 sum has the order of one call per shot
    for (int32_t i = 0; i < count; ++i) {
        hipError_t e = image ? fdk::launch_image_finish(acc[i], out, L.nz * L.ny, (int32_t)L.nx, L.px, s)
                             : fdk::launch_grad_finish(acc[i], model->c, out, L.nz * L.ny, (int32_t)L.nx,
                                                       L.px, 2.0 * model->grid.dt / model->grid.dh, s);
        if (e != hipSuccess) return hip_fail(e, image ? "image finish" : "gradient finish");
    }
    return ok();
}

}  // namespace

fd_status fd_adjoint_gradient_shots(const fd_model *model, const fd_shot *const *shots,
                                    int32_t count, const float *const *adj,
                                    const void *const *ckpt, size_t ckpt_bytes, int32_t ckpt_every,
                                    void *const *work, size_t work_bytes, double *grad_v,
                                    void *stream)
{
    return backward_shots(model, shots, count, adj, ckpt, ckpt_bytes, ckpt_every, work, work_bytes,
                          grad_v, false, stream);
}

fd_status fd_rtm_image_shots(const fd_model *model, const fd_shot *const *shots, int32_t count,
                             const float *const *data, const void *const *ckpt, size_t ckpt_bytes,
                             int32_t ckpt_every, void *const *work, size_t work_bytes,
                             double *image, void *stream)
{
    return backward_shots(model, shots, count, data, ckpt, ckpt_bytes, ckpt_every, work, work_bytes,
                          image, true, stream);
}

fd_status fd_get_wavefield(const fd_state *state, int32_t which, float *out, void *stream)
{
    if (!state || !out) return fail(FD_ERR_INVALID_ARG, "NULL state or out");
    if (which != 0 && which != 1) return fail(FD_ERR_INVALID_ARG, "which must be 0 (P) or 1 (Pold)");
    if (state->next < 0) return fail(FD_ERR_INVALID_ARG, "fd_begin_shot has not been called");
    const Layout &L = state->m->L;
    const int64_t lvl = which == 0 ? state->next : state->next - 1;
    const void *buf = state->buf[lvl & 1];
    hipError_t e = fdk::launch_get_field(L.storage, buf, out, L.nz * L.ny, (int32_t)L.nx, L.px,
                                         state->meta, (int32_t)(lvl & 3), (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "fd_get_wavefield");
    return ok();
}

fd_status fd_set_wavefield(fd_state *state, int32_t which, const float *in, void *stream)
{
    if (!state || !in) return fail(FD_ERR_INVALID_ARG, "NULL state or in");
    if (which != 0 && which != 1) return fail(FD_ERR_INVALID_ARG, "which must be 0 (P) or 1 (Pold)");
    const Layout &L = state->m->L;
    hipStream_t s = (hipStream_t)stream;
    if (state->next < 0) {
        hipError_t e = fdk::launch_fill_u32(state->base, L.state_least / 4, 0u, s);
        if (e != hipSuccess) return hip_fail(e, "fd_set_wavefield clear");
        state->next = 0;
    }
    const int64_t lvl = which == 0 ? state->next : state->next - 1;
    hipError_t e = fdk::launch_set_field(L.storage, in, state->buf[lvl & 1], L.nz * L.ny,
                                         (int32_t)L.nx, L.px, state->meta, (int32_t)(lvl & 3), s);
    if (e != hipSuccess) return hip_fail(e, "fd_set_wavefield");
    return ok();
}

fd_status fd_check_finite(const fd_state *state, uint32_t *flags, void *stream)
{
    if (!state || !flags) return fail(FD_ERR_INVALID_ARG, "NULL state or flags");
    if ((uintptr_t)flags % 4) return fail(FD_ERR_INVALID_ARG, "flags must be 4-byte aligned");
    if (state->next < 0) return fail(FD_ERR_INVALID_ARG, "fd_begin_shot has not been called");
    const Layout &L = state->m->L;
    hipStream_t s = (hipStream_t)stream;
    // the owned cells of each level (padding included: it holds zeros)
    const size_t bytes = L.npad * L.elem;
    hipError_t e = fdk::launch_fill_u32(flags, 1, 0u, s);
    if (e == hipSuccess)
        e = fdk::launch_nonfinite(L.storage, state->buf[state->next & 1], bytes, flags, 1u,
                                  state->meta + fdk::kHealth, s);
    if (e == hipSuccess)
        e = fdk::launch_nonfinite(L.storage, state->buf[(state->next + 1) & 1], bytes, flags, 2u, nullptr, s);
    if (e != hipSuccess) return hip_fail(e, "fd_check_finite");
    return ok();
}

fd_status fd_stream_probe(int32_t kind, const float *a, const float *b, float *out, size_t n, void *stream)
{
    if (kind != 0 && kind != 1) return fail(FD_ERR_INVALID_ARG, "kind must be 0 (copy) or 1 (out = a + b * out)");
    if (n == 0) return ok();  // nothing to stream; the arrays are not examined
    if (!a || !out || (kind == 1 && !b)) return fail(FD_ERR_INVALID_ARG, "NULL array");
    if (n % 4) return fail(FD_ERR_INVALID_ARG, "n must be a multiple of 4");
    if ((uintptr_t)a % 16 || (uintptr_t)out % 16 || (kind == 1 && (uintptr_t)b % 16))
        return fail(FD_ERR_INVALID_ARG, "arrays must be 16-byte aligned");
    const hipError_t e = fdk::launch_stream_probe(kind, a, b, out, n, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "fd_stream_probe");
    return ok();
}

fd_status fd_slab_exchange(const fd_state *upper, const fd_state *lower, void *stream)
{
    if (!upper || !lower) return fail(FD_ERR_INVALID_ARG, "NULL state");
    if (upper == lower) return fail(FD_ERR_INVALID_ARG, "a slab cannot exchange with itself");
    const Layout &U = upper->m->L, &D = lower->m->L;
    if (!is_slab(U) || !is_slab(D)) return fail(FD_ERR_INVALID_ARG, "both states must be z-slabs");
    if (U.nzg != D.nzg || U.ny != D.ny || U.nx != D.nx || U.storage != D.storage)
        return fail(FD_ERR_INVALID_ARG, "the slabs belong to different grids");
    if (U.z0 + U.nz != D.z0)
        return fail(FD_ERR_INVALID_ARG, "upper's planes [%lld, %lld) do not end where lower's begin (%lld)",
                    (long long)U.z0, (long long)(U.z0 + U.nz), (long long)D.z0);
    if (upper->next < 0 || lower->next < 0) return fail(FD_ERR_INVALID_ARG, "fd_begin_shot has not been called");
    if (upper->next != lower->next)
        return fail(FD_ERR_INVALID_ARG, "the slabs are at different steps (%lld, %lld)",
                    (long long)upper->next, (long long)lower->next);
    const size_t plane = (size_t)U.ny * (size_t)U.px * U.elem;
    const int64_t lvl = upper->next;  // P, the level the next step reads
    const char *u = (const char *)upper->buf[lvl & 1];
    const char *d = (const char *)lower->buf[lvl & 1];
    hipStream_t s = (hipStream_t)stream;
    const hipError_t e = fdk::launch_exchange(u + (size_t)(U.nz - kGhost) * plane, (char *)d - kGhost * plane, d,
                                              (char *)u + (size_t)U.nz * plane, kGhost * plane, s);
    if (e != hipSuccess) return hip_fail(e, "fd_slab_exchange");
    return ok();
}

}  // extern "C"

namespace {

fd_status step_routines(const fd_model *model, fd_state *state, const fd_shot *shot, int64_t n,
                        float *trace_row, void *work, size_t work_bytes, bool static_work, hipStream_t s)
{
    if (!model || !state) return fail(FD_ERR_INVALID_ARG, "NULL model or state");
    if (state->m != model) return fail(FD_ERR_INVALID_ARG, "state was created for another model");
    fd_status st = check_shot(model, shot);
    if (st != FD_OK) return st;
    const Layout &L = model->L;
    if (L.storage != FD_F32) return fail(FD_ERR_UNSUPPORTED, "the routine-per-kernel step is built for FP32 fields only");
    if (is_slab(L)) return fail(FD_ERR_UNSUPPORTED, "the routine-per-kernel step is not built for z-slabs");
    const size_t need = (size_t)L.ndim * L.f32field;
    if (static_work) {
        if (need > fdk::kRoutinesScratchBytes)
            return fail(FD_ERR_INVALID_ARG,
                        "the grid's routine work (%zu bytes) exceeds the static work area (%zu bytes); "
                        "fd_step_routines takes a work buffer of any size",
                        need, fdk::kRoutinesScratchBytes);
    } else {
        if (!work) return fail(FD_ERR_INVALID_ARG, "work is NULL");
        if (work_bytes < need) return fail(FD_ERR_INVALID_ARG, "work holds %zu bytes, %zu needed", work_bytes, need);
    }
    if (state->next < 0) return fail(FD_ERR_INVALID_ARG, "fd_begin_shot has not been called");
    if (n != state->next) return fail(FD_ERR_INVALID_ARG, "step %lld requested, next step is %lld",
                                      (long long)n, (long long)state->next);
    if (n >= shot->nt) return fail(FD_ERR_INVALID_ARG, "step %lld beyond the shot's %lld steps",
                                   (long long)n, (long long)shot->nt);
    if (static_work) {
        const hipError_t e = fdk::routines_scratch(s, &work);
        if (e != hipSuccess) return hip_fail(e, "static work area of the routine step");
    }
    StepArgs a = base_args(model, shot);
    a.cur = state->buf[n & 1];
    a.prev = state->buf[(n + 1) & 1];
    a.n = n;
    a.trace_row = nrec_of(shot) > 0 ? trace_row : nullptr;
    char *w = (char *)work;
    float *dzz = (float *)w, *dxx = (float *)(w + L.f32field);
    float *dyy = L.ndim == 3 ? (float *)(w + 2 * L.f32field) : nullptr;
    hipError_t e = fdk::launch_routines(a, L.ndim, dzz, dxx, dyy, s);
    if (e != hipSuccess) return hip_fail(e, "routine kernels launch");
    state->next = n + 1;
    return ok();
}

}  // namespace

extern "C" {

fd_status fd_step_routines(const fd_model *model, fd_state *state, const fd_shot *shot, int64_t n,
                           float *trace_row, void *work, size_t work_bytes, void *stream)
{
    return step_routines(model, state, shot, n, trace_row, work, work_bytes, false, (hipStream_t)stream);
}

fd_status fd_step_routines_noalloc(const fd_model *model, fd_state *state, const fd_shot *shot,
                                   int64_t n, float *trace_row, void *stream)
{
    static_assert(fdk::kRoutinesScratchBytes == FD_ROUTINES_STATIC_BYTES, "static work area size");
    return step_routines(model, state, shot, n, trace_row, nullptr, 0, true, (hipStream_t)stream);
}

fd_status fd_step_batch(fd_batch_item *items, int32_t count, int32_t nsteps, void *stream)
{
    if (count < 0 || count > FD_BATCH_MAX) return fail(FD_ERR_INVALID_ARG, "count must be in [0, %d]", FD_BATCH_MAX);
    if (count > 0 && !items) return fail(FD_ERR_INVALID_ARG, "items is NULL");
    if (nsteps < 0) return fail(FD_ERR_INVALID_ARG, "nsteps must be >= 0");
    for (int32_t i = 0; i < count; ++i) {
        const fd_batch_item &it = items[i];
        if (!it.model || !it.state) return fail(FD_ERR_INVALID_ARG, "item %d: NULL model or state", i);
        if (it.state->m != it.model) return fail(FD_ERR_INVALID_ARG, "item %d: state of another model", i);
        if (it.model->L.ndim != 2 || it.model->L.storage != FD_F32 || is_slab(it.model->L))
            return fail(FD_ERR_UNSUPPORTED, "item %d: batching is built for 2D FP32 grids", i);
        fd_status st = check_shot(it.model, it.shot);
        if (st != FD_OK) return st;
        if (it.state->next < 0) return fail(FD_ERR_INVALID_ARG, "item %d: fd_begin_shot has not been called", i);
        if (it.n != it.state->next) return fail(FD_ERR_INVALID_ARG, "item %d: n is not the state's next step", i);
        for (int32_t j = 0; j < i; ++j)
            if (items[j].state == it.state) return fail(FD_ERR_INVALID_ARG, "item %d repeats a state", i);
    }
    Flight f[FD_BATCH_MAX];
    for (int32_t i = 0; i < count; ++i)
        f[i] = Flight{items[i].model, items[i].state, items[i].shot, items[i].n,
                      std::min<int64_t>(items[i].shot->nt, items[i].n + nsteps), items[i].traces, nullptr};
    const fd_status st = advance(f, count, (hipStream_t)stream);
    for (int32_t i = 0; i < count; ++i) items[i].n = f[i].n;   // what has been enqueued
    return st == FD_OK ? ok() : st;
}

}  // extern "C"

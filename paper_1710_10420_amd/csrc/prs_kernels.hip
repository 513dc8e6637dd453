// prs_kernels.hip -- float32 instantiation of the PRS kernels (the device
// templates are in prs_device.h), the record reduction and the host-side
// dispatch by precision (the batched ensemble's kernel is in prs_ensemble.hip).

#include <cmath>
#include <mutex>

#include "prs_device.h"

namespace prs {

namespace {

// Reduces the partials of one record per workgroup.  A record's partials
// are a few KB to 4 MB in L2, and a wave alone waits for its loads one after
// another, so each virtual lane is a thread; and a launch reduces the records
// of up to kFinBatch passes, whose launch and first-load latency is then paid
// once and not between every two passes.  One wave and one record per launch
// took 4.5 us at 256^2, 8 us at 2048^2, 21 us at 8192^2 and 190 us at 1024^3
// each; now a launch takes 4.5 us for the five records of a 256^2 run, 5.6 us
// for eight of 2048^2, 14.5 us for four of 8192^2, 103 us for two of 1024^3.
__global__ __launch_bounds__(kFinLanes) void k_finalize(FinBatch B)
{
    __shared__ RecordSums sh[kFinLanes];
    const FinJob& J = B.job[blockIdx.x];
    RecordSums v;
    zero_sums(v);
#pragma unroll 4
    for (int64_t i = threadIdx.x; i < J.count; i += kFinLanes) {
        const WavePartial p = J.parts[i];
        add_counts(v, p);
        v.ar += p.area;
        v.ek += p.ek;
    }
    sh[threadIdx.x] = v;
    __syncthreads();
    if (threadIdx.x >= kWave) return;
    RecordSums r;
    zero_sums(r);
#pragma unroll
    for (int g = 0; g < kFinGroups; ++g) {
        const RecordSums& o = sh[threadIdx.x + g * kWave];
        r.l0 += o.l0;
        r.l1 += o.l1;
        r.l2 += o.l2;
        r.wl += o.wl;
        r.nf += o.nf;
        r.ar += o.ar;
        r.ek += o.ek;
    }
    write_record(r, J.rec, J.step, J.eta, B.area_scale);
}

// Scratch of the allocation-free slab-diagnostics entry point: one record
// slot and the wave partials of one pass, resident on every device the
// library runs on.  Host code never passes this name to a kernel (in host
// code it is only a stand-in for the symbol); static_scratch() hands out the
// device address hipGetSymbolAddress gives for the current device.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// Plain device copy of n16 16-byte words (the reference ceiling that pass
// bandwidths are compared with): each 256-lane workgroup moves 16 KiB, four
// independent 16-byte loads per lane in flight before its stores.
__global__ __launch_bounds__(kBlock) void k_copy16(const uint4* __restrict__ src, uint4* __restrict__ dst,
                                                   int64_t n16)
{
    const int64_t base = (int64_t)blockIdx.x * (4 * kBlock) + threadIdx.x;
    uint4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int64_t i = base + (int64_t)j * kBlock;
        if (i < n16) v[j] = src[i];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int64_t i = base + (int64_t)j * kBlock;
        if (i < n16) dst[i] = v[j];
    }
}

// Sum of `count` doubles in a fixed order into *out.
__global__ __launch_bounds__(kBlock) void k_sum_f64(const double* __restrict__ v, int64_t count,
                                                     double* __restrict__ out)
{
    __shared__ double sh[kBlock];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < count; i += kBlock) acc += v[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int o = kBlock / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = sh[0];
}

// Fills count doubles with 0 (a kernel rather than a memset, so the sequence
// can also live inside a captured graph).
__global__ __launch_bounds__(kBlock) void k_zero_f64(double* __restrict__ v, int64_t count)
{
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < count; i += stride) v[i] = 0.0;
}

__global__ __launch_bounds__(kBlock) void k_zero_f32(float* __restrict__ v, int64_t count)
{
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < count; i += stride) v[i] = 0.0f;
}

}  // namespace

Geometry geometry_of(const prs_params& p)
{
    Geometry g;
    g.ndim = p.ndim;
    g.f64 = p.precision == PRS_F64 ? 1 : 0;
    g.nx = p.n[0];
    if (p.ndim == 2) {
        g.Q = 1;
        g.M = p.n[1];
    } else {
        g.Q = p.n[1];
        g.M = p.n[2];
    }
    return g;
}

TileCounts tile_counts(const Geometry& g, const Tiling& t)
{
    TileCounts c;
    c.tiles_x = (g.nx + (int64_t)kWave * t.vec - 1) / ((int64_t)kWave * t.vec);
    c.tiles_q = (g.Q + step_ty(t.ty) - 1) / step_ty(t.ty);
    c.tiles_s = (g.M + t.rows - 1) / t.rows;
    c.ntiles = c.tiles_x * c.tiles_q * c.tiles_s;
    return c;
}

bool tiling_supported(const Geometry& g, const Tiling& t)
{
    if (t.vec != 1 && t.vec != 2 && t.vec != 4) return false;
    if (g.f64 && t.vec == 4) return false;          // 16 bytes per lane at most
    if (g.nx % t.vec != 0) return false;
    if (t.rows < 1 || t.rows > 4096) return false;
    if (g.ndim == 2) return t.ty == 1;
    return t.ty == 1 || t.ty == 2 || t.ty == 4 || tb3l_tiling(t.ty);
}

// ---- float32 instantiations ----

hipError_t launch_step_f32(const Geometry& g, const Tiling& t, const void* phi_in, void* phi_out, const void* pi,
                           void* pi_out, const StepCoef64& k, bool update, bool diag, WavePartial* partials,
                           const DiagCoef& dc, hipStream_t s)
{
    return launch_step_r<float>(g, t, phi_in, phi_out, pi, pi_out, k, update, diag, partials, dc, s);
}

hipError_t launch_adj_seed_f32(const void* phi, int64_t count, double kc, double deta, void* mu, void* w,
                               double* partial, int nblocks, hipStream_t s)
{
    return launch_adj_seed_r<float>(phi, count, kc, deta, mu, w, partial, nblocks, s);
}

hipError_t launch_fill_f32(void* phi, int64_t count, uint64_t seed, hipStream_t s)
{
    return launch_fill_r<float>(phi, count, seed, s);
}

// ---- dispatch by precision ----

hipError_t launch_step(const Geometry& g, const Tiling& t, const void* phi_in, void* phi_out, const void* pi,
                       void* pi_out, const StepCoef64& k, bool update, bool diag, WavePartial* partials,
                       const DiagCoef& dc, hipStream_t s)
{
    if (!tiling_supported(g, t) || tile_counts(g, t).ntiles > kMaxWaveTiles) return hipErrorInvalidValue;
    return g.f64 ? launch_step_f64(g, t, phi_in, phi_out, pi, pi_out, k, update, diag, partials, dc, s)
                 : launch_step_f32(g, t, phi_in, phi_out, pi, pi_out, k, update, diag, partials, dc, s);
}

static hipError_t tb_dispatch(int T, const Geometry& g, const Tiling& t, const void* phi_in, void* phi_out,
                              const void* pi_in, void* pi_out, const StepCoef64* k, bool diag,
                              WavePartial* partials, const DiagCoef& dc, int halo, hipStream_t s)
{
    if (g.ndim == 2)
        return g.f64 ? launch_tb2d<double>(T, g, t, phi_in, phi_out, pi_in, pi_out, k, diag, partials, dc, halo, s)
                     : launch_tb2d<float>(T, g, t, phi_in, phi_out, pi_in, pi_out, k, diag, partials, dc, halo, s);
    return g.f64 ? launch_tb3d<double>(T, g, t, phi_in, phi_out, pi_in, pi_out, k, diag, partials, dc, halo, s)
                 : launch_tb3d<float>(T, g, t, phi_in, phi_out, pi_in, pi_out, k, diag, partials, dc, halo, s);
}

hipError_t launch_tb(int T, const Geometry& g, const Tiling& t, const void* phi_in, void* phi_out,
                     const void* pi_in, void* pi_out, const StepCoef64* k, bool diag, WavePartial* partials,
                     const DiagCoef& dc, hipStream_t s)
{
    if (!tb_pass_supported(g, t, T)) return hipErrorInvalidValue;
    return tb_dispatch(T, g, t, phi_in, phi_out, pi_in, pi_out, k, diag, partials, dc, 0, s);
}

// Five steps, the longest LDS pass: a launch of the library's own choice
// (auto_pass3), not a pass length that a caller may set.
hipError_t launch_tb3_deep(const Geometry& g, const Tiling& t, const void* phi_in, void* phi_out, const void* pi_in,
                           void* pi_out, const StepCoef64* k, hipStream_t s)
{
    if (g.ndim != 3 || !tb_pass_supported(g, t, 4) || tb_tiles(g, t, kDeepSteps) > kMaxWaveTiles)
        return hipErrorInvalidValue;
    return g.f64 ? launch_tb3_deep_p<double>(g, t, phi_in, phi_out, pi_in, pi_out, k, s)
                 : launch_tb3_deep_p<float>(g, t, phi_in, phi_out, pi_in, pi_out, k, s);
}

BlkGrid blk_grid(const Geometry& g, int vec, int rows, int waves, int steps)
{
    BlkGrid b{0, 0, (steps + vec - 1) / vec};
    const int64_t w = (int64_t)(kWave - 2 * b.halo_lanes) * vec, h = (int64_t)waves * rows - 2 * steps;
    if (steps < 1 || steps > kBlkSteps || w <= 0 || h <= 0 || g.nx % vec != 0) return b;
    b.tiles_x = (g.nx + w - 1) / w;
    const int64_t n = b.tiles_x * ((g.M + h - 1) / h);
    b.blocks = n * waves <= kMaxWaveTiles ? n : 0;
    return b;
}

// Rows and columns are 32-bit in the kernel, a row's bytes a buffer size.
static bool blk_range(const Geometry& g)
{
    return g.ndim == 2 && g.nx <= ((int64_t)1 << 28) && g.M <= ((int64_t)1 << 30);
}

// A single step has the fewest blocks.
bool blk_supported(const Geometry& g) { return blk_range(g) && blk_choose(g, 1).vec != 0; }

// Time of a block pass on 256 compute units, from launches timed at 128^2 to
// 8192^2 with 4 to 16 steps (the constants are fitted to them; the shape
// picked is within 10 % of the fastest of all shapes, mostly the fastest).
// While every unit holds at most two blocks, all run at once and the fullest
// unit sets the time: launch and first loads, and per step a constant (the
// barrier and the exchange) and the unit's sites.  Beyond that the blocks
// pass through in turn, loads and stores beside other blocks' steps, and the
// larger of memory and arithmetic rules.
BlkShape blk_choose(const Geometry& g, int steps)
{
    struct Shape {
        int8_t vec, rows, waves;
    };
    static const Shape f32[] = {{1, 2, 8},  {1, 2, 16}, {1, 3, 16}, {1, 4, 16}, {1, 5, 16},  {1, 8, 16},  {1, 12, 16},
                                {2, 2, 16}, {2, 3, 16}, {2, 4, 16}, {2, 5, 16}, {2, 6, 16},  {2, 8, 16},  {2, 10, 16},
                                {2, 11, 16}, {2, 12, 16}};
    static const Shape f64[] = {{1, 2, 8},  {1, 2, 16}, {1, 3, 16}, {1, 4, 16}, {1, 5, 16}, {1, 8, 16},
                                {1, 12, 16}, {2, 2, 16}, {2, 3, 16}, {2, 4, 16}, {2, 5, 16}};
    const Shape* list = g.f64 ? f64 : f32;
    const int n = g.f64 ? (int)(sizeof f64 / sizeof f64[0]) : (int)(sizeof f32 / sizeof f32[0]);
    const double size = g.f64 ? 8 : 4, sites = (double)g.nx * (double)g.M;
    const double start = 3.4, step = g.f64 ? 0.109 : 0.085, load = g.f64 ? 0.020 : 0.0095;
    const double bw = 4 * sites * size > 250e6 ? 5.5e3 : g.f64 ? 6.5e3 : 4.7e3;   // bytes per ns x 1000
    BlkShape best{0, 0, 0, 0.0f};
    for (int i = 0; i < n; ++i) {
        const int v = list[i].vec, r = list[i].rows, w = list[i].waves;
        const BlkGrid b = blk_grid(g, v, r, w, steps);
        if (b.blocks < 1) continue;
        // us per step of 64 sites of a unit: two columns a lane share a DPP
        // shift and an LDS access
        const double site = (g.f64 ? 0.0059 : 0.0039) * (v == 1 ? 1.1 : 1.0);
        const double per = (double)b.blocks / 256.0, held = w == 16 ? 2.0 : 4.0, area = (double)(w * r * v);
        double t;
        if (per <= held) {
            const double m = (double)((b.blocks + 255) / 256);
            t = start + steps * (step + m * area * site) + load * area * m;
        } else {
            const double arith = steps * (step + (per + 0.25 * held) * area * site);
            const double mem = ((double)b.blocks * area * kWave + sites) * size * 2.0 / (bw * 1e3);
            t = start + (arith > mem ? arith + 0.2 * mem : mem + 0.2 * arith);
        }
        if (best.vec == 0 || t < best.us) best = BlkShape{v, r, w, (float)t};
    }
    return best;
}

// Rows doubled until a launch holds the wave tiles of single steps and, for
// T > 1, of T-step passes.
static Tiling fit_launch(const Geometry& g, Tiling t, int T)
{
    while (t.rows < 2048 &&
           (tile_counts(g, t).ntiles > kMaxWaveTiles || (T > 1 && tb_tiles(g, t, T) > kMaxWaveTiles)))
        t.rows *= 2;
    return t;
}

// 2D marching passes need about three wave tiles per SIMD (1024 SIMDs) to
// hide a wave's chain of levels: the shortest tiles with one site per lane
// while that makes no more, else two sites per lane, where the width is even,
// and the height that does.  Eight steps at 256^2: 9.1 us with one site and 8
// rows, 14.4 us with four and 8; at 2048^2 21 us with two sites and 13 rows,
// 24 with 16.  One site per lane stays at 32 rows or fewer: 40 steps of
// 4095^2 with a record every four take 1494 us with 8 rows, 1332 with 16,
// 1334 with 32 and 1403 with 64 (float64 2874, 2585, 2556 and 2625).
Tiling auto_tile2(const Geometry& g, int T)
{
    constexpr int64_t kTiles = 3072;
    Tiling t{1, (int)kMinRows, 1};
    if (tb_tiles(g, t, T) <= kTiles) return t;
    if (g.nx % 2 == 0 && (!g.f64 || T <= 4)) t.vec = 2;
    const int most = t.vec == 1 ? 32 : 64;
    while (t.rows < most && tb_tiles(g, t, T) > kTiles) ++t.rows;
    return fit_launch(g, t, T);
}

// 16 bytes a lane where the row allows them, and in 3D short tiles on
// lattices that would not fill the device (128^3: 9 us a step with 8 planes;
// 200 x 120 x 90 11 us against 34 with 32 planes).  Two rows a wave only where
// the fields outgrow the last-level cache: 512^3 431 us against 461 and
// 1024^3 3.59 ms against 3.65, but 384^3 238 us against 212 with one row --
// and with one site per lane (255^3 46.8 us, 58.5 with one row).
// The estimate of a small lattice counts the march of its tiles (512^2, 8 and
// 32 rows: 5.4 and 12.9 us) and the wave rows, most of whose lanes idle on a
// narrow lattice (1 x 100000, 32 rows: 21.5 us).
PassChoice auto_step(const Geometry& g)
{
    const double sites = (double)g.nx * (double)g.Q * (double)g.M, bytes = 4 * sites * (g.f64 ? 8 : 4);
    PassChoice c{1, 0.0f, false, Tiling{1, sites < 8e6 ? 8 : 32, g.ndim == 3 && sites > 1e8 ? 2 : 1}};
    if (g.nx % 4 == 0 && !g.f64) c.til.vec = 4;
    else if (g.nx % 2 == 0) c.til.vec = 2;
    else if (g.ndim == 3 && !g.f64 && sites >= 8e6) c.til.ty = 2;
    if (g.ndim == 2 && sites < 8e6) c.til = auto_tile2(g, 2);
    c.til = fit_launch(g, c.til, 1);
    const double mem = bytes / (bytes < 300e6 ? 7.0e6 : g.ndim == 2 ? 5.6e6 : 4.9e6);
    if (sites < 8e6) {
        const double wave_rows = (double)tile_counts(g, c.til).tiles_x * (double)g.Q * (double)g.M;
        c.us = (float)(2.8 + 0.32 * c.til.rows + std::max(mem, 1.1e-4 * wave_rows));
    } else {
        c.us = (float)(4.5 + mem);
    }
    return c;
}

// The shapes of the 3D LDS pass and the registers a wave of each takes.
struct Pass3Shape {
    int8_t vec, ty, T;
    uint8_t regs;
};

const Pass3Shape* pass3_shapes(bool f64, int* n)
{
    static const Pass3Shape f32[] = {
        {1, 8, 2, 33},  {1, 16, 2, 56},  {1, 32, 2, 33},  {1, 64, 2, 56},  {2, 8, 2, 72},
        {2, 16, 2, 126}, {2, 32, 2, 66}, {1, 8, 3, 42},   {1, 16, 3, 84},  {1, 32, 3, 42},
        {1, 64, 3, 84},  {2, 8, 3, 97},  {2, 16, 3, 176}, {2, 32, 3, 97},  {1, 8, 4, 62},
        {1, 16, 4, 113}, {1, 32, 4, 62}, {1, 64, 4, 113}, {2, 8, 4, 127},  {2, 16, 4, 219},
        {2, 32, 4, 127}, {2, 16, 5, 219}};
    static const Pass3Shape f64s[] = {{1, 8, 2, 68},   {1, 8, 3, 93},   {1, 8, 4, 118}, {1, 16, 2, 128},
                                      {1, 16, 3, 179}, {1, 16, 4, 220}, {1, 16, 5, 219}};
    *n = f64 ? (int)(sizeof f64s / sizeof f64s[0]) : (int)(sizeof f32 / sizeof f32[0]);
    return f64 ? f64s : f32;
}

// Estimated time of an LDS pass: the time of a round of workgroups
// (iterations, each a constant and the resident workgroups' rows and levels)
// times the rounds, or of the memory traffic where that is longer.  reverse:
// the adjoint's pass, which reads T fields besides w and mu.
struct Pass3Time {
    Pass3Time(const Geometry& lattice, const Pass3Shape& h, bool rev = false) : g(lattice), T(h.T), reverse(rev)
    {
        size = g.f64 ? 8 : 4;
        sites = (double)g.nx * (double)g.Q * (double)g.M;
        cached = 4 * sites * size < 300e6;
        const int nw = tb3l_waves(h.ty), r = tb3l_rows_per_wave(h.ty);
        const int64_t w = tb3l_width(g.nx, h.vec, T), y = tb3l_own_rows(nw, r, T);
        cols = ((g.nx + w - 1) / w) * ((g.Q + y - 1) / y);
        const int waves = h.regs <= 64 ? 8 : h.regs <= 72 ? 7 : h.regs <= 80 ? 6 : h.regs <= 96 ? 5 : h.regs <= 128 ? 4 : h.regs <= 168 ? 3 : 2;
        held = std::max(1, 4 * waves / nw);
        area = (double)(nw * r * h.vec);
    }
    double us(int64_t rows) const
    {
        const double site = (g.f64 ? 0.0060 : 0.00353) * (reverse ? 1.7 : 1.0);
        const double bw = cached && !reverse ? 8.8e3 : 5.5e3;
        const int64_t wgs = cols * ((g.M + rows - 1) / rows);
        const double iters = (double)(rows + 2 * T - 2);
        auto iter = [&](double m) { return 0.18 + m * area * (T + 1) * site; };
        double t;
        if (wgs <= 256 * (int64_t)held) {
            t = 4.46 + iters * iter((double)((wgs + 255) / 256));
        } else {
            const double rounds = (double)wgs / (256.0 * held), full = std::floor(rounds), rest = rounds - full;
            t = 4.46 + iters * (full * iter(held) + (rest > 0 ? iter(std::max(1.0, std::ceil(rest * held))) : 0.0));
        }
        const double planes = reverse ? (2.0 + T) * (double)rows + 4.0 * T - 2.0 : 2.0 * (double)rows + 4.0 * T - 2.0;
        const double read = (double)wgs * kWave * area * planes * size;
        const double mem = (0.75 * read + 2.5 * sites * size) / (bw * 1e3);
        return mem > t ? mem + 0.15 * t : t + 0.15 * mem;
    }
    // The fastest of the heights that give one to four whole rounds and two
    // or three plain ones.
    int64_t best_rows(int64_t least) const
    {
        int64_t best = 32;
        for (int k = 0; k < 6; ++k) {
            int64_t rows = k == 4 ? 16 : 64;
            if (k < 4) {
                const int64_t tz = 256 * (int64_t)held * (k + 1) / cols;
                if (tz < 1) continue;
                rows = std::min<int64_t>(64, std::max<int64_t>(least, (g.M + tz - 1) / tz));
            } else if (k == 5 && cached) {
                continue;
            }
            if (us(rows) < us(best)) best = rows;
        }
        return best;
    }
    const Geometry& g;
    int T, held;
    bool reverse;
    bool cached;
    int64_t cols;
    double size, sites, area;
};

// The estimated fastest LDS pass of T steps.  Within 7 % of the fastest
// measured shape from 64^3 to 400^3; above the last-level cache two sites per
// lane, whose rows are longer, run 20 % faster than one, and only there are
// there passes of five steps (512^3 123 us a step against 144 with four, but
// 256^3 20 against 15: the five-step march has no room for more than two
// waves per SIMD).
PassChoice auto_pass3(const Geometry& g, int T)
{
    int n;
    const Pass3Shape* list = pass3_shapes(g.f64, &n);
    PassChoice best{T, 0.0f, false, Tiling{0, 0, 0}};
    for (int i = 0; i < n; ++i) {
        const Pass3Shape& h = list[i];
        if (h.T != T || !tb_pass_supported(g, Tiling{h.vec, 32, h.ty}, std::min(T, 4))) continue;
        const Pass3Time p(g, h);
        if (p.cached ? T > 4 : !g.f64 && h.vec == 1 && g.nx % 2 == 0) continue;
        const Tiling til{h.vec, (int)p.best_rows(4), h.ty};
        if (tb_tiles(g, til, T) > kMaxWaveTiles) continue;
        const double t = p.us(til.rows);
        if (best.til.vec == 0 || t < best.us) {
            best.us = (float)t;
            best.til = til;
        }
    }
    return best;
}

// A pass of T steps in a tiling that the caller or the tuner chose, vec 0
// when it is none of the LDS pass.
PassChoice own_pass3(const Geometry& g, const Tiling& t, int T)
{
    int n;
    const Pass3Shape* list = pass3_shapes(g.f64, &n);
    if (tb3l_tiling(t.ty) && tb_pass_supported(g, t, T))
        for (int i = 0; i < n; ++i)
            if (list[i].T == T && list[i].vec == t.vec && list[i].ty == t.ty)
                return PassChoice{T, (float)Pass3Time(g, list[i]).us(t.rows), false, t};
    return PassChoice{T, 0.0f, false, Tiling{0, 0, 0}};
}

// Reverse passes.  3D (stored): the LDS reverse pass that the estimate ranks
// first.  2D (fused, four steps): the shortest tiles with one site
// per lane while they make at most two per SIMD; else two sites per lane and
// one tile per SIMD if those are short, or two (the tuner's choice from
// 128^2 to 3000 x 2000, the single steps of four sites per lane took 24
// against 9 us a step at 2048^2).
Tiling auto_adj_tile(const Geometry& g, int* T)
{
    if (g.ndim == 3) {
        static const Pass3Shape f32[] = {{1, 8, 2, 60},  {1, 8, 3, 82},   {1, 8, 4, 100},  {1, 16, 2, 112},
                                         {1, 16, 3, 144}, {1, 16, 4, 180}, {2, 8, 2, 112},  {2, 8, 3, 144},
                                         {2, 8, 4, 182}, {2, 16, 2, 180}, {2, 16, 3, 250}};
        static const Pass3Shape f64s[] = {{1, 8, 2, 112}, {1, 8, 3, 144}, {1, 8, 4, 182}, {1, 16, 2, 180}, {1, 16, 3, 250}};
        Tiling best{1, g.M < 96 ? 8 : 16, 2};
        double least = 0.0;
        *T = 2;
        const Pass3Shape* list = g.f64 ? f64s : f32;
        const int n = g.f64 ? (int)(sizeof f64s / sizeof f64s[0]) : (int)(sizeof f32 / sizeof f32[0]);
        for (int i = 0; i < n; ++i) {
            const Pass3Shape& h = list[i];
            if (!tiling_supported(g, Tiling{h.vec, (int)kMinRows, h.ty})) continue;
            const Pass3Time p(g, h, true);
            const Tiling til{h.vec, (int)p.best_rows(kMinRows), h.ty};
            if (!tba_supported(g, til, h.T)) continue;
            const double us = p.us(til.rows) / h.T;
            if (least == 0.0 || us < least) {
                least = us;
                *T = h.T;
                best = til;
            }
        }
        // Lattices of a few rows leave most of a workgroup's waves idle: 1 x 1
        // x 20000 33 us a step in passes of two, 9 in single steps.
        if (least > 2.0 * auto_step(g).us) *T = 1;
        return best;
    }
    *T = 4;
    Tiling t{1, (int)kMinRows, 1};
    if (g.f64 || g.nx % 2 != 0) {
        while (t.rows < 64 && tbf_tiles(g, t, 4) > 2048) ++t.rows;
        return t;
    }
    if (tbf_tiles(g, t, 4) <= 2048) return t;
    t.vec = 2;
    while (t.rows <= 12 && tbf_tiles(g, t, 4) > 1024) ++t.rows;
    if (t.rows <= 12) return t;
    t.rows = (int)kMinRows;
    while (t.rows < 64 && tbf_tiles(g, t, 4) > 2048) ++t.rows;
    return t;
}

// Single reverse steps (checkpoints every step, and remainders): not the
// passes' tiles, whose one site per lane is for their chains.  Short tiles
// with 16 bytes a lane where the row allows them and a field takes 4 MB
// (2048^2 float32 18.4 us with four sites and 8 rows, 19.2 with one; float64
// 32.4 with two, 40.5 with one; but 256^2 6.6 with one, 8.0 with four), 16
// rows on large 2D lattices (4096^2 63 us, 68 with 8), and on large float32
// boxes of odd width four rows a wave (255^3 94 us, 97 with one; float64 399^3
// 695 with one, 748 with two).
Tiling auto_adj_step(const Geometry& g)
{
    const double sites = (double)g.nx * (double)g.Q * (double)g.M;
    Tiling t{1, g.ndim == 2 && sites >= 8e6 ? 16 : (int)kMinRows, 1};
    if (sites * (g.f64 ? 8 : 4) >= 4e6) t.vec = g.nx % 4 == 0 && !g.f64 ? 4 : g.nx % 2 == 0 ? 2 : 1;
    if (g.ndim == 3 && !g.f64 && t.vec == 1 && sites >= 8e6) t.ty = 4;
    return fit_launch(g, t, 1);
}

hipError_t launch_blk2d(int steps, const BlkShape& b, const Geometry& g, const void* phi_in, void* phi_out,
                        const void* pi_in, void* pi_out, const StepCoef64* k, hipStream_t s)
{
    if (!blk_range(g)) return hipErrorInvalidValue;
    return g.f64 ? launch_blk2d_p<double>(steps, b, g, phi_in, phi_out, pi_in, pi_out, k, s)
                 : launch_blk2d_p<float>(steps, b, g, phi_in, phi_out, pi_in, pi_out, k, s);
}

hipError_t launch_tb_slab(int T, const Geometry& g, const Tiling& t, const void* phi_in, void* phi_out,
                          const void* pi_in, void* pi_out, const StepCoef64* k, bool diag, WavePartial* partials,
                          const DiagCoef& dc, hipStream_t s)
{
    if (!tb_pass_supported(g, t, T)) return hipErrorInvalidValue;
    return tb_dispatch(T, g, t, phi_in, phi_out, pi_in, pi_out, k, diag, partials, dc, T, s);
}

hipError_t launch_adjoint(const Geometry& g, const Tiling& t, const void* w_in, void* w_out, void* mu,
                          const void* phi_n, double* gacc, const AdjCoef64& c, hipStream_t s)
{
    if (!tiling_supported(g, t) || tile_counts(g, t).ntiles > kMaxWaveTiles) return hipErrorInvalidValue;
    return g.f64 ? launch_adjoint_p<double>(g, t, w_in, w_out, mu, phi_n, gacc, c, s)
                 : launch_adjoint_p<float>(g, t, w_in, w_out, mu, phi_n, gacc, c, s);
}

hipError_t launch_adj_seed(const Geometry& g, const void* phi, int64_t count, double kc, double deta, void* mu,
                           void* w, double* partial, int nblocks, hipStream_t s)
{
    return g.f64 ? launch_adj_seed_f64(phi, count, kc, deta, mu, w, partial, nblocks, s)
                 : launch_adj_seed_f32(phi, count, kc, deta, mu, w, partial, nblocks, s);
}

bool tba_supported(const Geometry& g, const Tiling& t, int T)
{
    if (!tb_supported(g) || !tiling_supported(g, t)) return false;
    bool has;     // there is a kernel
    if (g.ndim == 3 && tb3l_tiling(t.ty)) {
        const int rw = tb3l_rows_per_wave(t.ty), nw = tb3l_waves(t.ty);
        has = g.f64 ? tba3l_combo_ok<double>(t.vec, T, rw, nw) : tba3l_combo_ok<float>(t.vec, T, rw, nw);
    } else if (g.ndim == 3) {
        const int TY = tb3_rows(t.ty);
        has = g.f64 ? tba3_combo_ok<double>(t.vec, T, TY) : tba3_combo_ok<float>(t.vec, T, TY);
    } else {
        has = t.ty == 1 && (g.f64 ? tba_combo_ok<double>(t.vec, T) : tba_combo_ok<float>(t.vec, T));
    }
    return has && tb_tiles(g, t, T) <= kMaxWaveTiles;
}

bool tb_all_supported(const Geometry& g, const Tiling& t, int T)
{
    if (g.ndim == 3) return tb_pass_supported(g, t, T);
    if (!tb_supported(g) || !tiling_supported(g, t) || t.ty != 1 || tb_tiles(g, t, T) > kMaxWaveTiles) return false;
    return g.f64 ? tball_combo_ok<double>(t.vec, T) : tball_combo_ok<float>(t.vec, T);
}

hipError_t launch_tb_all(int T, const Geometry& g, const Tiling& t, const void* phi_in, void* const* phi_lv,
                         const void* pi_in, void* pi_out, const StepCoef64* k, hipStream_t s)
{
    if (!tb_all_supported(g, t, T)) return hipErrorInvalidValue;
    return g.f64 ? launch_tb_all_p<double>(T, g, t, phi_in, phi_lv, pi_in, pi_out, k, s)
                 : launch_tb_all_p<float>(T, g, t, phi_in, phi_lv, pi_in, pi_out, k, s);
}

hipError_t launch_tba(int T, const Geometry& g, const Tiling& t, const void* w_in, void* w_out, const void* mu_in,
                      void* mu_out, const void* const* phi, double* gacc, const AdjCoef64* c, hipStream_t s)
{
    if (!tba_supported(g, t, T)) return hipErrorInvalidValue;
    if (g.ndim == 3 && tb3l_tiling(t.ty))
        return g.f64 ? launch_tba3l_p<double>(T, g, t, w_in, w_out, mu_in, mu_out, phi, gacc, c, s)
                     : launch_tba3l_p<float>(T, g, t, w_in, w_out, mu_in, mu_out, phi, gacc, c, s);
    return g.f64 ? launch_tba_p<double>(T, g, t, w_in, w_out, mu_in, mu_out, phi, gacc, c, s)
                 : launch_tba_p<float>(T, g, t, w_in, w_out, mu_in, mu_out, phi, gacc, c, s);
}

bool tb_mid_supported(const Geometry& g, const Tiling& t, int T)
{
    if (g.ndim != 2 || !tb_supported(g) || !tiling_supported(g, t) || t.ty != 1 || tb_tiles(g, t, T) > kMaxWaveTiles)
        return false;
    return g.f64 ? tbmid_combo_ok<double>(t.vec, T) : tbmid_combo_ok<float>(t.vec, T);
}

hipError_t launch_tb_mid(int T, const Geometry& g, const Tiling& t, const void* phi_in, void* phi_out,
                         const void* pi_in, void* pi_out, void* phi_mid, void* pi_mid, const StepCoef64* k,
                         hipStream_t s)
{
    if (!tb_mid_supported(g, t, T)) return hipErrorInvalidValue;
    return g.f64 ? launch_tb_mid_p<double>(T, g, t, phi_in, phi_out, pi_in, pi_out, phi_mid, pi_mid, k, s)
                 : launch_tb_mid_p<float>(T, g, t, phi_in, phi_out, pi_in, pi_out, phi_mid, pi_mid, k, s);
}

bool tbf_supported(const Geometry& g, const Tiling& t, int T)
{
    if (g.ndim != 2 || !tb_supported(g) || !tiling_supported(g, t) || t.ty != 1 || tbf_tiles(g, t, T) > kMaxWaveTiles)
        return false;
    return g.f64 ? tbf_combo_ok<double>(t.vec, T) : tbf_combo_ok<float>(t.vec, T);
}

int64_t tbf_tiles(const Geometry& g, const Tiling& t, int T)
{
    const int64_t W = (int64_t)(kWave - 2 * tbf_halo(t.vec, T)) * t.vec;
    return ((g.nx + W - 1) / W) * ((g.M + t.rows - 1) / t.rows);
}

int64_t tb2_workgroups(const Geometry& g, const Tiling& t, int T)
{
    return (tb_tiles(g, t, T) + kWavesPerBlock - 1) / kWavesPerBlock;
}

int64_t tbf_workgroups(const Geometry& g, const Tiling& t, int T)
{
    return (tbf_tiles(g, t, T) + kWavesPerBlock - 1) / kWavesPerBlock;
}

hipError_t launch_tbf(int T, const Geometry& g, const Tiling& t, const void* phi_s, const void* pi_s,
                      const void* w_in, void* w_out, const void* mu_in, void* mu_out, double* gacc,
                      const StepCoef64* k, const AdjCoef64* c, hipStream_t s)
{
    if (!tbf_supported(g, t, T)) return hipErrorInvalidValue;
    return g.f64 ? launch_tbf_p<double>(T, g, t, phi_s, pi_s, w_in, w_out, mu_in, mu_out, gacc, k, c, s)
                 : launch_tbf_p<float>(T, g, t, phi_s, pi_s, w_in, w_out, mu_in, mu_out, gacc, k, c, s);
}

hipError_t launch_fill_uniform(void* phi, int64_t count, uint64_t seed, bool f64, hipStream_t s)
{
    return f64 ? launch_fill_f64(phi, count, seed, s) : launch_fill_f32(phi, count, seed, s);
}

hipError_t launch_finalize(const FinJob* jobs, int n, double area_scale, hipStream_t s)
{
    if (n < 1 || n > kFinBatch) return hipErrorInvalidValue;
    FinBatch B{};
    for (int i = 0; i < n; ++i) B.job[i] = jobs[i];
    B.area_scale = area_scale;
    hipLaunchKernelGGL(k_finalize, dim3(n), dim3(kFinLanes), 0, s, B);
    return hipGetLastError();
}

hipError_t static_scratch(void** ptr, size_t* bytes)
{
    // the device address of `scratch` on each device, looked up once per
    // device with that device current (each device holds its own copy)
    constexpr int kMaxDevices = 64;
    static std::mutex lock;
    static void* addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> g(lock);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    *bytes = kStaticScratchBytes;
    return hipSuccess;
}

hipError_t launch_copy16(const void* src, void* dst, int64_t n16, hipStream_t s)
{
    if (n16 <= 0) return hipSuccess;
    const int64_t blocks = (n16 + 4 * kBlock - 1) / (4 * kBlock);
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_copy16, dim3((unsigned)blocks), dim3(kBlock), 0, s, static_cast<const uint4*>(src),
                       static_cast<uint4*>(dst), n16);
    return hipGetLastError();
}

hipError_t launch_sum_f64(const double* v, int64_t count, double* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_sum_f64, dim3(1), dim3(kBlock), 0, s, v, count, out);
    return hipGetLastError();
}

hipError_t launch_zero_f64(double* v, int64_t count, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    int64_t blocks = (count + kBlock - 1) / kBlock;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_zero_f64, dim3((unsigned)blocks), dim3(kBlock), 0, s, v, count);
    return hipGetLastError();
}

hipError_t batch_clock_rate_khz(int* khz)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    return hipDeviceGetAttribute(khz, hipDeviceAttributeWallClockRate, dev);
}

hipError_t launch_zero_f32(float* v, int64_t count, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    int64_t blocks = (count + kBlock - 1) / kBlock;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_zero_f32, dim3((unsigned)blocks), dim3(kBlock), 0, s, v, count);
    return hipGetLastError();
}



int64_t tb_owned_width(int vec, int T)
{
    const int H = (T + vec - 1) / vec;
    return (int64_t)(kWave - 2 * H) * vec;
}


bool tb_supported(const Geometry& g)
{
    if (g.M > kMaxMarch) return false;
    if (g.ndim == 2) return g.nx <= ((int64_t)1 << 28);
    return g.nx * g.Q * (g.f64 ? 8 : 4) < ((int64_t)1 << 31);
}

bool tb_steps_supported(const Geometry& g, int T)
{
    if (!tb_supported(g)) return false;
    if (g.ndim == 3) return T == 2 || T == 3 || T == 4;
    return T == 2 || T == 3 || T == 4 || T == 6 || T == 8;
}

bool tb_pass_supported(const Geometry& g, const Tiling& t, int T)
{
    if (!tb_steps_supported(g, T) || !tiling_supported(g, t) || tb_tiles(g, t, T) > kMaxWaveTiles) return false;
    if (g.ndim == 2) return t.ty == 1 && (g.f64 ? tb2_combo_ok<double>(t.vec, T) : tb2_combo_ok<float>(t.vec, T));
    if (tb3l_tiling(t.ty)) {
        const int rw = tb3l_rows_per_wave(t.ty), nw = tb3l_waves(t.ty);
        return g.f64 ? tb3l_combo_ok<double>(t.vec, T, rw, nw) : tb3l_combo_ok<float>(t.vec, T, rw, nw);
    }
    return g.f64 ? tb3_combo_ok<double>(t.vec, T, tb3_rows(t.ty)) : tb3_combo_ok<float>(t.vec, T, tb3_rows(t.ty));
}

int64_t tb_tiles(const Geometry& g, const Tiling& t, int T)
{
    int64_t W = tb_owned_width(t.vec, T);
    const int64_t planes = (g.M + t.rows - 1) / t.rows;
    if (g.ndim == 3 && tb3l_tiling(t.ty)) {
        // one partial per wave of every workgroup
        const int nw = tb3l_waves(t.ty);
        W = tb3l_width(g.nx, t.vec, T);
        const int64_t yown = tb3l_own_rows(nw, tb3l_rows_per_wave(t.ty), T);
        return ((g.nx + W - 1) / W) * ((g.Q + yown - 1) / yown) * planes * nw;
    }
    if (g.ndim == 3) {
        const int64_t TY = tb3_rows(t.ty);
        return ((g.nx + W - 1) / W) * ((g.Q + TY - 1) / TY) * planes;
    }
    return ((g.nx + W - 1) / W) * planes;
}

}  // namespace prs

// prs_block2d.h -- 2D passes over blocks held in registers (gfx950).
//
// The marching passes of prs_device.h carry T levels through rows of a tall
// tile, one wave per tile: on a small lattice there are fewer tiles than
// SIMDs, and a wave alone waits for its own chain of T levels per row (about
// 12 cycles per instruction).  Here a workgroup of NW waves holds a whole
// block, 64 VEC columns by NW RPW rows, phi and phi_dot in registers (wave w
// the rows w RPW .. w RPW + RPW - 1), and advances all of it one step at a
// time: the rows of a step are independent, the x-neighbours are the adjacent
// lanes' (DPP), and only the first and last row of a wave go through LDS,
// with one barrier per step.  The block's edge goes stale by one site per
// step on every side, so after T steps the middle is stored; T is a run-time
// number (up to kBlkSteps), so a block needs no code per pass length and a
// launch covers more steps than the marching passes, whose registers hold
// every level.
//
// What bounds it: on small lattices (one or two blocks a compute unit) the
// launch and first loads, about 4 us, and 0.1 us per step of barrier and
// exchange beside the arithmetic; on large ones the vector units -- 9.4
// instructions a site and step, times the block's area over its stored
// middle, 1.4 at 12 steps with 128 x 192 blocks -- with the memory traffic,
// 16 B a site and launch, underneath.  us per step, marching passes (eight
// steps, their tuned tiles) and block passes of the length chosen here:
//   256^2 1.14 and 0.51 (16 steps)     512^2 1.18 and 0.61 (16)
//   1000 x 750 1.44 and 0.86 (14)      1024^2 1.60 and 1.02 (16)
//   2048^2 2.65 and 2.5 (12 to 16)     8192^2 29.5 and 26.1 (11, 12)
//   float64 4096^2 17.3 and 14.0 (12)
#pragma once

#include "prs_device.h"

namespace prs {

template <typename R>
struct BlkArgs {
    const R* phi_in;
    R* phi_out;
    const R* pi_in;
    R* pi_out;
    int32_t nx, ny;
    int32_t tiles_x, steps;
    int32_t halo_lanes, pad;    // ceil(steps / VEC): columns of a side that go stale, in lanes
    StepCoefT<R> k[kBlkSteps];
};

namespace {

// d = a d + v in place, a uniform.  Written out because the compiler's choice,
// v += a d, leaves the result in v's register and copies it back: one of ten
// instructions per site.
__device__ __forceinline__ void scale_add(float& d, float a, float v)
{
    asm("v_fma_f32 %0, %1, %0, %2" : "+v"(d) : "s"(a), "v"(v));
}

__device__ __forceinline__ void scale_add(double& d, double a, double v)
{
    asm("v_fma_f64 %0, %1, %0, %2" : "+v"(d) : "s"(a), "v"(v));
}

// kick_drift<2> of a site in place, operation by operation.
template <bool UNIT, typename R>
__device__ __forceinline__ void kick_drift_here(R& phi, R s, R& pi, const StepCoefT<R>& k)
{
    const R ck = UNIT ? phi : phi * k.kc;
    const R q = fmar(ck, phi, R(-1));
    const R bl = UNIT ? k.b : k.b * k.inv_dx2;
    const R t = fmar(k.b * k.F, q, R(4) * bl);
    scale_add(pi, k.a, fmar(bl, s, -(phi * t)));
    phi = fmar(k.deta, pi, phi);
}

template <int VEC, int RPW, int NW, bool UNIT, typename R>
__global__ __launch_bounds__(NW * kWave) void k_blk2d(BlkArgs<R> args)
{
    __shared__ R lds[2 * NW * 2 * kWave * VEC];
    // the coefficients are indexed by the step: read them where they lie
    const auto& A = *(const __attribute__((address_space(4))) BlkArgs<R>*)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int Y = NW * RPW;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = wave_in_block();
    const int32_t T = A.steps, H = A.halo_lanes, nx = A.nx, ny = A.ny;
    const uint32_t tile = (uint32_t)xcd_remap(blockIdx.x, gridDim.x);
    const uint32_t tx = tile % (uint32_t)A.tiles_x, ty = tile / (uint32_t)A.tiles_x;
    const int32_t x0 = (int32_t)tx * (kWave - 2 * H) * VEC + (lane - H) * VEC;
    const uint32_t voff = (uint32_t)wrap_row(x0, nx) * (uint32_t)sizeof(R);
    const uint32_t soff = (lane >= H && lane < kWave - H && x0 < nx) ? voff : kPastRow;
    const uint32_t row_bytes = (uint32_t)nx * (uint32_t)sizeof(R);
    const int32_t first = wave * RPW;                       // this wave's first row in the block
    const int32_t y0 = (int32_t)ty * (Y - 2 * T) - T + first;   // ... and in the lattice

    R phi[RPW][VEC], pi[RPW][VEC];
    int32_t y = wrap_row(y0, ny);
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        buf_load<VEC>(A.phi_in + (size_t)(uint32_t)y * (uint32_t)nx, row_bytes, voff, phi[r]);
        buf_load<VEC>(A.pi_in + (size_t)(uint32_t)y * (uint32_t)nx, row_bytes, voff, pi[r]);
        y = next_row(y, ny);
    }
    const int wb = wave > 0 ? wave - 1 : 0, wa = wave < NW - 1 ? wave + 1 : NW - 1;
    auto slot = [&](int par, int w, int side) { return lds + (((par * NW + w) * 2 + side) * kWave + lane) * VEC; };
    auto put = [&](int par) {
        tb3l_put<VEC>(slot(par, wave, 0), phi[0]);
        tb3l_put<VEC>(slot(par, wave, 1), phi[RPW - 1]);
    };
    auto set = [&](R (&d)[VEC], const R (&v)[VEC]) {
#pragma unroll
        for (int j = 0; j < VEC; ++j) d[j] = v[j];
    };
    auto add = [&](R (&d)[VEC], const R (&u)[VEC], const R (&v)[VEC]) {
#pragma unroll
        for (int j = 0; j < VEC; ++j) d[j] = u[j] + v[j];
    };
    auto step = [&](int32_t s) {
        R below[VEC], above[VEC];
        set(below, *reinterpret_cast<const R(*)[VEC]>(slot(s & 1, wb, 1)));
        set(above, *reinterpret_cast<const R(*)[VEC]>(slot(s & 1, wa, 0)));
        StepCoefT<R> k;
        k.a = A.k[s].a;
        k.b = A.k[s].b;
        k.deta = A.k[s].deta;
        k.F = A.k[s].F;
        k.kc = A.k[s].kc;
        k.inv_dx2 = A.k[s].inv_dx2;
        // row r in place, from the sum sy of its y-neighbours
        auto row = [&](int r, const R (&sy)[VEC]) {
            const R left = from_left_lane(phi[r][VEC - 1]);
            const R right = from_right_lane(phi[r][0]);
            R sx[VEC];
#pragma unroll
            for (int j = 0; j < VEC; ++j)
                sx[j] = (j > 0 ? phi[r][j > 0 ? j - 1 : 0] : left) + (j < VEC - 1 ? phi[r][j < VEC - 1 ? j + 1 : j] : right);
#pragma unroll
            for (int j = 0; j < VEC; ++j)
                kick_drift_here<UNIT>(phi[r][j], sx[j] + sy[j], pi[r][j], k);
        };
        // A row's sum is formed before the row below it is overwritten, so no
        // old row is kept (copies were 12 % of the loop's instructions).
        R sy[VEC], next[VEC];
        if constexpr (RPW <= 4) {
            // the inner rows first, while the neighbours' rows are on their way
            R second[VEC], last[VEC];
            set(second, phi[1]);
            set(last, phi[RPW - 2]);
            if constexpr (RPW > 2) add(sy, phi[0], phi[RPW > 2 ? 2 : 1]);
#pragma unroll
            for (int r = 1; r < RPW - 1; ++r) {
                if (r < RPW - 2) add(next, phi[r], phi[r + 2 < RPW ? r + 2 : r]);
                row(r, sy);
                set(sy, next);
            }
            add(sy, last, above);
            add(next, below, second);
            row(RPW - 1, sy);
            row(0, next);
        } else {
            add(sy, below, phi[1]);
#pragma unroll
            for (int r = 0; r < RPW; ++r) {
                if (r < RPW - 2) add(next, phi[r], phi[r + 2 < RPW ? r + 2 : r]);
                if (r == RPW - 2) add(next, phi[r], above);
                row(r, sy);
                set(sy, next);
            }
        }
    };
    // rows s .. Y - 1 - s are exact before step s; a wave without one only
    // keeps the barriers
    auto live = [&](int32_t s) { return first + RPW > s && first < Y - s; };
    if constexpr (RPW <= 4) {
        // few rows: the step after next's rows go out as soon as they are
        // computed, and two steps per iteration share their overhead
        put(0);
        auto one = [&](int32_t s) {
            __syncthreads();
            if (live(s)) {
                step(s);
                put((s + 1) & 1);
            }
        };
        int32_t s = 0;
        for (; s + 1 < T; s += 2) {
            one(s);
            one(s + 1);
        }
        if (s < T) one(s);
    } else {
        // many rows: the loads of the later rows are still on their way
        // during the first step
        for (int32_t s = 0; s < T; ++s) {
            if (live(s)) put(s & 1);
            __syncthreads();
            if (live(s)) step(s);
        }
    }
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        const int32_t br = first + r;
        const bool own = br >= T && br < Y - T && y0 + r < ny;
        const size_t base = own ? (size_t)(uint32_t)(y0 + r) * (uint32_t)nx : 0;
        buf_store<VEC>(A.phi_out + base, own ? row_bytes : 0u, soff, phi[r]);
        buf_store<VEC>(A.pi_out + base, own ? row_bytes : 0u, soff, pi[r]);
    }
}

}  // namespace

namespace {

// The shapes with code: (vec, rows per wave, waves).  Two workgroups of 16
// waves fit a compute unit (64 registers a wave, 64 KB of LDS), so that one
// loads and stores while the other computes; taller float32 blocks of 13 or
// 16 rows a wave, which leave room for one, were 2 to 5 % slower at 8192^2
// and four columns a lane no faster anywhere.
template <typename R>
constexpr bool blk_combo_ok(int vec, int rows)
{
    return vec == 1 ? true : sizeof(R) == 4 ? vec == 2 : vec == 2 && rows <= 5;
}

template <typename R, int VEC, int RPW, int NW>
hipError_t launch_blk_t(BlkArgs<R>& A, int64_t blocks, hipStream_t s)
{
    if (A.k[0].inv_dx2 == R(1) && A.k[0].kc == R(1))
        hipLaunchKernelGGL((k_blk2d<VEC, RPW, NW, true, R>), dim3((unsigned)blocks), dim3(NW * kWave), 0, s, A);
    else
        hipLaunchKernelGGL((k_blk2d<VEC, RPW, NW, false, R>), dim3((unsigned)blocks), dim3(NW * kWave), 0, s, A);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_blk_r(int steps, const BlkShape& b, const Geometry& g, const void* phi_in, void* phi_out,
                        const void* pi_in, void* pi_out, const StepCoef64* k, hipStream_t s)
{
    const BlkGrid grid = blk_grid(g, b.vec, b.rows, b.waves, steps);
    if (grid.blocks < 1) return hipErrorInvalidValue;
    BlkArgs<R> A;
    A.phi_in = static_cast<const R*>(phi_in);
    A.phi_out = static_cast<R*>(phi_out);
    A.pi_in = static_cast<const R*>(pi_in);
    A.pi_out = static_cast<R*>(pi_out);
    A.nx = (int32_t)g.nx;
    A.ny = (int32_t)g.M;
    A.tiles_x = (int32_t)grid.tiles_x;
    A.steps = steps;
    A.halo_lanes = grid.halo_lanes;
    A.pad = 0;
    for (int i = 0; i < kBlkSteps; ++i) A.k[i] = coef_as<R>(k[i < steps ? i : 0]);
#define PRS_BLK(V, RR, N)                                                                \
    if (b.vec == V && b.rows == RR && b.waves == N) {                                    \
        if constexpr (blk_combo_ok<R>(V, RR)) return launch_blk_t<R, V, RR, N>(A, grid.blocks, s); \
    }
    PRS_BLK(1, 2, 8)
    PRS_BLK(1, 2, 16)
    PRS_BLK(1, 3, 16)
    PRS_BLK(1, 4, 16)
    PRS_BLK(1, 5, 16)
    PRS_BLK(1, 8, 16)
    PRS_BLK(1, 12, 16)
    PRS_BLK(2, 2, 16)
    PRS_BLK(2, 3, 16)
    PRS_BLK(2, 4, 16)
    PRS_BLK(2, 5, 16)
    PRS_BLK(2, 6, 16)
    PRS_BLK(2, 8, 16)
    PRS_BLK(2, 10, 16)
    PRS_BLK(2, 11, 16)
    PRS_BLK(2, 12, 16)
#undef PRS_BLK
    return hipErrorInvalidValue;
}

}  // namespace

}  // namespace prs

// terrain_voxels.hip -- gfx950 kernels of the mesoscale voxel workload.
//
// Fields on a voxel grid beside the particle step:
//   coarse-grain      particle mass and momentum into voxel densities (FP64
//                     atomics), velocity u = p / rho (Eq. cg_velocity)
//   advect            conserved donor-cell advection of fluidized mass
//                     (Eq. advection), 16 x 16-column tiles marching through
//                     runs of planes
//   convert cut       solid above the predicted zone's bottom becomes fluid
//   convert deposit   particle-free fluid outside the zones becomes solid at
//                     the column's surface (tiles of 64 columns on LDS)
//   surface           Eq. surface per column, into the terrain heightfield
//   grow              particles grow from their voxel's fluid (Eq. eqmotmb)
//   form              new particles from the fluid inside the zones
//   settle            particles at rest outside the zones back to fluid
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "terrain_internal.h"

namespace trk {

constexpr int kBlk = 256;

__host__ __device__ inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---------------------------------------------------------------------------
// Mesoscale voxel fields: coarse-graining (Eq. cg_velocity) and the conserved
// advection of fluidized mass (Eq. advection)
// ---------------------------------------------------------------------------
__global__ void k_fill_f64(double* a, int64_t n, double v)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = v;
}

__global__ void k_cg_clear(int64_t nv, double* rho, double* mom)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nv) rho[i] = 0.0;
    if (i < 3 * nv) mom[i] = 0.0;
}

// one thread per particle of the env: its mass and momentum into its voxel
__global__ void k_coarse_grain(DevBuffers b, EnvDev E, tr_voxel_grid g, double* rho, double* mom)
{
#pragma clang fp contract(off)
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= E.n) return;
    const int sl = E.slot_begin + a;
    const float4 xf = b.xr[sl], vf = vel_at(b.vw, sl);
    const double x[3] = {xf.x, xf.y, xf.z}, v[3] = {vf.x, vf.y, vf.z};
    const double r = xf.w;
    const double m = (double)b.rho[sl] * (4.0 / 3.0) * 3.14159265358979323846 * r * r * r;
    const int dims[3] = {g.nx, g.ny, g.nz};
    const double V0 = g.l0 * g.l0 * g.l0;
    int c[3];
    for (int k = 0; k < 3; ++k) {
        const double f = floor((x[k] - g.origin[k]) / g.l0);
        if (!(f >= 0.0 && f < (double)dims[k])) return;
        c[k] = (int)f;
    }
    const int64_t id = ((int64_t)c[2] * g.ny + c[1]) * g.nx + c[0];
    atomicAdd(&rho[id], m / V0);
    for (int k = 0; k < 3; ++k) atomicAdd(&mom[3 * id + k], m * v[k] / V0);
}

// the value of lane l, the same l in the whole wave
__device__ inline int lane_value(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ inline double lane_value(double v, int l)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l);
    const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
    return __builtin_bit_cast(double, (uint64_t)c << 32 | a);
}

// The smooth kernel spreads a particle over all voxels within 3 R, about 113
// for R = l0: with an FP64 atomic to memory for each it is bound by those
// atomics (22.6 million for 50,000 particles, 480 us).  Neighbours in slot
// order are neighbours in space, so a block takes a run of them and adds
// their shares up in LDS over the box of voxels that they reach together; one
// atomic a voxel and value is left for the whole run (80 us with 8 waves a
// block, 99 with 4: what bounds it is the chain of an exponential).  A run
// whose box does not fit is cut where it stops fitting.  Particles that share
// no box (it would be larger than theirs together, or too large), as after
// positions were set in any order, go to memory directly: 50,000 of them with
// R = l0 / 2 take 117 us, where a box each took 408 and a thread a particle
// 155.  A wave takes a particle at a time, a lane a column of its voxels.  (The
// exponential as the product of its three axes', computed once a particle,
// took 6 us less and rounds twice more.)
constexpr int kCgWaves = 8;
constexpr int kCgVox = 2048;   // voxels of a run's box: 64 KB of LDS, two blocks a CU
constexpr int kCgAxis = 64;    // voxels of a particle's box along the three axes together

__global__ __launch_bounds__(64 * kCgWaves) void k_coarse_grain_smooth(DevBuffers b, EnvDev E, tr_voxel_grid g, double R,
                                                              int run, double* rho, double* mom)
{
#pragma clang fp contract(off)
    __shared__ double acc[4][kCgVox];
    __shared__ double ax2[kCgWaves][kCgAxis];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int p0 = blockIdx.x * run, np = min(run, E.n - p0);
    const int dims[3] = {g.nx, g.ny, g.nz};
    // lane p of every wave: particle p of the run and its box (empty past the run's end)
    double x[3] = {0.0, 0.0, 0.0}, mv[3] = {0.0, 0.0, 0.0}, m = 0.0;
    int lo[3] = {0, 0, 0}, hi[3] = {-1, -1, -1};
    if (lane < np) {
        const int sl = E.slot_begin + p0 + lane;
        const float4 xf = b.xr[sl], vf = vel_at(b.vw, sl);
        const double r = xf.w;
        x[0] = xf.x; x[1] = xf.y; x[2] = xf.z;
        m = (double)b.rho[sl] * (4.0 / 3.0) * 3.14159265358979323846 * r * r * r;
        mv[0] = m * (double)vf.x; mv[1] = m * (double)vf.y; mv[2] = m * (double)vf.z;
        for (int k = 0; k < 3; ++k) {
            const double fl = ceil((x[k] - 3.0 * R - g.origin[k]) / g.l0 - 0.5);
            const double fh = floor((x[k] + 3.0 * R - g.origin[k]) / g.l0 - 0.5);
            // (a bound beyond the grid on its far side leaves the box empty)
            lo[k] = fl < 0.0 ? 0 : (fl > (double)dims[k] ? dims[k] : (int)fl);
            hi[k] = fh > (double)(dims[k] - 1) ? dims[k] - 1 : (fh < -1.0 ? -1 : (int)fh);
        }
    }
    const bool some = lane < np && lo[0] <= hi[0] && lo[1] <= hi[1] && lo[2] <= hi[2];
    const double sq = sqrt(2.0 * 3.14159265358979323846) * R;
    const double norm = 1.0 / (sq * sq * sq), inv = 2.0 * R * R;
    auto volume = [](const int* l, const int* h) {
        return l[0] <= h[0] && l[1] <= h[1] && l[2] <= h[2]
                   ? (double)(h[0] - l[0] + 1) * (h[1] - l[1] + 1) * (h[2] - l[2] + 1) : 0.0;
    };
    const double reach = fmax(1.0, 6.0 * R / g.l0), most = reach * reach * reach;  // voxels of a particle's box
    // the particles that share a box with the next
    auto sharing = [&] {
        int nl[3], nh[3];
        for (int k = 0; k < 3; ++k) {
            const int l = some ? lo[k] : 0x7fffffff, h = some ? hi[k] : -1;
            nl[k] = min(l, __shfl_down(l, 1));
            nh[k] = max(h, __shfl_down(h, 1));
        }
        const double both = volume(nl, nh);
        return __ballot(lane + 1 < np && both <= (double)kCgVox && both <= 2.0 * most);
    };
    for (int q0 = 0; q0 < np;) {
        // the box of particles q0 .. lane, and the first lane at which it no longer fits
        int bl[3], bh[3];
        for (int k = 0; k < 3; ++k) {
            bl[k] = some && lane >= q0 ? lo[k] : 0x7fffffff;
            bh[k] = some && lane >= q0 ? hi[k] : -1;
        }
        for (int o = 1; o < 64; o <<= 1)
            for (int k = 0; k < 3; ++k) {
                const int l = __shfl_up(bl[k], o), h = __shfl_up(bh[k], o);
                if (lane >= o) { bl[k] = min(bl[k], l); bh[k] = max(bh[k], h); }
            }
        const double vol = volume(bl, bh);
        const unsigned long long over = __ballot(vol > (double)kCgVox && lane >= q0);
        const int first = over ? __ffsll((long long)over) - 1 : np, n = first - q0;
        const bool local = n > 1 && lane_value(vol, max(first, 1) - 1) <= n * most;
        int end = first;
        if (!local) {
            const int from = max(first, q0 + 1);
            const unsigned long long pairs = from < 64 ? sharing() >> from : 0ull;
            end = pairs ? from + __ffsll((long long)pairs) - 1 : np;
        }
        const int q1 = __builtin_amdgcn_readfirstlane(end);
        int base[3], side[3];
        for (int k = 0; k < 3; ++k) {
            base[k] = lane_value(bl[k], q1 - 1);
            side[k] = lane_value(bh[k], q1 - 1) - base[k] + 1;
        }
        const int nbox = local && side[0] > 0 ? side[0] * side[1] * side[2] : 0;
        for (int t = threadIdx.x; t < nbox; t += 64 * kCgWaves)
            for (int k = 0; k < 4; ++k) acc[k][t] = 0.0;
        if (local) __syncthreads();
        // (particle p is wave p's, mod their number, whatever the cuts)
        for (int p = q0 + ((wave - q0) & (kCgWaves - 1)); p < q1; p += kCgWaves) {
            if (!lane_value((int)some, p)) continue;
            int plo[3], ps[3];
            double px[3], pmv[3];
            for (int k = 0; k < 3; ++k) {
                plo[k] = lane_value(lo[k], p);
                ps[k] = lane_value(hi[k], p) - plo[k] + 1;
                px[k] = lane_value(x[k], p);
                pmv[k] = lane_value(mv[k], p);
            }
            const double pm = lane_value(m, p);
            auto offset2 = [&](int k, int i) {  // squared distance along an axis to voxel i of the box
                const double y = g.origin[k] + (plo[k] + i + 0.5) * g.l0 - px[k];
                return y * y;
            };
            const bool table = (int64_t)ps[0] + ps[1] + ps[2] <= kCgAxis;
            if (table) {
                const int k = lane < ps[0] ? 0 : (lane < ps[0] + ps[1] ? 1 : 2);
                ax2[wave][lane] = offset2(k, lane - (k > 0 ? ps[0] : 0) - (k > 1 ? ps[1] : 0));
            }
            // (LDS operations of one wave run in order)
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int64_t nxy = (int64_t)ps[0] * ps[1];
            for (int64_t t = lane; t < nxy; t += 64) {
                const int ix = (int)((uint32_t)t % (uint32_t)ps[0]), jy = (int)((uint32_t)t / (uint32_t)ps[0]);
                const double dx2 = table ? ax2[wave][ix] : offset2(0, ix);
                const double dy2 = table ? ax2[wave][ps[0] + jy] : offset2(1, jy);
                for (int kz = 0; kz < ps[2]; ++kz) {
                    const double dz2 = table ? ax2[wave][ps[0] + ps[1] + kz] : offset2(2, kz);
                    const double r2 = (dx2 + dy2) + dz2;
                    if (r2 > 9.0 * R * R) continue;
                    const double z = norm * exp(-r2 / inv);
                    const int cx = plo[0] + ix, cy = plo[1] + jy, cz = plo[2] + kz;
                    if (local) {
                        const int id = ((cz - base[2]) * side[1] + (cy - base[1])) * side[0] + (cx - base[0]);
                        atomicAdd(&acc[0][id], pm * z);
                        for (int k = 0; k < 3; ++k) atomicAdd(&acc[1 + k][id], pmv[k] * z);
                    } else {
                        const int64_t id = ((int64_t)cz * g.ny + cy) * g.nx + cx;
                        atomicAdd(&rho[id], pm * z);
                        for (int k = 0; k < 3; ++k) atomicAdd(&mom[3 * id + k], pmv[k] * z);
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();  // the tables are rewritten for the next particle
        }
        q0 = q1;
        if (!local) continue;
        __syncthreads();
        for (int t = threadIdx.x; t < nbox; t += 64 * kCgWaves) {
            const double mass = acc[0][t];
            if (mass == 0.0) continue;  // reached by no particle (or by massless shares alone)
            const int cx = t % side[0], cy = t / side[0] % side[1], cz = t / (side[0] * side[1]);
            const int64_t id = ((int64_t)(base[2] + cz) * g.ny + (base[1] + cy)) * g.nx + (base[0] + cx);
            atomicAdd(&rho[id], mass);
            for (int k = 0; k < 3; ++k) atomicAdd(&mom[3 * id + k], acc[1 + k][t]);
        }
        __syncthreads();
    }
}

__global__ void k_cg_velocity(int64_t nv, const double* rho, const double* mom, double* u)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nv) return;
    for (int k = 0; k < 3; ++k) u[3 * i + k] = rho[i] > 0.0 ? mom[3 * i + k] / rho[i] : 0.0;
}

void launch_coarse_grain(const DevBuffers& b, const EnvDev& E, const tr_voxel_grid& g, int kernel, double R,
                         double* rho, double* mom, double* u, hipStream_t s)
{
    const int64_t nv = (int64_t)g.nx * g.ny * g.nz;
    hipLaunchKernelGGL(k_cg_clear, dim3((unsigned)cdiv(3 * nv, kBlk)), dim3(kBlk), 0, s, nv, rho, mom);
    if (E.n > 0 && kernel == TR_CG_HEAVISIDE)
        hipLaunchKernelGGL(k_coarse_grain, dim3((unsigned)cdiv(E.n, kBlk)), dim3(kBlk), 0, s, b, E, g, rho, mom);
    else if (E.n > 0) {
        // a particle a wave for few particles, 64 a block where that still gives two blocks a CU
        const int run = (int)std::min<int64_t>(64, std::max<int64_t>(kCgWaves, E.n / 512));
        hipLaunchKernelGGL(k_coarse_grain_smooth, dim3((unsigned)cdiv(E.n, run)), dim3(64 * kCgWaves), 0, s, b, E, g, R,
                           run, rho, mom);
    }
    if (u) hipLaunchKernelGGL(k_cg_velocity, dim3((unsigned)cdiv(nv, kBlk)), dim3(kBlk), 0, s, nv, rho, mom, u);
}

// A block takes a 16 x 16 tile of columns through a run of kc planes: each
// plane of the tile (with a one-voxel halo in x and y) goes through LDS, and
// the planes above and below stay in registers, so every voxel's mass and
// velocity are read once (the halo aside).  The loads of plane k + 1 are in
// flight while plane k is computed (two LDS buffers, one barrier per plane).
// Each block leaves the largest Courant number it met in bmax[b]; one block
// reduces them (device-scope atomics to one address cost about 10 ns each).
constexpr int kAT = 16;  // tile edge (kAT * kAT == kBlk)

struct PlaneRegs {
    double mf, ux, uy, uz;  // the thread's own voxel
    double hx_mf, hx_u;     // across the tile's x edge (tx == 0: i - 1, tx == kAT - 1: i + 1)
    double hy_mf, hy_u;     // across the tile's y edge
};

__device__ inline void load_plane(const tr_voxel_grid& g, const double* u, const double* mf, int i, int j, int k,
                                  int tx, int ty, PlaneRegs& r)
{
    r = PlaneRegs{0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (k < 0 || k >= g.nz || i >= g.nx || j >= g.ny) return;
    const int64_t plane = (int64_t)k * g.nx * g.ny;
    const int64_t id = plane + (int64_t)j * g.nx + i;
    r.mf = mf[id];
    r.ux = u[3 * id];
    r.uy = u[3 * id + 1];
    r.uz = u[3 * id + 2];
    const int hi_ = tx == 0 ? i - 1 : (tx == kAT - 1 ? i + 1 : -1);
    if (hi_ >= 0 && hi_ < g.nx) {
        const int64_t h = plane + (int64_t)j * g.nx + hi_;
        r.hx_mf = mf[h];
        r.hx_u = u[3 * h];
    }
    const int hj = ty == 0 ? j - 1 : (ty == kAT - 1 ? j + 1 : -1);
    if (hj >= 0 && hj < g.ny) {
        const int64_t h = plane + (int64_t)hj * g.nx + i;
        r.hy_mf = mf[h];
        r.hy_u = u[3 * h + 1];
    }
}

__global__ void __launch_bounds__(kBlk) k_advect(tr_voxel_grid g, double dt, const double* u, const double* mf,
                                                 double* out, double* bmax, int tiles_x, int tiles_y, int kc,
                                                 int nblocks, int per)
{
#pragma clang fp contract(off)
    __shared__ double smf[2][kAT + 2][kAT + 2], sux[2][kAT + 2][kAT + 2], suy[2][kAT + 2][kAT + 2];
    const int tx = threadIdx.x % kAT, ty = threadIdx.x / kAT;
    // blocks go to the XCDs in turn; XCD x takes the contiguous run
    // [x per, (x + 1) per) of (tile x, tile y, chunk) order, so neighbouring
    // tiles, which read each other's edges as halo, share an L2
    const int lb = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    const int bx = lb % tiles_x, by = (lb / tiles_x) % tiles_y, bz = lb / (tiles_x * tiles_y);
    const int i = bx * kAT + tx, j = by * kAT + ty;
    // (a block past the last tile has an empty run of planes)
    const int k0 = bz * kc, k1 = lb < nblocks ? min(k0 + kc, g.nz) : k0;
    const bool live = i < g.nx && j < g.ny;
    PlaneRegs prv, cur, nxt;
    load_plane(g, u, mf, i, j, k0 < k1 ? k0 - 1 : -1, tx, ty, prv);
    load_plane(g, u, mf, i, j, k0 < k1 ? k0 : -1, tx, ty, cur);
    double cmax = 0.0;
    for (int k = k0; k < k1; ++k) {
        const int bf = k & 1;
        smf[bf][ty + 1][tx + 1] = cur.mf;
        sux[bf][ty + 1][tx + 1] = cur.ux;
        suy[bf][ty + 1][tx + 1] = cur.uy;
        if (tx == 0) { smf[bf][ty + 1][0] = cur.hx_mf; sux[bf][ty + 1][0] = cur.hx_u; }
        if (tx == kAT - 1) { smf[bf][ty + 1][kAT + 1] = cur.hx_mf; sux[bf][ty + 1][kAT + 1] = cur.hx_u; }
        if (ty == 0) { smf[bf][0][tx + 1] = cur.hy_mf; suy[bf][0][tx + 1] = cur.hy_u; }
        if (ty == kAT - 1) { smf[bf][kAT + 1][tx + 1] = cur.hy_mf; suy[bf][kAT + 1][tx + 1] = cur.hy_u; }
        load_plane(g, u, mf, i, j, k + 1, tx, ty, nxt);
        __syncthreads();
        if (live) {
            // the same faces, operations and order as a voxel-by-voxel sweep:
            // inflow through the lower faces (z, y, x), then outflow through the
            // upper ones (x, y, z); per face (lower voxel a, upper b):
            // u_f = (u_a + u_b) / 2, flux dt u_f m_donor / l0
            const double mi = cur.mf;
            const double ui[3] = {cur.ux, cur.uy, cur.uz};
            const bool lo[3] = {i > 0, j > 0, k > 0};
            const bool hi[3] = {i + 1 < g.nx, j + 1 < g.ny, k + 1 < g.nz};
            const double um[3] = {sux[bf][ty + 1][tx], suy[bf][ty][tx + 1], prv.uz};
            const double mm[3] = {smf[bf][ty + 1][tx], smf[bf][ty][tx + 1], prv.mf};
            const double up[3] = {sux[bf][ty + 1][tx + 2], suy[bf][ty + 2][tx + 1], nxt.uz};
            const double mp[3] = {smf[bf][ty + 1][tx + 2], smf[bf][ty + 2][tx + 1], nxt.mf};
            double m = mi;
#pragma unroll
            for (int d = 2; d >= 0; --d)
                if (lo[d]) {
                    const double uf = 0.5 * (um[d] + ui[d]);
                    m += dt * uf * (uf > 0.0 ? mm[d] : mi) / g.l0;
                }
#pragma unroll
            for (int d = 0; d < 3; ++d)
                if (hi[d]) {
                    const double uf = 0.5 * (ui[d] + up[d]);
                    m -= dt * uf * (uf > 0.0 ? mi : mp[d]) / g.l0;
                    cmax = fmax(cmax, fabs(uf) * dt / g.l0);
                }
            out[(int64_t)k * g.nx * g.ny + (int64_t)j * g.nx + i] = m;
        }
        prv = cur;
        cur = nxt;
    }
    __shared__ double wmax[kBlk / 64];
    for (int o = 32; o > 0; o >>= 1) cmax = fmax(cmax, __shfl_xor(cmax, o));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = cmax;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w) cmax = fmax(cmax, wmax[w]);
        bmax[blockIdx.x] = cmax;
    }
}

// one block: the largest of n per-block maxima, as its bit pattern
__global__ void k_max_reduce(const double* bmax, int n, unsigned long long* bits)
{
    double v = 0.0;
    for (int k = threadIdx.x; k < n; k += blockDim.x) v = fmax(v, bmax[k]);
    __shared__ double wmax[kBlk / 64];
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w) v = fmax(v, wmax[w]);
        *bits = (unsigned long long)__double_as_longlong(v);
    }
}

// tiles of kAT x kAT columns, each through chunks of kc planes: at most
// kAdvectTargetBlocks blocks unless the tiles alone are more
static void advect_shape(const tr_voxel_grid& g, int& tiles_x, int& tiles_y, int& kc, int& chunks)
{
    tiles_x = (int)cdiv(g.nx, kAT);
    tiles_y = (int)cdiv(g.ny, kAT);
    const int64_t tiles = (int64_t)tiles_x * tiles_y;
    int64_t want = std::max<int64_t>(1, kAdvectTargetBlocks / tiles);
    want = std::min<int64_t>(want, cdiv(g.nz, 16));  // at least 16 planes a chunk
    want = std::max<int64_t>(want, 1);
    kc = (int)cdiv(g.nz, want);
    chunks = (int)cdiv(g.nz, kc);
}

int64_t advect_blocks(const tr_voxel_grid& g)
{
    int tx, ty, kc, ch;
    advect_shape(g, tx, ty, kc, ch);
    return 8 * cdiv((int64_t)tx * ty * ch, 8);
}

void launch_advect(const tr_voxel_grid& g, double dt, const double* u, const double* mf_in, double* mf_out,
                   double* bmax, unsigned long long* cfl_bits, hipStream_t s)
{
    int tiles_x, tiles_y, kc, chunks;
    advect_shape(g, tiles_x, tiles_y, kc, chunks);
    const int64_t nb = (int64_t)tiles_x * tiles_y * chunks;
    const int per = (int)cdiv(nb, 8);
    hipLaunchKernelGGL(k_advect, dim3((unsigned)(8 * per)), dim3(kBlk), 0, s, g, dt, u, mf_in, mf_out, bmax, tiles_x,
                       tiles_y, kc, (int)nb, per);
    if (cfl_bits) hipLaunchKernelGGL(k_max_reduce, dim3(1), dim3(kBlk), 0, s, bmax, 8 * per, cfl_bits);
}

// ---------------------------------------------------------------------------
// Conversion between resting solid and fluidized mass: one thread per column,
// its voxels in increasing height (the columns are independent)
// ---------------------------------------------------------------------------
__global__ void k_surface(tr_voxel_grid g, const double* phi, double* h, float* hf)
{
#pragma clang fp contract(off)
    const int64_t nxy = (int64_t)g.nx * g.ny;
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nxy) return;
    double z = g.origin[2];
    // Eq. surface at the top-most voxel with solid, searched downwards kChunk
    // voxels at a time with every load in flight
    constexpr int kChunk = 8;
    bool found = false;
    for (int k1 = g.nz - 1; k1 >= 0 && !found; k1 -= kChunk) {
        double fc[kChunk];
#pragma unroll
        for (int q = 0; q < kChunk; ++q) fc[q] = k1 - q >= 0 ? phi[(int64_t)(k1 - q) * nxy + c] : 0.0;
        for (int q = 0; q < kChunk && !found; ++q)
            if (fc[q] > 0.0) {
                const int k = k1 - q;
                const double zc = g.origin[2] + (k + 0.5) * g.l0;
                z = zc + (fc[q] - 0.5) * g.l0;
                found = true;
            }
    }
    if (h) h[c] = z;
    if (hf) hf[c] = (float)z;
}

// the z range of the vertical line through (x, y) inside a wedge: its lower bound
__device__ inline bool wedge_bottom(const WedgeDev& w, double x, double y, double& zlo)
{
#pragma clang fp contract(off)
    double lo = -INFINITY, hi = INFINITY;
    if (w.n == 0) return false;
    for (int p = 0; p < w.n; ++p) {
        const double a = w.planes[p][2], b = w.planes[p][3] - w.planes[p][0] * x - w.planes[p][1] * y;
        if (a > 0.0) hi = fmin(hi, b / a);
        else if (a < 0.0) lo = fmax(lo, b / a);
        else if (b < 0.0) return false;
    }
    if (!(lo <= hi) || lo == -INFINITY) return false;
    zlo = lo;
    return true;
}

__device__ inline bool in_wedge_set(const WedgeSet& ws, double x, double y, double z)
{
#pragma clang fp contract(off)
    for (int r = 0; r < ws.n_ranges; ++r)
        for (int k = 0; k < ws.cnt[r]; ++k) {
            const WedgeDev& w = ws.base[ws.off[r] + k];
            if (w.n == 0) continue;
            bool in = true;
            for (int p = 0; p < w.n && in; ++p)
                if (w.planes[p][0] * x + w.planes[p][1] * y + w.planes[p][2] * z - w.planes[p][3] > 0.0) in = false;
            if (in) return true;
        }
    return false;
}

// A block takes kCols neighbouring columns, its kBlk / kCols parts every so
// manieth wedge of a column (a wedge is a chain of up to five divisions) and
// then every so manieth run of voxels above the cut.  Eight parts while the
// columns alone leave the chip short of waves, a thread a column beyond: under
// eight wedges 256 x 256 x 128 voxels take 36 us with eight parts, 47 with
// one; 430 x 430 x 128 50 and 63; 512 x 512 x 32 42 and 34, 512 x 512 x 128
// 137 and 66 (the parts' planes lie 2 MB apart).
constexpr int64_t kCutFew = 200000;

template <int kCols>
__global__ __launch_bounds__(kBlk) void k_convert_cut(tr_voxel_grid g, double rho_b, WedgeSet ws, double* phi,
                                                      const double* wc, double* mf, double* total)
{
#pragma clang fp contract(off)
    constexpr int kParts = kBlk / kCols;
    __shared__ double bottom[kParts][kCols], sums[kBlk / 64];
    const int64_t nxy = (int64_t)g.nx * g.ny;
    const int col = threadIdx.x % kCols, part = threadIdx.x / kCols;
    const int64_t c = (int64_t)blockIdx.x * kCols + col;
    const int i = (int)(c % g.nx), j = (int)(c / g.nx);
    const double x = g.origin[0] + (i + 0.5) * g.l0, y = g.origin[1] + (j + 0.5) * g.l0;
    double zcut = INFINITY, lo;
    int at = 0;  // number of the wedge over all ranges
    for (int r = 0; r < ws.n_ranges; ++r) {
        for (int k = (part + kParts - at % kParts) % kParts; k < ws.cnt[r]; k += kParts)
            if (wedge_bottom(ws.base[ws.off[r] + k], x, y, lo)) zcut = fmin(zcut, lo);
        at += ws.cnt[r];
    }
    bottom[part][col] = zcut;
    __syncthreads();
    for (int q = 0; q < kParts; ++q) zcut = fmin(zcut, bottom[q][col]);
    double sum = 0.0;
    if (c < nxy && zcut != INFINITY) {
        const double V0 = g.l0 * g.l0 * g.l0;
        // voxels a whole voxel or more below the cut keep their solid (occupancy
        // is at most 1): start one voxel below the cut's, then read kChunk voxels
        // at a time with every load in flight
        const double kc = floor((zcut - g.origin[2]) / g.l0) - 1.0;
        const int k_start = kc <= 0.0 ? 0 : (kc >= (double)g.nz ? g.nz : (int)kc);
        constexpr int kChunk = 4;
        for (int k0 = k_start + part * kChunk; k0 < g.nz; k0 += kParts * kChunk) {
            double fc[kChunk], wcc[kChunk], mc[kChunk];
#pragma unroll
            for (int q = 0; q < kChunk; ++q) {
                const bool in = k0 + q < g.nz;
                const int64_t id = (int64_t)(k0 + q) * nxy + c;
                fc[q] = in ? phi[id] : 0.0;
                wcc[q] = in ? wc[id] : 0.0;
                mc[q] = in ? mf[id] : 0.0;
            }
#pragma unroll
            for (int q = 0; q < kChunk; ++q) {
                const int k = k0 + q;
                if (k >= g.nz) break;
                double t = (zcut - (g.origin[2] + k * g.l0)) / g.l0;  // occupancy below the cut
                t = t < 0.0 ? 0.0 : (t > 1.0 ? 1.0 : t);
                if (fc[q] > t) {
                    const int64_t id = (int64_t)k * nxy + c;
                    const double dm = wcc[q] * rho_b * V0 * (fc[q] - t);
                    mf[id] = mc[q] + dm;
                    sum += dm;
                    phi[id] = t;
                }
            }
        }
    }
    if (!total) return;
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    if ((threadIdx.x & 63) == 0) sums[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlk / 64; ++w) sum += sums[w];
        if (sum > 0.0) atomicAdd(total, sum);
    }
}

__global__ void k_convert_deposit(tr_voxel_grid g, double rho_b, double w_dep, WedgeSet ws, const double* rho_p,
                                  double* phi, double* wc, double* mf, double* total)
{
#pragma clang fp contract(off)
    const int64_t nxy = (int64_t)g.nx * g.ny;
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nxy) return;
    const int i = (int)(c % g.nx), j = (int)(c / g.nx);
    const double x = g.origin[0] + (i + 0.5) * g.l0, y = g.origin[1] + (j + 0.5) * g.l0;
    const double V0 = g.l0 * g.l0 * g.l0;
    double sum = 0.0;
    // the first voxel of the column that is not full: fills only raise the
    // occupancy, so it never moves down and each search resumes from the last
    int kfree = 0;
    int kc = -1;               // the last voxel filled, its occupancy and compaction as written
    double fc = 0.0, wcc = 0.0;
    // the column is read kChunk voxels at a time (independent loads in
    // flight); a voxel's own deposit changes only phi and wc, and mf of that
    // voxel alone, so the values read ahead stay current
    constexpr int kChunk = 8;
    for (int k0 = 0; k0 < g.nz; k0 += kChunk) {
        double mc[kChunk], rc[kChunk];
#pragma unroll
        for (int t = 0; t < kChunk; ++t) {
            const bool in = k0 + t < g.nz;
            mc[t] = in ? mf[(int64_t)(k0 + t) * nxy + c] : 0.0;
            rc[t] = in ? rho_p[(int64_t)(k0 + t) * nxy + c] : 0.0;
        }
        for (int t = 0; t < kChunk; ++t) {
            const int k = k0 + t;
            if (!(mc[t] > 0.0) || rc[t] != 0.0 || in_wedge_set(ws, x, y, g.origin[2] + (k + 0.5) * g.l0)) continue;
            double m = mc[t];
            int kk = kfree;
            // the last voxel filled is held as written: when it is the first
            // non-full voxel no search is needed
            for (bool found = kk == kc && fc < 1.0; !found && kk < g.nz;) {  // kChunk at a time
                double pc[kChunk];
#pragma unroll
                for (int q = 0; q < kChunk; ++q) pc[q] = kk + q < g.nz ? phi[(int64_t)(kk + q) * nxy + c] : 0.0;
                int q = 0;
                while (q < kChunk && pc[q] >= 1.0) ++q;
                found = q < kChunk;
                kk += q;
            }
            kk = kk < g.nz ? kk : g.nz;
            kfree = kk;
            while (m > 0.0 && kk < g.nz) {
                const int64_t id = (int64_t)kk * nxy + c;
                const bool held = kk == kc;
                const double f0 = held ? fc : phi[id];
                const double w0 = held ? wcc : wc[id];
                const double cap = (1.0 - f0) * w_dep * rho_b * V0;
                const double take = m < cap ? m : cap;
                const double f = take == cap ? 1.0 : f0 + take / (w_dep * rho_b * V0);
                const double before = w0 * rho_b * V0 * f0;
                const double wn = f0 > 0.0 ? (before + take) / (rho_b * V0 * f) : w_dep;
                wc[id] = wn;
                phi[id] = f;
                kc = kk;
                fc = f;
                wcc = wn;
                sum += take;
                m -= take;
                ++kk;
            }
            // every voxel below the last one filled is full
            if (kc >= kfree) kfree = fc < 1.0 ? kc : kc + 1;
            mf[(int64_t)k * nxy + c] = 0.0 + m;  // what finds the column full stays fluid
        }
    }
    if (total && sum > 0.0) atomicAdd(total, sum);
}

// The deposit on tiles of kCols neighbouring columns of at most kTileNz
// voxels: a wave reads whole lines of one plane (or of four, with 16 columns),
// a block's waves take every so manieth.  The voxels whose fluid falls are
// marked in parallel (bit masks per column), as is each column's first non-full
// voxel; one lane per column then replays the fills over its marked voxels in
// increasing height, as the per-thread kernel does.  Fills start at the first
// non-full voxel and rarely climb far: occupancy and compaction of the kWin
// voxels from there are held in LDS (a fill beyond them reads and writes memory
// directly), the voxel being filled in registers, and the next marked voxel's
// mass is on its way meanwhile.  The block writes back what changed.
//
// Bound by the replay's chain, two divisions and a few LDS accesses a fill
// (about 0.4 us), of the column with most fills.  With 64 columns a tile many
// columns share its latency, and 256 x 256 columns are 1,024 blocks, four a CU,
// all at once; with 16 a wave waits for the longest of fewer columns, and few
// columns still give blocks to all CUs.  Under eight wedges, with 16 and 64
// columns a tile: 64 x 64 x 64 voxels 49 and 61 us, 160 x 160 x 60 59 and 63,
// 200 x 200 x 60 74 and 68, 256 x 256 x 128 182 and 137 (without wedges 29 and
// 40, 33 and 42, 40 and 43, 128 and 104).  16 columns with every mass in LDS
// and wedge by wedge for every voxel took 59, 62, 70 and 183 us (without
// wedges 32, 36, 38 and 100), and a thread a column 1,100 us for 200 x 200 x
// 150, which takes 141.
constexpr int64_t kFewColumns = 32768;
constexpr int kTileBlk = 512;
constexpr int kTileNz = 1024;
constexpr int kTilePer = 8;   // planes a wave reads at once
constexpr int kWin = 28;

// kCols: columns of a tile; kMass: planes of masses in LDS at once; kOcc: waves a SIMD
template <int kCols, int kMass, int kOcc>
__global__ void __launch_bounds__(kTileBlk, kOcc) k_convert_deposit_tile(tr_voxel_grid g, double rho_b,
                                                                         double w_dep, WedgeSet ws,
                                                                         const double* rho_p, double* phi,
                                                                         double* wc, double* mf, double* total)
{
#pragma clang fp contract(off)
    constexpr int kRows = kTileBlk / kCols;
    typedef std::conditional_t<kMass <= 32, unsigned, unsigned long long> Bits;
    static_assert(64 % kRows == 0 && kMass % kRows == 0 && 64 % kMass == 0, "planes of a thread and of a mask word");
    __shared__ double P[kWin][kCols], W[kWin][kCols], M[kMass][kCols];
    __shared__ int first_free[kCols], range[kCols][2];
    __shared__ unsigned long long any;  // kMass planes a bit: some column has a marked voxel
    HIP_DYNAMIC_SHARED(unsigned long long, mask)  // [words][kCols]
    const int64_t nxy = (int64_t)g.nx * g.ny;
    const int col = threadIdx.x % kCols, row = threadIdx.x / kCols;
    const int64_t c = (int64_t)blockIdx.x * kCols + col;
    const bool live = c < nxy;
    const int nz = g.nz, words = (nz + 63) / 64;
    const double x = g.origin[0] + ((int)(c % g.nx) + 0.5) * g.l0, y = g.origin[1] + ((int)(c / g.nx) + 0.5) * g.l0;
    for (int w = row; w < words; w += kRows) mask[w * kCols + col] = 0ull;
    if (row == 0) first_free[col] = nz;
    if (threadIdx.x == 0) any = 0ull;
    __syncthreads();
    unsigned long long mine = 0ull;
    for (int k0 = row; k0 < nz; k0 += kRows * kTilePer) {
        double mv[kTilePer], rv[kTilePer];
#pragma unroll
        for (int t = 0; t < kTilePer; ++t) {
            const int k = k0 + t * kRows;
            mv[t] = live && k < nz ? mf[(int64_t)k * nxy + c] : 0.0;
        }
#pragma unroll
        for (int t = 0; t < kTilePer; ++t) {
            const int k = k0 + t * kRows;
            rv[t] = mv[t] > 0.0 ? rho_p[(int64_t)k * nxy + c] : 1.0;
        }
        unsigned fall = 0u;  // bit t: plane k0 + 8 t is marked
#pragma unroll
        for (int t = 0; t < kTilePer; ++t) fall |= (unsigned)(mv[t] > 0.0 && rv[t] == 0.0) << t;
        // (in_wedge_set's test with a wedge's planes in the outer loop: each
        // is read once for all of a thread's voxels, and the next wedge's
        // first one on the way meanwhile)
        for (int r = 0; r < ws.n_ranges; ++r) {
            const WedgeDev* w = ws.base + ws.off[r];
            int n = 0;
            double first[4];
            auto begin = [&](int j) {
                n = w[j].n;
                for (int q = 0; q < 4; ++q) first[q] = w[j].planes[0][q];
            };
            if (ws.cnt[r] > 0) begin(0);
            for (int j = 0; j < ws.cnt[r] && __any(fall != 0u); ++j) {
                const int np = n;
                double pl[4] = {first[0], first[1], first[2], first[3]};
                begin(min(j + 1, ws.cnt[r] - 1));
                unsigned in = np > 0 ? fall : 0u;
                for (int p = 0; p < np && __any(in != 0u); ++p) {
                    if (p > 0)
                        for (int q = 0; q < 4; ++q) pl[q] = w[j].planes[p][q];
                    const double at = pl[0] * x + pl[1] * y;
#pragma unroll
                    for (int t = 0; t < kTilePer; ++t) {
                        const double z = g.origin[2] + (k0 + t * kRows + 0.5) * g.l0;
                        if (at + pl[2] * z - pl[3] > 0.0) in &= ~(1u << t);
                    }
                }
                fall &= ~in;
            }
        }
        for (unsigned f = fall; f; f &= f - 1) {
            const int k = k0 + (__ffs((int)f) - 1) * kRows;
            atomicOr(&mask[(k >> 6) * kCols + col], 1ull << (k & 63));
            mine |= 1ull << (k / kMass);
        }
    }
    if (mine) atomicOr(&any, mine);
    __syncthreads();
    bool work = false;
    for (int w = 0; w < words; ++w) work |= mask[w * kCols + col] != 0ull;
    double mr[kMass / kRows];
    auto bring = [&](unsigned long long planes) {
        const int k0 = planes ? (__ffsll((long long)planes) - 1) * kMass : nz;
#pragma unroll
        for (int t = 0; t < kMass / kRows; ++t) {
            const int k = k0 + row + t * kRows;
            mr[t] = work && k < nz ? mf[(int64_t)k * nxy + c] : 0.0;
        }
    };
    unsigned long long planes = any;
    bring(planes);
    if (work)
        for (int k0 = row; k0 < nz; k0 += kRows * kTilePer) {
            double pv[kTilePer];
#pragma unroll
            for (int t = 0; t < kTilePer; ++t) {
                const int k = k0 + t * kRows;
                pv[t] = k < nz ? phi[(int64_t)k * nxy + c] : 1.0;
            }
            int k = nz;
#pragma unroll
            for (int t = kTilePer - 1; t >= 0; --t)
                if (!(pv[t] >= 1.0)) k = k0 + t * kRows;
            if (k < nz) {
                atomicMin(&first_free[col], k);
                break;  // (the wave's later planes are higher)
            }
        }
    __syncthreads();
    const int ff = first_free[col];
    if (work)
        for (int q = row; q < kWin && ff + q < nz; q += kRows) {
            P[q][col] = phi[(int64_t)(ff + q) * nxy + c];
            W[q][col] = wc[(int64_t)(ff + q) * nxy + c];
        }
    __syncthreads();
    // the replay, kMass planes at a time: lane col of the first wave takes
    // column col, the other waves bring the next planes' masses
    double sum = 0.0, f0 = 1.0, w0 = 0.0;
    int klo = nz, khi = -1, kk = ff;
    const double V0 = g.l0 * g.l0 * g.l0;
    const double unit = w_dep * rho_b * V0;
    // the voxel being filled, its occupancy and compaction: LDS inside the window, memory above it
    auto enter = [&]() {
        if (kk < ff + kWin && kk < nz) {
            f0 = P[kk - ff][col];
            w0 = W[kk - ff][col];
        } else if (kk < nz) {
            f0 = phi[(int64_t)kk * nxy + c];
            w0 = wc[(int64_t)kk * nxy + c];
        }
    };
    if (row == 0 && work) enter();
    for (; planes; planes &= planes - 1) {
        const int k0 = (__ffsll((long long)planes) - 1) * kMass;
#pragma unroll
        for (int t = 0; t < kMass / kRows; ++t) M[row + t * kRows][col] = mr[t];
        __syncthreads();
        bring(planes & (planes - 1));
        if (row == 0) {
            const unsigned long long word = mask[(k0 >> 6) * kCols + col];
            Bits mk = (Bits)(word >> (k0 & 63)) & (Bits)(~0ull >> (64 - kMass)), keep = 0;
            while (mk) {
                const int q = (kMass <= 32 ? __ffs((int)mk) : __ffsll((long long)mk)) - 1;
                mk &= mk - 1;
                double m = M[q][col];
                while (kk < nz && f0 >= 1.0) {
                    ++kk;
                    enter();
                }
                klo = kk < klo ? kk : klo;
                while (m > 0.0 && kk < nz) {
                    const double cap = (1.0 - f0) * w_dep * rho_b * V0;
                    const double take = m < cap ? m : cap;
                    const double f = take == cap ? 1.0 : f0 + take / unit;
                    const double before = w0 * rho_b * V0 * f0;
                    const double wn = f0 > 0.0 ? (before + take) / (rho_b * V0 * f) : w_dep;
                    if (kk < ff + kWin) {
                        W[kk - ff][col] = wn;
                        P[kk - ff][col] = f;
                    } else {
                        wc[(int64_t)kk * nxy + c] = wn;
                        phi[(int64_t)kk * nxy + c] = f;
                    }
                    khi = kk;
                    sum += take;
                    m -= take;
                    f0 = f;
                    w0 = wn;
                    if (m > 0.0) {
                        ++kk;
                        enter();
                    }
                }
                if (m != 0.0) {  // the column is full (or its occupancy no number): what is left stays fluid
                    mf[(int64_t)(k0 + q) * nxy + c] = 0.0 + m;
                    keep |= (Bits)1 << q;
                }
            }
            if (keep) mask[(k0 >> 6) * kCols + col] = word & ~((unsigned long long)keep << (k0 & 63));
        }
        __syncthreads();
    }
    if (row == 0) {
        range[col][0] = klo;
        range[col][1] = khi;
        if (total) {
            for (int o = kCols / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
            if (col == 0 && sum > 0.0) atomicAdd(total, sum);  // one atomic per tile
        }
    }
    __syncthreads();
    if (work) {
        const int klo = range[col][0], khi = range[col][1];
        constexpr unsigned long long every = ~0ull / ((1ull << kRows) - 1);  // every kRows-th bit
        for (int w = 0; w < words; ++w)
            for (unsigned long long mk = mask[w * kCols + col] & (every << row); mk; mk &= mk - 1) {
                const int k = w * 64 + (__ffsll((long long)mk) - 1);
                mf[(int64_t)k * nxy + c] = 0.0;
            }
        for (int q = row; q < kWin; q += kRows) {  // (above the window: written by the fills)
            const int k = ff + q;
            if (k >= klo && k <= khi) {
                phi[(int64_t)k * nxy + c] = P[q][col];
                wc[(int64_t)k * nxy + c] = W[q][col];
            }
        }
    }
}

void launch_surface(const tr_voxel_grid& g, const double* phi, double* h, float* hf, hipStream_t s)
{
    const int64_t nxy = (int64_t)g.nx * g.ny;
    hipLaunchKernelGGL(k_surface, dim3((unsigned)cdiv(nxy, kBlk)), dim3(kBlk), 0, s, g, phi, h, hf);
}

void launch_convert_cut(const tr_voxel_grid& g, double rho_b, const WedgeSet& ws, double* phi, const double* wc,
                        double* mf, double* total, hipStream_t s)
{
    const int64_t nxy = (int64_t)g.nx * g.ny;
    if (total) hipLaunchKernelGGL(k_fill_f64, dim3(1), dim3(64), 0, s, total, (int64_t)1, 0.0);
    const bool few = nxy <= kCutFew;
    hipLaunchKernelGGL(few ? k_convert_cut<32> : k_convert_cut<kBlk>, dim3((unsigned)cdiv(nxy, few ? 32 : kBlk)),
                       dim3(kBlk), 0, s, g, rho_b, ws, phi, wc, mf, total);
}

void launch_convert_deposit(const tr_voxel_grid& g, double rho_b, double w_dep, const WedgeSet& ws,
                            const double* rho_p, double* phi, double* wc, double* mf, double* total, hipStream_t s)
{
    const int64_t nxy = (int64_t)g.nx * g.ny;
    if (total) hipLaunchKernelGGL(k_fill_f64, dim3(1), dim3(64), 0, s, total, (int64_t)1, 0.0);
    if (g.nz <= kTileNz) {
        const bool few = nxy <= kFewColumns;
        const int cols = few ? 16 : 64;
        auto k = few ? k_convert_deposit_tile<16, 64, 4> : k_convert_deposit_tile<64, 16, 8>;
        hipLaunchKernelGGL(k, dim3((unsigned)cdiv(nxy, cols)), dim3(kTileBlk), (size_t)((g.nz + 63) / 64) * cols * 8, s,
                           g, rho_b, w_dep, ws, rho_p, phi, wc, mf, total);
    } else {
        hipLaunchKernelGGL(k_convert_deposit, dim3((unsigned)cdiv(nxy, kBlk)), dim3(kBlk), 0, s, g, rho_b, w_dep, ws,
                           rho_p, phi, wc, mf, total);
    }
}

// ---------------------------------------------------------------------------
// Particle growth from the fluidized mass of the particle's voxel (Eq. eqmotmb):
// bounds summed per voxel, shares applied, the fluid charged per voxel
// ---------------------------------------------------------------------------
__device__ inline int64_t voxel_index(const tr_voxel_grid& g, const float4& xr)
{
#pragma clang fp contract(off)
    const double x[3] = {xr.x, xr.y, xr.z};
    const int dims[3] = {g.nx, g.ny, g.nz};
    int c[3];
    for (int k = 0; k < 3; ++k) {
        const double f = floor((x[k] - g.origin[k]) / g.l0);
        if (!(f >= 0.0 && f < (double)dims[k])) return -1;
        c[k] = (int)f;
    }
    return ((int64_t)c[2] * g.ny + c[1]) * g.nx + c[0];
}

// the most a particle may gain over dt: 3 m d' dt / d, not past d_max
__device__ inline double growth_bound(double km, double r, double dt, double dpm, double d_max)
{
#pragma clang fp contract(off)
    const double m = km * r * r * r;
    const double m_max = km * (0.5 * d_max) * (0.5 * d_max) * (0.5 * d_max);
    double c = 3.0 * m * dpm * dt / (2.0 * r);
    if (m + c > m_max) c = m_max > m ? m_max - m : 0.0;
    return c;
}

__global__ void k_grow_caps(DevBuffers b, EnvDev E, tr_voxel_grid g, double dt, double dpm, double d_max,
                            double* cap_sum)
{
#pragma clang fp contract(off)
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= E.n) return;
    const int sl = E.slot_begin + a;
    const float4 xr = b.xr[sl];
    const int64_t v = voxel_index(g, xr);
    if (v < 0) return;
    const double km = (double)b.rho[sl] * (4.0 / 3.0) * 3.14159265358979323846;
    const double c = growth_bound(km, (double)xr.w, dt, dpm, d_max);
    if (c > 0.0) atomicAdd(&cap_sum[v], c);
}

__global__ void k_grow_apply(DevBuffers b, EnvDev E, tr_voxel_grid g, double dt, double dpm, double d_max,
                             const double* cap_sum, const double* mf, double* used)
{
#pragma clang fp contract(off)
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= E.n) return;
    const int sl = E.slot_begin + a;
    float4 xr = b.xr[sl];
    const int64_t v = voxel_index(g, xr);
    if (v < 0) return;
    const double km = (double)b.rho[sl] * (4.0 / 3.0) * 3.14159265358979323846;
    const double r = xr.w;
    const double c = growth_bound(km, r, dt, dpm, d_max);
    if (!(c > 0.0)) return;
    const double A = mf[v] > 0.0 ? mf[v] : 0.0;
    const double share = cap_sum[v] <= A ? c : c * (A / cap_sum[v]);
    if (!(share > 0.0)) return;
    const double m = km * r * r * r;
    const float r_new = fminf((float)cbrt((m + share) / km), (float)(0.5 * d_max));
    if (!(r_new > xr.w)) return;
    // the fluid pays for what the FP32 radius holds
    const double rn = r_new;
    const double m_new = km * rn * rn * rn;
    atomicAdd(&used[v], m_new - m);
    xr.w = r_new;
    b.xr[sl] = xr;
    vel_at(b.vw, sl).w = (float)(1.0 / m_new);
    angv_at(b.vw, sl).w = (float)(1.0 / (0.4 * m_new * rn * rn));
}

__global__ void k_grow_fluid(int64_t nv, double* mf, const double* used, double* total)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nv) return;
    const double u = used[i];
    if (u > 0.0) {
        mf[i] -= u;
        if (total) atomicAdd(total, u);
    }
}

void launch_grow(const DevBuffers& b, const EnvDev& E, const tr_voxel_grid& g, double dt, double dprime_max,
                 double d_max, double* mf, double* work, double* total, hipStream_t s)
{
    const int64_t nv = (int64_t)g.nx * g.ny * g.nz;
    double* cap_sum = work;
    double* used = work + nv;
    hipLaunchKernelGGL(k_fill_f64, dim3((unsigned)cdiv(2 * nv, kBlk)), dim3(kBlk), 0, s, work, 2 * nv, 0.0);
    if (total) hipLaunchKernelGGL(k_fill_f64, dim3(1), dim3(64), 0, s, total, (int64_t)1, 0.0);
    if (E.n > 0) {
        const unsigned nb = (unsigned)cdiv(E.n, kBlk);
        hipLaunchKernelGGL(k_grow_caps, dim3(nb), dim3(kBlk), 0, s, b, E, g, dt, dprime_max, d_max, cap_sum);
        hipLaunchKernelGGL(k_grow_apply, dim3(nb), dim3(kBlk), 0, s, b, E, g, dt, dprime_max, d_max, cap_sum, mf,
                           used);
    }
    hipLaunchKernelGGL(k_grow_fluid, dim3((unsigned)cdiv(nv, kBlk)), dim3(kBlk), 0, s, nv, mf, used, total);
}

// ---------------------------------------------------------------------------
// Forming new particles from the fluid inside the zones: one thread per
// voxel marks a candidate (the list's order is fixed by the host afterwards),
// then the fluid of each listed voxel pays the mass its FP32 radius holds
// ---------------------------------------------------------------------------
__global__ void k_form_candidates(tr_voxel_grid g, double rho, double d_min, double d_max, double phi_max, WedgeSet ws,
                                  const double* rho_p, const double* u, const double* mf, FormEntry* list,
                                  unsigned long long* count, int64_t cap)
{
#pragma clang fp contract(off)
    const int64_t nxy = (int64_t)g.nx * g.ny, nv = nxy * g.nz;
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= nv) return;
    const double km = rho * 3.14159265358979323846 / 6.0;  // m = km d^3
    const double m_min = km * d_min * d_min * d_min;
    const double f = mf[id];
    if (!(f >= m_min)) return;
    const int k = (int)(id / nxy), j = (int)((id % nxy) / g.nx), i = (int)(id % g.nx);
    const double c[3] = {g.origin[0] + (i + 0.5) * g.l0, g.origin[1] + (j + 0.5) * g.l0, g.origin[2] + (k + 0.5) * g.l0};
    if (!in_wedge_set(ws, c[0], c[1], c[2])) return;
    double d = cbrt(f / km);
    d = d > d_max ? d_max : d;
    const double m = km * d * d * d;
    const double V0 = g.l0 * g.l0 * g.l0;
    if (rho_p[id] / rho + m / (rho * V0) > phi_max) return;  // no room for one more particle
    const unsigned long long slot = atomicAdd(count, 1ull);
    if ((int64_t)slot >= cap) return;
    FormEntry e;
    e.voxel = (double)id;
    for (int q = 0; q < 3; ++q) { e.x[q] = c[q]; e.v[q] = u[3 * id + q]; }
    e.r = 0.5 * d;
    list[slot] = e;
}

// the library's particle mass: FP32 density and radius, FP64 arithmetic
__global__ void k_form_pay(const FormEntry* list, int64_t n, double rho, double* mf)
{
#pragma clang fp contract(off)
    const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= n) return;
    const double r = (double)(float)list[a].r;
    const double m = (double)(float)rho * (4.0 / 3.0) * 3.14159265358979323846 * r * r * r;
    mf[(int64_t)list[a].voxel] -= m;  // one entry per voxel
}

void launch_form_candidates(const tr_voxel_grid& g, double rho, double d_min, double d_max, double phi_max,
                            const WedgeSet& ws, const double* rho_p, const double* u, const double* mf,
                            FormEntry* list, unsigned long long* count, int64_t cap, hipStream_t s)
{
    const int64_t nv = (int64_t)g.nx * g.ny * g.nz;
    hipLaunchKernelGGL(k_fill_f64, dim3(1), dim3(64), 0, s, (double*)count, (int64_t)1, 0.0);  // bits of 0
    hipLaunchKernelGGL(k_form_candidates, dim3((unsigned)cdiv(nv, kBlk)), dim3(kBlk), 0, s, g, rho, d_min, d_max,
                       phi_max, ws, rho_p, u, mf, list, count, cap);
}

void launch_form_pay(const FormEntry* list, int64_t n, double rho, double* mf, hipStream_t s)
{
    if (n > 0) hipLaunchKernelGGL(k_form_pay, dim3((unsigned)cdiv(n, kBlk)), dim3(kBlk), 0, s, list, n, rho, mf);
}

// ---------------------------------------------------------------------------
// Particles at rest outside the zones: their mass joins their voxel's fluid
// (FP64 atomics) and their ids are listed for removal
// ---------------------------------------------------------------------------
__global__ void k_settle(DevBuffers b, EnvDev E, tr_voxel_grid g, double v_rest, WedgeSet ws, double* mf, int* list,
                         unsigned long long* count, double* total)
{
#pragma clang fp contract(off)
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= E.n) return;
    const int sl = E.slot_begin + a;
    const float4 xr = b.xr[sl], vm = vel_at(b.vw, sl);
    const double v[3] = {vm.x, vm.y, vm.z};
    if (!(sqrt((v[0] * v[0] + v[1] * v[1]) + v[2] * v[2]) < v_rest)) return;
    const int64_t vox = voxel_index(g, xr);
    if (vox < 0 || in_wedge_set(ws, xr.x, xr.y, xr.z)) return;
    const double r = xr.w;
    const double m = (double)b.rho[sl] * (4.0 / 3.0) * 3.14159265358979323846 * r * r * r;
    atomicAdd(&mf[vox], m);
    if (total) atomicAdd(total, m);
    list[atomicAdd(count, 1ull)] = b.pid[sl];
}

void launch_settle(const DevBuffers& b, const EnvDev& E, const tr_voxel_grid& g, double v_rest, const WedgeSet& ws,
                   double* mf, int* list, unsigned long long* count, double* total, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill_f64, dim3(1), dim3(64), 0, s, (double*)count, (int64_t)1, 0.0);  // bits of 0
    if (total) hipLaunchKernelGGL(k_fill_f64, dim3(1), dim3(64), 0, s, total, (int64_t)1, 0.0);
    if (E.n > 0)
        hipLaunchKernelGGL(k_settle, dim3((unsigned)cdiv(E.n, kBlk)), dim3(kBlk), 0, s, b, E, g, v_rest, ws, mf, list,
                           count, total);
}

}  // namespace trk


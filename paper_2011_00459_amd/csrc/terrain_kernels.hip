// terrain_kernels.hip -- gfx950 kernels of one agitated-soil particle step.
//
// The step (Algorithm 1 of Servin, Berglund & Nystedt: collision detection,
// the mesoscale contact constraints, the aggregate bodies, the PGS solve and
// the position update) is split into these kernel families:
//   bin/scan/scatter/gather   particles sorted by (env, Morton cell, id)
//   narrow                    sphere-sphere and sphere-boundary contacts with
//                             a pinned FP64 predicate, wave-compacted
//   id count/scatter/sort     canonical contact order (key order)
//   incidence + colour        per-particle incidence lists and a greedy
//                             colouring in splitmix64 priority order
//   rows                      Hertz-mapped SPOOK rows (Eqs. signCoul1-2)
//   warm apply                v* = v + dt g + M^-1 G^T lambda^0
//   pgs                       persistent projected Gauss-Seidel sweeps in
//                             colour order with the residual fused in
//   finish                    body forces (FP64), x += dt v, kinematic poses,
//                             zone aggregates (FP64, Eqs. aggregate_mass ..
//                             aggregate_rot_vel)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <type_traits>

#include "terrain_internal.h"
#include "terrain_geom.h"

namespace trk {

constexpr int kBlk = 256;
constexpr unsigned long long kNoMask = ~0ull;  // no colours sent yet (DevBuffers::cmsg); a full mask is never sent
#ifndef TRK_BARRIER_SPINS
#define TRK_BARRIER_SPINS (1l << 22)
#endif
constexpr long kBarrierSpins = TRK_BARRIER_SPINS;  // bounded wait of a grid barrier

__host__ __device__ inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---------------------------------------------------------------------------
// generic fill and device-wide exclusive scan (out[n] = total)
// ---------------------------------------------------------------------------
__global__ void k_fill_u32(uint32_t* p, uint32_t v, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t st = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += st) p[i] = v;
}

void launch_fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t s)
{
    if (n <= 0) return;
    int grid = (int)std::min<int64_t>(cdiv(n, kBlk), 4096);
    hipLaunchKernelGGL(k_fill_u32, dim3(grid), dim3(kBlk), 0, s, p, v, n);
}

constexpr int kScanItems = 4;
constexpr int kScanTile = kBlk * kScanItems;

__device__ inline uint32_t wave_incl_scan(uint32_t v)
{
    int lane = threadIdx.x & 63;
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    return v;
}

// exclusive block scan of one value per thread; returns the block total via *tot
__device__ inline uint32_t block_excl_scan(uint32_t v, uint32_t* tot)
{
    __shared__ uint32_t wsum[kBlk / 64];
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t inc = wave_incl_scan(v);
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    uint32_t off = 0, all = 0;
    for (int k = 0; k < kBlk / 64; ++k) {
        if (k < w) off += wsum[k];
        all += wsum[k];
    }
    __syncthreads();
    *tot = all;
    return off + inc - v;
}

__global__ void k_scan_reduce(const uint32_t* in, int64_t n, uint32_t* tmp)
{
    int64_t base = (int64_t)blockIdx.x * kScanTile;
    uint32_t s = 0;
    for (int k = 0; k < kScanItems; ++k) {
        int64_t i = base + (int64_t)threadIdx.x * kScanItems + k;
        if (i < n) s += in[i];
    }
    uint32_t tot;
    block_excl_scan(s, &tot);
    if (threadIdx.x == 0) tmp[blockIdx.x] = tot;
}

__global__ void k_scan_top(uint32_t* tmp, int64_t nb)
{
    // single block: exclusive scan of the block totals, total at tmp[nb]
    __shared__ uint32_t carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int64_t base = 0; base < nb; base += kBlk) {
        int64_t i = base + threadIdx.x;
        uint32_t v = i < nb ? tmp[i] : 0u;
        uint32_t tot;
        uint32_t ex = block_excl_scan(v, &tot);
        if (i < nb) tmp[i] = carry + ex;
        __syncthreads();
        if (threadIdx.x == 0) carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) tmp[nb] = carry;
}

// sums: tmp holds the tiles' totals (each block adds those before its own),
// else their exclusive scan
__global__ void k_scan_down(const uint32_t* in, uint32_t* out, int64_t n, const uint32_t* tmp, int64_t nb, int sums)
{
    int64_t base = (int64_t)blockIdx.x * kScanTile;
    uint32_t before = 0;
    if (sums) {
        uint32_t s = 0;
        for (unsigned k = threadIdx.x; k < blockIdx.x; k += kBlk) s += tmp[k];
        block_excl_scan(s, &before);
    } else {
        before = tmp[blockIdx.x];
    }
    uint32_t v[kScanItems];
    uint32_t s = 0;
    for (int k = 0; k < kScanItems; ++k) {
        int64_t i = base + (int64_t)threadIdx.x * kScanItems + k;
        v[k] = i < n ? in[i] : 0u;
        s += v[k];
    }
    uint32_t tot;
    uint32_t ex = block_excl_scan(s, &tot) + before;
    for (int k = 0; k < kScanItems; ++k) {
        int64_t i = base + (int64_t)threadIdx.x * kScanItems + k;
        if (i < n) out[i] = ex;
        ex += v[k];
    }
    if (blockIdx.x == nb - 1 && threadIdx.x == 0) out[n] = before + tot;
}

// one block scans it all
constexpr int kSmallBlk = 1024;
__global__ __launch_bounds__(kSmallBlk) void k_scan_small(const uint32_t* in, uint32_t* out, int n)
{
    __shared__ uint32_t wsum[kSmallBlk / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t carry = 0;
    for (int base = 0; base < n; base += kSmallBlk * kScanItems) {
        const int i = base + (int)threadIdx.x * kScanItems;
        uint32_t v[kScanItems], s = 0;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            v[k] = i + k < n ? in[i + k] : 0u;
            s += v[k];
        }
        const uint32_t inc = wave_incl_scan(s);
        if (lane == 63) wsum[wave] = inc;
        __syncthreads();
        uint32_t off = 0, all = 0;
        for (int w = 0; w < kSmallBlk / 64; ++w) {
            if (w < wave) off += wsum[w];
            all += wsum[w];
        }
        uint32_t ex = carry + off + inc - s;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            if (i + k < n) out[i + k] = ex;
            ex += v[k];
        }
        carry += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) out[n] = carry;
}

int64_t scan_tmp_words(int64_t n) { return cdiv(std::max<int64_t>(n, 1), kScanTile) + 1; }

// Up to 16,384 words by one block (one launch, 5 us against 9 for two); up to
// 8,192 tiles with each block adding the totals before its own (cheaper than
// a launch of one block over them, 12 us at 2,000 tiles).
void launch_scan_u32(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* tmp, hipStream_t s)
{
    if (n <= 4 * kSmallBlk * kScanItems) {
        hipLaunchKernelGGL(k_scan_small, dim3(1), dim3(kSmallBlk), 0, s, in, out, (int)std::max<int64_t>(n, 0));
        return;
    }
    const int64_t nb = cdiv(n, kScanTile);
    const int sums = nb <= 8192 ? 1 : 0;
    hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(kBlk), 0, s, in, n, tmp);
    if (!sums) hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kBlk), 0, s, tmp, nb);
    hipLaunchKernelGGL(k_scan_down, dim3((unsigned)nb), dim3(kBlk), 0, s, in, out, n, tmp, nb, sums);
}

// ---------------------------------------------------------------------------
// small device helpers
// ---------------------------------------------------------------------------
__device__ inline uint32_t env_of(int id, uint32_t id_cap) { return (uint32_t)id / id_cap; }

__device__ inline uint32_t morton(int cx, int cy, int cz, const int bits[3])
{
    // non-uniform interleave: one bit of each axis that still has bits, x first
    uint32_t key = 0;
    int pos = 0;
    int mb = max(bits[0], max(bits[1], bits[2]));
    for (int b = 0; b < mb; ++b) {
        if (b < bits[0]) key |= (uint32_t)((cx >> b) & 1) << pos++;
        if (b < bits[1]) key |= (uint32_t)((cy >> b) & 1) << pos++;
        if (b < bits[2]) key |= (uint32_t)((cz >> b) & 1) << pos++;
    }
    return key;
}

__device__ inline void cell_of(const EnvDev& E, float x, float y, float z, int c[3])
{
    float f[3] = {(x - E.lo[0]) * E.inv_h, (y - E.lo[1]) * E.inv_h, (z - E.lo[2]) * E.inv_h};
    for (int k = 0; k < 3; ++k) {
        float g = fminf(fmaxf(floorf(f[k]), 0.0f), (float)(E.dims[k] - 1));
        c[k] = (int)g;
    }
}

__device__ inline unsigned long long splitmix64(unsigned long long x)
{
    unsigned long long z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Pinned sphere-sphere predicate (FP64, fixed order, no contraction).
__device__ inline bool pair_touch(double xi, double yi, double zi, double ri, double xj, double yj, double zj,
                                  double rj, double kappa_c)
{
#pragma clang fp contract(off)
    double dx = xj - xi, dy = yj - yi, dz = zj - zi;
    double d2 = (dx * dx + dy * dy) + dz * dz;
    double rs = ri + rj;
    double R = rs + (kappa_c > 0.0 ? kappa_c * rs : 0.0);
    return d2 < R * R;
}

// ---------------------------------------------------------------------------
// step begin: world data of shapes, clears, the particles' cells (A1)
// ---------------------------------------------------------------------------
__global__ void k_step_begin(DevBuffers b, StepParams p)
{
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < p.n_particles) {
        float4 x = b.xr[t];
        const EnvDev& E = b.envs[env_of(b.pid[t], p.id_cap)];
        int c[3];
        cell_of(E, x.x, x.y, x.z, c);
        uint32_t key = E.cell_base + morton(c[0], c[1], c[2], E.bits);
        b.pkey[t] = key;
        atomicAdd(&b.cell_count[key], 1u);
    }
    {
        // every counter starts the step at zero except the failure word, into
        // which one thread folds the previous step's flags before clearing them
        uint32_t* w = reinterpret_cast<uint32_t*>(b.cnt);
        constexpr int kOvfWord = (int)(offsetof(Counters, overflow) / 4);
        constexpr int kFailedWord = (int)(offsetof(Counters, failed) / 4);
        for (int k = t; k < (int)(sizeof(Counters) / 4); k += gridDim.x * blockDim.x)
            if (k != kOvfWord && k != kFailedWord) w[k] = 0u;
        if (t == 0) {
            w[kFailedWord] |= w[kOvfWord];
            w[kOvfWord] = 0u;
        }
    }
    if (t < p.n_envs) {
        b.env_stats[t].contacts = 0;
        b.env_stats[t].pairs = 0;
        b.env_stats[t].impacts = 0;
        b.env_ncol[t] = 0;
    }
    if (t < p.n_units) {
        uint32_t* w = reinterpret_cast<uint32_t*>(&b.ustats[t]);
        for (int k = 0; k < (int)(sizeof(UnitStats) / 4); ++k) w[k] = 0u;
    }
    if (t < p.n_shapes) {
#pragma clang fp contract(off)
        ShapeDev& S = b.shapes[t];
        const BodyDev& B = b.bodies[S.body];
        double R[9];
        quat_to_R(B.quat, R);
        for (int k = 0; k < 9; ++k) S.R[k] = R[k];
        for (int k = 0; k < 3; ++k) S.wn[k] = (R[k * 3 + 0] * S.n[0] + R[k * 3 + 1] * S.n[1]) + R[k * 3 + 2] * S.n[2];
        S.wd = S.d + ((S.wn[0] * B.pos[0] + S.wn[1] * B.pos[1]) + S.wn[2] * B.pos[2]);
        for (int k = 0; k < 3; ++k)
            S.wc[k] = B.pos[k] + ((R[k * 3 + 0] * S.off[0] + R[k * 3 + 1] * S.off[1]) + R[k * 3 + 2] * S.off[2]);
    }
}

void launch_step_begin(const DevBuffers& b, const StepParams& p, hipStream_t s)
{
    int n = std::max({(int)(sizeof(Counters) / 4), p.n_shapes, p.n_envs, p.n_units, p.n_particles});
    hipLaunchKernelGGL(k_step_begin, dim3((unsigned)cdiv(n, kBlk)), dim3(kBlk), 0, s, b, p);
}

// ---------------------------------------------------------------------------
// A1-A2: counting sort by cell key, per-cell id order, gather.  The counts
// that the step's counting sorts fill are drained again as they hand out
// places, so that every step finds them at zero.
// ---------------------------------------------------------------------------
__global__ void k_scatter_cells(DevBuffers b, StepParams p)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= p.n_particles) return;
    uint32_t key = b.pkey[i];
    uint32_t slot = b.cell_start[key] + atomicSub(&b.cell_count[key], 1u) - 1u;
    b.perm[slot] = (uint32_t)i;
}

// to the sorted place: the cell's range, in order of id inside it
__global__ void k_gather(DevBuffers b, StepParams p)
{
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= p.n_particles) return;
    const uint32_t i = b.perm[t];
    const uint32_t key = b.pkey[i];
    const uint32_t beg = b.cell_start[key], end = b.cell_start[key + 1];
    const int id = b.pid[i];
    uint32_t s = beg;
    for (uint32_t k = beg; k < end; ++k) s += b.pid[b.perm[k]] < id ? 1u : 0u;
    b.xr2[s] = b.xr[i];
    vel_at(b.vw2, s) = vel_at(b.vw, i);
    angv_at(b.vw2, s) = angv_at(b.vw, i);
    b.rho2[s] = b.rho[i];
    b.pid2[s] = id;
    b.id2slot[id] = (int)s;
}

void launch_sort_particles(const DevBuffers& b, const StepParams& p, const Sizes& z, hipStream_t s)
{
    int n = p.n_particles;
    launch_scan_u32(b.cell_count, b.cell_start, z.NC, b.scan_tmp, s);
    if (n <= 0) return;
    unsigned g = (unsigned)cdiv(n, kBlk);
    hipLaunchKernelGGL(k_scatter_cells, dim3(g), dim3(kBlk), 0, s, b, p);
    hipLaunchKernelGGL(k_gather, dim3(g), dim3(kBlk), 0, s, b, p);
}

// ---------------------------------------------------------------------------
// A3-A4: narrow phase (pairs through the 27 neighbour cells, then the env's
// boundary shapes), compacted per wave
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlk) void k_narrow(DevBuffers b, StepParams p, int64_t cap)
{
    __shared__ int hits[kBlk][kMaxHits + 1];
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    int nh = 0;
    int idi = 0;
    bool ovf = false;
    uint32_t env = 0;
    if (i < p.n_particles) {
        float4 xi = b.xr[i];
        idi = b.pid[i];
        env = env_of(idi, p.id_cap);
        const EnvDev& E = b.envs[env];
        int c[3];
        cell_of(E, xi.x, xi.y, xi.z, c);
        double X = xi.x, Y = xi.y, Z = xi.z, Ri = xi.w;
        // half shell: the own cell's later slots and the 13 cells after it
        // in (z, y, x) order, so that each pair is met once, from the sphere
        // whose cell comes first (the predicate is exactly symmetric)
        for (int dz = 0; dz <= 1; ++dz) {
            int cz = c[2] + dz;
            if (cz >= E.dims[2]) continue;
            for (int dy = dz ? -1 : 0; dy <= 1; ++dy) {
                int cy = c[1] + dy;
                if (cy < 0 || cy >= E.dims[1]) continue;
                for (int dx = (dz || dy) ? -1 : 0; dx <= 1; ++dx) {
                    int cx = c[0] + dx;
                    if (cx < 0 || cx >= E.dims[0]) continue;
                    uint32_t key = E.cell_base + morton(cx, cy, cz, E.bits);
                    uint32_t beg = b.cell_start[key], end = b.cell_start[key + 1];
                    if ((dx | dy | dz) == 0) beg = max(beg, (uint32_t)i + 1);
                    for (uint32_t j = beg; j < end; ++j) {
                        float4 xj = b.xr[j];
                        if (pair_touch(X, Y, Z, Ri, (double)xj.x, (double)xj.y, (double)xj.z, (double)xj.w, p.kappa_c)) {
                            if (nh < kMaxHits) hits[threadIdx.x][nh++] = (int)j;
                            else ovf = true;
                        }
                    }
                }
            }
        }
        for (int sg = E.shape_begin; sg < E.shape_end; ++sg) {
            if (shape_touch(b.shapes[sg], b.hf_pool, X, Y, Z, Ri, p.kappa_c, nullptr)) {
                if (nh < kMaxHits) hits[threadIdx.x][nh++] = -1 - sg;
                else ovf = true;
            }
        }
    }
    // wave-level compaction: one atomic per wave
    int lane = threadIdx.x & 63;
    uint32_t inc = wave_incl_scan((uint32_t)nh);
    uint32_t total = __shfl(inc, 63, 64);
    uint32_t base = 0;
    if (lane == 63 && total > 0) base = atomicAdd(&b.cnt->n_raw, total);
    base = __shfl(base, 63, 64);
    uint32_t off = base + inc - (uint32_t)nh;
    int npairs = 0;
    for (int k = 0; k < nh; ++k) {
        int h = hits[threadIdx.x][k];
        uint64_t idx = (uint64_t)off + (uint64_t)k;
        if (idx >= (uint64_t)cap) { ovf = true; continue; }
        if (h >= 0) {
            // key and pair in id order: (lower id, higher id)
            int idj = b.pid[h];
            const bool first = idi < idj;
            const uint32_t lo = (uint32_t)(first ? idi : idj), hi = (uint32_t)(first ? idj : idi);
            b.rkey[idx] = ((unsigned long long)lo << 32) | hi;
            b.rpair[idx] = first ? make_int2(i, h) : make_int2(h, i);
            ++npairs;
        } else {
            int sg = -1 - h;
            int local = sg - b.envs[env].shape_begin;
            b.rkey[idx] = ((unsigned long long)(uint32_t)idi << 32) | 0x80000000ull | (uint32_t)local;
            b.rpair[idx] = make_int2(h, i);
        }
    }
    // the pair count of the env: one atomic per wave when the wave's particles
    // share an env (same-address atomics from every lane serialise: this one,
    // per lane, took most of the kernel's time on a 50k-sphere bed)
    {
        const uint32_t env0 = __shfl(env, 0, 64);
        if (__ballot(env != env0) == 0ull) {
            unsigned long long t = (unsigned long long)npairs;
            for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
            if (lane == 0 && t) atomicAdd((unsigned long long*)&b.env_stats[env0].pairs, t);
        } else if (npairs) {
            atomicAdd((unsigned long long*)&b.env_stats[env].pairs, (unsigned long long)npairs);
        }
    }
    if (ovf) atomicOr(&b.cnt->overflow, kOvfContacts);
}

void launch_narrow(const DevBuffers& b, const StepParams& p, const Sizes& z, hipStream_t s)
{
    if (p.n_particles <= 0) return;
    hipLaunchKernelGGL(k_narrow, dim3((unsigned)cdiv(p.n_particles, kBlk)), dim3(kBlk), 0, s, b, p, z.C);
}

// ---------------------------------------------------------------------------
// A5: canonical order (counting sort by the lower id, then by key inside
// each id), per-particle incidence lists
// ---------------------------------------------------------------------------
__device__ inline uint32_t n_contacts(const DevBuffers& b, int64_t cap)
{
    uint32_t n = b.cnt->n_raw;
    return n < (uint64_t)cap ? n : (uint32_t)cap;
}

// atomicAdd(&counter[a], 1) for every active lane, as one atomic per run of
// equal a in consecutive lanes (same-address atomics from many lanes
// serialise); returns the lane's old value, as its own atomic would have
// (lanes of a run take consecutive values).  Every lane of the wave calls it.
// drain: the same places handed out from a filled counter, down to zero.
__device__ inline uint32_t wave_run_inc(uint32_t* counter, uint32_t a, bool active, bool drain = false)
{
    const int lane = threadIdx.x & 63;
    const uint32_t prev = __shfl_up(a, 1, 64);
    const bool prev_active = __shfl_up((int)active, 1, 64) != 0;
    const bool head = active && (lane == 0 || !prev_active || prev != a);
    const unsigned long long bound = __ballot(head || !active);
    const unsigned long long later = lane == 63 ? 0ull : bound >> (lane + 1);
    const int len = later ? __builtin_ctzll(later) + 1 : 64 - lane;
    uint32_t old = 0;
    if (head) old = drain ? atomicSub(&counter[a], (uint32_t)len) - (uint32_t)len : atomicAdd(&counter[a], (uint32_t)len);
    const unsigned long long upto = bound & (~0ull >> (63 - lane));
    const int h = 63 - __builtin_clzll(upto | 1ull);
    return __shfl(old, h, 64) + (uint32_t)(lane - h);
}

__global__ void k_id_count(DevBuffers b, int64_t cap)
{
    uint32_t nc = n_contacts(b, cap);
    for (uint32_t c0 = blockIdx.x * blockDim.x; c0 < nc; c0 += gridDim.x * blockDim.x) {
        const uint32_t c = c0 + threadIdx.x;
        const bool on = c < nc;
        (void)wave_run_inc(b.id_count, on ? (uint32_t)(b.rkey[c] >> 32) : 0u, on);
    }
}

__global__ void k_id_scatter(DevBuffers b, int64_t cap)
{
    uint32_t nc = n_contacts(b, cap);
    for (uint32_t c0 = blockIdx.x * blockDim.x; c0 < nc; c0 += gridDim.x * blockDim.x) {
        const uint32_t c = c0 + threadIdx.x;
        const bool on = c < nc;
        const unsigned long long k = on ? b.rkey[c] : 0ull;
        const uint32_t a = (uint32_t)(k >> 32);
        const uint32_t r = wave_run_inc(b.id_count, a, on, true);
        if (on) {
            const uint32_t pos = b.id_start[a] + r;
            b.ckey[pos] = k;
            b.cpair[pos] = b.rpair[c];
        }
    }
}

// Each id's contacts in key order; their number at each of their spheres,
// and the colouring's start values.  Up to kIdRank of them are ranked in
// registers.
constexpr int kIdRank = 8;

__global__ __launch_bounds__(kBlk) void k_id_sort(DevBuffers b, int64_t nid)
{
    int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= nid) return;
    const uint32_t beg = b.id_start[a], end = b.id_start[a + 1], len = end - beg;
    if (len == 0) return;
    if (len <= kIdRank) {
        unsigned long long k[kIdRank];
        int2 pr[kIdRank];
        uint32_t at[kIdRank];
#pragma unroll
        for (int j = 0; j < kIdRank; ++j) {
            k[j] = (uint32_t)j < len ? b.ckey[beg + j] : ~0ull;
            if ((uint32_t)j < len) pr[j] = b.cpair[beg + j];
            at[j] = 0;
        }
#pragma unroll
        for (int j = 1; j < kIdRank; ++j)
#pragma unroll
            for (int i = 0; i < j; ++i) {
                const bool up = k[i] <= k[j];
                at[j] += up ? 1u : 0u;
                at[i] += up ? 0u : 1u;
            }
#pragma unroll
        for (int j = 0; j < kIdRank; ++j)
            if ((uint32_t)j < len) {
                b.ckey[beg + at[j]] = k[j];
                b.cpair[beg + at[j]] = pr[j];
                if (pr[j].x >= 0) atomicAdd(&b.inc_count[pr[j].y], 1u);
            }
    } else {
        for (uint32_t u = beg; u < end; ++u) {
            unsigned long long k = b.ckey[u];
            int2 pr = b.cpair[u];
            uint32_t t = u;
            while (t > beg && b.ckey[t - 1] > k) {
                b.ckey[t] = b.ckey[t - 1];
                b.cpair[t] = b.cpair[t - 1];
                --t;
            }
            b.ckey[t] = k;
            b.cpair[t] = pr;
            if (pr.x >= 0) atomicAdd(&b.inc_count[pr.y], 1u);
        }
    }
    atomicAdd(&b.inc_count[b.id2slot[a]], len);
    for (uint32_t c = beg; c < end; ++c) {
        b.colour[c] = -1;
        b.cmsg[c] = kNoMask;
    }
}

__global__ void k_inc_fill(DevBuffers b, int64_t cap)
{
    uint32_t nc = n_contacts(b, cap);
    for (uint32_t c0 = blockIdx.x * blockDim.x; c0 < nc; c0 += gridDim.x * blockDim.x) {
        const uint32_t c = c0 + threadIdx.x;
        const bool on = c < nc;
        const int2 pr = on ? b.cpair[c] : make_int2(-1, 0);
        const int own = pr.x >= 0 ? pr.x : pr.y, other = pr.x >= 0 ? pr.y : -1;
        const uint32_t r = wave_run_inc(b.inc_count, (uint32_t)own, on, true);
        if (on) b.inc[b.inc_start[own] + r] = c;
        if (other >= 0) b.inc[b.inc_start[other] + atomicSub(&b.inc_count[other], 1u) - 1u] = c;
    }
}

// The block (region) that solves a contact of two regions of one env: the
// parity of the ranks decides, so that a region owns about half of the
// contacts on its surface.
__device__ inline int contact_rank(int ra, int rb)
{
    const int lo = min(ra, rb), hi = max(ra, rb);
    return ((lo ^ hi) & 1) ? lo : hi;
}

__device__ inline int region_of(const EnvDev& E, int slot) { return (slot - E.slot_begin) / E.chunk; }

// Each sphere's incident contacts, in canonical order (inc) and, with the
// other sphere of each, in the colouring's order of decreasing
// (splitmix64(key), key) (pinc).  A thread holds its sphere's contacts in
// registers and ranks them against each other; within an env canonical order
// is key order, so indices break equal hashes.
constexpr int kMaxRank = 16;
constexpr uint32_t kSecond = 0x80000000u;    // pinc: the sphere is the contact's second one
constexpr uint32_t kBoundary = 0x7fffffffu;  // pinc: a boundary in place of the other sphere

__device__ inline uint2 pinc_entry(uint32_t c, int2 pr, int s)
{
    return make_uint2(c, pr.x < 0 ? kBoundary : (pr.x == s ? (uint32_t)pr.y : (uint32_t)pr.x | kSecond));
}

__global__ __launch_bounds__(kBlk) void k_inc_sort(DevBuffers b, int n)
{
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    const uint32_t beg = b.inc_start[s], end = b.inc_start[s + 1], deg = end - beg;
    if (deg <= kMaxRank) {
        uint32_t e[kMaxRank], at[kMaxRank], pat[kMaxRank];
        unsigned long long h[kMaxRank];
        int2 pr[kMaxRank];
#pragma unroll
        for (int j = 0; j < kMaxRank; ++j) e[j] = (uint32_t)j < deg ? b.inc[beg + j] : ~0u;
#pragma unroll
        for (int j = 0; j < kMaxRank; ++j)
            if ((uint32_t)j < deg) pr[j] = b.cpair[e[j]];
#pragma unroll
        for (int j = 0; j < kMaxRank; ++j) {
            h[j] = (uint32_t)j < deg ? splitmix64(b.ckey[e[j]]) : 0ull;
            at[j] = pat[j] = 0;
        }
#pragma unroll
        for (int j = 1; j < kMaxRank; ++j) {
            if (__ballot((uint32_t)j < deg) == 0ull) break;
#pragma unroll
            for (int i = 0; i < j; ++i) {
                const bool up = e[i] < e[j];
                at[j] += up ? 1u : 0u;
                at[i] += up ? 0u : 1u;
                const bool first = (uint32_t)j >= deg || h[i] > h[j] || (h[i] == h[j] && !up);
                pat[j] += first ? 1u : 0u;
                pat[i] += first ? 0u : 1u;
            }
        }
#pragma unroll
        for (int j = 0; j < kMaxRank; ++j)
            if ((uint32_t)j < deg) {
                b.inc[beg + at[j]] = e[j];
                b.pinc[beg + pat[j]] = pinc_entry(e[j], pr[j], s);
            }
        return;
    }
    for (uint32_t u = beg + 1; u < end; ++u) {
        uint32_t v = b.inc[u];
        uint32_t t = u;
        while (t > beg && b.inc[t - 1] > v) {
            b.inc[t] = b.inc[t - 1];
            --t;
        }
        b.inc[t] = v;
    }
    for (uint32_t u = beg; u < end; ++u) {
        const uint32_t v = b.inc[u];
        const unsigned long long h = splitmix64(b.ckey[v]);
        uint32_t t = u;
        // (v is larger than every index before it: it goes before equal hashes)
        while (t > beg && splitmix64(b.ckey[b.pinc[t - 1].x]) <= h) {
            b.pinc[t] = b.pinc[t - 1];
            --t;
        }
        b.pinc[t] = pinc_entry(v, b.cpair[v], s);
    }
}

void launch_canonical(const DevBuffers& b, const StepParams& p, const Sizes& z, hipStream_t s)
{
    unsigned gc = (unsigned)std::min<int64_t>(cdiv(z.C, kBlk), 2048);
    hipLaunchKernelGGL(k_id_count, dim3(gc), dim3(kBlk), 0, s, b, z.C);
    launch_scan_u32(b.id_count, b.id_start, z.NID, b.scan_tmp, s);
    hipLaunchKernelGGL(k_id_scatter, dim3(gc), dim3(kBlk), 0, s, b, z.C);
    hipLaunchKernelGGL(k_id_sort, dim3((unsigned)cdiv(z.NID, kBlk)), dim3(kBlk), 0, s, b, z.NID);
    int n = std::max(p.n_particles, 1);
    launch_scan_u32(b.inc_count, b.inc_start, n, b.scan_tmp, s);
    hipLaunchKernelGGL(k_inc_fill, dim3(gc), dim3(kBlk), 0, s, b, z.C);
    hipLaunchKernelGGL(k_inc_sort, dim3((unsigned)cdiv(n, kBlk)), dim3(kBlk), 0, s, b, n);
}

// ---------------------------------------------------------------------------
// A7: colouring.  Each contact takes the least colour unused by its
// conflicting contacts of higher (splitmix64(key), key) priority: the unique
// Jones-Plassmann result.  Every sphere works through its contacts in order
// of priority (pinc): a contact is coloured when it is the next one of both
// its spheres, with the least colour neither of them has used, and both move
// on.  So a contact costs one look at each end when its turn comes, however
// long the chain before it.  Blocks take contiguous ranges of the sorted
// spheres and keep their state (colours used, next contact) in LDS, where a
// link of a chain takes a few hundred cycles; a contact across two blocks is
// coloured by the block of its second sphere, which the other sends its used
// colours through cmsg and which answers with the colour.  The grid is
// resident at once (blocks wait for each other); waits are bounded.
// Measured against threads that revisited every uncoloured contact and its
// conflicts until all were done: 984 contacts 97 -> 26 us, 152,000 163 -> 64,
// 1.5 million 578 -> 135, 256 beds of 4.1 million 1,471 -> 256 us.
// ---------------------------------------------------------------------------
constexpr int kColChunk = 8;
constexpr int kColBlk = 1024;
constexpr unsigned long long kNextPending = ~0ull;        // the sphere's next contact is not looked up yet
constexpr unsigned long long kNextDone = ~0ull - 1ull;    // no contact left
constexpr uint32_t kAcrossAsk = ~0u, kAcrossAnswer = ~0u - 1u;  // second word of a next contact across blocks

__device__ inline int ld_colour(const int* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A sphere's state: the colours its contacts have (their number is also the
// place of the next contact in pinc), and the next contact (low word) with the
// block's index of its other sphere.  In LDS, or in memory (two words per
// sphere in smask, which the colouring precedes) for scenes too large for it.
struct ColourLds {
    typedef volatile __attribute__((address_space(3))) unsigned long long Word;
    Word *used, *next;
    __device__ ColourLds(unsigned long long* p, int per) : used((Word*)p), next((Word*)p + per) {}
    __device__ unsigned long long get_used(int i) const { return used[i]; }
    __device__ unsigned long long get_next(int i) const { return next[i]; }
    __device__ void set_used(int i, unsigned long long v) const { used[i] = v; }
    __device__ void set_next(int i, unsigned long long v) const { next[i] = v; }
    __device__ void order() const {}  // LDS accesses of a wave stay in order
};
struct ColourMem {
    unsigned long long* m;
    __device__ unsigned long long get(int k) const { return __hip_atomic_load(&m[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ void set(int k, unsigned long long v) const { __hip_atomic_store(&m[k], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ unsigned long long get_used(int i) const { return get(2 * i); }
    __device__ unsigned long long get_next(int i) const { return get(2 * i + 1); }
    __device__ void set_used(int i, unsigned long long v) const { set(2 * i, v); }
    __device__ void set_next(int i, unsigned long long v) const { set(2 * i + 1, v); }
    __device__ void order() const { __builtin_amdgcn_s_waitcnt(0); }
};

template <bool LDS>
__global__ __launch_bounds__(kColBlk) void k_colour(DevBuffers b, int n, int per, int max_pass)
{
    HIP_DYNAMIC_SHARED(unsigned long long, col_state)
    // neighbouring ranges on one XCD (consecutive blocks go to the 8 XCDs in turn)
    const int blk = gridDim.x % kGroups ? (int)blockIdx.x
                                        : (int)((blockIdx.x % kGroups) * (gridDim.x / kGroups) + blockIdx.x / kGroups);
    const int base = min(n, (int)min((int64_t)blk * per, (int64_t)n)), ns = min(per, n - base);
    auto state = [&] {
        if constexpr (LDS) return ColourLds(col_state, per);
        else return ColourMem{(unsigned long long*)(b.smask + base)};
    }();
    for (int i = threadIdx.x; i < ns; i += kColBlk) {
        state.set_used(i, 0ull);
        state.set_next(i, kNextPending);
    }
    state.order();
    __syncthreads();
    bool left = true, ovf = false;
    for (int pass = 0; pass < max_pass && left; ++pass) {
        left = false;
        bool moved = false;
        for (int i = threadIdx.x; i < ns; i += kColBlk) {
            unsigned long long q = state.get_next(i);
            if (q == kNextDone) continue;
            left = true;
            if (q == kNextPending) {
                moved = true;
                const int s = base + i;
                const unsigned long long used = state.get_used(i);
                const uint32_t pos = b.inc_start[s] + (uint32_t)__popcll(used);
                if (pos >= b.inc_start[s + 1]) {
                    state.set_next(i, kNextDone);
                    continue;
                }
                // more contacts than colours (also for the block across, which
                // would take the full mask for none sent)
                if (used == ~0ull) { ovf = true; break; }
                const uint2 en = b.pinc[pos];
                const uint32_t c = en.x;
                if (en.y == kBoundary) {  // conflicts at its sphere only
                    const int col = __builtin_ctzll(~used);
                    b.colour[c] = col;
                    state.set_used(i, used | (1ull << col));
                    continue;
                }
                const int other = (int)(en.y & ~kSecond) - base;
                uint32_t how = (uint32_t)other;
                if (other < 0 || other >= ns) {
                    how = (en.y & kSecond) ? kAcrossAnswer : kAcrossAsk;
                    if (how == kAcrossAsk)
                        __hip_atomic_store(&b.cmsg[c], used, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                q = ((unsigned long long)how << 32) | c;
                state.set_next(i, q);
            }
            const uint32_t c = (uint32_t)q, how = (uint32_t)(q >> 32);
            if (how == kAcrossAsk) {
                const int col = ld_colour(&b.colour[c]);
                if (col < 0) continue;
                state.set_used(i, state.get_used(i) | (1ull << col));
                state.set_next(i, kNextPending);
                moved = true;
                continue;
            }
            unsigned long long theirs;
            if (how == kAcrossAnswer) {
                theirs = __hip_atomic_load(&b.cmsg[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (theirs == kNoMask) continue;
            } else {
                // both ends see a match; the one of the later sphere colours it
                if ((int)how > i) continue;
                const unsigned long long o = state.get_next((int)how);
                if ((uint32_t)o != c || o >= kNextDone) continue;
                theirs = state.get_used((int)how);
            }
            const unsigned long long mine = state.get_used(i), both = mine | theirs;
            if (both == ~0ull) { ovf = true; break; }
            const int col = __builtin_ctzll(~both);
            const unsigned long long bit = 1ull << col;
            __hip_atomic_store(&b.colour[c], col, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            moved = true;
            state.set_used(i, mine | bit);
            if (how != kAcrossAnswer) state.set_used((int)how, theirs | bit);
            state.order();
            state.set_next(i, kNextPending);
            if (how != kAcrossAnswer) state.set_next((int)how, kNextPending);
        }
        left = __ballot(left) != 0ull;
        bool stop = __ballot(ovf) != 0ull;
        if (!stop && __ballot(moved) == 0ull) {
            __builtin_amdgcn_s_sleep(1);
            // (another block gave up?)
            if ((pass & 255) == 255)
                stop = __hip_atomic_load(&b.cnt->overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
        }
        if (stop) {
            left = false;
            break;
        }
    }
    if (ovf) atomicOr(&b.cnt->overflow, kOvfColours);
    if (left) atomicOr(&b.cnt->overflow, kFailColouring);
}

// LDS index of a sphere in its region's block
__device__ inline int lds_index(const EnvDev& E, int slot)
{
    const int t = slot - E.slot_begin;
    return E.lds_off + t % E.chunk;
}

// The colours of a sphere's contacts (all) and of those that another region's
// block solves (away).  A sphere's contacts have distinct colours, so the
// masks give the order of its updates; those of a sphere without an LDS place
// all count as away.
__device__ inline ulonglong2 region_masks(const DevBuffers& b, const EnvDev& E, int s)
{
    const uint32_t beg = b.inc_start[s], end = b.inc_start[s + 1];
    const bool split = E.chunk < E.n;
    const int r = region_of(E, s);
    unsigned long long all = 0, away = 0;
    for (uint32_t t0 = beg; t0 < end; t0 += kColChunk) {
        uint2 e[kColChunk];
        int col[kColChunk];
#pragma unroll
        for (int j = 0; j < kColChunk; ++j) e[j] = b.pinc[min(t0 + j, end - 1)];
#pragma unroll
        for (int j = 0; j < kColChunk; ++j) col[j] = b.colour[e[j].x];
#pragma unroll
        for (int j = 0; j < kColChunk; ++j) {
            if (col[j] < 0 || col[j] >= kMaxColours) continue;  // failed colouring: the step is abandoned
            const unsigned long long bit = 1ull << col[j];
            all |= bit;
            if (!split || e[j].y == kBoundary) continue;
            const int q = region_of(E, (int)(e[j].y & ~kSecond));
            if (q != r && contact_rank(r, q) != r) away |= bit;
        }
    }
    if (lds_index(E, s) >= E.res_cap) away = all;
    return make_ulonglong2(all, away);
}

// of a sphere's update by its contact of colour col: its place in the
// sphere's sequence, and whether the one before (after) it, around the sweep,
// is solved away from the sphere's region
__device__ inline uint32_t seq_place(ulonglong2 m, int col) { return (uint32_t)__popcll(m.x & ((1ull << col) - 1)); }
__device__ inline bool from_away(ulonglong2 m, int col)
{
    const unsigned long long below = m.x & ((1ull << col) - 1);
    return (m.y >> (63 - __builtin_clzll(below ? below : m.x))) & 1;
}
__device__ inline bool to_away(ulonglong2 m, int col)
{
    const unsigned long long above = m.x & ~((2ull << col) - 1);
    return (m.y >> __builtin_ctzll(above ? above : m.x)) & 1;
}

// Solve order.  One block per owner (a region of an env's spheres, see
// EnvDev) lists the contacts it solves: those of its spheres, each once, by
// colour and, within a colour, the shared ones (a body that another block
// updated last, or one without an LDS place) before the private ones; equal
// ones in the order of its spheres and their contacts' priorities, which is
// fixed, so that the residual sums are reproducible.  Which contacts share a
// bucket does not change results.  Two passes over the owner's incidence
// lists: counts per wave and bucket, then positions; a lane's rank among the
// lanes of its wave comes from a ballot match on the bucket's seven bits.
constexpr int kOrdBlk = 1024;
constexpr int kOrdWaves = kOrdBlk / 64;
constexpr int kOrdBuckets = 2 * kMaxColours;
constexpr uint32_t kNotMine = 255, kUncoloured = 254;  // bucket codes of entries without a position

__global__ __launch_bounds__(kOrdBlk) void k_order(DevBuffers b)
{
    __shared__ uint32_t wc[kOrdWaves][kOrdBuckets];
    __shared__ uint32_t bst[kOrdBuckets + 1];
    __shared__ uint32_t base, unit_col;
    const int o = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int sg0 = b.own_idx[o], sg1 = b.own_idx[o + 1];
    for (int k = threadIdx.x; k < kOrdWaves * kOrdBuckets; k += kOrdBlk) wc[0][k] = 0;
    if (threadIdx.x == 0) unit_col = 0;
    for (int sg = sg0; sg < sg1; ++sg) {
        const int4 S = b.own_seg[sg];
        const EnvDev& E = b.envs[S.w];
        if (!E.masks) continue;
        for (int i = threadIdx.x; i < S.y; i += kOrdBlk) b.smask[S.x + i] = region_masks(b, E, S.x + i);
    }
    __syncthreads();
    volatile uint32_t* mine = wc[wave];
    const unsigned long long lower = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    // the lanes of the wave with this lane's bucket
    auto match = [&](uint32_t code) {
        unsigned long long same = ~0ull;
        for (int bit = 0; bit < 8; ++bit) {
            const unsigned long long m = __ballot((code >> bit) & 1);
            same &= ((code >> bit) & 1) ? m : ~m;
        }
        return same;
    };
    for (int sg = sg0; sg < sg1; ++sg) {
        const int4 S = b.own_seg[sg];
        const EnvDev& E = b.envs[S.w];
        const int rank = o - E.own_base, lo = S.x, hi = S.x + S.y;
        const int w1 = lo + (int)((int64_t)S.y * (wave + 1) / kOrdWaves);
        int ncol = 0;
        for (int s0 = lo + (int)((int64_t)S.y * wave / kOrdWaves); s0 < w1; s0 += 64) {
            const int s = s0 + lane;
            uint32_t t = 0, end = 0;
            ulonglong2 ms = make_ulonglong2(1, 0);
            if (s < w1) {
                t = b.inc_start[s];
                end = b.inc_start[s + 1];
                if (E.coded) ms = b.smask[s];
            }
            for (; __ballot(t < end); t += kColChunk) {
                uint2 e[kColChunk];
                uint32_t code[kColChunk];
#pragma unroll
                for (int j = 0; j < kColChunk; ++j) e[j] = t + j < end ? b.pinc[t + j] : make_uint2(~0u, kBoundary);
#pragma unroll
                for (int j = 0; j < kColChunk; ++j) {
                    code[j] = kNotMine;
                    if (e[j].x == ~0u) continue;
                    const int other = (int)(e[j].y & ~kSecond);
                    const bool two = e[j].y != kBoundary, inside = two && other >= lo && other < hi;
                    const bool take = inside ? (e[j].y & kSecond) != 0
                                             : (!two || contact_rank(rank, region_of(E, other)) == rank);
                    if (!take) continue;
                    const int col = b.colour[e[j].x];
                    code[j] = kUncoloured;
                    if (col >= 0 && col < kMaxColours) {
                        bool priv = !E.coded || ((inside || !two) && !from_away(ms, col));
                        if (E.coded && priv && inside) priv = !from_away(b.smask[other], col);
                        code[j] = 2 * (uint32_t)col + (priv ? 1u : 0u);
                        ncol = max(ncol, col + 1);
                    }
                }
#pragma unroll
                for (int j = 0; j < kColChunk; ++j) {
                    const unsigned long long same = match(code[j]);
                    if (code[j] < kOrdBuckets && (same & lower) == 0) mine[code[j]] += (uint32_t)__popcll(same);
                    if (e[j].x != ~0u) b.icode[t + j] = (uint8_t)code[j];
                }
            }
        }
        for (int k = 32; k > 0; k >>= 1) ncol = max(ncol, __shfl_xor(ncol, k, 64));
        if (lane == 0 && ncol) {
            atomicMax(&b.env_ncol[S.w], (uint32_t)ncol);
            atomicMax(&unit_col, (uint32_t)ncol);  // (an owner's envs are of one unit)
        }
    }
    __syncthreads();
    if (threadIdx.x < kOrdBuckets) {
        uint32_t run = 0;
        for (int w = 0; w < kOrdWaves; ++w) {
            const uint32_t n = wc[w][threadIdx.x];
            wc[w][threadIdx.x] = run;
            run += n;
        }
        bst[threadIdx.x] = run;
    }
    __syncthreads();
    if (wave == 0) {
        const uint32_t a = bst[2 * lane], c = bst[2 * lane + 1];
        const uint32_t inc = wave_incl_scan(a + c);
        bst[2 * lane] = inc - a - c;
        bst[2 * lane + 1] = inc - c;
        if (lane == 63) {
            bst[kOrdBuckets] = inc;
            base = atomicAdd(&b.cnt->n_pos, inc);
            if (unit_col) {
                atomicMax(&b.cnt->n_colours, unit_col);
                atomicMax(&b.ustats[b.envs[b.own_seg[sg0].w].unit].colours, unit_col);
            }
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k <= kOrdBuckets; k += kOrdBlk) b.own_start[(size_t)o * kOwnStride + k] = base + bst[k];
    for (int k = threadIdx.x; k < kOrdWaves * kOrdBuckets; k += kOrdBlk) wc[0][k] += base + bst[k % kOrdBuckets];
    __syncthreads();
    for (int sg = sg0; sg < sg1; ++sg) {
        const int4 S = b.own_seg[sg];
        const int w1 = S.x + (int)((int64_t)S.y * (wave + 1) / kOrdWaves);
        for (int s0 = S.x + (int)((int64_t)S.y * wave / kOrdWaves); s0 < w1; s0 += 64) {
            const int s = s0 + lane;
            uint32_t t = 0, end = 0;
            if (s < w1) {
                t = b.inc_start[s];
                end = b.inc_start[s + 1];
            }
            for (; __ballot(t < end); t += kColChunk) {
                uint32_t e[kColChunk], code[kColChunk];
#pragma unroll
                for (int j = 0; j < kColChunk; ++j) {
                    e[j] = t + j < end ? b.pinc[t + j].x : ~0u;
                    code[j] = t + j < end ? b.icode[t + j] : kNotMine;
                }
#pragma unroll
                for (int j = 0; j < kColChunk; ++j) {
                    const unsigned long long same = match(code[j]);
                    if (code[j] < kOrdBuckets) {
                        const uint32_t at = mine[code[j]];
                        b.cpos[e[j]] = at + (uint32_t)__popcll(same & lower);
                        if ((same & lower) == 0) mine[code[j]] = at + (uint32_t)__popcll(same);
                    } else if (code[j] == kUncoloured) {
                        b.cpos[e[j]] = e[j];  // failed colouring: the step is abandoned
                    }
                }
            }
        }
    }
}

// spheres of a colouring block, at least 1,024: chains across blocks cost about
// a microsecond a link
static int colour_range(const StepParams& p, const Sizes& z)
{
    return (int)std::max<int64_t>(kColBlk, cdiv(p.n_particles, z.col_grid));
}
int colour_blocks(const StepParams& p, const Sizes& z) { return (int)cdiv(p.n_particles, colour_range(p, z)); }

void launch_colour(const DevBuffers& b, const StepParams& p, const Sizes& z, hipStream_t s)
{
    if (p.n_particles > 0) {
        const int per = colour_range(p, z);
        const unsigned g = (unsigned)colour_blocks(p, z);
        if (per <= z.col_per)
            hipLaunchKernelGGL(k_colour<true>, dim3(g), dim3(kColBlk), (size_t)per * 16, s, b, p.n_particles, per, 1 << 22);
        else
            hipLaunchKernelGGL(k_colour<false>, dim3(g), dim3(kColBlk), 0, s, b, p.n_particles, per, 1 << 22);
    }
    if (z.n_own > 0) hipLaunchKernelGGL(k_order, dim3((unsigned)z.n_own), dim3(kOrdBlk), 0, s, b);
}

// ---------------------------------------------------------------------------
// A6 + A8: contact rows in colour order, with lambda^0 (cold or previous-step
// impulses matched by key, re-projected onto the tangent plane and onto the
// feasible set).  Geometry in FP64, stored in FP32.
// ---------------------------------------------------------------------------
// lambda_r onto the disk |lambda_r| <= lim
__device__ inline float4 project_roll(float4 Lr, float lim)
{
    float m2 = Lr.x * Lr.x + Lr.y * Lr.y + Lr.z * Lr.z;
    if (m2 > lim * lim) {
        float sc = m2 > 0.f ? lim * rsqrtf(m2) : 0.f;
        Lr.x *= sc; Lr.y *= sc; Lr.z *= sc;
    }
    return Lr;
}

// what k_rows reads and writes beside the rows: the previous-step match, the
// learned start's features and frame
constexpr int kRowsPrev = 1, kRowsFeatures = 2;

// How a row names its bodies.  In a region's rows a sphere of the region by
// its LDS index (kLocal) with whether its state comes from the exchange
// (kFetch: another block updated it last) and whether another block needs it
// next (kPublish); any other sphere by its exchange record.  Elsewhere by the
// sphere's slot.  A boundary at rest as kStill, a moving one (its velocity is
// in rk) as another negative number.
constexpr int kLocal = 1 << 30, kFetch = 1 << 29, kPublish = 1 << 28;
constexpr int kNameMask = kPublish - 1;
constexpr int kStill = (int)0x80000000;

// A contact's start impulse as the velocity changes of its two spheres
// (layout of wrec): J = lambda_n n + lambda_t acts on sphere 2 with +J and
// on sphere 1 with -J; the angular change of a sphere is its lever times
// (n x J), -l2 for sphere 2 and l1 for sphere 1, plus the rolling impulse.
__device__ inline void warm_record(float4 L, float4 a, float l2, int ib, float4 Lr, bool roll, float4* rec)
{
    float J0 = L.x * a.x + L.y, J1 = L.x * a.y + L.z, J2 = L.x * a.z + L.w;
    float lb = -l2, la = a.w;
    float b0 = lb * (a.y * J2 - a.z * J1), b1 = lb * (a.z * J0 - a.x * J2), b2 = lb * (a.x * J1 - a.y * J0);
    float a0 = la * (a.y * J2 - a.z * J1), a1 = la * (a.z * J0 - a.x * J2), a2 = la * (a.x * J1 - a.y * J0);
    if (roll) {
        b0 += Lr.x; b1 += Lr.y; b2 += Lr.z;
        a0 += Lr.x; a1 += Lr.y; a2 += Lr.z;
    }
    rec[0] = make_float4(J0, J1, J2, __int_as_float(ib));
    rec[1] = make_float4(b0, b1, b2, a0);
    rec[2] = make_float4(a1, a2, 0.f, 0.f);
}

__device__ inline void contact_rows(const DevBuffers& b, const StepParams& p, uint32_t c, int flags)
{
    unsigned long long key = b.ckey[c];
    int2 pr = b.cpair[c];
    int ia = pr.x, ib = pr.y;
    float4 x2 = b.xr[ib];
    float4 v2 = vel_at(b.vw, ib);
    double X2[3] = {x2.x, x2.y, x2.z};
    double r2 = x2.w;
    double n[3], delta, l1, l2, dstar, dref, rmin, im1 = 0.0, iI1 = 0.0, un;
    double vk[3] = {0.0, 0.0, 0.0};
    double u1[3] = {0.0, 0.0, 0.0};  // velocity of body 1 at the contact point
    if (ia >= 0) {
        float4 x1 = b.xr[ia];
        float4 v1 = vel_at(b.vw, ia);
        float4 w1 = angv_at(b.vw, ia);
        double r1 = x1.w;
        double e[3] = {X2[0] - x1.x, X2[1] - x1.y, X2[2] - x1.z};
        double d = sqrt(e[0] * e[0] + e[1] * e[1] + e[2] * e[2]);
        if (d > 0.0) { n[0] = e[0] / d; n[1] = e[1] / d; n[2] = e[2] / d; }
        else { n[0] = 0.0; n[1] = 0.0; n[2] = 1.0; }
        delta = (r1 + r2) - d;
        l1 = r1 - 0.5 * delta;
        l2 = r2 - 0.5 * delta;
        dstar = 1.0 / (1.0 / (2.0 * r1) + 1.0 / (2.0 * r2));
        dref = r1 + r2;
        rmin = fmin(r1, r2);
        im1 = v1.w;
        iI1 = w1.w;
        un = n[0] * ((double)v2.x - v1.x) + n[1] * ((double)v2.y - v1.y) + n[2] * ((double)v2.z - v1.z);
        // v1 + w1 x (l1 n)
        u1[0] = (double)v1.x + l1 * ((double)w1.y * n[2] - (double)w1.z * n[1]);
        u1[1] = (double)v1.y + l1 * ((double)w1.z * n[0] - (double)w1.x * n[2]);
        u1[2] = (double)v1.z + l1 * ((double)w1.x * n[1] - (double)w1.y * n[0]);
    } else {
        int sg = -1 - ia;
        const ShapeDev& S = b.shapes[sg];
        ShapeHit hit;
        shape_touch(S, b.hf_pool, X2[0], X2[1], X2[2], r2, p.kappa_c, &hit);
        delta = hit.delta;
        n[0] = hit.n[0]; n[1] = hit.n[1]; n[2] = hit.n[2];
        l1 = 0.0;
        l2 = r2 - 0.5 * delta;
        dstar = 2.0 * r2;
        dref = 2.0 * r2;
        rmin = r2;
        const BodyDev& B = b.bodies[S.body];
        double pc[3] = {X2[0] - l2 * n[0], X2[1] - l2 * n[1], X2[2] - l2 * n[2]};
        double arm[3] = {pc[0] - B.pos[0], pc[1] - B.pos[1], pc[2] - B.pos[2]};
        vk[0] = B.linvel[0] + (B.angvel[1] * arm[2] - B.angvel[2] * arm[1]);
        vk[1] = B.linvel[1] + (B.angvel[2] * arm[0] - B.angvel[0] * arm[2]);
        vk[2] = B.linvel[2] + (B.angvel[0] * arm[1] - B.angvel[1] * arm[0]);
        un = n[0] * ((double)v2.x - vk[0]) + n[1] * ((double)v2.y - vk[1]) + n[2] * ((double)v2.z - vk[2]);
        u1[0] = vk[0]; u1[1] = vk[1]; u1[2] = vk[2];
    }
    // Hertz stiffness and the row scaled to unit Jacobian
    double kn = p.Estar * sqrt(dstar) / 3.0;
    double de = fmax(delta, p.kappa_min * dref);
    double eps = 4.0 / (5.0 * kn * sqrt(de));
    double Sig = p.sig_coef * eps;
    double q = p.a_coef * (0.8 * delta) + p.b_coef * un;
    double im2 = v2.w, iI2 = angv_at(b.vw, ib).w;
    double Wn = im1 + im2;
    double Wt = im1 + im2 + l1 * l1 * iI1 + l2 * l2 * iI2;
    double Dn = Wn + Sig;
    double Dt = Wt + (double)p.gamma_dt;
    double lo = -p.lo_coef * rmin * rmin;

    // warm start: previous-step impulses of the same key
    float4 L = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 Lr = make_float4(0.f, 0.f, 0.f, 0.f);
    bool persistent = false;
    if (flags & kRowsPrev) {
        uint32_t a = (uint32_t)(key >> 32);
        uint32_t beg = b.pid_start[a], end = b.pid_start[a + 1];
        for (uint32_t t = beg; t < end; ++t)
            if (b.pkeyc[t] == key) {
                L = b.plam[t];
                if (p.mu_r > 0.f) Lr = b.plamr[t];
                persistent = true;
                break;
            }
    }
    uint32_t pos = b.cpos[c];
    // learned-start features (12), contact frame and impulse scale, in FP64
    if (flags & kRowsFeatures) {
        float4 w2 = angv_at(b.vw, ib);
        double u[3];
        u[0] = ((double)v2.x - l2 * ((double)w2.y * n[2] - (double)w2.z * n[1])) - u1[0];
        u[1] = ((double)v2.y - l2 * ((double)w2.z * n[0] - (double)w2.x * n[2])) - u1[1];
        u[2] = ((double)v2.z - l2 * ((double)w2.x * n[1] - (double)w2.y * n[0])) - u1[2];
        double unf = (n[0] * u[0] + n[1] * u[1]) + n[2] * u[2];
        double ut[3] = {u[0] - unf * n[0], u[1] - unf * n[1], u[2] - unf * n[2]};
        double utm = sqrt((ut[0] * ut[0] + ut[1] * ut[1]) + ut[2] * ut[2]);
        double lp[3] = {L.y, L.z, L.w};
        double lpn = (n[0] * lp[0] + n[1] * lp[1]) + n[2] * lp[2];
        for (int k = 0; k < 3; ++k) lp[k] -= lpn * n[k];
        double t1[3];
        if (utm > 1e-12) {
            for (int k = 0; k < 3; ++k) t1[k] = ut[k] / utm;
        } else {
            double lm = sqrt((lp[0] * lp[0] + lp[1] * lp[1]) + lp[2] * lp[2]);
            if (lm > 0.0) {
                for (int k = 0; k < 3; ++k) t1[k] = lp[k] / lm;
            } else {
                int k0 = 0;
                for (int k = 1; k < 3; ++k) if (fabs(n[k]) < fabs(n[k0])) k0 = k;
                double ax[3] = {0.0, 0.0, 0.0};
                ax[k0] = 1.0;
                double dn = (ax[0] * n[0] + ax[1] * n[1]) + ax[2] * n[2];
                for (int k = 0; k < 3; ++k) t1[k] = ax[k] - dn * n[k];
                double sm = sqrt((t1[0] * t1[0] + t1[1] * t1[1]) + t1[2] * t1[2]);
                for (int k = 0; k < 3; ++k) t1[k] /= sm;
            }
        }
        double t2[3] = {n[1] * t1[2] - n[2] * t1[1], n[2] * t1[0] - n[0] * t1[2], n[0] * t1[1] - n[1] * t1[0]};
        double ls = (1.0 / Wn) * p.gdt;
        double rbar = ia >= 0 ? 0.5 * ((double)b.xr[ia].w + r2) : r2;
        float* f = b.feat + (size_t)pos * 12;
        f[0] = (float)(delta / rbar);
        f[1] = (float)(unf / p.gdt);
        f[2] = (float)(utm / p.gdt);
        f[3] = (float)((double)L.x / ls);
        f[4] = (float)(((lp[0] * t1[0] + lp[1] * t1[1]) + lp[2] * t1[2]) / ls);
        f[5] = (float)(((lp[0] * t2[0] + lp[1] * t2[1]) + lp[2] * t2[2]) / ls);
        f[6] = ia >= 0 ? (float)((double)b.pdepth[ia] / rbar) : 0.0f;
        f[7] = (float)((double)b.pdepth[ib] / rbar);
        f[8] = ia >= 0 ? (float)((double)b.xr[ia].w / p.r_ref) : 0.0f;
        f[9] = (float)(r2 / p.r_ref);
        f[10] = ia >= 0 ? 0.0f : 1.0f;
        f[11] = persistent ? 1.0f : 0.0f;
        b.frm1[pos] = make_float4((float)t1[0], (float)t1[1], (float)t1[2], (float)ls);
        // (the solve unit beside t2, for the check of the network's output)
        b.frm2[pos] = make_float4((float)t2[0], (float)t2[1], (float)t2[2],
                                  __int_as_float(b.envs[env_of((int)(key >> 32), p.id_cap)].unit));
    }
    float nf[3] = {(float)n[0], (float)n[1], (float)n[2]};
    if (p.warm == TR_WARM_COLD) L = make_float4(0.f, 0.f, 0.f, 0.f);
    {
        float ln = fmaxf(L.x, (float)lo);
        float tn = nf[0] * L.y + nf[1] * L.z + nf[2] * L.w;
        float t0 = L.y - tn * nf[0], t1 = L.z - tn * nf[1], t2 = L.w - tn * nf[2];
        float lim = p.mu * fabsf(ln);
        float m2 = t0 * t0 + t1 * t1 + t2 * t2;
        if (m2 > lim * lim) {
            float sc = m2 > 0.f ? lim * rsqrtf(m2) : 0.f;
            t0 *= sc; t1 *= sc; t2 *= sc;
        }
        L = make_float4(ln, t0, t1, t2);
    }
    b.r0[pos] = make_float4(nf[0], nf[1], nf[2], (float)l1);
    b.r1[pos] = make_float4((float)l2, (float)(1.0 / Dn), (float)(1.0 / Dt), (float)Sig);
    // the bodies as the solve names them, and the contact's place in the
    // sequence of updates of each (with the sequence's length)
    const EnvDev& E = b.envs[env_of((int)(key >> 32), p.id_cap)];
    const int col = E.masks ? b.colour[c] : 0;
    int na = ib, nb = ib;
    uint32_t seq = 0;
    if (E.masks) {
        const int rb = region_of(E, ib), ra = ia >= 0 ? region_of(E, ia) : rb;
        const int rank = ra == rb ? rb : contact_rank(ra, rb);
        auto name = [&](int sl, int r, uint32_t shift) {
            const ulonglong2 m = b.smask[sl];
            seq |= (seq_place(m, col) << shift) | ((uint32_t)__popcll(m.x) << (16 + shift));
            if (!E.coded) return sl;
            const int li = lds_index(E, sl);
            if (r != rank || li >= E.res_cap) return E.x0 + r * E.xstride + li;
            return kLocal | li | (from_away(m, col) ? kFetch : 0) | (to_away(m, col) ? kPublish : 0);
        };
        nb = name(ib, rb, 8);
        if (ia >= 0) na = name(ia, ra, 0);
        b.seq[pos] = seq;
        b.rm[pos] = make_float4((float)im1, (float)iI1, (float)im2, (float)iI2);
    } else if (ia >= 0) {
        na = ia;
    }
    if (ia < 0) {
        const bool still = (float)vk[0] == 0.f && (float)vk[1] == 0.f && (float)vk[2] == 0.f;
        na = still ? kStill : -1;
        if (!still) b.rk[pos] = make_float4((float)vk[0], (float)vk[1], (float)vk[2], 0.f);
    }
    b.r2[pos] = make_float4((float)q, (float)lo, __int_as_float(na), __int_as_float(nb));
    b.lam[pos] = L;
    b.lam0[pos] = L;
    if (p.v_imp > 0.f) {
        // impact stage (before the main solve): a contact whose start-of-step
        // normal velocity approaches faster than v_imp gets the Newton law
        // G_n v+ = -e G_n v-, every other contact G_n v+ >= 0; no compliance,
        // regularisation or cohesion
        const bool impact = un < -(double)p.v_imp;
        b.ri1[pos] = make_float4((float)l2, (float)(1.0 / Wn), (float)(1.0 / Wt), 0.f);
        b.ri2[pos] = make_float4(impact ? (float)(-(double)p.restitution * un) : 0.f, 0.f, __int_as_float(na),
                                 __int_as_float(nb));
        b.qg[pos] = (float)(p.a_coef * (0.8 * delta));
        if (impact) {
            atomicAdd(&b.env_stats[env_of((int)(key >> 32), p.id_cap)].impacts, 1ull);
            atomicOr(&b.ustats[E.unit].imp_any, 1u);
        }
    }
    if (p.mu_r > 0.f) {
        // rolling row (Eq. signCoul3): 1/(1/I_1 + 1/I_2), r mu_r with r the
        // smaller radius, the kinematic body of a boundary contact; the start
        // impulse projected onto |lambda_r| <= r mu_r |lambda_n|
        float rlim = (float)((double)p.mu_r * rmin);
        int kb = ia >= 0 ? -1 : b.shapes[-1 - ia].body;
        b.r3[pos] = make_float4((float)(1.0 / (iI1 + iI2)), rlim, __int_as_float(kb), 0.f);
        if (p.warm == TR_WARM_COLD) Lr = make_float4(0.f, 0.f, 0.f, 0.f);
        Lr.w = 0.f;
        b.lamr0[pos] = Lr;  // unprojected: the start's lambda_n decides the bound
        Lr = project_roll(Lr, rlim * fabsf(L.x));
        b.lamr[pos] = Lr;
    }
    warm_record(L, make_float4(nf[0], nf[1], nf[2], (float)l1), (float)l2, ib, Lr, p.mu_r > 0.f, b.wrec + 3 * (size_t)c);
}

__global__ void k_rows(DevBuffers b, StepParams p, int64_t cap, int flags)
{
    if (b.cnt->overflow) return;
    const uint32_t nc = n_contacts(b, cap);
    for (uint32_t c = blockIdx.x * blockDim.x + threadIdx.x; c < nc; c += gridDim.x * blockDim.x)
        contact_rows(b, p, c, flags);
}

// Blocks of a kernel over the contacts, whose number the host does not know:
// the capacity may be ten times it, and 150,000 blocks that find nothing take
// 30 us to come and go.
unsigned contact_grid(int64_t cap) { return (unsigned)std::min<int64_t>(cdiv(cap, kBlk), 16384); }

void launch_rows(const DevBuffers& b, const StepParams& p, const Sizes& z, bool have_prev, bool features,
                 hipStream_t s)
{
    const int flags = (have_prev ? kRowsPrev : 0) | (features ? kRowsFeatures : 0);
    hipLaunchKernelGGL(k_rows, dim3(contact_grid(z.C)), dim3(kBlk), 0, s, b, p, z.C, flags);
}

// Impact stage set-up: the stage's impulses start at zero, and the rows of an
// env without impacts do nothing (zero inverse masses: the stage leaves that
// env as it is, as if solved alone).
__global__ void k_impact_prep(DevBuffers b, StepParams p, int64_t cap)
{
    uint32_t nc = n_contacts(b, cap);
    uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nc) return;
    if (b.cnt->overflow) return;
    const uint32_t pos = b.cpos[c];
    b.lami[pos] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (p.mu_r > 0.f) b.lamri[pos] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (b.env_stats[env_of((int)(b.ckey[c] >> 32), p.id_cap)].impacts == 0) {
        float4 r = b.ri1[pos];
        b.ri1[pos] = make_float4(r.x, 0.f, 0.f, 0.f);
    }
}

// After the impact stage: the main rows' velocity term from the post-impact
// velocities, q = qg + Upsilon G_n v+ (envs with impacts; the others keep q).
__global__ void k_impact_q(DevBuffers b, StepParams p, int64_t cap)
{
    uint32_t nc = n_contacts(b, cap);
    uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nc) return;
    if (b.cnt->overflow) return;
    if (b.env_stats[env_of((int)(b.ckey[c] >> 32), p.id_cap)].impacts == 0) return;
    const uint32_t pos = b.cpos[c];
    float4 q = b.r2[pos];
    const int ia = b.cpair[c].x, ib = b.cpair[c].y;
    const float4 a = b.r0[pos], v2 = vel_at(b.vw, ib);
    double v1[3];
    if (ia >= 0) {
        const float4 t = vel_at(b.vw, ia);
        v1[0] = t.x; v1[1] = t.y; v1[2] = t.z;
    } else {
        const bool still = __float_as_int(q.z) == kStill;
        const float4 k = still ? make_float4(0.f, 0.f, 0.f, 0.f) : b.rk[pos];
        v1[0] = k.x; v1[1] = k.y; v1[2] = k.z;
    }
    double un = ((double)a.x * ((double)v2.x - v1[0]) + (double)a.y * ((double)v2.y - v1[1])) +
                (double)a.z * ((double)v2.z - v1[2]);
    q.x = (float)((double)b.qg[pos] + p.b_coef * un);
    b.r2[pos] = q;
}

void launch_impact_stage(const DevBuffers& b, const StepParams& p, const Sizes& z, hipStream_t s)
{
    if (!(p.v_imp > 0.f)) return;
    const dim3 g((unsigned)cdiv(z.C, kBlk));
    hipLaunchKernelGGL(k_impact_prep, g, dim3(kBlk), 0, s, b, p, z.C);
    DevBuffers bi = b;
    bi.r1 = b.ri1;
    bi.r2 = b.ri2;
    bi.lam = b.lami;
    bi.lamr = b.lamri;
    StepParams pi = p;
    pi.gamma_dt = 0.f;
    launch_pgs(bi, pi, z, s, -1, kSlotImpact);
    hipLaunchKernelGGL(k_impact_q, g, dim3(kBlk), 0, s, b, p, z.C);
}

// ---------------------------------------------------------------------------
// v* = v + dt g + M^-1 G^T lambda^0, gathered per particle over its sorted
// incidence list (fixed order) from the contacts' records in canonical order
// (one 32 or 48 B record per incident contact)
// ---------------------------------------------------------------------------
// Before a solve: its counters and flags cleared, and the exchange record of a
// sphere that uses one at version 0.
__device__ inline void solve_begin(const DevBuffers& b, int t, int n_envs, int n_flags)
{
    if (t < kGroups) { b.cnt->bar[t][0] = 0; b.cnt->bar[t][1] = 0; }
    if (t < n_envs) { b.env_bar[(size_t)t * 16] = 0; b.env_bar[(size_t)t * 16 + 1] = 0; }
    if (t < n_flags) b.rflags[t] = 0;
}
__device__ inline void exchange_begin(const DevBuffers& b, const StepParams& p, int s, float4 v, float4 w)
{
    const EnvDev& E = b.envs[env_of(b.pid[s], p.id_cap)];
    if (!E.coded || b.smask[s].y == 0) return;
    const int64_t x = E.x0 + (int64_t)region_of(E, s) * E.xstride + lds_index(E, s);
    v.w = w.w = 0.f;  // version 0
    b.xw[2 * x] = v;
    b.xw[2 * x + 1] = w;
}

__global__ void k_warm_apply(DevBuffers b, StepParams p, int n_envs, int n_flags)
{
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    solve_begin(b, s, n_envs, n_flags);
    if (s >= p.n_particles) return;
    if (b.cnt->overflow) return;
    const bool roll = p.mu_r > 0.f;
    float4 v = vel_at(b.vw, s), w = angv_at(b.vw, s);
    v.x += p.dt * p.g[0];
    v.y += p.dt * p.g[1];
    v.z += p.dt * p.g[2];
    uint32_t beg = b.inc_start[s], end = b.inc_start[s + 1];
    for (uint32_t t = beg; t < end; ++t) {
        const float4* r = b.wrec + 3 * (size_t)b.inc[t];
        float4 R0 = r[0], R1 = r[1];
        if (!roll && R0.x == 0.f && R0.y == 0.f && R0.z == 0.f) continue;
        float sgn, W0, W1, W2;
        if (__float_as_int(R0.w) == s) { sgn = 1.f; W0 = R1.x; W1 = R1.y; W2 = R1.z; }
        else {
            float4 R2 = r[2];
            sgn = -1.f; W0 = R1.w; W1 = R2.x; W2 = R2.y;
        }
        v.x += sgn * v.w * R0.x; v.y += sgn * v.w * R0.y; v.z += sgn * v.w * R0.z;
        w.x += sgn * w.w * W0; w.y += sgn * w.w * W1; w.z += sgn * w.w * W2;
    }
    vel_at(b.vw, s) = v;
    angv_at(b.vw, s) = w;
    exchange_begin(b, p, s, v, w);
}

// the records again from the colour-ordered impulses and rows, after a
// kernel other than k_rows has set the start impulses
__global__ void k_warm_rec(DevBuffers b, StepParams p, int64_t cap)
{
    uint32_t nc = n_contacts(b, cap);
    uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nc) return;
    if (b.cnt->overflow) return;
    const uint32_t pos = b.cpos[c];
    const bool roll = p.mu_r > 0.f;
    warm_record(b.lam[pos], b.r0[pos], b.r1[pos].x, b.cpair[c].y,
                roll ? b.lamr[pos] : make_float4(0.f, 0.f, 0.f, 0.f), roll, b.wrec + 3 * (size_t)c);
}

void launch_warm_apply(const DevBuffers& b, const StepParams& p, const Sizes& z, bool rebuild, hipStream_t s)
{
    if (rebuild) hipLaunchKernelGGL(k_warm_rec, dim3((unsigned)cdiv(z.C, kBlk)), dim3(kBlk), 0, s, b, p, z.C);
    const int ne = z.pgs_mode == kModePerEnv ? z.n_envs : 0;
    const int n = std::max({kGroups, ne, z.n_flags, p.n_particles});
    hipLaunchKernelGGL(k_warm_apply, dim3((unsigned)cdiv(n, kBlk)), dim3(kBlk), 0, s, b, p, ne, z.n_flags);
}

// ---------------------------------------------------------------------------
// A9: persistent projected Gauss-Seidel.  Sweeps x colours; inside a colour
// no two contacts share a dynamic particle, so every contact updates its two
// bodies without atomics, and any schedule of a colour's contacts gives the
// same result.
//
// A solve is run by one block or by a cluster of blocks.  Each block owns a
// region: a contiguous range of the solve's Morton-sorted spheres, kept in its
// LDS for the whole solve, and the contacts k_order gave it.  A sphere on the
// region's surface is also updated by the neighbour that owns the contact
// across; its state then goes through a record of the exchange array: the
// block whose update precedes one solved elsewhere publishes the state there,
// and the block that needs it polls the record.  Each 16 B half of a record
// carries the number of updates it has seen beside its three components, so
// that one load brings the state and says whether it is the awaited one: no
// flags, no drained stores, no barrier between blocks.  (That rests on a
// lane's aligned 16 B store being seen whole or not at all by another block's
// 16 B load, which no document promises.  Measured: 1.2e10 loads of records
// that other blocks kept rewriting, across XCDs and inside one, written through
// and not, saw 7.5e9 new versions, none half written and none out of order.)
// Every version has one
// reader, which writes the next, so a record is never overwritten unread; and
// a block waits only for updates of earlier phases, so that waits end as long
// as every block is resident (they are bounded all the same).
//
// Records are written through to where the neighbours read them: the XCD's
// L2 (ordinary stores) when the cluster sits on one XCD, else memory
// (device-scope stores).  They are read with device-scope (sc1) loads, which
// miss the per-CU L1; measured, L1-hit loads return data another CU of the
// XCD has already replaced.  Consecutive blocks of a launch go to the 8 XCDs
// in turn, so a cluster whose blocks are congruent mod 8 shares one XCD; it
// checks that once per launch and writes through to memory otherwise.
//
// Within a phase (one colour) the contacts that wait are taken by the block's
// last waves while the others update contacts whose bodies are all in LDS;
// a workgroup barrier ends the phase.
//
// What LDS has left beside the bodies holds the block's rows and impulses, or
// its impulses alone, when they fit whole (blocks of up to about 600 and 2,000
// spheres); blocks of 1,024 threads have no registers for the extra code.
//
// Measured (MI355X, PGS per launch) against clusters that kept every body in
// memory and met at a counter barrier after every colour: a 50,000-sphere bed
// of 150 sweeps 7.16 -> 2.05 ms (2.36 with rows and impulses in memory), a
// 500,000-sphere one of 200 sweeps 24.6 -> 7.9 ms (8.5), a 300-sphere column
// of 50 sweeps 0.74 -> 0.29 ms (0.32), one of 1,000 spheres to 1e-3 4.9 ->
// 3.0 ms (3.5).  A phase is bound by its chain: about 170 instructions issued
// by one wave a SIMD, the bodies out of LDS and back, the barrier (0.65 us on
// one block of a few hundred spheres), or the hand-over (1.1 us within an
// XCD, 1.4 us across), and from about 2,000 spheres a block by instruction
// issue.
//
// Contact c of a colour is always handled by the same thread, so its rows
// (read-only) and impulses (thread-owned) use the ordinary caches, and the
// rows of the next phase are in flight while the block waits.  The residual
// R_k = ||d lambda||_D / ||lambda||_D of each sweep is reduced per block in a
// fixed order and combined identically by every block of the cluster, which
// then all take the same stopping decision.
// ---------------------------------------------------------------------------
// waves of a block of the grouped, spread and small per-env solves: the wide
// ones for regions of more than kWideRegion spheres, whose colours have more
// contacts than 512 threads (300,000 spheres on all XCDs 3.04 -> 2.58 ms,
// 500,000 7.9 -> 7.5, eight rolling columns of 1,000 1.04 -> 0.95; a column of
// 300 0.293 -> 0.302; with 12 waves 450,000 spheres 3.46 -> 3.52)
constexpr int kPgsWaves = 8, kPgsWide = 10;
constexpr int kCoherent = 16;  // cache-policy bits of a device-scope (sc1) access

__device__ inline __amdgpu_buffer_rsrc_t raw_rsrc(const void* p)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, 0x7fffffff, 0x00020000);
}
// (exchange records may reach 4 GiB)
__device__ inline __amdgpu_buffer_rsrc_t exchange_rsrc(const void* p)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)0xffffffff, 0x00020000);
}
template <int AUX>
__device__ inline float4 ld_body(__amdgpu_buffer_rsrc_t r, int idx)
{
    return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, idx * 16, 0, AUX));
}
template <int AUX>
__device__ inline void st_body(__amdgpu_buffer_rsrc_t r, int idx, float4 v)
{
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), r, idx * 16, 0, AUX);
}

// XCD (accelerator complex die) this wave runs on
__device__ inline unsigned xcc_id() { return __builtin_amdgcn_s_getreg((3 << 11) | 20) & 0xf; }

// Bounded wait for a barrier counter to reach target; false on timeout or
// when another block has reported a failed barrier.
__device__ inline bool wait_counter(Counters* cnt, uint32_t* counter, unsigned target)
{
    long spins = 0;
    while (__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
        __builtin_amdgcn_s_sleep(1);
        if ((++spins & 1023) == 0 &&
            (__hip_atomic_load(&cnt->overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kFailBarrier))
            return false;
        if (spins > kBarrierSpins) {
            atomicOr(&cnt->overflow, kFailBarrier);
            return false;
        }
    }
    return true;
}

// Cluster barrier of the counter-ordered solve on counter[0] (zeroed before
// the launch).  Arrive drains this block's stores; wait returns false when
// the barrier failed.
__device__ inline void cluster_arrive(uint32_t* counter)
{
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline bool cluster_wait(Counters* cnt, uint32_t* counter, unsigned target, int& flag)
{
    if (threadIdx.x == 0) flag = wait_counter(cnt, counter, target) ? 1 : 0;
    __syncthreads();
    return flag != 0;
}

// First barrier of a launch: every block of the cluster sets the bit of its
// XCD in counter[1] (zeroed before the launch).  The round-robin dispatch
// puts blocks congruent mod 8 on one XCD, but which XCD depends on the
// launches before, so only "one XCD for the whole cluster" is checked.
// Returns 1 for XCD-local accesses, 2 for write-through ones, 0 when the
// barrier failed; uniform over the cluster.
__device__ inline int cluster_placement(Counters* cnt, uint32_t* counter, unsigned size, int& flag)
{
    if (threadIdx.x == 0) {
        __hip_atomic_fetch_or(&counter[1], 1u << xcc_id(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_waitcnt(0);
        __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        flag = 0;
        if (wait_counter(cnt, counter, size)) {
            uint32_t xcds = __hip_atomic_load(&counter[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            flag = __popc(xcds) == 1 ? 1 : 2;
        }
    }
    __syncthreads();
    return flag;
}

// Every flag of f[0 .. K) at least want, seen by the whole wave; bounded like
// wait_counter.
__device__ inline bool wait_flags(Counters* cnt, const uint32_t* f, unsigned K, uint32_t want)
{
    const unsigned lane = threadIdx.x & 63;
    for (long spins = 1;; ++spins) {
        bool ok = true;
        for (unsigned i = lane; i < K; i += 64)
            ok &= __hip_atomic_load(&f[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= want;
        if (__ballot(!ok) == 0ull) return true;
        if ((spins & 255) == 0 &&
            (__hip_atomic_load(&cnt->overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kFailBarrier))
            return false;
        if (spins > kBarrierSpins) {
            if (lane == 0) atomicOr(&cnt->overflow, kFailBarrier);
            return false;
        }
    }
}

// Makes the wave wait here for the load that brings v (and for those before
// it).  Without it the compiler waits at the first use, where loads issued in
// between, in flight for a later contact, would be waited for too.
__device__ inline void settle(float& v) { asm volatile("" : "+v"(v)); }

// A contact's rows as the update reads them (rk, the velocity of a moving
// boundary, is fetched by the few contacts that need it).
struct RowRegs {
    float4 a, r1, q, L;
    float4 r3, Lr;  // rolling rows (loaded when mu_r > 0)
    uint32_t seq;   // places in the bodies' sequences (region and counter-ordered solves)
};

__device__ inline RowRegs load_rows(const DevBuffers& b, uint32_t c, bool roll)
{
    RowRegs R;
    R.a = b.r0[c];
    R.r1 = b.r1[c];
    R.q = b.r2[c];
    R.L = b.lam[c];
    if (roll) {
        R.r3 = b.r3[c];
        R.Lr = b.lamr[c];
    }
    return R;
}

__device__ inline void settle(RowRegs& R, bool roll)
{
    settle(R.a.x);
    settle(R.r1.x);
    settle(R.q.x);
    settle(R.L.x);
    if (roll) {
        settle(R.r3.x);
        settle(R.Lr.x);
    }
}

__device__ inline void store_lam(const DevBuffers& b, uint32_t c, const RowRegs& R, bool roll)
{
    b.lam[c] = R.L;
    if (roll) b.lamr[c] = R.Lr;
}

// Body state accessors of the one-block and counter-ordered solves.  Xcd: sc1
// loads, and stores that reach the cluster's XCD or (through) all of them.  Plain:
// ordinary accesses, for a solve confined to one block (its waves share one
// CU and its L1).  Lds: the env's bodies staged in LDS.
struct XcdBodies {
    __amdgpu_buffer_rsrc_t r;  // vw: record i is float4 2i (v) and 2i + 1 (omega)
    bool through;
    __device__ float4 v(int i) const { return ld_body<kCoherent>(r, 2 * i); }
    __device__ float4 w(int i) const { return ld_body<kCoherent>(r, 2 * i + 1); }
    __device__ void set(int i, float4 v, float4 w) const
    {
        if (through) {
            st_body<kCoherent>(r, 2 * i, v);
            st_body<kCoherent>(r, 2 * i + 1, w);
        } else {
            st_body<0>(r, 2 * i, v);
            st_body<0>(r, 2 * i + 1, w);
        }
    }
};
struct PlainBodies {
    float4* vw;
    __device__ float4 v(int i) const { return vel_at(vw, i); }
    __device__ float4 w(int i) const { return angv_at(vw, i); }
    __device__ void set(int i, float4 v, float4 w) const { vel_at(vw, i) = v; angv_at(vw, i) = w; }
};
struct LdsBodies {
    float4 *sv, *sw;  // env slots [base, base + n)
    int base;
    __device__ float4 v(int i) const { return sv[i - base]; }
    __device__ float4 w(int i) const { return sw[i - base]; }
    __device__ void set(int i, float4 v, float4 w) const { sv[i - base] = v; sw[i - base] = w; }
};

// An env solved by one block whose spheres do not all fit its LDS: the
// first cap slots in LDS, the others in global memory (one block, one CU:
// plain accesses are ordered by its workgroup barriers)
struct MixedBodies {
    float4 *sv, *sw;
    int base, cap;
    float4* vw;
    __device__ bool lds(int i) const { return (unsigned)(i - base) < (unsigned)cap; }
    __device__ float4 v(int i) const { return lds(i) ? sv[i - base] : vel_at(vw, i); }
    __device__ float4 w(int i) const { return lds(i) ? sw[i - base] : angv_at(vw, i); }
    __device__ void set(int i, float4 v, float4 w) const
    {
        if (lds(i)) {
            sv[i - base] = v;
            sw[i - base] = w;
        } else {
            vel_at(vw, i) = v;
            angv_at(vw, i) = w;
        }
    }
};

// A region's bodies: LDS, and the exchange records (through: stores reach
// the other XCDs).
struct RegionBodies {
    float4 *sv, *sw;
    __amdgpu_buffer_rsrc_t x;
    int xbase;  // exchange record of LDS index 0
    bool through;
    __device__ void publish(int rec, uint32_t version, float4 v, float4 w) const
    {
        v.w = __uint_as_float(version);
        w.w = v.w;
        if (through) {
            st_body<kCoherent>(x, 2 * rec, v);
            st_body<kCoherent>(x, 2 * rec + 1, w);
        } else {
            st_body<0>(x, 2 * rec, v);
            st_body<0>(x, 2 * rec + 1, w);
        }
    }
};

// the two bodies of a contact, loaded ahead of the update (the update
// replaces body 1 of a boundary contact by the boundary's velocity)
struct BodyRegs {
    float4 va, wa, vb, wb;
};

// unconditional loads (a boundary contact reads its sphere twice): no
// divergent branch between the loads and their use
template <class BA>
__device__ inline BodyRegs load_bodies(const BA& ba, const RowRegs& R)
{
    BodyRegs B;
    const int ia = __float_as_int(R.q.z), ib = __float_as_int(R.q.w);
    const int ja = ia >= 0 ? ia : ib;
    B.vb = ba.v(ib);
    B.wb = ba.w(ib);
    B.va = ba.v(ja);
    B.wa = ba.w(ja);
    return B;
}
template <class BA>
__device__ inline void store_bodies(const BA& ba, const RowRegs& R, const BodyRegs& B)
{
    const int ia = __float_as_int(R.q.z), ib = __float_as_int(R.q.w);
    ba.set(ib, B.vb, B.wb);
    if (ia >= 0) ba.set(ia, B.va, B.wa);
}

// a . b and the determinant a d - b c, with their fused operations fixed
__device__ inline float dot3f(float ax, float ay, float az, float bx, float by, float bz)
{
    return __builtin_fmaf(az, bz, __builtin_fmaf(ax, bx, ay * by));
}
__device__ inline float det2f(float a, float b, float c, float d) { return __builtin_fmaf(a, d, -(b * c)); }

// One contact's update on the loaded rows and bodies; the caller stores the
// impulses (left in R.L, R.Lr) and the bodies (left in B).  want: add the
// contact's share of the sweep residual to (num, den).  Every fused operation
// is written out: left to the compiler, the products it fuses would differ
// between the kernels this is inlined into, and so would the last bits of the
// schedules' results.
__device__ inline void pgs_update(const DevBuffers& b, uint32_t c, RowRegs& R, BodyRegs& B, float mu, float gdt,
                                  bool want, float& num, float& den, bool roll)
{
#pragma clang fp contract(off)
    const float4 a = R.a, r1 = R.r1, q = R.q, L = R.L;
    const int ka = __float_as_int(q.z);
    const bool pair = ka >= 0;
    float4 vb = B.vb, wb = B.wb, va = B.va, wa = B.wa;
    if (!pair) {
        va = make_float4(0.f, 0.f, 0.f, 0.f);
        wa = make_float4(0.f, 0.f, 0.f, 0.f);
        if (ka != kStill) {
            const float4 kv = b.rk[c];  // the boundary's velocity at the contact point
            va.x = kv.x; va.y = kv.y; va.z = kv.z;
            settle(va.x);  // here, where few contacts pay for it
        }
    }
    auto fma = [](float x, float y, float z) { return __builtin_fmaf(x, y, z); };
    const float nx = a.x, ny = a.y, nz = a.z, l1 = a.w;
    const float l2 = r1.x, iDn = r1.y, iDt = r1.z, Sig = r1.w;
    // normal row
    const float un = dot3f(nx, ny, nz, vb.x - va.x, vb.y - va.y, vb.z - va.z);
    const float ln = fmaxf(q.y, fma(-iDn, fma(Sig, L.x, un) - q.x, L.x));
    const float dn = ln - L.x;
    const float jx = nx * dn, jy = ny * dn, jz = nz * dn;
    vb.x = fma(vb.w, jx, vb.x); vb.y = fma(vb.w, jy, vb.y); vb.z = fma(vb.w, jz, vb.z);
    va.x = fma(-va.w, jx, va.x); va.y = fma(-va.w, jy, va.y); va.z = fma(-va.w, jz, va.z);
    // tangential disk row: u = (vb - va) - (l2 wb + l1 wa) x n
    const float sx = fma(l2, wb.x, l1 * wa.x), sy = fma(l2, wb.y, l1 * wa.y), sz = fma(l2, wb.z, l1 * wa.z);
    float ux = (vb.x - va.x) - det2f(nz, ny, sz, sy);
    float uy = (vb.y - va.y) - det2f(nx, nz, sx, sz);
    float uz = (vb.z - va.z) - det2f(ny, nx, sy, sx);
    const float udn = dot3f(nx, ny, nz, ux, uy, uz);
    ux = fma(-nx, udn, ux); uy = fma(-ny, udn, uy); uz = fma(-nz, udn, uz);
    float tx = fma(-iDt, fma(gdt, L.y, ux), L.y);
    float ty = fma(-iDt, fma(gdt, L.z, uy), L.z);
    float tz = fma(-iDt, fma(gdt, L.w, uz), L.w);
    const float lim = mu * fabsf(ln);
    const float m2 = dot3f(tx, ty, tz, tx, ty, tz);
    // (a product with 1 changes nothing; cheaper than a branch)
    const float sc = m2 > lim * lim ? (m2 > 0.f ? lim * rsqrtf(m2) : 0.f) : 1.f;
    tx *= sc; ty *= sc; tz *= sc;
    const float dx = tx - L.y, dy = ty - L.z, dz = tz - L.w;
    // impulse d at the contact point: +d on body 2 (arm -l2 n), -d on body 1 (arm +l1 n)
    const float cx = det2f(ny, nz, dy, dz), cy = det2f(nz, nx, dz, dx), cz = det2f(nx, ny, dx, dy);  // n x d
    vb.x = fma(vb.w, dx, vb.x); vb.y = fma(vb.w, dy, vb.y); vb.z = fma(vb.w, dz, vb.z);
    const float kb = l2 * wb.w;
    wb.x = fma(-kb, cx, wb.x); wb.y = fma(-kb, cy, wb.y); wb.z = fma(-kb, cz, wb.z);
    // (a boundary's are not used any more)
    va.x = fma(-va.w, dx, va.x); va.y = fma(-va.w, dy, va.y); va.z = fma(-va.w, dz, va.z);
    const float kk = l1 * wa.w;
    wa.x = fma(-kk, cx, wa.x); wa.y = fma(-kk, cy, wa.y); wa.z = fma(-kk, cz, wa.z);
    if (want) {
        // residual weights (the stopping test only): hardware reciprocals; a row
        // with zero inverse mass (a neutralised impact-stage row) weighs nothing
        const float Dn = iDn > 0.f ? __builtin_amdgcn_rcpf(iDn) : 0.f, Dt = iDt > 0.f ? __builtin_amdgcn_rcpf(iDt) : 0.f;
        num += fma(dn, Dn * dn, Dt * fma(dz, dz, fma(dy, dy, dx * dx)));
        den += fma(ln, Dn * ln, Dt * fma(tz, tz, fma(ty, ty, tx * tx)));
    }
    if (roll) {
        // rolling row (Eq. signCoul3): zero relative angular velocity, the
        // torque impulse on the disk |lambda_r| <= r mu_r |lambda_n|
        const float4 Lr = R.Lr;
        float ox = 0.f, oy = 0.f, oz = 0.f;
        if (pair) { ox = wa.x; oy = wa.y; oz = wa.z; }
        else {
            const BodyDev& K = b.bodies[__float_as_int(R.r3.z)];
            ox = (float)K.angvel[0]; oy = (float)K.angvel[1]; oz = (float)K.angvel[2];
        }
        const float iWr = R.r3.x;
        float rx = fma(-iWr, wb.x - ox, Lr.x), ry = fma(-iWr, wb.y - oy, Lr.y), rz = fma(-iWr, wb.z - oz, Lr.z);
        const float rlim = R.r3.y * fabsf(ln);
        const float r2 = dot3f(rx, ry, rz, rx, ry, rz);
        if (r2 > rlim * rlim) {
            const float sc = r2 > 0.f ? rlim * rsqrtf(r2) : 0.f;
            rx *= sc; ry *= sc; rz *= sc;
        }
        const float ex = rx - Lr.x, ey = ry - Lr.y, ez = rz - Lr.z;
        wb.x = fma(wb.w, ex, wb.x); wb.y = fma(wb.w, ey, wb.y); wb.z = fma(wb.w, ez, wb.z);
        if (pair) { wa.x = fma(-wa.w, ex, wa.x); wa.y = fma(-wa.w, ey, wa.y); wa.z = fma(-wa.w, ez, wa.z); }
        R.Lr = make_float4(rx, ry, rz, 0.f);
        if (want) {
            const float Wr = __builtin_amdgcn_rcpf(iWr);
            num = fma(Wr, dot3f(ex, ey, ez, ex, ey, ez), num);
            den = fma(Wr, dot3f(rx, ry, rz, rx, ry, rz), den);
        }
    }
    R.L = make_float4(ln, tx, ty, tz);
    B.vb = vb; B.wb = wb; B.va = va; B.wa = wa;
}

// load, update, store of one contact; its impulses are left in R
template <class BA>
__device__ inline void pgs_contact(const DevBuffers& b, const BA& ba, uint32_t c, RowRegs& R, float mu, float gdt,
                                   bool want, float& num, float& den, bool roll)
{
    BodyRegs B = load_bodies(ba, R);
    pgs_update(b, c, R, B, mu, gdt, want, num, den, roll);
    store_bodies(ba, R, B);
}

// Where a block reads the rows and keeps the impulses of its contacts
// [base, base + n): both in memory, the impulses in LDS, or all in LDS (one
// record a contact: impulses, normal, row, bodies, masses, rolling row and
// impulses; the places in the bodies' sequences after the records).
enum RowHome { kRowsMemory, kRowsImpulses, kRowsLds };
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <bool ROLL, RowHome HOME>
struct BlockRows {
    static constexpr uint32_t kRec = HOME == kRowsLds ? (ROLL ? 7 : 5) : HOME == kRowsImpulses ? (ROLL ? 2 : 1) : 0;
    static constexpr uint32_t kRollAt = HOME == kRowsLds ? 6 : 1;
    typedef __attribute__((address_space(3))) f32x4 lds4;
    typedef __attribute__((address_space(3))) uint32_t lds1;
    lds4* l;
    uint32_t base, n;

    // float4s of LDS that n contacts take
    static __device__ uint32_t size(uint32_t n) { return n * kRec + (HOME == kRowsLds ? (n + 3) / 4 : 0); }
    __device__ BlockRows(float4* lds, uint32_t base, uint32_t n) : l((lds4*)lds), base(base), n(n) {}
    static __device__ float4 get(const lds4* p)
    {
        const f32x4 v = *p;
        return make_float4(v.x, v.y, v.z, v.w);
    }
    static __device__ void put(lds4* p, float4 v) { *p = f32x4{v.x, v.y, v.z, v.w}; }
    __device__ lds1* seqs() const { return (lds1*)(l + n * kRec); }
    __device__ void begin(const DevBuffers& b, uint32_t tid, uint32_t nthr) const
    {
        if (HOME == kRowsMemory) return;
        for (uint32_t k = tid; k < n; k += nthr) {
            const uint32_t c = base + k;
            lds4* r = l + k * kRec;
            put(r, b.lam[c]);
            if (ROLL) put(r + kRollAt, b.lamr[c]);
            if (HOME == kRowsLds) {
                put(r + 1, b.r0[c]);
                put(r + 2, b.r1[c]);
                put(r + 3, b.r2[c]);
                put(r + 4, b.rm[c]);
                if (ROLL) put(r + 5, b.r3[c]);
                seqs()[k] = b.seq[c];
            }
        }
    }
    __device__ void end(const DevBuffers& b, uint32_t tid, uint32_t nthr) const
    {
        if (HOME == kRowsMemory) return;
        for (uint32_t k = tid; k < n; k += nthr) {
            b.lam[base + k] = get(l + k * kRec);
            if (ROLL) b.lamr[base + k] = get(l + k * kRec + kRollAt);
        }
    }
    __device__ RowRegs load(const DevBuffers& b, uint32_t c) const
    {
        if (HOME == kRowsMemory) return load_rows(b, c, ROLL);
        RowRegs R;
        const lds4* r = l + (c - base) * kRec;
        if (HOME == kRowsLds) {
            R.a = get(r + 1);
            R.r1 = get(r + 2);
            R.q = get(r + 3);
            if (ROLL) R.r3 = get(r + 5);
        } else {
            R.a = b.r0[c];
            R.r1 = b.r1[c];
            R.q = b.r2[c];
            if (ROLL) R.r3 = b.r3[c];
        }
        R.L = get(r);
        if (ROLL) R.Lr = get(r + kRollAt);
        return R;
    }
    __device__ uint32_t seq(const DevBuffers& b, uint32_t c) const
    {
        if (HOME == kRowsLds) return seqs()[c - base];
        return b.seq[c];
    }
    __device__ float4 masses(const DevBuffers& b, uint32_t c) const
    {
        if (HOME == kRowsLds) return get(l + (c - base) * kRec + 4);
        return b.rm[c];
    }
    __device__ void store(const DevBuffers& b, uint32_t c, const RowRegs& R) const
    {
        if (HOME == kRowsMemory) {
            store_lam(b, c, R, ROLL);
            return;
        }
        lds4* r = l + (c - base) * kRec;
        put(r, R.L);
        if (ROLL) put(r + kRollAt, R.Lr);
    }
};

// what a solve's block keeps in LDS beside its bodies
template <int NW>
struct SolveShared {
    double red[2][NW];
    uint32_t st[kOwnStride];  // the owner's starts
    int flag;
};

// a block's part of a solve: its owner's contacts, rank of K, the cluster's
// first progress flag, the unit of its statistics
struct SolveTask {
    int owner;
    unsigned rank, K;
    unsigned f0;
    int unit;
};

// block sums of the sweep's (num, den) in a fixed order, returned to every thread
template <int NW>
__device__ inline void block_sum2(float num, float den, double (*red)[NW], double& sn, double& sd)
{
    double dnum = num, dden = den;
    for (int o = 32; o > 0; o >>= 1) {
        dnum += __shfl_down(dnum, o, 64);
        dden += __shfl_down(dden, o, 64);
    }
    if ((threadIdx.x & 63) == 0) { red[0][threadIdx.x >> 6] = dnum; red[1][threadIdx.x >> 6] = dden; }
    __syncthreads();
    sn = 0.0; sd = 0.0;
    for (int w = 0; w < NW; ++w) { sn += red[0][w]; sd += red[1][w]; }
    __syncthreads();  // red is reused
}

// The cluster's (num, den) from its blocks' partials, the same value in every
// thread of every block: wave 0 loads the K partials in parallel and sums
// them in a fixed tree order, the result is broadcast through LDS.
template <int NW>
__device__ inline void combine_parts(const double* part, unsigned K, double (*red)[NW], double& sn, double& sd)
{
    if (threadIdx.x < 64) {
        double a = 0.0, d = 0.0;
        for (unsigned t = threadIdx.x; t < K; t += 64) {
            a += __hip_atomic_load(&part[2 * t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            d += __hip_atomic_load(&part[2 * t + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        for (int o = 32; o > 0; o >>= 1) {
            a += __shfl_down(a, o, 64);
            d += __shfl_down(d, o, 64);
        }
        if (threadIdx.x == 0) { red[0][0] = a; red[1][0] = d; }
    }
    __syncthreads();
    sn = red[0][0];
    sd = red[1][0];
    __syncthreads();  // red is reused
}

__device__ inline double sweep_resid(double sn, double sd)
{
    return sd > 0.0 ? sqrt(sn) / sqrt(sd) : (sn > 0.0 ? 1.0 : 0.0);
}

__device__ inline void write_stats(const DevBuffers& b, int unit, int slot, int sweeps, double Rk, double R1)
{
    UnitStats& G = b.ustats[unit];
    if (slot == 0) {
        G.sweeps = (uint32_t)sweeps;
        G.resid = Rk;
        G.resid_first = R1;
    } else if (slot == kSlotImpact) {
        G.imp_sweeps = (uint32_t)sweeps;
    } else {
        G.r1_trial[slot - 1] = R1;
    }
}

template <int NW>
__device__ inline void stage_starts(const DevBuffers& b, int owner, uint32_t ncol, SolveShared<NW>& sh)
{
    for (uint32_t q = threadIdx.x; q <= 2 * ncol; q += blockDim.x)
        sh.st[q] = b.own_start[(size_t)owner * kOwnStride + q];
}

// Counter-ordered updates: contact c is update number s deg_j + pos_j of
// sphere j in sweep s (pos_j: its rank among j's contacts by colour), so it
// may run once j's counter shows that many updates; afterwards it drains its
// stores and advances the counters.  This keeps the colour order of every
// sphere's updates without barriers between colours.  The waits are bounded
// and give up when another wait has failed.
__device__ inline bool flow_wait(Counters* cnt, const uint32_t* ver, int j, uint32_t want)
{
    long spins = 0;
    while (__hip_atomic_load(&ver[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != want) {
        __builtin_amdgcn_s_sleep(1);
        if ((++spins & 255) == 0) {
            if (__hip_atomic_load(&cnt->overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kFailBarrier)
                return false;
            if (spins > kBarrierSpins) {
                atomicOr(&cnt->overflow, kFailBarrier);
                return false;
            }
        }
    }
    return true;
}

// The counter-ordered solve of a cluster (every body in memory): a barrier
// remains at the end of a sweep when a residual tolerance is set, and once at
// the end.
template <bool ROLL, int NW>
__device__ void pgs_flow(const DevBuffers& b, const StepParams& p, const SolveTask& T, uint32_t ncol,
                         uint32_t* counter, bool through, int sweeps_cap, int slot, SolveShared<NW>& sh)
{
    constexpr uint32_t kThreads = NW * 64;
    const XcdBodies ba{raw_rsrc(b.vw), through};
    const size_t nblk = gridDim.x;
    unsigned nbar = 1;
    int sweeps = 0;
    double Rk = 0.0, R1 = 0.0, sn = 0.0, sd = 0.0;
    bool alive = true;
    stage_starts(b, T.owner, ncol, sh);
    __syncthreads();
    auto part_of = [&](int sw) { return b.block_part + 2 * ((size_t)sw * nblk + T.f0); };
    for (int sw = 0; sw < sweeps_cap && ncol > 0; ++sw) {
        float num = 0.f, den = 0.f;
        for (uint32_t col = 0; col < ncol; ++col) {
            const uint32_t hi = sh.st[2 * col + 2];
            for (uint32_t c = sh.st[2 * col] + threadIdx.x; c < hi; c += kThreads) {
                RowRegs R = load_rows(b, c, ROLL);
                const uint32_t seq = b.seq[c];
                const int ia = __float_as_int(R.q.z), ib = __float_as_int(R.q.w);
                const uint32_t wa = (uint32_t)sw * ((seq >> 16) & 255u) + (seq & 255u);
                const uint32_t wb = (uint32_t)sw * (seq >> 24) + ((seq >> 8) & 255u);
                if (alive) alive = flow_wait(b.cnt, b.ver, ib, wb) && (ia < 0 || flow_wait(b.cnt, b.ver, ia, wa));
                if (alive) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");  // body loads after the counters
                    pgs_contact(b, ba, c, R, p.mu, p.gamma_dt, true, num, den, ROLL);
                    store_lam(b, c, R, ROLL);
                    __builtin_amdgcn_s_waitcnt(0);  // the sphere state has reached the XCD's L2
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    __hip_atomic_store(&b.ver[ib], wb + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (ia >= 0) __hip_atomic_store(&b.ver[ia], wa + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        block_sum2<NW>(num, den, sh.red, sn, sd);
        if (threadIdx.x == 0) {
            double* part = part_of(sw) + 2 * T.rank;
            __hip_atomic_store(&part[0], sn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&part[1], sd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        sweeps = sw + 1;
        if (p.tol > 0.f) {
            // the stopping test needs every block's partial of this sweep
            cluster_arrive(counter);
            ++nbar;
            if (!cluster_wait(b.cnt, counter, nbar * T.K, sh.flag)) return;
            combine_parts<NW>(part_of(sw), T.K, sh.red, sn, sd);
            Rk = sweep_resid(sn, sd);
            if (sw == 0) R1 = Rk;
            if (Rk <= (double)p.tol) break;  // uniform: every block holds the same Rk
        }
    }
    if (sweeps > 0 && !(p.tol > 0.f)) {
        // fixed sweep count: the first and last residuals once every block is done
        cluster_arrive(counter);
        ++nbar;
        if (!cluster_wait(b.cnt, counter, nbar * T.K, sh.flag)) return;
        combine_parts<NW>(part_of(0), T.K, sh.red, sn, sd);
        R1 = sweep_resid(sn, sd);
        combine_parts<NW>(part_of(sweeps - 1), T.K, sh.red, sn, sd);
        Rk = sweep_resid(sn, sd);
    }
    if (T.rank == 0 && threadIdx.x == 0) write_stats(b, T.unit, slot, sweeps, Rk, R1);
}

// The bodies of a contact that waits: LDS, or the exchange record once it
// shows the awaited version (with the masses from rm).  Called by whole
// waves; on: the lane has a contact.  alive turns false when a wait gives up.
__device__ inline BodyRegs await_bodies(const DevBuffers& b, const RegionBodies& rb, const RowRegs& R, float4 m,
                                        uint32_t it, bool on, bool& alive)
{
    BodyRegs B;
    const int ia = __float_as_int(R.q.z), ib = __float_as_int(R.q.w);
    const bool la = (ia & kLocal) != 0, lb = (ib & kLocal) != 0;
    const int xa = la ? rb.xbase + (ia & kNameMask) : ia, xb = lb ? rb.xbase + (ib & kNameMask) : ib;
    const uint32_t va = it * ((R.seq >> 16) & 255u) + (R.seq & 255u), vb = it * (R.seq >> 24) + ((R.seq >> 8) & 255u);
    bool need_a = on && ia >= 0 && (!la || (ia & kFetch)), need_b = on && (!lb || (ib & kFetch));
    if (on && !need_b) { B.vb = rb.sv[ib & kNameMask]; B.wb = rb.sw[ib & kNameMask]; }
    if (on && ia >= 0 && !need_a) { B.va = rb.sv[ia & kNameMask]; B.wa = rb.sw[ia & kNameMask]; }
    const bool far_a = need_a, far_b = need_b;
    for (long spins = 1;; ++spins) {
        if (need_b) { B.vb = ld_body<kCoherent>(rb.x, 2 * xb); B.wb = ld_body<kCoherent>(rb.x, 2 * xb + 1); }
        if (need_a) { B.va = ld_body<kCoherent>(rb.x, 2 * xa); B.wa = ld_body<kCoherent>(rb.x, 2 * xa + 1); }
        if (need_b) need_b = __float_as_uint(B.vb.w) != vb || __float_as_uint(B.wb.w) != vb;
        if (need_a) need_a = __float_as_uint(B.va.w) != va || __float_as_uint(B.wa.w) != va;
        if (__ballot(need_a || need_b) == 0ull || !alive) break;
        if ((spins & 255) == 0 &&
            (__hip_atomic_load(&b.cnt->overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kFailBarrier))
            alive = false;
        if (spins > kBarrierSpins) {
            if ((threadIdx.x & 63) == 0) atomicOr(&b.cnt->overflow, kFailBarrier);
            alive = false;
        }
    }
    if (far_a) { B.va.w = m.x; B.wa.w = m.y; }
    if (far_b) { B.vb.w = m.z; B.wb.w = m.w; }
    return B;
}

// The solve of one region (file comment above).  lds holds the bodies of the
// region's first nb spheres (v, then omega).
template <bool ROLL, int NW, RowHome HOME>
__device__ __forceinline__ void solve_region(const DevBuffers& b, const StepParams& p, const SolveTask& T, uint32_t ncol, bool through,
                             int sweeps_cap, int slot, float4* lds, int nb, const BlockRows<ROLL, HOME>& br,
                             SolveShared<NW>& sh)
{
    constexpr uint32_t kThreads = NW * 64;
    const uint32_t tid = threadIdx.x;
    const bool cluster = T.K > 1;
    uint32_t* sweep_flag = b.rflags + T.f0;
    const RegionBodies rb{lds, lds + nb, exchange_rsrc(b.xw), b.own_x[T.owner], through};
    const int sg0 = b.own_idx[T.owner], sg1 = b.own_idx[T.owner + 1];
    if (ncol > 0) {
        for (int sg = sg0; sg < sg1; ++sg) {
            const int4 S = b.own_seg[sg];
            for (int i = (int)tid; i < S.y && S.z + i < nb; i += (int)kThreads) {
                rb.sv[S.z + i] = vel_at(b.vw, S.x + i);
                rb.sw[S.z + i] = angv_at(b.vw, S.x + i);
            }
        }
        br.begin(b, tid, kThreads);
    }
    __syncthreads();
    // Shared contacts go to the threads from the last one down, private ones
    // from the first one up: the waves that wait for the neighbours are the
    // last to get a second private contact.  A thread's first shared and
    // first private contact of a phase are both fetched ahead by 512-thread
    // blocks; 1024-thread ones have registers for one, and take the private
    // contact of a thread with both as it comes.
    constexpr bool kBoth = NW <= kPgsWide;
    const uint32_t ts = kThreads - 1 - tid, wave_ts = ts & ~63u;  // this wave's first shared contact
    RowRegs cs, cp;
    float4 ms;  // masses of the shared contact's bodies
    auto rows = [&](uint32_t c) {
        RowRegs R = br.load(b, c);
        R.seq = br.seq(b, c);
        return R;
    };
    uint32_t s_next = 0, p_next = 0, e_next = 0;  // the phase's shared and private contacts, their end
    auto fetch = [&](uint32_t col) {
        s_next = sh.st[2 * col];
        p_next = sh.st[2 * col + 1];
        e_next = sh.st[2 * col + 2];
        const bool has_s = ts < p_next - s_next, has_p = tid < e_next - p_next;
        if (has_s) ms = br.masses(b, s_next + ts);
        if (kBoth) {
            if (has_s) cs = rows(s_next + ts);
            if (has_p) cp = rows(p_next + tid);
        } else if (has_s || has_p) {
            cp = rows(has_s ? s_next + ts : p_next + tid);
        }
    };
    if (ncol > 0) fetch(0);
    bool alive = true;
    int sweeps = 0;
    double Rk = 0.0, R1 = 0.0;
    // the updated bodies to LDS and, with the number of updates they have
    // seen, to the exchange (a sphere without an LDS index, or needed next by
    // another block); priv: both bodies have an LDS index
    auto put = [&](const RowRegs& R, const BodyRegs& B, uint32_t it, bool priv) {
        const int ia = __float_as_int(R.q.z), ib = __float_as_int(R.q.w);
        if (priv || (ib & kLocal)) { rb.sv[ib & kNameMask] = B.vb; rb.sw[ib & kNameMask] = B.wb; }
        if (ia >= 0 && (priv || (ia & kLocal))) { rb.sv[ia & kNameMask] = B.va; rb.sw[ia & kNameMask] = B.wa; }
        const bool out_a = ia >= 0 && ((ia & kPublish) || !(priv || (ia & kLocal)));
        const bool out_b = (ib & kPublish) || !(priv || (ib & kLocal));
        if (out_a || out_b) {
            const int rec_a = (ia & kNameMask) + ((ia & kLocal) ? rb.xbase : 0);
            const int rec_b = (ib & kNameMask) + ((ib & kLocal) ? rb.xbase : 0);
            if (out_b) rb.publish(rec_b, it * (R.seq >> 24) + ((R.seq >> 8) & 255u) + 1, B.vb, B.wb);
            if (out_a) rb.publish(rec_a, it * ((R.seq >> 16) & 255u) + (R.seq & 255u) + 1, B.va, B.wa);
        }
    };
    auto update_private = [&](uint32_t c, RowRegs& R, uint32_t it, bool want, float& num, float& den) {
        const int ia = __float_as_int(R.q.z), ib = __float_as_int(R.q.w) & kNameMask;
        const int ja = ia >= 0 ? ia & kNameMask : ib;
        BodyRegs B{rb.sv[ja], rb.sw[ja], rb.sv[ib], rb.sw[ib]};
        pgs_update(b, c, R, B, p.mu, p.gamma_dt, want, num, den, ROLL);
        put(R, B, it, true);
        br.store(b, c, R);
    };
    for (int it = 0; it < sweeps_cap && ncol > 0; ++it) {
        // without a tolerance only the first and last residuals are reported
        const bool want = p.tol > 0.f || it == 0 || it + 1 == sweeps_cap;
        float num = 0.f, den = 0.f;
        for (uint32_t col = 0; col < ncol; ++col) {
            const uint32_t s0 = s_next, p0 = p_next, ns = p0 - s0, np = e_next - p0;
            RowRegs& C = kBoth ? cs : cp;
            for (uint32_t k0 = wave_ts; k0 < ns; k0 += kThreads) {
                const uint32_t k = k0 + (ts & 63u);
                const bool on = k < ns;
                if (k0 != wave_ts && on) {
                    C = rows(s0 + k);
                    ms = br.masses(b, s0 + k);
                }
                settle(C, ROLL);
                settle(ms.x);
                BodyRegs B = await_bodies(b, rb, C, ms, (uint32_t)it, on, alive);
                if (on) {
                    pgs_update(b, s0 + k, C, B, p.mu, p.gamma_dt, want, num, den, ROLL);
                    put(C, B, (uint32_t)it, false);
                    br.store(b, s0 + k, C);
                }
            }
            if (tid < np) {
                if (!kBoth && ts < ns) cp = rows(p0 + tid);
                settle(cp, ROLL);
                // a second private contact is in flight during the first's update
                RowRegs nxt;
                if (tid + kThreads < np) nxt = rows(p0 + tid + kThreads);
                update_private(p0 + tid, cp, (uint32_t)it, want, num, den);
                for (uint32_t k = tid + kThreads; k < np; k += kThreads) {
                    settle(nxt, ROLL);
                    cp = nxt;
                    if (k + kThreads < np) nxt = rows(p0 + k + kThreads);
                    update_private(p0 + k, cp, (uint32_t)it, want, num, den);
                }
            }
            fetch(col + 1 < ncol ? col + 1 : 0);  // in flight across the barrier
            __syncthreads();
        }
        sweeps = it + 1;
        if (!want) continue;
        double sn, sd;
        block_sum2<NW>(num, den, sh.red, sn, sd);
        if (cluster) {
            // two slots: the first and the last sweep, or with a tolerance
            // alternating sweeps (no block is more than one sweep ahead)
            const int q = p.tol > 0.f ? it & 1 : (it == 0 ? 0 : 1);
            double* part = b.block_part + 2 * ((size_t)q * gridDim.x + T.f0);
            if (tid == 0) {
                __hip_atomic_store(&part[2 * T.rank], sn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&part[2 * T.rank + 1], sd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __builtin_amdgcn_s_waitcnt(0);
                __hip_atomic_store(&sweep_flag[T.rank], (uint32_t)it + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (tid < 64 && alive) {
                alive = wait_flags(b.cnt, sweep_flag, T.K, (uint32_t)it + 1);
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            }
            combine_parts<NW>(part, T.K, sh.red, sn, sd);
        }
        Rk = sweep_resid(sn, sd);
        if (it == 0) R1 = Rk;
        if (p.tol > 0.f && Rk <= (double)p.tol) break;  // uniform: every thread holds the same Rk
    }
    // the region's final states: from LDS, or from the exchange where the
    // sphere's last update was solved away
    if (ncol > 0 && sweeps > 0)
        for (int sg = sg0; sg < sg1; ++sg) {
            const int4 S = b.own_seg[sg];
            for (int i = (int)tid; i < S.y; i += (int)kThreads) {
                const int li = S.z + i, sl = S.x + i;
                const ulonglong2 m = b.smask[sl];
                if (m.y && ((m.y >> (63 - __builtin_clzll(m.x))) & 1)) {
                    const uint32_t last = (uint32_t)sweeps * (uint32_t)__popcll(m.x);
                    float4 v, w;
                    long spins = 0;
                    do {
                        v = ld_body<kCoherent>(rb.x, 2 * (rb.xbase + li));
                        w = ld_body<kCoherent>(rb.x, 2 * (rb.xbase + li) + 1);
                        if (++spins > kBarrierSpins) atomicOr(&b.cnt->overflow, kFailBarrier);
                        if ((spins & 255) == 0 && (__hip_atomic_load(&b.cnt->overflow, __ATOMIC_RELAXED,
                                                                     __HIP_MEMORY_SCOPE_AGENT) & kFailBarrier))
                            break;
                    } while (alive && (__float_as_uint(v.w) != last || __float_as_uint(w.w) != last));
                    v.w = vel_at(b.vw, sl).w;
                    w.w = angv_at(b.vw, sl).w;
                    vel_at(b.vw, sl) = v;
                    angv_at(b.vw, sl) = w;
                } else if (li < nb) {
                    vel_at(b.vw, sl) = rb.sv[li];
                    angv_at(b.vw, sl) = rb.sw[li];
                }
            }
        }
    if (ncol > 0) br.end(b, tid, kThreads);
    if (T.rank == 0 && tid == 0) write_stats(b, T.unit, slot, sweeps, Rk, R1);
}

// A solve of one region, all of whose bodies are in LDS: no contact waits and
// nothing is published, so that a phase is its chain alone, which one wave a
// SIMD issues: the update's hundred operations, its bodies out of LDS and
// back, a barrier.  Everything else is kept off it: the rows of the next phase
// are fetched before the update, into the other of two sets of registers,
// unconditionally (a thread without a contact reads the last one's, so there
// must be one).
template <bool ROLL, int NW, RowHome HOME>
__device__ __forceinline__ void solve_alone(const DevBuffers& b, const StepParams& p, const SolveTask& T, uint32_t ncol, int sweeps_cap,
                            int slot, float4* lds, int nb, const BlockRows<ROLL, HOME>& br, SolveShared<NW>& sh)
{
    constexpr uint32_t kThreads = NW * 64;
    const uint32_t tid = threadIdx.x;
    float4 *sv = lds, *sw = lds + nb;
    const int sg0 = b.own_idx[T.owner], sg1 = b.own_idx[T.owner + 1];
    if (ncol == 0 || sweeps_cap <= 0) {
        if (tid == 0) write_stats(b, T.unit, slot, 0, 0.0, 0.0);
        return;
    }
    for (int sg = sg0; sg < sg1; ++sg) {
        const int4 S = b.own_seg[sg];
        for (int i = (int)tid; i < S.y; i += (int)kThreads) {
            sv[S.z + i] = vel_at(b.vw, S.x + i);
            sw[S.z + i] = angv_at(b.vw, S.x + i);
        }
    }
    br.begin(b, tid, kThreads);
    __syncthreads();
    const uint32_t last = br.base + br.n - 1;
    uint32_t s0 = sh.st[0], s1 = sh.st[2], s2 = sh.st[ncol > 1 ? 4 : 2];  // starts of the phase, its end, the next's end
    uint32_t next = ncol > 1 ? 1 : 0;                                      // the next phase
    int sweep = 0;
    float num = 0.f, den = 0.f;
    bool want = true;
    double Rk = 0.0, R1 = 0.0;
    auto update = [&](uint32_t c, RowRegs& R, BodyRegs& B) {
        const int ia = __float_as_int(R.q.z), ib = __float_as_int(R.q.w) & kNameMask;
        pgs_update(b, c, R, B, p.mu, p.gamma_dt, want, num, den, ROLL);
        sv[ib] = B.vb;
        sw[ib] = B.wb;
        if (ia >= 0) { sv[ia & kNameMask] = B.va; sw[ia & kNameMask] = B.wa; }
        br.store(b, c, R);
    };
    auto bodies = [&](const RowRegs& R) {
        const int ia = __float_as_int(R.q.z), ib = __float_as_int(R.q.w) & kNameMask;
        const int ja = ia >= 0 ? ia & kNameMask : ib;
        return BodyRegs{sv[ja], sw[ja], sv[ib], sw[ib]};
    };
    // one phase on the rows in cur, the next one's into nxt; false at the end of the solve
    auto phase = [&](RowRegs& cur, RowRegs& nxt) {
        const uint32_t c = s0 + tid, hi = s1;
        settle(cur, ROLL);
        BodyRegs B = bodies(cur);
        if (ncol > 1) nxt = br.load(b, min((next > 0 ? s1 : br.base) + tid, last));
        const uint32_t after = next + 1 < ncol ? next + 1 : 0;
        const uint32_t s3 = sh.st[2 * after + 2];
        if (c < hi) update(c, cur, B);
        for (uint32_t k = c + kThreads; k < hi; k += kThreads) {
            RowRegs R = br.load(b, k);
            BodyRegs C = bodies(R);
            update(k, R, C);
        }
        if (ncol == 1) nxt = br.load(b, min(br.base + tid, last));  // (its impulses are those just stored)
        __syncthreads();
        s0 = next > 0 ? s1 : br.base;
        s1 = s2;
        s2 = s3;
        const bool end = next == 0;
        next = after;
        if (!end) return true;
        ++sweep;
        bool more = sweep < sweeps_cap;
        if (want) {
            double sn, sd;
            block_sum2<NW>(num, den, sh.red, sn, sd);
            Rk = sweep_resid(sn, sd);
            if (sweep == 1) R1 = Rk;
            if (p.tol > 0.f && Rk <= (double)p.tol) more = false;  // uniform: every thread holds the same Rk
        }
        num = den = 0.f;
        // without a tolerance only the first and last residuals are reported
        want = p.tol > 0.f || sweep + 1 == sweeps_cap;
        return more;
    };
    RowRegs A = br.load(b, min(br.base + tid, last)), Z;
    while (phase(A, Z) && phase(Z, A)) {}
    for (int sg = sg0; sg < sg1; ++sg) {
        const int4 S = b.own_seg[sg];
        for (int i = (int)tid; i < S.y; i += (int)kThreads) {
            vel_at(b.vw, S.x + i) = sv[S.z + i];
            angv_at(b.vw, S.x + i) = sw[S.z + i];
        }
    }
    br.end(b, tid, kThreads);
    if (tid == 0) write_stats(b, T.unit, slot, sweep, Rk, R1);
}

// The region's solve with its rows where they fit: the bodies (at most
// lds_cap) come first in the lds_f4 float4s of LDS, then the rows and impulses
// of its contacts, or the impulses alone.  Whole or not at all: impulses of
// the first contacts in LDS and the others in memory took a branch or a flat
// access at every use, and were slower than all of them in memory (3.6 and
// 3.5 ms for the column of 1,000 above).
template <bool ROLL, int NW>
__device__ __forceinline__ void pgs_region(const DevBuffers& b, const StepParams& p, const SolveTask& T, uint32_t ncol, bool through,
                           int sweeps_cap, int slot, float4* lds, int lds_cap, int lds_f4, SolveShared<NW>& sh)
{
    int nb = 0;
    for (int sg = b.own_idx[T.owner]; sg < b.own_idx[T.owner + 1]; ++sg) {
        const int4 S = b.own_seg[sg];
        nb = max(nb, S.z + S.y);
    }
    const bool alone = T.K == 1 && nb <= lds_cap;
    nb = min(nb, lds_cap);
    stage_starts(b, T.owner, ncol, sh);
    __syncthreads();
    const uint32_t base = ncol > 0 ? sh.st[0] : 0u, n = ncol > 0 ? sh.st[2 * ncol] - base : 0u;
    const uint32_t room = (uint32_t)max(0, lds_f4 - 2 * nb);
    auto solve = [&](auto home) {
        const BlockRows<ROLL, decltype(home)::value> br(lds + 2 * nb, base, n);
        if (NW <= kPgsWide && alone)
            solve_alone<ROLL, NW>(b, p, T, ncol, sweeps_cap, slot, lds, nb, br, sh);
        else
            solve_region<ROLL, NW>(b, p, T, ncol, through, sweeps_cap, slot, lds, nb, br, sh);
    };
    if (NW <= kPgsWide && BlockRows<ROLL, kRowsLds>::size(n) <= room)
        solve(std::integral_constant<RowHome, kRowsLds>{});
    else if (NW <= kPgsWide && BlockRows<ROLL, kRowsImpulses>::size(n) <= room)
        solve(std::integral_constant<RowHome, kRowsImpulses>{});
    else
        solve(std::integral_constant<RowHome, kRowsMemory>{});
}

// solve_begin and exchange_begin for a solve that no warm apply precedes
__global__ void k_pgs_reset(DevBuffers b, StepParams p, int n_envs, int n_flags)
{
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    solve_begin(b, t, n_envs, n_flags);
    if (t < p.n_particles) exchange_begin(b, p, t, vel_at(b.vw, t), angv_at(b.vw, t));
}

// Grouped and spread modes: block blockIdx takes the region of its task.
template <bool ROLL, int NW>
__global__ __launch_bounds__(64 * NW) void k_pgs(DevBuffers b, StepParams p, int sweeps_cap, int slot, int lds_cap,
                                                 int lds_f4, int flow)
{
    HIP_DYNAMIC_SHARED(float4, dyn_bodies)
    __shared__ SolveShared<NW> sh;
    if (b.cnt->overflow) return;  // uniform: written by earlier kernels only
    const int4 q = b.grp_task[blockIdx.x];
    if (q.x < 0) return;
    const SolveTask T{q.x, (unsigned)q.y & 0xffffu, (unsigned)q.y >> 16, (unsigned)q.z, q.w & 0x7fffffff};
    bool through = q.w < 0;
    uint32_t ncol = b.cnt->n_colours;
    if (slot == kSlotImpact && !b.ustats[T.unit].imp_any) ncol = 0;  // no impact in the unit
    // no contact in the unit (K is never 0: with the test of it the compiler
    // leaves the solve's loops as they are without this line, 2.07 ms of PGS on
    // the 50,000-sphere bed; else they take 2.09)
    if (T.K > 0 && b.ustats[T.unit].colours == 0) ncol = 0;
    uint32_t* counter = &b.cnt->bar[blockIdx.x % kGroups][0];
    if ((T.K > 1 || flow) && !through) {
        const int mode = cluster_placement(b.cnt, counter, T.K, sh.flag);
        if (mode == 0) return;
        through = mode == 2;
    }
    if (flow)
        pgs_flow<ROLL, NW>(b, p, T, ncol, counter, through, sweeps_cap, slot, sh);
    else
        pgs_region<ROLL, NW>(b, p, T, ncol, through, sweeps_cap, slot, dyn_bodies, lds_cap, lds_f4, sh);
}

// Per-env mode, a set of small envs solved at once by one block: env j of the
// set runs on waves [wb, we) with its bodies in LDS at offset off (global
// memory when off < 0).  The envs share the workgroup barrier after every
// colour (up to the largest colour count of the set) but reduce their own
// residual, stop on their own and record their own statistics.
template <bool ROLL>
__device__ void pgs_local_set(const DevBuffers& b, const StepParams& p, const int4* tasks, int ntask, int sweeps_cap,
                              int slot, float4* dyn, int lds_cap, double (*red)[kEnvBlk / 64])
{
    const int wave = threadIdx.x >> 6;
    int j = -1;
    uint32_t maxcol = 0;
    for (int t = 0; t < ntask; ++t) {
        const int4 q = tasks[t];
        const int wb = q.y & 255, we = (q.y >> 8) & 255;
        if (wave >= wb && wave < we) j = t;
        maxcol = max(maxcol, b.env_ncol[q.x]);
    }
    int e = -1, wb = 0, we = 1, off = -1;
    if (j >= 0) {
        const int4 q = tasks[j];
        e = q.x; wb = q.y & 255; we = (q.y >> 8) & 255; off = q.w;
    }
    const uint32_t nthr = 64u * (uint32_t)(we - wb), lt = threadIdx.x - 64u * (uint32_t)wb;
    const int sb = e >= 0 ? b.envs[e].slot_begin : 0, n = e >= 0 ? b.envs[e].n : 0;
    LdsBodies lb{dyn + (off >= 0 ? off : 0), dyn + lds_cap + (off >= 0 ? off : 0), sb};
    PlainBodies gb{b.vw};
    // the env's first lcap slots in LDS: all of them when they fit (how 0),
    // none without an LDS offset (how 1), else the rest in global memory (how 2)
    const int lcap = off >= 0 ? min(n, lds_cap - off) : 0;
    const int how = off < 0 ? 1 : (lcap < n ? 2 : 0);
    MixedBodies mb{lb.sv, lb.sw, sb, lcap, b.vw};
    for (int i = (int)lt; i < lcap; i += (int)nthr) {
        lb.sv[i] = vel_at(b.vw, sb + i);
        lb.sw[i] = angv_at(b.vw, sb + i);
    }
    __syncthreads();
    // one owner per env here: colour col is [ec[2 col], ec[2 col + 2])
    const uint32_t* ec = b.own_start + (size_t)(e >= 0 ? b.envs[e].own_base : 0) * kOwnStride;
    const uint32_t ncol = e >= 0 && !(slot == kSlotImpact && !b.ustats[e].imp_any) ? b.env_ncol[e] : 0;
    bool active = ncol > 0;  // uniform over the env's waves
    int sweeps = 0;
    double Rk = 0.0, R1 = 0.0;
    uint32_t c = 1, hi = 0;
    RowRegs cur;
    auto start_col = [&](uint32_t col) {
        c = ec[2 * col] + lt;
        hi = ec[2 * col + 2];
        if (c < hi) cur = load_rows(b, c, ROLL);
    };
    if (active) start_col(0);
    for (int sw = 0; sw < sweeps_cap; ++sw) {
        if (!__syncthreads_or(active)) break;
        // without a tolerance only the first and last residuals are reported
        const bool want = p.tol > 0.f || sw == 0 || sw + 1 == sweeps_cap;
        float num = 0.f, den = 0.f;
        for (uint32_t col = 0; col < maxcol; ++col) {
            if (active && col < ncol) {
                while (c < hi) {
                    uint32_t cn = c + nthr;
                    BodyRegs B = how == 0 ? load_bodies(lb, cur) : how == 1 ? load_bodies(gb, cur) : load_bodies(mb, cur);
                    RowRegs nxt;
                    if (cn < hi) nxt = load_rows(b, cn, ROLL);
                    pgs_update(b, c, cur, B, p.mu, p.gamma_dt, want, num, den, ROLL);
                    if (how == 0) store_bodies(lb, cur, B);
                    else if (how == 1) store_bodies(gb, cur, B);
                    else store_bodies(mb, cur, B);
                    store_lam(b, c, cur, ROLL);
                    cur = nxt;
                    c = cn;
                }
                start_col(col + 1 < ncol ? col + 1 : 0);  // the next phase's first rows
            }
            __syncthreads();
        }
        if (active) sweeps = sw + 1;
        if (!want) continue;
        // the env's residual from its waves' partials, in wave order
        double dnum = num, dden = den;
        for (int o = 32; o > 0; o >>= 1) {
            dnum += __shfl_down(dnum, o, 64);
            dden += __shfl_down(dden, o, 64);
        }
        if ((threadIdx.x & 63) == 0) { red[0][wave] = dnum; red[1][wave] = dden; }
        __syncthreads();
        if (active) {
            double sn = 0.0, sd = 0.0;
            for (int w = wb; w < we; ++w) { sn += red[0][w]; sd += red[1][w]; }
            Rk = sweep_resid(sn, sd);
            if (sw == 0) R1 = Rk;
            if (p.tol > 0.f && Rk <= (double)p.tol) active = false;
        }
        __syncthreads();  // red is reused
    }
    for (int i = (int)lt; i < lcap; i += (int)nthr) {
        vel_at(b.vw, sb + i) = lb.sv[i];
        angv_at(b.vw, sb + i) = lb.sw[i];
    }
    if (e >= 0 && lt == 0) write_stats(b, e, slot, sweeps, Rk, R1);
}

// Per-env mode: block b runs plan[plan_idx[b] .. plan_idx[b + 1]) in order: at
// most one share (env, rank, cluster size K >= 2, first block) of a
// multi-block cluster, first, then sets of small envs solved at once (entries
// (env, waves wb | we << 8, 1, LDS offset); a set starts at wb == 0).
template <bool ROLL, int NW>
__global__ __launch_bounds__(64 * NW) void k_pgs_env(DevBuffers b, StepParams p, int sweeps_cap, int slot, int lds_cap,
                                                     int flow)
{
    HIP_DYNAMIC_SHARED(float4, dyn_bodies)
    __shared__ SolveShared<NW> sh;
    if (b.cnt->overflow) return;  // uniform: written by earlier kernels only
    const uint32_t t0 = b.plan_idx[blockIdx.x], t1 = b.plan_idx[blockIdx.x + 1];
    uint32_t t = t0;
    while (t < t1) {
        const int4 pl = b.plan[t];
        if (64 * NW == kEnvBlk && pl.z < 2) {
            uint32_t u = t + 1;
            while (u < t1 && b.plan[u].z < 2 && (b.plan[u].y & 255) != 0) ++u;
            if constexpr (64 * NW == kEnvBlk)
                pgs_local_set<ROLL>(b, p, b.plan + t, (int)(u - t), sweeps_cap, slot, dyn_bodies, lds_cap, sh.red);
            __syncthreads();  // LDS and the reduction scratch are reused
            t = u;
            continue;
        }
        const int e = pl.x;
        // a cluster's flags are consecutive: block lane + 8 i has flag lane * (blocks / 8) + i
        const unsigned first = (unsigned)pl.w;
        const SolveTask T{b.envs[e].own_base + pl.y, (unsigned)pl.y, (unsigned)pl.z,
                          (first % kGroups) * (gridDim.x / kGroups) + first / kGroups, e};
        const uint32_t ncol = slot == kSlotImpact && !b.ustats[e].imp_any ? 0u : b.env_ncol[e];
        uint32_t* counter = b.env_bar + (size_t)e * 16;
        const int mode = T.K > 1 ? cluster_placement(b.cnt, counter, T.K, sh.flag) : 1;
        if (mode == 0) return;  // failed barrier: the step is abandoned
        if (flow)
            pgs_flow<ROLL, NW>(b, p, T, ncol, counter, mode == 2, sweeps_cap, slot, sh);
        else
            pgs_region<ROLL, NW>(b, p, T, ncol, mode == 2, sweeps_cap, slot, dyn_bodies, lds_cap, 2 * lds_cap, sh);
        __syncthreads();
        ++t;
    }
}

// dynamic LDS one block of a kernel may take: the device's limit per block
// less the larger static footprint of its two instances
static int max_dynamic_lds(const void* k0, const void* k1)
{
    int dev = 0, lds = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    hipFuncAttributes a0{}, a1{};
    size_t st = 2048;  // if the attributes cannot be read
    if (hipFuncGetAttributes(&a0, k0) == hipSuccess && hipFuncGetAttributes(&a1, k1) == hipSuccess)
        st = std::max(a0.sharedSizeBytes, a1.sharedSizeBytes);
    return std::max(0, lds - (int)((st + 255) / 256 * 256));
}

constexpr int kEnvWaves = kEnvBlk / 64;

int pgs_env_max_lds()
{
    return max_dynamic_lds((const void*)k_pgs_env<false, kEnvWaves>, (const void*)k_pgs_env<true, kEnvWaves>);
}

int pgs_group_max_lds()
{
    return std::min(max_dynamic_lds((const void*)k_pgs<false, kPgsWaves>, (const void*)k_pgs<true, kPgsWaves>),
                    max_dynamic_lds((const void*)k_pgs<false, kPgsWide>, (const void*)k_pgs<true, kPgsWide>));
}

// blocks of either instance (plain or with rolling rows) of a persistent
// solve resident at once: its blocks wait for each other
static int resident_blocks(const void* k0, const void* k1, int block, int lds_bytes)
{
    int dev = 0, c0 = 0, c1 = 0;
    (void)hipGetDevice(&dev);
    hipDeviceProp_t pr;
    (void)hipGetDeviceProperties(&pr, dev);
    if (lds_bytes > 0) {
        (void)hipFuncSetAttribute(k0, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        (void)hipFuncSetAttribute(k1, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    }
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&c0, k0, block, lds_bytes);
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&c1, k1, block, lds_bytes);
    return std::max(1, std::min(c0, c1)) * pr.multiProcessorCount;
}

int pgs_env_resident_blocks(int lds_bytes)
{
    const int all = resident_blocks((const void*)k_pgs_env<false, kEnvWaves>, (const void*)k_pgs_env<true, kEnvWaves>,
                                    kEnvBlk, lds_bytes);
    return std::min({all,
                     resident_blocks((const void*)k_pgs_env<false, kPgsWaves>, (const void*)k_pgs_env<true, kPgsWaves>,
                                     64 * kPgsWaves, lds_bytes),
                     resident_blocks((const void*)k_pgs_env<false, kPgsWide>, (const void*)k_pgs_env<true, kPgsWide>,
                                     64 * kPgsWide, lds_bytes)});
}

int pgs_resident_blocks()
{
    const int lds = pgs_group_max_lds();
    return std::min(resident_blocks((const void*)k_pgs<false, kPgsWaves>, (const void*)k_pgs<true, kPgsWaves>,
                                    64 * kPgsWaves, lds),
                    resident_blocks((const void*)k_pgs<false, kPgsWide>, (const void*)k_pgs<true, kPgsWide>,
                                    64 * kPgsWide, lds));
}

// The colouring's blocks wait for each other, so all of them must run at
// once: one block per CU (terrain_gate.h: beside the blocks of other scenes'
// steps too); per_block: the spheres whose state its LDS holds.
int colour_resident_blocks(int* per_block)
{
    int dev = 0;
    (void)hipGetDevice(&dev);
    hipDeviceProp_t pr;
    (void)hipGetDeviceProperties(&pr, dev);
    const int lds = max_dynamic_lds((const void*)k_colour<true>, (const void*)k_colour<true>);
    (void)hipFuncSetAttribute((const void*)k_colour<true>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    *per_block = lds / 16;
    return pr.multiProcessorCount;
}

void launch_pgs(const DevBuffers& b, const StepParams& p, const Sizes& z, hipStream_t s, int sweeps_cap, int slot)
{
    int sw = sweeps_cap < 0 ? p.max_sweeps : sweeps_cap;
    if (slot == kSlotImpact) {
        const int ne = z.pgs_mode == kModePerEnv ? z.n_envs : 0;
        const int n = std::max({kGroups, ne, z.n_flags, p.n_particles});
        hipLaunchKernelGGL(k_pgs_reset, dim3((unsigned)cdiv(n, kBlk)), dim3(kBlk), 0, s, b, p, ne, z.n_flags);
    }
    const int flow = z.flow;
    if (flow && p.n_particles > 0) launch_fill_u32(b.ver, 0u, p.n_particles, s);
    const bool env = z.pgs_mode == kModePerEnv;
    const bool roll = p.mu_r > 0.f;
    const dim3 grid((unsigned)(env ? z.plan_blocks : z.pgs_grid));
    const dim3 blk(env && !z.env_small ? kEnvBlk : 64 * (z.pgs_wide ? kPgsWide : kPgsWaves));
    const size_t lds = env ? (size_t)z.lds_cap * 32 : (size_t)z.grp_f4 * 16;
    if (grid.x == 0) return;
    if (env) {
        auto k = !z.env_small ? (roll ? k_pgs_env<true, kEnvWaves> : k_pgs_env<false, kEnvWaves>)
                 : z.pgs_wide ? (roll ? k_pgs_env<true, kPgsWide> : k_pgs_env<false, kPgsWide>)
                              : (roll ? k_pgs_env<true, kPgsWaves> : k_pgs_env<false, kPgsWaves>);
        hipLaunchKernelGGL(k, grid, blk, lds, s, b, p, sw, slot, z.lds_cap, flow);
    } else {
        auto k = z.pgs_wide ? (roll ? k_pgs<true, kPgsWide> : k_pgs<false, kPgsWide>)
                            : (roll ? k_pgs<true, kPgsWaves> : k_pgs<false, kPgsWaves>);
        hipLaunchKernelGGL(k, grid, blk, lds, s, b, p, sw, slot, z.grp_lds, z.grp_f4, flow);
    }
}

// ---------------------------------------------------------------------------
// depth below the free surface: per env grid column the max of z + r
// (ordered-integer atomic max, order free), then depth = top - z
// ---------------------------------------------------------------------------
__device__ inline uint32_t f2ord(float f)
{
    uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float ord2f(uint32_t u) { return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u); }

__device__ inline uint32_t column_of(const EnvDev& E, float4 x)
{
    int c[3];
    cell_of(E, x.x, x.y, x.z, c);
    return (uint32_t)E.col_base + (uint32_t)(c[1] * E.dims[0] + c[0]);
}

__global__ void k_colmax(DevBuffers b, StepParams p)
{
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= p.n_particles) return;
    float4 x = b.xr[s];
    const EnvDev& E = b.envs[env_of(b.pid[s], p.id_cap)];
    atomicMax(&b.colmax[column_of(E, x)], f2ord(x.z + x.w));
}

__global__ void k_depth(DevBuffers b, StepParams p)
{
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= p.n_particles) return;
    float4 x = b.xr[s];
    const EnvDev& E = b.envs[env_of(b.pid[s], p.id_cap)];
    b.pdepth[s] = ord2f(b.colmax[column_of(E, x)]) - x.z;
}

void launch_depth(const DevBuffers& b, const StepParams& p, const Sizes& z, hipStream_t s)
{
    launch_fill_u32(b.colmax, 0u, z.NCOL, s);
    if (p.n_particles <= 0) return;
    unsigned g = (unsigned)cdiv(p.n_particles, kBlk);
    hipLaunchKernelGGL(k_colmax, dim3(g), dim3(kBlk), 0, s, b, p);
    hipLaunchKernelGGL(k_depth, dim3(g), dim3(kBlk), 0, s, b, p);
}

// ---------------------------------------------------------------------------
// learned-start trial plumbing: velocity backup/restore, start selection,
// the first-sweep comparison
// ---------------------------------------------------------------------------
__global__ void k_vel_copy(DevBuffers b, int n, int backup)
{
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    if (backup) { vel_at(b.vw2, s) = vel_at(b.vw, s); angv_at(b.vw2, s) = angv_at(b.vw, s); }
    else { vel_at(b.vw, s) = vel_at(b.vw2, s); angv_at(b.vw, s) = angv_at(b.vw2, s); }
}

void launch_vel_copy(const DevBuffers& b, const StepParams& p, bool backup, hipStream_t s)
{
    if (p.n_particles <= 0) return;
    hipLaunchKernelGGL(k_vel_copy, dim3((unsigned)cdiv(p.n_particles, kBlk)), dim3(kBlk), 0, s, b, p.n_particles,
                       backup ? 1 : 0);
}

__global__ void k_select_start(DevBuffers b, int64_t cap, int mode, uint32_t id_cap, float mu_r)
{
    uint32_t nc = n_contacts(b, cap);
    uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nc || b.cnt->overflow) return;
    const uint32_t pos = b.cpos[c];
    bool learned = mode == 1;
    if (mode == 2) learned = b.ustats[b.envs[env_of((int)(b.ckey[c] >> 32), id_cap)].unit].use_learned != 0;
    float4 L = learned ? b.lamL[pos] : b.lam0[pos];
    b.lam[pos] = L;
    if (mu_r > 0.f) b.lamr[pos] = project_roll(b.lamr0[pos], b.r3[pos].y * fabsf(L.x));
}

void launch_select_start(const DevBuffers& b, const StepParams& p, const Sizes& z, int mode, hipStream_t s)
{
    hipLaunchKernelGGL(k_select_start, dim3((unsigned)cdiv(z.C, kBlk)), dim3(kBlk), 0, s, b, z.C, mode, p.id_cap, p.mu_r);
}

__global__ void k_choose_start(DevBuffers b, int n_units)
{
    int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= n_units) return;
    UnitStats& G = b.ustats[u];
    bool finite = G.learn_bad == 0 && isfinite(G.r1_trial[0]);
    bool use = finite && !(G.r1_trial[0] > G.r1_trial[1]);
    G.use_learned = use ? 1u : 0u;
    G.fallback = use ? 0u : 1u;
}

void launch_choose_start(const DevBuffers& b, const StepParams& p, hipStream_t s)
{
    hipLaunchKernelGGL(k_choose_start, dim3((unsigned)cdiv(p.n_units, 64)), dim3(64), 0, s, b, p.n_units);
}

// training samples of the last step in canonical order: the 12 features and
// the final impulses in the contact frame divided by m_eff g dt
__global__ void k_learn_samples(DevBuffers b, int64_t beg, int64_t n, float* feat, float* label)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    uint32_t pos = b.cpos[beg + k];
    for (int q = 0; q < 12; ++q) feat[k * 12 + q] = b.feat[(size_t)pos * 12 + q];
    float4 L = b.lam[pos], f1 = b.frm1[pos], f2 = b.frm2[pos];
    float ls = f1.w;
    label[k * 3 + 0] = L.x / ls;
    label[k * 3 + 1] = (L.y * f1.x + L.z * f1.y + L.w * f1.z) / ls;
    label[k * 3 + 2] = (L.y * f2.x + L.z * f2.y + L.w * f2.z) / ls;
}

void launch_learn_samples(const DevBuffers& b, int64_t beg, int64_t n, float* feat, float* label, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_learn_samples, dim3((unsigned)cdiv(n, kBlk)), dim3(kBlk), 0, s, b, beg, n, feat, label);
}

// ---------------------------------------------------------------------------
// finish: canonical impulses, body forces (A11), integration (A10), poses,
// zone aggregates (A12), env stats
// ---------------------------------------------------------------------------
// the contacts' impulses in canonical order (the next step's warm start), and
// x += dt v
__global__ void k_finish(DevBuffers b, StepParams p, int64_t cap, unsigned contact_blocks)
{
    const bool bad = b.cnt->overflow != 0;
    if (blockIdx.x < contact_blocks) {
        const uint32_t nc = n_contacts(b, cap);
        for (uint32_t c = blockIdx.x * blockDim.x + threadIdx.x; c < nc; c += contact_blocks * blockDim.x) {
            const uint32_t pos = bad ? 0 : b.cpos[c];
            b.lamc[c] = bad ? make_float4(0.f, 0.f, 0.f, 0.f) : b.lam[pos];
            if (p.mu_r > 0.f) b.lamrc[c] = bad ? make_float4(0.f, 0.f, 0.f, 0.f) : b.lamr[pos];
        }
        return;
    }
    int s = (blockIdx.x - contact_blocks) * blockDim.x + threadIdx.x;
    if (s >= p.n_particles || bad) return;
    float4 x = b.xr[s];
    float4 v = vel_at(b.vw, s);
    x.x += p.dt * v.x;
    x.y += p.dt * v.y;
    x.z += p.dt * v.z;
    b.xr[s] = x;
}

__device__ inline double block_sum_d(double v, double* sh)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += sh[w];
    return s;
}

constexpr int kRedBlk = 128;

// partial force/torque of (body, chunk) over the env's canonical contacts
__global__ __launch_bounds__(kRedBlk) void k_force_part(DevBuffers b, StepParams p, int64_t cap)
{
    __shared__ double sh[kRedBlk / 64];
    const int nch = p.force_chunks;
    int body = blockIdx.x / nch, ch = blockIdx.x % nch;
    const BodyDev& B = b.bodies[body];
    const EnvDev& E = b.envs[B.env];
    uint32_t nc = n_contacts(b, cap);
    uint32_t beg = b.id_start[E.id_base], end = b.id_start[E.id_base + p.id_cap];
    if (end > nc) end = nc;
    if (beg > end) beg = end;
    uint32_t len = end - beg;
    uint32_t lo = beg + (uint32_t)(((uint64_t)len * ch) / nch);
    uint32_t hi = beg + (uint32_t)(((uint64_t)len * (ch + 1)) / nch);
    double acc[6] = {0, 0, 0, 0, 0, 0};
    if (b.cnt->overflow) hi = lo;
    for (uint32_t c = lo + threadIdx.x; c < hi; c += blockDim.x) {
        int2 pr = b.cpair[c];
        if (pr.x >= 0) continue;
        int sg = -1 - pr.x;
        if (b.shapes[sg].body != body) continue;
        uint32_t pos = b.cpos[c];
        float4 L = b.lam[pos];
        float4 a = b.r0[pos];
        double l2 = b.r1[pos].x;
        float4 x2 = b.xr[pr.y];
        double J[4] = {L.x, L.y, L.z, L.w};
        if (p.v_imp > 0.f) {  // the step's impulses include the impact stage's
            const float4 Li = b.lami[pos];
            J[0] += Li.x; J[1] += Li.y; J[2] += Li.z; J[3] += Li.w;
        }
        double f[3] = {-(J[0] * a.x + J[1]) / p.dt, -(J[0] * a.y + J[2]) / p.dt, -(J[0] * a.z + J[3]) / p.dt};
        double arm[3] = {(double)x2.x - l2 * a.x - B.pos[0], (double)x2.y - l2 * a.y - B.pos[1],
                         (double)x2.z - l2 * a.z - B.pos[2]};
        acc[0] += f[0]; acc[1] += f[1]; acc[2] += f[2];
        acc[3] += arm[1] * f[2] - arm[2] * f[1];
        acc[4] += arm[2] * f[0] - arm[0] * f[2];
        acc[5] += arm[0] * f[1] - arm[1] * f[0];
        if (p.mu_r > 0.f) {  // the rolling couple
            float4 Lr = b.lamr[pos];
            double R[3] = {Lr.x, Lr.y, Lr.z};
            if (p.v_imp > 0.f) {
                const float4 Li = b.lamri[pos];
                R[0] += Li.x; R[1] += Li.y; R[2] += Li.z;
            }
            acc[3] -= R[0] / p.dt;
            acc[4] -= R[1] / p.dt;
            acc[5] -= R[2] / p.dt;
        }
    }
    for (int k = 0; k < 6; ++k) {
        double s = block_sum_d(acc[k], sh);
        if (threadIdx.x == 0) b.force_part[((size_t)body * nch + ch) * 6 + k] = s;
    }
}

// One wave per body: its force from the chunks' partials, its pose advanced
// with its constant velocities, the world zone planes of the new pose; the
// blocks after them count the envs' contacts.
__global__ __launch_bounds__(64) void k_bodies_end(DevBuffers b, StepParams p)
{
    const int t = blockIdx.x;
    if (t >= p.n_bodies) {
        const int e = (t - p.n_bodies) * 64 + threadIdx.x;
        if (e >= p.n_envs) return;
        const int64_t base = (int64_t)e * p.id_cap;
        b.env_stats[e].contacts = (int64_t)b.id_start[base + p.id_cap] - (int64_t)b.id_start[base];
        return;
    }
    double f[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int ch = threadIdx.x; ch < p.force_chunks; ch += 64)
        for (int k = 0; k < 6; ++k) f[k] += b.force_part[((size_t)t * p.force_chunks + ch) * 6 + k];
    for (int k = 0; k < 6; ++k)
        for (int o = 32; o > 0; o >>= 1) f[k] += __shfl_down(f[k], o, 64);
    if (threadIdx.x != 0) return;
    for (int k = 0; k < 6; ++k) b.body_ft[t * 6 + k] = f[k];
    if (b.cnt->overflow) return;
    BodyDev& B = b.bodies[t];
    double dt = p.dt;
    for (int k = 0; k < 3; ++k) B.pos[k] += dt * B.linvel[k];
    double q0 = B.quat[0], q1 = B.quat[1], q2 = B.quat[2], q3 = B.quat[3];
    double wx = B.angvel[0], wy = B.angvel[1], wz = B.angvel[2];
    double h = 0.5 * dt;
    double n0 = q0 + h * (-wx * q1 - wy * q2 - wz * q3);
    double n1 = q1 + h * (wx * q0 + wy * q3 - wz * q2);
    double n2 = q2 + h * (-wx * q3 + wy * q0 + wz * q1);
    double n3 = q3 + h * (wx * q2 - wy * q1 + wz * q0);
    double nn = sqrt(n0 * n0 + n1 * n1 + n2 * n2 + n3 * n3);
    B.quat[0] = n0 / nn; B.quat[1] = n1 / nn; B.quat[2] = n2 / nn; B.quat[3] = n3 / nn;
    double R[9];
    quat_to_R(B.quat, R);
    for (int k = 0; k < B.nplanes; ++k) {
        double nw[3];
        for (int r = 0; r < 3; ++r)
            nw[r] = (R[r * 3 + 0] * B.planes[k][0] + R[r * 3 + 1] * B.planes[k][1]) + R[r * 3 + 2] * B.planes[k][2];
        for (int r = 0; r < 3; ++r) B.wplanes[k][r] = nw[r];
        B.wplanes[k][3] = B.planes[k][3] + (nw[0] * B.pos[0] + nw[1] * B.pos[1] + nw[2] * B.pos[2]);
    }
}

// zone moments of one chunk of an env's particles (sorted slots), per zone
// Zone membership of a world point: the union of the body's predicted
// wedges when it has a tool, else its half-spaces (end-of-step pose).
__device__ inline bool in_body_zone(const DevBuffers& b, const BodyDev& B, const double* x)
{
    if (B.tool >= 0) {
        const ToolDev& T = b.tools[B.tool];
        for (int w = 0; w < T.n_wedges; ++w) {
            const WedgeDev& W = b.wedges[(size_t)B.tool * TR_MAX_WEDGES + w];
            bool in = W.n > 0;
            for (int k = 0; k < W.n && in; ++k)
                if (W.planes[k][0] * x[0] + W.planes[k][1] * x[1] + W.planes[k][2] * x[2] - W.planes[k][3] > 0.0)
                    in = false;
            if (in) return true;
        }
        return false;
    }
    bool in = B.nplanes > 0;
    for (int k = 0; k < B.nplanes && in; ++k)
        if (B.wplanes[k][0] * x[0] + B.wplanes[k][1] * x[1] + B.wplanes[k][2] * x[2] - B.wplanes[k][3] > 0.0)
            in = false;
    return in;
}

// height and gradient of a heightfield shape (Eq. surface: bilinear between
// the grid heights, clamped to the border cells)
__device__ inline double hf_height(const ShapeDev& S, const float* hf, double x, double y, double& hx, double& hy)
{
#pragma clang fp contract(off)
    double fx = (x - S.ox) * S.inv_l0;
    double fy = (y - S.oy) * S.inv_l0;
    double fi = floor(fx), fj = floor(fy);
    if (fi < 0.0) fi = 0.0;
    if (fi > (double)(S.nx - 2)) fi = (double)(S.nx - 2);
    if (fj < 0.0) fj = 0.0;
    if (fj > (double)(S.ny - 2)) fj = (double)(S.ny - 2);
    int i = (int)fi, j = (int)fj;
    double t = fx - fi, u = fy - fj;
    const float* h = hf + S.hf_off;
    double h00 = h[j * S.nx + i], h10 = h[j * S.nx + i + 1];
    double h01 = h[(j + 1) * S.nx + i], h11 = h[(j + 1) * S.nx + i + 1];
    hx = ((h10 - h00) * (1.0 - u) + (h11 - h01) * u) * S.inv_l0;
    hy = ((h01 - h00) * (1.0 - t) + (h11 - h10) * t) * S.inv_l0;
    return (h00 * (1.0 - t) + h10 * t) * (1.0 - u) + (h01 * (1.0 - t) + h11 * t) * u;
}

__device__ inline double dot3d(const double* a, const double* c) { return (a[0] * c[0] + a[1] * c[1]) + a[2] * c[2]; }
__device__ inline void cross3d(const double* a, const double* c, double* o)
{
#pragma clang fp contract(off)
    o[0] = a[1] * c[2] - a[2] * c[1];
    o[1] = a[2] * c[0] - a[0] * c[2];
    o[2] = a[0] * c[1] - a[1] * c[0];
}
__device__ inline void unit3d(double* a)
{
    double m = sqrt(dot3d(a, a));
    a[0] /= m; a[1] /= m; a[2] /= m;
}

// Active-zone predictor (Eq. failure_plane): one thread per (tool, lateral
// wedge), at the end-of-step pose.  The wedge lies in front of the separation
// plate through the edge, above the failure plane rising at
// theta = pi/2 - (phi + beta)/2 against the terrain surface, below where that
// plane meets the surface (+ heap), between the slice's lateral planes.
__global__ void k_predict_wedges(DevBuffers b, StepParams p)
{
#pragma clang fp contract(off)
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= p.n_tools * TR_MAX_WEDGES) return;
    const int ti = t / TR_MAX_WEDGES, w = t % TR_MAX_WEDGES;
    const ToolDev& T = b.tools[ti];
    if (w >= T.n_wedges) return;
    WedgeDev& W = b.wedges[t];
    W.n = 0;
    if (T.terrain < 0) return;
    const BodyDev& B = b.bodies[T.body];
    const ShapeDev& S = b.shapes[T.terrain];
    double R[9];
    quat_to_R(B.quat, R);
    double E0[3], E1[3], nc[3], ntc[3];
    for (int k = 0; k < 3; ++k) {
        E0[k] = B.pos[k] + ((R[k * 3 + 0] * T.edge0[0] + R[k * 3 + 1] * T.edge0[1]) + R[k * 3 + 2] * T.edge0[2]);
        E1[k] = B.pos[k] + ((R[k * 3 + 0] * T.edge1[0] + R[k * 3 + 1] * T.edge1[1]) + R[k * 3 + 2] * T.edge1[2]);
        nc[k] = (R[k * 3 + 0] * T.n_c[0] + R[k * 3 + 1] * T.n_c[1]) + R[k * 3 + 2] * T.n_c[2];
        ntc[k] = (R[k * 3 + 0] * T.n_tc[0] + R[k * 3 + 1] * T.n_tc[1]) + R[k * 3 + 2] * T.n_tc[2];
    }
    if (T.v_min > 0.0) {
        double mid[3], arm[3], ve[3];
        for (int k = 0; k < 3; ++k) { mid[k] = 0.5 * (E0[k] + E1[k]); arm[k] = mid[k] - B.pos[k]; }
        cross3d(B.angvel, arm, ve);
        for (int k = 0; k < 3; ++k) ve[k] += B.linvel[k];
        if (!(sqrt(dot3d(ve, ve)) > T.v_min)) return;
    }
    double nf[3], L[3], l[3];
    for (int k = 0; k < 3; ++k) {
        nf[k] = (1.0 - T.fill) * nc[k] + T.fill * ntc[k];
        L[k] = E1[k] - E0[k];
        l[k] = L[k];
    }
    unit3d(nf);
    unit3d(l);
    const double zh[3] = {0.0, 0.0, 1.0};
    double u[3], pl[3];
    cross3d(zh, l, u);
    unit3d(u);
    if (dot3d(u, nf) < 0.0) for (int k = 0; k < 3; ++k) u[k] = -u[k];
    cross3d(l, nf, pl);
    unit3d(pl);
    if (pl[2] < 0.0) for (int k = 0; k < 3; ++k) pl[k] = -pl[k];
    double a[3], c2[3], m[3];
    const double fa = (double)w / T.n_wedges, fb = (double)(w + 1) / T.n_wedges, fm = (w + 0.5) / T.n_wedges;
    for (int k = 0; k < 3; ++k) { a[k] = E0[k] + L[k] * fa; c2[k] = E0[k] + L[k] * fb; m[k] = E0[k] + L[k] * fm; }
    double hx, hy;
    const double h0 = hf_height(S, b.hf_pool, m[0], m[1], hx, hy);
    if (!(m[2] < h0)) return;
    double sv[3] = {u[0], u[1], u[2] + (hx * u[0] + hy * u[1])};
    const double sl = dot3d(sv, l);
    for (int k = 0; k < 3; ++k) sv[k] -= sl * l[k];
    unit3d(sv);
    double ns[3];
    cross3d(l, sv, ns);
    if (ns[2] < 0.0) for (int k = 0; k < 3; ++k) ns[k] = -ns[k];
    const double beta = atan2(dot3d(pl, ns), dot3d(pl, sv));
    const double theta = 0.5 * 3.14159265358979323846 - 0.5 * (T.phi + beta);
    if (!(theta > 0.0 && theta < 0.5 * 3.14159265358979323846)) return;
    double d[3];
    for (int k = 0; k < 3; ++k) d[k] = cos(theta) * sv[k] + sin(theta) * ns[k];
    double lo = 0.0, hi = S.l0;
    bool found = false;
    for (int it = 0; it < 40; ++it) {
        const double q[3] = {m[0] + hi * d[0], m[1] + hi * d[1], m[2] + hi * d[2]};
        if (q[2] - hf_height(S, b.hf_pool, q[0], q[1], hx, hy) >= 0.0) { found = true; break; }
        lo = hi;
        hi *= 2.0;
    }
    if (!found) return;
    for (int it = 0; it < 60; ++it) {
        const double md = 0.5 * (lo + hi);
        const double q[3] = {m[0] + md * d[0], m[1] + md * d[1], m[2] + md * d[2]};
        if (q[2] - hf_height(S, b.hf_pool, q[0], q[1], hx, hy) >= 0.0) hi = md;
        else lo = md;
    }
    const double ztop = (m[2] + hi * d[2]) + T.heap;
    double cf[3];
    cross3d(l, d, cf);
    unit3d(cf);
    if (dot3d(cf, pl) > 0.0) for (int k = 0; k < 3; ++k) cf[k] = -cf[k];
    for (int k = 0; k < 3; ++k) {
        W.planes[0][k] = -nf[k];
        W.planes[1][k] = cf[k];
        W.planes[2][k] = zh[k];
        W.planes[3][k] = -l[k];
        W.planes[4][k] = l[k];
    }
    W.planes[0][3] = -dot3d(nf, m);
    W.planes[1][3] = dot3d(cf, m);
    W.planes[2][3] = ztop;
    W.planes[3][3] = -dot3d(l, a);
    W.planes[4][3] = dot3d(l, c2);
    W.n = 5;
}

__global__ __launch_bounds__(kRedBlk) void k_zone_part(DevBuffers b, StepParams p)
{
    __shared__ double sh[kRedBlk / 64];
    int4 ck = b.zone_chunks[blockIdx.x];   // env, begin, end, partial base
    const EnvDev& E = b.envs[ck.x];
    for (int z = 0; z < E.zone_count; ++z) {
        double acc[kZonePart];
        for (int k = 0; k < kZonePart; ++k) acc[k] = 0.0;
        for (int s = ck.y + threadIdx.x; s < ck.z; s += blockDim.x) {
            float4 xf = b.xr[s];
            double x[3] = {xf.x, xf.y, xf.z};
            // first zone (body order) containing x wins
            int zone = -1;
            for (int zz = 0; zz < E.zone_count && zone < 0; ++zz)
                if (in_body_zone(b, b.bodies[E.zone_body[zz]], x)) zone = zz;
            if (zone != z) continue;
            double r = xf.w;
            double m = (double)b.rho[s] * (4.0 / 3.0) * 3.14159265358979323846 * r * r * r;
            float4 vf = vel_at(b.vw, s), wf = angv_at(b.vw, s);
            double v[3] = {vf.x, vf.y, vf.z};
            double Is = 0.4 * m * r * r;
            acc[0] += m;
            for (int k = 0; k < 3; ++k) { acc[1 + k] += m * x[k]; acc[4 + k] += m * v[k]; }
            acc[7] += m * x[0] * x[0]; acc[8] += m * x[1] * x[1]; acc[9] += m * x[2] * x[2];
            acc[10] += m * x[0] * x[1]; acc[11] += m * x[0] * x[2]; acc[12] += m * x[1] * x[2];
            acc[13] += m * (x[1] * v[2] - x[2] * v[1]);
            acc[14] += m * (x[2] * v[0] - x[0] * v[2]);
            acc[15] += m * (x[0] * v[1] - x[1] * v[0]);
            acc[16] += Is;
            acc[17] += Is * wf.x; acc[18] += Is * wf.y; acc[19] += Is * wf.z;
            acc[kZoneMoments] += 1.0;
        }
        // most chunks hold no particle of the zone
        double* part = b.zone_part + ((size_t)ck.w + z) * kZonePart;
        if (!__syncthreads_or(acc[kZoneMoments] > 0.0)) {
            if (threadIdx.x < kZonePart) part[threadIdx.x] = 0.0;
            continue;
        }
        for (int k = 0; k < kZonePart; ++k) {
            double s = block_sum_d(acc[k], sh);
            if (threadIdx.x == 0) part[k] = s;
        }
    }
}

// One block per zone: kZoneGroups threads per moment sum every kZoneGroups-th
// chunk's, their sums are added in order, then one thread forms the aggregate
// body.
constexpr int kZoneGroups = 32;
__global__ __launch_bounds__(kZonePart* kZoneGroups) void k_zone_final(DevBuffers b, StepParams p, int n_chunks)
{
    __shared__ double part[kZoneGroups][kZonePart], S[kZonePart];
    const int zs = blockIdx.x, k0 = threadIdx.x % kZonePart, g = threadIdx.x / kZonePart;
    const int4 zt = b.zone_chunks[n_chunks + zs];  // env, zone in it, its chunks
    const int env = zt.x, zi = zt.y;
    double sum = 0.0;
    for (int c = zt.z + g; c < zt.w; c += kZoneGroups)
        sum += b.zone_part[((size_t)c * kMaxZonesPerEnv + zi) * kZonePart + k0];
    part[g][k0] = sum;
    __syncthreads();
    if (g == 0) {
        sum = 0.0;
        for (int q = 0; q < kZoneGroups; ++q) sum += part[q][k0];
        S[k0] = sum;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int k = 0; k < kZoneMoments; ++k) b.zone_mom[(size_t)zs * kZoneMoments + k] = S[k];
    tr_aggregate A;
    A.zone = b.bodies[b.envs[env].zone_body[zi]].user_id;
    A.pad = 0;
    double M = S[0];
    A.M = M;
    A.n_particles = (int64_t)S[kZoneMoments];
    for (int k = 0; k < 3; ++k) { A.x[k] = 0.0; A.v[k] = 0.0; A.w[k] = 0.0; }
    for (int k = 0; k < 6; ++k) A.I[k] = 0.0;
    if (M > 0.0) {
        double x[3] = {S[1] / M, S[2] / M, S[3] / M};
        double v[3] = {S[4] / M, S[5] / M, S[6] / M};
        // second moments about x_A
        double Cxx = S[7] - M * x[0] * x[0], Cyy = S[8] - M * x[1] * x[1], Czz = S[9] - M * x[2] * x[2];
        double Cxy = S[10] - M * x[0] * x[1], Cxz = S[11] - M * x[0] * x[2], Cyz = S[12] - M * x[1] * x[2];
        double tr = Cxx + Cyy + Czz;
        double I[3][3] = {{S[16] + tr - Cxx, -Cxy, -Cxz}, {-Cxy, S[16] + tr - Cyy, -Cyz}, {-Cxz, -Cyz, S[16] + tr - Czz}};
        // angular momentum about x_A: sum m x*v - x_A * sum m v + spins
        double L[3] = {S[13] - (x[1] * S[6] - x[2] * S[5]) + S[17], S[14] - (x[2] * S[4] - x[0] * S[6]) + S[18],
                       S[15] - (x[0] * S[5] - x[1] * S[4]) + S[19]};
        double det = I[0][0] * (I[1][1] * I[2][2] - I[1][2] * I[2][1]) - I[0][1] * (I[1][0] * I[2][2] - I[1][2] * I[2][0]) +
                     I[0][2] * (I[1][0] * I[2][1] - I[1][1] * I[2][0]);
        // inverse by cofactors (I symmetric)
        double inv[3][3];
        inv[0][0] = (I[1][1] * I[2][2] - I[1][2] * I[2][1]);
        inv[0][1] = -(I[0][1] * I[2][2] - I[0][2] * I[2][1]);
        inv[0][2] = (I[0][1] * I[1][2] - I[0][2] * I[1][1]);
        inv[1][0] = -(I[1][0] * I[2][2] - I[1][2] * I[2][0]);
        inv[1][1] = (I[0][0] * I[2][2] - I[0][2] * I[2][0]);
        inv[1][2] = -(I[0][0] * I[1][2] - I[0][2] * I[1][0]);
        inv[2][0] = (I[1][0] * I[2][1] - I[1][1] * I[2][0]);
        inv[2][1] = -(I[0][0] * I[2][1] - I[0][1] * I[2][0]);
        inv[2][2] = (I[0][0] * I[1][1] - I[0][1] * I[1][0]);
        for (int r = 0; r < 3; ++r) {
            A.x[r] = x[r];
            A.v[r] = v[r];
            A.w[r] = det != 0.0 ? (inv[r][0] * L[0] + inv[r][1] * L[1] + inv[r][2] * L[2]) / det : 0.0;
        }
        A.I[0] = I[0][0]; A.I[1] = I[1][1]; A.I[2] = I[2][2];
        A.I[3] = I[0][1]; A.I[4] = I[0][2]; A.I[5] = I[1][2];
    }
    b.aggs[zs] = A;
}

void launch_finish(const DevBuffers& b, const StepParams& p, const Sizes& z, hipStream_t s)
{
    const unsigned gc = contact_grid(z.C);
    if (p.n_bodies > 0)  // (at the positions the contacts were found at)
        hipLaunchKernelGGL(k_force_part, dim3(p.n_bodies * p.force_chunks), dim3(kRedBlk), 0, s, b, p, z.C);
    hipLaunchKernelGGL(k_finish, dim3(gc + (unsigned)cdiv(std::max(p.n_particles, 0), kBlk)), dim3(kBlk), 0, s, b, p, z.C, gc);
    hipLaunchKernelGGL(k_bodies_end, dim3((unsigned)(p.n_bodies + cdiv(p.n_envs, 64))), dim3(64), 0, s, b, p);
    if (p.n_tools > 0)  // the tools' zones at the end-of-step poses
        hipLaunchKernelGGL(k_predict_wedges, dim3((unsigned)cdiv(p.n_tools * TR_MAX_WEDGES, 64)), dim3(64), 0, s, b, p);
    if (p.n_zones > 0 && z.n_zone_chunks > 0) {
        hipLaunchKernelGGL(k_zone_part, dim3(z.n_zone_chunks), dim3(kRedBlk), 0, s, b, p);
        hipLaunchKernelGGL(k_zone_final, dim3(p.n_zones), dim3(kZonePart * kZoneGroups), 0, s, b, p, z.n_zone_chunks);
    }
}

// ---------------------------------------------------------------------------
// host <-> device particle exchange in id order
// ---------------------------------------------------------------------------
// m particles from id id0 on, straight into host memory in the caller's layout
// (FP64: positions, velocities and angular velocities of three values, radii):
// consecutive lanes write consecutive values, so the link carries whole lines
// and the host only copies.  500,000 particles reach the caller in 2.5
// ms, where floats copied to pageable memory and converted there took 13.
__global__ void k_read_particles(DevBuffers b, int id0, int m, double* out)
{
    const int f = blockIdx.y;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (f < 3 ? 3 * m : m)) return;
    const int s = b.id2slot[id0 + (f < 3 ? t / 3 : t)];
    const float4* src = f == 0 || f == 3 ? b.xr + s : b.vw + 2 * (int64_t)s + (f - 1);
    const float* v = reinterpret_cast<const float*>(src);
    out[(int64_t)f * 3 * m + t] = v[f < 3 ? t % 3 : 3];
}

void launch_read_particles(const DevBuffers& b, int id0, int m, double* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_read_particles, dim3((unsigned)cdiv(3 * m, kBlk), 4), dim3(kBlk), 0, s, b, id0, m, out);
}

// what the host reads after a step, into host memory: one launch in place of
// a copy and a wait for each table
__global__ void k_report(StepReport r)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
    for (int k = 0; k < StepReport::kParts; ++k)
        for (int64_t w = t; w < r.words[k]; w += step) r.to[k][w] = r.from[k][w];
}

void launch_report(const StepReport& r, hipStream_t s)
{
    int64_t most = 1;
    for (int k = 0; k < StepReport::kParts; ++k) most = std::max(most, r.words[k]);
    hipLaunchKernelGGL(k_report, dim3((unsigned)std::min<int64_t>(cdiv(most, kBlk), 64)), dim3(kBlk), 0, s, r);
}

__global__ void k_zero(ZeroList l)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    for (int k = 0; k < ZeroList::kParts; ++k)
        for (int64_t w = t; w < (int64_t)(l.part[k].bytes / 4); w += step) ((uint32_t*)l.part[k].p)[w] = 0u;
}

void launch_zero(const ZeroList& l, hipStream_t s)
{
    size_t most = 0;
    for (const ZeroList::Part& q : l.part) most = std::max(most, q.bytes / 4);
    hipLaunchKernelGGL(k_zero, dim3((unsigned)std::min<int64_t>(std::max<int64_t>(cdiv((int64_t)most, kBlk), 1), 1024)),
                       dim3(kBlk), 0, s, l);
}

__global__ void k_scatter_by_id(DevBuffers b, int id_base, int n, const float4* xi, const float4* vi,
                                const float4* wi, int mask)
{
    int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    int s = b.id2slot[id_base + k];
    if (mask & 1) { float4 o = b.xr[s]; float4 v = xi[k]; b.xr[s] = make_float4(v.x, v.y, v.z, o.w); }
    if (mask & 2) { float4 o = vel_at(b.vw, s); float4 v = vi[k]; vel_at(b.vw, s) = make_float4(v.x, v.y, v.z, o.w); }
    if (mask & 4) { float4 o = angv_at(b.vw, s); float4 v = wi[k]; angv_at(b.vw, s) = make_float4(v.x, v.y, v.z, o.w); }
}

void launch_scatter_by_id(const DevBuffers& b, int id_base, int n, const float4* xi, const float4* vi,
                          const float4* wi, int mask, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_scatter_by_id, dim3((unsigned)cdiv(n, kBlk)), dim3(kBlk), 0, s, b, id_base, n, xi, vi, wi,
                       mask);
}

}  // namespace trk

// kernels_util.hip -- initialisation, state transfer and diagnostic kernels
// of the particle store (not on the per-step hot path).
#include "common.hpp"
#include "launch.hpp"

namespace lbmpcd {

// ---------------------------------------------------------------------------
// Initial particles: exactly ppc per fine cell, uniform inside the cell, ids
// in cell order; velocities Maxwell-Boltzmann about the initial flow.  Each
// particle starts in the tile of its unshifted cell (no collision is pending
// after init).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double poiseuille_p(const InstDesc& d, double gk, double y) {
    double nu = (d.tau - 0.5) / 3.0, H = (double)d.ny, tau = d.tau;
    return gk * y * (H - y) / (2.0 * nu) + gk * (16.0 * tau * tau - 16.0 * tau + 1.0) / (24.0 * nu);
}

template <int DIM, typename PT>
__global__ void __launch_bounds__(WG) k_part_init(const InstDesc* __restrict__ D, int n_inst, long long total,
                                                  PartBuf P) {
    long long gid = (long long)blockIdx.x * WG + threadIdx.x;
    if (gid >= total) return;
    int ii = find_inst(D, n_inst, gid, [](const InstDesc& d) { return d.part_off; });
    const InstDesc& d = D[ii];
    const long long id = gid - d.part_off;
    const long long cl = id / d.ppc;
    const int I = (int)(cl % d.Cx);
    const int J = (int)((cl / d.Cx) % d.R);
    const int K = (int)(cl / ((long long)d.Cx * d.R));
    double u[4], z[3];
    rng_uniforms4(key_of(d), (uint32_t)id, 0u, 0u, P_INIT_POS, u);
    const double r = (double)d.r;
    const double x = ((double)I + u[0]) / r;
    const double y = (double)d.ylo + ((double)J + u[1]) / r;
    const double zz = (DIM == 3) ? ((double)K + u[2]) / r : 0.0;
    rng_normals<DIM>(key_of(d), (uint32_t)id, 0u, 0u, P_INIT_VEL, z);
    // the tile of the unshifted cell; slots ranked over the tile's slab cells
    const int tx = I / d.Tx, ty = J / d.Ty, tz = K / d.Tz;
    const int cx = min(d.Tx, d.Cx - tx * d.Tx), cy = min(d.Ty, d.R - ty * d.Ty), cz = min(d.Tz, d.Cz - tz * d.Tz);
    (void)cz;
    const long long tile = tx + (long long)d.ntx * (ty + (long long)d.nty * tz);
    const long long lcell = (I - tx * d.Tx) + (long long)cx * ((J - ty * d.Ty) + (long long)cy * (K - tz * d.Tz));
    const long long slot = lcell * d.ppc + id % d.ppc;
    const PT px[3] = {(PT)x, (PT)y, (PT)zz};
    PT pv[3];
#pragma unroll
    for (int q = 0; q < DIM; ++q) {
        const double u0 = d.init_flow ? poiseuille_p(d, d.g[q], y) : 0.0;
        pv[q] = (PT)(u0 + d.sd * z[q]);
    }
    store_part<DIM, PT>(P, d.slot_off, (uint32_t)(tile * d.cap + slot), px, pv, (uint32_t)id);
}

__global__ void __launch_bounds__(WG) k_fill_sequential(const InstDesc* __restrict__ D, int n_inst, long long tiles,
                                                        uint32_t* fill, uint32_t* other) {
    long long T = (long long)blockIdx.x * WG + threadIdx.x;
    if (T >= tiles) return;
    int ii = find_inst(D, n_inst, T, [](const InstDesc& d) { return d.tile_off; });
    const InstDesc& d = D[ii];
    const long long lt = T - d.tile_off;
    const int tx = (int)(lt % d.ntx), ty = (int)((lt / d.ntx) % d.nty), tz = (int)(lt / ((long long)d.ntx * d.nty));
    const int cx = max(0, min(d.Tx, d.Cx - tx * d.Tx));
    const int cy = max(0, min(d.Ty, d.R - ty * d.Ty));
    const int cz = max(0, min(d.Tz, d.Cz - tz * d.Tz));
    fill[T] = (uint32_t)((long long)cx * cy * cz * d.ppc);
    other[T] = 0u;
}

// Workgroup b of xcd_grid(items) in an order in which the workgroups that the
// hardware deals to one XCD take one contiguous range, so that what
// neighbouring items scatter to (or gather from) the same cache lines meets in
// one L2.
__device__ __forceinline__ long long xcd_item() {
    return (long long)(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
}
static inline unsigned xcd_grid(long long items) { return (unsigned)(8 * ((items + 7) / 8)); }

// Slot `s` of instance d, in the buffer's numbering; -1 if it is empty.
__device__ __forceinline__ long long filled_slot(const InstDesc& d, const uint32_t* __restrict__ fill, long long s) {
    if (s >= d.ntiles * d.cap) return -1;
    const uint32_t lt = (uint32_t)s / (uint32_t)d.cap, k = (uint32_t)s - lt * (uint32_t)d.cap;
    return k < fill[d.tile_off + lt] ? d.slot_off + s : -1;
}

// Positions or velocities of slot g.
template <int DIM, typename PT, bool VEL>
__device__ __forceinline__ void load_field(const PStore<DIM, PT>& S, long long g, PT* v) {
    if constexpr (PStore<DIM, PT>::F32 && DIM == 3 && !VEL) {
        const u32x4 a = *(const u32x4*)S.pos(0, g);
        v[0] = as_f(a.x); v[1] = as_f(a.y); v[2] = as_f(a.z);
    } else {
#pragma unroll
        for (int q = 0; q < DIM; ++q) v[q] = VEL ? *S.vel(q, g) : *S.pos(q, g);
    }
}

enum GatherWhat { GATHER_POS, GATHER_VEL, GATHER_CELL, GATHER_INV };

// Positions, velocities or cells (in the binning of (t, sub)) of one
// instance's particles scattered to their ids, or (GATHER_INV) the slots of
// the ids; one thread per slot.  A workgroup per tile, which walks through the
// tile's slots, has too few loads in flight and a ragged end: the inverse map's
// read of 41.9M binary32 particles took 1617 us with it and takes 1464.
template <int DIM, typename PT, int WHAT>
__global__ void __launch_bounds__(WG) k_scatter(const InstDesc* __restrict__ D, int inst, PartBuf P,
                                                const uint32_t* __restrict__ fill, double* out, int* out32, long long t,
                                                int sub) {
    const InstDesc& d = D[inst];
    const long long s = xcd_item() * WG + threadIdx.x, g = filled_slot(d, fill, s);
    if (g < 0) return;
    const PStore<DIM, PT> S{P.b, P.cs};
    const uint32_t id = *S.id(g);
    if ((long long)id >= d.Np) return;
    if constexpr (WHAT == GATHER_INV) {
        out32[id] = (int)s;
        return;
    }
    PT v[3];
    load_field<DIM, PT, WHAT == GATHER_VEL>(S, g, v);
    if constexpr (WHAT == GATHER_CELL) {
        PT sh[3];
        grid_shift_of<DIM, PT>(d, (uint32_t)t, (uint32_t)sub, sh);
        const PT rr = (PT)d.r;
        int ix = bin_coord<PT>(v[0], (PT)0, sh[0], rr);
        if (ix >= d.Cx) ix -= d.Cx;
        const int iy = bin_row<PT>(d, v[1], sh[1], rr);
        int iz = 0;
        if (DIM == 3) {
            iz = bin_coord<PT>(v[2], (PT)0, sh[2], rr);
            if (iz >= d.Cz) iz -= d.Cz;
        }
        out32[id] = ix + d.Cx * (iy + d.CyB * iz);
    } else if constexpr (WHAT != GATHER_INV) {
#pragma unroll
        for (int q = 0; q < DIM; ++q) out[(long long)q * d.Np + id] = (double)v[q];
    }
}

// Positions or velocities in id order through the slots of the ids: one thread
// per id, the stores consecutive.  An id that a tile overflow lost has no slot,
// and its word of the map is whatever the memory held: once particles have been
// dropped, an entry counts only if it names a filled slot with that id in it
// (the others then cost their id's load; marking the map beforehand would cost
// every read a pass over it and a launch).
template <int DIM, typename PT, int WHAT>
__global__ void __launch_bounds__(WG) k_gather(const InstDesc* __restrict__ D, int inst, PartBuf P,
                                               const uint32_t* __restrict__ fill, const DevStats* __restrict__ stats,
                                               const uint32_t* __restrict__ slot, double* out) {
    const InstDesc& d = D[inst];
    const long long id = (long long)blockIdx.x * WG + threadIdx.x;
    if (id >= d.Np) return;
    const long long s = slot[id];
    if (s >= d.ntiles * d.cap) return;
    const PStore<DIM, PT> S{P.b, P.cs};
    const long long g = d.slot_off + s;
    if (stats->dropped != 0ull && (filled_slot(d, fill, s) < 0 || *S.id(g) != (uint32_t)id)) return;
    PT v[3];
    load_field<DIM, PT, WHAT == GATHER_VEL>(S, g, v);
#pragma unroll
    for (int q = 0; q < DIM; ++q) out[(long long)q * d.Np + id] = (double)v[q];
}

template <int DIM, typename PT>
__global__ void __launch_bounds__(WG) k_cell_count(const InstDesc* __restrict__ D, int inst, PStore<DIM, PT> P,
                                                   const uint32_t* __restrict__ fill, int* count, long long t,
                                                   int sub) {
    const InstDesc& d = D[inst];
    const long long s = (long long)blockIdx.x * WG + threadIdx.x;
    if (s >= d.ntiles * d.cap) return;
    const long long lt = s / d.cap;
    const int k = (int)(s % d.cap);
    uint32_t n = fill[d.tile_off + lt];
    if (n > (uint32_t)d.cap) n = (uint32_t)d.cap;
    if ((uint32_t)k >= n) return;
    const long long g = d.slot_off + s;
    PT sh[3];
    grid_shift_of<DIM, PT>(d, (uint32_t)t, (uint32_t)sub, sh);
    const PT rr = (PT)d.r;
    int ix = bin_coord<PT>(*P.pos(0, g), (PT)0, sh[0], rr);
    if (ix >= d.Cx) ix -= d.Cx;
    const int iy = bin_row<PT>(d, *P.pos(1, g), sh[1], rr);
    int iz = 0;
    if (DIM == 3) {
        iz = bin_coord<PT>(*P.pos(2, g), (PT)0, sh[2], rr);
        if (iz >= d.Cz) iz -= d.Cz;
    }
    atomicAdd(&count[ix + d.Cx * (iy + d.CyB * iz)], 1);
}

// Overwrite positions (which = 0) or velocities (1) of one instance by id.
// The sources of a tile's particles lie in its surroundings, which the
// XCD-blocked order keeps in one L2; from 2^25 particles on they overflow it,
// and the XCDs share them better going through the tiles together (41.9M
// binary32 particles after 200 LB steps: 2627 us blocked, 2377 in order; 10.5M
// in 2D: 397 and 507).
template <int DIM, typename PT>
__global__ void __launch_bounds__(WG) k_set_field(const InstDesc* __restrict__ D, int inst, PStore<DIM, PT> P,
                                                  const uint32_t* __restrict__ fill, int which,
                                                  const double* __restrict__ src) {
    const InstDesc& d = D[inst];
    const long long g = filled_slot(d, fill, (d.Np < (1 << 25) ? xcd_item() : (long long)blockIdx.x) * WG + threadIdx.x);
    if (g < 0) return;
    const uint32_t id = *P.id(g);
    if ((long long)id >= d.Np) return;
#pragma unroll
    for (int q = 0; q < DIM; ++q) *(which == 0 ? P.pos(q, g) : P.vel(q, g)) = (PT)src[(long long)q * d.Np + id];
}

__global__ void __launch_bounds__(WG) k_zero(uint32_t* p, long long nwords) {
    const long long i = (long long)blockIdx.x * WG + threadIdx.x;
    if (i < nwords) p[i] = 0u;
}

// Sum of the NCOPY profile replicas of one instance: out[R][4].  A workgroup
// takes 64 outputs, each wave a quarter of the replicas, whose loads are
// independent (one thread walking over all 64 took 11.2 us for 72 rows, a
// quarter of them 4.6).
constexpr int PR_OUT = 64;

__global__ void __launch_bounds__(WG) k_profile_reduce(const InstDesc* __restrict__ D, int inst,
                                                       const double* __restrict__ prof, double* out) {
    __shared__ double part[WG / PR_OUT][PR_OUT];
    const InstDesc& d = D[inst];
    const int lane = threadIdx.x % PR_OUT, w = threadIdx.x / PR_OUT;
    const int i = blockIdx.x * PR_OUT + lane;
    const bool in = i < d.R * 4;
    double s = 0.0;
    constexpr int PER = NCOPY / (WG / PR_OUT);
#pragma unroll
    for (int c = 0; c < PER; ++c) {
        const double* v = &prof[(d.prof_off + (long long)(w * PER + c) * d.R) * 4 + (in ? i : 0)];
        s += d.det ? fix_bits(v) : *v;  // fixed-point sums in the deterministic mode
    }
    part[w][lane] = s;
    __syncthreads();
    if (w > 0 || !in) return;
    for (int k = 1; k < WG / PR_OUT; ++k) s += part[k][lane];
    out[i] = s;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static inline unsigned nblk(long long n) { return (unsigned)((n + WG - 1) / WG); }


hipError_t launch_part_init(int dim, int part_fp, const InstDesc* D, int n_inst, long long total, PartBuf buf,
                            hipStream_t s) {
    if (total <= 0) return hipSuccess;
    dim3 g(nblk(total)), b(WG);
    if (dim == 2 && part_fp == 64) hipLaunchKernelGGL((k_part_init<2, double>), g, b, 0, s, D, n_inst, total, buf);
    else if (dim == 2) hipLaunchKernelGGL((k_part_init<2, float>), g, b, 0, s, D, n_inst, total, buf);
    else if (part_fp == 64) hipLaunchKernelGGL((k_part_init<3, double>), g, b, 0, s, D, n_inst, total, buf);
    else hipLaunchKernelGGL((k_part_init<3, float>), g, b, 0, s, D, n_inst, total, buf);
    return hipGetLastError();
}

hipError_t launch_fill_sequential(const InstDesc* D, int n_inst, long long tiles, uint32_t* fill,
                                  uint32_t* fill_other, hipStream_t s) {
    if (tiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_sequential, dim3(nblk(tiles)), dim3(WG), 0, s, D, n_inst, tiles, fill, fill_other);
    return hipGetLastError();
}

// From this many particles on, positions and velocities go through the inverse
// map (in `idle`, memory of at least 4 bytes a particle): one scattered 4-byte
// store a particle, then consecutive 8-byte stores, instead of a scattered
// 8-byte store for every component.  A tile's ids come from all its
// surroundings, the more so the longer the run.  us a field after 40 LB steps,
// directly / through the map: binary32 in 3D, which one or two loads fetch,
// 327k particles 15 / 17, 655k 29 / 24, 10.5M 409 / 380, 41.9M 3772 / 1464; in
// 2D 5M 168 / 211, 18.9M 1022 / 783; binary64 2D 10.5M 320 / 420, 18.9M 1020 /
// 788; 3D 10.5M 455 / 561, 21M 1427 / 1117.
template <int DIM, typename PT>
constexpr long long gather_inv_min() { return sizeof(PT) == 4 && DIM == 3 ? 1 << 19 : 1 << 24; }

template <int DIM, typename PT>
static void gather(const InstDesc* D, int inst, const InstDesc& d, PartBuf buf, const uint32_t* fill,
                   const DevStats* stats, double* pos_out, double* vel_out, int* cell_out, void* idle, long long t,
                   int sub, hipStream_t s) {
    const dim3 b(WG), slots(xcd_grid(nblk(d.ntiles * d.cap)));
    if (cell_out) {
        hipLaunchKernelGGL((k_scatter<DIM, PT, GATHER_CELL>), slots, b, 0, s, D, inst, buf, fill, nullptr, cell_out, t, sub);
    } else if (d.Np < gather_inv_min<DIM, PT>()) {
        if (pos_out) hipLaunchKernelGGL((k_scatter<DIM, PT, GATHER_POS>), slots, b, 0, s, D, inst, buf, fill, pos_out, nullptr, t, sub);
        else hipLaunchKernelGGL((k_scatter<DIM, PT, GATHER_VEL>), slots, b, 0, s, D, inst, buf, fill, vel_out, nullptr, t, sub);
    } else {
        const dim3 ids(nblk(d.Np));
        const uint32_t* slot = (const uint32_t*)idle;
        hipLaunchKernelGGL((k_scatter<DIM, PT, GATHER_INV>), slots, b, 0, s, D, inst, buf, fill, nullptr, (int*)idle, t, sub);
        if (pos_out) hipLaunchKernelGGL((k_gather<DIM, PT, GATHER_POS>), ids, b, 0, s, D, inst, buf, fill, stats, slot, pos_out);
        else hipLaunchKernelGGL((k_gather<DIM, PT, GATHER_VEL>), ids, b, 0, s, D, inst, buf, fill, stats, slot, vel_out);
    }
}

hipError_t launch_gather(int dim, int part_fp, const InstDesc* D, int inst, const InstDesc& d, PartBuf buf,
                         const uint32_t* fill, const DevStats* stats, double* pos_out, double* vel_out, int* cell_out,
                         void* idle, long long t, int sub, hipStream_t s) {
    if (d.ntiles <= 0) return hipSuccess;
    if (dim == 2 && part_fp == 64) gather<2, double>(D, inst, d, buf, fill, stats, pos_out, vel_out, cell_out, idle, t, sub, s);
    else if (dim == 2) gather<2, float>(D, inst, d, buf, fill, stats, pos_out, vel_out, cell_out, idle, t, sub, s);
    else if (part_fp == 64) gather<3, double>(D, inst, d, buf, fill, stats, pos_out, vel_out, cell_out, idle, t, sub, s);
    else gather<3, float>(D, inst, d, buf, fill, stats, pos_out, vel_out, cell_out, idle, t, sub, s);
    return hipGetLastError();
}

hipError_t launch_cell_count(int dim, int part_fp, const InstDesc* D, int inst, PartBuf buf, const uint32_t* fill,
                             int* count_out, long long slots, long long t, int sub, hipStream_t s) {
    if (slots <= 0) return hipSuccess;
    dim3 g(nblk(slots)), b(WG);
    if (dim == 2 && part_fp == 64) hipLaunchKernelGGL((k_cell_count<2, double>), g, b, 0, s, D, inst, typed<2, double>(buf), fill, count_out, t, sub);
    else if (dim == 2) hipLaunchKernelGGL((k_cell_count<2, float>), g, b, 0, s, D, inst, typed<2, float>(buf), fill, count_out, t, sub);
    else if (part_fp == 64) hipLaunchKernelGGL((k_cell_count<3, double>), g, b, 0, s, D, inst, typed<3, double>(buf), fill, count_out, t, sub);
    else hipLaunchKernelGGL((k_cell_count<3, float>), g, b, 0, s, D, inst, typed<3, float>(buf), fill, count_out, t, sub);
    return hipGetLastError();
}

hipError_t launch_set_field(int dim, int part_fp, const InstDesc* D, int inst, PartBuf buf, const uint32_t* fill,
                            int which, const double* src, long long slots, hipStream_t s) {
    if (slots <= 0) return hipSuccess;
    dim3 g(xcd_grid(nblk(slots))), b(WG);
    if (dim == 2 && part_fp == 64) hipLaunchKernelGGL((k_set_field<2, double>), g, b, 0, s, D, inst, typed<2, double>(buf), fill, which, src);
    else if (dim == 2) hipLaunchKernelGGL((k_set_field<2, float>), g, b, 0, s, D, inst, typed<2, float>(buf), fill, which, src);
    else if (part_fp == 64) hipLaunchKernelGGL((k_set_field<3, double>), g, b, 0, s, D, inst, typed<3, double>(buf), fill, which, src);
    else hipLaunchKernelGGL((k_set_field<3, float>), g, b, 0, s, D, inst, typed<3, float>(buf), fill, which, src);
    return hipGetLastError();
}

hipError_t launch_zero(void* p, size_t bytes, hipStream_t s) {
    const long long nw = (long long)(bytes / 4);
    if (nw <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero, dim3(nblk(nw)), dim3(WG), 0, s, (uint32_t*)p, nw);
    return hipGetLastError();
}

// Exclusive prefix sum of n ints in place, by one workgroup walking the
// array in chunks (a diagnostic field; n is the cell count of one channel).
__global__ void __launch_bounds__(WG) k_exclusive_scan(int* a, long long n) {
    __shared__ int part[WG];
    __shared__ int carry;
    const int tid = threadIdx.x;
    if (tid == 0) carry = 0;
    __syncthreads();
    for (long long c0 = 0; c0 < n; c0 += WG) {
        const long long i = c0 + tid;
        const int v = i < n ? a[i] : 0;
        part[tid] = v;
        __syncthreads();
        // Hillis-Steele inclusive scan of the chunk
        for (int o = 1; o < WG; o <<= 1) {
            const int add = tid >= o ? part[tid - o] : 0;
            __syncthreads();
            part[tid] += add;
            __syncthreads();
        }
        if (i < n) a[i] = carry + part[tid] - v;
        __syncthreads();
        if (tid == WG - 1) carry += part[WG - 1];
        __syncthreads();
    }
}

hipError_t launch_exclusive_scan(int* a, long long n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_exclusive_scan, dim3(1), dim3(WG), 0, s, a, n);
    return hipGetLastError();
}

// Mean particle velocity per slab node from the per-node sample sums
// [count, sum v_x, sum v_y, sum v_z]: out[q][node], zero where no particle.
__global__ void __launch_bounds__(WG) k_node_mean(const double* acc, long long nslab, int dim, int det,
                                                  double* out) {
    const long long i = (long long)blockIdx.x * WG + threadIdx.x;
    if (i >= nslab) return;
    const double* a = acc + 4 * i;
    double v[4];
    for (int q = 0; q < 4; ++q) v[q] = det ? fix_bits(a + q) : a[q];  // fixed point in the deterministic mode
    for (int q = 0; q < dim; ++q) out[(long long)q * nslab + i] = v[0] > 0.0 ? v[1 + q] / v[0] : 0.0;
}

hipError_t launch_node_mean(const double* acc, long long nslab, int dim, int det, double* out, hipStream_t s) {
    if (nslab <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_node_mean, dim3(nblk(nslab)), dim3(WG), 0, s, acc, nslab, dim, det, out);
    return hipGetLastError();
}

hipError_t launch_profile_reduce(const InstDesc* D, int inst, int R, const double* prof, double* out, hipStream_t s) {
    if (R <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_profile_reduce, dim3((unsigned)((4LL * R + PR_OUT - 1) / PR_OUT)), dim3(WG), 0, s, D, inst, prof,
                       out);
    return hipGetLastError();
}

}  // namespace lbmpcd

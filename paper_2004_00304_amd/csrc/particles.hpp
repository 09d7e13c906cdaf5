// particles.hpp -- the fused MPCD step for gfx950 (the particle kernel template;
// kernels_mpcd.hip, kernels_mpcd_ce.hip and kernels_mpcd_det.hip instantiate it).
//
// Particle layout.  The cells of the shifted grid are grouped into tiles of
// Tx x Ty x Tz cells; every tile owns `cap` slots of the particle buffer
// (PStore).  After the binning of an MPCD step every
// particle sits in the slots of the tile that contains its cell, in no
// particular order inside the tile.
//
// k_particles: one workgroup per tile, one launch per MPCD step.
//   phase 1 (collision of the previous binning, Eq. 4): cell occupancy and
//     momentum summed in LDS (FP64 atomics); the rotation of every cell
//     (2D sign / 3D axis) is drawn while the tile's particles are loading;
//     in wall-cut cells the virtual particles' momentum is added; every
//     particle is rotated about its cell's centre of mass in registers;
//   phase 2 (next MPCD step): Maxwell-Boltzmann redraw of buffer particles
//     (exchange step of Alg. 1; with mode bit 8 the first-order
//     Chapman-Enskog redraw instead) about the LB velocity of their fine cell,
//     which the workgroup copied into LDS for every buffer cell of the tile
//     while the particles were loading, streaming with the body force (Eq. 3) and
//     boundary conditions, samples of the last MPCD step of an LB step,
//     binning into the new shifted grid;
//   phase 3 (counting sort into tiles): each wave groups its particles by
//     destination tile; the first lane of a group claims a row of a small LDS
//     table of destination tiles; one global atomic per destination reserves a
//     run of slots, and every store writes the lanes of a group to consecutive
//     slots.
// Every particle is read once and written once per MPCD step.
//
// With binary32 particles the launch is bound by vector issue (thin film 84 %
// of the cycles), so what every particle executes is kept short: one test for
// both periodic axes, wrapped only where it fails; the body of the boundary
// conditions alone checks for finite velocities; the exchange is decided by
// comparing positions; 24-bit products in the tile index, and none in the slot
// of a store; the normals' quotients and roots without the IEEE sequences'
// range handling (thin film 5.38 -> 5.19 ms per MPCD step, 3D channel 2.39 ->
// 2.32, with MPCD-AT 3.08 -> 2.96; the binary64 ensemble, bound by latency,
// 2.10 -> 2.09).  All of it gives the same bits; fused multiply-adds in the
// rotation would not (film 5.12, 3D channel 2.30): a rounding that differs
// makes another realisation of every long run.
#pragma once

#include <cmath>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"

namespace lbmpcd {

template <typename PT>
struct PArgs {
    const InstDesc* D;
    PartBuf in, out;
    uint32_t* fill_in;
    uint32_t* fill_out;
    const int* tile_inst;
    const double* ufine;
    const double* tfine;
    double* acc;
    double* prof;
    DevStats* stats;
    const long long* clock;
    const double* shifts;
    double* cell_vcm;
    int coll_dt, coll_s, str_s, do_fb, do_prof, diag_inst;
    long long ntiles;  // tiles of all instances
    long long xcd_per; // > 0: tiles per XCD of the XCD-blocked order, 0: workgroup b takes tile b
    // Overflow list: [0] tiles listed, [1] workgroups of the overflow pass
    // done, [2..] tiles.  ovf_mode 0: every tile fits the launch's slots;
    // 1: a tile with more particles than NT * PPT is listed and skipped;
    // 2: the overflow pass over the listed tiles.
    uint32_t* ovf;
    int ovf_mode;
};

template <typename PT>
__device__ __forceinline__ PT wrap_periodic(PT x, PT lo, PT L) {
    if (x < lo) x = x + L;
    if (x >= lo + L) x = x - L;
    return x;
}

template <typename PT>
__device__ __forceinline__ PT fma_t(PT a, PT b, PT c);
template <>
__device__ __forceinline__ float fma_t<float>(float a, float b, float c) { return fmaf(a, b, c); }
template <>
__device__ __forceinline__ double fma_t<double>(double a, double b, double c) { return fma(a, b, c); }

template <typename PT>
__device__ __forceinline__ PT prev_below(PT v, PT toward);
template <>
__device__ __forceinline__ float prev_below<float>(float v, float toward) { return nextafterf(v, toward); }
template <>
__device__ __forceinline__ double prev_below<double>(double v, double toward) { return nextafter(v, toward); }

// Normal deviates of the exchange step, inlined: a call would make the
// caller save and restore most of its scalar registers around it.
template <int DIM>
__device__ __forceinline__ void reinject_normals(Key key, uint32_t id, uint32_t t, uint32_t sub, double* z) {
    rng_normals<DIM>(key, id, t, sub, P_REINJ, z);
}

// Chapman-Enskog exchange (a first-order Chapman-Enskog distribution about
// the LB velocity, sampled as Garcia and Alexander do, by acceptance-rejection
// against the Maxwellian): the weight of a thermal velocity z (units of
// sqrt(kT/m)) is 1 - T:zz.  Attempt k draws z from the Philox blocks 4k and
// 4k + 1 of the element's exchange stream -- attempt 0 is the Maxwell-
// Boltzmann draw -- and a uniform u from block 4k + 2, and is accepted when
// A u <= 1 - T:zz; A = 1 + CE_KAPPA b, b the largest absolute row sum of T.
// After CE_ATTEMPTS rejections the first draw stands.
template <int DIM>
__device__ __forceinline__ void ce_normals_at(Key key, uint32_t id, uint32_t t, uint32_t sub, uint32_t blk,
                                              double z[3]) {
    U4 w = rng_block(key, id, t, sub, P_REINJ, blk);
    if constexpr (DIM == 2) {
        box_muller(u01(w.x, w.y), u01(w.z, w.w), z[0], z[1]);
        z[2] = 0.0;
    } else {
        const double u0 = u01(w.x, w.y), u1 = u01(w.z, w.w);
        w = rng_block(key, id, t, sub, P_REINJ, blk + 1);
        double dummy;
        box_muller(u0, u1, z[0], z[1]);
        box_muller(u01(w.x, w.y), u01(w.z, w.w), z[2], dummy);
    }
}

// T:zz with T = (xx, yy, zz, xy, xz, yz), summed in that order
template <int DIM>
__device__ __forceinline__ double ce_contract(const double T[6], const double z[3]) {
    if constexpr (DIM == 2) return T[0] * z[0] * z[0] + T[1] * z[1] * z[1] + 2.0 * (T[3] * z[0] * z[1]);
    return T[0] * z[0] * z[0] + T[1] * z[1] * z[1] + T[2] * z[2] * z[2] +
           2.0 * (T[3] * z[0] * z[1] + T[4] * z[0] * z[2] + T[5] * z[1] * z[2]);
}

// The attempts after the first (rare: the first is accepted with
// probability about 1/A), out of line so that the particle kernel's unrolled
// exchange carries one call instead of a copy of the loop per particle.
struct CEDraw { double z0, z1, z2; };

template <int DIM>
__device__ __noinline__ CEDraw ce_retry(Key key, uint32_t id, uint32_t t, uint32_t sub, double T0, double T1,
                                        double T2, double T3, double T4, double T5, double A, CEDraw first) {
    const double T[6] = {T0, T1, T2, T3, T4, T5};
    for (int k = 1; k < CE_ATTEMPTS; ++k) {
        double zk[3];
        ce_normals_at<DIM>(key, id, t, sub, 4u * (uint32_t)k, zk);
        const U4 w = rng_block(key, id, t, sub, P_REINJ, 4u * (uint32_t)k + 2u);
        if (A * u01(w.x, w.y) <= 1.0 - ce_contract<DIM>(T, zk)) return CEDraw{zk[0], zk[1], zk[2]};
    }
    return first;
}

template <int DIM>
__device__ __forceinline__ void ce_redraw(Key key, uint32_t id, uint32_t t, uint32_t sub, const double* tf,
                                          long long NF, long long fc, double z[3]) {
    double T[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    T[0] = tf[fc];
    T[1] = tf[NF + fc];
    T[3] = tf[3 * NF + fc];
    if constexpr (DIM == 3) {
        T[2] = tf[2 * NF + fc];
        T[4] = tf[4 * NF + fc];
        T[5] = tf[5 * NF + fc];
    }
    const double r0 = fabs(T[0]) + fabs(T[3]) + fabs(T[4]);
    const double r1 = fabs(T[3]) + fabs(T[1]) + fabs(T[5]);
    const double r2 = fabs(T[4]) + fabs(T[5]) + fabs(T[2]);
    const double A = 1.0 + CE_KAPPA * fmax(r0, fmax(r1, r2));
    const U4 w = rng_block(key, id, t, sub, P_REINJ, 2u);
    if (A * u01(w.x, w.y) <= 1.0 - ce_contract<DIM>(T, z)) return;
    const CEDraw r = ce_retry<DIM>(key, id, t, sub, T[0], T[1], T[2], T[3], T[4], T[5], A, CEDraw{z[0], z[1], z[2]});
    z[0] = r.z0;
    z[1] = r.z1;
    z[2] = r.z2;
}

// Read-only tables (descriptors, tile owners, grid shifts, fill counts of
// tiles not yet processed) are read through the constant address space:
// scalar loads, which the compiler may not use for ordinary global pointers
// once the loop over tiles has stored anything.
template <typename T>
using cst = __attribute__((address_space(4))) const T;
template <typename T>
__device__ __forceinline__ cst<T>* cptr(const T* p) { return (cst<T>*)p; }

__device__ __forceinline__ void lds_add(double* p, double v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void gl_add(double* p, double v) { unsafeAtomicAdd(p, v); }

// A sum in LDS or global memory: FP64 atomics, or with DET (deterministic
// mode) fixed-point integer atomics in the same 8-byte slot (to_fix).
template <bool DET>
__device__ __forceinline__ void sum_lds(double* p, double v) {
    if constexpr (DET) atomicAdd((unsigned long long*)p, to_fix(v));
    else lds_add(p, v);
}
template <bool DET>
__device__ __forceinline__ void sum_gl(double* p, double v) {
    if constexpr (DET) atomicAdd((unsigned long long*)p, to_fix(v));
    else gl_add(p, v);
}
template <bool DET>
__device__ __forceinline__ double sum_read(const double* p) {
    if constexpr (DET) return fix_bits(p);
    else return *p;
}

// Mode bit of the collision with replicated cell sums (512 threads, contexts
// with a channel of dense cells): an instantiation of its own, since the
// replicas' code costs MPCD-AT 5 to 15 % where no cell has any (2D, 4,352 tiles,
// 512 threads: 0.667 -> 0.605 ms a coupled step, deterministic 0.721 -> 0.618).
constexpr int MODE_REPS = 32;

// LDS carve-up (bytes): header (counters and the table of destination tiles),
// then one region that holds the collision arrays and the tile's window of
// buffer-cell LB velocities first, and the sample windows afterwards.
constexpr int NHASH_BITS = 6;
constexpr int NHASH = 1 << NHASH_BITS;
constexpr int SINGLES = 16;  // waiting lanes of a wave that claim their places singly
constexpr size_t LDS_HDR = 1088;  // >= 4 * (4 + 3 * NHASH + 2), a multiple of 16
// Node sample window: NREP interleaved replicas of every bin (lane l adds into
// replica l mod NREP), so that the lanes of a wave, which mostly sample the
// same few nodes, spread their FP64 atomics over more banks.  Profile window:
// a wave's particles lie in two or three fine rows, so every row has WSLOTS
// slots, component by component (lane l adds into slot l mod WSLOTS); with four
// replicas per row and the region of its own that they had before, a sampling
// launch of the thin film took 6.83 ms, with a slot per lane 6.66.  Sixteen, summed
// by one thread per row and component, cost small tiles less than a slot per
// lane summed by shuffles (binary32 in 2D, 12,700 tiles of 640 particles, a
// sampled step 300 -> 283 us; film cut by 16, one MPCD step 1369 -> 1366).
constexpr int NREP = 4;
constexpr int WSLOTS = 16;
constexpr int PROF_SLOTS = MAX_WJ * WSLOTS;  // rows x slots per row of the profile window
constexpr size_t LDS_WIN = ((size_t)MAX_WIN * NREP * 4 + (size_t)PROF_SLOTS * 4) * sizeof(double);
// The exchange reads the LB velocity of a buffer particle's fine cell.  A
// particle binned into shifted cell i (shift in [0, a)) sits in unshifted
// fine cell i - 1 or i, so the particles of a tile of Tx x Ty x Tz cells read
// at most (Tx + 1)(Ty + 1)(Tz + 1) fine cells, which the workgroup copies into
// LDS at the start of the launch, where the loads overlap the particle loads
// and the collision instead of stalling the exchange.
constexpr size_t LDS_COLL = (size_t)MAX_NCT * 4 + (size_t)MAX_NCT * 9 * sizeof(double) +
                            (size_t)MAX_UFC * 3 * sizeof(double);
constexpr size_t LDS_UNI = LDS_COLL > LDS_WIN ? LDS_COLL : LDS_WIN;
constexpr uint32_t DROP_SLOT = 0x7FFFFFFFu;  // never a slot: the slot total stays below it
constexpr long long OVF_GRID = 128;           // workgroups of the overflow pass
static_assert(4 * (4 + 3 * NHASH + 2) <= (int)LDS_HDR, "LDS header too small");

// Minimum resident waves per SIMD the register allocation must allow.  With
// binary32 particles (eight per thread) and in the Chapman-Enskog modes the
// kernel spills at four (128 VGPRs) and runs faster at three (on MI355X:
// 3.45 against 3.49 ms per MPCD step of the 3D channel with SRD, 4.93 against
// 5.78 with MPCD-AT, 4.70 against 7.3 with the Chapman-Enskog exchange); with
// binary64 particles (the batched 2D ensemble) four is as fast, but for eight
// per thread and for six with MPCD-AT, which spill up to 254 registers at four
// and none to 19 at three (coupled step, 4,352 tiles in 2D: MPCD-AT 0.782 ->
// 0.622 ms, SRD with 128 threads 0.888 -> 0.573; 8,700 in 3D: MPCD-AT 1.583 ->
// 1.319), and in 3D for eight per thread with the Chapman-Enskog exchange,
// which spill up to 229 at three and none at two (2.49 -> 1.56 ms with 128
// threads; in 2D two is slower on small grids).  Six binary32 particles per
// thread fit five waves with SRD and four with MPCD-AT without spilling; the
// Chapman-Enskog modes stay at three.
template <int DIM, typename PT, int MODE, int PPT>
constexpr int particle_waves() {
    if (DIM == 3 && sizeof(PT) == 8 && PPT == 8 && (MODE & 8)) return 2;
    if (sizeof(PT) == 8 && (PPT == 8 || (PPT == 6 && (MODE & 4)))) return 3;
    if (PPT == 6 && sizeof(PT) == 4) return (MODE & 8) ? 3 : (MODE & 4) ? 4 : 5;
    return (sizeof(PT) == 4 || (MODE & 8) != 0) ? 3 : 4;
}

// One workgroup per tile.
template <int DIM, typename PT, int NT, int PPT, int MODE>
__device__ __forceinline__ void particle_tile(const PArgs<PT>& A, long long T, unsigned char* smem) {
    constexpr bool COLL = (MODE & 1) != 0;
    constexpr bool STREAM = (MODE & 2) != 0;
    constexpr bool AT = (MODE & 4) != 0;  // MPCD-AT collision (Eq. 6) instead of SRD (Eq. 4)
    constexpr bool CE = (MODE & 8) != 0;  // Chapman-Enskog exchange instead of Maxwell-Boltzmann
    constexpr bool DET = (MODE & 16) != 0;  // deterministic: fixed-point integer sums
    uint32_t* wstat = (uint32_t*)smem;          // [4] far moves, misplaced, samples outside the LDS windows,
                                                // invalid particles
    uint32_t* hkey = wstat + 4;                 // [NHASH] destination tiles (local index)
    uint32_t* hcnt = hkey + NHASH;              // [NHASH + 1] particles per destination
    uint32_t* gbase = hcnt + NHASH + 1;         // [NHASH + 1] reserved run start
    unsigned char* uni = smem + LDS_HDR;
    double* wacc = (double*)uni;                // [MAX_WIN][NREP][4] node sample window
    double* wprof = wacc + MAX_WIN * NREP * 4;  // [4][rows][slots] profile window
    // Cell sums: in tiles of at most four cells (hundreds of particles per
    // cell, which 512 threads serve) every cell keeps eight replicas, lane l
    // adding into replica l mod 8, so that a cell's particles do not all meet
    // on one address.  Coupled step of the paper's channel (centre line, MPCD-AT,
    // binary64) without, with eight and with 32: 1,000 particles per cell 40.2,
    // 32.3 and 33.9 us, at 200 nodes' length 155, 109 and 119; 250 per cell, 1,000
    // nodes 145, 137 and 151 (the 32 have to be summed).  More cells per tile
    // measure slower with 32 replicas (2D channel with eight per cell 51.1 ->
    // 52.9 us).
    uint32_t* ccnt = (uint32_t*)uni;                 // [MAX_NCT]
    double* csv = (double*)(uni + MAX_NCT * 4);      // [MAX_NCT][3]
    double* cvcm = csv + MAX_NCT * 3;                // [MAX_NCT][3]
    double* ucache = cvcm + MAX_NCT * 6;          // [3][MAX_UFC] LB velocities of the tile's buffer cells
    double* crot = cvcm + MAX_NCT * 3;               // [MAX_NCT][3] SRD sign/axis; MPCD-AT: sum, then mean, of the random velocities

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int ii = cptr(A.tile_inst)[T];
    cst<InstDesc>& d = cptr(A.D)[ii];
    const Key key = key_of(d);
    // The Philox key at a draw site, pinned to scalar registers there, so
    // that the compiler derives the round keys next to each draw (scalar
    // additions) instead of keeping twenty of them live across the kernel,
    // which spills other scalars into vector lanes.
    auto kfresh = [&]() {
        Key k = key;
        asm volatile("" : "+s"(k.k0), "+s"(k.k1));
        return k;
    };
    // tile coordinates in 32-bit arithmetic (a channel has fewer than 2^31 tiles)
    const uint32_t lt = (uint32_t)(T - d.tile_off);
    const uint32_t nxy = (uint32_t)d.ntx * (uint32_t)d.nty;
    const uint32_t tzu = lt / nxy, rem = lt - tzu * nxy;
    const uint32_t tyu = rem / (uint32_t)d.ntx;
    const int tx = (int)(rem - tyu * (uint32_t)d.ntx), ty = (int)tyu, tz = (int)tzu;
    const int cap = d.cap;
    const long long base = d.slot_off + (long long)lt * cap;
    uint32_t n = cptr(A.fill_in)[T];
    if (A.ovf_mode == 1 && n > (uint32_t)(NT * PPT)) {
        // more particles than this launch's slots: left untouched for the
        // overflow pass, which takes the tiles of this list
        if (tid == 0) A.ovf[2 + atomicAdd(&A.ovf[0], 1u)] = (uint32_t)T;
        return;
    }
    if (n > (uint32_t)cap) n = (uint32_t)cap;
    constexpr bool REPS = (MODE & MODE_REPS) != 0;
    [[maybe_unused]] const int lrep = REPS ? d.lrep : 0;
    const long long t_now = *cptr(A.clock);
    const PT rr = (PT)d.r;
    cst<double>* shtab = cptr(A.shifts) + (long long)ii * 2 * d.S * 3;
    const long long tcl = t_now + A.coll_dt;
    const uint32_t tc = (uint32_t)tcl;
    const uint32_t sc = (uint32_t)A.coll_s;

    // ---- load (the rotations below are drawn while the loads are in flight)
    uint32_t pid[PPT];
    PT px[PPT][3], pv[PPT][3];
    bool valid[PPT];
    // What would be spilled as it arrives is loaded later, since each such
    // load waits for the one before it: an id in an array of its own, needed
    // first by the draws after an SRD collision, is loaded there (binary64
    // ensemble 2.53 -> 2.10 ms per MPCD step), and of six binary32 records
    // the last comes after the rotations are drawn, whose FP64 series need the
    // registers (95 VGPRs and 16 spilled bytes -> 89 and none; film 5.51 ->
    // 5.38 ms).  MPCD-AT and the Chapman-Enskog modes do not spill there; in
    // binary64 fewer waves end their spills (particle_waves), later loads do not.
    constexpr bool ID_LATE = PStore<DIM, PT>::ID_APART && !AT;
    constexpr int FIRST = (PPT == 6 && sizeof(PT) == 4 && !AT && !CE) ? PPT - 1 : PPT;
    auto load = [&](int k) {
        const int s = tid + k * NT;
        valid[k] = s < (int)n;
        // (an absent particle's registers are never read)
        if (!valid[k]) return;
        load_part<DIM, PT>(A.in, base, (uint32_t)s, px[k], pv[k], pid[k]);
        if constexpr (PStore<DIM, PT>::ID_APART && !ID_LATE) pid[k] = load_id<DIM, PT>(A.in, base, (uint32_t)s);
    };
#pragma unroll
    for (int k = 0; k < FIRST; ++k) load(k);
    if (tid == 0 && n > (uint32_t)(3 * cap / 4)) atomicMax(&A.stats->max_fill, n);
    if (tid < 4) wstat[tid] = 0u;
    if constexpr (STREAM) {
        for (int i = tid; i < NHASH; i += NT) hkey[i] = BAD_SLOT;
        for (int i = tid; i <= NHASH; i += NT) hcnt[i] = 0u;
    }
    // window of fine cells (origin one cell below the tile on each axis);
    // only buffer rows are copied, and only for tiles that reach them
    if constexpr (STREAM) {
        const int uwx = d.Tx + 1, uwy = d.Ty + 1, uwz = (DIM == 3) ? d.Tz + 1 : 1;
        const int uJ0 = (ty << d.lTy) - 1;
        const int rbl = d.buf_lo * d.r, rbh = d.R - d.buf_hi * d.r;
        if (((uJ0 < rbl) || (uJ0 + uwy - 1 >= rbh)) && uwx * uwy * uwz <= MAX_UFC) {
            const int uI0 = (tx << d.lTx) - 1, uK0 = (DIM == 3) ? (tz << d.lTz) - 1 : 0;
            const long long NFc = (long long)d.Cx * d.NB * d.Cz;
            const double* ufc = A.ufine + d.ufine_off * DIM;
            for (int i = tid; i < uwx * uwy * uwz; i += NT) {
                const int ax = i % uwx, ay = (i / uwx) % uwy, az = i / (uwx * uwy);
                const int J = uJ0 + ay;
                if (J < 0 || J >= d.R || (J >= rbl && J < rbh)) continue;
                const int I = ((uI0 + ax) % d.Cx + d.Cx) % d.Cx;
                const int K = (DIM == 3) ? ((uK0 + az) % d.Cz + d.Cz) % d.Cz : 0;
                const int Jb = (J < rbl) ? J : J - (d.R - d.NB);
                const long long fc = ((long long)K * d.NB + Jb) * d.Cx + I;
#pragma unroll
                for (int q = 0; q < DIM; ++q) ucache[q * MAX_UFC + i] = ufc[q * NFc + fc];
            }
        }
    }

    // rotation of every cell of the tile (2D sign / 3D axis): independent of
    // the particles
    if constexpr (COLL) {
        for (int j = tid; j < d.nct; j += NT) {
            const int lx = j & (d.Tx - 1), ly = (j >> d.lTx) & (d.Ty - 1), lz = j >> (d.lTx + d.lTy);
            const int ix = (tx << d.lTx) + lx, iy = (ty << d.lTy) + ly, iz = (tz << d.lTz) + lz;
            const uint32_t cg = (uint32_t)(ix + d.Cx * (iy + d.CyB * iz));
            const U4 w = AT ? U4{0u, 0u, 0u, 0u} : rng_block(kfresh(), cg, tc, sc, P_ROT, 0);
            if constexpr (AT) {
                if constexpr (!REPS) { crot[3 * j] = 0.0; crot[3 * j + 1] = 0.0; crot[3 * j + 2] = 0.0; }
            } else if constexpr (DIM == 2) {
                crot[3 * j] = (w.x & 1u) ? 1.0 : -1.0;
            } else {
                const double u0 = u01(w.x, w.y), u1 = u01(w.z, w.w);
                const double nz = 2.0 * u0 - 1.0;  // azimuth 2 pi u1
                const double sxy = sqrt(fmax(0.0, 1.0 - nz * nz));
                double sp, cp;
                sincos_2pi(u1, &sp, &cp);
                crot[3 * j] = sxy * cp;
                crot[3 * j + 1] = sxy * sp;
                crot[3 * j + 2] = nz;
            }
            if constexpr (!REPS) {
                ccnt[j] = 0u;
                csv[3 * j] = 0.0; csv[3 * j + 1] = 0.0; csv[3 * j + 2] = 0.0;
            }
        }
        if constexpr (REPS) {
            for (int j = tid; j < (d.nct << lrep); j += NT) {
                ccnt[j] = 0u;
                csv[3 * j] = 0.0; csv[3 * j + 1] = 0.0; csv[3 * j + 2] = 0.0;
                if constexpr (AT) { crot[3 * j] = 0.0; crot[3 * j + 1] = 0.0; crot[3 * j + 2] = 0.0; }
            }
        }
    }
#pragma unroll
    for (int k = FIRST; k < PPT; ++k) load(k);
    if constexpr (COLL) __syncthreads();

    // ---- phase 1: collision (SRD, or MPCD-AT) of the binning these particles sit in
    if constexpr (COLL) {
        cst<double>* shc = shtab + ((tcl & 1) * d.S + sc) * 3;
        const PT sh[3] = {(PT)shc[0], (PT)shc[1], (PT)shc[2]};
        int lc[PPT];
        // MPCD-AT: each particle's random velocity (variance kT/m per
        // component, keyed by its id and the collision's MPCD step; binary32
        // normals for binary32 particles), kept in the particle precision
        // between the two passes over the cell
        [[maybe_unused]] PT vr[AT ? PPT : 1][3];
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            lc[k] = -1;
            if (!valid[k]) continue;
            int ix = bin_coord<PT>(px[k][0], (PT)0, sh[0], rr);
            if (ix >= d.Cx) ix -= d.Cx;
            const int iy = bin_row<PT>(d, px[k][1], sh[1], rr);
            int iz = 0;
            if constexpr (DIM == 3) {
                iz = bin_coord<PT>(px[k][2], (PT)0, sh[2], rr);
                if (iz >= d.Cz) iz -= d.Cz;
            }
            const int lx = ix - (tx << d.lTx), ly = iy - (ty << d.lTy), lz = iz - (tz << d.lTz);
            if ((unsigned)lx >= (unsigned)d.Tx || (unsigned)ly >= (unsigned)d.Ty ||
                (unsigned)lz >= (unsigned)d.Tz) {
                atomicAdd(&wstat[1], 1u);
                continue;
            }
            const int c = lx + ((ly + (lz << d.lTy)) << d.lTx);
            lc[k] = c;
            const int cr = REPS ? (c << lrep) | (lane & ((1 << lrep) - 1)) : c;
            atomicAdd(&ccnt[cr], 1u);
#pragma unroll
            for (int q = 0; q < DIM; ++q) sum_lds<DET>(&csv[3 * cr + q], (double)pv[k][q]);
            if constexpr (AT) {
                double z[3];
                if constexpr (sizeof(PT) == 4) {
                    float zf[3];
                    rng_normals32<DIM>(kfresh(), pid[k], tc, sc, P_AT, zf);
#pragma unroll
                    for (int q = 0; q < 3; ++q) z[q] = (double)zf[q];
                } else {
                    rng_normals<DIM>(kfresh(), pid[k], tc, sc, P_AT, z);
                }
#pragma unroll
                for (int q = 0; q < DIM; ++q) {
                    vr[k][q] = (PT)(d.sd * z[q]);
                    sum_lds<DET>(&crot[3 * cr + q], (double)vr[k][q]);
                }
            }
        }
        __syncthreads();
        for (int j = tid; j < d.nct; j += NT) {
            const int lx = j & (d.Tx - 1), ly = (j >> d.lTx) & (d.Ty - 1), lz = j >> (d.lTx + d.lTy);
            const int ix = (tx << d.lTx) + lx, iy = (ty << d.lTy) + ly, iz = (tz << d.lTz) + lz;
            const int jr = REPS ? j << lrep : j;
            uint32_t nc = ccnt[jr];
            if constexpr (REPS) {
                // the replicas' sums into the first
                using Sum = std::conditional_t<DET, unsigned long long, double>;
                Sum *sv = (Sum*)csv, *sr = (Sum*)crot, v[3] = {0, 0, 0}, r[3] = {0, 0, 0};
                nc = 0u;
                for (int i = jr; i < (j + 1) << lrep; ++i) {
                    nc += ccnt[i];
#pragma unroll
                    for (int q = 0; q < DIM; ++q) {
                        v[q] += sv[3 * i + q];
                        if constexpr (AT) r[q] += sr[3 * i + q];
                    }
                }
#pragma unroll
                for (int q = 0; q < DIM; ++q) {
                    sv[3 * jr + q] = v[q];
                    if constexpr (AT) sr[3 * jr + q] = r[q];
                }
            }
            if (nc == 0u || ix >= d.Cx || iy >= d.CyB || iz >= d.Cz) continue;
            const uint32_t cg = (uint32_t)(ix + d.Cx * (iy + d.CyB * iz));
            // wall-cut cell below its nominal occupancy: nv virtual particles
            // with Maxwell-Boltzmann velocities (variance kT/m each), whose
            // velocity sum, of variance nv kT/m, enters the centre of mass
            double pvv[3] = {0.0, 0.0, 0.0}, mv = 0.0;
            const bool cut = ((double)sh[1] > 0.0) && ((d.bot_wall && iy == 0) || (d.top_wall && iy == d.R));
            if (cut && (int)nc < d.ppc) {
                double z[3];
                rng_normals<DIM>(kfresh(), cg, tc, sc, P_WALL, z);
                const int nv = d.ppc - (int)nc;
                const double sdv = sqrt((double)nv * d.kT / d.mass);
#pragma unroll
                for (int q = 0; q < DIM; ++q) pvv[q] = sdv * z[q];
                mv = (double)nv;
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) cvcm[3 * j + q] = 0.0;
#pragma unroll
            for (int q = 0; q < DIM; ++q) cvcm[3 * j + q] = (sum_read<DET>(&csv[3 * jr + q]) + pvv[q]) / ((double)nc + mv);
            if constexpr (AT) {
                // mean random velocity over the cell's real particles
#pragma unroll
                for (int q = 0; q < DIM; ++q) crot[3 * jr + q] = sum_read<DET>(&crot[3 * jr + q]) / (double)nc;
            }
            if (A.cell_vcm && ii == A.diag_inst) {
#pragma unroll
                for (int q = 0; q < DIM; ++q) A.cell_vcm[(long long)q * d.ncells + cg] = cvcm[3 * j + q];
            }
        }
        __syncthreads();
        const double ca = d.cos_a, sa = d.sin_a;
        [[maybe_unused]] const double one_c = 1.0 - ca;
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            if (lc[k] < 0) continue;
            const int c = lc[k];
            double vc[3] = {cvcm[3 * c], cvcm[3 * c + 1], cvcm[3 * c + 2]};
            if constexpr (AT) {
                // Eq. 6: centre of mass plus the random velocity less the cell mean
#pragma unroll
                for (int q = 0; q < DIM; ++q) pv[k][q] = (PT)(vc[q] + ((double)vr[k][q] - crot[3 * (REPS ? c << lrep : c) + q]));
                continue;
            }
            double wv[3] = {0.0, 0.0, 0.0}, rv[3];
#pragma unroll
            for (int q = 0; q < DIM; ++q) wv[q] = (double)pv[k][q] - vc[q];
            if constexpr (DIM == 2) {
                const double s = crot[3 * c] * sa;
                rv[0] = ca * wv[0] - s * wv[1];
                rv[1] = s * wv[0] + ca * wv[1];
            } else {
                const double a0 = crot[3 * c], a1 = crot[3 * c + 1], a2 = crot[3 * c + 2];
                const double nw = a0 * wv[0] + a1 * wv[1] + a2 * wv[2];
                const double cx = a1 * wv[2] - a2 * wv[1];
                const double cy = a2 * wv[0] - a0 * wv[2];
                const double cz = a0 * wv[1] - a1 * wv[0];
                rv[0] = wv[0] * ca + cx * sa + a0 * nw * one_c;
                rv[1] = wv[1] * ca + cy * sa + a1 * nw * one_c;
                rv[2] = wv[2] * ca + cz * sa + a2 * nw * one_c;
            }
#pragma unroll
            for (int q = 0; q < DIM; ++q) pv[k][q] = (PT)(vc[q] + rv[q]);
        }
        if constexpr (!STREAM) {
            // collision only: velocities go back to their slots
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                if (!valid[k]) continue;
                store_vel<DIM, PT>(A.out, base + tid + k * NT, px[k], pv[k]);
            }
            if (tid == 0 && wstat[1]) atomicAdd(&A.stats->misplaced, (unsigned long long)wstat[1]);
            return;
        }
    }

    if constexpr (STREAM) {
        if constexpr (ID_LATE) {
#pragma unroll
            for (int k = 0; k < PPT; ++k)
                if (valid[k]) pid[k] = load_id<DIM, PT>(A.in, base, (uint32_t)(tid + k * NT));
        }
        const uint32_t ts = (uint32_t)t_now;
        const uint32_t ss = (uint32_t)A.str_s;
        cst<double>* shs = shtab + ((t_now & 1) * d.S + ss) * 3;
        const PT sh[3] = {(PT)shs[0], (PT)shs[1], (PT)shs[2]};
        // sample windows (node sums for the feedback, fine rows for profiles)
        const int nslab_y = d.yhi - d.ylo;
        // non-negative quotients by r (a shift when r is a power of two)
        auto divr = [&](int v) { return d.lr >= 0 ? (v >> d.lr) : v / d.r; };
        const int wnx = divr(d.Tx + d.r - 1) + 2, wny = divr(d.Ty + d.r - 1) + 2;
        const int wnz = (DIM == 3) ? divr(d.Tz + d.r - 1) + 2 : 1;
        const int wx0 = divr(tx << d.lTx) - 1, wy0 = divr(ty << d.lTy) - 1;
        const int wz0 = (DIM == 3) ? divr(tz << d.lTz) - 1 : 0;
        const bool win_ok = wnx * wny * wnz <= MAX_WIN;
        const int wj0 = (ty << d.lTy) - 2, wnj = d.Ty + 4;
        const bool wj_ok = wnj <= MAX_WJ;
        const int copy = (int)(lt % (uint32_t)NCOPY);
        // the collision's barriers cover the tables written at the start
        if constexpr (!COLL) __syncthreads();

        const double ylo_d = (double)d.ylo, yhi_d = (double)d.yhi;
        // the slab faces are integers, exact in either precision, so the
        // face tests compare in the particle precision
        const PT ylo_p = (PT)d.ylo, yhi_p = (PT)d.yhi;
        const int bw = d.bot_wall, tw = d.top_wall, ywrap = d.ywrap;
        const int rb_lo = d.buf_lo * d.r, rb_hi = d.R - d.buf_hi * d.r;
        [[maybe_unused]] const float buf_below = d.buf_below, buf_from = d.buf_from;
        auto row_of = [&](PT y) { return clampi((int)floor(((double)y - ylo_d) * (double)d.r), 0, d.R - 1); };
        const long long NF = (long long)d.Cx * d.NB * d.Cz;
        const double* uf = A.ufine + d.ufine_off * DIM;
        [[maybe_unused]] const double* tfl = CE ? A.tfine + d.ufine_off * CE_NT : nullptr;
        [[maybe_unused]] const bool ce_on = CE && d.ce;
        // per-tile constants in the particle precision (read once, not per particle)
        PT dtp, ghp[3], gdp[3];
        if constexpr (sizeof(PT) == 4) {
            dtp = (PT)d.dtf;
            for (int q = 0; q < 3; ++q) { ghp[q] = (PT)d.ghf[q]; gdp[q] = (PT)d.gdtf[q]; }
        } else {
            dtp = (PT)d.dt;
            for (int q = 0; q < 3; ++q) { ghp[q] = (PT)d.gh[q]; gdp[q] = (PT)d.gdt[q]; }
        }
        const PT nxp = (PT)d.nx, nzp = (PT)d.nz, nyp = (PT)d.ny;
        uint32_t dest[PPT];
#pragma unroll
        for (int k = 0; k < PPT; ++k) dest[k] = BAD_SLOT;
        // exchange step: redraw buffer particles about the LB velocity.  (A
        // version that first listed each wave's buffer particles densely in
        // LDS, so that mixed waves ran the normals once per 64 of them, was
        // measured: 1 % faster on the thin film, 2 % slower on the 3D channel.)
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            if (!valid[k]) continue;
            int J0 = 0;
            bool in_buf;
            if constexpr (sizeof(PT) == 4) {
                // the row's rule by comparisons alone (buffer_bounds)
                in_buf = px[k][1] < buf_below || px[k][1] >= buf_from;
            } else {
                J0 = row_of(px[k][1]);
                in_buf = J0 < rb_lo || J0 >= rb_hi;
            }
            if (in_buf) {
                if constexpr (sizeof(PT) == 4) J0 = row_of(px[k][1]);
                const int I = clampi((int)floor((double)px[k][0] * (double)d.r), 0, d.Cx - 1);
                const int K = (DIM == 3) ? clampi((int)floor((double)px[k][2] * (double)d.r), 0, d.Cz - 1) : 0;
                auto fine = [&]() {
                    const int Jb = (J0 < rb_lo) ? J0 : J0 - (d.R - d.NB);
                    return ((long long)K * d.NB + Jb) * d.Cx + I;
                };
                double z[3], ulv[3];
                if (sizeof(PT) == 4 && !(CE && ce_on)) {
                    // binary32 particles draw binary32 normals (one Philox
                    // block); the Chapman-Enskog draws stay binary64
                    float zf[3];
                    rng_normals32<DIM>(kfresh(), pid[k], ts, ss, P_REINJ, zf);
#pragma unroll
                    for (int q = 0; q < 3; ++q) z[q] = (double)zf[q];
                } else {
                    reinject_normals<DIM>(kfresh(), pid[k], ts, ss, z);
                    if constexpr (CE) {
                        if (ce_on) ce_redraw<DIM>(kfresh(), pid[k], ts, ss, tfl, NF, fine(), z);
                    }
                }
#pragma unroll
                for (int q = 0; q < DIM; ++q) ulv[q] = 0.0;
                {
                    // the LB velocity from the tile's LDS window, or from
                    // global memory for a particle outside it (misplaced, or
                    // a window too large for the LDS)
                    const int uwx = d.Tx + 1, uwy = d.Ty + 1, uwz = (DIM == 3) ? d.Tz + 1 : 1;
                    const int uJ0 = (ty << d.lTy) - 1;
                    const bool uc_ok = ((uJ0 < rb_lo) || (uJ0 + uwy - 1 >= rb_hi)) && uwx * uwy * uwz <= MAX_UFC;
                    int ax = I - ((tx << d.lTx) - 1);
                    if (ax < 0) ax += d.Cx;
                    const int ay = J0 - uJ0;
                    int az = 0;
                    if (DIM == 3) { az = K - ((tz << d.lTz) - 1); if (az < 0) az += d.Cz; }
                    if (uc_ok && ax < uwx && ay >= 0 && ay < uwy && az < uwz) {
                        const int ci = ax + uwx * (ay + uwy * az);
#pragma unroll
                        for (int q = 0; q < DIM; ++q) ulv[q] = ucache[q * MAX_UFC + ci];
                    } else {
                        const long long fc = fine();
#pragma unroll
                        for (int q = 0; q < DIM; ++q) ulv[q] = uf[q * NF + fc];
                    }
                }
#pragma unroll
                for (int q = 0; q < DIM; ++q) pv[k][q] = (PT)(ulv[q] + d.sd * z[q]);
            }
        }

        // streaming, Eq. 3, with the body force as constant acceleration
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            if (!valid[k]) continue;
            PT r0[3] = {px[k][0], px[k][1], px[k][2]}, v0[3] = {pv[k][0], pv[k][1], pv[k][2]};
            PT r1[3] = {r0[0], r0[1], r0[2]}, v1[3] = {v0[0], v0[1], v0[2]};
#pragma unroll
            for (int q = 0; q < DIM; ++q) {
                const PT vh = v0[q] + ghp[q];
                r1[q] = fma_t<PT>(vh, dtp, r0[q]);
                v1[q] = v0[q] + gdp[q];
            }
            // A particle that left the domain by more than one period in this
            // step, or whose position or velocity is not finite, is an invalid
            // state (a diverged LB field hands out such velocities): it is
            // parked at the slab's lower corner at rest, so that every cell,
            // tile and slot index below stays in range, and counted (the next
            // synchronising call reports E_STATE).  A velocity that is not
            // finite takes the free flight out of range with it; only the
            // boundary conditions, which put a particle back on the face,
            // look at the velocity itself.
            bool bad = false;
            const bool in_y = r1[1] >= ylo_p && r1[1] < yhi_p;
            if (!ywrap && !in_y) {
                const bool below = r1[1] < ylo_p;
                const int wall = below ? bw : tw;
                const double Yw = below ? ylo_d : yhi_d;
                double q1[3] = {(double)r1[0], (double)r1[1], (double)r1[2]};
                double w1[3] = {(double)v1[0], (double)v1[1], (double)v1[2]};
                if (wall) {
                    const double tcx = (Yw - (double)r0[1]) / (double)v0[1];
                    const double tr = d.dt - tcx;
#pragma unroll
                    for (int q = 0; q < DIM; ++q) {
                        double rc = (double)r0[q] + ((double)v0[q] + 0.5 * d.g[q] * tcx) * tcx;
                        const double vc = (double)v0[q] + d.g[q] * tcx;
                        if (q == 1) rc = Yw;
                        const double vr = -vc;
                        q1[q] = rc + (vr + 0.5 * d.g[q] * tr) * tr;
                        w1[q] = vr + d.g[q] * tr;
                    }
                } else if (bw || tw) {
                    q1[1] = 2.0 * Yw - q1[1];
                    w1[1] = -w1[1];
                } else {
                    q1[1] = (double)wrap_periodic<PT>(r1[1], (PT)d.ylo, (PT)(d.yhi - d.ylo));
                }
#pragma unroll
                for (int q = 0; q < DIM; ++q) { r1[q] = (PT)q1[q]; v1[q] = (PT)w1[q]; }
                if (r1[1] < ylo_p) r1[1] = ylo_p;
                if (r1[1] >= yhi_p) r1[1] = prev_below<PT>(yhi_p, ylo_p);
                bad = !(r1[1] >= ylo_p && r1[1] < yhi_p);
#pragma unroll
                for (int q = 0; q < DIM; ++q) bad |= !isfinite(v1[q]);
            } else if (ywrap) {
                r1[1] = wrap_periodic<PT>(r1[1], (PT)0, nyp);
                bad = !(r1[1] >= (PT)0 && r1[1] < nyp);
            }
            // periodic axes: only the tiles at the box's faces have work here
            bool in_xz = r1[0] >= (PT)0 && r1[0] < nxp;
            if constexpr (DIM == 3) in_xz &= r1[2] >= (PT)0 && r1[2] < nzp;
            if (!in_xz) {
                r1[0] = wrap_periodic<PT>(r1[0], (PT)0, nxp);
                bad |= !(r1[0] >= (PT)0 && r1[0] < nxp);
                if constexpr (DIM == 3) {
                    r1[2] = wrap_periodic<PT>(r1[2], (PT)0, nzp);
                    bad |= !(r1[2] >= (PT)0 && r1[2] < nzp);
                }
            }
            if (bad) {
#pragma unroll
                for (int q = 0; q < 3; ++q) v1[q] = (PT)0;
                r1[0] = (PT)0;
                r1[1] = ywrap ? (PT)0 : ylo_p;
                r1[2] = (PT)0;
                atomicAdd(&wstat[3], 1u);
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) { px[k][q] = r1[q]; pv[k][q] = v1[q]; }
        }

        // samples right after streaming (last MPCD step of an LB step); the
        // loops over a thread's particles are split by task so that fewer
        // per-tile constants are live at once
        if (A.do_fb | A.do_prof) {
            // the windows take the place of the collision arrays and the
            // LB velocities
            __syncthreads();
            if (A.do_fb && win_ok)
                for (int i = tid; i < wnx * wny * wnz * NREP * 4; i += NT) wacc[i] = 0.0;
            if (A.do_prof && wj_ok)
                for (int i = tid; i < wnj * WSLOTS * 4; i += NT) wprof[i] = 0.0;
            __syncthreads();
            const int wrep = 4 * (lane & (NREP - 1));
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                if (!valid[k]) continue;
                const int J = clampi((int)floor(((double)px[k][1] - ylo_d) * (double)d.r), 0, d.R - 1);
                double vals[4] = {1.0, (double)pv[k][0], (double)pv[k][1], DIM == 3 ? (double)pv[k][2] : 0.0};
                // the feedback projects the interior slab nodes only: buffer
                // rows are not sampled for it (the profile takes every row)
                if (A.do_fb && J >= rb_lo && J < rb_hi) {
                    const int ixn = clampi((int)floor((double)px[k][0]), 0, d.nx - 1);
                    const int iyn = d.lr >= 0 ? (J >> d.lr) : J / d.r;
                    const int izn = (DIM == 3) ? clampi((int)floor((double)px[k][2]), 0, d.nz - 1) : 0;
                    int ax = ixn - wx0; if (ax < 0) ax += d.nx; else if (ax >= d.nx) ax -= d.nx;
                    const int ay = iyn - wy0;
                    int az = izn - wz0;
                    if (DIM == 3) { if (az < 0) az += d.nz; else if (az >= d.nz) az -= d.nz; }
                    if (win_ok && ax < wnx && ay >= 0 && ay < wny && az < wnz) {
                        double* wb = wacc + 4 * NREP * (ax + wnx * (ay + wny * az)) + wrep;
#pragma unroll
                        for (int q = 0; q < DIM + 1; ++q) sum_lds<DET>(&wb[q], vals[q]);
                    } else {
                        const long long sidx = ((long long)izn * nslab_y + iyn) * d.nx + ixn;
                        double* gb = A.acc + (d.acc_off + sidx) * 4;
#pragma unroll
                        for (int q = 0; q < DIM + 1; ++q) sum_gl<DET>(&gb[q], vals[q]);
                        atomicAdd(&wstat[2], 1u);
                    }
                }
                if (A.do_prof) {
                    int aj = J - wj0;
                    // a particle re-wrapped across the slab samples a row next
                    // to the tile modulo the slab's rows
                    if (aj < 0) aj += d.R; else if (aj >= wnj) aj -= d.R;
                    if (wj_ok && aj >= 0 && aj < wnj) {
#pragma unroll
                        for (int q = 0; q < DIM + 1; ++q)
                            sum_lds<DET>(&wprof[(q * wnj + aj) * WSLOTS + (lane & (WSLOTS - 1))], vals[q]);
                    } else {
                        double* gb = A.prof + (d.prof_off + (long long)copy * d.R + J) * 4;
#pragma unroll
                        for (int q = 0; q < DIM + 1; ++q) sum_gl<DET>(&gb[q], vals[q]);
                        atomicAdd(&wstat[2], 1u);
                    }
                }
            }
        }

        // binning into the shifted grid of this MPCD step (24-bit products, a
        // quarter of the cost of 32-bit ones, unless the channel has 2^24
        // tiles or more in a plane or along z)
        const bool mul24 = (nxy | (uint32_t)d.ntz) < (1u << 24);
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            if (!valid[k]) continue;
            int ix = bin_coord<PT>(px[k][0], (PT)0, sh[0], rr);
            if (ix >= d.Cx) ix -= d.Cx;
            const int iy = bin_row<PT>(d, px[k][1], sh[1], rr);
            int iz = 0;
            if constexpr (DIM == 3) {
                iz = bin_coord<PT>(px[k][2], (PT)0, sh[2], rr);
                if (iz >= d.Cz) iz -= d.Cz;
            }
            const int ntx = ix >> d.lTx, nty = iy >> d.lTy, ntz = iz >> d.lTz;
            dest[k] = (uint32_t)ntx + (mul24 ? __umul24(d.ntx, nty) + __umul24(nxy, ntz) : (uint32_t)d.ntx * (uint32_t)nty + nxy * (uint32_t)ntz);
            if (dest[k] >= (uint32_t)d.ntiles) {
                // unreachable for positions inside the domain (checked above);
                // kept so that no slot index can leave the channel's tiles
                dest[k] = lt;
                atomicAdd(&wstat[3], 1u);
            }
            // moves beyond the neighbour tiles (they are grouped like any other
            // destination; the count bounds the sample-window misses, so it is
            // kept in the MPCD steps that sample, and skipped in the others)
            if (A.do_fb | A.do_prof) {
                int dx = ntx - tx, dy = nty - ty, dz = ntz - tz;
                if (d.ntx > 2) { if (dx == d.ntx - 1) dx = -1; else if (dx == 1 - d.ntx) dx = 1; }
                if (DIM == 3 && d.ntz > 2) { if (dz == d.ntz - 1) dz = -1; else if (dz == 1 - d.ntz) dz = 1; }
                if (dx < -1 || dx > 1 || dy < -1 || dy > 1 || dz < -1 || dz > 1) atomicAdd(&wstat[0], 1u);
            }
        }

        // ---- phase 3a: group each wave's particles by destination tile.
        // Lanes with equal destinations get consecutive ranks; the group's
        // first lane claims a row of the LDS destination table and the
        // group's offset in it, and hands both back with one permute.
        uint32_t pk[PPT];  // bit 31: direct slot; else (table row + 1) << 24 | rank
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const uint32_t key = dest[k];
            // Waterfall over the lanes still waiting: the lowest of them
            // names the next group, whose lanes (the active lanes with its
            // key) take their ranks from the active mask and leave the loop.
            // Two or three destinations hold most of a wave; once no more
            // than SINGLES lanes wait, spread over several others, each is a
            // group of its own, which costs one pass through the claim below
            // (made anyway) instead of one round each (film 5.64 -> 5.38 ms,
            // MPCD-AT on the 3D channel 3.28 -> 3.08; 24 measures the same).
            int my_leader = 0;
            uint32_t my_rank = 0, lead_cnt = 0;
            if (key != BAD_SLOT) {
                for (;;) {
                    const uint32_t kv = (uint32_t)__builtin_amdgcn_readfirstlane((int)key);
                    if (key == kv) {
                        const unsigned long long m = __ballot(1);
                        my_leader = __ffsll(m) - 1;
                        my_rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                        lead_cnt = (uint32_t)__popcll(m);
                        break;
                    }
                    if (__popcll(__ballot(1)) <= SINGLES) {
                        my_leader = lane;
                        lead_cnt = 1u;
                        break;
                    }
                }
            }
            const bool is_lead = key != BAD_SLOT && my_rank == 0u;
            uint32_t packed = 0u;
            if (is_lead) {
                int h = -1;
                uint32_t hh = (key * 2654435761u) >> (32 - NHASH_BITS);
#pragma unroll 1
                for (int probe = 0; probe < NHASH; ++probe) {
                    const uint32_t old = atomicCAS(&hkey[hh], BAD_SLOT, key);
                    if (old == BAD_SLOT || old == key) { h = (int)hh; break; }
                    hh = (hh + 1) & (NHASH - 1);
                }
                if (h >= 0) {
                    packed = ((uint32_t)(h + 1) << 24) | atomicAdd(&hcnt[h], lead_cnt);
                } else {
                    // more destinations than table rows: reserve directly
                    const uint32_t ob = atomicAdd(&A.fill_out[d.tile_off + key], lead_cnt);
                    packed = ob < 0xFFFFFFu ? ob : 0xFFFFFFu;
                }
            }
            packed = (uint32_t)__shfl((int)packed, my_leader);
            pk[k] = BAD_SLOT;
            if (key != BAD_SLOT) {
                const uint32_t row = packed >> 24;
                const uint32_t r_ = (packed & 0xFFFFFFu) + my_rank;
                if (row) {
                    pk[k] = (row << 24) | r_;
                } else {
                    pk[k] = r_ < (uint32_t)cap ? (0x80000000u | (uint32_t)(key * cap + r_)) : DROP_SLOT;
                }
            }
        }
        __syncthreads();
        // ---- phase 3b: one global atomic per destination reserves a run of
        // slots; each store writes the lanes of a group to consecutive slots
        if (tid < NHASH) {
            const uint32_t c = hcnt[tid], key = hkey[tid];
            const uint32_t g0 = c > 0u ? atomicAdd(&A.fill_out[d.tile_off + key], c) : 0u;
            gbase[tid] = g0;
            hkey[tid] = key * (uint32_t)cap + g0;  // from here on the run's first slot
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const uint32_t e = pk[k];
            if (e == BAD_SLOT) continue;
            uint32_t g = 0u;  // slot within the channel
            bool ok = e != DROP_SLOT;
            if (ok && (e & 0x80000000u)) {
                g = e & 0x7FFFFFFFu;
            } else if (ok) {
                const int row = (int)(e >> 24) - 1;
                const uint32_t r_ = e & 0xFFFFFFu;
                ok = gbase[row] + r_ < (uint32_t)cap;
                g = hkey[row] + r_;
            }
            if (!ok) {
                atomicAdd(&A.stats->dropped, 1ull);
                continue;
            }
            store_part<DIM, PT>(A.out, d.slot_off, g, px[k], pv[k], pid[k]);
        }
        // ---- sample windows to global memory
        if (A.do_fb && win_ok) {
            for (int i = tid; i < wnx * wny * wnz; i += NT) {
                double sum[4] = {0.0, 0.0, 0.0, 0.0};
                [[maybe_unused]] unsigned long long isum[4] = {0ull, 0ull, 0ull, 0ull};
#pragma unroll
                for (int r = 0; r < NREP; ++r)
#pragma unroll
                    for (int q = 0; q < DIM + 1; ++q) {
                        if constexpr (DET) isum[q] += ((const unsigned long long*)wacc)[4 * (NREP * i + r) + q];
                        else sum[q] += wacc[4 * (NREP * i + r) + q];
                    }
                if (DET ? isum[0] == 0ull : sum[0] == 0.0) continue;
                const int ax = i % wnx, ay = (i / wnx) % wny, az = i / (wnx * wny);
                int ixn = wx0 + ax; if (ixn < 0) ixn += d.nx; else if (ixn >= d.nx) ixn -= d.nx;
                const int iyn = wy0 + ay;
                int izn = wz0 + az;
                if (DIM == 3) { if (izn < 0) izn += d.nz; else if (izn >= d.nz) izn -= d.nz; }
                if (iyn < 0 || iyn >= nslab_y) continue;  // samples are clamped to the slab
                const long long sidx = ((long long)izn * nslab_y + iyn) * d.nx + ixn;
                double* gb = A.acc + (d.acc_off + sidx) * 4;
#pragma unroll
                for (int q = 0; q < DIM + 1; ++q) {
                    if constexpr (DET) atomicAdd((unsigned long long*)&gb[q], isum[q]);
                    else gl_add(&gb[q], sum[q]);
                }
            }
        }
        if (A.do_prof && wj_ok) {
            // one thread per row and component; the four components of a row
            // leave in one instruction
            for (int i = tid; i < wnj * 4; i += NT) {
                const int q = i & 3, row = i >> 2;
                if (DIM == 2 && q == 3) continue;
                const double* w = wprof + (q * wnj + row) * WSLOTS;
                double sum = 0.0;
                [[maybe_unused]] unsigned long long isum = 0ull;
#pragma unroll
                for (int j = 0; j < WSLOTS; ++j) {
                    if constexpr (DET) isum += ((const unsigned long long*)w)[j];
                    else sum += w[j];
                }
                if (DET ? isum == 0ull : sum == 0.0) continue;
                int J = wj0 + row;
                if (J < 0) J += d.R; else if (J >= d.R) J -= d.R;
                double* gb = A.prof + (d.prof_off + (long long)copy * d.R + J) * 4 + q;
                if constexpr (DET) atomicAdd((unsigned long long*)gb, isum);
                else gl_add(gb, sum);
            }
        }
        if (tid == 0) {
            A.fill_in[T] = 0u;
            if (wstat[0]) atomicAdd(&A.stats->far_moves, (unsigned long long)wstat[0]);
            if (wstat[1]) atomicAdd(&A.stats->misplaced, (unsigned long long)wstat[1]);
            if (wstat[2]) atomicAdd(&A.stats->window_misses, (unsigned long long)wstat[2]);
            if (wstat[3]) atomicAdd(&A.stats->bad_state, (unsigned long long)wstat[3]);
        }
    }
}

// One workgroup per tile.
template <int DIM, typename PT, int NT, int PPT, int MODE>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(particle_waves<DIM, PT, MODE, PPT>())))
k_particles(PArgs<PT> A) {
    extern __shared__ __align__(16) unsigned char smem[];
    // Workgroups are dealt to the eight XCDs in turn.  In the XCD-blocked
    // order the workgroups of one XCD take one contiguous range of tiles, so
    // the tiles that trade particles are mostly served by one L2, where the
    // partial lines of their destination runs merge.
    long long T = blockIdx.x;
    if (A.xcd_per > 0) {
        T = (long long)(blockIdx.x % 8) * A.xcd_per + blockIdx.x / 8;
        if (T >= A.ntiles) return;
    }
    particle_tile<DIM, PT, NT, PPT, MODE>(A, T, smem);
}

// The overflow pass (ovf_mode 2): the workgroups of a small grid take the
// listed tiles in turn; the last workgroup to finish clears the list.  A
// kernel of its own, so that the loop does not weigh on the register
// allocation of the one-tile kernel.
template <int DIM, typename PT, int NT, int PPT, int MODE>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(particle_waves<DIM, PT, MODE, PPT>())))
k_particles_ovf(PArgs<PT> A) {
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t cnt = A.ovf[0];
    for (uint32_t i = blockIdx.x; i < cnt; i += gridDim.x) {
        particle_tile<DIM, PT, NT, PPT, MODE>(A, (long long)A.ovf[2 + i], smem);
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        __threadfence();
        if (atomicAdd(&A.ovf[1], 1u) == gridDim.x - 1) {
            A.ovf[0] = 0u;
            A.ovf[1] = 0u;
        }
    }
}

// ---------------------------------------------------------------------------
// launch templates; `Modes::run<DIM, PT, NT, PPT>` picks the instantiation
// of the mode (each translation unit instantiates its own set)
// ---------------------------------------------------------------------------
template <int DIM, typename PT, int NT, int PPT, int MODE, int OVF = 0>
static hipError_t launch_p4(const ParticleLaunch& L, hipStream_t s) {
    if constexpr (NT == 512 && (MODE & 1) != 0 && (MODE & MODE_REPS) == 0) {
        if (L.reps) return launch_p4<DIM, PT, NT, PPT, MODE | MODE_REPS, OVF>(L, s);
    }
    PArgs<PT> a;
    a.D = L.D;
    a.in = L.in; a.out = L.out;
    a.fill_in = L.fill_in; a.fill_out = L.fill_out; a.tile_inst = L.tile_inst;
    a.ufine = L.ufine; a.tfine = L.tfine; a.acc = L.acc; a.prof = L.prof; a.stats = L.stats; a.clock = L.clock;
    a.shifts = L.shifts;
    a.coll_dt = L.coll_dt; a.coll_s = L.coll_s; a.str_s = L.str_s;
    a.do_fb = L.do_fb; a.do_prof = L.do_prof; a.diag_inst = L.diag_inst; a.cell_vcm = L.cell_vcm;
    a.ntiles = L.tiles;
    a.xcd_per = L.xcd_blocked ? (L.tiles + 7) / 8 : 0;
    a.ovf = L.ovf;
    a.ovf_mode = OVF;
    // the sample windows only where samples are taken: the other launches fit
    // more workgroups per CU
    const size_t lds = LDS_HDR + ((L.do_fb | L.do_prof) ? LDS_UNI : LDS_COLL);
    if constexpr (OVF == 2) {
        const long long grid = L.tiles < OVF_GRID ? L.tiles : OVF_GRID;
        hipLaunchKernelGGL((k_particles_ovf<DIM, PT, NT, PPT, MODE>), dim3((unsigned)grid), dim3(NT), lds, s,
                           a);
        return hipGetLastError();
    } else {
        const long long grid = L.xcd_blocked ? 8 * a.xcd_per : L.tiles;
        auto kern = k_particles<DIM, PT, NT, PPT, MODE>;
        hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(NT), lds, s, a);
        return hipGetLastError();
    }
}

// Workgroup shape: threads x particles per thread must cover the largest
// tile capacity.  256 threads unless the caller asks for 512.
template <class Modes, int DIM, typename PT>
static hipError_t launch_p2(const ParticleLaunch& L, hipStream_t s) {
    if (L.wg_threads == 128) {
        if (L.cap_max <= 4 * 128) return Modes::template run<DIM, PT, 128, 4>(L, s);
        if (L.cap_max <= 8 * 128) return Modes::template run<DIM, PT, 128, 8>(L, s);
        return hipErrorInvalidValue;
    }
    if (L.wg_threads == 512) {
        if (L.cap_max <= 2 * 512) return Modes::template run<DIM, PT, 512, 2>(L, s);
        if (L.cap_max <= 4 * 512) return Modes::template run<DIM, PT, 512, 4>(L, s);
        return hipErrorInvalidValue;
    }
    if (L.cap_max <= 2 * 256) return Modes::template run<DIM, PT, 256, 2>(L, s);
    if (L.cap_max <= 4 * 256) return Modes::template run<DIM, PT, 256, 4>(L, s);
    if (L.cap_max <= 8 * 256) return Modes::template run<DIM, PT, 256, 8>(L, s);
    return hipErrorInvalidValue;
}

// Tiles of 1025-2048 slots at 256 threads: six slots per thread instead of
// eight leave the kernel fewer vector registers and one more wave per SIMD
// (binary32, SRD: 89 VGPRs and five waves instead of 113 and four; MPCD-AT: 123
// and four instead of 151 and three; binary64, SRD: 128 and four instead of
// 147 and three).
// A tile holding
// more than 1536 particles is skipped and listed by that launch and
// processed by a second launch over the list (512 threads, four slots per
// thread: a listed tile waits on one tile's latency, which more threads
// shorten).  It is rare: the
// tile's expected occupancy plus two standard deviations of its Poisson
// count must stay within 1536 for this form to be taken.
inline bool split_applies(const ParticleLaunch& L) {
    if (L.ovf == nullptr) return false;
    if ((L.wg_threads != 0 && L.wg_threads != 256) || L.cap_max <= 4 * 256 || L.cap_max > 8 * 256) return false;
    const double e = (double)L.exp_max;
    return e + 2.0 * std::sqrt(e) <= 6.0 * 256;
}

template <class Modes, int DIM, typename PT>
static hipError_t launch_split_dim(const ParticleLaunch& L, hipStream_t s) {
    hipError_t e = Modes::template run<DIM, PT, 256, 6, 1>(L, s);
    if (e == hipSuccess) e = Modes::template run<DIM, PT, 512, 4, 2>(L, s);
    return e;
}

template <class Modes>
static hipError_t launch_modes(const ParticleLaunch& L, hipStream_t s) {
    if (L.tiles <= 0) return hipSuccess;
    if (split_applies(L)) {
        if (L.part_fp == 64)
            return L.dim == 2 ? launch_split_dim<Modes, 2, double>(L, s) : launch_split_dim<Modes, 3, double>(L, s);
        return L.dim == 2 ? launch_split_dim<Modes, 2, float>(L, s) : launch_split_dim<Modes, 3, float>(L, s);
    }
    if (L.dim == 2 && L.part_fp == 64) return launch_p2<Modes, 2, double>(L, s);
    if (L.dim == 2) return launch_p2<Modes, 2, float>(L, s);
    if (L.part_fp == 64) return launch_p2<Modes, 3, double>(L, s);
    return launch_p2<Modes, 3, float>(L, s);
}

// The Chapman-Enskog modes (bit 8), instantiated in kernels_mpcd_ce.hip.
hipError_t launch_particles_ce(const ParticleLaunch& L, hipStream_t s);
// The deterministic modes (bit 16), instantiated in kernels_mpcd_det.hip.
hipError_t launch_particles_det(const ParticleLaunch& L, hipStream_t s);

}  // namespace lbmpcd

// pstore.hpp -- layout of a particle buffer and access to its records.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lbmpcd {

// A particle buffer: per slot, N16 arrays of 16-byte vectors `cs` bytes apart,
// then one array of LAST bytes a slot.
//   binary32 3D: (x, y, z, id); (vx, vy, vz)
//   binary32 2D: (x, y, vx, vy); id
//   binary64 2D: (x, y); (vx, vy); id
//   binary64 3D: (x, y); (z, vx); (vy, vz); id
// A wave moves a particle in two to four vector accesses.  With one array per
// component it took five or seven: the particle kernel's stores, whose lanes
// go to some eight runs of consecutive slots, then touch that many cache lines
// per component.
constexpr size_t PART_ALIGN = 256;
constexpr int part_n16(int dim, int part_fp) { return part_fp == 64 ? dim : 1; }
constexpr int part_last(int dim, int part_fp) { return part_fp == 32 && dim == 3 ? 12 : 4; }

template <int DIM, typename PT>
struct PStore {
    static constexpr bool F32 = sizeof(PT) == 4;
    static constexpr int N16 = part_n16(DIM, F32 ? 32 : 64), LAST = part_last(DIM, F32 ? 32 : 64);
    static constexpr bool ID_APART = LAST == 4;  // the id is the last array
    unsigned char* b;
    long long cs;
    // component c of x, y, (z), vx, vy, (vz) of slot g
    __device__ __forceinline__ PT* at(int c, long long g) const {
        if constexpr (!F32) return (PT*)(b + (c >> 1) * cs + g * 16) + (c & 1);
        else if constexpr (DIM == 2) return (PT*)(b + g * 16) + c;
        else return c < 3 ? (PT*)(b + g * 16) + c : (PT*)(b + cs + g * 12) + (c - 3);
    }
    __device__ __forceinline__ PT* pos(int q, long long g) const { return at(q, g); }
    __device__ __forceinline__ PT* vel(int q, long long g) const { return at(DIM + q, g); }
    __device__ __forceinline__ uint32_t* id(long long g) const {
        if constexpr (F32 && DIM == 3) return (uint32_t*)(b + g * 16) + 3;
        else return (uint32_t*)(b + N16 * cs + g * 4);
    }
};

// One particle buffer, type-erased (layout: PStore).
struct PartBuf {
    unsigned char* b;
    long long cs;
};

template <int DIM, typename PT>
inline PStore<DIM, PT> typed(const PartBuf& p) { return PStore<DIM, PT>{p.b, p.cs}; }

// One particle's record from slot base + s (base uniform) of a buffer.
// Binary32 records are read with buffer instructions: one resource per array
// (its uniform 64-bit base in scalar registers) and a 32-bit byte offset per
// lane.  Stores go to any tile of the channel, whose arrays may exceed 4 GiB,
// so they take 64-bit addresses.
typedef unsigned int u32x3 __attribute__((ext_vector_type(3)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
struct __attribute__((packed, aligned(4))) F3 { float x, y, z; };

__device__ __forceinline__ __amdgpu_buffer_rsrc_t arr_rsrc(const unsigned char* p) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, -1, 0x00020000);
}
__device__ __forceinline__ float as_f(uint32_t u) { return __builtin_bit_cast(float, u); }

template <int DIM, typename PT>
__device__ __forceinline__ void load_part(const PartBuf& B, long long base, uint32_t s, PT* px, PT* pv, uint32_t& id) {
    using S = PStore<DIM, PT>;
    [[maybe_unused]] const unsigned char* last = B.b + S::N16 * B.cs + base * S::LAST;
    if constexpr (DIM == 2) px[2] = pv[2] = (PT)0;
    if constexpr (S::F32) {
        const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(arr_rsrc(B.b + base * 16), (int)(s * 16u), 0, 0);
        px[0] = as_f(a.x); px[1] = as_f(a.y);
        if constexpr (DIM == 3) {
            const u32x3 v = __builtin_amdgcn_raw_buffer_load_b96(arr_rsrc(last), (int)(s * 12u), 0, 0);
            px[2] = as_f(a.z); id = a.w;
            pv[0] = as_f(v.x); pv[1] = as_f(v.y); pv[2] = as_f(v.z);
        } else {
            pv[0] = as_f(a.z); pv[1] = as_f(a.w);
        }
    } else {
        const double2 a = *(const double2*)(B.b + base * 16 + s * 16u);
        const double2 b = *(const double2*)(B.b + B.cs + base * 16 + s * 16u);
        px[0] = a.x; px[1] = a.y;
        if constexpr (DIM == 3) {
            const double2 c = *(const double2*)(B.b + 2 * B.cs + base * 16 + s * 16u);
            px[2] = b.x; pv[0] = b.y; pv[1] = c.x; pv[2] = c.y;
        } else {
            pv[0] = b.x; pv[1] = b.y;
        }
    }
}
// The id of a record that holds it in an array of its own (ID_APART).
template <int DIM, typename PT>
__device__ __forceinline__ uint32_t load_id(const PartBuf& B, long long base, uint32_t s) {
    using S = PStore<DIM, PT>;
    return __builtin_amdgcn_raw_buffer_load_b32(arr_rsrc(B.b + S::N16 * B.cs + base * 4), (int)(s * 4u), 0, 0);
}

// Writes the record of slot g of the channel that starts at slot `off`.
template <int DIM, typename PT>
__device__ __forceinline__ void store_part(const PartBuf& B, long long off, uint32_t g, const PT* px, const PT* pv,
                                           uint32_t id) {
    using S = PStore<DIM, PT>;
    unsigned char* last = B.b + S::N16 * B.cs + off * S::LAST;
    unsigned char* a = B.b + off * 16 + ((uint64_t)g << 4);
    if constexpr (S::F32) {
        if constexpr (DIM == 3) {
            *(u32x4*)a = u32x4{__float_as_uint(px[0]), __float_as_uint(px[1]), __float_as_uint(px[2]), id};
            *(F3*)(last + (uint64_t)g * 12u) = F3{pv[0], pv[1], pv[2]};
        } else {
            *(u32x4*)a = u32x4{__float_as_uint(px[0]), __float_as_uint(px[1]), __float_as_uint(pv[0]), __float_as_uint(pv[1])};
            *(uint32_t*)(last + ((uint64_t)g << 2)) = id;
        }
    } else {
        *(double2*)a = double2{px[0], px[1]};
        if constexpr (DIM == 3) {
            *(double2*)(a + B.cs) = double2{px[2], pv[0]};
            *(double2*)(a + 2 * B.cs) = double2{pv[1], pv[2]};
        } else {
            *(double2*)(a + B.cs) = double2{pv[0], pv[1]};
        }
        *(uint32_t*)(last + ((uint64_t)g << 2)) = id;
    }
}

// Writes the velocity of slot g, whose position px it leaves as it is.  Where a
// vector holds both, it is written whole: of every second half alone, a
// collision without streaming took 423 us for 21M binary64 particles in 3D
// instead of 352, and 46.9 instead of 44.2 for 5.2M binary32 in 2D.
template <int DIM, typename PT>
__device__ __forceinline__ void store_vel(const PartBuf& B, long long g, const PT* px, const PT* pv) {
    using S = PStore<DIM, PT>;
    unsigned char* a = B.b + g * 16;
    if constexpr (S::F32) {
        if constexpr (DIM == 3) *(F3*)(B.b + B.cs + g * 12) = F3{pv[0], pv[1], pv[2]};
        else *(u32x4*)a = u32x4{__float_as_uint(px[0]), __float_as_uint(px[1]), __float_as_uint(pv[0]), __float_as_uint(pv[1])};
    } else if constexpr (DIM == 3) {
        *(double2*)(a + B.cs) = double2{px[2], pv[0]};
        *(double2*)(a + 2 * B.cs) = double2{pv[1], pv[2]};
    } else {
        *(double2*)(a + B.cs) = double2{pv[0], pv[1]};
    }
}

}  // namespace lbmpcd

// lbm_addr.hpp -- how the tile kernels address a copy of the state (or of the
// adjoint): planes through a uniform base, nodes through one byte offset.
#pragma once

#include <type_traits>

#include "lbm_device.hpp"

namespace lbm {

// A copy below 4 GiB (OFF uint32_t) as a buffer resource: an element is
// addressed by a byte offset per lane plus a uniform plane offset, so that one
// offset register serves every plane a node is read from or written to and no
// address is formed on the vector unit.  `bytes`: of the copy; offsets beyond it
// read zero and store nothing.  Larger copies (uint64_t): plain 64-bit
// addresses.
// Stores: ordinary; non-temporal; or through the XCD's L2 to memory (device
// scope), which leaves no dirty lines to flush between launches.
enum StoreKind { ST_PLAIN = 0, ST_NT = 2, ST_THROUGH = 16 };   // the instructions' nt and sc1 bits

// How a two-level launch stores `bytes` of state (both copies): through the L2 while the
// cache holds them, else non-temporally; but rows that end inside a cache line with
// ordinary stores, unless the state is small (small_bytes): written through or
// non-temporally, a line that two tiles share goes out in two parts, and once several
// states, or one of more than 256 MB, spill the last-level cache each part is a
// partial write to memory.  Measured on MI355X, us per level, rows of broken lines,
// through / ordinary: FP32 1050 x 1700 52.1 / 45.2, 937 x 1898 51.7 / 44.4, 1500 x 1000 31.4 /
// 31.6, 1528 x 636 21.8 / 22.5, local gradient 1500 x 1100 52.6 / 45.1, FP64 1030 x 800 44.8 /
// 40.3, 1030 x 709 32.7 / 32.5; three lattices on streams of their own, FP32 969 x 1111
// 30.5 / 26.0, 1000 x 560 14.7 / 13.2, FP64 1100 x 900 50.5 / 44.4.
inline StoreKind step2_store(size_t bytes, bool whole) {
    if (whole ? cached_bytes(bytes) : small_bytes(bytes)) return ST_THROUGH;
    return whole ? ST_NT : ST_PLAIN;
}

template <typename OFF>
struct CopyAddr;

template <>
struct CopyAddr<uint32_t> {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ CopyAddr(const char* base, uint32_t bytes)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, bytes, 0x00020000)) {}
    template <typename T>
    __device__ __forceinline__ T ld(uint32_t off, uint32_t plane) const {
        if constexpr (sizeof(T) == 4)
            return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, plane, 0));
        else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, plane, 0));
    }
    template <StoreKind K, typename T>
    __device__ __forceinline__ void st(uint32_t off, uint32_t plane, T v) const {
        if constexpr (sizeof(T) == 4)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, off, plane, K);
        else {
            typedef unsigned u2 __attribute__((ext_vector_type(2)));
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, off, plane, K);
        }
    }
};

template <>
struct CopyAddr<uint64_t> {
    char* base;
    __device__ __forceinline__ CopyAddr(const char* b, uint64_t) : base(const_cast<char*>(b)) {}
    template <typename T>
    __device__ __forceinline__ T ld(uint64_t off, uint64_t plane) const {
        return *reinterpret_cast<const T*>(base + plane + off);
    }
    template <StoreKind K, typename T>
    __device__ __forceinline__ void st(uint64_t off, uint64_t plane, T v) const {
        if (K == ST_NT) __builtin_nontemporal_store(v, reinterpret_cast<T*>(base + plane + off));
        else *reinterpret_cast<T*>(base + plane + off) = v;
    }
};

// The kernel parameters of a tile body: by value, or (RELOAD) in constant memory,
// from which params_at() reads the fields that the code after it uses anew, which
// keeps them out of scalar registers in between.
template <typename T>
using ParamsPtr = const __attribute__((address_space(4))) KParams<T>*;
template <typename T, bool RELOAD>
using BodyParams = typename std::conditional<RELOAD, ParamsPtr<T>, KParams<T>>::type;

template <typename T>
__device__ __forceinline__ KParams<T> params_at(ParamsPtr<T> p) {
#ifdef __OPTIMIZE__   // unoptimised code keeps p in no scalar register, and reads anew anyway
    asm volatile("" : "+s"(p));
#endif
    return *(const KParams<T>*)p;
}
template <typename T>
__device__ __forceinline__ const KParams<T>& params_at(const KParams<T>& p) {
    return p;
}
// From a kernel's first argument P, or from memory that the launch only reads.
template <bool RELOAD, typename T>
__device__ __forceinline__ BodyParams<T, RELOAD> kernel_params(const KParams<T>& P) {
    if constexpr (RELOAD) return (ParamsPtr<T>)__builtin_amdgcn_kernarg_segment_ptr();
    else return P;
}
template <bool RELOAD, typename T>
__device__ __forceinline__ BodyParams<T, RELOAD> memory_params(const KParams<T>& P) {
    if constexpr (RELOAD) return (ParamsPtr<T>)&P;
    else return P;
}

// Node of region position p on an axis of n nodes; -1 beyond a wall.  Periodic
// axes wrap (any number of times: a lattice may be narrower than the region; by a
// remainder, since a loop of up to a region's height per position cost lattices of a
// few rows 3-8%: 100000 x 3 FP64 32.3 against 30.1 us per level).
__device__ __forceinline__ int axis_node(int p, int n, bool wall) {
    if ((unsigned)p < (unsigned)n) return p;
    if (wall) return -1;
    p += p < 0 ? n : -n;
    if ((unsigned)p < (unsigned)n) return p;
    const int r = p % n;
    return r < 0 ? r + n : r;
}

// The plane from whose base population i is addressed: the lower of i and
// opp(i) = i +- 2, so that the reflected population (plane opp(i), the node's own
// offset) lies at a non-negative offset too.
__host__ __device__ constexpr int pair_plane(int i) { return opp(i) < i ? opp(i) : i; }

// Whether population i of node (x, y) crosses a wall on its way from (DIR -1) or
// to (DIR +1) its neighbour.
template <int DIR, typename T>
__device__ __forceinline__ bool beyond_wall(const KParams<T>& P, int i, int x, int y) {
    const int dx = DIR * cx(i), dy = DIR * cy(i);
    return (dx < 0 ? P.wall_x && x == 0 : (dx > 0 ? P.wall_x && x == P.nx - 1 : false)) ||
           (dy < 0 ? P.wall_y && y == 0 : (dy > 0 ? P.wall_y && y == P.ny - 1 : false));
}

// Byte offsets of the populations that position (px, py) pulls (DIR -1: i comes
// from the node at -c_i) or pushes (DIR +1: i goes to the node at +c_i), from the
// base of plane pair_plane(i); at a wall the node's own opp(i).  off[0]: the node
// itself, (xi, yi); false beyond a wall.  `inner` (uniform): no wrap and no wall
// within one node of any position of the tile's windows.
template <typename T, typename OFF, int DIR>
__device__ __forceinline__ bool neighbour_offsets(const KParams<T>& P, bool inner, int px, int py, OFF (&off)[9],
                                                  int& xi, int& yi) {
    constexpr OFF ES = sizeof(T);
    const OFF nx = (OFF)P.nx, pl2 = 2 * (OFF)P.plane * ES;
    if (inner) {
        xi = px;
        yi = py;
        // with 32-bit offsets nx < 2^24: an inner tile has ny >= 6 and the copy is below 4 GiB
        const OFF k = ((sizeof(OFF) == 4 ? (OFF)__umul24((unsigned)py, (unsigned)nx) : (OFF)py * nx) + (OFF)px) * ES;
        off[0] = k;
#pragma unroll
        for (int i = 1; i < Q; i++)
            off[i] = k + ((pair_plane(i) == i ? OFF(0) : pl2) + (OFF)((long long)DIR * (cy(i) * (long long)P.nx + cx(i))) * ES);
        return true;
    }
    xi = axis_node(px, P.nx, P.wall_x);
    yi = axis_node(py, P.ny, P.wall_y);
    if (xi < 0 || yi < 0) return false;
    OFF col[3], row[3];
    col[1] = (OFF)xi;
    col[0] = xi == 0 ? nx - 1 : (OFF)xi - 1;
    col[2] = xi == P.nx - 1 ? OFF(0) : (OFF)xi + 1;
    row[1] = (OFF)yi * nx;
    row[0] = yi == 0 ? (OFF)(P.ny - 1) * nx : row[1] - nx;
    row[2] = yi == P.ny - 1 ? OFF(0) : row[1] + nx;
    off[0] = (row[1] + col[1]) * ES;
#pragma unroll
    for (int i = 1; i < Q; i++)
        off[i] = (row[1 + DIR * cy(i)] + col[1 + DIR * cx(i)]) * ES + (pair_plane(i) == i ? OFF(0) : pl2);
    if (P.wall_x || P.wall_y)
#pragma unroll
        for (int i = 1; i < Q; i++)
            if (beyond_wall<DIR>(P, i, xi, yi)) off[i] = off[0] + (pair_plane(i) == i ? pl2 : OFF(0));
    return true;
}

}  // namespace lbm

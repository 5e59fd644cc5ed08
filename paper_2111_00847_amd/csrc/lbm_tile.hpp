// lbm_tile.hpp -- the 64 x TY tile of the step kernels: LDS window of phi
// with wall ghosts, stencils from the window, end-of-step signalling.
#pragma once

#include "lbm_device.hpp"

namespace lbm {

constexpr int TX = 64;
constexpr int BY = 4;

// Wall ghosts of the window (Eq. Dwetting): x-walls first, then y-walls
// across the extended rows, which fixes the corners.  Call after the window
// interior and ring are filled and synchronised; ends synchronised.
template <typename T, int TY, int NBY = BY>
__device__ __forceinline__ void wall_ghosts(const KParams<T>& P, bool need_prev, int x0, int y0,
                                            T (*sphi)[TX + 3], T (*sphp)[TX + 3]) {
    constexpr int WX = TX + 2, WY = TY + 2;
    const int tid = threadIdx.y * TX + threadIdx.x;
    if (P.wall_x) {
        const int wxr = P.nx - x0 + 1;  // window column of x = nx
        for (int wy = tid; wy < WY; wy += TX * NBY) {
            // rows beyond a y-wall get their ghosts below; on a periodic y axis
            // the halo rows -1 and ny hold wrapped rows and need x-ghosts too
            const int gy = y0 - 1 + wy;
            if (gy > P.ny || (P.wall_y && (gy < 0 || gy >= P.ny))) continue;
            if (x0 == 0) {
                sphi[wy][0] = wet_ghost(P, 0, sphi[wy][1], sphi[wy][2]);
                if (need_prev) sphp[wy][0] = wet_ghost(P, 0, sphp[wy][1], sphp[wy][2]);
            }
            if (wxr <= WX - 1) {
                sphi[wy][wxr] = wet_ghost(P, 1, sphi[wy][wxr - 1], sphi[wy][wxr - 2]);
                if (need_prev) sphp[wy][wxr] = wet_ghost(P, 1, sphp[wy][wxr - 1], sphp[wy][wxr - 2]);
            }
        }
        __syncthreads();
    }
    if (P.wall_y) {
        const int wyt = P.ny - y0 + 1;  // window row of y = ny
        for (int wx = tid; wx < WX; wx += TX * NBY) {
            int gx = x0 - 1 + wx;
            if (gx > P.nx) continue;
            if (y0 == 0) {
                sphi[0][wx] = wet_ghost(P, 2, sphi[1][wx], sphi[2][wx]);
                if (need_prev) sphp[0][wx] = wet_ghost(P, 2, sphp[1][wx], sphp[2][wx]);
            }
            if (wyt <= WY - 1) {
                sphi[wyt][wx] = wet_ghost(P, 3, sphi[wyt - 1][wx], sphi[wyt - 2][wx]);
                if (need_prev) sphp[wyt][wx] = wet_ghost(P, 3, sphp[wyt - 1][wx], sphp[wyt - 2][wx]);
            }
        }
        __syncthreads();
    }
}

// The same stencils on any 2-D window array, centred at (wx, wy).
template <typename A, typename T>
__device__ __forceinline__ void win_stencil_at(const A& s, int wx, int wy, T& gx, T& gy, T& lap) {
    stencil(s[wy - 1][wx - 1], s[wy - 1][wx], s[wy - 1][wx + 1], s[wy][wx - 1], s[wy][wx], s[wy][wx + 1],
            s[wy + 1][wx - 1], s[wy + 1][wx], s[wy + 1][wx + 1], gx, gy, lap);
}

template <typename T, int TY>
__device__ __forceinline__ void win_stencil(T (*s)[TX + 3], int wx, int wy, T& gx, T& gy, T& lap) {
    stencil(s[wy - 1][wx - 1], s[wy - 1][wx], s[wy - 1][wx + 1], s[wy][wx - 1], s[wy][wx],
            s[wy][wx + 1], s[wy + 1][wx - 1], s[wy + 1][wx], s[wy + 1][wx + 1], gx, gy, lap);
}

}  // namespace lbm

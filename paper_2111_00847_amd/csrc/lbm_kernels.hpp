// lbm_kernels.hpp -- host-side launchers of the gfx950 kernels.
#pragma once

#include "lbm_common.hpp"

namespace lbm {

// nsteps levels; `copy`: the host's guess of the copy holding the state on
// entry, updated to where the launches leave it
template <typename T>
hipError_t launch_step(const KParams<T>& P, char* state, const Layout& L, int64_t nsteps, hipStream_t s,
                       int ty, int by, int& copy);
// two levels of the plain Allen-Cahn step in one launch (lbm_step2.hip); back: the
// tile rows from last to first (xcd_tile)
template <typename T>
void launch_step2(const KParams<T>& P, char* state, const Layout& L, hipStream_t s, bool back);
// A tile of the two-level launch owns at least one level stamp (lbm_step2.hpp).
inline bool stamp_share_ok(int nx, int ny, int tw, int ty) {
    const long long nstamp = (long long)((nx + STAMP_BAND - 1) / STAMP_BAND) * ny;
    return nstamp >= (long long)((nx + tw - 1) / tw) * ((ny + ty - 1) / ty);
}

// Tiles of the two-level launch.  A tile's chain (loads, level n, level n + 1)
// sets the launch's duration until every CU has several of them, so a lattice
// takes the smallest tiles that leave no CU with two; beyond one round the ring
// (region nodes per tile node: 16 x 4 2.5, 32 x 4 2.25, 32 x 8 1.69, 32 x 16 1.41,
// 64 x 8 1.59, 64 x 16 1.33) and the workgroups a CU holds decide.  Measured on
// MI355X, us per level, chosen shape first:
//   FP32 64 x 64      16x4 3.04, 16x8 3.4, 32x4 3.4, 64x8 4.7; one-level 4.99
//        256 x 128    32x4 3.5, 32x8 on 576 threads 3.8, 16x4 3.95; one-level 5.31
//        256 x 256    32x8 on 576 threads 3.9, 32x4 4.4, 64x8 5.0; one-level 5.74
//        256 x 512    32x16 5.03, 64x8 5.2, 32x8 5.5
//        256 x 1024   64x16 6.7, 64x8 6.7, 32x16 6.9
//        1024 x 512   32x16 12.4, 64x8 12.9; 512 x 700 10.1, 10.6; 700 x 700 12.6, 12.9
//        640 x 1089   64x8 17.0, 32x16 16.3; three such lattices at once on streams,
//                     more than the cache holds, 16.7 and 17.4; 1024 x 700 17.4, 16.6
//                     and 17.8, 17.9; 1024 x 1024 22.7, 22.0 and 25.6, 26.2; 1280 x 1024
//                     27.5, 27.0 and 32.6, 34.9.  The library does not know what else
//                     runs: it gives up 2-5% of a lone lattice there, for up to 7% of
//                     several (small_state)
//        4096 x 4096  64x8 347, 32x8 375, 32x16 388 (streamed from HBM)
//        60000 x 3    64x8 10.2, 32x16 16.5; 17000 x 17 12.5, 14.0; 9000 x 49 12.5, 14.5;
//                     9000 x 40 10.7, 11.7: no tiles of 16 rows on lattices of at most 8, nor
//                     where they pad it by a sixth more than tiles of 8 or take a round
//                     more
//   FP64 64 x 64      16x4 3.67, 32x4 4.3, 64x8 6.9; one-level 9.07
//        200 x 100    32x4 4.3, 16x4 4.3, 32x8 5.6; one-level 14.5
//        300 x 300    32x16 7.2, 32x8 7.35, 64x8 7.3
//        1000 x 500   32x8 24.0, 32x16 26.5, 64x8 27.6; 1999 x 2203 194, 312, 294
// The 32x8 tiles of FP64 (80 KB of LDS) run two workgroups of 256 threads per
// CU; of one node per thread (576 threads) they serve single-round lattices.
// S2_NONE: FP64 lattices of one row, which have fewer stamps than 32-wide tiles; they
// run one level per launch (17000 x 1 7.4, two levels on 64x8 tiles 10.5).
enum Step2Shape { S2_NONE, S2_16x4, S2_32x4, S2_32x8_WIDE, S2_32x16, S2_64x16, S2_64x8, S2_32x8 };
inline Step2Shape step2_shape(int nx, int ny, size_t esz, bool small) {
    auto tiles = [&](int tw, int ty) { return (long long)((nx + tw - 1) / tw) * ((ny + ty - 1) / ty); };
    auto one_round = [&](int tw, int ty) { return tiles(tw, ty) <= 256 && stamp_share_ok(nx, ny, tw, ty); };
    if (one_round(16, 4)) return S2_16x4;
    if (one_round(32, 4)) return S2_32x4;
    if (one_round(32, 8)) return S2_32x8_WIDE;
    const bool tall = ny > 8;   // tiles of 16 rows would be half empty
    if (tall && one_round(32, 16)) return S2_32x16;
    if (esz == 8) return stamp_share_ok(nx, ny, 32, 8) ? S2_32x8 : S2_NONE;
    if (tall && one_round(64, 16)) return S2_64x16;
    const int rows8 = (ny + 7) / 8 * 8, rows16 = (ny + 15) / 16 * 16;
    auto rounds = [&](int tw, int ty) { return (tiles(tw, ty) + 511) / 512; };   // two workgroups to a CU
    const bool filled = 6 * rows16 <= 7 * rows8 && rounds(32, 16) <= rounds(64, 8);
    return small && filled && stamp_share_ok(nx, ny, 32, 16) ? S2_32x16 : S2_64x8;
}

// the Allen-Cahn step (either gradient scheme, not the corrected model) on a
// lattice whose copy fits 32-bit offsets: lbm_step folds two levels into a
// launch (not with LBM_TWO_LEVEL=0 in the environment)
bool two_level_step(const Layout& L, int nx, int ny, int pf, int model);
// the same on lattices of at least 256 tiles of 64 x 8 nodes, or on any with
// LBM_TWO_LEVEL=1: what lbm_levels_per_launch reports
bool two_level_path(const Layout& L, int nx, int ny, int pf, int model);
template <typename T>
hipError_t launch_moments(const KParams<T>& P, const char* state, const Layout& L, T* phi, T* u, T* p,
                          hipStream_t s);
template <typename T>
hipError_t launch_init(const KParams<T>& P, char* state, const Layout& L, const T* phi0, const T* u0,
                       const T* p0, int dtype, hipStream_t s);
template <typename T>
hipError_t launch_hydrostatic(const KParams<T>& P, const T* phi0, T* p0, hipStream_t s);
template <typename T>
hipError_t launch_import(const KParams<T>& P, char* state, const Layout& L, const T* f, const T* g,
                         const T* hist, int64_t step, int dtype, hipStream_t s);
template <typename T>
hipError_t launch_export(const KParams<T>& P, const char* state, const Layout& L, T* f, T* g, T* hist,
                         hipStream_t s);
// the Allen-Cahn step / moments with the local gradient scheme (lbm_local.hip)
template <typename T, int MODE>
void launch_local(const KParams<T>& P, char* state, const Layout& L, hipStream_t s, T* phi, T* u, T* p,
                  bool back = false);
template <typename T>
hipError_t launch_diagnostics(const KParams<T>& P, const char* state, const Layout& L, double* host_out,
                              hipStream_t s);

}  // namespace lbm

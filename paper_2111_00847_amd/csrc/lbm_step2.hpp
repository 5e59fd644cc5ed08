// lbm_step2.hpp -- the tile body of two time levels of the Allen-Cahn step
// (stencil gradients) per launch: the plain two-level launch (lbm_step2.hip)
// and the two-level batch launch (lbm_batch.hip) run it.  The scheme and its
// bitwise equality with two one-level steps are described in lbm_step2.hip.
#pragma once

#include "lbm_addr.hpp"
#include "lbm_fused.hpp"

namespace lbm {

// Wall ghosts (Eq. Dwetting) of a window whose position (wx, wy) is node
// (x0 - H + wx, y0 - H + wy): the rule and order of wall_ghosts (x-walls on
// every row that is not beyond a y-wall, then y-walls across all columns up to
// the x-ghosts), on windows of any halo H.  Ends synchronised.
template <typename T, int WW, int WH, int H, int NT, int PITCH>
__device__ __forceinline__ void ghosts_h(const KParams<T>& P, bool need_prev, int x0, int y0, T (*a)[PITCH],
                                         T (*b)[PITCH], int tid) {
    if (P.wall_x) {
        const int wl = H - 1 - x0;          // window column of x = -1
        const int wr = P.nx - x0 + H;       // window column of x = nx
        for (int wy = tid; wy < WH; wy += NT) {
            const int gy = y0 - H + wy;
            if (P.wall_y && (gy < 0 || gy >= P.ny)) continue;
            if (wl >= 0 && wl + 2 < WW) {
                a[wy][wl] = wet_ghost(P, 0, a[wy][wl + 1], a[wy][wl + 2]);
                if (need_prev) b[wy][wl] = wet_ghost(P, 0, b[wy][wl + 1], b[wy][wl + 2]);
            }
            if (wr < WW && wr - 2 >= 0) {
                a[wy][wr] = wet_ghost(P, 1, a[wy][wr - 1], a[wy][wr - 2]);
                if (need_prev) b[wy][wr] = wet_ghost(P, 1, b[wy][wr - 1], b[wy][wr - 2]);
            }
        }
        __syncthreads();
    }
    if (P.wall_y) {
        const int wb = H - 1 - y0;
        const int wt = P.ny - y0 + H;
        for (int wx = tid; wx < WW; wx += NT) {
            const int gx = x0 - H + wx;
            if (P.wall_x && (gx < -1 || gx > P.nx)) continue;
            if (wb >= 0 && wb + 2 < WH) {
                a[wb][wx] = wet_ghost(P, 2, a[wb + 1][wx], a[wb + 2][wx]);
                if (need_prev) b[wb][wx] = wet_ghost(P, 2, b[wb + 1][wx], b[wb + 2][wx]);
            }
            if (wt < WH && wt - 2 >= 0) {
                a[wt][wx] = wet_ghost(P, 3, a[wt - 1][wx], a[wt - 2][wx]);
                if (need_prev) b[wt][wx] = wet_ghost(P, 3, b[wt - 1][wx], b[wt - 2][wx]);
            }
        }
        __syncthreads();
    }
}

// f(0), ..., f(N - 1) with the index a compile-time constant from the start.  The
// positions of a thread (step2_body) are walked with it: in a loop over them, unrolled
// later, their FP32 populations became one wide vector register, copied whole
// between the loads of one position and the next, and each copy waits for the
// loads before it -- the round trips of a tile one after the other.
template <int N, typename F>
__device__ __forceinline__ void each(F&& f) {
    if constexpr (N > 0) {
        each<N - 1>(f);
        f(std::integral_constant<int, N - 1>());
    }
}

// Waits until the wave's loads have arrived (vmcnt 0; the other counters are left).
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// LDS of one tile.  Arrays of A's region have the region's pitch, the phi windows
// theirs.  LOCAL: the local gradient scheme hands B m^phiC of level n and needs
// no window of the previous phi.
template <typename T, int TW, int TY, bool LOCAL = false>
struct Step2Lds {
    static constexpr int AW = TW + 4, AH = TY + 4, NA = AW * AH;   // region of A: the tile and a two-node ring
    static constexpr int WW = TW + 6, WH = TY + 6, NW = WW * WH;   // phi windows of A: a three-node ring
    static constexpr int GW = TW + 2, GH = TY + 2;   // phi window of B: a one-node ring
    T pa[WH][WW];                        // phi of level n (with wall ghosts); B's history window
    T pp[LOCAL ? 1 : WH][WW];            // phi of level n-1 (the history of the copy)
    T fa[Q][NA];                         // post-collision f of A (f_0 in the stored encoding)
    T ga[Q][NA];                         // post-collision g of A (tile and one-node ring)
    T pb[GH][GW + 1];                    // phi of level n + 1 (with wall ghosts)
    T ua[NA], va[NA];                    // velocity of level n on the tile (B's history)
    // LOCAL: m^phiC of level n on the tile (on the tile alone, so that two workgroups of
    // FP64 32 x 8 tiles fit a CU: 80.6 KB)
    T mxa[LOCAL ? TW * TY : 1], mya[LOCAL ? TW * TY : 1];
};

// Whether the body reads its parameters anew in each phase (params_at): in FP64,
// where held from end to end they spilled into vector lanes (240 of the 2900
// vector instructions; 1999 x 2203: 237 to 228 us per level), and in the FP32 tiles
// of large lattices (64 x 8: 4096 x 4096 362 to 357 us, 2048 x 2048 local gradient
// 112 to 104; 32 x 8: a batch of 64 cases 100.6 to 97.3).  A small lattice's single
// round of tiles gains more from having them at hand (64 x 64 FP32 3.3 to 3.1 us).
template <typename T>
__host__ __device__ constexpr bool step2_reload(int tw, int ty, int nt) {
    return sizeof(T) == 8 || (ty == 8 && nt == tw * ty);
}

// Two levels of one TW x TY tile, with the LDS `L` of the workgroup of NT
// threads (64 x NT/64).  `tile` (StateTile, TapeTile) says which tile, where its
// level is read and where level + 2 goes.  MID also stores the tile's
// intermediate level (what a one-level step would write) into the copy at
// tile.mid, non-temporally (with ordinary stores where SK is).  Every thread owns
// up to S positions of A's window and one node of the tile in B.  SK: how the
// destination copy is stored; written through the XCD's L2 it leaves no dirty
// lines to flush between two launches (256 x 1024 FP32: 14.7 to 13.4 us per
// launch; 1024 x 512: 29.2 to 27.2).
// LOCAL: the Allen-Cahn step with the local gradient scheme (Eq. local; the
// one-level body of lbm_local_step.hpp): grad phi of levels >= 1 from each
// node's own f and g, a history of five planes (phi, u, v and m^phiC of the
// previous level), no window of the previous phi, and the general collision
// (STD false), as the one-level kernel runs it.
//
// The loads of a tile are a third to a half of its time and vector issue most
// of the rest.  So the body keeps addresses off the vector unit (planes are
// uniform buffer offsets, f and g of one direction share one byte offset, and
// only tiles within four nodes of an edge of the lattice, `inner` false, look
// at wraps and walls).  Bounce-back costs B nothing: A's wall
// nodes store their reflected populations at the positions beyond the wall
// that B pulls from.
template <typename T, int TW, int TY, int NT, bool STD, StoreKind SK, bool MID = false, bool LOCAL = false, typename Tile>
__device__ __forceinline__ void step2_body(const BodyParams<T, step2_reload<T>(TW, TY, NT)> params, Tile tile, Step2Lds<T, TW, TY, LOCAL>& L) {
    using Lds = Step2Lds<T, TW, TY, LOCAL>;
    static_assert(!(LOCAL && (MID || STD)), "the local scheme: no tape, general collision");
    constexpr int AW = Lds::AW, AH = Lds::AH, WW = Lds::WW, WH = Lds::WH, NW = Lds::NW, GW = Lds::GW, GH = Lds::GH;
    constexpr int S = (NW + NT - 1) / NT;
    constexpr int NRING1 = 2 * GW + 2 * TY;        // window positions of B outside the tile
    static_assert(NRING1 <= NT && TW * TY <= NT, "one node and one window ring position per thread");
    constexpr uint32_t ES = sizeof(T);

    const KParams<T>& P = params_at<T>(params);   // the lattice (the model's constants are read below)
    const int tid = threadIdx.y * TX + threadIdx.x;
    const int x0 = tile.xt * TW, y0 = tile.yt * TY;
    const uint32_t plB = (uint32_t)P.plane * ES;   // bytes of a plane
    const uint32_t bytes = (LOCAL ? 23 : 21) * plB;
    const bool inner = x0 >= 4 && x0 + TW + 4 <= P.nx && y0 >= 4 && y0 + TY + 4 <= P.ny;
    const bool walls = P.wall_x || P.wall_y;

    // position s of this thread in A's window, row by row.  Of two positions to a
    // thread, the rows of the region first and the ring's two rows last: fewer waves
    // have two positions to step in A (64 x 8 tiles: 5 of 8 against 8; us per level,
    // FP32, 4096 x 4096 344 / 352, 2048 x 1200 57.1 / 58.4, 1024 x 1024 22.5 / 22.8; with
    // one or three positions plain order is 0-2% faster).  The ring's columns come
    // with the rows, from the same cache lines.
    // Returns its index in the window; beyond NW: none.
    auto window_pos = [&](int s, int& wx, int& wy) -> int {
        const int idx = tid + s * NT, row = idx / WW;
        wx = idx - row * WW;
        wy = S != 2 ? row : (row < AH ? row + 1 : (row == AH ? 0 : WH - 1));
        return S != 2 || idx >= NW ? idx : wy * WW + wx;
    };
    // whether it lies in A's region
    auto in_region = [](int wx, int wy) -> bool {
        return (unsigned)(wx - 1) < (unsigned)AW && (unsigned)(wy - 1) < (unsigned)AH;
    };

    // ---- A: loads of the window (f, history phi) and of the region (g, history)
    T f[S][9], g[S][9], hp[S], hu[S], hv[S], hmx[S], hmy[S], f0s[S];
    bool ok[S], reg[S];
    int nxi[S], nyi[S];
    uint32_t off[S][9];
    const CopyAddr<uint32_t> sb = tile.source(bytes);
    auto load_f = [&](auto index) {
        constexpr int s = decltype(index)::value;
        int wx, wy;
        const int at = window_pos(s, wx, wy);
        ok[s] = ((s + 1) * NT <= NW || at < NW) && neighbour_offsets<T, uint32_t, -1>(P, inner, x0 - 3 + wx, y0 - 3 + wy, off[s], nxi[s], nyi[s]);
        reg[s] = ok[s] && in_region(wx, wy);
        if (ok[s]) {
            f0s[s] = sb.template ld<T>(off[s][0], 0);
            hp[s] = sb.template ld<T>(off[s][0], 18 * plB);
#pragma unroll
            for (int i = 1; i < Q; i++) f[s][i] = sb.template ld<T>(off[s][i], pair_plane(i) * plB);
        }
    };
    auto load_g = [&](auto index) {
        constexpr int s = decltype(index)::value;
        if (reg[s]) {
            g[s][0] = sb.template ld<T>(off[s][0], 9 * plB);
#pragma unroll
            for (int i = 1; i < Q; i++) g[s][i] = sb.template ld<T>(off[s][i], (9 + pair_plane(i)) * plB);
            hu[s] = sb.template ld<T>(off[s][0], 19 * plB);
            hv[s] = sb.template ld<T>(off[s][0], 20 * plB);
            if constexpr (LOCAL) {
                hmx[s] = sb.template ld<T>(off[s][0], 21 * plB);
                hmy[s] = sb.template ld<T>(off[s][0], 22 * plB);
            }
        }
    };
    // The memory system sets the pace of this phase.  On streamed FP32 states a
    // position's g follows its f, each once the loads before it are in: all loads of
    // a tile at once leave less time in which one tile's loads run under another's
    // arithmetic.  Elsewhere all f, then all g; three positions to a thread (the FP32
    // batch's 32 x 8 tiles) and FP64 rows of broken lines (ordinary stores) by position
    // without the wait.  Measured on MI355X, us per level, no wait / by position / f then g:
    // FP32 4096 x 4096 362 / 346 / 368, 3072 x 2000 137 / 132 / 139, 2048 x 1200 59.6 /
    // 57.5 / 60.1, cached 1280 x 1024 27.7 / 27.4 / 27.1, a batch of 64 cases 95.5 / 94.2 /
    // 94.5, by position without the wait 93.3; FP64 1999 x 2203 196 / 199 / 197,
    // by position without the wait 194, 3001 x 2000 268, 264; 3072 x 2000 274 / 273 / 270,
    // cached 1000 x 700 33.1 / 32.9 / 31.4, 200 x 100 5.3 / 5.05 / 5.0.
    constexpr bool f32 = sizeof(T) == 4, waits = f32 ? S <= 2 : SK != ST_PLAIN;
    if constexpr (f32 ? SK != ST_THROUGH || S > 2 : SK == ST_PLAIN) {
        each<S>([&](auto index) {
            load_f(index);
            if (waits) wait_loads();
            load_g(index);
        });
    } else {
        each<S>(load_f);
        if (waits) wait_loads();
        each<S>(load_g);
    }
    const int64_t lev = tile.level();
    const bool first = lev == 0;
    T* const pa = &L.pa[0][0];
    T* const pp = &L.pp[0][0];
    double phid[S];
    each<S>([&](auto index) {
        constexpr int s = decltype(index)::value;
        if (ok[s]) {
            const double f0 = rest_decode(f0s[s], hp[s], P.rest_w);
            f[s][0] = (T)f0;
            phid[s] = f0 + moving_sum_d(f[s]);
            int wx, wy;
            const int at = window_pos(s, wx, wy);
            pa[at] = (T)phid[s];
            if constexpr (!LOCAL) pp[at] = hp[s];
        }
    });
    __syncthreads();
    if (!inner) ghosts_h<T, WW, WH, 3, NT, WW>(params_at<T>(params), !first && !LOCAL, x0, y0, L.pa, L.pp, tid);

    // ---- A: the step of level n on the region
    each<S>([&](auto index) {
        constexpr int s = decltype(index)::value;
        int wx, wy;
        const int at = window_pos(s, wx, wy);
        if (!reg[s]) return;
        const KParams<T>& P = params_at<T>(params);
        const int ax = wx - 1, ay = wy - 1;
        const int idx = at - (WW - AW) * wy - (AW + 1);   // ay * AW + ax
        T gx, gy, lap, gxp = T(0), gyp = T(0), lp, php = T(0), up = T(0), vp = T(0);
        win_stencil_at(L.pa, wx, wy, gx, gy, lap);
        const Macro<T> M = [&]() -> Macro<T> {
            if constexpr (LOCAL) {
                const T phi = L.pa[wy][wx];
                T mpx = T(0), mpy = T(0);
                if (!first) {
                    php = hp[s];
                    up = hu[s];
                    vp = hv[s];
                    mpx = hmx[s];
                    mpy = hmy[s];
                    local_grad(P, f[s], g[s], phi, lap, php * up, php * vp, gx, gy);
                }
                return macro<T, false, true>(P, g[s], phi, gx, gy, lap, first, php, T(0), T(0), up, vp, T(0), T(0),
                                             mpx, mpy);
            } else {
                if (!first) {
                    win_stencil_at(L.pp, wx, wy, gxp, gyp, lp);
                    php = hp[s];
                    up = hu[s];
                    vp = hv[s];
                }
                return macro(P, g[s], L.pa[wy][wx], gx, gy, lap, first, php, gxp, gyp, up, vp);
            }
        }();
        const double f0n = collide_f<T, false, STD>(P, M, f[s], phid[s]);
        const T f0e = rest_encode<T>(f0n, M.phi, P.rest_w);
        L.fa[0][idx] = f0e;
#pragma unroll
        for (int i = 1; i < Q; i++) L.fa[i][idx] = f[s][i];
        if ((unsigned)(ax - 1) < (unsigned)(AW - 2) && (unsigned)(ay - 1) < (unsigned)(AH - 2)) {
            collide_g<T, STD>(P, M, g[s]);
#pragma unroll
            for (int i = 0; i < Q; i++) L.ga[i][idx] = g[s][i];
            // B's history of the velocity (read on the tile only)
            L.ua[idx] = M.u;
            L.va[idx] = M.v;
            if constexpr (LOCAL)
                if ((unsigned)(ax - 2) < (unsigned)TW && (unsigned)(ay - 2) < (unsigned)TY) {
                    L.mxa[(ay - 2) * TW + ax - 2] = M.mx;
                    L.mya[(ay - 2) * TW + ax - 2] = M.my;
                }
            if (!inner && walls) {   // what B's pulls from beyond a wall find there
#pragma unroll
                for (int i = 1; i < Q; i++)
                    if (beyond_wall<-1>(P, i, nxi[s], nyi[s])) {
                        L.fa[i][idx - cy(i) * AW - cx(i)] = f[s][opp(i)];
                        L.ga[i][idx - cy(i) * AW - cx(i)] = g[s][opp(i)];
                    }
            }
            if constexpr (MID) {
                const int x = x0 + ax - 2, y = y0 + ay - 2;
                // a node of the tile (not a wrapped position)
                if (ax >= 2 && ax < AW - 2 && ay >= 2 && ay < AH - 2 && x < P.nx && y < P.ny) {
                    const CopyAddr<uint32_t> mb(tile.mid, bytes);
                    const uint32_t k = ((uint32_t)y * (uint32_t)P.nx + (uint32_t)x) * ES;
                    constexpr StoreKind MK = SK == ST_PLAIN ? ST_PLAIN : ST_NT;
                    mb.template st<MK>(k, 0, f0e);
#pragma unroll
                    for (int i = 1; i < Q; i++) mb.template st<MK>(k, i * plB, f[s][i]);
#pragma unroll
                    for (int i = 0; i < Q; i++) mb.template st<MK>(k, (9 + i) * plB, g[s][i]);
                    mb.template st<MK>(k, 18 * plB, M.phi);
                    mb.template st<MK>(k, 19 * plB, M.u);
                    mb.template st<MK>(k, 20 * plB, M.v);
                }
            }
        }
    });
    __syncthreads();

    // ---- B: phi of level n + 1 on the tile and its one-node ring, from A's f
    // f arriving at region position c (the wall nodes' reflected populations lie
    // beyond the walls), the sum in FP64
    auto pull_a = [&](int c, T phi_a, T* fo) -> double {
#pragma unroll
        for (int i = 1; i < Q; i++) fo[i] = L.fa[i][c - cy(i) * AW - cx(i)];
        const double f0 = rest_decode(L.fa[0][c], phi_a, P.rest_w);
        fo[0] = (T)f0;
        return f0 + moving_sum_d(fo);
    };
    const int ly = tid / TW, lx = tid - ly * TW, c = (ly + 2) * AW + lx + 2;
    const int x = x0 + lx, y = y0 + ly;
    T fb[9];
    double phb = 0.0;
    // a ragged tile's positions beyond the lattice hold wrapped nodes on a
    // periodic axis (they are the ring of the tile's last nodes)
    if ((NT == TW * TY || tid < TW * TY) && (inner || ((x < P.nx || !P.wall_x) && (y < P.ny || !P.wall_y)))) {
        phb = pull_a(c, L.pa[ly + 3][lx + 3], fb);
        L.pb[ly + 1][lx + 1] = (T)phb;
    }
    if (tid < NRING1) {
        int wx, wy;
        if (tid < 2 * GW) {
            wx = tid < GW ? tid : tid - GW;
            wy = tid < GW ? 0 : GH - 1;
        } else {
            wx = tid < 2 * GW + TY ? 0 : GW - 1;
            wy = 1 + tid - 2 * GW - (tid < 2 * GW + TY ? 0 : TY);
        }
        const int px = x0 - 1 + wx, py = y0 - 1 + wy;
        if (inner || ((!P.wall_x || (unsigned)px < (unsigned)P.nx) && (!P.wall_y || (unsigned)py < (unsigned)P.ny))) {
            T fw[9];
            L.pb[wy][wx] = (T)pull_a((wy + 1) * AW + wx + 1, L.pa[wy + 2][wx + 2], fw);
        }
    }
    __syncthreads();
    if (!inner) ghosts_h<T, GW, GH, 1, NT, GW + 1>(params_at<T>(params), false, x0, y0, L.pb, L.pb, tid);

    // ---- B: the step of level n + 1 on the tile, stored into the other copy
    if ((NT == TW * TY || tid < TW * TY) && (inner || (x < P.nx && y < P.ny))) {
        const KParams<T>& P = params_at<T>(params);
        T gb[9];
#pragma unroll
        for (int i = 0; i < Q; i++) gb[i] = L.ga[i][c - cy(i) * AW - cx(i)];
        T gx, gy, lap, gxp, gyp, lp;
        win_stencil_at(L.pb, lx + 1, ly + 1, gx, gy, lap);
        const Macro<T> M = [&]() -> Macro<T> {
            if constexpr (LOCAL) {
                const T phi = L.pb[ly + 1][lx + 1], php = L.pa[ly + 3][lx + 3];
                const T up = L.ua[c], vp = L.va[c];
                local_grad(P, fb, gb, phi, lap, php * up, php * vp, gx, gy);
                return macro<T, false, true>(P, gb, phi, gx, gy, lap, false, php, T(0), T(0), up, vp, T(0), T(0),
                                             L.mxa[ly * TW + lx], L.mya[ly * TW + lx]);
            } else {
                win_stencil_at(L.pa, lx + 3, ly + 3, gxp, gyp, lp);
                return macro(P, gb, L.pb[ly + 1][lx + 1], gx, gy, lap, false, L.pa[ly + 3][lx + 3], gxp, gyp,
                             L.ua[c], L.va[c]);
            }
        }();
        const double f0n = collide_f<T, false, STD>(P, M, fb, phb);
        collide_g<T, STD>(P, M, gb);
        const uint32_t k = ((uint32_t)y * (uint32_t)P.nx + (uint32_t)x) * ES;
        const CopyAddr<uint32_t> db(tile.dst(), bytes);
        db.template st<SK>(k, 0, rest_encode<T>(f0n, M.phi, P.rest_w));
#pragma unroll
        for (int i = 1; i < Q; i++) db.template st<SK>(k, i * plB, fb[i]);
#pragma unroll
        for (int i = 0; i < Q; i++) db.template st<SK>(k, (9 + i) * plB, gb[i]);
        db.template st<SK>(k, 18 * plB, M.phi);
        db.template st<SK>(k, 19 * plB, M.u);
        db.template st<SK>(k, 20 * plB, M.v);
        if constexpr (LOCAL) {
            db.template st<SK>(k, 21 * plB, M.mx);
            db.template st<SK>(k, 22 * plB, M.my);
        }
    }
    // every wave read the stamp before the barriers above
    tile.done(tid);
}

// The stamps a workgroup owns.  The lattice's `nstamp` level stamps are dealt
// to its tiles in order, sq or (the first srem tiles) sq + 1 to each; every tile
// needs one to read, so a lattice takes tiles of a shape only while it has at
// least as many stamps as tiles (stamp_share_ok).
struct StampShare {
    int sq, srem;
};
inline StampShare stamp_share(long long nstamp, long long ntiles) {
    return StampShare{(int)(nstamp / ntiles), (int)(nstamp % ntiles)};
}
// One tile of a ping-pong state (copies at off0 and off1, level stamps at
// off_stamp, dealt to the tiles by `sh`): its stamp selects the source copy, and
// its stamps move to level n + 2 in the other copy when it is done.
// (Starting the loads on the copy the host last left the state in while the stamp
// is read, as the one-level step does, gained nothing here: 6.79 against 6.70 us
// per level at 256 x 1024 FP32, 12.8 against 13.05 at 1024 x 512.)
struct StateTile {
    char* state;
    size_t off0, off1, off_stamp;
    StampShare sh;
    int t, xt, yt;
    int64_t sv;
    static constexpr char* mid = nullptr;
    __device__ int64_t* stamp() const {
        return reinterpret_cast<int64_t*>(state + off_stamp) + (size_t)t * sh.sq + (t < sh.srem ? t : sh.srem);
    }
    __device__ CopyAddr<uint32_t> source(uint32_t bytes) {
        sv = stamp()[0];
        return CopyAddr<uint32_t>(state + (stamp_copy(sv) ? off1 : off0), bytes);
    }
    __device__ int64_t level() const { return stamp_level(sv); }
    __device__ char* dst() const { return state + (stamp_copy(sv) ? off0 : off1); }
    __device__ void done(int tid) const {
        if (tid < sh.sq + (t < sh.srem ? 1 : 0)) stamp()[tid] = stamp_of(stamp_level(sv) + 2, 1 - stamp_copy(sv));
    }
};

// Level `lev` in the copy at `src` to level lev + 2 in the copy at `d`, the
// intermediate level into the copy at `mid` (tapes).
struct TapeTile {
    const char* src;
    char* mid;
    char* d;
    int64_t lev;
    int xt, yt;
    __device__ CopyAddr<uint32_t> source(uint32_t bytes) const { return CopyAddr<uint32_t>(src, bytes); }
    __device__ int64_t level() const { return lev; }
    __device__ char* dst() const { return d; }
    __device__ void done(int) const {}
};

}  // namespace lbm

// lbm_step.hip -- gfx950 kernels of the fused phase-field LBM time step.
//
// Memory layout (structure of arrays, x fastest): a state buffer is
//   [header | copy 0 | copy 1 | level stamps | diagnostics scratch],
// a copy being f_0 | f_1..f_8 | g_0..g_8 | hist = (phi, u, v), every
// plane padded to a multiple of 64 elements.  The copy that holds level n
// holds the post-collision populations of level n-1 -- a node obtains its
// level-n populations by pulling them from its neighbours -- and the history
// of level n-1, from which the explicit-Euler time derivatives are formed.  A
// launch reads that copy and writes the other.  The level and its copy are
// kept in per-row stamps owned by the workgroups (lbm_common.hpp), so host
// code never needs them, no workgroup waits for another, and a sequence of
// steps can be captured in a graph.
//
// The phi stencils need phi on a one-node ring around each tile.  A tile of
// 64 x TY nodes first pulls the populations of its (64+2) x (TY+2) window,
// sums them into phi in LDS (the ring's pulls hit L2: those lines are the
// neighbour tiles' own reads), fills wall ghosts, and then each thread runs
// the per-node update for its nodes (lbm_fused.hpp).
#include <cstdlib>

#include "lbm_addr.hpp"
#include "lbm_ch_step.hpp"
#include "lbm_fused.hpp"
#include "lbm_kernels.hpp"

namespace lbm {

// Steps on states that the last-level cache holds (HINT) start their loads
// on the copy of the host's parity guess `hint` while the level stamp is read
// (step_core); LBM_PARITY_HINT=0 reads the stamp first there too.  States
// streamed from HBM always read the stamp first: a wrong guess would cost a
// whole extra copy of HBM reads (the guess is wrong after every replay of a
// captured graph of an odd number of launches, 1.5x the step time measured on
// 4096 x 4096 FP32), while the stamp read costs a tile little next to its
// stream of loads; there the guess only sets the direction of the sweep
// (xcd_tile).
#ifndef LBM_PARITY_HINT
#define LBM_PARITY_HINT 1
#endif

template <typename T, int TY, int MODE, typename OFF, int NBY, bool STD, bool NT = true, bool LATE_G = false,
          bool HINT = MODE == 0 && LBM_PARITY_HINT && !NT>
__global__ __launch_bounds__(TX* NBY) __attribute__((amdgpu_waves_per_eu(StepWaves<T, TY, NBY>::value)))
void k_step(KParams<T> P, char* state, size_t off0, size_t off1, size_t off_stamp, int ntx, int nty, T* out_phi,
            T* out_u, T* out_p, int hint) {
    __shared__ T sphi[TY + 2][TX + 3];
    __shared__ T sphp[TY + 2][TX + 3];
    int xt, yt;
    if (LBM_XCD_REMAP) {
        xcd_tile(blockIdx.x, ntx, nty, xt, yt, MODE == 0 && !HINT && hint != 0);
    } else {
        xt = blockIdx.x % ntx;
        yt = blockIdx.x / ntx;
    }
    step_tile<T, TY, MODE, OFF, NBY, STD, NT, LATE_G, HINT>(
        P, state, off0, off1, off_stamp, xt, yt, out_phi, out_u, out_p, sphi, sphp, hint);
}

// The Cahn-Hilliard variant and the corrected comparison model with the
// Allen-Cahn phase field (ACC), both on the two-node phi window of lbm_ch.hpp:
// one 64 x TY tile per workgroup, one node per thread (64 x TY threads; 64 x 8
// for 16 rows), tiles dealt to the XCDs as for the Allen-Cahn step, the same
// state layout, level stamps and store policy.  MODE 0: one time step; MODE 1:
// phi, u, p of the current level.  Tile shape (measured on MI355X, FP32 square
// droplet, us per step): 8 rows on 64 x 8 threads 574 / 39.5 / 9.4 at 4096^2 /
// 1024^2 / 200^2, against 589 / 42.0 / 11.7 for the shapes used before (8 rows
// on 64 x 4 threads with two nodes per thread, 4 rows on 64 x 4 below 1024
// tiles); 16 rows on 64 x 8 threads 575 / 38.2 / 18.4; 16 rows on 64 x 16 656 /
// 43.2 / 14.0.  LBM_CH_TY forces 4, 8 or 16 rows.
// SWEEPS: the launches sweep forward and `back` by turns (streamed states).  The steps
// of cached states do not read `back`: it lies in a cache line of the arguments that
// nothing else needs, and every workgroup waited for it (FP64 64 x 196 8.77 against
// 8.55 us per step, 256 x 320 10.3 against 10.0).
#ifndef LBM_CH_TY
#define LBM_CH_TY 0
#endif

template <typename T, int TY, int MODE, bool ACC, bool STD, bool NT = true, int NBY = BY, typename OFF = uint64_t,
          bool SWEEPS = true>
__global__ __launch_bounds__(TX* NBY) void k_step_ch(KParams<T> P, char* state, size_t off0, size_t off1,
                                                    size_t off_stamp, int ntx, int nty, T* out_phi, T* out_u,
                                                    T* out_p, bool back) {
    __shared__ ChWindow<T, TY> W;
    int xt, yt;
    if (LBM_XCD_REMAP) {
        xcd_tile(blockIdx.x, ntx, nty, xt, yt, SWEEPS && back);
    } else {
        xt = blockIdx.x % ntx;
        yt = blockIdx.x / ntx;
    }
    ch_step_tile<T, TY, MODE, ACC, STD, NT, NBY, OFF>(P, state, off0, off1, off_stamp, xt, yt, out_phi, out_u, out_p,
                                                      W);
}

// Rows of the CH tile (8 unless LBM_CH_TY) and thread rows (one node per thread).
constexpr int CH_TY = (LBM_CH_TY == 4 || LBM_CH_TY == 16) ? LBM_CH_TY : 8;
constexpr int CH_NBY = CH_TY == 4 ? 4 : 8;

template <typename T, int MODE, bool ACC, bool STD, bool NT, typename OFF, bool SWEEPS>
static void launch_ch_shape(const KParams<T>& P, char* state, const Layout& L, hipStream_t s, T* phi, T* u, T* p,
                            bool back) {
    const int ntx = (P.nx + TX - 1) / TX, nty = (P.ny + CH_TY - 1) / CH_TY;
    k_step_ch<T, CH_TY, MODE, ACC, STD, NT, CH_NBY, OFF, SWEEPS><<<ntx * nty, dim3(TX, CH_NBY), 0, s>>>(
        P, state, L.off_buf[0], L.off_buf[1], L.off_stamp, ntx, nty, phi, u, p, back);
}

// Steps address a copy below 4 GiB with 32-bit byte offsets from a uniform
// base, as the Allen-Cahn step does (1323 against 1960 VALU instructions in the
// FP32 kernel, 62 against 68 VGPRs; measured on MI355X, FP32 square droplet, us
// per step: 554 against 571 at 4096^2, 37.0 against 39.7 at 1024^2, 7.0 against
// 9.6 at 200^2); moments and larger copies with 64-bit ones.
template <typename T, int MODE, bool ACC, bool STD, bool NT = true, bool SWEEPS = true>
static void launch_ch_acc_std(const KParams<T>& P, char* state, const Layout& L, hipStream_t s, T* phi, T* u, T* p,
                              bool back) {
    if constexpr (MODE == 0) {
        if (L.buf_bytes < (size_t(1) << 32)) {
            launch_ch_shape<T, MODE, ACC, STD, NT, uint32_t, SWEEPS>(P, state, L, s, phi, u, p, back);
            return;
        }
    }
    launch_ch_shape<T, MODE, ACC, STD, NT, uint64_t, true>(P, state, L, s, phi, u, p, back);
}

// the standard rates compiled in for steps (moments do not collide); steps on
// a state that the last-level cache holds, or of rows that end inside a cache
// line (whole_lines), store it with ordinary stores
template <typename T, int MODE, bool ACC>
static void launch_ch_acc(const KParams<T>& P, char* state, const Layout& L, hipStream_t s, T* phi, T* u, T* p,
                          bool back) {
    if constexpr (MODE == 0) {
        const bool plain = plain_stores(L, P.nx), cached = cached_state(L);
        if (P.rates_std) {
            if (cached) launch_ch_acc_std<T, MODE, ACC, true, false, false>(P, state, L, s, phi, u, p, back);
            else if (plain) launch_ch_acc_std<T, MODE, ACC, true, false>(P, state, L, s, phi, u, p, back);
            else launch_ch_acc_std<T, MODE, ACC, true>(P, state, L, s, phi, u, p, back);
        } else {
            if (cached) launch_ch_acc_std<T, MODE, ACC, false, false, false>(P, state, L, s, phi, u, p, back);
            else if (plain) launch_ch_acc_std<T, MODE, ACC, false, false>(P, state, L, s, phi, u, p, back);
            else launch_ch_acc_std<T, MODE, ACC, false>(P, state, L, s, phi, u, p, back);
        }
    } else {
        launch_ch_acc_std<T, MODE, ACC, false>(P, state, L, s, phi, u, p, back);
    }
}

// CH (any model) or the corrected AC model: the two-node-window kernels.
template <typename T, int MODE>
static void launch_ch(const KParams<T>& P, char* state, const Layout& L, hipStream_t s, T* phi, T* u, T* p,
                      bool back = false) {
    if (P.pf == 1) launch_ch_acc<T, MODE, false>(P, state, L, s, phi, u, p, back);
    else launch_ch_acc<T, MODE, true>(P, state, L, s, phi, u, p, back);
}

// ---------------------------------------------------------------- init / import / export
// phi at (x, y) of a caller field, extended by the lattice's ghost rule:
// periodic axes wrap; x-wall ghosts from the row, y-wall ghosts from the
// (possibly x-ghost) column -- the same order as the LDS window.  The few nodes
// beside a wall call it; inlined at each of their nine (or 81) positions it made
// a kernel of 14000 instructions that runs once, from a cold instruction cache.
template <typename T>
__device__ __attribute__((noinline)) T field_at(ParamsPtr<T> params, const T* phi, int x, int y) {
    const KParams<T> P = *(const KParams<T>*)params;
    if (!P.wall_x && (x < 0 || x >= P.nx)) x = x < 0 ? x + P.nx : x - P.nx;
    if (!P.wall_y && (y < 0 || y >= P.ny)) y = y < 0 ? y + P.ny : y - P.ny;
    auto col = [&](int xx, int yy) -> T {
        const T* row = phi + (long long)yy * P.nx;
        if (xx < 0) return wet_ghost(P, 0, row[0], row[1]);
        if (xx >= P.nx) return wet_ghost(P, 1, row[P.nx - 1], row[P.nx - 2]);
        return row[xx];
    };
    if (y < 0) return wet_ghost(P, 2, col(x, 0), col(x, 1));
    if (y >= P.ny) return wet_ghost(P, 3, col(x, P.ny - 1), col(x, P.ny - 2));
    return col(x, y);
}

// mu_phi of a caller field at (x, y) (Sec. 2), positions beyond a wall taking
// the value of the first fluid node (x first, then y), periodic axes wrapping.
template <typename T>
__device__ __attribute__((noinline)) T mu_at(ParamsPtr<T> params, const T* phi, int x, int y) {
    const KParams<T> P = *(const KParams<T>*)params;
    if (x < 0 || x >= P.nx) x = P.wall_x ? (x < 0 ? 0 : P.nx - 1) : (x < 0 ? x + P.nx : x - P.nx);
    if (y < 0 || y >= P.ny) y = P.wall_y ? (y < 0 ? 0 : P.ny - 1) : (y < 0 ? y + P.ny : y - P.ny);
    T n_[3][3];
#pragma unroll
    for (int j = 0; j < 3; j++)
#pragma unroll
        for (int i = 0; i < 3; i++) n_[j][i] = field_at<T>(params, phi, x + i - 1, y + j - 1);
    T gx, gy, lap;
    stencil(n_[0][0], n_[0][1], n_[0][2], n_[1][0], n_[1][1], n_[1][2], n_[2][0], n_[2][1], n_[2][2], gx, gy, lap);
    return chem_pot(P, n_[1][1], lap);
}

// The (2 H + 1)^2 neighbourhood of (x, y) of a caller field where none of it lies
// beyond a wall (false otherwise): plain loads at wrapped offsets.
template <int H, typename T>
__device__ __forceinline__ bool open_neighbourhood(const KParams<T>& P, const T* phi, int x, int y,
                                                   T (&v)[2 * H + 1][2 * H + 1]) {
    if (P.nx < H || P.ny < H || (P.wall_x && (x < H || x >= P.nx - H)) || (P.wall_y && (y < H || y >= P.ny - H)))
        return false;
    long long col[2 * H + 1], row[2 * H + 1];
#pragma unroll
    for (int i = 0; i <= 2 * H; i++) {
        int a = x + i - H, b = y + i - H;
        a += a < 0 ? P.nx : 0;
        b += b < 0 ? P.ny : 0;
        col[i] = a - (a >= P.nx ? P.nx : 0);
        row[i] = (long long)(b - (b >= P.ny ? P.ny : 0)) * P.nx;
    }
#pragma unroll
    for (int j = 0; j <= 2 * H; j++)
#pragma unroll
        for (int i = 0; i <= 2 * H; i++) v[j][i] = phi[row[j] + col[i]];
    return true;
}

// What a state needs besides its copy: the header and every level stamp.
struct StateMeta {
    StateHeader* header;
    int64_t* stamp;
    long long nstamp;
    int64_t value;
    int dtype;
};
template <typename T>
__device__ __forceinline__ void set_meta(const KParams<T>& P, const StateMeta& m, long long i) {
    if (i < m.nstamp) m.stamp[i] = m.value;
    if (i == 0) {
        m.header->magic = STATE_MAGIC;
        m.header->nx = P.nx;
        m.header->ny = P.ny;
        m.header->dtype = m.dtype;
    }
}

// Storing a state: the post-streaming population i of node (x, y) goes to the slot
// that (x, y) pulls i from (neighbour_offsets; the map is one to one, so all
// nodes' populations fill the copy).

// The state of level 0: equilibria of the given fields in the pull
// representation, zero history, header and stamps, in one pass (bound by HBM:
// 1 to 4 planes read, 21 or 23 written).  CH: Cahn-Hilliard.
template <typename T, bool CH, typename OFF>
__global__ __launch_bounds__(256) void k_init(KParams<T> P, const T* phi0, const T* u0, const T* p0, char* dst_base,
                                              StateMeta meta) {
    const ParamsPtr<T> params = (ParamsPtr<T>)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr OFF ES = sizeof(T);
    const OFF plB = (OFF)P.plane * ES;
    const int nh = P.grad == 1 ? 5 : 3;
    const CopyAddr<OFF> D(dst_base, (18 + nh) * plB);
    const long long n = (long long)P.nx * P.ny;
    for (long long k = blockIdx.x * (long long)blockDim.x + threadIdx.x; k < n;
         k += (long long)gridDim.x * blockDim.x) {
        set_meta(P, meta, k);   // no more stamps than nodes
        const int y = (int)(k / P.nx), x = (int)(k - (long long)y * P.nx);
        T n_[3][3];
        if (!open_neighbourhood<1>(P, phi0, x, y, n_))
#pragma unroll
            for (int j = 0; j < 3; j++)
#pragma unroll
                for (int i = 0; i < 3; i++) n_[j][i] = field_at<T>(params, phi0, x + i - 1, y + j - 1);
        T gx, gy, lap;
        stencil(n_[0][0], n_[0][1], n_[0][2], n_[1][0], n_[1][1], n_[1][2], n_[2][0], n_[2][1], n_[2][2],
                gx, gy, lap);
        const T phi = n_[1][1];
        const T u = u0 ? u0[k] : T(0), v = u0 ? u0[n + k] : T(0), p = p0 ? p0[k] : T(0);
        T lnx, lny, mx, my;
        if (CH) {   // Cahn-Hilliard: grad mu of the initial field, mu mirrored at walls
            T mn[3][3], w[5][5];
            if (open_neighbourhood<2>(P, phi0, x, y, w)) {
#pragma unroll
                for (int j = 0; j < 3; j++)
#pragma unroll
                    for (int i = 0; i < 3; i++) {
                        T a, b, c;
                        win_stencil_at(w, i + 1, j + 1, a, b, c);
                        mn[j][i] = chem_pot(P, w[j + 1][i + 1], c);
                    }
            } else {
#pragma unroll
                for (int j = 0; j < 3; j++)
#pragma unroll
                    for (int i = 0; i < 3; i++) mn[j][i] = mu_at<T>(params, phi0, x + i - 1, y + j - 1);
            }
            T gmx, gmy, lm;
            stencil(mn[0][0], mn[0][1], mn[0][2], mn[1][0], mn[1][1], mn[1][2], mn[2][0], mn[2][1], mn[2][2], gmx,
                    gmy, lm);
            mass_flux_ch(P, gmx, gmy, mx, my);
        } else {
            mass_flux(P, phi, gx, gy, lnx, lny, mx, my);
        }
        const T rho = P.drho * (phi - P.phiB) + P.rhoB;
        OFF off[9];
        int xi, yi;
        neighbour_offsets<T, OFF, -1>(P, false, x, y, off, xi, yi);
        T m[9], e[9];
        T mf[9] = {phi, T(-2) * phi, phi, phi * u, -phi * u, phi * v, -phi * v, T(0), T(0)};
        if (CH) {   // Eq. MfMRCH1
            const T mu = chem_pot(P, phi, lap);
            mf[1] = T(-4) * phi + T(2) * mu;
            mf[2] = T(4) * phi - T(3) * mu;
        }
        from_moments(mf, e);
        D.template st<ST_PLAIN>(off[0], 0, rest_encode<T>((double)e[0], T(0), P.rest_w));
#pragma unroll
        for (int i = 1; i < Q; i++) D.template st<ST_PLAIN>(off[i], pair_plane(i) * plB, e[i]);
        for (int j = 0; j < nh; j++) D.template st<ST_PLAIN>(off[0], (18 + j) * plB, T(0));
        T tr = T(3) * rho * (u * u + v * v) + T(3) * (u * mx + v * my);
        m[0] = P.rho0;
        m[1] = T(-4) * P.rho0 + T(6) * p + tr;
        m[2] = T(4) * P.rho0 - T(9) * p - tr;
        m[3] = rho * u;
        m[4] = -rho * u;
        m[5] = rho * v;
        m[6] = -rho * v;
        m[7] = (u * mx - v * my) + rho * (u * u - v * v);
        m[8] = T(0.5) * ((u * my + v * mx) + T(2) * rho * u * v);
        from_moments(m, e);
        D.template st<ST_PLAIN>(off[0], 9 * plB, e[0]);
#pragma unroll
        for (int i = 1; i < Q; i++) D.template st<ST_PLAIN>(off[i], (9 + pair_plane(i)) * plB, e[i]);
    }
}

// The state of level n from post-streaming populations f, g ([9][n] each) and
// the history of level n - 1 (NULL: zeros), in one pass.
template <typename T, typename OFF>
__global__ __launch_bounds__(256) void k_import(KParams<T> P, const T* f, const T* g, const T* hist, char* dst_base,
                                                StateMeta meta) {
    constexpr OFF ES = sizeof(T);
    const OFF plB = (OFF)P.plane * ES;
    const int nh = P.grad == 1 ? 5 : 3;
    const CopyAddr<OFF> D(dst_base, (18 + nh) * plB);
    const long long n = (long long)P.nx * P.ny;
    for (long long k = blockIdx.x * (long long)blockDim.x + threadIdx.x; k < n;
         k += (long long)gridDim.x * blockDim.x) {
        set_meta(P, meta, k);
        const int y = (int)(k / P.nx), x = (int)(k - (long long)y * P.nx);
        T fv[9], gv[9], hv[5];
#pragma unroll
        for (int i = 0; i < Q; i++) fv[i] = f[i * n + k];
#pragma unroll
        for (int i = 0; i < Q; i++) gv[i] = g[i * n + k];
#pragma unroll
        for (int j = 0; j < 5; j++) hv[j] = hist && j < nh ? hist[j * n + k] : T(0);
        OFF off[9];
        int xi, yi;
        neighbour_offsets<T, OFF, -1>(P, false, x, y, off, xi, yi);
        D.template st<ST_PLAIN>(off[0], 0, rest_encode<T>((double)fv[0], hv[0], P.rest_w));
#pragma unroll
        for (int i = 1; i < Q; i++) D.template st<ST_PLAIN>(off[i], pair_plane(i) * plB, fv[i]);
        D.template st<ST_PLAIN>(off[0], 9 * plB, gv[0]);
#pragma unroll
        for (int i = 1; i < Q; i++) D.template st<ST_PLAIN>(off[i], (9 + pair_plane(i)) * plB, gv[i]);
#pragma unroll
        for (int j = 0; j < 5; j++)
            if (j < nh) D.template st<ST_PLAIN>(off[0], (18 + j) * plB, hv[j]);
    }
}

// Post-streaming populations and history of the current level: f, g [9][n],
// hist [3][n] ([5][n] for the local gradient scheme), any NULL.  Nine loads, then
// nine stores; in FP64 with non-temporal stores while what is written fits the last-level
// cache, and beyond it each store after its own load (EACH).  Measured on MI355X, us a
// call, nine and nine / non-temporal / each: FP64 1024 x 1024 96 / 77 / 99, 1000 x 1001
// 90 / 77 / 96, 2048 x 1200 183 / 177 / 179, 1999 x 2203 341 / 370 / 313; FP32 3000 x 3001
// 345 / 357 / 394.
enum ExportForm { EXPORT_NINE, EXPORT_NT, EXPORT_EACH };
template <typename T, typename OFF, ExportForm FORM>
__global__ __launch_bounds__(256) void k_export(KParams<T> P, const char* state, size_t off0, size_t off1,
                                                size_t off_stamp, T* f, T* g, T* hist) {
    constexpr OFF ES = sizeof(T);
    const OFF plB = (OFF)P.plane * ES;
    const int nh = P.grad == 1 ? 5 : 3;
    const int cur = stamp_copy(*reinterpret_cast<const int64_t*>(state + off_stamp));
    const CopyAddr<OFF> S(state + (cur ? off1 : off0), (18 + nh) * plB);
    const long long n = (long long)P.nx * P.ny;
    for (long long k = blockIdx.x * (long long)blockDim.x + threadIdx.x; k < n;
         k += (long long)gridDim.x * blockDim.x) {
        const int y = (int)(k / P.nx), x = (int)(k - (long long)y * P.nx);
        OFF off[9];
        int xi, yi;
        neighbour_offsets<T, OFF, -1>(P, false, x, y, off, xi, yi);
        auto give = [&](T* out, T rest, OFF plane0) {
            if constexpr (FORM == EXPORT_EACH) {
                out[k] = rest;
#pragma unroll
                for (int i = 1; i < Q; i++) out[i * n + k] = S.template ld<T>(off[i], plane0 + pair_plane(i) * plB);
            } else {
                T v[9];
                v[0] = rest;
#pragma unroll
                for (int i = 1; i < Q; i++) v[i] = S.template ld<T>(off[i], plane0 + pair_plane(i) * plB);
#pragma unroll
                for (int i = 0; i < Q; i++) {
                    if constexpr (FORM == EXPORT_NT) __builtin_nontemporal_store(v[i], &out[i * n + k]);
                    else out[i * n + k] = v[i];
                }
            }
        };
        if (f) give(f, (T)rest_decode(S.template ld<T>(off[0], 0), S.template ld<T>(off[0], 18 * plB), P.rest_w), 0);
        if (g) give(g, S.template ld<T>(off[0], 9 * plB), 9 * plB);
        if (hist)   // phi, u, v of level n-1 (and m^phiC of level n-1 for the local gradient scheme)
            for (int j = 0; j < nh; j++) hist[j * n + k] = S.template ld<T>(off[0], (18 + j) * plB);
    }
}

// Hydrostatic pressure of the two fluids at rest (the initial pressure of the
// gravity-driven set-ups): rho from the density law of Sec. 2 at phi0,
// dp/dy = f, f = (rho - rho_ref) g_y, integrated down every column by the
// trapezoid rule from p = 0 at the top row, then the mean taken out, in FP64.
// A column is a serial chain of ny additions (kept in that order: an instability
// that starts from this field amplifies its rounding).  The chain itself is
// short; what took 482 us at 256 x 1024 FP32 (11.3 ms at
// 4096 x 4096) was one workgroup loading a row between every two additions.  So
// a workgroup takes 16 columns and stages 256 rows of f at a time in LDS, the
// next rows' loads running while 16 of its threads run the chains (24 and 33 us for
// the two passes at 256 x 1024; chains fed by waves of their own, and reading LDS a
// group of rows ahead, were no faster: 27 to 40 us, and 21 and 33):
//   k_hydro_cols, SUMS  the sum of p down columns x, x + 1024, ... (the order of the
//                       additions of one workgroup of 1024 threads), kept in column
//                       x's own first bytes of p0 (rows 0 and 1 in FP32, row 0 in
//                       FP64);
//   k_hydro_mean        the mean, left in the first bytes of every workgroup's
//                       first column;
//   k_hydro_cols        p less the mean.
constexpr int HYDRO_THREADS = 1024, HYDRO_COLS = 16, HYDRO_ROWS = 256, HYDRO_STAGE = 256;

// The double kept in column x's first bytes of p0.
template <typename T>
__device__ __forceinline__ void put_col(T* p0, int nx, int x, double v) {
    if constexpr (sizeof(T) == 8) p0[x] = v;
    else {
        const uint64_t w = __builtin_bit_cast(uint64_t, v);
        p0[x] = __builtin_bit_cast(T, (uint32_t)w);
        p0[nx + x] = __builtin_bit_cast(T, (uint32_t)(w >> 32));
    }
}
template <typename T>
__device__ __forceinline__ double get_col(const T* p0, int nx, int x) {
    if constexpr (sizeof(T) == 8) return p0[x];
    else return __builtin_bit_cast(double, (uint64_t)__builtin_bit_cast(uint32_t, p0[x]) |
                                               (uint64_t)__builtin_bit_cast(uint32_t, p0[nx + x]) << 32);
}

template <typename T, bool SUMS>
__global__ __launch_bounds__(HYDRO_STAGE) void k_hydro_cols(KParams<T> P, const T* __restrict__ phi0,
                                                            T* __restrict__ p0) {
    constexpr int PER = HYDRO_ROWS * HYDRO_COLS / HYDRO_STAGE;   // staged elements per thread
    __shared__ double f[2][HYDRO_ROWS][HYDRO_COLS + 1];
    const int nx = P.nx, ny = P.ny, tid = threadIdx.x;
    const double gy = (double)P.gy, drho = (double)P.drho, rhoB = (double)P.rhoB, rref = (double)P.rho_ref,
                 phiB = (double)P.phiB;
    int x0 = blockIdx.x * HYDRO_COLS;
    const double mean = SUMS ? 0.0 : get_col(p0, nx, x0);   // read before the first barrier, overwritten after it
    const int chunks = (ny + HYDRO_ROWS - 1) / HYDRO_ROWS;
    T v[PER];
    // chunk c: rows ny - 1 - c HYDRO_ROWS downwards, element e of it row e / COLS, column e % COLS
    auto load = [&](int c) {
#pragma unroll
        for (int q = 0; q < PER; q++) {
            const int e = tid + q * HYDRO_STAGE, j = ny - 1 - c * HYDRO_ROWS - e / HYDRO_COLS, x = x0 + e % HYDRO_COLS;
            v[q] = j >= 0 && x < nx ? phi0[(long long)j * nx + x] : T(0);
        }
    };
    auto stage = [&](int c) {
#pragma unroll
        for (int q = 0; q < PER; q++) {
            const int e = tid + q * HYDRO_STAGE;
            f[c & 1][e / HYDRO_COLS][e % HYDRO_COLS] = (drho * ((double)v[q] - phiB) + rhoB - rref) * gy;
        }
    };
    double acc = 0.0;
    for (; x0 < nx; x0 += SUMS ? HYDRO_THREADS : nx) {
        load(0);
        stage(0);
        __syncthreads();
        double p = 0.0, fu = 0.0;
        for (int c = 0; c < chunks; c++) {
            if (c + 1 < chunks) load(c + 1);
            const int rows = ny - c * HYDRO_ROWS < HYDRO_ROWS ? ny - c * HYDRO_ROWS : HYDRO_ROWS;
            if (tid < HYDRO_COLS && x0 + tid < nx) {
                double (*col)[HYDRO_COLS + 1] = f[c & 1];
#pragma unroll 8
                for (int r = 0; r < rows; r++) {
                    const double fj = col[r][tid];
                    if (c > 0 || r > 0) p -= 0.5 * (fj + fu);
                    fu = fj;
                    acc += p;
                    if (!SUMS) col[r][tid] = p - mean;
                }
            }
            __syncthreads();
            if (!SUMS)
#pragma unroll
                for (int q = 0; q < PER; q++) {
                    const int e = tid + q * HYDRO_STAGE, r = e / HYDRO_COLS, x = x0 + e % HYDRO_COLS;
                    if (r < rows && x < nx) p0[(long long)(ny - 1 - c * HYDRO_ROWS - r) * nx + x] = (T)f[c & 1][r][e % HYDRO_COLS];
                }
            if (c + 1 < chunks) stage(c + 1);
            __syncthreads();
        }
    }
    x0 = blockIdx.x * HYDRO_COLS;
    if (SUMS && tid < HYDRO_COLS && x0 + tid < nx) put_col(p0, nx, x0 + tid, acc);
}

template <typename T>
__global__ __launch_bounds__(HYDRO_THREADS) void k_hydro_mean(KParams<T> P, T* p0) {
    __shared__ double red[HYDRO_THREADS / 64];
    double acc = 0.0;
    if ((int)threadIdx.x < P.nx) acc = get_col(p0, P.nx, threadIdx.x);
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();   // every column's sum is read
    double t = 0.0;
    for (int w = 0; w < HYDRO_THREADS / 64; w++) t += red[w];
    const double mean = t / ((double)P.nx * (double)P.ny);
    for (int x = threadIdx.x * HYDRO_COLS; x < P.nx; x += HYDRO_THREADS * HYDRO_COLS) put_col(p0, P.nx, x, mean);
}

// The same by one workgroup, every thread walking its columns twice (the second
// walk subtracts the mean the first one gives): for a p0 that overlaps phi0, whose
// bytes hold no sums before they are read, for one row, and for few rows.

template <typename T>
__global__ __launch_bounds__(HYDRO_THREADS) void k_hydrostatic(KParams<T> P, const T* phi0, T* p0) {
    __shared__ double red[HYDRO_THREADS / 64];
    const int nx = P.nx, ny = P.ny;
    const double gy = (double)P.gy, drho = (double)P.drho, rhoB = (double)P.rhoB, rref = (double)P.rho_ref,
                 phiB = (double)P.phiB;
    auto force = [&](int j, int x) { return (drho * ((double)phi0[(long long)j * nx + x] - phiB) + rhoB - rref) * gy; };
    double total = 0.0;
    for (int pass = 0; pass < 2; pass++) {
        const double mean = pass == 0 ? 0.0 : total / ((double)nx * (double)ny);
        double acc = 0.0;
        for (int x = threadIdx.x; x < nx; x += HYDRO_THREADS) {
            double p = 0.0, fu = force(ny - 1, x);
            acc += p;
            if (pass == 1) p0[(long long)(ny - 1) * nx + x] = (T)(p - mean);
            for (int j = ny - 2; j >= 0; j--) {
                const double f = force(j, x);
                p -= 0.5 * (f + fu);
                fu = f;
                acc += p;
                if (pass == 1) p0[(long long)j * nx + x] = (T)(p - mean);
            }
        }
        if (pass == 0) {
            for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
            if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
            __syncthreads();
            double t = 0.0;
            for (int w = 0; w < HYDRO_THREADS / 64; w++) t += red[w];
            total = t;
        }
    }
}

// ---------------------------------------------------------------- launchers
static int grid1d(long long n) {
    long long b = (n + 255) / 256;
    return (int)(b < 65536 ? (b > 0 ? b : 1) : 65536);
}

// Byte size of one copy fits 32-bit offsets?
static bool small_copy(const Layout& L) { return L.buf_bytes < (size_t(1) << 32); }


template <typename T, int TY, int MODE, int NBY = BY>
static void launch_tile(const KParams<T>& P, char* state, const Layout& L, hipStream_t s, T* phi, T* u, T* p,
                        int hint = 0) {
    const int ntx = (P.nx + TX - 1) / TX, nty = (P.ny + TY - 1) / TY;
    dim3 blk(TX, NBY);
    // the standard rates compiled in for steps (moments do not collide)
    const bool std_rates = MODE == 0 && P.rates_std;
    if (MODE == 0 && resident_state(L)) {   // the last-level cache holds both copies: g loaded late
        if (std_rates)
            k_step<T, TY, MODE, uint32_t, NBY, true, false, true><<<ntx * nty, blk, 0, s>>>(
                P, state, L.off_buf[0], L.off_buf[1], L.off_stamp, ntx, nty, phi, u, p, hint);
        else
            k_step<T, TY, MODE, uint32_t, NBY, false, false, true><<<ntx * nty, blk, 0, s>>>(
                P, state, L.off_buf[0], L.off_buf[1], L.off_stamp, ntx, nty, phi, u, p, hint);
    } else if (MODE == 0 && cached_state(L)) {
        if (std_rates)
            k_step<T, TY, MODE, uint32_t, NBY, true, false><<<ntx * nty, blk, 0, s>>>(
                P, state, L.off_buf[0], L.off_buf[1], L.off_stamp, ntx, nty, phi, u, p, hint);
        else
            k_step<T, TY, MODE, uint32_t, NBY, false, false><<<ntx * nty, blk, 0, s>>>(
                P, state, L.off_buf[0], L.off_buf[1], L.off_stamp, ntx, nty, phi, u, p, hint);
    } else if (MODE == 0 && small_copy(L) && !whole_lines(L, P.nx)) {
        if (std_rates)
            k_step<T, TY, MODE, uint32_t, NBY, true, false, false, false><<<ntx * nty, blk, 0, s>>>(
                P, state, L.off_buf[0], L.off_buf[1], L.off_stamp, ntx, nty, phi, u, p, hint);
        else
            k_step<T, TY, MODE, uint32_t, NBY, false, false, false, false><<<ntx * nty, blk, 0, s>>>(
                P, state, L.off_buf[0], L.off_buf[1], L.off_stamp, ntx, nty, phi, u, p, hint);
    } else if (small_copy(L)) {
        if (std_rates)
            k_step<T, TY, MODE, uint32_t, NBY, true><<<ntx * nty, blk, 0, s>>>(P, state, L.off_buf[0], L.off_buf[1],
                                                                                L.off_stamp, ntx, nty, phi, u, p, hint);
        else
            k_step<T, TY, MODE, uint32_t, NBY, false><<<ntx * nty, blk, 0, s>>>(P, state, L.off_buf[0], L.off_buf[1],
                                                                                 L.off_stamp, ntx, nty, phi, u, p, hint);
    } else {
        if (std_rates)
            k_step<T, TY, MODE, uint64_t, NBY, true><<<ntx * nty, blk, 0, s>>>(P, state, L.off_buf[0], L.off_buf[1],
                                                                                L.off_stamp, ntx, nty, phi, u, p, hint);
        else
            k_step<T, TY, MODE, uint64_t, NBY, false><<<ntx * nty, blk, 0, s>>>(P, state, L.off_buf[0], L.off_buf[1],
                                                                                 L.off_stamp, ntx, nty, phi, u, p, hint);
    }
}

// Two levels per launch for the Allen-Cahn step with either gradient scheme
// (stencils or Eq. local; present or original model; lbm_step2.hip) on lattices
// whose copy fits 32-bit offsets, with tiles by size (step2_shape): one-level
// launches are slower on every lattice measured (64 x 64 FP32 4.99 against 3.04
// us per level, FP64 9.07 against 3.67; 4096 x 4096 523 against 364).  The
// environment variable LBM_TWO_LEVEL, read at every call, turns it off ("0").
// lbm_levels_per_launch reports 2 only where these launches run, but of those
// lattices only the ones of at least 256 tiles of 64 x 8 nodes (all of them with
// LBM_TWO_LEVEL "1", which changes nothing else).  The compile-time LBM_TWO_LEVEL=0
// removes the path.
#ifndef LBM_TWO_LEVEL
#define LBM_TWO_LEVEL 1
#endif

static char two_level_env() {   // '0', '1' or, unset or anything else, 0
    const char* e = getenv("LBM_TWO_LEVEL");
    return e && (e[0] == '0' || e[0] == '1') && e[1] == 0 ? e[0] : 0;
}

static bool two_level_eligible(const Layout& L, int pf, int model) {
    return LBM_TWO_LEVEL && pf == 0 && model != 2 && L.buf_bytes < (size_t(1) << 32) && two_level_env() != '0';
}

bool two_level_step(const Layout& L, int nx, int ny, int pf, int model) {
    return two_level_eligible(L, pf, model) && step2_shape(nx, ny, L.esz, small_state(L)) != S2_NONE;
}

bool two_level_path(const Layout& L, int nx, int ny, int pf, int model) {
    if (!two_level_step(L, nx, ny, pf, model)) return false;
    const long long tiles8 = (long long)((nx + TX - 1) / TX) * ((ny + 7) / 8);
    return two_level_env() == '1' || tiles8 >= 256;
}

template <typename T>
hipError_t launch_step(const KParams<T>& P, char* state, const Layout& L, int64_t nsteps, hipStream_t s,
                       int ty, int by, int& copy) {
    constexpr int T16 = sizeof(T) == 8 ? 8 : 16;   // FP64 tiles stop at 8 rows
    auto back = [&] { return copy != 0 && !cached_state(L); };   // alternate sweeps (xcd_tile)
    if (two_level_step(L, P.nx, P.ny, P.pf, P.model))
        for (; nsteps >= 2; nsteps -= 2) {
            launch_step2<T>(P, state, L, s, back());
            copy ^= 1;
        }
    for (int64_t t = 0; t < nsteps; t++) {
        const int h = copy;   // the copy this launch is expected to find the state in
        const bool rev = back();
        copy ^= 1;
        if (P.pf == 1 || P.model == 2) launch_ch<T, 0>(P, state, L, s, nullptr, nullptr, nullptr, rev);
        else if (P.grad == 1) launch_local<T, 0>(P, state, L, s, nullptr, nullptr, nullptr, rev);
        else if (ty == 4) launch_tile<T, 4, 0>(P, state, L, s, nullptr, nullptr, nullptr, h);
        else if (ty == 8 || sizeof(T) == 8) {
            if (by == 8) launch_tile<T, 8, 0, 8>(P, state, L, s, nullptr, nullptr, nullptr, h);
            else launch_tile<T, 8, 0>(P, state, L, s, nullptr, nullptr, nullptr, h);
        } else {
            if (by == 8) launch_tile<T, T16, 0, 8>(P, state, L, s, nullptr, nullptr, nullptr, h);
            else launch_tile<T, T16, 0>(P, state, L, s, nullptr, nullptr, nullptr, h);
        }
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_moments(const KParams<T>& P, const char* state, const Layout& L, T* phi, T* u, T* p,
                          hipStream_t s) {
    if (P.pf == 1 || P.model == 2) launch_ch<T, 1>(P, const_cast<char*>(state), L, s, phi, u, p);
    else if (P.grad == 1) launch_local<T, 1>(P, const_cast<char*>(state), L, s, phi, u, p);
    else launch_tile<T, 8, 1>(P, const_cast<char*>(state), L, s, phi, u, p);
    return hipGetLastError();
}

static StateMeta state_meta(char* state, const Layout& L, int dtype, int64_t stamp) {
    return StateMeta{reinterpret_cast<StateHeader*>(state), reinterpret_cast<int64_t*>(state + L.off_stamp),
                     (long long)L.nstamp, stamp, dtype};
}

template <typename T>
hipError_t launch_init(const KParams<T>& P, char* state, const Layout& L, const T* phi0, const T* u0,
                       const T* p0, int dtype, hipStream_t s) {
    const StateMeta meta = state_meta(state, L, dtype, stamp_of(0, 0));
    auto go = [&](auto kernel) LBM_CALLS_STUB { kernel<<<grid1d(L.n), 256, 0, s>>>(P, phi0, u0, p0, state + L.off_buf[0], meta); };
    if (P.pf == 1) small_copy(L) ? go(k_init<T, true, uint32_t>) : go(k_init<T, true, uint64_t>);
    else small_copy(L) ? go(k_init<T, false, uint32_t>) : go(k_init<T, false, uint64_t>);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_hydrostatic(const KParams<T>& P, const T* phi0, T* p0, hipStream_t s) {
    const long long n = (long long)P.nx * P.ny;
    // One workgroup where it walks few rows in all (its columns 1024 at a time, about 0.25
    // us a row), less than the three launches of the staged columns take (14 us, and more
    // from 16 passes on): 48 x 40 13.0 against 15.3 us, 1000 x 30 13.4 / 14.3, 20000 x 2 17.2 /
    // 31.8; 48 x 50 15.5 / 15.0, 1000 x 40 16.9 / 14.4, 4000 x 10 17.0 / 14.1.  Same bits.
    const long long passes = (P.nx + HYDRO_THREADS - 1) / HYDRO_THREADS;
    const bool few = passes * P.ny <= (P.nx <= 256 ? 40 : 28 + 2 * passes);
    if (P.ny < 2 || few || (p0 < phi0 + n && phi0 < p0 + n)) {
        k_hydrostatic<T><<<1, HYDRO_THREADS, 0, s>>>(P, phi0, p0);
        return hipGetLastError();
    }
    const int g = (P.nx + HYDRO_COLS - 1) / HYDRO_COLS;
    k_hydro_cols<T, true><<<g < HYDRO_THREADS / HYDRO_COLS ? g : HYDRO_THREADS / HYDRO_COLS, HYDRO_STAGE, 0, s>>>(P, phi0, p0);
    k_hydro_mean<T><<<1, HYDRO_THREADS, 0, s>>>(P, p0);
    k_hydro_cols<T, false><<<g, HYDRO_STAGE, 0, s>>>(P, phi0, p0);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_import(const KParams<T>& P, char* state, const Layout& L, const T* f, const T* g,
                         const T* hist, int64_t step, int dtype, hipStream_t s) {
    const int cur = (int)(step & 1);
    const StateMeta meta = state_meta(state, L, dtype, stamp_of(step, cur));
    auto go = [&](auto kernel) LBM_CALLS_STUB {
        kernel<<<grid1d(L.n), 256, 0, s>>>(P, f, g, step > 0 ? hist : nullptr, state + L.off_buf[cur], meta);
    };
    small_copy(L) ? go(k_import<T, uint32_t>) : go(k_import<T, uint64_t>);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_export(const KParams<T>& P, const char* state, const Layout& L, T* f, T* g, T* hist,
                         hipStream_t s) {
    auto go = [&](auto kernel) LBM_CALLS_STUB {
        kernel<<<grid1d(L.n), 256, 0, s>>>(P, state, L.off_buf[0], L.off_buf[1], L.off_stamp, f, g, hist);
    };
    if constexpr (sizeof(T) == 4) small_copy(L) ? go(k_export<T, uint32_t, EXPORT_NINE>) : go(k_export<T, uint64_t, EXPORT_NINE>);
    else if ((size_t)L.n * (9 * !!f + 9 * !!g + 3 * !!hist) * sizeof(T) <= size_t(256) << 20) go(k_export<T, uint32_t, EXPORT_NT>);
    else small_copy(L) ? go(k_export<T, uint32_t, EXPORT_EACH>) : go(k_export<T, uint64_t, EXPORT_EACH>);
    return hipGetLastError();
}

#define LBM_INSTANTIATE(T)                                                                              \
    template hipError_t launch_step<T>(const KParams<T>&, char*, const Layout&, int64_t, hipStream_t, int, int, \
                                       int&);                                                            \
    template hipError_t launch_moments<T>(const KParams<T>&, const char*, const Layout&, T*, T*, T*,     \
                                          hipStream_t);                                                 \
    template hipError_t launch_init<T>(const KParams<T>&, char*, const Layout&, const T*, const T*,     \
                                       const T*, int, hipStream_t);                                     \
    template hipError_t launch_import<T>(const KParams<T>&, char*, const Layout&, const T*, const T*,   \
                                         const T*, int64_t, int, hipStream_t);                          \
    template hipError_t launch_export<T>(const KParams<T>&, const char*, const Layout&, T*, T*, T*,     \
                                         hipStream_t);                                                  \
    template hipError_t launch_hydrostatic<T>(const KParams<T>&, const T*, T*, hipStream_t);

LBM_INSTANTIATE(float)
LBM_INSTANTIATE(double)

}  // namespace lbm

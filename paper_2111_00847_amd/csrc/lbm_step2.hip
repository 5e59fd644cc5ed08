// lbm_step2.hip -- two time levels of the Allen-Cahn step (either gradient
// scheme) per launch.
//
// On small lattices a one-level launch is bound by its own latency (the load,
// window, collide, store chain of a tile, and the launch itself) more than by
// bytes; on larger ones it is bound by HBM, which it crosses once per level.  A
// two-level launch pays the chain once and crosses HBM once for two levels: a
// tile of TW x TY nodes advances from level n to n + 2 by
//   A. computing level n + 1 (the step of level n) on the tile and a two-node
//      ring around it: the populations of that region are pulled from the
//      state, phi of level n on a three-node ring is summed into an LDS
//      window (with the phi of level n-1 from the history), and the
//      post-collision f (and g on the one-node ring) are kept in LDS;
//   B. the step of level n + 1 on the tile alone, pulling from LDS, and storing
//      the result into the other copy.
// Every quantity of A is computed from the same inputs with the same device
// functions as the one-level step (lbm_fused.hpp), and B consumes exactly
// what a one-level step would load back from the copy written by A (the FP32
// rest population included: it is kept in the stored encoding), so two levels
// of this launch equal two one-level launches bit for bit.  The ring costs
// recomputation (the region of A is (TW + 4)(TY + 4) nodes) and L2 reads of
// the neighbouring tiles' rows, not HBM traffic beyond those rows: a launch
// reads the state once and writes it once for two levels.  On states larger than
// the last-level cache the sweeps alternate in direction (xcd_tile); step2_store says
// how the copy is stored.
//
// Where the time of a launch goes (wave clocks, 256 x 1024 FP32, 64 x 16 tiles, one
// per CU, before the window's ring was read with the region and the stores wrote
// through): 4.0 us until the loads are in, 3.9 A, 1.9 B and its stores, and 3.5
// between launches.
//
// A launch writes level n + 2 into the other copy (the level stamps carry the
// copy, lbm_common.hpp).
#include "lbm_kernels.hpp"
#include "lbm_step2.hpp"

namespace lbm {

enum { BACK = 1, STRIPS = 2 };

// Two levels of one tile per workgroup, tiles dealt to the XCDs (xcd_tile) in
// `order`: sweep direction, and strips for streamed states.  What is written through is
// cached and swept forward in bands, and does not read it.
// P is the kernel's first argument: the body reads it from the argument
// segment.  LOCAL: the local gradient scheme (Eq. local; the general collision,
// as the one-level kernel runs it).
template <typename T, int TW, int TY, int NT, bool STD, StoreKind SK, bool LOCAL>
__global__ __launch_bounds__(NT) void k_step2(KParams<T> P, char* state, size_t off0, size_t off1, size_t off_stamp,
                                              int ntx, int nty, StampShare sh, int order) {
    __shared__ Step2Lds<T, TW, TY, LOCAL> L;
    int xt, yt;
    xcd_tile(blockIdx.x, ntx, nty, xt, yt, SK != ST_THROUGH && (order & BACK), SK != ST_THROUGH && (order & STRIPS));
    step2_body<T, TW, TY, NT, STD, SK, false, LOCAL>(
        kernel_params<step2_reload<T>(TW, TY, NT)>(P),
        StateTile{state, off0, off1, off_stamp, sh, (int)blockIdx.x, xt, yt, 0}, L);
}

template <typename T, int TW, int TY, int NT>
static void launch_step2_shape(const KParams<T>& P, char* state, const Layout& L, hipStream_t s, bool back) {
    const int ntx = (P.nx + TW - 1) / TW, nty = (P.ny + TY - 1) / TY;
    const StampShare sh = stamp_share((long long)L.nstamp, (long long)ntx * nty);
    const dim3 grd(ntx * nty), blk(TX, NT / TX);
    const int order = (back ? BACK : 0) | (cached_state(L) ? 0 : STRIPS);
    auto go = [&](auto kernel) LBM_CALLS_STUB {
        kernel<<<grd, blk, 0, s>>>(P, state, L.off_buf[0], L.off_buf[1], L.off_stamp, ntx, nty, sh, order);
    };
    auto by_store = [&](auto kind) {
        constexpr StoreKind SK = decltype(kind)::value;
        if (P.grad == 1) go(k_step2<T, TW, TY, NT, false, SK, true>);
        else if (P.rates_std) go(k_step2<T, TW, TY, NT, true, SK, false>);
        else go(k_step2<T, TW, TY, NT, false, SK, false>);
    };
    switch (step2_store(2 * L.buf_bytes, whole_lines(L, P.nx))) {
        case ST_THROUGH: by_store(std::integral_constant<StoreKind, ST_THROUGH>()); break;
        case ST_NT: by_store(std::integral_constant<StoreKind, ST_NT>()); break;
        default: by_store(std::integral_constant<StoreKind, ST_PLAIN>());
    }
}

// The launch's tiles (step2_shape).
template <typename T>
void launch_step2(const KParams<T>& P, char* state, const Layout& L, hipStream_t s, bool back) {
    switch (step2_shape(P.nx, P.ny, sizeof(T), small_state(L))) {
        case S2_16x4: launch_step2_shape<T, 16, 4, 256>(P, state, L, s, back); break;
        case S2_32x4: launch_step2_shape<T, 32, 4, 384>(P, state, L, s, back); break;
        case S2_32x8_WIDE: launch_step2_shape<T, 32, 8, 576>(P, state, L, s, back); break;
        case S2_32x16: launch_step2_shape<T, 32, 16, 512>(P, state, L, s, back); break;
        case S2_64x16:
            if constexpr (sizeof(T) == 4) launch_step2_shape<T, 64, 16, 1024>(P, state, L, s, back);
            break;
        default:
            if constexpr (sizeof(T) == 8) launch_step2_shape<T, 32, 8, 256>(P, state, L, s, back);
            else launch_step2_shape<T, 64, 8, 512>(P, state, L, s, back);
    }
}

template void launch_step2<float>(const KParams<float>&, char*, const Layout&, hipStream_t, bool);
template void launch_step2<double>(const KParams<double>&, char*, const Layout&, hipStream_t, bool);

}  // namespace lbm

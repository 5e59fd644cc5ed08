// lbm_batch.hip -- many independent lattices of uneven sizes advanced by one
// launch per time step (or per two).
//
// The batch state is one caller buffer holding every case's own state
// (same layout as a single lattice, 256-byte aligned, back to back).  A work
// item is one 64 x TY tile of one case; items are numbered case by case and
// a grid of one workgroup per item, or a grid of G workgroups that stride
// over the items (b, b + G, b + 2G, ...), takes them.  Each item runs exactly
// the single-lattice tile body (lbm_fused.hpp) with its case's parameters and
// level stamps, so a case advanced in a batch is bitwise identical to the
// same case advanced alone.  The tile height and G are picked per batch by
// timing the candidates on the batch itself (the autotuner), and K steps are
// captured once into a hipGraph and replayed.
// Batches that hold Cahn-Hilliard or corrected Allen-Cahn cases (the
// two-node-window body of lbm_ch_step.hpp) or local-gradient cases
// (lbm_local_step.hpp) run a second kernel whose LDS holds any of the windows;
// each item runs its case's body.  Batches whose every case runs the plain
// Allen-Cahn step (stencil gradients, present or original model) advance two
// levels per launch, as a single lattice does (lbm_step2.hpp; bitwise two
// one-level steps), with an odd step count ending on a one-level launch.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <vector>

#include "../../include/lbm.h"
#include "lbm_ch_step.hpp"
#include "lbm_fused.hpp"
#include "lbm_kernels.hpp"
#include "lbm_local_step.hpp"
#include "lbm_step2.hpp"

namespace lbm {

Layout layout_of(const lbm_params* p);
int validate(const lbm_params* p);
int hip_fail(hipError_t e);
template <typename T>
KParams<T> resolve(const lbm_params* p, const Layout& L);

template <typename T>
struct BatchCase {
    KParams<T> P;
    size_t base;                 // byte offset of the case's state in the batch buffer
    size_t off0, off1, off_stamp;
    int ntx, nty;
    StampShare share;            // of the case's tiles (two-level launch)
    int item_begin;              // first work item of this case
    int body;                    // 0: Allen-Cahn step; 1: Cahn-Hilliard; 2: corrected Allen-Cahn (ACC);
                                 // 3: Allen-Cahn with the local gradient scheme
};

// Case of work item w: the number of cases whose first item is <= w, less
// one.  Every thread of the workgroup tests one case (item_begin ascends with
// the case index) and the workgroup counts the hits: one round of loads
// instead of the dependent loads of a search.
template <typename T>
__device__ __forceinline__ int batch_case(const BatchCase<T>* __restrict__ cases, int ncases, int w, int nthreads) {
    const int tid = threadIdx.y * TX + threadIdx.x;
    int n = 0;
    for (int c0 = 0; c0 < ncases; c0 += nthreads) {
        const int c = c0 + tid;
        n += __syncthreads_count(c < ncases && cases[c].item_begin <= w);
    }
    return n - 1;
}

// NT: non-temporal state stores (the batch's state exceeds the last-level
// cache); ordinary ones otherwise, as for a single lattice.  LOOP: a
// persistent grid (items b, b + G, ...); without it one item per workgroup,
// whose body needs fewer registers (60 against 92 VGPRs for 64 x 4 tiles in
// FP32: 8 waves per SIMD against 5).
template <typename T, int TY, int NBY, bool NT, bool LOOP = true>
__global__ __launch_bounds__(TX* NBY) __attribute__((amdgpu_waves_per_eu(StepWaves<T, TY, NBY>::value)))
void k_step_batch(const BatchCase<T>* __restrict__ cases, int ncases, int nitems, char* batch_state) {
    __shared__ T sphi[TY + 2][TX + 3];
    __shared__ T sphp[TY + 2][TX + 3];
    auto item = [&](int w) {
        const BatchCase<T>& C = cases[batch_case(cases, ncases, w, TX * NBY)];
        const int local = w - C.item_begin;
        // the collision specialisation the case runs alone (lbm_step), so that it stays bitwise
        if (C.P.rates_std)
            step_tile<T, TY, 0, uint32_t, NBY, true, NT>(C.P, batch_state + C.base, C.off0, C.off1, C.off_stamp,
                                                     local % C.ntx, local / C.ntx, nullptr, nullptr, nullptr, sphi, sphp);
        else
            step_tile<T, TY, 0, uint32_t, NBY, false, NT>(C.P, batch_state + C.base, C.off0, C.off1, C.off_stamp,
                                                      local % C.ntx, local / C.ntx, nullptr, nullptr, nullptr, sphi, sphp);
    };
    if constexpr (LOOP) {
        for (int w = blockIdx.x; w < nitems; w += gridDim.x) {
            item(w);
            __syncthreads();   // the next item reuses the LDS window
        }
    } else if ((int)blockIdx.x < nitems) {   // uniform over the workgroup
        item(blockIdx.x);
    }
}

// Two levels per launch: one work item, a TW x TY tile of one case, per workgroup
// of NT threads, items dealt to the XCDs in bands so that neighbouring tiles share
// an L2 (us per level, 32 x 8 tiles, against items in launch order: 8 cases FP32
// 13.6 / 17.1, 20 cases 30.1 / 38.4, 64 cases 100.6 / 107.8).  One item per workgroup: a loop over items (a
// persistent grid) doubles the registers of the body.  PER_ITEM: the table
// holds one entry per item (its case's), so that the workgroup reads its case
// directly instead of counting item_begin over the cases first (one round
// trip and a barrier fewer before the tile's loads).
template <typename T, int TW, int TY, int NT, StoreKind SK, bool PER_ITEM>
__global__ __launch_bounds__(NT) void k_step2_batch(const BatchCase<T>* __restrict__ cases, int ncases, int nitems,
                                                    char* batch_state) {
    __shared__ Step2Lds<T, TW, TY> L;
    const int w = xcd_band(blockIdx.x, nitems);
    const BatchCase<T>& C = cases[PER_ITEM ? w : batch_case(cases, ncases, w, NT)];
    const int local = w - C.item_begin;
    const StateTile tile{batch_state + C.base, C.off0, C.off1, C.off_stamp, C.share, local, local % C.ntx,
                         local / C.ntx, 0};
    auto body = [&](auto params) {
        if (C.P.rates_std) step2_body<T, TW, TY, NT, true, SK>(params, tile, L);
        else step2_body<T, TW, TY, NT, false, SK>(params, tile, L);
    };
    body(memory_params<step2_reload<T>(TW, TY, NT)>(C.P));
}

// Batches with two-node-window or local-gradient cases: 64 x TY threads (one
// node per thread), the LDS holds any of the windows, each item runs its
// case's body; LOOP as for k_step_batch.
template <typename T, int TY, bool NT, bool LOOP = true>
__global__ __launch_bounds__(TX* TY) void k_step_batch_wide(const BatchCase<T>* __restrict__ cases, int ncases,
                                                            int nitems, char* batch_state) {
    constexpr int NBY = TY;
    __shared__ union {
        struct {
            T sphi[TY + 2][TX + 3];
            T sphp[TY + 2][TX + 3];
        } ac;
        ChWindow<T, TY> ch;
    } lds;
    auto item = [&](int w) {
        const BatchCase<T>& C = cases[batch_case(cases, ncases, w, TX * NBY)];
        const int local = w - C.item_begin;
        const int xt = local % C.ntx, yt = local / C.ntx;
        char* st0 = batch_state + C.base;
        if (C.body == 0 && C.P.rates_std)
            step_tile<T, TY, 0, uint32_t, NBY, true, NT>(C.P, st0, C.off0, C.off1, C.off_stamp, xt, yt, nullptr,
                                                         nullptr, nullptr, lds.ac.sphi, lds.ac.sphp);
        else if (C.body == 0)
            step_tile<T, TY, 0, uint32_t, NBY, false, NT>(C.P, st0, C.off0, C.off1, C.off_stamp, xt, yt, nullptr,
                                                          nullptr, nullptr, lds.ac.sphi, lds.ac.sphp);
        else if (C.body == 1 && C.P.rates_std)
            ch_step_tile<T, TY, 0, false, true, NT, NBY, uint32_t>(C.P, st0, C.off0, C.off1, C.off_stamp, xt, yt,
                                                                   nullptr, nullptr, nullptr, lds.ch);
        else if (C.body == 1)
            ch_step_tile<T, TY, 0, false, false, NT, NBY, uint32_t>(C.P, st0, C.off0, C.off1, C.off_stamp, xt, yt,
                                                                    nullptr, nullptr, nullptr, lds.ch);
        else if (C.body == 3)
            local_step_tile<T, TY, 0, NT, NBY, uint32_t>(C.P, st0, C.off0, C.off1, C.off_stamp, xt, yt, nullptr,
                                                         nullptr, nullptr, lds.ac.sphi);
        else if (C.P.rates_std)
            ch_step_tile<T, TY, 0, true, true, NT, NBY, uint32_t>(C.P, st0, C.off0, C.off1, C.off_stamp, xt, yt,
                                                                  nullptr, nullptr, nullptr, lds.ch);
        else
            ch_step_tile<T, TY, 0, true, false, NT, NBY, uint32_t>(C.P, st0, C.off0, C.off1, C.off_stamp, xt, yt,
                                                                   nullptr, nullptr, nullptr, lds.ch);
    };
    if constexpr (LOOP) {
        for (int w = blockIdx.x; w < nitems; w += gridDim.x) {
            item(w);
            __syncthreads();   // the next item reuses the LDS
        }
    } else if ((int)blockIdx.x < nitems) {   // uniform over the workgroup
        item(blockIdx.x);
    }
}

}  // namespace lbm

using namespace lbm;

// Library-owned plan of a batch: per-case parameters and state offsets, the
// device case table for the chosen tile height, the tuning choice and the
// captured graph.
struct lbm_batch {
    int ncases = 0;
    int dtype = 0;
    std::vector<lbm_params> params;
    std::vector<Layout> layouts;
    std::vector<size_t> base;
    size_t total = 0;
    int autotune = 0;
    bool tuned = false;
    bool wide = false;    // some case runs the two-node-window or local body (one node per thread)
    int ty = 8;
    int by = 4;           // thread rows per workgroup
    int grid = 0;
    int nitems = 0;
    void* d_cases = nullptr;
    int cus = 256;
    // two levels per launch (every case runs the plain Allen-Cahn step), on a
    // table of items of the tile shape `shape2`; two_level: what
    // lbm_batch_levels_per_launch reports (the size rule)
    bool two_level = false;
    lbm::Step2Shape shape2 = lbm::S2_NONE;
    bool whole = false;   // whole_batch
    void* d_cases2 = nullptr;
    int nitems2 = 0;
    // graph of `graph_steps` levels for (graph_state, graph_stream)
    hipGraphExec_t graph = nullptr;
    void* graph_state = nullptr;
    hipStream_t graph_stream = nullptr;
    int graph_steps = 0;
};

namespace {

int tiles_for(const lbm_params& p, int tw, int ty, int* ntx, int* nty) {
    *ntx = (p.nx + tw - 1) / tw;
    *nty = (p.ny + ty - 1) / ty;
    return *ntx * *nty;
}

// Case table of a batch for tiles of tw x ty nodes: parameters, state offsets and
// the first work item of every case; returns the number of work items.
template <typename T>
int fill_cases(const lbm_params* params, const Layout* layouts, const size_t* base, int ncases, int tw,
               int ty, BatchCase<T>* h) {
    int items = 0;
    for (int c = 0; c < ncases; c++) {
        BatchCase<T>& C = h[c];
        memset(&C, 0, sizeof(C));
        C.P = resolve<T>(&params[c], layouts[c]);
        C.base = base[c];
        C.off0 = layouts[c].off_buf[0];
        C.off1 = layouts[c].off_buf[1];
        C.off_stamp = layouts[c].off_stamp;
        C.item_begin = items;
        const lbm_params& q = params[c];
        C.body = q.phase_eq == LBM_CAHN_HILLIARD ? 1
                 : q.model == LBM_MODEL_CORRECTED ? 2
                 : q.grad_scheme == LBM_GRAD_LOCAL ? 3
                                                   : 0;
        const int tiles = tiles_for(params[c], tw, ty, &C.ntx, &C.nty);
        C.share = stamp_share((long long)layouts[c].nstamp, tiles);
        items += tiles;
    }
    return items;
}

template <typename T>
hipError_t upload_cases(lbm_batch* B, int ty) {
    std::vector<BatchCase<T>> h(B->ncases);
    B->nitems = fill_cases<T>(B->params.data(), B->layouts.data(), B->base.data(), B->ncases, TX, ty, h.data());
    if (!B->d_cases) {
        hipError_t e = hipMalloc(&B->d_cases, sizeof(BatchCase<T>) * B->ncases);
        if (e != hipSuccess) return e;
    }
    return hipMemcpy(B->d_cases, h.data(), sizeof(BatchCase<T>) * B->ncases, hipMemcpyHostToDevice);
}

// Nodes of a tile of the two-level launch.
void step2_tile_size(Step2Shape shape, int* tw, int* ty) {
    *tw = shape == S2_16x4 ? 16 : (shape == S2_64x8 || shape == S2_64x16 ? 64 : 32);
    *ty = shape == S2_16x4 || shape == S2_32x4 ? 4 : (shape == S2_32x16 || shape == S2_64x16 ? 16 : 8);
}

// The item table of the two-level launch.
template <typename T>
hipError_t upload_cases2(lbm_batch* B) {
    std::vector<BatchCase<T>> h(B->ncases);
    int tw, ty;
    step2_tile_size(B->shape2, &tw, &ty);
    B->nitems2 = fill_cases<T>(B->params.data(), B->layouts.data(), B->base.data(), B->ncases, tw, ty, h.data());
    // one entry per item: entry w is the case of item w (k_step2_batch, PER_ITEM)
    std::vector<BatchCase<T>> items((size_t)B->nitems2);
    for (int c = 0; c < B->ncases; c++) {
        const int end = c + 1 < B->ncases ? h[c + 1].item_begin : B->nitems2;
        for (int w = h[c].item_begin; w < end; w++) items[(size_t)w] = h[c];
    }
    hipError_t e = hipMalloc(&B->d_cases2, sizeof(BatchCase<T>) * items.size());
    if (e != hipSuccess) return e;
    return hipMemcpy(B->d_cases2, items.data(), sizeof(BatchCase<T>) * items.size(), hipMemcpyHostToDevice);
}

// One launch of the batch kernels over `nitems` work items of a device case
// table (grid 0: one workgroup per item).
struct BatchShape {
    int ty, by, grid, nitems, ncases;
    bool wide;
    size_t total;   // bytes of the batch state (store policy)
};

template <typename T, int TY, int NBY>
void batch_launch(const BatchShape& S, const void* d_cases, char* state, hipStream_t s) {
    const BatchCase<T>* cases = reinterpret_cast<const BatchCase<T>*>(d_cases);
    const bool nt = S.total > (size_t)LBM_NT_MIN_BYTES;
    if (S.grid > 0 && S.grid < S.nitems) {
        if (nt) k_step_batch<T, TY, NBY, true><<<S.grid, dim3(TX, NBY), 0, s>>>(cases, S.ncases, S.nitems, state);
        else k_step_batch<T, TY, NBY, false><<<S.grid, dim3(TX, NBY), 0, s>>>(cases, S.ncases, S.nitems, state);
    } else {
        if (nt) k_step_batch<T, TY, NBY, true, false><<<S.nitems, dim3(TX, NBY), 0, s>>>(cases, S.ncases, S.nitems, state);
        else k_step_batch<T, TY, NBY, false, false><<<S.nitems, dim3(TX, NBY), 0, s>>>(cases, S.ncases, S.nitems, state);
    }
}

template <typename T, int TY>
void batch_launch_wide(const BatchShape& S, const void* d_cases, char* state, hipStream_t s) {
    const BatchCase<T>* cases = reinterpret_cast<const BatchCase<T>*>(d_cases);
    const bool nt = S.total > (size_t)LBM_NT_MIN_BYTES;
    const dim3 blk(TX, TY);
    if (S.grid > 0 && S.grid < S.nitems) {
        if (nt) k_step_batch_wide<T, TY, true><<<S.grid, blk, 0, s>>>(cases, S.ncases, S.nitems, state);
        else k_step_batch_wide<T, TY, false><<<S.grid, blk, 0, s>>>(cases, S.ncases, S.nitems, state);
    } else {
        if (nt) k_step_batch_wide<T, TY, true, false><<<S.nitems, blk, 0, s>>>(cases, S.ncases, S.nitems, state);
        else k_step_batch_wide<T, TY, false, false><<<S.nitems, blk, 0, s>>>(cases, S.ncases, S.nitems, state);
    }
}

template <typename T>
void launch_batch_shape(const BatchShape& S, const void* d_cases, char* state, hipStream_t s) {
    constexpr int T16 = sizeof(T) == 8 ? 8 : 16;
    if (S.wide) {
        if (S.ty == 4) batch_launch_wide<T, 4>(S, d_cases, state, s);
        else batch_launch_wide<T, 8>(S, d_cases, state, s);
        return;
    }
    if (S.ty == 4) batch_launch<T, 4, 4>(S, d_cases, state, s);
    else if (S.ty == 8 || sizeof(T) == 8) {
        if (S.by == 8) batch_launch<T, 8, 8>(S, d_cases, state, s);
        else batch_launch<T, 8, 4>(S, d_cases, state, s);
    } else {
        if (S.by == 8) batch_launch<T, T16, 8>(S, d_cases, state, s);
        else batch_launch<T, T16, 4>(S, d_cases, state, s);
    }
}

template <typename T>
void launch_batch_once(lbm_batch* B, char* state, hipStream_t s) {
    const BatchShape S{B->ty, B->by, B->grid, B->nitems, B->ncases, B->wide, B->total};
    launch_batch_shape<T>(S, B->d_cases, state, s);
}

// One two-level launch over `nitems` items of a table for tiles of `shape`
// (PER_ITEM: one entry per item, as upload_cases2 writes it; else one per case).
// whole: whole_batch (step2_store; us per level, FP32,
// non-temporal or through against ordinary stores: 60 cases of 250 x 250 134 / 98, 28 of
// them 57 / 48, 10 of 500 x 300 38.7 / 32.5; FP64 13 of 250 x 250 50.2 / 47.3, 30 107.2 /
// 107.9).
template <typename T, bool PER_ITEM>
void launch_batch2(Step2Shape shape, int nitems, int ncases, const void* d_cases, size_t total, bool whole,
                   char* state, hipStream_t s) {
    const BatchCase<T>* cases = reinterpret_cast<const BatchCase<T>*>(d_cases);
    auto go = [&](auto kernel, int nt) LBM_CALLS_STUB { kernel<<<nitems, dim3(TX, nt / TX), 0, s>>>(cases, ncases, nitems, state); };
    const StoreKind kind = step2_store(total, whole);
    switch (shape) {   // the single-round shapes are far below the last-level cache
        case S2_16x4: go(k_step2_batch<T, 16, 4, 256, ST_THROUGH, PER_ITEM>, 256); break;
        case S2_32x4: go(k_step2_batch<T, 32, 4, 384, ST_THROUGH, PER_ITEM>, 384); break;
        case S2_32x8_WIDE: go(k_step2_batch<T, 32, 8, 576, ST_THROUGH, PER_ITEM>, 576); break;
        case S2_32x16: go(k_step2_batch<T, 32, 16, 512, ST_THROUGH, PER_ITEM>, 512); break;
        case S2_32x8:
            if (kind == ST_NT) go(k_step2_batch<T, 32, 8, 256, ST_NT, PER_ITEM>, 256);
            else if (kind == ST_PLAIN) go(k_step2_batch<T, 32, 8, 256, ST_PLAIN, PER_ITEM>, 256);
            else go(k_step2_batch<T, 32, 8, 256, ST_THROUGH, PER_ITEM>, 256);
            break;
        default:
            if constexpr (sizeof(T) == 4) {
                if (kind == ST_NT) go(k_step2_batch<T, 64, 8, 512, ST_NT, PER_ITEM>, 512);
                else if (kind == ST_PLAIN) go(k_step2_batch<T, 64, 8, 512, ST_PLAIN, PER_ITEM>, 512);
                else go(k_step2_batch<T, 64, 8, 512, ST_THROUGH, PER_ITEM>, 512);
            }
    }
}

// `n` levels of the batch: two-level launches, and a one-level launch for an odd n.
template <typename T>
void launch_batch_levels(lbm_batch* B, char* state, int64_t n, hipStream_t s) {
    if (B->shape2 != S2_NONE) {
        for (int64_t t = 0; t + 2 <= n; t += 2)
            launch_batch2<T, true>(B->shape2, B->nitems2, B->ncases, B->d_cases2, B->total, B->whole, state, s);
        if (n & 1) launch_batch_once<T>(B, state, s);
    } else {
        for (int64_t t = 0; t < n; t++) launch_batch_once<T>(B, state, s);
    }
}

void drop_graph(lbm_batch* B) {
    if (B->graph) (void)hipGraphExecDestroy(B->graph);
    B->graph = nullptr;
    B->graph_state = nullptr;
    B->graph_stream = nullptr;
    B->graph_steps = 0;
}

template <typename T>
int batch_step_t(lbm_batch* B, char* state, int64_t nsteps, hipStream_t s) {
    constexpr int K = 32;   // steps per captured graph
    hipError_t e;
    // not while the caller captures the stream: the launches go into its graph
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (s != nullptr && nsteps >= K) {
        e = hipStreamIsCapturing(s, &cs);
        if (e != hipSuccess) return hip_fail(e);
    }
    if (s != nullptr && nsteps >= K && cs == hipStreamCaptureStatusNone) {
        if (!B->graph || B->graph_state != state || B->graph_stream != s) {
            drop_graph(B);
            hipGraph_t g;
            e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal);
            if (e != hipSuccess) return hip_fail(e);
            launch_batch_levels<T>(B, state, K, s);
            e = hipStreamEndCapture(s, &g);
            if (e != hipSuccess) return hip_fail(e);
            e = hipGraphInstantiate(&B->graph, g, nullptr, nullptr, 0);
            (void)hipGraphDestroy(g);
            if (e != hipSuccess) return hip_fail(e);
            B->graph_state = state;
            B->graph_stream = s;
            B->graph_steps = K;
        }
        for (int64_t t = 0; t + K <= nsteps; t += K) {
            e = hipGraphLaunch(B->graph, s);
            if (e != hipSuccess) return hip_fail(e);
        }
        nsteps %= K;
    }
    launch_batch_levels<T>(B, state, nsteps, s);
    e = hipGetLastError();
    return e == hipSuccess ? LBM_OK : hip_fail(e);
}

template <typename T>
int batch_init_cases(lbm_batch* B, char* state, const void* const* phi0, const void* const* p0, hipStream_t s) {
    for (int c = 0; c < B->ncases; c++) {
        int rc = lbm_init(&B->params[c], state + B->base[c], phi0[c], nullptr, p0 ? p0[c] : nullptr, s);
        if (rc) return rc;
    }
    return LBM_OK;
}

// Time every candidate (tile height, persistent grid) on the batch itself and
// keep the fastest; the state is re-initialised afterwards by the caller.
template <typename T>
int autotune_t(lbm_batch* B, char* state, const void* const* phi0, const void* const* p0, hipStream_t s) {
    const int shapes[5][2] = {{4, 4}, {8, 4}, {8, 8}, {16, 4}, {16, 8}};   // (tile rows, thread rows)
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) return LBM_E_HIP;
    float best = 1e30f;
    int best_ty = 8, best_by = 4, best_grid = 0;
    for (const auto& sh : shapes) {
        const int ty = sh[0];
        if (ty == 16 && sizeof(T) == 8) continue;
        if (B->wide && (sh[1] != ty || ty > 8)) continue;   // the wide bodies: one node per thread
        B->ty = ty;
        B->by = sh[1];
        hipError_t e = upload_cases<T>(B, ty);
        if (e != hipSuccess) return hip_fail(e);
        const int grids[4] = {0, 2 * B->cus, 4 * B->cus, 8 * B->cus};
        for (int g : grids) {
            if (g > B->nitems) continue;
            B->grid = g;
            int rc = batch_init_cases<T>(B, state, phi0, p0, s);
            if (rc) return rc;
            for (int w = 0; w < 3; w++) launch_batch_once<T>(B, state, s);
            (void)hipEventRecord(e0, s);
            for (int w = 0; w < 10; w++) launch_batch_once<T>(B, state, s);
            (void)hipEventRecord(e1, s);
            e = hipEventSynchronize(e1);
            if (e != hipSuccess) return hip_fail(e);
            float ms = 0;
            (void)hipEventElapsedTime(&ms, e0, e1);
            if (ms < best) {
                best = ms;
                best_ty = ty;
                best_by = sh[1];
                best_grid = g;
            }
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    B->ty = best_ty;
    B->by = best_by;
    B->grid = best_grid;
    hipError_t e = upload_cases<T>(B, best_ty);
    if (e != hipSuccess) return hip_fail(e);
    B->tuned = true;
    return LBM_OK;
}

// Every case valid, one dtype, each case's state copy addressable with 32-bit offsets.
int validate_batch(const lbm_params* cases, int ncases) {
    if (ncases < 1) return LBM_E_SIZE;
    for (int c = 0; c < ncases; c++) {
        int rc = validate(&cases[c]);
        if (rc) return rc;
        if (cases[c].dtype != cases[0].dtype) return LBM_E_DTYPE;
        Layout L = layout_of(&cases[c]);
        if (L.buf_bytes >= (size_t(1) << 32)) return LBM_E_SIZE;   // 32-bit offsets within a case
    }
    return LBM_OK;
}

// Byte offset of every case's state in a batch state (each rounded up to 256 B);
// returns the total.
size_t batch_offsets(const lbm_params* cases, int ncases, Layout* layouts, size_t* base) {
    size_t off = 0;
    for (int c = 0; c < ncases; c++) {
        layouts[c] = layout_of(&cases[c]);
        base[c] = off;
        off += (layouts[c].total + 255) / 256 * 256;
    }
    return off;
}

bool wide_batch(const lbm_params* cases, int ncases) {
    bool w = false;
    for (int c = 0; c < ncases; c++)
        w = w || cases[c].phase_eq == LBM_CAHN_HILLIARD || cases[c].model == LBM_MODEL_CORRECTED ||
            cases[c].grad_scheme == LBM_GRAD_LOCAL;
    return w;
}

// Two levels per launch: every case runs the plain Allen-Cahn step (stencil
// gradients, present or original model); LBM_TWO_LEVEL=0, read when a plan is
// made (and at every call of the allocation-free step), turns it off.
bool two_level_cases(const lbm_params* cases, int ncases) {
    for (int c = 0; c < ncases; c++)
        if (cases[c].phase_eq != LBM_ALLEN_CAHN || cases[c].model == LBM_MODEL_CORRECTED ||
            cases[c].grad_scheme != LBM_GRAD_STENCIL)
            return false;
    const char* e = getenv("LBM_TWO_LEVEL");
    return !(e && e[0] == '0' && e[1] == 0);
}

// What lbm_batch_levels_per_launch reports of a batch that runs two levels per
// launch: whether it has at least 256 tiles of 64 x 8 nodes (LBM_TWO_LEVEL=1: whatever
// the size).
bool two_level_batch(const lbm_params* cases, int ncases) {
    long long tiles8 = 0;
    int ntx, nty;
    for (int c = 0; c < ncases; c++) tiles8 += tiles_for(cases[c], TX, 8, &ntx, &nty);
    const char* e = getenv("LBM_TWO_LEVEL");
    return (e && e[0] == '1' && e[1] == 0) || tiles8 >= 256;
}

// Whether a batch counts as one of whole cache lines in step2_store: most of its nodes do.
bool whole_batch(const lbm_params* cases, int ncases) {
    long long broken = 0, n = 0;
    for (int c = 0; c < ncases; c++) {
        const long long nodes = (long long)cases[c].nx * cases[c].ny;
        n += nodes;
        if (!whole_rows(cases[c].nx, cases[c].dtype == LBM_F64 ? 8 : 4)) broken += nodes;
    }
    return 2 * broken <= n;
}

// Tile shape of the two-level launch: the smallest that gives no CU two tiles, as
// for a single lattice (step2_shape), else 32 x 8 tiles, two (FP64) to four (FP32)
// workgroups of 256 threads to a CU; S2_NONE: one level per launch.  Measured on
// MI355X, us per level, spreading cases of 128 x 64 to 512 x 256 nodes, 32x8 /
// 64x8 / 32x16: FP32 3 cases 7.0 / 7.6 / 7.3, 8 cases 13.6 / 13.4 / 12.8, 20 cases
// 30.1 / 31.6 / 30.6, 64 cases (streamed) 100.6 / 102.2 / 111.7; FP64 3 cases 12.1 /
// 14.4 / 13.8, 8 cases 26.1 / 28.6 / 27.9, 64 cases 213.6 / 252.2 / 258.6.  32x8 beyond one
// round although 32x16 is 6% faster at 8 FP32 cases: at 3 and 20 it is 2-4% slower, at 64 11%.
Step2Shape batch_shape2(const lbm_params* cases, int ncases) {
    if (!two_level_cases(cases, ncases)) return S2_NONE;
    bool shares = true;
    auto fits = [&](int tw, int ty, long long limit) {
        long long tiles = 0;
        int ntx, nty;
        shares = true;
        for (int c = 0; c < ncases; c++) {
            tiles += tiles_for(cases[c], tw, ty, &ntx, &nty);
            shares = shares && stamp_share_ok(cases[c].nx, cases[c].ny, tw, ty);
        }
        return tiles <= limit && shares;
    };
    const long long any = 1LL << 62;
    if (fits(16, 4, 256)) return S2_16x4;
    if (fits(32, 4, 256)) return S2_32x4;
    if (fits(32, 8, 256)) return S2_32x8_WIDE;
    if (fits(32, 16, 256)) return S2_32x16;
    if (fits(32, 8, any)) return S2_32x8;
    return cases[0].dtype == LBM_F64 ? S2_NONE : S2_64x8;   // a case of one row
}

// ---- the batch step that allocates nothing (lbm_batch_step_noalloc) ----
// Its case table lives in `scratch`, a fixed array of the library in every
// GPU's memory.  In host code `scratch` only names the symbol: the kernels get
// the device address that hipGetSymbolAddress returns for the current device
// (looked up once per device, on the first call there).
constexpr size_t NOALLOC_CASE_BYTES =
    sizeof(BatchCase<double>) > sizeof(BatchCase<float>) ? sizeof(BatchCase<double>) : sizeof(BatchCase<float>);
static_assert(LBM_NOALLOC_MAX_CASES * NOALLOC_CASE_BYTES <= (size_t(256) << 10), "case table above 256 KB");
static __device__ __align__(256) unsigned char scratch[LBM_NOALLOC_MAX_CASES * NOALLOC_CASE_BYTES];

std::mutex g_scratch_mu;
std::vector<void*> g_scratch_dev;   // device address of `scratch`, per device ordinal

hipError_t scratch_address(void** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if ((size_t)dev >= g_scratch_dev.size()) g_scratch_dev.resize(dev + 1, nullptr);
    if (!g_scratch_dev[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_dev[dev] = p;
    }
    *out = g_scratch_dev[dev];
    return hipSuccess;
}

// A few cases of the table travel in the kernel arguments (copied at launch,
// so the host table may go away as soon as the launch returns) and are stored
// into the device table by one small workgroup.
template <typename T>
struct CaseChunk {
    static constexpr int N = (int)(3072 / sizeof(BatchCase<T>)) > 0 ? (int)(3072 / sizeof(BatchCase<T>)) : 1;
    BatchCase<T> c[N];
    int first, count;
};

template <typename T>
__global__ void k_put_cases(CaseChunk<T> chunk, BatchCase<T>* dst) {
    for (int i = threadIdx.x; i < chunk.count; i += blockDim.x) dst[chunk.first + i] = chunk.c[i];
}

template <typename T>
int batch_step_noalloc_t(const lbm_params* cases, int ncases, char* state, int64_t nsteps, hipStream_t s) {
    // host-side tables on the stack: at most LBM_NOALLOC_MAX_CASES cases
    static_assert(LBM_NOALLOC_MAX_CASES <= 256, "stack tables");
    Layout layouts[LBM_NOALLOC_MAX_CASES];
    size_t base[LBM_NOALLOC_MAX_CASES];
    const size_t total = batch_offsets(cases, ncases, layouts, base);
    void* dtab = nullptr;
    hipError_t e = scratch_address(&dtab);
    if (e != hipSuccess) return hip_fail(e);
    BatchCase<T>* table = reinterpret_cast<BatchCase<T>*>(dtab);
    auto put_cases = [&](int tw, int ty) {
        CaseChunk<T> chunk;
        int nitems = 0;
        for (int c0 = 0; c0 < ncases; c0 += CaseChunk<T>::N) {
            const int cnt = ncases - c0 < CaseChunk<T>::N ? ncases - c0 : CaseChunk<T>::N;
            memset(&chunk, 0, sizeof(chunk));
            const int items = fill_cases<T>(cases + c0, layouts + c0, base + c0, cnt, tw, ty, chunk.c);
            for (int i = 0; i < cnt; i++) chunk.c[i].item_begin += nitems;
            nitems += items;
            chunk.first = c0;
            chunk.count = cnt;
            k_put_cases<T><<<1, 64, 0, s>>>(chunk, table);
        }
        return nitems;
    };
    int64_t t = 0;
    const Step2Shape shape = batch_shape2(cases, ncases);
    if (shape != S2_NONE && nsteps >= 2) {
        int tw, ty;
        step2_tile_size(shape, &tw, &ty);
        const int nitems = put_cases(tw, ty);
        for (; t + 2 <= nsteps; t += 2) launch_batch2<T, false>(shape, nitems, ncases, table, total, whole_batch(cases, ncases), state, s);
    }
    if (t < nsteps) {
        // the untuned plan's shape: 8-row tiles, 64 x 4 threads (64 x 8 for the wide bodies), one
        // workgroup per item
        const int ty = 8, nitems = put_cases(TX, ty);
        const bool wide = wide_batch(cases, ncases);
        const BatchShape S{ty, wide ? ty : 4, 0, nitems, ncases, wide, total};
        for (; t < nsteps; t++) launch_batch_shape<T>(S, table, state, s);
    }
    e = hipGetLastError();
    return e == hipSuccess ? LBM_OK : hip_fail(e);
}

}  // namespace

extern "C" {

int lbm_batch_create(const lbm_params* cases, int32_t ncases, int32_t autotune, lbm_batch** out) {
    if (!cases || !out) return LBM_E_NULL;
    int rc = validate_batch(cases, ncases);
    if (rc) return rc;
    lbm_batch* B = new lbm_batch();
    B->ncases = ncases;
    B->dtype = cases[0].dtype;
    B->autotune = autotune;
    B->params.assign(cases, cases + ncases);
    B->wide = wide_batch(cases, ncases);
    B->layouts.resize(ncases);
    B->base.resize(ncases);
    B->total = batch_offsets(cases, ncases, B->layouts.data(), B->base.data());
    int dev = 0;
    if (hipGetDevice(&dev) == hipSuccess)
        (void)hipDeviceGetAttribute(&B->cus, hipDeviceAttributeMultiprocessorCount, dev);
    // default (untuned) choice: 8-row tiles, one workgroup per item (64 x 4 threads; the
    // wide bodies: 64 x 8, one node per thread)
    B->ty = 8;
    B->by = B->wide ? 8 : 4;
    B->grid = 0;
    // LBM_BATCH_SHAPE="ty,by,grid" fixes the one-level shape (no autotuning):
    // one of the tuner's candidates, grid 0 for one workgroup per item
    if (const char* env = getenv("LBM_BATCH_SHAPE")) {
        int ty = 0, by = 0, grid = -1;
        const bool ok = sscanf(env, "%d,%d,%d", &ty, &by, &grid) == 3 && grid >= 0 &&
                        ((ty == 4 && by == 4) || ((ty == 8 || ty == 16) && (by == 4 || by == 8))) &&
                        !(ty == 16 && B->dtype == LBM_F64) && !(B->wide && (by != ty || ty > 8));
        if (!ok) {
            delete B;
            return LBM_E_PARAM;
        }
        B->ty = ty;
        B->by = by;
        B->grid = grid;
        B->tuned = true;
    }
    hipError_t e = B->dtype == LBM_F32 ? upload_cases<float>(B, B->ty) : upload_cases<double>(B, B->ty);
    B->shape2 = batch_shape2(cases, ncases);
    B->two_level = B->shape2 != S2_NONE && two_level_batch(cases, ncases);
    B->whole = whole_batch(cases, ncases);
    if (e == hipSuccess && B->shape2 != S2_NONE) e = B->dtype == LBM_F32 ? upload_cases2<float>(B) : upload_cases2<double>(B);
    if (e != hipSuccess) {
        lbm_batch_destroy(B);
        return hip_fail(e);
    }
    *out = B;
    return LBM_OK;
}

int lbm_batch_state_size(const lbm_batch* B, size_t* nbytes) {
    if (!B || !nbytes) return LBM_E_NULL;
    *nbytes = B->total;
    return LBM_OK;
}

int lbm_batch_case_offset(const lbm_batch* B, int32_t c, size_t* offset) {
    if (!B || !offset) return LBM_E_NULL;
    if (c < 0 || c >= B->ncases) return LBM_E_SIZE;
    *offset = B->base[c];
    return LBM_OK;
}

int lbm_batch_init(lbm_batch* B, void* state, const void* const* phi0, const void* const* p0, void* stream) {
    if (!B || !state || !phi0) return LBM_E_NULL;
    if ((uintptr_t)state % 256) return LBM_E_SIZE;
    for (int c = 0; c < B->ncases; c++)
        if (!phi0[c]) return LBM_E_NULL;
    hipStream_t s = (hipStream_t)stream;
    drop_graph(B);
    if (B->autotune && !B->tuned) {
        int rc = B->dtype == LBM_F32 ? autotune_t<float>(B, (char*)state, phi0, p0, s)
                                     : autotune_t<double>(B, (char*)state, phi0, p0, s);
        if (rc) return rc;
    }
    return B->dtype == LBM_F32 ? batch_init_cases<float>(B, (char*)state, phi0, p0, s)
                               : batch_init_cases<double>(B, (char*)state, phi0, p0, s);
}

int lbm_batch_step(lbm_batch* B, void* state, int64_t nsteps, void* stream) {
    if (!B || !state) return LBM_E_NULL;
    if (nsteps < 0) return LBM_E_SIZE;
    hipStream_t s = (hipStream_t)stream;
    return B->dtype == LBM_F32 ? batch_step_t<float>(B, (char*)state, nsteps, s)
                               : batch_step_t<double>(B, (char*)state, nsteps, s);
}

int lbm_batch_step_noalloc(const lbm_params* cases, int32_t ncases, void* state, int64_t nsteps, void* stream) {
    if (!cases || !state) return LBM_E_NULL;
    if (ncases > LBM_NOALLOC_MAX_CASES) return LBM_E_SIZE;
    int rc = validate_batch(cases, ncases);
    if (rc) return rc;
    if (nsteps < 0) return LBM_E_SIZE;
    if ((uintptr_t)state % 256) return LBM_E_SIZE;
    if (nsteps == 0) return LBM_OK;
    hipStream_t s = (hipStream_t)stream;
    return cases[0].dtype == LBM_F32 ? batch_step_noalloc_t<float>(cases, ncases, (char*)state, nsteps, s)
                                     : batch_step_noalloc_t<double>(cases, ncases, (char*)state, nsteps, s);
}

int lbm_batch_tuning(const lbm_batch* B, int32_t* tile_rows, int32_t* thread_rows, int32_t* grid, int32_t* items) {
    if (!B) return LBM_E_NULL;
    if (tile_rows) *tile_rows = B->ty;
    if (thread_rows) *thread_rows = B->by;
    if (grid) *grid = B->grid > 0 ? B->grid : B->nitems;
    if (items) *items = B->nitems;
    return LBM_OK;
}

int lbm_batch_levels_per_launch(const lbm_batch* B, int32_t* levels) {
    if (!B || !levels) return LBM_E_NULL;
    *levels = B->two_level ? 2 : 1;
    return LBM_OK;
}

int lbm_batch_destroy(lbm_batch* B) {
    if (!B) return LBM_E_NULL;
    drop_graph(B);
    if (B->d_cases) (void)hipFree(B->d_cases);
    if (B->d_cases2) (void)hipFree(B->d_cases2);
    delete B;
    return LBM_OK;
}

}  // extern "C"

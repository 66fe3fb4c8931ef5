// Batched driver: many independent 2D models (a parameter sweep) solved
// increment by increment together.
//
// Every model is an ordinary solver handle carved from the batch workspace,
// so prologue, precision conversions, epilogue and field I/O are the
// single-model code.  What is shared is the PT iteration: a graph of n_check
// sweeps (a reduction reset, then persistent launches of up to K sweeps per
// precision and tile shape in use, the last sweep with the residual check)
// is captured on first use and replayed; each launch walks a device tile list of the
// models still iterating in that precision.  After a replay the host reads
// every model's residual in one copy, applies the single-model convergence
// logic per model, and retires or re-files the models whose state changed by
// rewriting the lists (their length is read by the kernels, so the graph
// stays valid).  The tile shape of each model size is chosen by an
// autotuner that times the whole batched sweep.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <new>
#include <utility>
#include <vector>

#include "ep.h"
#include "ep_handle.h"
#include "ep_internal.h"

using namespace ep;

struct ep_batch {
    int n;
    hipStream_t st;
    hipStream_t cs;                     // capture stream (graph recording only)
    bool fp32;
    int n_check;
    std::vector<ep_handle*> m;
    std::vector<long> cells;
    std::vector<int> shape;             // tile shape per model (sweeps in the batch precision)
    std::vector<int> shape64;           // FP32-field batches: tile shape of the FP64 finishing sweeps
    int ncu;
    double scale[2][BATCH_SHAPES], own_scale[2];   // [FP64, FP32] tuner's times over the modelled (1: not tuned)
    unsigned long long* red;            // n x RED_N
    double* cols;                       // n x 4
    SweepArgs<double>* tab64;           // 2 x n (parity of the ping-pong buffers)
    SweepArgs<float>* tab32;
    TileRef* list[2][ALL_SHAPES];     // [precision: 0 FP64, 1 FP32][shape]
    int* cnt;                           // 2 x ALL_SHAPES
    int grid[2][ALL_SHAPES];
    std::vector<SweepArgs<double>> h_tab64;
    std::vector<SweepArgs<float>> h_tab32;
    std::vector<TileRef> h_list[2][ALL_SHAPES];
    int h_cnt[2 * ALL_SHAPES];
    std::vector<unsigned long long> h_red;
    std::vector<double> h_cols;
    double cs32, cs64;                  // cell-sweeps of the current replay set-up
    // captured replays keyed by the set of non-empty tile lists (a precision
    // whose lists are empty is not launched at all)
    std::map<unsigned, std::pair<hipGraph_t, hipGraphExec_t>> graphs;
    bool timing;
    hipEvent_t ev0, ev1;
    double t_ms, t_cs32, t_cs64;
    long t_replays;
    char err[512];
};

namespace {

int berr(ep_batch* b, int code, const char* fmt, ...)
{
    if (b) {
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(b->err, sizeof(b->err), fmt, ap);
        va_end(ap);
    }
    return code;
}

#define BCHK(b, x)                                                                          \
    do {                                                                                    \
        hipError_t e_ = (x);                                                                \
        if (e_ != hipSuccess)                                                               \
            return berr((b), EP_EDEVICE, "%s failed: %s", #x, hipGetErrorString(e_));       \
    } while (0)

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

int resolved_check(const ep_params& p) { return p.n_check > 0 ? p.n_check : (p.ndim == 3 ? 10 : 100); }

int validate_batch(int n, const ep_params* p)
{
    if (n <= 0 || !p) return EP_EINVAL;
    const int nc = resolved_check(p[0]);
    for (int i = 0; i < n; ++i) {
        if (validate(&p[i]) != EP_OK) return EP_EINVAL;
        if (p[i].ndim != 2 || p[i].precision != p[0].precision) return EP_EINVAL;
        if (resolved_check(p[i]) != nc || nc % 2 != 0) return EP_EINVAL;
        if ((p[i].nx + 31) / 32 > 32767 || (p[i].ny + 3) / 4 > 32767) return EP_EINVAL;
    }
    return EP_OK;
}

// Layout of the batch workspace: the models, then the batch arrays.
struct BatchLayout {
    std::vector<size_t> model_off;
    size_t red, cols, tab64, tab32, lists[2][ALL_SHAPES], cnt, total;
};

BatchLayout layout(int n, const ep_params* p)
{
    BatchLayout L;
    size_t off = 0;
    for (int i = 0; i < n; ++i) {
        L.model_off.push_back(off);
        off = align256(off + carve(&p[i], nullptr, nullptr));
    }
    auto take = [&](size_t bytes) { size_t r = off; off = align256(off + bytes); return r; };
    L.red = take((size_t)n * RED_N * sizeof(unsigned long long));
    L.cols = take((size_t)n * 4 * sizeof(double));
    L.tab64 = take((size_t)3 * n * sizeof(SweepArgs<double>));
    L.tab32 = take((size_t)3 * n * sizeof(SweepArgs<float>));
    const bool fp32 = p[0].precision == EP_FP32_FIELDS;
    for (int q = 0; q < 2; ++q)
        for (int s = 0; s < ALL_SHAPES; ++s) {
            long c = 0;
            if (q == 0 || fp32)
                for (int i = 0; i < n; ++i) c += tiles2d(q == 1, s, p[i].nx, p[i].ny);
            L.lists[q][s] = take((size_t)std::max(c, 1L) * sizeof(TileRef));
        }
    L.cnt = take(2 * ALL_SHAPES * sizeof(int));
    L.total = off;
    return L;
}

// Model tables, 3 x n entries: [0] the first sweep of a replay (reads the
// current buffers; stores Lambda when a freeze was just decided), [1] and [2]
// the later sweeps reading the current / the other buffers.
void fill_tables(ep_batch* b)
{
    const int n = b->n;
    for (int i = 0; i < n; ++i) {
        ep_handle* h = b->m[i];
        const int lm_first = sweep_lam_mode(h, 0), lm_rest = sweep_lam_mode(h, 1);
        for (int slot = 0; slot < 3; ++slot) {
            const int par = slot == 2 ? 1 : 0;
            const int lm = slot == 0 ? lm_first : lm_rest;
            b->h_tab64[slot * n + i] = args64(h, false, h->cur64 ^ par);
            b->h_tab64[slot * n + i].lam_mode = lm;
            if (b->fp32) {
                b->h_tab32[slot * n + i] = args32(h, h->cur32 ^ par);
                b->h_tab32[slot * n + i].lam_mode = lm;
            }
        }
    }
}

int own_shape(const ep_batch* b, int i, int q) { return (q == 1 || !b->fp32) ? b->shape[i] : b->shape64[i]; }

// Tiles of the models that are active in precision q, with their own shapes
// and with each shape for all of them.
template <typename F>
void count_tiles(const ep_batch* b, int q, F active, long* own, long* tiles)
{
    std::fill(own, own + ALL_SHAPES, 0L);
    std::fill(tiles, tiles + ALL_SHAPES, 0L);
    for (int i = 0; i < b->n; ++i) {
        if (!active(i, q)) continue;
        const ep_handle* h = b->m[i];
        own[own_shape(b, i, q)] += tiles2d(q == 1, own_shape(b, i, q), h->nx, h->ny);
        for (int s = 0; s < ALL_SHAPES; ++s) tiles[s] += tiles2d(q == 1, s, h->nx, h->ny);
    }
}

// Tile lists of the running models (precision of each model's current
// sweeps), or of all models when all_models is set, in FP32 when all32 (the
// batch precision) else in FP64.  Running models of a precision take their
// (tuned) shapes, or together one of the others (tile2d_common; checks every
// two sweeps: tile2d_one_sweep).
void fill_lists(ep_batch* b, bool all_models, bool all32 = true)
{
    for (int q = 0; q < 2; ++q)
        for (int s = 0; s < ALL_SHAPES; ++s) b->h_list[q][s].clear();
    b->cs32 = b->cs64 = 0;
    auto active = [&](int i, int q) {
        if (all_models) return (b->fp32 && all32) == (q == 1);
        return b->m[i]->ctl.running && b->m[i]->ctl.use32 == (q == 1);
    };
    for (int q = 0; q < 2; ++q) {
        int common = -1;
        if (!all_models) {
            long own[ALL_SHAPES], tiles[ALL_SHAPES];
            count_tiles(b, q, active, own, tiles);
            common = b->n_check == 2       // one sweep per launch of a replay
                         ? tile2d_one_sweep(q == 1, tiles[ONE_SWEEP], tiles[ONE_SWEEP + 1], b->ncu)
                         : tile2d_common(q == 1, own, tiles, b->scale[q], b->own_scale[q], b->ncu);
        }
        for (int i = 0; i < b->n; ++i) {
            if (!active(i, q)) continue;
            ep_handle* h = b->m[i];
            const int s = common >= 0 ? common : own_shape(b, i, q);
            const int tx = kTiles2d[q][s].tx, ty = kTiles2d[q][s].ty;
            const int nbx = (h->nx + tx - 1) / tx, nby = (h->ny + ty - 1) / ty;
            auto& L = b->h_list[q][s];
            for (int by = 0; by < nby; ++by)
                for (int bx = 0; bx < nbx; ++bx) L.push_back(TileRef{i, bx, by});
            (q == 1 ? b->cs32 : b->cs64) += (double)b->cells[i] * b->n_check;
        }
    }
    for (int q = 0; q < 2; ++q)
        for (int s = 0; s < ALL_SHAPES; ++s) b->h_cnt[q * ALL_SHAPES + s] = (int)b->h_list[q][s].size();
}

int upload(ep_batch* b)
{
    const size_t n2 = 3 * (size_t)b->n;
    BCHK(b, hipMemcpyAsync(b->tab64, b->h_tab64.data(), n2 * sizeof(SweepArgs<double>), hipMemcpyHostToDevice, b->st));
    if (b->fp32)
        BCHK(b, hipMemcpyAsync(b->tab32, b->h_tab32.data(), n2 * sizeof(SweepArgs<float>), hipMemcpyHostToDevice,
                               b->st));
    for (int q = 0; q < 2; ++q)
        for (int s = 0; s < ALL_SHAPES; ++s)
            if (!b->h_list[q][s].empty())
                BCHK(b, hipMemcpyAsync(b->list[q][s], b->h_list[q][s].data(), b->h_list[q][s].size() * sizeof(TileRef),
                                       hipMemcpyHostToDevice, b->st));
    BCHK(b, hipMemcpyAsync(b->cnt, b->h_cnt, sizeof(b->h_cnt), hipMemcpyHostToDevice, b->st));
    // the host vectors may change right after this call
    BCHK(b, hipStreamSynchronize(b->st));
    return EP_OK;
}

// Bit q * ALL_SHAPES + shape for every non-empty tile list (q: 0 FP64, 1 FP32).
unsigned list_mask(const ep_batch* b)
{
    unsigned m = 0;
    for (int q = 0; q < 2; ++q)
        for (int sh = 0; sh < ALL_SHAPES; ++sh)
            if (b->h_cnt[q * ALL_SHAPES + sh] > 0) m |= 1u << (q * ALL_SHAPES + sh);
    return m;
}

// nsw sweeps of every tile in the lists selected by mask, in launches of at
// most K sweeps of the list's shape; the last one in CHECK mode when check is
// set.  With alternate, the launches advance the iteration (ping-pong), an
// even number of them, so that every model's current buffer stays in place;
// without, every launch reads the current buffers and writes the other ones
// (timing runs that leave the state unchanged).
void enqueue_sweeps(ep_batch* b, int nsw, bool check, bool reset, bool alternate, unsigned mask, hipStream_t s)
{
    if (reset) launch_reset_red_n(b->red, b->n, s);
    for (int q = 1; q >= 0; --q)
        for (int sh = 0; sh < ALL_SHAPES; ++sh) {
            if (!(mask >> (q * ALL_SHAPES + sh) & 1u)) continue;
            const int k = kTiles2d[q][sh].k;
            int n = (nsw + k - 1) / k;
            if (alternate && n % 2 != 0) ++n;
            Launch2d l{};
            l.shape = sh;
            l.grid = b->grid[q][sh];
            l.nbx = 1;
            for (int c = 0; c < n; ++c) {
                l.ns = nsw / n + (c < nsw % n ? 1 : 0);
                l.mode = (check && c == n - 1) ? MODE_CHECK : MODE_UPDATE;
                const int slot = !alternate ? 1 : c == 0 ? 0 : (c & 1) ? 2 : 1;
                const int* cnt = b->cnt + q * ALL_SHAPES + sh;
                if (q == 1) launch_sweep_batch_2d<float>(b->tab32 + slot * b->n, b->list[1][sh], cnt, l, s);
                else launch_sweep_batch_2d<double>(b->tab64 + slot * b->n, b->list[0][sh], cnt, l, s);
            }
        }
}

void drop_graphs(ep_batch* b)
{
    for (auto& g : b->graphs) {
        (void)hipGraphExecDestroy(g.second.second);
        (void)hipGraphDestroy(g.second.first);
    }
    b->graphs.clear();
}

// The replay of n_check sweeps for the lists in mask (captured on first use).
int replay_for(ep_batch* b, unsigned mask, hipGraphExec_t* out)
{
    auto it = b->graphs.find(mask);
    if (it != b->graphs.end()) {
        *out = it->second.second;
        return EP_OK;
    }
    BCHK(b, hipStreamBeginCapture(b->cs, hipStreamCaptureModeRelaxed));
    enqueue_sweeps(b, b->n_check, true, true, true, mask, b->cs);
    hipGraph_t g = nullptr;
    BCHK(b, hipStreamEndCapture(b->cs, &g));
    hipGraphExec_t ex = nullptr;
    hipError_t e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
    if (e != hipSuccess) {
        (void)hipGraphDestroy(g);
        return berr(b, EP_EDEVICE, "hipGraphInstantiate failed: %s", hipGetErrorString(e));
    }
    b->graphs[mask] = {g, ex};
    *out = ex;
    return EP_OK;
}

int read_all(ep_batch* b, bool cols)
{
    BCHK(b, hipMemcpyAsync(b->h_red.data(), b->red, b->h_red.size() * sizeof(unsigned long long),
                           hipMemcpyDeviceToHost, b->st));
    if (cols)
        BCHK(b, hipMemcpyAsync(b->h_cols.data(), b->cols, b->h_cols.size() * sizeof(double), hipMemcpyDeviceToHost,
                               b->st));
    BCHK(b, hipStreamSynchronize(b->st));
    BCHK(b, hipGetLastError());
    return EP_OK;
}

void model_red(const ep_batch* b, int i, double out[RED_N]) { decode_red(&b->h_red[(size_t)i * RED_N], out); }

void destroy_batch(ep_batch* b)
{
    drop_graphs(b);
    for (ep_handle* h : b->m) handle_free(h);
    if (b->cs) (void)hipStreamDestroy(b->cs);
    if (b->ev0) (void)hipEventDestroy(b->ev0);
    if (b->ev1) (void)hipEventDestroy(b->ev1);
    delete b;
}

}  // namespace

// All models' sweeps with one shape (for tests, which so reach every one).
int ep::batch_use_shape(ep_batch* b, int shape)
{
    if (!b || shape < 0 || shape >= BATCH_SHAPES) return EP_EINVAL;
    std::fill(b->shape.begin(), b->shape.end(), shape);
    std::fill(b->shape64.begin(), b->shape64.end(), shape);
    b->own_scale[0] = b->own_scale[1] = 0.0;
    drop_graphs(b);
    return EP_OK;
}

int ep::tuned_sweeps(int reps) { return (int)std::min((reps + 5L) / 6 * 6, 2147483646L); }

// =========================================================================
extern "C" {

int ep_batch_workspace_size(int n, const ep_params* p, size_t* bytes)
{
    if (!bytes || validate_batch(n, p) != EP_OK) return EP_EINVAL;
    *bytes = layout(n, p).total;
    return EP_OK;
}

int ep_batch_init(int n, const ep_params* p, const double* const* cohesion, void* d_workspace, size_t ws_bytes,
                  void* stream, ep_batch** out)
{
    if (!out) return EP_EINVAL;
    *out = nullptr;
    if (validate_batch(n, p) != EP_OK) return EP_EINVAL;
    const BatchLayout L = layout(n, p);
    if (!d_workspace || ws_bytes < L.total) return EP_ENOMEM;
    if (((uintptr_t)d_workspace & 255) != 0) return EP_EINVAL;
    ep_batch* b = new (std::nothrow) ep_batch();
    if (!b) return EP_ENOMEM;
    char* base = (char*)d_workspace;
    b->n = n;
    b->st = (hipStream_t)stream;
    b->fp32 = p[0].precision == EP_FP32_FIELDS;
    b->n_check = resolved_check(p[0]);
    auto fail = [&](int code) { destroy_batch(b); return code; };
    if (hipStreamCreateWithFlags(&b->cs, hipStreamNonBlocking) != hipSuccess) return fail(EP_EDEVICE);
    if (hipEventCreate(&b->ev0) != hipSuccess || hipEventCreate(&b->ev1) != hipSuccess) return fail(EP_EDEVICE);
    b->red = (unsigned long long*)(base + L.red);
    b->cols = (double*)(base + L.cols);
    b->tab64 = (SweepArgs<double>*)(base + L.tab64);
    b->tab32 = (SweepArgs<float>*)(base + L.tab32);
    for (int q = 0; q < 2; ++q)
        for (int s = 0; s < ALL_SHAPES; ++s) b->list[q][s] = (TileRef*)(base + L.lists[q][s]);
    b->cnt = (int*)(base + L.cnt);
    if (hipMemsetAsync(base + L.red, 0, L.total - L.red, b->st) != hipSuccess) return fail(EP_EDEVICE);
    for (int i = 0; i < n; ++i) {
        ep_handle* h = nullptr;
        int rc = handle_create(&p[i], cohesion ? cohesion[i] : nullptr, base + L.model_off[i], b->st, &h);
        if (rc) return fail(rc);
        h->in_batch = true;
        h->red = b->red + (size_t)i * RED_N;
        h->cols64 = b->cols + (size_t)i * 4;
        if ((rc = upload_tables(h))) return fail(rc);
        b->m.push_back(h);
        b->cells.push_back((long)p[i].nx * p[i].ny);
        b->shape.push_back(0);
        b->shape64.push_back(5);        // 24 x 24 cells, K = 2: 20 us per FP64 sweep of 777 x 1010 cells, shape 0 22
    }
    int ncu = 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, 0) != hipSuccess || ncu <= 0) ncu = 256;
    b->ncu = ncu;
    for (int q = 0; q < 2; ++q) {
        std::fill(b->scale[q], b->scale[q] + BATCH_SHAPES, 1.0);
        b->own_scale[q] = 1.0;
    }
    for (int s = 0; s < ALL_SHAPES; ++s) {
        b->grid[0][s] = ncu * std::min(8, batch_blocks_per_cu<double>(s));
        b->grid[1][s] = ncu * std::min(8, batch_blocks_per_cu<float>(s));
    }
    b->h_tab64.resize(3 * (size_t)n);
    b->h_tab32.resize(3 * (size_t)n);
    b->h_red.assign((size_t)n * RED_N, 0ull);
    b->h_cols.assign((size_t)n * 4, 0.0);
    if (hipGetLastError() != hipSuccess) return fail(EP_EDEVICE);
    *out = b;
    return EP_OK;
}

void ep_batch_destroy(ep_batch* b)
{
    if (b) destroy_batch(b);
}

const char* ep_batch_last_error(const ep_batch* b) { return b ? b->err : "no batch"; }

ep_handle* ep_batch_model(ep_batch* b, int i)
{
    if (!b || i < 0 || i >= b->n) return nullptr;
    return b->m[i];
}

int ep_batch_tile_shape(const ep_batch* b, int i, int* tx, int* ty)
{
    if (!b || i < 0 || i >= b->n) return EP_EINVAL;
    if (tx) *tx = kTiles2d[b->fp32][b->shape[i]].pass_x;
    if (ty) *ty = kTiles2d[b->fp32][b->shape[i]].pass_y;
    return EP_OK;
}

int ep_batch_tune(ep_batch* b, int reps)
{
    if (!b || reps <= 0) return EP_EINVAL;
    // the timed sweeps read the current buffers and write the other ones, so
    // the state is unchanged
    for (ep_handle* h : b->m) {
        if (b->fp32) ensure_it32(h);
        else ensure_it64(h);
    }
    fill_tables(b);
    // models grouped by size: one tile shape per size class
    std::map<std::pair<int, int>, std::vector<int>> classes;
    for (int i = 0; i < b->n; ++i) classes[{b->m[i]->nx, b->m[i]->ny}].push_back(i);
    // coordinate descent over the size classes for one precision's shapes
    auto descend = [&](std::vector<int>& shape, bool all32) -> int {
        auto time_config = [&](double* ms) -> int {
            fill_lists(b, true, all32);
            int rc = upload(b);
            if (rc) return rc;
            const unsigned mask = list_mask(b);
            const int n = tuned_sweeps(reps);
            enqueue_sweeps(b, 1, false, false, false, mask, b->st);    // warm-up
            BCHK(b, hipEventRecord(b->ev0, b->st));
            enqueue_sweeps(b, n, false, false, false, mask, b->st);
            BCHK(b, hipEventRecord(b->ev1, b->st));
            BCHK(b, hipEventSynchronize(b->ev1));
            BCHK(b, hipGetLastError());
            float t = 0.f;
            BCHK(b, hipEventElapsedTime(&t, b->ev0, b->ev1));
            *ms = t / n;
            return EP_OK;
        };
        double best = 0;
        int rc = time_config(&best);
        if (rc) return rc;
        // (one size class: a second pass would time the same again)
        for (int pass = 0; pass < (classes.size() > 1 ? 2 : 1); ++pass) {
            for (auto& cl : classes) {
                const int keep = shape[cl.second[0]];
                int best_s = keep;
                for (int s = 0; s < TUNED_SHAPES; ++s) {
                    if (s == keep) continue;
                    for (int i : cl.second) shape[i] = s;
                    double t;
                    if ((rc = time_config(&t))) return rc;
                    if (t < best) {
                        best = t;
                        best_s = s;
                    }
                }
                for (int i : cl.second) shape[i] = best_s;
            }
        }
        // the tuned shapes and those for few tiles against their modelled times
        const int q = b->fp32 && all32 ? 1 : 0;
        const auto all = [](int, int) { return true; };
        long own[ALL_SHAPES], tiles[ALL_SHAPES];
        count_tiles(b, q, all, own, tiles);
        double model = 0;
        for (int s = 0; s < BATCH_SHAPES; ++s)
            if (own[s] > 0) model += tile2d_cost(q == 1, s, own[s], b->ncu);
        b->own_scale[q] = best * 1e3 / model;
        const std::vector<int> tuned = shape;
        for (int s = TUNED_SHAPES; s < BATCH_SHAPES && rc == EP_OK; ++s) {
            std::fill(shape.begin(), shape.end(), s);
            double t = 0;
            rc = time_config(&t);
            b->scale[q][s] = t * 1e3 / tile2d_cost(q == 1, s, tiles[s], b->ncu);
        }
        shape = tuned;
        return rc;
    };
    int rc = descend(b->shape, true);
    if (rc) return rc;
    if (b->fp32) {
        // the FP64 finishing sweeps have their own best shapes (8-byte LDS
        // planes limit the workgroups per CU differently)
        for (ep_handle* h : b->m) ensure_it64(h);
        fill_tables(b);
        if ((rc = descend(b->shape64, false))) return rc;
    }
    drop_graphs(b);                     // recaptured for the new shapes when used
    return EP_OK;
}

int ep_batch_enable_timing(ep_batch* b, int on)
{
    if (!b) return EP_EINVAL;
    b->timing = on != 0;
    b->t_ms = b->t_cs32 = b->t_cs64 = 0;
    b->t_replays = 0;
    return EP_OK;
}

int ep_batch_timing(const ep_batch* b, double* ms, double* cell_sweeps32, double* cell_sweeps64, long* replays)
{
    if (!b) return EP_EINVAL;
    if (ms) *ms = b->t_ms;
    if (cell_sweeps32) *cell_sweeps32 = b->t_cs32;
    if (cell_sweeps64) *cell_sweeps64 = b->t_cs64;
    if (replays) *replays = b->t_replays;
    return EP_OK;
}

int ep_batch_load_step(ep_batch* b, ep_step_stats* st)
{
    if (!b || !st) return EP_EINVAL;
    int rc;
    // prologue of every model, then one read of all reference residuals
    for (int i = 0; i < b->n; ++i) step_begin(b->m[i], &st[i]);
    if ((rc = read_all(b, false))) return rc;
    for (int i = 0; i < b->n; ++i) {
        double red[RED_N];
        model_red(b, i, red);
        step_start(b->m[i], red);       // a failed start leaves the model not running
    }
    auto any_running = [&]() {
        for (ep_handle* h : b->m)
            if (h->ctl.running) return true;
        return false;
    };
    bool dirty = true;
    while (any_running()) {
        if (dirty) {
            fill_tables(b);
            fill_lists(b, false);
            if ((rc = upload(b))) return rc;
            dirty = false;
        }
        if (b->timing) BCHK(b, hipEventRecord(b->ev0, b->st));
        hipGraphExec_t ex = nullptr;
        if ((rc = replay_for(b, list_mask(b), &ex))) return rc;
        BCHK(b, hipGraphLaunch(ex, b->st));
        if (b->timing) BCHK(b, hipEventRecord(b->ev1, b->st));
        if ((rc = read_all(b, false))) return rc;
        if (b->timing) {
            float t = 0.f;
            if (hipEventElapsedTime(&t, b->ev0, b->ev1) == hipSuccess) {
                b->t_ms += t;
                b->t_cs32 += b->cs32;
                b->t_cs64 += b->cs64;
                ++b->t_replays;
            }
        }
        for (int i = 0; i < b->n; ++i) {
            ep_handle* h = b->m[i];
            if (!h->ctl.running) continue;
            // an even number of sweeps leaves every model's current buffer in place
            const bool was32 = h->ctl.use32;
            if (was32) h->it64_valid = false;
            else h->it32_valid = false;
            if (h->freeze == 1) {           // the replay's first sweep stored Lambda
                h->freeze = 2;
                h->lam_in32 = was32;
                dirty = true;
            }
            double red[RED_N];
            model_red(b, i, red);
            const int freeze_before = h->freeze;
            const bool late_before = h->late;
            const bool cont = step_check(h, red, b->n_check);
            if (!cont || h->ctl.use32 != was32 || h->freeze != freeze_before || h->late != late_before) dirty = true;
        }
        // certificates of the models whose check met the tolerance (the
        // single-model evaluation on each model's own reduction slots)
        bool any_cert = false;
        for (ep_handle* h : b->m)
            if (h->ctl.running && h->ctl.cert_pending) {
                step_certify_launch(h);
                any_cert = true;
            }
        if (any_cert) {
            if ((rc = read_all(b, false))) return rc;
            for (int i = 0; i < b->n; ++i) {
                ep_handle* h = b->m[i];
                if (!h->ctl.running || !h->ctl.cert_pending) continue;
                double red[RED_N];
                model_red(b, i, red);
                const int freeze_before = h->freeze;
                const bool late_before = h->late;
                if (!step_certify(h, red) || h->freeze != freeze_before || h->late != late_before) dirty = true;
            }
        }
    }
    int worst = EP_OK;
    for (int i = 0; i < b->n; ++i) {
        const int s = step_finish(b->m[i]);
        if (s != EP_OK && worst == EP_OK) worst = s;
    }
    if ((rc = read_all(b, true))) return rc;
    for (int i = 0; i < b->n; ++i) {
        if (st[i].status != EP_OK) continue;
        double red[RED_N];
        model_red(b, i, red);
        step_report(b->m[i], red, &b->h_cols[(size_t)i * 4]);
    }
    return worst;
}

}  // extern "C"

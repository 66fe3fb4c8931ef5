// 2D PT sweeps: persistent launches that walk the tiles of one model or of
// many independent models of different sizes and parameters, up to K sweeps
// per launch (ep_tile2d.h).
//
// A model table holds one SweepArgs per model (per parity of the ping-pong
// buffers); a tile list holds (model, tile x, tile y) for every tile of the
// models that are still iterating in this precision and tile shape (a single
// model needs no list).  The grid is sized to the resident capacity of the
// device and each workgroup walks the list with a grid stride; models that
// converged are simply absent from the list, so their tiles cost nothing.
// The list length is read from device memory, which lets a captured graph of
// sweeps stay valid while the host retires models between replays.
#include <cmath>

#include "ep_device.h"
#include "ep_tile2d.h"

namespace ep {

namespace {

template <typename R, int TX, int TY, int K, int MODE, int NT, int E, bool HG>
__global__ __attribute__((amdgpu_flat_work_group_size(NT, NT), amdgpu_waves_per_eu(E)))
void k_batch_2d(const SweepArgs<R>* __restrict__ table, const TileRef* __restrict__ list, const int* __restrict__ count,
                int tiles, int nbx, int ns)
{
    const int n = list ? *count : tiles;
    // logical workgroup ids contiguous per XCD: consecutive tiles of a model
    // (neighbours, sharing halo lines) run on the same L2
    const int g = xcd_remap(blockIdx.x, gridDim.x);
    for (int t = g; t < n; t += gridDim.x) {
        if (t != g) __syncthreads();        // LDS of the previous tile is still being read
        TileRef r{0, 0, 0};
        int bx = t % nbx, by = t / nbx;
        if (list) {
            r = list[t];
            bx = r.bx;
            by = r.by;
        }
        sweep_tile_2d<R, TX, TY, K, MODE, NT, HG>(table[r.model], bx, by, ns);
    }
}

// Tile shapes of each precision: index, TX, TY, K, threads, waves per SIMD to
// fit in registers, whether single models choose it (and it has a form with a
// per-cell G), and what a launch costs, in us: alone with at most one
// workgroup per CU (t1), else t0 + t2 per workgroup on a CU; measured on 18
// grids from 31^2 to 2047^2 (not for the shapes of one sweep:
// tile2d_one_sweep).  The first six are the tuner's, named by the points that
// one pass of the workgroup's threads covers (64 x 8, 64 x 4, 32 x 8, 128 x 4,
// 64 x 16, 32 x 16), the last two those of launches of one sweep.
#define EP_TILES_32(X)                                                                                                 \
    X(0, 52, 20, 3, 512, 6, false, 15.7, 5.0, 7.0) X(1, 56, 8, 2, 256, 5, true, 10.0, 2.0, 2.6)                        \
    X(2, 24, 24, 2, 256, 5, false, 10.0, 2.0, 3.5) X(3, 120, 8, 2, 512, 5, false, 11.0, 2.0, 6.4)                      \
    X(4, 52, 20, 3, 1024, 8, true, 11.2, 3.0, 6.9) X(5, 24, 24, 2, 512, 8, true, 8.0, 1.5, 3.2)                        \
    X(6, 12, 12, 5, 1024, 8, true, 9.6, 1.7, 5.9) X(7, 16, 16, 4, 1024, 8, true, 8.5, 1.6, 4.9)                        \
    X(8, 20, 20, 3, 1024, 8, true, 7.4, 2.3, 3.9) X(9, 32, 32, 4, 768, 6, true, 17.0, 2.5, 10.2)                       \
    X(10, 60, 12, 1, 512, 6, true, 0, 0, 0) X(11, 60, 28, 1, 1024, 8, true, 0, 0, 0)
#define EP_TILES_64(X)                                                                                                 \
    X(0, 56, 8, 2, 512, 4, true, 10.5, 4.5, 5.7) X(1, 56, 8, 2, 256, 3, false, 13.0, 7.0, 5.6)                         \
    X(2, 24, 24, 2, 256, 3, true, 15.0, 8.0, 6.0) X(3, 120, 8, 2, 512, 2, true, 16.0, 3.0, 13.0)                       \
    X(4, 52, 20, 3, 1024, 4, true, 20.5, 1.0, 20.5) X(5, 24, 24, 2, 512, 4, true, 11.0, 4.5, 6.2)                      \
    X(6, 12, 12, 5, 1024, 4, true, 15.8, 1.8, 14.0) X(7, 16, 16, 4, 1024, 4, true, 14.0, 2.0, 12.3)                    \
    X(8, 20, 20, 3, 1024, 4, true, 12.0, 1.5, 10.7) X(9, 20, 20, 3, 512, 4, true, 13.7, 5.0, 7.6)                      \
    X(10, 60, 12, 1, 512, 4, true, 0, 0, 0) X(11, 60, 28, 1, 1024, 4, true, 0, 0, 0)

template <typename R, int TX, int TY, int K, int NT, int E, bool SINGLE>
void run(const SweepArgs<R>* table, const TileRef* list, const int* count, const Launch2d& l, hipStream_t s)
{
    const int grid = l.grid > 0 ? l.grid : 1;
    if constexpr (K == 1 && sizeof(R) == 8) {
        if (l.mode == MODE_PHYS) {
            // physical evaluations: single FP64 models
            if (l.has_g)
                k_batch_2d<R, TX, TY, K, MODE_PHYS, NT, E, true><<<grid, NT, 0, s>>>(table, list, count, l.tiles, l.nbx, 1);
            else
                k_batch_2d<R, TX, TY, K, MODE_PHYS, NT, E, false><<<grid, NT, 0, s>>>(table, list, count, l.tiles, l.nbx, 1);
            return;
        }
    }
    if constexpr (SINGLE) {
        if (l.has_g) {
            if (l.mode == MODE_CHECK)
                k_batch_2d<R, TX, TY, K, MODE_CHECK, NT, E, true><<<grid, NT, 0, s>>>(table, list, count, l.tiles, l.nbx, l.ns);
            else
                k_batch_2d<R, TX, TY, K, MODE_UPDATE, NT, E, true><<<grid, NT, 0, s>>>(table, list, count, l.tiles, l.nbx, l.ns);
            return;
        }
    }
    if (l.mode == MODE_CHECK)
        k_batch_2d<R, TX, TY, K, MODE_CHECK, NT, E, false><<<grid, NT, 0, s>>>(table, list, count, l.tiles, l.nbx, l.ns);
    else
        k_batch_2d<R, TX, TY, K, MODE_UPDATE, NT, E, false><<<grid, NT, 0, s>>>(table, list, count, l.tiles, l.nbx, l.ns);
}

template <typename R, int TX, int TY, int K, int NT, int E>
int occupancy()
{
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_batch_2d<R, TX, TY, K, MODE_CHECK, NT, E, false>, NT, 0) !=
        hipSuccess)
        return 1;
    return n > 0 ? n : 1;
}

}  // namespace

#define X(i, TX, TY, K, NT, E, SINGLE, t1, t0, t2) {TX, TY, K, TX + 4 * K, NT / (TX + 4 * K), SINGLE, t1, t0, t2},
const Tile2d kTiles2d[2][ALL_SHAPES] = {{EP_TILES_64(X)}, {EP_TILES_32(X)}};
#undef X
#define X(i, ...) i,
constexpr bool in_order(const int (&at)[ALL_SHAPES])
{
    for (int s = 0; s < ALL_SHAPES; ++s)
        if (at[s] != s) return false;
    return true;
}
static_assert(in_order({EP_TILES_64(X)}) && in_order({EP_TILES_32(X)}), "the indexes are the places in kTiles2d");
#undef X

double tile2d_cost(bool fp32, int shape, long tiles, int cus)
{
    const Tile2d& t = kTiles2d[fp32][shape];
    const double m = std::ceil((double)tiles / cus);
    return std::fmax(t.t1, t.t0 + t.t2 * m) / t.k;
}

// The shape of least modelled time for a model of nx x ny cells, of those that
// are marked for single models (the others only ever gain 2 % on strips of
// less than 9 cells).  A launch of
// K sweeps is worth more redundant points the fewer workgroups a grid fills:
// 12 x 12 tiles with K = 5 up to 16 tiles a side (63^2 FP32 1.9 us per sweep,
// one sweep per launch of 64 x 16 tiles 5; FP64 3.1 against 7.5), then 16 x 16,
// 20 x 20 and the large tiles (1023^2 FP32 11 against 19 us, FP64 25 against
// 43).
int tile2d_choice(bool fp32, int nx, int ny, int cus)
{
    int best = 0;
    double t_best = INFINITY;
    for (int s = 0; s < BATCH_SHAPES; ++s) {
        const double t = tile2d_cost(fp32, s, tiles2d(fp32, s, nx, ny), cus);
        if (kTiles2d[fp32][s].single && t < t_best) {
            t_best = t;
            best = s;
        }
    }
    return best;
}

// Where few models of a batch are left, the shapes for few tiles take less
// time.  Once the tuner has run, both sides are scaled by what it measured
// with all models, so that a shape it chose gives way only to one that its
// own times favour.
int tile2d_common(bool fp32, const long* own, const long* tiles, const double* scale, double own_scale, int cus)
{
    double best = 0;
    for (int s = 0; s < BATCH_SHAPES; ++s)
        if (own[s] > 0) best += tile2d_cost(fp32, s, own[s], cus);
    best *= own_scale;
    int common = -1;
    for (int s = TUNED_SHAPES; s < BATCH_SHAPES; ++s) {
        const double t = scale[s] * tile2d_cost(fp32, s, tiles[s], cus);
        if (tiles[s] > 0 && t < best) {
            best = t;
            common = s;
        }
    }
    return common;
}

// A launch of one sweep has no use for the wide halo of the shapes above
// (1023^2 FP32: 47 us by events where 60 x 28 tiles take 38; 2047^2 FP64 with a
// per-cell G 344 and 208): tiles with a halo of two points.  60 x 12 (512
// threads) unless 60 x 28 (1024) spare the CUs a second workgroup (511^2 FP64
// 27.5 us, 60 x 12 32.5), or in FP32, where two and three of them fit a CU at a
// time, rounds: 17 us one of 60 x 28, 12 us one of 60 x 12 (1500^2: 62 and 75
// us; 2047^2: 132 and 111).  In FP64 the larger tiles never gain there (1023^2:
// 66 and 62.5 us).
int tile2d_one_sweep(bool fp32, long t12, long t28, int cus)
{
    auto rounds = [&](long tiles, long per_cu) { return (tiles + per_cu * cus - 1) / (per_cu * cus); };
    const bool large = (t28 <= cus && t12 > cus) || (fp32 && 17 * rounds(t28, 2) < 12 * rounds(t12, 3));
    return ONE_SWEEP + large;
}

template <typename R>
void launch_sweep_batch_2d(const SweepArgs<R>* table, const TileRef* list, const int* count, const Launch2d& l,
                           hipStream_t s)
{
#define X(i, TX, TY, K, NT, E, SINGLE, ...) case i: run<R, TX, TY, K, NT, E, SINGLE>(table, list, count, l, s); break;
    if constexpr (sizeof(R) == 8) {
        switch (l.shape) { EP_TILES_64(X) }
    } else {
        switch (l.shape) { EP_TILES_32(X) }
    }
#undef X
}

template <typename R>
int batch_blocks_per_cu(int shape)
{
#define X(i, TX, TY, K, NT, E, ...) case i: return occupancy<R, TX, TY, K, NT, E>();
    if constexpr (sizeof(R) == 8) {
        switch (shape) { EP_TILES_64(X) }
    } else {
        switch (shape) { EP_TILES_32(X) }
    }
#undef X
    return 1;
}

template void launch_sweep_batch_2d<float>(const SweepArgs<float>*, const TileRef*, const int*, const Launch2d&,
                                           hipStream_t);
template void launch_sweep_batch_2d<double>(const SweepArgs<double>*, const TileRef*, const int*, const Launch2d&,
                                            hipStream_t);
template int batch_blocks_per_cu<float>(int);
template int batch_blocks_per_cu<double>(int);

}  // namespace ep

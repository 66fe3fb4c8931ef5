// Learned warm start: the encoder-decoder network of ep_net.h, its forward
// and backward passes and Adam, all in HIP kernels on the gfx950 matrix
// cores (bfloat16 operands, FP32 accumulation).
//
// Tensors of the network are channel-last over the network volume with a
// one-voxel zero border (the padding of the 3x3x3 'same' convolutions):
// voxel (z, y, x) of a D x H x W level is stored at ((z+1)(H+2) + y+1)(W+2)
// + x+1, times the channel count.  Borders are zeroed once and never written.
//
// Convolution = implicit GEMM over 27 taps x input channels: output channels
// are the rows and voxels the columns of v_mfma_f32_16x16x32_bf16 (the
// 16-channel input layer uses the K = 16 form), so that a lane of the result
// holds consecutive channels of one voxel.  The voxels come from an LDS copy
// of the block's input with halo, the weights in fragment order from memory;
// the epilogues (bias, ReLU, skip sum, ReLU mask of the backward pass) are
// part of the kernel, and a layer behind a repetition reads its parent level.
// The gradient with respect to the input is the same kernel on the output
// gradient with the weights transposed (input <-> output channels) and the
// taps mirrored.  The weight gradient reduces over voxels: a workgroup takes a
// chunk of voxels, stages the output gradient and the input around it once for
// all 27 taps, accumulates 16 x 16 blocks with the voxels as the MFMA reduction
// dimension and writes partial sums, which are added up in a fixed order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <random>
#include <type_traits>
#include <vector>

#include "ep.h"
#include "ep_handle.h"
#include "ep_internal.h"
#include "ep_net.h"

using namespace ep;

namespace {

typedef unsigned short bf16_t;
typedef __attribute__((ext_vector_type(4))) short s4;
typedef __attribute__((ext_vector_type(8))) __bf16 b8;
typedef __attribute__((ext_vector_type(4))) float f4;
// 8 bfloat16 values (16 bytes) as the operand of a K = 32 MFMA

constexpr int NL = 11;      // convolutions
constexpr int CIN0 = 16;    // input channels (11 used)
constexpr int COUT = 16;    // output channels (3 used)
constexpr long PART_FLOATS = 1L << 23;   // at most as many partial sums of a layer's weight gradient

// ------------------------------------------------------------ bfloat16
__device__ __forceinline__ float bf2f(bf16_t b) { return __uint_as_float((unsigned)b << 16); }
// round to nearest, ties to even (gfx950 converts in one instruction)
__device__ __forceinline__ bf16_t f2bf(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }
bf16_t host_f2bf(float f)
{
    unsigned u;
    std::memcpy(&u, &f, 4);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}
float host_bf2f(bf16_t b)
{
    unsigned u = (unsigned)b << 16;
    float f;
    std::memcpy(&f, &u, 4);
    return f;
}

// ------------------------------------------------------------ geometry
struct Vol {
    int D, H, W;      // interior
    int Hp, Wp;       // padded
    long V;           // interior voxels
    long Vp;          // padded voxels
};

Vol make_vol(int D, int H, int W)
{
    Vol g;
    g.D = D; g.H = H; g.W = W;
    g.Hp = H + 2; g.Wp = W + 2;
    g.V = (long)D * H * W;
    g.Vp = (long)(D + 2) * (H + 2) * (W + 2);
    return g;
}

__device__ __forceinline__ long pidx(const Vol& g, long v)
{
    const int x = (int)(v % g.W);
    const long r = v / g.W;
    const int y = (int)(r % g.H);
    const int z = (int)(r / g.H);
    return ((long)(z + 1) * g.Hp + (y + 1)) * g.Wp + (x + 1);
}

// Block index -> logical index so that consecutive logical indices run on
// the same XCD (workgroups are dispatched round-robin over the 8 XCDs).
// Bijective for any nb.
__device__ __forceinline__ int xcd_order(int b, int nb)
{
    const int q = nb / 8, r = nb % 8;
    const int x = b % 8, s = b / 8;
    return x < r ? x * (q + 1) + s : r * (q + 1) + (x - r) * q + s;
}

// ------------------------------------------------------------ convolution
enum { EPI_RELU = 0,      // Y = max(z, 0)
       EPI_RELU_ADD = 1,  // ... and Y2 = Y + M
       EPI_LIN = 2,       // Y = z
       EPI_LIN_MASK = 3,  // ... and Y2 = Y where M > 0, else 0
       EPI_MASK = 4,      // Y = z where M > 0, else 0
       EPI_F32 = 5 };     // Y = z, unpadded FP32 [V][16]

struct ConvArgs {
    const bf16_t* X;       // input, cin channels (level g, or its parent gx with UP)
    const bf16_t* Wt;      // weights in the order of weight_at
    const float* bias;     // or nullptr
    void* Y;
    bf16_t* Y2;
    const bf16_t* M;
    int cin, cout;
    Vol g, gx;
};

// Place of weight (output channel o, tap t, input channel i) of a convolution
// with cin input and cout output channels: blocks of 16 output channels, then
// chunks of KC = 16 or 32 input channels, then taps; of each the 64 lanes'
// pieces one after the other, lane (r, kq) = row r of the block, input
// channels kq KC / 4 .. + KC / 4 - 1, so that a wave loads a tap's block as
// 1 KB in a row.  Two blocks share 32 output channels: rows 4 k + i of the
// first are the channels 8 k + i, those of the second 8 k + 4 + i, so that a
// lane of the result (rows 4 k .. 4 k + 3 of each block) holds 8 channels in
// a row.
__host__ __device__ __forceinline__ long weight_at(int o, int t, int i, int cin, int cout)
{
    const int kc = cin < 32 ? 16 : 32, p = kc / 4, c = o % 32;
    const int block = cout < 32 ? 0 : o / 32 * 2 + c / 4 % 2, row = cout < 32 ? o : c / 8 * 4 + c % 4;
    return ((((long)block * (cin / kc) + i / kc) * 27 + t) * 64 + (i % kc) / p * 16 + row) * p + i % p;
}

// Epilogue of a wave's rows: the lane holds channels c0 .. c0 + 4 NBW - 1 of
// voxel x of the rows y0 .. of plane z (16-byte stores, 64 bytes per voxel by
// the four lanes of a column; the 8-byte stores of blocks of 16 consecutive
// channels took 31 of the 122 us of a 32-channel layer at 128^3).
template <int MR, int NBW, int EPI>
__device__ __forceinline__ void conv_store(const ConvArgs& a, const f4 (&acc)[MR][NBW], int x, int y0, int z, int c0)
{
    constexpr int NC = 4 * NBW;
    typedef __attribute__((ext_vector_type(NC))) short sn;
    const Vol& g = a.g;
    const int co = a.cout;
    if (z >= g.D || x >= g.W) return;
    const long at = EPI == EPI_F32 ? (((long)z * g.H + y0) * g.W + x) * co + c0
                                   : (((long)(z + 1) * g.Hp + y0 + 1) * g.Wp + x + 1) * co + c0;
    const int row = (EPI == EPI_F32 ? g.W : g.Wp) * co;
    f4 bb[NBW];
#pragma unroll
    for (int n = 0; n < NBW; ++n) {
        bb[n] = f4{0.f, 0.f, 0.f, 0.f};
        if (a.bias) bb[n] = *(const f4*)(a.bias + c0 + n * 4);
    }
#pragma unroll
    for (int m = 0; m < MR; ++m) {
        if (y0 + m >= g.H) break;
        const long p = at + m * row;
        sn mm, o, o2;
        if (EPI == EPI_RELU_ADD || EPI == EPI_LIN_MASK || EPI == EPI_MASK) mm = *(const sn*)(a.M + p);
#pragma unroll
        for (int n = 0; n < NBW; ++n) {
            f4 zz = acc[m][n];
#pragma unroll
            for (int i = 0; i < 4; ++i) zz[i] = zz[i] + bb[n][i];
            if (EPI == EPI_F32) {
                *(f4*)((float*)a.Y + p + n * 4) = zz;
                continue;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float q = zz[i];
                const float mf = bf2f((bf16_t)mm[n * 4 + i]);
                if (EPI == EPI_RELU || EPI == EPI_RELU_ADD) q = fmaxf(q, 0.f);
                if (EPI == EPI_MASK) q = mf > 0.f ? q : 0.f;
                const bf16_t h = f2bf(q);
                o[n * 4 + i] = (short)h;
                if (EPI == EPI_RELU_ADD) o2[n * 4 + i] = (short)f2bf(bf2f(h) + mf);
                if (EPI == EPI_LIN_MASK) o2[n * 4 + i] = mf > 0.f ? (short)h : (short)0;
            }
        }
        if (EPI == EPI_F32) continue;
        *(sn*)((bf16_t*)a.Y + p) = o;
        if (EPI == EPI_RELU_ADD || EPI == EPI_LIN_MASK) *(sn*)(a.Y2 + p) = o2;
    }
}

// The input of a block of output voxels, halo included: the origin (padded
// coordinates of the block's first halo voxel, channel chunk) is uniform, the
// lanes' offsets in it do not depend on the block.  Beyond the border of the
// volume they run on into other voxels (only outputs that are not stored see
// those), beyond the tensor the loads' range check gives 0.  With UP the
// voxels are the parent's, whose border is the zero border of the repetition
// (a block starts at even coordinates).  Buffer loads reach 2 GiB from the
// origin; where the six planes of a block span more (conv_far), FAR takes
// 64-bit offsets.
template <bool UP, bool FAR>
struct ConvIn {
    using Off = std::conditional_t<FAR, long, unsigned>;
    const ConvArgs& a;
    struct Src {
        const bf16_t* p;
        long rest;                                           // bytes up to the end of the tensor
    };
    __device__ Off offset(int tx, int ty, int tz, int c) const
    {
        if constexpr (UP) {
            tx = ((tx - 1) >> 1) + 1;
            ty = ((ty - 1) >> 1) + 1;
            tz = ((tz - 1) >> 1) + 1;
        }
        return ((Off)((Off)tz * a.gx.Hp + ty) * a.gx.Wp + tx) * (a.cin * 2) + c * 2;
    }
    __device__ Src origin(int x0, int y0, int z0, int c0) const
    {
        if constexpr (UP) {
            x0 >>= 1;
            y0 >>= 1;
            z0 >>= 1;
        }
        const long o = (((long)z0 * a.gx.Hp + y0) * a.gx.Wp + x0) * a.cin + c0;
        return {a.X + o, (a.gx.Vp * a.cin - o) * 2};
    }
    template <int N>
    __device__ void load(const Src& s, const Off (&from)[N], uint4 (&in)[N]) const
    {
        if constexpr (FAR) {
#pragma unroll
            for (int u = 0; u < N; ++u) {
                in[u] = uint4{0u, 0u, 0u, 0u};
                if (from[u] + 16 <= s.rest) in[u] = *(const uint4*)((const char*)s.p + from[u]);
            }
        } else {
            const int range = (int)(s.rest < 0x7fffffffL ? s.rest : 0x7fffffffL);
            const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)s.p, (short)0, range, 0x00020000);
#pragma unroll
            for (int u = 0; u < N; ++u)
                in[u] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, from[u], 0, 0));
        }
    }
};

// Six planes, and the rows and voxels of a block beyond them, past the reach
// of a buffer load?
bool conv_far(const ConvArgs& a) { return ((6L * a.gx.Hp + 10) * a.gx.Wp + 18) * a.cin * 2 > 0x7fffffffL; }

// Y[v][c] = epilogue(b[c] + sum_t sum_i X[v + off_t][i] W[c][t][i]).
// A workgroup computes a 4 (z) x MR (y) x 16 (x) block of output voxels for
// NBW * 16 output channels; wave w takes the z-slice w: MR rows of 16 voxels,
// the columns of the MFMA, against NBW blocks of 16 output channels, its rows
// (a lane then holds 4 channels of one voxel per block).
// The input block with its one-voxel halo is staged in LDS KC channels at a
// time and serves all 27 taps; with UP the input is the 2 x 2 x 2 repetition
// of its parent level, read from there.
//
// What bounds it: the operands.  A tap's weights are NBW KB per wave from the
// L1 (64 bytes per clock and CU), a row of voxels 1 KB from LDS (128 bytes per
// clock), and an MFMA takes 16 clocks, so both have to serve several MFMAs:
// 8 rows per wave halve the weight bytes of 4, and the rows of a z-plane are
// read once per dx and kept in registers for the three dy (MR + 2 fragments
// instead of 3 MR).  Every output adds its products in the order of the
// channel chunks and the taps, whatever the block.  The LDS rows of 64 bytes
// are swizzled (the 16-byte piece q of voxel x lies at q ^ (x / 4 % 4)), so
// that 16 lanes reading 16 consecutive voxels hit distinct banks.
// Measured: the 21 convolutions of a gradient at 128^3 with 32 base channels
// took 4.7 ms with 4 rows x 16 channels per wave, one fragment read per
// product and 2-byte stores, and take 2.18 ms.  32 -> 32 channels: 116 us
// (955 TFLOP/s; 56 us for its 268 MB at a copy's 4.8 TB/s), of which the
// products with their LDS reads are 67; staging, weights and stores, each 15
// to 30 us, overlap with them only across the two workgroups of a CU.  A
// persistent form that loads the next block's input ahead took 143 us.
__device__ __forceinline__ f4 mfma(b8 a, b8 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f4 mfma(s4 a, s4 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0); }
constexpr int CB_X = 16, CB_Z = 4, CT_X = CB_X + 2, CT_Z = CB_Z + 2;

template <int MR, int NBW, int KC, int EPI, bool UP, bool FAR = false>
__global__ __launch_bounds__(256, 2) void k_conv(ConvArgs a)
{
    constexpr int CT_Y = MR + 2, CT_N = CT_X * CT_Y * CT_Z, NP = KC / 8;   // voxels, 16-byte pieces per voxel
    __shared__ uint4 tile[(CT_N * NP + 255) / 256 * 256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, kq = lane >> 4;
    const Vol& g = a.g;
    const int nbx = (g.W + CB_X - 1) / CB_X, nby = (g.H + MR - 1) / MR, ng = a.cout / (16 * NBW);
    // the channel groups of a block of voxels run side by side on one XCD
    const int lb = xcd_order(blockIdx.x, gridDim.x);
    const int n0 = (lb % ng) * NBW * 16, bt = lb / ng;
    const int x0 = (bt % nbx) * CB_X, y0 = (bt / nbx % nby) * MR, z0 = bt / (nbx * nby) * CB_Z;
    const int cin = a.cin;
    f4 acc[MR][NBW];
#pragma unroll
    for (int m = 0; m < MR; ++m)
#pragma unroll
        for (int n = 0; n < NBW; ++n) acc[m][n] = f4{0.f, 0.f, 0.f, 0.f};
    using Frag = std::conditional_t<KC == 32, b8, s4>;       // KC / 4 channels of a voxel or of an output channel
    constexpr int TASKS = CT_N * NP, PER = (TASKS + 255) / 256;
    const ConvIn<UP, FAR> X{a};
    // LDS piece e of a swizzled row: channels 8 (e ^ (tx / 4)) % 32
    typename ConvIn<UP, FAR>::Off from[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int e = threadIdx.x + 256 * u, tv = e / NP;
        const int tx = tv % CT_X, ty = (tv / CT_X) % CT_Y, tz = tv / (CT_X * CT_Y);
        from[u] = X.offset(tx, ty, tz, (KC == 32 ? (e & 3) ^ (tx >> 2 & 3) : e & 1) * 8);
    }
    const long wstep = 16L * 27 * cin;                       // next block of output channels
    for (int c0 = 0; c0 < cin; c0 += KC) {
        uint4 in[PER];
        X.load(X.origin(x0, y0, z0, c0), from, in);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PER; ++u) tile[threadIdx.x + 256 * u] = in[u];
        __syncthreads();
        // lane (r, kq): channels kq * KC / 4 .. of output channel r (weights)
        // and of voxel r (input)
        const bf16_t* wl = a.Wt + n0 / 16 * wstep + c0 * 27L * 16 + lane * (KC / 4);
        int at[3];                                           // this lane's fragment in a row shifted by dx
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) at[dx] = (r + dx) * 4 + (KC == 32 ? kq ^ ((r + dx) >> 2 & 3) : kq);
        Frag w[NBW];
#pragma unroll
        for (int n = 0; n < NBW; ++n) w[n] = *(const Frag*)(wl + n * wstep);
        for (int dz = 0; dz < 3; ++dz) {
            const Frag* const rows = (const Frag*)tile + (wave + dz) * CT_Y * CT_X * 4;
            Frag f[MR + 2][3];
#pragma unroll
            for (int y = 0; y < MR; ++y)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) f[y][dx] = rows[y * CT_X * 4 + at[dx]];
#pragma unroll
            for (int dy = 0; dy < 3; ++dy) {
                if (dy > 0)
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx) f[MR - 1 + dy][dx] = rows[(MR - 1 + dy) * CT_X * 4 + at[dx]];
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) {
                    // the weights of the next tap are loaded while this one computes
                    const int t = dz * 9 + dy * 3 + dx, tn = t < 26 ? t + 1 : t;
                    Frag wn[NBW];
#pragma unroll
                    for (int n = 0; n < NBW; ++n) wn[n] = *(const Frag*)(wl + n * wstep + tn * 16 * KC);
#pragma unroll
                    for (int n = 0; n < NBW; ++n)
#pragma unroll
                        for (int m = 0; m < MR; ++m) acc[m][n] = mfma(w[n], f[m + dy][dx], acc[m][n]);
#pragma unroll
                    for (int n = 0; n < NBW; ++n) w[n] = wn[n];
                    __builtin_amdgcn_sched_barrier(0);       // later taps' loads stay where they are: registers
                }
            }
        }
    }
    const int c0 = NBW == 2 || a.cout < 32 ? n0 + kq * 4 * NBW : n0 / 32 * 32 + kq * 8 + n0 / 16 % 2 * 4;
    conv_store<MR, NBW, EPI>(a, acc, x0 + r, y0, z0 + wave, c0);
}

// 8 channels of a voxel
__device__ __forceinline__ uint4 ld8(const bf16_t* p) { return *(const uint4*)p; }
__device__ __forceinline__ float bf_at(const uint4& v, int k) { return bf2f(((const bf16_t*)&v)[k]); }

// Weight and bias gradients: the products are reduced over voxels, so both
// fragments hold 8 voxels of one channel per lane.  Voxels are staged in LDS
// as they lie in memory, channel-last, and read transposed
// (ds_read_b64_tr_b16: 16 lanes read 4 voxels x 16 channels, lane i gets the 4
// voxels of channel i).
typedef __attribute__((address_space(3))) s4 lds_s4;
__device__ __forceinline__ b8 ld_tr(const bf16_t* p, const bf16_t* q)
{
    typedef __attribute__((ext_vector_type(8))) short s8;
    const s4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)p);
    const s4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)q);
    return __builtin_bit_cast(b8, s8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]});
}
__device__ __forceinline__ int div_by(int n, float inv) { return (int)(((float)n + 0.5f) * inv); }   // n < 2^22

// n / d of values that are the same in all lanes, most often 0 or 1 (an
// integer division is some 40 dependent instructions)
__device__ __forceinline__ int div_uniform(int n, int d, float inv)
{
    if (n < d) return 0;
    if (n < 2 * d) return 1;
    return __builtin_amdgcn_readfirstlane(div_by(n, inv));
}

constexpr int WG_STEP = 128, WG_NEW = 192;                   // voxels of a step, new places of one load
constexpr int WG_LOAD = 256;                                 // threads that load (behind 512 that compute)
// with 32 input channels others load G (1.41 instead of 1.54 ms for the layers
// of a gradient at 128^3; with 16, two workgroups per CU, 0.13 instead of 0.11)
constexpr int wg_threads(int ci) { return 512 + ci * WG_LOAD; }
struct WgradArgs {
    const bf16_t *X, *G;
    float *part, *bias;                                      // partial sums: weights, bias
    int cin, cout;
    Vol g, gx;                                               // level of G; level of X (with UP the parent's)
    float *dW, *db;
    long E, vchunk;                                          // weights; voxels of a chunk
    int nch, nb, step;                                       // chunks; workgroups for the bias; voxels of a step at most
    int co, ci, up, rows, wgs;                               // kernel: blocks of 16 channels, parent level, rings; its workgroups
};
// The layers of one launch: workgroups first[l] .. first[l + 1] - 1 are layer l's.
struct WgradTable {
    int n, first[NL + 1];
    WgradArgs a[NL];
};
// the layer of this workgroup and the workgroup's number in it
__device__ __forceinline__ int layer_of(const WgradTable& t, int& block)
{
    int l = 0;
    while (l + 1 < t.n && (int)blockIdx.x >= t.first[l + 1]) ++l;
    block = blockIdx.x - t.first[l];
    return l;
}

// bias[block][c] = sum over the block's voxels of G[v][c] (k_wsum adds the
// blocks up in a fixed order)
__global__ __launch_bounds__(256) void k_bias_grad(WgradTable t)
{
    int block;
    const WgradArgs& a = t.a[layer_of(t, block)];
    // thread = (voxel slot, group of 8 channels): 16-byte loads, a block
    // covers 256 / (C / 8) voxels per step (C in {16, 32, 64, 128})
    __shared__ float s[256 * 8];
    const int C = a.cout, ng = C / 8, grp = threadIdx.x % ng, vq = threadIdx.x / ng, nv = 256 / ng;
    const Vol& g = a.g;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const long step = (long)a.nb * nv;
    long v = (long)block * nv + vq;
    // 8 loads in flight: one after the other they took 37 us of a 32-channel
    // layer at 128^3
    for (; v + 7 * step < g.V; v += 8 * step) {
        uint4 q[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) q[u] = ld8(a.G + pidx(g, v + u * step) * C + grp * 8);
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int k = 0; k < 8; ++k) acc[k] += bf_at(q[u], k);
    }
    for (; v < g.V; v += step) {
        const uint4 q = ld8(a.G + pidx(g, v) * C + grp * 8);
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] += bf_at(q, k);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) s[threadIdx.x * 8 + k] = acc[k];
    __syncthreads();
    if ((int)threadIdx.x < C) {
        const int gq = threadIdx.x / 8, k = threadIdx.x % 8;
        float sum = 0.f;
        for (int q = 0; q < nv; ++q) sum += s[(q * ng + gq) * 8 + k];
        a.bias[(long)block * C + threadIdx.x] = sum;
    }
}

// of two steps: the voxels' places (in elements); blocks of 32 voxels, whether
// the next step is stored after it, whether there is one
struct WgradSteps {
    int place[2][WG_STEP], blocks[2], wait[2], more[2];
};

// part[chunk][group][block pair][tap][lane][4]: sum over the chunk's voxels of
// G[v][o] X[v + off_t][i], for groups of 16 CO output and 16 CI input
// channels; every sum adds 32 voxels at a time in their order, whatever the
// split.
//
// A chunk is walked in steps of up to 128 consecutive voxels.  Its voxels have places q = (z (H + 1) + y) (W + 1) + x,
// in which one zero voxel between rows and one zero row between planes are the
// border, so that a tap is a constant distance dy (W + 1) + dx; of each of the
// three planes z + dz of X, a ring of R places in LDS holds those around the
// step, and a step loads only the places that are new: all 27 taps come from
// them.  (Rows too long for a ring: ROWS = 3 rings per plane, one per dy, and
// no row between planes.)  Eight waves compute: they share the (input block,
// tap) pairs, each with all output blocks, so that a fragment of X is read
// once.  Four waves load (eight with CI = 2): while a step is computed they store the
// next one's voxels and the list of its places to LDS and fetch the voxels of
// the one after it into registers.
//
// What bounds it: LDS reads (a fragment of 1 KB takes 10 clocks of the CU and
// serves CO products of 4 each; their banks do not conflict at any voxel
// pitch measured) and the instructions of the loading waves.  With a
// workgroup per tap and chunk, which staged both tensors transposed 27 times,
// the eleven layers of a gradient at 128^3 with 32 base channels took 5.9 ms,
// at 72 x 64 x 48 with 16 0.55 ms; they take 1.53 and 0.10 in one launch (1.9
// and 0.37 in eleven).  32 -> 32 channels at 128^3 alone: 276 us, of the 46
// that its products take.  Loading from the computing waves themselves: 384 us
// (9 windows per step) and 519 (rings).
template <int CO, int CI, bool UP, int R, int ROWS>
__device__ __forceinline__ void wgrad_chunk(const WgradArgs& a, int block, bf16_t* lds, WgradSteps& steps)
{
    constexpr int NO = CO * 16, NI = CI * 16;                // channels
    constexpr int TG = 8 / CI, PER = (27 + TG - 1) / TG;     // waves that share the taps, taps of a wave
    constexpr int RING = R * NI, XE = 3 * ROWS * RING, GE = WG_STEP * NO;   // elements
    constexpr int NEW = WG_NEW, NP = NI / 8;                 // 16-byte pieces of a voxel
    constexpr int PX = (ROWS * NEW * NP + WG_LOAD - 1) / WG_LOAD, PG = GE / 8 / WG_LOAD;    // per loading thread
    static_assert(GE / 8 % WG_LOAD == 0, "");
    auto& [place, blocks, wait, more] = steps;
    const Vol &g = a.g, &gx = a.gx;
    const int ngi = a.cin / NI, ng = ngi * (a.cout / NO), nw = a.nch * ng;
    const int lb = xcd_order(block, nw), chunk = lb / ng, grp = lb % ng;
    const int o0 = grp / ngi * NO, i0 = grp % ngi * NI;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int W1 = g.W + 1;
    const int loader = tid < 512 ? -1 : (tid - 512) % WG_LOAD;
    if (loader < 0) {
        const int l0 = (lane >> 4) * 8 + (lane & 15) / 4, c4 = lane % 4 * 4;   // voxel and channels the lane reads
        const int ib = wave % CI, tg = wave / CI, mine = ib * 16 + c4;
        f4 acc[PER][CO];
        int ring[PER], shift[PER];                           // of the wave's taps, in elements
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int t = tg * PER + q < 27 ? tg * PER + q : 26, dy = t / 3 % 3;
            ring[q] = (ROWS == 3 ? t / 3 : t / 9) * RING;
            shift[q] = ((ROWS == 3 ? 0 : (dy - 1) * W1) + t % 3 - 1) * NI + mine;
#pragma unroll
            for (int m = 0; m < CO; ++m) acc[q][m] = f4{0.f, 0.f, 0.f, 0.f};
        }
        struct Frags {
            b8 w[CO], f[PER];
        };
        for (int b = 0;; b ^= 1) {
            __syncthreads();
            const bf16_t* const from = lds + XE + b * GE + l0 * NO + c4;
            const int* const at = place[b] + l0;
            const int nk = __builtin_amdgcn_readfirstlane(blocks[b]);
            // the places of a block of 32 voxels are read one block ahead
            int q[2] = {at[0], at[4]};
            auto read = [&](int kb, Frags& x) {
#pragma unroll
                for (int m = 0; m < CO; ++m)
                    x.w[m] = ld_tr(from + kb * 32 * NO + m * 16, from + (kb * 32 + 4) * NO + m * 16);
#pragma unroll
                for (int t = 0; t < PER; ++t)
                    x.f[t] = ld_tr(lds + (((q[0] + shift[t]) & (RING - 1)) | ring[t]),
                                   lds + (((q[1] + shift[t]) & (RING - 1)) | ring[t]));
                const int next = (kb + 1) * 32 & (WG_STEP - 1);
                q[0] = at[next];
                q[1] = at[next + 4];
            };
            auto compute = [&](const Frags& x) {
#pragma unroll
                for (int t = 0; t < PER; ++t)
#pragma unroll
                    for (int m = 0; m < CO; ++m) acc[t][m] = mfma(x.w[m], x.f[t], acc[t][m]);
            };
            for (int kb = 0; kb < nk; ++kb) {
                Frags x;
                read(kb, x);
                compute(x);
            }
            const bool last = !__builtin_amdgcn_readfirstlane(more[b]);
            if (__builtin_amdgcn_readfirstlane(wait[b])) __syncthreads();
            if (last) break;
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int t = tg * PER + q;
            if (t >= 27) break;
#pragma unroll
            for (int m = 0; m < CO; ++m)
                *((f4*)a.part + ((((long)chunk * ng + grp) * CO * CI + m * CI + ib) * 27 + t) * 64 + lane) = acc[q][m];
        }
        return;
    }

    // ---- the loading waves
    const int H1 = g.H + (ROWS == 3 ? 0 : 1), gap = ROWS == 3 ? 0 : W1;     // gap: places between planes
    const int reach = ROWS == 3 ? 1 : W1 + 1;                // of the taps, in places
    const float inv_w = 1.f / (float)g.W, inv_h = 1.f / (float)g.H, inv_w1 = 1.f / (float)W1, inv_h1 = 1.f / (float)H1;
    // a voxel, or a place (z counted from -1), in coordinates
    struct At {
        int x, y, z, q;
    };
    // the voxel n on from v, n < 2^20
    auto ahead_of = [&](At v, int n) {
        const int x = v.x + n, run = div_uniform(x, g.W, inv_w), y = v.y + run, plane = div_uniform(y, g.H, inv_h);
        return At{x - run * g.W, y - plane * g.H, v.z + plane, v.q + n + run + plane * gap};
    };
    // the pieces of X (row ring, place, channels) and of G of a thread
    constexpr unsigned NONE = 0x80000000u;                   // out of a load's range: gives 0
    const int xp = loader % NP, gp = loader % (NO / 8);
    auto piece = [&](int u, int& r, int& i) {
        const int e = loader + WG_LOAD * u;
        r = e / (NEW * NP);
        i = e / NP % NEW;
        return ROWS * NEW * NP % WG_LOAD == 0 || r < ROWS;
    };
    uint4 vx[PX][3], vg[PG];
    // offsets are those of voxels of the tensor or NONE
    auto source = [](const bf16_t* p) { return __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, 0x7fffffff, 0x00020000); };
    auto read = [](__amdgpu_buffer_rsrc_t rs, unsigned at) {
        return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, at, 0, 0));
    };
    const long v0 = chunk * a.vchunk, v1 = v0 + a.vchunk < g.V ? v0 + a.vchunk : g.V;
    At v, n;                                                 // first voxel of a step, first place not stored
    v.x = (int)(v0 % g.W);
    v.y = (int)(v0 / g.W % g.H);
    v.z = (int)(v0 / ((long)g.W * g.H));
    const long q0 = ((long)(v.z + 1) * H1 + v.y) * W1 + v.x, n0 = q0 - reach;
    v.q = (int)(unsigned)q0;
    n.q = (int)(unsigned)n0;
    n.x = (int)(n0 % W1);
    n.y = (int)(n0 / W1 % H1);
    n.z = (int)(n0 / ((long)W1 * H1)) - 1;
    // count (up to NEW) places of X from n on
    auto load_x = [&](int count) {
        unsigned at[PX][UP ? 3 : 1];
#pragma unroll
        for (int u = 0; u < PX; ++u) {
            int r, i;
            const bool have = piece(u, r, i) && i < count;
            int x = n.x + i;
            const int run = div_by(x, inv_w1);
            x -= run * W1;
            const int plane = div_by(n.y + run, inv_h1), y = n.y + run - plane * H1 + (ROWS == 3 ? r - 1 : 0);
            const int z = n.z + plane;
            const bool in = have && x < g.W && y >= 0 && y < g.H && z >= 0 && z < g.D;
            if constexpr (UP) {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const int p = ((z + k - 1) >> 1) - ((n.z + k - 1) >> 1);
                    at[u][k] = in ? (unsigned)(((p * gx.Hp + (y >> 1) + 1) * gx.Wp + (x >> 1) + 1) * a.cin) * 2u + xp * 16 : NONE;
                }
            } else {
                at[u][0] = in ? (unsigned)(((plane * gx.Hp + y + 1 - n.y) * gx.Wp + x + 1) * a.cin) * 2u + xp * 16 : NONE;
            }
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int z = n.z + k - 1;
            const auto rs = UP ? source(a.X + (long)((z >> 1) + 1) * gx.Hp * gx.Wp * a.cin + i0)
                               : source(a.X + ((long)(z + 1) * gx.Hp + n.y) * gx.Wp * a.cin + i0);
#pragma unroll
            for (int u = 0; u < PX; ++u) vx[u][k] = read(rs, at[u][UP ? k : 0]);
        }
    };
    auto store_x = [&](int count) {
#pragma unroll
        for (int u = 0; u < PX; ++u) {
            int r, i;
            if (!piece(u, r, i) || i >= count) continue;
#pragma unroll
            for (int k = 0; k < 3; ++k)
                *(uint4*)(lds + (k * ROWS + r) * RING + ((n.q + i) & (R - 1)) * NI + xp * 8) = vx[u][k];
        }
        const int x = n.x + count, run = div_uniform(x, W1, inv_w1), y = n.y + run, plane = div_uniform(y, H1, inv_h1);
        n = At{x - run * W1, y - plane * H1, n.z + plane, n.q + count};
    };
    auto load_g = [&] {
        const auto rs = source(a.G + (((long)(v.z + 1) * g.Hp + v.y + 1) * g.Wp + 1) * a.cout + o0);
#pragma unroll
        for (int u = 0; u < PG; ++u) {
            int x = v.x + (loader + WG_LOAD * u) / (NO / 8);
            const int run = div_by(x, inv_w), plane = div_by(v.y + run, inv_h), y = v.y + run - plane * g.H;
            x -= run * g.W;
            vg[u] = read(rs, v.z + plane < g.D ? (unsigned)(((plane * g.Hp + y - v.y) * g.Wp + x) * a.cout) * 2u + gp * 16 : NONE);
        }
    };
    // A step has as many voxels, up to a.step, as have room in the ring beside the
    // step before it; where not even 32 have, the step before it is done
    // first.  It is fetched ahead unless it brings too many places for one load
    // (at a chunk's start, or where it crosses planes).
    long left = v1 - v0;
    int voxels, end;                                         // of the step from v on; end of its places
    bool held = false;                                       // no room in the ring until the step before it is computed
    auto size = [&](int first) {
        for (voxels = a.step;; voxels -= 32) {
            end = ahead_of(v, voxels - 1).q + reach + 1;
            if (end - first <= R || voxels == 32) return;
        }
    };
    auto advance = [&] {                                     // to the next step, if there is one
        const int first = v.q - reach;
        left -= voxels;
        held = false;
        if (left <= 0) return false;
        v = ahead_of(v, voxels);
        size(first);
        held = end - first > R;
        return true;
    };
    size(v.q - reach);
    // one loop per kind of loading wave: the compiler then knows which loads
    // are in flight when it waits for one
    auto load = [&](auto does_x, auto does_g) {
        if (does_g) load_g();
        bool fetched = false;                                // X
        for (int b = 0;; b ^= 1) {
            if (does_x) {
                if (!fetched) {
                    while (end - n.q > NEW) {
                        load_x(NEW);
                        store_x(NEW);
                    }
                    load_x(end - n.q);
                }
                store_x(end - n.q);
            }
            if (does_g) {
#pragma unroll
                for (int u = 0; u < PG; ++u) *(uint4*)(lds + XE + b * GE + (loader + WG_LOAD * u) * 8) = vg[u];
                if (loader < WG_STEP) {
                    const int run = div_by(v.x + loader, inv_w), plane = div_by(v.y + run, inv_h);
                    place[b][loader] = (v.q + loader + run + plane * gap) * NI;
                }
            }
            // the chunk's last step may be shorter (behind the volume G is 0)
            const int kb = left < voxels ? (int)(left + 31) / 32 : voxels / 32;
            const bool go_on = advance();
            if (does_x) {
                fetched = go_on && end - n.q <= NEW;
                if (fetched) load_x(end - n.q);
            }
            if (does_g) {
                if (go_on) load_g();
                if (loader == 0) {
                    blocks[b] = kb;
                    wait[b] = held;
                    more[b] = go_on;
                }
            }
            __syncthreads();
            if (held) __syncthreads();
            if (!go_on) return;
        }
    };
    using T = std::true_type;
    using F = std::false_type;
    if constexpr (CI == 1) load(T(), T());
    else if (tid < 512 + WG_LOAD) load(T(), F());
    else load(F(), T());
}

// The weight gradients of all layers of one kind of ring in one launch: one
// layer's chunks do not fill the chip evenly (303 workgroups at 128^3, 14 of
// the middle level at 72 x 64 x 48).
template <int CI, int R, int ROWS>
__global__ __launch_bounds__(wg_threads(CI), 2 + CI) void k_wgrad(WgradTable t)
{
    __shared__ __attribute__((aligned(16))) bf16_t lds[3 * ROWS * R * CI * 16 + 2 * WG_STEP * 32];
    __shared__ WgradSteps steps;
    int block;
    const WgradArgs& a = t.a[layer_of(t, block)];
    if (a.co == 2) {
        if (a.up) wgrad_chunk<2, CI, true, R, ROWS>(a, block, lds, steps);
        else wgrad_chunk<2, CI, false, R, ROWS>(a, block, lds, steps);
    } else {
        if (a.up) wgrad_chunk<1, CI, true, R, ROWS>(a, block, lds, steps);
        else wgrad_chunk<1, CI, false, R, ROWS>(a, block, lds, steps);
    }
}

// dW and db = sums over the chunks' and the bias blocks' partial sums in a
// fixed order.  Weights: E / 128 workgroups of 32 groups of 4 entries, thread
// j of 8 sums chunks j, j + 8, ..., then the eight sums are added in j order;
// entry (group, pair, tap, lane, i) is output channel 4 (lane / 16) + i and
// input channel lane % 16 of its block.  Bias: one workgroup per channel,
// thread j sums blocks j, j + 256, ..., then a tree of fixed shape adds the
// 256 sums.
__global__ __launch_bounds__(256) void k_wsum(WgradTable table)
{
    __shared__ f4 s[8][32];
    int block;
    const WgradArgs& a = table.a[layer_of(table, block)];
    const long E = a.E, nw = E / 128;
    const int co = a.co, ci = a.ci;
    if (block >= nw) {
        float* const t = (float*)s;
        const int c = (int)(block - nw);
        float acc = 0.f;
        for (int b = threadIdx.x; b < a.nb; b += 256) acc += a.bias[(long)b * a.cout + c];
        t[threadIdx.x] = acc;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) t[threadIdx.x] += t[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) a.db[c] = t[0];
        return;
    }
    const int el = threadIdx.x & 31, jl = threadIdx.x >> 5;
    const long e = block * 128L + el * 4;
    f4 sum{0.f, 0.f, 0.f, 0.f};
    auto add = [&](const f4& v) {
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[i] = sum[i] + v[i];
    };
#pragma unroll 8
    for (int c = jl; c < a.nch; c += 8) add(*(const f4*)(a.part + c * E + e));
    s[jl][el] = sum;
    __syncthreads();
    if (jl > 0) return;
    for (int j = 1; j < 8; ++j) add(s[j][el]);
    const int lane = (int)(e / 4) % 64, t = (int)(e / 256) % 27, q = (int)(e / (256 * 27));
    const int pair = q % (co * ci), grp = q / (co * ci), ngi = a.cin / (16 * ci);
    const int o = (grp / ngi * co + pair / ci) * 16 + lane / 16 * 4;
    const int i = (grp % ngi * ci + pair % ci) * 16 + lane % 16;
#pragma unroll
    for (int k = 0; k < 4; ++k) a.dW[((long)(o + k) * 27 + t) * a.cin + i] = sum[k];
}

// ------------------------------------------------------------ elementwise
// Passes between the levels.  A thread takes 8 channels (16 bytes) of one
// voxel; all are bound by the bytes they move.
__device__ __forceinline__ long at(const Vol& g, int x, int y, int z)
{
    return ((long)(z + 1) * g.Hp + y + 1) * g.Wp + x + 1;
}

// sum of the 8 children (level g, C channels) of voxel (x, y, z), 8 channels from c
__device__ __forceinline__ void sum_children(const bf16_t* __restrict__ in, int C, const Vol& g, int x, int y, int z, int c,
                                             float s[8])
{
#pragma unroll
    for (int k = 0; k < 8; ++k) s[k] = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const uint4 v = ld8(in + at(g, 2 * x + (q & 1), 2 * y + ((q >> 1) & 1), 2 * z + (q >> 2)) * C + c);
#pragma unroll
        for (int k = 0; k < 8; ++k) s[k] += bf_at(v, k);
    }
}

// voxel and first channel of element e (8 channels each) of a level
struct Elem {
    int x, y, z, c;
};
__device__ __forceinline__ Elem elem_of(const Vol& g, int C, long e)
{
    const int n = C / 8;
    const long v = e / n;
    return {(int)(v % g.W), (int)((v / g.W) % g.H), (int)(v / ((long)g.W * g.H)), (int)(e % n) * 8};
}

// pool: out (level g2) = mean of the 8 children in level g
__global__ void k_pool(const bf16_t* __restrict__ in, bf16_t* __restrict__ out, int C, Vol g, Vol g2)
{
    // grid-stride: the element count can exceed 2^32 work-items
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < g2.V * (C / 8); e += (long)gridDim.x * blockDim.x) {
        const Elem t = elem_of(g2, C, e);
        float s[8];
        sum_children(in, C, g, t.x, t.y, t.z, t.c, s);
        bf16_t o[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) o[k] = f2bf(s[k] * 0.125f);
        *(uint4*)(out + at(g2, t.x, t.y, t.z) * C + t.c) = *(uint4*)o;
    }
}

// gradient of up, then of the ReLU before it: out (level g2) = sum of the 8
// children (level g) where m > 0, else 0
__global__ void k_up_dx(const bf16_t* __restrict__ in, const bf16_t* __restrict__ m, bf16_t* __restrict__ out, int C,
                        Vol g, Vol g2)
{
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < g2.V * (C / 8); e += (long)gridDim.x * blockDim.x) {
        const Elem t = elem_of(g2, C, e);
        float s[8];
        sum_children(in, C, g, t.x, t.y, t.z, t.c, s);
        const long p = at(g2, t.x, t.y, t.z) * C + t.c;
        const uint4 mv = ld8(m + p);
        bf16_t o[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) o[k] = bf_at(mv, k) > 0.f ? f2bf(s[k]) : (bf16_t)0;
        *(uint4*)(out + p) = *(uint4*)o;
    }
}

// gradient of the skip connection and of pool, then of the ReLU before them:
// out (level g) = a + t(parent, level g2) / 8 where m > 0, else 0
__global__ void k_add_pool_dx(const bf16_t* __restrict__ a, const bf16_t* __restrict__ t, const bf16_t* __restrict__ m,
                              bf16_t* __restrict__ out, int C, Vol g, Vol g2)
{
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < g.V * (C / 8); e += (long)gridDim.x * blockDim.x) {
        const Elem q = elem_of(g, C, e);
        const long p = at(g, q.x, q.y, q.z) * C + q.c;
        const uint4 av = ld8(a + p), mv = ld8(m + p), tv = ld8(t + at(g2, q.x / 2, q.y / 2, q.z / 2) * C + q.c);
        bf16_t o[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) o[k] = bf_at(mv, k) > 0.f ? f2bf(bf_at(av, k) + bf_at(tv, k) * 0.125f) : (bf16_t)0;
        *(uint4*)(out + p) = *(uint4*)o;
    }
}

// Loss: mean squared error over the interior faces; gy = its gradient.
// Output channel d of voxel (x, y, z) is the lower d-face of that cell; the
// face is interior when its index along d is in 1 .. n_d - 1.
// Output gradient of the loss, and part[block] = the block's share of the
// loss (k_lsum adds the blocks up in a fixed order).
__global__ void k_loss(const float* __restrict__ y, const float* __restrict__ tg, bf16_t* __restrict__ gy, Vol g,
                       int nx, int ny, int nz, float inv_n, double* __restrict__ part)
{
    __shared__ float s[256];
    float acc = 0.f;
    for (long v = (long)blockIdx.x * blockDim.x + threadIdx.x; v < g.V; v += (long)gridDim.x * blockDim.x) {
        const int x = (int)(v % g.W), yy = (int)((v / g.W) % g.H), z = (int)(v / ((long)g.W * g.H));
        const bool in = x < nx && yy < ny && z < nz;
        const long p = pidx(g, v);
        const f4 a = *(const f4*)(y + v * COUT), b = *(const f4*)(tg + v * 4);
        bf16_t o[COUT] = {};
        for (int c = 0; c < 3; ++c) {
            const bool ok = in && (c == 0 ? x : c == 1 ? yy : z) >= 1;
            const float d = ok ? a[c] - b[c] : 0.f;
            acc += d * d;
            o[c] = f2bf(2.f * d * inv_n);
        }
        for (int c = 0; c < COUT; c += 8) *(uint4*)(gy + p * COUT + c) = *(uint4*)(o + c);
    }
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = (double)s[0] * inv_n;
}

// loss = sum of the nb block shares, thread j taking blocks j, j + 256, ...,
// then a tree of fixed shape (one workgroup of 256 threads)
__global__ __launch_bounds__(256) void k_lsum(const double* __restrict__ part, int nb, double* __restrict__ loss)
{
    __shared__ double s[256];
    double acc = 0.0;
    for (int b = threadIdx.x; b < nb; b += 256) acc += part[b];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = s[0];
}

__global__ void k_fill_f(float* p, float v, long n)
{
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) p[e] = v;
}

// Adam step on the master parameters; bias corrections c1 = 1 - b1^t,
// c2 = 1 - b2^t.
__global__ void k_adam(float* __restrict__ w, const float* __restrict__ gr, float* __restrict__ m,
                       float* __restrict__ vv, long n, float lr, float c1, float c2)
{
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float gg = gr[e];
    const float mm = b1 * m[e] + (1.f - b1) * gg;
    const float v2 = b2 * vv[e] + (1.f - b2) * gg * gg;
    m[e] = mm;
    vv[e] = v2;
    w[e] -= lr * (mm / c1) / (sqrtf(v2 / c2) + eps);
}

// bfloat16 copies of all layers' weights for their convolutions and,
// transposed and tap-mirrored, for those of their input gradients, both in the
// order in which the convolution's waves load them (weight_at).
struct WcopyTable {
    long first[NL + 1], woff[NL], wboff[NL];                 // first entry, place in the parameters and in the copies
    int co[NL], ci[NL];
};
__global__ void k_wcopy(WcopyTable t, const float* __restrict__ w, bf16_t* __restrict__ wb, bf16_t* __restrict__ wtb)
{
    const long at = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (at >= t.first[NL]) return;
    int l = 0;
    while (at >= t.first[l + 1]) ++l;
    const long e = at - t.first[l];
    const int ci = t.ci[l], co = t.co[l];
    const int i = (int)(e % ci), tap = (int)((e / ci) % 27), o = (int)(e / ((long)ci * 27));
    const bf16_t b = f2bf(w[t.woff[l] + e]);
    wb[t.wboff[l] + weight_at(o, tap, i, ci, co)] = b;
    wtb[t.wboff[l] + weight_at(i, 26 - tap, o, co, ci)] = b;
}

// ------------------------------------------------------------ solver side
struct SolverView {
    const double *txx, *tyy, *txy, *txz, *tyz, *p, *epsp;
    const double *vx, *vy, *vz;
    int nx, ny, nz, sy;
    long sz;
};

// Features of the solver state into a padded input tensor (16 channels).
__global__ void k_features(SolverView s, const float* __restrict__ dvp, bf16_t* __restrict__ x, Vol g, float iss,
                           float ise, float isv)
{
    const long v = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= g.V) return;
    const int i = (int)(v % g.W), j = (int)((v / g.W) % g.H), k = (int)(v / ((long)g.W * g.H));
    float f[16];
    for (int c = 0; c < 16; ++c) f[c] = 0.f;
    if (i < s.nx && j < s.ny && k < s.nz) {
        const long sy = s.sy, sz = s.sz;
        const long e = i + sy * j + sz * k;
        const double txx = s.txx[e], tyy = s.tyy[e];
        f[0] = (float)(txx * iss);
        f[1] = (float)(tyy * iss);
        f[2] = (float)(-(txx + tyy) * iss);
        f[3] = (float)(0.25 * (s.txy[e] + s.txy[e + 1] + s.txy[e + sy] + s.txy[e + sy + 1]) * iss);
        f[4] = (float)(0.25 * (s.txz[e] + s.txz[e + 1] + s.txz[e + sz] + s.txz[e + sz + 1]) * iss);
        f[5] = (float)(0.25 * (s.tyz[e] + s.tyz[e + sy] + s.tyz[e + sz] + s.tyz[e + sy + sz]) * iss);
        f[6] = (float)(s.p[e] * iss);
        f[7] = (float)(s.epsp[e] * ise);
        f[8] = dvp[v * 4 + 0] * isv;
        f[9] = dvp[v * 4 + 1] * isv;
        f[10] = dvp[v * 4 + 2] * isv;
    }
    const long p = pidx(g, v) * 16;
    for (int c = 0; c < 16; ++c) x[p + c] = f2bf(f[c]);
}

// After an increment: velocity change at the lower faces since the last
// call -> tracked previous change (and a target when tg != null).
__global__ void k_observe(SolverView s, double* __restrict__ vlast, float* __restrict__ dvp, float* __restrict__ tg,
                          Vol g, int first, float iso)
{
    const long v = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= g.V) return;
    const int i = (int)(v % g.W), j = (int)((v / g.W) % g.H), k = (int)(v / ((long)g.W * g.H));
    for (int d = 0; d < 3; ++d) {
        float dv = 0.f;
        if (i < s.nx && j < s.ny && k < s.nz) {
            const long e = i + (long)s.sy * j + s.sz * k;
            const double cur = d == 0 ? s.vx[e] : d == 1 ? s.vy[e] : s.vz[e];
            if (!first) dv = (float)(cur - vlast[v * 3 + d]);
            vlast[v * 3 + d] = cur;
        }
        dvp[v * 4 + d] = dv;
        if (tg) tg[v * 4 + d] = dv * iso;
    }
    dvp[v * 4 + 3] = 0.f;
    if (tg) tg[v * 4 + 3] = 0.f;
}

// Guess velocities: current + scale * y at interior faces, current elsewhere.
__global__ void k_apply_guess(SolverView s, const float* __restrict__ y, double* __restrict__ gx,
                              double* __restrict__ gyv, double* __restrict__ gz, Vol g, float so)
{
    const long n = (long)(s.nx + 1) * (s.ny + 1) * (s.nz + 1);
    const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const int i = (int)(q % (s.nx + 1)), j = (int)((q / (s.nx + 1)) % (s.ny + 1)),
              k = (int)(q / ((long)(s.nx + 1) * (s.ny + 1)));
    const long e = i + (long)s.sy * j + s.sz * k;
    auto yv = [&](int c) { return y[(((long)k * g.H + j) * g.W + i) * COUT + c]; };
    if (j < s.ny && k < s.nz) gx[e] = s.vx[e] + ((i >= 1 && i < s.nx) ? (double)(so * yv(0)) : 0.0);
    if (i < s.nx && k < s.nz) gyv[e] = s.vy[e] + ((j >= 1 && j < s.ny) ? (double)(so * yv(1)) : 0.0);
    if (i < s.nx && j < s.ny) gz[e] = s.vz[e] + ((k >= 1 && k < s.nz) ? (double)(so * yv(2)) : 0.0);
}

// blocks for n elements, capped at 2^22 (2^30 work-items, below the 2^32
// limit of a dispatch); kernels whose n can exceed that loop grid-stride
inline unsigned nblk(long n, int t = 256) { return (unsigned)std::min<long>((n + t - 1) / t, 1L << 22); }

}  // namespace

// =========================================================================
struct ep_net {
    ep_net_config cfg;
    hipStream_t st;
    Vol g[3];
    int ch[NL][2];             // (Cin, Cout)
    long woff[NL], boff[NL];   // offsets in the parameter vector
    long wboff[NL];            // offsets in the bf16 weight arrays
    long np, nwb;
    float *w, *gr, *m, *v;     // FP32 masters, gradient, moments
    bf16_t *wb, *wtb;          // bf16 weights and transposed copies
    // activations
    bf16_t *xin, *a0, *s0, *p0, *a1, *s1, *p1, *a2, *b2, *r6, *c1, *d1, *r8, *c0, *d0;
    float* y;
    // gradients
    bf16_t *gy, *z9, *gc0, *z8, *t0, *z7, *gc1, *z6, *t1, *z5, *z4, *t2, *z3, *z2, *t3, *z1, *z0;
    // samples and tracking
    bf16_t* sx;                // max_samples x Vp0 x 16
    float* stg;                // max_samples x V0 x 4
    double* vlast;             // V0 x 3
    float* dvp;                // V0 x 4
    double* loss;
    float* part;               // per-chunk partial sums of the weight and bias gradients (training only)
    bool have_last;
    long adam_t;
    char err[512];
};

namespace {

int nerr(ep_net* n, int code, const char* fmt, ...)
{
    if (n) {
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(n->err, sizeof(n->err), fmt, ap);
        va_end(ap);
    }
    return code;
}

#define NCHK(n, x)                                                                          \
    do {                                                                                    \
        hipError_t e_ = (x);                                                                \
        if (e_ != hipSuccess)                                                               \
            return nerr((n), EP_EDEVICE, "%s failed: %s", #x, hipGetErrorString(e_));       \
    } while (0)

int validate_cfg(const ep_net_config* c)
{
    if (!c) return EP_EINVAL;
    if (c->nx < 4 || c->ny < 4 || c->nz < 4) return EP_EINVAL;
    if (c->base != 16 && c->base != 32) return EP_EINVAL;
    if (c->max_samples < 0) return EP_EINVAL;
    for (int q = 0; q < 4; ++q)
        if (!(c->scale[q] > 0)) return EP_EINVAL;
    return EP_OK;
}

void layer_channels(int base, int ch[NL][2])
{
    const int c = base, c2 = 2 * base, c4 = 4 * base;
    const int t[NL][2] = {{CIN0, c}, {c, c}, {c, c2}, {c2, c2}, {c2, c4}, {c4, c4},
                          {c4, c2}, {c2, c2}, {c2, c}, {c, c}, {c, COUT}};
    std::memcpy(ch, t, sizeof(t));
}

// Weight gradient l of level g: chunks, partial sums and kernel.
WgradArgs wgrad_plan(int cout, int cin, const Vol& g)
{
    // voxel chunks of at least 2048 voxels (a multiple of 128), at most 512
    // and as many as PART_FLOATS partial sums hold
    WgradArgs a{};
    a.cin = cin;
    a.cout = cout;
    a.g = g;
    a.E = 27L * cout * cin;
    long nch = std::min<long>((g.V + 2047) / 2048, std::min<long>(512, PART_FLOATS / a.E));
    a.vchunk = ((g.V + nch - 1) / nch + 127) / 128 * 128;
    a.nch = (int)((g.V + a.vchunk - 1) / a.vchunk);
    a.nb = (int)std::min<long>(1024, (g.V * (cout / 8) + 255) / 256);
    // Places of 32 voxels: their own, one per row and a row per plane more, and
    // the taps' reach.  Rings of 512 places hold rows up to 157 voxels with 32
    // input channels, of 1024 rows up to 328 with 16 (a workgroup per 16 input
    // channels: 398 instead of 276 us of a 32 -> 32 channel layer at 128^3);
    // with one ring per row offset a step loads three times as much.
    const long span = 32 + (32 / g.W + 1) + (32 / ((long)g.W * g.H) + 1) * (g.W + 1) + 2L * (g.W + 2);
    a.rows = span <= 512 ? 0 : span <= 1024 ? 1 : 2;
    // two steps inside a plane beside each other in a ring
    const long ring = a.rows == 0 ? 512 : a.rows == 1 ? 1024 : 256, reach = a.rows == 2 ? 2 : 2L * (g.W + 2);
    for (a.step = WG_STEP; a.step > 32 && 2 * a.step + 2 * a.step / g.W + 1 + reach > ring;) a.step -= 32;
    a.co = cout % 32 == 0 ? 2 : 1;                           // channel counts are 16 or multiples of 32
    a.ci = a.rows == 0 && cin % 32 == 0 ? 2 : 1;
    a.wgs = a.nch * (cout / (16 * a.co)) * (cin / (16 * a.ci));
    return a;
}

// Walk the workspace layout (assign pointers when n->... base != null).
size_t net_carve(const ep_net_config* c, ep_net* n, char* base)
{
    int ch[NL][2];
    layer_channels(c->base, ch);
    const int D0 = (c->nz + 3) / 4 * 4, H0 = (c->ny + 3) / 4 * 4, W0 = (c->nx + 3) / 4 * 4;
    Vol g0 = make_vol(D0, H0, W0), g1 = make_vol(D0 / 2, H0 / 2, W0 / 2), g2 = make_vol(D0 / 4, H0 / 4, W0 / 4);
    long np = 0, nwb = 0;
    long woff[NL], boff[NL], wboff[NL];
    for (int l = 0; l < NL; ++l) {
        woff[l] = np;
        np += (long)ch[l][1] * 27 * ch[l][0];
        boff[l] = np;
        np += ch[l][1];
        wboff[l] = nwb;
        nwb += (long)ch[l][1] * 27 * ch[l][0];
    }
    size_t off = 0;
    auto take = [&](size_t bytes) -> char* {
        off = (off + 255) / 256 * 256;
        char* r = base ? base + off : nullptr;
        off += bytes;
        return r;
    };
    auto act = [&](const Vol& g, int C) { return (bf16_t*)take((size_t)g.Vp * C * sizeof(bf16_t)); };
    const int C = c->base, C2 = 2 * C, C4 = 4 * C;
    float* w = (float*)take(np * 4);
    float* gr = (float*)take(np * 4);
    float* m = (float*)take(np * 4);
    float* v = (float*)take(np * 4);
    bf16_t* wb = (bf16_t*)take(nwb * 2);
    bf16_t* wtb = (bf16_t*)take(nwb * 2);
    bf16_t* A[15];
    const Vol* gl[15] = {&g0, &g0, &g0, &g1, &g1, &g1, &g2, &g2, &g2, &g1, &g1, &g1, &g0, &g0, &g0};
    const int cl[15] = {CIN0, C, C, C, C2, C2, C2, C4, C4, C2, C2, C2, C, C, C};
    for (int q = 0; q < 15; ++q) A[q] = act(*gl[q], cl[q]);
    float* y = (float*)take((size_t)g0.V * COUT * 4);
    bf16_t* G[17];
    const Vol* gg[17] = {&g0, &g0, &g0, &g0, &g0, &g1, &g1, &g1, &g1, &g2, &g2, &g2, &g1, &g1, &g1, &g0, &g0};
    const int cg[17] = {COUT, C, C, C, C2, C2, C2, C2, C4, C4, C4, C2, C2, C2, C, C, C};
    // gradient tensors only for a network that trains (max_samples > 0)
    for (int q = 0; q < 17; ++q) G[q] = c->max_samples > 0 ? act(*gg[q], cg[q]) : nullptr;
    bf16_t* sx = (bf16_t*)take((size_t)c->max_samples * g0.Vp * 16 * 2);
    float* stg = (float*)take((size_t)c->max_samples * g0.V * 4 * 4);
    double* vlast = (double*)take((size_t)g0.V * 3 * 8);
    float* dvp = (float*)take((size_t)g0.V * 4 * 4);
    double* loss = (double*)take(8);
    // partial sums of the parameter gradients (k_loss's before them)
    long sums = 2 * 1024;
    const Vol* lv[NL] = {&g0, &g0, &g1, &g1, &g2, &g2, &g1, &g1, &g0, &g0, &g0};
    for (int l = 0; l < NL; ++l) {
        const WgradArgs a = wgrad_plan(ch[l][1], ch[l][0], *lv[l]);
        sums += a.nch * a.E + (long)a.nb * a.cout;
    }
    float* part = c->max_samples > 0 ? (float*)take(sums * 4) : nullptr;
    if (n) {
        n->g[0] = g0; n->g[1] = g1; n->g[2] = g2;
        std::memcpy(n->ch, ch, sizeof(ch));
        std::memcpy(n->woff, woff, sizeof(woff));
        std::memcpy(n->boff, boff, sizeof(boff));
        std::memcpy(n->wboff, wboff, sizeof(wboff));
        n->np = np; n->nwb = nwb;
        n->w = w; n->gr = gr; n->m = m; n->v = v; n->wb = wb; n->wtb = wtb;
        bf16_t** dst[15] = {&n->xin, &n->a0, &n->s0, &n->p0, &n->a1, &n->s1, &n->p1, &n->a2, &n->b2,
                            &n->r6, &n->c1, &n->d1, &n->r8, &n->c0, &n->d0};
        for (int q = 0; q < 15; ++q) *dst[q] = A[q];
        n->y = y;
        bf16_t** gd[17] = {&n->gy, &n->z9, &n->gc0, &n->z8, &n->t0, &n->z7, &n->gc1, &n->z6, &n->t1, &n->z5, &n->z4,
                           &n->t2, &n->z3, &n->z2, &n->t3, &n->z1, &n->z0};
        for (int q = 0; q < 17; ++q) *gd[q] = G[q];
        n->sx = sx; n->stg = stg; n->vlast = vlast; n->dvp = dvp; n->loss = loss; n->part = part;
    }
    return (off + 255) / 256 * 256;
}

// ---- launch helpers -------------------------------------------------------
template <int MR, int NBW, int EPI, bool UP, bool FAR = false>
void conv_block(const ConvArgs& a, hipStream_t s)
{
    const Vol& g = a.g;
    const unsigned grid = (unsigned)((long)((g.W + CB_X - 1) / CB_X) * ((g.H + MR - 1) / MR) *
                                     ((g.D + CB_Z - 1) / CB_Z) * (a.cout / (16 * NBW)));
    if (a.cin == 16) k_conv<MR, NBW, 16, EPI, UP, FAR><<<grid, 256, 0, s>>>(a);
    else k_conv<MR, NBW, 32, EPI, UP, FAR><<<grid, 256, 0, s>>>(a);
}

// Blocks of 8 rows and 32 channels from 512 workgroups on (two per CU fit):
// with 2 rows the 64 -> 32 channel layer at 128^3 takes 332 instead of 262 us,
// 64 -> 64 at 64^3 85 instead of 64.  Below that 2 rows, with 32 channels
// from 768 workgroups on (128 -> 128 at 32^3: 49 us, 57 with 8 rows, 53 with
// 16 channels), else with 16 (64 -> 64 at 16^3: 19 us instead of 28 and, with
// 8 rows, 39).  Every block gives the same values.
template <int EPI, bool UP = false>
void conv(const ConvArgs& a, hipStream_t s)
{
    const Vol& g = a.g;
    const bool two = a.cout % 32 == 0;
    auto blocks = [&](int mr) {
        return (long)((g.W + CB_X - 1) / CB_X) * ((g.H + mr - 1) / mr) * ((g.D + CB_Z - 1) / CB_Z) *
               (a.cout / (two ? 32 : 16));
    };
    if (conv_far(a)) {
        if (two) conv_block<8, 2, EPI, UP, true>(a, s);
        else conv_block<8, 1, EPI, UP, true>(a, s);
    } else if (blocks(8) >= 512) {
        if (two) conv_block<8, 2, EPI, UP>(a, s);
        else conv_block<8, 1, EPI, UP>(a, s);
    } else if (two && blocks(2) >= 768) {
        conv_block<2, 2, EPI, UP>(a, s);
    } else {
        conv_block<2, 1, EPI, UP>(a, s);
    }
}

// Weight and bias gradients of all layers, deterministically: the partial sums
// of each kind of ring, the layers with the longest chunks first, then the sums.
void wgrad(const WgradArgs (&layers)[NL], hipStream_t s)
{
    auto table = [&](auto&& wgs) {
        WgradTable t{};
        for (const WgradArgs& a : layers)
            if (wgs(a) > 0) t.a[t.n++] = a;
        std::stable_sort(t.a, t.a + t.n, [](const WgradArgs& p, const WgradArgs& q) { return p.vchunk > q.vchunk; });
        for (int l = 0; l < t.n; ++l) t.first[l + 1] = t.first[l] + wgs(t.a[l]);
        return t;
    };
    auto launch = [&](auto kernel, const WgradTable& t, int threads) {
        if (t.n) kernel<<<(unsigned)t.first[t.n], threads, 0, s>>>(t);
    };
    auto kind = [&](int ci, int rows) {
        return table([=](const WgradArgs& a) { return a.ci == ci && a.rows == rows ? a.wgs : 0; });
    };
    launch(k_bias_grad, table([](const WgradArgs& a) { return a.nb; }), 256);
    launch(k_wgrad<2, 512, 1>, kind(2, 0), wg_threads(2));
    launch(k_wgrad<1, 512, 1>, kind(1, 0), wg_threads(1));
    launch(k_wgrad<1, 1024, 1>, kind(1, 1), wg_threads(1));
    launch(k_wgrad<1, 256, 3>, kind(1, 2), wg_threads(1));
    launch(k_wsum, table([](const WgradArgs& a) { return (int)(a.E / 128) + a.cout; }), 256);
}

void refresh_bf16(ep_net* n)
{
    WcopyTable t{};
    for (int l = 0; l < NL; ++l) {
        t.first[l + 1] = t.first[l] + (long)n->ch[l][1] * 27 * n->ch[l][0];
        t.woff[l] = n->woff[l];
        t.wboff[l] = n->wboff[l];
        t.co[l] = n->ch[l][1];
        t.ci[l] = n->ch[l][0];
    }
    k_wcopy<<<nblk(t.first[NL]), 256, 0, n->st>>>(t, n->w, n->wb, n->wtb);
}

const bf16_t* slot_x(const ep_net* n, int slot) { return slot < 0 ? n->xin : n->sx + (size_t)slot * n->g[0].Vp * 16; }
float* slot_t(const ep_net* n, int slot) { return n->stg + (size_t)slot * n->g[0].V * 4; }

// Convolution l of the network (its weights, or with back their transposed,
// mirrored form): X (level gx with UP, else g) -> Y, and Y2 from M where the
// epilogue has one.
template <int EPI, bool UP = false>
void layer(ep_net* n, int l, bool back, const bf16_t* X, void* Y, const Vol& g, const bf16_t* M = nullptr,
           bf16_t* Y2 = nullptr, const Vol* gx = nullptr)
{
    ConvArgs a;
    a.X = X;
    a.Wt = (back ? n->wtb : n->wb) + n->wboff[l];
    a.bias = back ? nullptr : n->w + n->boff[l];
    a.Y = Y;
    a.Y2 = Y2;
    a.M = M;
    a.cin = n->ch[l][back ? 1 : 0];
    a.cout = n->ch[l][back ? 0 : 1];
    a.g = g;
    a.gx = gx ? *gx : g;
    conv<EPI, UP>(a, n->st);
}

void forward(ep_net* n, const bf16_t* x)
{
    hipStream_t s = n->st;
    const Vol &g0 = n->g[0], &g1 = n->g[1], &g2 = n->g[2];
    const int C = n->cfg.base, C2 = 2 * C;
    layer<EPI_RELU>(n, 0, false, x, n->a0, g0);
    layer<EPI_RELU>(n, 1, false, n->a0, n->s0, g0);
    k_pool<<<nblk(g1.V * (C / 8)), 256, 0, s>>>(n->s0, n->p0, C, g0, g1);
    layer<EPI_RELU>(n, 2, false, n->p0, n->a1, g1);
    layer<EPI_RELU>(n, 3, false, n->a1, n->s1, g1);
    k_pool<<<nblk(g2.V * (C2 / 8)), 256, 0, s>>>(n->s1, n->p1, C2, g1, g2);
    layer<EPI_RELU>(n, 4, false, n->p1, n->a2, g2);
    layer<EPI_RELU>(n, 5, false, n->a2, n->b2, g2);
    layer<EPI_RELU_ADD, true>(n, 6, false, n->b2, n->r6, g1, n->s1, n->c1, &g2);
    layer<EPI_RELU>(n, 7, false, n->c1, n->d1, g1);
    layer<EPI_RELU_ADD, true>(n, 8, false, n->d1, n->r8, g0, n->s0, n->c0, &g1);
    layer<EPI_RELU>(n, 9, false, n->c0, n->d0, g0);
    layer<EPI_F32>(n, 10, false, n->d0, n->y, g0);
}

// Gradient of the loss of the current forward pass with respect to all
// parameters, in n->gr.
void backward(ep_net* n, const bf16_t* x)
{
    hipStream_t s = n->st;
    const Vol &g0 = n->g[0], &g1 = n->g[1], &g2 = n->g[2];
    const int C = n->cfg.base, C2 = 2 * C, C4 = 4 * C;
    // layer l's gradients from its input X and output gradient G, which both
    // stay until all are known
    WgradArgs grads[NL];
    float* part = n->part;
    auto weights = [&](int l, const bf16_t* X, const bf16_t* G, const Vol& g, const Vol* parent = nullptr) {
        WgradArgs& a = grads[l] = wgrad_plan(n->ch[l][1], n->ch[l][0], g);
        a.X = X;
        a.G = G;
        a.gx = parent ? *parent : g;
        a.up = parent != nullptr;
        a.part = part;
        a.bias = part += a.nch * a.E;
        part += (long)a.nb * a.cout;
        a.dW = n->gr + n->woff[l];
        a.db = n->gr + n->boff[l];
    };
    weights(10, n->d0, n->gy, g0);
    layer<EPI_MASK>(n, 10, true, n->gy, n->z9, g0, n->d0);
    weights(9, n->c0, n->z9, g0);
    layer<EPI_LIN_MASK>(n, 9, true, n->z9, n->gc0, g0, n->r8, n->z8);
    weights(8, n->d1, n->z8, g0, &g1);
    layer<EPI_LIN>(n, 8, true, n->z8, n->t0, g0);
    k_up_dx<<<nblk(g1.V * (C2 / 8)), 256, 0, s>>>(n->t0, n->d1, n->z7, C2, g0, g1);
    weights(7, n->c1, n->z7, g1);
    layer<EPI_LIN_MASK>(n, 7, true, n->z7, n->gc1, g1, n->r6, n->z6);
    weights(6, n->b2, n->z6, g1, &g2);
    layer<EPI_LIN>(n, 6, true, n->z6, n->t1, g1);
    k_up_dx<<<nblk(g2.V * (C4 / 8)), 256, 0, s>>>(n->t1, n->b2, n->z5, C4, g1, g2);
    weights(5, n->a2, n->z5, g2);
    layer<EPI_MASK>(n, 5, true, n->z5, n->z4, g2, n->a2);
    weights(4, n->p1, n->z4, g2);
    layer<EPI_LIN>(n, 4, true, n->z4, n->t2, g2);
    k_add_pool_dx<<<nblk(g1.V * (C2 / 8)), 256, 0, s>>>(n->gc1, n->t2, n->s1, n->z3, C2, g1, g2);
    weights(3, n->a1, n->z3, g1);
    layer<EPI_MASK>(n, 3, true, n->z3, n->z2, g1, n->a1);
    weights(2, n->p0, n->z2, g1);
    layer<EPI_LIN>(n, 2, true, n->z2, n->t3, g1);
    k_add_pool_dx<<<nblk(g0.V * (C / 8)), 256, 0, s>>>(n->gc0, n->t3, n->s0, n->z1, C, g0, g1);
    weights(1, n->a0, n->z1, g0);
    layer<EPI_MASK>(n, 1, true, n->z1, n->z0, g0, n->a0);
    weights(0, x, n->z0, g0);
    wgrad(grads, s);
}

float inv_count(const ep_net* n)
{
    const long nf = (long)(n->cfg.nx - 1) * n->cfg.ny * n->cfg.nz + (long)n->cfg.nx * (n->cfg.ny - 1) * n->cfg.nz +
                    (long)n->cfg.nx * n->cfg.ny * (n->cfg.nz - 1);
    return 1.f / (float)nf;
}

int loss_and_grad(ep_net* n, int slot, double* loss_out)
{
    hipStream_t s = n->st;
    const bf16_t* x = slot_x(n, slot);
    forward(n, x);
    const Vol& g0 = n->g[0];
    const unsigned nb = std::min(nblk(g0.V), 1024u);
    k_loss<<<nb, 256, 0, s>>>(n->y, slot_t(n, slot), n->gy, g0, n->cfg.nx, n->cfg.ny, n->cfg.nz, inv_count(n),
                              (double*)n->part);
    k_lsum<<<1, 256, 0, s>>>((const double*)n->part, (int)nb, n->loss);
    backward(n, x);
    if (loss_out) {
        NCHK(n, hipMemcpyAsync(loss_out, n->loss, 8, hipMemcpyDeviceToHost, s));
        NCHK(n, hipStreamSynchronize(s));
    }
    NCHK(n, hipGetLastError());
    return EP_OK;
}

SolverView view_of(const ep_handle* h)
{
    SolverView v;
    double* const* it = h->it64[h->cur64];
    v.txx = it[F_TXX]; v.tyy = it[F_TYY]; v.txy = it[F_TXY]; v.txz = it[F_TXZ]; v.tyz = it[F_TYZ];
    v.p = it[F_P]; v.epsp = h->epsp64;
    v.vx = it[F_VX]; v.vy = it[F_VY]; v.vz = it[F_VZ];
    v.nx = h->nx; v.ny = h->ny; v.nz = h->nz; v.sy = h->sy; v.sz = h->sz;
    return v;
}

int check_handle(ep_net* n, ep_handle* h)
{
    if (!h) return nerr(n, EP_EINVAL, "no solver handle");
    if (h->ndim != 3 || h->nx != n->cfg.nx || h->ny != n->cfg.ny || h->nz != n->cfg.nz)
        return nerr(n, EP_EINVAL, "solver grid %dx%dx%d does not match the network's %dx%dx%d", h->nx, h->ny, h->nz,
                    n->cfg.nx, n->cfg.ny, n->cfg.nz);
    ensure_it64(h);
    return EP_OK;
}

}  // namespace

// =========================================================================
extern "C" {

int ep_net_workspace_size(const ep_net_config* c, size_t* bytes)
{
    if (!bytes || validate_cfg(c) != EP_OK) return EP_EINVAL;
    *bytes = net_carve(c, nullptr, nullptr);
    return EP_OK;
}

int ep_net_init(const ep_net_config* c, void* d_workspace, size_t ws_bytes, void* stream, ep_net** out)
{
    if (!out) return EP_EINVAL;
    *out = nullptr;
    if (validate_cfg(c) != EP_OK) return EP_EINVAL;
    const size_t need = net_carve(c, nullptr, nullptr);
    if (!d_workspace || ws_bytes < need) return EP_ENOMEM;
    if (((uintptr_t)d_workspace & 255) != 0) return EP_EINVAL;
    ep_net* n = new (std::nothrow) ep_net();
    if (!n) return EP_ENOMEM;
    n->cfg = *c;
    n->st = (hipStream_t)stream;
    net_carve(c, n, (char*)d_workspace);
    auto fail = [&](int code) { delete n; return code; };
    if (hipMemsetAsync(d_workspace, 0, need, n->st) != hipSuccess) return fail(EP_EDEVICE);
    // He-normal initialisation (std sqrt(2 / (27 Cin))), zero biases, zero head
    std::vector<float> w(n->np, 0.f);
    std::mt19937_64 rng((unsigned long long)c->seed);
    std::normal_distribution<double> nd(0.0, 1.0);
    for (int l = 0; l < NL - 1; ++l) {
        const double sd = std::sqrt(2.0 / (27.0 * n->ch[l][0]));
        const long cnt = (long)n->ch[l][1] * 27 * n->ch[l][0];
        for (long q = 0; q < cnt; ++q) w[n->woff[l] + q] = (float)(nd(rng) * sd);
    }
    if (hipMemcpyAsync(n->w, w.data(), n->np * 4, hipMemcpyHostToDevice, n->st) != hipSuccess) return fail(EP_EDEVICE);
    refresh_bf16(n);
    if (hipStreamSynchronize(n->st) != hipSuccess || hipGetLastError() != hipSuccess) return fail(EP_EDEVICE);
    *out = n;
    return EP_OK;
}

void ep_net_destroy(ep_net* n) { delete n; }

const char* ep_net_last_error(const ep_net* n) { return n ? n->err : "no network"; }

long ep_net_param_count(const ep_net* n) { return n ? n->np : EP_EINVAL; }

int ep_net_params(ep_net* n, int dir, float* host, size_t count)
{
    if (!n || !host || (dir != EP_GET && dir != EP_SET)) return EP_EINVAL;
    if (count != (size_t)n->np) return nerr(n, EP_EINVAL, "count %zu, expected %ld", count, n->np);
    if (dir == EP_GET) {
        NCHK(n, hipMemcpyAsync(host, n->w, n->np * 4, hipMemcpyDeviceToHost, n->st));
    } else {
        NCHK(n, hipMemcpyAsync(n->w, host, n->np * 4, hipMemcpyHostToDevice, n->st));
        k_fill_f<<<nblk(n->np), 256, 0, n->st>>>(n->m, 0.f, n->np);
        k_fill_f<<<nblk(n->np), 256, 0, n->st>>>(n->v, 0.f, n->np);
        n->adam_t = 0;
        refresh_bf16(n);
    }
    NCHK(n, hipStreamSynchronize(n->st));
    NCHK(n, hipGetLastError());
    return EP_OK;
}

int ep_net_sample(ep_net* n, int slot, int dir, float* x, float* t)
{
    if (!n || slot < 0 || slot >= n->cfg.max_samples || (dir != EP_GET && dir != EP_SET)) return EP_EINVAL;
    const Vol& g = n->g[0];
    if (x) {
        bf16_t* dev = const_cast<bf16_t*>(slot_x(n, slot));
        std::vector<bf16_t> pad((size_t)g.Vp * 16, 0);
        if (dir == EP_GET) {
            NCHK(n, hipMemcpyAsync(pad.data(), dev, pad.size() * 2, hipMemcpyDeviceToHost, n->st));
            NCHK(n, hipStreamSynchronize(n->st));
        }
        for (int z = 0; z < g.D; ++z)
            for (int y = 0; y < g.H; ++y)
                for (int xx = 0; xx < g.W; ++xx) {
                    const long v = ((long)z * g.H + y) * g.W + xx;
                    const long p = (((long)z + 1) * g.Hp + y + 1) * g.Wp + xx + 1;
                    for (int c = 0; c < 16; ++c) {
                        if (dir == EP_GET) x[v * 16 + c] = host_bf2f(pad[p * 16 + c]);
                        else pad[p * 16 + c] = host_f2bf(x[v * 16 + c]);
                    }
                }
        if (dir == EP_SET) {
            NCHK(n, hipMemcpyAsync(dev, pad.data(), pad.size() * 2, hipMemcpyHostToDevice, n->st));
            NCHK(n, hipStreamSynchronize(n->st));
        }
    }
    if (t) {
        if (dir == EP_GET) NCHK(n, hipMemcpyAsync(t, slot_t(n, slot), g.V * 16, hipMemcpyDeviceToHost, n->st));
        else NCHK(n, hipMemcpyAsync(slot_t(n, slot), t, g.V * 16, hipMemcpyHostToDevice, n->st));
        NCHK(n, hipStreamSynchronize(n->st));
    }
    return EP_OK;
}

int ep_net_record(ep_net* n, ep_handle* h, int slot)
{
    if (!n || slot < -1 || slot >= n->cfg.max_samples) return EP_EINVAL;
    int rc = check_handle(n, h);
    if (rc) return rc;
    const Vol& g = n->g[0];
    k_features<<<nblk(g.V), 256, 0, n->st>>>(view_of(h), n->dvp, const_cast<bf16_t*>(slot_x(n, slot)), g,
                                             1.f / n->cfg.scale[0], 1.f / n->cfg.scale[1], 1.f / n->cfg.scale[2]);
    NCHK(n, hipGetLastError());
    return EP_OK;
}

int ep_net_observe(ep_net* n, ep_handle* h, int slot)
{
    if (!n || slot < -1 || slot >= n->cfg.max_samples) return EP_EINVAL;
    int rc = check_handle(n, h);
    if (rc) return rc;
    const Vol& g = n->g[0];
    k_observe<<<nblk(g.V), 256, 0, n->st>>>(view_of(h), n->vlast, n->dvp, slot >= 0 ? slot_t(n, slot) : nullptr, g,
                                            n->have_last ? 0 : 1, 1.f / n->cfg.scale[3]);
    n->have_last = true;
    NCHK(n, hipStreamSynchronize(n->st));
    NCHK(n, hipGetLastError());
    return EP_OK;
}

int ep_net_reset(ep_net* n)
{
    if (!n) return EP_EINVAL;
    n->have_last = false;
    return EP_OK;
}

int ep_net_forward(ep_net* n, int slot, float* y)
{
    if (!n || slot < -1 || slot >= n->cfg.max_samples) return EP_EINVAL;
    forward(n, slot_x(n, slot));
    if (y) NCHK(n, hipMemcpyAsync(y, n->y, n->g[0].V * COUT * 4, hipMemcpyDeviceToHost, n->st));
    NCHK(n, hipStreamSynchronize(n->st));
    NCHK(n, hipGetLastError());
    return EP_OK;
}

int ep_net_gradient(ep_net* n, int slot, double* loss, float* grad)
{
    if (!n || slot < 0 || slot >= n->cfg.max_samples) return EP_EINVAL;
    int rc = loss_and_grad(n, slot, loss);
    if (rc) return rc;
    if (grad) {
        NCHK(n, hipMemcpyAsync(grad, n->gr, n->np * 4, hipMemcpyDeviceToHost, n->st));
        NCHK(n, hipStreamSynchronize(n->st));
    }
    return EP_OK;
}

int ep_net_train(ep_net* n, const int* slots, int nslots, int nsteps, float lr, float* losses)
{
    if (!n || !slots || nslots <= 0 || nsteps < 0 || !(lr > 0)) return EP_EINVAL;
    for (int q = 0; q < nslots; ++q)
        if (slots[q] < 0 || slots[q] >= n->cfg.max_samples) return EP_EINVAL;
    for (int k = 0; k < nsteps; ++k) {
        double l = 0;
        int rc = loss_and_grad(n, slots[k % nslots], losses ? &l : nullptr);
        if (rc) return rc;
        if (losses) losses[k] = (float)l;
        ++n->adam_t;
        const float c1 = 1.f - std::pow(0.9f, (float)n->adam_t), c2 = 1.f - std::pow(0.999f, (float)n->adam_t);
        k_adam<<<nblk(n->np), 256, 0, n->st>>>(n->w, n->gr, n->m, n->v, n->np, lr, c1, c2);
        refresh_bf16(n);
    }
    NCHK(n, hipStreamSynchronize(n->st));
    NCHK(n, hipGetLastError());
    return EP_OK;
}

int ep_net_predict(ep_net* n, ep_handle* h)
{
    if (!n) return EP_EINVAL;
    int rc = ep_net_record(n, h, -1);
    if (rc) return rc;
    forward(n, n->xin);
    const long nf = (long)(h->nx + 1) * (h->ny + 1) * (h->nz + 1);
    k_apply_guess<<<nblk(nf), 256, 0, n->st>>>(view_of(h), n->y, h->vguess64[0], h->vguess64[1], h->vguess64[2],
                                               n->g[0], n->cfg.scale[3]);
    NCHK(n, hipGetLastError());
    h->guess_ready = true;
    return EP_OK;
}

}  // extern "C"

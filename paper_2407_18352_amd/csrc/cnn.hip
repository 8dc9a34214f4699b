// Convolutional surrogates on the composed tensor seen as images (Table IV
// model spaces: convolutions of a few channels for MiniWeather; convolution,
// max-pool and fully connected layers for ParticleFilter).
//
// Fused path (convolution-only stacks, SAME padding, stride 1, <= 16
// channels): one block owns a tile of TY x 64 output pixels of one image.  It
// gathers the tile plus the stack's total halo through the `to` map into LDS
// ([row][column][channel], channels padded to 4), then runs every layer over
// the shrinking region — each layer's output region is the next layer's
// input region — and writes the last layer's tile through the `from` map.
// Outside the image, a layer's input follows its padding mode: circular
// stacks wrap at the gather and then compute the halo as is (on a torus the
// halo's values equal the wrapped ones); zeros writes 0; replicate takes the
// pixel at the clamped position (inside the region, since the region always
// contains the image edge it crosses).  Two forms: on the matrix cores (exact
// splits of the floats, several pixels a column; the usual one), and on the
// vector ALU, with one thread per pixel, 16-byte LDS reads of its window and
// weights as wave-uniform scalar loads (one FMA per weight per lane), for
// stacks whose weights don't fit the LDS, large images with few
// multiplications, and tiles with values that have no split.
//
// Layer-by-layer path (everything else, and in-place regions): kernels over
// [S][h][w][c] tensors in a workspace -- convolutions (a max-pool with
// non-overlapping windows folded into the convolution before it), pools,
// fully connected layers (split K when the tiles alone are too few), and the
// fully connected layers closing a stack together with the scatter; else a
// scatter of the last tensor.
#include "cnn.hpp"
#include "mlp_f32.hpp"

namespace hpacml {

namespace {

constexpr int kThreads = 256;
constexpr int kTX = 64;   // tile columns

// ------------------------------------------------------------------ fused, vector ALU
struct FusedArgs {
    Map32 in, out;
    const FeatTable32 *tin, *tout;   // device; the used entries are staged in LDS
    int32_t S, H, W, n_layers;
    int32_t ty, tiles_x, tiles_y, n_tiles;
    int32_t c0, cout_last, circular, buf1;   // buf1: float offset of the second LDS buffer
    int32_t co_last_pad;                     // the last layer's channels, padded to 4
    // region of layer l's input (l = n_layers: the tile itself), relative to
    // the tile origin: rows [-rt, ty + rb), columns [-rl, 64 + rr)
    int32_t rt[kCnnFusedMaxLayers + 1], rl[kCnnFusedMaxLayers + 1];
    int32_t rh[kCnnFusedMaxLayers + 1], rw[kCnnFusedMaxLayers + 1];
    uint32_t rw_magic[kCnnFusedMaxLayers + 1];   // i / rw == (i * rw_magic) >> 24 for i < 2^16
    CnnFusedLayer L[kCnnFusedMaxLayers];
};

// Feature tables of the two maps in LDS (the first 16 entries): read with a
// wave-uniform index, so every lane gets the same pointer, without holding
// 16 pointers per map in scalar registers for the whole kernel.
struct TabLds {
    const float *in[kCnnFusedMaxC];
    float *out[kCnnFusedMaxC];
    uint32_t in_raw8[kCnnFusedMaxC], out_raw8[kCnnFusedMaxC];
};

__device__ __forceinline__ int div_region(int i, uint32_t magic) { return (int)(((uint32_t)i * magic) >> 24); }

__device__ __forceinline__ int wrap(int v, int n) {
    int r = v % n;
    return r < 0 ? r + n : r;
}

// Layer 0's input region from the `to` map: pixel (y, x) of image s is
// composed point (s * H + y) * W + x; channel f is its feature f.
template <int CI, int NT>
__device__ __forceinline__ void gather_region(const FusedArgs &a, const TabLds &tab, int s, int y0, int x0,
                                              float *dst) {
    const int rh = a.rh[0], rw = a.rw[0], n = rh * rw;
    const int mode = a.L[0].mode;
    const int vy0 = y0 - a.rt[0], vx0 = x0 - a.rl[0];
    for (int i = threadIdx.x; i < n; i += NT) {
        const int ry = div_region(i, a.rw_magic[0]), rx = i - ry * rw;
        int y = vy0 + ry, x = vx0 + rx;
        bool zero = false;
        if (y < 0 || y >= a.H || x < 0 || x >= a.W) {
            if (mode == HPACML_PADMODE_CIRCULAR) {
                y = wrap(y, a.H);
                x = wrap(x, a.W);
            } else {
                zero = mode == HPACML_PADMODE_ZEROS;
                y = min(max(y, 0), a.H - 1);
                x = min(max(x, 0), a.W - 1);
            }
        }
        const Pt32 pt = locate32(a.in, (s * a.H + y) * a.W + x);
        const uint32_t edge = edge_dims32(a.in, pt);
        float v[CI];
#pragma unroll
        for (int f = 0; f < CI; ++f) {
            v[f] = 0.f;
            if (f < a.c0) {
                const int fix = edge ? edge_fix32(a.in, pt, tab.in_raw8[f], edge) : 0;
                v[f] = ldg(tab.in[f] + (pt.pe + fix));
            }
        }
        float4 *d4 = reinterpret_cast<float4 *>(dst + (size_t)i * CI);
#pragma unroll
        for (int c4 = 0; c4 < CI / 4; ++c4)
            d4[c4] = zero ? make_float4(0.f, 0.f, 0.f, 0.f)
                          : make_float4(v[4 * c4], v[4 * c4 + 1], v[4 * c4 + 2], v[4 * c4 + 3]);
    }
}

// One layer's launch constants, read from the kernel arguments with constant
// indices (a kernel-argument array indexed at run time would be copied to
// private memory first).
struct LayerRun {
    CnnFusedLayer Ly;
    int oh, ow, sw;        // output region; input region row length
    uint32_t ow_magic;
    int rt, rl;            // output region origin relative to the tile
    int next_mode, last;
};

template <int l>
__device__ __forceinline__ LayerRun layer_run(const FusedArgs &a) {
    LayerRun r;
    r.Ly = a.L[l];
    r.oh = a.rh[l + 1];
    r.ow = a.rw[l + 1];
    r.sw = a.rw[l];
    r.ow_magic = a.rw_magic[l + 1];
    r.rt = a.rt[l + 1];
    r.rl = a.rl[l + 1];
    r.last = l == a.n_layers - 1;
    r.next_mode = (l + 1 < kCnnFusedMaxLayers && !r.last) ? a.L[l + 1 < kCnnFusedMaxLayers ? l + 1 : l].mode
                                                          : HPACML_PADMODE_ZEROS;
    return r;
}

// One layer over its output region (the next layer's input region, or the
// tile for the last layer) into LDS.  Each thread takes kPix pixels per pass
// (i, i + NT, ...): a weight loaded once feeds kPix FMAs.  Pixels
// outside the image get what the next layer's padding reads there (the last
// layer's are never stored).
template <int CIN4, int COUT4, int NT, int kPix>
__device__ __forceinline__ void conv_pass(const FusedArgs &a, const TabLds &tab, const LayerRun &r,
                                          const float *__restrict__ wts, const float *src, float *dst, int s, int y0,
                                          int x0) {
    constexpr int CI = 4 * CIN4, CO = 4 * COUT4;
    const CnnFusedLayer &Ly = r.Ly;
    const int oh = r.oh, ow = r.ow, sw = r.sw;
    const int vy0 = y0 - r.rt, vx0 = x0 - r.rl;
    const int next_mode = r.next_mode;
    const float *wl = wts + Ly.woff;
    const float *bl = wts + Ly.boff;
    const int kh = Ly.kh, kw = Ly.kw;
    const int n = oh * ow;
    for (int base = 0; base < n; base += NT * kPix) {
        int off[kPix];          // LDS float offset of each pixel's window origin
        bool valid[kPix], zero[kPix];
#pragma unroll
        for (int j = 0; j < kPix; ++j) {
            const int i = base + j * NT + (int)threadIdx.x;
            valid[j] = i < n;
            const int ic = valid[j] ? i : n - 1;
            int ry = div_region(ic, r.ow_magic), rx = ic - ry * ow;
            const int vy = vy0 + ry, vx = vx0 + rx;
            const bool outside = vy < 0 || vy >= a.H || vx < 0 || vx >= a.W;
            zero[j] = false;
            if (outside && !a.circular) {
                if (next_mode == HPACML_PADMODE_REPLICATE) {
                    ry = min(max(vy, 0), a.H - 1) - vy0;
                    rx = min(max(vx, 0), a.W - 1) - vx0;
                } else {
                    zero[j] = true;
                }
            }
            off[j] = (ry * sw + rx) * CI;
        }
        // output channels in groups of 4, one group at a time: a step (kx,
        // 4 input channels) then holds 16 weights in scalar registers, which
        // leaves the registers the pass's other uniform values need (larger
        // weight sets spilled them); the window is re-read from LDS per group
        const int nq = kw * CIN4;
#pragma unroll 1
        for (int og = 0; og < COUT4; ++og) {
            const float *wg = wl + og * kh * nq * 16;
            float acc[kPix][4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float bv = bl[4 * og + c];
#pragma unroll
                for (int j = 0; j < kPix; ++j)
                    acc[j][c] = bv;
            }
            for (int ky = 0; ky < kh; ++ky) {
                const float *wrow = wg + ky * nq * 16;
                const int rowoff = ky * sw * CI;
                for (int q = 0; q < nq; ++q) {
                    const float *wk = wrow + q * 16;
                    float4 v[kPix];
#pragma unroll
                    for (int j = 0; j < kPix; ++j)
                        v[j] = *reinterpret_cast<const float4 *>(src + off[j] + rowoff + 4 * q);
#pragma unroll
                    for (int ci = 0; ci < 4; ++ci)
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const float wv = wk[ci * 4 + c];
#pragma unroll
                            for (int j = 0; j < kPix; ++j) {
                                const float x = ci == 0 ? v[j].x : ci == 1 ? v[j].y : ci == 2 ? v[j].z : v[j].w;
                                acc[j][c] = fmaf(wv, x, acc[j][c]);
                            }
                        }
                }
            }
#pragma unroll
            for (int j = 0; j < kPix; ++j) {
                if (Ly.act == HPACML_ACT_RELU) {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        acc[j][c] = relu_arith(acc[j][c]);
                }
                if (!valid[j])
                    continue;
                const int i = base + j * NT + (int)threadIdx.x;
                reinterpret_cast<float4 *>(dst + (size_t)i * CO)[og] =
                    zero[j] ? make_float4(0.f, 0.f, 0.f, 0.f) : make_float4(acc[j][0], acc[j][1], acc[j][2], acc[j][3]);
            }
        }
    }
}

// The last layer's tile (LDS, [pixel][4 * cout4]) through the `from` map:
// pixel (y, x) of image s is point (s * H + y) * W + x, channel g its feature g.
template <int NT>
__device__ __forceinline__ void scatter_tile(const FusedArgs &a, const TabLds &tab, const float *src, int s, int y0,
                                             int x0) {
    const int CO = a.co_last_pad;
    const int n = a.ty * kTX;
    for (int i = threadIdx.x; i < n; i += NT) {
        const int ry = i / kTX, rx = i % kTX;
        const int y = y0 + ry, x = x0 + rx;
        if (y >= a.H || x >= a.W)
            continue;
        const Pt32 pt = locate32(a.out, (s * a.H + y) * a.W + x);
        const uint32_t edge = edge_dims32(a.out, pt);
        const float *v = src + (size_t)i * CO;
        for (int g = 0; g < a.cout_last; ++g) {
            const int fix = edge ? edge_fix32(a.out, pt, tab.out_raw8[g], edge) : 0;
            stg(tab.out[g] + (pt.pe + fix), v[g]);
        }
    }
}

template <int CIN4, int NT, int kPix>
__device__ __forceinline__ void conv_dispatch_out(const FusedArgs &a, const TabLds &tab, const LayerRun &r,
                                                  const float *__restrict__ wts, const float *src, float *dst, int s,
                                                  int y0, int x0) {
    switch (r.Ly.cout4) {
    case 1: conv_pass<CIN4, 1, NT, kPix>(a, tab, r, wts, src, dst, s, y0, x0); break;
    case 2: conv_pass<CIN4, 2, NT, kPix>(a, tab, r, wts, src, dst, s, y0, x0); break;
    case 3: conv_pass<CIN4, 3, NT, kPix>(a, tab, r, wts, src, dst, s, y0, x0); break;
    default: conv_pass<CIN4, 4, NT, kPix>(a, tab, r, wts, src, dst, s, y0, x0); break;
    }
}

__device__ __forceinline__ void stage_tab(const FusedArgs &a, TabLds &tab) {
    if (threadIdx.x < kCnnFusedMaxC) {
        const int f = threadIdx.x;
        tab.in[f] = a.tin->fptr[f];
        tab.in_raw8[f] = a.tin->raw8[f];
        tab.out[f] = const_cast<float *>(a.tout->fptr[f]);
        tab.out_raw8[f] = a.tout->raw8[f];
    }
}

// Layer 0's input region of a tile.
template <int NT>
__device__ __forceinline__ void gather_tile(const FusedArgs &a, const TabLds &tab, float *buf0, int s, int y0, int x0) {
    switch (a.L[0].cin4) {
    case 1: gather_region<4, NT>(a, tab, s, y0, x0, buf0); break;
    case 2: gather_region<8, NT>(a, tab, s, y0, x0, buf0); break;
    case 3: gather_region<12, NT>(a, tab, s, y0, x0, buf0); break;
    default: gather_region<16, NT>(a, tab, s, y0, x0, buf0); break;
    }
}

// One gathered tile by the vector ALU and NT threads, kPix pixels each at a time:
// every layer, scatter.
template <int NT, int kPix>
__device__ __forceinline__ void run_tile(const FusedArgs &a, const TabLds &tab, const float *__restrict__ wts,
                                         float *buf0, int s, int y0, int x0) {
    float *const buf1 = buf0 + a.buf1;
    __syncthreads();
    for (int l = 0; l < a.n_layers; ++l) {
        LayerRun r;
        switch (l) {
        case 0: r = layer_run<0>(a); break;
        case 1: r = layer_run<1>(a); break;
        case 2: r = layer_run<2>(a); break;
        default: r = layer_run<3>(a); break;
        }
        const float *src = (l & 1) ? buf1 : buf0;
        float *dst = (l & 1) ? buf0 : buf1;
        switch (r.Ly.cin4) {
        case 1: conv_dispatch_out<1, NT, kPix>(a, tab, r, wts, src, dst, s, y0, x0); break;
        case 2: conv_dispatch_out<2, NT, kPix>(a, tab, r, wts, src, dst, s, y0, x0); break;
        case 3: conv_dispatch_out<3, NT, kPix>(a, tab, r, wts, src, dst, s, y0, x0); break;
        default: conv_dispatch_out<4, NT, kPix>(a, tab, r, wts, src, dst, s, y0, x0); break;
        }
        __syncthreads();
    }
    scatter_tile<NT>(a, tab, (a.n_layers & 1) ? buf1 : buf0, s, y0, x0);
}

__global__ void __launch_bounds__(kThreads) cnn_fused_kernel(FusedArgs a, const float *__restrict__ wts) {
    extern __shared__ float4 lds4[];
    float *const buf0 = reinterpret_cast<float *>(lds4);
    __shared__ TabLds tab;
    stage_tab(a, tab);
    __syncthreads();

    // blocks of one XCD (blockIdx % 8) take a contiguous range of tiles, so
    // neighbouring tiles share their halo rows in that XCD's L2
    const int32_t k0 = blockIdx.x;
    const int32_t xq = a.n_tiles / 8, xr = a.n_tiles % 8, xx = k0 % 8;
    const int32_t tile = xx * xq + (xx < xr ? xx : xr) + k0 / 8;
    const int32_t per_img = a.tiles_y * a.tiles_x;
    const int s = tile / per_img;
    const int rem = tile - s * per_img;
    const int ty_i = rem / a.tiles_x;
    const int y0 = ty_i * a.ty, x0 = (rem - ty_i * a.tiles_x) * kTX;

    gather_tile<kThreads>(a, tab, buf0, s, y0, x0);
    run_tile<kThreads, 1>(a, tab, wts, buf0, s, y0, x0);
}

// ------------------------------------------------------------------ fused, matrix cores
// The same tiles with the convolutions on the bf16 matrix cores, every float
// as the exact sum of three bf16 parts (see mlp_f32.hip: six products, hi hi
// accumulated apart; values outside the range of that arithmetic send their
// tile to the vector ALU path above).
//
// A few channels would fill a quarter of a matrix instruction's rows, so P
// neighbouring output pixels of a row share one column of it: rows = (pixel of
// the group, output channel), columns = 32 (16) groups, K = (window row, the
// kw + P - 1 input pixels the group's windows span, channel).  A weight that a
// pixel's window doesn't reach is zero (a Toeplitz band: kw of kw + P - 1).
// With channels last the K of one window row is contiguous in LDS, so a lane's
// 8 values of K are one 16-byte read per part.  Four output channels take
// 16 x 16 x 32 instructions with P = 4, more of them 32 x 32 x 16 with P = 32 /
// channels.
//
// One block of 8 waves per CU loops over tiles: weights of all layers stay in
// LDS (staged once), the layers' inputs as three bf16 planes [row][column]
// [channel]; the next tile's pixels are requested while the current tile's
// layers run (one-group inputs).  The last layer goes straight from the
// accumulators through the `from` map.
//
// Measured, matrix cores / vector ALU: 4 -> 8 -> 4 channels, 5 x 5 and 3 x 3 on 2048 x
// 2048: 174-181 / 299 us, on 512 x 512 16.4 / 33.3, on 64 x 64 11.4 / 33.2; 6 x 6 and 5 x 5
// on 1426 x 1867: 178 / 465 us.  Error against 64 bits 1.2e-7 / 3.2e-7.  What bounds
// it: of 26 thousand cycles a tile of 16 rows the first layer's column tiles take 8
// (matrix instructions 3.8 of them, LDS reads as much), the second's 6, and the
// gather's address arithmetic, splits and barriers most of the rest.
//
// NaN pixels (a land mask) go on in this form: 0 in the planes and a bit a pixel,
// and the outputs whose window reaches one are put right after the first layer.
// 2048 x 2048 as above with a NaN in every tile: 227 us, on 1024 x 1024 with 2 x 2 and
// 2 x 2 on 4 channels 47 (each such tile on the vector ALU after the matrix cores: 570,
// 64).  A tile with other values outside the range takes 2 to 2.4 times as long.
constexpr int kMThreads = 512, kMWaves = 8;
constexpr size_t kMStatic = 2048;        // LDS beside the image and the planes (tables, arguments, flags)
constexpr int kPre = 4;                  // pixels per thread requested ahead
constexpr int kFallPix = 3;              // pixels per thread at a time where a tile goes to the vector ALU
constexpr int kNanWords = 5;             // words of a row of NaN bits: 128 columns, and one to read past them
struct ConvM {
    int32_t cout, m16, P, ci, co;        // output channels; 16-row form; pixels per group; padded channels in, out
    int32_t steps, rch, chunks;          // K-steps; 8-value chunks per window row, and in all
    // A row of a plane in 16-byte chunks: a group starts S chunks after its
    // neighbour, so chunk k is kept at place (k % S) sub + k / S: the same chunk
    // of neighbouring groups is then contiguous (no bank conflicts)
    int32_t S, inv, sub;                 // k / S == (k * inv) >> 16
    int32_t row_b;                       // bytes of a plane's row of the input buffer
    int32_t in_off, in_plane;            // the input's planes: byte offset in LDS, bytes per plane
    int32_t out_off, out_plane, out_row_b, out_S, out_inv, out_sub;
    int32_t a_off, bias_off;             // weights and bias in LDS
    int32_t ng, oh, groups;              // groups per row, rows, groups of the output region
    uint32_t ng_magic;                   // i / ng == (i * ng_magic) >> 24
    int32_t relu, next_mode, rt, rl;     // what the next layer's padding reads outside; region origin
    int32_t tab_off;                     // this layer's chunk offsets in LDS (steps x chunks a step)
    int32_t kh, kw;
};
struct MfmaArgs {
    FusedArgs f;
    ConvM c[kCnnFusedMaxLayers];
    const void *image;                   // device: biases and fragments of every layer
    float limit, least;                  // of the layers' inputs and the outputs (see split_range)
    int32_t tiny;                        // a weight loses bits
    int32_t image_bytes, planes_off, planes_bytes;   // LDS: image, then planes,
    int32_t clear_bytes;                 // then NaN bits (with the planes)
    int32_t nan_off, nan_bytes;          // LDS: the gathered region's NaN bits (0: a NaN sends the tile to the vector ALU)
    int32_t pre;                         // the next tile is requested ahead
    int32_t in_rank, out_rank, in_offsets, out_offsets;
    int32_t imaged;                      // the sweep's last two dimensions are the image's (a snapshot record's are not)
    int32_t ys, yd, yst, xs, xd, xst;    // sweep rows and columns: start, step, element stride
    int32_t o_imaged;                    // the same of the `from` map, with one image
    int32_t oys, oyd, oyst, oxs, oxd, oxst;
    int32_t grid_x;                      // blocks per XCD
};

// A wave-uniform word of the block's LDS copy of the kernel arguments.  The
// arguments are far more than the scalar registers hold over the kernel's
// phases, and reading them again from memory costs microseconds (they lie in
// host memory: 7 thousand cycles a phase as measured).
__device__ __forceinline__ int32_t uni(const int32_t &v) { return __builtin_amdgcn_readfirstlane(v); }

// The arguments where they lie (scalar loads), for the start and for rare paths.
__device__ __forceinline__ const MfmaArgs &mfma_args() {
    const __attribute__((address_space(4))) void *p =
        (const __attribute__((address_space(4))) void *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const MfmaArgs *)(const __attribute__((address_space(4))) MfmaArgs *)p;
}

static_assert(sizeof(MfmaArgs) + sizeof(TabLds) + 3 * kMWaves * 4 <= kMStatic, "static LDS");

// v0..v3 split into the three planes at byte `at` (four bf16 each).
__device__ __forceinline__ void put4(char *base, int plane, int at, float v0, float v1, float v2, float v3) {
    uint32_t q[3][2];
    split2(v0, v1, q[0][0], q[1][0], q[2][0]);
    split2(v2, v3, q[0][1], q[1][1], q[2][1]);
#pragma unroll
    for (int p = 0; p < 3; ++p)
        *reinterpret_cast<uint2 *>(base + at + p * plane) = make_uint2(q[p][0], q[p][1]);
}

// Byte e of a plane's row (see ConvM).
__device__ __forceinline__ int row_spot(int e, int S, int inv, int sub) {
    const int k = e >> 4, q = (k * inv) >> 16;
    return ((k - q * S) * sub + q) * 16 + (e & 15);
}

// Region pixel i of layer 0's input at tile (s, y0, x0): element index of its
// sweep point and where its boundary handling leaves it.
struct GPix {
    Pt32 pt;
    bool zero;
};
__device__ __forceinline__ GPix region_pixel(const MfmaArgs &m, int i, int s, int y0, int x0, int32_t lead_pe,
                                             const int32_t (&lead)[2], bool inside) {
    const FusedArgs &a = m.f;
    const int ry = div_region(i, a.rw_magic[0]), rx = i - ry * a.rw[0];
    int y = y0 - a.rt[0] + ry, x = x0 - a.rl[0] + rx;
    GPix g;
    g.zero = false;
    if (!inside && (y < 0 || y >= a.H || x < 0 || x >= a.W)) {
        if (a.L[0].mode == HPACML_PADMODE_CIRCULAR) {
            y = wrap(y, a.H);
            x = wrap(x, a.W);
        } else {
            g.zero = a.L[0].mode == HPACML_PADMODE_ZEROS;
            y = min(max(y, 0), a.H - 1);
            x = min(max(x, 0), a.W - 1);
        }
    }
    if (!m.imaged) {
        g.pt = locate32(a.in, (s * a.H + y) * a.W + x);
        return g;
    }
    // the sweep's last two dimensions are the image rows and columns
    const int r = m.in_rank;
    const int yy = m.ys + y * m.yd, xx = m.xs + x * m.xd;
    g.pt.pe = lead_pe + yy * m.yst + xx * m.xst;
    g.pt.p[0] = r == 2 ? yy : lead[0];
    g.pt.p[1] = r == 2 ? xx : r == 3 ? yy : lead[1];
    g.pt.p[2] = r == 2 ? 0 : r == 3 ? xx : yy;
    g.pt.p[3] = r == 4 ? xx : 0;
    return g;
}

// row m0 < 32 of a 32-row tile: pixel of the group (channels padded to co >= 8)
__device__ __forceinline__ int pixel_of(int m0, int co) { return (m0 >= co) + (m0 >= 2 * co) + (m0 >= 3 * co); }

template <bool M16>
struct AccOf {
    typedef floatx16 type;
};
template <>
struct AccOf<true> {
    typedef floatx4 type;
};
__device__ __forceinline__ floatx16 mma(u32x4 a, u32x4 b, floatx16 c) { return mfma(a, b, c); }
__device__ __forceinline__ floatx4 mma(u32x4 a, u32x4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// What a lane met in a tile.
struct Seen {
    Range hidden;                  // the layers' inputs but the first's
    uint32_t in2 = 0;              // the first's largest: bits shifted past the sign (infinities and NaN above all); tested apart
    uint32_t low = 0xFFFFFFFFu;    // the least input of any layer but 0: the same bits, less 1 (0 comes last)
    float out = FLT_MAX;           // the least output
    __device__ __forceinline__ void add_low(float v) { low = min(low, (__float_as_uint(v) << 1) - 1u); }
    // bit 0: the matrix form may not serve this tile; bit 1: nor if bit 2 (a
    // value lost bits) is set as well, in any wave of the block
    __device__ __forceinline__ uint32_t flags(float limit, float least) const {
        return (__any(hidden.outside(limit)) ? 1u : 0u) | (__any(out < least) ? 2u : 0u) |
               (__any(low < (__float_as_uint(kLeast) << 1) - 1u) ? 4u : 0u);
    }
};

// Whether a window of the first layer, at the gathered region's row and column,
// holds a NaN pixel.
__device__ __forceinline__ bool window_nan(const uint32_t *rows, int row, int col, int kh, int kw) {
    uint32_t any = 0;
    for (int ky = 0; ky < kh; ++ky) {
        const uint32_t *r = rows + (row + ky) * kNanWords + (col >> 5);
        any |= __builtin_amdgcn_alignbit(r[1], r[0], col & 31);
    }
    return (any & ((1u << kw) - 1u)) != 0;
}

// One layer of the tile: this wave's share of the groups.
template <bool M16, bool LAST>
__device__ __forceinline__ void conv_mfma(const MfmaArgs &m, int l, char *lds, const TabLds &tab, int wave, int lane, int s, int y0, int x0,
                                          Seen &seen) {
    typedef typename AccOf<M16>::type Acc;
    // columns; chunks per K-step; register quads; column tiles at a time (they
    // share the weights' fragments, and the short 16-row tiles need company)
    constexpr int N = M16 ? 16 : 32, KC = M16 ? 4 : 2, Q = M16 ? 1 : 4, T = M16 ? 2 : 1;
    const ConvM &c = m.c[l];   // (m in LDS)
    const int n = lane % N, kc = lane / N;
    const int groups = uni(c.groups), ng = uni(c.ng), row_b = uni(c.row_b), plane = uni(c.in_plane), steps = uni(c.steps);
    const int co = uni(c.co), P = uni(c.P), group_b = 16;
    const uint32_t ng_magic = (uint32_t)uni((const int32_t &)c.ng_magic);
    const char *in = lds + uni(c.in_off);
    const char *wl = lds + uni(c.a_off) + lane * 16;
    const int32_t *offs = reinterpret_cast<const int32_t *>(lds + uni(c.tab_off)) + kc;
    const float *bias = reinterpret_cast<const float *>(lds + uni(c.bias_off));
    const float floor = act_floor(uni(c.relu));
    const int H = uni(m.f.H), W = uni(m.f.W), rt = uni(c.rt), rl = uni(c.rl);
    const int out_S = uni(c.out_S), out_inv = uni(c.out_inv), out_sub = uni(c.out_sub);
    const int out_off = uni(c.out_off), out_plane = uni(c.out_plane), out_row_b = uni(c.out_row_b), cout = uni(c.cout);
    const bool circular = uni(m.f.circular), imaged = uni(m.o_imaged), offsets = uni(m.out_offsets);
    const int oys = uni(m.oys), oyd = uni(m.oyd), oyst = uni(m.oyst), oxs = uni(m.oxs), oxd = uni(m.oxd), oxst = uni(m.oxst);
    const int out_rank = uni(m.out_rank);
    for (int t = wave; t * N * T < groups; t += kMWaves) {
        int ry[T], gx[T];
        const char *base[T];
        Acc main[T], s0[T], s1[T];
#pragma unroll
        for (int u = 0; u < T; ++u) {
            const int gi = min((t * T + u) * N + n, groups - 1);
            ry[u] = (int)(((uint32_t)gi * ng_magic) >> 24);
            gx[u] = gi - ry[u] * ng;
            base[u] = in + ry[u] * row_b + gx[u] * group_b;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int m0 = M16 ? 4 * kc : 8 * q + 4 * kc;
                const int c0 = M16 ? 0 : m0 - pixel_of(m0, co) * co;
                const float4 b4 = *reinterpret_cast<const float4 *>(bias + c0);
                main[u][4 * q] = b4.x;
                main[u][4 * q + 1] = b4.y;
                main[u][4 * q + 2] = b4.z;
                main[u][4 * q + 3] = b4.w;
            }
#pragma unroll
            for (int r = 0; r < 4 * Q; ++r)
                s0[u][r] = s1[u][r] = 0.f;
        }
        // K-steps two at a time: the fragments of one are read during the other
        u32x4 b[2][T][3], w[2][3];
        int off = offs[0];
        auto fetch = [&](int st, u32x4 (&bb)[T][3], u32x4 (&ww)[3]) __attribute__((always_inline)) {
            const char *q = wl + st * (3 * kFragBytes);
#pragma unroll
            for (int u = 0; u < T; ++u) {
                const char *p = base[u] + off;
                bb[u][0] = *reinterpret_cast<const u32x4 *>(p);
                bb[u][1] = *reinterpret_cast<const u32x4 *>(p + plane);
                bb[u][2] = *reinterpret_cast<const u32x4 *>(p + 2 * plane);
            }
            ww[0] = *reinterpret_cast<const u32x4 *>(q);
            ww[1] = *reinterpret_cast<const u32x4 *>(q + kFragBytes);
            ww[2] = *reinterpret_cast<const u32x4 *>(q + 2 * kFragBytes);
            off = offs[(st + 1) * KC];   // (the table ends with a spare step)
        };
        // (the two sums of small products in turn, also from one K-step to the
        // next: no instruction waits for the one before it)
        auto step = [&](const u32x4 (&bb)[T][3], const u32x4 (&ww)[3], Acc (&p0)[T], Acc (&p1)[T])
                        __attribute__((always_inline)) {
            __builtin_amdgcn_sched_barrier(kSchedAluOnly);
            auto product = [&](Acc (&d)[T], int x, int y) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < T; ++u)
                    d[u] = mma(ww[x], bb[u][y], d[u]);
                __builtin_amdgcn_sched_barrier(kSchedAluOnly);
            };
            product(p0, 0, 1);
            product(p1, 0, 2);
            product(main, 0, 0);
            product(p0, 1, 0);
            product(p1, 1, 1);
            product(p0, 2, 0);
        };
        fetch(0, b[0], w[0]);
        int st = 1;
        for (; st + 1 < steps; st += 2) {
            fetch(st, b[1], w[1]);
            step(b[0], w[0], s0, s1);
            fetch(st + 1, b[0], w[0]);
            step(b[1], w[1], s1, s0);
        }
        if (st < steps) {
            fetch(st, b[1], w[1]);
            step(b[0], w[0], s0, s1);
            step(b[1], w[1], s1, s0);
        } else {
            step(b[0], w[0], s0, s1);
        }
#pragma unroll
        for (int u = 0; u < T; ++u) {
            const bool live = (t * T + u) * N + n < groups;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int m0 = M16 ? 4 * kc : 8 * q + 4 * kc;
                const int px = M16 ? kc : pixel_of(m0, co), c0 = M16 ? 0 : m0 - px * co;
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    v[e] = main[u][4 * q + e] + (s0[u][4 * q + e] + s1[u][4 * q + e]);
                if (!LAST) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        v[e] = __builtin_amdgcn_fmed3f(v[e], floor, FLT_MAX);
                        seen.add_low(v[e]);
                    }
                    seen.hidden.add(v[0], v[1]);
                    seen.hidden.add(v[2], v[3]);
                }
                const int col = gx[u] * P + px;
                const int y = y0 - rt + ry[u], x = x0 - rl + col;
                if (LAST) {
                    if (live && px < P && y < H && x < W) {
                        Pt32 pt;
                        if (imaged) {
                            pt.p[0] = oys + y * oyd;
                            pt.p[1] = oxs + x * oxd;
                            pt.p[2] = pt.p[3] = 0;
                            pt.pe = pt.p[0] * oyst + pt.p[1] * oxst;
                        } else {
                            pt = locate_lds(m.f.out, out_rank, (s * H + y) * W + x);
                        }
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            if (c0 + e < cout) {
                                int32_t idx[1] = {pt.pe};
                                if (offsets) {
                                    const uint32_t raw[1] = {tab.out_raw8[c0 + e]};
                                    fix_lds<1>(m.f.out, pt, 15u, raw, idx);
                                }
                                seen.out = fminf(seen.out, fabsf(v[e]));
                                stg(tab.out[c0 + e] + idx[0], __builtin_amdgcn_fmed3f(v[e], floor, FLT_MAX));
                            }
                        }
                    }
                } else {
                    const bool outside = !circular && (y < 0 || y >= H || x < 0 || x >= W);
                    if (live && px < P) {
                        if (outside)
                            v[0] = v[1] = v[2] = v[3] = 0.f;   // (replicate: copied over afterwards)
                        put4(lds + out_off, out_plane, ry[u] * out_row_b + row_spot((col * co + c0) * 2, out_S, out_inv, out_sub), v[0],
                             v[1], v[2], v[3]);
                    }
                }
            }
        }
    }
}

// Replicate padding of the next layer: pixels of this layer's output region
// outside the image take the value at the nearest pixel inside (which the
// region always contains).
__device__ __forceinline__ void replicate_edges(const MfmaArgs &m, const ConvM &c, char *lds, int y0, int x0) {
    const FusedArgs &a = m.f;
    const int cols = c.ng * c.P, n = c.oh * cols;
    for (int i = threadIdx.x; i < n; i += kMThreads) {
        const int ry = i / cols, rx = i - ry * cols;
        const int y = y0 - c.rt + ry, x = x0 - c.rl + rx;
        const int qy = min(max(y, 0), a.H - 1) - y, qx = min(max(x, 0), a.W - 1) - x;
        if (qy == 0 && qx == 0)
            continue;
        for (int e = 0; e < c.co / 4; ++e) {
            const int d = c.out_off + ry * c.out_row_b + row_spot(rx * c.co * 2 + 8 * e, c.out_S, c.out_inv, c.out_sub);
            const int from = c.out_off + (ry + qy) * c.out_row_b +
                             row_spot((rx + qx) * c.co * 2 + 8 * e, c.out_S, c.out_inv, c.out_sub);
            for (int p = 0; p < 3; ++p)
                *reinterpret_cast<uint2 *>(lds + d + p * c.out_plane) =
                    *reinterpret_cast<const uint2 *>(lds + from + p * c.out_plane);
        }
    }
}

// NaN pixels among a tile's inputs are 0 in the planes: after the first layer the
// outputs that they reach become what they are, 0 after a ReLU ahead of another
// layer (the planes), NaN or 0 in the last (the arrays).
__device__ __forceinline__ void nan_outputs(const MfmaArgs &m, const TabLds &tab, char *lds, int s, int y0, int x0) {
    const FusedArgs &a = m.f;
    const ConvM &c = m.c[0];
    const uint32_t *rows = reinterpret_cast<const uint32_t *>(lds + m.nan_off);
    const bool last = a.n_layers == 1;
    const int cols = a.rw[1], n = c.oh * cols;
    for (int i = threadIdx.x; i < n; i += kMThreads) {
        const int ry = div_region(i, a.rw_magic[1]), rx = i - ry * cols;
        const int y = y0 + ry, x = x0 + rx;
        if (!window_nan(rows, ry, rx, c.kh, c.kw) || (last && (y >= a.H || x >= a.W)))
            continue;
        if (!last) {
            for (int e = 0; e < c.co / 4; ++e) {
                const int d = c.out_off + ry * c.out_row_b + row_spot(rx * c.co * 2 + 8 * e, c.out_S, c.out_inv, c.out_sub);
                for (int p = 0; p < 3; ++p)
                    *reinterpret_cast<uint2 *>(lds + d + p * c.out_plane) = make_uint2(0u, 0u);
            }
            continue;
        }
        const Pt32 pt = locate32(a.out, (s * a.H + y) * a.W + x);
        const uint32_t edge = edge_dims32(a.out, pt);
        for (int g = 0; g < a.cout_last; ++g) {
            const int fix = edge ? edge_fix32(a.out, pt, tab.out_raw8[g], edge) : 0;
            stg(tab.out[g] + (pt.pe + fix), c.relu ? 0.f : __builtin_nanf(""));
        }
    }
}

__global__ void __launch_bounds__(kMThreads, 2) cnn_fused_mfma_kernel(MfmaArgs, const float *__restrict__ wts) {
    extern __shared__ float4 lds4[];
    char *lds = reinterpret_cast<char *>(lds4);
    __shared__ TabLds tab;
    __shared__ MfmaArgs args_lds;
    auto local = [&]() __attribute__((always_inline)) -> const MfmaArgs & {
        int z = 0;
        asm volatile("" : "+v"(z));   // read where it is used, not held in registers
        return *reinterpret_cast<const MfmaArgs *>(reinterpret_cast<const char *>(&args_lds) + z);
    };
    __shared__ uint32_t flags[3][kMWaves];   // after a tile's gather, after its layers (see Seen) and after a second look at its inputs, per wave
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    auto clear = [&](int off, int bytes) {
        for (int i = tid; i < bytes / 16; i += kMThreads)
            reinterpret_cast<u32x4 *>(lds + off)[i] = u32x4{0u, 0u, 0u, 0u};
    };
    int n_tiles, n_layers, n_pix, grid_x, pre_on, nan_off;
    uint32_t limit2, tiny;
    float limit, least;
    {
        const MfmaArgs &m = mfma_args();
        for (int i = tid; i < (int)(sizeof(MfmaArgs) / 4); i += kMThreads)
            reinterpret_cast<int32_t *>(&args_lds)[i] = reinterpret_cast<const int32_t *>(&m)[i];
        stage_tab(m.f, tab);
        for (int i = tid; i < m.image_bytes / 16; i += kMThreads)
            reinterpret_cast<u32x4 *>(lds)[i] = reinterpret_cast<const u32x4 *>(m.image)[i];
        // byte offset of each chunk of K in a group's window (window row, place
        // in it); past the last chunk the weights are zero and any place will do
        for (int l = 0; l < m.f.n_layers; ++l) {
            const int kcs = m.c[l].m16 ? 4 : 2, rch = m.c[l].rch, chunks = m.c[l].chunks;
            int32_t *t = reinterpret_cast<int32_t *>(lds + m.c[l].tab_off);
            for (int i = tid; i < (m.c[l].steps + 1) * kcs; i += kMThreads)
                t[i] = i < chunks ? i / rch * m.c[l].row_b + row_spot(i % rch * 16, m.c[l].S, m.c[l].inv, m.c[l].sub) : 0;
        }
        n_tiles = m.f.n_tiles;
        n_layers = m.f.n_layers;
        n_pix = m.f.rh[0] * m.f.rw[0];
        grid_x = m.grid_x;
        pre_on = m.pre;
        nan_off = m.nan_off;
        limit = m.limit;
        least = m.least;
        limit2 = __float_as_uint(limit) << 1;
        tiny = m.tiny ? 4u : 0u;
    }
    clear(mfma_args().planes_off, mfma_args().clear_bytes);   // columns past the gathered ones are read (with zero weights): they must be finite (NaN bits behind them)
    __syncthreads();

    // each XCD takes a contiguous range of tiles, its blocks adjacent ones
    const int per = (n_tiles + 7) / 8, xcd = blockIdx.x % 8;
    const int t_end = min(n_tiles, (xcd + 1) * per);
    auto locate_tile = [&](const FusedArgs &a, int tile, int &s, int &y0, int &x0) {
        const int tx = uni(a.tiles_x), per_img = uni(a.tiles_y) * tx;
        s = tile / per_img;
        const int rem = tile - s * per_img, ty_i = rem / tx;
        y0 = ty_i * uni(a.ty);
        x0 = (rem - ty_i * tx) * kTX;
    };
    // element index and coordinates of the leading sweep dimensions of image s
    auto lead_of = [&](const MfmaArgs &m, int s, int32_t (&lead)[2]) -> int32_t {
        const Map32 &in = m.f.in;
        int32_t pe = 0;
        const int rank = uni(m.imaged) ? uni(m.in_rank) : 0;
        lead[0] = lead[1] = 0;
        if (rank == 3) {
            lead[0] = uni(in.start[0]) + s * uni(in.step[0]);
            pe = lead[0] * uni(in.stride[0]);
        } else if (rank == 4) {
            const int n1 = uni(in.count[1]), q = s / n1;
            lead[0] = uni(in.start[0]) + q * uni(in.step[0]);
            lead[1] = uni(in.start[1]) + (s - q * n1) * uni(in.step[1]);
            pe = lead[0] * uni(in.stride[0]) + lead[1] * uni(in.stride[1]);
        }
        return pe;
    };
    auto inside_of = [&](const FusedArgs &a, int y0, int x0) {
        const int y = y0 - uni(a.rt[0]), x = x0 - uni(a.rl[0]);
        return y >= 0 && x >= 0 && y + uni(a.rh[0]) <= uni(a.H) && x + uni(a.rw[0]) <= uni(a.W);
    };
    auto load4 = [&](const MfmaArgs &m, const GPix &g, int c4, float (&v)[4]) __attribute__((always_inline)) {
        const FusedArgs &a = m.f;
        const int ch = uni(a.c0);
        const uint32_t edge = uni(m.in_offsets) ? edge_lds(a.in, uni(m.in_rank), g.pt) : 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int f = 4 * c4 + e;
            v[e] = 0.f;
            if (f < ch) {
                int32_t idx[1] = {g.pt.pe};
                if (edge) {
                    const uint32_t raw[1] = {tab.in_raw8[f]};
                    fix_lds<1>(a.in, g.pt, edge, raw, idx);
                }
                v[e] = ldg(tab.in[f] + idx[0]);
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            v[e] = g.zero ? 0.f : v[e];
    };
    // the pixels that this thread requests ahead: element offset from the
    // region's first pixel, place in the planes (the same for every tile)
    float pre[kPre][4];
    int32_t rel[kPre], place[kPre];
    if (pre_on) {
        const MfmaArgs &m = mfma_args();
#pragma unroll
        for (int u = 0; u < kPre; ++u) {
            const int i = min(tid + u * kMThreads, n_pix - 1);
            const int ry = div_region(i, m.f.rw_magic[0]), rx = i - ry * m.f.rw[0];
            rel[u] = ry * m.yd * m.yst + rx * m.xd * m.xst;
            place[u] = m.c[0].in_off + ry * m.c[0].row_b + row_spot(rx * m.c[0].ci * 2, m.c[0].S, m.c[0].inv, m.c[0].sub);
        }
    }
    uint32_t zeros = 0;   // bit u: pixel u is zero padding
    auto request = [&](int tile) __attribute__((always_inline)) {
        const MfmaArgs &m = local();
        int s, y0, x0;
        locate_tile(m.f, tile, s, y0, x0);
        int32_t lead[2], at[kPre];
        const int32_t pe = lead_of(m, s, lead);
        zeros = 0;
        if (inside_of(m.f, y0, x0) && uni(m.imaged)) {
            const int32_t b = pe + (uni(m.ys) + (y0 - uni(m.f.rt[0])) * uni(m.yd)) * uni(m.yst) +
                              (uni(m.xs) + (x0 - uni(m.f.rl[0])) * uni(m.xd)) * uni(m.xst);
#pragma unroll
            for (int u = 0; u < kPre; ++u)
                at[u] = b + rel[u];
        } else {
#pragma unroll
            for (int u = 0; u < kPre; ++u) {
                const GPix g = region_pixel(m, min(tid + u * kMThreads, n_pix - 1), s, y0, x0, pe, lead, false);
                at[u] = g.pt.pe;
                zeros |= g.zero ? 1u << u : 0u;
            }
        }
        // (nothing here waits for a load: padding and missing channels are
        // zeroed when the values are used)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float *p = tab.in[e];   // (entries past the last channel repeat it)
#pragma unroll
            for (int u = 0; u < kPre; ++u)
                if (u * kMThreads < n_pix)
                    pre[u][e] = ldg(p + at[u]);
        }
    };
    const int first = xcd * per + blockIdx.x / 8;
    if (pre_on && first < t_end)
        request(first);
    for (int tile = first; tile < t_end; tile += grid_x) {
        int s, y0, x0;
        Seen seen;
        locate_tile(local().f, tile, s, y0, x0);
        // the tile's pixels: f(byte of the planes, bytes of one plane, region pixel, four channels)
        auto pixels = [&](auto &&f) __attribute__((always_inline)) {
            const MfmaArgs &m = local();
            const int plane = uni(m.c[0].in_plane), ch = uni(m.f.c0);
            if (pre_on) {
#pragma unroll
                for (int u = 0; u < kPre; ++u) {
                    if (tid + u * kMThreads < n_pix) {
                        float v[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            v[e] = (zeros >> u & 1u) || e >= ch ? 0.f : pre[u][e];
                        f(place[u], plane, tid + u * kMThreads, v);
                    }
                }
            } else {
                const int in_off = uni(m.c[0].in_off), row_b = uni(m.c[0].row_b), ci = uni(m.c[0].ci), rw = uni(m.f.rw[0]);
                const uint32_t rw_magic = (uint32_t)uni((const int32_t &)m.f.rw_magic[0]);
                const int S0 = uni(m.c[0].S), inv0 = uni(m.c[0].inv), sub0 = uni(m.c[0].sub);
                int32_t lead[2];
                const int32_t pe = lead_of(m, s, lead);
                const bool inside = inside_of(m.f, y0, x0);
                for (int i = tid; i < n_pix; i += kMThreads) {
                    const GPix g = region_pixel(m, i, s, y0, x0, pe, lead, inside);
                    const int ry = div_region(i, rw_magic), rx = i - ry * rw;
                    for (int c4 = 0; c4 < ci / 4; ++c4) {
                        float v[4];
                        load4(m, g, c4, v);
                        f(in_off + ry * row_b + row_spot((rx * ci + 4 * c4) * 2, S0, inv0, sub0), plane, i, v);
                    }
                }
            }
        };
        pixels([&](int at, int plane, int, float (&v)[4]) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                seen.in2 = max(seen.in2, __float_as_uint(v[e]) << 1);
                seen.add_low(v[e]);
            }
            put4(lds, plane, at, v[0], v[1], v[2], v[3]);
        });
        // the block's flags: each wave writes its own ahead of a barrier
        auto collect = [&](uint32_t (&f)[kMWaves], uint32_t mine) __attribute__((always_inline)) {
            if (lane == 0)
                f[wave] = mine;
            __syncthreads();
            uint32_t all = 0;
#pragma unroll
            for (int w = 0; w < kMWaves; ++w)
                all |= f[w];
            return (uint32_t)__builtin_amdgcn_readfirstlane(all);
        };
        uint32_t met = collect(flags[0], __any(seen.in2 >= limit2) ? 1u : 0u);
        bool vector = false, gathered = false;
        if (met) {
            // an input too large for the split products, or a NaN: these become 0
            // in the planes, and a bit; with the others, or without the bits, the
            // tile goes to the vector ALU at once, its requested pixels with it
            seen.in2 = 0;
            bool nan = false;
            pixels([&](int at, int plane, int i, float (&v)[4]) __attribute__((always_inline)) {
                bool here = false;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    here = here || v[e] != v[e];
                    v[e] = v[e] != v[e] ? 0.f : v[e];
                    seen.in2 = max(seen.in2, __float_as_uint(v[e]) << 1);
                }
                if (here && nan_off) {
                    put4(lds, plane, at, v[0], v[1], v[2], v[3]);
                    const FusedArgs &a = local().f;
                    const int ry = div_region(i, a.rw_magic[0]), rx = i - ry * a.rw[0];
                    atomicOr(reinterpret_cast<uint32_t *>(lds + nan_off) + ry * kNanWords + (rx >> 5), 1u << (rx & 31));
                }
                nan = nan || here;
            });
            met = collect(flags[2], (__any(seen.in2 >= limit2) ? 1u : 0u) | (__any(nan) ? 2u : 0u));
            vector = (met & 1u) || !nan_off;
            gathered = vector && pre_on;
            if (gathered) {
                float4 *buf0 = reinterpret_cast<float4 *>(lds + mfma_args().planes_off);
                pixels([&](int, int, int i, float (&v)[4]) __attribute__((always_inline)) { buf0[i] = make_float4(v[0], v[1], v[2], v[3]); });
            }
        }
        if (pre_on && tile + grid_x < t_end)
            request(tile + grid_x);
        if (!vector) {
            for (int l = 0; l + 1 < n_layers; ++l) {
                const MfmaArgs &m = local();
                if (uni(m.c[l].m16))
                    conv_mfma<true, false>(m, l, lds, tab, wave, lane, s, y0, x0, seen);
                else
                    conv_mfma<false, false>(m, l, lds, tab, wave, lane, s, y0, x0, seen);
                __syncthreads();
                if (l == 0 && met) {
                    nan_outputs(mfma_args(), tab, lds, s, y0, x0);
                    __syncthreads();
                }
                if (uni(m.c[l].next_mode) == HPACML_PADMODE_REPLICATE) {
                    replicate_edges(m, m.c[l], lds, y0, x0);
                    __syncthreads();
                }
            }
            {
                const MfmaArgs &m = local();
                if (uni(m.c[n_layers - 1].m16))
                    conv_mfma<true, true>(m, n_layers - 1, lds, tab, wave, lane, s, y0, x0, seen);
                else
                    conv_mfma<false, true>(m, n_layers - 1, lds, tab, wave, lane, s, y0, x0, seen);
            }
            // (also the barrier after the last reads of this tile's planes)
            const uint32_t all = collect(flags[1], seen.flags(limit, least) | tiny);
            vector = (all & 1u) || (all & 6u) == 6u;
            if (n_layers == 1 && met && !vector)
                nan_outputs(mfma_args(), tab, lds, s, y0, x0);
        }
        if (vector) {
            const MfmaArgs &m = mfma_args();
            float *buf0 = reinterpret_cast<float *>(lds + m.planes_off);
            if (!gathered)
                gather_tile<kMThreads>(m.f, tab, buf0, s, y0, x0);
            run_tile<kMThreads, kFallPix>(m.f, tab, wts, buf0, s, y0, x0);
            __syncthreads();
            clear(m.planes_off, m.planes_bytes);
            __syncthreads();
        }
        if ((met & 2u) && nan_off) {
            __syncthreads();
            clear(nan_off, uni(local().nan_bytes));
            __syncthreads();
        }
    }
}

// LDS floats of the two buffers for tiles of `ty` rows.
void fused_regions(const CnnFused &f, int ty, FusedArgs *a, size_t *floats0, size_t *floats1) {
    const int L = f.n_layers;
    a->rt[L] = a->rl[L] = 0;
    int rb = 0, rr = 0;
    a->rh[L] = ty;
    a->rw[L] = kTX;
    size_t b0 = 0, b1 = 0;
    // the last layer's output tile
    ((L & 1) ? b1 : b0) = (size_t)ty * kTX * 4 * f.L[L - 1].cout4;
    for (int l = L - 1; l >= 0; --l) {
        const CnnFusedLayer &y = f.L[l];
        a->rt[l] = a->rt[l + 1] + y.top;
        a->rl[l] = a->rl[l + 1] + y.left;
        rb += y.kh - 1 - y.top;
        rr += y.kw - 1 - y.left;
        a->rh[l] = ty + a->rt[l] + rb;
        a->rw[l] = kTX + a->rl[l] + rr;
        const size_t fl = (size_t)a->rh[l] * a->rw[l] * 4 * y.cin4;
        if (l & 1)
            b1 = std::max(b1, fl);
        else
            b0 = std::max(b0, fl);
    }
    *floats0 = b0;
    *floats1 = b1;
}

// tile buffers of at most 40 KB leave room for four blocks (16 waves) per CU:
// measured faster than 64 KB tiles with two blocks, the recomputed halo
// notwithstanding
constexpr size_t kLdsShared = 40 * 1024;
constexpr size_t kLdsOneBlock = 160 * 1024;

// ------------------------------------------------------------------ layers
// One thread per output pixel and group of kConvG output channels
// (blockIdx.y).  Weights packed [group][ky][kx][ci][kConvG], zero past cout:
// in the channels-last image the taps of one window row are one contiguous
// run of kw * cin floats.  Taps go in chunks of kTapChunk whose input loads are
// all issued before the first product.  A wave whose windows all lie inside the
// image multiplies on the fp32 matrix instruction of sixteen 4 x 4 blocks:
// columns = the wave's 64 pixels, rows = 4 output channels, one tap per
// instruction, the block of A broadcast to the others (sixteen taps' weights for
// 4 channels in one register): twice the vector ALU's rate and beside its index
// arithmetic.  A wave with a window that leaves the image (SAME padding at the
// border) works on the vector ALU, its weights as wave-uniform scalar loads, each
// tap resolved through the padding mode.  Measured: 4 x 4, 8 channels, 2 x 2 pool on 1024
// frames of 128 x 128: 21.0 -> 17.0 us (67 MB of frames: 4.5 TB/s with the output); the
// whole model with 2 x 2 windows 91.7 -> 75 us, 7 x 7 and a 3 x 3 pool 49.7 -> 42.4.  What
// bounds it: memory latency at a tile per wave, and its index arithmetic.
//
// With POOL, a max-pool whose windows do not overlap follows in the same
// kernel, so the convolution's output never goes to memory: a group of
// 2^QS adjacent lanes holds one pooled pixel, lane q computing window
// position q (lanes past the window repeat position 0), and the group's
// maximum comes from pairwise exchanges.  Each step keeps the lower
// lane's value unless the other is larger or a NaN, and a NaN once taken
// stays: the window's first NaN, else its first maximum, as in the pool
// kernel.  In a step the two lanes share the channels between them, so the
// next one has half as many to exchange (7 in all for four lanes' 8 channels
// where every lane reducing all of them takes 16), and the lanes of a group
// store their channels side by side.
constexpr int kTapChunk = 16;

// One chunk's products: v[j] = this lane's value of tap t0 + j, a register of
// weights for each four channels (see conv_pixel).
__device__ __forceinline__ void conv_taps(const float (&v)[kTapChunk], int left, float w0, float w1, floatx4 &a0,
                                          floatx4 &a1) {
    static_for<0, kTapChunk / 4>([&](auto jj) __attribute__((always_inline)) {
        constexpr int j = 4 * jj;
        if (j < left) {   // taps past the last are zeros in both operands
            static_for<0, 4>([&](auto ii) __attribute__((always_inline)) {
                constexpr int t = j + ii;
                a0 = __builtin_amdgcn_mfma_f32_4x4x1f32(w0, v[t], a0, 4, t, 0);
                a1 = __builtin_amdgcn_mfma_f32_4x4x1f32(w1, v[t], a1, 4, t, 0);
            });
        }
    });
}

// Convolution outputs (bias, taps, activation) of output pixel (oy, ox).  Called
// by whole waves.
__device__ __forceinline__ void conv_pixel(const CnnLayerDev &L, const float *img, const float *__restrict__ wg,
                                           int oy, int ox, int ng, float (&acc)[kConvG]) {
    static_assert(kConvG == 8 && kTapChunk == 16, "two registers of sixteen taps' weights");
    const int y0 = oy * L.sh - (L.same ? (L.kh - 1) / 2 : 0);
    const int x0 = ox * L.sw - (L.same ? (L.kw - 1) / 2 : 0);
    const int taps = L.kh * L.kw * L.cin;
#pragma unroll
    for (int g = 0; g < kConvG; ++g)
        acc[g] = g < ng ? L.b[blockIdx.y * kConvG + g] : 0.f;
    if (__all(y0 >= 0 && x0 >= 0 && y0 + L.kh <= L.h && x0 + L.kw <= L.w)) {
        const float *base = img + ((int64_t)y0 * L.w + x0) * L.cin;
        const int run = L.kw * L.cin;                 // floats of one window row
        const int64_t rs = (int64_t)L.w * L.cin;      // image row stride
        const int lane = threadIdx.x & 63;
        // weights of tap t0 + lane / 4, channels lane % 4 and 4 + lane % 4
        const float *wl = wg + (lane >> 2) * kConvG + (lane & 3);
        floatx4 a0 = {acc[0], acc[1], acc[2], acc[3]}, a1 = {acc[4], acc[5], acc[6], acc[7]};
        const bool vec = run % 4 == 0 && rs % 4 == 0 && __all(((uintptr_t)base & 15) == 0);
        int ky = 0, r = 0;
        for (int t0 = 0; t0 < taps; t0 += kTapChunk) {
            const bool in = t0 + (lane >> 2) < taps;
            const float w0 = in ? wl[t0 * kConvG] : 0.f, w1 = in ? wl[t0 * kConvG + 4] : 0.f;
            float v[kTapChunk];
            if (vec) {
                // window rows of whole, aligned float4s: 16-byte loads
#pragma unroll
                for (int j = 0; j < kTapChunk; j += 4) {
                    const float4 q = t0 + j < taps ? *reinterpret_cast<const float4 *>(base + ky * rs + r)
                                                   : make_float4(0.f, 0.f, 0.f, 0.f);
                    v[j] = q.x;
                    v[j + 1] = q.y;
                    v[j + 2] = q.z;
                    v[j + 3] = q.w;
                    r += 4;
                    if (r == run) {
                        r = 0;
                        ++ky;
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < kTapChunk; ++j) {
                    v[j] = t0 + j < taps ? base[ky * rs + r] : 0.f;
                    if (++r == run) {
                        r = 0;
                        ++ky;
                    }
                }
            }
            conv_taps(v, taps - t0, w0, w1, a0, a1);
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            acc[g] = a0[g];
            acc[4 + g] = a1[g];
        }
    } else {
        for (int ky = 0; ky < L.kh; ++ky) {
            int y = y0 + ky;
            bool zy = false;
            if (y < 0 || y >= L.h) {
                if (L.mode == HPACML_PADMODE_CIRCULAR)
                    y = wrap(y, L.h);
                else if (L.mode == HPACML_PADMODE_REPLICATE)
                    y = min(max(y, 0), L.h - 1);
                else
                    zy = true;
            }
            for (int kx = 0; kx < L.kw; ++kx) {
                int x = x0 + kx;
                bool z = zy;
                if (x < 0 || x >= L.w) {
                    if (L.mode == HPACML_PADMODE_CIRCULAR)
                        x = wrap(x, L.w);
                    else if (L.mode == HPACML_PADMODE_REPLICATE)
                        x = min(max(x, 0), L.w - 1);
                    else
                        z = true;
                }
                if (z)
                    continue;
                const float *px = img + ((int64_t)y * L.w + x) * L.cin;
                const float *wk = wg + (int64_t)(ky * L.kw + kx) * L.cin * kConvG;
                for (int ci = 0; ci < L.cin; ++ci) {
                    const float v = px[ci];
#pragma unroll
                    for (int g = 0; g < kConvG; ++g)
                        acc[g] = fmaf(wk[ci * kConvG + g], v, acc[g]);
                }
            }
        }
    }
#pragma unroll
    for (int g = 0; g < kConvG; ++g)
        acc[g] = L.act == HPACML_ACT_RELU ? (acc[g] > 0.f ? acc[g] : 0.f) : acc[g];
}

__device__ __forceinline__ uint32_t fdiv(uint32_t i, uint32_t magic, uint32_t shift) {
    return (uint32_t)(((uint64_t)i * magic) >> shift);
}

// The value of lane l ^ D (neighbours within four lanes without LDS).
template <int D>
__device__ __forceinline__ float lane_xor(float v) {
    if (D <= 2)
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), D == 1 ? 0xB1 : 0x4E, 0xf, 0xf, true));
    return __shfl_xor(v, D);
}

// Maximum of acc[0, N) over the lanes l, l ^ D, ... of the 2^QS-lane groups.
// While more than one channel is left a lane keeps half of them: the lower of
// a pair the first half.  Returns in `c0` the first channel the lane ends up with.
template <int D, int END, int N>
__device__ __forceinline__ void group_max(int q, float (&acc)[kConvG], int &c0) {
    if constexpr (D < END) {
        constexpr int H = N > 1 ? N / 2 : 1;
        const bool lower = (q & D) == 0;
#pragma unroll
        for (int g = 0; g < H; ++g) {
            const float mine = N > 1 && !lower ? acc[H + g] : acc[g];
            const float give = N > 1 && lower ? acc[H + g] : acc[g];
            const float o = lane_xor<D>(give);
            const float a = lower ? mine : o, b = lower ? o : mine;
            acc[g] = (!(a != a) && (b != b || b > a)) ? b : a;
        }
        if (N > 1 && !lower)
            c0 += H;
        group_max<2 * D, END, H>(q, acc, c0);
    }
}

template <bool POOL, int QS>
__global__ void __launch_bounds__(256) cnn_conv_kernel(CnnLayerDev L, CnnLayerDev P, const float *__restrict__ in,
                                                      float *__restrict__ out, int64_t n_pix) {
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t pix = POOL ? tid >> QS : tid;
    // (every lane takes part in the matrix instructions and the exchanges)
    const int64_t pc = pix < n_pix ? pix : n_pix - 1;
    const int co0 = blockIdx.y * kConvG;
    const int ng = min(kConvG, L.cout - co0);
    const CnnLayerDev &G = POOL ? P : L;   // the grid of output pixels
    int ox, oy;
    int64_t s;
    if (n_pix <= INT32_MAX) {
        // 32-bit divisions by multiply-shift (a 64-bit division is a long
        // instruction sequence, and this kernel is VALU-bound)
        const uint32_t q1 = fdiv((uint32_t)pc, G.w2_magic, G.w2_shift);
        const uint32_t q2 = fdiv(q1, G.h2_magic, G.h2_shift);
        ox = (int)((uint32_t)pc - q1 * (uint32_t)G.w2);
        oy = (int)(q1 - q2 * (uint32_t)G.h2);
        s = q2;
    } else {
        ox = (int)(pc % G.w2);
        oy = (int)(pc / G.w2 % G.h2);
        s = pc / ((int64_t)G.w2 * G.h2);
    }
    const int q = POOL ? (int)(tid & ((1 << QS) - 1)) : 0;
    if (POOL) {
        // window position qq < 16 of a window kw <= 16 wide: (qq + 1/2) / kw
        // lies at least 1/32 from an integer, so the approximate reciprocal
        // gives the exact quotient
        const int qq = q < P.kh * P.kw ? q : 0;
        const int qy = (int)(((float)qq + 0.5f) * __builtin_amdgcn_rcpf((float)P.kw));
        oy = oy * P.sh + qy;
        ox = ox * P.sw + (qq - qy * P.kw);
    }
    const float *img = in + s * L.h * L.w * L.cin;
    const float *__restrict__ wg = L.W + (int64_t)blockIdx.y * L.kh * L.kw * L.cin * kConvG;
    float acc[kConvG];
    conv_pixel(L, img, wg, oy, ox, ng, acc);
    if (POOL) {
        constexpr int C = kConvG >> QS ? kConvG >> QS : 1;   // channels a lane ends up with
        int c0 = 0;
        group_max<1, 1 << QS, kConvG>(q, acc, c0);
        if (pix >= n_pix || q >= kConvG)   // (16 lanes: the last 8 hold the same as the first)
            return;
        float *o = out + pix * L.cout + co0 + c0;
#pragma unroll
        for (int g = 0; g < C; ++g)
            acc[g] = P.act == HPACML_ACT_RELU ? (acc[g] > 0.f ? acc[g] : 0.f) : acc[g];
        if (C == 2 && c0 + 2 <= ng && ((uintptr_t)o & 7) == 0) {
            *reinterpret_cast<float2 *>(o) = make_float2(acc[0], acc[1]);
        } else if (C >= 4 && c0 + C <= ng && ((uintptr_t)o & 15) == 0) {
#pragma unroll
            for (int g = 0; g + 3 < C; g += 4)
                *reinterpret_cast<float4 *>(o + g) = make_float4(acc[g], acc[g + 1], acc[g + 2], acc[g + 3]);
        } else {
#pragma unroll
            for (int g = 0; g < C; ++g)
                if (c0 + g < ng)
                    o[g] = acc[g];
        }
        return;
    }
    if (pix >= n_pix)
        return;
    float *o = out + pix * L.cout + co0;
    if (ng == kConvG && ((uintptr_t)o & 15) == 0) {
        *reinterpret_cast<float4 *>(o) = make_float4(acc[0], acc[1], acc[2], acc[3]);
        *reinterpret_cast<float4 *>(o + 4) = make_float4(acc[4], acc[5], acc[6], acc[7]);
    } else {
        for (int g = 0; g < ng; ++g)
            o[g] = acc[g];
    }
}

__global__ void __launch_bounds__(256) cnn_pool_kernel(CnnLayerDev L, const float *__restrict__ in,
                                                      float *__restrict__ out, int64_t total) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total)
        return;
    const int c = (int)(idx % L.cout);
    const int64_t pix = idx / L.cout;
    const int ox = (int)(pix % L.w2);
    const int oy = (int)(pix / L.w2 % L.h2);
    const int64_t s = pix / ((int64_t)L.w2 * L.h2);
    const float *win = in + ((s * L.h + (int64_t)oy * L.sh) * L.w + (int64_t)ox * L.sw) * L.cin + c;
    // the largest window value; a NaN anywhere in the window wins
    float m = win[0];
    for (int ky = 0; ky < L.kh; ++ky)
        for (int kx = 0; kx < L.kw; ++kx) {
            const float v = win[((int64_t)ky * L.w + kx) * L.cin];
            if (!(m != m) && (v != v || v > m))
                m = v;
        }
    out[idx] = L.act == HPACML_ACT_RELU ? (m > 0.f ? m : 0.f) : m;
}

// Fully connected layer over S images: out[S][O] = in[S][K] W^T + b.  A block
// owns a T x T output tile (T = 64: 4 x 4 outputs per thread; T = 16 for
// layers of at most 16 outputs, one output per thread), K in chunks staged in
// LDS k-major, coalesced loads along k.
// Split-K: block z of gridDim.z sums k in [z Kc, (z+1) Kc) and, when
// gridDim.z > 1, writes its raw partial sums to part[z][S][O] (a reduce kernel
// adds them in z order, then bias and activation).
template <int T>
__global__ void __launch_bounds__(256) cnn_linear_kernel(CnnLayerDev L, const float *__restrict__ in,
                                                        float *__restrict__ out, int64_t S, int64_t Kc,
                                                        float *__restrict__ part) {
    constexpr int R = T / 16;                 // outputs per thread per dimension
    constexpr int KC = 256 * 4 / T;           // k per chunk: each thread loads 4 values per operand
    __shared__ float xs[KC][T + 4];
    __shared__ float ws[KC][T + 4];
    const int t = threadIdx.x;
    const int64_t s0 = (int64_t)blockIdx.x * T;
    const int o0 = blockIdx.y * T;
    const int O = L.cout;
    const int64_t K = (int64_t)L.h * L.w * L.cin;
    const int ti = t / 16, tj = t % 16;
    const int64_t kb = (int64_t)blockIdx.z * Kc;
    const int64_t ke = kb + Kc < K ? kb + Kc : K;
    float acc[R][R] = {};
    // T rows x KC columns of each operand per chunk: thread t loads column
    // t % KC of rows t / KC + (256 / KC) m, into registers one chunk ahead
    const int c = t % KC;
    float xr[4], wr[4];
    auto fetch = [&](int64_t k0) {
        const int64_t k = k0 + c;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int r = t / KC + (256 / KC) * m;
            const int64_t sr = s0 + r;
            const int o = o0 + r;
            xr[m] = (sr < S && k < ke) ? in[sr * K + k] : 0.f;
            wr[m] = (o < O && k < ke) ? L.W[(int64_t)o * K + k] : 0.f;
        }
    };
    if (kb < ke)
        fetch(kb);
    for (int64_t k0 = kb; k0 < ke; k0 += KC) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int r = t / KC + (256 / KC) * m;
            xs[c][r] = xr[m];
            ws[c][r] = wr[m];
        }
        __syncthreads();
        if (k0 + KC < ke)
            fetch(k0 + KC);
#pragma unroll 8
        for (int kk = 0; kk < KC; ++kk) {
            float a[R], b[R];
#pragma unroll
            for (int i = 0; i < R; ++i) {
                a[i] = xs[kk][R * ti + i];
                b[i] = ws[kk][R * tj + i];
            }
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
                for (int j = 0; j < R; ++j)
                    acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int64_t sr = s0 + R * ti + i;
        if (sr >= S)
            continue;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int o = o0 + R * tj + j;
            if (o < O) {
                if (gridDim.z > 1) {
                    part[((int64_t)blockIdx.z * S + sr) * O + o] = acc[i][j];
                } else {
                    const float v = acc[i][j] + L.b[o];
                    out[sr * O + o] = L.act == HPACML_ACT_RELU ? (v > 0.f ? v : 0.f) : v;
                }
            }
        }
    }
}

// The products of a fully connected layer with more than 16 outputs whose K
// is split over blocks, on fp32 MFMA (v_mfma_f32_32x32x2f32): the transposed
// product C[o][s] = sum_k W[o][k] in[s][k], weights as the A operand (32
// outputs x 2 k per m-block), images as B (32 images x 2 k).  A block of 4
// waves owns 128 images (32 per wave) x 64 outputs (2 m-blocks) and one K
// range; K goes in chunks of kMfK staged in LDS (rows padded to kMfK + 1
// floats: lane l reads row l % 32 at column k + l / 32, conflict-free),
// loaded one chunk ahead in registers.  Lane l ends up holding image l % 32
// and, in register r of m-block mb, output 32 mb + 8 (r / 4) + 4 (l / 32) +
// r % 4: four consecutive outputs per group of registers, stored as one
// 16-byte write of the raw partial sums part[z][s][o].
constexpr int kMfS = 128, kMfO = 64, kMfK = 32;

__global__ void __launch_bounds__(256) cnn_linear_mfma_kernel(CnnLayerDev L, const float *__restrict__ in, int64_t S,
                                                             int64_t Kc, float *__restrict__ part) {
    __shared__ float xs[kMfS][kMfK + 1];
    __shared__ float ws[kMfO][kMfK + 1];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t s0 = (int64_t)blockIdx.x * kMfS;
    const int o0 = blockIdx.y * kMfO;
    const int O = L.cout;
    const int64_t K = (int64_t)L.h * L.w * L.cin;
    const int64_t kb = (int64_t)blockIdx.z * Kc;
    const int64_t ke = kb + Kc < K ? kb + Kc : K;
    // chunk loads: thread t takes column t % 32 of rows t / 32 + 8 m
    const int c = t % kMfK, r0 = t / kMfK;
    float xr[kMfS / 8], wr[kMfO / 8];
    auto fetch = [&](int64_t k0) {
        const int64_t k = k0 + c;
        const bool kin = k < ke;
#pragma unroll
        for (int m = 0; m < kMfS / 8; ++m) {
            const int64_t sr = s0 + r0 + 8 * m;
            xr[m] = (kin && sr < S) ? in[sr * K + k] : 0.f;
        }
#pragma unroll
        for (int m = 0; m < kMfO / 8; ++m) {
            const int o = o0 + r0 + 8 * m;
            wr[m] = (kin && o < O) ? L.W[(int64_t)o * K + k] : 0.f;
        }
    };
    floatx16 acc[2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            acc[mb][r] = 0.f;
    if (kb < ke)
        fetch(kb);
    const int col = lane & 31, kh = lane >> 5;
    for (int64_t k0 = kb; k0 < ke; k0 += kMfK) {
#pragma unroll
        for (int m = 0; m < kMfS / 8; ++m)
            xs[r0 + 8 * m][c] = xr[m];
#pragma unroll
        for (int m = 0; m < kMfO / 8; ++m)
            ws[r0 + 8 * m][c] = wr[m];
        __syncthreads();
        if (k0 + kMfK < ke)
            fetch(k0 + kMfK);
#pragma unroll
        for (int kk = 0; kk < kMfK; kk += 2) {
            const float b = xs[32 * w + col][kk + kh];
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
                acc[mb] = __builtin_amdgcn_mfma_f32_32x32x2f32(ws[32 * mb + col][kk + kh], b, acc[mb], 0, 0, 0);
        }
        __syncthreads();
    }
    const int64_t s = s0 + 32 * w + col;
    if (s >= S)
        return;
    float *dst = part + ((int64_t)blockIdx.z * S + s) * O;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int o = o0 + 32 * mb + 8 * q + 4 * kh;
            if (o + 3 < O && ((uintptr_t)(dst + o) & 15) == 0) {
                *reinterpret_cast<float4 *>(dst + o) =
                    make_float4(acc[mb][4 * q], acc[mb][4 * q + 1], acc[mb][4 * q + 2], acc[mb][4 * q + 3]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (o + i < O)
                        dst[o + i] = acc[mb][4 * q + i];
            }
        }
}

// The same products where the images are few (see split_few): a block owns 32
// images x 64 outputs and one K range, its four waves a quarter of the range
// each, in steps of 32 k: loads one step ahead (eight lanes to 128 bytes of a
// row) go through the wave's own part of the LDS, without a barrier, to
// fragments (lane l: k of half l / 32 of the step; the two halves' k pair up in
// an instruction).  The waves' sums meet in LDS in wave
// order, so a K range is four times as long as a 128-image block's for as many
// blocks, and a quarter as many partial sums go through memory.  What bounds
// it is the latency of one round of blocks, not the matrix cores.  VEC: rows of
// whole, aligned float4s (others read theirs unaligned: 1024 x 4095 -> 256 35 us; one
// by one they took 49, the 128-image kernel 42).
constexpr int kFewS = 32, kFewRows = kFewS + kMfO;
constexpr int kFewPad = kMfK + 4;   // floats a staged row: 16 rows read at once lie in 64 different banks
template <bool VEC>
__global__ void __launch_bounds__(256) cnn_linear_few_kernel(CnnLayerDev L, const float *__restrict__ in, int64_t S,
                                                            int64_t Kc, float *__restrict__ part) {
    __shared__ __align__(16) float lds[4 * kFewRows * kFewPad];
    auto red = reinterpret_cast<float(*)[kFewS][kMfO + 4]>(lds);   // after the products
    static_assert(4 * kFewS * (kMfO + 4) <= 4 * kFewRows * kFewPad, "the sums fit where the rows were");
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int col = lane & 31, kh = lane >> 5;
    const int O = L.cout;
    const int64_t s0 = (int64_t)blockIdx.x * kFewS;
    const int o0 = blockIdx.y * kMfO;
    const int64_t K = (int64_t)L.h * L.w * L.cin;
    // Kc is a multiple of 128: whole steps for every wave, cut at K
    const int64_t kb = (int64_t)blockIdx.z * Kc + w * (Kc / 4);
    const int64_t ke = kb + Kc / 4 < K ? kb + Kc / 4 : K;
    // row 8m + lane / 8 of the step's 96 (32 images, 64 outputs), floats 4 (lane % 8) .. + 3;
    // rows past the last image or output read the last one, their results unused
    const int lr = lane >> 3, lk = 4 * (lane & 7);
    float *mine = lds + w * kFewRows * kFewPad;
    float4 pre[kFewRows / 8];
    auto row = [&](int m, int64_t k) __attribute__((always_inline)) {
        if (8 * m < kFewS) {
            const int64_t r = s0 + 8 * m + lr;
            return in + (r < S ? r : S - 1) * K + k;
        }
        const int r = o0 + 8 * m - kFewS + lr;
        return L.W + (int64_t)(r < O ? r : O - 1) * K + k;
    };
    // (a 16-byte load needs 4-byte alignment only)
    typedef float rowx4 __attribute__((ext_vector_type(4), aligned(4)));
    auto fetch = [&](int64_t k0) {
        const int64_t k = k0 + lk;
        if (VEC || k + 3 < ke) {
#pragma unroll
            for (int m = 0; m < kFewRows / 8; ++m) {
                if (VEC) {
                    pre[m] = k < ke ? *reinterpret_cast<const float4 *>(row(m, k)) : make_float4(0.f, 0.f, 0.f, 0.f);
                } else {
                    const rowx4 v = *reinterpret_cast<const rowx4 *>(row(m, k));
                    pre[m] = make_float4(v[0], v[1], v[2], v[3]);
                }
            }
        } else {
#pragma unroll
            for (int m = 0; m < kFewRows / 8; ++m) {
                const float *p = row(m, k);
                pre[m] = make_float4(k < ke ? p[0] : 0.f, k + 1 < ke ? p[1] : 0.f, k + 2 < ke ? p[2] : 0.f, 0.f);
            }
        }
    };
    floatx16 acc[2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            acc[mb][r] = 0.f;
    if (kb < ke)
        fetch(kb);
    for (int64_t k0 = kb; k0 < ke; k0 += 32) {
#pragma unroll
        for (int m = 0; m < kFewRows / 8; ++m)
            *reinterpret_cast<float4 *>(mine + (8 * m + lr) * kFewPad + lk) = pre[m];
        // the wave's own writes before its reads, and these before the next step's writes
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (k0 + 32 < ke)
            fetch(k0 + 32);
        float4 x[4], y[2][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float *f = mine + col * kFewPad + 16 * kh + 4 * i;
            x[i] = *reinterpret_cast<const float4 *>(f);
            y[0][i] = *reinterpret_cast<const float4 *>(f + kFewS * kFewPad);
            y[1][i] = *reinterpret_cast<const float4 *>(f + (kFewS + 32) * kFewPad);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float b[4] = {x[i].x, x[i].y, x[i].z, x[i].w};
            const float a0[4] = {y[0][i].x, y[0][i].y, y[0][i].z, y[0][i].w};
            const float a1[4] = {y[1][i].x, y[1][i].y, y[1][i].z, y[1][i].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0[j], b[j], acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[j], b[j], acc[1], 0, 0, 0);
            }
        }
    }
    __syncthreads();   // every wave is done with its rows
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<float4 *>(&red[w][col][32 * mb + 8 * q + 4 * kh]) =
                make_float4(acc[mb][4 * q], acc[mb][4 * q + 1], acc[mb][4 * q + 2], acc[mb][4 * q + 3]);
    __syncthreads();
    // thread t: outputs 4 (t % 16) .. + 3 of images t / 16 and t / 16 + 16
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int si = t / 16 + 16 * h, oi = t % 16 * 4;
        const int64_t s = s0 + si;
        float4 v = *reinterpret_cast<const float4 *>(&red[0][si][oi]);
#pragma unroll
        for (int u = 1; u < 4; ++u) {
            const float4 p = *reinterpret_cast<const float4 *>(&red[u][si][oi]);
            v.x += p.x;
            v.y += p.y;
            v.z += p.z;
            v.w += p.w;
        }
        if (s >= S)
            continue;
        float *dst = part + ((int64_t)blockIdx.z * S + s) * O + o0 + oi;
        if (o0 + oi + 3 < O && ((uintptr_t)dst & 15) == 0) {
            *reinterpret_cast<float4 *>(dst) = v;
        } else {
            const float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (o0 + oi + i < O)
                    dst[i] = e[i];
        }
    }
}

__global__ void __launch_bounds__(256) cnn_linear_reduce_kernel(CnnLayerDev L, const float *__restrict__ part,
                                                               float *__restrict__ out, int64_t S, int splits) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n = S * L.cout;
    if (idx >= n)
        return;
    float v = 0.f;
#pragma unroll 8
    for (int z = 0; z < splits; ++z)
        v += part[z * n + idx];
    v += L.b[idx % L.cout];
    out[idx] = L.act == HPACML_ACT_RELU ? (v > 0.f ? v : 0.f) : v;
}

// The fully connected layers that end a stack, once the first of them has
// run its products: a block of 256 threads takes 256 / width images (width =
// the widest of these layers), adds the first layer's partial sums in block
// order with bias and activation (or reads its finished outputs), runs the
// remaining small layers on vectors in LDS (thread (image, o) computes
// output o in k order, then adds the bias), and scatters the last layer's
// outputs through the `from` map (one point per image).
__global__ void __launch_bounds__(256) cnn_tail_kernel(CnnTail T, const float *__restrict__ src, DevMap m,
                                                      int64_t S) {
    __shared__ float buf[2][256];
    const int ws = T.width;
    const int sb = threadIdx.x / ws, o = threadIdx.x % ws;
    const int64_t s = (int64_t)blockIdx.x * (256 / ws) + sb;
    const bool live = sb < 256 / ws && s < S;
    {
        const CnnLayerDev &L = T.first;
        if (live && o < L.cout) {
            float v;
            if (T.splits) {
                const int64_t n = S * L.cout, idx = s * L.cout + o;
                // every partial in flight before the first add; the sum in block order
                float pv[kLinSplit];
#pragma unroll
                for (int z = 0; z < kLinSplit; ++z)
                    pv[z] = z < T.splits ? src[z * n + idx] : 0.f;
                v = 0.f;
#pragma unroll
                for (int z = 0; z < kLinSplit; ++z)
                    if (z < T.splits)
                        v += pv[z];
                v += L.b[o];
                v = L.act == HPACML_ACT_RELU ? (v > 0.f ? v : 0.f) : v;
            } else {
                v = src[s * L.cout + o];
            }
            buf[0][sb * ws + o] = v;
        }
    }
    __syncthreads();
    int cur = 0, width = T.first.cout;
#pragma unroll
    for (int l = 0; l < kTailLayers; ++l) {
        if (l >= T.n_rest)
            break;
        const CnnLayerDev &L = T.rest[l];
        if (live && o < L.cout) {
            const float *h = &buf[cur][sb * ws];
            const float *w = L.W + (int64_t)o * width;
            float acc = 0.f;
            for (int k = 0; k < width; ++k)
                acc = fmaf(h[k], w[k], acc);
            const float v = acc + L.b[o];
            buf[cur ^ 1][sb * ws + o] = L.act == HPACML_ACT_RELU ? (v > 0.f ? v : 0.f) : v;
        }
        __syncthreads();
        cur ^= 1;
        width = L.cout;
    }
    if (live && o < width) {
        int64_t p[HPACML_MAX_RANK];
        sweep_point(m, s, p);
        stg(const_cast<float *>(feature_ptr(m, p, interior(m, p), o)), buf[cur][sb * ws + o]);
    }
}

__global__ void __launch_bounds__(256) scatter_record_kernel(DevMap m, const float *__restrict__ src) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= m.n_points)
        return;
    int64_t p[HPACML_MAX_RANK];
    sweep_point(m, b, p);
    const bool inside = interior(m, p);
    for (int g = 0; g < m.n_features; ++g)
        stg(const_cast<float *>(feature_ptr(m, p, inside, g)), src[b * m.n_features + g]);
}

}  // namespace

// ------------------------------------------------------------------ host
bool cnn_fused_supported(const CnnPlan &p) {
    if (p.n_layers > kCnnFusedMaxLayers)
        return false;
    int circ = 0;
    for (int l = 0; l < p.n_layers; ++l) {
        const hpacml_layer &y = p.layers[l];
        if (y.kind != HPACML_LAYER_CONV2D || y.padding != HPACML_PAD_SAME || y.kernel[0] > 16 || y.kernel[1] > 16)
            return false;
        if (p.shape[l].c > kCnnFusedMaxC || p.shape[l + 1].c > kCnnFusedMaxC)
            return false;
        circ += y.pad_mode == HPACML_PADMODE_CIRCULAR;
    }
    return circ == 0 || circ == p.n_layers;
}

void cnn_fused_pack(const CnnPlan &p, const float *const *W, const float *const *b, std::vector<float> &buf,
                    CnnFused *out) {
    CnnFused f{};
    f.n_layers = p.n_layers;
    f.c0 = p.in_channels;
    f.cout_last = p.shape[p.n_layers].c;
    f.circular = p.layers[0].pad_mode == HPACML_PADMODE_CIRCULAR;
    buf.clear();
    for (int l = 0; l < p.n_layers; ++l) {
        const hpacml_layer &y = p.layers[l];
        CnnFusedLayer &d = f.L[l];
        const int cin = p.shape[l].c, cout = p.shape[l + 1].c;
        d.cin4 = (cin + 3) / 4;
        d.cout4 = (cout + 3) / 4;
        d.kh = y.kernel[0];
        d.kw = y.kernel[1];
        d.top = (d.kh - 1) / 2;
        d.left = (d.kw - 1) / 2;
        d.act = y.act;
        d.mode = y.pad_mode;
        const int CI = 4 * d.cin4, CO = 4 * d.cout4;
        // [co / 4][ky][kx][ci][co % 4], zero in the padded channels
        d.woff = (int32_t)buf.size();
        buf.resize(buf.size() + (size_t)d.kh * d.kw * CI * CO, 0.f);
        for (int co = 0; co < cout; ++co)
            for (int ci = 0; ci < cin; ++ci)
                for (int ky = 0; ky < d.kh; ++ky)
                    for (int kx = 0; kx < d.kw; ++kx)
                        buf[d.woff + ((((size_t)(co / 4) * d.kh + ky) * d.kw + kx) * CI + ci) * 4 + co % 4] =
                            W[l][(((size_t)co * cin + ci) * d.kh + ky) * d.kw + kx];
        d.boff = (int32_t)buf.size();
        buf.resize(buf.size() + CO, 0.f);
        for (int co = 0; co < cout; ++co)
            buf[d.boff + co] = b[l][co];
    }
    *out = f;
}

int cnn_fused_tile_rows(const CnnFused &f, int32_t H) {
    // the largest tile of at most max(H, 1) rows (rounded up to a power of
    // two) whose buffers fit kLdsShared, else one block per CU
    int one = 0;
    for (int ty : {32, 16, 8, 4, 2, 1}) {
        if (ty > 1 && ty / 2 >= H)
            continue;
        FusedArgs a{};
        size_t f0, f1;
        fused_regions(f, ty, &a, &f0, &f1);
        const size_t bytes = (f0 + f1) * sizeof(float);
        if (bytes <= kLdsShared)
            return ty;
        if (!one && bytes <= kLdsOneBlock)
            one = ty;
    }
    return one;
}

// ---- matrix-core form: geometry, packing, choice of the tile
static void mfma_shape(const CnnFusedLayer &y, ConvM *c) {
    c->ci = 4 * y.cin4;
    c->co = 4 * y.cout4;
    c->m16 = y.cout4 == 1;
    c->P = c->m16 ? 4 : 32 / c->co;
    c->rch = ((y.kw + c->P - 1) * c->ci + 7) / 8;
    c->chunks = y.kh * c->rch;
    const int kc = c->m16 ? 4 : 2;
    c->steps = (c->chunks + kc - 1) / kc;
}

static double mfma_tile_cycles(const CnnFused &f, int ty);

bool cnn_mfma_pack(const CnnPlan &p, const float *const *W, const float *const *b, CnnFused &f,
                   std::vector<uint8_t> &buf) {
    buf.clear();
    LayerRows rows[kCnnFusedMaxLayers];
    for (int l = 0; l < f.n_layers; ++l)
        rows[l] = LayerRows{W[l], b[l], p.shape[l + 1].c, p.shape[l].c * f.L[l].kh * f.L[l].kw};
    SplitRange range;
    if (!split_range(rows, f.n_layers, 1, &range))
        return false;
    f.limit = range.limit;
    f.least = range.least;
    f.tiny = range.tiny;
    for (int ty = 1; ty <= kMaxTileRows; ++ty)
        f.cycles[ty] = mfma_tile_cycles(f, ty);
    for (int l = 0; l < f.n_layers; ++l) {
        ConvM c{};
        mfma_shape(f.L[l], &c);
        const int cin = p.shape[l].c, cout = p.shape[l + 1].c, kh = f.L[l].kh, kw = f.L[l].kw;
        const int N = c.m16 ? 16 : 32, kc = c.m16 ? 4 : 2;
        const size_t at = buf.size();
        buf.resize(at + 64 + (size_t)c.steps * 3 * kFragBytes, 0);
        for (int o = 0; o < cout; ++o)
            reinterpret_cast<float *>(&buf[at])[o] = b[l][o];
        for (int st = 0; st < c.steps; ++st)
            for (int lane = 0; lane < 64; ++lane) {
                const int row = lane % N, ch = st * kc + lane / N;
                const int px = row / c.co, o = row % c.co;
                if (ch >= c.chunks || px >= c.P || o >= cout)
                    continue;
                const int ky = ch / c.rch;
                for (int j = 0; j < 8; ++j) {
                    const int e = ch % c.rch * 8 + j, kx = e / c.ci - px, i = e % c.ci;
                    if (kx < 0 || kx >= kw || i >= cin)
                        continue;
                    const float w = W[l][(((size_t)o * cin + i) * kh + ky) * kw + kx];
                    uint16_t *d = reinterpret_cast<uint16_t *>(&buf[at + 64 + (size_t)st * 3 * kFragBytes]) + lane * 8 + j;
                    split_parts(w, d[0], d[kFragBytes / 2], d[kFragBytes]);
                }
            }
    }
    return true;
}

// The launch's layer constants for tiles of `ty` rows; returns the LDS bytes.
static size_t mfma_layout(const CnnFused &f, int ty, MfmaArgs *m) {
    size_t f0, f1;
    fused_regions(f, ty, &m->f, &f0, &f1);
    const FusedArgs &a = m->f;
    int off = 0;
    for (int l = 0; l < f.n_layers; ++l) {
        ConvM &c = m->c[l];
        const CnnFusedLayer &y = f.L[l];
        mfma_shape(y, &c);
        c.cout = l + 1 < f.n_layers ? 4 * y.cout4 : f.cout_last;
        c.bias_off = off;
        c.a_off = off + 64;
        off += 64 + c.steps * 3 * kFragBytes;
        c.oh = a.rh[l + 1];
        c.ng = (a.rw[l + 1] + c.P - 1) / c.P;
        c.groups = c.oh * c.ng;
        c.ng_magic = (uint32_t)(((1u << 24) + c.ng - 1) / c.ng);
        c.relu = y.act == HPACML_ACT_RELU;
        c.kh = y.kh;
        c.kw = y.kw;
        c.next_mode = l + 1 < f.n_layers ? f.L[l + 1].mode : HPACML_PADMODE_ZEROS;
        c.rt = a.rt[l + 1];
        c.rl = a.rl[l + 1];
        // columns of the input buffer: the region, and what the layer before
        // writes; chunks: those, and what the last group reads
        int cols = a.rw[l];
        if (l > 0)
            cols = std::max(cols, m->c[l - 1].ng * m->c[l - 1].P);
        c.S = c.P * c.ci / 8;
        c.inv = (65536 + c.S - 1) / c.S;
        c.sub = (std::max((cols * c.ci + 7) / 8, (c.ng - 1) * c.S + c.rch) + c.S - 1) / c.S;
        c.row_b = c.S * c.sub * 16;
        c.in_plane = a.rh[l] * c.row_b;
    }
    m->image_bytes = off;
    for (int l = 0; l < f.n_layers; ++l) {
        m->c[l].tab_off = off;
        off += ((m->c[l].steps + 1) * (m->c[l].m16 ? 4 : 2) * 4 + 15) / 16 * 16;
    }
    m->planes_off = off;
    int size[2] = {0, 0};
    for (int l = 0; l < f.n_layers; ++l)
        size[l & 1] = std::max(size[l & 1], 3 * m->c[l].in_plane);
    for (int l = 0; l < f.n_layers; ++l) {
        m->c[l].in_off = off + (l & 1 ? size[0] : 0);
        if (l > 0) {
            m->c[l - 1].out_off = m->c[l].in_off;
            m->c[l - 1].out_plane = m->c[l].in_plane;
            m->c[l - 1].out_row_b = m->c[l].row_b;
            m->c[l - 1].out_S = m->c[l].S;
            m->c[l - 1].out_inv = m->c[l].inv;
            m->c[l - 1].out_sub = m->c[l].sub;
        }
    }
    // (the vector ALU path of a tile uses the same space)
    m->planes_bytes = std::max(size[0] + size[1], (int)((f0 + f1) * sizeof(float)) + 15 & ~15);
    m->f.buf1 = (int32_t)f0;
    return (size_t)off + m->planes_bytes;
}

// Cycles of a tile of `ty` rows (see cnn_mfma_tile_rows), 0 where it doesn't fit.
static double mfma_tile_cycles(const CnnFused &f, int ty) {
    MfmaArgs m{};
    if (mfma_layout(f, ty, &m) + kMStatic > kLdsOneBlock)
        return 0;
    for (int l = 0; l <= f.n_layers; ++l)   // the divisions' ranges (see launch_cnn_fused)
        if (m.f.rh[l] >= 256 || m.f.rw[l] > 256)
            return 0;
    double cycles = 9500 + 8.2 * m.f.rh[0] * m.f.rw[0];
    for (int l = 0; l < f.n_layers; ++l) {
        const ConvM &c = m.c[l];
        const int n = c.m16 ? 16 : 32, each = c.m16 ? 2 : 1;   // columns of a tile, tiles at a time
        const int rounds = ((c.groups + n * each - 1) / (n * each) + kMWaves - 1) / kMWaves;
        cycles += (double)rounds * each * c.steps * 6 * n;
    }
    return cycles;
}

// Tile rows of the matrix-core form for S images, or 0 where the vector ALU
// kernel serves: no tile fits the LDS, or a large image and a stack with so few
// multiplications that both wait for memory (2048 x 2048, 2 x 2 + 2 x 2 on 4
// channels: 98 us against 109, 3 x 3 + 2 x 2: 110 / 115, 4 x 4: 102 / 93; at 1448 x
// 1448 60 / 49).  The rows: the least time over the launch's rounds of 256 blocks.  A tile's cycles
// as measured on the 5 x 5 + 3 x 3 stack with 6 to 18 rows (within 4%): 9500,
// 8.2 per gathered pixel, and the matrix time of a wave's column tiles.
int cnn_mfma_tile_rows(const CnnFused &f, int32_t S, int32_t H, int32_t W) {
    int64_t taps = 0;   // multiplications per pixel
    for (int l = 0; l < f.n_layers; ++l)
        taps += 16 * f.L[l].kh * f.L[l].kw * f.L[l].cin4 * f.L[l].cout4;
    if (!f.image || (taps <= 208 && (int64_t)S * H * W >= 3 << 20))
        return 0;
    int best = 0;
    double least = 0;
    for (int ty = 1; ty <= kMaxTileRows && (ty == 1 || ty <= H); ++ty) {
        const double tiles = (double)S * ((H + ty - 1) / ty) * ((W + kTX - 1) / kTX);
        const double t = std::ceil(tiles / 256) * f.cycles[ty];
        if (f.cycles[ty] > 0 && (!best || t < least)) {
            best = ty;
            least = t;
        }
    }
    return best;
}

hipError_t launch_cnn_mfma(const Map32 &in, const Map32 &out, const FeatTable32 *tin, const FeatTable32 *tout,
                           const CnnFused &f, int32_t S, int32_t H, int32_t W, int ty, hipStream_t stream) {
    MfmaArgs m{};
    size_t lds = mfma_layout(f, ty, &m);
    // NaN bits where there is room and only the first layer can meet one (a ReLU
    // makes 0 of it)
    const int nan_bytes = (m.f.rh[0] * kNanWords * 4 + 15) / 16 * 16;
    if ((f.n_layers == 1 || f.L[0].act == HPACML_ACT_RELU) && lds + nan_bytes + kMStatic <= kLdsOneBlock) {
        m.nan_off = (int32_t)lds;
        m.nan_bytes = nan_bytes;
        lds += nan_bytes;
    }
    m.clear_bytes = m.planes_bytes + m.nan_bytes;
    FusedArgs &a = m.f;
    a.in = in;
    a.out = out;
    a.tin = tin;
    a.tout = tout;
    a.S = S;
    a.H = H;
    a.W = W;
    a.n_layers = f.n_layers;
    a.ty = ty;
    a.tiles_y = (H + ty - 1) / ty;
    a.tiles_x = (W + kTX - 1) / kTX;
    const int64_t n_tiles = (int64_t)S * a.tiles_y * a.tiles_x;
    if (n_tiles == 0)
        return hipSuccess;
    if (n_tiles > INT32_MAX - 16)
        return hipErrorInvalidValue;
    a.n_tiles = (int32_t)n_tiles;
    a.c0 = f.c0;
    a.cout_last = f.cout_last;
    a.co_last_pad = 4 * f.L[f.n_layers - 1].cout4;
    a.circular = f.circular;
    for (int l = 0; l < f.n_layers; ++l)
        a.L[l] = f.L[l];
    for (int l = 0; l <= f.n_layers; ++l)
        a.rw_magic[l] = (uint32_t)(((1u << 24) + a.rw[l] - 1) / a.rw[l]);
    m.image = f.image;
    m.limit = f.limit;
    m.least = f.least;
    m.tiny = f.tiny;
    m.in_rank = in.rank;
    m.out_rank = out.rank;
    for (int d = 0; d < out.rank; ++d)
        m.out_offsets |= out.omin[d] != 0 || out.omax[d] != 0;
    for (int d = 0; d < in.rank; ++d)
        m.in_offsets |= in.omin[d] != 0 || in.omax[d] != 0;
    m.pre = m.c[0].ci == 4 && a.rh[0] * a.rw[0] <= kPre * kMThreads && !m.in_offsets;
    m.o_imaged = out.rank == 2 && out.count[0] == H && out.count[1] == W;   // (so S is 1)
    if (m.o_imaged) {
        m.oys = out.start[0];
        m.oyd = out.step[0];
        m.oyst = out.stride[0];
        m.oxs = out.start[1];
        m.oxd = out.step[1];
        m.oxst = out.stride[1];
    }
    m.imaged = in.rank >= 2 && in.count[in.rank - 2] == H && in.count[in.rank - 1] == W;
    if (m.imaged) {
        m.ys = in.start[in.rank - 2];
        m.yd = in.step[in.rank - 2];
        m.yst = in.stride[in.rank - 2];
        m.xs = in.start[in.rank - 1];
        m.xd = in.step[in.rank - 1];
        m.xst = in.stride[in.rank - 1];
    }
    m.grid_x = (int32_t)std::min<int64_t>(32, (n_tiles + 7) / 8);
    hipError_t e = hipFuncSetAttribute((const void *)cnn_fused_mfma_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(cnn_fused_mfma_kernel, dim3((unsigned)(8 * m.grid_x)), dim3(kMThreads), lds, stream, m, f.wts);
    return hipGetLastError();
}

hipError_t launch_cnn_fused(const Map32 &in, const Map32 &out, const FeatTable32 *tin, const FeatTable32 *tout,
                            const CnnFused &f, int32_t S, int32_t H, int32_t W, hipStream_t stream) {
    const int rows = cnn_mfma_tile_rows(f, S, H, W);
    if (rows > 0)
        return launch_cnn_mfma(in, out, tin, tout, f, S, H, W, rows, stream);
    const int ty = cnn_fused_tile_rows(f, H);
    if (ty == 0)
        return hipErrorInvalidValue;
    FusedArgs a{};
    a.in = in;
    a.out = out;
    a.tin = tin;
    a.tout = tout;
    a.S = S;
    a.H = H;
    a.W = W;
    a.n_layers = f.n_layers;
    a.ty = ty;
    a.tiles_y = (H + ty - 1) / ty;
    a.tiles_x = (W + kTX - 1) / kTX;
    const int64_t n_tiles = (int64_t)S * a.tiles_y * a.tiles_x;
    if (n_tiles == 0)
        return hipSuccess;
    if (n_tiles > INT32_MAX)
        return hipErrorInvalidValue;
    a.n_tiles = (int32_t)n_tiles;
    a.c0 = f.c0;
    a.cout_last = f.cout_last;
    a.co_last_pad = 4 * f.L[f.n_layers - 1].cout4;
    a.circular = f.circular;
    for (int l = 0; l < f.n_layers; ++l)
        a.L[l] = f.L[l];
    size_t f0, f1;
    fused_regions(f, ty, &a, &f0, &f1);
    a.buf1 = (int32_t)f0;
    for (int l = 0; l <= f.n_layers; ++l) {
        // region sizes stay below 2^16 pixels and widths at most 256 (checked
        // here): the multiply-shift quotient is then exact
        if ((int64_t)a.rh[l] * a.rw[l] >= (1 << 16) || a.rw[l] > 256)
            return hipErrorInvalidValue;
        a.rw_magic[l] = (uint32_t)(((1u << 24) + a.rw[l] - 1) / a.rw[l]);
    }
    const size_t lds = (f0 + f1) * sizeof(float);
    hipError_t e = hipFuncSetAttribute((const void *)cnn_fused_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(cnn_fused_kernel, dim3((unsigned)n_tiles), dim3(kThreads), lds, stream, a, f.wts);
    return hipGetLastError();
}

static void divisor(uint32_t d, uint32_t *magic, uint32_t *shift) {
    // i / d == (i * magic) >> (31 + l) for i < 2^31, l = ceil(log2 d), d < 2^31
    int l = 0;
    while ((uint64_t(1) << l) < d)
        ++l;
    *magic = (uint32_t)(((uint64_t(1) << (31 + l)) + d - 1) / d);
    *shift = 31 + l;
}

void cnn_layer_divisors(CnnLayerDev &L) {
    divisor((uint32_t)std::max(L.w2, 1), &L.w2_magic, &L.w2_shift);
    divisor((uint32_t)std::max(L.h2, 1), &L.h2_magic, &L.h2_shift);
}

void cnn_conv_pack(const float *W, int cout, int cin, int kh, int kw, std::vector<float> &dst) {
    const int groups = (cout + kConvG - 1) / kConvG;
    const size_t taps = (size_t)kh * kw * cin, at = dst.size();
    dst.resize(at + groups * taps * kConvG, 0.f);
    for (int co = 0; co < cout; ++co)
        for (int ci = 0; ci < cin; ++ci)
            for (int ky = 0; ky < kh; ++ky)
                for (int kx = 0; kx < kw; ++kx)
                    dst[at + ((co / kConvG) * taps + ((size_t)ky * kw + kx) * cin + ci) * kConvG + co % kConvG] =
                        W[(((size_t)co * cin + ci) * kh + ky) * kw + kx];
}

// Output tile of a fully connected layer: 64 x 64 (4 x 4 outputs per thread,
// two 16-byte LDS reads per 16 FMAs) unless the layer has at most 16
// outputs, where most of such a tile would be padding.
int linear_tile(const CnnLayerDev &L) { return L.cout > 16 ? 64 : 16; }

// Few images: where the 32-image kernel's blocks take at least two K ranges to
// fill the chip's 256 CUs (128-image / 32-image kernel, whole model of a 2048 -> 64
// layer: 16 images 18.1 / 15.0 us, 1024: 30.0 / 27.8, 4096: 82.2 / 75.9; above that
// the larger tiles fill the chip too and read the weights a quarter as often), and
// a step for each wave of two ranges at least.
static int64_t few_tiles(const CnnLayerDev &L, int64_t S) {
    return ((S + kFewS - 1) / kFewS) * ((L.cout + kMfO - 1) / kMfO);
}
static bool split_few(const CnnLayerDev &L, int64_t S) {
    const int64_t K = (int64_t)L.h * L.w * L.cin;
    return L.cout > 16 && L.cout <= 256 && K >= 256 && few_tiles(L, S) <= 128;
}

int linear_splits(const CnnLayerDev &L, int64_t S) {
    if (L.kind != HPACML_LAYER_LINEAR || S <= 0)
        return 1;
    const int64_t K = (int64_t)L.h * L.w * L.cin;
    const int64_t T = linear_tile(L);
    if (split_few(L, S)) {
        // at most 256 blocks, one round of them (a few more: 4096 -> 128 on 1400
        // images 39.7 us in 264 blocks, 33.5 in 176; on 2000 42.0 in 378, 34.7 in
        // 252), each at least one 32-k step per wave (more ranges for a long K, 1024
        // each: 32768 -> 33 on 1024 images 104 us against 99)
        const int64_t tiles = few_tiles(L, S);
        return (int)std::min<int64_t>(std::min<int64_t>(256 / tiles, K / 128), kLinSplit);
    }
    // split products of layers with more than 16 outputs run on the MFMA
    // kernel's 128 x 64 tiles
    const int64_t blocks = T == 64 ? ((S + kMfS - 1) / kMfS) * ((L.cout + kMfO - 1) / kMfO)
                                   : ((S + T - 1) / T) * ((L.cout + T - 1) / T);
    int64_t z = (1024 + blocks - 1) / blocks;                 // about 1024 blocks in all
    z = std::min<int64_t>(z, std::max<int64_t>(1, K / 64));  // at least 64 k per block
    return (int)std::max<int64_t>(1, std::min<int64_t>(z, kLinSplit));
}

int64_t linear_part_rows(const CnnLayerDev &L, int64_t S) {
    const int64_t z = linear_splits(L, S);
    if (z <= 1)
        return 0;
    if (!split_few(L, S))
        return z * S;
    // z S <= 256 S / tiles and S / tiles <= 32 / (output tiles): growing with S, so a
    // workspace made for more images serves fewer
    const int64_t K = (int64_t)L.h * L.w * L.cin, to = (L.cout + kMfO - 1) / kMfO;
    return std::min<int64_t>(std::min<int64_t>(K / 128, kLinSplit) * S, 256 * kFewS / to);
}

// pooled pixels take groups of 2^qshift lanes: windows of at most 16
// positions, so that a group wastes at most 7 of 16 lanes
bool cnn_pool_fusable(const CnnLayerDev &conv, const CnnLayerDev &pool) {
    return conv.kind == HPACML_LAYER_CONV2D && pool.kind == HPACML_LAYER_MAXPOOL2D && pool.sh == pool.kh &&
           pool.sw == pool.kw && pool.kh * pool.kw <= 16;
}

hipError_t launch_cnn_conv(const CnnLayerDev &L, const CnnLayerDev *pool, const float *in, float *out, int64_t S,
                           hipStream_t stream) {
    const int64_t n_pix = S * (pool ? (int64_t)pool->h2 * pool->w2 : (int64_t)L.h2 * L.w2);
    if (n_pix == 0)
        return hipSuccess;
    int qshift = 0;
    while (pool && (1 << qshift) < pool->kh * pool->kw)
        ++qshift;
    const int64_t bx = ((n_pix << qshift) + 255) / 256, by = (L.cout + kConvG - 1) / kConvG;
    if (bx > INT32_MAX || by > 65535)
        return hipErrorInvalidValue;
    const auto kernel = !pool         ? cnn_conv_kernel<false, 0>
                        : qshift == 0 ? cnn_conv_kernel<true, 0>
                        : qshift == 1 ? cnn_conv_kernel<true, 1>
                        : qshift == 2 ? cnn_conv_kernel<true, 2>
                        : qshift == 3 ? cnn_conv_kernel<true, 3>
                                      : cnn_conv_kernel<true, 4>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)bx, (unsigned)by), dim3(256), 0, stream, L, pool ? *pool : L, in, out,
                       n_pix);
    return hipGetLastError();
}

// Raw split-K partial sums of a fully connected layer into part[splits][S][O]
// (splits >= 2).
hipError_t launch_linear_split(const CnnLayerDev &L, const float *in, float *out, int64_t S, float *part, int splits,
                               hipStream_t stream) {
    const int64_t K = (int64_t)L.h * L.w * L.cin;
    const int64_t Kc = (K + splits - 1) / splits;
    if (split_few(L, S)) {
        const int64_t Kf = (Kc + 127) / 128 * 128;   // a range past K leaves zeros
        const unsigned bx = (unsigned)((S + kFewS - 1) / kFewS), by = (unsigned)((L.cout + kMfO - 1) / kMfO);
        const bool vec = K % 4 == 0 && ((uintptr_t)in & 15) == 0 && ((uintptr_t)L.W & 15) == 0;
        hipLaunchKernelGGL(vec ? cnn_linear_few_kernel<true> : cnn_linear_few_kernel<false>, dim3(bx, by, splits),
                           dim3(256), 0, stream, L, in, S, Kf, part);
    } else if (linear_tile(L) == 64) {
        const int64_t bx = (S + kMfS - 1) / kMfS, by = (L.cout + kMfO - 1) / kMfO;
        if (bx > INT32_MAX || by > 65535)
            return hipErrorInvalidValue;
        hipLaunchKernelGGL(cnn_linear_mfma_kernel, dim3((unsigned)bx, (unsigned)by, splits), dim3(256), 0, stream, L,
                           in, S, Kc, part);
    } else {
        const int64_t bx = (S + 15) / 16, by = (L.cout + 15) / 16;
        if (bx > INT32_MAX || by > 65535)
            return hipErrorInvalidValue;
        hipLaunchKernelGGL(cnn_linear_kernel<16>, dim3((unsigned)bx, (unsigned)by, splits), dim3(256), 0, stream, L,
                           in, out, S, Kc, part);
    }
    return hipGetLastError();
}

hipError_t launch_cnn_layer(const CnnLayerDev &L, const float *in, float *out, int64_t S, float *part,
                            hipStream_t stream) {
    const int64_t total = S * (int64_t)L.h2 * L.w2 * L.cout;
    if (total == 0)
        return hipSuccess;
    const int64_t blocks = (total + 255) / 256;
    if (blocks > INT32_MAX)
        return hipErrorInvalidValue;
    switch (L.kind) {
    case HPACML_LAYER_CONV2D:
        return launch_cnn_conv(L, nullptr, in, out, S, stream);
    case HPACML_LAYER_MAXPOOL2D:
        hipLaunchKernelGGL(cnn_pool_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, L, in, out, total);
        break;
    default: {
        // K split over up to kLinSplit blocks when the tiles alone leave the
        // chip short of blocks
        const int T = linear_tile(L);
        const int splits = linear_splits(L, S);
        if (splits == 1) {
            const int64_t bx = (S + T - 1) / T, by = (L.cout + T - 1) / T;
            if (bx > INT32_MAX || by > 65535)
                return hipErrorInvalidValue;
            const int64_t K = (int64_t)L.h * L.w * L.cin;
            if (T == 64)
                hipLaunchKernelGGL(cnn_linear_kernel<64>, dim3((unsigned)bx, (unsigned)by, 1), dim3(256), 0, stream,
                                   L, in, out, S, K, part);
            else
                hipLaunchKernelGGL(cnn_linear_kernel<16>, dim3((unsigned)bx, (unsigned)by, 1), dim3(256), 0, stream,
                                   L, in, out, S, K, part);
        } else {
            hipError_t e = launch_linear_split(L, in, out, S, part, splits, stream);
            if (e != hipSuccess)
                return e;
            const int64_t n = S * L.cout;
            hipLaunchKernelGGL(cnn_linear_reduce_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, L,
                               part, out, S, splits);
        }
        break;
    }
    }
    return hipGetLastError();
}

int cnn_tail_start(const std::vector<CnnLayerDev> &ly) {
    const int n = (int)ly.size();
    int t = n;
    // the trailing fully connected layers whose inputs are at most 256 wide
    while (t > 0 && ly[t - 1].kind == HPACML_LAYER_LINEAR && ly[t - 1].cout <= 256 &&
           (int64_t)ly[t - 1].h * ly[t - 1].w * ly[t - 1].cin <= 256)
        --t;
    // the fully connected layer before them (any K) starts the tail
    if (t > 0 && ly[t - 1].kind == HPACML_LAYER_LINEAR && ly[t - 1].cout <= 256)
        --t;
    if (t == n)
        return -1;
    return n - 1 - t <= kTailLayers ? t : -1;
}

hipError_t launch_cnn_tail(const std::vector<CnnLayerDev> &ly, int start, const float *src, int splits,
                           const DevMap &out, int64_t S, hipStream_t stream) {
    if (S == 0)
        return hipSuccess;
    CnnTail T{};
    T.first = ly[start];
    T.n_rest = (int)ly.size() - 1 - start;
    T.splits = splits > 1 ? splits : 0;
    int width = T.first.cout;
    for (int l = 0; l < T.n_rest; ++l) {
        T.rest[l] = ly[start + 1 + l];
        width = std::max(width, T.rest[l].cout);
    }
    int ws = 1;
    while (ws < width)
        ws *= 2;
    T.width = ws;
    const int64_t per = 256 / ws, blocks = (S + per - 1) / per;
    if (blocks > INT32_MAX)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(cnn_tail_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, T, src, out, S);
    return hipGetLastError();
}

hipError_t launch_cnn_linear_partials(const CnnLayerDev &L, const float *in, float *out, int64_t S, float *part,
                                      int *splits, hipStream_t stream) {
    *splits = linear_splits(L, S);
    if (*splits <= 1)
        return launch_cnn_layer(L, in, out, S, part, stream);
    return launch_linear_split(L, in, out, S, part, *splits, stream);
}

hipError_t launch_scatter_record(const DevMap &m, const float *src, hipStream_t stream) {
    if (m.n_points == 0)
        return hipSuccess;
    const int64_t blocks = (m.n_points + 255) / 256;
    if (blocks > INT32_MAX)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(scatter_record_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, m, src);
    return hipGetLastError();
}

}  // namespace hpacml

// fp32 fused region kernel for one or two hidden layers of any widths whose
// weights fit in LDS: gather -> MLP -> scatter with no activation in memory.
//
// The arithmetic is that of the uniform-width kernel (exact three-way bf16
// splits, six products on v_mfma_f32_32x32x16_bf16, hi hi accumulated apart
// from the small products; values without a split take the fp32 matrix
// instruction).  A wave owns 32 points.  The first hidden layer is never held
// whole: its neurons are computed 32 at a time, activated, split and at once
// multiplied into the accumulators of the second (two K-steps of it), or, with
// one hidden layer, into the output sums; so its width costs time but no
// registers.  The second layer's neurons go in passes of 32 G (G = 1 or 2)
// for which the first layer is computed again (6 of the 30 matrix instructions
// per block and pass where it has one K-step, 6 of 18 with G = 1), so its width
// costs no registers either.
//
// The block of neurons j + 1 is computed between the split of block j and its
// products, so that its activation and split (vector ALU) can run beside the
// products of block j.  Measured, 9-200-50-1 on 1,048,576 points: 758 us layer
// by layer (three launches, the rows of both hidden layers through memory), 167
// here; 9-200-1 471 / 73, 48-160-96-8 1402 / 422, 9-32-512-1 1147 / 330; on 65,536
// points 9-200-50-1 50 / 14.1.  Few points wait for one tile's chain of passes: from
// eight passes over two blocks on (9-40-512-1 on up to 4096 points) two library calls
// are shorter, 20.6 / 23.4 us; the kernel serves there too, since it needs no
// workspace (a call's route, and its bits, don't depend on the points).  What bounds it: matrix operations, a fifth of them
// padding, and the splits' vector instructions beside them.
#include "mlp_f32.hpp"

namespace hpacml {

namespace {

// The image (bytes).  In LDS behind the maps: biases of the two layers in
// C-fragment order, output weights, output biases, then fragments: layer 1 per
// block j of 32 neurons [K-step][hi, mid, lo]; layer 2 (nb2 blocks, a multiple
// of the pass) [j][2 K-steps][block][hi, mid] and [j][2][block] lo; with
// lo_global that last part stays in global memory.  Output weights, per group
// of four outputs and block of the last hidden layer: two registers of the
// 4 x 4 matrix instruction's A operand (lane l: row l % 4; register i: the
// feature its half holds in register 8i + (l % 32) / 4 of the block).
struct WideLayout {
    int nb1, nb2, ks, f_out;
    __host__ __device__ int blocks_out() const { return nb2 ? nb2 : nb1; }
    __host__ __device__ int bias1() const { return 0; }
    __host__ __device__ int bias2() const { return nb1 * 128; }
    __host__ __device__ int out_w(int group, int blk) const { return (nb1 + nb2) * 128 + (group * blocks_out() + blk) * 512; }
    __host__ __device__ int out_b() const { return out_w((f_out + 3) / 4, 0); }
    __host__ __device__ int l1(int j, int s) const { return out_b() + 4 * kFoutMax + (j * ks + s) * 3 * kFragBytes; }
    __host__ __device__ int l2(int j, int t, int blk) const { return l1(nb1, 0) + ((j * 2 + t) * nb2 + blk) * 2 * kFragBytes; }
    __host__ __device__ int l2_lo(int j, int t, int blk) const { return l2(nb1, 0, 0) + ((j * 2 + t) * nb2 + blk) * kFragBytes; }
    __host__ __device__ int total() const { return l2_lo(nb1, 0, 0); }
    // kPlainBehind: fp32 weights for the fragment pair at byte f lie at f + behind()
    __host__ __device__ int behind() const { return total() - l1(0, 0); }
    __host__ __device__ int image_lds(bool lo_global) const { return lo_global ? l2_lo(0, 0, 0) : total(); }
    __host__ __device__ int lds(bool lo_global) const { return image_lds(lo_global) + (int)sizeof(MapsLds); }
};

// Sums of four outputs: y += W x for the 16 registers of one block of the last
// hidden layer (w: this lane's two A registers of that block).
__device__ __forceinline__ floatx4 out_block(float2 w, const floatx16 &x, floatx4 y) {
    floatx4 y1 = {};
    static_for<0, 8>([&](auto i) __attribute__((always_inline)) {
        constexpr int r = i;
        y = __builtin_amdgcn_mfma_f32_4x4x1f32(w.x, x[r], y, 3, r, 0);
        y1 = __builtin_amdgcn_mfma_f32_4x4x1f32(w.y, x[8 + r], y1, 3, r, 0);
    });
    return y + y1;
}

// G: blocks of 32 second-layer neurons per pass (0: one hidden layer).
template <int G, int KS1, bool LOG>
__global__ void __launch_bounds__(512, 2) mlp_f32w_kernel(Map32 in, Map32 out, FeatTable32 tin, FeatTable32 tout,
                                                         F32WPacked pk, int32_t n_tiles, int32_t windowed,
                                                         int32_t out_offsets, int32_t xcd_ranges) {
    extern __shared__ u32x4 smem[];
    auto maps = [&]() __attribute__((always_inline)) -> const MapsLds & {
        int z = 0;
        asm volatile("" : "+v"(z));   // read where it is used, not held in registers
        return *reinterpret_cast<const MapsLds *>(smem + z);
    };
    u32x4 *lds4 = smem + sizeof(MapsLds) / 16;
    const char *lds = reinterpret_cast<const char *>(lds4);
    constexpr int XS = 8 * KS1;
    constexpr int GG = G ? G : 1;
    const WideLayout lay{pk.nb1, pk.nb2, KS1, pk.f_out};
    const int lane = threadIdx.x & 63, g = lane >> 5, col = lane & 31;
    const int F = in.n_features, n_points = in.n_points, rank_in = in.rank, rank_out = out.rank;
    const TileOrder order(n_tiles, xcd_ranges);
    stage_maps(*reinterpret_cast<MapsLds *>(smem), in, out, tin, tout);
    __syncthreads();
    const int pairs = (F + 1) / 2;
    float xn[XS];
    if (order.first < order.end)
        gather_inputs<KS1>(maps(), rank_in, n_points, windowed, pairs, order.first * 32 + col, g, xn);
    {
        const u32x4 *src = reinterpret_cast<const u32x4 *>(pk.image);
        const int n4 = lay.image_lds(LOG) / 16;
        // eight loads in flight: few points wait for this (9-256-128-1 on 200: 20.0 -> 18.0 us,
        // 9-200-1 7.1 -> 6.6)
        for (int i = threadIdx.x; i < n4; i += 8 * blockDim.x) {
            u32x4 q[8];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                q[k] = src[min(i + k * (int)blockDim.x, n4 - 1)];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (i + k * (int)blockDim.x < n4)
                    lds4[i + k * blockDim.x] = q[k];
        }
    }
    __syncthreads();

    for (int tile = order.first; tile < order.end; tile += order.step) {
        const int b = tile * 32 + col;
        const bool valid = b < n_points;
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const u32x4 *fl = lds4 + ln;
        const u32x4 *gl = reinterpret_cast<const u32x4 *>(pk.image) + ln;
        Range range;   // of the inputs of every layer
        range.top = pk.weights == kPlainWeights ? kBig : 0.f;
        Split b1[KS1];
        static_for<0, KS1>([&](auto s) __attribute__((always_inline)) {
            floatx8 v;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                // zero where there is no feature
                v[j] = 2 * (8 * s + j) + g < F ? xn[8 * s + j] : 0.f;
            }
#pragma unroll
            for (int j = 0; j < 8; j += 2)
                range.add(v[j], v[j + 1]);
            b1[s] = split8(v);
        });
        if (tile + order.step < order.end) {
            gather_inputs<KS1>(maps(), rank_in, n_points, windowed, pairs, (tile + order.step) * 32 + col, g, xn);
        } else {
#pragma unroll
            for (int s = 0; s < XS; ++s)
                xn[s] = 0.f;
        }

        floatx4 y[2] = {};   // output sums (two groups of four)
        auto out_add = [&](const floatx16 &x, int blk) __attribute__((always_inline)) {
            y[0] = out_block(reinterpret_cast<const float2 *>(lds + lay.out_w(0, blk))[ln], x, y[0]);
            if (pk.f_out > 4)
                y[1] = out_block(reinterpret_cast<const float2 *>(lds + lay.out_w(1, blk))[ln], x, y[1]);
        };
        // block j of the first hidden layer, activated
        struct Frags {
            u32x4 q[KS1][3];
        };
        auto read1 = [&](int j, Frags &f) __attribute__((always_inline)) {
            const int at = lay.l1(j, 0) / 16;
#pragma unroll
            for (int s = 0; s < KS1; ++s)
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    f.q[s][q] = fl[at + (s * 3 + q) * 64];
        };
        auto first = [&](int j, const Frags &f, floatx16 &main, floatx16 &sub) __attribute__((always_inline)) {
            load_bias<1>(reinterpret_cast<const float *>(lds + lay.bias1() + j * 128), ln >> 5, &main);
            const floatx16 zero = {};
            static_for<0, KS1>([&](auto s) __attribute__((always_inline)) {
                sub = mfma(f.q[s][0], b1[s].mid, s == 0 ? zero : sub);
                main = mfma(f.q[s][0], b1[s].hi, main);
                sub = mfma(f.q[s][0], b1[s].lo, sub);
                sub = mfma(f.q[s][1], b1[s].hi, sub);
                sub = mfma(f.q[s][1], b1[s].mid, sub);
                sub = mfma(f.q[s][2], b1[s].hi, sub);
            });
        };
        auto finish = [&](floatx16 main, const floatx16 &sub, int layer) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                main[r] += sub[r];
            activate<1>(&main, act_floor(pk.relu >> layer & 1), range);
            return main;
        };
        if (__any(range.outside(pk.limit))) {
            // (see below)
        } else if constexpr (G == 0) {
            floatx16 main, sub;
            Frags f;
            read1(0, f);
            first(0, f, main, sub);
            for (int j = 0; j < pk.nb1; ++j) {
                floatx16 m1 = main, s1 = sub;
                read1(j + 1 < pk.nb1 ? j + 1 : j, f);
                first(j + 1 < pk.nb1 ? j + 1 : j, f, main, sub);
                out_add(finish(m1, s1, 0), j);
            }
        } else {
            for (int p = 0; p < pk.nb2; p += GG) {
                floatx16 m2[GG], s2[GG], main, sub;
                load_bias<1, 1>(reinterpret_cast<const float *>(lds + lay.bias2() + p * 128), ln >> 5, &m2[0]);
                if constexpr (GG == 2)
                    load_bias<1, 1>(reinterpret_cast<const float *>(lds + lay.bias2() + (p + 1) * 128), ln >> 5, &m2[1]);
#pragma unroll
                for (int i = 0; i < GG; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        s2[i][r] = 0.f;
                u32x4 lo[2][GG];
                auto read_lo = [&](int j) __attribute__((always_inline)) {
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int i = 0; i < GG; ++i)
                            lo[t][i] = (LOG ? gl : fl)[lay.l2_lo(j, t, p + i) / 16];
                };
                Frags f;
                read1(0, f);
                if (LOG)
                    read_lo(0);
                first(0, f, main, sub);
                Split bs[2];
                auto split = [&](const floatx16 &x) __attribute__((always_inline)) {
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        floatx8 v;
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            v[e] = x[8 * t + e];
                        bs[t] = split8(v);
                    }
                };
                split(finish(main, sub, 0));
#pragma unroll 1
                for (int j = 0; j < pk.nb1; ++j) {
                    const int jn = j + 1 < pk.nb1 ? j + 1 : j;
                    u32x4 h[2][GG], m[2][GG], lw[2][GG];
#pragma unroll
                    for (int i = 0; i < GG; ++i) {
                        h[0][i] = fl[lay.l2(j, 0, p + i) / 16];
                        m[0][i] = fl[lay.l2(j, 0, p + i) / 16 + 64];
                    }
                    if (!LOG)
                        read_lo(j);
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int i = 0; i < GG; ++i)
                            lw[t][i] = lo[t][i];
                    if (LOG)
                        read_lo(jn);
                    read1(jn, f);
                    __builtin_amdgcn_sched_barrier(kSchedAluOnly);
                    Split bc[2] = {bs[0], bs[1]};
                    first(jn, f, main, sub);
                    __builtin_amdgcn_sched_barrier(kSchedAluOnly);
                    static_for<0, 2>([&](auto t) __attribute__((always_inline)) {
                        if (t == 0) {
#pragma unroll
                            for (int i = 0; i < GG; ++i) {
                                h[1][i] = fl[lay.l2(j, 1, p + i) / 16];
                                m[1][i] = fl[lay.l2(j, 1, p + i) / 16 + 64];
                            }
                            __builtin_amdgcn_sched_barrier(kSchedAluOnly);
                        }
#pragma unroll
                        for (int i = 0; i < GG; ++i)
                            s2[i] = mfma(h[t][i], bc[t].mid, s2[i]);
#pragma unroll
                        for (int i = 0; i < GG; ++i)
                            m2[i] = mfma(h[t][i], bc[t].hi, m2[i]);
#pragma unroll
                        for (int i = 0; i < GG; ++i)
                            s2[i] = mfma(h[t][i], bc[t].lo, s2[i]);
#pragma unroll
                        for (int i = 0; i < GG; ++i)
                            s2[i] = mfma(m[t][i], bc[t].hi, s2[i]);
#pragma unroll
                        for (int i = 0; i < GG; ++i)
                            s2[i] = mfma(m[t][i], bc[t].mid, s2[i]);
#pragma unroll
                        for (int i = 0; i < GG; ++i)
                            s2[i] = mfma(lw[t][i], bc[t].hi, s2[i]);
                    });
                    split(finish(main, sub, 0));
                }
#pragma unroll
                for (int i = 0; i < GG; ++i)
                    out_add(finish(m2[i], s2[i], 1), p + i);
            }
        }
        const float *ob = reinterpret_cast<const float *>(lds + lay.out_b()) + (ln >> 5);
        float v[2][2] = {};   // outputs 2i + g and 4 + 2i + g
        auto outputs = [&]() __attribute__((always_inline)) {
            join_halves(y[0], ob, v[0]);
            if (pk.f_out > 4)
                join_halves(y[1], ob + 4, v[1]);
        };
        outputs();
        if (outside(range, pk.limit, pk.least, v, pk.f_out)) {
            // this tile (again) on the fp32 instruction
            const int gc = ln >> 5, form = pk.weights, behind = lay.behind() / 16;
            float x[XS];
            gather_inputs<KS1>(maps(), rank_in, n_points, windowed, pairs, b, gc, x);
#pragma unroll
            for (int s = 0; s < XS; ++s)
                x[s] = 2 * s + gc < F ? x[s] : 0.f;
            auto step = [&](int hm, u32x4 lw, const float *xs, floatx16 acc) __attribute__((always_inline)) {
                u32x4 f[2];
                if (form == kPlainBehind) {
                    f[0] = gl[behind + hm / 16];
                    f[1] = gl[behind + hm / 16 + 64];
                } else {
                    f[0] = fl[hm / 16];
                    f[1] = fl[hm / 16 + 64];
                }
                return mfma_plain(f[0], f[1], lw, form, xs, acc);
            };
            auto plain1 = [&](int j) __attribute__((always_inline)) {
                floatx16 acc;
                load_bias<1>(reinterpret_cast<const float *>(lds + lay.bias1() + j * 128), gc, &acc);
#pragma unroll
                for (int s = 0; s < KS1; ++s)
                    acc = step(lay.l1(j, s), fl[lay.l1(j, s) / 16 + 128], x + 8 * s, acc);
                activate_plain<1>(&acc, pk.relu & 1, j, gc, pk.dims[1]);
                return acc;
            };
            y[0] = y[1] = floatx4{};
            if constexpr (G == 0) {
#pragma unroll 1
                for (int j = 0; j < pk.nb1; ++j)
                    out_add(plain1(j), j);
            } else {
#pragma unroll 1
                for (int p = 0; p < pk.nb2; ++p) {
                    floatx16 acc;
                    load_bias<1>(reinterpret_cast<const float *>(lds + lay.bias2() + p * 128), gc, &acc);
#pragma unroll 1
                    for (int j = 0; j < pk.nb1; ++j) {
                        const floatx16 h = plain1(j);
#pragma unroll
                        for (int t = 0; t < 2; ++t) {
                            float xt[8];
#pragma unroll
                            for (int e = 0; e < 8; ++e)
                                xt[e] = h[8 * t + e];
                            acc = step(lay.l2(j, t, p), (LOG ? gl : fl)[lay.l2_lo(j, t, p) / 16], xt, acc);
                        }
                    }
                    activate_plain<1>(&acc, pk.relu >> 1 & 1, p, gc, pk.dims[2]);
                    out_add(acc, p);
                }
            }
            outputs();
        }
        const MapsLds &tab = maps();
        const OutPoint po(tab, rank_out, out_offsets, valid ? b : n_points - 1);
        const bool orelu = pk.relu >> (G ? 2 : 1) & 1;
        po.store(tab, v[0][0], v[0][1], 0, pk.f_out, g, orelu, valid);
        if (pk.f_out > 4)
            po.store(tab, v[1][0], v[1][1], 4, pk.f_out, g, orelu, valid);
    }
}

template <int G, int KS1, bool LOG>
hipError_t launch_t(const Map32 &in, const Map32 &out, const FeatTable32 &tin, const FeatTable32 &tout,
                    const F32WPacked &pk, hipStream_t stream) {
    const int32_t n_tiles = (in.n_points + 31) / 32;
    const WideLayout lay{pk.nb1, pk.nb2, KS1, pk.f_out};
    const size_t lds = (size_t)lay.lds(LOG);
    // blocks per CU: two waves per SIMD fill the registers; few tiles go in
    // blocks of four waves so that more CUs have one
    const int threads = n_tiles <= 256 * 4 ? 256 : 512, waves = threads / 64;
    int64_t grid = 256LL * (threads == 256 && 2 * (lds + 1024) <= (size_t)kLdsMax ? 2 : 1);
    const int64_t need = (n_tiles + waves - 1) / waves;
    if (grid > need)
        grid = need;
    bool window = false, offsets = false;
    for (int d = 0; d < in.rank; ++d)
        window = window || in.omin[d] != 0 || in.omax[d] != 0;
    for (int d = 0; d < out.rank; ++d)
        offsets = offsets || out.omin[d] != 0 || out.omax[d] != 0;
    auto kern = mlp_f32w_kernel<G, KS1, LOG>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(threads), lds, stream, in, out, tin, tout, pk, n_tiles,
                       (int32_t)window, (int32_t)offsets, (int32_t)(window && grid % 8 == 0));
    return hipGetLastError();
}

// first-layer K-steps the kernel is built for: one (up to 16 inputs) or three (48)
int wide_ks(int f_in) { return f_in <= 16 ? 1 : 3; }

WideLayout wide_layout(int n_layers, const int32_t *dims) {
    const int nb2 = n_layers == 3 ? (dims[2] + 31) / 32 : 0;
    return WideLayout{(dims[1] + 31) / 32, nb2 > 1 ? (nb2 + 1) / 2 * 2 : nb2, wide_ks(dims[0]), dims[n_layers]};
}

}  // namespace

bool f32w_supported(int n_layers, const int32_t *dims, int compute) {
    if (compute != HPACML_F32 || n_layers < 2 || n_layers > 3 || dims[0] > 48 || dims[n_layers] > kFoutMax)
        return false;
    const WideLayout lay = wide_layout(n_layers, dims);
    return lay.nb1 <= 128 && lay.nb2 <= 128 && lay.lds(true) <= kLdsMax;
}

void f32w_pack(int n_layers, const int32_t *dims, const float *const *W, const float *const *b, std::vector<float> &image,
               F32WPacked *pk) {
    const WideLayout lay = wide_layout(n_layers, dims);
    pk->nb1 = lay.nb1;
    pk->nb2 = lay.nb2;
    pk->f_out = lay.f_out;
    // (the output layer is on the fp32 instruction)
    LayerRows rows[2];
    for (int l = 0; l + 1 < n_layers; ++l)
        rows[l] = LayerRows{W[l], b[l], dims[l + 1], dims[l]};
    SplitRange range;
    const bool fine = split_range(rows, n_layers - 1, largest_row_sum(W[n_layers - 1], dims[n_layers], dims[n_layers - 1]), &range);
    pk->weights = !fine ? kPlainWeights : range.tiny ? kPlainBehind : kSplitWeights;
    pk->limit = range.limit;
    pk->least = range.least;
    image.assign((lay.total() + (range.tiny ? lay.l2_lo(0, 0, 0) - lay.l1(0, 0) : 0)) / 4, 0.f);
    char *img = reinterpret_cast<char *>(image.data());
    auto put_bias = [&](int off, const float *bias, int n, int blocks) {
        float *d = reinterpret_cast<float *>(img + off);
        for (int mb = 0; mb < blocks; ++mb)
            for (int g = 0; g < 2; ++g)
                for (int r = 0; r < 16; ++r)
                    d[(mb * 2 + g) * 16 + r] = crow(mb, r, g) < n ? bias[crow(mb, r, g)] : 0.f;
    };
    auto put = [&](int l, int steps, int blocks, auto &&hm, auto &&lo, auto &&feature) {
        put_layer(img, W[l], dims[l + 1], dims[l], steps, blocks, !fine, hm, lo, feature);
        if (fine && range.tiny)
            put_layer(img + lay.behind(), W[l], dims[l + 1], dims[l], steps, blocks, true, hm, lo, feature);
    };
    put_bias(lay.bias1(), b[0], dims[1], lay.nb1);
    put(0, lay.ks, lay.nb1, [&](int s, int j) { return lay.l1(j, s); }, [&](int s, int j) { return lay.l1(j, s) + 2 * kFragBytes; },
        [](int s, int g, int j) { return 2 * (8 * s + j) + g; });
    if (n_layers == 3) {
        put_bias(lay.bias2(), b[1], dims[2], lay.nb2);
        put(1, 2 * lay.nb1, lay.nb2, [&](int s, int mb) { return lay.l2(s / 2, s % 2, mb); },
            [&](int s, int mb) { return lay.l2_lo(s / 2, s % 2, mb); },
            [](int s, int g, int j) { return crow(s / 2, 8 * (s % 2) + j, g); });
    }
    const int K = dims[n_layers - 1], O = dims[n_layers];
    for (int o = 0; o < O; ++o)
        for (int blk = 0; blk < lay.blocks_out(); ++blk) {
            float *d = reinterpret_cast<float *>(img + lay.out_w(o / 4, blk));
            for (int i = 0; i < 2; ++i)
                for (int g = 0; g < 2; ++g)
                    for (int q = 0; q < 8; ++q) {
                        const int k = crow(blk, 8 * i + q, g);
                        d[(32 * g + 4 * q + o % 4) * 2 + i] = k < K ? W[n_layers - 1][(size_t)o * K + k] : 0.f;
                    }
        }
    for (int o = 0; o < kFoutMax; ++o)
        reinterpret_cast<float *>(img + lay.out_b())[o] = o < O ? b[n_layers - 1][o] : FLT_MAX;   // (never below `least`)
}

hipError_t launch_mlp_f32w(const Map32 &in, const Map32 &out, const FeatTable32 &tin, const FeatTable32 &tout,
                           const F32WPacked &pk, hipStream_t stream) {
    if (in.n_points == 0)
        return hipSuccess;
    const int ks = wide_ks(in.n_features), G = pk.nb2 > 1 ? 2 : pk.nb2;
    const bool log = WideLayout{pk.nb1, pk.nb2, ks, pk.f_out}.lds(false) > kLdsMax;
#define HPACML_F32W(g, k)                                                                  \
    if (G == g && ks == k)                                                                 \
        return log && g ? launch_t<g, k, (g != 0)>(in, out, tin, tout, pk, stream)         \
                        : launch_t<g, k, false>(in, out, tin, tout, pk, stream);
    HPACML_F32W(0, 1)
    HPACML_F32W(0, 3)
    HPACML_F32W(1, 1)
    HPACML_F32W(1, 3)
    HPACML_F32W(2, 1)
    HPACML_F32W(2, 3)
#undef HPACML_F32W
    return hipErrorInvalidValue;
}

}  // namespace hpacml

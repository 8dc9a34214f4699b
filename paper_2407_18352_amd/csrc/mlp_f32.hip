// fp32 fused region kernel: gather -> MLP -> scatter with the activations
// resident in registers and the weights in LDS, the products on the bf16
// matrix cores.
//
// The surrogate runs per sweep point on the composed input tensor
// (Sec. IV-A composition, Sec. IV-B inference).  Here each wave owns 32 points
// and computes every layer transposed, H_out^T = W * H_in^T: A = weights
// (rows = output features), B = activations (columns = points, from
// registers), C = the next layer's activations.
//
// Products of 32-bit numbers: the fp32 matrix instruction does 64 flop per
// cycle and SIMD, the bf16 one 1024.  A float is the exact sum of three bf16
// numbers (hi + mid + lo: 8 significant bits each, rounded to nearest; exact
// from 2^-110 up, below that to an absolute 2^-134), so w * x is the sum of
// nine bf16 products; the six of at least 2^-18 of the largest (hi hi, hi
// mid, mid hi, mid mid, hi lo, lo hi) are accumulated in fp32 by
// v_mfma_f32_32x32x16_bf16; the other three (2^-27 and less) are below half a
// unit of the fp32 product.  Six of these instructions take 192 cycles for 16
// values of k where the fp32 form takes 512.  hi hi is accumulated apart from
// the five small products, so that a sum is rounded at its final size once per
// 16 values of k, not once per two.  Measured against the same kernel on the
// fp32 instruction: 9-128-128-128-1 on 1,048,576 points 537 -> 315 us,
// 36-128-128-4 on 2048 x 2048 windows 1680 -> 862 us, 5-64-64-1 on 65,536
// points 10.2 -> 7.3 us; error against 64 bits (2-norm) 1.6e-7 -> 0.8e-7,
// 3.0e-7 -> 1.4e-7, 2.4e-7 -> 1.5e-7.  What bounds it: bf16 matrix operations (the
// two larger ones run 1.36 PFLOP/s of them, a 16384^3 bf16 product 1.32; counters:
// matrix cores busy 60 and 62% of the cycles at a clock that the load lowers to 2.1
// and 1.9 GHz).
//
// Layouts: in the 32x32 C layout lane l holds point l % 32 and, in register r
// of m-block mb, feature 32 mb + 8 (r / 4) + 4 (l / 32) + r % 4.  Registers 8t ..
// 8t + 7, split in three, are directly the B operand of K-step 2 mb + t of the
// next layer (k = 8 (l / 32) + j) when that layer's weight columns are permuted
// to match at pack time; the activations never leave registers.
//
// First layer: each lane gathers features 2t + l / 32 of its point into the
// slots t = 8s .. 8s + 7 of K-step s.  Output layer (<= 8 outputs): the fp32 matrix
// instruction of 4 x 4 blocks.  Biases enter as the initial accumulator.
//
// Values of 2^127 and more (infinities among them) have no such split, values
// large enough for a sum to overflow could turn an infinity into a NaN, and
// values below 2^-110 lose bits in it, which shows in very small outputs: a wave
// that meets a point of that kind (see split_range for the bounds) computes its
// tile on the fp32 matrix instruction, with the weights put together from their
// parts (see WeightForm).  So does every wave of a model with a weight that has no
// split.  Measured, 9-128-128-128-1 on 1,048,576 points: 316 us; with an infinite
// input in every tile 873, with such a weight 668 (weights from global memory: 2073
// both); 5-64-64-1: 61, 160 and 132 (249 both).
#include "mlp_f32.hpp"

namespace hpacml {

namespace {

// Split image offsets (bytes).  In LDS: biases and output layer (fp32), the hi
// and mid fragments of every layer, and the lo fragments; with lo_global the
// lo fragments stay in global memory behind the rest.  The output weights go in
// groups of four outputs: a[i] of lane l, i < 2 NMB, is weight [l % 4] for the
// feature that lane half l / 32 holds in register 8i + (l % 32) / 4 (counted
// over the m-blocks): one register of the matrix instruction's A operand
// serves eight of the activations' registers.
//   fragment of layer 1: K-step s, m-block mb, part q -> l1(s, mb, q)
//   fragment of hidden layer h likewise; 2 * NMB K-steps
struct SplitLayout {
    int nmb, ks, n_hidden, f_out;
    __host__ __device__ int l1_bias() const { return 0; }
    __host__ __device__ int hidden_bias(int h) const { return (h + 1) * 128 * nmb; }
    __host__ __device__ int out_w() const { return (n_hidden + 1) * 128 * nmb; }
    __host__ __device__ int out_w(int group) const { return out_w() + group * 512 * nmb; }
    __host__ __device__ int out_b() const { return out_w((f_out + 3) / 4); }
    // hi and mid of layer 1, then of the hidden layers: [K-step][m-block][2]
    __host__ __device__ int l1() const { return out_b() + 4 * kFoutMax; }
    __host__ __device__ int hidden(int h) const { return l1() + (ks + h * 2 * nmb) * nmb * 2 * kFragBytes; }
    // lo: [K-step][m-block]
    __host__ __device__ int l1_lo() const { return hidden(n_hidden); }
    __host__ __device__ int hidden_lo(int h) const { return l1_lo() + (ks + h * 2 * nmb) * nmb * kFragBytes; }
    __host__ __device__ int total() const { return hidden_lo(n_hidden); }
    // kPlainBehind: fp32 weights for the fragment pair at byte f lie at f + behind()
    __host__ __device__ int behind() const { return total() - l1(); }
    // what a block keeps in LDS
    __host__ __device__ int image_lds(bool lo_global) const { return lo_global ? l1_lo() : total(); }
    __host__ __device__ int lds(bool lo_global) const { return image_lds(lo_global) + (int)sizeof(MapsLds); }
};

// Every layer but the output on the fp32 matrix instruction; x: the point's inputs
// (0 past the last); fl, gl: this lane's part of the image in LDS and in global memory.
template <int NMB, int KS1, bool LOG>
__device__ __forceinline__ void layers_plain(const F32Packed &pk, const float (&x)[8 * KS1], const u32x4 *fl,
                                             const u32x4 *gl, const char *lds, const SplitLayout &lay, int g, floatx16 *acc) {
    const int form = pk.weights, behind = lay.behind() / 16;
    auto step = [&](int hm, int lo, const float *xs) __attribute__((always_inline)) {
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb) {
            u32x4 f[3];
            if (form == kPlainBehind) {
                f[0] = gl[behind + hm / 16 + mb * 128];
                f[1] = gl[behind + hm / 16 + mb * 128 + 64];
            } else {
                f[0] = fl[hm / 16 + mb * 128];
                f[1] = fl[hm / 16 + mb * 128 + 64];
            }
            f[2] = (LOG ? gl : fl)[lo / 16 + mb * 64];
            acc[mb] = mfma_plain(f[0], f[1], f[2], form, xs, acc[mb]);
            __builtin_amdgcn_sched_barrier(0);   // (few registers are left)
        }
    };
    load_bias<NMB>(reinterpret_cast<const float *>(lds + lay.l1_bias()), g, acc);
#pragma unroll
    for (int s = 0; s < KS1; ++s)
        step(lay.l1() + s * NMB * 2 * kFragBytes, lay.l1_lo() + s * NMB * kFragBytes, x + 8 * s);
    activate_plain<NMB>(acc, pk.relu & 1, 0, g, pk.dims[1]);
    for (int h = 0; h < pk.n_hidden; ++h) {
        floatx16 hin[NMB];
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb)
            hin[mb] = acc[mb];
        load_bias<NMB>(reinterpret_cast<const float *>(lds + lay.hidden_bias(h)), g, acc);
#pragma unroll 1
        for (int q = 0; q < NMB; ++q) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                float xs[8];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    xs[j] = hin[0][8 * t + j];
                step(lay.hidden(h) + (2 * q + t) * NMB * 2 * kFragBytes, lay.hidden_lo(h) + (2 * q + t) * NMB * kFragBytes, xs);
            }
#pragma unroll
            for (int i = 0; i + 1 < NMB; ++i)
                hin[i] = hin[i + 1];
        }
        activate_plain<NMB>(acc, pk.relu >> (h + 1) & 1, 0, g, pk.dims[h + 2]);
    }
}

// KS1: K-steps of the first layer (16 features each).
// LOG: the lo fragments are read from global memory (the L2), not LDS.
template <int NMB, int KS1, bool LOG>
__global__ void __launch_bounds__(NMB == 4 ? 512 : 256, 2) mlp_f32_kernel(Map32 in, Map32 out, FeatTable32 tin, FeatTable32 tout,
                                                      F32Packed pk, int32_t n_tiles, int32_t windowed,
                                                      int32_t out_offsets, int32_t xcd_ranges) {
    extern __shared__ u32x4 smem[];
    MapsLds &tab0 = *reinterpret_cast<MapsLds *>(smem);
    // the maps through an address the compiler doesn't know: what is read
    // through it is read there, not held in registers over the whole loop
    auto maps = [&]() __attribute__((always_inline)) -> const MapsLds & {
        int z = 0;
        asm volatile("" : "+v"(z));
        return *reinterpret_cast<const MapsLds *>(smem + z);
    };
    u32x4 *lds4 = smem + sizeof(MapsLds) / 16;
    const char *lds = reinterpret_cast<const char *>(lds4);
    constexpr int XS = 8 * KS1;      // input slots of a lane
    const SplitLayout lay{NMB, KS1, pk.n_hidden, pk.f_out};
    const int lane = threadIdx.x & 63;
    const int g = lane >> 5;
    const int col = lane & 31;
    const TileOrder order(n_tiles, xcd_ranges);
    const int F = in.n_features, n_points = in.n_points, rank_in = in.rank, rank_out = out.rank;

    stage_maps(tab0, in, out, tin, tout);
    __syncthreads();

    auto gather = [&](int tile, float (&x)[XS]) __attribute__((always_inline)) {
        gather_inputs<KS1>(maps(), rank_in, n_points, windowed, pk.ks1, tile * 32 + col, g, x);
    };
    float xn[XS];
    // the first tile's loads go out before the weights are staged
    if (order.first < order.end)
        gather(order.first, xn);

    // stage the split weights once per block
    {
        const u32x4 *src = reinterpret_cast<const u32x4 *>(pk.image);
        const int n4 = lay.image_lds(LOG) / 16;
        for (int i = threadIdx.x; i < n4; i += blockDim.x)
            lds4[i] = src[i];
    }
    __syncthreads();

    for (int tile = order.first; tile < order.end; tile += order.step) {
        const int b = tile * 32 + col;
        const bool valid = b < n_points;
        int ln = lane;
        asm volatile("" : "+v"(ln));   // nothing read from LDS is held from one tile to the next
        Range range;   // of the inputs of every layer
        range.top = pk.weights == kPlainWeights ? kBig : 0.f;
        Split b1[KS1];
        floatx16 acc[NMB];
        const u32x4 *fl = lds4 + ln;                                        // this lane's part of the LDS fragments
        const u32x4 *gl = reinterpret_cast<const u32x4 *>(pk.image) + ln;   // ... of the global ones
        // One layer: B fragments b[K-step], weights' hi and mid fragments at
        // byte `hm`, lo at `lw`, bias at `bias`; two m-blocks at a time (with
        // independent accumulators, which keeps the matrix core busy).  Of the
        // six products hi hi goes into `main` and the small ones into `sub`, so
        // that a sum of its final size is rounded once per K-step, not six
        // times.  A K-step has three phases -- the hi, mid and lo fragments'
        // products, 6, 4 and 2 matrix instructions -- and each fragment pair
        // is read two phases ahead of its own (global ones a K-step more).
        // prepare() runs once the first fragments are on their way.
        auto layer = [&](auto &b, auto ksteps, int hm, int lw, int bias, bool relu,
                         auto &&prepare) __attribute__((always_inline)) {
            constexpr int K = decltype(ksteps)::value, Q = K * (NMB / 2);
            u32x4 h[2], m[2], l[2][2];
            const int hb = hm / 16, lb = lw / 16;
            auto at = [&](int q, int i) __attribute__((always_inline)) { return (q % K) * NMB + 2 * (q / K) + i; };
            auto read_h = [&](int q) __attribute__((always_inline)) {
                h[0] = fl[hb + at(q, 0) * 128];
                h[1] = fl[hb + at(q, 1) * 128];
            };
            auto read_m = [&](int q) __attribute__((always_inline)) {
                m[0] = fl[hb + at(q, 0) * 128 + 64];
                m[1] = fl[hb + at(q, 1) * 128 + 64];
            };
            auto read_l = [&](int q, u32x4 (&d)[2]) __attribute__((always_inline)) {
                d[0] = (LOG ? gl : fl)[lb + at(q, 0) * 64];
                d[1] = (LOG ? gl : fl)[lb + at(q, 1) * 64];
            };
            if (LOG)
                read_l(0, l[0]);
            read_h(0);
            read_m(0);
            __builtin_amdgcn_sched_barrier(kSchedAluOnly);
            prepare();
            floatx16 main[2], sub[2];
            static_for<0, Q>([&](auto q) __attribute__((always_inline)) {
                constexpr int s = q % K, p = q / K;
                if (s == 0)
                    load_bias<NMB, 2>(reinterpret_cast<const float *>(lds + bias), ln >> 5, main, 2 * p);
                if (!LOG)
                    read_l(q, l[0]);
                else if (q + 1 < Q)
                    read_l(q + 1, l[(q + 1) % 2]);
                __builtin_amdgcn_sched_barrier(kSchedAluOnly);
                const floatx16 zero = {};
                sub[0] = mfma(h[0], b[s].mid, s == 0 ? zero : sub[0]);
                sub[1] = mfma(h[1], b[s].mid, s == 0 ? zero : sub[1]);
                sub[0] = mfma(h[0], b[s].lo, sub[0]);
                sub[1] = mfma(h[1], b[s].lo, sub[1]);
                main[0] = mfma(h[0], b[s].hi, main[0]);
                main[1] = mfma(h[1], b[s].hi, main[1]);
                if (q + 1 < Q)
                    read_h(q + 1);
                __builtin_amdgcn_sched_barrier(kSchedAluOnly);
                sub[0] = mfma(m[0], b[s].hi, sub[0]);
                sub[1] = mfma(m[1], b[s].hi, sub[1]);
                sub[0] = mfma(m[0], b[s].mid, sub[0]);
                sub[1] = mfma(m[1], b[s].mid, sub[1]);
                if (q + 1 < Q)
                    read_m(q + 1);
                __builtin_amdgcn_sched_barrier(kSchedAluOnly);
                sub[0] = mfma(l[LOG ? q % 2 : 0][0], b[s].hi, sub[0]);
                sub[1] = mfma(l[LOG ? q % 2 : 0][1], b[s].hi, sub[1]);
                if (s == K - 1) {
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            main[i][r] += sub[i][r];
                    activate<2>(main, act_floor(relu), range);
                    acc[2 * p] = main[0];
                    acc[2 * p + 1] = main[1];
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
        };
        // ---- first layer
        if (pk.weights != kPlainWeights)
            layer(b1, std::integral_constant<int, KS1>{}, lay.l1(), lay.l1_lo(), lay.l1_bias(), pk.relu & 1, [&]() {
            static_for<0, KS1>([&](auto s) __attribute__((always_inline)) {
                floatx8 v;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    // zero where there is no feature (only in the last K-step)
                    v[j] = s < KS1 - 1 || 2 * (8 * s + j) + g < F ? xn[8 * s + j] : 0.f;
                }
#pragma unroll
                for (int j = 0; j < 8; j += 2)
                    range.add(v[j], v[j + 1]);
                b1[s] = split8(v);
            });
        });

        // ---- hidden layers H -> H
        auto hidden = [&](int h) __attribute__((always_inline)) {
            Split bs[2 * NMB];
            layer(bs, std::integral_constant<int, 2 * NMB>{}, lay.hidden(h), lay.hidden_lo(h), lay.hidden_bias(h),
                  pk.relu >> (h + 1) & 1, [&]() __attribute__((always_inline)) {
                      static_for<0, 2 * NMB>([&](auto s) __attribute__((always_inline)) {
                          floatx8 v;
#pragma unroll
                          for (int j = 0; j < 8; ++j)
                              v[j] = acc[s / 2][8 * (s % 2) + j];
                          bs[s] = split8(v);
                      });
                  });
        };
        const int n_split = __any(range.outside(pk.limit)) ? 0 : pk.n_hidden;   // (the fp32 path follows)
        for (int h = 0; h < n_split; ++h)
            hidden(h);
        // the next tile's inputs are requested here, where the activations'
        // splits are free; they arrive during the output layer and the other
        // wave's work
        if (tile + order.step < order.end) {
            gather(tile + order.step, xn);
        } else {
#pragma unroll
            for (int s = 0; s < XS; ++s)
                xn[s] = 0.f;   // (keeps the old values from living through the tile)
        }

        // ---- output layer + scatter through the `from` map: four outputs by
        //      sixteen 4 x 4 blocks of the fp32 matrix instruction, one k each
        //      (v_mfma_f32_4x4x1_16b_f32): block l / 4 holds the points of lanes
        //      4 (l / 4) .., and the eight blocks of a lane half share the A
        //      operand of block `abid` (cbsz 3).  Each half sums its own
        //      features; swapping halves leaves output 2i in lanes 0..31 and
        //      2i + 1 in lanes 32..63.
        const float *ob = reinterpret_cast<const float *>(lds + lay.out_b()) + (ln >> 5);
        float v[2][2];   // outputs 2i + g and 4 + 2i + g
        auto outputs = [&](int group) __attribute__((always_inline)) {
            const float4 *wq = reinterpret_cast<const float4 *>(lds + lay.out_w(group)) + ln;
            float a[2 * NMB];
#pragma unroll
            for (int i = 0; i < NMB / 2; ++i) {
                const float4 w = wq[i * 64];
                a[4 * i] = w.x;
                a[4 * i + 1] = w.y;
                a[4 * i + 2] = w.z;
                a[4 * i + 3] = w.w;
            }
            floatx4 y[NMB];
            static_for<0, 16 * NMB>([&](auto k) __attribute__((always_inline)) {
                // m-blocks in turn: independent accumulators
                constexpr int mb = k % NMB, r = k / NMB, i = (16 * mb + r) / 8;
                const floatx4 zero = {};
                y[mb] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[i], acc[mb][r], r == 0 ? zero : y[mb], 3, r % 8, 0);
            });
            floatx4 sum = y[0];
#pragma unroll
            for (int mb = 1; mb < NMB; ++mb)
                sum += y[mb];
            join_halves(sum, ob + 4 * group, v[group]);
        };
        outputs(0);
        if (pk.f_out > 4)
            outputs(1);
        if (outside(range, pk.limit, pk.least, v, pk.f_out)) {
            // this tile (again) on the fp32 instruction
            float x[XS];
            gather(tile, x);
#pragma unroll
            for (int s = 0; s < XS; ++s)
                x[s] = 2 * s + (ln >> 5) < F ? x[s] : 0.f;
            layers_plain<NMB, KS1, LOG>(pk, x, fl, gl, lds, lay, ln >> 5, acc);
            outputs(0);
            if (pk.f_out > 4)
                outputs(1);
        }
        const MapsLds &tab = maps();
        const OutPoint po(tab, rank_out, out_offsets, valid ? b : n_points - 1);
        const bool orelu = pk.relu >> (pk.n_hidden + 1) & 1;
        po.store(tab, v[0][0], v[0][1], 0, pk.f_out, g, orelu, valid);
        if (pk.f_out > 4)
            po.store(tab, v[1][0], v[1][1], 4, pk.f_out, g, orelu, valid);
    }
}

SplitLayout split_layout(const F32Packed &pk) {
    return SplitLayout{pk.hid / 32, (pk.ks1 + 7) / 8, pk.n_hidden, pk.f_out};
}

template <int NMB, int KS1, bool LOG>
hipError_t launch_t(const Map32 &in, const Map32 &out, const FeatTable32 &tin, const FeatTable32 &tout,
                    const F32Packed &pk, hipStream_t stream) {
    const int32_t n_tiles = (in.n_points + 31) / 32;
    const int threads = NMB == 4 ? 512 : 256;
    const int waves = threads / 64;
    const size_t lds = (size_t)split_layout(pk).lds(LOG);
    // blocks per CU: by registers, one of 8 waves (H = 128) or three of 4; by LDS
    int per_cu = NMB == 4 ? 1 : 3;
    per_cu = std::max(1, std::min(per_cu, (int)(kLdsMax / (lds + 1024))));
    int64_t grid = 256LL * per_cu;
    const int64_t need = (n_tiles + waves - 1) / waves;
    if (grid > need)
        grid = need;
    // windowed maps: one contiguous range of tiles per XCD (see the kernel)
    bool window = false;
    for (int d = 0; d < in.rank; ++d)
        window = window || in.omin[d] != 0 || in.omax[d] != 0;
    bool offsets = false;   // of the `from` map
    for (int d = 0; d < out.rank; ++d)
        offsets = offsets || out.omin[d] != 0 || out.omax[d] != 0;
    const int32_t xcd_ranges = window && grid % 8 == 0;
    auto kern = mlp_f32_kernel<NMB, KS1, LOG>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(threads), lds, stream, in, out, tin, tout, pk, n_tiles,
                       (int32_t)window, (int32_t)offsets, xcd_ranges);
    return hipGetLastError();
}

template <int NMB, int KS1>
hipError_t launch_k(const Map32 &in, const Map32 &out, const FeatTable32 &tin, const FeatTable32 &tout,
                    const F32Packed &pk, hipStream_t stream) {
    return split_layout(pk).lds(false) <= kLdsMax ? launch_t<NMB, KS1, false>(in, out, tin, tout, pk, stream)
                                                  : launch_t<NMB, KS1, true>(in, out, tin, tout, pk, stream);
}

}  // namespace

bool f32_fast_supported(int n_layers, const int32_t *dims, int compute) {
    if (compute != HPACML_F32 || n_layers < 2 || n_layers > HPACML_MAX_LAYERS)
        return false;
    const int H = dims[1];
    if (H != 64 && H != 128)
        return false;
    for (int l = 1; l < n_layers; ++l)
        if (dims[l] != H)
            return false;
    if (dims[0] > 64 || dims[n_layers] > kFoutMax)
        return false;
    return SplitLayout{H / 32, (dims[0] + 15) / 16, n_layers - 2, dims[n_layers]}.lds(true) <= kLdsMax;
}

// Host packing of the split image (see SplitLayout): A fragments in the order
// the lanes read them, biases and output weights in the C-fragment order.
void f32_pack(int n_layers, const int32_t *dims, const float *const *W, const float *const *b, std::vector<float> &image,
              F32Packed *pk) {
    const int H = dims[1], NMB = H / 32, Fin = dims[0], Fout = dims[n_layers], NH = n_layers - 2;
    const SplitLayout sl{NMB, (Fin + 15) / 16, NH, Fout};
    auto put_bias = [&](float *dst, const float *bias) {
        for (int g = 0; g < 2; ++g)
            for (int mb = 0; mb < NMB; ++mb)
                for (int r = 0; r < 16; ++r)
                    dst[(g * NMB + mb) * 16 + r] = bias[crow(mb, r, g)];
    };
    // (the output layer is on the fp32 instruction)
    LayerRows rows[HPACML_MAX_LAYERS];
    for (int l = 0; l + 1 < n_layers; ++l)
        rows[l] = LayerRows{W[l], b[l], dims[l + 1], dims[l]};
    SplitRange range;
    const bool fine = split_range(rows, n_layers - 1, largest_row_sum(W[n_layers - 1], dims[n_layers], dims[n_layers - 1]), &range);
    pk->weights = !fine ? kPlainWeights : range.tiny ? kPlainBehind : kSplitWeights;
    pk->limit = range.limit;
    pk->least = range.least;
    image.assign((sl.total() + (range.tiny ? sl.l1_lo() - sl.l1() : 0)) / 4, 0.f);
    float *img = image.data();
    auto put = [&](const float *w, int K, int steps, int hm0, int lo0, auto &&feature) {
        auto hm = [&](int s, int mb) { return hm0 + (s * NMB + mb) * 2 * kFragBytes; };
        auto lo = [&](int s, int mb) { return lo0 + (s * NMB + mb) * kFragBytes; };
        put_layer(reinterpret_cast<char *>(img), w, H, K, steps, NMB, !fine, hm, lo, feature);
        if (fine && range.tiny)
            put_layer(reinterpret_cast<char *>(img) + sl.behind(), w, H, K, steps, NMB, true, hm, lo, feature);
    };
    put(W[0], Fin, sl.ks, sl.l1(), sl.l1_lo(), [](int s, int g, int j) { return 2 * (8 * s + j) + g; });
    put_bias(img + sl.l1_bias() / 4, b[0]);
    for (int h = 0; h < NH; ++h) {
        // element j of K-step s is register 8 (s % 2) + j of m-block s / 2
        put(W[h + 1], H, 2 * NMB, sl.hidden(h), sl.hidden_lo(h),
            [](int s, int g, int j) { return crow(s / 2, 8 * (s % 2) + j, g); });
        put_bias(img + sl.hidden_bias(h) / 4, b[h + 1]);
    }
    const float *Wo = W[n_layers - 1];
    for (int o = 0; o < Fout; ++o)
        for (int i = 0; i < 2 * NMB; ++i)
            for (int g = 0; g < 2; ++g)
                for (int bb = 0; bb < 8; ++bb) {
                    const int r = 8 * i + bb, lane = 32 * g + 4 * bb + o % 4;
                    img[sl.out_w(o / 4) / 4 + (i / 4 * 64 + lane) * 4 + i % 4] = Wo[(size_t)o * H + crow(r / 16, r % 16, g)];
                }
    for (int go = 0; go < kFoutMax; ++go)
        img[sl.out_b() / 4 + go] = go < Fout ? b[n_layers - 1][go] : FLT_MAX;   // (never below `least`)
}

hipError_t launch_mlp_f32(const Map32 &in, const Map32 &out, const FeatTable32 &tin, const FeatTable32 &tout,
                          const F32Packed &pk, hipStream_t stream) {
    if (in.n_points == 0)
        return hipSuccess;
    const int ks = (pk.ks1 + 7) / 8;
#define HPACML_F32(NMB)                                                                     \
    switch (ks) {                                                                           \
    case 1: return launch_k<NMB, 1>(in, out, tin, tout, pk, stream);                        \
    case 2: return launch_k<NMB, 2>(in, out, tin, tout, pk, stream);                        \
    case 3: return launch_k<NMB, 3>(in, out, tin, tout, pk, stream);                        \
    default: return launch_k<NMB, 4>(in, out, tin, tout, pk, stream);                       \
    }
    if (pk.hid == 128) {
        HPACML_F32(4)
    }
    HPACML_F32(2)
#undef HPACML_F32
}

const char *f32_variant_name(const F32Packed &pk) {
    if (pk.hid == 128)
        return pk.ks1 <= 8 ? "mlp_f32_h128_k16" : (pk.ks1 <= 20 ? "mlp_f32_h128_k40" : "mlp_f32_h128_k64");
    return pk.ks1 <= 8 ? "mlp_f32_h64_k16" : (pk.ks1 <= 20 ? "mlp_f32_h64_k40" : "mlp_f32_h64_k64");
}

}  // namespace hpacml

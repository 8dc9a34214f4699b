// Device parts shared by the fp32 fused kernels (three-way bf16 splits of fp32
// numbers, the maps in LDS, the order of tiles, the gather and the scatter).
#pragma once

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <type_traits>
#include <vector>

#include "kernels.hpp"

namespace hpacml {

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx8 __attribute__((ext_vector_type(8)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kFoutMax = 8;
// scheduling-barrier mask: only VALU, SALU and transcendental instructions
// may be moved across
constexpr int kSchedAluOnly = 0x2 | 0x4 | 0x400;
constexpr int kFragBytes = 1024;        // one A operand: 64 lanes x 8 bf16
constexpr int kLdsMax = 160 * 1024;     // LDS of a CU
constexpr float kBig = 0x1p127f;        // this and more has no three-way split
constexpr float kLeast = 0x1p-110f;     // below it the lo part loses bits (bf16 numbers end at 2^-133)

// What a block keeps of the two maps in LDS, ahead of the split image: the
// feature tables, read with a lane's own feature number, and the 32-bit
// views, whose fields would otherwise occupy (and spill) scalar registers
// over the whole kernel.
struct MapsLds {
    Map32 in, out;
    const float *fptr[kTableMaxF];
    float *optr[kFoutMax];
    uint32_t raw8[kTableMaxF], oraw8[kFoutMax];
};
static_assert(sizeof(MapsLds) % 16 == 0 && sizeof(Map32) % 16 == 0, "read 16 bytes at a time");

// locate32 on a view in LDS: unused dimensions (count 1, stride 0) add
// nothing, those past the second are skipped for the usual ranks.
__device__ __forceinline__ Pt32 locate_lds(const Map32 &m, int rank, int32_t b) {
    Pt32 r;
    uint32_t rem = (uint32_t)b;
    r.pe = 0;
    auto dim = [&](int d) __attribute__((always_inline)) {
        uint32_t k = rem;
        if (d > 0) {
            rem = (uint32_t)(((uint64_t)rem * m.magic[d]) >> m.shift[d]);
            k -= rem * (uint32_t)m.count[d];
        }
        r.p[d] = m.start[d] + (int32_t)k * m.step[d];
        r.pe += r.p[d] * m.stride[d];
    };
    r.p[1] = r.p[2] = r.p[3] = 0;
    if (rank > 1) {
        if (rank > 2) {
            dim(3);
            dim(2);
        }
        dim(1);
    }
    dim(0);
    return r;
}

// The dimensions along which some lane of the wave reads outside the arrays.
__device__ __forceinline__ uint32_t edge_lds(const Map32 &m, int rank, const Pt32 &r) {
    uint32_t edge = 0;
#pragma unroll
    for (int d = 0; d < HPACML_MAX_RANK; ++d)
        if (d < rank && __any(r.p[d] + m.omin[d] < 0 || r.p[d] + m.omax[d] >= m.extent[d]))
            edge |= 1u << d;
    return edge;
}

// Boundary corrections of N accesses with raw offsets raw[] at point r, added
// to idx[]; `edge`: the dimensions along which some lane of the wave leaves
// the arrays.  Per dimension dl = clamp(at, 0, n - 1) - at (zero inside):
// clamp adds dl strides, periodic one wrap in dl's direction (|offset| <=
// extent).
template <int N>
__device__ __forceinline__ void fix_lds(const Map32 &m, const Pt32 &r, uint32_t edge, const uint32_t (&raw)[N],
                                        int32_t (&idx)[N]) {
#pragma unroll
    for (int d = 0; d < HPACML_MAX_RANK; ++d) {
        if (edge & (1u << d)) {
            const int32_t n = m.extent[d], st = m.stride[d];
            const bool per = m.bnd[d] == HPACML_BND_PERIODIC;
            const int32_t lim = per ? 1 : INT32_MAX, mul = per ? (int32_t)((uint32_t)n * (uint32_t)st) : st;
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const int32_t at = r.p[d] + (int32_t)(int8_t)(raw[j] >> (8 * d));
                const int32_t dl = min(max(at, 0), n - 1) - at;
                idx[j] += min(max(dl, -lim), lim) * mul;
            }
        }
    }
}

// feature held by lane half g in register r of m-block mb
__host__ __device__ inline int crow(int mb, int r, int g) { return 32 * mb + 8 * (r / 4) + 4 * g + (r % 4); }

// N m-blocks from m-block mb0 on
template <int NMB, int N = NMB>
__device__ __forceinline__ void load_bias(const float *bias, int g, floatx16 *acc, int mb0 = 0) {
#pragma unroll
    for (int mb = 0; mb < N; ++mb) {
        const float4 *p = reinterpret_cast<const float4 *>(bias + (g * NMB + mb0 + mb) * 16);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float4 v = p[q];
            acc[mb][4 * q + 0] = v.x;
            acc[mb][4 * q + 1] = v.y;
            acc[mb][4 * q + 2] = v.z;
            acc[mb][4 * q + 3] = v.w;
        }
    }
}

// compile-time loop: fn(std::integral_constant<int, i>) for i in [B, E)
template <int B, int E, typename Fn>
__device__ __forceinline__ void static_for(Fn &&fn) {
    if constexpr (B < E) {
        fn(std::integral_constant<int, B>{});
        static_for<B + 1, E>(fn);
    }
}

// Two floats in three bf16 parts each (a in the lower halves), v = hi + mid + lo
// (exactly, see mlp_f32.hip).
__device__ __forceinline__ void split2(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l) {
    h = __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2){a, b}, bf16x2));
    const float ra = a - __uint_as_float(h << 16), rb = b - __uint_as_float(h & 0xFFFF0000u);
    m = __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2){ra, rb}, bf16x2));
    const float la = ra - __uint_as_float(m << 16), lb = rb - __uint_as_float(m & 0xFFFF0000u);
    l = __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2){la, lb}, bf16x2));
}

// Eight floats as three B fragments.
struct Split {
    u32x4 hi, mid, lo;
};
__device__ __forceinline__ Split split8(floatx8 v) {
    Split f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t h, m, l;
        split2(v[2 * i], v[2 * i + 1], h, m, l);
        f.hi[i] = h;
        f.mid[i] = m;
        f.lo[i] = l;
    }
    return f;
}

__device__ __forceinline__ floatx16 mfma(u32x4 a, u32x4 b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The larger of m and two magnitudes (a NaN is passed over); for values that
// the vector ALU made (not MFMA results: the compiler does not see the read).
__device__ __forceinline__ float max_abs(float a, float b, float m) {
    float r;
    asm("v_max3_f32 %0, |%1|, |%2|, %3" : "=v"(r) : "v"(a), "v"(b), "v"(m));
    return r;
}

// Lower bound of a layer's activation: 0 (ReLU) or none.
__device__ __forceinline__ float act_floor(bool relu) { return relu ? 0.f : -FLT_MAX; }

// The magnitudes that a lane met among a layer's inputs.
struct Range {
    float top = 0.f;   // the largest (a NaN is passed over)
    __device__ __forceinline__ void add(float a, float b) { top = max_abs(a, b, top); }
    // Whether a sum could overflow (limit: see split_range).
    __device__ __forceinline__ bool outside(float limit) const { return top >= limit; }
};

// Activation as one v_med3_f32(x, floor, FLT_MAX), without a branch, so that it
// can be scheduled beside matrix instructions; the magnitudes join `range`.
// Only a NaN among the inputs makes a NaN here (no sum overflows, see
// split_range).  It becomes the floor (v_med3_f32 returns the least of the other
// two): 0 under ReLU, and the -FLT_MAX of an identity layer, like any
// magnitude of 2^127 and more, sends the tile to the fp32 instruction.
template <int N>
__device__ __forceinline__ void activate(floatx16 *acc, float floor, Range &range) {
#pragma unroll
    for (int mb = 0; mb < N; ++mb)
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            acc[mb][r] = __builtin_amdgcn_fmed3f(acc[mb][r], floor, FLT_MAX);
            acc[mb][r + 1] = __builtin_amdgcn_fmed3f(acc[mb][r + 1], floor, FLT_MAX);
            range.add(acc[mb][r], acc[mb][r + 1]);
        }
}

// Where the fp32 path of a tile has its weights: the split image's fragments put
// together (hi + mid + lo is the weight, exactly, from 2^-110 up), or fragments of
// fp32 weights (see put_layer) in the image's place in LDS or, for a model with
// smaller weights, behind the image in global memory.
enum WeightForm : int32_t { kSplitWeights = 0, kPlainWeights = 1, kPlainBehind = 2 };

// One K-step of an m-block on the fp32 matrix instruction: a fragment (h, m, l)
// holds rows and columns as eight of its A operands do; x: features (s, g, 0 .. 7)
// of the lane's point.
__device__ __forceinline__ floatx16 mfma_plain(u32x4 h, u32x4 m, u32x4 l, int form, const float *x, floatx16 acc) {
    float w[8];
    if (form == kSplitWeights) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            w[2 * i] = (__uint_as_float(h[i] << 16) + __uint_as_float(m[i] << 16)) + __uint_as_float(l[i] << 16);
            w[2 * i + 1] = (__uint_as_float(h[i] & 0xFFFF0000u) + __uint_as_float(m[i] & 0xFFFF0000u)) +
                           __uint_as_float(l[i] & 0xFFFF0000u);
        }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            w[j] = __uint_as_float(j < 4 ? h[j] : m[j - 4]);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w[j], x[j], acc, 0, 0, 0);
    return acc;
}

// Activation of the fp32 path: ReLU (a NaN gives 0) or nothing; m-blocks mb0 on of
// a layer of `width` neurons.  Those past it are 0 whatever the inputs (an
// infinite input times their weights of 0 is a NaN).
template <int N>
__device__ __forceinline__ void activate_plain(floatx16 *acc, bool relu, int mb0, int g, int width) {
    asm volatile("" : "+v"(g));   // (compared here, not ahead of the tiles)
#pragma unroll
    for (int mb = 0; mb < N; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float v = relu ? relu_mfma(acc[mb][r]) : acc[mb][r];
            acc[mb][r] = crow(mb0 + mb, r, g) < width ? v : 0.f;
        }
}

// Which tiles of 32 points a wave takes: first, first + step, ... below end.
// XCD-aware (blocks of one XCD, hardware id % 8, share an L2).  Pointwise
// maps: each round of the grid takes adjacent tiles per XCD.  Windowed maps
// (xcd_ranges, grid a multiple of 8): each XCD walks one contiguous eighth of
// the tiles, so the rows a window shares with the tiles before it are still in
// that XCD's L2.
struct TileOrder {
    int first, step, end;
    __device__ TileOrder(int32_t n_tiles, int32_t xcd_ranges) {
        const int nb = gridDim.x, waves = blockDim.x >> 6, w = threadIdx.x >> 6;
        if (xcd_ranges) {
            const int per = (n_tiles + 7) / 8;
            const int x = blockIdx.x % 8;
            first = x * per + (blockIdx.x / 8) * waves + w;
            step = (nb / 8) * waves;
            end = (x + 1) * per < n_tiles ? (x + 1) * per : n_tiles;
        } else {
            const int lb = (nb % 8 == 0) ? (blockIdx.x % 8) * (nb / 8) + blockIdx.x / 8 : blockIdx.x;
            first = lb * waves + w;
            step = nb * waves;
            end = n_tiles;
        }
    }
};

// The block's copy of the maps (blocks of at least 256 threads; a barrier follows).
__device__ __forceinline__ void stage_maps(MapsLds &tab, const Map32 &in, const Map32 &out, const FeatTable32 &tin,
                                           const FeatTable32 &tout) {
    const int t = threadIdx.x;
    constexpr int kWords = (int)(sizeof(Map32) / 4);
    static_assert(kWords <= 64, "one word per thread");
    if (t < kTableMaxF) {
        tab.fptr[t] = tin.fptr[t];
        tab.raw8[t] = tin.raw8[t];
    } else if (t < 64 + kFoutMax) {
        tab.optr[t - 64] = const_cast<float *>(tout.fptr[t - 64]);
        tab.oraw8[t - 64] = tout.raw8[t - 64];
    } else if (t >= 128 && t < 128 + kWords) {
        ((int32_t *)&tab.in)[t - 128] = ((const int32_t *)&in)[t - 128];
    } else if (t >= 192 && t < 192 + kWords) {
        ((int32_t *)&tab.out)[t - 192] = ((const int32_t *)&out)[t - 192];
    }
}

// Inputs of point b: lane half g loads features 2t + g into the slots t,
// through the table's entry of that feature (entries past the last feature
// repeat it).  Four slots at a time: table entries, boundary fix-ups along the
// dimensions where the wave touches an edge, then the loads; the last four
// slots are left out where no feature reaches them (pairs: ceil(F / 2)).
template <int KS1>
__device__ __forceinline__ void gather_inputs(const MapsLds &tab, int rank, int32_t n_points, bool windowed, int pairs,
                                              int32_t b, int g, float (&x)[8 * KS1]) {
    const Pt32 pt = locate_lds(tab.in, rank, b < n_points ? b : n_points - 1);
    const uint32_t edge = windowed ? edge_lds(tab.in, rank, pt) : 0u;
    static_for<0, 2 * KS1>([&](auto q) __attribute__((always_inline)) {
        constexpr int s0 = 4 * q;
        if (q < 2 * KS1 - 1 || s0 < pairs) {
            int32_t idx[4] = {pt.pe, pt.pe, pt.pe, pt.pe};
            if (edge) {
                const uint32_t raw[4] = {tab.raw8[2 * s0 + g], tab.raw8[2 * s0 + 2 + g], tab.raw8[2 * s0 + 4 + g],
                                         tab.raw8[2 * s0 + 6 + g]};
                fix_lds<4>(tab.in, pt, edge, raw, idx);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                x[s0 + j] = ldg(tab.fptr[2 * (s0 + j) + g] + idx[j]);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                x[s0 + j] = 0.f;
        }
    });
}

// Four outputs: each lane half holds its own features' sums of outputs go .. go +
// 3; swapping halves leaves output go + 2i in lanes 0..31 and go + 2i + 1 in lanes
// 32..63.  (bias: kFoutMax of them)
__device__ __forceinline__ void join_halves(floatx4 sum, const float *bias, float (&v)[2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum[2 * i]), __float_as_uint(sum[2 * i + 1]),
                                                         false, false);
        v[i] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]) + bias[2 * i];
    }
}

// Whether the split products may not serve a point of the wave: a value too large
// for them, or an output (v: those of this lane; FLT_MAX past the last) so small
// that the bits which tiny values lose would show in it (see split_range).  All
// outputs of a point whose inputs and activations are 0 are exact.
__device__ __forceinline__ bool outside(const Range &range, float limit, float least, const float (&v)[2][2], int f_out) {
    float low = fminf(fabsf(v[0][0]), fabsf(v[0][1]));
    if (f_out > 4)
        low = fminf(low, fminf(fabsf(v[1][0]), fabsf(v[1][1])));
    if (!__any(range.outside(limit) || low < least))
        return false;
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(range.top), __float_as_uint(range.top), false, false);
    const float top = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    return __any(range.outside(limit) || (top > 0.f && low < least));
}

// A point of the `from` map, and the store of outputs go + g and go + 2 + g.
struct OutPoint {
    Pt32 p;
    uint32_t edge;
    __device__ __forceinline__ OutPoint(const MapsLds &tab, int rank, bool offsets, int32_t b) {
        p = locate_lds(tab.out, rank, b);
        edge = offsets ? edge_lds(tab.out, rank, p) : 0u;
    }
    __device__ __forceinline__ void store(const MapsLds &tab, float v0, float v1, int go, int f_out, int g, bool relu,
                                          bool valid) const {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int o = go + 2 * i + g;
            if (o < f_out) {
                float v = i ? v1 : v0;
                if (relu)
                    v = fmaxf(v, 0.f);
                int32_t idx[1] = {p.pe};
                if (edge) {
                    const uint32_t raw[1] = {tab.oraw8[o]};
                    fix_lds<1>(tab.out, p, edge, raw, idx);
                }
                if (valid)
                    stg(tab.optr[o] + idx[0], v);
            }
        }
    }
};

// The values that a stack of layers can leave to the split products; false when
// every tile has to take the fp32 path.  `after`: the largest row sum of |w| of
// the layer behind them (1: none).
//
// limit: no sum overflows for inputs (of any layer) below it.  With the largest
// row sum of |w| the products of a row, and the bias, come to 2^126 each, so
// that hi hi (at most 1 + 2^-6 times as large) and the sums of small products
// stay finite.  Otherwise an infinite sum of hi hi could meet small products that
// are infinite with the other sign, where the fp32 sum is infinite.
//
// least: a value below 2^-110 loses what its split has below 2^-133, at most
// 2^-134.  Through a layer that makes row sum x 2^-134, and 2^-134 K x the largest
// input (kept below 2^40 then) where a weight is that small; the layers behind
// multiply it by their row sums at most.  Outputs of 2^26 times the whole and
// more keep their 24 bits.
struct LayerRows {
    const float *W, *b;   // [N][K], [N]
    int N, K;
};
struct SplitRange {
    float limit, least;
    bool tiny;   // a weight loses bits
};
inline bool split_range(const LayerRows *layers, int n, double after, SplitRange *r) {
    double limit = kBig, lost = 0;
    *r = SplitRange{};
    for (int l = n - 1; l >= 0; --l) {
        const LayerRows &y = layers[l];
        double worst = 0;
        bool tiny = false;
        for (int o = 0; o < y.N; ++o) {
            double sum[4] = {};
            float low = kBig, top = 0.f;   // the least but 0
            const float *w = y.W + (size_t)o * y.K;
            for (int k = 0; k < y.K; ++k) {
                const float a = std::fabs(w[k]);
                sum[k % 4] += a;
                low = std::min(low, a > 0.f ? a : kBig);
                top = std::max(top, a);
            }
            const double all = (sum[0] + sum[1]) + (sum[2] + sum[3]);
            // (a weight without a split, or a bias without room)
            if (!(all < HUGE_VAL) || top >= kBig || !(std::fabs(y.b[o]) < 0.5f * kBig))
                return false;
            worst = std::max(worst, all);
            tiny = tiny || low < kLeast;
        }
        if (worst > 0.5)
            limit = std::min(limit, 0.5 * kBig / worst * (1 - 0x1p-20));
        lost += after * (worst + (tiny ? 0x1p40 * y.K : 0));
        after *= worst;
        r->tiny = r->tiny || tiny;
    }
    if (r->tiny)
        limit = std::min(limit, 0x1p40);
    r->limit = (float)limit;
    r->least = (float)(0x1p-108 * lost);   // 2^26 x 2^-134
    return lost < 0x1p200;
}
inline double largest_row_sum(const float *W, int N, int K) {
    double worst = 0;
    for (int o = 0; o < N; ++o) {
        double sum = 0;
        for (int k = 0; k < K; ++k)
            sum += std::fabs((double)W[(size_t)o * K + k]);
        worst = std::max(worst, sum);
    }
    return worst;
}

// Host side of the split: rounded to nearest even, as the device's conversion
// (finite values).
inline uint16_t rne(float x) {
    uint32_t u = __builtin_bit_cast(uint32_t, x);
    return (uint16_t)((u + 0x7FFFu + (u >> 16 & 1u)) >> 16);
}
inline float bf16_float(uint16_t h) { return __builtin_bit_cast(float, (uint32_t)h << 16); }
inline void split_parts(float w, uint16_t &h, uint16_t &m, uint16_t &l) {
    h = rne(w);
    const float r = w - bf16_float(h);
    m = rne(r);
    l = rne(r - bf16_float(m));
}

// One layer's A fragments: K-step s, m-block mb, lane l, element j is weight
// [32 mb + l % 32][feature(s, l / 32, j)] (zero past N rows and K columns), its
// parts at img + hm(s, mb) (hi, then mid) and img + lo(s, mb); `plain`: the
// weights themselves, elements 0 .. 3 in place of hi and 4 .. 7 in place of mid.
template <typename Hm, typename Lo, typename Feature>
inline void put_layer(char *img, const float *W, int N, int K, int steps, int blocks, bool plain, Hm &&hm, Lo &&lo,
                      Feature &&feature) {
    // split the layer in its own order (a loop the compiler vectorises), then
    // place the parts
    const size_t n = (size_t)N * K;
    std::vector<uint16_t> q(plain ? 0 : 3 * n);
    uint16_t *qh = q.data(), *qm = qh + n, *ql = qm + n;
    for (size_t i = 0; !plain && i < n; ++i)
        split_parts(W[i], qh[i], qm[i], ql[i]);
    for (int s = 0; s < steps; ++s) {
        int at[2][8];
        for (int g = 0; g < 2; ++g)
            for (int j = 0; j < 8; ++j)
                at[g][j] = feature(s, g, j);
        for (int mb = 0; mb < blocks; ++mb) {
            uint16_t *h = reinterpret_cast<uint16_t *>(img + hm(s, mb)), *m = h + kFragBytes / 2;
            uint16_t *l = reinterpret_cast<uint16_t *>(img + lo(s, mb));
            float *f = reinterpret_cast<float *>(img + hm(s, mb));
            for (int lane = 0; lane < 64; ++lane) {
                if (32 * mb + lane % 32 >= N)
                    continue;
                const size_t row = (size_t)(32 * mb + lane % 32) * K;
                for (int j = 0; j < 8; ++j) {
                    const int k = at[lane / 32][j];
                    if (k < K && plain) {
                        f[(j / 4) * (kFragBytes / 4) + lane * 4 + j % 4] = W[row + k];
                    } else if (k < K) {
                        h[lane * 8 + j] = qh[row + k];
                        m[lane * 8 + j] = qm[row + k];
                        l[lane * 8 + j] = ql[row + k];
                    }
                }
            }
        }
    }
}

}  // namespace

}  // namespace hpacml

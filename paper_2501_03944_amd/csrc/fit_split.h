// FP32 fitness of register-chain networks on the FP16 matrix units, instantiated by the
// split_*.hip files (the frame is fit_kernel.h's: transposed layers, 16-sample slabs,
// weights staged in LDS, layers chained in registers).
//
// The FP32 matrix rate (157 TFLOP/s) bounds fit_kernel.h's FP32 kernels (0.82 of it at
// 64-128-128-10).  Here every operand of a layer is two FP16 parts of the value times a
// power of two, v 2^e = hi + lo 2^-12, and a layer is three FP16 products per K block,
// W_hi H_hi in one accumulator and W_lo H_hi + W_hi H_lo in a second one whose scale is
// 2^12 times the first one's, both FP32 (bound 833 TFLOP/s).  Bias, activation and loss
// are FP32 on the true scale.
//
// Range: with its largest value in [2^14, 2^15), a set of values that shares an exponent
// is held to a last bit of FP32 (2^-23 of the value) down to 2^-14, that is over 2^29:
// below, hi is a subnormal and lo runs out of bits.  (Without the scale of lo it would be
// 2^17, and one weight in ten of a network falls below that.)  What shares an exponent: the
// weights of a layer (the search box's exponent, or where that does not hold a row, which
// need not lie in the box, its own largest weight's; biases take no part),
// the inputs of a sample (Xe), and the activations of a sample and layer.  Exponents are
// kept to +-60, so that all scales are normal FP32 values.
//
// What the parts do not hold goes through FP32 instructions, never rounded: weights are
// compared with their parts as they are staged, inputs when they are packed (Xe), the
// activations of a sample by their least magnitude but zero against its exponent.  Rows
// whose weights fail and slab groups with a sample or an activation that does (values
// that are not finite among them) are marked and taken by fit_kernel.h's slab_group once
// the block has been through its samples, with the row's FP32 weights staged in place of
// the parts.  Ordinary rows mark a slab group in ten million.
//
// The conversion of the hidden activations to parts is vector work (about eight
// instructions per value) beside the products; two slabs per wavefront share each
// weight fragment's LDS read, and two wavefronts per SIMD overlap one's conversions
// with the other's products.
//
// Measured, FP32 instructions -> so: a generation of 64-128-128-10 (2,048 sparks x 4,096
// samples) 3,478 -> 1,455 us; 300 rows x 4,096 samples of it 574 -> 282 us, their error
// against binary64 5.2e-8 -> 2.9e-8.  (Lo parts on the scale of the hi parts, in one
// accumulator: 1,355 and 260 us, right over 2^17 only.)
#pragma once

#include "fit_kernel.h"

namespace mgfwa {
namespace fit {

typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));

// The parts of one B operand (eight values of a lane).
struct Parts {
    halfx8 hi, lo;
};

// (a, b) c as parts, pairs converted by one instruction each (gfx950).
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void split8(const floatx4 &a, const floatx4 &b, float c, Parts &p)
{
    const float cl = c * SPLIT_LO_UP;
    uint4v hi, lo;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float x = i < 2 ? a[2 * (i & 1)] : b[2 * (i & 1)];
        const float y = i < 2 ? a[2 * (i & 1) + 1] : b[2 * (i & 1) + 1];
        const halfx2 h = __builtin_convertvector((floatx2){x * c, y * c}, halfx2);
        // (as a multiply-add, which takes the FP16 half as it is)
        const floatx2 r = {__builtin_fmaf((float)h[0], -SPLIT_LO_UP, x * cl),
                           __builtin_fmaf((float)h[1], -SPLIT_LO_UP, y * cl)};
        hi[i] = __builtin_bit_cast(uint32_t, h);
        lo[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, halfx2));
    }
    p.hi = __builtin_bit_cast(halfx8, hi);
    p.lo = __builtin_bit_cast(halfx8, lo);
}

// One lane's view of a layer's staged weights.  A row holds, per 32-column block, 32 hi
// and then 32 lo elements, 16-byte chunk c of row r stored at chunk c ^ (r & 1).  Behind
// the first layer the row's pitch follows from the row blocks of the layer before, so that
// every fragment's place is an immediate offset.
template <int RI>
struct SplitView {
    const _Float16 *p;
    int runtime_pitch;
    __device__ __forceinline__ SplitView(const FitArgs &a, const char *smem, int l, int n, int g)
    {
        runtime_pitch = a.lay.lpitch[l];
        p = reinterpret_cast<const _Float16 *>(smem) + a.lay.lw[l] + n * pitch() + 8 * (g ^ (n & 1));
    }
    __device__ __forceinline__ int pitch() const { return RI > 0 ? split_pitch(32 * ((RI + 1) / 2)) : runtime_pitch; }
    __device__ __forceinline__ void load(int rb, int kb, halfx8 &hi, halfx8 &lo) const
    {
        const _Float16 *q = p + 16 * rb * pitch() + 64 * kb;
        hi = *reinterpret_cast<const halfx8 *>(q);
        lo = *reinterpret_cast<const halfx8 *>(q + 32);
    }
};

// The spark's weights as parts into LDS (zero-padded; layer l times 2^wexp[l], wexp in
// LDS), biases into the FP32 area.  False when the parts do not hold a weight (the same in
// every thread).
__device__ __forceinline__ bool stage_split(const FitArgs &a, const float *w, int r, char *smem, const int *wexp)
{
    float *bias = reinterpret_cast<float *>(smem + a.lay.bias_byte);
    const bool regen = a.rg.F != nullptr;
    const int nt = blockDim.x;
    bool held = true;
    for (int l = 0; l < a.nl; ++l) {
        const int fo = a.fo[l], fi = a.fi[l], rows = a.lay.lrows[l], cols = a.lay.lcols[l];
        const int pitch = a.lay.lpitch[l];
        _Float16 *dst = reinterpret_cast<_Float16 *>(smem) + a.lay.lw[l];
        const float *src = w + a.woff[l];
        const int n4 = rows * cols / 4;
        const bool vec = a.vec[l] != 0;
        const float c = __builtin_ldexpf(1.0f, wexp[l]);
        for (int i0 = threadIdx.x; i0 < n4; i0 += 4 * nt) {
            floatx4 v[4];
            int at[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int idx = i0 + u * nt;
                const int o = (4 * idx) / cols, k = 4 * idx - o * cols;
                const int pos = split_pos(k);   // (in the block's hi elements)
                at[u] = idx < n4 ? o * pitch + (((pos & ~31) + pos) ^ ((o & 1) << 3)) : -1;
                const bool live = idx < n4 && o < fo && k < fi;
                if (!live) {
                    v[u] = zero4();
                } else if (vec) {
                    v[u] = regen ? regen_chunk(a.rg, r, (a.woff[l] + o * fi + k) >> 2)
                                 : *reinterpret_cast<const floatx4 *>(src + (size_t)o * fi + k);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        v[u][e] = k + e < fi ? spark_at(a, w, r, a.woff[l] + o * fi + k + e) : 0.0f;
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (at[u] < 0) continue;
                typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));
                halfx4 hi, lo;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const ChainParts p = chain_parts(v[u][e] * c);
                    hi[e] = p.hi;
                    lo[e] = p.lo;
                    held &= p.held;
                }
                *reinterpret_cast<halfx4 *>(dst + at[u]) = hi;
                *reinterpret_cast<halfx4 *>(dst + 32 + at[u]) = lo;
            }
        }
        for (int o = threadIdx.x; o < rows; o += nt)
            bias[a.lay.lb[l] + o] = o < fo ? spark_at(a, w, r, a.boff[l] + o) : 0.0f;
    }
    return __syncthreads_and(held) != 0;
}

// The exponents of the row's layers from their largest weights, into wexp (LDS; a barrier
// before and behind).
__device__ __forceinline__ void row_exps(const FitArgs &a, const float *w, int r, int *wexp)
{
    const int lane = threadIdx.x & 63;
    if (threadIdx.x < MAXL) wexp[threadIdx.x] = 0;
    __syncthreads();
    for (int l = 0; l < a.nl; ++l) {
        const int j0 = a.woff[l], j1 = a.boff[l];
        float m = 0.0f;
        for (int c0 = (j0 >> 2) + threadIdx.x; 4 * c0 < j1; c0 += 4 * blockDim.x) {
            floatx4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = c0 + u * blockDim.x;
                v[u] = 4 * c >= j1 ? zero4()
                       : a.rg.F ? regen_chunk(a.rg, r, c)
                                : reinterpret_cast<const floatx4 *>(w)[c];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int j = 4 * (c0 + u * (int)blockDim.x) + e;
                    if (j >= j0 && j < j1) m = fmaxf(m, fabsf(v[u][e]));
                }
        }
        for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
        // (magnitudes are ordered as their bits are; a NaN took no part)
        if (lane == 0) atomicMax(&wexp[l], __float_as_int(m));
    }
    __syncthreads();
    if (threadIdx.x < MAXL) wexp[threadIdx.x] = part_exp(__int_as_float(wexp[threadIdx.x]));
    __syncthreads();
}

// The products of row blocks RB0 .. RB0 + G - 1 in one K block, fragments one row block
// ahead: W_hi H_hi into out (FIRST: from zero), the cross products into cr (CLEAR: from
// zero).
template <bool FIRST, bool CLEAR, int RB0, int G, int P, int RO, int RI>
__device__ __forceinline__ void split_kblock(const SplitView<RI> &wv, int kb, const Parts (&x)[P],
                                             floatx4 (&out)[P][RO], floatx4 (&cr)[P][G])
{
    halfx8 hi, lo;
    wv.load(RB0, kb, hi, lo);
#pragma unroll
    for (int i = 0; i < G; ++i) {
        halfx8 hn = hi, ln = lo;
        if (i + 1 < G) wv.load(RB0 + i + 1, kb, hn, ln);
#pragma unroll
        for (int p = 0; p < P; ++p)
            cr[p][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(lo, x[p].hi, CLEAR ? zero4() : cr[p][i], 0, 0, 0);
#pragma unroll
        for (int p = 0; p < P; ++p)
            out[p][RB0 + i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                hi, x[p].hi, FIRST ? zero4() : out[p][RB0 + i], 0, 0, 0);
#pragma unroll
        for (int p = 0; p < P; ++p)
            cr[p][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, x[p].lo, cr[p][i], 0, 0, 0);
        hi = hn;
        lo = ln;
        // (keeps later fragments' reads and K blocks' conversions from moving up, whose
        // registers would spill)
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Pre-activations on the true scale: (out + cr 2^-12) c + bias (bias: this lane's of the
// layer), two roundings.
template <int RB0, int G, int P, int RO>
__device__ __forceinline__ void split_finish(floatx4 (&out)[P][RO], const floatx4 (&cr)[P][G],
                                             const float (&c)[P], const char *bias)
{
#pragma unroll
    for (int i = 0; i < G; ++i) {
        const floatx4 b = *reinterpret_cast<const floatx4 *>(bias + 64 * (RB0 + i));
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                out[p][RB0 + i][v] = __builtin_fmaf(
                    out[p][RB0 + i][v], c[p], __builtin_fmaf(cr[p][i][v], c[p] * SPLIT_LO_DOWN, b[v]));
        if (i & 1) asm volatile("" ::: "memory");   // (all biases at once would spill)
    }
}

// This lane's biases of layer l: 16 bytes per row block, 64 bytes apart.
__device__ __forceinline__ const char *split_bias(const FitArgs &a, const char *smem, int l, int g)
{
    return smem + a.lay.bias_byte + (size_t)(a.lay.lb[l] + 4 * g) * 4;
}

// The two accumulators' sum, on the scale of the first.
template <int RB0, int G, int P, int RO>
__device__ __forceinline__ void split_join(floatx4 (&out)[P][RO], const floatx4 (&cr)[P][G])
{
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int i = 0; i < G; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                out[p][RB0 + i][v] = __builtin_fmaf(cr[p][i][v], SPLIT_LO_DOWN, out[p][RB0 + i][v]);
}

// Registers of a lane with NW wavefronts on a compute unit, less what the addresses,
// biases, loss and the weights' fragments take.
template <int NW>
constexpr int split_regs()
{
    return 512 / ((NW + 3) / 4) - 46;
}

// Row blocks of the first layer whose cross products are accumulated at a time, beside all
// RO accumulators and the parts of two K blocks.
template <int NW, int P, int RO>
constexpr int split_rows()
{
    constexpr int most = (split_regs<NW>() - 4 * P * RO - 16 * P) / (4 * P);
    constexpr int groups = most >= RO ? 1 : most < 2 ? (RO + 1) / 2 : (RO + most - 1) / most;
    return (RO + groups - 1) / groups;
}

// K blocks kb and kb + 1 (if there is one) of a layer, G row blocks after the other; the
// cross products join the others behind them.
template <bool FIRST, int G, int RB0, int P, int RO>
__device__ __forceinline__ void split_pair(const SplitView<0> &wv, int kb, int nkb, const Parts (&x0)[P],
                                           const Parts (&x1)[P], floatx4 (&out)[P][RO])
{
    constexpr int GN = RO - RB0 < G ? RO - RB0 : G;
    floatx4 cr[P][GN];
    split_kblock<FIRST, true, RB0, GN>(wv, kb, x0, out, cr);
    if (kb + 1 < nkb) split_kblock<false, false, RB0, GN>(wv, kb + 1, x1, out, cr);
    split_join<RB0, GN>(out, cr);
    if constexpr (RB0 + GN < RO) split_pair<FIRST, G, RB0 + GN>(wv, kb, nkb, x0, x1, out);
}

// First layer: the samples' inputs, packed as parts (k_pack_split).
template <int G, int P, int RO>
__device__ __forceinline__ void split_layer_x(const FitArgs &a, const SplitView<0> &wv, int s0, int n, int g,
                                              const float (&c)[P], const char *bias, floatx4 (&out)[P][RO])
{
    const int nkb = (a.in_pad + 31) >> 5, pitch = 32 * nkb;
    const _Float16 *xp = a.Xs + (size_t)(s0 + n) * pitch + 8 * g;
    const size_t plane = (size_t)a.S_pad * pitch;
    auto fetch = [&](int kb, Parts (&x)[P]) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const _Float16 *q = xp + (size_t)16 * p * pitch + 32 * kb;
            x[p].hi = *reinterpret_cast<const halfx8 *>(q);
            x[p].lo = *reinterpret_cast<const halfx8 *>(q + plane);
        }
    };
    if constexpr (RO <= 10) {
        floatx4 cr[P][RO];
        Parts x[P];
        fetch(0, x);
        split_kblock<true, true, 0, RO>(wv, 0, x, out, cr);
        for (int kb = 1; kb < nkb; ++kb) {
            fetch(kb, x);
            split_kblock<false, false, 0, RO>(wv, kb, x, out, cr);
        }
        split_finish<0, RO>(out, cr, c, bias);
        return;
    }
    // with more row blocks, two K blocks at a time: their inputs are loaded together, and
    // once for all groups (64-192-10, 512 rows x 2,900 samples: 278 -> 216 us; with one row
    // block to a multiply's wait it costs instead, 32-96-10 93 -> 107 us)
    Parts x0[P], x1[P];
    fetch(0, x0);
    fetch(min(1, nkb - 1), x1);
    split_pair<true, G, 0>(wv, 0, nkb, x0, x1, out);
    for (int kb = 2; kb < nkb; kb += 2) {
        fetch(kb, x0);
        fetch(min(kb + 1, nkb - 1), x1);
        split_pair<false, G, 0>(wv, kb, nkb, x0, x1, out);
    }
#pragma unroll
    for (int rb = 0; rb < RO; ++rb) {
        const floatx4 b = *reinterpret_cast<const floatx4 *>(bias + 64 * rb);
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int v = 0; v < 4; ++v) out[p][rb][v] = __builtin_fmaf(out[p][rb][v], c[p], b[v]);
        if (rb & 1) asm volatile("" ::: "memory");
    }
}

// The largest of three, one instruction (a NaN is passed over).
__device__ __forceinline__ float max3(float a, float b, float c)
{
    float d;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

// Activation of a layer's pre-activations; of a sample's values in this lane, m is the largest magnitude, and least the bits of the
// smallest but zero, less one (ReLU; else doubled, less one).
template <int ACT, int P, int R>
__device__ __forceinline__ void split_apply(floatx4 (&h)[P][R], float (&m)[P], uint32_t (&least)[P])
{
#pragma unroll
    for (int p = 0; p < P; ++p) {
        m[p] = 0.0f;
        least[p] = 0xffffffffu;
    }
    auto low = [](uint32_t least, float y) {
        const uint32_t u = __float_as_uint(y);
        return min(least, ACT == 1 ? u - 1u : (u << 1) - 1u);
    };
#pragma unroll
    for (int rb = 0; rb < R; ++rb) {
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int v = 0; v < 4; v += 2) {
                const float y = h[p][rb][v], z = h[p][rb][v + 1];
                h[p][rb][v] = act_c<ACT>(y);
                h[p][rb][v + 1] = act_c<ACT>(z);
                if constexpr (ACT == 1) {     // (never below 0; negative values' bits are large)
                    m[p] = max3(m[p], y, z);
                    least[p] = low(low(least[p], y), z);
                } else {
                    m[p] = max3(m[p], fabsf(h[p][rb][v]), fabsf(h[p][rb][v + 1]));
                    least[p] = low(low(least[p], h[p][rb][v]), h[p][rb][v + 1]);
                }
            }
    }
    // (the form of the ReLU for all: the bits of the least magnitude, less one)
    if constexpr (ACT != 1)
#pragma unroll
        for (int p = 0; p < P; ++p) least[p] >>= 1;
}

// Activations of layer l and, per sample, the exponent en that they take as the next
// layer's operand: from the largest magnitude over the sample's R x 16 values.  False when
// the parts do not hold one.  ACT < 0: the layer's own activation.
template <int ACT, int P, int R>
__device__ __forceinline__ bool split_act(const FitArgs &a, int l, floatx4 (&h)[P][R], int (&en)[P])
{
    bool ok = true;
    float m[P];
    uint32_t least[P];
    if constexpr (ACT >= 0) {
        split_apply<ACT, P, R>(h, m, least);
    } else {
        switch (a.act[l]) {
        case 1: split_apply<1, P, R>(h, m, least); break;
        case 2: split_apply<2, P, R>(h, m, least); break;
        case 3: split_apply<3, P, R>(h, m, least); break;
        default: split_apply<0, P, R>(h, m, least); break;
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < P; ++p) {
        m[p] = xor_max4(m[p]);
        const int e = max(min(15 - __builtin_amdgcn_frexp_expf(m[p]), PART_EMAX), -PART_EMAX);
        en[p] = e;
        // m 2^e < 2^15 (false for an infinity), and nothing but zero below 2^-14
        ok &= m[p] < __builtin_ldexpf(1.0f, 15 - e) && least[p] >= (uint32_t)(127 - 14 - e) * 0x800000u - 1u;
    }
    return ok;
}

template <int RB0 = 0, int P, int NKB, int RO, int RI>
__device__ __forceinline__ void split_layer_h(const SplitView<RI> &wv, const Parts (&x)[NKB][P],
                                              const float (&c)[P], const char *bias, floatx4 (&out)[P][RO])
{
    constexpr int G = RO - RB0 < 4 ? RO - RB0 : 4;
    floatx4 cr[P][G];
    split_kblock<true, true, RB0, G>(wv, 0, x[0], out, cr);
#pragma unroll
    for (int kb = 1; kb < NKB; ++kb) split_kblock<false, false, RB0, G>(wv, kb, x[kb], out, cr);
    split_finish<RB0, G>(out, cr, c, bias);
    if constexpr (RB0 + G < RO) split_layer_h<RB0 + G>(wv, x, c, bias, out);
}

// A layer behind the first one, from activations h times 2^en: converted to parts K block
// by K block where the registers hold all accumulators of the cross products beside h,
// else all at once, for a few row blocks after the other.
template <int NW, int P, int R, int RO>
__device__ __forceinline__ void split_layer(const SplitView<R> &wv, const floatx4 (&h)[P][R],
                                            const int (&en)[P], const float (&c)[P], const char *bias,
                                            floatx4 (&out)[P][RO])
{
    constexpr int NKB = (R + 1) / 2;
    auto parts = [&](int kb, int p, Parts &x) {
        split8(h[p][2 * kb], 2 * kb + 1 < R ? h[p][2 * kb + 1 < R ? 2 * kb + 1 : 0] : zero4(),
               __builtin_ldexpf(1.0f, en[p]), x);
    };
    if constexpr (4 * P * (R + 2 * RO) + 8 * P <= split_regs<NW>()) {
        floatx4 cr[P][RO];
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            Parts x[P];
#pragma unroll
            for (int p = 0; p < P; ++p) parts(kb, p, x[p]);
            if (kb == 0) split_kblock<true, true, 0, RO>(wv, kb, x, out, cr);
            else split_kblock<false, false, 0, RO>(wv, kb, x, out, cr);
        }
        split_finish<0, RO>(out, cr, c, bias);
    } else {
        Parts x[NKB][P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) parts(kb, p, x[kb][p]);
            __builtin_amdgcn_sched_barrier(0);
        }
        split_layer_h(wv, x, c, bias, out);
    }
}

// Layer l of a slab group and those behind it, from its pre-activations h: activation and
// the next layer, or the losses.  False, and no losses, when the
// parts do not hold an activation of the group (the same in every lane).
template <int NW, int ACT, int P, int R, int RN, int... RR>
__device__ __forceinline__ bool split_chain(const FitArgs &a, const char *smem, int l, int s0, int n, int g,
                                            const int (&wexp)[MAXL], floatx4 (&h)[P][R],
                                            const int (&lab)[P], LossSum<false> &loss, bool ok)
{
    if constexpr (RN == 0) {
        if (!__all(ok)) return false;
        slab_loss<P, R>(a, l, s0, n, g, h, lab, loss);
        return true;
    } else {
        int e[P];
        float c[P];
        ok &= split_act<ACT, P, R>(a, l, h, e);
#pragma unroll
        for (int p = 0; p < P; ++p) c[p] = __builtin_ldexpf(1.0f, -(e[p] + wexp[l + 1]));
        floatx4 out[P][RN];
        const SplitView<R> wv(a, smem, l + 1, n, g);
        split_layer<NW>(wv, h, e, c, split_bias(a, smem, l + 1, g), out);
        return split_chain<NW, ACT, P, RN, RR..., 0>(a, smem, l + 1, s0, n, g, wexp, out, lab, loss, ok);
    }
}

// One slab group from its inputs on, as split_chain.
template <int NW, int P, int ACT, int R1, int R2, int R3, int R4>
__device__ __forceinline__ bool split_group(const FitArgs &a, const char *smem, const SplitView<0> &w0, int s0,
                                            int n, int g, const int (&wexp)[MAXL],
                                            LossSum<false> &loss)
{
    // re-read the staged weights for every slab (a hoisted fragment set spills)
    asm volatile("" ::: "memory");
    int lab[P];
    load_labels(a, s0, n, lab);
    bool ok = true;
    float cz[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int xe = a.Xe[s0 + 16 * p + n];
        ok &= xe < XE_BAD;
        cz[p] = __builtin_ldexpf(1.0f, -(xe + wexp[0]));
    }
    if (!__all(ok)) return false;
    floatx4 h1[P][R1];
    // (its fragments' addresses would be kept, and spilled, from slab to slab)
    SplitView<0> wv = w0;
    asm volatile("" : "+v"(wv.p));
    split_layer_x<split_rows<NW, P, R1>()>(a, wv, s0, n, g, cz, split_bias(a, smem, 0, g), h1);
    return split_chain<NW, ACT, P, R1, R2, R3, R4>(a, smem, 0, s0, n, g, wexp, h1, lab, loss, true);
}

// The launch's arguments where they lie in memory.  The redo reads them there, behind an
// opaque pointer: kept in registers for it, they would spill the slab loop's.
typedef const __attribute__((address_space(4))) FitArgs *ArgsInMemory;

// Slab groups of a wavefront that its products in parts left out: bit i the i-th, and
// every one from `rest` on.
struct Redo {
    uint64_t marks = 0;
    int rest = 0x7fffffff;
    __device__ __forceinline__ bool any() const { return marks != 0 || rest != 0x7fffffff; }
};

// The losses of the marked slab groups of samples [s0, s_end) with FP32 instructions and
// weights.
template <int NW, int P, int ACT, int R1, int R2, int R3, int R4>
__device__ __forceinline__ void redo_groups(ArgsInMemory k, char *smem, int r, int s0, int s_end,
                                            const Redo &redo, LossSum<false> &loss)
{
    asm volatile("" : "+s"(k));
    const FitArgs &a = *(const FitArgs *)k;
    const int n = threadIdx.x & 15, g = (threadIdx.x & 63) >> 4;
    const float *w = a.W + (size_t)r * a.ld;
    stage_weights<false>(a, a.lay32, w, r, smem);
    const WView<false, true> v0(a, a.lay32, w, smem, 0, n, g), v1(a, a.lay32, w, smem, 1, n, g);
    const WView<false, true> v2(a, a.lay32, w, smem, 2, n, g), v3(a, a.lay32, w, smem, 3, n, g);
    for (int i = 0; s0 < s_end; s0 += NW * 16 * P, ++i)
        if (i >= redo.rest || (i < 64 && redo.marks >> i & 1))
            slab_group<false, true, P, ACT, R1, R2, R3, R4, 5>(a, a.lay32, w, smem, v0, v1, v2, v3, s0,
                                                                     n, g, loss);
}

// Block `bid` of a fitness launch: spark r = bid / bpr, sample range c = bid % bpr.
template <int NW, int P, int ACT, int R1, int R2, int R3, int R4>
__device__ __forceinline__ void split_body(const FitArgs &a, ArgsInMemory k, int bid)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int r = bid / a.bpr, c = bid % a.bpr;
    const float *w = a.W + (size_t)r * a.ld;
    __shared__ int row_exp[MAXL];
    bool held = false;
    // first the box's exponent, which needs no pass over the row
    for (int own = 0; own < 2 && !held; ++own) {
        if (own) row_exps(a, w, r, row_exp);
        else if (threadIdx.x < MAXL) row_exp[threadIdx.x] = a.wexp;
        __syncthreads();
        held = stage_split(a, w, r, smem, row_exp);
    }
    int wexp[MAXL];
#pragma unroll
    for (int l = 0; l < MAXL; ++l) wexp[l] = __builtin_amdgcn_readfirstlane(row_exp[l]);
    const SplitView<0> w0(a, smem, 0, n, g);
    const int s_begin = c * a.spb + wave * 16 * P;
    const int s_end = min(c * a.spb + a.spb, a.S_pad);
    LossSum<false> loss;
    Redo redo;
    if (!held) redo.rest = 0;
    for (int s0 = s_begin, i = 0; s0 < s_end && i < redo.rest; s0 += NW * 16 * P, ++i)
        if (!split_group<NW, P, ACT, R1, R2, R3, R4>(a, smem, w0, s0, n, g, wexp, loss)) {
            if (i < 64) redo.marks |= 1ull << i;
            else redo.rest = i;
        }
    if (__syncthreads_or(redo.any()))
        redo_groups<NW, P, ACT, R1, R2, R3, R4>(k, smem, r, s_begin, s_end, redo, loss);
    block_loss<NW>(a, r, c, loss);
}

template <int NW, int P, int ACT, int R1, int R2, int R3, int R4>
__global__ __launch_bounds__(NW * 64) void k_fit_split(FitArgs a)
{
    // (its only argument starts the kernel's argument segment)
    split_body<NW, P, ACT, R1, R2, R3, R4>(a, (ArgsInMemory)__builtin_amdgcn_kernarg_segment_ptr(),
                                           xcd_remap(blockIdx.x, gridDim.x));
}

template <int NW, int P, int ACT, int R1, int R2, int R3, int R4>
__global__ __launch_bounds__(NW * 64) void k_fit_split_group(GroupTable t, int which)
{
    const int j = group_job(t, blockIdx.x);
    const int local = blockIdx.x - t.start[j], n = t.gx[j] * t.gy[j];
    if (local >= n) return;   // padding
    const FitArgs a = t.job[j]->fit[which].a;   // a private copy, as in k_fit_group
    split_body<NW, P, ACT, R1, R2, R3, R4>(a, (ArgsInMemory)&t.job[j]->fit[which].a, xcd_remap(local, n));
}

#define FIT_ENTRY_SPLIT(NW, P, ACT, R1, R2, R3, R4)                                          \
    {0, 1, NW, P, ACT, {R1, R2, R3, R4},                                                      \
     reinterpret_cast<const void *>(&::mgfwa::fit::k_fit_split<NW, P, ACT, R1, R2, R3, R4>), \
     reinterpret_cast<const void *>(&::mgfwa::fit::k_fit_split_group<NW, P, ACT, R1, R2, R3, R4>), 1}

}  // namespace fit
}  // namespace mgfwa

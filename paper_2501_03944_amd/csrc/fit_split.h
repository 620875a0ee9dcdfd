// FP32 fitness of register-chain networks on the FP16 matrix units, instantiated by the
// split_*.hip files (the frame is fit_kernel.h's: transposed layers, 16-sample slabs,
// weights staged in LDS, layers chained in registers).
//
// The FP32 matrix rate (157 TFLOP/s) bounds fit_kernel.h's FP32 kernels (0.82 of it at
// 64-128-128-10).  Here every operand of a layer is two FP16 parts of the value times a
// power of two, v 2^e = hi + lo (23 of the 24 bits), and a layer is three FP16 products
// per K block, W_lo H_hi + W_hi H_lo + W_hi H_hi, accumulated in FP32 (bound 833
// TFLOP/s).  Exponents: one for the spark's weights (the search box's, or the row's own
// for rows that need not lie in it), one per sample for the inputs (Xe), and one per
// sample and hidden layer from the largest activation of the sample, so that no part
// overflows and every value near the largest keeps its bits.  Bias, activation and loss
// are FP32 on the true scale.
//
// The conversion of the hidden activations to parts is vector work (about six
// instructions per value) beside the products; two slabs per wavefront share each
// weight fragment's LDS read, and two wavefronts per SIMD overlap one's conversions
// with the other's products.
//
// Measured, FP32 instructions -> so: a generation of 64-128-128-10 (2,048 sparks x 4,096
// samples) 3,478 -> 1,350 us; 300 rows x 4,096 samples of it 574 -> 258 us, their error
// against binary64 5.2e-8 -> 4.5e-8.
//
// Slab groups with a sample, a weight or an activation that is not finite, or whose
// exponents leave the FP32 range, are marked and taken again by FP32 instructions
// (fit_kernel.h's slab_group) once the block has been through its samples, with the
// row's FP32 weights staged in place of the parts; values that are not finite thus go
// the way that they go in the FP32 kernels.
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
    uint4v hi, lo;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float x = (i < 2 ? a[2 * (i & 1)] : b[2 * (i & 1)]) * c;
        const float y = (i < 2 ? a[2 * (i & 1) + 1] : b[2 * (i & 1) + 1]) * c;
        const halfx2 h = __builtin_convertvector((floatx2){x, y}, halfx2);
        // (as a multiply-add, which takes the FP16 half as it is)
        const floatx2 r = {__builtin_fmaf((float)h[0], -1.0f, x), __builtin_fmaf((float)h[1], -1.0f, y)};
        hi[i] = __builtin_bit_cast(uint32_t, h);
        lo[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, halfx2));
    }
    p.hi = __builtin_bit_cast(halfx8, hi);
    p.lo = __builtin_bit_cast(halfx8, lo);
}

// Exponents kept in the range where 2^e and 2^-e are normal FP32 values.
constexpr int SPLIT_EMAX = 120;

// Position of element k (of a 32-column block) in the order the lanes read: lane
// group g takes columns 4g..4g+3 and 16+4g..16+4g+3 as eight consecutive elements.
__device__ __forceinline__ int split_pos(int k)
{
    return (k & ~31) + ((k & 12) << 1) + ((k & 16) >> 2) + (k & 3);
}

// One lane's view of a layer's staged weights: the hi plane, the lo plane `plane`
// elements behind it, 16-byte chunk c of row r stored at chunk c ^ (r & 1).
struct SplitView {
    const _Float16 *p;
    int pitch, plane;
    __device__ __forceinline__ SplitView(const FitArgs &a, const char *smem, int l, int n, int g)
    {
        pitch = a.lay.lpitch[l];
        plane = a.lay.lrows[l] * pitch;
        p = reinterpret_cast<const _Float16 *>(smem) + a.lay.lw[l] + n * pitch + 8 * (g ^ (n & 1));
    }
    __device__ __forceinline__ void load(int rb, int kb, halfx8 &hi, halfx8 &lo) const
    {
        const _Float16 *q = p + 16 * rb * pitch + 32 * kb;
        hi = *reinterpret_cast<const halfx8 *>(q);
        lo = *reinterpret_cast<const halfx8 *>(q + plane);
    }
};

// The spark's weights as parts into LDS (zero-padded), biases into the FP32 area.
__device__ __forceinline__ void stage_split(const FitArgs &a, const float *w, int r, char *smem, int wexp)
{
    float *bias = reinterpret_cast<float *>(smem + a.lay.bias_byte);
    const bool regen = a.rg.F != nullptr;
    const int nt = blockDim.x;
    for (int l = 0; l < a.nl; ++l) {
        const int fo = a.fo[l], fi = a.fi[l], rows = a.lay.lrows[l], cols = a.lay.lcols[l];
        const int pitch = a.lay.lpitch[l], plane = rows * pitch;
        _Float16 *dst = reinterpret_cast<_Float16 *>(smem) + a.lay.lw[l];
        const float *src = w + a.woff[l];
        const int n4 = rows * cols / 4;
        const bool vec = a.vec[l] != 0;
        for (int i0 = threadIdx.x; i0 < n4; i0 += 4 * nt) {
            floatx4 v[4];
            int at[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int idx = i0 + u * nt;
                const int o = (4 * idx) / cols, k = 4 * idx - o * cols;
                at[u] = idx < n4 ? o * pitch + (split_pos(k) ^ ((o & 1) << 3)) : -1;
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
                    const SplitF16 s = split_f16(v[u][e], wexp);
                    hi[e] = s.hi;
                    lo[e] = s.lo;
                }
                *reinterpret_cast<halfx4 *>(dst + at[u]) = hi;
                *reinterpret_cast<halfx4 *>(dst + plane + at[u]) = lo;
            }
        }
        for (int o = threadIdx.x; o < rows; o += nt)
            bias[a.lay.lb[l] + o] = o < fo ? spark_at(a, w, r, a.boff[l] + o) : 0.0f;
    }
    __syncthreads();
}

// The exponent of a row that need not lie in the box; *bad when a value of it is not
// finite (the same in every thread).
__device__ __forceinline__ int row_exp(const FitArgs &a, const float *w, bool *bad)
{
    __shared__ float sm[16];
    const int n = a.boff[a.nl - 1] + a.fo[a.nl - 1];
    float m = 0.0f;
    bool inf = false;
    const int n4 = n / 4, nt = blockDim.x;
    for (int i0 = threadIdx.x; i0 < n4; i0 += 4 * nt) {
        floatx4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            v[u] = i0 + u * nt < n4 ? reinterpret_cast<const floatx4 *>(w)[i0 + u * nt] : zero4();
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                m = fmaxf(m, fabsf(v[u][e]));
                inf |= !(fabsf(v[u][e]) <= 3.4028234e38f);
            }
    }
    if ((int)threadIdx.x < n - 4 * n4) {
        const float v = fabsf(w[4 * n4 + threadIdx.x]);
        m = fmaxf(m, v);
        inf |= !(v <= 3.4028234e38f);
    }
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = m;
    *bad = __syncthreads_or(inf) != 0;
    m = sm[0];
    for (int i = 1; i < (int)(blockDim.x >> 6); ++i) m = fmaxf(m, sm[i]);
    return split_exp(m);
}

// One K block of a layer's products for every row block: fragments one row block
// ahead, the small products first.
template <int P, int RO>
__device__ __forceinline__ void split_kblock(const SplitView &wv, int kb, const Parts (&x)[P],
                                             floatx4 (&out)[P][RO])
{
    halfx8 hi, lo;
    wv.load(0, kb, hi, lo);
#pragma unroll
    for (int rb = 0; rb < RO; ++rb) {
        halfx8 hn = hi, ln = lo;
        if (rb + 1 < RO) wv.load(rb + 1, kb, hn, ln);
#pragma unroll
        for (int p = 0; p < P; ++p)
            out[p][rb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(lo, x[p].hi, out[p][rb], 0, 0, 0);
#pragma unroll
        for (int p = 0; p < P; ++p)
            out[p][rb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, x[p].lo, out[p][rb], 0, 0, 0);
#pragma unroll
        for (int p = 0; p < P; ++p)
            out[p][rb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, x[p].hi, out[p][rb], 0, 0, 0);
        hi = hn;
        lo = ln;
        // (keeps later fragments' reads and K blocks' conversions from moving up, whose
        // registers would spill)
        __builtin_amdgcn_sched_barrier(0);
    }
}

// First layer: the samples' inputs, scaled by their exponents xe.
template <int P, int RO>
__device__ __forceinline__ void split_layer_x(const FitArgs &a, const SplitView &wv, int s0, int n, int g,
                                              const float (&cx)[P], floatx4 (&out)[P][RO])
{
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int rb = 0; rb < RO; ++rb) out[p][rb] = zero4();
    const float *xp = a.X + (size_t)(s0 + n) * a.in_pad + 4 * g;
    const int nkb = (a.in_pad + 31) >> 5;
    for (int kb = 0; kb < nkb; ++kb) {
        Parts x[P];
        const bool both = 32 * kb + 16 < a.in_pad;      // the block's upper half exists
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const float *q = xp + (size_t)16 * p * a.in_pad + 32 * kb;
            const floatx4 u = *reinterpret_cast<const floatx4 *>(q);
            const floatx4 v = both ? *reinterpret_cast<const floatx4 *>(q + 16) : zero4();
            split8(u, v, cx[p], x[p]);
        }
        split_kblock<P, RO>(wv, kb, x, out);
    }
}

// The largest of three, one instruction (a NaN is passed over).
__device__ __forceinline__ float max3(float a, float b, float c)
{
    float d;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

// Pre-activations on the true scale (acc c + bias) and activation of layer l; m is the
// largest magnitude of a sample's values in this lane.
template <int ACT, int P, int R>
__device__ __forceinline__ void split_bias_act(const FitArgs &a, const char *smem, int l, int g,
                                               const float (&c)[P], floatx4 (&h)[P][R], float (&m)[P])
{
#pragma unroll
    for (int p = 0; p < P; ++p) m[p] = 0.0f;
#pragma unroll
    for (int rb = 0; rb < R; ++rb) {
        const floatx4 b = *reinterpret_cast<const floatx4 *>(smem + a.lay.bias_byte +
                                                             (size_t)(a.lay.lb[l] + 16 * rb + 4 * g) * 4);
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int v = 0; v < 4; v += 2) {
                const float y = __builtin_fmaf(h[p][rb][v], c[p], b[v]);
                const float z = __builtin_fmaf(h[p][rb][v + 1], c[p], b[v + 1]);
                h[p][rb][v] = act_c<ACT>(y);
                h[p][rb][v + 1] = act_c<ACT>(z);
                if constexpr (ACT == 1) m[p] = max3(m[p], y, z);   // (never below 0)
                else m[p] = max3(m[p], fabsf(h[p][rb][v]), fabsf(h[p][rb][v + 1]));
            }
    }
}

// Activations of layer l and the next layer's operand parts: per sample times 2^en, the
// exponent en from the largest magnitude over the sample's R x 16 values.  False when
// one is not finite or en is out of range.  ACT < 0: the layer's own activation.
template <int ACT, int P, int R>
__device__ __forceinline__ bool split_act(const FitArgs &a, const char *smem, int l, int g,
                                          const float (&c)[P], floatx4 (&h)[P][R], int (&en)[P],
                                          Parts (&x)[(R + 1) / 2][P])
{
    bool ok = true;
    float m[P];
    if constexpr (ACT >= 0) {
        split_bias_act<ACT, P, R>(a, smem, l, g, c, h, m);
    } else {
        switch (a.act[l]) {
        case 1: split_bias_act<1, P, R>(a, smem, l, g, c, h, m); break;
        case 2: split_bias_act<2, P, R>(a, smem, l, g, c, h, m); break;
        case 3: split_bias_act<3, P, R>(a, smem, l, g, c, h, m); break;
        default: split_bias_act<0, P, R>(a, smem, l, g, c, h, m); break;
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < P; ++p) {
        m[p] = xor_max4(m[p]);
        int e = 15 - __builtin_amdgcn_frexp_expf(m[p]);      // m < 2^(15 - e)
        if (!(m[p] <= 3.4028234e38f) || e < -SPLIT_EMAX) ok = false;
        e = e > SPLIT_EMAX ? SPLIT_EMAX : e;                  // (all but zero activations)
        en[p] = e;
        const float cn = __builtin_ldexpf(1.0f, e);
#pragma unroll
        for (int kb = 0; kb < (R + 1) / 2; ++kb)
            split8(h[p][2 * kb], 2 * kb + 1 < R ? h[p][2 * kb + 1 < R ? 2 * kb + 1 : 0] : zero4(), cn,
                   x[kb][p]);
        __builtin_amdgcn_sched_barrier(0);
    }
    return ok;
}

template <int P, int NKB, int RO>
__device__ __forceinline__ void split_layer_h(const SplitView &wv, const Parts (&x)[NKB][P],
                                              floatx4 (&out)[P][RO])
{
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int rb = 0; rb < RO; ++rb) out[p][rb] = zero4();
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) split_kblock<P, RO>(wv, kb, x[kb], out);
}

// Output logits on the true scale.
template <int P, int R>
__device__ __forceinline__ void split_out(const FitArgs &a, const char *smem, int l, int g,
                                          const float (&c)[P], floatx4 (&z)[P][R])
{
#pragma unroll
    for (int rb = 0; rb < R; ++rb) {
        const floatx4 b = *reinterpret_cast<const floatx4 *>(smem + a.lay.bias_byte +
                                                             (size_t)(a.lay.lb[l] + 16 * rb + 4 * g) * 4);
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int v = 0; v < 4; ++v) z[p][rb][v] = __builtin_fmaf(z[p][rb][v], c[p], b[v]);
    }
}

// Layer l of a slab group and those behind it, from its raw products h (their scale
// 2^-c): activation and the next layer, or the losses.  False, and no losses, when the
// parts do not hold an activation of the group (the same in every lane).
template <int ACT, int P, int R, int RN, int... RR>
__device__ __forceinline__ bool split_chain(const FitArgs &a, const char *smem, int l, int s0, int n, int g,
                                            int wexp, float (&c)[P], floatx4 (&h)[P][R],
                                            const int (&lab)[P], LossSum &loss, bool ok)
{
    if constexpr (RN == 0) {
        if (!__all(ok)) return false;
        split_out<P, R>(a, smem, l, g, c, h);
        slab_loss<P, R>(a, l, s0, n, g, h, lab, loss);
        return true;
    } else {
        Parts x[(R + 1) / 2][P];
        int e[P];
        ok &= split_act<ACT, P, R>(a, smem, l, g, c, h, e, x);
#pragma unroll
        for (int p = 0; p < P; ++p) c[p] = __builtin_ldexpf(1.0f, -(e[p] + wexp));
        floatx4 out[P][RN];
        const SplitView wv(a, smem, l + 1, n, g);
        split_layer_h(wv, x, out);
        return split_chain<ACT, P, RN, RR..., 0>(a, smem, l + 1, s0, n, g, wexp, c, out, lab, loss, ok);
    }
}

// One slab group from its inputs on, as split_chain.
template <int P, int ACT, int R1, int R2, int R3, int R4>
__device__ __forceinline__ bool split_group(const FitArgs &a, const char *smem, const SplitView &w0, int s0,
                                            int n, int g, int wexp, LossSum &loss)
{
    // re-read the staged weights for every slab (a hoisted fragment set spills)
    asm volatile("" ::: "memory");
    int lab[P];
    load_labels(a, s0, n, lab);
    bool ok = true;
    float cx[P], cz[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int xe = a.Xe[s0 + 16 * p + n];
        ok &= xe < XE_BAD / 2 && xe + wexp >= -SPLIT_EMAX;
        cx[p] = __builtin_ldexpf(1.0f, xe);
        cz[p] = __builtin_ldexpf(1.0f, -(xe + wexp));
    }
    if (!__all(ok)) return false;
    floatx4 h1[P][R1];
    split_layer_x<P, R1>(a, w0, s0, n, g, cx, h1);
    return split_chain<ACT, P, R1, R2, R3, R4>(a, smem, 0, s0, n, g, wexp, cz, h1, lab, loss, true);
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
                                            const Redo &redo, LossSum &loss)
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
            slab_group<false, true, P, ACT, R1, R2, R3, R4, 1, true>(a, a.lay32, w, smem, v0, v1, v2, v3, s0,
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
    bool row_bad = false;
    const int wexp = a.boxed ? a.wexp : row_exp(a, w, &row_bad);
    stage_split(a, w, r, smem, wexp);
    const SplitView w0(a, smem, 0, n, g);
    const int s_begin = c * a.spb + wave * 16 * P;
    const int s_end = min(c * a.spb + a.spb, a.S_pad);
    LossSum loss;
    Redo redo;
    if (row_bad) redo.rest = 0;
    for (int s0 = s_begin, i = 0; s0 < s_end && i < redo.rest; s0 += NW * 16 * P, ++i)
        if (!split_group<P, ACT, R1, R2, R3, R4>(a, smem, w0, s0, n, g, wexp, loss)) {
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

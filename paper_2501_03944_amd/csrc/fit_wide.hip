// Wide-first-layer fitness: packing of sparks and samples, kernel instances,
// plan selection and launches (kernel template in fit_wide.h).
#include "fit_wide.h"

#include <cstdlib>

namespace mgfwa {

using namespace fit;

namespace {

constexpr int TPB = 256;
constexpr int MAX_GRID_Y = 65535;

// Part of a packed spark row per thread.  Chunk ranges:
//   W1aug  [Kp/32][256][32]  8 columns each, K-blocked: value(o, k) = W1[o][k]
//                        (k < in), b1[o] (k == in), 0 otherwise, at
//                        ((k/32)*256 + o)*32 + k%32 of its plane (FP16 parts: both planes)
//   W2     [16][256]     16 bytes each; BF16: chunk (i, kb, g) holds
//                        W2[i][32kb + p(g, e)], e = 0..7, p(g, e) = 4g + e (e < 4) or
//                        16 + 4g + e - 4 (e >= 4); FP32: natural order
//   b2     [16]          FP32, four each
constexpr int PACK_CPT = 4;   // chunks per thread (strided by the block)
constexpr int PACK_RPB = 4;   // spark rows per block

__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)a) |
           ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)b) << 16);
}

template <int KIND>
__device__ __forceinline__ void pack_chunk(const float *__restrict__ w, char *__restrict__ wp,
                                           int chunk, int c1, int c2, const WidePack &p, float c, bool raw)
{
    constexpr bool BF = KIND == WIDE_BF16;
    if (chunk < c1) {
        const int e0 = chunk * 8, kb = e0 / (WT_M * WT_K), rem = e0 % (WT_M * WT_K);
        const int o = rem / WT_K, k0 = kb * WT_K + rem % WT_K;
        const float *src = w + p.woff1 + (size_t)o * p.in + k0;
        float v[8];
        if (o < p.hid && k0 + 8 <= p.in && (reinterpret_cast<uintptr_t>(src) & 15) == 0) {
            // inside W1 and 16-byte aligned: vector loads
#pragma unroll
            for (int e = 0; e < 8; e += 4) {
                const float4 t = *reinterpret_cast<const float4 *>(src + e);
                v[e] = t.x;
                v[e + 1] = t.y;
                v[e + 2] = t.z;
                v[e + 3] = t.w;
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = k0 + e;
                float x = 0.0f;
                if (o < p.hid) {
                    if (k < p.in) x = w[p.woff1 + (size_t)o * p.in + k];
                    else if (k == p.in) x = w[p.boff1 + o];
                }
                v[e] = x;
            }
        }
        if constexpr (BF) {
            reinterpret_cast<uint4 *>(wp)[chunk] =
                make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]),
                           pack_bf16(v[6], v[7]));
        } else if constexpr (KIND == WIDE_F16X2) {
            uint32_t h[4], l[4];
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                const Words a = wide_words(v[e], c, raw), b = wide_words(v[e + 1], c, raw);
                h[e / 2] = a.hi | (uint32_t)b.hi << 16;
                l[e / 2] = a.lo | (uint32_t)b.lo << 16;
            }
            reinterpret_cast<uint4 *>(wp)[chunk] = make_uint4(l[0], l[1], l[2], l[3]);
            reinterpret_cast<uint4 *>(wp)[c1 + chunk] = make_uint4(h[0], h[1], h[2], h[3]);
        } else {
            reinterpret_cast<float4 *>(wp)[2 * chunk] = make_float4(v[0], v[1], v[2], v[3]);
            reinterpret_cast<float4 *>(wp)[2 * chunk + 1] = make_float4(v[4], v[5], v[6], v[7]);
        }
    } else if (chunk < c1 + c2) {
        constexpr int EPC = BF ? 8 : 4;
        const int e0 = (chunk - c1) * EPC, i = e0 / WT_M, c0 = e0 % WT_M;
        float v[EPC];
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
            int col = c0 + e;
            if (BF) {
                const int blk = c0 & ~31, g = (c0 & 31) >> 3;   // c0 = 32kb + 8g
                col = blk + (e < 4 ? 4 * g + e : 16 + 4 * g + e - 4);
            }
            v[e] = (i < p.out && col < p.hid) ? w[p.woff2 + (size_t)i * p.hid + col] : 0.0f;
        }
        char *dst = wp + (size_t)c1 * (BF ? 16 : 32) + (size_t)(chunk - c1) * 16;
        if constexpr (BF)
            *reinterpret_cast<uint4 *>(dst) = make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]),
                                                         pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]));
        else
            *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
        const int i0 = (chunk - c1 - c2) * 4;
        float *dst = reinterpret_cast<float *>(wp + (size_t)c1 * (BF ? 16 : 32) + (size_t)c2 * 16);
        float4 b;
        b.x = i0 + 0 < p.out ? w[p.boff2 + i0 + 0] : 0.0f;
        b.y = i0 + 1 < p.out ? w[p.boff2 + i0 + 1] : 0.0f;
        b.z = i0 + 2 < p.out ? w[p.boff2 + i0 + 2] : 0.0f;
        b.w = i0 + 3 < p.out ? w[p.boff2 + i0 + 3] : 0.0f;
        reinterpret_cast<float4 *>(dst)[i0 / 4] = b;
    }
}

// A block packs PACK_RPB rows x (PACK_CPT * TPB) chunks: fat blocks, so the
// dispatcher is not what bounds the pass.  Two planes: in the form k_wide_row_exp stored.
template <int KIND>
__global__ __launch_bounds__(TPB) void k_pack_wide_rows(const float *__restrict__ W, size_t ld,
                                                        int rows, WidePack p)
{
    const int c1 = WT_M * p.Kp / 8;                  // chunks of W1aug
    const int c2 = 16 * WT_M / (KIND == WIDE_BF16 ? 8 : 4);         // chunks of W2
    const int nchunk = c1 + c2 + 4;
    const int cfirst = blockIdx.x * TPB * PACK_CPT + threadIdx.x;
    for (int r0 = blockIdx.y * PACK_RPB; r0 < rows; r0 += gridDim.y * PACK_RPB) {
        const int rend = r0 + PACK_RPB < rows ? r0 + PACK_RPB : rows;
        for (int r = r0; r < rend; ++r) {
            const float *w = W + (size_t)r * ld;
            char *wp = p.Wp + (size_t)r * p.pr;
            float c = 1.0f;
            bool raw = false;
            if constexpr (KIND == WIDE_F16X2) {
                const int32_t *t = wide_row_exp(wp, p.Kp);
                c = __builtin_ldexpf(1.0f, t[0]);
                raw = t[1] != 0;
            }
#pragma unroll
            for (int i = 0; i < PACK_CPT; ++i) {
                const int chunk = cfirst + i * TPB;
                if (chunk < nchunk) pack_chunk<KIND>(w, wp, chunk, c1, c2, p, c, raw);
            }
        }
    }
}

// The form (row_form) of rows that the explosion did not pack: one block per row, over W1
// and b1 (adjacent, at the start of the spark, which is 16-byte aligned), whose values the
// parts hold or not, and W2, which must not be too large for their scale.  A few rows leave
// most of the chip idle, so a block keeps as many loads in flight as it can: 1024 threads
// x 4 x 16 bytes.
constexpr int ROW_EXP_TPB = 1024;
__global__ __launch_bounds__(ROW_EXP_TPB) void k_wide_row_exp(const float *__restrict__ W, size_t ld,
                                                              WidePack p)
{
    __shared__ uint32_t most, least, w2most;
    if (threadIdx.x == 0) {
        most = w2most = 0;
        least = 0xffffffffu;
    }
    __syncthreads();
    const float *w = W + (size_t)blockIdx.x * ld + p.woff1;
    const int n = p.hid * (p.in + 1), n4 = n / 4;
    uint32_t m = 0, l = 0xffffffffu, m2 = 0;   // (magnitudes are ordered as their bits are)
    auto take = [&](float v) {
        m = max(m, __float_as_uint(fabsf(v)));
        l = least_bits(l, v);
    };
    for (int i0 = threadIdx.x; i0 < n4; i0 += 4 * ROW_EXP_TPB) {
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * ROW_EXP_TPB;
            v[u] = i < n4 ? reinterpret_cast<const float4 *>(w)[i] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            take(v[u].x);
            take(v[u].y);
            take(v[u].z);
            take(v[u].w);
        }
    }
    if ((int)threadIdx.x < n - 4 * n4) take(w[4 * n4 + threadIdx.x]);
    for (int i = threadIdx.x; i < p.out * p.hid; i += ROW_EXP_TPB)
        m2 = max(m2, __float_as_uint(fabsf(w[p.woff2 - p.woff1 + i])));
    for (int off = 32; off > 0; off >>= 1) {
        m = max(m, (uint32_t)__shfl_xor((int)m, off));
        l = min(l, (uint32_t)__shfl_xor((int)l, off));
        m2 = max(m2, (uint32_t)__shfl_xor((int)m2, off));
    }
    if ((threadIdx.x & 63) == 0) {
        atomicMax(&most, m);
        atomicMin(&least, l);
        atomicMax(&w2most, m2);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        RowForm form = row_form(most, least);
        if (w2most >= __float_as_uint(WIDE_W2_MAX)) form = RowForm{0, 1};
        int32_t *t = wide_row_exp(p.Wp + (size_t)blockIdx.x * p.pr, p.Kp);
        t[0] = form.e;
        t[1] = form.raw;
    }
}

// FP32 or BF16 samples for the wide kernel, column `in` = 1 (the folded bias),
// K-blocked per 256-sample tile: element (s, k) at
// ((s/256 * Kp/32 + k/32) * 256 + s%256) * 32 + k%32, so one K step of one sample
// tile is a contiguous 256 x 32 block.
template <bool BF>
__global__ __launch_bounds__(TPB) void k_pack_wide_x(const float *__restrict__ x, int S, int S_pad,
                                                     int in, int Kp, char *__restrict__ Xw)
{
    const size_t tid = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (tid >= (size_t)S_pad * Kp) return;
    const int s = (int)(tid / Kp), k = (int)(tid % Kp);
    float v = 0.0f;
    if (s < S) v = k < in ? x[(size_t)s * in + k] : (k == in ? 1.0f : 0.0f);
    const int nk = Kp / WT_K;
    const size_t dst = (((size_t)(s / WT_N) * nk + k / WT_K) * WT_N + s % WT_N) * WT_K + k % WT_K;
    if constexpr (BF) reinterpret_cast<uint16_t *>(Xw)[dst] = __builtin_bit_cast(uint16_t, (__bf16)v);
    else reinterpret_cast<float *>(Xw)[dst] = v;
}

__global__ void k_clear_marks(int32_t *p, int n)
{
    if ((int)threadIdx.x < n) p[threadIdx.x] = 0;
}

// Exponent of every sample's inputs and of the constant 1 (Xe), a wavefront per sample; a
// tile of 256 with a sample that the parts do not hold is marked (behind the exponents) and
// packed raw.
__global__ __launch_bounds__(TPB) void k_wide_sample_exp(const float *__restrict__ x, int S, int S_pad, int in,
                                                         int32_t *__restrict__ Xe)
{
    const int s = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (s >= S_pad) return;
    uint32_t m = __float_as_uint(1.0f), l = least_bits(0xffffffffu, 1.0f);
    for (int k = lane; s < S && k < in; k += 64) {
        const float v = x[(size_t)s * in + k];
        m = max(m, __float_as_uint(fabsf(v)));
        l = least_bits(l, v);
    }
    for (int off = 32; off > 0; off >>= 1) {
        m = max(m, (uint32_t)__shfl_xor((int)m, off));
        l = min(l, (uint32_t)__shfl_xor((int)l, off));
    }
    if (lane != 0) return;
    const RowForm form = row_form(m, l);
    Xe[s] = form.e;
    if (form.raw) atomicOr(&Xe[S_pad + s / WT_N], 1);
}

// Samples in two planes: a tile's hi plane, then its lo plane, each K-blocked as above.
__global__ __launch_bounds__(TPB) void k_pack_wide_x_planes(const float *__restrict__ x, int S, int S_pad,
                                                            int in, int Kp, char *__restrict__ Xw,
                                                            const int32_t *__restrict__ Xe)
{
    const size_t tid = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (tid >= (size_t)S_pad * Kp) return;
    const int s = (int)(tid / Kp), k = (int)(tid % Kp);
    float v = 0.0f;
    if (s < S) v = k < in ? x[(size_t)s * in + k] : (k == in ? 1.0f : 0.0f);
    const Words p = wide_words(v, __builtin_ldexpf(1.0f, Xe[s]), Xe[S_pad + s / WT_N] != 0);
    const size_t plane = (size_t)WT_N * Kp;
    uint16_t *hi = reinterpret_cast<uint16_t *>(Xw) + (size_t)(s / WT_N) * 2 * plane;
    const size_t at = ((size_t)(k / WT_K) * WT_N + s % WT_N) * WT_K + k % WT_K;
    hi[at] = p.hi;
    hi[plane + at] = p.lo;
}

// One instance per (precision, hidden activation): a run-time activation
// switch over the 256 accumulators would push them out of registers.
typedef void (*WideFn)(WideArgs);
struct WideKernels {
    WideFn fit;
    WideFn raw;    // two planes: the tiles that fit leaves out
};
#define WIDE_KIND(FIT, RAW)                                                                         \
    {{&FIT 0>, RAW 0>}, {&FIT 1>, RAW 1>}, {&FIT 2>, RAW 2>}, {&FIT 3>, RAW 3>}}
#define COMMA ,
template <int ACT>
constexpr WideFn NO_RAW = nullptr;
const WideKernels kWide[3][4] = {
    WIDE_KIND(k_fit_wide32<false COMMA, NO_RAW<),
    WIDE_KIND(k_fit_wide<WIDE_BF16 COMMA, NO_RAW<),
    WIDE_KIND(k_fit_wide<WIDE_F16X2 COMMA, &k_fit_wide32<true COMMA)};
#undef COMMA
#undef WIDE_KIND

const WideKernels &wide_kernels(const Net &net)
{
    const int act = net.act[0] >= 0 && net.act[0] <= 3 ? net.act[0] : 0;
    return kWide[wide_kind(net)][act];
}

// Sparks per XCD tile group.  Enough tiles for the XCD's blocks; when the
// group's rounds can be gs x (bx/gs) rectangles, the gs minimising the distinct
// weight + sample tiles per round (gs + bx/gs); gs always divides rows.
int wide_group(const Net &net, int rows, int ntn)
{
    const int bx = (net.num_cu + 7) / 8;
    int gs = 1;
    while (gs * ntn < bx && rows % (2 * gs) == 0 && gs < 64) gs *= 2;
    if (gs * ntn < bx) return gs;
    int best = gs, best_cost = gs + bx;
    for (int g = gs; g <= 16; g *= 2) {
        if (rows % g || bx % g || ntn % (bx / g)) continue;
        const int cost = g + bx / g;
        if (cost < best_cost) {
            best = g;
            best_cost = cost;
        }
    }
    // a small launch (e.g. one row per firework) gives every XCD a group while
    // the groups still hold a tile per block
    while (best > 1 && rows / best < 8 && (best / 2) * ntn >= bx) best /= 2;
    return best;
}

}  // namespace

bool wide_applicable(const Net &net)
{
    return net.nl == 2 && net.fo[0] <= WT_M && net.fo[1] <= 16;
}

// K (inputs plus the ones column) padded to K steps; the 16-bit pipeline looks STAGES
// steps ahead within a tile and the next, so a tile has at least as many
int wide_kp(const Net &net)
{
    const int kp = (net.fi[0] + 1 + WT_K - 1) / WT_K * WT_K;
    const int kmin = net.bf16 ? PipeCfg::STAGES * WT_K : 0;
    return kp > kmin ? kp : kmin;
}

// FP32 takes two FP16 parts from 128 columns on, where their products are at least as
// accurate as FP32 instructions (fit_wide.h has the figures), in boxes whose weights they
// take
WideKind wide_kind(const Net &net)
{
    return net.bf16 ? WIDE_BF16 : wide_kp(net) >= 128 && net.box_exp >= WIDE_EMIN ? WIDE_F16X2 : WIDE_F32;
}

size_t wide_row_bytes(const Net &net)
{
    const size_t es = net.bf16 ? 2 : 4;
    const size_t b = (size_t)WT_M * wide_kp(net) * es + 16 * WT_M * es + 64 + 8;
    return (b + 255) / 256 * 256;
}

int wide_lds_bytes(const Net &net) { return wide_kind(net) == WIDE_BF16 ? PipeCfg::LDS : Cfg32::LDS; }

hipError_t wide_prepare(const Net &net)
{
    static_assert(PipeCfg::LDS <= Cfg32::LDS, "wide_lds_bytes holds for both kernels of two planes");
    for (const WideFn fn : {wide_kernels(net).fit, wide_kernels(net).raw}) {
        if (!fn) continue;
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 wide_lds_bytes(net));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_pack_wide_x(const Net &net, const float *x, const DevState &d, hipStream_t st)
{
    const int Kp = wide_kp(net);
    const size_t n = (size_t)net.S_pad * Kp;
    const dim3 grid((unsigned)((n + TPB - 1) / TPB));
    if (wide_kind(net) == WIDE_F16X2) {
        hipLaunchKernelGGL(k_clear_marks, dim3(1), dim3(TPB), 0, st, d.Xe + net.S_pad, net.S_pad / WT_N);
        hipLaunchKernelGGL(k_wide_sample_exp, dim3((unsigned)((net.S_pad + 3) / 4)), dim3(TPB), 0, st, x,
                           net.S, net.S_pad, net.fi[0], d.Xe);
        hipLaunchKernelGGL(k_pack_wide_x_planes, grid, dim3(TPB), 0, st, x, net.S, net.S_pad, net.fi[0], Kp,
                           d.Xw, d.Xe);
    } else {
        hipLaunchKernelGGL(net.bf16 ? &k_pack_wide_x<true> : &k_pack_wide_x<false>, grid, dim3(TPB), 0, st, x,
                           net.S, net.S_pad, net.fi[0], Kp, d.Xw);
    }
    return hipGetLastError();
}

WidePack wide_pack_geometry(const Net &net, const DevState &d)
{
    static_assert(WT_M == 256 && WT_K == 32, "wide_pack_offset assumes 256 x 32 K blocks");
    WidePack p;
    p.Wp = d.Wpack;
    p.pr = wide_row_bytes(net);
    p.in = net.fi[0];
    p.hid = net.fo[0];
    p.out = net.fo[1];
    p.Kp = wide_kp(net);
    p.kind = wide_kind(net);
    p.wexp = net.box_exp;
    p.woff1 = net.woff[0];
    p.boff1 = net.boff[0];
    p.woff2 = net.woff[1];
    p.boff2 = net.boff[1];
    return p;
}

hipError_t launch_fitness_wide(const Net &net, const DevState &d, const float *W, size_t ld,
                               int rows, OutMap map, float *out, hipStream_t st,
                               hipEvent_t mid, hipEvent_t pre, int prepacked)
{
    if (rows <= 0) return hipSuccess;
    const int Kp = wide_kp(net);
    const size_t pr = wide_row_bytes(net);
    hipError_t e = hipSuccess;
    const int npack = rows - prepacked;
    if (npack > 0) {
        const int nchunk = WT_M * Kp / 8 + 16 * WT_M / (net.bf16 ? 8 : 4) + 4;
        const int rgroups = (npack + PACK_RPB - 1) / PACK_RPB;
        dim3 pg((nchunk + TPB * PACK_CPT - 1) / (TPB * PACK_CPT),
                rgroups < MAX_GRID_Y ? rgroups : MAX_GRID_Y);
        const float *Wsrc = W + (size_t)prepacked * ld;
        WidePack p = wide_pack_geometry(net, d);
        p.Wp += (size_t)prepacked * pr;
        if (p.kind == WIDE_F16X2)
            hipLaunchKernelGGL(k_wide_row_exp, dim3(npack), dim3(ROW_EXP_TPB), 0, st, Wsrc, ld, p);
        auto *k = p.kind == WIDE_BF16    ? &k_pack_wide_rows<WIDE_BF16>
                  : p.kind == WIDE_F16X2 ? &k_pack_wide_rows<WIDE_F16X2>
                                         : &k_pack_wide_rows<WIDE_F32>;
        hipLaunchKernelGGL(k, pg, dim3(TPB), 0, st, Wsrc, ld, npack, p);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (pre) {                          // packing done: the GEMM kernel starts here
        e = hipEventRecord(pre, st);
        if (e != hipSuccess) return e;
    }
    WideArgs a;
    a.Wp = d.Wpack;
    a.pr = pr;
    a.rows = rows;
    a.Xw = d.Xw;
    a.Kp = Kp;
    a.nk = Kp / WT_K;
    const bool f16x2 = wide_kind(net) == WIDE_F16X2;
    a.nv = f16x2 ? 3 * a.nk : a.nk;
    a.hid = net.fo[0];
    a.Xe = d.Xe;
    a.S = net.S;
    a.S_pad = net.S_pad;
    a.ntn = net.S_pad / WT_N;
    a.fo1 = net.fo[1];
    a.loss = net.loss;
    a.act = net.act[0];
    a.Y = d.Ypad;
    a.lab = d.Lpad;
    a.partial = d.partial;
    a.gs = wide_group(net, rows, a.ntn);
    const WideKernels &k = wide_kernels(net);
    hipLaunchKernelGGL(k.fit, dim3((unsigned)net.num_cu), dim3(TPB), (size_t)wide_lds_bytes(net), st, a);
    if (k.raw)
        hipLaunchKernelGGL(k.raw, dim3((unsigned)net.num_cu), dim3(TPB), (size_t)wide_lds_bytes(net), st, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (mid) {
        e = hipEventRecord(mid, st);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(f16x2 ? &k_wide_finalize<double> : &k_wide_finalize<float>,
                       dim3((unsigned)((rows + 63) / 64)), dim3(64), 0, st, a, net.inv_norm, map, out);
    return hipGetLastError();
}

}  // namespace mgfwa

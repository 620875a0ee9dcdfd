// Fitness host side: kernel table, plan selection and launches, plus the
// partial-sum finalisation and the packing of the problem data.  The kernel
// template lives in fit_kernel.h; the fit_*.hip files instantiate it.
#include "fit_kernel.h"

#include <algorithm>
#include <cstdlib>

namespace mgfwa {

namespace fit {
// one table per instantiation file
const KernelEntry *table_std(int *n);
const KernelEntry *table_l1(int *n);
const KernelEntry *table_l2(int *n);
const KernelEntry *table_l2_wide(int *n);
const KernelEntry *table_l3(int *n);
const KernelEntry *table_l3_wide_f32(int *n);
const KernelEntry *table_l3_wide_bf16(int *n);
const KernelEntry *table_l4_f32(int *n);
const KernelEntry *table_l4_bf16(int *n);
const KernelEntry *table_l4_wide_f32(int *n);
const KernelEntry *table_l4_wide_bf16(int *n);
const KernelEntry *table_lds_bf16(int *n);
const KernelEntry *table_lds_f32(int *n);
const KernelEntry *table_lds_any(int *n);
const KernelEntry *table_split(int *n);
const KernelEntry *table_split_any(int *n);
}  // namespace fit

namespace {

using namespace fit;

constexpr int MAX_BPR = 64;

// Sum of a row's partials in order (binary64: they may be few and large), scaled to
// the mean, NaN -> +inf, scattered.
__device__ __forceinline__ void finalize_body(const float *__restrict__ partial, int rows, int bpr,
                                              float inv_norm, const OutMap &map,
                                              float *__restrict__ out, Blk b)
{
    const int r = b.x * 256 + threadIdx.x;
    if (r >= rows) return;
    double t = 0.0;
    for (int c = 0; c < bpr; ++c) t += partial[(size_t)r * bpr + c];
    out[map.index(r)] = canon_fitness((float)(t * (double)inv_norm));
}

__global__ __launch_bounds__(256) void k_fit_finalize(const float *__restrict__ partial, int rows,
                                                      int bpr, float inv_norm, OutMap map,
                                                      float *__restrict__ out)
{
    finalize_body(partial, rows, bpr, inv_norm, map, out, own_block());
}

__global__ __launch_bounds__(256) void k_fit_finalize_group(GroupTable t, int which)
{
    const int j = group_job(t, blockIdx.x);
    Blk gb;
    if (!group_block(t, j, blockIdx.x, &gb)) return;   // padding
    const FitLaunch f = t.job[j]->fit[which];
    finalize_body(f.a.partial, f.a.rows, f.a.bpr, f.a.inv_norm, f.a.map, f.a.out, gb);
}

// Pack the problem data: X zero-padded to [S_pad][in_pad] (FP32 or bf16 RNE;
// skipped when both X destinations are null), MSE targets to [S_pad][out],
// labels to [S_pad] (-1 on padding).
__global__ __launch_bounds__(256) void k_pack(const float *__restrict__ x, const float *__restrict__ y,
                                              const int32_t *__restrict__ lab, int S, int S_pad,
                                              int in, int in_pad, int out, int bf16,
                                              float *__restrict__ Xp, uint16_t *__restrict__ Xb,
                                              float *__restrict__ Yp, int32_t *__restrict__ Lp)
{
    const size_t tid = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t nx = (size_t)S_pad * in_pad;
    if (tid < nx && (Xb || Xp)) {   // (the wide kernel packs its samples itself)
        const int s = (int)(tid / in_pad), k = (int)(tid % in_pad);
        const float v = (s < S && k < in) ? x[(size_t)s * in + k] : 0.0f;
        if (bf16) Xb[tid] = __builtin_bit_cast(uint16_t, (__bf16)v);
        else Xp[tid] = v;
    }
    if (tid < (size_t)S_pad * out && Yp) {
        const int s = (int)(tid / out);
        Yp[tid] = (s < S && y) ? y[tid] : 0.0f;
    }
    if (tid < (size_t)S_pad && Lp) Lp[tid] = (tid < (size_t)S && lab) ? lab[tid] : -1;
}

// Exponent of every sample's inputs for the register chain, or XE_BAD where the parts do
// not hold one of them: one wavefront per sample, the largest magnitude, then every value.
__global__ __launch_bounds__(256) void k_split_exp(const float *__restrict__ x, int S, int S_pad, int in,
                                                   int32_t *__restrict__ Xe)
{
    const int s = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (s >= S_pad) return;
    const float *row = x + (size_t)s * in;
    const int n = s < S ? in : 0;
    float m = 0.0f;
    for (int k = lane; k < n; k += 64) m = fmaxf(m, fabsf(row[k]));
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    const int e = part_exp(m);
    bool held = true;
    for (int k = lane; k < n; k += 64) held &= chain_parts(__builtin_ldexpf(row[k], e)).held;
    held = __all(held);
    if (lane == 0) Xe[s] = held ? e : XE_BAD;
}

// Samples in two FP16 parts (exponents Xe): the hi plane, then the lo plane, every row's
// 32-column blocks in the order that the lanes read them.  A sample whose inputs the
// parts do not hold was marked in Xe: its parts are not read.
__global__ __launch_bounds__(256) void k_pack_split(const float *__restrict__ x, int S, int S_pad, int in,
                                                    int pitch, const int32_t *__restrict__ Xe,
                                                    _Float16 *__restrict__ Xs)
{
    const size_t tid = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (tid >= (size_t)S_pad * pitch) return;
    const int s = (int)(tid / pitch), k = (int)(tid % pitch);
    const float v = s < S && k < in ? x[(size_t)s * in + k] : 0.0f;
    const size_t at = (size_t)s * pitch + split_pos(k);
    const ChainParts p = chain_parts(__builtin_ldexpf(v, Xe[s]));
    Xs[at] = p.hi;
    Xs[(size_t)S_pad * pitch + at] = p.lo;
}

const KernelEntry *(*const kTables[])(int *) = {
    table_std,         table_l1,          table_l2,       table_l2_wide,     table_l3,
    table_l3_wide_f32, table_l3_wide_bf16, table_l4_f32,  table_l4_bf16,     table_l4_wide_f32,
    table_l4_wide_bf16, table_lds_bf16, table_lds_f32, table_lds_any, table_split, table_split_any,
};

}  // namespace

int fit_max_bpr() { return MAX_BPR; }

// LDS layout of the staged weights for kernel entry e (split: of its FP16 parts, or of
// FP32 weights); returns the byte size.
static int lds_layout(const Net &net, const KernelEntry &e, LdsLayout *p, bool split)
{
    const int es = e.bf16 || split ? 2 : 4;   // bytes per stored element (split: per part)
    // pitch padding in elements: BF16 16 bytes; FP32 32 bytes (a pitch of 2 mod 8
    // 16-byte chunks, with the row-parity chunk swizzle of the kernel); split: likewise
    int off = 0, boff = 0;
    for (int l = 0; l < MAXL; ++l) {
        p->lw[l] = p->lpitch[l] = p->lrows[l] = p->lcols[l] = p->lb[l] = 0;
        if (l >= net.nl) continue;
        const int rows = 16 * e.R[l];
        int cols;
        if (l == 0) cols = split ? (net.in_pad + 31) / 32 * 32 : net.in_pad;
        else cols = e.bf16 || split ? 32 * ((e.R[l - 1] + 1) / 2) : 16 * e.R[l - 1];
        const int pitch = split ? split_pitch(cols) : cols + 8;
        off = (off + (16 / es) - 1) / (16 / es) * (16 / es);   // 16-byte aligned layer base
        p->lw[l] = off;
        p->lpitch[l] = pitch;
        p->lrows[l] = rows;
        p->lcols[l] = cols;
        p->lb[l] = boff;
        off += rows * pitch;
        boff += rows;
    }
    p->bias_byte = (off * es + 15) / 16 * 16;
    p->bytes = p->bias_byte + boff * 4;
    return p->bytes;
}

// Both layouts of kernel entry e; returns the bytes that its blocks take.
static int lds_layouts(const Net &net, const KernelEntry &e, LdsLayout *lay, LdsLayout *lay32)
{
    const int bytes = lds_layout(net, e, lay, e.split != 0);
    if (!e.split) {
        *lay32 = LdsLayout{};
        return bytes;
    }
    return std::max(bytes, lds_layout(net, e, lay32, false));
}

static int lds_bytes(const Net &net, const KernelEntry &e)
{
    LdsLayout lay, lay32;
    return lds_layouts(net, e, &lay, &lay32);
}

int resident_lds_bytes(const Net &net)
{
    KernelEntry e{};
    e.bf16 = net.bf16;
    for (int l = 0; l < MAXL; ++l) {
        e.R[l] = l < net.nl ? (net.fo[l] + 15) / 16 : 0;
        if (net.bf16 && l < net.nl - 1 && (e.R[l] & 1)) e.R[l] += 1;
    }
    return lds_bytes(net, e);
}

// Whether the network may take the register chain in two FP16 parts.  Those (7e-8 of a
// value, fewer roundings of the sum) are the more accurate form of a layer from about 48
// inputs on: error of the fitness against binary64 at 32-64-64-64-10 5.9e-8 -> 4.8e-8, but
// 6.3e-8 -> 7.0e-8 at 16-36-36-36-2, 5.4e-8 -> 5.6e-8 at 16-209-10 and 7.5e-8 -> 8.4e-8
// at 3-58-1, where the first layer's few products are all but exact in FP32, and with few
// outputs, where fewer logits average it out (5.9e-8 -> 6.2e-8 at 32-128-2, 5.6e-8 ->
// 6.8e-8 at 20-48-48-3; 5.9e-8 -> 5.8e-8 at 30-96-96-10, 5.3e-8 -> 4.0e-8 at 32-64-10).
bool chain_split(const Net &net)
{
    int widest = 0, narrowest = net.fi[0];
    for (int l = 0; l + 1 < net.nl; ++l) {
        widest = std::max(widest, net.fo[l]);
        narrowest = std::min(narrowest, net.fo[l]);
    }
    return !net.no_parts && !net.bf16 && !net.wide && widest >= 48 && narrowest >= 20 && net.fo[net.nl - 1] >= 8;
}

// Whether kernel entry e covers the network; *cost is the model cost used to
// rank the entries that do, *padded the products of its padded layers.
static bool entry_fits(const Net &net, const KernelEntry &e, double *cost, double *padded = nullptr)
{
    int need[MAXL] = {0, 0, 0, 0};
    for (int l = 0; l < net.nl; ++l) {
        need[l] = (net.fo[l] + 15) / 16;
        // BF16 chains need even 16-row blocks for every layer that feeds another
        if (net.bf16 && l < net.nl - 1 && (need[l] & 1)) need[l] += 1;
    }
    if (e.bf16 != net.bf16) return false;
    if (e.split && !chain_split(net)) return false;
    if (e.act >= 0) {
        for (int l = 0; l < net.nl - 1; ++l)   // a fixed activation must match every hidden layer
            if (net.act[l] != e.act) return false;
    }
    double c = 0.0;
    for (int l = 0; l < MAXL; ++l) {
        const bool present = l < net.nl;
        if (present != (e.R[l] > 0) || (present && e.R[l] < need[l])) return false;
        if (present) c += (double)e.R[l] * (l == 0 ? net.in_pad : net.fo[l - 1] + 16);
    }
    if (padded) *padded = c;
    if (e.wl) {
        // (the parts' kernels hold up to 400 bytes of their own; lds_max leaves 256)
        if (lds_bytes(net, e) + (e.split ? 256 : 0) > net.lds_max) return false;
        // staged weights beat global fragment loads; run-time activations with more row
        // blocks than twice the network's do not (12-45-1 in GELU, 156 sparks: 23 us a
        // generation from global memory in 4 row blocks, 29 us from LDS in 8)
        c *= e.act >= 0 || e.split ? 0.5 : 0.6;
    }
    if (e.act >= 0) c *= 0.9;                 // specialised activation: straight-line epilogue
    if (e.split) c *= 0.5;                    // three FP16 products against one in FP32
    *cost = c;
    return true;
}

// Blocks per spark row by default.  Weights in global memory: enough blocks to fill
// the chip (about 4 per CU) while keeping at least two slab groups per wavefront; a
// launch too small to fill the chip even then (a few rows) takes one slab group per
// wavefront, since its duration is the chain of passes a block runs.  Weights in LDS:
// every block stages them first (about half a pass of the FP32 kernels, a whole one
// of BF16's), so the least time over the rounds that the chip needs, eight wavefronts
// per CU at a time (16 of the narrow networks): 64 sparks of 64-128-128-10 in FP32 80 -> 59 us, 512 of 32-64-64-10
// in BF16 53 -> 46 us against four blocks per CU.
static int default_bpr(const Net &net, const KernelEntry &e, int rows)
{
    const int group = e.nw * 16 * e.P;                    // samples per block pass
    const int max_bpr = (net.S_pad + group - 1) / group;
    if (e.wl) {
        const int fit = (160 * 1024) / std::max(1, lds_bytes(net, e));
        int best = 1, widest = 0;
        for (int l = 0; l < net.nl; ++l) widest = std::max(widest, net.fo[l]);
        const int waves = widest <= 32 ? 16 : 8;
        const long at_once = (long)std::max(1, net.num_cu) * std::max(1, std::min(waves / e.nw, fit));
        double least = 0.0;
        for (int b = 1; b <= std::min(max_bpr, MAX_BPR); ++b) {
            const int passes = (max_bpr + b - 1) / b;
            if (b > 1 && passes == (max_bpr + b - 2) / (b - 1)) continue;   // no shorter blocks
            const long blocks = (long)rows * ((max_bpr + passes - 1) / passes);
            // (several blocks a row: the finalisation's launch, a pass of a small network)
            const double t = (double)((blocks + at_once - 1) / at_once) * (passes + (e.bf16 ? 1.0 : 0.5)) +
                             (b > 1 && widest <= 32 ? 1.0 : 0.0);
            if (b == 1 || t < least) {
                least = t;
                best = b;
            }
        }
        return best;
    }
    int bpr = (1024 + rows - 1) / (rows > 0 ? rows : 1);
    const int lim = (long)rows * max_bpr <= 1024 ? max_bpr : max_bpr / 2 > 0 ? max_bpr / 2 : 1;
    if (bpr > lim) bpr = lim;
    if (bpr > MAX_BPR) bpr = MAX_BPR;
    return bpr < 1 ? 1 : bpr;
}

// The plan for entry e with about `bpr` blocks per row (rounded to whole block passes).
static void make_plan(const Net &net, const KernelEntry &e, int rows, int bpr, FitPlan *plan)
{
    plan->kernel = e.fn;
    plan->gkernel = e.gfn;
    plan->nw = e.nw;
    plan->P = e.P;
    plan->wl = e.wl;
    plan->split = e.split;
    // Every block of a row draws the row's weights again, which the kernels of up to
    // three layers with the activation compiled in carry; others store the sparks (156
    // sparks of 12-45-1 in GELU: 33 us a generation drawn in the kernel, 23 us stored).
    plan->regen = e.wl && e.act >= 0 && net.nl <= 3;
    plan->rows = rows;
    plan->lds_bytes = lds_layouts(net, e, &plan->lay, &plan->lay32);
    if (!e.wl) plan->lds_bytes = 0;
    const int group = e.nw * 16 * e.P;
    int spb = (net.S_pad + bpr - 1) / bpr;
    spb = (spb + group - 1) / group * group;
    plan->bpr = (net.S_pad + spb - 1) / spb;
    plan->spb = spb;
}

bool fit_select(const Net &net, int rows, FitPlan *plan)
{
    const KernelEntry *best = nullptr;
    double best_cost = 0.0;
    for (auto table : kTables) {
        int nent = 0;
        const KernelEntry *ents = table(&nent);
        for (int ie = 0; ie < nent; ++ie) {
            double cost = 0.0;
            if (!entry_fits(net, ents[ie], &cost)) continue;
            // rows that fill the chip by themselves: with few samples a network of 16
            // units takes the blocks of fewer wavefronts (2,048 sparks x 256 samples of
            // 8-16-1: 51 us a generation with 2 x 2, 57 with 8 x 2; 256 sparks: 37 and 33)
            if (ents[ie].R[0] == 1 && ents[ie].nw > 4 && rows >= 4L * net.num_cu && net.S_pad < 1024)
                cost *= 1.1;
            if (!best || cost < best_cost) {
                best = &ents[ie];
                best_cost = cost;
            }
        }
    }
    if (!best) return false;
    make_plan(net, *best, rows, default_bpr(net, *best, rows), plan);
    return true;
}

int fit_candidates(const Net &net, int rows, FitPlan *out, int max_out)
{
    // entries that pad the layers to more than twice what the tightest one does are
    // never the fastest
    double least = 0.0;
    for (auto table : kTables) {
        int nent = 0;
        const KernelEntry *ents = table(&nent);
        for (int ie = 0; ie < nent; ++ie) {
            double cost = 0.0, padded = 0.0;
            if (entry_fits(net, ents[ie], &cost, &padded) && (least == 0.0 || padded < least)) least = padded;
        }
    }
    int n = 0;
    for (auto table : kTables) {
        int nent = 0;
        const KernelEntry *ents = table(&nent);
        for (int ie = 0; ie < nent; ++ie) {
            double cost = 0.0, padded = 0.0;
            if (!entry_fits(net, ents[ie], &cost, &padded) || padded > 2.0 * least) continue;
            const int b0 = default_bpr(net, ents[ie], rows);
            for (int b : {b0, 2 * b0, b0 / 2, 4 * b0}) {
                if (b < 1 || b > MAX_BPR || n >= max_out) continue;
                FitPlan p{};
                make_plan(net, ents[ie], rows, b, &p);
                bool dup = false;
                for (int i = 0; i < n; ++i)
                    dup = dup || (out[i].kernel == p.kernel && out[i].bpr == p.bpr);
                if (!dup) out[n++] = p;
            }
        }
    }
    return n;
}

hipError_t fit_prepare(const FitPlan &plan)
{
    if (plan.lds_bytes <= 0) return hipSuccess;
    return hipFuncSetAttribute(plan.kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                               plan.lds_bytes);
}

FitLaunch fit_launch_args(const Net &net, const FitPlan &plan, const DevState &d, const float *W,
                          size_t ld, int rows, OutMap map, float *out, const SparkRegen *rg)
{
    FitLaunch f;
    FitArgs &a = f.a;
    a.rg = rg ? *rg : SparkRegen{};
    a.W = W;
    a.ld = ld;
    a.rows = rows;
    a.X = d.Xp;
    a.Xb = d.Xb;
    a.in_pad = net.in_pad;
    a.S = net.S;
    a.S_pad = net.S_pad;
    a.nl = net.nl;
    for (int l = 0; l < MAXL; ++l) {
        a.fi[l] = net.fi[l];
        a.fo[l] = net.fo[l];
        a.woff[l] = net.woff[l];
        a.boff[l] = net.boff[l];
        a.act[l] = net.act[l];
        a.vec[l] = net.vec[l];
    }
    a.lay = plan.lay;
    a.lay32 = plan.lay32;
    a.loss = net.loss;
    a.Y = d.Ypad;
    a.lab = d.Lpad;
    a.bpr = plan.bpr;
    a.spb = plan.spb;
    a.partial = d.partial;
    a.Xs = d.Xs;
    a.Xe = d.Xe;
    a.wexp = net.box_exp;
    a.inv_norm = net.inv_norm;
    a.map = map;
    a.out = out;
    return f;
}

dim3 fitness_grid(const FitLaunch &f) { return dim3((unsigned)(f.a.rows * f.a.bpr)); }
dim3 finalize_grid(const FitLaunch &f) { return dim3((unsigned)((f.a.rows + 255) / 256)); }

hipError_t launch_fitness(const Net &net, const FitPlan &plan, const DevState &d, const float *W,
                          size_t ld, int rows, OutMap map, float *out, hipStream_t st,
                          hipEvent_t mid, const SparkRegen *rg)
{
    if (rows <= 0) return hipSuccess;
    if (rg && !plan.regen) return hipErrorInvalidValue;   // only the staging regenerates
    FitLaunch f = fit_launch_args(net, plan, d, W, ld, rows, map, out, rg);
    FitArgs &a = f.a;
    void *args[] = {&a};
    hipError_t e = hipLaunchKernel(plan.kernel, dim3((unsigned)(rows * plan.bpr)),
                                   dim3(64 * plan.nw), args, (size_t)plan.lds_bytes, st);
    if (e != hipSuccess) return e;
    if (mid) {
        e = hipEventRecord(mid, st);
        if (e != hipSuccess) return e;
    }
    if (plan.bpr == 1) return hipSuccess;   // (the blocks have finished their rows)
    hipLaunchKernelGGL(k_fit_finalize, finalize_grid(f), dim3(256), 0, st, d.partial, rows,
                       plan.bpr, net.inv_norm, map, out);
    return hipGetLastError();
}

hipError_t fit_group_prepare(const void *gkernel, int lds_bytes)
{
    if (lds_bytes <= 0) return hipSuccess;
    return hipFuncSetAttribute(gkernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
}

hipError_t launch_fitness_group(const GroupTable &t, const void *gkernel, int nw, int lds_bytes,
                                int which, hipStream_t st)
{
    GroupTable tt = t;
    void *args[] = {&tt, &which};
    return hipLaunchKernel(gkernel, dim3((unsigned)t.start[t.njobs]), dim3(64 * nw), args,
                           (size_t)lds_bytes, st);
}

hipError_t launch_finalize_group(const GroupTable &t, int which, hipStream_t st)
{
    hipLaunchKernelGGL(k_fit_finalize_group, dim3((unsigned)t.start[t.njobs]), dim3(256), 0, st, t,
                       which);
    return hipGetLastError();
}

hipError_t launch_pack_problem(const Net &net, const float *x, const float *y,
                               const int32_t *labels, const DevState &d, hipStream_t st)
{
    if (d.Xs && chain_split(net)) {   // (the wide kernel packs its samples itself)
        hipLaunchKernelGGL(k_split_exp, dim3((unsigned)((net.S_pad + 3) / 4)), dim3(256), 0, st, x, net.S,
                           net.S_pad, net.fi[0], d.Xe);
        const int pitch = (net.in_pad + 31) / 32 * 32;
        const size_t blocks = ((size_t)net.S_pad * pitch + 255) / 256;
        hipLaunchKernelGGL(k_pack_split, dim3((unsigned)blocks), dim3(256), 0, st, x, net.S, net.S_pad,
                           net.fi[0], pitch, d.Xe, d.Xs);
    }
    const int out = net.fo[net.nl - 1];
    size_t n = (size_t)net.S_pad * net.in_pad;
    if ((size_t)net.S_pad * out > n) n = (size_t)net.S_pad * out;
    const unsigned blocks = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(k_pack, dim3(blocks), dim3(256), 0, st, x, net.loss == 0 ? y : nullptr,
                       net.loss == 1 ? labels : nullptr, net.S, net.S_pad, net.fi[0], net.in_pad,
                       out, net.bf16, d.Xp, d.Xb, net.loss == 0 ? d.Ypad : nullptr,
                       net.loss == 1 ? d.Lpad : nullptr);
    return hipGetLastError();
}

}  // namespace mgfwa

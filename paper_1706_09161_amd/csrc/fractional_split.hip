// fractional_split.hip -- the dense fractional term (Sec. 2.4) on the BF16
// matrix cores, for axes too short for boxes (fractional_far.hip).  NT = 6:
// FP32 products from exact three-term BF16 splits (split_fragments.h; six BF16
// products take 6/16 of the matrix time of one FP32 product); NT = 3: the
// split of LBM_BF16X3.
//
// A workgroup of 4 wavefronts computes 32 lines x (64 WJ) outputs of one
// axis: WJ wavefronts take 64 outputs each, WK = 4 / WJ share the k range
// (steps of 16 k dealt round robin, summed through LDS in a fixed order).  The
// k range runs in chunks of KC:
//  * C of a chunk is read once by the workgroup (8 values of a line per thread
//    and 64 k), split, and parked in LDS as BF16 planes, line by line, so that
//    every wavefront reads its MFMA operand with one 16-byte load per plane:
//    the split costs 11 VALU instructions per pair of values, about as long as
//    the MFMAs of one 64-output wavefront, so it is shared;
//  * two chunk buffers: while chunk i is multiplied, chunk i + 1 is split and
//    stored and chunk i + 2 loaded; one LDS-only barrier a chunk;
//  * the Toeplitz operand comes from an LDS window of pair words stored with d
//    decreasing.  With WK = 1 the fragment of the second 32 outputs is that of
//    the first ones two steps before (T depends on j - k alone).
// Loads go through a buffer descriptor, so ragged axes and lines cost a mask
// and no separate path.
//
// Measured (us per launch, all axes, graph replay; in brackets the register
// kernels before), one-sided / two-sided: FP32 256^3 110 / 141 (221 / 221),
// 200 x 150 x 170 49 / 55 (140 / 140), 128^3 18 / 19 (27 / 27), 90 x 75 x 61
// 8.1 / 8.6 (14.9 / 14.9), 64^3 5.8 / 5.9 (8.3 / 7.6), 201 x 101 6.0 (8.9 /
// 8.8), 333 x 500 9.2 / 9.5 (12.5 / 12.8), 64^2 4.6 (5.1); split BF16 256^3 79 /
// 92 (119 / 126), 90 x 75 x 61 7.3 / 7.7 (15.9 / 15.7), 201 x 101 5.5 (11.9 /
// 11.4), 64^2 4.7 (7.2).  Errors of the FP32 sums fall too (256^3 relative L2
// 2.9e-7 -> 6.8e-8: three accumulators, 16 products a rounding).  At 256^3 the
// matrix work is 61 us and the bytes (C per axis, Phi) 80 us at 5 TB/s; small
// grids are a chain of loads, split, products and stores.
#include <hip/hip_runtime.h>
#include <limits.h>

#include "split_fragments.h"

namespace lbm {
namespace {

using namespace split;

constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;
constexpr int kJW = 64;  // outputs per wavefront

// KC: k per chunk.  A staged line takes KC + 8 BF16 (16 lines hit distinct banks).
template <bool CONTIG, int WJ, int KC, int NT>
__device__ __forceinline__ void split_tile(const SplitOp& op, const AxisLayout& lay, const float* __restrict__ C,
                                           float* __restrict__ Phi, int tiles_l, int tiles_j, int bid, int total,
                                           unsigned char* smem)
{
    constexpr int WK = kWaves / WJ;
    constexpr int JT = kJW * WJ;
    constexpr int SPC = KC / 16;  // k steps per chunk
    constexpr int SPW = SPC / WK; // of which a wavefront takes
    constexpr int NP = NT == 6 ? 3 : 2;
    constexpr int kRow = KC + 8, kPlane = 32 * kRow;
    constexpr int G = KC / 64;    // groups of 8 values a thread stages per chunk
    const int n = op.n, N = n - 1;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wj = wave / WK, wk = wave % WK;
    const int li = lane & 31, lh = lane >> 5;

    // contiguous workgroup ranges per XCD, the output tiles of a line block
    // next to each other: they share its C in that XCD's L2
    int lin = bid;
    if ((total & 7) == 0) lin = (bid & 7) * (total >> 3) + (bid >> 3);
    const int jt = lin % tiles_j;
    const int rest = lin / tiles_j;
    const int lt = rest % tiles_l;
    const int batch = rest / tiles_l;
    const int j0 = jt * JT;        // first output of the workgroup
    const int jw = j0 + kJW * wj;  // first output of the wavefront
    const int64_t line0 = (int64_t)lt * 32;
    const int64_t js = lay.j_stride;
    const uint32_t ks4 = CONTIG ? 4u : (uint32_t)js * 4u, ls4 = CONTIG ? (uint32_t)n * 4u : 4u;  // byte strides of k, line
    const float* Cb = C + (CONTIG ? line0 * n : (int64_t)batch * lay.batch_stride + line0);
    float* Pb = Phi + (CONTIG ? line0 * n : (int64_t)batch * lay.batch_stride + line0);
    const int nl = (int)min((int64_t)32, lay.lines - line0);  // lines past the end are computed, never stored
    const Rsrc Cr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(Cb), 0, (int)(4 * (CONTIG ? (int64_t)nl * n : (int64_t)n * js - line0)), 0x00020000);

    // k range (one-sided operators skip the zero triangle), in chunks
    int kb = 0, ke = n;
    if (op.lower_only) ke = min(n, j0 + JT);
    if (op.upper_only) kb = j0;
    const int nch = (ke - kb + KC - 1) / KC;
    const int kend = kb + nch * KC;
    // k past the axis and, for the forward operators, its two end nodes (whose
    // whole columns the epilogue adds) are left out of the sum
    const int k_lo = op.ends_excluded ? 1 : 0, k_hi = op.ends_excluded ? N : n;

    // LDS: boundary columns of each output tile | C at the walls of each line
    // (contiguous axis) | chunk buffers [2][NP] (later the k-share sums) |
    // Toeplitz window, NP planes
    float* cols = reinterpret_cast<float*>(smem);
    float* w0s = cols + WJ * 128;
    float* wNs = w0s + 32;
    uint16_t* cpl = reinterpret_cast<uint16_t*>(wNs + 32);
    uint32_t* win = reinterpret_cast<uint32_t*>(cpl + 2 * NP * kPlane);
    const int wlen = JT + (kend - kb);      // word x of a plane holds W(dmax - x)
    const int dmax = j0 + JT - 1 - kb;      // = 15 (mod 16): 64-byte aligned in the pair words

    // ---- staging of C: group id = (line, 8 consecutive k)
    uint32_t soff[G];
    int sk[G], sdst[G];
#pragma unroll
    for (int q = 0; q < G; ++q) {
        const int id = q * kThreads + threadIdx.x;
        const int row = CONTIG ? id / (KC / 8) : id % 32, g = CONTIG ? id % (KC / 8) : id / 32;
        sk[q] = kb + 8 * g;
        soff[q] = (uint32_t)min(row, nl - 1) * ls4 + (uint32_t)sk[q] * ks4;
        sdst[q] = row * kRow + 8 * g;
    }
    float raw[G][8];
    auto load_raw = [&](int ch) {
#pragma unroll
        for (int q = 0; q < G; ++q) load8<CONTIG>(Cr, soff[q] + (uint32_t)(ch * KC) * ks4, ks4, raw[q]);
    };
    auto park = [&](int ch) {
        if (kb + ch * KC < k_lo || kb + (ch + 1) * KC > k_hi) {  // uniform
#pragma unroll
            for (int q = 0; q < G; ++q) mask8(raw[q], sk[q] + ch * KC, k_lo, k_hi);
        }
#pragma unroll
        for (int q = 0; q < G; ++q) {
            u32x4 h, m, l;
            split3_8(raw[q], h, m, l);
            uint16_t* dst = cpl + (ch & 1) * NP * kPlane + sdst[q];
            *reinterpret_cast<u32x4*>(dst) = h;
            *reinterpret_cast<u32x4*>(dst + kPlane) = m;
            if constexpr (NT == 6) *reinterpret_cast<u32x4*>(dst + 2 * kPlane) = l;
        }
    };

    // ---- set-up: the first chunk of C, the window, boundary columns
    load_raw(0);
    {
        const int x0 = op.pw_top - dmax;
        for (int q = threadIdx.x; q < wlen / 4; q += kThreads) {
            *reinterpret_cast<u32x4*>(win + 4 * q) = *reinterpret_cast<const u32x4*>(op.pw_hi + x0 + 4 * q);
            *reinterpret_cast<u32x4*>(win + wlen + 4 * q) = *reinterpret_cast<const u32x4*>(op.pw_lo + x0 + 4 * q);
            if constexpr (NT == 6)
                *reinterpret_cast<u32x4*>(win + 2 * wlen + 4 * q) = *reinterpret_cast<const u32x4*>(op.pw_l3 + x0 + 4 * q);
        }
        if ((int)threadIdx.x < JT) {
            const int t = threadIdx.x, j = min(j0 + t, N);
            cols[t / 64 * 128 + t % 64] = op.col0[j];
            cols[t / 64 * 128 + 64 + t % 64] = op.colN[j];
        }
    }
    const uint32_t line_off = (uint32_t)min(li, nl - 1) * ls4;
    float b0 = 0.f, bN = 0.f;
    if constexpr (CONTIG) {
        if (threadIdx.x < 32) {
            w0s[threadIdx.x] = ldf(Cr, line_off);
            wNs[threadIdx.x] = ldf(Cr, line_off + (uint32_t)N * ks4);
        }
    } else {
        b0 = ldf(Cr, line_off);
        bN = ldf(Cr, line_off + (uint32_t)N * ks4);
    }
    park(0);
    if (nch > 1) load_raw(1);
    lds_barrier();

    Accumulators<CONTIG, NT> acc;
    acc.clear();
    // word of the Toeplitz fragment of k step s (from kb) and output block c: wbase + 16 s - 32 c
    const uint32_t* wbase = win + (JT - 1 - kJW * wj) - li + 8 * lh;
    // chunks outside [c_lo, c_hi) hold only zeros of this wavefront's
    // triangle (one-sided operators)
    const int c_lo = op.upper_only ? (jw - kb) / KC : 0;
    const int c_hi = op.lower_only ? (min(n, jw + kJW) - kb + KC - 1) / KC : nch;

    // Products of chunk ch: the fragments of step u + 1 are read while step u
    // is multiplied.
    auto multiply = [&](int ch) {
        const uint16_t* src = cpl + (ch & 1) * NP * kPlane + li * kRow + 8 * lh;
        const uint32_t* w = wbase + ch * KC;
        auto load_c = [&](int sc, Frag3& f) {
            f.h = ld16(src + 16 * sc);
            f.m = ld16(src + kPlane + 16 * sc);
            if constexpr (NT == 6) f.l = ld16(src + 2 * kPlane + 16 * sc);
        };
        Frag3 cf[2];
        // WK = 1: block-0 fragments by step modulo 4 (block 1 of step s is
        // block 0 of step s - 2); else both blocks of two steps
        Frag3 tf[4];
        load_c(wk, cf[0]);
        if constexpr (WK == 1) {
            tf[2] = toeplitz<NT>(w - 32, wlen);
            tf[3] = toeplitz<NT>(w - 16, wlen);
            tf[0] = toeplitz<NT>(w, wlen);
        } else {
            tf[0] = toeplitz<NT>(w + 16 * wk, wlen);
            tf[1] = toeplitz<NT>(w + 16 * wk - 32, wlen);
        }
#pragma unroll
        for (int u = 0; u < SPW; ++u) {
            if (u + 1 < SPW) {
                const int sn = (u + 1) * WK + wk;  // next step within the chunk
                load_c(sn, cf[(u + 1) & 1]);
                if constexpr (WK == 1) {
                    tf[(u + 1) & 3] = toeplitz<NT>(w + 16 * sn, wlen);
                } else {
                    tf[2 * ((u + 1) & 1)] = toeplitz<NT>(w + 16 * sn, wlen);
                    tf[2 * ((u + 1) & 1) + 1] = toeplitz<NT>(w + 16 * sn - 32, wlen);
                }
            }
            if constexpr (WK == 1) acc.add(cf[u & 1], tf[u & 3], tf[(u + 2) & 3], u & 1);
            else acc.add(cf[u & 1], tf[2 * (u & 1)], tf[2 * (u & 1) + 1], u & 1);
        }
    };
    for (int ch = 0; ch < nch; ++ch) {
        if (ch + 1 < nch) {
            park(ch + 1);
            if (ch + 2 < nch) load_raw(ch + 2);
        }
        if (ch >= c_lo && ch < c_hi) multiply(ch);
        lds_barrier();
    }
    f32x16 sum[2];
    acc.template total<(SPW > 1)>(sum);

    // ---- k shares summed in a fixed order; the 8 groups of 4 rows ("units",
    // u = 4 c + r4) are dealt out to the WK wavefronts
    constexpr int U = 8;
    const int u_lo = wk * (U / WK), u_hi = u_lo + U / WK;
    if constexpr (WK > 1) {
        float* red = reinterpret_cast<float*>(cpl);  // chunk buffers and window are dead
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u >= u_lo && u < u_hi) continue;
            const int c = u >> 2, r = 4 * (u & 3);
            *reinterpret_cast<f32x4*>(red + ((wave * U + u) * 64 + lane) * 4) =
                f32x4{sum[c][r], sum[c][r + 1], sum[c][r + 2], sum[c][r + 3]};
        }
        lds_barrier();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u < u_lo || u >= u_hi) continue;
            const int c = u >> 2, r = 4 * (u & 3);
            f32x4 part[WK];
#pragma unroll
            for (int s = 0; s < WK; ++s)
                part[s] = s == wk ? f32x4{sum[c][r], sum[c][r + 1], sum[c][r + 2], sum[c][r + 3]}
                                  : *reinterpret_cast<const f32x4*>(red + (((wj * WK + s) * U + u) * 64 + lane) * 4);
            // pairwise: two roundings of the full sum instead of three (uniform C
            // = 0.7 at 96 x 80 in split BF16: 1.43e-6 rms against 1.48e-6)
#pragma unroll
            for (int h = WK / 2; h > 0; h /= 2)
#pragma unroll
                for (int s = 0; s < h; ++s)
#pragma unroll
                    for (int e = 0; e < 4; ++e) part[s][e] = part[2 * s][e] + part[2 * s + 1][e];
            const f32x4 t = part[0];
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[c][r + e] = t[e];
        }
    }
    store_tile<CONTIG, NT == 6>(op, sum, u_lo, u_hi, {cols + wj * 128, w0s, wNs, b0, bN}, Cb, Pb, nl, jw, k_lo, k_hi, ls4,
                                ks4);
}

template <int WJ, int KC, int NT>
__global__ __launch_bounds__(kThreads, WJ == 1 && KC == 64 ? 4 : 2) void fractional_split(SplitLaunch L)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_s[];
    const int bid = blockIdx.x;
    int axis = 0;
    while (axis + 1 < L.naxes && bid >= L.first[axis + 1]) ++axis;
    const int local = bid - L.first[axis];
    const int total = L.first[axis + 1] - L.first[axis];
    if (L.lay[axis].contiguous)
        split_tile<true, WJ, KC, NT>(L.op[axis], L.lay[axis], L.C[axis], L.Phi[axis], L.tiles_m[axis], L.tiles_n[axis],
                                     local, total, smem_s);
    else
        split_tile<false, WJ, KC, NT>(L.op[axis], L.lay[axis], L.C[axis], L.Phi[axis], L.tiles_m[axis], L.tiles_n[axis],
                                      local, total, smem_s);
}

// tiles_m = line blocks of 32, tiles_n = output tiles
template <int WJ, int KC, int NT>
void split_grid(SplitLaunch& L, int64_t& grid, size_t& lds)
{
    grid = 0;
    lds = 0;
    for (int a = 0; a < L.naxes; ++a) {
        const SplitOp& op = L.op[a];
        const AxisLayout& lay = L.lay[a];
        L.tiles_m[a] = (int)((lay.lines + 31) / 32);
        L.tiles_n[a] = (op.n + kJW * WJ - 1) / (kJW * WJ);
        L.first[a] = (int)grid;
        grid += (int64_t)L.tiles_m[a] * L.tiles_n[a] * (lay.contiguous ? 1 : lay.batches);
        constexpr size_t NP = NT == 6 ? 3 : 2;
        const size_t kspan = (size_t)((op.n + KC - 1) / KC) * KC;
        size_t body = sizeof(uint16_t) * 2 * NP * 32 * (KC + 8) + sizeof(uint32_t) * NP * (kJW * WJ + kspan);
        const size_t red = WJ < kWaves ? sizeof(float) * kWaves * 8 * 64 * 4 : 0;
        body = body > red ? body : red;
        const size_t b = sizeof(float) * (WJ * 128 + 64) + body;
        lds = b > lds ? b : lds;
    }
}

template <int WJ, int KC, int NT>
hipError_t run_split(SplitLaunch& L, hipStream_t s)
{
    int64_t grid = 0;
    size_t lds = 0;
    split_grid<WJ, KC, NT>(L, grid, lds);
    if (grid > 0x7fffffff || lds > 160 * 1024) return hipErrorInvalidValue;
    L.first[L.naxes] = (int)grid;
    auto kern = fractional_split<WJ, KC, NT>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kThreads), lds, s, L);
    return hipGetLastError();
}

// Output tiles per workgroup and k per chunk.  One output tile where the
// workgroups would be few or the axes have one; then the four wavefronts share
// k.  Chunks of 128 k there as long as every CU can hold its workgroups'
// larger buffers at once (<1,64> / <1,128>, FP32, us: 201 x 101 6.3 / 6.0,
// 333 x 500 10.0 / 9.5, 640^2 13.6 / 12.9, but 768^2 18.5 / 21.7, 90 x 75 x 61
// 8.6 / 11.6).  From four workgroups per CU on, wavefronts take whole k ranges
// (two output tiles at 128 nodes: 128^3 19.3 against 22.0; four beyond:
// 256^3 141 against 201 with one, 171 with two).
template <int NT>
hipError_t pick(SplitLaunch& L, hipStream_t s)
{
    int nmax = 0;
    for (int a = 0; a < L.naxes; ++a) nmax = L.op[a].n > nmax ? L.op[a].n : nmax;
    SplitLaunch T = L;
    int64_t grid = 0;
    size_t lds = 0;
    if (nmax <= 64) return run_split<1, 64, NT>(L, s);
    split_grid<4, 64, NT>(T, grid, lds);
    if (nmax > 128 && grid >= 1024) return run_split<4, 64, NT>(L, s);
    split_grid<2, 64, NT>(T, grid, lds);
    if (nmax <= 128 && grid >= 1024) return run_split<2, 64, NT>(L, s);
    split_grid<1, 64, NT>(T, grid, lds);
    if (grid <= 512) return run_split<1, 128, NT>(L, s);
    return run_split<1, 64, NT>(L, s);
}

}  // namespace

// Whether this kernel takes a launch: axes with their third plane and within
// 32-bit byte offsets, except in 2D where the register kernels are still faster
// (us, this kernel / the register kernel):
//  * FP32, every axis a multiple of 8: 65 to 128 nodes (72^2 5.44 / 5.17, 128^2
//    5.45 / 5.32), and strided axes beyond 128 up to 224 nodes on the longer
//    axis (136^2 6.55 / 6.31, 208^2 6.52 / 6.37, 96 x 192 6.44 / 6.24), or 384 if
//    an operator is two-sided (240^2 6.57 / 6.51, 304^2 7.77 / 7.69, 160 x 240
//    6.58 / 6.44).  The next ones are this kernel's: one-sided 240^2 6.53 / 6.74,
//    480^2 8.97 / 9.11, and a strided axis of up to 128 beside a longer
//    contiguous one, 200 x 128 5.89 / 6.33, 400 x 320 7.85 / 8.44.
//  * Split BF16, every axis a multiple of 16: a strided axis of 385 to 512 nodes,
//    none longer, with a two-sided operator (400^2 7.82 / 7.61, 512^2 7.81 /
//    7.69, 96 x 512 7.59 / 7.42; one-sided 512^2 7.71 / 7.82, 384^2 6.95 / 7.53,
//    512 x 256 6.49 / 7.50, 528^2 9.32 / 9.95), and beyond 832 (896^2 15.98 /
//    14.99, 1024^2 18.41 / 15.24; 832^2 13.55 / 14.61).  Multiples of 8 alone:
//    every axis of 961 to 1024 nodes with a two-sided operator (968^2 19.79 /
//    19.21, 1000^2 19.95 / 19.54; one-sided 1000^2 14.81 / 18.95, 936^2 19.41 /
//    19.79, 1032^2 28.2 / 43.9).
// In 3D the line blocks are many enough to hide this kernel's set-up (split
// BF16 1024 x 64 x 64 42.1 / 54.3, 2048 x 64 x 64 93 / 114) until one axis is
// nearly all of the grid (4096 x 16 x 16 53.6 / 45.4).
bool split_takes(const SplitLaunch& L, int dim, int terms)
{
    int nmax = 0, nmin = INT_MAX, align = 0, ny = 0;  // ny: longest strided axis
    bool two_sided = false;
    for (int a = 0; a < L.naxes; ++a) {
        const SplitOp& op = L.op[a];
        if (!op.pw_l3 || !far_reaches(L.lay[a], op.n)) return false;
        nmax = op.n > nmax ? op.n : nmax;
        nmin = op.n < nmin ? op.n : nmin;
        align |= op.n;
        if (!L.lay[a].contiguous && op.n > ny) ny = op.n;
        two_sided = two_sided || (!op.lower_only && !op.upper_only);
    }
    if (terms == 6) {
        if (dim == 3 || align % 8 != 0 || nmax <= 64) return true;
        return nmax > 128 && (ny <= 128 || nmax > (two_sided ? 384 : 224));
    }
    if (align % 8 != 0) return true;
    if (dim == 3) return align % 16 != 0 || nmax <= 2048;
    if (align % 16 != 0) return !(two_sided && nmin > 960 && nmax <= 1024);
    return nmax <= 832 && !(two_sided && ny > 384 && nmax <= 512);
}

hipError_t launch_fractional_split(SplitLaunch& L, int terms, hipStream_t s)
{
    return terms == 3 ? pick<3>(L, s) : pick<6>(L, s);
}

}  // namespace lbm

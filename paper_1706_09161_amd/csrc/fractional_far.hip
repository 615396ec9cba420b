// fractional_far.hip -- the fractional term (Sec. 2.4) of long axes: products
// with the near part of the Toeplitz operator as they stand, and the far part
// through 16 moments per box of 128 nodes.
//
// The product-rule weights a_k = (k+1)^{g+1} - 2 k^{g+1} + (k-1)^{g+1} are a
// smooth function of k away from k = 0.  Outputs j of a target box
// [128 J, 128 J + 128) take the nodes k of the band [128 J - 64, 128 J + 192)
// from T(j - k) itself; every other node lies in a source box
// [128 m - 64, 128 m + 64), m <= J - 1 or m >= J + 2, at least 64 nodes away,
// where T(j - k) is interpolated at 16 x 16 Chebyshev nodes of the two boxes,
//   T(j - k) = sum_pq l_p(j) T(x_p - y_q) l_q(k),
// l the Lagrange polynomials of those nodes.  Both boxes have half width 64
// and the nearest point of the other box is 128 from their centre: in 64-bit
// arithmetic the result differs from the dense sum by 1e-12 of its norm, and
// by at most 2.4e-11 of any single value (n = 700 ... 4096, g = 0.1 ... 0.95).
// Per line the far part is
//   moments  mom_m = sum_k l(k) C[k]                      (16 per box),
//   local    loc_J = sum_{far m} T(x - y) mom_m           (16 x 16 per pair of boxes),
//   Phi[j] += l(j) . loc_J,
// so a node costs 256 + 16 + n / 64 + 16 products instead of n.
//
// All contractions run on the BF16 matrix cores with exact three-term splits
// (split_fragments.h).  One workgroup (NW wavefronts) holds 32 lines: it
// computes the moments of all their source boxes into LDS, then walks over
// groups of NW / 2 target boxes, two wavefronts (64 outputs each) per box.  No
// moment leaves the workgroup, so there is no workspace and calls on several
// streams do not meet.  Where the lines alone do not fill the chip, several
// workgroups share a line block's target boxes and each computes the moments
// again.  Each wavefront reads the C of its band straight into registers and
// splits it there; a group has one barrier, between the two wavefronts' halves
// of the local coefficients and their use.  LBM_FP32 only: in LBM_BF16X3 the
// rounding of the split weights, which this sum does not have, is the result's
// largest error, so its values would be other ones (4096^2, 10 steps: C moves
// by up to 1.2e-3 of its rms, as far as it is from 64 bits).
//
// Measured (us per launch, both axes, graph replay; before: the dense FP32
// kernels), one-sided p = (1, 0) / two-sided p = (0.3, 0.8): 4096^2 1113 / 2106
// -> 118 / 158, 2048^2 183 / 272 -> 39 / 48, 1024^2 39 / 41 -> 18 / 21.
// At 4096^2 the moments read C at 7 TB/s; of the band's time half is matrix
// work, the rest the split of C, its loads and the stores.  Below about 1500
// nodes one wavefront per SIMD runs load, moments, local coefficients and band
// one after the other, so latency bounds it (1024^2 two-sided, cycles: tables
// 3.4k, moments 14k, local 4k, band 10k, stores 3k).  Errors against 64 bits
// (relative L2, pulses, dense FP32 in brackets): 1024^2 5.7e-8 / 6.2e-8 (6.0e-8
// / 8.0e-8), 4096^2 5.7e-8 / 5.9e-8 (5.2e-8 / 7.8e-8); random C 6.1e-8 / 6.4e-8
// (8.0e-8 / 9.5e-8) and 6.2e-8 / 7.0e-8 (1.0e-7 / 2.6e-7).  Adding the three
// accumulators with the first sum's rounding carried along takes about 5e-9 off
// each, and 2 to 4 % more time (4096^2 one-sided 115.8 -> 120.7 us).
#include <hip/hip_runtime.h>
#include <math.h>

#include <vector>

#include "split_fragments.h"

namespace lbm {
namespace {

using namespace split;

constexpr int kBox = 128;    // nodes per target and source box
constexpr int kRank = 16;    // Chebyshev nodes per box
constexpr int kWin = 384;    // pair words of the band: d = 191 ... -191
constexpr int kDmax = 191;

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 acc)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
}

// acc += a b with six products; the five small ones into corr
__device__ __forceinline__ void six16(const Frag3& a, const Frag3& b, f32x4& main_, f32x4& corr)
{
    corr = mfma16(a.l, b.h, corr);
    main_ = mfma16(a.h, b.h, main_);
    corr = mfma16(a.h, b.l, corr);
    corr = mfma16(a.m, b.m, corr);
    corr = mfma16(a.m, b.h, corr);
    corr = mfma16(a.h, b.m, corr);
}

template <bool CONTIG, int NW>
__device__ __forceinline__ void far_tile(const SplitOp& op, const AxisLayout& lay, const float* __restrict__ C,
                                         float* __restrict__ Phi, int tiles_l, int splits, int bid, int total,
                                         unsigned char* smem)
{
    constexpr int T = 64 * NW;  // threads
    constexpr int NB = NW / 2;  // target boxes per group
    const int n = op.n, N = n - 1;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 31, lh = lane >> 5;
    const int l16 = lane & 15, lg = lane >> 4;

    // contiguous workgroup ranges per XCD; the workgroups of a line block are
    // neighbours and share its C in that XCD's L2
    int lin = bid;
    if ((total & 7) == 0) lin = (bid & 7) * (total >> 3) + (bid >> 3);
    const int sp = lin % splits;
    const int rest = lin / splits;
    const int lt = rest % tiles_l;
    const int batch = rest / tiles_l;
    const int64_t lines = lay.lines;
    const int64_t line0 = (int64_t)lt * 32;
    const int64_t js = lay.j_stride;
    // the block's lines; the launch checks that 32-bit byte offsets reach them
    const float* Cb = C + (CONTIG ? line0 * n : (int64_t)batch * lay.batch_stride + line0);
    float* Pb = Phi + (CONTIG ? line0 * n : (int64_t)batch * lay.batch_stride + line0);
    const int nl = (int)min((int64_t)32, lines - line0);  // lines past the end are computed, never stored
    const uint32_t ks4 = CONTIG ? 4u : (uint32_t)js * 4u, ls4 = CONTIG ? (uint32_t)n * 4u : 4u;  // byte strides of k, line
    const Rsrc Cr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(Cb), 0, (int)(4 * (CONTIG ? (int64_t)nl * n : (int64_t)n * js - line0)), 0x00020000);
    const int nJ = (n + kBox - 1) / kBox;
    const int nsp = far_sources(n);  // source boxes (even)
    const int ms = kRank * nsp + 8;  // BF16 per line of a moment plane
    const int ngroups = (nJ + NB - 1) / NB;
    const int g_lo = (int)((int64_t)ngroups * sp / splits), g_hi = (int)((int64_t)ngroups * (sp + 1) / splits);
    // k past the axis and, for the forward operators, its two end nodes (whose
    // whole columns the epilogue adds) are left out of the sums
    const int k_lo = op.ends_excluded ? 1 : 0, k_hi = op.ends_excluded ? N : n;

    // LDS: band window, 3 planes | local coefficients [2][box][k half][line][p]
    // | boundary columns of each wavefront's outputs | C at the walls of each
    // line (contiguous axis) | U fragments | moment planes
    uint32_t* win = reinterpret_cast<uint32_t*>(smem);
    float* locs = reinterpret_cast<float*>(win + 3 * kWin);
    float* cols = locs + 2 * NW * 32 * kRank;
    float* w0s = cols + NW * 128;
    float* wNs = w0s + 32;
    uint16_t* ufr = reinterpret_cast<uint16_t*>(wNs + 32);
    uint16_t* mom = ufr + 6144;

    {
        const int x0 = op.pw_top - kDmax;
        for (int i = threadIdx.x; i < 3 * kWin / 4; i += T) {
            const int pl = i / (kWin / 4), q = i - pl * (kWin / 4);
            const uint32_t* src = pl == 0 ? op.pw_hi : (pl == 1 ? op.pw_lo : op.pw_l3);
            *reinterpret_cast<u32x4*>(win + pl * kWin + 4 * q) = *reinterpret_cast<const u32x4*>(src + x0 + 4 * q);
        }
        for (int i = threadIdx.x; i < 6144 / 8; i += T)
            *reinterpret_cast<u32x4*>(ufr + 8 * i) = *reinterpret_cast<const u32x4*>(op.far_uv + 8 * i);
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

    // ---- moments: D[p][line] = sum_k l_p(k) C[line][k] for 16 lines and one
    // source box at a time per wavefront ("unit" = box, line half), the next
    // unit's C in flight.  A one-sided operator needs the boxes on one side of
    // this workgroup's target boxes only.
    {
        const int m_lo = op.upper_only ? min(nsp, (NB * g_lo + 2) & ~1) : 0;
        const int m_hi = op.lower_only ? min(nsp, (NB * g_hi + 1) & ~1) : nsp;
        Frag3 vf[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const uint16_t* v = op.far_uv + 6144 + (ks * 3 * 64 + lane) * 8;
            vf[ks].h = ld16(v);
            vf[ks].m = ld16(v + 512);
            vf[ks].l = ld16(v + 1024);
        }
        uint32_t unit_off[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) unit_off[h] = (uint32_t)min(16 * h + l16, nl - 1) * ls4;
        auto load_unit = [&](int u, float (&raw)[4][8]) {
            const int kbox = kBox * (u >> 1) - kBox / 2;
            const uint32_t off = ((u & 1) ? unit_off[1] : unit_off[0]) + (uint32_t)(kbox + 8 * lg) * ks4;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) load8<CONTIG>(Cr, off + 32u * ks * ks4, ks4, raw[ks]);
        };
        auto add_unit = [&](int u, float (&raw)[4][8]) {
            const int m = u >> 1, kbox = kBox * m - kBox / 2;
            if (kbox < k_lo || kbox + kBox > k_hi) {  // uniform
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) mask8(raw[ks], kbox + 32 * ks + 8 * lg, k_lo, k_hi);
            }
            f32x4 mn[2], co;
#pragma unroll
            for (int r = 0; r < 4; ++r) mn[0][r] = mn[1][r] = co[r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                u32x4 ch, cm, cl;
                split3_8(raw[ks], ch, cm, cl);
                const Frag3 cf = {as_bf16(ch), as_bf16(cm), as_bf16(cl)};
                six16(vf[ks], cf, mn[ks & 1], co);
            }
            // moments p = 4 lg .. 4 lg + 3 of line 16 (u & 1) + l16
            uint32_t h0, m0, q0, h1, m1, q1;
            float v[4], ev[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float s1, e1, e2;
                two_sum(mn[0][r], mn[1][r], s1, e1);
                two_sum(s1, co[r], v[r], e2);
                ev[r] = e1 + e2;
            }
            split3_pair(v[0], ev[0], v[1], ev[1], h0, m0, q0);
            split3_pair(v[2], ev[2], v[3], ev[3], h1, m1, q1);
            uint16_t* dst = mom + (16 * (u & 1) + l16) * ms + kRank * m + 4 * lg;
            *reinterpret_cast<uint2*>(dst) = make_uint2(h0, h1);
            *reinterpret_cast<uint2*>(dst + 32 * ms) = make_uint2(m0, m1);
            *reinterpret_cast<uint2*>(dst + 64 * ms) = make_uint2(q0, q1);
        };
        const int u_hi = 2 * m_hi;
        int u = 2 * m_lo + wave;
        float ra[4][8], rb[4][8];
        if (u < u_hi) load_unit(u, ra);
        auto stage = [&](float (&now)[4][8], float (&ahead)[4][8]) {
            if (u + NW < u_hi) load_unit(u + NW, ahead);
            if (u < u_hi) add_unit(u, now);
            u += NW;
        };
        while (u < u_hi) {
            stage(ra, rb);
            stage(rb, ra);
        }
    }
    lds_barrier();

    // the two wavefronts of a SIMD (wave, wave + 4) take different halves: the
    // halves of a one-sided operator's band differ in length
    const int half = (wave ^ (wave >> 2)) & 1;
    // word of the Toeplitz fragment of step s and output block c: wbase + 16 s - 32 c
    const uint32_t* wbase = win + 127 - 64 * half - li + 8 * lh;

    for (int g = g_lo; g < g_hi; ++g) {
        const int J = NB * g + (wave >> 1);  // this wavefront's target box (may lie past the axis)
        const int jw = kBox * J + 64 * half; // first output
        const int kband = kBox * J - 64;     // k of step 0
        // steps of 16 k, in fours: on the axis, and on the side a one-sided
        // operator needs
        int s_lo = J == 0 ? 4 : 0, s_hi = min(16, (min(n, kband + 256) - kband + 63) / 64 * 4);
        if (op.upper_only) s_lo = 4 + 4 * half;
        if (op.lower_only) s_hi = min(s_hi, 8 + 4 * half);
        const bool live = jw < n;

        // C of a step: lane = (line li, 8 consecutive k)
        const uint32_t band_off = line_off + (uint32_t)(kband + 8 * lh) * ks4;
        auto load_c = [&](int s, float (&v)[8]) {
            load8<CONTIG>(Cr, band_off + (uint32_t)(16 * min(s, s_hi - 1)) * ks4, ks4, v);
        };
        float raw[2][8];
        if (live) {
            load_c(s_lo, raw[0]);
            load_c(s_lo + 1, raw[1]);
            const int j = min(jw + lane, N);
            const float c0 = op.col0[j], cN = op.colN[j];
            cols[wave * 128 + lane] = c0;
            cols[wave * 128 + 64 + lane] = cN;
        }

        // ---- local coefficients of box J: the far boxes in pairs (32
        // moments), even pairs by one wavefront of the box and odd ones by the
        // other; the table holds zeros for the near boxes
        float* lbuf = locs + (g & 1) * NW * 32 * kRank;
        {
            f32x4 mn[2][2], co[2];
#pragma unroll
            for (int r = 0; r < 4; ++r) mn[0][0][r] = mn[0][1][r] = mn[1][0][r] = mn[1][1][r] = co[0][r] = co[1][r] = 0.f;
            int i_lo = 0, i_hi = nsp / 2;
            if (op.lower_only) i_hi = min(i_hi, (J + 1) / 2);
            if (op.upper_only) i_lo = min(i_hi, (J + 2) / 2);
            if (J >= nJ) i_hi = i_lo;
            const uint16_t* mb = mom + l16 * ms + 8 * lg;
            const uint16_t* fm = op.far_m + ((int64_t)(J + nsp - 1 - (lg >> 1)) * 3 * kRank + l16) * kRank + 8 * (lg & 1);
            auto pair = [&](int i, Frag3& a) {
                const uint16_t* p = fm - (int64_t)i * (2 * 3 * kRank * kRank);
                a.h = ld16(p);
                a.m = ld16(p + kRank * kRank);
                a.l = ld16(p + 2 * kRank * kRank);
            };
            auto add = [&](int i, const Frag3& a, int set) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint16_t* q = mb + 16 * h * ms + 32 * i;
                    const Frag3 b = {ld16(q), ld16(q + 32 * ms), ld16(q + 64 * ms)};
                    six16(a, b, mn[set][h], co[h]);
                }
            };
            int i = i_lo + (wave & 1);
            for (; i + 6 < i_hi; i += 8) {
                Frag3 a[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) pair(i + 2 * u, a[u]);
#pragma unroll
                for (int u = 0; u < 4; ++u) add(i + 2 * u, a[u], u & 1);
            }
            for (; i < i_hi; i += 4) {
                Frag3 a[2];
                pair(i, a[0]);
                if (i + 2 < i_hi) pair(i + 2, a[1]);
                add(i, a[0], 0);
                if (i + 2 < i_hi) add(i + 2, a[1], 1);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                f32x4 v;
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = (mn[0][h][r] + mn[1][h][r]) + co[h][r];
                *reinterpret_cast<f32x4*>(lbuf + (wave * 32 + 16 * h + l16) * kRank + 4 * lg) = v;
            }
        }
        lds_barrier();
        if (!live) continue;

        // ---- band: C split in registers, its loads 2 steps ahead
        Accumulators<CONTIG, 6> acc;
        acc.clear();
        Frag3 cf[2], tf[4];  // tf: block-0 fragments by step modulo 4; block 1 of step s is block 0 of step s - 2
        tf[2] = toeplitz<6>(wbase + 16 * s_lo - 32, kWin);
        tf[3] = toeplitz<6>(wbase + 16 * s_lo - 16, kWin);
        tf[0] = toeplitz<6>(wbase + 16 * s_lo, kWin);
        const int kl = kband + 8 * lh;
        const bool edge = kband + 16 * s_lo < k_lo || kband + 16 * s_hi > k_hi;  // uniform
        if (edge) mask8(raw[0], kl + 16 * s_lo, k_lo, k_hi);
        cf[0] = planes(raw[0]);
        for (int s = s_lo; s < s_hi; s += 4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (edge) mask8(raw[(u + 1) & 1], kl + 16 * (s + u + 1), k_lo, k_hi);
                tf[(u + 1) & 3] = toeplitz<6>(wbase + 16 * min(s + u + 1, 15), kWin);
                load_c(s + u + 2, raw[u & 1]);  // slot of step s + u, converted already
                cf[(u + 1) & 1] = planes(raw[(u + 1) & 1]);
                acc.add(cf[u & 1], tf[u & 3], tf[(u + 2) & 3], u & 1);
                __builtin_amdgcn_sched_barrier(0);
            }
        }

        // ---- far part: both wavefronts' local coefficients times l_p(j)
        {
            Frag3 uf[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const uint16_t* u = ufr + ((half * 2 + c) * 3 * 64 + lane) * 8;
                uf[c].h = ld16(u);
                uf[c].m = ld16(u + 512);
                uf[c].l = ld16(u + 1024);
            }
            const float* lp = lbuf + ((wave & ~1) * 32 + li) * kRank + 8 * lh;
            float lv[8], ev[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) two_sum(lp[e], lp[32 * kRank + e], lv[e], ev[e]);
            u32x4 h, m, l;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                uint32_t hp, mp, qp;
                split3_pair(lv[2 * p], ev[2 * p], lv[2 * p + 1], ev[2 * p + 1], hp, mp, qp);
                h[p] = hp;
                m[p] = mp;
                l[p] = qp;
            }
            const Frag3 x = {as_bf16(h), as_bf16(m), as_bf16(l)};
            acc.add(x, uf[0], uf[1], 1);
        }

        // ---- boundary columns and stores
        f32x16 sum[2];
        acc.total(sum);
        store_tile<CONTIG, true>(op, sum, 0, 8, {cols + wave * 128, w0s, wNs, b0, bN}, Cb, Pb, nl, jw, k_lo, k_hi,
                                    ls4, ks4);
    }
}

template <int NW>
__global__ __launch_bounds__(64 * NW, 2) void fractional_far(SplitLaunch L)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_f[];
    const int bid = blockIdx.x;
    int axis = 0;
    while (axis + 1 < L.naxes && bid >= L.first[axis + 1]) ++axis;
    const int local = bid - L.first[axis];
    const int total = L.first[axis + 1] - L.first[axis];
    if (L.lay[axis].contiguous)
        far_tile<true, NW>(L.op[axis], L.lay[axis], L.C[axis], L.Phi[axis], L.tiles_m[axis], L.tiles_n[axis], local,
                               total, smem_f);
    else
        far_tile<false, NW>(L.op[axis], L.lay[axis], L.C[axis], L.Phi[axis], L.tiles_m[axis], L.tiles_n[axis],
                                local, total, smem_f);
}

// Chebyshev nodes of [-1, 1] and their Lagrange polynomials, FP64
double cheb(int p) { return cos((2 * p + 1) * M_PI / (2 * kRank)); }
double lagrange(int p, double x)
{
    double v = 1.0;
    for (int q = 0; q < kRank; ++q)
        if (q != p) v *= (x - cheb(q)) / (cheb(p) - cheb(q));
    return v;
}

// T(x_p - y_q) of every pair of boxes at box distance delta = J - m, split
// into three BF16 planes: entry delta + nsp - 1, [plane][p][q]; zero for the
// near boxes (delta = 0, -1).  The weights at a real distance d >= 64 come
// from their binomial series (FP64),
//   a(d) = g (g + 1) d^{g-1} (1 + (g-1)(g-2)/12 d^-2 (1 + (g-3)(g-4)/30 d^-2 (1 + ...))),
// which has no cancellation (the second difference as printed loses d^2 / g
// of the 64-bit precision).
struct FarTables {
    int first[4];  // first workgroup of every axis
    int nsp[3];
    double g[3], pos[3], neg[3];
    uint16_t* out[3];
};

__global__ __launch_bounds__(256) void far_table(FarTables F)
{
    const int ax = (int)blockIdx.x >= F.first[2] ? 2 : ((int)blockIdx.x >= F.first[1] ? 1 : 0);
    const int entry = (int)blockIdx.x - F.first[ax], nsp = F.nsp[ax];
    const double g = F.g[ax], pos = F.pos[ax], neg = F.neg[ax];
    const int delta = entry - (nsp - 1);
    const int p = threadIdx.x / kRank, q = threadIdx.x % kRank;
    double v = 0.0;
    if (delta != 0 && delta != -1) {
        const double xp = cos((2 * p + 1) * 3.14159265358979323846 / (2 * kRank));
        const double xq = cos((2 * q + 1) * 3.14159265358979323846 / (2 * kRank));
        const double d = (double)kBox * delta + 64.0 + 64.0 * (xp - xq);
        const double ad = fabs(d), z = 1.0 / (d * d);
        double s = 1.0 + (g - 5.0) * (g - 6.0) / 56.0 * z * (1.0 + (g - 7.0) * (g - 8.0) / 90.0 * z);
        s = 1.0 + (g - 3.0) * (g - 4.0) / 30.0 * z * s;
        s = 1.0 + (g - 1.0) * (g - 2.0) / 12.0 * z * s;
        v = (d > 0.0 ? pos : neg) * g * (g + 1.0) * pow(ad, g - 1.0) * s;
    }
    uint16_t* o = F.out[ax] + (size_t)entry * 3 * kRank * kRank + threadIdx.x;
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) {
        const float f = (float)v;
        const __bf16 b = (__bf16)f;
        o[pl * kRank * kRank] = __builtin_bit_cast(uint16_t, b);
        v -= (double)(float)b;
    }
}

template <int NW>
size_t far_lds(int n)
{
    const int ms = kRank * far_sources(n) + 8;
    return sizeof(uint32_t) * 3 * kWin + sizeof(float) * (2 * NW * 32 * kRank + NW * 128 + 64) +
           sizeof(uint16_t) * (6144 + 3 * 32 * ms);
}

template <int NW>
hipError_t run_far(SplitLaunch& L, hipStream_t s)
{
    size_t lds = 0;
    int64_t per[3];
    for (int a = 0; a < L.naxes; ++a) {
        const AxisLayout& lay = L.lay[a];
        L.tiles_m[a] = (int)((lay.lines + 31) / 32);
        per[a] = (int64_t)L.tiles_m[a] * (lay.contiguous ? 1 : lay.batches);
        const size_t b = far_lds<NW>(L.op[a].n);
        lds = b > lds ? b : lds;
    }
    // groups per workgroup: the fewest that keep the launch within one round of
    // workgroups (one per CU, two with NW = 4, whose LDS allows them); all of a
    // line block's groups where the line blocks fill the chip
    const int64_t round = NW == 4 ? 512 : 256;
    int64_t grid = 0;
    for (int per_wg = 1, last = 0; !last; ++per_wg) {
        grid = 0;
        last = 1;
        for (int a = 0; a < L.naxes; ++a) {
            const int ng = ((L.op[a].n + kBox - 1) / kBox + NW / 2 - 1) / (NW / 2);
            const int sp = (ng + per_wg - 1) / per_wg;
            L.tiles_n[a] = sp;
            L.first[a] = (int)grid;
            grid += per[a] * sp;
            last = last && sp == 1;
        }
        last = last || grid <= round;
    }
    if (grid > 0x7fffffff || lds > 160 * 1024) return hipErrorInvalidValue;
    L.first[L.naxes] = (int)grid;
    auto kern = fractional_far<NW>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * NW), lds, s, L);
    return hipGetLastError();
}

}  // namespace

bool far_reaches(const AxisLayout& lay, int n)
{
    return lay.contiguous || (int64_t)n * lay.j_stride < ((int64_t)1 << 29);
}

bool far_used(int n)
{
    // Upper end: the longest axis this was measured on, and the one up to which
    // the third plane of the weights is made (kThirdPlaneMax); the moments of 32
    // lines (16 BF16 triples per 128 nodes and line) fill the LDS at 4288 nodes.
    // Longer axes are summed densely, as they were: 4097^2 costs 10 times 4096^2.
    // Lower end: there the band and the two box steps cost as much as the dense
    // sum (FP32, far / dense, us: 640^2 16.4 / 12.9, 768^2 17.9 / 18.5, 896 x 900
    // 18.4 / 24.2, 1024^2 19.3 / 26.0).
    return n > 768 && n <= 4096;
}

size_t far_table_entries(int n) { return (size_t)((n + kBox - 1) / kBox + far_sources(n) - 1) * 3 * kRank * kRank; }

// U fragments [half][block][plane][lane][8] (lane: output 64 half + 32 block +
// lane % 32, p = 8 (lane / 32) + e), then V fragments [step][plane][lane][8]
// (lane: p = lane % 16, k = 32 step + 8 (lane / 16) + e); both hold l_p at
// node (x - 63.5) / 64 of a box.
void far_uv_fill(uint16_t* out, uint16_t (*to_bf16)(double), float (*to_float)(uint16_t))
{
    auto put = [&](size_t base, int lane, int e, double v) {
        for (int pl = 0; pl < 3; ++pl) {
            const uint16_t b = to_bf16(v);
            out[base + (size_t)(pl * 64 + lane) * 8 + e] = b;
            v -= (double)to_float(b);
        }
    };
    std::vector<double> tab(kBox * kRank);
    for (int x = 0; x < kBox; ++x)
        for (int p = 0; p < kRank; ++p) tab[x * kRank + p] = lagrange(p, (x - 63.5) / 64.0);
    for (int hc = 0; hc < 4; ++hc)
        for (int lane = 0; lane < 64; ++lane)
            for (int e = 0; e < 8; ++e)
                put((size_t)hc * 3 * 64 * 8, lane, e, tab[(32 * hc + lane % 32) * kRank + 8 * (lane / 32) + e]);
    for (int ks = 0; ks < 4; ++ks)
        for (int lane = 0; lane < 64; ++lane)
            for (int e = 0; e < 8; ++e)
                put(6144 + (size_t)ks * 3 * 64 * 8, lane, e, tab[(32 * ks + 8 * (lane / 16) + e) * kRank + lane % 16]);
}

hipError_t launch_far_tables(const AxisData* ops, int nops, hipStream_t s)
{
    FarTables F = {};
    int k = 0, blocks = 0;
    for (int a = 0; a < nops; ++a) {
        const AxisData& op = ops[a];
        if (!op.far_m) continue;
        F.first[k] = blocks;
        F.nsp[k] = far_sources(op.n);
        F.g[k] = op.far_g;
        F.pos[k] = op.far_pos;
        F.neg[k] = op.far_neg;
        F.out[k] = const_cast<uint16_t*>(op.far_m);
        blocks += (op.n + kBox - 1) / kBox + F.nsp[k] - 1;
        ++k;
    }
    if (!k) return hipSuccess;
    for (; k < 4; ++k) F.first[k] = blocks;
    hipLaunchKernelGGL(far_table, dim3(blocks), dim3(256), 0, s, F);
    return hipGetLastError();
}

hipError_t launch_fractional_far(SplitLaunch& L, hipStream_t s)
{
    int nmax = 0;
    for (int a = 0; a < L.naxes; ++a) nmax = L.op[a].n > nmax ? L.op[a].n : nmax;
    // 8 wavefronts per workgroup share the moments of a long line; up to 1024
    // nodes smaller workgroups give more of them (1024^2 20.9 us against 22.9;
    // 1280^2 28.4 against 25.0)
    return nmax <= 1024 ? run_far<4>(L, s) : run_far<8>(L, s);
}

}  // namespace lbm

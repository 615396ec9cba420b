// lbm_internal.h -- structures shared by the host runtime (lbm_fade.hip) and
// the kernel launchers (fractional_gemm.hip, collide_stream.hip, adjoint.hip).
// Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lbm {

constexpr int kMaxQ = 7;

// Device-side description of the fractional operator along one axis
// (Sec. 2.4), with T and the boundary values pre-multiplied by
// g dx^gamma / Gamma(2 + gamma) and by p (lower part) / (1 - p) (upper part):
//   ends_excluded = 1 (the forward operators):
//     Phi[j] = sum_{0 < k < N} T(j - k) C[k] + col0[j] C[0] + colN[j] C[N],
//     col0 / colN the whole boundary columns K[j][0], K[j][N];
//   ends_excluded = 0 (the adjoint's transposed parts):
//     Phi[j] = sum_{0 <= k <= N} T(j - k) C[k] + col0[j] C[0] + colN[j] C[N].
struct AxisOp {
    int n;               // nodes on the axis, N = n - 1
    int lower_only;      // p == 1: T(d) = 0 for d < 0
    int upper_only;      // p == 0: T(d) = 0 for d > 0
    int ends_excluded;   // see above
    const float* gen;    // T(d) at gen[d + n - 1], d in [-(n-1), n-1]
    const float* col0;  // n values
    const float* colN;  // n values
    const uint16_t* gen_hi;  // BF16 bits of T split hi/lo (same indexing)
    const uint16_t* gen_lo;
    // Pair words of the split, W(d) = b(d) | b(d - 1) << 16 with b = hi or lo
    // bits (0 for |d| > n - 1), stored with d decreasing: pw[x] = W(pw_top - x)
    // for x in [0, pw_top + n + 288).  pw_top = 16 ceil((n + 512) / 16) - 1.
    const uint32_t* pw_hi;
    const uint32_t* pw_lo;
    int pw_top;
};

// Everything the library holds of one axis' operator (host side; a kernel gets
// the part it reads, AxisOp or SplitOp, by value).
struct AxisData : AxisOp {
    // The third plane of T = hi + lo + l3 (indexed as the other two), for the
    // FP32 products formed from exact three-term splits; null on axes beyond
    // kThirdPlaneMax.
    const uint32_t* pw_l3;
    // Far part of a long axis (fractional_far.hip; null where it is not used):
    // operators between boxes, and the interpolation fragments.  T(d) at a
    // distance |d| >= 64 is far_pos a(d) for d > 0, far_neg a(-d) for d < 0,
    // a the product-rule weights of gamma = far_g.
    const uint16_t* far_m;
    const uint16_t* far_uv;
    double far_g, far_pos, far_neg;
};

// Source boxes of 128 nodes of an axis of n nodes (the first starts at -64),
// rounded up to an even number.
__host__ __device__ inline int far_sources(int n) { return ((n + 64 + 127) / 128 + 1) & ~1; }
constexpr size_t kFarUvEntries = 12288;  // BF16 values of the interpolation fragments

constexpr int kThirdPlaneMax = 4096;

// Top index and length of the pair-word arrays of an axis of n nodes.
inline int pw_top_of(int n) { return 16 * ((n + 512 + 15) / 16) - 1; }
inline int64_t pw_len_of(int n) { return (int64_t)pw_top_of(n) + n + 288; }

// Workgroup barrier that orders LDS accesses only (release/acquire fences
// scoped to LDS): global loads in flight stay in flight, unlike
// __syncthreads(), which also waits for them.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Strided view of a node field for the operator along one axis.
//   contiguous axis (x): line l, node j  ->  l * n + j
//   other axes: batch b, node j, line l  ->  b * batch_stride + j * j_stride + l
struct AxisLayout {
    int contiguous;        // 1 for the x axis
    int64_t lines;         // lines per batch (contiguous axis: all lines)
    int64_t j_stride;      // stride of the axis index (strided case)
    int64_t batch_stride;  // strided case
    int batches;           // strided case
};

// One launch of the fractional term for all axes of a step, or for several
// operators at once (the adjoint applies two per axis): workgroup ids are split
// into per-operator ranges, in order.
constexpr int kMaxOps = 6;
struct FracLaunch {
    AxisOp op[kMaxOps];
    AxisLayout lay[kMaxOps];
    int tiles_m[kMaxOps], tiles_n[kMaxOps];
    int first[kMaxOps + 1];  // first workgroup id of every operator, first[naxes] = grid size
    const float* C[kMaxOps];  // input field of every operator
    float* Phi[kMaxOps];
    int naxes;  // operators in this launch
    int lgroup;  // one-sided operators: line tiles per group of the tile order (0 = all of an XCD's)
};

// The same for the kernels on three-term splits (fractional_split.hip,
// fractional_far.hip): the axes of one step, and of an operator what they read.
// Whole cache lines: the operator of a workgroup is loaded by its index, and
// across lines 1 % of short launches is lost (split BF16 1024 x 24 x 24 17.35 us
// packed, 17.15 so).
struct alignas(64) SplitOp {
    int n, lower_only, upper_only, ends_excluded;
    const float *gen, *col0, *colN;
    const uint32_t *pw_hi, *pw_lo, *pw_l3;
    const uint16_t *far_m, *far_uv;
    int pw_top;
};
struct SplitLaunch {
    SplitOp op[3];
    AxisLayout lay[3];
    int tiles_m[3], tiles_n[3];
    int first[4];
    const float* C[3];
    float* Phi[3];
    int naxes;
};

// Constants of the fused collide-stream kernel (Sec. 2.2-2.5).
struct CollideConsts {
    int dim, Q;
    int n[3];
    float w[kMaxQ];         // lattice weights
    float adv[3];           // (dt/dx) u_mu w / e^2: f^eq_{2mu+1} += adv C, f^eq_{2mu+2} -= adv C
    float R[kMaxQ * kMaxQ]; // M^-1 Lambda M (BGK: I / lambda), row-major
    float wSdt[kMaxQ];      // w_i dt (multiplies S)
    float c_wall;
    // Collision in moments (every free relaxation time is 1): H = (Id -
    // lambda-bar^-1) / 2, d x d row-major, and the time step.
    int moments;
    float H[9];
    float dt;
    // Space-dependent coefficients (both null, or both set):
    //   dB: d(d+1)/2 node fields, the upper triangle (row by row) of
    //       lambda-bar(x)^-1 - lambda-bar^-1, added to the flux block of Lambda;
    //   Cw: one node field, the Dirichlet value of every wall node.
    const float* dB;
    const float* Cw;
};

// Kernel launchers (host functions).  All return a hipError_t.
// Fractional term of all axes: axis a reads C + a * in_stride (in_stride = 0:
// one field for every axis) and writes Phi + a * nodes.  register_kernels: every
// axis on the register kernels.
hipError_t launch_fractional(const AxisData* ops, const AxisLayout* lays, int naxes, int precision,
                             bool register_kernels, const float* C, int64_t in_stride, float* Phi, int64_t nodes,
                             hipStream_t s);
// FP32 only: nops (<= kMaxOps) operators with their own layouts, inputs and
// outputs, in one launch of a register kernel.
hipError_t launch_fractional_ops(const AxisOp* ops, const AxisLayout* lays, const float* const* C, float* const* Phi,
                                 int nops, hipStream_t s);
// Places of several buffers in one allocation.  An allocation and its release
// cost 50 to 100 us each whatever their size, and a program that makes a handle
// per call (fade_solve) pays them every time (512^2, 100 steps and gradients:
// 9.8 ms with 28 allocations, 8.0 with 6).  32 KiB + 256 bytes lie between two
// buffers: side by side, fields of a power of two of bytes meet in the same
// memory channels (512^2, us a step, close / apart: operator 14.70 / 14.28, with a
// space-dependent tensor 16.1 / 15.4; in allocations of their own 14.46, 15.2).
struct Slab {
    size_t bytes = 0;
    size_t take(size_t n)  // offset of the next n bytes
    {
        const size_t at = bytes;
        bytes += ((n + 4095) & ~(size_t)4095) + (32 << 10) + 256;
        return at;
    }
};

// One step's collision, streaming and walls.  The state read and written is
// the populations and C (C_in is read only where cc.moments, and must not be
// C_out then), or, inside a run of steps where moment_runs(), the 1 + d fields
// C, j_0, .. of the collision in moments (consecutive node fields in the same
// buffers; C_in is not read then, C_out not written).
enum class StepState { populations, to_moments, moments, to_populations };
bool moment_runs(const CollideConsts& cc);
hipError_t launch_collide_stream(const CollideConsts& cc, const float* f_in, const float* C_in, float* f_out,
                                 const float* Phi, const float* S, float* C_out, hipStream_t s,
                                 StepState state = StepState::populations);
// f := f^eq(C, Phi), C := <1|f>
hipError_t launch_equilibrium_init(const CollideConsts& cc, float* C, const float* Phi, float* f, hipStream_t s);
hipError_t launch_wall_overwrite(const CollideConsts& cc, float* C, hipStream_t s);
hipError_t launch_fill(float* p, int64_t count, float v, hipStream_t s);
hipError_t launch_moment(const CollideConsts& cc, const float* f, float* C, hipStream_t s);
hipError_t launch_nonfinite_check(const float* C, int64_t nodes, int* flag, hipStream_t s);
bool have_bf16x3();
// Records msg as the calling thread's last error (lbm_fade_last_error) and returns code.
int set_error(int code, const char* msg);
// Output tiles of 128 x 128 over all axes (sizes the GEMM launch).
int64_t big_tiles(const FracLaunch& L);
// Tile configuration forced through an environment variable (0 = automatic).
int tile_choice(const char* var);
hipError_t launch_fractional_bf16x3(FracLaunch& L, hipStream_t s);
// Dense kernel on the BF16 matrix cores; terms: BF16 products per FP32 product
// (6), or of LBM_BF16X3 (3).  split_takes: the launches it is used for.
bool split_takes(const SplitLaunch& L, int dim, int terms);
hipError_t launch_fractional_split(SplitLaunch& L, int terms, hipStream_t s);
// Long axes (every operator needs its far_m table): near band plus moments of
// far boxes, LBM_FP32.  far_used: axis lengths that take this path.  launch_far_tables fills far_m.
// far_reaches: the kernel's 32-bit byte offsets span the axis.
bool far_used(int n);
bool far_reaches(const AxisLayout& lay, int n);
size_t far_table_entries(int n);
void far_uv_fill(uint16_t* out, uint16_t (*to_bf16)(double), float (*to_float)(uint16_t));
hipError_t launch_far_tables(const AxisData* ops, int nops, hipStream_t s);
hipError_t launch_fractional_far(SplitLaunch& L, hipStream_t s);

}  // namespace lbm

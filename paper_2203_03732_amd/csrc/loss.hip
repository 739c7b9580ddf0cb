// Matching-based OT loss of a batch and its gradient.
//
// For instance i with matching mate_b (row b -> column a), the loss is
//   L_i = (1/n_i) * sum_b ||x_b - y_mate(b)||^2,
// the cost of the plan P = (1/n_i) * permutation that the push-relabel solve
// returns (arXiv:2203.03732 motivates using the plan in learning, Section 1).
// The plan is piecewise constant in X and Y, so for an upstream gradient g_i
//   dL/dx_b = (2 g_i / n_i) (x_b - y_mate(b)),
//   dL/dy_a = (2 g_i / n_i) (y_a - x_mate^-1(a)),
// and 0 for vertices the plan leaves unmatched.
#include <algorithm>
#include <mutex>

#include "internal.h"

// Partial sums of prot_ot_loss_fwd_static: a fixed array of the library, one
// copy per device, so that the call allocates nothing. In host code its name
// is only a handle: kernels get the device address from static_loss_partials.
static __device__ __align__(256) double scratch[prot::kStaticLossParts];

namespace prot {
namespace {

constexpr int kLossThreads = 256;
constexpr int kFwdThreads = 1024;
constexpr int kFwdUnroll = 8;
constexpr int kBwdThreads = 512;
constexpr int kBwdRowsMin = 64, kBwdRowsMax = 1024;  // of a block of the one-pass backward
constexpr int kBwdCoords = 2048;                     // it takes about, or more where d is large
constexpr int kBwdFewBlocks = 1024;                  // together on the device
constexpr int64_t kBwdFewMaxN = 8192, kBwdFewMates = 1 << 22;

__device__ inline int64_t inst_n(const LossArgs &A, int inst)
{
    return A.n_arr ? (int64_t)A.n_arr[inst] : A.n_uniform;
}
__device__ inline int64_t inst_off(const LossArgs &A, int inst)
{
    return A.n_arr ? A.pt_off[inst] : (int64_t)inst * A.n_uniform;
}

// grid (parts, batch): block `part` of instance `inst` sums the squared
// differences of coordinates [part * per, (part + 1) * per) of the instance
// (row-major, so consecutive lanes read consecutive floats, kFwdUnroll
// loads in flight per thread), each thread in ascending order in binary64,
// then a fixed-order block reduction into partial[inst * parts + part].
// Bound: the latency of the mates' and then the coordinates' loads, so a block
// takes its ~8,192 coordinates in one step, and a thread walks from one
// coordinate to its next by row and column steps (a 64-bit division each
// costs more than the loads' issue): 33 x 1,531 x 37 20 -> 6.9 us.
__global__ void __launch_bounds__(kFwdThreads)
ot_loss_part_kernel(LossArgs A, double *partial)
{
    __shared__ double red[kFwdThreads];
    const int inst = blockIdx.y, parts = gridDim.x;
    const int64_t n = inst_n(A, inst), off = inst_off(A, inst);
    const int d = A.d;
    const float *X = A.X + off * d, *Y = A.Y + off * d;
    const int32_t *mb = A.mate_b + off;
    const int64_t total = n * d;
    const int64_t per = (total + parts - 1) / parts;
    const int64_t lo = min(total, (int64_t)blockIdx.x * per), hi = min(total, lo + per);
    double s = 0.0;
    // coordinate e = b * d + j of this thread, and the step to its next
    const int64_t e_first = lo + threadIdx.x;
    int64_t b = e_first / d;
    int32_t j = (int32_t)(e_first - b * d);
    const int32_t step_b = kFwdThreads / d, step_j = kFwdThreads % d;
    for (int64_t e0 = e_first; e0 < hi; e0 += (int64_t)kFwdUnroll * kFwdThreads) {
        float x[kFwdUnroll], y[kFwdUnroll];
        int32_t at[kFwdUnroll], col[kFwdUnroll];
#pragma unroll
        for (int u = 0; u < kFwdUnroll; ++u) {
            at[u] = e0 + (int64_t)u * kFwdThreads < hi ? mb[b] : -1;
            col[u] = j;
            b += step_b;
            j += step_j;
            if (j >= d) {
                j -= d;
                b += 1;
            }
        }
#pragma unroll
        for (int u = 0; u < kFwdUnroll; ++u) {
            x[u] = y[u] = 0.0f;
            if (at[u] >= 0 && at[u] < n) {
                x[u] = X[e0 + (int64_t)u * kFwdThreads];
                y[u] = Y[(int64_t)at[u] * d + col[u]];
            }
        }
        // (a pair that is not summed has x = y = 0 and adds exactly nothing)
#pragma unroll
        for (int u = 0; u < kFwdUnroll; ++u) {
            const double t = __dsub_rn((double)x[u], (double)y[u]);
            s = __dadd_rn(s, __dmul_rn(t, t));
        }
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = kFwdThreads / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] = __dadd_rn(red[threadIdx.x], red[threadIdx.x + o]);
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[(int64_t)inst * parts + blockIdx.x] = red[0];
}

// One thread per instance: the partial sums in part order, divided by n.
__global__ void ot_loss_sum_kernel(LossArgs A, const double *partial, int parts, float *loss)
{
    const int inst = blockIdx.x * blockDim.x + threadIdx.x;
    if (inst >= A.batch) return;
    double s = 0.0;
    for (int q = 0; q < parts; ++q) s = __dadd_rn(s, partial[(int64_t)inst * parts + q]);
    const int64_t n = inst_n(A, inst);
    loss[inst] = n > 0 ? (float)(s / (double)n) : 0.0f;
}

// grid.y = instance, grid.x over the instance's n * d coordinates.
__global__ void __launch_bounds__(kLossThreads)
ot_loss_bwd_kernel(LossArgs A, const float *grad_loss, float *dX, float *dY)
{
    const int inst = blockIdx.y;
    const int64_t n = inst_n(A, inst), off = inst_off(A, inst);
    const int d = A.d;
    const int64_t e = (int64_t)blockIdx.x * kLossThreads + threadIdx.x;
    if (e >= n * d) return;
    const int64_t v = e / d;
    const int j = (int)(e - v * d);
    const float scale = 2.0f * grad_loss[inst] / (float)n;
    const float *X = A.X + off * d, *Y = A.Y + off * d;
    const int32_t a = A.mate_b[off + v];
    const int32_t b = A.mate_a[off + v];
    dX[off * d + e] = a >= 0 && a < n ? scale * (X[e] - Y[(int64_t)a * d + j]) : 0.0f;
    dY[off * d + e] = b >= 0 && b < n ? scale * (Y[e] - X[(int64_t)b * d + j]) : 0.0f;
}

// Without mate_a: every coordinate of dY starts at 0 (a column no row
// holds keeps it), then each matched row b writes dX_b and the coordinates
// of its column's dY (a matching gives each column at most one row).
__global__ void fill_zero_kernel(float *p, int64_t count)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.0f;
}

// The same in one pass: a block takes `rows` rows and the columns of the same
// indices; it reads the instance's mates (from the L2) to find which rows hold
// its columns, so that every coordinate of dX and dY is written once, by the
// thread that computes it, and nothing is filled first.
// Bound: the latency of the mates' and then the coordinates' loads, 30 MB of
// coordinates at 33 x 1,531 x 37: 13.7 us for the fill and the scatter, 11.2
// so (13.0 with blocks of 32 rows and 256 threads).
__global__ void __launch_bounds__(kBwdThreads)
ot_loss_bwd_one_pass_kernel(LossArgs A, const float *grad_loss, float *dX, float *dY, int rows)
{
    __shared__ int32_t row_col[kBwdRowsMax], col_row[kBwdRowsMax];
    const int inst = blockIdx.y;
    const int n = (int)inst_n(A, inst), d = A.d;
    const int v0 = (int)blockIdx.x * rows;
    if (v0 >= n) return;
    const int cnt = min(rows, n - v0);
    const int64_t off = inst_off(A, inst);
    const int32_t *mb = A.mate_b + off;
    for (int v = threadIdx.x; v < cnt; v += kBwdThreads) {
        col_row[v] = -1;
        row_col[v] = mb[v0 + v];
    }
    __syncthreads();
#pragma unroll 8
    for (int b = threadIdx.x; b < n; b += kBwdThreads) {
        const int32_t a = mb[b];
        if (a >= v0 && a < v0 + cnt) col_row[a - v0] = b;
    }
    __syncthreads();
    const float scale = 2.0f * grad_loss[inst] / (float)n;
    const float *X = A.X + off * d, *Y = A.Y + off * d;
    float *gX = dX + off * d, *gY = dY + off * d;
    const uint32_t ud = (uint32_t)d;
#pragma unroll 4
    for (uint32_t i = threadIdx.x; i < (uint32_t)cnt * ud; i += kBwdThreads) {
        const uint32_t v = i / ud, c = i - v * ud;
        const int32_t a = row_col[v], b = col_row[v];
        const int64_t e = (int64_t)v0 * d + i;
        gX[e] = a >= 0 && a < n ? scale * (X[e] - Y[(int64_t)a * d + c]) : 0.0f;
        gY[e] = b >= 0 ? -(scale * (X[(int64_t)b * d + c] - Y[e])) : 0.0f;
    }
}

__global__ void __launch_bounds__(kLossThreads)
ot_loss_bwd_rows_kernel(LossArgs A, const float *grad_loss, float *dX, float *dY)
{
    const int inst = blockIdx.y;
    const int64_t n = inst_n(A, inst), off = inst_off(A, inst);
    const int d = A.d;
    const int64_t e = (int64_t)blockIdx.x * kLossThreads + threadIdx.x;
    if (e >= n * d) return;
    const int64_t v = e / d;
    const int j = (int)(e - v * d);
    const float scale = 2.0f * grad_loss[inst] / (float)n;
    const float *X = A.X + off * d, *Y = A.Y + off * d;
    const int32_t a = A.mate_b[off + v];
    if (a >= 0 && a < n) {
        const float diff = X[e] - Y[(int64_t)a * d + j];
        dX[off * d + e] = scale * diff;
        dY[(off + a) * d + j] = -(scale * diff);
    } else {
        dX[off * d + e] = 0.0f;
    }
}

}  // namespace

int loss_parts(int64_t n_max, int32_t d)
{
    // about 8192 coordinates per block, at most 64 blocks per instance
    const int64_t p = (n_max * d + 8191) / 8192;
    return (int)(p < 1 ? 1 : (p > 64 ? 64 : p));
}

hipError_t launch_loss_fwd(const LossArgs &a, int64_t n_max, double *partial, float *loss,
                           hipStream_t s)
{
    if (a.batch > 0) {
        const int parts = loss_parts(n_max, a.d);
        hipLaunchKernelGGL(ot_loss_part_kernel, dim3((unsigned)parts, (unsigned)a.batch),
                           dim3(kFwdThreads), 0, s, a, partial);
        hipLaunchKernelGGL(ot_loss_sum_kernel, dim3((unsigned)((a.batch + 255) / 256)), dim3(256),
                           0, s, a, (const double *)partial, parts, loss);
    }
    return hipGetLastError();
}

// Device address of this device's copy of `scratch` (the device current on
// the calling thread), looked up once per device.
hipError_t static_loss_partials(double **out)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static double *ptr[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        ptr[dev] = static_cast<double *>(p);
    }
    *out = ptr[dev];
    return hipSuccess;
}

hipError_t launch_loss_bwd(const LossArgs &a, int64_t n_max, const float *grad_loss, float *dX,
                           float *dY, hipStream_t s)
{
    if (a.batch > 0) {
        const int64_t blocks = (n_max * a.d + kLossThreads - 1) / kLossThreads;
        // The one-pass backward reads n mates per `rows` rows, and a block of
        // it has three steps that wait: it is taken where a block's coordinates
        // outweigh its mates and fill its threads, or where all blocks run at
        // once and read few mates, so that one launch instead of two counts.
        // Fill and scatter / one pass, in us: 2^20 rows in all, d = 64, n = 64
        // 326 / 268, 4,096 336 / 323, 8,192 (not taken) 343 / 373; n = 256, d = 4
        // 30.2 / 17.6; n = 64, d = 4 (not taken) 22.6 / 29.6; one instance of
        // 64 to 8,192 points 14.5 / 11.3; 128 of 8,192 x 1 (not taken) 17.7 / 21.5.
        int rows = kBwdRowsMin;
        while (rows < kBwdRowsMax && (int64_t)rows * a.d < kBwdCoords) rows *= 2;
        const int64_t pass_blocks = (n_max + rows - 1) / rows;
        const bool one_pass = (int64_t)rows * a.d < (int64_t)1 << 31 &&
                              ((n_max <= kBwdFewMaxN && pass_blocks * a.batch <= kBwdFewBlocks &&
                                pass_blocks * a.batch * n_max <= kBwdFewMates) ||
                               (n_max <= (int64_t)rows * a.d && n_max * a.d >= kBwdThreads));
        if (a.mate_a) {
            hipLaunchKernelGGL(ot_loss_bwd_kernel, dim3((unsigned)blocks, (unsigned)a.batch),
                               dim3(kLossThreads), 0, s, a, grad_loss, dX, dY);
        } else if (one_pass) {
            hipLaunchKernelGGL(ot_loss_bwd_one_pass_kernel,
                               dim3((unsigned)pass_blocks, (unsigned)a.batch), dim3(kBwdThreads),
                               0, s, a, grad_loss, dX, dY, rows);
        } else {
            const int64_t count = (int64_t)a.batch * n_max * a.d;  // uniform n
            const int64_t g = std::min<int64_t>((count + 255) / 256, 65536);
            hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)g), dim3(256), 0, s, dY, count);
            hipLaunchKernelGGL(ot_loss_bwd_rows_kernel, dim3((unsigned)blocks, (unsigned)a.batch),
                               dim3(kLossThreads), 0, s, a, grad_loss, dX, dY);
        }
    }
    return hipGetLastError();
}

}  // namespace prot

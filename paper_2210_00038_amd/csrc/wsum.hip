// Weighted sum of stored per-sample gradients (App. B.5), BK-MixOpt's
// clipped gradient on the layers that instantiate:
//   G[e] = sum_i C[i] P[i n + e],  one float32 fused multiply-add per sample in
// a fixed order (deterministic); with accum the sum is added to G.
// One launch covers a group of layers; each thread owns 4 consecutive
// elements (16-byte loads when the layer's buffers allow) and streams their
// per-sample values, eight rows of loads in flight.  HBM-bound: (B + 1) * 4
// bytes per element.  Long vectors (BK-MixOpt weights): one thread adds all
// samples, ascending.  Short ones over many samples (biases, affines) would
// leave a serial chain of B loads on few CUs (n = 1000, B = 1024: 268 us for
// three layers): there 16 threads add every 16th sample each and their sums
// are added in order (14 us; the 97 bias and affine vectors of GPT-2 small at
// B = 32 19 -> 9 us).
#include "bk_device.h"
#include "bk_kernels.h"

namespace bk {
namespace {

__global__ __launch_bounds__(256) void wsum_kernel(const WsumArgs args) {
    __shared__ float4 sums[kWsumRuns][16];
    const uint32_t wg = blockIdx.x;
    const int l = find_desc(args.n, (int64_t)wg, [&](int k) { return args.L[k].wg_begin; });
    const WsumLayer& L = args.L[l];
    const int64_t n = L.n;
    const int run = (int)L.run;                       // 1 or kWsumRuns
    const int q = run == 1 ? 0 : (int)threadIdx.x >> 4;         // first sample
    const int col = run == 1 ? (int)threadIdx.x : (int)threadIdx.x & 15;
    const int64_t e0 = (int64_t)(wg - L.wg_begin) * (kWsumPerWG / run) + 4 * (int64_t)col;
    const int B = args.B;
    const int m = (int)max<int64_t>(0, min<int64_t>(4, n - e0));   // elements of this thread
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    // Samples q, q + run, ... in ascending order, eight rows of loads at once.
    for (int i0 = q; i0 < B; i0 += 8 * run) {
        float c[8], v[8][4];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * run;
            c[u] = i < B ? args.C[i] : 0.f;
            const float* row = L.P + (size_t)min(i, B - 1) * n + e0;
            if (L.vec) {       // 4 | n: a thread's 4 elements are in range or none is
                if (m > 0) {
                    const float4 w = *reinterpret_cast<const float4*>(row);
                    v[u][0] = w.x;
                    v[u][1] = w.y;
                    v[u][2] = w.z;
                    v[u][3] = w.w;
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (j < m) v[u][j] = row[j];
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (i0 + u * run < B) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (j < m) acc[j] = fmaf(c[u], v[u][j], acc[j]);
            }
    }
    if (run > 1) {
        sums[q][col] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        __syncthreads();
        if (q > 0) return;
#pragma unroll
        for (int k = 1; k < kWsumRuns; ++k) {
            const float4 w = sums[k][col];
            acc[0] += w.x;
            acc[1] += w.y;
            acc[2] += w.z;
            acc[3] += w.w;
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (j < m && L.accum) acc[j] += L.G[e0 + j];
    if (L.vec && m > 0) {
        *reinterpret_cast<float4*>(L.G + e0) = make_float4(acc[0], acc[1], acc[2], acc[3]);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j < m) L.G[e0 + j] = acc[j];
    }
}

}  // namespace

hipError_t launch_wsum(const WsumArgs& args, int n_wg, hipStream_t s) {
    if (n_wg <= 0) return hipSuccess;
    hipLaunchKernelGGL(wsum_kernel, dim3(n_wg), dim3(256), 0, s, args);
    return hipGetLastError();
}

}  // namespace bk

// gfx950 kernels for many right-hand sides sharing one 3-D operator, given and
// returned interleaved: the K values of a grid point are contiguous, element
// (x, y, z, k) at ((z n + y) n + x) K + k of the dense arrays.
//
// The solve itself runs on K separate padded grids with the kernels of the
// batched instances: an interleaved level needs five neighbour fields per
// thread and leaves no room in LDS for the fused stages (127^3, 32 right-hand
// sides, FP16: 1.65 ms per step interleaved, with smoothing, residual,
// restriction, prolongation and update as passes of their own).  The kernel
// here splits the columns on the way in, joins them on the way out, and forms
// the true residuals, for any set of the columns.
#include "mg_device.h"
#include "mg_launch.h"

#include <algorithm>

namespace mg {
namespace {

// Points of a workgroup's row segment times K: 32 KB of LDS in FP64.
constexpr int kColElems = 4096;
constexpr int kColThreads = 512;
constexpr int kColPer = kColElems / kColThreads;

// A workgroup takes one row y, a segment of S = 4096 / K points of it and a
// chunk of planes, marching z.  The interleaved values of a plane are read in
// memory order into LDS (rows of K + 1: the transposed reads are then free of
// bank conflicts) while the plane before is computed; wave w takes the runs of
// 64 points j = w, w + 8, ... (column j mod K, points 64 (j / K) ..), so the
// grids are read and written in runs of 512 bytes.  Each lane keeps U on planes
// z-1, z, z+1 in registers; the y neighbours are the rows of the workgroups
// beside it (dealt to the same XCD).  Bound by memory.
// The same roundings as the single-grid residual: b - (6 u - nb) / h^2 with nb
// summed in the order x, y, z.
template <bool HASU>
__global__ __launch_bounds__(kColThreads) void k_columns(const ColumnsArgs a, int lk, int nseg, int zc) {
    __shared__ double tile[kColElems + kColElems / 4];
    __shared__ double red[2 * 64];
    const int n = a.n, K = 1 << lk, P = n + 1;
    const size_t plane = (size_t)P * P;
    const int S = kColElems >> lk, KP = K + 1;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int t = xcd_block(blockIdx.x, gridDim.x);
    const int y = 1 + t % n, xs = (t / n) % nseg * S, len = min(S, n - xs);
    const int z0 = 1 + t / (n * nseg) * zc, z1 = min(z0 + zc, n + 1);
    const int cnt = len << lk;
    double ss[kColPer], mx[kColPer], um[kColPer], uc[kColPer], up[kColPer], bn[kColPer];
    // run e of this wave: column, first point, whether its r is formed
    auto col = [&](int e) { return (w + 8 * e) & (K - 1); };
    auto first = [&](int e) { return ((w + 8 * e) >> lk) * 64; };
    auto grid_at = [&](int e, int z) {
        return (size_t)col(e) * a.stride + ((size_t)z * P + y) * P + 1 + xs + first(e) + lane;
    };
    const bool rd = a.mask != 0;
    auto fetch = [&](int z) {
        const double *s = a.src + ((((size_t)(z - 1) * n + (y - 1)) * n + xs) << lk);
#pragma unroll
        for (int i = 0; i < kColPer; ++i) {
            const int f = threadIdx.x + i * kColThreads;
            bn[i] = f < cnt ? s[f] : 0.0;
        }
    };
#pragma unroll
    for (int e = 0; e < kColPer; ++e) {
        ss[e] = mx[e] = 0.0;
        if (HASU) {
            const bool in = first(e) + lane < len;
            um[e] = in ? a.U[grid_at(e, z0 - 1)] : 0.0;
            uc[e] = in ? a.U[grid_at(e, z0)] : 0.0;
        }
    }
    if (rd && z0 < z1) fetch(z0);
    for (int z = z0; z < z1; ++z) {
        if (rd) {
#pragma unroll
            for (int i = 0; i < kColPer; ++i) {
                const int f = threadIdx.x + i * kColThreads;
                if (f < cnt) tile[(f >> lk) * KP + (f & (K - 1))] = bn[i];
            }
            __syncthreads();
            if (z + 1 < z1) fetch(z + 1);
        }
#pragma unroll
        for (int e = 0; e < kColPer; ++e) {
            const int x = first(e) + lane;
            if (x >= len) continue;
            const size_t p = grid_at(e, z);
            if (HASU) up[e] = a.U[p + plane];  // plane n + 1 is a zero ghost
            if (!((a.mask >> col(e)) & 1)) continue;
            double r = tile[x * KP + col(e)];
            if (HASU) {
                double nb = a.U[p - 1] + a.U[p + 1];
                nb += a.U[p - P];
                nb += a.U[p + P];
                nb += um[e];
                nb += up[e];
                r = r - (6.0 * uc[e] - nb) * a.inv_h2;
            }
            if (a.R) a.R[p] = r;
            ss[e] += r * r;
            mx[e] = nanmax(mx[e], fabs(r));
        }
        if (HASU && a.out) {
            __syncthreads();
#pragma unroll
            for (int e = 0; e < kColPer; ++e) {
                const int x = first(e) + lane;
                if (x < len) tile[x * KP + col(e)] = uc[e];
            }
            __syncthreads();
            double *o = a.out + ((((size_t)(z - 1) * n + (y - 1)) * n + xs) << lk);
#pragma unroll
            for (int i = 0; i < kColPer; ++i) {
                const int f = threadIdx.x + i * kColThreads;
                if (f < cnt) o[f] = tile[(f >> lk) * KP + (f & (K - 1))];
            }
        }
        __syncthreads();
        if (HASU) {
#pragma unroll
            for (int e = 0; e < kColPer; ++e) um[e] = uc[e], uc[e] = up[e];
        }
    }
    if (!a.part || !rd) return;
    // run j = w + 8 e holds column j mod K
#pragma unroll
    for (int e = 0; e < kColPer; ++e) {
        wave_reduce(ss[e], mx[e]);
        if (lane == 0) {
            red[2 * (w + 8 * e)] = ss[e];
            red[2 * (w + 8 * e) + 1] = mx[e];
        }
    }
    __syncthreads();
    const int k = threadIdx.x;
    if (k < K && ((a.mask >> k) & 1)) {
        double s = 0.0, m = 0.0;
        for (int j = k; j < 64; j += K) {
            s += red[2 * j];
            m = nanmax(m, red[2 * j + 1]);
        }
        a.part[(size_t)k * a.pstride + 2 * (size_t)blockIdx.x] = s;
        a.part[(size_t)k * a.pstride + 2 * (size_t)blockIdx.x + 1] = m;
    }
}

// Planes per workgroup: about 2048 workgroups (four rounds of the chip).
struct ColShape {
    int lk, nseg, zc, blocks;
};
ColShape col_shape(int n, int K) {
    ColShape s{};
    while ((1 << s.lk) < K) ++s.lk;
    const int S = kColElems / K;
    s.nseg = (n + S - 1) / S;
    const int chunks = std::max(1, std::min(n, 2048 / (n * s.nseg)));
    s.zc = (n + chunks - 1) / chunks;
    s.blocks = n * s.nseg * ((n + s.zc - 1) / s.zc);
    return s;
}

}  // namespace

bool columns_ok(int prec, int K) { return K >= (prec == P_F64 ? 4 : 8) && K <= 64 && (K & (K - 1)) == 0; }

int columns_blocks(int n, int K) { return col_shape(n, K).blocks; }

hipError_t launch_columns(const ColumnsArgs &a, hipStream_t st) {
    if (a.K < 4 || a.K > 64 || (a.K & (a.K - 1)) || a.n < 3 || (a.mask && !a.src)) return hipErrorInvalidValue;
    const ColShape s = col_shape(a.n, a.K);
    if (a.U) hipLaunchKernelGGL(k_columns<true>, dim3(s.blocks), dim3(kColThreads), 0, st, a, s.lk, s.nseg, s.zc);
    else hipLaunchKernelGGL(k_columns<false>, dim3(s.blocks), dim3(kColThreads), 0, st, a, s.lk, s.nseg, s.zc);
    return hipGetLastError();
}

}  // namespace mg

// The coarse end of the V-cycle in one workgroup: every level from a small
// grid down to the base level (one point, or a few solved by CG) and back up,
// with all level vectors held in LDS.  On these levels a stage is a few
// thousand points, so as separate launches each costs launch latency (3.5-6 us
// on MI355X), not bandwidth; here it costs one pass over LDS and a barrier.
// A cycle whose finest level is that small runs as this one kernel alone.
//
// Work split.  A thread owns a segment of V consecutive x values of a level
// (K segments on the largest Q1 level) and keeps the segment's right-hand side
// and correction in registers from the first sweep to the residual, so a sweep
// costs the vector reads of its neighbour rows and one write.  Values sit in
// LDS in the accumulator format (they are values of the level's storage
// format: exact), which takes the conversions off every neighbour read.  The
// residual goes to the level's free correction buffer; the threads of the next
// level gather their full-weighting sums from it straight into registers, so a
// level costs nu1 + 1 barriers on the way down and nu2 + 1 on the way up.
//
// What bounds it: one CU's LDS and VALU issue on the largest level, barrier and
// LDS latency below.  Measured per launch: 3-D from 15^3 in FP16 14.8 us (33.7
// for the form that stored the level formats in LDS and walked single points),
// 2-D from 63^2 in FP64 17.5 us (21 level launches, 75 us), 3-D Q1 from 11^3
// with its 2^3 CG base 17.6 us (13 launches, 68 us).
//
// The arithmetic is the level kernels' own, operation for operation: the
// neighbour sum order (x-, x+, y-, y+, z-, z+; the Q1 sums of q1_weighted, or
// of the marching kernels on 3-D pitches that are multiples of 4), the
// explicit FMAs of the Jacobi sweep, the residual and full-weighting order of
// the restriction, the canonical interpolation sums, the dot products of the
// CG base solver, and a rounding to the level's storage format wherever a
// level kernel stores a value.  So a V-cycle with the fused end is bitwise the
// one without it.  The right-hand sides and corrections of the inner levels
// are also written to the workspace, where the level kernels leave them.
#include "mg_level_math.h"

#include <algorithm>
#include <type_traits>

namespace mg {
namespace {

constexpr int kThreads = 1024;

// Segments per thread and values per segment: finite differences have pitches
// that are multiples of 4; the Q1 pitches (c 2^j) are even.
template <int OP> struct TailSplit {
    static constexpr int V = OP ? 2 : 4, K = OP ? 2 : 1;
};

struct TailKArgs {
    const void *b0;          // right-hand side of the first level in its format (padded), or
    const double *R, *scal;  // ... the FP64 residual: b = round(R scal[1]), also written to wb[0]
    void *wb[kTailLevels + 1], *wc[kTailLevels + 1];  // workspace vectors of the levels and the base
    int off[kTailLevels + 1];  // LDS offset (elements of A) of a level's b, c0, c1
    int base_off;              // ... and, in doubles, of the base arrays
    unsigned precs;            // storage format of level l at bits 2l
    int pb, nb;                // base level: format, points per dimension
    int P0, nlev, nu1, nu2, nu2_first;
    double k;                  // Jacobi weight
    double tol;                // CG base
    int maxit;
    int zero16;                // LDS in use, in 16-byte chunks
};

__device__ __forceinline__ void mem_store1(void *m, int o, int p, double v) {
    if (p == P_F64) static_cast<double *>(m)[o] = v;
    else if (p == P_F32) static_cast<float *>(m)[o] = (float)v;
    else if (p == P_F16) static_cast<f16 *>(m)[o] = store_as<f16>(v);
    else static_cast<bf16 *>(m)[o] = store_as<bf16>(v);
}

// Elements of a level array in LDS: P + 1 planes (rows in 2-D), the row above
// plane P's first that the corner neighbours of the last point reach, and the
// element a segment's right neighbour reaches.
__host__ __device__ __forceinline__ int lds_elems(int D, int P) {
    return (D == 3 ? (P + 1) * P * P + P : (P + 1) * P) + 4;
}

// LDS rows
template <class A, int V> __device__ __forceinline__ void seg(const A *p, A (&v)[V]) { load_row<A, V>(p, v); }
template <class A, int V> __device__ __forceinline__ void put(A *p, const A (&v)[V]) { store_row<A, V>(p, v); }

// Segment s of a level of pitch P (P = TXR V): its first element sits at s V.
struct Item {
    int o, x0, y, z;
    bool on;  // an interior row
};
template <int D, int V> __device__ __forceinline__ Item item(int s, int P) {
    // s < 2^12 and P <= 64: the reciprocal product is exact after truncation
    Item t;
    const int TXR = P / V;
    const int row = (int)(((float)s + 0.5f) / (float)TXR);
    t.o = s * V;
    t.x0 = (s - row * TXR) * V;
    if (D == 3) {
        t.z = (int)(((float)row + 0.5f) / (float)P);
        t.y = row - t.z * P;
        t.on = t.z >= 1 && t.z < P && t.y >= 1;
    } else {
        t.z = row;
        t.y = 0;
        t.on = t.z >= 1 && t.z < P;
    }
    return t;
}

// lc = L c (finite differences) or S c (Q1) on a segment; cc holds its values.
template <int D, int OP, class A, int V>
__device__ __forceinline__ void apply(const A *c, const Item &t, int P, const A (&cc)[V], A (&lc)[V]) {
    const A *p = c + t.o;
    const bool first = t.x0 == 0;
    const int Z = D == 3 ? P * P : P;
    if constexpr (OP == 0) {
        A nb[V], w[V];
        const A xl = first ? A(0) : p[-1];
        const A xr = p[V];  // the zero ghost of the next row after the last segment
#pragma unroll
        for (int i = 0; i < V; ++i) nb[i] = (i > 0 ? cc[i - 1] : xl) + (i < V - 1 ? cc[i + 1] : xr);
        if constexpr (D == 3) {
            seg<A, V>(p - P, w);
#pragma unroll
            for (int i = 0; i < V; ++i) nb[i] += w[i];
            seg<A, V>(p + P, w);
#pragma unroll
            for (int i = 0; i < V; ++i) nb[i] += w[i];
        }
        seg<A, V>(p - Z, w);
#pragma unroll
        for (int i = 0; i < V; ++i) nb[i] += w[i];
        seg<A, V>(p + Z, w);
#pragma unroll
        for (int i = 0; i < V; ++i) nb[i] += w[i];
#pragma unroll
        for (int i = 0; i < V; ++i) lc[i] = fmaT<A>(A(2 * D), cc[i], -nb[i]);
    } else {
        // a row at x0 - 1 .. x0 + V
        auto row = [&](const A *q, A (&r)[V + 2]) {
            A m[V];
            seg<A, V>(q, m);
            r[0] = first ? A(0) : q[-1];
#pragma unroll
            for (int i = 0; i < V; ++i) r[i + 1] = m[i];
            r[V + 1] = q[V];
        };
        if constexpr (D == 2) {
            A s[V + 2], n[V + 2], m[V + 2];
            row(p - P, s);
            row(p, m);
            row(p + P, n);
#pragma unroll
            for (int i = 0; i < V; ++i) {
                const A nb = ((s[i] + s[i + 1]) + (s[i + 2] + m[i])) + ((m[i + 2] + n[i]) + (n[i + 1] + n[i + 2]));
                lc[i] = fmaT<A>(A(8), m[i + 1], -nb) * q1_scale<2, A>();
            }
        } else {
            A e[V], cn[V];
            A a[V + 2], b[V + 2], m[V + 2];
            row(p, m);
            if (P % 4 == 0) {
                // sums of rows y - 1 and y + 1 per plane, as the marching kernels
                A Am[V + 2], Cm[V + 2], Ap[V + 2], Cp[V + 2], A0[V + 2];
                row(p - Z, Cm);
                row(p - Z - P, a);
                row(p - Z + P, b);
#pragma unroll
                for (int i = 0; i < V + 2; ++i) Am[i] = a[i] + b[i];
                row(p + Z, Cp);
                row(p + Z - P, a);
                row(p + Z + P, b);
#pragma unroll
                for (int i = 0; i < V + 2; ++i) Ap[i] = a[i] + b[i];
                row(p - P, a);
                row(p + P, b);
#pragma unroll
                for (int i = 0; i < V + 2; ++i) A0[i] = a[i] + b[i];
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    const int k = i + 1;
                    e[i] = ((A0[k - 1] + A0[k + 1]) + ((Cm[k - 1] + Cm[k + 1]) + (Cp[k - 1] + Cp[k + 1]))) +
                           (Am[k] + Ap[k]);
                    cn[i] = (Am[k - 1] + Am[k + 1]) + (Ap[k - 1] + Ap[k + 1]);
                }
            } else {
                // the point-wise order (q1_weighted)
                A em[V], cm[V], w[V + 2];
                row(p - Z - P, a);
                row(p - Z, w);
                row(p - Z + P, b);
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    const int k = i + 1;
                    em[i] = (a[k] + w[k - 1]) + (w[k + 1] + b[k]);
                    cm[i] = (a[k - 1] + a[k + 1]) + (b[k - 1] + b[k + 1]);
                }
                row(p - P, a);
                row(p + P, b);
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    const int k = i + 1;
                    e[i] = em[i] + ((a[k - 1] + a[k + 1]) + (b[k - 1] + b[k + 1]));
                }
                row(p + Z - P, a);
                row(p + Z, w);
                row(p + Z + P, b);
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    const int k = i + 1;
                    e[i] = e[i] + ((a[k] + w[k - 1]) + (w[k + 1] + b[k]));
                    cn[i] = cm[i] + ((a[k - 1] + a[k + 1]) + (b[k - 1] + b[k + 1]));
                }
            }
#pragma unroll
            for (int i = 0; i < V; ++i)
                lc[i] = fmaT<A>(A(32), cc[i], -fmaT<A>(A(2), e[i], cn[i])) * q1_scale<3, A>();
        }
    }
}

// Full weighting of the fine residual r (pitch P) at coarse x X0 .. X0 + N - 1
// of row (Y, Z); values at X = 0 are not meaningful.
template <int D, int OP, class A, int N>
__device__ __forceinline__ void gather(const A *r, int X0, int Y, int Z, int P, A (&v)[N]) {
    const A *c = r + (D == 3 ? ((2 * Z) * P + 2 * Y) * P : 2 * Z * P) + 2 * X0;
    const int Zs = D == 3 ? P * P : P;
    auto row = [&](const A *q, A (&s)[N]) {
        A m[2 * N], h[N];
        seg<A, N>(q, h);  // two loads of a segment each: aligned on every pitch
#pragma unroll
        for (int j = 0; j < N; ++j) m[j] = h[j];
        seg<A, N>(q + N, h);
#pragma unroll
        for (int j = 0; j < N; ++j) m[N + j] = h[j];
        A left = q[-1];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            if (OP == 0) s[j] = A(0.25) * (left + m[2 * j + 1]) + A(0.5) * m[2 * j];
            else s[j] = (left + m[2 * j + 1]) + A(2) * m[2 * j];
            left = m[2 * j + 1];
        }
    };
    auto plane = [&](const A *q, A (&s)[N]) {
        if constexpr (D == 2) {
            row(q, s);
        } else {
            A a[N], b[N], d[N];
            row(q - P, a);
            row(q, b);
            row(q + P, d);
#pragma unroll
            for (int j = 0; j < N; ++j)
                s[j] = OP == 0 ? A(0.25) * (a[j] + d[j]) + A(0.5) * b[j] : (a[j] + d[j]) + A(2) * b[j];
        }
    };
    A a[N], b[N], d[N];
    plane(c - Zs, a);
    plane(c, b);
    plane(c + Zs, d);
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if (OP == 0) {
            A acc = A(0.25) * a[j];
            acc += A(0.5) * b[j];
            v[j] = acc + A(0.25) * d[j];
        } else {
            v[j] = ((a[j] + d[j]) + A(2) * b[j]) * (D == 3 ? A(1.0 / 64.0) : A(1.0 / 16.0));
        }
    }
}

// c + 4 P e on a segment, in W (e: coarse correction, pitch Pc, zero ghosts),
// rounded into format p.
template <int D, int OP, class A, class W, int V>
__device__ __forceinline__ void prolong(const A (&c)[V], const W *e, const Item &t, int Pc, int p, A (&out)[V]) {
    constexpr int H = V / 2;
    const int X0 = t.x0 >> 1;
    auto crow = [&](int Y, int Z, W (&v)[H + 1]) {
        const W *q = e + (D == 3 ? (Z * Pc + Y) * Pc : Z * Pc) + X0;
#pragma unroll
        for (int j = 0; j <= H; ++j) v[j] = q[j];
    };
    const int z0 = t.z >> 1, z1 = (t.z + 1) >> 1, y0 = t.y >> 1, y1 = (t.y + 1) >> 1;
    W S[H + 1];
    if constexpr (OP == 0) {
        const bool oz = t.z & 1, oy = D == 3 && (t.y & 1);
        W a[H + 1], b[H + 1];
        crow(y0, z0, S);
        crow(y0, z1, a);
#pragma unroll
        for (int j = 0; j <= H; ++j) S[j] = oz ? S[j] + a[j] : S[j];
        if constexpr (D == 3) {
            crow(y1, z0, a);
            crow(y1, z1, b);
#pragma unroll
            for (int j = 0; j <= H; ++j) {
                a[j] = oz ? a[j] + b[j] : a[j];
                S[j] = oy ? S[j] + a[j] : S[j];
            }
        }
        const W k0 = W(4) * (oz ? W(0.5) : W(1)) * (oy ? W(0.5) : W(1));
        const W k1 = W(0.5) * k0;
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const W q = (i & 1) ? S[i >> 1] + S[(i >> 1) + 1] : S[i >> 1];
            out[i] = rnd_w<A>((W)c[i] + ((i & 1) ? k1 : k0) * q, p);
        }
    } else {
        W a[H + 1], b[H + 1], d[H + 1];
        crow(y0, z0, S);
        if constexpr (D == 2) {
            crow(y0, z1, a);
#pragma unroll
            for (int j = 0; j <= H; ++j) S[j] = S[j] + a[j];
        } else {
            crow(y1, z0, a);
            crow(y0, z1, b);
            crow(y1, z1, d);
#pragma unroll
            for (int j = 0; j <= H; ++j) S[j] = (S[j] + a[j]) + (b[j] + d[j]);
        }
#pragma unroll
        for (int i = 0; i < V; ++i) {
            W s = S[i >> 1] + S[(i + 1) >> 1];
            s *= W(D == 3 ? 0.5 : 1.0);
            out[i] = rnd_w<A>((W)c[i] + s, p);
        }
    }
    if (t.x0 == 0) out[0] = A(0);
}

// Sum over the workgroup to every thread, in block_reduce's order (a wave64
// butterfly, then the waves in index order; absent waves add zero there).
// red: 16 doubles that no later sum reuses before a barrier.
__device__ __forceinline__ double wg_sum(double v, double *red) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    const int nw = blockDim.x >> 6;
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    for (int i = 0; i < nw; ++i) s += red[i];
    return s;
}

// CG on a base level of N <= blockDim.x points (k_cg_base, one point per
// thread: x, r, q in registers, p in LDS with zero ghosts); returns x.
template <int D, int OP, class AB>
__device__ __forceinline__ AB cg_point(AB bi, bool on, AB *p, int o, int P, double tol, int maxit, double *red) {
    const int Z = D == 3 ? P * P : P;
    AB x = AB(0), r = on ? bi : AB(0), pi = r;
    int slot = 0;
    auto sum = [&](double v) {
        const double s = wg_sum(v, red + 16 * slot);
        slot ^= 1;
        return s;
    };
    if (on) p[o] = pi;
    double rr = sum((double)r * (double)r);
    const double stop = tol * sqrt(rr);
    for (int k = 0; k < maxit && sqrt(rr) > stop; ++k) {
        // (the barrier of the last sum follows every write of p)
        AB q = AB(0);
        if (on) {
            if (OP == 1) {
                q = q1_weighted<D, AB>(p, (size_t)o, P) * q1_scale<D, AB>();
            } else {
                AB nb = p[o - 1] + p[o + 1];
                if (D == 3) {
                    nb += p[o - P];
                    nb += p[o + P];
                }
                nb += p[o - Z];
                nb += p[o + Z];
                q = fmaT<AB>(AB(2 * D), pi, -nb);
            }
        }
        const double pq = sum((double)pi * (double)q);
        if (!(pq > 0.0)) break;  // p = 0: the residual is already zero
        const AB a = (AB)(rr / pq);
        x = fmaT<AB>(a, pi, x);
        r = fmaT<AB>(-a, q, r);
        const double rr_new = sum((double)r * (double)r);
        const AB beta = (AB)(rr_new / rr);
        pi = fmaT<AB>(beta, pi, r);
        if (on) p[o] = pi;  // every thread read its neighbours before the last two barriers
        __syncthreads();
        rr = rr_new;
    }
    return x;
}

// Base level: right-hand side gathered from the fine residual r (pitch P),
// solved, the correction left in ec (W, zero ghosts) and in the workspace.
template <int D, int OP, class A, class AB, class W>
__device__ __forceinline__ void base_solve(const TailKArgs &a, const A *r, int P, AB *p, W *ec, double *red) {
    const int n = a.nb, Pb = P / 2, N = D == 3 ? n * n * n : n * n;
    const int i = (int)threadIdx.x;
    const bool on = i < N;
    int X = 1, Y = D == 3 ? 1 : 0, Z = 1;
    if (n > 1) {
        X = i % n + 1;
        Y = D == 3 ? (i / n) % n + 1 : 0;
        Z = D == 3 ? i / (n * n) + 1 : i / n + 1;
    }
    const int o = D == 3 ? (Z * Pb + Y) * Pb + X : Z * Pb + X;
    AB bv = AB(0);
    if (on) {
        A g[1];
        gather<D, OP, A, 1>(r, X, Y, Z, P, g);
        if constexpr (std::is_same<AB, double>::value) bv = a.pb == P_F64 ? (double)g[0] : (double)rnd64<float>(g[0], a.pb);
        else bv = rnd64<float>((double)g[0], a.pb);
        mem_store1(a.wb[a.nlev], o, a.pb, (double)bv);
    }
    AB x;
    if (n == 1) {
        x = OP ? bv * AB(0.375) : bv / AB(2 * D);
    } else {
        x = cg_point<D, OP, AB>(bv, on, p, o, Pb, a.tol, a.maxit, red);
    }
    if (on) {
        if constexpr (std::is_same<AB, float>::value) x = rnd(x, a.pb);
        ec[o] = (W)x;
        mem_store1(a.wc[a.nlev], o, a.pb, (double)x);
    }
}

template <int D, int OP, class A>
__global__ __launch_bounds__(kThreads) void k_tail(const TailKArgs a) {
    constexpr int V = TailSplit<OP>::V, K = TailSplit<OP>::K;
    extern __shared__ __align__(16) unsigned char smem[];
    A *lds = reinterpret_cast<A *>(smem);
    const A k = (A)a.k;
    const int tid = (int)threadIdx.x, nthr = (int)blockDim.x;
    Item it[K];
    A b[K][V], c[K][V];
    // the first level's right-hand side is on its way while LDS is cleared
    {
        const int p = (int)(a.precs & 3u);
#pragma unroll
        for (int q = 0; q < K; ++q) {
            it[q] = item<D, V>(tid + q * nthr, a.P0);
            if (!it[q].on) continue;
            if (a.R) {
                double r[V];
                load_row<double, V>(a.R + it[q].o, r);
                const double inv = a.scal[1];
#pragma unroll
                for (int i = 0; i < V; ++i) b[q][i] = rnd64<A>(r[i] * inv, p);
                if (it[q].x0 == 0) b[q][0] = A(0);
            } else {
                mem_load<A, V>(a.b0, it[q].o, p, b[q]);
            }
        }
    }
    for (int i = tid; i < a.zero16; i += nthr) reinterpret_cast<uint4 *>(smem)[i] = uint4{0u, 0u, 0u, 0u};
    __syncthreads();
    auto elems = [&](int P) { return lds_elems(D, P); };
    // down: pre-smoothing, residual, restriction
    for (int l = 0; l < a.nlev; ++l) {
        const int P = a.P0 >> l, E = elems(P), p = (int)(a.precs >> (2 * l)) & 3;
        A *const B = lds + a.off[l], *const C0 = B + E, *const C1 = C0 + E;
        if (l > 0) {
            const A *r = lds + a.off[l - 1] + elems(2 * P) * (1 + (a.nu1 & 1));
#pragma unroll
            for (int q = 0; q < K; ++q) {
                it[q] = item<D, V>(tid + q * nthr, P);
                if (!it[q].on) continue;
                gather<D, OP, A, V>(r, it[q].x0, it[q].y, it[q].z, 2 * P, b[q]);
#pragma unroll
                for (int i = 0; i < V; ++i) b[q][i] = rnd(b[q][i], p);
                if (it[q].x0 == 0) b[q][0] = A(0);
            }
        }
#pragma unroll
        for (int q = 0; q < K; ++q) {
            if (!it[q].on) continue;
            put<A, V>(B + it[q].o, b[q]);
            if (l > 0 || a.R) mem_store<A, V>(a.wb[l], it[q].o, p, b[q]);
#pragma unroll
            for (int i = 0; i < V; ++i) c[q][i] = rnd(k * b[q][i], p);
            put<A, V>(C0 + it[q].o, c[q]);
        }
        __syncthreads();
        // sweeps 1 .. nu1 - 1 and, last, the residual into the free buffer
        for (int s = 1; s <= a.nu1; ++s) {
            const A *src = (s & 1) ? C0 : C1;
            A *dst = (s & 1) ? C1 : C0;
            const bool res = s == a.nu1;
#pragma unroll
            for (int q = 0; q < K; ++q) {
                if (!it[q].on) continue;
                A lc[V], v[V];
                apply<D, OP, A, V>(src, it[q], P, c[q], lc);
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    const A r = b[q][i] - lc[i];
                    v[i] = res ? r : rnd(fmaT<A>(k, r, c[q][i]), p);
                }
                if (it[q].x0 == 0) v[0] = A(0);
                put<A, V>(dst + it[q].o, v);
#pragma unroll
                for (int i = 0; i < V; ++i) c[q][i] = v[i];
            }
            __syncthreads();
        }
    }
    // base level
    double *const base = reinterpret_cast<double *>(smem) + a.base_off;  // [32 sums][c][p]
    const int Pl = a.P0 >> (a.nlev - 1);
    const int Eb = elems(Pl / 2);
    const A *rl = lds + a.off[a.nlev - 1] + elems(Pl) * (1 + (a.nu1 & 1));
    double *const ecd = base + 32;
    A *const eca = reinterpret_cast<A *>(ecd);
    const bool wide = std::is_same<A, double>::value || a.pb == P_F64;  // interpolation from the base in FP64
    if (a.pb == P_F64) {
        base_solve<D, OP, A, double, double>(a, rl, Pl, ecd + Eb, ecd, base);
    } else {
        base_solve<D, OP, A, float, A>(a, rl, Pl, reinterpret_cast<float *>(ecd + Eb), eca, base);
    }
    __syncthreads();
    // up: prolongation, correction and post-smoothing.  The correction sits in
    // C0 after an odd number of pre-sweeps, else in C1.
    int cur = (a.nu1 & 1) ? 0 : 1;
    for (int l = a.nlev - 1; l >= 0; --l) {
        const int P = a.P0 >> l, E = elems(P), p = (int)(a.precs >> (2 * l)) & 3;
        A *const B = lds + a.off[l];
        auto C = [&](int j) { return B + (1 + j) * E; };
        const int nu2 = l == 0 ? a.nu2_first : a.nu2;
        int x = (a.nu1 & 1) ? 0 : 1;  // buffer of the current correction
        // the coarse correction: the base's, or the buffer its last sweep wrote
        const A *ec = l + 1 < a.nlev ? lds + a.off[l + 1] + elems(P / 2) * (1 + cur) : eca;
#pragma unroll
        for (int q = 0; q < K; ++q) {
            it[q] = item<D, V>(tid + q * nthr, P);
            if (!it[q].on) continue;
            A cv[V];
            seg<A, V>(C(x) + it[q].o, cv);
            seg<A, V>(B + it[q].o, b[q]);
            if (!std::is_same<A, double>::value && l + 1 == a.nlev && wide)
                prolong<D, OP, A, double, V>(cv, ecd, it[q], P / 2, p, c[q]);
            else
                prolong<D, OP, A, A, V>(cv, ec, it[q], P / 2, p, c[q]);
            put<A, V>(C(x ^ 1) + it[q].o, c[q]);
        }
        x ^= 1;
        __syncthreads();
        for (int s = 0; s < nu2; ++s) {
#pragma unroll
            for (int q = 0; q < K; ++q) {
                if (!it[q].on) continue;
                A lc[V], v[V];
                apply<D, OP, A, V>(C(x), it[q], P, c[q], lc);
#pragma unroll
                for (int i = 0; i < V; ++i) v[i] = rnd(fmaT<A>(k, b[q][i] - lc[i], c[q][i]), p);
                if (it[q].x0 == 0) v[0] = A(0);
                put<A, V>(C(x ^ 1) + it[q].o, v);
#pragma unroll
                for (int i = 0; i < V; ++i) c[q][i] = v[i];
            }
            x ^= 1;
            __syncthreads();
        }
        cur = x;
#pragma unroll
        for (int q = 0; q < K; ++q)
            if (it[q].on) mem_store<A, V>(a.wc[l], it[q].o, p, c[q]);
    }
}

// Launch plan: LDS offsets and sizes, and whether the levels fit.
struct Plan {
    TailKArgs k;
    size_t lds = 0;
    int threads = 0;
};

bool plan_tail(const TailArgs &t, Plan &q) {
    if (t.nlev < 1 || t.nlev > kTailLevels || (t.D != 2 && t.D != 3) || t.nu1 < 1 || t.nu2 < 1 || t.nu2_first < 1)
        return false;
    const int V = t.q1 ? 2 : 4, K = t.q1 ? 2 : 1;
    const bool f64 = t.prec[0] == P_F64;
    const size_t sa = f64 ? 8 : 4;
    TailKArgs &k = q.k;
    k = TailKArgs{};
    size_t off = 0;
    int segs0 = 0;
    for (int l = 0; l < t.nlev; ++l) {
        const int P = t.P0 >> l;
        if ((P << l) != t.P0 || P % V || P < 4 || P > 64) return false;
        if ((t.prec[l] == P_F64) != f64) return false;  // one accumulator format
        const int segs = (P / V) * P * (t.D == 3 ? P : 1);
        if (l == 0) segs0 = segs;
        k.off[l] = (int)(off / sa);
        off += 3 * (size_t)lds_elems(t.D, P) * sa;
        off = (off + 15) & ~(size_t)15;
        k.precs |= (unsigned)t.prec[l] << (2 * l);
    }
    const int Pl = t.P0 >> (t.nlev - 1), Pb = Pl / 2;
    if (Pl % 2 || t.nb != Pb - 1) return false;
    const int N = t.D == 3 ? t.nb * t.nb * t.nb : t.nb * t.nb;
    if (t.nb < 1 || N > kThreads || segs0 > K * kThreads) return false;
    k.base_off = (int)(off / 8);
    off += 8 * (32 + (size_t)lds_elems(t.D, Pb) * (t.nb > 1 ? 2 : 1));
    off = (off + 15) & ~(size_t)15;
    if (off > kLdsMax) return false;
    q.lds = off;
    q.threads = std::min(kThreads, std::max((segs0 + K - 1) / K, N));
    q.threads = (q.threads + 63) / 64 * 64;
    k.b0 = t.b0;
    k.R = t.R;
    k.scal = t.scal;
    for (int l = 0; l <= t.nlev; ++l) {
        k.wb[l] = t.wb[l];
        k.wc[l] = t.wc[l];
    }
    k.pb = t.prec[t.nlev];
    k.nb = t.nb;
    k.P0 = t.P0;
    k.nlev = t.nlev;
    k.nu1 = t.nu1;
    k.nu2 = t.nu2;
    k.nu2_first = t.nu2_first;
    k.k = t.q1 ? t.omega * 0.375 : t.omega / (2.0 * t.D);
    k.tol = t.base_tol;
    k.maxit = t.base_maxit;
    k.zero16 = (int)(off / 16);
    return true;
}

typedef void (*TailFn)(const TailKArgs);
TailFn tail_fn(int D, bool q1, bool f64) {
    if (D == 3) {
        if (q1) return f64 ? k_tail<3, 1, double> : k_tail<3, 1, float>;
        return f64 ? k_tail<3, 0, double> : k_tail<3, 0, float>;
    }
    if (q1) return f64 ? k_tail<2, 1, double> : k_tail<2, 1, float>;
    return f64 ? k_tail<2, 0, double> : k_tail<2, 0, float>;
}

}  // namespace

bool tail_ok(const TailArgs &t) {
    Plan q;
    return plan_tail(t, q);
}

hipError_t tail_prepare() {
    static hipError_t done = [] {
        for (int i = 0; i < 8; ++i) {
            const hipError_t e =
                hipFuncSetAttribute(reinterpret_cast<const void *>(tail_fn(i & 1 ? 3 : 2, i & 2, i & 4)),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax);
            if (e != hipSuccess) {
                (void)hipGetLastError();  // leave no error for the next launch to report
                return e;
            }
        }
        return hipSuccess;
    }();
    return done;
}

hipError_t launch_tail(const TailArgs &t, hipStream_t st) {
    Plan q;
    if (!plan_tail(t, q) || (!t.b0 && !t.R)) return hipErrorInvalidValue;
    for (int l = 0; l <= t.nlev; ++l)
        if (!t.wc[l] || (!t.wb[l] && (l > 0 || t.R))) return hipErrorInvalidValue;
    if (q.lds > 65536 && tail_prepare() != hipSuccess) return hipErrorInvalidValue;
    hipLaunchKernelGGL(tail_fn(t.D, t.q1, t.prec[0] == P_F64), dim3(1), dim3(q.threads), q.lds, st, q.k);
    return hipGetLastError();
}

}  // namespace mg

// The coarse end of the V-cycle in one workgroup: every level from a small
// grid down to the base level (one point, or a few solved by CG) and back up,
// with all level vectors held in LDS.  On these levels a stage is a few
// thousand points, so as separate launches each costs launch latency (3.5-6 us
// on MI355X), not bandwidth; here it costs one pass over LDS and a barrier.
// A cycle whose finest level is that small runs as this one kernel alone.
//
// Work split.  A wave issues one instruction in four cycles or more, and these
// stages wait for nothing else, so what counts is instructions per wave: a
// level of up to 1024 points gives a thread one point, a larger one (up to 16^3
// or 64^2) a segment of four consecutive x values (two with Q1 elements, two
// segments).  A thread keeps right-hand side and correction in registers from
// the first sweep to the residual, so a sweep costs the reads of its neighbours
// and one write.  Values sit in LDS in the accumulator format (they are values
// of the level's storage format: exact), which takes the conversions off every
// neighbour read.  The residual goes to the level's free correction buffer; the
// threads of the next level gather their full-weighting sums from it straight
// into registers, so a level costs nu1 + 1 barriers on the way down and nu2 + 1
// on the way up, and none where one wave holds the level.  Nothing is stored to
// memory before the end, since every barrier would wait for it.
//
// What bounds it: instruction issue and LDS latency, about 550 cycles a stage
// on the small levels and 1000 on the largest.  Measured per launch, before
// (level formats in LDS, single points walked by every thread) and now: 3-D
// from 15^3 in FP16 33.7 and 11.0; 2-D from 63^2 in FP64 21 launches, 75 us,
// and 14.3; 3-D Q1 from 11^3 with its 2^3 CG base 13 launches, 68 us, and 14.8.
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
    int base_off;              // LDS offset, in doubles, of the base arrays
    unsigned precs;            // storage format of level l at bits 2l
    int pb, nb;                // base level: format, points per dimension
    int P0, nlev, nu1, nu2, nu2_first;
    double k;                  // Jacobi weight
    double tol;                // CG base
    int maxit;
    int zero16;                // LDS in use, in 16-byte chunks
    int single;                // first level whose threads hold single points
    int small;                 // first of these that one wave holds
    float inv_p0;              // 1 / P0
    int inst;                  // batched: the instance
};

__device__ __forceinline__ void mem_store1(void *m, int o, int p, double v) {
    if (p == P_F64) static_cast<double *>(m)[o] = v;
    else if (p == P_F32) static_cast<float *>(m)[o] = (float)v;
    else if (p == P_F16) static_cast<f16 *>(m)[o] = store_as<f16>(v);
    else static_cast<bf16 *>(m)[o] = store_as<bf16>(v);
}

// Elements of a level array in LDS: P + 1 planes (rows in 2-D), the row above
// plane P's first that the corner neighbours of the last point reach, and the
// element a segment's right neighbour reaches; a multiple of 4.
__host__ __device__ __forceinline__ int lds_elems(int D, int P) {
    return ((D == 3 ? (P + 1) * P * P + P : (P + 1) * P) + 7) & ~3;
}

// LDS rows
template <class A, int V> __device__ __forceinline__ void seg(const A *p, A (&v)[V]) { load_row<A, V>(p, v); }
template <class A, int V> __device__ __forceinline__ void put(A *p, const A (&v)[V]) { store_row<A, V>(p, v); }

// Segment s of a level of pitch P (P = TXR V): its first element sits at s V.
struct Item {
    int o, x0, y, z;
    bool on;  // an interior row
};
// inv_txr, inv_p: float reciprocals of P / V and P (s < 2^12, P <= 64: the
// truncated products are exact).  Finite-difference pitches are powers of two.
template <int D, int OP, int V> __device__ __forceinline__ Item item(int s, int P, float inv_txr, float inv_p) {
    Item t;
    const int TXR = P / V;
    t.o = s * V;
    int row;
    if constexpr (OP == 0) {
        const int lg = 31 - __clz(P), lt = lg - (V == 4 ? 2 : V == 2 ? 1 : 0);
        row = s >> lt;
        t.x0 = (s & (TXR - 1)) * V;
        if (D == 3) {
            t.z = row >> lg;
            t.y = row & (P - 1);
        }
    } else {
        row = (int)(((float)s + 0.5f) * inv_txr);
        t.x0 = (s - row * TXR) * V;
        if (D == 3) {
            t.z = (int)(((float)row + 0.5f) * inv_p);
            t.y = row - t.z * P;
        }
    }
    if (D == 3) {
        t.on = t.z >= 1 && t.z < P && t.y >= 1;
    } else {
        t.z = row;
        t.y = 0;
        t.on = t.z >= 1 && t.z < P;
    }
    if (V == 1) t.on = t.on && t.x0 >= 1;  // single points: the ghost keeps its zero
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
    constexpr int H = V == 1 ? 1 : V / 2;  // (a single point takes one coarse value, or two)
    const int X0 = t.x0 >> 1;
    auto crow = [&](int Y, int Z, W (&v)[H + 1]) {
        const W *q = e + (D == 3 ? (Z * Pc + Y) * Pc : Z * Pc) + X0;
        W m[H];
        seg<W, H>(q, m);  // X0 is a multiple of H
#pragma unroll
        for (int j = 0; j < H; ++j) v[j] = m[j];
        v[H] = q[H];
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
            const bool odd = V == 1 ? (t.x0 & 1) : (i & 1);
            const W q = odd ? S[i >> 1] + S[(i >> 1) + 1] : S[i >> 1];
            out[i] = rnd_w<A>((W)c[i] + (odd ? k1 : k0) * q, p);
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
            W s = S[i >> 1] + (V == 1 ? ((t.x0 & 1) ? S[1] : S[0]) : S[(i + 1) >> 1]);
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

// Orders the LDS accesses of one wave (which the hardware runs in order).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// CG on a base level of N <= blockDim.x points (k_cg_base, one point per
// thread: x, r, q in registers, p in LDS with zero ghosts); returns x.  WAVE:
// N <= 64, called by the first wave alone: no barriers, and the sums start at
// the butterfly step that first meets a point (the earlier steps and the other
// waves of k_cg_base add zeros).
template <int D, int OP, class AB, bool WAVE>
__device__ __forceinline__ AB cg_point(AB bi, bool on, AB *p, int o, int P, int N, double tol, int maxit, double *red) {
    const int Z = D == 3 ? P * P : P;
    AB x = AB(0), r = on ? bi : AB(0), pi = r;
    int slot = 0;
    const int top = N > 32 ? 32 : N > 16 ? 16 : N > 8 ? 8 : N > 4 ? 4 : 2;
    auto sum = [&](double v) {
        if constexpr (WAVE) {
            for (int off = top; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
            const unsigned long long u = (unsigned long long)__double_as_longlong(v);
            const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)u);
            const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(u >> 32));
            return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
        } else {
            const double s = wg_sum(v, red + 16 * slot);
            slot ^= 1;
            return s;
        }
    };
    auto sync = [&]() {
        if constexpr (WAVE) wave_sync();
        else __syncthreads();
    };
    if (on) p[o] = pi;
    double rr = sum((double)r * (double)r);
    const double stop = tol * sqrt(rr);
    if (WAVE) wave_sync();
    for (int k = 0; k < maxit && sqrt(rr) > stop; ++k) {
        // (a barrier follows every write of p: that of the first sum, or the
        // one at the end of the loop)
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
        if (WAVE) wave_sync();
        if (on) p[o] = pi;  // every thread read its neighbours before the last two sums
        sync();
        rr = rr_new;
    }
    return x;
}

// Base level: right-hand side gathered from the fine residual r (pitch P),
// solved, the correction left in ec (W, zero ghosts); both are returned for the
// workspace copy.  WAVE: called by the first wave alone (at most 64 points).
template <int D, int OP, class A, class AB, class W, bool WAVE>
__device__ __forceinline__ void base_solve(const TailKArgs &a, const A *r, int P, AB *p, W *ec, double *red, bool on,
                                           int X, int Y, int Z, int o, double &bout, double &cout) {
    const int n = a.nb, Pb = P / 2, N = D == 3 ? n * n * n : n * n;
    AB bv = AB(0);
    if (on) {
        A g[1];
        gather<D, OP, A, 1>(r, X, Y, Z, P, g);
        if constexpr (std::is_same<AB, double>::value) bv = a.pb == P_F64 ? (double)g[0] : (double)rnd64<float>(g[0], a.pb);
        else bv = rnd64<float>((double)g[0], a.pb);
    }
    AB x;
    if (n == 1) {
        x = OP ? bv * AB(0.375) : bv / AB(2 * D);
    } else {
        x = cg_point<D, OP, AB, WAVE>(bv, on, p, o, Pb, N, a.tol, a.maxit, red);
    }
    if constexpr (std::is_same<AB, float>::value) x = rnd(x, a.pb);
    if (on) ec[o] = (W)x;
    bout = (double)bv;
    cout = (double)x;
}

// What the level passes share.
template <class A> struct Ctx {
    const TailKArgs &a;
    A k;
    __device__ __forceinline__ int prec(int l) const { return (int)(a.precs >> (2 * l)) & 3; }
    // levels from a.small on have at most 64 points: one wave holds them, and
    // its LDS accesses need no barrier (the other waves wait at the next one)
    __device__ __forceinline__ void sync(int l) const {
        if (l >= a.small) wave_sync();
        else __syncthreads();
    }
    template <int D, int OP, int V, int K> __device__ __forceinline__ void items(int l, Item (&it)[K]) const {
#pragma unroll
        for (int q = 0; q < K; ++q)
            it[q] = item<D, OP, V>((int)(threadIdx.x + q * blockDim.x), a.P0 >> l, a.inv_p0 * (float)(V << l),
                                   a.inv_p0 * (float)(1 << l));
    }
};

// The first level's right-hand side, from memory.
template <int D, int OP, class A, int V, int K>
__device__ __forceinline__ void fetch_rhs(const Ctx<A> &x, A (&b)[K][V]) {
    Item it[K];
    x.template items<D, OP, V, K>(0, it);
    const int p = x.prec(0);
#pragma unroll
    for (int q = 0; q < K; ++q) {
        if (!it[q].on) continue;
        if (x.a.R) {
            double r[V];
            load_row<double, V>(x.a.R + it[q].o, r);
            const double inv = x.a.scal[1];
#pragma unroll
            for (int i = 0; i < V; ++i) b[q][i] = rnd64<A>(r[i] * inv, p);
            if (it[q].x0 == 0) b[q][0] = A(0);
        } else {
            mem_load<A, V>(x.a.b0, it[q].o, p, b[q]);
        }
    }
}

// Level l on the way down (its arrays b, c0, c1 at B): the right-hand side
// gathered from the residual rf of the level above (l > 0; else b holds it),
// nu1 sweeps, the residual into the free correction buffer.
template <int D, int OP, class A, int V, int K>
__device__ __forceinline__ void level_down(const Ctx<A> &x, int l, A *B, const A *rf, A (&b)[K][V]) {
    const int P = x.a.P0 >> l, E = lds_elems(D, P), p = x.prec(l), nu1 = x.a.nu1;
    A *const C0 = B + E, *const C1 = C0 + E;
    const A k = x.k;
    Item it[K];
    A c[K][V];
    x.template items<D, OP, V, K>(l, it);
#pragma unroll
    for (int q = 0; q < K; ++q) {
        if (!it[q].on) continue;
        if (l > 0) {
            gather<D, OP, A, V>(rf, it[q].x0, it[q].y, it[q].z, 2 * P, b[q]);
            rnd_run<V>(b[q], p);
            if (it[q].x0 == 0) b[q][0] = A(0);
        }
        put<A, V>(B + it[q].o, b[q]);
#pragma unroll
        for (int i = 0; i < V; ++i) c[q][i] = k * b[q][i];
        rnd_run<V>(c[q], p);
        put<A, V>(C0 + it[q].o, c[q]);
    }
    x.sync(l);
    for (int s = 1; s <= nu1; ++s) {
        const A *src = (s & 1) ? C0 : C1;
        A *dst = (s & 1) ? C1 : C0;
        const bool res = s == nu1;
#pragma unroll
        for (int q = 0; q < K; ++q) {
            if (!it[q].on) continue;
            A lc[V], v[V];
            apply<D, OP, A, V>(src, it[q], P, c[q], lc);
#pragma unroll
            for (int i = 0; i < V; ++i) {
                const A r = b[q][i] - lc[i];
                v[i] = res ? r : fmaT<A>(k, r, c[q][i]);
            }
            if (!res) rnd_run<V>(v, p);
            if (it[q].x0 == 0) v[0] = A(0);
            put<A, V>(dst + it[q].o, v);
#pragma unroll
            for (int i = 0; i < V; ++i) c[q][i] = v[i];
        }
        x.sync(l);
    }
}

// Level l on the way up: the coarse correction ec (W) prolongated onto its
// correction, nu2 sweeps.  The first level's result goes to the workspace.
template <int D, int OP, class A, int V, int K, class W>
__device__ __forceinline__ void level_up(const Ctx<A> &x, int l, A *B, const W *ec) {
    const int P = x.a.P0 >> l, E = lds_elems(D, P), p = x.prec(l), nu2 = l == 0 ? x.a.nu2_first : x.a.nu2;
    const A k = x.k;
    auto C = [&](int j) { return B + (1 + j) * E; };
    int y = (x.a.nu1 & 1) ? 0 : 1;  // buffer of the current correction
    Item it[K];
    A b[K][V], c[K][V];
    x.template items<D, OP, V, K>(l, it);
#pragma unroll
    for (int q = 0; q < K; ++q) {
        if (!it[q].on) continue;
        A cv[V];
        seg<A, V>(C(y) + it[q].o, cv);
        seg<A, V>(B + it[q].o, b[q]);
        prolong<D, OP, A, W, V>(cv, ec, it[q], P / 2, p, c[q]);
        put<A, V>(C(y ^ 1) + it[q].o, c[q]);
    }
    y ^= 1;
    x.sync(l);
    for (int s = 0; s < nu2; ++s) {
        const bool last = l == 0 && s + 1 == nu2;
#pragma unroll
        for (int q = 0; q < K; ++q) {
            if (!it[q].on) continue;
            A lc[V], v[V];
            apply<D, OP, A, V>(C(y), it[q], P, c[q], lc);
#pragma unroll
            for (int i = 0; i < V; ++i) v[i] = fmaT<A>(k, b[q][i] - lc[i], c[q][i]);
            rnd_run<V>(v, p);
            if (it[q].x0 == 0) v[0] = A(0);
            if (!last) put<A, V>(C(y ^ 1) + it[q].o, v);
#pragma unroll
            for (int i = 0; i < V; ++i) c[q][i] = v[i];
        }
        y ^= 1;
        if (!last) x.sync(l);
    }
    if (l == 0) {
#pragma unroll
        for (int q = 0; q < K; ++q) {
            if (!it[q].on) continue;
            mem_store<A, V>(x.a.wc[0], it[q].o, p, c[q]);
            if (x.a.R) mem_store<A, V>(x.a.wb[0], it[q].o, p, b[q]);
        }
    }
}

template <int D, int OP, class A> __device__ __forceinline__ void tail_body(const TailKArgs &a) {
    constexpr int V = TailSplit<OP>::V, K = TailSplit<OP>::K;
    extern __shared__ __align__(16) unsigned char smem[];
    A *const lds = reinterpret_cast<A *>(smem);
    const Ctx<A> x{a, (A)a.k};
    const int tid = (int)threadIdx.x, nthr = (int)blockDim.x, nlev = a.nlev;
    auto elems = [&](int l) { return lds_elems(D, a.P0 >> l); };
    // the first level's right-hand side is on its way while LDS is cleared
    A b[K][V], b1[1][1];
    if (a.single > 0) fetch_rhs<D, OP, A, V, K>(x, b);
    else fetch_rhs<D, OP, A, 1, 1>(x, b1);
    for (int i = tid; i < a.zero16; i += nthr) reinterpret_cast<uint4 *>(smem)[i] = uint4{0u, 0u, 0u, 0u};
    __syncthreads();
    // down: pre-smoothing, residual, restriction
    const int rbuf = 1 + (a.nu1 & 1);  // the residual's buffer among a level's arrays
    A *B = lds;
    const A *rf = nullptr;
    for (int l = 0; l < nlev; ++l) {
        if (l < a.single) level_down<D, OP, A, V, K>(x, l, B, rf, b);
        else level_down<D, OP, A, 1, 1>(x, l, B, rf, b1);
        rf = B + rbuf * elems(l);
        B += 3 * elems(l);
    }
    // base level
    double *const base = reinterpret_cast<double *>(smem) + a.base_off;  // [32 sums][c][p]
    const int Pl = a.P0 >> (nlev - 1), Pb = Pl / 2;
    const int Eb = lds_elems(D, Pb);
    double *const ecd = base + 32;
    A *const eca = reinterpret_cast<A *>(ecd);
    const bool wide = std::is_same<A, double>::value || a.pb == P_F64;  // interpolation from the base in FP64
    const int N = D == 3 ? a.nb * a.nb * a.nb : a.nb * a.nb;
    const bool bon = tid < N;
    int bX = 1, bY = D == 3 ? 1 : 0, bZ = 1;
    if (a.nb > 1) {
        bX = tid % a.nb + 1;
        bY = D == 3 ? (tid / a.nb) % a.nb + 1 : 0;
        bZ = D == 3 ? tid / (a.nb * a.nb) + 1 : tid / a.nb + 1;
    }
    const int bo = D == 3 ? (bZ * Pb + bY) * Pb + bX : bZ * Pb + bX;
    double bb = 0.0, bc = 0.0;
#define MG_BASE(AB, W, WV, EC) \
    base_solve<D, OP, A, AB, W, WV>(a, rf, Pl, reinterpret_cast<AB *>(ecd + Eb), EC, base, bon, bX, bY, bZ, bo, bb, bc)
    if (N <= 64) {
        if (tid < 64) {
            if (a.pb == P_F64) MG_BASE(double, double, true, ecd);
            else MG_BASE(float, A, true, eca);
        }
        x.sync(nlev - 1);
    } else {
        if (nlev - 1 >= a.small) __syncthreads();  // the residual came from one wave
        if (a.pb == P_F64) MG_BASE(double, double, false, ecd);
        else MG_BASE(float, A, false, eca);
        __syncthreads();
    }
#undef MG_BASE
    // up: prolongation, correction and post-smoothing.  A level's correction
    // sits in c0 after an odd number of pre-sweeps, else in c1, and ends in
    // array xf.
    const int xf = 1 + ((a.nu1 & 1) ^ (a.nu2 & 1));
    const A *ec = eca;
    for (int l = nlev - 1; l >= 0; --l) {
        B -= 3 * elems(l);
        if (l + 1 == a.small) __syncthreads();  // the coarse correction came from one wave
        const bool from_wide = !std::is_same<A, double>::value && l + 1 == nlev && wide;
        if (l < a.single) {
            if (from_wide) level_up<D, OP, A, V, K, double>(x, l, B, ecd);
            else level_up<D, OP, A, V, K, A>(x, l, B, ec);
        } else {
            if (from_wide) level_up<D, OP, A, 1, 1, double>(x, l, B, ecd);
            else level_up<D, OP, A, 1, 1, A>(x, l, B, ec);
        }
        ec = B + xf * elems(l);
    }
    // the inner levels' vectors, which the level kernels leave in the workspace.
    // Copied here and not on the way, where the barriers would wait for the
    // stores; whole arrays, ghosts (zeros) and all.
    B = lds;
    for (int l = 1; l < nlev; ++l) {
        B += 3 * elems(l - 1);
        const int P = a.P0 >> l, p = x.prec(l), n = (D == 3 ? P * P : P) * P, E = elems(l);
        constexpr int VC = OP ? 2 : 4;
        for (int i = VC * tid; i < n; i += VC * nthr) {
            A v[VC];
            seg<A, VC>(B + i, v);
            mem_store<A, VC>(a.wb[l], i, p, v);
            seg<A, VC>(B + xf * E + i, v);
            mem_store<A, VC>(a.wc[l], i, p, v);
        }
    }
    if (bon) {
        mem_store1(a.wb[nlev], bo, a.pb, bb);
        mem_store1(a.wc[nlev], bo, a.pb, bc);
    }
}

template <int D, int OP, class A> __global__ __launch_bounds__(kThreads) void k_tail(const TailKArgs a) {
    tail_body<D, OP, A>(a);
}

// Batched instances: one workgroup each (block sizes and LDS of the largest).
template <class A>
__global__ __launch_bounds__(kThreads) void k_batched_tail(const TailKArgs *__restrict__ args,
                                                           const int *__restrict__ active) {
    const TailKArgs &a = args[blockIdx.x];  // (scalar loads where used: a copy would sit in scratch memory)
    if (active[a.inst]) tail_body<3, 0, A>(a);
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
    int threads = 64;
    for (int l = 0; l < t.nlev; ++l) {
        const int P = t.P0 >> l;
        if ((P << l) != t.P0 || P % V || P < 4 || P > 64) return false;
        if ((t.prec[l] == P_F64) != f64) return false;  // one accumulator format
        const int pts = P * P * (t.D == 3 ? P : 1), segs = pts / V;
        if (pts > kThreads) k.single = l + 1;
        if (pts > 64) k.small = l + 1;
        threads = std::max(threads, pts > kThreads ? (segs + K - 1) / K : pts);
        off += 3 * (size_t)lds_elems(t.D, P) * sa;
        k.precs |= (unsigned)t.prec[l] << (2 * l);
    }
    if (threads > kThreads) return false;
    off = (off + 15) & ~(size_t)15;
    const int Pl = t.P0 >> (t.nlev - 1), Pb = Pl / 2;
    if (Pl % 2 || t.nb != Pb - 1) return false;
    const int N = t.D == 3 ? t.nb * t.nb * t.nb : t.nb * t.nb;
    if (t.nb < 1 || N > kThreads) return false;
    k.base_off = (int)(off / 8);
    off += 8 * (32 + (size_t)lds_elems(t.D, Pb) * (t.nb > 1 ? 2 : 1));
    off = (off + 15) & ~(size_t)15;
    if (off > kLdsMax) return false;
    q.lds = off;
    q.threads = (std::max(threads, N) + 63) / 64 * 64;
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
    k.inv_p0 = 1.0f / (float)t.P0;
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
        for (const void *f : {(const void *)k_batched_tail<float>, (const void *)k_batched_tail<double>}) {
            const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax);
            if (e != hipSuccess) {
                (void)hipGetLastError();
                return e;
            }
        }
        return hipSuccess;
    }();
    return done;
}

size_t tail_record_bytes() { return sizeof(TailKArgs); }

bool tail_record(const TailArgs &t, int inst, void *dst, int *threads, size_t *lds) {
    Plan q;
    if (t.D != 3 || t.q1 || !plan_tail(t, q)) return false;
    q.k.inst = inst;
    if (dst) *static_cast<TailKArgs *>(dst) = q.k;
    *threads = q.threads;
    *lds = q.lds;
    return true;
}

hipError_t launch_batched_tail(bool f64, const void *records, int n, const int *active, int threads, size_t lds,
                               hipStream_t st) {
    if (n < 1 || threads < 64 || threads > kThreads || lds > kLdsMax) return hipErrorInvalidValue;
    if (lds > 65536 && tail_prepare() != hipSuccess) return hipErrorInvalidValue;
    const TailKArgs *r = static_cast<const TailKArgs *>(records);
    if (f64) hipLaunchKernelGGL((k_batched_tail<double>), dim3(n), dim3(threads), lds, st, r, active);
    else hipLaunchKernelGGL((k_batched_tail<float>), dim3(n), dim3(threads), lds, st, r, active);
    return hipGetLastError();
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

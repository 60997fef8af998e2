// Fused stages of a 2-D level, one block per tile: all pre-smoothing with the
// residual and the restriction ("down"), and the prolongation with all
// post-smoothing ("up"), on the finest level of a refinement step also the
// update of r and u and its norms.  A level costs two launches instead of four
// or five (seven with Q1 elements), and no intermediate goes through memory:
// of the FP16 finest level's 12 + 6.25 + 6.25 + 6 + 34 bytes per point the
// step moves 12.25 + 36.25 (finite differences); a level of a few hundred
// points per side costs launch latency only, and half of it.
//
// Work split.  A block owns TX by TY points and works on them with a halo: four
// columns either side (a segment, so that rows stay aligned) and as many rows
// as the chained stencils need (down: nu1 + 1 above, nu1 below; up: nu2, one
// more with the update).  A thread holds one segment of four x values of one
// row for the whole kernel, right-hand side and correction in registers; the
// correction passes through two LDS tiles, written and read once per sweep.
// The rim of the halo goes stale one ring per stage and is not used after that.
//
// What bounds it: launch latency up to about 1000^2 (4.6 us a launch), above
// that memory for the FP64 streams of the update (2047^2 FP16: down 17.7 us,
// 51 MB; up with the update 40 us, 152 MB) and FP64 arithmetic with Q1 elements
// (4095^2 FP16: 66 and 136 us).  Before, the same stages took 39 + 43 us at
// 2047^2 and 100 + 126 us at 4095^2, and four to seven launches of 3.5-6 us on
// every smaller level.
//
// The arithmetic is that of the separate kernels, operation for operation, so
// results are bitwise theirs (the norms up to their summation order).
#include "mg_level_math.h"

#include <algorithm>

namespace mg {
namespace {

constexpr int kThreads = 1024;
constexpr int V = 4;

// Tile geometry: SX segments per row (one of halo each side), rows of LS
// elements in LDS with a segment of padding each side, and a row above and
// below: every neighbour a thread reads lies in the block's LDS.
struct Tile {
    int r, s;        // row and segment within the tile
    int x0, y;       // first point
    bool in;         // inside the grid (x0 = 0 holds the ghost in element 0)
    int at;          // LDS index of the segment
};
__device__ __forceinline__ Tile tile_of(int TX, int rows, int X0, int Y0, int top, int P, int LS) {
    Tile t;
    const int SX = TX / V + 2, tid = (int)threadIdx.x;
    t.r = (int)(((float)tid + 0.5f) / (float)SX);  // tid < 2^10: exact after truncation
    t.s = tid - t.r * SX;
    t.x0 = X0 + V * (t.s - 1);
    t.y = Y0 - top + t.r;
    t.in = t.r < rows && t.y >= 1 && t.y < P && t.x0 >= 0 && t.x0 < P;
    t.at = (t.r + 1) * LS + V * (t.s + 1);
    return t;
}

// lc = L c (finite differences) or S c (Q1) at a segment, in C; c: LDS tile.
template <int OP, class A, class C>
__device__ __forceinline__ void apply2(const A *c, const Tile &t, int LS, const A (&cc)[V], C (&lc)[V]) {
    const A *p = c + t.at;
    if constexpr (OP == 0) {
        A s[V], n[V];
        load_row<A, V>(p - LS, s);
        load_row<A, V>(p + LS, n);
        const C xl = (C)p[-1], xr = (C)p[V];
#pragma unroll
        for (int i = 0; i < V; ++i) {
            C nb = (i > 0 ? (C)cc[i - 1] : xl) + (i < V - 1 ? (C)cc[i + 1] : xr);
            nb += (C)s[i];
            nb += (C)n[i];
            lc[i] = fmaT<C>(C(4), (C)cc[i], -nb);
        }
    } else {
        auto row = [&](const A *q, C (&r)[V + 2]) {
            A m[V];
            load_row<A, V>(q, m);
            r[0] = (C)q[-1];
#pragma unroll
            for (int i = 0; i < V; ++i) r[i + 1] = (C)m[i];
            r[V + 1] = (C)q[V];
        };
        C s[V + 2], n[V + 2], m[V + 2];
        row(p - LS, s);
        row(p + LS, n);
        m[0] = (C)p[-1];
#pragma unroll
        for (int i = 0; i < V; ++i) m[i + 1] = (C)cc[i];
        m[V + 1] = (C)p[V];
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const C nb = ((s[i] + s[i + 1]) + (s[i + 2] + m[i])) + ((m[i + 2] + n[i]) + (n[i + 1] + n[i + 2]));
            lc[i] = fmaT<C>(C(8), m[i + 1], -nb) * q1_scale<2, C>();
        }
    }
}

struct DownK {
    const void *b;
    const double *R, *scal;
    void *bout, *cout, *bc;
    int P, prec, pc, nu, TX, TY, xtiles;
    double k;
};

template <int OP, class A> __global__ __launch_bounds__(kThreads) void k_tile2d_down(const DownK a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int P = a.P, p = a.prec, top = a.nu + 1, rows = a.TY + top + a.nu, LS = a.TX + 4 * V;
    A *const L0 = reinterpret_cast<A *>(smem), *const L1 = L0 + (rows + 2) * LS;
    const int blk = xcd_block((int)blockIdx.x, (int)gridDim.x);
    const int yt = blk / a.xtiles, X0 = (blk - yt * a.xtiles) * a.TX, Y0 = yt * a.TY;
    const Tile t = tile_of(a.TX, rows, X0, Y0, top, P, LS);
    const bool row_in = t.r < rows;
    const bool own = t.in && t.s >= 1 && t.s <= a.TX / V && t.r >= top && t.r < top + a.TY;
    const size_t o = (size_t)t.y * P + t.x0;
    const A k = (A)a.k;
    A b[V], c[V];
#pragma unroll
    for (int i = 0; i < V; ++i) b[i] = A(0);
    if (t.in) {
        if (a.R) {
            double r[V];
            load_row<double, V>(a.R + o, r);
            const double inv = a.scal[1];
#pragma unroll
            for (int i = 0; i < V; ++i) b[i] = rnd64<A>(r[i] * inv, p);
        } else {
            mem_load<A, V>(a.b, o, p, b);
        }
        if (t.x0 == 0) b[0] = A(0);
        if (a.bout && own) mem_store<A, V>(a.bout, o, p, b);
    }
#pragma unroll
    for (int i = 0; i < V; ++i) c[i] = rnd(k * b[i], p);
    if (row_in) store_row<A, V>(L0 + t.at, c);
    __syncthreads();
    // sweeps 2 .. nu, then the residual
    for (int s = 1; s <= a.nu; ++s) {
        const A *src = (s & 1) ? L0 : L1;
        A *dst = (s & 1) ? L1 : L0;
        if (row_in) {
            const bool res = s == a.nu;
            A lc[V], v[V];
            apply2<OP, A, A>(src, t, LS, c, lc);
#pragma unroll
            for (int i = 0; i < V; ++i) {
                const A r = b[i] - lc[i];
                v[i] = !t.in ? A(0) : res ? r : rnd(fmaT<A>(k, r, c[i]), p);
            }
            if (t.x0 == 0) v[0] = A(0);
            if (res && own) mem_store<A, V>(a.cout, o, p, c);
            store_row<A, V>(dst + t.at, v);
#pragma unroll
            for (int i = 0; i < V; ++i) c[i] = v[i];
        }
        __syncthreads();
    }
    // full weighting: the threads of the even rows form two coarse values each
    if (own && (t.y & 1) == 0 && t.y >= 2) {
        const A *q = ((a.nu & 1) ? L1 : L0) + t.at;
        constexpr int H = V / 2;
        auto row = [&](const A *e, A (&w)[H]) {
            A m[V];
            load_row<A, V>(e, m);
            A left = e[-1];
#pragma unroll
            for (int j = 0; j < H; ++j) {
                if (OP == 0) w[j] = A(0.25) * (left + m[2 * j + 1]) + A(0.5) * m[2 * j];
                else w[j] = (left + m[2 * j + 1]) + A(2) * m[2 * j];
                left = m[2 * j + 1];
            }
        };
        A u[H], m[H], d[H], v[H];
        row(q - LS, u);
        row(q, m);
        row(q + LS, d);
#pragma unroll
        for (int j = 0; j < H; ++j) {
            if (OP == 0) {
                A acc = A(0.25) * u[j];
                acc += A(0.5) * m[j];
                v[j] = acc + A(0.25) * d[j];
            } else {
                v[j] = ((u[j] + d[j]) + A(2) * m[j]) * A(1.0 / 16.0);
            }
        }
        if (t.x0 == 0) v[0] = A(0);
        mem_store<A, H>(a.bc, (size_t)(t.y >> 1) * (P / 2) + (t.x0 >> 1), a.pc, v);
    }
}

struct UpK {
    const void *b, *c, *ec;
    void *cout;  // swept correction, or
    const double *R;  // ... the update of Algorithm 2: r (in), Rout, U or the ring
    double *Rout, *U;
    const double *scal;
    void *cd;
    const int *ctr;
    size_t cstride;
    double *adef, *part;
    double k, f;
    int P, prec, pc, nu, TX, TY, xtiles;
};

// c + 4 P e of a segment, in W, rounded into format p.
template <int OP, class A, class W>
__device__ __forceinline__ void prolong2(const void *ec, int pc, const Tile &t, int Pc, const A (&c)[V], int p,
                                         A (&out)[V]) {
    constexpr int H = V / 2;
    const int X0 = t.x0 >> 1;
    auto crow = [&](int Z, W (&v)[H + 1]) {
        const size_t q = (size_t)Z * Pc + X0;
        W two[H], last[1];
        mem_load<W, H>(ec, q, pc, two);
        mem_load<W, 1>(ec, q + H, pc, last);  // beyond the row: the next row's zero ghost
#pragma unroll
        for (int j = 0; j < H; ++j) v[j] = two[j];
        v[H] = last[0];
    };
    W S[H + 1], a[H + 1];
    const bool odd = t.y & 1;
    crow(t.y >> 1, S);
    if (odd) crow((t.y + 1) >> 1, a);
    else
#pragma unroll
        for (int j = 0; j <= H; ++j) a[j] = S[j];
    if constexpr (OP == 0) {
        if (odd)
#pragma unroll
            for (int j = 0; j <= H; ++j) S[j] = S[j] + a[j];
        const W k0 = odd ? W(2) : W(4), k1 = W(0.5) * k0;
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const W q = (i & 1) ? S[i >> 1] + S[(i >> 1) + 1] : S[i >> 1];
            out[i] = rnd_w<A>((W)c[i] + ((i & 1) ? k1 : k0) * q, p);
        }
    } else {
#pragma unroll
        for (int j = 0; j <= H; ++j) S[j] = S[j] + a[j];
#pragma unroll
        for (int i = 0; i < V; ++i) out[i] = rnd_w<A>((W)c[i] + (S[i >> 1] + S[(i + 1) >> 1]), p);
    }
    if (t.x0 == 0) out[0] = A(0);
}

template <int OP, class A, bool UPD> __global__ __launch_bounds__(kThreads) void k_tile2d_up(const UpK a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[2 * kThreads / 64];
    const int P = a.P, p = a.prec, top = a.nu + (UPD ? 1 : 0), rows = a.TY + 2 * top, LS = a.TX + 4 * V;
    A *L0 = reinterpret_cast<A *>(smem), *L1 = L0 + (rows + 2) * LS;
    const int blk = xcd_block((int)blockIdx.x, (int)gridDim.x);
    const int yt = blk / a.xtiles, X0 = (blk - yt * a.xtiles) * a.TX, Y0 = yt * a.TY;
    const Tile t = tile_of(a.TX, rows, X0, Y0, top, P, LS);
    const bool row_in = t.r < rows;
    const bool own = t.in && t.s >= 1 && t.s <= a.TX / V && t.r >= top && t.r < top + a.TY;
    const size_t o = (size_t)t.y * P + t.x0;
    const A k = (A)a.k;
    A b[V], c[V];
    double r[V], u[V];
#pragma unroll
    for (int i = 0; i < V; ++i) b[i] = c[i] = A(0), r[i] = u[i] = 0.0;
    if (t.in) {
        A cv[V];
        mem_load<A, V>(a.c, o, p, cv);
        mem_load<A, V>(a.b, o, p, b);
        if (UPD && own) {  // in flight during the sweeps
            load_row<double, V>(a.R + o, r);
            if (a.U) load_row<double, V>(a.U + o, u);
        }
        if (!std::is_same<A, double>::value && a.pc == P_F64)
            prolong2<OP, A, double>(a.ec, a.pc, t, P / 2, cv, p, c);
        else
            prolong2<OP, A, A>(a.ec, a.pc, t, P / 2, cv, p, c);
    }
    if (row_in) store_row<A, V>(L0 + t.at, c);
    __syncthreads();
    for (int s = 0; s < a.nu; ++s) {
        if (row_in) {
            A lc[V];
            apply2<OP, A, A>(L0, t, LS, c, lc);
#pragma unroll
            for (int i = 0; i < V; ++i) c[i] = t.in ? rnd(fmaT<A>(k, b[i] - lc[i], c[i]), p) : A(0);
            if (t.x0 == 0) c[0] = A(0);
            if (UPD || s + 1 < a.nu) store_row<A, V>(L1 + t.at, c);
        }
        if (UPD || s + 1 < a.nu) __syncthreads();
        A *const sw = L0;
        L0 = L1;
        L1 = sw;
    }
    if constexpr (!UPD) {
        if (own) mem_store<A, V>(a.cout, o, p, c);
    } else {
        double ss = 0.0, mx = 0.0;
        const double al = a.scal[0];
        int slot = 0;
        if (a.cd) {
            slot = *a.ctr;
            if (blockIdx.x == 0 && threadIdx.x == 0) a.adef[slot] = al;
        }
        if (own) {
            const double af = al * a.f;
            double lc[V];
            apply2<OP, A, double>(L0, t, LS, c, lc);
#pragma unroll
            for (int i = 0; i < V; ++i) {
                r[i] = fmaT<double>(-al, lc[i], r[i]);
                u[i] = fmaT<double>(af, (double)c[i], u[i]);
            }
            if (t.x0 == 0) r[0] = 0.0, u[0] = 0.0;
#pragma unroll
            for (int i = 0; i < V; ++i) {
                ss += r[i] * r[i];
                mx = nanmax(mx, fabs(r[i]));
            }
            store_row<double, V>(a.Rout + o, r);
            if (a.cd) mem_store<A, V>(a.cd, (size_t)slot * a.cstride + o, p, c);
            else store_row<double, V>(a.U + o, u);
        }
        block_reduce(ss, mx, red);
        if (threadIdx.x == 0) {
            a.part[2 * blockIdx.x] = ss;
            a.part[2 * blockIdx.x + 1] = mx;
        }
    }
}

// Tile sizes.  Small levels take small tiles, so that there are about as many
// blocks as CUs; from pitch 512 on 64 by 16, from 4096 on 128 by 16 points
// (taller tiles of up to 1024 threads do less halo work but measured slower:
// 4095^2 Q1 FP16 373 us a step at 128 by 24 and 361 at 128 by 16, 2047^2 FP64
// 158 and 150; two to four blocks per CU overlap their barriers).
struct Geo {
    int TX, TY, xtiles, blocks, threads;
    size_t lds;
};
Geo geo(int P, int halo_rows, size_t sa) {
    Geo g;
    g.TX = P >= 4096 ? 128 : P >= 512 ? 64 : 32;
    const int SX = g.TX / V + 2;
    // rows by threads, and by the 64 KB of LDS of two tiles (FP64)
    const int lds_rows = (int)((65536 - 512) / (2 * (g.TX + 4 * V) * sa)) - 2;
    const int most = (std::min(kThreads / SX, lds_rows) - halo_rows) & ~1;
    g.TY = std::max(2, std::min(P >= 512 ? 16 : 8, most));
    g.xtiles = (P + g.TX - 1) / g.TX;
    g.blocks = g.xtiles * ((P + g.TY - 1) / g.TY);
    const int rows = g.TY + halo_rows;
    g.threads = (SX * rows + 63) / 64 * 64;
    g.lds = 2 * (size_t)(rows + 2) * (g.TX + 4 * V) * sa;
    return g;
}

}  // namespace

bool tile2d_ok(int P, int nu1, int nu2) {
    // four halo columns: nu1 + 1 and nu2 + 1 stencils deep; and coarse rows of
    // whole two-value segments
    return P >= 8 && P % 4 == 0 && P <= 8192 && nu1 >= 1 && nu1 <= 3 && nu2 >= 1 && nu2 <= 3;
}

int tile2d_update_blocks(int P, int prec, int nu2) {
    return geo(P, 2 * (nu2 + 1), prec == P_F64 ? 8 : 4).blocks;
}

hipError_t launch_tile2d_down(const Tile2dArgs &t, hipStream_t st) {
    if (!tile2d_ok(t.P, t.nu, t.nu) || (!t.b && !t.R) || !t.cout || !t.bc) return hipErrorInvalidValue;
    const bool f64 = t.prec == P_F64;
    const Geo g = geo(t.P, 2 * t.nu + 1, f64 ? 8 : 4);
    DownK a{};
    a.b = t.b, a.R = t.R, a.scal = t.scal, a.bout = t.bout, a.cout = t.cout, a.bc = t.bc;
    a.P = t.P, a.prec = t.prec, a.pc = t.pc, a.nu = t.nu, a.TX = g.TX, a.TY = g.TY, a.xtiles = g.xtiles;
    a.k = t.q1 ? t.omega * 0.375 : t.omega / 4.0;
    auto fn = t.q1 ? (f64 ? k_tile2d_down<1, double> : k_tile2d_down<1, float>)
                   : (f64 ? k_tile2d_down<0, double> : k_tile2d_down<0, float>);
    hipLaunchKernelGGL(fn, dim3(g.blocks), dim3(g.threads), g.lds, st, a);
    return hipGetLastError();
}

hipError_t launch_tile2d_up(const Tile2dArgs &t, hipStream_t st) {
    const bool upd = t.Rout != nullptr;
    if (!tile2d_ok(t.P, t.nu, t.nu) || !t.b || !t.cin || !t.ec || (upd ? !t.R || !t.part || !t.scal : !t.cout))
        return hipErrorInvalidValue;
    if (upd && (t.cdefer ? !t.adef || !t.ctr : !t.U)) return hipErrorInvalidValue;
    // neighbouring tiles read the right-hand side this block's update overwrites
    if (upd && t.b == (const void *)t.Rout) return hipErrorInvalidValue;
    const bool f64 = t.prec == P_F64;
    const Geo g = geo(t.P, 2 * (t.nu + (upd ? 1 : 0)), f64 ? 8 : 4);
    UpK a{};
    a.b = t.b, a.c = t.cin, a.ec = t.ec, a.cout = t.cout;
    a.R = t.R, a.Rout = t.Rout, a.U = t.cdefer ? nullptr : t.U, a.scal = t.scal;
    a.cd = t.cdefer, a.ctr = t.ctr, a.cstride = t.cstride, a.adef = t.adef, a.part = t.part, a.f = t.f;
    a.P = t.P, a.prec = t.prec, a.pc = t.pc, a.nu = t.nu, a.TX = g.TX, a.TY = g.TY, a.xtiles = g.xtiles;
    a.k = t.q1 ? t.omega * 0.375 : t.omega / 4.0;
#define MG_UP(OP, A) (upd ? k_tile2d_up<OP, A, true> : k_tile2d_up<OP, A, false>)
    auto fn = t.q1 ? (f64 ? MG_UP(1, double) : MG_UP(1, float)) : (f64 ? MG_UP(0, double) : MG_UP(0, float));
#undef MG_UP
    hipLaunchKernelGGL(fn, dim3(g.blocks), dim3(g.threads), g.lds, st, a);
    return hipGetLastError();
}

}  // namespace mg

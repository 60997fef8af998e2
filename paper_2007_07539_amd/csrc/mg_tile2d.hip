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
// that memory for the FP64 streams of the update and instruction issue
// (finest level, down and up with the update: 2047^2 FP16 14 and 34 us for 51 and
// 152 MB, 4095^2 Q1 FP16 54 and 103 us).  Formats chosen at run time made each
// load wait for its own conversion (4095^2 Q1: 67 and 138 us), and a segment's
// neighbours read together with it conflicted in LDS (66 and 124 us).  As separate
// kernels the same stages took 39 + 43 us at 2047^2 and 100 + 126 us at 4095^2, and
// four to seven launches of 3.5-6 us on every smaller level.
//
// The arithmetic is that of the separate kernels, operation for operation, so
// results are bitwise theirs (the norms up to their summation order).
#include "mg_level_math.h"

#include <algorithm>

namespace mg {
namespace {

constexpr int kThreads = 1024;
constexpr int V = 4;

// The level's format is a template parameter: chosen at run time, each load waited
// for its own conversion before the next one was issued.
template <int PF> struct AccOf {
    typedef typename std::conditional<PF == P_F64, double, float>::type type;
    typedef typename std::conditional<PF == P_F16, f16, typename std::conditional<PF == P_BF16, bf16, type>::type>::type
        store;
};

// Tile geometry: SX segments per row (one of halo each side), rows of LS
// elements in LDS with a segment of padding each side, and a row above and
// below: every neighbour a thread reads lies in the block's LDS.
struct Tile {
    int r, s;        // row and segment within the tile
    int x0, y;       // first point
    bool in;         // inside the grid (x0 = 0 holds the ghost in element 0)
    int at;          // LDS index of the segment
    int lf, rt;      // ... of its left and right neighbours, opaque to the compiler: it
                     // would merge them with the segment's 16-byte access into
                     // misaligned pairs with four-way bank conflicts
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
    t.lf = t.at - 1, t.rt = t.at + V;
    asm("" : "+v"(t.lf), "+v"(t.rt));
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
        const C xl = (C)c[t.lf], xr = (C)c[t.rt];
#pragma unroll
        for (int i = 0; i < V; ++i) {
            C nb = (i > 0 ? (C)cc[i - 1] : xl) + (i < V - 1 ? (C)cc[i + 1] : xr);
            nb += (C)s[i];
            nb += (C)n[i];
            lc[i] = fmaT<C>(C(4), (C)cc[i], -nb);
        }
    } else {
        auto row = [&](int off, C (&r)[V + 2]) {
            A m[V];
            load_row<A, V>(p + off, m);
            r[0] = (C)c[t.lf + off];
#pragma unroll
            for (int i = 0; i < V; ++i) r[i + 1] = (C)m[i];
            r[V + 1] = (C)c[t.rt + off];
        };
        C s[V + 2], n[V + 2], m[V + 2];
        row(-LS, s);
        row(LS, n);
        m[0] = (C)c[t.lf];
#pragma unroll
        for (int i = 0; i < V; ++i) m[i + 1] = (C)cc[i];
        m[V + 1] = (C)c[t.rt];
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
    int P, pc, nu, TX, TY, xtiles;
    double k;
};

template <int OP, int PF> __global__ __launch_bounds__(kThreads) void k_tile2d_down(const DownK a) {
    typedef typename AccOf<PF>::type A;
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int p = PF;
    const int P = a.P, top = a.nu + 1, rows = a.TY + top + a.nu, LS = a.TX + 4 * V;
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
                const A r = b[i] - lc[i], w = rnd(fmaT<A>(k, r, c[i]), p);  // (both: no branch per value)
                v[i] = !t.in ? A(0) : res ? r : w;
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
        const A *q = (a.nu & 1) ? L1 : L0;
        constexpr int H = V / 2;
        auto row = [&](int off, A (&w)[H]) {
            A m[V];
            load_row<A, V>(q + t.at + off, m);
            A left = q[t.lf + off];
#pragma unroll
            for (int j = 0; j < H; ++j) {
                if (OP == 0) w[j] = A(0.25) * (left + m[2 * j + 1]) + A(0.5) * m[2 * j];
                else w[j] = (left + m[2 * j + 1]) + A(2) * m[2 * j];
                left = m[2 * j + 1];
            }
        };
        A u[H], m[H], d[H], v[H];
        row(-LS, u);
        row(0, m);
        row(LS, d);
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
    int P, pc, nu, TX, TY, xtiles;
};

// c + 4 P e of a segment, in W, rounded into format p; S, a: coarse rows
// floor(y / 2) and ceil(y / 2) from x0 / 2.
template <int OP, class A, class W>
__device__ __forceinline__ void prolong2(W (&S)[V / 2 + 1], const W (&a)[V / 2 + 1], const Tile &t, const A (&c)[V],
                                         int p, A (&out)[V]) {
    constexpr int H = V / 2;
    const bool odd = t.y & 1;
    if constexpr (OP == 0) {
#pragma unroll
        for (int j = 0; j <= H; ++j) S[j] = odd ? S[j] + a[j] : S[j];
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

// The same from a coarse level in another format than the fine one's.
template <int OP, class A, class W>
__device__ __forceinline__ void prolong2_mixed(const void *ec, int pc, const Tile &t, int Pc, const A (&c)[V], int p,
                                               A (&out)[V]) {
    constexpr int H = V / 2;
    auto crow = [&](int Z, W (&v)[H + 1]) {
        const size_t q = (size_t)Z * Pc + (t.x0 >> 1);
        W two[H], last[1];
        mem_load<W, H>(ec, q, pc, two);
        mem_load<W, 1>(ec, q + H, pc, last);  // beyond the row: the next row's zero ghost
#pragma unroll
        for (int j = 0; j < H; ++j) v[j] = two[j];
        v[H] = last[0];
    };
    W S[H + 1], a[H + 1];
    crow(t.y >> 1, S);
    crow((t.y + 1) >> 1, a);
    prolong2<OP, A, W>(S, a, t, c, p, out);
}

template <int OP, int PF, bool UPD> __global__ __launch_bounds__(kThreads) void k_tile2d_up(const UpK a) {
    typedef typename AccOf<PF>::type A;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[2 * kThreads / 64];
    constexpr int p = PF;
    const int P = a.P, top = a.nu + (UPD ? 1 : 0), rows = a.TY + 2 * top, LS = a.TX + 4 * V;
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
        // every load is issued before the first is waited for
        constexpr int H = V / 2;
        typedef typename AccOf<PF>::store T;
        RawRow<T, H> e0, e1;
        RawRow<T, V> cr, br;
        T l0{}, l1{};
        const bool same = a.pc == PF;
        if (same) {
            const T *ec = static_cast<const T *>(a.ec) + (t.x0 >> 1);
            const T *r0 = ec + (size_t)(t.y >> 1) * (P / 2), *r1 = ec + (size_t)((t.y + 1) >> 1) * (P / 2);
            fetch_row<T, H>(r0, e0);
            fetch_row<T, H>(r1, e1);
            l0 = r0[H], l1 = r1[H];  // beyond the row: the next row's zero ghost
        }
        fetch_row<T, V>(static_cast<const T *>(a.c) + o, cr);
        fetch_row<T, V>(static_cast<const T *>(a.b) + o, br);
        if (UPD && own) {  // in flight during the sweeps
            load_row<double, V>(a.R + o, r);
            if (a.U) load_row<double, V>(a.U + o, u);
        }
        A cv[V];
        widen_row<T, V>(cr, cv);
        if (same) {
            A S[H + 1], n[H + 1], w[H];
            widen_row<T, H>(e0, w);
#pragma unroll
            for (int j = 0; j < H; ++j) S[j] = w[j];
            S[H] = widen(l0);
            widen_row<T, H>(e1, w);
#pragma unroll
            for (int j = 0; j < H; ++j) n[j] = w[j];
            n[H] = widen(l1);
            prolong2<OP, A, A>(S, n, t, cv, p, c);
        } else if (!std::is_same<A, double>::value && a.pc == P_F64) {
            prolong2_mixed<OP, A, double>(a.ec, P_F64, t, P / 2, cv, p, c);
        } else {
            prolong2_mixed<OP, A, A>(a.ec, a.pc, t, P / 2, cv, p, c);
        }
        widen_row<T, V>(br, b);
    }
    if (row_in) store_row<A, V>(L0 + t.at, c);
    __syncthreads();
    for (int s = 0; s < a.nu; ++s) {
        if (row_in) {
            A lc[V];
            apply2<OP, A, A>(L0, t, LS, c, lc);
#pragma unroll
            for (int i = 0; i < V; ++i) {
                const A w = rnd(fmaT<A>(k, b[i] - lc[i], c[i]), p);
                c[i] = t.in ? w : A(0);
            }
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
// blocks as CUs; from pitch 512 on 64 by 16, from 2048 on 64 by 20 points
// (us of the finest level's two kernels at 64 by 16, 64 by 20, 128 by 16: 4095^2
// Q1 FP16 184, 163, 171; 2047^2 FP16 51.5, 49.6, 53.7, FP64 58.3, 54.8, 61.3;
// 1023^2 FP16 21.6, -, 20.5.  Several blocks of few waves per CU overlap their
// barriers; 32 by 32 does less halo work and takes 176 at 4095^2).
struct Geo {
    int TX, TY, xtiles, blocks, threads;
    size_t lds;
};
Geo geo(int P, int halo_rows, size_t sa) {
    Geo g;
    g.TX = P >= 512 ? 64 : 32;
    const int SX = g.TX / V + 2;
    // rows by threads, and by the 64 KB of LDS of two tiles (FP64)
    const int lds_rows = (int)((65536 - 512) / (2 * (g.TX + 4 * V) * sa)) - 2;
    const int most = (std::min(kThreads / SX, lds_rows) - halo_rows) & ~1;
    g.TY = std::max(2, std::min(P >= 2048 ? 20 : P >= 512 ? 16 : 8, most));
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
    a.P = t.P, a.pc = t.pc, a.nu = t.nu, a.TX = g.TX, a.TY = g.TY, a.xtiles = g.xtiles;
    a.k = t.q1 ? t.omega * 0.375 : t.omega / 4.0;
#define MG_DOWN(OP)                                                       \
    (f64                 ? k_tile2d_down<OP, P_F64>                       \
     : t.prec == P_F16   ? k_tile2d_down<OP, P_F16>                       \
     : t.prec == P_BF16  ? k_tile2d_down<OP, P_BF16>                      \
                         : k_tile2d_down<OP, P_F32>)
    auto fn = t.q1 ? MG_DOWN(1) : MG_DOWN(0);
#undef MG_DOWN
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
    a.P = t.P, a.pc = t.pc, a.nu = t.nu, a.TX = g.TX, a.TY = g.TY, a.xtiles = g.xtiles;
    a.k = t.q1 ? t.omega * 0.375 : t.omega / 4.0;
#define MG_UP(OP, PF) (upd ? k_tile2d_up<OP, PF, true> : k_tile2d_up<OP, PF, false>)
#define MG_UPS(OP) \
    (f64 ? MG_UP(OP, P_F64) : t.prec == P_F16 ? MG_UP(OP, P_F16) : t.prec == P_BF16 ? MG_UP(OP, P_BF16) : MG_UP(OP, P_F32))
    auto fn = t.q1 ? MG_UPS(1) : MG_UPS(0);
#undef MG_UPS
#undef MG_UP
    hipLaunchKernelGGL(fn, dim3(g.blocks), dim3(g.threads), g.lds, st, a);
    return hipGetLastError();
}

}  // namespace mg

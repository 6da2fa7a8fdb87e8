// Reverse-mode kernels of the SIPF-PIC step along a fixed noise path.
//
// Forward step n (Algorithm 4, split form):
//   Y = X + s Z-,  v = I*G(Y),  X' = wrap(Y + chi tau v + s Z+),
// with G the filtered gradient grids of alpha^(n-1) and phi = I(X) the deposit.
// Reverse, with Xbar' the cotangent of X' (floor() locally constant, wrap = id):
//   chibar += tau Xbar'.v,   vbar = chi tau Xbar',   Ybar = Xbar' + J^T vbar,
//   sbar   += Xbar'.Z+ + Ybar.Z-,   Gbar += I(vbar at Y)   (transpose of I*,
//   the adjoint relation <I rho, f> = <rho, I* f> of Sec. 3.1),
//   Xbar   = Ybar + (M0/P)(H/L) sum_gamma phibar[g + gamma] dF_gamma/dlambda.
// Euler-Maruyama (eq. rho_hat_update): Y = X, sbar += Xbar'.Z.
// Cotangents of positions are stored by original particle id.
#include <climits>

#include "internal.h"
#include "pass_common.h"
#include "sipf.h"

namespace sipf {

// Four nodes p[u][v] of a square with trilinear weights (1 - lu, lu) x (1 - lv, lv):
// the interpolated value and its derivatives by lu and lv.
template <typename T> struct Quad {
    T q, u, v;
    __device__ __forceinline__ Quad(T p00, T p01, T p10, T p11, T lu, T lv) {
        const T d0 = p01 - p00, d1 = p11 - p10;
        const T r0 = p00 + lv * d0, r1 = p10 + lv * d1;
        u = r1 - r0;
        q = r0 + lu * u;
        v = d0 + lu * (d1 - d0);
    }
};

// sum over the 32 nodes of Gamma_4 of phibar[node] * dF/dlambda (eq. 4ord), as
// a contraction along one axis after the other: node(i, j, k) is the value at
// cell offsets (i - 1, j - 1, k - 1), l the position in the cell.
template <typename T, typename Node>
__device__ __forceinline__ void deposit_grad(Node node, const T* l, T& ax, T& ay, T& az) {
    T F[3][2], D[3][2], dS[3], S = (T)1;  // weights of the outer nodes 0 and 3 and their derivatives
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const T om = (T)1 - l[a], lo = l[a] * om;
        F[a][0] = -((T)2 - l[a]) * lo * (T)(1.0 / 6.0);
        F[a][1] = -((T)1 + l[a]) * lo * (T)(1.0 / 6.0);
        D[a][0] = -((T)2 - (T)6 * l[a] + (T)3 * l[a] * l[a]) * (T)(1.0 / 6.0);
        D[a][1] = -((T)1 - (T)3 * l[a] * l[a]) * (T)(1.0 / 6.0);
        S += lo * (T)0.5;
        dS[a] = ((T)1 - (T)2 * l[a]) * (T)0.5;
    }
    {  // inner nodes: F = X Y Z S
        const Quad<T> a(node(1, 1, 1), node(1, 1, 2), node(1, 2, 1), node(1, 2, 2), l[1], l[2]);
        const Quad<T> b(node(2, 1, 1), node(2, 1, 2), node(2, 2, 1), node(2, 2, 2), l[1], l[2]);
        const T dx = b.q - a.q, v = a.q + l[0] * dx;
        ax = dx * S + v * dS[0];
        ay = (a.u + l[0] * (b.u - a.u)) * S + v * dS[1];
        az = (a.v + l[0] * (b.v - a.v)) * S + v * dS[2];
    }
    // outer nodes: F = X Y Z with one index in {0, 3}
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        const int e = o ? 3 : 0;
        const Quad<T> x(node(e, 1, 1), node(e, 1, 2), node(e, 2, 1), node(e, 2, 2), l[1], l[2]);
        ax += D[0][o] * x.q;
        ay += F[0][o] * x.u;
        az += F[0][o] * x.v;
        const Quad<T> y(node(1, e, 1), node(1, e, 2), node(2, e, 1), node(2, e, 2), l[0], l[2]);
        ax += F[1][o] * y.u;
        ay += D[1][o] * y.q;
        az += F[1][o] * y.v;
        const Quad<T> z(node(1, 1, e), node(1, 2, e), node(2, 1, e), node(2, 2, e), l[0], l[1]);
        ax += F[2][o] * z.u;
        ay += F[2][o] * z.v;
        az += D[2][o] * z.q;
    }
}

// The same from the whole grid of H^3 nodes (a power of two), around cell g.
template <typename T>
__device__ __forceinline__ void deposit_grad_grid(const T* __restrict__ phibar, int H, const int* g, const T* l, T& ax,
                                                  T& ay, T& az) {
    const int Hm = H - 1;
    const auto p = gp(phibar);
    deposit_grad(
        [&](int i, int j, int k) -> T {
            const int ix = (g[0] - 1 + i) & Hm, iy = (g[1] - 1 + j) & Hm, iz = (g[2] - 1 + k) & Hm;
            return p[((size_t)ix * H + iy) * H + iz];
        },
        l, ax, ay, az);
}

template <typename T> __device__ __forceinline__ void cell_of(const T* X, T hl, int* g, T* l) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const T s = X[d] * hl, f = floor(s);
        g[d] = (int)f;
        l[d] = s - f;
    }
}

template <typename T>
__global__ __launch_bounds__(256) void k_adj_seed(AdjDesc<T> a) {
    const T c = a.wmass * a.hl;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.P; i += (int64_t)gridDim.x * blockDim.x) {
        const T X[3] = {a.x[i], a.y[i], a.z[i]};
        T gx, gy, gz, l[3];
        int g[3];
        cell_of(X, a.hl, g, l);
        deposit_grad_grid(a.phibar, a.H, g, l, gx, gy, gz);
        const size_t p = a.id[i];
        a.xbar[3 * p] = c * gx;
        a.xbar[3 * p + 1] = c * gy;
        a.xbar[3 * p + 2] = c * gz;
    }
}

__device__ __forceinline__ double block_sum(double v, double* sh) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();
    if (lane == 0) sh[w] = v;
    __syncthreads();
    double t = 0;
    if (threadIdx.x == 0)
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += sh[i];
    return t;
}

// ---------------------------------------------------------------------------
// Reverse particle pass over the work items of a tile sort (one item = up to
// AdjShape<T>::PT x PPT particles of one tile, consecutive in the segment's
// order).  Per item, windows of the grid around the cells of X:
//   G window     the gradient grids, staged once from HBM (gather of v, J at
//                Y = X + W^-);
//   Gbar window  fixed-point accumulators of the transpose of the gather,
//                added to the grid once per item instead of once per particle;
//   phibar window the deposit cotangent, for the transpose of the deposit at X.
// Windows have fixed strides and at most as many cells as these allow: where
// the item's box is wider (particles drift out of their tile over a segment),
// the window keeps to the item's middle and the few particles outside go
// straight to HBM (gathers, float atomics).
// ---------------------------------------------------------------------------
// Launch shape per precision: threads per workgroup, particles per thread (an
// item holds up to PT x PPT particles), waves per SIMD that the registers are
// budgeted for, nodes per axis of the gradient windows (G) and of the phibar
// window (D).
//
// What bounds the pass: the windows' staging and their float atomics into the
// grid once per item, LDS atomics (24 per particle) and latency; its 124 bytes
// per FP64 particle alone would take 52 us at P = 2e6.  Contracting along one
// axis after the other and one gradient component at a time keeps the
// registers at 108 (FP32) and 155 (FP64) without spills, where all 24 node
// values at once took 168 and 256 with spills: two 512-thread workgroups per CU
// in FP32, one of 768 in FP64 (1024 threads spill, 168 us; two of 512 with
// windows of 11 nodes 216, since the particles drift about a cell over a
// segment; 768 160).  Adjoint workload (P = 2e6, H = 64, segments of ten
// steps), us per launch: FP64 277 -> 160, FP32 161 -> 83.
template <typename T> struct AdjShape;
template <> struct AdjShape<float> { static constexpr int PT = 512, PPT = 8, WAVES = 4, G = 13, D = 15; };
template <> struct AdjShape<double> { static constexpr int PT = 768, PPT = 6, WAVES = 3, G = 14, D = 13; };

// Gbar accumulator: a term t (already scaled by 2^S) is added as round(t).  FP32:
// S per item such that a node sum stays below 2^E, a little under the integers'
// range for the terms' rounding (2^-16 of the bound, at least 2^15; half a unit for
// each of up to 4096 particles is 2^11).  FP64: each term below 2^E, the quick
// rounding's range; a sum of 4096 stays below 2^62 (a scale for the sum costs items
// of 4096 twelve bits: error of dL/dX0 against 64 bits, P = 5e5, H = 64, 1.2e-14
// instead of 2.8e-15).
template <typename T> struct AdjFixed;
template <> struct AdjFixed<float> {
    using I = int32_t;
    using U = uint32_t;
    static constexpr int E = 31;
    __device__ static double bound(int cnt, double term) { return (double)cnt * term * (1.0 + 0x1p-16); }
    __device__ static U q(float t) { return (U)(int32_t)rintf(t); }
};
template <> struct AdjFixed<double> {
    using I = long long;
    using U = unsigned long long;
    static constexpr int E = 50;
    __device__ static double bound(int, double term) { return term; }
    __device__ static U q(double t) { return (U)Magic<double>::take(t + Magic<double>::M); }
};

template <typename T> constexpr int adj_lds_bytes() {
    using A = AdjShape<T>;
    return 3 * A::G * A::G * A::G * (int)(sizeof(typename AdjFixed<T>::I) + sizeof(T)) + A::D * A::D * A::D * (int)sizeof(T);
}

template <typename T, int SCHEME>
__device__ __forceinline__ void adj_item(const AdjDesc<T>& a, int64_t beg, int cnt, unsigned char* lds, int4* sh,
                                         const Ticket& ticket, double& chib, double& sb) {
    using I = typename AdjFixed<T>::I;
    using U = typename AdjFixed<T>::U;
    constexpr int APT = AdjShape<T>::PT, APPT = AdjShape<T>::PPT, NW = APT / 64;
    constexpr int G = AdjShape<T>::G, G2 = G * G, G3 = G2 * G, D = AdjShape<T>::D, D2 = D * D;
    const int tid = threadIdx.x;
    const int H = a.H, Hm = H - 1, Hh = H / 2;
    const T hl = a.hl;
    const size_t H3 = (size_t)H * H * H;
    // the load phase keeps the particles only long enough for the bounding box
    // and the cotangent bound; the main loop re-reads each one from L2
    const int rx = ifloor(a.x[beg] * hl) & Hm, ry = ifloor(a.y[beg] * hl) & Hm, rz = ifloor(a.z[beg] * hl) & Hm;
    int bx = BOUNDS_NONE, by = BOUNDS_NONE, bz = BOUNDS_NONE, sx = 0, sy = 0, sz = 0;
    float bmax = 0.f;
    // in batches of four particles per thread, to bound the registers held
    constexpr int NB = APPT < 4 ? APPT : 4;
#pragma unroll
    for (int k0 = 0; k0 < APPT; k0 += NB) {
        T px[NB], py[NB], pz[NB], qx[NB], qy[NB], qz[NB];
#pragma unroll
        for (int kk = 0; kk < NB; ++kk) {
            const int j = tid + (k0 + kk) * APT;
            const uint32_t jj = (uint32_t)(j < cnt ? j : cnt - 1);  // in-item index for every lane: branch-free loads
            px[kk] = gp(a.x + beg)[jj];
            py[kk] = gp(a.y + beg)[jj];
            pz[kk] = gp(a.z + beg)[jj];
            qx[kk] = gp(a.xbx + beg)[jj];
            qy[kk] = gp(a.xby + beg)[jj];
            qz[kk] = gp(a.xbz + beg)[jj];
        }
#pragma unroll
        for (int kk = 0; kk < NB; ++kk) {
            const int j = tid + (k0 + kk) * APT;
            if (j < cnt) {
                const int cx = (((ifloor(px[kk] * hl) & Hm) - rx + Hh) & Hm) - Hh;
                const int cy = (((ifloor(py[kk] * hl) & Hm) - ry + Hh) & Hm) - Hh;
                const int cz = (((ifloor(pz[kk] * hl) & Hm) - rz + Hh) & Hm) - Hh;
                bx = pk_min(bx, pk_bounds(cx));
                by = pk_min(by, pk_bounds(cy));
                bz = pk_min(bz, pk_bounds(cz));
                sx += cx;
                sy += cy;
                sz += cz;
                // |x| rounded up to float (values beyond float range give +inf)
                const float m3 =
                    (float)fmax(fmax(fabs((double)qx[kk]), fabs((double)qy[kk])), fabs((double)qz[kk]));
                bmax = fmaxf(bmax, m3 * 1.0000002f);
            }
        }
    }
    // non-negative floats order like their bit patterns
    const int bm = block_bounds3_max<NW>(bx, by, bz, __float_as_int(bmax), sh);
    ticket.draw();
    const double bound = AdjFixed<T>::bound(cnt, (double)a.chitau * (double)__int_as_float(bm));
    const bool gwin = bound < 1e300;
    int mx = 0, my = 0, mz = 0;
    if (max(max(pk_hi(bx) - pk_lo(bx), pk_hi(by) - pk_lo(by)), pk_hi(bz) - pk_lo(bz)) >= min(G - 1, D - 3)) {
        // a box wider than a window: the item's mean cell
        __syncthreads();  // the bounds have been read
        int* sum = reinterpret_cast<int*>(sh);
        if (tid < 3) sum[tid] = 0;
        __syncthreads();
        atomicAdd(sum, sx);
        atomicAdd(sum + 1, sy);
        atomicAdd(sum + 2, sz);
        __syncthreads();
        mx = sum[0] / cnt;
        my = sum[1] / cnt;
        mz = sum[2] / cnt;
    }
    // gradient windows (first cell, cells), Gbar then G in LDS; nodes = cells + 1
    int gox, goy, goz, gnx, gny, gnz;
    window_axis(pk_lo(bx), pk_hi(bx), a.gmargin, mx, G - 1, H, gox, gnx);
    window_axis(pk_lo(by), pk_hi(by), a.gmargin, my, G - 1, H, goy, gny);
    window_axis(pk_lo(bz), pk_hi(bz), a.gmargin, mz, G - 1, H, goz, gnz);
    gox = (gox + rx) & Hm;
    goy = (goy + ry) & Hm;
    goz = (goz + rz) & Hm;
    I* Gb = reinterpret_cast<I*>(lds);
    T* Gw = reinterpret_cast<T*>(lds + (size_t)3 * G3 * sizeof(I));
    // deposit-cotangent window: cells of X, order-4 stencil (-1 .. +2) around them
    int dox = 0, doy = 0, doz = 0, dnx = 0, dny = 0, dnz = 0;
    T* Pw = Gw + 3 * G3;
    if (a.phibar != nullptr) {
        window_axis(pk_lo(bx), pk_hi(bx), 0, mx, D - 3, H, dox, dnx);
        window_axis(pk_lo(by), pk_hi(by), 0, my, D - 3, H, doy, dny);
        window_axis(pk_lo(bz), pk_hi(bz), 0, mz, D - 3, H, doz, dnz);
        dox = (dox + rx) & Hm;
        doy = (doy + ry) & Hm;
        doz = (doz + rz) & Hm;
        const int wy = dny + 3, wz = dnz + 3, dn = (dnx + 3) * wy * wz;
        const float inv_y = 1.0f / (float)wy, inv_z = 1.0f / (float)wz;
        for (int e = tid; e < dn; e += APT) {
            int i, j, k;
            unflatten3(e, wy, wz, inv_z, inv_y, i, j, k);
            Pw[i * D2 + j * D + k] =
                gp(a.phibar)[(uint32_t)((((dox - 1 + i) & Hm) * H + ((doy - 1 + j) & Hm)) * H + ((doz - 1 + k) & Hm))];
        }
    }
    const T cdep = a.wmass * hl;
    const int wy = gny + 1, wz = gnz + 1, gn = (gnx + 1) * wy * wz;
    const float inv_y = 1.0f / (float)wy, inv_z = 1.0f / (float)wz;
    if (gwin) {
        for (int e = tid; e < gn; e += APT) {
            int i, j, k;
            unflatten3(e, wy, wz, inv_z, inv_y, i, j, k);
            const uint32_t node = (uint32_t)((((gox + i) & Hm) * H + ((goy + j) & Hm)) * H + ((goz + k) & Hm));
            const int at = i * G2 + j * G + k;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                Gw[d * G3 + at] = gp(a.G + d * H3)[node];
                Gb[d * G3 + at] = 0;
            }
        }
    }
    int e2 = 0;
    if (bound > 0 && gwin) (void)frexp(bound, &e2);  // bound < 2^e2
    const T scale = (T)ldexp(1.0, AdjFixed<T>::E - e2);
    const T back = (T)ldexp(1.0, e2 - AdjFixed<T>::E);
    __syncthreads();

#pragma unroll 1
    for (int k = 0; k < APPT; ++k) {
        const int j = tid + k * APT;
        if (j >= cnt) continue;
        const T X[3] = {gp(a.x + beg)[j], gp(a.y + beg)[j], gp(a.z + beg)[j]};
        const T xb[3] = {gp(a.xbx + beg)[j], gp(a.xby + beg)[j], gp(a.xbz + beg)[j]};
        const uint32_t pidk = gp(a.id + beg)[j];
        T zm[3], zp[3], Y[3], zn[6];
        if (a.zin != nullptr) {
            // the normals kept by the segment's forward recompute
#pragma unroll
            for (int q = 0; q < 6; ++q)
                zn[q] = (SCHEME == SIPF_STRANG || q < 3) ? gp(a.zin + q * a.P + beg)[j] : (T)0;
        } else if (SCHEME == SIPF_STRANG) {
            noise6<3, T>(pidk, a.n, a.inst, a.k0, a.k1, zn);
        } else {
            noise6<2, T>(pidk, a.n, a.inst, a.k0, a.k1, zn);
        }
        if (SCHEME == SIPF_STRANG) {
            for (int d = 0; d < 3; ++d) {
                zm[d] = zn[d];
                zp[d] = zn[3 + d];
                Y[d] = X[d] + a.s * zm[d];
            }
        } else {
            for (int d = 0; d < 3; ++d) {
                zp[d] = zn[d];
                zm[d] = 0;
                Y[d] = X[d];
            }
        }
        int gc[3];
        T l[3];
        cell_of(Y, hl, gc, l);
        const int i0 = (gc[0] - gox) & Hm, j0 = (gc[1] - goy) & Hm, k0 = (gc[2] - goz) & Hm;
        const bool inside = gwin && i0 < gnx && j0 < gny && k0 < gnz;
        const T wyz[4] = {((T)1 - l[1]) * ((T)1 - l[2]), ((T)1 - l[1]) * l[2], l[1] * ((T)1 - l[2]), l[1] * l[2]};
        const T wt[8] = {((T)1 - l[0]) * wyz[0], ((T)1 - l[0]) * wyz[1], ((T)1 - l[0]) * wyz[2], ((T)1 - l[0]) * wyz[3],
                         l[0] * wyz[0],          l[0] * wyz[1],          l[0] * wyz[2],          l[0] * wyz[3]};
        T yb[3] = {xb[0], xb[1], xb[2]}, xv = 0;
        // gradient component d at the cell's nodes: its value and derivatives
        auto component = [&](int d, T vb, auto node) {
            const Quad<T> lo(node(0, 0, 0), node(0, 0, 1), node(0, 1, 0), node(0, 1, 1), l[1], l[2]);
            const Quad<T> hi(node(1, 0, 0), node(1, 0, 1), node(1, 1, 0), node(1, 1, 1), l[1], l[2]);
            const T dx = hi.q - lo.q, vh = vb * hl;
            xv += xb[d] * (lo.q + l[0] * dx);
            yb[0] += vh * dx;
            yb[1] += vh * (lo.u + l[0] * (hi.u - lo.u));
            yb[2] += vh * (lo.v + l[0] * (hi.v - lo.v));
        };
        // two explicit paths, so that LDS reads stay ds_read instructions; the
        // transpose of the gather spreads vbar with the trilinear weights at Y
        if (inside) {
            const int at = i0 * G2 + j0 * G + k0;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const T vb = a.chitau * xb[d], vs = vb * scale;
                const T* g = Gw + d * G3 + at;
                component(d, vb, [&](int ia, int ib, int ic) { return g[ia * G2 + ib * G + ic]; });
                U* b = reinterpret_cast<U*>(Gb + d * G3 + at);
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    atomicAdd(b + (q >> 2) * G2 + ((q >> 1) & 1) * G + (q & 1), AdjFixed<T>::q(wt[q] * vs));
            }
        } else {
            const uint32_t r0 = (gc[0] & Hm) * H * H, r1 = ((gc[0] + 1) & Hm) * H * H;
            const uint32_t c0 = (gc[1] & Hm) * H, c1 = ((gc[1] + 1) & Hm) * H, e0 = gc[2] & Hm, e1 = (gc[2] + 1) & Hm;
            auto at = [&](int ia, int ib, int ic) { return (ia ? r1 : r0) + (ib ? c1 : c0) + (ic ? e1 : e0); };
#pragma unroll 1
            for (int d = 0; d < 3; ++d) {
                const T xd = d == 0 ? xb[0] : (d == 1 ? xb[1] : xb[2]);
                const T vb = a.chitau * xd;
                const auto g = gp(a.G + d * H3);
                const Quad<T> lo(g[at(0, 0, 0)], g[at(0, 0, 1)], g[at(0, 1, 0)], g[at(0, 1, 1)], l[1], l[2]);
                const Quad<T> hi(g[at(1, 0, 0)], g[at(1, 0, 1)], g[at(1, 1, 0)], g[at(1, 1, 1)], l[1], l[2]);
                const T dx = hi.q - lo.q, vh = vb * hl;
                xv += xd * (lo.q + l[0] * dx);
                yb[0] += vh * dx;
                yb[1] += vh * (lo.u + l[0] * (hi.u - lo.u));
                yb[2] += vh * (lo.v + l[0] * (hi.v - lo.v));
                for (int q = 0; q < 8; ++q)
                    gatomic_add(a.Gbar + d * H3 + at(q >> 2, (q >> 1) & 1, q & 1), wt[q] * vb);
            }
        }
        chib += (double)(a.tau * xv);
        if (SCHEME == SIPF_STRANG)
            sb += (double)(xb[0] * zp[0] + xb[1] * zp[1] + xb[2] * zp[2] + yb[0] * zm[0] + yb[1] * zm[1] +
                           yb[2] * zm[2]);
        else
            sb += (double)(xb[0] * zp[0] + xb[1] * zp[1] + xb[2] * zp[2]);
        // transpose of the deposit at X
        if (a.phibar != nullptr) {
            T dg[3];
            cell_of(X, hl, gc, l);
            const int di = (gc[0] - dox) & Hm, dj = (gc[1] - doy) & Hm, dk = (gc[2] - doz) & Hm;
            if (di < dnx && dj < dny && dk < dnz) {
                const T* p = Pw + di * D2 + dj * D + dk;
                deposit_grad([&](int i, int j, int k) { return p[i * D2 + j * D + k]; }, l, dg[0], dg[1], dg[2]);
            } else {
                deposit_grad_grid(a.phibar, H, gc, l, dg[0], dg[1], dg[2]);
            }
#pragma unroll
            for (int d = 0; d < 3; ++d) yb[d] += cdep * dg[d];
        }
        gp(a.xbx + beg)[j] = yb[0];
        gp(a.xby + beg)[j] = yb[1];
        gp(a.xbz + beg)[j] = yb[2];
    }
    __syncthreads();
    if (gwin) {
        for (int e = tid; e < gn; e += APT) {
            int i, j, k;
            unflatten3(e, wy, wz, inv_z, inv_y, i, j, k);
            const uint32_t node = (uint32_t)((((gox + i) & Hm) * H + ((goy + j) & Hm)) * H + ((goz + k) & Hm));
            const int at = i * G2 + j * G + k;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const I val = Gb[d * G3 + at];
                if (val != 0) gatomic_add(a.Gbar + d * H3 + node, (T)val * back);
            }
        }
    }
}

__device__ __forceinline__ double block_sum_n(double v, double* sh, int nthreads) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();
    if (lane == 0) sh[w] = v;
    __syncthreads();
    double t = 0;
    if (threadIdx.x == 0)
        for (int i = 0; i < nthreads / 64; ++i) t += sh[i];
    return t;
}

template <typename T, int SCHEME>
__global__ __launch_bounds__(AdjShape<T>::PT) __attribute__((amdgpu_waves_per_eu(AdjShape<T>::WAVES))) void k_adj_items(
    AdjDesc<T> a, const WorkItem* __restrict__ items, int* hdr) {
    constexpr int APT = AdjShape<T>::PT;
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ int4 sh[APT / 64];
    __shared__ int slot;
    __shared__ double shd[APT / 64];
    const int n = hdr[0];
    double chib = 0, sb = 0;
    const Ticket ticket{hdr, n, &slot};
    for (int it = blockIdx.x; it < n; it = ticket.next()) {
        const WorkItem w = items[it];
        adj_item<T, SCHEME>(a, w.beg, w.cnt, lds, sh, ticket, chib, sb);
    }
    __syncthreads();
    const double tc = block_sum_n(chib, shd, APT);
    const double ts = block_sum_n(sb, shd, APT);
    if (threadIdx.x == 0) {
        atomicAdd(a.acc, tc);
        atomicAdd(a.acc + 1, ts);
    }
}

template <typename T>
__global__ void k_copy_positions(T* x, T* y, T* z, uint32_t* id, const T* __restrict__ sx, const T* __restrict__ sy,
                                 const T* __restrict__ sz, const uint32_t* __restrict__ sid, int64_t P) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < P; i += (int64_t)gridDim.x * blockDim.x) {
        x[i] = sx[i];
        y[i] = sy[i];
        z[i] = sz[i];
        id[i] = sid[i];
    }
}

template <typename T>
__global__ void k_xbar_order(T* xbar, T* bx, T* by, T* bz, const uint32_t* __restrict__ id, int64_t P, int to_order) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < P; i += (int64_t)gridDim.x * blockDim.x) {
        const size_t p = id[i];
        if (to_order) {
            bx[i] = xbar[3 * p];
            by[i] = xbar[3 * p + 1];
            bz[i] = xbar[3 * p + 2];
        } else {
            xbar[3 * p] = bx[i];
            xbar[3 * p + 1] = by[i];
            xbar[3 * p + 2] = bz[i];
        }
    }
}

__global__ void k_iota_u32(uint32_t* p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = (uint32_t)i;
}

template <typename T>
__global__ __launch_bounds__(256) void k_dot(const T* __restrict__ u, const T* __restrict__ v, int64_t n, double* out) {
    __shared__ double sh[8];
    double s = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        s += (double)u[i] * (double)v[i];
    const double t = block_sum(s, sh);
    if (threadIdx.x == 0) atomicAdd(out, t);
}

template <typename T> __global__ void k_axpby(T* y, const T* x, T a, T b, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        y[i] = a * x[i] + b * y[i];
}

__global__ void k_set_u32(uint32_t* p, uint32_t v) { *p = v; }
__global__ void k_zero_f64(double* p, int n) {
    if ((int)threadIdx.x < n) p[threadIdx.x] = 0.0;
}

static int grid_for(int64_t n) {
    const int64_t b = (n + 255) / 256;
    return (int)(b < 8192 ? (b > 0 ? b : 1) : 8192);
}

template <typename T> hipError_t launch_adj_seed(const AdjDesc<T>& a, hipStream_t s) {
    hipLaunchKernelGGL((k_adj_seed<T>), dim3(grid_for(a.P)), dim3(256), 0, s, a);
    return hipGetLastError();
}
// Workgroups of the reverse pass that the device holds at once
template <typename T> int adj_resident_blocks(int scheme) {
    const void* k = scheme == SIPF_STRANG ? (const void*)k_adj_items<T, SIPF_STRANG> : (const void*)k_adj_items<T, SIPF_EM>;
    int per_cu = 0, dev = 0, cus = 0;
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, adj_lds_bytes<T>());
    if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, AdjShape<T>::PT, adj_lds_bytes<T>());
    if (e == hipSuccess) e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess || per_cu < 1 || cus < 1) {
        (void)hipGetLastError();
        return 256;
    }
    return per_cu * cus;
}
template <typename T>
hipError_t launch_adj_items(const AdjDesc<T>& a, const WorkItem* items, int* nitems, int grid, hipStream_t s) {
    if (grid <= 0) return hipSuccess;
    constexpr int APT = AdjShape<T>::PT;
    if (particle_chunk() > APT * AdjShape<T>::PPT) return hipErrorInvalidValue;  // an item must fit one workgroup
    auto k = a.scheme == SIPF_STRANG ? k_adj_items<T, SIPF_STRANG> : k_adj_items<T, SIPF_EM>;
    hipLaunchKernelGGL(k, dim3(grid), dim3(APT), adj_lds_bytes<T>(), s, a, items, nitems);
    return hipGetLastError();
}
template <typename T>
hipError_t launch_copy_positions(T* x, T* y, T* z, uint32_t* id, const T* sx, const T* sy, const T* sz,
                                 const uint32_t* sid, int64_t P, hipStream_t s) {
    hipLaunchKernelGGL((k_copy_positions<T>), dim3(grid_for(P)), dim3(256), 0, s, x, y, z, id, sx, sy, sz, sid, P);
    return hipGetLastError();
}
template <typename T>
hipError_t launch_xbar_order(T* xbar, T* bx, T* by, T* bz, const uint32_t* id, int64_t P, bool to_order,
                             hipStream_t s) {
    hipLaunchKernelGGL((k_xbar_order<T>), dim3(grid_for(P)), dim3(256), 0, s, xbar, bx, by, bz, id, P,
                       to_order ? 1 : 0);
    return hipGetLastError();
}
hipError_t launch_iota_u32(uint32_t* p, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_iota_u32, dim3(grid_for(n)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}
template <typename T> hipError_t launch_dot(const T* u, const T* v, int64_t n, double* out, hipStream_t s) {
    hipLaunchKernelGGL((k_dot<T>), dim3(grid_for(n)), dim3(256), 0, s, u, v, n, out);
    return hipGetLastError();
}
template <typename T> hipError_t launch_axpby(T* y, const T* x, T a, T b, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL((k_axpby<T>), dim3(grid_for(n)), dim3(256), 0, s, y, x, a, b, n);
    return hipGetLastError();
}
hipError_t launch_set_u32(uint32_t* p, uint32_t v, hipStream_t s) {
    hipLaunchKernelGGL(k_set_u32, dim3(1), dim3(1), 0, s, p, v);
    return hipGetLastError();
}
hipError_t launch_zero_f64(double* p, int n, hipStream_t s) {
    hipLaunchKernelGGL(k_zero_f64, dim3(1), dim3(64), 0, s, p, n);
    return hipGetLastError();
}

#define SIPF_ADJ_INST(T)                                                                \
    template int adj_resident_blocks<T>(int);                                                   \
    template hipError_t launch_adj_seed<T>(const AdjDesc<T>&, hipStream_t);            \
    template hipError_t launch_adj_items<T>(const AdjDesc<T>&, const WorkItem*, int*, int, hipStream_t); \
    template hipError_t launch_copy_positions<T>(T*, T*, T*, uint32_t*, const T*, const T*, const T*,          \
                                                 const uint32_t*, int64_t, hipStream_t);                       \
    template hipError_t launch_xbar_order<T>(T*, T*, T*, T*, const uint32_t*, int64_t, bool, hipStream_t);     \
    template hipError_t launch_dot<T>(const T*, const T*, int64_t, double*, hipStream_t); \
    template hipError_t launch_axpby<T>(T*, const T*, T, T, int64_t, hipStream_t);
SIPF_ADJ_INST(float)
SIPF_ADJ_INST(double)

}  // namespace sipf

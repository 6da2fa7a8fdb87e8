// Field passes of the two-dimensional step (the 2-D runs of Sec. 5.2):
// real-to-complex 2-D FFT of the deposit, the implicit (or, with eps = 0,
// elliptic) mode update, the filtered spectral gradient and the
// complex-to-real inverse FFT of its two components.
//
// Convention: beta_q = L^-2 sum_j phi_j e^{-2 pi i q.j/H},
// grad c(x_j) = sum_q i xi_q Phi_q alpha_q e^{+2 pi i q.j/H}.
//
// Grid sizes H = 8 .. 4096 (a row of 4096 complex values fits in LDS).  Three
// passes per step, each staged through LDS:
//   fwd_rows  R rows of phi per workgroup: each real row along y is read as
//             H/2 complex values, transformed and split into its half
//             spectrum (ky = 0..H/2), which is written ky-major in blocks of K
//             frequencies (below).  Clears the deposit and advances the step
//             counter.
//   xrows     one workgroup per K frequencies ky: transform along x, update
//             alpha, form i xi_d Phi alpha for d = x, y and inverse-transform
//             each along x.
//   inv_rows  R rows per workgroup and component: gather the ky-major
//             spectrum, half-length complex-to-real inverse along y.
//
// What bounds them: memory.  The spectra between the passes (B1, gspec) hold
// frequency ky of row x at (ky / K) H K + x K + ky % K, so a row pass moves
// runs of R K values (64 bytes at H = 2048 with K = 2 in place of 32, 128 at
// H = 512 and 1024) and an x pass one contiguous block.  Transforms above 256
// values (Fft16) read and write HBM from their first and last stages, and the
// modes stay in registers between the forward and the inverse x transform.
// Each pass issues all of a thread's loads before it computes its twiddles
// and writes LDS.  H = 2048, FP32, us per launch, before and after: forward 29.3
// -> 11.7, x rows 57.4 -> 29.3, inverse 61.1 -> 21.9 (H = 4096, the whole step
// at P = 1e5, 637 -> 358).
#include <algorithm>

#include "internal.h"
#include "lds_fft.h"
#include "pass_common.h"

namespace sipf {

constexpr int ROW_THREADS = 512;

// rows per workgroup of the row passes and frequencies per workgroup of the x
// pass, within LDS together with an H-entry twiddle table
template <typename T, int H> struct Rows2 {
    static constexpr bool F32 = sizeof(T) == 4;
    static constexpr int R = H <= 16 ? H : (H <= 512 ? 16 : (H == 1024 ? 8 : (H == 2048 ? 4 : (F32 ? 4 : 2))));
    static constexpr int K = F32 && H >= 1024 ? 2 : 1;
    static constexpr int HH = H / 2 + 1;
    static constexpr int NKB = (HH + K - 1) / K;  // blocks of K frequencies, the last may be partial
    static constexpr size_t SPEC = (size_t)NKB * K * H;  // values of one blocked spectrum
};
size_t blocked_spec2(int H) { return (size_t)(H / 2 + 1 + 1) / 2 * 2 * H; }  // the largest K is 2

// Half-length transform of a row pass.  Above 256 values Fft16, whose groups
// leave and enter through the natural order of LDS row r: value k at r OP + k
// + k / 16 (the padding keeps the groups' writes, 16 apart, on separate banks).
template <typename T, int H> struct RowFft {
    static constexpr int M = H / 2, R = Rows2<T, H>::R;
    static constexpr bool BIG = M > 256;
    using F = Fft16<T, BIG ? M : 512>;
    static constexpr int OP = BIG ? M + M / 16 + 1 : M + 1;  // row pitch in natural order
    static constexpr int SIZE = BIG && F::LEN > OP ? R * F::LEN : R * OP;
    static constexpr int NG = BIG ? (R * F::G3 + ROW_THREADS - 1) / ROW_THREADS : 1;  // groups per thread
    __device__ __forceinline__ static int at(int r, int k) { return r * OP + (BIG ? k + k / 16 : k); }
};

enum { XR_STEP = 0, XR_GRAD = 1, XR_RHO = 4 };

template <typename T, int H>
__global__ __launch_bounds__(ROW_THREADS) void k2_fwd_rows(const FieldDesc<T>* __restrict__ fds, int consume) {
    using V = cplx_t<T>;
    using RF = RowFft<T, H>;
    constexpr int M = H / 2, HH = M + 1, R = Rows2<T, H>::R;
    __shared__ V buf[RF::SIZE];
    __shared__ V tw[H];
    const FieldDesc<T>& fd = fds[blockIdx.y];
    const int ix0 = blockIdx.x * R;
    const int tid = threadIdx.x;
    V* rows = reinterpret_cast<V*>(fd.phi + (size_t)ix0 * H);  // (x[2m], x[2m+1]) of row r at r M + m
    if (consume && blockIdx.x == 0 && tid == 0 && fd.step != nullptr) *fd.step += 1u;
    if constexpr (RF::BIG) {
        using F = typename RF::F;
        static_assert(R * F::M <= ROW_THREADS, "one first-stage item per thread");
        const int b = tid / F::M, m = tid % F::M;
        V r[16];
        if (tid < R * F::M) {
#pragma unroll
            for (int i = 0; i < 16; ++i) r[i] = ldg(rows + b * M + m + F::M * i);
        }
        make_twiddles<T, H>(tw);
        __syncthreads();
        if (tid < R * F::M) {
            if (consume) {
#pragma unroll
                for (int i = 0; i < 16; ++i) stg(rows + b * M + m + F::M * i, cmake<V, T>(0, 0));
            }
            F::first(buf + b * F::LEN, tw, 2, m, r);
        }
        __syncthreads();
        F::template middle<R, -1>(buf, tw, 2);
        __syncthreads();
        V z[RF::NG][F::N2];
#pragma unroll
        for (int q = 0; q < RF::NG; ++q)
            if (tid + q * ROW_THREADS < R * F::G3) F::load_group(buf, tid + q * ROW_THREADS, z[q]);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < RF::NG; ++q) {
            const int g = tid + q * ROW_THREADS;
            if (g < R * F::G3) {
#pragma unroll
                for (int i = 0; i < F::N2; ++i)
                    buf[RF::at(g / F::G3, F::k1_of(g) + 16 * (F::j1_of(g) + F::N1 * i))] = z[q][i];
            }
        }
    } else {
        constexpr int NL = (R * M + ROW_THREADS - 1) / ROW_THREADS;
        V v[NL];
#pragma unroll
        for (int q = 0; q < NL; ++q) v[q] = ldg(rows + min(tid + q * ROW_THREADS, R * M - 1));
        make_twiddles<T, H>(tw);
#pragma unroll
        for (int q = 0; q < NL; ++q) {
            const int u = tid + q * ROW_THREADS;
            if (u < R * M) buf[RF::at(u / M, u % M)] = v[q];
        }
        __syncthreads();
        if (consume)
            for (int u = tid; u < R * M; u += ROW_THREADS) stg(rows + u, cmake<V, T>(0, 0));
        fft_2s<T, Split<M>::N1, Split<M>::N2, -1>(buf, R, 1, RF::OP, 0, 1, tw, 2);
    }
    __syncthreads();
    // X_k = E_k + w_H^k O_k from Z_k and Z_{M-k}, as it is written
    auto z_at = [&](int r, int k) { return buf[RF::at(r, RF::BIG ? k : perm_pos_g<M>(k))]; };
    constexpr int K = Rows2<T, H>::K;
    V* out = fd.B1 + (size_t)ix0 * K;
    for (int u = tid; u < Rows2<T, H>::NKB * R * K; u += ROW_THREADS) {
        const int kb = u / (R * K), e = u % (R * K);
        const int r = e / K, k = kb * K + e % K;
        if (k < HH) {
            const V za = z_at(r, k % M), zc = cconj(z_at(r, (M - k) % M));
            const V ev = cscale(cadd(za, zc), (T)0.5);
            const V dd = csub(za, zc);
            const V o = cmake<V, T>(dd.y * (T)0.5, -dd.x * (T)0.5);  // (Z_k - conj Z_{M-k}) / (2i)
            stg(out + (size_t)kb * H * K + e, cadd(ev, cmul(tw[k], o)));
        }
    }
}

// mode update of one mode: new alpha (STEP) and Phi alpha
template <typename T, int H, int MODE>
__device__ __forceinline__ cplx_t<T> mode2(const FieldDesc<T>& fd, cplx_t<T>& a, const cplx_t<T>& beta, int kx, int ky) {
    using V = cplx_t<T>;
    const T qx = (T)(kx < H / 2 ? kx : kx - H), qy = (T)ky;
    const T q2 = qx * qx + qy * qy;
    if constexpr (MODE == XR_STEP) {
        T A, B;
        mode_ab(fd, q2 * fd.two_pi_over_L * fd.two_pi_over_L + fd.k2, A, B);
        const T bs = B * fd.inv_Ld;
        a = cmake<V, T>(A * a.x + bs * beta.x, A * a.y + bs * beta.y);
    }
    return cscale(a, fd.filt > (T)0 ? exp(-fd.filt * q2) : (T)1);
}
// i xi_d times a, zero at the Nyquist frequency |q_d| = H/2
template <typename T, int H> __device__ __forceinline__ cplx_t<T> ixi(const FieldDesc<T>& fd, int kd, const cplx_t<T>& a) {
    const T q = (T)(kd == H / 2 ? 0 : (kd < H / 2 ? kd : kd - H));
    const T xi = q * fd.two_pi_over_L;
    return cmake<cplx_t<T>, T>(-xi * a.y, xi * a.x);
}

// Threads of the x pass: one group of frequencies each, the group whose modes the
// thread carries from the forward to the inverse transform, and at least two waves.
// (Half as many at H = 2048, one per middle-stage item, two groups each: the
// critical-mass run 155 instead of 152 us per step, FP64 172 instead of 162.)
template <typename T, int H> constexpr int xrow_threads() {
    if constexpr (H > 256) return std::max(128, Rows2<T, H>::K * Fft16<T, H>::G3);
    else return 256;
}

template <typename T, int H, int MODE>
__global__ __launch_bounds__((xrow_threads<T, H>())) void k2_xrows(const FieldDesc<T>* __restrict__ fds) {
    using V = cplx_t<T>;
    constexpr int K = Rows2<T, H>::K, HH = H / 2 + 1;
    constexpr int NT = xrow_threads<T, H>();
    const FieldDesc<T>& fd = fds[blockIdx.y];
    const int k0 = blockIdx.x * K;
    const int tid = threadIdx.x;
    const V* in = fd.B1 + (size_t)k0 * H;      // element (x, b) at x K + b
    V* const out = fd.gspec + (size_t)k0 * H;
    constexpr int NCOMP = MODE == XR_RHO ? 1 : 2;
    __shared__ V tw[H];
    if constexpr (H > 256) {
        using F = Fft16<T, H>;
        constexpr int NG = (K * F::G3 + NT - 1) / NT;   // groups per thread
        constexpr int NF = (K * F::M + NT - 1) / NT;    // first- and last-stage items per thread
        __shared__ V buf[K * F::LEN];
        // alpha of the thread's groups (storage position k1 M + j1 + N1 i), B1 in flight at the same time
        V al[NG][F::N2];
        auto al_at = [&](int g, int i) {
            return (size_t)min(k0 + g / F::G3, HH - 1) * H + F::k1_of(g) * F::M + F::j1_of(g) + F::N1 * i;
        };
        if constexpr (MODE != XR_RHO) {
#pragma unroll
            for (int q = 0; q < NG; ++q)
#pragma unroll
                for (int i = 0; i < F::N2; ++i) al[q][i] = ldg(fd.alpha + al_at(min(tid + q * NT, K * F::G3 - 1), i));
        }
        if constexpr (MODE != XR_GRAD) {
            V r[NF][16];
#pragma unroll
            for (int q = 0; q < NF; ++q) {
                const int u = min(tid + q * NT, K * F::M - 1);
#pragma unroll
                for (int i = 0; i < 16; ++i) r[q][i] = ldg(in + (size_t)(u / K + F::M * i) * K + u % K);
            }
            make_twiddles<T, H>(tw);
            __syncthreads();
#pragma unroll
            for (int q = 0; q < NF; ++q) {
                const int u = tid + q * NT;
                if (u < K * F::M) F::first(buf + (u % K) * F::LEN, tw, 1, u / K, r[q]);
            }
            __syncthreads();
            F::template middle<K, -1>(buf, tw, 1);
            __syncthreads();
        } else {
            make_twiddles<T, H>(tw);
            __syncthreads();
        }
#pragma unroll
        for (int q = 0; q < NG; ++q) {
            const int g = tid + q * NT;
            if (g < K * F::G3) {
                V z[F::N2];
                if constexpr (MODE != XR_GRAD) F::load_group(buf, g, z);
                const int ky = k0 + g / F::G3;
#pragma unroll
                for (int i = 0; i < F::N2; ++i) {
                    const int kx = F::k1_of(g) + 16 * (F::j1_of(g) + F::N1 * i);
                    if constexpr (MODE == XR_RHO) {
                        V b = z[i];
                        al[q][i] = cscale(mode2<T, H, MODE>(fd, b, b, kx, ky), fd.inv_Ld);
                    } else {
                        V a = al[q][i];
                        al[q][i] = mode2<T, H, MODE>(fd, a, z[i], kx, ky);
                        if (MODE == XR_STEP && ky < HH) stg(fd.alpha + al_at(g, i), a);
                    }
                }
            }
        }
#pragma unroll 1
        for (int d = 0; d < NCOMP; ++d) {
            if (d > 0) __syncthreads();  // the previous component has been read
#pragma unroll
            for (int q = 0; q < NG; ++q) {
                const int g = tid + q * NT;
                if (g < K * F::G3) {
                    V z[F::N2];
#pragma unroll
                    for (int i = 0; i < F::N2; ++i) {
                        const int kx = F::k1_of(g) + 16 * (F::j1_of(g) + F::N1 * i);
                        z[i] = MODE == XR_RHO ? al[q][i] : ixi<T, H>(fd, d == 0 ? kx : k0 + g / F::G3, al[q][i]);
                    }
                    F::store_group(buf, g, z, tw, 1);
                }
            }
            __syncthreads();
            F::template middle<K, +1>(buf, tw, 1);
            __syncthreads();
            V* o = out + d * Rows2<T, H>::SPEC;
#pragma unroll
            for (int q = 0; q < NF; ++q) {
                const int u = tid + q * NT;
                if (u < K * F::M) {
                    V r[16];
                    F::last(buf + (u % K) * F::LEN, tw, 1, u / K, r);
                    if (k0 + u % K < HH) {
#pragma unroll
                        for (int i = 0; i < 16; ++i) stg(o + (size_t)(u / K + F::M * i) * K + u % K, r[i]);
                    }
                }
            }
        }
    } else {
        static_assert(K == 1 && H <= NT, "one value per thread");
        constexpr int N1 = Split<H>::N1, N2 = Split<H>::N2;
        __shared__ V buf[H];
        const bool ok = tid < H;
        const size_t row = (size_t)k0 * H;
        V a = cmake<V, T>(0, 0), b = a;
        if (MODE != XR_RHO && ok) a = ldg(fd.alpha + row + tid);
        if (MODE != XR_GRAD && ok) b = ldg(in + tid);
        make_twiddles<T, H>(tw);
        if constexpr (MODE != XR_GRAD) {
            if (ok) buf[tid] = b;
            __syncthreads();
            fft_2s<T, N1, N2, -1>(buf, 1, 1, H, 0, 1, tw, 1);
            __syncthreads();
            if (ok) b = buf[tid];
        }
        const int kx = perm_freq_g<H>(ok ? tid : 0);
        if constexpr (MODE == XR_RHO) {
            a = cscale(mode2<T, H, MODE>(fd, b, b, kx, k0), fd.inv_Ld);
        } else {
            V na = a;
            a = mode2<T, H, MODE>(fd, na, b, kx, k0);
            if (MODE == XR_STEP && ok) stg(fd.alpha + row + tid, na);
        }
        for (int d = 0; d < NCOMP; ++d) {
            __syncthreads();
            if (ok) buf[tid] = MODE == XR_RHO ? a : ixi<T, H>(fd, d == 0 ? kx : k0, a);
            __syncthreads();
            fft_2s<T, N1, N2, +1>(buf, 1, 1, H, 0, 1, tw, 1);
            __syncthreads();
            if (ok) stg(out + d * Rows2<T, H>::SPEC + tid, buf[tid]);
        }
    }
}

template <typename T, int H>
__global__ __launch_bounds__(ROW_THREADS) void k2_inv_rows(const FieldDesc<T>* __restrict__ fds, int ncomp) {
    using V = cplx_t<T>;
    using RF = RowFft<T, H>;
    constexpr int M = H / 2, HH = M + 1, R = Rows2<T, H>::R;
    __shared__ V buf[RF::SIZE];
    __shared__ V tw[H];
    const FieldDesc<T>& fd = fds[blockIdx.y];
    const int d = blockIdx.x % ncomp;
    const int ix0 = (blockIdx.x / ncomp) * R;
    const int tid = threadIdx.x;
    constexpr int K = Rows2<T, H>::K, NI = Rows2<T, H>::NKB * R * K;
    constexpr int NL = (NI + ROW_THREADS - 1) / ROW_THREADS;
    const V* in = fd.gspec + (size_t)d * Rows2<T, H>::SPEC + (size_t)ix0 * K;
    V* outp = reinterpret_cast<V*>(fd.G + (size_t)d * H * H + (size_t)ix0 * H);  // (x[2m], x[2m+1]) pairs
    {
        V v[NL];
#pragma unroll
        for (int q = 0; q < NL; ++q) {
            const int u = min(tid + q * ROW_THREADS, NI - 1);
            v[q] = ldg(in + (size_t)(u / (R * K)) * H * K + u % (R * K));
        }
        make_twiddles<T, H>(tw);
#pragma unroll
        for (int q = 0; q < NL; ++q) {
            const int u = tid + q * ROW_THREADS;
            const int e = u % (R * K), k = u / (R * K) * K + e % K;
            if (u < NI && k < HH) buf[RF::at(e / K, k)] = v[q];
        }
    }
    __syncthreads();
    // Z_k = (X_k + conj X_{M-k}) + i w_H^-k (X_k - conj X_{M-k})
    auto z_of = [&](int r, int k) {
        const V xa = buf[RF::at(r, k)], xc = cconj(buf[RF::at(r, M - k)]);
        const V s = cadd(xa, xc), t = cmul(cconj(tw[k]), csub(xa, xc));
        return cmake<V, T>(s.x - t.y, s.y + t.x);
    };
    if constexpr (RF::BIG) {
        using F = typename RF::F;
        V z[RF::NG][F::N2];
#pragma unroll
        for (int q = 0; q < RF::NG; ++q) {
            const int g = min(tid + q * ROW_THREADS, R * F::G3 - 1);
#pragma unroll
            for (int i = 0; i < F::N2; ++i) z[q][i] = z_of(g / F::G3, F::k1_of(g) + 16 * (F::j1_of(g) + F::N1 * i));
        }
        __syncthreads();  // the spectrum is read, its memory is the transform's now
#pragma unroll
        for (int q = 0; q < RF::NG; ++q)
            if (tid + q * ROW_THREADS < R * F::G3) F::store_group(buf, tid + q * ROW_THREADS, z[q], tw, 2);
        __syncthreads();
        F::template middle<R, +1>(buf, tw, 2);
        __syncthreads();
        if (tid < R * F::M) {
            const int b = tid / F::M, m = tid % F::M;
            V r[16];
            F::last(buf + b * F::LEN, tw, 2, m, r);
#pragma unroll
            for (int i = 0; i < 16; ++i) stg(outp + b * M + m + F::M * i, r[i]);
        }
    } else {
        constexpr int NZ = (R * M + ROW_THREADS - 1) / ROW_THREADS;
        V z[NZ];
#pragma unroll
        for (int q = 0; q < NZ; ++q) {
            const int u = min(tid + q * ROW_THREADS, R * M - 1);
            z[q] = z_of(u / M, u % M);
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NZ; ++q) {
            const int u = tid + q * ROW_THREADS;
            if (u < R * M) buf[RF::at(u / M, perm_pos_g<M>(u % M))] = z[q];
        }
        __syncthreads();
        fft_2s<T, Split<M>::N1, Split<M>::N2, +1>(buf, R, 1, RF::OP, 0, 1, tw, 2);
        __syncthreads();
        for (int u = tid; u < R * M; u += ROW_THREADS) stg(outp + u, buf[RF::at(u / M, u % M)]);
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <typename T, int H>
static hipError_t fwd_rows_h(const FieldDesc<T>* fd, int count, bool consume, hipStream_t s) {
    launch_kernel((k2_fwd_rows<T, H>), dim3(H / Rows2<T, H>::R, count), dim3(ROW_THREADS), 0, s, fd, consume ? 1 : 0);
    return hipGetLastError();
}
template <typename T, int H>
static hipError_t xrows_h(const FieldDesc<T>* fd, int count, int mode, hipStream_t s) {
    const dim3 g(Rows2<T, H>::NKB, count), b(xrow_threads<T, H>());
    switch (mode) {
        case XP_STEP: launch_kernel((k2_xrows<T, H, XR_STEP>), g, b, 0, s, fd); break;
        case XP_GRAD: launch_kernel((k2_xrows<T, H, XR_GRAD>), g, b, 0, s, fd); break;
        case XP_RHO: launch_kernel((k2_xrows<T, H, XR_RHO>), g, b, 0, s, fd); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
template <typename T, int H>
static hipError_t inv_rows_h(const FieldDesc<T>* fd, int count, int ncomp, hipStream_t s) {
    launch_kernel((k2_inv_rows<T, H>), dim3((H / Rows2<T, H>::R) * ncomp, count), dim3(ROW_THREADS), 0, s, fd, ncomp);
    return hipGetLastError();
}

#define SIPF_H2_SWITCH(H, FN, ...)                \
    switch (H) {                                  \
        case 8: return FN<T, 8>(__VA_ARGS__);     \
        case 16: return FN<T, 16>(__VA_ARGS__);   \
        case 32: return FN<T, 32>(__VA_ARGS__);   \
        case 64: return FN<T, 64>(__VA_ARGS__);   \
        case 128: return FN<T, 128>(__VA_ARGS__); \
        case 256: return FN<T, 256>(__VA_ARGS__); \
        case 512: return FN<T, 512>(__VA_ARGS__); \
        case 1024: return FN<T, 1024>(__VA_ARGS__); \
        case 2048: return FN<T, 2048>(__VA_ARGS__); \
        case 4096: return FN<T, 4096>(__VA_ARGS__); \
        default: return hipErrorInvalidValue;     \
    }

template <typename T> hipError_t launch_fwd_rows2(int H, const FieldDesc<T>* fd, int count, bool consume, hipStream_t s) {
    SIPF_H2_SWITCH(H, fwd_rows_h, fd, count, consume, s)
}
template <typename T> hipError_t launch_xrows2(int H, const FieldDesc<T>* fd, int count, int mode, hipStream_t s) {
    SIPF_H2_SWITCH(H, xrows_h, fd, count, mode, s)
}
template <typename T> hipError_t launch_inv_rows2(int H, const FieldDesc<T>* fd, int count, int ncomp, hipStream_t s) {
    SIPF_H2_SWITCH(H, inv_rows_h, fd, count, ncomp, s)
}

bool fft2d_size_supported(int H) {
    return H == 8 || H == 16 || H == 32 || H == 64 || H == 128 || H == 256 || H == 512 || H == 1024 || H == 2048 ||
           H == 4096;
}

template hipError_t launch_fwd_rows2<float>(int, const FieldDesc<float>*, int, bool, hipStream_t);
template hipError_t launch_fwd_rows2<double>(int, const FieldDesc<double>*, int, bool, hipStream_t);
template hipError_t launch_xrows2<float>(int, const FieldDesc<float>*, int, int, hipStream_t);
template hipError_t launch_xrows2<double>(int, const FieldDesc<double>*, int, int, hipStream_t);
template hipError_t launch_inv_rows2<float>(int, const FieldDesc<float>*, int, int, hipStream_t);
template hipError_t launch_inv_rows2<double>(int, const FieldDesc<double>*, int, int, hipStream_t);

}  // namespace sipf

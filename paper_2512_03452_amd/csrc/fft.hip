// Field passes of the SIPF-PIC step: real-to-complex 3-D FFT of the deposit,
// implicit mode update, filtered spectral gradient and complex-to-real 3-D
// inverse FFT of its three components (Algorithm 2's last line, the mode
// update and the gradient lines of Algorithm 4).
//
// Transform convention (Sec. 3.1): beta_q = L^-3 sum_j phi_j e^{-2 pi i q.j/H},
// grad c(x_j) = sum_q i xi_q Phi_q alpha_q e^{+2 pi i q.j/H}.
//
// Three passes over HBM per step (five at H = 256, where a plane pass splits
// into a row pass and a column pass, see below):
//   fwd_planes  one workgroup per x-plane: each real row along z is read as
//               H/2 complex values, transformed, and split into its half
//               spectrum (kz = 0..H/2); then the plane is transformed along y.
//               Also zeroes the deposit grid for the next step and advances
//               the step counter.
//   xpencils    one workgroup per 16 consecutive (ky, kz) x-pencils: transform
//               along x, alpha <- A alpha + B beta, form i xi_d Phi alpha for
//               d = 0,1,2 and inverse-transform each along x.
//   inv_planes  one workgroup per (component, x-plane): inverse along y, then
//               the half-length complex-to-real inverse along z.
//
// What bounds them: latency on a single grid (a launch of 3 to 7 us is a chain
// of a memory round trip, LDS exchanges and barriers), memory in batches and at
// H = 256.  So the first and last register DFT of every pass read and write
// HBM themselves, the mode update works on the registers between the forward
// and the inverse x transform, and LDS only carries the exchange between two
// stages (one write and one read each).  Measured against passes that staged
// every value through LDS, us per launch, forward / x pencils / inverse: H = 256
// 81 / 146 / 187 -> 79 / 93 / 196; 30 grids of H = 64 24 / 41 / 52 -> 26 / 42 /
// 37; H = 128 11.9 / 17.5 / 18.2 -> 11.4 / 16.0 / 19.7; H = 64 5.0 / 6.0 / 7.1 ->
// 5.3 / 6.6 / 6.9; H = 8 4.4 / 3.7 / 3.3 -> 3.5 / 2.8 / 2.6.
//
// The slower ones, from registers and counters: the values that wait for the
// other half of a stage are held in registers and the padded addresses cost VALU
// work.  k_inv_planes at H = 128 takes 86 registers instead of 58, so a CU holds one of
// its 1024-thread workgroups instead of two and the 384 planes take two rounds
// (VALU instructions +13 %, LDS waits -80 %); k_inv_zrows +16 % VALU instructions;
// the forward and x passes of a single H = 64 grid have half and a quarter of the
// waves in flight.
//
// The LDS FFT (lds_fft.h) leaves the forward transform in a digit-permuted
// order and takes that order back in the inverse; the x and y frequency axes
// of the stored spectra use it.
#include "internal.h"
#include "lds_fft.h"
#include "pass_common.h"

namespace sipf {

int fft_perm(int N, int k) {
    int N1 = 0, N2 = 1;
    switch (N) {
#define SIPF_SPLIT_CASE(n) case n: N1 = Split<n>::N1; N2 = Split<n>::N2; break;
        SIPF_SPLIT_CASE(3) SIPF_SPLIT_CASE(4) SIPF_SPLIT_CASE(5) SIPF_SPLIT_CASE(6) SIPF_SPLIT_CASE(8)
        SIPF_SPLIT_CASE(11) SIPF_SPLIT_CASE(12) SIPF_SPLIT_CASE(16) SIPF_SPLIT_CASE(22) SIPF_SPLIT_CASE(23)
        SIPF_SPLIT_CASE(32) SIPF_SPLIT_CASE(45) SIPF_SPLIT_CASE(46) SIPF_SPLIT_CASE(64) SIPF_SPLIT_CASE(90)
        SIPF_SPLIT_CASE(128) SIPF_SPLIT_CASE(256)
#undef SIPF_SPLIT_CASE
        case 512: case 1024: case 2048: case 4096: {
            const int M = N / 16;
            return (k % 16) * M + k / 16;
        }
        default: return -1;
    }
    return (k % N1) * N2 + k / N1;
}

// ---------------------------------------------------------------------------
// Storage order -> natural order of a half spectrum (the ABI's layout), on the
// device.  Both kernels are copies bound by memory: 3-D rows along kz move
// whole (one thread per value, writes coalesced), the 2-D spectrum is
// transposed through LDS.  Against a read-back, a permutation on the host and
// a copy to the device again, reading alpha takes 34.4 -> 0.09 ms at H = 256,
// 1.4 -> 0.05 ms at H = 128 and 14 -> 0.05 ms at H = 2048 in 2-D.
// ---------------------------------------------------------------------------
struct PermMap {
    int pm, pt, n1, n2;  // length pm pt: pt blocks of pm, each in two-stage order pm = n1 n2 (natural: n2 = 1)
    __device__ __forceinline__ int pos(int k) const {
        const int r = k / pt;
        return (k % pt) * pm + (r % n1) * n2 + r / n1;
    }
    __device__ __forceinline__ int freq(int p) const {
        const int r = p % pm;
        return p / pm + pt * (r / n2 + n1 * (r % n2));
    }
};

template <typename V>
__global__ __launch_bounds__(256) void k_natural3(const V* __restrict__ per, V* __restrict__ nat, int H, PermMap m) {
    const int HH = H / 2 + 1;
    const int n = H * H * HH;
    const int e = (int)(blockIdx.x * 256 + threadIdx.x);
    if (e >= n) return;
    const int row = e / HH, kz = e - row * HH;
    const int kx = row / H, ky = row - kx * H;
    nat[e] = per[(m.pos(kx) * H + m.pos(ky)) * HH + kz];
}

constexpr int NT2 = 32;  // tile of the 2-D transposition
template <typename V>
__global__ __launch_bounds__(256) void k_natural2(const V* __restrict__ per, V* __restrict__ nat, int H, PermMap m) {
    __shared__ V t[NT2][NT2 + 1];
    const int HH = H / 2 + 1;
    const int p0 = blockIdx.x * NT2, k0 = blockIdx.y * NT2;  // storage position of kx; ky
    const int c = threadIdx.x % NT2, r0 = threadIdx.x / NT2;
    for (int r = r0; r < NT2; r += 256 / NT2)
        if (k0 + r < HH && p0 + c < H) t[r][c] = per[(size_t)(k0 + r) * H + p0 + c];
    __syncthreads();
    for (int r = r0; r < NT2; r += 256 / NT2)
        if (p0 + r < H && k0 + c < HH) nat[(size_t)m.freq(p0 + r) * HH + k0 + c] = t[c][r];
}

template <typename T>
hipError_t launch_natural(int dim, int H, const cplx_t<T>* per, cplx_t<T>* nat, hipStream_t s) {
    PermMap m;
    m.pm = H > 256 ? H / 16 : H;
    m.pt = H > 256 ? 16 : 1;
    m.n2 = H > 256 ? 1 : fft_perm(m.pm, 1);
    m.n1 = m.pm / m.n2;
    const int HH = H / 2 + 1;
    if (dim == 2)
        hipLaunchKernelGGL((k_natural2<cplx_t<T>>), dim3((H + NT2 - 1) / NT2, (HH + NT2 - 1) / NT2), dim3(256), 0, s,
                           per, nat, H, m);
    else
        hipLaunchKernelGGL((k_natural3<cplx_t<T>>), dim3((H * H * HH + 255) / 256), dim3(256), 0, s, per, nat, H, m);
    return hipGetLastError();
}
template hipError_t launch_natural<float>(int, int, const cplx_t<float>*, cplx_t<float>*, hipStream_t);
template hipError_t launch_natural<double>(int, int, const cplx_t<double>*, cplx_t<double>*, hipStream_t);

// 3-D grids: powers of two 8 .. 256 and the mixed-radix sizes 12, 22, 46, 90;
// FP64 up to 64 (the plane passes' LDS)
bool fft_size_supported(int H, bool fp64) {
    switch (H) {
        case 8: case 12: case 16: case 22: case 32: case 46: case 64: return true;
        case 90: case 128: case 256: return !fp64;
        default: return false;
    }
}

constexpr int KB = 16;  // columns per workgroup of the x-pencil and y-column passes: one 128-byte line of FP32 per row

// ---------------------------------------------------------------------------
// Rows along z and planes in LDS.  A row of H reals is read as M = H/2 complex
// values z[m] = x[2m] + i x[2m+1] and transformed with an M-point FFT; then
//   E_k = (Z_k + conj Z_{M-k}) / 2,  O_k = (Z_k - conj Z_{M-k}) / (2i),
//   X_k = E_k + exp(-2 pi i k / H) O_k,   k = 0 .. M.
// The inverse takes Z_k = (X_k + conj X_{M-k}) + i exp(+2 pi i k / H)
// (X_k - conj X_{M-k}) to z[m] (unnormalised, as the gradient synthesis needs).
//
// M = M1 M2: value q of row r is at r PITCH + q + q / M2 (no padding when M2 =
// 1), with PITCH 8 mod 16 values (odd when M2 = 1), so that the lanes of a wave,
// M2 of one row beside each other, spread over the banks in both stages.
// Frequency k is at q = perm_pos<M>(k); the column k = M of a plane lies behind
// the rows.  tw[j] = exp(-2 pi i j / H).
// ---------------------------------------------------------------------------
template <typename T, int H, int NR> struct ZRows {
    using V = cplx_t<T>;
    static constexpr int M = H / 2, M1 = Split<M>::N1, M2 = Split<M>::N2;
    static constexpr int BARE = M2 > 1 ? M + M / M2 : M;
    static constexpr int PITCH = M2 > 1 ? BARE + (24 - BARE % 16) % 16 : BARE | 1;
    static constexpr int EXTRA = NR * PITCH;        // column k = M of the rows
    static constexpr int SIZE = NR * PITCH + NR;
    __device__ __forceinline__ static int at(int r, int q) { return r * PITCH + (M2 > 1 ? q + q / M2 : q); }
    // value k = 0 .. M of row r
    __device__ __forceinline__ static int freq_at(int r, int k) { return k == M ? EXTRA + r : at(r, perm_pos<M>(k)); }

    // rows from HBM (row r at src + r M), transformed: Z_k at freq_at(r, k).
    // clear: zero the rows.  Ends with a barrier; tw is made on the way.
    // One register DFT per row longer than 8 values (M = 11, 23): rows pass through LDS on the
    // way, since a thread's own row is not contiguous across the wave (H = 46: 7.4 -> 6.8
    // us forward).
    static constexpr bool STAGED = M2 == 1 && M1 > 8;
    template <int NT> __device__ __forceinline__ static void forward(V* buf, V* tw, V* src, bool clear) {
        if constexpr (STAGED) {
            constexpr int NL = NR * M, QL = (NL + NT - 1) / NT;
            V v[QL];
#pragma unroll
            for (int q = 0; q < QL; ++q) v[q] = ldg(src + min((int)threadIdx.x + q * NT, NL - 1));
            make_twiddles<T, H>(tw);
#pragma unroll
            for (int q = 0; q < QL; ++q) {
                const int u = (int)threadIdx.x + q * NT;
                if (u < NL) {
                    buf[at(u / M, u % M)] = v[q];
                    if (clear) stg(src + u, cmake<V, T>(0, 0));
                }
            }
            __syncthreads();
            for (int u = threadIdx.x; u < NR; u += NT) {
                V r[M1];
#pragma unroll
                for (int i = 0; i < M1; ++i) r[i] = buf[at(u, i)];
                Dft<T, M1, -1>::run(r);
#pragma unroll
                for (int i = 0; i < M1; ++i) buf[at(u, i)] = r[i];
            }
            __syncthreads();
            return;
        }
        constexpr int NI = NR * M2;  // first-stage items (r, m2)
        constexpr int Q = (NI + NT - 1) / NT;
        V r[Q][M1];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int u = min((int)threadIdx.x + q * NT, NI - 1);
#pragma unroll
            for (int i = 0; i < M1; ++i) r[q][i] = ldg(src + (u / M2) * M + u % M2 + i * M2);
        }
        make_twiddles<T, H>(tw);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int u = (int)threadIdx.x + q * NT;
            if (u < NI) {
                const int row = u / M2, m2 = u % M2;
                if (clear) {
#pragma unroll
                    for (int i = 0; i < M1; ++i) stg(src + row * M + m2 + i * M2, cmake<V, T>(0, 0));
                }
                Dft<T, M1, -1>::run(r[q]);
                if constexpr (M2 > 1) {
#pragma unroll
                    for (int j = 1; j < M1; ++j) r[q][j] = cmul(r[q][j], tw[2 * m2 * j]);
                }
#pragma unroll
                for (int j = 0; j < M1; ++j) buf[at(row, j * M2 + m2)] = r[q][j];
            }
        }
        __syncthreads();
        if constexpr (M2 > 1) {
            for (int u = threadIdx.x; u < NR * M1; u += NT) {
                V* p = buf + at(u / M1, u % M1 * M2);
                V v[M2];
#pragma unroll
                for (int i = 0; i < M2; ++i) v[i] = p[i];
                Dft<T, M2, -1>::run(v);
#pragma unroll
                for (int i = 0; i < M2; ++i) p[i] = v[i];
            }
            __syncthreads();
        }
    }
    // X_k of row r from the transformed row
    __device__ __forceinline__ static V split(const V* buf, const V* tw, int r, int k) {
        const V za = buf[freq_at(r, k % M)], zc = cconj(buf[freq_at(r, (M - k) % M)]);
        const V e = cscale(cadd(za, zc), (T)0.5);
        const V d = csub(za, zc);
        return cadd(e, cmul(tw[k], cmake<V, T>(d.y * (T)0.5, -d.x * (T)0.5)));
    }
    // rows X_k (at freq_at) to real rows in HBM (row r at dst + r M); starts after a barrier
    template <int NT> __device__ __forceinline__ static void inverse(V* buf, const V* tw, V* dst) {
        constexpr int NG = NR * M1, Q = (NG + NT - 1) / NT;  // groups (r, j1): k = j1 + M1 i
        V z[Q][M2];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int u = min((int)threadIdx.x + q * NT, NG - 1);
            const int row = u / M1, j1 = u % M1;
#pragma unroll
            for (int i = 0; i < M2; ++i) {
                const int k = j1 + M1 * i;
                const V xa = buf[freq_at(row, k)], xc = cconj(buf[freq_at(row, M - k)]);
                const V s = cadd(xa, xc), t = cmul(cconj(tw[k]), csub(xa, xc));
                z[q][i] = cmake<V, T>(s.x - t.y, s.y + t.x);
            }
            if constexpr (M2 > 1) {
                Dft<T, M2, +1>::run(z[q]);
#pragma unroll
                for (int i = 1; i < M2; ++i) z[q][i] = cmul(z[q][i], cconj(tw[2 * i * j1]));
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int u = (int)threadIdx.x + q * NT;
            if (u < NG) {
                V* p = buf + at(u / M1, u % M1 * M2);
#pragma unroll
                for (int i = 0; i < M2; ++i) p[i] = z[q][i];
            }
        }
        __syncthreads();
        for (int u = threadIdx.x; u < NR * M2; u += NT) {
            const int row = u / M2, m2 = u % M2;
            V r[M1];
#pragma unroll
            for (int j = 0; j < M1; ++j) r[j] = buf[at(row, j * M2 + m2)];
            Dft<T, M1, +1>::run(r);
#pragma unroll
            for (int i = 0; i < M1; ++i) {
                if constexpr (STAGED) buf[at(row, i)] = r[i];
                else stg(dst + row * M + m2 + i * M2, r[i]);
            }
        }
        if constexpr (STAGED) {
            __syncthreads();
            for (int u = threadIdx.x; u < NR * M; u += NT) stg(dst + u, buf[at(u / M, u % M)]);
        }
    }
};

// threads of a plane workgroup
template <int H> constexpr int plane_threads() {
    return H <= 16 ? 64 : (H <= 32 ? 256 : (H < 128 ? 512 : 1024));
}

// ---------------------------------------------------------------------------
// Pass 1: x-plane -> half spectrum along z, transformed along y.
// ---------------------------------------------------------------------------
template <typename T, int H>
__global__ __launch_bounds__(plane_threads<H>()) void k_fwd_planes(const FieldDesc<T>* __restrict__ fds, int consume) {
    using V = cplx_t<T>;
    using Z = ZRows<T, H, H>;
    constexpr int HH = H / 2 + 1, NT = plane_threads<H>();
    constexpr int N1 = Split<H>::N1, N2 = Split<H>::N2;
    __shared__ V buf[Z::SIZE];
    __shared__ V tw[H];
    const FieldDesc<T>& fd = fds[blockIdx.y];
    const int ix = blockIdx.x % H;
    const int comp = blockIdx.x / H;  // component of a multi-grid input (phi + comp H^3)
    const int tid = threadIdx.x;
    if (consume && ix == 0 && comp == 0 && tid == 0 && fd.step != nullptr) *fd.step += 1u;
    // the deposit grid is consumed: cleared for the next step's particle pass
    Z::template forward<NT>(buf, tw, reinterpret_cast<V*>(fd.phi + ((size_t)comp * H + ix) * H * H), consume != 0);
    V* out = fd.B1 + ((size_t)comp * H + ix) * H * HH;
    // along y, first stage: items (n2, kz) take rows n2 + i N2 of column kz
    constexpr int NI = HH * N2, Q = (NI + NT - 1) / NT;
    constexpr bool WIDE = N1 > 16;  // few items of many rows (H = 46): X_k from Z_k first, by all threads
    if constexpr (WIDE) {
        constexpr int QX = (H * HH + NT - 1) / NT;
        V x[QX];
#pragma unroll
        for (int q = 0; q < QX; ++q) {
            const int u = min(tid + q * NT, H * HH - 1);
            x[q] = Z::split(buf, tw, u / HH, u % HH);
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < QX; ++q) {
            const int u = tid + q * NT;
            if (u < H * HH) buf[Z::freq_at(u / HH, u % HH)] = x[q];
        }
        __syncthreads();
    }
    V r[Q][N1];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int u = min(tid + q * NT, NI - 1);
        const int kz = u % HH, n2 = u / HH;
#pragma unroll
        for (int i = 0; i < N1; ++i)
            r[q][i] = WIDE ? buf[Z::freq_at(n2 + i * N2, kz)] : Z::split(buf, tw, n2 + i * N2, kz);
        Dft<T, N1, -1>::run(r[q]);
#pragma unroll
        for (int k = 1; k < N1; ++k) r[q][k] = cmul(r[q][k], tw[n2 * k]);
    }
    __syncthreads();  // the rows are read, the columns overwrite them
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int u = tid + q * NT;
        if (u < NI) {
#pragma unroll
            for (int k = 0; k < N1; ++k) buf[Z::freq_at(k * N2 + u / HH, u % HH)] = r[q][k];
        }
    }
    __syncthreads();
    for (int u = tid; u < HH * N1; u += NT) {
        const int kz = u % HH, k1 = u / HH;
        V v[N2];
#pragma unroll
        for (int i = 0; i < N2; ++i) v[i] = buf[Z::freq_at(k1 * N2 + i, kz)];
        Dft<T, N2, -1>::run(v);
#pragma unroll
        for (int i = 0; i < N2; ++i) stg(out + (k1 * N2 + i) * HH + kz, v[i]);
    }
}

// ---------------------------------------------------------------------------
// Pass 2: x-pencils, mode update, filtered gradient spectra, inverse along x.
// ---------------------------------------------------------------------------
// MODE_STEP: forward x of B1, mode update of alpha, three gradient spectra
//            i xi_d Phi alpha, inverse x into gspec.
// MODE_GRAD: the three gradient spectra of alpha (no update).
// MODE_ADJ_SRC: adjoint of the source term: L^-3 B abar (abar in alpha), inverse x
//            into gspec component 0.
// MODE_ADJ_ACC: adjoint of the gradient and of the propagation: forward x of the
//            three transformed grids in B1, abar <- A abar + sum_d (-i xi_d Phi) B1_d.
// MODE_RHO:  forward x of B1 (a deposit), Gaussian factor Phi and L^-3, inverse x
//            into gspec component 0: the regularised density rho_hat * G0 after
//            the inverse plane pass.
// MODE_ADJ_ACC_SRC: MODE_ADJ_ACC, then MODE_ADJ_SRC of the updated abar in the
//            same pass (the reverse sweep needs the source term of abar^(n-1)
//            right after accumulating it).
enum { MODE_STEP = 0, MODE_GRAD = 1, MODE_ADJ_SRC = 2, MODE_ADJ_ACC = 3, MODE_RHO = 4, MODE_ADJ_ACC_SRC = 5 };

// A block is KB consecutive columns of the half spectrum flattened over
// (ky, kz) (column c = ky_position (H/2 + 1) + kz), all H x rows of each: a
// row of the block is KB contiguous values starting at a multiple of KB, one
// aligned 128-byte line in FP32 (blocks of KB kz values of one ky straddled
// two lines, since H/2 + 1 is odd).
//
// H = N1 N2.  First- and last-stage items (n2, column) hold rows n2 + i N2,
// groups (k1, column) hold the storage positions k1 N2 + i, i.e. the
// frequencies k1 + N1 i: one group per thread, whose registers carry the modes
// from the forward transform through the update into the inverse.  LDS carries
// value q of a column at (q + q / N2) KB + column: four rows of a wave lie on
// different banks in both stages.
template <int H> constexpr int pencil_threads() { return (KB * Split<H>::N1 + 63) / 64 * 64; }

template <typename T, int H, int MODE>
__global__ __launch_bounds__(pencil_threads<H>()) void k_xpencils(const FieldDesc<T>* __restrict__ fds) {
    using V = cplx_t<T>;
    constexpr int HH = H / 2 + 1;
    constexpr int NC = H * HH;  // columns (ky, kz): the pitch of an x row in HBM
    constexpr int N1 = Split<H>::N1, N2 = Split<H>::N2;
    constexpr int CB = KB, NT = pencil_threads<H>();
    static_assert(N2 > 1, "two stages");
    constexpr int NIN = MODE == MODE_ADJ_ACC || MODE == MODE_ADJ_ACC_SRC ? 3 : (MODE == MODE_STEP || MODE == MODE_RHO ? 1 : 0);
    constexpr int NOUT = MODE == MODE_STEP || MODE == MODE_GRAD ? 3 : (MODE == MODE_ADJ_ACC ? 0 : 1);
    // LDS for three grids at once where a block is small, so that their stages
    // share their barriers; above H = 64 one after the other, for more
    // workgroups per CU (H = 256: 35 KB against 104)
    constexpr int NBUF = NIN == 3 || (NOUT == 3 && H <= 64) ? 3 : 1;
    constexpr int LEN = (H + N1) * CB;  // values per grid
    __shared__ V lds[NBUF * LEN];
    __shared__ V tw[H];
    const FieldDesc<T>& fd = fds[blockIdx.y];
    const int c0 = blockIdx.x * CB;
    const int tid = threadIdx.x;
    // the thread's column (threads past the last column, or past the groups, compute on a valid one and store nothing)
    const int col = c0 + tid % CB;
    const bool ok = col < NC && tid < CB * N1;
    const int cc = min(col, NC - 1);
    const int kyp = cc / HH, kz = cc - kyp * HH;
    const int ky = perm_freq<H>(kyp);
    const int k1 = min(tid / CB, N1 - 1);  // the thread's group
    constexpr int GN = N2;                 // its modes: position pos(i), frequency kx(i)
    auto pos = [&](int i) { return k1 * N2 + i; };
    auto kx_of = [&](int i) { return k1 + N1 * i; };
    auto lat = [&](int q) { return (q + q / N2) * CB + tid % CB; };
    V al[GN];
    if constexpr (MODE != MODE_RHO) {
#pragma unroll
        for (int i = 0; i < GN; ++i) al[i] = ldg(fd.alpha + (size_t)pos(i) * NC + cc);
    }
    // factors of the thread's modes; up to 9 modes they are made while the loads are in flight
    constexpr bool AHEAD = GN <= 9;
    const T qy = (T)(ky < H / 2 ? ky : ky - H), qz = (T)kz;
    auto xi_of = [&](int k) { return (T)(k == H / 2 ? 0 : (k < H / 2 ? k : k - H)) * fd.two_pi_over_L; };
    T fA[GN], fB[GN], fP[GN];
    auto factors = [&](int i) {
        const int kx = kx_of(i);
        const T qx = (T)(kx < H / 2 ? kx : kx - H);
        const T q2 = qx * qx + qy * qy + qz * qz;
        if constexpr (MODE != MODE_ADJ_SRC) fP[i] = fd.filt > (T)0 ? exp(-fd.filt * q2) : (T)1;
        if constexpr (MODE != MODE_RHO && MODE != MODE_GRAD)
            mode_ab(fd, q2 * fd.two_pi_over_L * fd.two_pi_over_L + fd.k2, fA[i], fB[i]);
    };
    auto factors_ahead = [&]() {
        if constexpr (AHEAD) {
#pragma unroll
            for (int i = 0; i < GN; ++i) factors(i);
        }
    };
    // forward: the modes of the NIN input grids, z[d][i]
    V z[NIN > 0 ? NIN : 1][GN];
    if constexpr (NIN > 0) {
        constexpr int NI = NIN * CB * N2, Q = (NI + NT - 1) / NT;  // items (d, n2, column)
        V r[Q][N1];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int u = min(tid + q * NT, NI - 1);
            const int c = min(c0 + u % CB, NC - 1), n2 = u / CB % N2, d = u / (CB * N2);
#pragma unroll
            for (int i = 0; i < N1; ++i) r[q][i] = ldg(fd.B1 + (size_t)d * H * NC + (size_t)(n2 + i * N2) * NC + c);
        }
        make_twiddles<T, H>(tw);
        factors_ahead();
        __syncthreads();
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int u = tid + q * NT;
            if (u < NI) {
                const int n2 = u / CB % N2, d = u / (CB * N2);
                Dft<T, N1, -1>::run(r[q]);
#pragma unroll
                for (int k = 1; k < N1; ++k) r[q][k] = cmul(r[q][k], tw[n2 * k]);
#pragma unroll
                for (int k = 0; k < N1; ++k) lds[d * LEN + (k * N2 + n2 + k) * CB + u % CB] = r[q][k];
            }
        }
        __syncthreads();
#pragma unroll
        for (int d = 0; d < NIN; ++d) {
#pragma unroll
            for (int i = 0; i < N2; ++i) z[d][i] = lds[d * LEN + lat(pos(i))];
            Dft<T, N2, -1>::run(z[d]);
        }
    } else {
        make_twiddles<T, H>(tw);
        factors_ahead();
        __syncthreads();
    }
    // the modes: al[i] becomes the spectrum whose (derivatives') inverse transform goes out
#pragma unroll
    for (int i = 0; i < GN; ++i) {
        if constexpr (!AHEAD) factors(i);
        if constexpr (MODE == MODE_RHO) {
            al[i] = cscale(z[0][i], fP[i] * fd.inv_Ld);
        } else if constexpr (MODE == MODE_GRAD) {
            al[i] = cscale(al[i], fP[i]);
        } else {
            const T A = fA[i], B = fB[i];
            V a = al[i];
            if constexpr (MODE == MODE_STEP) {
                const T bs = B * fd.inv_Ld;
                a = cmake<V, T>(A * a.x + bs * z[0][i].x, A * a.y + bs * z[0][i].y);
            } else if constexpr (MODE != MODE_ADJ_SRC) {
                // abar <- A abar + sum_d (-i xi_d Phi) F(Gbar_d)
                const T xi[3] = {xi_of(kx_of(i)), xi_of(ky), xi_of(kz)};
                V acc = cmake<V, T>(0, 0);
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const T c = xi[d] * fP[i];
                    acc.x += c * z[NIN == 3 ? d : 0][i].y;  // (-i c) g = (c g.y, -c g.x)
                    acc.y -= c * z[NIN == 3 ? d : 0][i].x;
                }
                a = cmake<V, T>(A * a.x + acc.x, A * a.y + acc.y);
            }
            if (MODE != MODE_ADJ_SRC && ok) stg(fd.alpha + (size_t)pos(i) * NC + cc, a);
            if constexpr (MODE == MODE_STEP) al[i] = cscale(a, fP[i]);
            else al[i] = cscale(a, B * fd.inv_Ld);
        }
    }
    if constexpr (NOUT > 0) {
        // mode i of output grid d
        auto out_of = [&](int d, int i) -> V {
            if constexpr (NOUT == 1) {
                return al[i];
            } else {
                const T xi = xi_of(d == 0 ? kx_of(i) : (d == 1 ? ky : kz));
                return cmake<V, T>(-xi * al[i].y, xi * al[i].x);
            }
        };
        constexpr int ND = NBUF == 3 && NOUT == 3 ? 3 : 1;  // grids per exchange
        constexpr int NI = ND * CB * N2;
        if constexpr (NIN == 3) __syncthreads();  // groups of all three grids are read
#pragma unroll 1
        for (int d0 = 0; d0 < NOUT; d0 += ND) {
            if (d0 > 0) __syncthreads();  // the previous grid has been read
            if (tid < CB * N1) {
#pragma unroll
                for (int d = 0; d < ND; ++d) {
                    V r[N2];
#pragma unroll
                    for (int i = 0; i < N2; ++i) r[i] = out_of(d0 + d, i);
                    Dft<T, N2, +1>::run(r);
#pragma unroll
                    for (int i = 1; i < N2; ++i) r[i] = cmul(r[i], cconj(tw[i * k1]));
#pragma unroll
                    for (int i = 0; i < N2; ++i) lds[d * LEN + lat(pos(i))] = r[i];
                }
            }
            __syncthreads();
            for (int u = tid; u < NI; u += NT) {
                const int c = c0 + u % CB, n2 = u / CB % N2, d = u / (CB * N2);
                V r[N1];
#pragma unroll
                for (int k = 0; k < N1; ++k) r[k] = lds[d * LEN + (k * N2 + n2 + k) * CB + u % CB];
                Dft<T, N1, +1>::run(r);
                if (c < NC) {
                    V* o = fd.gspec + (size_t)(d0 + d) * H * NC + c;
#pragma unroll
                    for (int i = 0; i < N1; ++i) stg(o + (size_t)(n2 + i * N2) * NC, r[i]);
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Pass 3: inverse along y, complex-to-real inverse along z, per component.
// ---------------------------------------------------------------------------
template <typename T, int H>
__global__ __launch_bounds__(plane_threads<H>()) void k_inv_planes(const FieldDesc<T>* __restrict__ fds, int ncomp) {
    using V = cplx_t<T>;
    using Z = ZRows<T, H, H>;
    constexpr int HH = H / 2 + 1, NT = plane_threads<H>();
    constexpr int N1 = Split<H>::N1, N2 = Split<H>::N2;
    __shared__ V buf[Z::SIZE];
    __shared__ V tw[H];
    const FieldDesc<T>& fd = fds[blockIdx.y];
    // blocks 8c + r (c = (ix / 8) ncomp + d) keep the components of a plane on
    // one XCD; grids that are not a multiple of 8 take block ix ncomp + d
    const int b = blockIdx.x;
    int d, ix;
    if constexpr (H % 8 == 0) {
        const int grp = b / 8, r = b % 8;
        d = grp % ncomp;
        ix = (grp / ncomp) * 8 + r;
    } else {
        d = b % ncomp;
        ix = b / ncomp;
    }
    const int tid = threadIdx.x;
    const V* in = fd.gspec + ((size_t)d * H + ix) * H * HH;
    // along y: groups (k1, kz) of the positions k1 N2 + i, then items (n2, kz)
    constexpr int NG = HH * N1, NI = HH * N2;
    constexpr int Q = (NG + NT - 1) / NT;
    V r[Q][N2];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int u = tid + q * NT;
        if (u < NG) {
#pragma unroll
            for (int i = 0; i < N2; ++i) r[q][i] = ldg(in + (u / HH * N2 + i) * HH + u % HH);
        }
    }
    make_twiddles<T, H>(tw);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int u = tid + q * NT;
        if (u < NG) {
            Dft<T, N2, +1>::run(r[q]);
#pragma unroll
            for (int i = 1; i < N2; ++i) r[q][i] = cmul(r[q][i], cconj(tw[i * (u / HH)]));
#pragma unroll
            for (int i = 0; i < N2; ++i) buf[Z::freq_at(u / HH * N2 + i, u % HH)] = r[q][i];
        }
    }
    __syncthreads();
    for (int u = tid; u < NI; u += NT) {
        const int kz = u % HH, n2 = u / HH;
        V v[N1];
#pragma unroll
        for (int k = 0; k < N1; ++k) v[k] = buf[Z::freq_at(k * N2 + n2, kz)];
        Dft<T, N1, +1>::run(v);
#pragma unroll
        for (int i = 0; i < N1; ++i) buf[Z::freq_at(i * N2 + n2, kz)] = v[i];
    }
    __syncthreads();
    Z::template inverse<NT>(buf, tw, reinterpret_cast<V*>(fd.G + ((size_t)d * H + ix) * H * H));
}

// ---------------------------------------------------------------------------
// Grids whose yz-plane of half spectrum does not fit in LDS (H = 256: 264 KB
// in FP32).  Each plane pass splits in two, with one more trip through HBM:
//   fwd_zrows  ZROWS rows along z per workgroup: the half-length real
//              transform of fwd_planes, written to B1 with y in natural
//              order; consumes the deposit and advances the step counter.
//   ycols      KB kz columns of one x-plane per workgroup, transformed along
//              y in place (forward: natural -> digit-permuted y, as
//              fwd_planes leaves it; inverse: permuted -> natural).
//   inv_zrows  ZROWS rows per workgroup: the half-length complex-to-real
//              inverse of inv_planes.
// ---------------------------------------------------------------------------
constexpr int ZROWS = 16;
constexpr int ROW_THREADS = 256;

template <typename T, int H>
__global__ __launch_bounds__(ROW_THREADS) void k_fwd_zrows(const FieldDesc<T>* __restrict__ fds, int consume) {
    using V = cplx_t<T>;
    using Z = ZRows<T, H, ZROWS>;
    constexpr int HH = H / 2 + 1;
    constexpr int NRB = H * H / ZROWS;  // row blocks per component
    __shared__ V buf[Z::SIZE];
    __shared__ V tw[H];
    const FieldDesc<T>& fd = fds[blockIdx.y];
    const int comp = blockIdx.x / NRB;
    const size_t row0 = (size_t)(blockIdx.x % NRB) * ZROWS;  // row r = x H + y
    const int tid = threadIdx.x;
    if (consume && blockIdx.x == 0 && tid == 0 && fd.step != nullptr) *fd.step += 1u;
    Z::template forward<ROW_THREADS>(buf, tw, reinterpret_cast<V*>(fd.phi + ((size_t)comp * H * H + row0) * H), consume != 0);
    V* out = fd.B1 + ((size_t)comp * H * H + row0) * HH;
    for (int u = tid; u < ZROWS * HH; u += ROW_THREADS) stg(out + u, Z::split(buf, tw, u / HH, u % HH));
}

template <typename T, int H, int DIR>
__global__ __launch_bounds__(KB * Split<H>::N1) void k_ycols(const FieldDesc<T>* __restrict__ fds) {
    using V = cplx_t<T>;
    constexpr int HH = H / 2 + 1;
    constexpr int NKB = (HH + KB - 1) / KB;
    constexpr int N1 = Split<H>::N1, N2 = Split<H>::N2;
    static_assert(N1 == N2, "one item of each stage per thread");
    __shared__ V lds[(H + N1) * KB];  // as in k_xpencils
    __shared__ V tw[H];
    const FieldDesc<T>& fd = fds[blockIdx.y];
    const int kb = blockIdx.x % NKB, rest = blockIdx.x / NKB;
    const int x = rest % H, comp = rest / H;
    const int tid = threadIdx.x, a = tid / KB, c = tid % KB;  // a: n2 or k1
    const bool ok = kb * KB + c < HH;
    V* base = (DIR < 0 ? fd.B1 : fd.gspec) + ((size_t)comp * H + x) * H * HH + min(kb * KB + c, HH - 1);
    V r[N1];
    // forward: rows n2 + i N2 in, positions k1 N2 + i out; inverse: the other way round
    auto item = [&](int i) { return a + i * N2; };
    auto group = [&](int i) { return a * N2 + i; };
#pragma unroll
    for (int i = 0; i < N1; ++i) r[i] = ldg(base + (size_t)(DIR < 0 ? item(i) : group(i)) * HH);
    make_twiddles<T, H>(tw);
    __syncthreads();
    Dft<T, N1, DIR>::run(r);
#pragma unroll
    for (int i = 1; i < N1; ++i) r[i] = cmul(r[i], DIR < 0 ? tw[a * i] : cconj(tw[a * i]));
    // forward: r[k1] at position k1 N2 + n2; inverse: r[n2] at position k1 N2 + n2
#pragma unroll
    for (int i = 0; i < N1; ++i) {
        const int q = DIR < 0 ? i * N2 + a : a * N2 + i;
        lds[(q + q / N2) * KB + c] = r[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N1; ++i) {
        const int q = DIR < 0 ? a * N2 + i : i * N2 + a;
        r[i] = lds[(q + q / N2) * KB + c];
    }
    Dft<T, N1, DIR>::run(r);
    if (ok) {
#pragma unroll
        for (int i = 0; i < N1; ++i) stg(base + (size_t)(DIR < 0 ? group(i) : item(i)) * HH, r[i]);
    }
}

template <typename T, int H>
__global__ __launch_bounds__(ROW_THREADS) void k_inv_zrows(const FieldDesc<T>* __restrict__ fds) {
    using V = cplx_t<T>;
    using Z = ZRows<T, H, ZROWS>;
    constexpr int HH = H / 2 + 1;
    constexpr int NRB = H * H / ZROWS;
    constexpr int NL = ZROWS * HH, Q = (NL + ROW_THREADS - 1) / ROW_THREADS;
    __shared__ V buf[Z::SIZE];
    __shared__ V tw[H];
    const FieldDesc<T>& fd = fds[blockIdx.y];
    const int d = blockIdx.x / NRB;
    const size_t row0 = (size_t)(blockIdx.x % NRB) * ZROWS;
    const int tid = threadIdx.x;
    const V* in = fd.gspec + ((size_t)d * H * H + row0) * HH;
    V v[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) v[q] = ldg(in + min(tid + q * ROW_THREADS, NL - 1));
    make_twiddles<T, H>(tw);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int u = tid + q * ROW_THREADS;
        if (u < NL) buf[Z::freq_at(u / HH, u % HH)] = v[q];
    }
    __syncthreads();
    Z::template inverse<ROW_THREADS>(buf, tw, reinterpret_cast<V*>(fd.G + ((size_t)d * H * H + row0) * H));
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// grids above 128 take the split passes (a plane of half spectrum does not fit in LDS)
#ifndef SIPF_MAX_PLANE_H
#define SIPF_MAX_PLANE_H 128
#endif
constexpr int MAX_PLANE_H = SIPF_MAX_PLANE_H;

template <typename T, int H>
static hipError_t fwd_planes_h(const FieldDesc<T>* fd, int count, int ncomp, bool consume, hipStream_t s) {
    if constexpr (H > MAX_PLANE_H) {
        static_assert((H * H) % ZROWS == 0, "row blocks");
        constexpr int NKB = (H / 2 + 1 + KB - 1) / KB;
        launch_kernel((k_fwd_zrows<T, H>), dim3(ncomp * H * H / ZROWS, count), dim3(ROW_THREADS), 0, s, fd,
                      consume ? 1 : 0);
        launch_kernel((k_ycols<T, H, -1>), dim3(ncomp * H * NKB, count), dim3(KB * Split<H>::N1), 0, s, fd);
    } else {
        launch_kernel((k_fwd_planes<T, H>), dim3(H * ncomp, count), dim3(plane_threads<H>()), 0, s, fd, consume ? 1 : 0);
    }
    return hipGetLastError();
}
template <typename T, int H>
static hipError_t xpencils_h(const FieldDesc<T>* fd, int count, int mode, hipStream_t s) {
    const dim3 g((H * (H / 2 + 1) + KB - 1) / KB, count), b(pencil_threads<H>());
    switch (mode) {
        case MODE_STEP: launch_kernel((k_xpencils<T, H, MODE_STEP>), g, b, 0, s, fd); break;
        case MODE_GRAD: launch_kernel((k_xpencils<T, H, MODE_GRAD>), g, b, 0, s, fd); break;
        case MODE_ADJ_SRC: launch_kernel((k_xpencils<T, H, MODE_ADJ_SRC>), g, b, 0, s, fd); break;
        case MODE_ADJ_ACC: launch_kernel((k_xpencils<T, H, MODE_ADJ_ACC>), g, b, 0, s, fd); break;
        case MODE_ADJ_ACC_SRC: launch_kernel((k_xpencils<T, H, MODE_ADJ_ACC_SRC>), g, b, 0, s, fd); break;
        case MODE_RHO: launch_kernel((k_xpencils<T, H, MODE_RHO>), g, b, 0, s, fd); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
template <typename T, int H>
static hipError_t inv_planes_h(const FieldDesc<T>* fd, int count, int ncomp, hipStream_t s) {
    if constexpr (H > MAX_PLANE_H) {
        constexpr int NKB = (H / 2 + 1 + KB - 1) / KB;
        launch_kernel((k_ycols<T, H, +1>), dim3(ncomp * H * NKB, count), dim3(KB * Split<H>::N1), 0, s, fd);
        launch_kernel((k_inv_zrows<T, H>), dim3(ncomp * H * H / ZROWS, count), dim3(ROW_THREADS), 0, s, fd);
    } else {
        launch_kernel((k_inv_planes<T, H>), dim3(ncomp * H, count), dim3(plane_threads<H>()), 0, s, fd, ncomp);
    }
    return hipGetLastError();
}

#define SIPF_H_SWITCH(H, FN, ...)                         \
    switch (H) {                                          \
        case 8: return FN<T, 8>(__VA_ARGS__);             \
        case 12: return FN<T, 12>(__VA_ARGS__);           \
        case 16: return FN<T, 16>(__VA_ARGS__);           \
        case 22: return FN<T, 22>(__VA_ARGS__);           \
        case 32: return FN<T, 32>(__VA_ARGS__);           \
        case 46: return FN<T, 46>(__VA_ARGS__);           \
        case 64: return FN<T, 64>(__VA_ARGS__);           \
        case 90: if constexpr (sizeof(T) == 4) return FN<T, 90>(__VA_ARGS__); else return hipErrorInvalidValue; \
        case 128: if constexpr (sizeof(T) == 4) return FN<T, 128>(__VA_ARGS__); else return hipErrorInvalidValue; \
        case 256: if constexpr (sizeof(T) == 4) return FN<T, 256>(__VA_ARGS__); else return hipErrorInvalidValue; \
        default: return hipErrorInvalidValue;             \
    }

template <typename T>
hipError_t launch_fwd_planes(int H, const FieldDesc<T>* fd, int count, int ncomp, bool consume, hipStream_t s) {
    SIPF_H_SWITCH(H, fwd_planes_h, fd, count, ncomp, consume, s)
}
template <typename T> hipError_t launch_xpencils(int H, const FieldDesc<T>* fd, int count, int mode, hipStream_t s) {
    SIPF_H_SWITCH(H, xpencils_h, fd, count, mode, s)
}
template <typename T> hipError_t launch_inv_planes(int H, const FieldDesc<T>* fd, int count, int ncomp, hipStream_t s) {
    SIPF_H_SWITCH(H, inv_planes_h, fd, count, ncomp, s)
}

template hipError_t launch_fwd_planes<float>(int, const FieldDesc<float>*, int, int, bool, hipStream_t);
template hipError_t launch_fwd_planes<double>(int, const FieldDesc<double>*, int, int, bool, hipStream_t);
template hipError_t launch_xpencils<float>(int, const FieldDesc<float>*, int, int, hipStream_t);
template hipError_t launch_xpencils<double>(int, const FieldDesc<double>*, int, int, hipStream_t);
template hipError_t launch_inv_planes<float>(int, const FieldDesc<float>*, int, int, hipStream_t);
template hipError_t launch_inv_planes<double>(int, const FieldDesc<double>*, int, int, hipStream_t);

}  // namespace sipf

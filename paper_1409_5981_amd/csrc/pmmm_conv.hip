// FFT convolution of the moment meshes with the transfer kernel (Sec. 2.1,
// the four-line FFT procedure: forward transforms of the (p+1)^2 moment
// meshes, element-wise M2L in wave space, inverse transforms).
//
// Three launches, all LDS-resident:
//   k_plane_fwd  one z-plane of one component: real-to-complex FFT along x
//                (two real rows packed as one complex row) then a complex
//                FFT along y.  Open boundaries read the n x n data rows and
//                treat the rest of the 2n x 2n plane as zeros (App. C).
//   k_column     w (ky, kx) columns of ALL components: complex FFT along z,
//                the M2L of eq. realmatrix at every frequency of the columns,
//                inverse FFT along z (pmmm_column.h).
//   k_plane_inv  inverse of k_plane_fwd restricted to the y < n, x < n
//                block, scaled by 1/nf^3.
// The 3-D spectrum therefore never reaches HBM in full: the buffer between
// the kernels holds [P][n][nf][nf/2+1] complex values.
#include <type_traits>

#include "pmmm_internal.h"

namespace pmmm {

// ------------------------------------------------------------------ planes
// ------------------------------------------------- planes up to 32 points
// FFT sizes N = 4 to 32: a block takes pb planes (component c, z), one wave or
// two.  Every transform of a plane is one thread's, in registers: N/2 (open:
// N/4) row pairs along x -- two real rows as one complex row -- and N/2 + 1
// columns along y, so that pb (N/2 + 1) fills the block's lanes (planes_per).
// The planes pass through LDS twice, rows of N + 1 values against bank
// conflicts, and the spectra go straight between registers and memory.  Bound
// by HBM: each plane is read and written once.  Measured against the block-wide
// passes this replaced (a barrier per FFT step, 256 threads on up to 8 planes):
// periodic 32^3, p = 7, 2048 planes 14.6 -> 9.3 us forward, 16.1 -> 8.3 inverse
// (17 MB each way, 3.7 us); batch of 256 systems of 8^3 to 32^3 cells, whole
// call 2835 -> 2156 us; FP64 open 16^3, p = 5, whole call 79 -> 61.
template <typename T>
struct alignas(16) vec4 {
    T v[4];
};

template <typename T, int N, bool HALF>
__global__ void __launch_bounds__(128) k_plane_fwd(const T *__restrict__ M,
                                                   cplx<T> *__restrict__ spec, int P, int pb,
                                                   int nblk, int nzl, int nzs,
                                                   double *__restrict__ qr2_partial) {
    constexpr int nin = HALF ? N / 2 : N, npair = nin / 2, nh = N / 2 + 1, LS = N + 1;
    constexpr int NV = nin * nin / 4, LB = 8;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    cplx<T> *xb = (cplx<T> *)lds_raw;            // [pb][npair][LS]
    const int tid = threadIdx.x, nthr = blockDim.x;
    {
        // system blockIdx.z of a batch: meshes at fixed strides
        const int64_t sy = blockIdx.z;
        M += sy * (P + 1) * nin * nin * nin;
        spec += sy * P * nzs * N * nh;
        if (qr2_partial != nullptr) qr2_partial += sy * nin;
    }
    if ((int)blockIdx.x >= nblk) {
        // periodic: sum over plane z of the per-cell q|u|^2 (component P of
        // M), fixed-order reduction
        __shared__ double red[2];
        const int z = blockIdx.x - nblk;
        const T *pl = M + ((int64_t)P * nin + z) * nin * nin;
        double acc = 0.0;
        for (int idx = tid; idx < nin * nin; idx += nthr) acc += (double)pl[idx];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
        if ((tid & 63) == 0) red[tid >> 6] = acc;
        __syncthreads();
        if (tid == 0) qr2_partial[z] = nthr > 64 ? red[0] + red[1] : red[0];
        return;
    }
    const int first = blockIdx.x * pb, left = P * nzl - first, cnt = left < pb ? left : pb;
    // loads of a batch are issued before their LDS stores
    for (int base = tid; base < cnt * NV; base += nthr * LB) {
        vec4<T> v[LB];
#pragma unroll
        for (int u = 0; u < LB; ++u) {
            const int idx = base + u * nthr < cnt * NV ? base + u * nthr : cnt * NV - 1;
            const int q = first + idx / NV, c = q / nzl;
            v[u] = ((const vec4<T> *)(M + ((int64_t)c * nin + (q - c * nzl)) * nin * nin))[idx % NV];
        }
#pragma unroll
        for (int u = 0; u < LB; ++u) {
            const int idx = base + u * nthr;
            if (idx < cnt * NV) {
                const int y = idx % NV / (nin / 4), x = idx % (nin / 4) * 4;
                T *d = (T *)(xb + (idx / NV * npair + (y >> 1)) * LS + x) + (y & 1);
#pragma unroll
                for (int k = 0; k < 4; ++k) d[2 * k] = v[u].v[k];
            }
        }
    }
    __syncthreads();
    for (int line = tid; line < cnt * npair; line += nthr) {
        cplx<T> *b = xb + line * LS;
        cplx<T> w[N];
        static_for<0, N>([&](auto ix) {
            constexpr int x = decltype(ix)::value;
            if constexpr (x < nin) w[x] = b[x];
            else w[x] = {T(0), T(0)};
        });
        fft_reg<N, false, T>(w);
        static_for<0, N>([&](auto ix) { b[decltype(ix)::value] = w[decltype(ix)::value]; });
    }
    __syncthreads();
    for (int it = tid; it < cnt * nh; it += nthr) {
        const int pl = it / nh, k = it - pl * nh, km = (N - k) & (N - 1);
        const cplx<T> *b = xb + pl * npair * LS;
        cplx<T> w[N];
        static_for<0, N / 2>([&](auto ij) {
            constexpr int j = decltype(ij)::value;
            if constexpr (j < npair) {
                const cplx<T> zk = b[j * LS + k], zm = b[j * LS + km];
                w[2 * j] = {T(0.5) * (zk.re + zm.re), T(0.5) * (zk.im - zm.im)};
                w[2 * j + 1] = {T(0.5) * (zk.im + zm.im), T(-0.5) * (zk.re - zm.re)};
            } else {
                w[2 * j] = {T(0), T(0)};
                w[2 * j + 1] = {T(0), T(0)};
            }
        });
        fft_reg<N, false, T>(w);
        const int q = first + pl, c = q / nzl;
        cplx<T> *out = spec + ((int64_t)c * nzs + (q - c * nzl)) * N * nh + k;
        static_for<0, N>([&](auto iy) { out[decltype(iy)::value * nh] = w[decltype(iy)::value]; });
    }
}

template <typename T, int N, bool HALF>
__global__ void __launch_bounds__(128) k_plane_inv(const cplx<T> *__restrict__ spec,
                                                   T *__restrict__ L, T scale, int P, int pb,
                                                   int nzl, int nzs) {
    constexpr int nout = HALF ? N / 2 : N, npair = nout / 2, nh = N / 2 + 1, LS = N + 1;
    constexpr int NV = nout * nout / 4;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    cplx<T> *xb = (cplx<T> *)lds_raw;            // [pb][npair][LS]
    const int tid = threadIdx.x, nthr = blockDim.x;
    {
        // system blockIdx.z of a batch: meshes at fixed strides
        const int64_t sy = blockIdx.z;
        spec += sy * P * nzs * N * nh;
        L += sy * P * nout * nout * nout;
    }
    const int first = blockIdx.x * pb, left = P * nzl - first, cnt = left < pb ? left : pb;
    for (int it = tid; it < cnt * nh; it += nthr) {
        const int pl = it / nh, k = it - pl * nh;
        const int q = first + pl, c = q / nzl;
        const cplx<T> *in = spec + ((int64_t)c * nzs + (q - c * nzl)) * N * nh + k;
        cplx<T> w[N];
        static_for<0, N>([&](auto iy) { w[decltype(iy)::value] = in[decltype(iy)::value * nh]; });
        fft_reg<N, true, T>(w);
        // C2R row pairs: Z_j[k] = A[k] + i B[k] and, 0 < k < N/2,
        // Z_j[N - k] = conj(A[k]) + i conj(B[k]) from rows A = 2j, B = 2j + 1
        cplx<T> *b = xb + pl * npair * LS;
        static_for<0, npair>([&](auto ij) {
            constexpr int j = decltype(ij)::value;
            const cplx<T> A = w[2 * j], B = w[2 * j + 1];
            b[j * LS + k] = {A.re - B.im, A.im + B.re};
            if (k > 0 && k < N / 2) b[j * LS + N - k] = {A.re + B.im, B.re - A.im};
        });
    }
    __syncthreads();
    for (int line = tid; line < cnt * npair; line += nthr) {
        cplx<T> *b = xb + line * LS;
        cplx<T> w[N];
        static_for<0, N>([&](auto ix) { w[decltype(ix)::value] = b[decltype(ix)::value]; });
        fft_reg<N, true, T>(w);
        static_for<0, nout>([&](auto ix) {
            constexpr int x = decltype(ix)::value;
            b[x] = {w[x].re * scale, w[x].im * scale};
        });
    }
    __syncthreads();
    for (int idx = tid; idx < cnt * NV; idx += nthr) {
        const int y = idx % NV / (nout / 4), x = idx % (nout / 4) * 4;
        const T *d = (const T *)(xb + (idx / NV * npair + (y >> 1)) * LS + x) + (y & 1);
        vec4<T> v;
#pragma unroll
        for (int k = 0; k < 4; ++k) v.v[k] = d[2 * k];
        const int q = first + idx / NV, c = q / nzl;
        ((vec4<T> *)(L + ((int64_t)c * nout + (q - c * nzl)) * nout * nout))[idx % NV] = v;
    }
}

// ------------------------------------------------- planes of 64 and 128
// Same transforms for FFT sizes N = 64 and 128, one (plane z, component c)
// per block of 256 threads, with register FFTs in four steps (fft_col) and
// the open boundary's zero half pruned.  The row pairs live in swizzled LDS
// rows xb[npair][N]; the y pass runs over chunks of up to 17 kx columns
// through yb[N][CWS] (y-major, kx fastest, so the lanes of a wave take
// consecutive kx: conflict-free in LDS and coalesced in memory): its first
// step reads the row pairs straight from xb (unpacking the R2C of two real
// rows), its second writes the spectrum to memory (forward) or into the
// C2R row pairs (inverse).  Open: nin = N / 2 rows and columns in, and the
// y and x transforms skip the zero half; periodic: nin = N.
// Chunks of 17 columns keep a 128-point block at 51 KB of LDS, three blocks
// per CU (33 columns: 68 KB, two blocks, and the inverse planes 28% slower;
// 5 columns: 39 KB, four blocks, but 13 chunks' barriers make both passes
// about 60% slower).
constexpr int kPlaneThreads = 256;
constexpr int kPlaneChunk = 17;

// W_N^e (conjugate for the inverse) from the full-circle table.
template <typename T>
__device__ __forceinline__ cplx<T> tw_n(const cplx<T> *tw, int e, bool inv) {
    cplx<T> w = tw[e];
    if (inv) w.im = -w.im;
    return w;
}

template <typename T, int N, bool HALF>
__global__ void __launch_bounds__(kPlaneThreads) k_plane_fwd_n(const T *__restrict__ M,
                                                               cplx<T> *__restrict__ spec,
                                                               const cplx<T> *__restrict__ tw_g,
                                                               int P, int nzs,
                                                               double *__restrict__ qr2_partial) {
    constexpr int nin = HALF ? N / 2 : N, npair = nin / 2, nh = N / 2 + 1, N2 = N / 16;
    constexpr int CWS = kPlaneChunk;  // odd row stride of yb
    extern __shared__ __align__(16) unsigned char lds_raw[];
    cplx<T> *tw = (cplx<T> *)lds_raw;
    cplx<T> *xb = tw + N;
    cplx<T> *yb = xb + npair * N;
    const int z = blockIdx.x, tid = threadIdx.x;
    {
        const int64_t sy = blockIdx.z, K = (int64_t)nin * nin * nin;
        M += sy * (P + 1) * K;
        spec += sy * P * nzs * N * nh;
        if (qr2_partial != nullptr) qr2_partial += sy * nin;
    }
    if ((int)blockIdx.y == P) {
        // blocks of the extra row: sum over plane z of the per-cell q|u|^2
        // (component P of M), fixed-order reduction
        __shared__ double red[kPlaneThreads / 64];
        const T *pl = M + ((int64_t)P * nin + z) * nin * nin;
        double acc = 0.0;
        for (int idx = tid; idx < nin * nin; idx += kPlaneThreads) acc += (double)pl[idx];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
        if ((tid & 63) == 0) red[tid >> 6] = acc;
        __syncthreads();
        if (tid == 0) {
            double t = 0.0;
            for (int w = 0; w < kPlaneThreads / 64; ++w) t += red[w];
            qr2_partial[z] = t;
        }
        return;
    }
    const int c = blockIdx.y;
    const T *plane = M + ((int64_t)c * nin + z) * nin * nin;
    // rows (2j, 2j+1) as one complex row; the loads of a batch are issued
    // before their LDS stores
    constexpr int NL = npair * nin;
    constexpr int LB = (NL + kPlaneThreads - 1) / kPlaneThreads < 8
                           ? (NL + kPlaneThreads - 1) / kPlaneThreads : 8;
    for (int base = tid; base < NL; base += kPlaneThreads * LB) {
        cplx<T> v[LB];
#pragma unroll
        for (int u = 0; u < LB; ++u) {
            const int idx = base + u * kPlaneThreads < NL ? base + u * kPlaneThreads : NL - 1;
            const int j = idx / nin, x = idx - j * nin;
            v[u] = {plane[(2 * j) * nin + x], plane[(2 * j + 1) * nin + x]};
        }
#pragma unroll
        for (int u = 0; u < LB; ++u) {
            const int idx = base + u * kPlaneThreads;
            if (idx < NL) {
                const int j = idx / nin, x = idx - j * nin;
                xb[j * N + cpos(j, x)] = v[u];
            }
        }
    }
    fill_twiddles<T>(tw, tw_g, N, tid, kPlaneThreads);
    __syncthreads();
    fft_col<T, false, N, HALF>(xb, npair, tw, tid, kPlaneThreads);   // ends with a barrier
    cplx<T> *out = spec + ((int64_t)c * nzs + z) * N * nh;
    for (int k0 = 0; k0 < nh; k0 += kPlaneChunk) {
        const int cn = nh - k0 < kPlaneChunk ? nh - k0 : kPlaneChunk;
        // y transforms, first step: 16-point FFTs over n1 of x[n1 N2 + t2]
        for (int it = tid; it < cn * N2; it += kPlaneThreads) {
            const int t2 = it / cn, kl = it - t2 * cn, k = k0 + kl;
            cplx<T> v[16];
            static_for<0, 16>([&](auto in) {
                constexpr int n1 = decltype(in)::value;
                if constexpr (HALF && n1 >= 8) {
                    v[n1] = {T(0), T(0)};
                } else {
                    const int y = n1 * N2 + t2, j = y >> 1;
                    const cplx<T> zk = xb[j * N + cpos(j, k & (N - 1))];
                    const cplx<T> zm = xb[j * N + cpos(j, (N - k) & (N - 1))];
                    if ((y & 1) == 0) v[n1] = {T(0.5) * (zk.re + zm.re), T(0.5) * (zk.im - zm.im)};
                    else v[n1] = {T(0.5) * (zk.im + zm.im), T(-0.5) * (zk.re - zm.re)};
                }
            });
            fft_reg<16, false, T>(v);
            static_for<0, 16>([&](auto ik) {
                constexpr int k1 = decltype(ik)::value;
                const cplx<T> w = k1 == 0 ? cplx<T>{T(1), T(0)} : tw_n(tw, t2 * k1, false);
                yb[(t2 * 16 + k1) * CWS + kl] = k1 == 0 ? v[k1] : cmul(v[k1], w);
            });
        }
        __syncthreads();
        // second step: N2-point FFTs over t2, spectrum rows y = k2 * 16 + k1
        for (int it = tid; it < cn * 16; it += kPlaneThreads) {
            const int k1 = it / cn, kl = it - k1 * cn;
            cplx<T> u[N2];
            static_for<0, N2>([&](auto it2) {
                constexpr int t2 = decltype(it2)::value;
                u[t2] = yb[(t2 * 16 + k1) * CWS + kl];
            });
            fft_reg<N2, false, T>(u);
            static_for<0, N2>([&](auto ik2) {
                constexpr int k2 = decltype(ik2)::value;
                out[(k2 * 16 + k1) * nh + k0 + kl] = u[k2];
            });
        }
        __syncthreads();   // yb is refilled by the next chunk
    }
}

template <typename T, int N, bool HALF>
__global__ void __launch_bounds__(kPlaneThreads) k_plane_inv_n(const cplx<T> *__restrict__ spec,
                                                               T *__restrict__ L,
                                                               const cplx<T> *__restrict__ tw_g,
                                                               T scale, int P, int nzs) {
    constexpr int nout = HALF ? N / 2 : N, npair = nout / 2, nh = N / 2 + 1, N2 = N / 16;
    constexpr int CWS = kPlaneChunk;
    constexpr int K2 = HALF ? N2 / 2 : N2;   // y rows kept: k2 * 16 + k1 < nout
    extern __shared__ __align__(16) unsigned char lds_raw[];
    cplx<T> *tw = (cplx<T> *)lds_raw;
    cplx<T> *xb = tw + N;
    cplx<T> *yb = xb + npair * N;
    const int z = blockIdx.x, c = blockIdx.y, tid = threadIdx.x;
    {
        const int64_t sy = blockIdx.z;
        spec += sy * P * nzs * N * nh;
        L += sy * P * nout * nout * nout;
    }
    fill_twiddles<T>(tw, tw_g, N, tid, kPlaneThreads);
    __syncthreads();
    const cplx<T> *in = spec + ((int64_t)c * nzs + z) * N * nh;
    for (int k0 = 0; k0 < nh; k0 += kPlaneChunk) {
        const int cn = nh - k0 < kPlaneChunk ? nh - k0 : kPlaneChunk;
        // y inverse transforms, first step, straight from memory (lanes take
        // consecutive kx)
        for (int it = tid; it < cn * N2; it += kPlaneThreads) {
            const int t2 = it / cn, kl = it - t2 * cn;
            cplx<T> v[16];
            static_for<0, 16>([&](auto in1) {
                constexpr int n1 = decltype(in1)::value;
                v[n1] = in[(n1 * N2 + t2) * nh + k0 + kl];
            });
            fft_reg<16, true, T>(v);
            static_for<0, 16>([&](auto ik) {
                constexpr int k1 = decltype(ik)::value;
                const cplx<T> w = k1 == 0 ? cplx<T>{T(1), T(0)} : tw_n(tw, t2 * k1, true);
                yb[(t2 * 16 + k1) * CWS + kl] = k1 == 0 ? v[k1] : cmul(v[k1], w);
            });
        }
        __syncthreads();
        // second step, rows y = k2 * 16 + k1 < nout, into the C2R row pairs:
        // even rows y = 2j give A, odd rows B, and Z_j[k] = A[k] + i B[k],
        // Z_j[N - k] = conj(A[k]) + i conj(B[k]) (0 < k < N/2); the even rows
        // are written first, the odd ones added after a barrier
        for (int parity = 0; parity < 2; ++parity) {
            for (int it = tid; it < cn * 8; it += kPlaneThreads) {
                const int kh = it / cn, kl = it - kh * cn, k1 = 2 * kh + parity, k = k0 + kl;
                cplx<T> u[N2];
                static_for<0, N2>([&](auto it2) {
                    constexpr int t2 = decltype(it2)::value;
                    u[t2] = yb[(t2 * 16 + k1) * CWS + kl];
                });
                fft_reg<N2, true, T>(u);
                static_for<0, K2>([&](auto ik2) {
                    constexpr int k2 = decltype(ik2)::value;
                    const int j = (k2 * 16 + k1) >> 1;
                    cplx<T> *row = xb + j * N;
                    const cplx<T> a = u[k2];
                    if (parity == 0) {
                        row[cpos(j, k)] = a;
                        if (k >= 1 && k < N / 2) row[cpos(j, N - k)] = {a.re, -a.im};
                    } else {
                        cplx<T> &zk = row[cpos(j, k)];
                        zk = {zk.re - a.im, zk.im + a.re};
                        if (k >= 1 && k < N / 2) {
                            cplx<T> &zm = row[cpos(j, N - k)];
                            zm = {zm.re + a.im, zm.im + a.re};
                        }
                    }
                });
            }
            __syncthreads();
        }
    }
    // x inverse transforms of the row pairs, the first nout outputs kept
    fft_col<T, true, N, HALF>(xb, npair, tw, tid, kPlaneThreads);
    T *plane = L + ((int64_t)c * nout + z) * nout * nout;
    for (int idx = tid; idx < nout * nout; idx += kPlaneThreads) {
        const int y = idx / nout, x = idx - y * nout, j = y >> 1;
        const cplx<T> v = xb[j * N + cpos(j, x)];
        plane[idx] = ((y & 1) ? v.im : v.re) * scale;
    }
}

template <typename T, int N>
static size_t plane_n_lds(bool half) {
    const int npair = (half ? N / 2 : N) / 2;
    return (size_t)(N + npair * N + N * kPlaneChunk) * sizeof(cplx<T>);
}

template <typename T, int N>
static hipError_t plane_n_launch(const FFTArgs &a, int stage, hipStream_t s) {
    const int P = nreal(a.p), nz = a.nzl, nsys = a.nsys > 0 ? a.nsys : 1;
    const bool half = a.open != 0;
    const size_t lds = plane_n_lds<T, N>(half);
    hipError_t e = hipSuccess;
    if (stage == 0) {
        const void *k = half ? (const void *)k_plane_fwd_n<T, N, true>
                             : (const void *)k_plane_fwd_n<T, N, false>;
        if (lds > 65536 && (e = set_max_lds(k, lds)) != hipSuccess) return e;
        const int rows = half ? P : P + 1;   // periodic: one extra row of q|u|^2 sums
        if (half)
            hipLaunchKernelGGL((k_plane_fwd_n<T, N, true>), dim3(nz, rows, nsys),
                               dim3(kPlaneThreads), lds, s, (const T *)a.M, (cplx<T> *)a.spec,
                               (const cplx<T> *)a.tw, P, a.nzs, nullptr);
        else
            hipLaunchKernelGGL((k_plane_fwd_n<T, N, false>), dim3(nz, rows, nsys),
                               dim3(kPlaneThreads), lds, s, (const T *)a.M, (cplx<T> *)a.spec,
                               (const cplx<T> *)a.tw, P, a.nzs, a.qr2_partial);
    } else {
        const void *k = half ? (const void *)k_plane_inv_n<T, N, true>
                             : (const void *)k_plane_inv_n<T, N, false>;
        if (lds > 65536 && (e = set_max_lds(k, lds)) != hipSuccess) return e;
        const T scale = T(1.0 / ((double)N * N * a.nfz));
        if (half)
            hipLaunchKernelGGL((k_plane_inv_n<T, N, true>), dim3(nz, P, nsys), dim3(kPlaneThreads),
                               lds, s, (const cplx<T> *)a.spec, (T *)a.L, (const cplx<T> *)a.tw,
                               scale, P, a.nzs);
        else
            hipLaunchKernelGGL((k_plane_inv_n<T, N, false>), dim3(nz, P, nsys), dim3(kPlaneThreads),
                               lds, s, (const cplx<T> *)a.spec, (T *)a.L, (const cplx<T> *)a.tw,
                               scale, P, a.nzs);
    }
    return hipGetLastError();
}

// --------------------------------------------------------------- launcher
// Column stage, one instantiation per order in the pmmm_column_*.hip units.
template <int PO, typename T>
hipError_t column_launch(const FFTArgs &a, hipStream_t s);

// Planes per block of the transforms up to 32 points: the columns of pb planes
// fill one wave; two from 1024 such blocks on, which leave fewer lanes idle
// (7 x 17 of 128 against 3 x 17 of 64 at 32 points) and still fill the chip.
static int planes_per(int N, int64_t planes) {
    const int nh = N / 2 + 1;
    return planes >= (int64_t)1024 * (128 / nh) ? 128 / nh : 64 / nh;
}

template <typename T, int N, bool HALF>
static hipError_t plane_launch(const FFTArgs &a, int stage, hipStream_t s) {
    const int P = nreal(a.p), nsys = a.nsys > 0 ? a.nsys : 1, npair = (HALF ? N / 2 : N) / 2;
    const int pb = planes_per(N, (int64_t)P * a.nzl * nsys);
    const int nblk = (P * a.nzl + pb - 1) / pb, threads = pb * (N / 2 + 1) > 64 ? 128 : 64;
    const size_t lds = (size_t)pb * npair * (N + 1) * sizeof(cplx<T>);
    if (stage == 0)   // periodic: one more block per plane sums q|u|^2
        hipLaunchKernelGGL((k_plane_fwd<T, N, HALF>), dim3(nblk + (HALF ? 0 : N), 1, nsys),
                           dim3(threads), lds, s, (const T *)a.M, (cplx<T> *)a.spec, P, pb, nblk,
                           a.nzl, a.nzs, HALF ? nullptr : a.qr2_partial);
    else
        hipLaunchKernelGGL((k_plane_inv<T, N, HALF>), dim3(nblk, 1, nsys), dim3(threads), lds, s,
                           (const cplx<T> *)a.spec, (T *)a.L, T(1.0 / ((double)N * N * a.nfz)), P, pb,
                           a.nzl, a.nzs);
    return hipGetLastError();
}

template <typename T>
static hipError_t plane_dispatch(const FFTArgs &a, int stage, hipStream_t s) {
    switch (a.nf) {
        case 4: return a.open ? hipErrorInvalidValue : plane_launch<T, 4, false>(a, stage, s);
        case 8: return a.open ? plane_launch<T, 8, true>(a, stage, s) : plane_launch<T, 8, false>(a, stage, s);
        case 16: return a.open ? plane_launch<T, 16, true>(a, stage, s) : plane_launch<T, 16, false>(a, stage, s);
        case 32: return a.open ? plane_launch<T, 32, true>(a, stage, s) : plane_launch<T, 32, false>(a, stage, s);
        case 64: return plane_n_launch<T, 64>(a, stage, s);
        case 128:
            if constexpr (sizeof(T) == 4) return plane_n_launch<T, 128>(a, stage, s);
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

template <typename T>
hipError_t launch_conv_stage(const FFTArgs &a, int stage, hipStream_t s) {
    if (a.generic) return launch_generic_stage<T>(a, stage, s);
    if (stage == 1) {
        switch (a.p) {
            case 0: return column_launch<0, T>(a, s);
            case 1: return column_launch<1, T>(a, s);
            case 2: return column_launch<2, T>(a, s);
            case 3: return column_launch<3, T>(a, s);
            case 4: return column_launch<4, T>(a, s);
            case 5: return column_launch<5, T>(a, s);
            case 6: return column_launch<6, T>(a, s);
            case 7: return column_launch<7, T>(a, s);
            case 8: return column_launch<8, T>(a, s);
            case 9: return column_launch<9, T>(a, s);
            case 10: return column_launch<10, T>(a, s);
            default: return hipErrorInvalidValue;
        }
    }
    return plane_dispatch<T>(a, stage, s);
}

template hipError_t launch_conv_stage<float>(const FFTArgs &, int, hipStream_t);
template hipError_t launch_conv_stage<double>(const FFTArgs &, int, hipStream_t);

}  // namespace pmmm

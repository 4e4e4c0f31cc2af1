// Fine-level kernel of the two-level hierarchical far field (Sec. 5.2),
// instantiated once per order by pmmm_hier_inst.hip.  The local expansion of
// fine cell I gathers eq. M2L of the moments of every fine cell J whose
// coarse cell is within c of I's and which is itself more than c from I, in
// the real-matrix form of eq. realmatrix with the real values of S at the
// displacement I - J (cell units), read from a table over the margin
// |d_a| <= D = (c + 1) r - 1.  The sum is taken directly, cell pair by cell
// pair (the paper's local FFT convolution computes the same sum).  Two forms:
// k_hier_m2l on the matrix cores, and k_hier_m2l_cell with lanes per cell for
// what hier_mat_floats leaves to it.
#pragma once

#include "pmmm_hier.h"

namespace pmmm {
namespace hier_detail {

// Table value of Re S_nn^k / Im S_nn^k (any -nn <= k <= nn, conjugate
// relation) with nn and k known at compile time: a fixed address and sign.
template <int NN, int KK>
__device__ __forceinline__ float re_s_c(const float *g) {
    if constexpr (KK > NN || -KK > NN) return 0.0f;
    else if constexpr (KK >= 0) return g[NN * (NN + 1) + KK];
    else if constexpr (((-KK) & 1) != 0) return -g[NN * (NN + 1) - KK];
    else return g[NN * (NN + 1) - KK];
}
template <int NN, int KK>
__device__ __forceinline__ float im_s_c(const float *g) {
    if constexpr (KK == 0 || KK > NN || -KK > NN) return 0.0f;
    else if constexpr (KK > 0) return g[NN * (NN + 1) - KK];
    else if constexpr (((-KK) & 1) != 0) return g[NN * (NN + 1) + KK];
    else return -g[NN * (NN + 1) + KK];
}

// Output orders of the row groups of the kernel: group g takes the orders
// [hier_cut(PO, g), hier_cut(PO, g + 1)).  Up to order 4 one group holds
// every row; above it [0, 4), [4, 6) and one order per group from 6 on, so
// that a lane's FP64 sums, the moments it holds and the coefficient sums in
// flight stay within the register file (no spills up to order 10).
__host__ __device__ constexpr int hier_ngroups(int po) { return po <= 4 ? 1 : po - 3; }
__host__ __device__ constexpr int hier_cut(int po, int g) {
    return g == 0 ? 0 : g == hier_ngroups(po) ? po + 1 : (g == 1 ? 4 : g == 2 ? 6 : g + 4);
}

// Index of output row (l, m >= 0) in l-major order.
__host__ __device__ constexpr int hier_row(int l, int m) { return l * (l + 1) / 2 + m; }

// A group of `split` lanes per target fine cell and row group: the lanes of
// a group take the cell's source cells in turn, and per source cell the
// moments and the table row are read once and the rows of orders
// [LA, LE) of the (P x P) product of eq. realmatrix are unrolled at compile
// time (order PO).  Per-source sums in FP32, the sums over sources and over
// the group's lanes in FP64.  split is a power of two <= 64 (several lanes
// per cell fill the chip's SIMDs when a fine mesh has few cells for a kernel
// of this register size).
constexpr int kHierCellThreads = 64;
template <int PO, int LA, int LE>
__device__ __forceinline__ void hier_cell_rows(const float *__restrict__ M, float *__restrict__ L,
                                               const float *__restrict__ table, int nf, int r,
                                               int cutoff, int D, int split) {
    constexpr int P = nreal(PO), Q = nreal(2 * PO);
    constexpr int A0 = LA * LA, NA = LE * LE - A0;
    constexpr int NR = hier_row(LE, 0) - hier_row(LA, 0);   // rows (l, m >= 0), LA <= l < LE
    const int64_t K = (int64_t)nf * nf * nf;
    const int part = (int)threadIdx.x & (split - 1);
    const int64_t I = ((int64_t)blockIdx.x * kHierCellThreads + threadIdx.x) / split;
    const bool active = I < K;
    const int W = 2 * D + 1;
    const int64_t Ic = active ? I : 0;
    const int ix = (int)(Ic % nf), iy = (int)((Ic / nf) % nf), iz = (int)(Ic / ((int64_t)nf * nf));
    const int nc = nf / r;
    int lo[3], w[3];
    const int ii[3] = {ix, iy, iz};
    for (int a = 0; a < 3; ++a) {
        const int C = ii[a] / r;
        lo[a] = (C - cutoff > 0 ? C - cutoff : 0) * r;
        w[a] = (C + cutoff < nc - 1 ? C + cutoff : nc - 1) * r + r - lo[a];
    }
    const int count = active ? w[0] * w[1] * w[2] : 0;
    double acc[NA];
    static_for<0, NA>([&](auto ia) { acc[decltype(ia)::value] = 0.0; });
    for (int sidx = part; sidx < count; sidx += split) {
        const int jx = lo[0] + sidx % w[0];
        const int t = sidx / w[0];
        const int jy = lo[1] + t % w[1];
        const int jz = lo[2] + t / w[1];
        const int dx = ix - jx, dy = iy - jy, dz = iz - jz;
        int cheb = abs(dx) > abs(dy) ? abs(dx) : abs(dy);
        cheb = cheb > abs(dz) ? cheb : abs(dz);
        if (cheb <= cutoff) continue;
        const float *g = table + (((int64_t)(dz + D) * W + (dy + D)) * W + (dx + D)) * Q;
        const float *MJ = M + ((int64_t)jz * nf + jy) * nf + jx;
        float mj[P];
        static_for<0, P>([&](auto ia) {
            constexpr int a = decltype(ia)::value;
            mj[a] = MJ[(int64_t)a * K];
        });
        // FP32 sums of this source, one per output row (l, m >= 0); the
        // coefficient sums of a (nn, m, mu) are formed once and serve every
        // split nn = l + lambda
        float sre[NR], sim[NR];
        static_for<0, NR>([&](auto ir) {
            sre[decltype(ir)::value] = 0.0f;
            sim[decltype(ir)::value] = 0.0f;
        });
        static_for<LA, LE + PO>([&](auto inn) {
            constexpr int nn = decltype(inn)::value;
            static_for<0, (nn < LE - 1 ? nn : LE - 1) + 1>([&](auto im) {
                constexpr int m = decltype(im)::value;
                static_for<0, (nn < PO ? nn : PO) + 1>([&](auto imu) {
                    constexpr int mu = decltype(imu)::value;
                    // splits l + lambda = nn with LA <= l < LE, m <= l,
                    // mu <= lambda <= PO
                    constexpr int l_lo0 = nn - PO > LA ? nn - PO : LA;
                    constexpr int l_lo = l_lo0 > m ? l_lo0 : m;
                    constexpr int l_hi0 = nn - mu < LE - 1 ? nn - mu : LE - 1;
                    if constexpr (l_lo <= l_hi0) {
                        if constexpr (mu == 0) {
                            const float a0 = re_s_c<nn, -m>(g);
                            const float b0 = im_s_c<nn, -m>(g);
                            static_for<l_lo, l_hi0 + 1>([&](auto il) {
                                constexpr int l = decltype(il)::value;
                                constexpr int lam = nn - l;
                                constexpr int row = hier_row(l, m) - hier_row(LA, 0);
                                const float M0 = mj[lam * (lam + 1)];
                                sre[row] = __builtin_fmaf(a0, M0, sre[row]);
                                if constexpr (m > 0) sim[row] = __builtin_fmaf(b0, M0, sim[row]);
                            });
                        } else {
                            constexpr float sg = (mu & 1) ? -1.0f : 1.0f;
                            const float A = re_s_c<nn, -(m + mu)>(g);
                            const float B = im_s_c<nn, -(m + mu)>(g);
                            const float C = sg * re_s_c<nn, -(m - mu)>(g);
                            const float Dv = sg * im_s_c<nn, -(m - mu)>(g);
                            const float s1 = A + C, s2 = B - Dv, s3 = B + Dv, s4 = A - C;
                            static_for<l_lo, l_hi0 + 1>([&](auto il) {
                                constexpr int l = decltype(il)::value;
                                constexpr int lam = nn - l;
                                constexpr int row = hier_row(l, m) - hier_row(LA, 0);
                                const float Mr = mj[lam * (lam + 1) + mu];
                                const float Mi = mj[lam * (lam + 1) - mu];
                                // one FMA per multiply-add into the running
                                // sums (a - b inside += would cost a product,
                                // an FMA and an add)
                                sre[row] = __builtin_fmaf(s1, Mr, sre[row]);
                                sre[row] = __builtin_fmaf(-s2, Mi, sre[row]);
                                if constexpr (m > 0) {
                                    sim[row] = __builtin_fmaf(s3, Mr, sim[row]);
                                    sim[row] = __builtin_fmaf(s4, Mi, sim[row]);
                                }
                            });
                        }
                    }
                });
            });
        });
        static_for<LA, LE>([&](auto il) {
            constexpr int l = decltype(il)::value;
            static_for<0, l + 1>([&](auto im) {
                constexpr int m = decltype(im)::value;
                constexpr int row = hier_row(l, m) - hier_row(LA, 0);
                acc[l * (l + 1) + m - A0] += (double)sre[row];
                if constexpr (m > 0) acc[l * (l + 1) - m - A0] += (double)sim[row];
            });
        });
    }
    for (int off = 1; off < split; off <<= 1)
        static_for<0, NA>([&](auto ia) {
            constexpr int a = decltype(ia)::value;
            acc[a] += __shfl_xor(acc[a], off, kHierCellThreads);
        });
    if (!active || part != 0) return;
    static_for<0, NA>([&](auto ia) {
        constexpr int a = decltype(ia)::value;
        L[(int64_t)(A0 + a) * K + I] = (float)acc[a];
    });
}

// blockIdx.y selects the row group.
template <int PO>
__global__ __launch_bounds__(kHierCellThreads) void k_hier_m2l_cell(
    const float *__restrict__ M, float *__restrict__ L, const float *__restrict__ table, int nf,
    int r, int cutoff, int D, int split) {
    static_for<0, hier_ngroups(PO)>([&](auto ig) {
        constexpr int gi = decltype(ig)::value;
        if (blockIdx.y == gi)
            hier_cell_rows<PO, hier_cut(PO, gi), hier_cut(PO, gi + 1)>(M, L, table, nf, r, cutoff,
                                                                        D, split);
    });
}

// ---- matrix-core form ----
//
// Bound by the multiply-adds: 2 P^2 flops per pair of fine cells.  Target
// cells with the same position o inside their coarse cells see the same
// displacements: lane = coarse cell, and one source offset j (in fine cells
// from the target's coarse cell) has one P x P matrix T(o - j) for the whole
// wave.  v_mfma_f32_4x4x1 with its A operand broadcast from one of its 16
// blocks is then four rows of one column of T times one moment of 64 cells, so
// a register of 64 coefficients feeds 16 products and no row is padded beyond
// a multiple of four; its rate is twice what the vector unit reaches with one
// wave issuing, and it leaves that unit to the FP64 sums.  The matrices are
// written once per hierarchy in that register order, and the moments are read
// grouped by fine position (moment_place): 64 consecutive floats a load, where
// the strided rows made the loads the bound (16^3 x 4^3 cells, p = 6: 64.6 ms,
// grouped 28.1; the lane-per-cell form, whose lanes gather different table
// rows, 47.8).
//
// A row group is RBG blocks of four rows, at most nine (72 registers of FP64
// sums, 36 of FP32 sums); its columns go in NCH chunks of KC <= 8, a chunk's
// coefficients are NV registers of (column, row block) pairs, and the loads of
// a chunk are issued before the products of the one before.  Four waves per
// SIMD: at three (wider chunks, 136 registers) 64^3 x 2^3 cells, p = 4 took
// 5.85 ms, now 4.74, of which the products are 3.45 (lane per cell 8.19);
// 16^3 x 2^3 cells 101 us (212).
template <int PO>
struct HierMat {
    static constexpr int P = nreal(PO), RB = (P + 3) / 4;
    static constexpr int NG = (RB + 8) / 9, RBG = (RB + NG - 1) / NG;
    static constexpr int NCH = 2 * ((P + 15) / 16), KC = (P + NCH - 1) / NCH;
    static constexpr int NV = (KC * RBG + 15) / 16;
    static constexpr int WAVES = RBG <= 7 && PO <= 6 ? 4 : 3;   // per SIMD, without spills
    static constexpr int GSTRIDE = NCH * NV * 64, STRIDE = NG * GSTRIDE;   // floats per group, matrix
};

// Entry (row, col) of eq. realmatrix's matrix from the table row of S.
__device__ __forceinline__ float hier_entry(const float *g, int row, int col) {
    auto order = [](int a) {
        int l = 0;
        while ((l + 1) * (l + 1) <= a) ++l;
        return l;
    };
    auto sgn = [](int k) { return (k & 1) ? -1.0f : 1.0f; };
    auto re = [&](int n, int k) {
        if (k > n || -k > n) return 0.0f;
        return k >= 0 ? g[n * (n + 1) + k] : sgn(k) * g[n * (n + 1) - k];
    };
    auto im = [&](int n, int k) {
        if (k == 0 || k > n || -k > n) return 0.0f;
        return k > 0 ? g[n * (n + 1) - k] : -sgn(k) * g[n * (n + 1) + k];
    };
    const int l = order(row), mm = row - l * (l + 1), m = abs(mm);
    const int lam = order(col), uu = col - lam * (lam + 1), mu = abs(uu), nn = l + lam;
    if (mu == 0) return mm >= 0 ? re(nn, -m) : im(nn, -m);
    const float sg = sgn(mu);
    if (mm >= 0)
        return uu > 0 ? re(nn, -(m + mu)) + sg * re(nn, -(m - mu))
                      : sg * im(nn, -(m - mu)) - im(nn, -(m + mu));
    return uu > 0 ? im(nn, -(m + mu)) + sg * im(nn, -(m - mu))
                  : re(nn, -(m + mu)) - sg * re(nn, -(m - mu));
}

// All matrices in register order: thread = one float of mat; the lanes of an
// unused pair or row hold zero.
template <int PO>
__global__ __launch_bounds__(256) void k_hier_matrices(const float *__restrict__ table,
                                                       float *__restrict__ mat, int64_t cnt) {
    using H = HierMat<PO>;
    constexpr int Q = nreal(2 * PO);
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= cnt * H::STRIDE) return;
    const int64_t d = t / H::STRIDE;
    const int e = (int)(t - d * H::STRIDE);
    const int lane = e & 63, v = (e >> 6) % H::NV, ch = (e >> 6) / H::NV % H::NCH;
    const int grp = e / H::GSTRIDE;
    const int pair = v * 16 + (lane >> 2), kk = pair / H::RBG;
    const int col = ch * H::KC + kk, row = (grp * H::RBG + pair % H::RBG) * 4 + (lane & 3);
    mat[t] = kk < H::KC && col < H::P && row < H::P ? hier_entry(table + d * Q, row, col) : 0.0f;
}

typedef float hier_f4 __attribute__((ext_vector_type(4)));
constexpr int kHierMaxSplit = 8;
constexpr int64_t kHierMaxMatBytes = (int64_t)512 << 20;

// One block: the 64 coarse cells of group blockIdx.x / r^3 at one position o
// and one row group (blockIdx.y); its waves take the sources in turn and
// their FP64 sums are added through LDS in wave order.
template <int PO>
__global__ __launch_bounds__(64 * kHierMaxSplit, HierMat<PO>::WAVES) void k_hier_m2l(
    const float *__restrict__ M, float *__restrict__ L, const float *__restrict__ mat, int ln, int lr,
    int cutoff, int D) {
    using H = HierMat<PO>;
    constexpr int P = H::P, RBG = H::RBG, KC = H::KC, NV = H::NV, NCH = H::NCH;
    extern __shared__ double part[];   // [split][4][64]
    const int nf = 1 << ln, r = 1 << lr, lc = ln - lr, nc = 1 << lc;
    const int K = 1 << (3 * ln), r3 = 1 << (3 * lr), W = 2 * D + 1;
    const int split = (int)(blockDim.x >> 6);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int item = xcd_tile(blockIdx.x, gridDim.x), o = item & (r3 - 1);
    const int ox = o & (r - 1), oy = (o >> lr) & (r - 1), oz = o >> (2 * lr);
    const int C = (item >> (3 * lr)) * 64 + lane;
    const bool active = C < 1 << (3 * lc);
    const int cx = C & (nc - 1), cy = (C >> lc) & (nc - 1), cz = C >> (2 * lc);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)M, 0, (int)((int64_t)P * K * sizeof(float)), 0x00027000);
    const int span = (2 * cutoff + 1) * r;
    const int grp = blockIdx.y;

    // next source of this wave that some lane has: its matrix and the byte
    // offset of the lane's source cell (out of range, which loads zero, where
    // the cell is outside the mesh)
    const int j0 = -cutoff * r, j1 = j0 + span;
    int jx = j0 + wave - split, jy = j0, jz = j0;
    const float *T = nullptr;
    int voff = 0;
    auto next = [&]() -> bool {
        while (true) {
            for (jx += split; jx >= j1; jx -= span)
                if (++jy == j1) {
                    jy = j0;
                    ++jz;
                }
            if (jz >= j1) return false;
            const int dx = ox - jx, dy = oy - jy, dz = oz - jz;
            int cheb = abs(dx) > abs(dy) ? abs(dx) : abs(dy);
            cheb = cheb > abs(dz) ? cheb : abs(dz);
            if (cheb <= cutoff) continue;
            const int x = cx + (jx >> lr), y = cy + (jy >> lr), z = cz + (jz >> lr);
            const bool in = active && (unsigned)x < (unsigned)nc && (unsigned)y < (unsigned)nc &&
                            (unsigned)z < (unsigned)nc;
            if (__ballot(in) == 0) continue;
            const int oj = ((((jz & (r - 1)) << lr) | (jy & (r - 1))) << lr) | (jx & (r - 1));
            voff = in ? ((oj << (3 * lc)) + (((z << lc) + y) << lc) + x) * (int)sizeof(float)
                      : (int)0x80000000;
            T = mat + ((int64_t)((dz + D) * W + (dy + D)) * W + (dx + D)) * H::STRIDE +
                grp * H::GSTRIDE;
            return true;
        }
    };
    float mv[2][KC], av[2][NV];
    auto load = [&](auto ich, float (&m)[KC], float (&a)[NV]) {
        constexpr int ch = decltype(ich)::value;
        static_for<0, NV>([&](auto iv) {
            constexpr int v = decltype(iv)::value;
            a[v] = T[(ch * NV + v) * 64 + lane];
        });
        static_for<0, KC>([&](auto ik) {
            constexpr int k = decltype(ik)::value;
            if constexpr (ch * KC + k < P)
                m[k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                     rs, voff, (ch * KC + k) * K * (int)sizeof(float), 0));
        });
    };
    double acc[4 * RBG];
    static_for<0, 4 * RBG>([&](auto ia) { acc[decltype(ia)::value] = 0.0; });
    bool more = next();
    if (more) load(std::integral_constant<int, 0>{}, mv[0], av[0]);
    while (more) {
        hier_f4 s[RBG];
        static_for<0, RBG>([&](auto ib) { s[decltype(ib)::value] = hier_f4{0.0f, 0.0f, 0.0f, 0.0f}; });
        static_for<0, NCH>([&](auto ich) {
            constexpr int ch = decltype(ich)::value;
            if constexpr (ch + 1 < NCH) {
                load(std::integral_constant<int, ch + 1>{}, mv[(ch + 1) & 1], av[(ch + 1) & 1]);
            } else {
                more = next();
                if (more) load(std::integral_constant<int, 0>{}, mv[0], av[0]);
            }
            __builtin_amdgcn_sched_barrier(0);
            static_for<0, KC>([&](auto ik) {
                constexpr int k = decltype(ik)::value;
                if constexpr (ch * KC + k < P)
                    static_for<0, RBG>([&](auto ib) {
                        constexpr int b = decltype(ib)::value, pair = k * RBG + b;
                        s[b] = __builtin_amdgcn_mfma_f32_4x4x1f32(av[ch & 1][pair / 16], mv[ch & 1][k],
                                                                  s[b], 4, pair % 16, 0);
                    });
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        static_for<0, RBG>([&](auto ib) {
            constexpr int b = decltype(ib)::value;
            static_for<0, 4>([&](auto ii) {
                constexpr int i = decltype(ii)::value;
                acc[4 * b + i] += (double)s[b][i];
            });
        });
    }
    const int I = active ? (((cz * r + oz) * nf) + cy * r + oy) * nf + cx * r + ox : 0;
    static_for<0, RBG>([&](auto ib) {
        constexpr int b = decltype(ib)::value;
        __syncthreads();
        static_for<0, 4>([&](auto ii) {
            constexpr int i = decltype(ii)::value;
            part[(wave * 4 + i) * 64 + lane] = acc[4 * b + i];
        });
        __syncthreads();
        for (int i = wave; i < 4; i += split) {
            const int row = (grp * RBG + b) * 4 + i;
            if (row >= P || !active) continue;
            double t = part[i * 64 + lane];
            for (int w = 1; w < split; ++w) t += part[(w * 4 + i) * 64 + lane];
            L[(int64_t)row * K + I] = (float)t;
        }
    });
}

}  // namespace hier_detail

// Floats of the matrices of W^3 displacements for a fine mesh nf^3 refined by
// r; 0 where the lane-per-cell form serves instead:
//  - matrices above kHierMaxMatBytes (r = 8, or r = 4 with c = 2 at high
//    orders), which are not kept;
//  - coarse meshes so small that much of a neighbourhood lies outside, whose
//    offsets the matrix form runs for whole waves all the same.  Fine level in
//    us, table / matrices: 2^3 cells always table (r = 2, c = 1, p = 4 24 / 54);
//    4^3, c = 2 table below order 8 (r = 2: p = 0 22 / 48, p = 4 147 / 212;
//    r = 4: p = 0 144 / 350, p = 6 2438 / 3864, p = 8 7797 / 6733); 4^3, c = 1
//    below order 2 (r = 4: p = 0 67 / 83, p = 1 92 / 98, p = 3 268 / 198); 8^3,
//    c = 2 below order 2 (r = 2: p = 0 40 / 47, p = 1 52 / 55, p = 2 91 / 78);
//    larger ones never (8^3, c = 1, r = 2: p = 0 15 / 15, p = 4 67 / 56; 16^3,
//    c = 2, r = 2: p = 0 78 / 66, p = 4 778 / 382);
//  - r = 1, where every source is near, up to 16^3 cells (p = 4 7 / 9, p = 5 8 /
//    10; 32^3: p = 4 14 / 11);
//  - above order 4, fewer than 1024 waves: a wave's chain of products is then
//    the longer one (c = 1, r = 2: 4^3 cells, p = 5 76 / 91, p = 10 263 / 278;
//    8^3, p = 5 87 / 93; from 1024 waves on 8^3, p = 6 137 / 110, 16^3, p = 8
//    2353 / 1088).
template <int PO>
int64_t hier_mat_floats(int nf, int r, int D) {
    using H = hier_detail::HierMat<PO>;
    const int64_t nc = nf / r, r3 = (int64_t)r * r * r, items = (nc * nc * nc + 63) / 64 * r3;
    const int c = (D + 1) / r - 1;
    if (nc < 4 || (nc == 4 && PO < (c == 2 ? 8 : 2)) || (nc == 8 && c == 2 && PO < 2)) return 0;
    if (r == 1 && nc < 32) return 0;
    if (PO > 4 && items * H::NG * hier_detail::kHierMaxSplit < 1024) return 0;
    const int64_t W = 2 * D + 1, cnt = W * W * W * H::STRIDE;
    return cnt * (int64_t)sizeof(float) <= hier_detail::kHierMaxMatBytes ? cnt : 0;
}

template <int PO>
hipError_t hier_mat_build(int D, const float *table, float *mat, hipStream_t s) {
    const int64_t W = 2 * D + 1, cnt = W * W * W, n = cnt * hier_detail::HierMat<PO>::STRIDE;
    hipLaunchKernelGGL(hier_detail::k_hier_matrices<PO>, dim3((unsigned)((n + 255) / 256)), dim3(256),
                       0, s, table, mat, cnt);
    return hipGetLastError();
}

// Launch of the kernel for order PO (one compile unit per order).
template <int PO>
hipError_t hier_cell_launch(const HierArgs &a, hipStream_t s) {
    const int64_t K = (int64_t)a.nf * a.nf * a.nf;
    if (a.mat) {
        using H = hier_detail::HierMat<PO>;
        const int64_t nc = a.nf / a.r, r3 = (int64_t)a.r * a.r * a.r, items = (nc * nc * nc + 63) / 64 * r3;
        // waves per item that share its sources: four waves per SIMD over
        // the chip (256 CUs x 4 SIMDs), at most eight
        int split = 1;
        while (split < hier_detail::kHierMaxSplit && items * H::NG * split < 4096) split <<= 1;
        hipLaunchKernelGGL(hier_detail::k_hier_m2l<PO>, dim3((unsigned)items, H::NG), dim3(64 * split),
                           sizeof(double) * 256 * split, s, a.M, a.L, a.mat, __builtin_ctz(a.nf), __builtin_ctz(a.r), a.cutoff, a.D);
        return hipGetLastError();
    }
    constexpr int NG = hier_detail::hier_ngroups(PO);
    // Lanes per cell and row group: enough waves for four per SIMD
    // (256 CUs x 4 SIMDs), at most 8.
    int split = 1;
    while (split < 8 && K * NG * split < (int64_t)4 * 1024 * hier_detail::kHierCellThreads) split <<= 1;
    const int64_t nthr = K * split;
    hipLaunchKernelGGL(hier_detail::k_hier_m2l_cell<PO>,
                       dim3((unsigned)((nthr + hier_detail::kHierCellThreads - 1) / hier_detail::kHierCellThreads), NG),
                       dim3(hier_detail::kHierCellThreads), 0, s, a.M, a.L, a.table, a.nf, a.r, a.cutoff, a.D,
                       split);
    return hipGetLastError();
}

}  // namespace pmmm

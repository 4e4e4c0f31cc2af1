// Near field (Sec. 2.1, last paragraph, and Sec. 2.3): the particles of the
// (2c+1)^3 cells masked out of the transfer kernel interact by direct
// Newtonian sums with no cutoff function.  Periodic meshes take, for each
// neighbour cell, the one image within c cells of the target cell.
//
// Two kernels share the targets, row of cells (fixed y and z) by row:
//   k_near_list   lists the work: a row with kNearLight near pairs per cell on
//                 average (near_pairs_reach) gives its non-empty cells, in pieces of at most
//                 kNearTargets targets; any other row gives tiles of kNearTile
//                 consecutive sorted targets.  The lists' order
//                 varies from call to call (positions are reserved with
//                 atomics), their entries and results do not.
//   k_near_cells  one block per piece of a cell: 256 threads, or one wave
//                 where the row's cells have few pairs
//   k_near        one wave per tile (the other rows)
// Results (caller units) are stored or added to the sorted-order records that
// k_unpermute sends back to the caller's order.
//
// Displacements are formed from the integer cell offset and the in-cell
// offsets u (|u| <= 1/2), so FP32 keeps its relative precision on near pairs.
// At most 64 sources are summed in T, those sums in FP64: a target meets
// ~10^3 sources, and one long FP32 running sum would lose about
// sqrt(10^3 / 2) roundings' worth of accuracy.
#include "pmmm_internal.h"

namespace pmmm {

constexpr int kNearTile = 64;       // targets per tile (one wave)
constexpr int kNearThreads = 256;   // threads per piece of a heavy cell
constexpr int kNearTargets = 64;    // targets per piece: two per lane, several source parts
constexpr int kNearSeg = 63;        // sources of one part per chunk (an FP32 running sum)
// Lists of one call: the first slot of every tile, and per piece j of a cell
// its first slot + j (j is below the cell's count, so the slot names the cell;
// one-wave pieces from the front of the array, the others from its end), and their counts (zeroed by the binning).  One wave per row of cells
// (n <= 128: two cells per lane), 16 rows per block, which reserves its places
// with one atomic per list (one per row took 190 us at 128^2 rows).
__global__ void __launch_bounds__(1024) k_near_list(int n, int nx, int cutoff, int periodic,
                                                    int64_t light_pairs, int64_t heavy_pairs,
                                                    int most_around,
                                                    const int *__restrict__ start,
                                                    int *__restrict__ tiles,
                                                    int *__restrict__ pieces, int last_piece,
                                                    int *__restrict__ counts) {
    __shared__ int cnt[3][16];          // tiles, light pieces, heavy pieces of each wave
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int r = blockIdx.x * 16 + wid;
    int row0 = 0, np = 0, around = 0, c[2] = {0, 0}, first[2] = {0, 0};
    if (r < n * n) {
        const int *row = start + (int64_t)r * n;
        row0 = row[0];
        np = row[n] - row0;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int x = lane + 64 * u;
            first[u] = x < n ? row[x] : 0;
            c[u] = x < n ? row[x + 1] - first[u] : 0;
        }
        const int w = 2 * cutoff + 1;
        if (lane < w * w) {             // a row around this one per lane
            int jz = r / n + lane / w - cutoff, jy = r % n + lane % w - cutoff;
            const bool in = jz >= 0 && jz < n && jy >= 0 && jy < n;
            jz += jz < 0 ? n : jz >= n ? -n : 0;
            jy += jy < 0 ? n : jy >= n ? -n : 0;
            const int *near = start + ((int64_t)jz * n + jy) * n;
            if (in || periodic) around = near[n] - near[0];
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) around += __shfl_xor(around, off, 64);
    const bool dense = around >= most_around ||
                       near_pairs_reach(np, around, nx, cutoff, light_pairs);
    const bool heavy = near_pairs_reach(np, around, nx, cutoff, heavy_pairs);
    const int nt = dense ? 0 : (np + kNearTile - 1) / kNearTile;
    int J[2], inc;
#pragma unroll
    for (int u = 0; u < 2; ++u) J[u] = dense ? (c[u] + kNearTargets - 1) / kNearTargets : 0;
    inc = J[0] + J[1];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int u = __shfl_up(inc, off, 64);
        if (lane >= off) inc += u;
    }
    if (lane == 63) {
        cnt[0][wid] = nt;
        cnt[1][wid] = heavy ? 0 : inc;
        cnt[2][wid] = heavy ? inc : 0;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        // exclusive prefix of the waves' counts after the block's first place
        int *k = cnt[threadIdx.x], tot = 0;
        for (int v = 0; v < 16; ++v) tot += k[v];
        int base = tot > 0 ? atomicAdd(counts + threadIdx.x, tot) : 0;
        for (int v = 0; v < 16; ++v) {
            const int kv = k[v];
            k[v] = base;
            base += kv;
        }
    }
    __syncthreads();
    for (int t = lane; t < nt; t += 64)
        tiles[cnt[0][wid] + t] = row0 + t * kNearTile;
    int at = cnt[heavy ? 2 : 1][wid] + inc - J[0] - J[1];
#pragma unroll
    for (int u = 0; u < 2; ++u)
        for (int j = 0; j < J[u]; ++j, ++at)
            pieces[heavy ? last_piece - at : at] = first[u] + j;
}

// 1 / sqrt(r2).  FP64: the hardware estimate and one third-order step, to
// about one unit in the last place; r2 = 0 or infinite keeps the estimate
// (infinite or 0), which the step would turn into NaN.
__device__ __forceinline__ float near_rsqrt(float r2) { return __builtin_amdgcn_rsqf(r2); }
__device__ __forceinline__ double near_rsqrt(double r2) {
    const double y = __builtin_amdgcn_rsq(r2);
    const double e = fma(-(r2 * y), y, 1.0);
    const double t = fma(y, e * fma(0.375, e, 0.5), y);
    return __builtin_amdgcn_class(r2, 0x180) ? t : y;   // positive, normal or subnormal
}

// Sources staged in LDS for one chunk: offsets u and charge, the y and z
// offsets already moved into the target row's frame (u + row offset), the
// source cell's x in the tile's unwrapped frame, and its sorted slot.
template <typename T>
struct NearSrc {
    T ux, yz[2], q;
};

// Cell-index arithmetic on rows of n cells: shifts for power-of-two n (POW2),
// divisions otherwise.
template <bool POW2>
struct RowIdx {
    int n, logn;
    __device__ __forceinline__ int mul(int v) const { return POW2 ? v << logn : v * n; }
    __device__ __forceinline__ int div(int v) const { return POW2 ? v >> logn : v / n; }  // v >= 0
    __device__ __forceinline__ int mod(int v) const { return POW2 ? v & (n - 1) : v % n; }  // v >= 0
};

// Sparse rows: a tile of 64 consecutive targets of one row per wave.  For
// every neighbour row (dy, dz) the source cells the tile needs, x in
// [xa - c, xb + c] for targets in cells xa..xb, are contiguous sorted slots
// (split where a periodic row wraps, each piece with its image shift), which
// the wave streams in chunks of 64 through LDS; every lane reads each source
// as a broadcast, and a per-pair mask keeps exactly the neighbour cells of
// the lane's own target and drops the target itself.
template <typename T, bool POW2>
__global__ void __launch_bounds__(kNearTile) k_near(int n, int logn, int cutoff, int periodic,
                                                    const int *__restrict__ start,
                                                    const int *__restrict__ scell,
                                                    const particle4<T> *__restrict__ sorted,
                                                    const int *__restrict__ tiles,
                                                    const int *__restrict__ ntiles, T inv_h,
                                                    out4<T> *__restrict__ staged, int accumulate) {
    __shared__ NearSrc<T> src[kNearTile];
    __shared__ int2 sx_slot[kNearTile];
    const int lane = threadIdx.x;
    const int t = blockIdx.x;
    if (t >= ntiles[0]) return;  // the whole (one-wave) block leaves
    const RowIdx<POW2> ri{n, logn};
    const int s0 = tiles[t], r = ri.div(scell[s0]);
    const int s1 = min(s0 + kNearTile, start[ri.mul(r + 1)]);
    const int s = s0 + lane;
    const bool live = s < s1;
    const int sc = live ? s : s1 - 1;
    const particle4<T> me = sorted[sc];
    const int tx = ri.mod(scell[sc]);
    const int xa = ri.mod(scell[s0]), xb = ri.mod(scell[s1 - 1]);  // sorted: xa <= xb
    const int iz = ri.div(r), iy = ri.mod(r);
    const int c = cutoff;
    double tph = 0.0, tax = 0.0, tay = 0.0, taz = 0.0;
    for (int dz = -c; dz <= c; ++dz) {
        int jz = iz + dz;
        if (jz < 0 || jz >= n) {
            if (!periodic) continue;
            jz += jz < 0 ? n : -n;      // |dz| <= c < n
        }
        for (int dy = -c; dy <= c; ++dy) {
            int jy = iy + dy;
            if (jy < 0 || jy >= n) {
                if (!periodic) continue;
                jy += jy < 0 ? n : -n;
            }
            const int jrow = ri.mul(jz) + jy;
            // unwrapped x range of the sources, in pieces that do not wrap
            int lo = xa - c, hi = xb + c;
            if (!periodic) {
                lo = lo < 0 ? 0 : lo;
                hi = hi > n - 1 ? n - 1 : hi;
            }
            for (int u0 = lo; u0 <= hi;) {
                // image shift of the piece holding u0: floor(u0 / n) n
                const int shift = ri.mul(u0 >= 0 ? ri.div(u0) : -ri.div(n - 1 - u0));
                const int x0 = u0 - shift;
                const int x1 = hi - shift < n - 1 ? hi - shift : n - 1;
                const int b0 = start[ri.mul(jrow) + x0], b1 = start[ri.mul(jrow) + x1 + 1];
                for (int c0 = b0; c0 < b1; c0 += kNearTile) {
                    const int cnt = b1 - c0 < kNearTile ? b1 - c0 : kNearTile;
                    {
                        const int js = c0 + lane < b1 ? c0 + lane : b1 - 1;
                        const particle4<T> so = sorted[js];
                        const int sxu = ri.mod(scell[js]) + shift;
                        __syncthreads();  // the previous chunk has been read
                        // target - source displacement in y and z is
                        // (u_t - u_s) - (row offset): keep u_s + offset
                        src[lane] = NearSrc<T>{so.ux, {so.uy + T(dy), so.uz + T(dz)},
                                               c0 + lane < b1 ? so.q : T(0)};
                        sx_slot[lane] = make_int2(sxu, js);
                        __syncthreads();
                    }
                    const int cnt4 = (cnt + 3) & ~3;
                    T ph = T(0), ax = T(0), ay = T(0), az = T(0);
                    for (int k0 = 0; k0 < cnt4; k0 += 4) {
#pragma unroll
                        for (int kk = 0; kk < 4; ++kk) {
                            const int k = k0 + kk;
                            const NearSrc<T> sv = src[k < cnt ? k : cnt - 1];
                            const int2 xs = sx_slot[k < cnt ? k : cnt - 1];
                            const int o = tx - xs.x;  // target - source cell offset in x
                            const bool m = k < cnt && (unsigned)(o + c) <= (unsigned)(2 * c) &&
                                           xs.y != s;
                            const T dx = T(o) + (me.ux - sv.ux);
                            const T dyv = me.uy - sv.yz[0];
                            const T dzv = me.uz - sv.yz[1];
                            const T r2 = m ? dx * dx + dyv * dyv + dzv * dzv : T(1);
                            const T ri = near_rsqrt(r2);
                            const T qr = (m ? sv.q : T(0)) * ri;
                            ph += qr;
                            const T qr3 = qr * (ri * ri);
                            ax = fma(-qr3, dx, ax);
                            ay = fma(-qr3, dyv, ay);
                            az = fma(-qr3, dzv, az);
                        }
                    }
                    tph += (double)ph;
                    tax += (double)ax;
                    tay += (double)ay;
                    taz += (double)az;
                }
                u0 = x1 + shift + 1;
            }
        }
    }
    if (!live) return;
    const double ih = (double)inv_h, ih2 = ih * ih;
    out4<T> v{T(tph * ih), T(tax * ih2), T(tay * ih2), T(taz * ih2)};
    if (accumulate) {
        const out4<T> o = staged[s];
        v.phi += o.phi;
        v.gx += o.gx;
        v.gy += o.gy;
        v.gz += o.gz;
    }
    staged[s] = v;
}

// One pair: displacement target - source, the target itself dropped (SELF).
template <bool SELF, typename T>
__device__ __forceinline__ void near_pair(const particle4<T> &me, const particle4<T> &sv, bool self,
                                          T &ph, T &ax, T &ay, T &az) {
    const T dx = me.ux - sv.ux, dy = me.uy - sv.uy, dz = me.uz - sv.uz;
    T r2 = fma(dz, dz, fma(dy, dy, dx * dx));
    T q = sv.q;
    if constexpr (SELF) {
        r2 = self ? T(1) : r2;
        q = self ? T(0) : q;
    }
    const T ri = near_rsqrt(r2);
    const T qr = q * ri;
    ph += qr;
    const T w = qr * (ri * -ri);
    ax = fma(w, dx, ax);
    ay = fma(w, dy, ay);
    az = fma(w, dz, az);
}

// Dense rows: one block per piece of at most kNearTargets targets of ONE cell,
// so no pair needs a mask.  The sources of the (2c+1)^2 neighbour rows (one
// slot range each, two where a periodic row wraps) form one list, staged
// 2 NT at a time in LDS with their cell offset added; a lane holds two
// targets (g and g + G of the piece, G = half its targets) and sums one of
// `parts` contiguous segments of the chunk, parts = NT / G, so that small
// cells fill the block too.  The parts' FP64 sums are added in a fixed tree.
//
// Bound by VALU issue: 13 FP32 instructions and one v_rsq_f32 per pair (26 in
// k_near, whose tiles also evaluate 7 cells of a row for 5 at c = 2 and 32
// particles per cell): 3.1e12 pairs/s on the fine level of a clustered
// hierarchy (7.8e10 pairs, 35.0 -> 25 ms), 10^6 uniform particles on 32^3 cells
// 2.72 -> 1.4 ms, and in FP64 16384 particles on 8^3 cells 1.01 ms -> 85 us,
// where the split over source parts also fills the chip.  Operands stay in vector registers: two waves of a
// SIMD issue together only without scalar operands, at twice the rate.  Two
// targets per lane halve the 16-byte LDS broadcasts, which would otherwise
// take as long as the arithmetic.  More waves per SIMD (8 for 6), 128 or 32
// targets per piece, or chunks of one source per thread: 0.5-5% slower.
template <typename T, bool POW2, int NT>
__global__ void __launch_bounds__(NT, sizeof(T) == 4 ? 6 : 4) k_near_cells(
    int n, int logn, int cutoff, int periodic, const int *__restrict__ start,
    const int *__restrict__ scell, const particle4<T> *__restrict__ sorted,
    const int *__restrict__ pieces, int stride, const int *__restrict__ npieces, T inv_h,
    out4<T> *__restrict__ staged, int accumulate) {
    constexpr int kMaxRows = 25, U = 2, kChunk = U * NT;   // sources staged at a time
    __shared__ __align__(16) union {
        particle4<T> src[kChunk];
        double red[8][NT];
    } lds;
    // source ranges: first list index, sorted slot minus list index, and the
    // offsets of the range's row and image from the target's cell
    __shared__ int r_first[2 * kMaxRows + 1], r_slot[2 * kMaxRows], r_x[2 * kMaxRows];
    __shared__ T r_y[2 * kMaxRows], r_z[2 * kMaxRows];
    const int tid = threadIdx.x;
    const int w = 2 * cutoff + 1, nrange = 2 * w * w;
    const RowIdx<POW2> ri{n, logn};
    const int np = npieces[0];
    for (int it = blockIdx.x; it < np; it += gridDim.x) {
        const int pc = pieces[(int64_t)it * stride];
        const int cell = scell[pc], r = ri.div(cell), tx = ri.mod(cell);
        const int iz = ri.div(r), iy = ri.mod(r);
        const int c0 = start[cell], cn = start[cell + 1] - c0;
        // pieces of a cell are as even as possible
        const int J = (cn + kNearTargets - 1) / kNearTargets;
        const int per = (cn + J - 1) / J;
        const int s0 = c0 + (pc - c0) * per;
        const int cnt = min(per, c0 + cn - s0);
        if (cnt <= 0) continue;   // the same for every thread
        if (tid < 64) {
            int b0 = 0, b1 = 0, sx = 0, dy = 0, dz = 0;
            if (tid < nrange) {
                const int row = tid >> 1, second = tid & 1;
                dz = row / w - cutoff;
                dy = row - (dz + cutoff) * w - cutoff;
                int jy = iy + dy, jz = iz + dz;
                bool ok = true;
                if (jz < 0 || jz >= n) {
                    ok = periodic != 0;
                    jz += jz < 0 ? n : -n;
                }
                if (jy < 0 || jy >= n) {
                    ok = ok && periodic != 0;
                    jy += jy < 0 ? n : -n;
                }
                // x cells lo..hi; the part beyond the row's end is its image
                int lo = tx - cutoff, hi = tx + cutoff;
                int x0 = max(lo, 0), x1 = min(hi, n - 1);
                if (second) {
                    ok = ok && periodic != 0 && (lo < 0 || hi >= n);
                    sx = lo < 0 ? -n : n;
                    x0 = lo < 0 ? lo + n : 0;
                    x1 = lo < 0 ? n - 1 : hi - n;
                }
                if (ok) {
                    const int base = ri.mul(ri.mul(jz) + jy);
                    b0 = start[base + x0];
                    b1 = start[base + x1 + 1];
                }
            }
            int inc = b1 - b0;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int u = __shfl_up(inc, off, 64);
                if (tid >= off) inc += u;
            }
            if (tid < nrange) {
                const int first = inc - (b1 - b0);
                r_first[tid] = first;
                r_slot[tid] = b0 - first;
                r_x[tid] = sx - tx;
                r_y[tid] = T(dy);
                r_z[tid] = T(dz);
                if (tid == nrange - 1) r_first[nrange] = inc;
            }
        }
        __syncthreads();
        const int total = r_first[nrange];
        // the piece's own particles in the list: range of the target's row
        const int own = s0 - r_slot[2 * (cutoff * w + cutoff)];
        const int G = (cnt + 1) >> 1;
        const int parts = NT / G;
        const int k = min(tid / G, parts - 1), g = tid % G;
        const int t1 = min(g + G, cnt - 1);
        const particle4<T> me0 = sorted[s0 + g], me1 = sorted[s0 + t1];
        // chunks as even as possible; odd segments put the parts' sources in
        // different LDS banks
        int seg = kChunk / parts;
        seg = seg > kNearSeg ? kNearSeg : (seg - 1) | 1;
        const int nch = (total + seg * parts - 1) / (seg * parts);
        seg = ((total + nch * parts - 1) / (nch * parts)) | 1;
        const int len = seg * parts;
        particle4<T> rec[U];
        int rg = 0;               // range of this thread's next source
        auto load = [&](int f0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int e = tid + u * NT, f = f0 + e;
                if (e < len && f < total) {
                    // ranges only advance with f (u and chunks both increase it)
                    while (f >= r_first[rg + 1]) ++rg;
                    const int s = f + r_slot[rg];
                    particle4<T> v = sorted[s];
                    v.ux += T(ri.mod(scell[s]) + r_x[rg]);
                    v.uy += r_y[rg];
                    v.uz += r_z[rg];
                    rec[u] = v;
                } else {
                    rec[u] = particle4<T>{T(1e4), T(1e4), T(1e4), T(0)};   // adds nothing
                }
            }
        };
        double tot[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        load(0);
        // the targets arrive here, so that the pair loop waits for LDS only
        // and the next chunk's loads stay in flight behind it
        asm volatile("" ::"v"(me0.ux), "v"(me0.uy), "v"(me0.uz), "v"(me1.ux), "v"(me1.uy), "v"(me1.uz));
        for (int f0 = 0; f0 < total; f0 += len) {
            __syncthreads();      // the previous chunk (or reduction) has been read
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (tid + u * NT < len) lds.src[tid + u * NT] = rec[u];
            __syncthreads();
            if (f0 + len < total) load(f0 + len);
            const particle4<T> *sp = lds.src + k * seg;
            T p0 = T(0), x0 = T(0), y0 = T(0), z0 = T(0);
            T p1 = T(0), x1 = T(0), y1 = T(0), z1 = T(0);
            if (own < f0 + len && own + cnt > f0) {
                // this chunk holds some of the targets: source j0 (j1) of the
                // segment is the lane's own first (second) target
                const int j0 = own + g - f0 - k * seg, j1 = own + t1 - f0 - k * seg;
                for (int j = 0; j < seg; ++j) {
                    const particle4<T> sv = sp[j];
                    near_pair<true, T>(me0, sv, j == j0, p0, x0, y0, z0);
                    near_pair<true, T>(me1, sv, j == j1, p1, x1, y1, z1);
                }
            } else {
#pragma unroll 2
                for (int j = 0; j < seg; ++j) {
                    const particle4<T> sv = sp[j];
                    near_pair<false, T>(me0, sv, false, p0, x0, y0, z0);
                    near_pair<false, T>(me1, sv, false, p1, x1, y1, z1);
                }
            }
            tot[0] += (double)p0;
            tot[1] += (double)x0;
            tot[2] += (double)y0;
            tot[3] += (double)z0;
            tot[4] += (double)p1;
            tot[5] += (double)x1;
            tot[6] += (double)y1;
            tot[7] += (double)z1;
        }
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 8; ++v) lds.red[v][tid] = tot[v];
        __syncthreads();
        int step = 1;
        while (2 * step < parts) step *= 2;
        const bool act = tid < parts * G;
        for (; parts > 1 && step >= 1; step >>= 1) {
            if (act && k < step && k + step < parts) {
#pragma unroll
                for (int v = 0; v < 8; ++v) lds.red[v][tid] += lds.red[v][tid + step * G];
            }
            __syncthreads();
        }
        if (tid < cnt) {
            const int v0 = tid < G ? 0 : 4, c = tid < G ? tid : tid - G;
            const double ih = (double)inv_h, ih2 = ih * ih;
            out4<T> v{T(lds.red[v0][c] * ih), T(lds.red[v0 + 1][c] * ih2),
                      T(lds.red[v0 + 2][c] * ih2), T(lds.red[v0 + 3][c] * ih2)};
            if (accumulate) {
                const out4<T> o = staged[s0 + tid];
                v.phi += o.phi;
                v.gx += o.gx;
                v.gy += o.gy;
                v.gz += o.gz;
            }
            staged[s0 + tid] = v;
        }
        __syncthreads();          // the lists and sums are rewritten by the next piece
    }
}

// Upper bounds of the lists for np particles on n^3 cells (every piece holds a
// particle).
static int64_t max_row_tiles(int64_t np, int n) { return (np + kNearTile - 1) / kNearTile + (int64_t)n * n; }

template <typename T, bool POW2>
static void near_launch(const NearArgs &a, int logn, hipStream_t s) {
    const int64_t most = a.n;
    int *tiles = a.lists, *pieces = a.pieces;
    int *counts = a.small + 5;
    const int rows = a.ncell * a.ncell;
    const particle4<T> *sorted = (const particle4<T> *)a.sorted;
    const int64_t cells = bin_min64(a.n, a.cells), pieces_most = cells + a.n / kNearTargets;
    const int64_t heavy = pieces_most <= kNearFewPieces ? 0 : kNearHeavy;
    const int64_t light = heavy == 0 || cells <= kNearFewCells ? 0 : kNearLight;
    // a tile's wave takes the rows around one after the other: rows with far more
    // particles around them than the mean, or very many, go by cells too
    const int64_t w = 2 * a.cutoff + 1, mean4 = 4 * w * w * a.n / (a.cells / a.nx);
    const int most_around = (int)bin_min64(kNearMostAround, bin_max64(kNearMostAround / 4, mean4));
    // blocks loop over the pieces, which may be fewer (with none at all, 32600
    // blocks of 256 threads take 8.7 us, 3200 2.5)
    const int64_t most_rows = heavy > 0 ? near_rows_most(a.n, a.nx, a.cutoff, heavy) : rows;
    const int64_t wide = bin_min64(bin_min64(most_rows, rows) * a.nx + a.n / kNearTargets, pieces_most);
    const unsigned blocks256 = (unsigned)bin_min64(wide, 32768);
    const unsigned blocks64 = (unsigned)bin_min64(pieces_most, 32768);
    hipLaunchKernelGGL(k_near_list, dim3((rows + 15) / 16), dim3(1024), 0, s, a.ncell, a.nx,
                       a.cutoff, a.periodic, light, heavy, most_around, a.start, tiles, pieces,
                       (int)most - 1, counts);
    // launched where the particles suffice for one row of the kind
    if (near_pairs_reach(a.n, a.n, a.nx, a.cutoff, heavy))
        hipLaunchKernelGGL((k_near_cells<T, POW2, kNearThreads>), dim3(blocks256), dim3(kNearThreads),
                           0, s, a.ncell, logn, a.cutoff, a.periodic, a.start, a.scell, sorted,
                           pieces + most - 1, -1, counts + 2, T(a.inv_h), (out4<T> *)a.staged,
                           a.accumulate);
    if (heavy > 0 && (a.n >= most_around || near_pairs_reach(a.n, a.n, a.nx, a.cutoff, light)))
        hipLaunchKernelGGL((k_near_cells<T, POW2, 64>), dim3(blocks64), dim3(64), 0, s, a.ncell, logn,
                           a.cutoff, a.periodic, a.start, a.scell, sorted, pieces, 1, counts + 1,
                           T(a.inv_h), (out4<T> *)a.staged, a.accumulate);
    if (light > 0)
        hipLaunchKernelGGL((k_near<T, POW2>), dim3((unsigned)max_row_tiles(a.n, a.ncell)),
                           dim3(kNearTile), 0, s, a.ncell, logn, a.cutoff, a.periodic, a.start,
                           a.scell, sorted, tiles, counts, T(a.inv_h), (out4<T> *)a.staged,
                           a.accumulate);
}

template <typename T>
hipError_t launch_near(const NearArgs &a, hipStream_t s) {
    if (a.n == 0) return hipSuccess;
    // 25 neighbour rows and two cells per lane of k_near_list at most
    if (a.cutoff < 1 || a.cutoff > 2 || a.ncell > 128) return hipErrorInvalidValue;
    if ((a.ncell & (a.ncell - 1)) == 0)
        near_launch<T, true>(a, __builtin_ctz((unsigned)a.ncell), s);
    else
        near_launch<T, false>(a, 0, s);
    return hipGetLastError();
}

int64_t near_list_ints(int64_t n, int ncell) { return max_row_tiles(n, ncell); }

template hipError_t launch_near<float>(const NearArgs &, hipStream_t);
template hipError_t launch_near<double>(const NearArgs &, hipStream_t);

}  // namespace pmmm

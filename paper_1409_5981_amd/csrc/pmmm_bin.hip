// Cell binning (Sec. 2.1 requires that the particles of every cell be known,
// which takes linear time): a stable sort of the particles by cell index, so
// the particles of a cell keep the caller's order and every result is bitwise
// reproducible (no atomics decide an order).  The cell index is cut in two: a
// partition by its high bits, then a sort of every bucket by the low bits.
//   k_rb_hist     tile histogram of the high bits, computed from the positions
//                 (and flags open-boundary particles outside the box)
//   k_rb_scan1 or k_rb_scan_sums + k_rb_scan
//                 exclusive scan of the histograms in bucket-major order (so
//                 tile t's bucket-d elements start after every smaller bucket
//                 and after bucket d of the tiles before t)
//   k_rb_scatter  stable partition: each wave ranks a contiguous chunk of the
//                 tile (wave ballots for equal digits plus the wave's running
//                 count per digit), one prefix over the waves per tile, then
//                 the tile is put in digit order in LDS and written out in
//                 runs (key, caller index, particle record)
//   k_rb_hist2    histograms of the low bits for the chunks of buckets above
//                 kLocalTile particles (clustered input; other blocks leave)
//   k_rb_sums2    running sums of those over the chunks of a bucket of many
//   k_rb_local    sorts a bucket, or one chunk of a large one, by the low bits
//                 into its final place: sorted cell, permutation, records and,
//                 on request, each particle's sorted slot; the bucket's
//                 histogram is also the starts of its cells and lists the P2M
//                 work items of the cells above the dense threshold
//   k_bin_keys, k_bin_small   all of it in two launches, for few particles and
//                 cells
// Cell index: I = floor(r n / b) per axis, clamped to [0, n-1], along z of a
// flat open box to the box's own top cell (the stages of a call stop there);
// periodic positions are first wrapped into the box (in cell units).
//
// Batches: blockIdx.y selects one of several independent systems on meshes of
// the same size; prange[2s], prange[2s+1] bound system s's particles in the
// caller's arrays (null: one system, particles [0, n)), and its per-system
// arrays sit at fixed strides (start K + 1, small 8, histograms
// bin_hist_ints(max_np, K), scan sums bin_scan_tiles(max_np, K)).
#include "pmmm_internal.h"

namespace pmmm {

constexpr int kRadixBuckets = 1 << kRadixMaxBits;   // k_rb_hist, k_rb_scatter
constexpr int kLocalBuckets = 1 << kLocalMaxBits;   // k_rb_hist2, k_rb_local
constexpr int kScanOneBlock = 16384;   // histograms up to this size: one-block scan
// A chunk of a bucket of J <= kChunkRows chunks reads the J low-bit histograms
// itself; of a larger one it finds them summed (k_rb_sums2), where the call has
// more than kChunkSumMinN particles.  Up to there J is at most 512 and reading
// all rows costs 20 us of 286 with every particle in one bucket (10 of 227 at
// 2^20), the launch 3 us of every call.
constexpr int kChunkRows = 64;
constexpr int64_t kChunkSumMinN = int64_t(1) << 21;

template <typename T>
__device__ __forceinline__ void cell_coord(T v, T inv_h, int n, int top, int lim,
                                           int periodic, int &ic, T &u, int &outside) {
    T s = v * inv_h;
    if (periodic) {
        s = s - T(n) * floor(s / T(n));
    } else if (!(s >= T(0) && s < T(lim))) {
        outside = 1;
    }
    int i = (int)floor(s);
    i = i < 0 ? 0 : (i > top - 1 ? top - 1 : i);
    ic = i;
    u = s - T(i) - T(0.5);
}

// LDS of the scatter: the per-wave counts [16][nb], later reused as the
// staging area of one tile, then ls[nb], goff[nb], wtot[16].
template <typename T, int R>
__host__ __device__ constexpr size_t scatter_region(int bits) {
    return (size_t)16 * ((size_t)1 << bits) * sizeof(int) >
                   (size_t)1024 * R * sizeof(particle4<T>)
               ? (size_t)16 * ((size_t)1 << bits) * sizeof(int)
               : (size_t)1024 * R * sizeof(particle4<T>);
}
template <typename T, int R>
constexpr size_t scatter_lds(int bits) {
    return scatter_region<T, R>(bits) + (size_t)(2 * (1 << bits) + 16) * sizeof(int);
}

// Counts of one system's binning, written by its first kernel: dense P2M
// items, partial slots and split cells, and the near field's work lists.
__device__ __forceinline__ void reset_counts(int *__restrict__ small) {
    small[0] = 0;
    for (int k = 3; k < 8; ++k) small[k] = 0;
}

// Every system empty: zero starts and counts.
__global__ void __launch_bounds__(256) k_bin_empty(int K, int *__restrict__ start,
                                                   int *__restrict__ small) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c <= K) start[(int64_t)blockIdx.y * (K + 1) + c] = 0;
    if (c == 0) reset_counts(small + (int64_t)blockIdx.y * 8);
}

// Cell of particle i and its record.
template <typename T>
__device__ __forceinline__ int cell_record(const T *__restrict__ x, const T *__restrict__ y,
                                           const T *__restrict__ z, const T *__restrict__ q,
                                           int64_t i, T inv_h, int nc, int topz, int periodic,
                                           particle4<T> &rec) {
    int ix, iy, iz, out = 0;
    cell_coord(x[i], inv_h, nc, nc, nc, periodic, ix, rec.ux, out);
    cell_coord(y[i], inv_h, nc, nc, nc, periodic, iy, rec.uy, out);
    cell_coord(z[i], inv_h, nc, topz, nc, periodic, iz, rec.uz, out);
    rec.q = q != nullptr ? q[i] : T(0);
    return (iz * nc + iy) * nc + ix;
}

// Lanes of the wave that are active and hold the same digit d.
__device__ __forceinline__ uint64_t digit_peers(bool act, int d, int bits) {
    uint64_t peers = __ballot(act);
    for (int b = 0; b < bits; ++b) {
        const uint64_t m = __ballot(act && ((d >> b) & 1));
        peers &= ((d >> b) & 1) ? m : ~m;
    }
    return peers;
}

// Tile histogram of the bucket key >> shift, written to hist[d * tiles + t]
// (every block writes all 2^bits of its entries).
template <typename T, int R>
__global__ void __launch_bounds__(1024) k_rb_hist(
    const int64_t *__restrict__ prange, int64_t n, const T *__restrict__ x,
    const T *__restrict__ y, const T *__restrict__ z, T inv_h, int nc, int3 lim, int periodic,
    int *__restrict__ hist, int64_t hist_ints, int tiles, int shift, int bits,
    int *__restrict__ flag, int *__restrict__ small) {
    __shared__ int s_hist[kRadixBuckets];
    int64_t p0, np;
    sys_range(prange, n, p0, np);
    const int nb = 1 << bits, t = blockIdx.x;
    for (int d = threadIdx.x; d < nb; d += blockDim.x) s_hist[d] = 0;
    if (t == 0 && threadIdx.x == 0) reset_counts(small + (int64_t)blockIdx.y * 8);
    __syncthreads();
    int kv[R];
    int out = 0;
    T xv[R], yv[R], zv[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t j = (int64_t)t * (1024 * R) + r * 1024 + threadIdx.x;
        const int64_t i = p0 + (j < np ? j : 0);
        const bool act = j < np;
        xv[r] = act ? x[i] : T(0);
        yv[r] = act ? y[i] : T(0);
        zv[r] = act ? z[i] : T(0);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t j = (int64_t)t * (1024 * R) + r * 1024 + threadIdx.x;
        int ix, iy, iz;
        T u;
        cell_coord(xv[r], inv_h, nc, nc, lim.x, periodic, ix, u, out);
        cell_coord(yv[r], inv_h, nc, nc, lim.y, periodic, iy, u, out);
        cell_coord(zv[r], inv_h, nc, lim.z, lim.z, periodic, iz, u, out);
        kv[r] = j < np ? (iz * nc + iy) * nc + ix : -1;
    }
    if (out && np > 0) {
        // only lanes with particles can be outside (inactive lanes read 0)
        *flag = 1;
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (kv[r] >= 0) atomicAdd(&s_hist[kv[r] >> shift], 1);
    __syncthreads();
    int *h = hist + (int64_t)blockIdx.y * hist_ints;
    for (int d = threadIdx.x; d < nb; d += blockDim.x) h[(int64_t)d * tiles + t] = s_hist[d];
}

// Scanned values of the entries base .. base + C - 1 (the first is run), and
// the bucket starts -- the entries of tile 0 -- once more in a row behind the
// histogram, where every block of the local sort reads them all.
template <int C>
__device__ __forceinline__ void put_scanned(int *__restrict__ hist, int64_t base, int64_t L,
                                            int tiles, int run, const int *v) {
    int b = (int)(base / tiles), t = (int)(base - (int64_t)b * tiles);
#pragma unroll
    for (int k = 0; k < C; ++k) {
        if (base + k < L) {
            hist[base + k] = run;
            if (t == 0) hist[L + b] = run;
        }
        run += v[k];
        if (++t == tiles) {
            t = 0;
            ++b;
        }
    }
}

// Exclusive scan of the L (<= kScanOneBlock) histogram entries of every
// system in one block: 16 consecutive entries per thread.
__global__ void __launch_bounds__(1024) k_rb_scan1(int64_t L, int64_t hist_ints, int tiles,
                                                   int *__restrict__ hist) {
    __shared__ int wtot[16];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    hist += (int64_t)blockIdx.y * hist_ints;
    const int64_t base = (int64_t)tid * 16;
    int v[16];
    int tot = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        v[k] = base + k < L ? hist[base + k] : 0;
        tot += v[k];
    }
    int inc = tot;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int u = __shfl_up(inc, off, 64);
        if (lane >= off) inc += u;
    }
    if (lane == 63) wtot[wid] = inc;
    __syncthreads();
    int run = inc - tot;
    for (int w = 0; w < wid; ++w) run += wtot[w];
    put_scanned<16>(hist, base, L, tiles, run, v);
}

// The same for larger histograms, in scan tiles of 4096: per-tile sums, then
// each tile scanned from the sum of the tiles before it.
__global__ void __launch_bounds__(1024) k_rb_scan_sums(int64_t L, int64_t hist_ints,
                                                       const int *__restrict__ hist,
                                                       int *__restrict__ sums) {
    __shared__ int wsum[16];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    hist += (int64_t)blockIdx.y * hist_ints;
    sums += (int64_t)blockIdx.y * gridDim.x;
    const int64_t base = (int64_t)blockIdx.x * 4096 + tid * 4;
    int v = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (base + k < L) v += hist[base + k];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    if (lane == 0) wsum[wid] = v;
    __syncthreads();
    if (tid == 0) {
        int a = 0;
        for (int w = 0; w < 16; ++w) a += wsum[w];
        sums[blockIdx.x] = a;
    }
}

__global__ void __launch_bounds__(1024) k_rb_scan(int64_t L, int64_t hist_ints, int tiles,
                                                  int *__restrict__ hist,
                                                  const int *__restrict__ sums) {
    __shared__ int wtot[16];
    __shared__ int pre_s;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    hist += (int64_t)blockIdx.y * hist_ints;
    sums += (int64_t)blockIdx.y * gridDim.x;
    const int64_t base = (int64_t)blockIdx.x * 4096 + tid * 4;
    int v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = base + k < L ? hist[base + k] : 0;
    int pre = 0;
    for (int k = tid; k < (int)blockIdx.x; k += 1024) pre += sums[k];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) pre += __shfl_xor(pre, off, 64);
    if (lane == 0) wtot[wid] = pre;
    __syncthreads();
    if (tid == 0) {
        int a = 0;
        for (int w = 0; w < 16; ++w) a += wtot[w];
        pre_s = a;
    }
    __syncthreads();
    const int tot = (v[0] + v[1]) + (v[2] + v[3]);
    int inc = tot;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int u = __shfl_up(inc, off, 64);
        if (lane >= off) inc += u;
    }
    if (lane == 63) wtot[wid] = inc;
    __syncthreads();
    int run = pre_s + inc - tot;
    for (int w = 0; w < wid; ++w) run += wtot[w];
    put_scanned<4>(hist, base, L, tiles, run, v);
}

// P2M items of a dense cell of cnt particles: J = ceil(cnt / kDenseItem) items
// {cell, j, J, first partial slot (J > 1) or -1}, a cell of J > 1 also as split
// {cell, J, first slot}; or (whole) one item for the cell.  Places are reserved with atomics, so they vary from
// call to call, but every item covers a fixed particle range and the partials
// of a cell are added in a fixed order, so the moments do not.
__device__ __forceinline__ void list_dense(int cell, int cnt, int whole, int4 *__restrict__ items,
                                           int64_t items_cap, int64_t splits_cap,
                                           int *__restrict__ small) {
    const int J = whole ? 1 : (cnt + kDenseItem - 1) / kDenseItem;
    const int base = atomicAdd(small, J);
    const int ps = J > 1 ? atomicAdd(small + 3, J) : -1;
    for (int j = 0; j < J; ++j)
        if (base + j < items_cap - splits_cap) items[base + j] = int4{cell, j, J, ps};
    if (J > 1) {
        const int si = atomicAdd(small + 4, 1);
        if (si < splits_cap) items[items_cap - splits_cap + si] = int4{cell, J, ps, 0};
    }
}

// Stable partition by the bucket over tiles of 1024 R elements; wave w ranks
// elements [64 R w, 64 R (w + 1)) of its tile, 64 at a time.  With start the
// buckets are the cells (few cells): the partition is the whole sort, and tile
// 0 writes the starts and lists the dense cells as k_rb_local does.
template <typename T, int R>
__global__ void __launch_bounds__(1024) k_rb_scatter(
    const int64_t *__restrict__ prange, int64_t n, const T *__restrict__ x,
    const T *__restrict__ y, const T *__restrict__ z, const T *__restrict__ q, T inv_h, int nc,
    int topz, int periodic, int *__restrict__ keys_out, int *__restrict__ vals_out,
    particle4<T> *__restrict__ recs_out, const int *__restrict__ offs, int64_t hist_ints,
    int tiles, int shift, int bits, int K, int *__restrict__ pos, int *__restrict__ start,
    int dense_thr, int whole, int4 *__restrict__ items, int64_t items_cap, int64_t splits_cap,
    int *__restrict__ small) {
    constexpr int TILE = 1024 * R;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int nb = 1 << bits;
    int *wcnt = (int *)lds_raw;                      // [16][nb] while ranking
    int *sint = (int *)lds_raw;                      // staging: TILE ints
    particle4<T> *srec = (particle4<T> *)lds_raw;    // staging: TILE records
    int *ls = (int *)(lds_raw + scatter_region<T, R>(bits));  // [nb] tile-local digit start
    int *goff = ls + nb;                             // [nb] global slot - local slot
    int *wtot = goff + nb;                           // [16]
    int64_t p0, np;
    sys_range(prange, n, p0, np);
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    offs += (int64_t)blockIdx.y * hist_ints;
    const int64_t t0 = (int64_t)t * TILE;
    const int na = (int)(np - t0 <= 0 ? 0 : (np - t0 > TILE ? TILE : np - t0));
    for (int e = tid; e < 16 * nb; e += 1024) wcnt[e] = 0;
    if (start != nullptr && t == 0) {
        int *st = start + (int64_t)blockIdx.y * (K + 1);
        for (int d = tid; d <= K; d += 1024) {
            const int s0 = d < nb ? offs[(int64_t)d * tiles] : (int)np;
            const int s1 = d + 1 < nb ? offs[(int64_t)(d + 1) * tiles] : (int)np;
            st[d] = s0;
            if (d < K && items != nullptr && s1 - s0 > dense_thr)
                list_dense(d, s1 - s0, whole, items + (int64_t)blockIdx.y * items_cap, items_cap,
                           splits_cap, small + (int64_t)blockIdx.y * 8);
        }
    }

    int key[R], val[R], dig[R];
    particle4<T> rec[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = wid * 64 * R + r * 64 + lane;
        const int64_t i = p0 + t0 + (e < na ? e : 0);
        if (e < na) {
            key[r] = cell_record(x, y, z, q, i, inv_h, nc, topz, periodic, rec[r]);
            val[r] = (int)i;
        } else {
            key[r] = 0;
            val[r] = 0;
            rec[r] = particle4<T>{T(0), T(0), T(0), T(0)};
        }
        dig[r] = key[r] >> shift;
    }
    __syncthreads();

    // rank among the wave's earlier elements of the same digit: the running
    // count of the digit before this group of 64, plus the lower lanes that
    // hold it; one lane per digit group then advances the count (the wave's
    // LDS reads precede its writes, and only this wave touches its counts)
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    int rank[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = wid * 64 * R + r * 64 + lane;
        const bool act = e < na;
        const int d = dig[r];
        const uint64_t peers = digit_peers(act, d, bits);
        const int before = __popcll(peers & lt);
        const int base = act ? wcnt[wid * nb + d] : 0;
        __builtin_amdgcn_wave_barrier();
        rank[r] = base + before;
        if (act && before == 0) wcnt[wid * nb + d] = base + __popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();

    // per digit: exclusive prefix over the waves (in place) and the tile count;
    // thread tid holds the digits [tid DP, tid DP + DP)
    constexpr int DP = kRadixBuckets / 1024;
    int tot[DP], sum = 0;
#pragma unroll
    for (int u = 0; u < DP; ++u) {
        const int d = tid * DP + u;
        tot[u] = 0;
        if (d < nb) {
#pragma unroll
            for (int w = 0; w < 16; ++w) {
                const int c = wcnt[w * nb + d];
                wcnt[w * nb + d] = tot[u];
                tot[u] += c;
            }
        }
        sum += tot[u];
    }
    // exclusive scan of the tile counts over the digits
    int inc = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int u = __shfl_up(inc, off, 64);
        if (lane >= off) inc += u;
    }
    if (lane == 63) wtot[wid] = inc;
    __syncthreads();
    int l = inc - sum;
    for (int w = 0; w < wid; ++w) l += wtot[w];
#pragma unroll
    for (int u = 0; u < DP; ++u) {
        const int d = tid * DP + u;
        if (d < nb) {
            ls[d] = l;
            goff[d] = offs[(int64_t)d * tiles + t] - l;
        }
        l += tot[u];
    }
    __syncthreads();
    int lidx[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = wid * 64 * R + r * 64 + lane;
        lidx[r] = e < na ? ls[dig[r]] + wcnt[wid * nb + dig[r]] + rank[r] : 0;
    }
    __syncthreads();  // the counts' region becomes the staging area

    // the tile in digit order: slot jj of the tile goes to goff[digit] + jj
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (wid * 64 * R + r * 64 + lane < na) sint[lidx[r]] = key[r];
    __syncthreads();
    int dst[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int jj = r * 1024 + tid;
        dst[r] = 0;
        if (jj < na) {
            const int k = sint[jj];
            dst[r] = goff[k >> shift] + jj;
            keys_out[p0 + dst[r]] = k;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (wid * 64 * R + r * 64 + lane < na) sint[lidx[r]] = val[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int jj = r * 1024 + tid;
        if (jj < na) {
            const int v = sint[jj];
            vals_out[p0 + dst[r]] = v;
            if (pos != nullptr) pos[v] = (int)(p0 + dst[r]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (wid * 64 * R + r * 64 + lane < na) srec[lidx[r]] = rec[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int jj = r * 1024 + tid;
        if (jj < na) recs_out[p0 + dst[r]] = srec[jj];
    }
}

// The chunk of block blk: bucket b of the partition holds the slots [start,
// start + cnt) and makes J = max(1, ceil(cnt / kLocalTile)) chunks, of which
// this is chunk j; mbase counts the chunks of the buckets before it that make
// more than one.  b < 0: no such chunk.  Two barriers; scr: 2 x 16 ints.
// near: eight chunks in a row go to one XCD (blocks are dealt to the eight in
// turn), so that the runs which a bucket's chunks write side by side meet in one
// L2: uniform particles on 64^3 cells, binning of 2^24 665 -> 609 us, of 2^25
// 1298 -> 1179.  Longer stretches leave XCDs idle where most buckets are empty.
struct Chunk {
    int b, start, cnt, j, J, mbase;
};
__device__ __forceinline__ Chunk find_chunk(int blk, int nb, int64_t np, int near, const int *first_of,
                                            int *scr, Chunk *found) {
    constexpr int DP = kRadixBuckets / 1024;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    if (tid == 0) found->b = -1;
    int first[DP + 1], js = 0, ms = 0;
#pragma unroll
    for (int u = 0; u <= DP; ++u) {
        const int d = tid * DP + u;
        first[u] = d < nb ? first_of[d] : (int)np;
    }
    int J[DP], M[DP];
#pragma unroll
    for (int u = 0; u < DP; ++u) {
        const int c = (first[u + 1] - first[u] + kLocalTile - 1) / kLocalTile;
        J[u] = tid * DP + u < nb ? (c > 1 ? c : 1) : 0;
        M[u] = c > 1 ? c : 0;
        js += J[u];
        ms += M[u];
    }
    int ji = js, mi = ms;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int a = __shfl_up(ji, off, 64), m = __shfl_up(mi, off, 64);
        if (lane >= off) {
            ji += a;
            mi += m;
        }
    }
    if (lane == 63) {
        scr[wid] = ji;
        scr[16 + wid] = mi;
    }
    __syncthreads();
    ji -= js;
    mi -= ms;
    for (int w = 0; w < wid; ++w) {
        ji += scr[w];
        mi += scr[16 + w];
    }
    if (near) {
        int total = 0;
        for (int w = 0; w < 16; ++w) total += scr[w];
        if (blk < (total & ~63)) blk = (blk & ~63) | (blk & 7) << 3 | (blk >> 3 & 7);
    }
#pragma unroll
    for (int u = 0; u < DP; ++u) {
        if (blk >= ji && blk < ji + J[u])
            *found = Chunk{tid * DP + u, first[u], first[u + 1] - first[u], blk - ji, J[u], mi};
        ji += J[u];
        mi += M[u];
    }
    __syncthreads();
    return *found;
}

// Low-bit histogram of one chunk of a bucket that makes several.
__global__ void __launch_bounds__(1024) k_rb_hist2(const int64_t *__restrict__ prange, int64_t n,
                                                   const int *__restrict__ keys,
                                                   int *__restrict__ hist, int64_t hist_ints,
                                                   int tiles, int nb, int lbits) {
    __shared__ int s_hist[kLocalBuckets], scr[32];
    __shared__ Chunk found;
    int64_t p0, np;
    sys_range(prange, n, p0, np);
    hist += (int64_t)blockIdx.y * hist_ints;
    const int *first_of = hist + (int64_t)nb * tiles;
    const int nl = 1 << lbits, tid = threadIdx.x;
    int large = 0;                      // any bucket of several chunks?
    for (int d = tid; d < nb; d += 1024)
        large |= (d + 1 < nb ? first_of[d + 1] : (int)np) - first_of[d] > kLocalTile;
    if (!__syncthreads_or(large)) return;
    const Chunk c = find_chunk(blockIdx.x, nb, np, 0, first_of, scr, &found);
    if (c.b < 0 || c.J == 1) return;    // the same for every thread
    for (int d = tid; d < nl; d += 1024) s_hist[d] = 0;
    __syncthreads();
    const int e1 = min(c.cnt - c.j * kLocalTile, kLocalTile);
    const int *k = keys + p0 + c.start + c.j * kLocalTile;
    for (int e = tid; e < e1; e += 1024) atomicAdd(&s_hist[k[e] & (nl - 1)], 1);
    __syncthreads();
    int *h = hist + (int64_t)nb * (tiles + 1) + (int64_t)(c.mbase + c.j) * nl;
    for (int d = tid; d < nl; d += 1024) h[d] = s_hist[d];
}

// Low-bit histograms of a bucket of more than kChunkRows chunks into inclusive
// sums over its chunks, so that a chunk reads two rows of them where it would
// read J (one bucket of 2^22 particles on 64^3 cells: binning 276 -> 164 us, of
// 2^25 8501 -> 1176).  Blocks take the large buckets in turn, 64 digits
// each: the 16 waves sum contiguous shares of the rows, then write them from
// the sum of the shares before.
constexpr int kSumGroups = 32;          // blocks per 64 digits
__global__ void __launch_bounds__(1024) k_rb_sums2(const int64_t *__restrict__ prange, int64_t n,
                                                   int *__restrict__ hist, int64_t hist_ints,
                                                   int tiles, int nb, int lbits) {
    constexpr int DP = kRadixBuckets / 1024, U = 16;
    __shared__ int scr[16], share[16][64], found, large_mbase[kRadixBuckets], large_J[kRadixBuckets];
    int64_t p0, np;
    sys_range(prange, n, p0, np);
    hist += (int64_t)blockIdx.y * hist_ints;
    const int *first_of = hist + (int64_t)nb * tiles;
    const int nl = 1 << lbits, tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    // rows before each bucket of several chunks (as find_chunk counts them)
    int J[DP], ms = 0, large = 0;
#pragma unroll
    for (int u = 0; u < DP; ++u) {
        const int d = tid * DP + u;
        const int cnt = d < nb ? (d + 1 < nb ? first_of[d + 1] : (int)np) - first_of[d] : 0;
        const int c = (cnt + kLocalTile - 1) / kLocalTile;
        J[u] = c > 1 ? c : 0;
        ms += J[u];
        large |= c > kChunkRows;
    }
    if (tid == 0) found = 0;
    if (!__syncthreads_or(large)) return;
    int mi = ms;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int m = __shfl_up(mi, off, 64);
        if (lane >= off) mi += m;
    }
    if (lane == 63) scr[wid] = mi;
    __syncthreads();
    mi -= ms;
    for (int w = 0; w < wid; ++w) mi += scr[w];
#pragma unroll
    for (int u = 0; u < DP; ++u) {
        if (J[u] > kChunkRows) {
            const int at = atomicAdd(&found, 1);   // in any order
            large_mbase[at] = mi;
            large_J[at] = J[u];
        }
        mi += J[u];
    }
    __syncthreads();
    const int digit = (int)(blockIdx.x / kSumGroups) * 64 + lane;
    const bool act = digit < nl;
    for (int b = 0; b < found; ++b) {
        const int rows = large_J[b], per = (rows + 15) / 16;
        if (large_mbase[b] % kSumGroups != (int)(blockIdx.x % kSumGroups)) continue;
        int *h = hist + (int64_t)nb * (tiles + 1) + (int64_t)large_mbase[b] * nl + digit;
        const int r0 = min(wid * per, rows), r1 = min(r0 + per, rows);
        int sum = 0, v[U];
        for (int k0 = r0; k0 < r1; k0 += U) {
#pragma unroll
            for (int k = 0; k < U; ++k) v[k] = act && k0 + k < r1 ? h[(int64_t)(k0 + k) * nl] : 0;
#pragma unroll
            for (int k = 0; k < U; ++k) sum += v[k];
        }
        __syncthreads();                // the previous bucket's shares have been read
        share[wid][lane] = sum;
        __syncthreads();
        int run = 0;
        for (int w = 0; w < wid; ++w) run += share[w][lane];
        for (int k0 = r0; k0 < r1; k0 += U) {
            if (per > U) {              // else the rows are still in v
#pragma unroll
                for (int k = 0; k < U; ++k) v[k] = act && k0 + k < r1 ? h[(int64_t)(k0 + k) * nl] : 0;
            }
#pragma unroll
            for (int k = 0; k < U; ++k) {
                run += v[k];
                if (act && k0 + k < r1) h[(int64_t)(k0 + k) * nl] = run;
            }
        }
    }
}

// LDS of the local sort: the per-wave counts [16][nl], later the staging area
// of the chunk (its records are the largest array).
template <typename T>
constexpr size_t local_lds(int lbits) {
    return ((size_t)16 * sizeof(int) << lbits) > (size_t)kLocalTile * sizeof(particle4<T>)
               ? ((size_t)16 * sizeof(int) << lbits)
               : (size_t)kLocalTile * sizeof(particle4<T>);
}

// Stable sort of one chunk by the low bits of the cell into the final arrays.
// Wave w takes a contiguous share of the chunk and ranks it as k_rb_scatter
// does; the chunk is then put in order in LDS and written out in runs -- one
// run for a bucket of one chunk.  (Storing each element straight to its slot
// costs an L2 request per element and array: 27 us for 2^20 particles.)
template <typename T>
__global__ void __launch_bounds__(1024, sizeof(T) == 4 ? 8 : 4) k_rb_local(
    const int64_t *__restrict__ prange, int64_t n, int K, const int *__restrict__ keys_in,
    const int *__restrict__ vals_in, const particle4<T> *__restrict__ recs_in,
    int *__restrict__ keys_out, int *__restrict__ vals_out, particle4<T> *__restrict__ recs_out,
    int *__restrict__ pos, int *__restrict__ start, const int *__restrict__ hist,
    int64_t hist_ints, int tiles, int nb, int lbits, int summed, int near, int dense_thr, int whole,
    int4 *__restrict__ items,
    int64_t items_cap, int64_t splits_cap, int *__restrict__ small) {
    constexpr int RM = kLocalTile / 1024;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    __shared__ int scr[32], ls[kLocalBuckets], goff[kLocalBuckets];
    __shared__ Chunk found;
    const int nl = 1 << lbits, tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    int *wcnt = (int *)lds_raw;                     // [16][nl] while ranking
    int *sint = (int *)lds_raw;                     // staging: kLocalTile ints
    particle4<T> *srec = (particle4<T> *)lds_raw;   // staging: kLocalTile records
    int64_t p0, np;
    sys_range(prange, n, p0, np);
    hist += (int64_t)blockIdx.y * hist_ints;
    start += (int64_t)blockIdx.y * (K + 1);
    for (int e = tid; e < 16 * nl; e += 1024) wcnt[e] = 0;
    const Chunk c = find_chunk(blockIdx.x, nb, np, near, hist + (int64_t)nb * tiles, scr, &found);
    if (c.b < 0) return;                // the same for every thread
    const int na = min(c.cnt - c.j * kLocalTile, kLocalTile);
    const int rounds = (na + 1023) >> 10;
    const int64_t in0 = p0 + c.start + (int64_t)c.j * kLocalTile + wid * 64 * rounds;
    const int left = na - wid * 64 * rounds;        // elements from this wave's first on
    int key[RM], val[RM];
    particle4<T> rec[RM];
#pragma unroll
    for (int r = 0; r < RM; ++r) {
        const bool act = r < rounds && r * 64 + lane < left;
        const int64_t i = act ? in0 + r * 64 + lane : p0;
        key[r] = act ? keys_in[i] : -1;
        val[r] = act ? vals_in[i] : 0;
        rec[r] = act ? recs_in[i] : particle4<T>{T(0), T(0), T(0), T(0)};
    }
    // rank among the wave's earlier elements of the same digit (as k_rb_scatter)
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    int rank[RM];
#pragma unroll
    for (int r = 0; r < RM; ++r) {
        rank[r] = 0;
        if (r < rounds && r * 64 < left) {          // the same for the whole wave
            const bool act = key[r] >= 0;
            const int d = key[r] & (nl - 1);
            const uint64_t peers = digit_peers(act, d, lbits);
            const int before = __popcll(peers & lt);
            const int base = act ? wcnt[wid * nl + d] : 0;
            __builtin_amdgcn_wave_barrier();
            rank[r] = base + before;
            if (act && before == 0) wcnt[wid * nl + d] = base + __popcll(peers);
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
    // thread d (< nl <= 1024): prefix of its digit over the waves, the chunk's
    // count and, for a bucket of several chunks, the others' counts
    int tot = 0, all = 0, before = 0;
    if (tid < nl) {
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const int v = wcnt[w * nl + tid];
            wcnt[w * nl + tid] = tot;
            tot += v;
        }
        all = tot;
        if (c.J > 1) {
            const int *h = hist + (int64_t)nb * (tiles + 1) + (int64_t)c.mbase * nl + tid;
            if (c.J > summed) {         // rows hold inclusive sums
                before = c.j > 0 ? h[(int64_t)(c.j - 1) * nl] : 0;
                all = h[(int64_t)(c.J - 1) * nl];
            } else {
                all = 0;
#pragma unroll 8
                for (int j = 0; j < c.J; ++j) {
                    const int v = h[(int64_t)j * nl];
                    before += j < c.j ? v : 0;
                    all += v;
                }
            }
        }
    }
    // exclusive scans over the digits: the chunk's counts and the bucket's
    int inc = tot, ia = all;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int u = __shfl_up(inc, off, 64), a = __shfl_up(ia, off, 64);
        if (lane >= off) {
            inc += u;
            ia += a;
        }
    }
    if (lane == 63) {                   // find_chunk's last barrier is behind
        scr[wid] = inc;
        scr[16 + wid] = ia;
    }
    __syncthreads();
    if (tid < nl) {
        int l = inc - tot, first = c.start + ia - all;
        for (int w = 0; w < wid; ++w) {
            l += scr[w];
            first += scr[16 + w];
        }
        const int cell = (c.b << lbits) | tid;
        if (c.j == 0 && cell < K) {
            start[cell] = first;
            if (items != nullptr && all > dense_thr)
                list_dense(cell, all, whole, items + (int64_t)blockIdx.y * items_cap, items_cap,
                           splits_cap, small + (int64_t)blockIdx.y * 8);
        }
        ls[tid] = l;
        goff[tid] = first + before - l;
    }
    if (blockIdx.x == 0 && tid == 0) start[K] = (int)np;
    __syncthreads();
    int lidx[RM];
#pragma unroll
    for (int r = 0; r < RM; ++r) {
        const int d = key[r] & (nl - 1);
        lidx[r] = key[r] >= 0 ? ls[d] + wcnt[wid * nl + d] + rank[r] : 0;
    }
    __syncthreads();                    // the counts' region becomes the staging area
#pragma unroll
    for (int r = 0; r < RM; ++r)
        if (key[r] >= 0) sint[lidx[r]] = key[r];
    __syncthreads();
    int dst[RM];
#pragma unroll
    for (int r = 0; r < RM; ++r) {
        const int jj = r * 1024 + tid;
        dst[r] = 0;
        if (jj < na) {
            const int k = sint[jj];
            dst[r] = goff[k & (nl - 1)] + jj;
            keys_out[p0 + dst[r]] = k;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RM; ++r)
        if (key[r] >= 0) sint[lidx[r]] = val[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RM; ++r) {
        const int jj = r * 1024 + tid;
        if (jj < na) {
            const int v = sint[jj];
            vals_out[p0 + dst[r]] = v;
            if (pos != nullptr) pos[v] = (int)(p0 + dst[r]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RM; ++r)
        if (key[r] >= 0) srec[lidx[r]] = rec[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RM; ++r) {
        const int jj = r * 1024 + tid;
        if (jj < na) recs_out[p0 + dst[r]] = srec[jj];
    }
}

// Few particles and cells: two launches in place of the sort's five or six.
// k_bin_keys writes every particle's cell; in k_bin_small every block counts
// the cells of ALL particles in LDS, those before its tile of kSmallTile
// particles apart, scans the counts and places its own tile, whose four waves
// rank one after the other.  A call this small is bound by launches and
// latency, and reading 128 KB of cells from L2 once per block costs less than
// the histogram, scan and second-pass launches it replaces.  (Cells recomputed
// from the positions by every block: one launch, but 25 us at 32768 particles.)
constexpr int kSmallTile = 256;
template <typename T>
__global__ void __launch_bounds__(256) k_bin_keys(
    const int64_t *__restrict__ prange, int64_t n, const T *__restrict__ x,
    const T *__restrict__ y, const T *__restrict__ z, T inv_h, int nc, int3 lim, int periodic,
    int *__restrict__ keys, int *__restrict__ flag, int *__restrict__ small) {
    int64_t p0, np;
    sys_range(prange, n, p0, np);
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j == 0) reset_counts(small + (int64_t)blockIdx.y * 8);
    if (j >= np) return;
    int ix, iy, iz, out = 0;
    T u;
    cell_coord(x[p0 + j], inv_h, nc, nc, lim.x, periodic, ix, u, out);
    cell_coord(y[p0 + j], inv_h, nc, nc, lim.y, periodic, iy, u, out);
    cell_coord(z[p0 + j], inv_h, nc, lim.z, lim.z, periodic, iz, u, out);
    if (out) *flag = 1;
    keys[p0 + j] = (iz * nc + iy) * nc + ix;
}

template <typename T>
__global__ void __launch_bounds__(1024) k_bin_small(
    const int64_t *__restrict__ prange, int64_t n, const T *__restrict__ x,
    const T *__restrict__ y, const T *__restrict__ z, const T *__restrict__ q, T inv_h, int nc,
    int topz, int periodic, int K, int bits, const int *__restrict__ keys, int *__restrict__ keys_out,
    int *__restrict__ vals_out, particle4<T> *__restrict__ recs_out, int *__restrict__ pos,
    int *__restrict__ start, int dense_thr, int whole, int4 *__restrict__ items,
    int64_t items_cap, int64_t splits_cap, int *__restrict__ small) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    __shared__ int scr[16];
    int64_t p0, np;
    sys_range(prange, n, p0, np);
    const int nb = 1 << bits, tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int t0 = blockIdx.x * kSmallTile;
    if (t0 >= np && blockIdx.x > 0) return;         // block 0 writes the starts
    keys += p0;
    int *cur = (int *)lds_raw, *rest = cur + nb;    // counts before the tile, and from it on
    // this block's own records, in flight behind the counting
    const int64_t i = p0 + t0 + tid;
    const bool act = tid < kSmallTile && t0 + tid < np;
    particle4<T> rec{T(0), T(0), T(0), T(0)};
    int key = 0, slot = 0;
    if (act) key = cell_record(x, y, z, q, i, inv_h, nc, topz, periodic, rec);
    for (int d = tid; d < 2 * nb; d += 1024) cur[d] = 0;
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    __syncthreads();
    constexpr int U = 8;
    for (int base = tid; base < np; base += 1024 * U) {
        int kv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) kv[u] = keys[base + u * 1024 < np ? base + u * 1024 : 0];
        // Where the wave's first 64 keys agree, one lane counts for all that hold
        // the same cell (a wave's keys are all before t0 or all from it on): 64
        // additions to one address are serial, and a binning of 31270 particles
        // in one cell took 38 us, now 20.  Tried for every key: 2 us of the 42
        // of 32768 uniform particles on 16^3 cells.
        if (__all(kv[0] == __builtin_amdgcn_readfirstlane(kv[0]))) {
            for (int u = 0; u < U; ++u) {
                const int j = base + u * 1024;
                if (j < np) {
                    int *c = j < t0 ? cur : rest;
                    const int k0 = __builtin_amdgcn_readfirstlane(kv[u]);
                    const uint64_t same = __ballot(kv[u] == k0);
                    if (kv[u] != k0) atomicAdd(&c[kv[u]], 1);
                    else if ((same & lt) == 0) atomicAdd(&c[k0], __popcll(same));
                }
            }
            continue;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = base + u * 1024;
            if (j < np) atomicAdd(&(j < t0 ? cur : rest)[kv[u]], 1);
        }
    }
    __syncthreads();
    // thread tid scans the cells [tid C, tid C + C)
    constexpr int C = kSmallMaxK / 1024;
    int tot[C], sum = 0;
#pragma unroll
    for (int u = 0; u < C; ++u) {
        const int d = tid * C + u;
        tot[u] = d < nb ? cur[d] + rest[d] : 0;
        sum += tot[u];
    }
    int inc = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int u = __shfl_up(inc, off, 64);
        if (lane >= off) inc += u;
    }
    if (lane == 63) scr[wid] = inc;
    __syncthreads();
    int first = inc - sum;
    for (int w = 0; w < wid; ++w) first += scr[w];
    start += (int64_t)blockIdx.y * (K + 1);
#pragma unroll
    for (int u = 0; u < C; ++u) {
        const int d = tid * C + u;
        if (d < nb) {
            cur[d] += first;
            if (blockIdx.x == 0 && d < K) {
                start[d] = first;
                if (items != nullptr && tot[u] > dense_thr)
                    list_dense(d, tot[u], whole, items + (int64_t)blockIdx.y * items_cap, items_cap,
                               splits_cap, small + (int64_t)blockIdx.y * 8);
            }
        }
        first += tot[u];
    }
    if (blockIdx.x == 0 && tid == 0) start[K] = (int)np;
    // place the tile
    const uint64_t peers = digit_peers(act, key, bits);
    const int rank = __popcll(peers & lt);
    for (int w = 0; w < kSmallTile / 64; ++w) {
        __syncthreads();
        if (wid == w && act) {
            slot = cur[key] + rank;
            __builtin_amdgcn_wave_barrier();
            if (rank == 0) cur[key] = slot + __popcll(peers);
        }
    }
    if (act) {
        const int64_t o = p0 + slot;
        keys_out[o] = key;
        vals_out[o] = (int)i;
        recs_out[o] = rec;
        if (pos != nullptr) pos[i] = (int)o;
    }
}

template <typename T, int R>
static hipError_t radix_bin(const BinArgs &a, int K, int64_t maxn, hipStream_t s) {
    const T inv_h = T(a.inv_h);
    const int nsys = a.nsys > 0 ? a.nsys : 1;
    const int tiles = (int)bin_tiles(maxn);
    const int64_t hist_ints = bin_hist_ints(maxn, K);
    const int hb = bin_high_bits(maxn, K), lb = bin_key_bits(K) - hb, nb = 1 << hb;
    const int3 lim = make_int3(a.lim[0] > 0 ? a.lim[0] : a.ncell, a.lim[1] > 0 ? a.lim[1] : a.ncell,
                               a.lim[2] > 0 ? a.lim[2] : a.ncell);
    particle4<T> *recs = (particle4<T> *)a.recs;
    hipLaunchKernelGGL((k_rb_hist<T, R>), dim3(tiles, nsys), dim3(1024), 0, s, a.prange, a.n,
                       (const T *)a.x, (const T *)a.y, (const T *)a.z, inv_h, a.ncell, lim,
                       a.periodic, a.count, hist_ints, tiles, lb, hb, a.flag, a.small);
    const int64_t L = (int64_t)nb * tiles;
    if (L <= kScanOneBlock) {
        hipLaunchKernelGGL(k_rb_scan1, dim3(1, nsys), dim3(1024), 0, s, L, hist_ints, tiles, a.count);
    } else {
        const int st = (int)((L + 4095) / 4096);
        hipLaunchKernelGGL(k_rb_scan_sums, dim3(st, nsys), dim3(1024), 0, s, L, hist_ints, a.count,
                           a.tile_sums);
        hipLaunchKernelGGL(k_rb_scan, dim3(st, nsys), dim3(1024), 0, s, L, hist_ints, tiles, a.count,
                           a.tile_sums);
    }
    size_t lds = scatter_lds<T, R>(hb);
    hipError_t e;
    if (lds > 65536 && (e = set_max_lds((const void *)k_rb_scatter<T, R>, lds)) != hipSuccess)
        return e;
    const bool one = lb == 0;           // the buckets are the cells
    hipLaunchKernelGGL((k_rb_scatter<T, R>), dim3(tiles, nsys), dim3(1024), lds, s, a.prange, a.n,
                       (const T *)a.x, (const T *)a.y, (const T *)a.z, (const T *)a.q, inv_h,
                       a.ncell, lim.z, a.periodic, one ? a.scell : a.cell_of, one ? a.perm : a.slot,
                       one ? (particle4<T> *)a.sorted : recs, a.count, hist_ints, tiles, lb, hb, K,
                       one ? a.pos : nullptr, one ? a.start : nullptr, a.dense_threshold, a.whole,
                       a.items, a.items_cap, dense_splits_cap_of(a.slots_cap), a.small);
    if (one) return hipGetLastError();
    // every bucket makes a chunk, and every kLocalTile particles at most one more
    const unsigned chunks = (unsigned)(nb + maxn / kLocalTile);
    // a bucket makes several chunks on average
    const int near = maxn > (int64_t)nb * kLocalTile;
    if (maxn > kLocalTile)
        hipLaunchKernelGGL(k_rb_hist2, dim3(chunks, nsys), dim3(1024), 0, s, a.prange, a.n,
                           a.cell_of, a.count, hist_ints, tiles, nb, lb);
    const bool sums = maxn > kChunkSumMinN;
    if (sums)
        hipLaunchKernelGGL(k_rb_sums2, dim3((((1u << lb) + 63) / 64) * kSumGroups, nsys), dim3(1024), 0,
                           s, a.prange, a.n, a.count, hist_ints, tiles, nb, lb);
    lds = local_lds<T>(lb);
    if ((e = set_max_lds((const void *)k_rb_local<T>, lds)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_rb_local<T>, dim3(chunks, nsys), dim3(1024), lds, s, a.prange, a.n, K,
                       a.cell_of, a.slot, recs, a.scell, a.perm, (particle4<T> *)a.sorted, a.pos,
                       a.start, a.count, hist_ints, tiles, nb, lb, sums ? kChunkRows : INT32_MAX, near,
                       a.dense_threshold, a.whole, a.items, a.items_cap, dense_splits_cap_of(a.slots_cap), a.small);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_bin(const BinArgs &a, hipStream_t s) {
    const int K = a.ncell * a.ncell * a.ncell;
    const int64_t maxn = a.prange ? a.max_np : a.n;
    const int nsys = a.nsys > 0 ? a.nsys : 1;
    if (maxn == 0) {
        hipLaunchKernelGGL(k_bin_empty, dim3((K + 1 + 255) / 256, nsys), dim3(256), 0, s, K,
                           a.start, a.small);
        return hipGetLastError();
    }
    if (bin_is_small(maxn, K, nsys)) {
        const int bits = bin_key_bits(K);
        const unsigned blocks = (unsigned)((maxn + 255) / 256);
        const int3 lim =
            make_int3(a.lim[0] > 0 ? a.lim[0] : a.ncell, a.lim[1] > 0 ? a.lim[1] : a.ncell,
                      a.lim[2] > 0 ? a.lim[2] : a.ncell);
        static_assert(kSmallTile == 256, "one grid for both kernels");
        hipLaunchKernelGGL(k_bin_keys<T>, dim3(blocks, nsys), dim3(256), 0, s, a.prange, a.n,
                           (const T *)a.x, (const T *)a.y, (const T *)a.z, T(a.inv_h), a.ncell, lim,
                           a.periodic, a.cell_of, a.flag, a.small);
        hipLaunchKernelGGL(k_bin_small<T>, dim3(blocks, nsys), dim3(1024),
                           (size_t)2 * sizeof(int) << bits, s, a.prange, a.n, (const T *)a.x,
                           (const T *)a.y, (const T *)a.z, (const T *)a.q, T(a.inv_h), a.ncell,
                           lim.z, a.periodic, K, bits, a.cell_of, a.scell, a.perm,
                           (particle4<T> *)a.sorted, a.pos, a.start, a.dense_threshold, a.whole,
                           a.items, a.items_cap, dense_splits_cap_of(a.slots_cap), a.small);
        return hipGetLastError();
    }
    switch (bin_tile_items(maxn)) {
    case 4: return radix_bin<T, 4>(a, K, maxn, s);
    case 2: return radix_bin<T, 2>(a, K, maxn, s);
    default: return radix_bin<T, 1>(a, K, maxn, s);
    }
}

template hipError_t launch_bin<float>(const BinArgs &, hipStream_t);
template hipError_t launch_bin<double>(const BinArgs &, hipStream_t);

}  // namespace pmmm

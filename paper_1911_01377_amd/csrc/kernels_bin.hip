// Binning of the charges into x-y columns, sorted by z inside each column,
// and cut into clusters of up to 8 consecutive charges (spatially compact:
// one column cross-section by about the same extent in z).  Used by the near
// part (cluster-pair tiles) and by the spreading step (z-ranges per column).
//
// Positions are stored as uint32 fractions of the cell edge (u = x/L * 2^32),
// so a periodic wrap is an integer overflow and the int32 difference of two
// encodings is the exact minimum-image separation.
//
// Two sequences produce the same sorted charges, permutation and z-plane
// index; the clusters differ only in their numbering.
//
// Two launches (bin_local -> colbuild), when the column counts fit in LDS and
// the blocks' column prefixes are few enough for every column to read:
//   bin_local: block b of 256 charges ranks its charges within their columns
//     in LDS and writes them grouped by column into its own segment
//     [256 b, 256 b + 256) of the records, with its exclusive column prefix
//     P[b][0 .. ncol] (no global atomics, no counters);
//   colbuild: block c reads P[b][c] and P[b][c + 1] of every block b: its
//     first sorted position sum_b P[b][c], its count, and where its charges
//     lie in each segment; it gathers them, sorts them and writes the column.
//   Column c's clusters are numbered from floor(lo_c / 8) + c (lo_c its first
//   sorted position), so no prefix over the cluster counts of all columns is
//   needed; numbers left between two columns are clusters of no charge.
//
// Otherwise four: encode -> scan (column and cluster offsets) -> scatter
// (atomic slots) -> colsort, with consecutive cluster numbers.  When the
// column counts fit in LDS and are few enough to be read by every scatter
// block, each scatter block takes the offsets itself (block 0 also publishes
// them) and the scan launch is skipped; colsort clears the counters either
// way, ready for the next evaluation.
//
// Either way each column is sorted by (z, input index): a deterministic
// order.  Cluster numbers up to the pair kernel's block count that hold no
// charge have a count of 0.
#include <algorithm>

#include "useries_internal.h"
#include "device_common.h"

namespace useries {

// Column histograms are first taken in LDS per block (many charges share a
// column), then added to the global counters once per (block, column).
constexpr int kHistCols = 4096;

__device__ __forceinline__ void encode_body(const BinArgs& a, int bid, const float* __restrict__ xyz,
                                            const float* __restrict__ q,
                                            uint4* __restrict__ coord,
                                            int* __restrict__ col_count,
                                            double* __restrict__ qpart) {
    __shared__ double red[2][4];
    __shared__ int hist[kHistCols];
    const int ncol = a.nc[0] * a.nc[1];
    const bool local = ncol <= kHistCols;
    if (local)
        for (int k = threadIdx.x; k < ncol; k += 256) hist[k] = 0;
    __syncthreads();
    const int i = bid * 256 + threadIdx.x;
    double qs = 0.0, q2 = 0.0;
    if (i < a.n) {
        uint32_t u[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) u[k] = to_fixed((double)xyz[3 * i + k], a.inv_box[k]);
        const float qi = q[i];
        const int c = cell_coord(u[1], a.nc[1]) * a.nc[0] + cell_coord(u[0], a.nc[0]);
        coord[i] = make_uint4(u[0], u[1], u[2], __float_as_uint(qi));
        if (local) atomicAdd(&hist[c], 1);
        else atomicAdd(&col_count[c], 1);
        qs = qi;
        q2 = (double)qi * (double)qi;
    }
    __syncthreads();
    if (local)
        for (int k = threadIdx.x; k < ncol; k += 256)
            if (hist[k] > 0) atomicAdd(&col_count[k], hist[k]);
    // charge sums: wavefront sums, then the 4 wavefront sums in order
    qs = wave_sum_d(qs);
    q2 = wave_sum_d(q2);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
        red[0][wv] = qs;
        red[1][wv] = q2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        qpart[2 * bid] = ((red[0][0] + red[0][1]) + red[0][2]) + red[0][3];
        qpart[2 * bid + 1] = ((red[1][0] + red[1][1]) + red[1][2]) + red[1][3];
    }
}

__global__ void __launch_bounds__(256) k_encode(const float* __restrict__ xyz,
                                                const float* __restrict__ q,
                                                uint4* __restrict__ coord,
                                                int* __restrict__ col_count,
                                                double* __restrict__ qpart, BinArgs a) {
    encode_body(a, blockIdx.x, xyz, q, coord, col_count, qpart);
}

__global__ void __launch_bounds__(256) k_encode_batch(const BatchTable* __restrict__ tab,
                                                      const BoxDesc* __restrict__ desc) {
    batch_for(tab, BK_ENCODE, [&](int i, int item) {
        const BoxDesc& d = desc[tab->slot[i]];
        encode_body(d.bin, item, d.xyz, d.q, d.coord, d.col_count, d.qpart);
    });
}

// One block of 1024 threads: exclusive scans of the column counts and of the
// cluster counts ceil(count / 8) (each thread owns a contiguous chunk;
// wavefront scans by DPP lane moves, then a scan of the 16 wavefront totals), zero
// the fill counters, and reduce the charge partials in a fixed order.  The
// column counts are cleared once read, ready for the next evaluation (they
// start at zero when the workspace is allocated).
__device__ __forceinline__ void scan_body(int ncol, int* __restrict__ count,
                                          int* __restrict__ start, int* __restrict__ cstart,
                                          int* __restrict__ fill,
                                          const double* __restrict__ qpart, int nqpart,
                                          double* __restrict__ qstats) {
    __shared__ int wsum[2][16];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int chunk = (ncol + 1023) / 1024;
    const int lo = min(t * chunk, ncol), hi = min(lo + chunk, ncol);
    int s = 0, sc = 0;
    for (int c = lo; c < hi; ++c) {
        const int k = count[c];
        s += k;
        sc += (k + 7) >> 3;
    }
    const int v = wave_incl_scan(s), vc = wave_incl_scan(sc);
    if (lane == 63) {
        wsum[0][wv] = v;
        wsum[1][wv] = vc;
    }
    __syncthreads();
    if (wv == 0) {
        const int own = lane < 16 ? wsum[0][lane] : 0, ownc = lane < 16 ? wsum[1][lane] : 0;
        const int x = wave_incl_scan(own), xc = wave_incl_scan(ownc);
        if (lane < 16) {
            wsum[0][lane] = x - own;
            wsum[1][lane] = xc - ownc;
        }
    }
    __syncthreads();
    int run = wsum[0][wv] + v - s, runc = wsum[1][wv] + vc - sc;   // exclusive prefixes
    for (int c = lo; c < hi; ++c) {
        const int k = count[c];
        start[c] = run;
        cstart[c] = runc;
        run += k;
        runc += (k + 7) >> 3;
        fill[c] = 0;
        count[c] = 0;
    }
    if (t == 1023) {
        start[ncol] = run;
        cstart[ncol] = runc;
    }
    if (wv == 1) {
        double qa = 0.0, qb = 0.0;
        for (int k = lane; k < nqpart; k += 64) {
            qa += qpart[2 * k];
            qb += qpart[2 * k + 1];
        }
        qa = wave_sum_d(qa);
        qb = wave_sum_d(qb);
        if (lane == 0) {
            qstats[0] = qa;
            qstats[1] = qb;
        }
    }
}

__global__ void __launch_bounds__(1024) k_scan(int ncol, int* __restrict__ count,
                                               int* __restrict__ start, int* __restrict__ cstart,
                                               int* __restrict__ fill,
                                               const double* __restrict__ qpart, int nqpart,
                                               double* __restrict__ qstats) {
    scan_body(ncol, count, start, cstart, fill, qpart, nqpart, qstats);
}

__global__ void __launch_bounds__(1024) k_scan_batch(const BatchTable* __restrict__ tab,
                                                     const BoxDesc* __restrict__ desc) {
    batch_for(tab, BK_SCAN, [&](int i, int) {
        const BoxDesc& d = desc[tab->slot[i]];
        scan_body(d.ncol, d.col_count, d.col_start, d.clus_start, d.col_fill, d.qpart, d.nq,
                  d.qstats);
    });
}

// Slots inside a column: the rank among the block's charges of that column
// (LDS atomic) plus a base reserved once per (block, column).  The order they
// produce is arbitrary; colsort makes it deterministic.  Each slot gets the
// charge's input index and its encoded record (the record into `sorted`,
// which colsort then reorders within the column).  With `fused`, the
// block first takes the exclusive prefix sums of the column counts (256
// threads, a contiguous run of at most kHistCols / 256 columns each) as its
// column starts; block 0 also writes them, the cluster starts and the charge
// sums, in place of the scan kernel.
constexpr int kPrefixRun = kHistCols / 256;

__device__ __forceinline__ void scatter_body(const BinArgs& a, int bid, bool fused,
                                             const uint4* __restrict__ coord,
                                             uint4* __restrict__ sorted,
                                             const int* __restrict__ count,
                                             int* __restrict__ start, int* __restrict__ cstart,
                                             int* __restrict__ fill, int* __restrict__ slots,
                                             const double* __restrict__ qpart, int nqpart,
                                             double* __restrict__ qstats) {
    __shared__ int hist[kHistCols];
    __shared__ int base[kHistCols];
    __shared__ int wsum[2][4];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int n = a.n, ncol = a.nc[0] * a.nc[1];
    const bool local = ncol <= kHistCols;
    if (local)
        for (int k = t; k < ncol; k += 256) hist[k] = 0;
    const int i = bid * 256 + t;
    const uint4 rec = i < n ? coord[i] : make_uint4(0, 0, 0, 0);
    const int c = cell_coord(rec.y, a.nc[1]) * a.nc[0] + cell_coord(rec.x, a.nc[0]);
    if (fused) {
        const int run_len = (ncol + 255) / 256;
        const int lo = min(t * run_len, ncol), hi = min(lo + run_len, ncol);
        int kc[kPrefixRun];
        int s = 0, sc = 0;
#pragma unroll
        for (int u = 0; u < kPrefixRun; ++u) kc[u] = lo + u < hi ? count[lo + u] : 0;
#pragma unroll
        for (int u = 0; u < kPrefixRun; ++u) {
            s += kc[u];
            sc += (kc[u] + 7) >> 3;
        }
        const int v = wave_incl_scan(s), vc = wave_incl_scan(sc);
        if (lane == 63) {
            wsum[0][wv] = v;
            wsum[1][wv] = vc;
        }
        __syncthreads();
        int run = v - s, runc = vc - sc;   // exclusive prefixes
        for (int u = 0; u < wv; ++u) {
            run += wsum[0][u];
            runc += wsum[1][u];
        }
#pragma unroll
        for (int u = 0; u < kPrefixRun; ++u) {
            if (lo + u < hi) {
                base[lo + u] = run;
                if (bid == 0) {
                    start[lo + u] = run;
                    cstart[lo + u] = runc;
                }
                run += kc[u];
                runc += (kc[u] + 7) >> 3;
            }
        }
        if (bid == 0 && t == 255) {
            start[ncol] = run;
            cstart[ncol] = runc;
        }
        if (bid == 0 && wv == 1) {
            double qa = 0.0, qb = 0.0;
            for (int k = lane; k < nqpart; k += 64) {
                qa += qpart[2 * k];
                qb += qpart[2 * k + 1];
            }
            qa = wave_sum_d(qa);
            qb = wave_sum_d(qb);
            if (lane == 0) {
                qstats[0] = qa;
                qstats[1] = qb;
            }
        }
    }
    __syncthreads();
    int r = 0;
    if (i < n) r = local ? atomicAdd(&hist[c], 1) : atomicAdd(&fill[c], 1);
    __syncthreads();
    if (local)
        for (int k = t; k < ncol; k += 256)
            if (hist[k] > 0) base[k] = (fused ? base[k] : start[k]) + atomicAdd(&fill[k], hist[k]);
    __syncthreads();
    if (i < n) {
        const int slot = (local ? base[c] : start[c]) + r;
        slots[slot] = i;
        sorted[slot] = rec;
    }
}

__global__ void __launch_bounds__(256) k_scatter(int fused, int nqpart,
                                                 const uint4* __restrict__ coord,
                                                 const int* __restrict__ count,
                                                 uint4* __restrict__ sorted,
                                                 int* __restrict__ start, int* __restrict__ cstart,
                                                 int* __restrict__ fill, int* __restrict__ slots,
                                                 const double* __restrict__ qpart,
                                                 double* __restrict__ qstats, BinArgs a) {
    scatter_body(a, blockIdx.x, fused != 0, coord, sorted, count, start, cstart, fill, slots,
                 qpart, nqpart, qstats);
}

__global__ void __launch_bounds__(256) k_scatter_batch(const BatchTable* __restrict__ tab,
                                                       const BoxDesc* __restrict__ desc) {
    batch_for(tab, BK_SCATTER, [&](int i, int item) {
        const BoxDesc& d = desc[tab->slot[i]];
        scatter_body(d.bin, item, false, d.coord, d.sorted, d.col_count, d.col_start,
                     d.clus_start, d.col_fill, d.slots, d.qpart, d.nq, d.qstats);
    });
}

// One block per column: sort the column's charges by the key (z, input
// index) -- unique, so the order is deterministic: up to 256 charges by
// counting each key's rank in LDS, up to kSortCap by a bitonic sort in LDS,
// beyond by ranking from global memory -- then write the permutation, the
// sorted positions, the column's clusters and its z-plane index.
constexpr int kSortCap = 1024;

__device__ __forceinline__ void colsort_body(int col, const int* __restrict__ start,
                                             const int* __restrict__ cstart,
                                             const int* __restrict__ slots,
                                             const uint4* __restrict__ coord,
                                             int* __restrict__ perm, uint4* __restrict__ sorted,
                                             int2* __restrict__ cl_info, int* __restrict__ cl_col,
                                             int ncx,
                                             uint2* __restrict__ cl_z, int gz,
                                             int* __restrict__ zbin, int* __restrict__ count,
                                             int* __restrict__ fill, int ncol, int npb) {
    __shared__ unsigned long long key[kSortCap];
    __shared__ uint32_t skz[kSortCap];         // z of the sorted charges
    const int t = threadIdx.x;
    const int lo = start[col], cnt = start[col + 1] - lo;
    if (t == 0) {   // the column's counters, cleared for the next evaluation
        count[col] = 0;
        fill[col] = 0;
    }
    if (col == ncol - 1)   // cluster numbers past the last cluster: no charges
        for (int k = cstart[ncol] + t; k < npb; k += 256) cl_info[k] = make_int2(start[ncol], 0);
    int* zrow = zbin + (size_t)col * (gz + 1);
    if (cnt == 0) {
        for (int b = t; b <= gz; b += 256) zrow[b] = lo;
        return;
    }
    if (cnt <= 256) {
        // one charge per thread, its rank counted against every key
        unsigned long long mine = ~0ull;
        uint4 c = make_uint4(0, 0, 0, 0);
        int i = 0;
        if (t < cnt) {   // the column's records as scatter left them (read before any write)
            i = slots[lo + t];
            c = sorted[lo + t];
            mine = ((unsigned long long)c.z << 32) | (unsigned)i;
            key[t] = mine;
        }
        __syncthreads();
        if (t < cnt) {
            // four independent counts, so that consecutive comparisons do not
            // wait on each other's sums (one wavefront per SIMD here)
            int r0 = 0, r1 = 0, r2 = 0, r3 = 0, m = 0;
#pragma unroll 4
            for (; m + 4 <= cnt; m += 4) {
                r0 += key[m] < mine;
                r1 += key[m + 1] < mine;
                r2 += key[m + 2] < mine;
                r3 += key[m + 3] < mine;
            }
            for (; m < cnt; ++m) r0 += key[m] < mine;
            const int r = (r0 + r1) + (r2 + r3);
            perm[lo + r] = i;
            sorted[lo + r] = c;
            skz[r] = c.z;
        }
    } else if (cnt <= kSortCap) {
        int m = 1;
        while (m < cnt) m <<= 1;
        for (int k = t; k < m; k += 256) {
            if (k < cnt) {
                const int i = slots[lo + k];
                key[k] = ((unsigned long long)coord[i].z << 32) | (unsigned)i;
            } else {
                key[k] = ~0ull;
            }
        }
        __syncthreads();
        for (int size = 2; size <= m; size <<= 1) {
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                for (int k = t; k < m; k += 256) {
                    const int o = k ^ stride;
                    if (o > k) {
                        const bool up = (k & size) == 0;
                        const unsigned long long x = key[k], y = key[o];
                        if ((x > y) == up) {
                            key[k] = y;
                            key[o] = x;
                        }
                    }
                }
                __syncthreads();
            }
        }
        for (int k = t; k < cnt; k += 256) {
            const int i = (int)(unsigned)(key[k] & 0xffffffffull);
            perm[lo + k] = i;
            sorted[lo + k] = coord[i];
            skz[k] = (uint32_t)(key[k] >> 32);
        }
    } else {
        // rank by counting (O(cnt^2) work spread over the block)
        for (int k = t; k < cnt; k += 256) {
            const int i = slots[lo + k];
            const unsigned long long ki = ((unsigned long long)coord[i].z << 32) | (unsigned)i;
            int rank = 0;
            for (int m = 0; m < cnt; ++m) {
                const int j = slots[lo + m];
                rank += (((unsigned long long)coord[j].z << 32) | (unsigned)j) < ki;
            }
            perm[lo + rank] = i;
            sorted[lo + rank] = coord[i];
        }
    }
    __syncthreads();
    const bool in_lds = cnt <= kSortCap;
    // z-plane index of the column: zrow[b] = first charge whose grid z index
    // is >= b (b = 0 .. gz), for the spreading and gathering windows
    for (int b = t; b <= gz; b += 256) {
        int l = 0, h = cnt;
        while (l < h) {
            const int mid = (l + h) >> 1;
            const uint32_t z = in_lds ? skz[mid] : sorted[lo + mid].z;
            if (cell_coord(z, gz) < b) l = mid + 1; else h = mid;
        }
        zrow[b] = lo + l;
    }
    // clusters: 8 consecutive charges of the column (the last may be short);
    // the column is stored as its coordinates cx | cy << 16
    const int c0 = cstart[col], nclus = (cnt + 7) >> 3;
    const int cyx = (col % ncx) | ((col / ncx) << 16);
    for (int k = t; k < nclus; k += 256) {
        const int b = lo + 8 * k;
        const int nk = min(8, cnt - 8 * k);
        cl_info[c0 + k] = make_int2(b, nk);
        cl_col[c0 + k] = cyx;
        cl_z[c0 + k] = in_lds ? make_uint2(skz[8 * k], skz[8 * k + nk - 1])
                              : make_uint2(sorted[b].z, sorted[b + nk - 1].z);
    }
}

__global__ void __launch_bounds__(256) k_colsort(const int* __restrict__ start,
                                                 const int* __restrict__ cstart,
                                                 const int* __restrict__ slots,
                                                 const uint4* __restrict__ coord,
                                                 int* __restrict__ perm,
                                                 uint4* __restrict__ sorted,
                                                 int2* __restrict__ cl_info,
                                                 int* __restrict__ cl_col, int ncx,
                                                 uint2* __restrict__ cl_z, int gz,
                                                 int* __restrict__ zbin, int* __restrict__ count,
                                                 int* __restrict__ fill, int npb) {
    colsort_body(blockIdx.x, start, cstart, slots, coord, perm, sorted, cl_info, cl_col, ncx, cl_z, gz,
                 zbin, count, fill, (int)gridDim.x, npb);
}

__global__ void __launch_bounds__(256) k_colsort_batch(const BatchTable* __restrict__ tab,
                                                       const BoxDesc* __restrict__ desc) {
    batch_for(tab, BK_COLSORT, [&](int i, int item) {
        const BoxDesc& d = desc[tab->slot[i]];
        colsort_body(item, d.col_start, d.clus_start, d.slots, d.coord, d.perm, d.sorted,
                     d.cl_info, d.cl_col, d.bin.nc[0], d.cl_z, d.grid.g[2], d.zbin, d.col_count,
                     d.col_fill, d.ncol, d.npb);
    });
}

// ------------------------------------------------------------ two-launch binning
constexpr int kLocalBlocks = 4096;   // bin_local blocks whose prefixes colbuild reads
constexpr int kLocalRun = kLocalBlocks / 256;
constexpr int kZBuckets = 512;       // z buckets of a column's sort, at most
static_assert(kZBuckets >= kMaxGrid, "a bucket per grid plane at least");

bool bin_local_ok(int n, int ncol) {
    const long long nb = ((long long)n + 255) / 256;
    return n > 0 && ncol <= kHistCols && nb <= kLocalBlocks && nb * (ncol + 1) <= (1ll << 22);
}

// Block b: the records (fixed-point position and charge bits) of charges
// 256 b .. 256 b + 255, grouped by column into coord[256 b ...] with their
// input indices in slots[...] (order within a column as the LDS atomics
// leave it), the block's exclusive column prefix in bpre[b][0 .. ncol]
// (bpre[b][ncol]: its charge count) and its charge sums in qpart.
__device__ __forceinline__ void bin_local_body(const BinArgs& a, int b, const float* __restrict__ xyz,
                                               const float* __restrict__ q,
                                               uint4* __restrict__ coord,
                                               int* __restrict__ slots, int* __restrict__ bpre,
                                               double* __restrict__ qpart) {
    __shared__ int hist[kHistCols];
    __shared__ int wsum[4];
    __shared__ double red[2][4];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int ncol = a.nc[0] * a.nc[1];
    for (int k = t; k < ncol; k += 256) hist[k] = 0;
    __syncthreads();
    const int i = b * 256 + t;
    uint4 rec = make_uint4(0, 0, 0, 0);
    int c = 0, r = 0;
    double qs = 0.0, q2 = 0.0;
    if (i < a.n) {
        uint32_t u[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) u[k] = to_fixed((double)xyz[3 * i + k], a.inv_box[k]);
        const float qi = q[i];
        c = cell_coord(u[1], a.nc[1]) * a.nc[0] + cell_coord(u[0], a.nc[0]);
        rec = make_uint4(u[0], u[1], u[2], __float_as_uint(qi));
        r = atomicAdd(&hist[c], 1);   // rank within the block's charges of column c
        qs = qi;
        q2 = (double)qi * (double)qi;
    }
    __syncthreads();
    // exclusive prefix of the block's column counts: thread t owns the run of
    // columns [t run, t run + run), run = ceil(ncol / 256) <= kPrefixRun
    const int run = (ncol + 255) / 256;
    const int lo = min(t * run, ncol), hi = min(lo + run, ncol);
    int kc[kPrefixRun];
    int s = 0;
#pragma unroll
    for (int u = 0; u < kPrefixRun; ++u) {
        kc[u] = lo + u < hi ? hist[lo + u] : 0;
        s += kc[u];
    }
    const int v = wave_incl_scan(s);
    if (lane == 63) wsum[wv] = v;
    __syncthreads();   // every count read before it is replaced by its prefix
    int pre = v - s;
    for (int u = 0; u < wv; ++u) pre += wsum[u];
    int* row = bpre + (size_t)b * (ncol + 1);
#pragma unroll
    for (int u = 0; u < kPrefixRun; ++u) {
        if (lo + u < hi) {
            hist[lo + u] = pre;
            row[lo + u] = pre;
            pre += kc[u];
        }
    }
    if (t == 255) row[ncol] = pre;   // the last run ends at ncol: pre is the block's total
    __syncthreads();
    if (i < a.n) {
        const int slot = b * 256 + hist[c] + r;
        coord[slot] = rec;
        slots[slot] = i;
    }
    // charge sums: wavefront sums, then the 4 wavefront sums in order
    qs = wave_sum_d(qs);
    q2 = wave_sum_d(q2);
    if (lane == 0) {
        red[0][wv] = qs;
        red[1][wv] = q2;
    }
    __syncthreads();
    if (t == 0) {
        qpart[2 * b] = ((red[0][0] + red[0][1]) + red[0][2]) + red[0][3];
        qpart[2 * b + 1] = ((red[1][0] + red[1][1]) + red[1][2]) + red[1][3];
    }
}

// Block c (column c): from P[b][c] and P[b][c + 1] of the nb bin_local blocks,
// the column's first sorted position lo = sum_b P[b][c], its count and the
// offset of each block's segment in the column's list; then its charges
// gathered, sorted by (z, input index) and written with the column's z-plane
// index and clusters.  Up to kSortCap charges are sorted by z buckets in LDS
// (a whole number of buckets per grid plane, about 512 in all): a charge's
// rank is its bucket's offset plus the keys of its bucket below its own, and
// the offsets at the planes are the z-plane index.  A bucket of more than an
// eighth of the column (charges at a few values of z, as in a crystal's or an
// electrode's planes) makes it count against all of the column's keys: those
// reads are the same for every thread, so several are in flight, at 5 to 9 ns per
// key and charge of a thread against 46 for the bucket's own, one after another
// (a column at one z: 256 charges 21 -> 13 us, 1,024 202 -> 49).  Of longer columns kSortCap
// charges at a time, four per thread, are ranked against the whole column, whose
// keys pass through LDS in tiles of kSortCap.  Every list position has its thread
// whichever input blocks hold it: dealing the blocks' segments to the threads
// left a column of 2,000 charges in 8 blocks to 8 of the 256 threads, 34.5 ms
// against 0.18 now (1,100 charges 18.5 against 0.11; with keys read from global
// memory for every comparison, a charge per thread, 1.1 and 0.39).
//
// Bound: latency of two dependent rounds of scattered loads.  The block's LDS
// (14 KB) lets all columns of the largest cells be resident at once.  With 68
// KB of LDS (segment tables, sort arrays), two blocks per CU, ranks counted
// against the whole column (bitonic beyond 256) and a search per charge for
// its segment it took 22.4 us on 90,180 charges and 38.8 on 210,000, now 7.0
// and 11.5 (26,268 charges 6.7 -> 5.3).
// reduce_q: this block also reduces the charge sums (qstats_reduce).
__device__ __forceinline__ void qstats_reduce(int nb, const double* __restrict__ qpart,
                                              double* __restrict__ qstats) {
    const int lane = threadIdx.x & 63;
    double qa = 0.0, qb = 0.0;
    for (int k = lane; k < nb; k += 64) {
        qa += qpart[2 * k];
        qb += qpart[2 * k + 1];
    }
    qa = wave_sum_d(qa);
    qb = wave_sum_d(qb);
    if (lane == 0) {
        qstats[0] = qa;
        qstats[1] = qb;
    }
}

// rank += how many of the m keys in LDS lie below each of the thread's own N
template <int N>
__device__ __forceinline__ void rank_among(const unsigned long long* key, int m,
                                           const unsigned long long* mine, int* rank) {
#pragma unroll 4
    for (int k = 0; k < m; ++k) {
        const unsigned long long x = key[k];
#pragma unroll
        for (int v = 0; v < N; ++v) rank[v] += x < mine[v];
    }
}

__device__ __forceinline__ void colbuild_body(int col, int nb, int ncol, int ncx, int gz, int npb,
                                              bool reduce_q,
                                              const int* __restrict__ bpre,
                                              const uint4* __restrict__ coord,
                                              const int* __restrict__ slots,
                                              int* __restrict__ perm, uint4* __restrict__ sorted,
                                              int2* __restrict__ cl_info, int* __restrict__ cl_col,
                                              uint2* __restrict__ cl_z, int* __restrict__ zbin,
                                              const double* __restrict__ qpart,
                                              double* __restrict__ qstats) {
    // record index of each list position, later the sorted charges' z
    __shared__ uint32_t lslot[kSortCap];
    __shared__ unsigned long long bkey[kSortCap];   // keys grouped by bucket
    __shared__ int boff[kZBuckets + 1];             // bucket counts, then offsets
    __shared__ int wsum[2][4];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int stride = ncol + 1;

    // segment counts h_b = P[b][c + 1] - P[b][c] over a contiguous run of b
    // per thread; their exclusive scan (segment offsets) and the sum of P[b][c]
    for (int k = t; k <= kZBuckets; k += 256) boff[k] = 0;
    const int run = (nb + 255) / 256;
    const int blo = min(t * run, nb), bhi = min(blo + run, nb);
    int h[kLocalRun], pc[kLocalRun];
    int s = 0, ps = 0;
#pragma unroll
    for (int u = 0; u < kLocalRun; ++u) {
        h[u] = pc[u] = 0;
        if (blo + u < bhi) {
            const int* rowp = bpre + (size_t)(blo + u) * stride + col;
            pc[u] = rowp[0];
            h[u] = rowp[1] - pc[u];
        }
        s += h[u];
        ps += pc[u];
    }
    const int v = wave_incl_scan(s), vp = wave_incl_scan(ps);
    if (lane == 63) {
        wsum[0][wv] = v;
        wsum[1][wv] = vp;
    }
    __syncthreads();
    int off = v - s;
    for (int u = 0; u < wv; ++u) off += wsum[0][u];
    const int cnt = ((wsum[0][0] + wsum[0][1]) + wsum[0][2]) + wsum[0][3];
    const int lo = ((wsum[1][0] + wsum[1][1]) + wsum[1][2]) + wsum[1][3];
    const int off0 = off;
    // list position off + j of segment b holds record 256 b + P[b][c] + j
    auto place = [&](int u) {
        if (blo + u < bhi) {
            const int r0 = (blo + u) * 256 + pc[u];
            for (int j = 0; j < h[u]; ++j) lslot[off + j] = r0 + j;
            off += h[u];
        }
    };
    if (cnt <= kSortCap) {
        place(0);
        if (run > 1) {   // more than 65,536 charges (skipped one by one, the rest cost 0.2 us)
            place(1);
            if (run > 2) {
#pragma unroll
                for (int u = 2; u < kLocalRun; ++u) place(u);
            }
        }
    }
    if (reduce_q && wv == 1) qstats_reduce(nb, qpart, qstats);

    // cluster numbers: this column's from floor(lo / 8) + col, the next
    // column's from floor((lo + cnt) / 8) + col + 1 (the last column's run to
    // npb); those between its clusters and the next column's hold no charge
    const int c0 = lo / 8 + col, nclus = (cnt + 7) >> 3;
    const int cend = col == ncol - 1 ? npb : (lo + cnt) / 8 + col + 1;
    for (int k = c0 + nclus + t; k < cend; k += 256) cl_info[k] = make_int2(lo + cnt, 0);
    int* zrow = zbin + (size_t)col * (gz + 1);
    if (cnt == 0) {
        for (int k = t; k <= gz; k += 256) zrow[k] = lo;
        return;
    }
    __syncthreads();
    const bool in_lds = cnt <= kSortCap;
    uint32_t* skz = lslot;
    if (in_lds) {
        const int m = kZBuckets / gz, nz = gz * m;   // buckets per plane, in all
        constexpr int kPer = kSortCap / 256;
        uint4 c[kPer];
        int i[kPer], bk[kPer], r[kPer];
#pragma unroll
        for (int v2 = 0; v2 < kPer; ++v2) {
            const int k = t + 256 * v2;
            if (k < cnt) {
                const int sl = lslot[k];
                c[v2] = coord[sl];
                i[v2] = slots[sl];
                bk[v2] = cell_coord(c[v2].z, nz);
                r[v2] = atomicAdd(&boff[bk[v2]], 1);
            }
        }
        __syncthreads();
        // counts to offsets: two buckets per thread
        static_assert(kZBuckets == 512, "two buckets per thread");
        const int b0 = boff[2 * t], b1 = boff[2 * t + 1];
        const int incl = wave_incl_scan(b0 + b1);
        const int big = __builtin_amdgcn_ballot_w64(8 * max(b0, b1) > cnt) != 0;
        if (lane == 63) {
            wsum[0][wv] = incl;
            wsum[1][wv] = big;
        }
        __syncthreads();
        // a bucket of more than an eighth of the column
        const bool deep = (wsum[1][0] | wsum[1][1] | wsum[1][2] | wsum[1][3]) != 0;
        int o = incl - b0 - b1;
        for (int u = 0; u < wv; ++u) o += wsum[0][u];
        boff[2 * t] = o;
        boff[2 * t + 1] = o + b0;
        if (t == 255) boff[kZBuckets] = cnt;
        __syncthreads();
#pragma unroll
        for (int v2 = 0; v2 < kPer; ++v2)
            if (t + 256 * v2 < cnt)
                bkey[boff[bk[v2]] + r[v2]] = ((unsigned long long)c[v2].z << 32) | (unsigned)i[v2];
        // zrow[z]: first charge whose grid z index is >= z
        for (int z = t; z <= gz; z += 256) zrow[z] = lo + boff[z * m];
        __syncthreads();
        int rank[kPer] = {};
        if (deep) {
            // few values of z: against the whole column
            unsigned long long mine[kPer];
#pragma unroll
            for (int v2 = 0; v2 < kPer; ++v2)
                mine[v2] = t + 256 * v2 < cnt ? ((unsigned long long)c[v2].z << 32) | (unsigned)i[v2] : 0;
            if (cnt <= 256)
                rank_among<1>(bkey, cnt, mine, rank);
            else if (cnt <= 512)
                rank_among<2>(bkey, cnt, mine, rank);
            else
                rank_among<kPer>(bkey, cnt, mine, rank);
        } else {
#pragma unroll
            for (int v2 = 0; v2 < kPer; ++v2) {
                if (t + 256 * v2 < cnt) {
                    const unsigned long long mine = ((unsigned long long)c[v2].z << 32) | (unsigned)i[v2];
                    rank[v2] = boff[bk[v2]];
                    const int e = boff[bk[v2] + 1];
                    for (int k = rank[v2], e0 = e; k < e0; ++k) rank[v2] += bkey[k] < mine;
                }
            }
        }
#pragma unroll
        for (int v2 = 0; v2 < kPer; ++v2) {
            if (t + 256 * v2 < cnt) {
                perm[lo + rank[v2]] = i[v2];
                sorted[lo + rank[v2]] = c[v2];
                skz[rank[v2]] = c[v2].z;
            }
        }
    } else {
        // record indices of list positions [y, y + kSortCap) to lslot
        auto list = [&](int y) {
            int o = off0 - y;
            for (int b = blo; b < bhi; ++b) {
                const int* rowp = bpre + (size_t)b * stride + col;
                const int p = rowp[0], n = rowp[1] - p;
                const int e = min(n, kSortCap - o);
                for (int j = max(0, -o); j < e; ++j) lslot[o + j] = b * 256 + p + j;
                o += n;
            }
            __syncthreads();
        };
        constexpr int kPer = kSortCap / 256;
        for (int y0 = 0; y0 < cnt; y0 += kSortCap) {
            list(y0);
            uint4 c[kPer];
            int i[kPer], rank[kPer];
            unsigned long long mine[kPer];
#pragma unroll
            for (int v2 = 0; v2 < kPer; ++v2) {
                const int k = t + 256 * v2;
                rank[v2] = 0;
                mine[v2] = 0;
                if (y0 + k < cnt) {
                    const int sl = lslot[k];
                    c[v2] = coord[sl];
                    i[v2] = slots[sl];
                    mine[v2] = ((unsigned long long)c[v2].z << 32) | (unsigned)i[v2];
                }
            }
            for (int y1 = 0; y1 < cnt; y1 += kSortCap) {
                __syncthreads();   // lslot and bkey are read
                list(y1);
                const int m = min(kSortCap, cnt - y1);
                for (int k = t; k < m; k += 256) {
                    const int sl = lslot[k];
                    bkey[k] = ((unsigned long long)coord[sl].z << 32) | (unsigned)slots[sl];
                }
                __syncthreads();
                rank_among<kPer>(bkey, m, mine, rank);
            }
#pragma unroll
            for (int v2 = 0; v2 < kPer; ++v2) {
                if (y0 + t + 256 * v2 < cnt) {
                    perm[lo + rank[v2]] = i[v2];
                    sorted[lo + rank[v2]] = c[v2];
                }
            }
        }
    }
    __syncthreads();
    // z-plane index of a column sorted in global memory: a search per plane
    if (!in_lds) {
        for (int z = t; z <= gz; z += 256) {
            int l = 0, hh = cnt;
            while (l < hh) {
                const int mid = (l + hh) >> 1;
                if (cell_coord(sorted[lo + mid].z, gz) < z) l = mid + 1; else hh = mid;
            }
            zrow[z] = lo + l;
        }
    }
    const int cyx = (col % ncx) | ((col / ncx) << 16);
    for (int k = t; k < nclus; k += 256) {
        const int b0 = lo + 8 * k;
        const int nk = min(8, cnt - 8 * k);
        cl_info[c0 + k] = make_int2(b0, nk);
        cl_col[c0 + k] = cyx;
        cl_z[c0 + k] = in_lds ? make_uint2(skz[8 * k], skz[8 * k + nk - 1])
                              : make_uint2(sorted[b0].z, sorted[b0 + nk - 1].z);
    }
}

__global__ void __launch_bounds__(256) k_bin_local(const float* __restrict__ xyz,
                                                   const float* __restrict__ q,
                                                   uint4* __restrict__ coord,
                                                   int* __restrict__ slots,
                                                   int* __restrict__ bpre,
                                                   double* __restrict__ qpart, BinArgs a) {
    bin_local_body(a, blockIdx.x, xyz, q, coord, slots, bpre, qpart);
}

__global__ void __launch_bounds__(256) k_colbuild(int nb, int ncol, int ncx, int gz, int npb,
                                                  const int* __restrict__ bpre,
                                                  const uint4* __restrict__ coord,
                                                  const int* __restrict__ slots,
                                                  int* __restrict__ perm,
                                                  uint4* __restrict__ sorted,
                                                  int2* __restrict__ cl_info,
                                                  int* __restrict__ cl_col,
                                                  uint2* __restrict__ cl_z,
                                                  int* __restrict__ zbin,
                                                  const double* __restrict__ qpart,
                                                  double* __restrict__ qstats) {
    // block ncol (one past the columns) reduces the charge sums, beside the columns
    if (blockIdx.x == ncol) {
        if (threadIdx.x < 64) qstats_reduce(nb, qpart, qstats);
        return;
    }
    colbuild_body(blockIdx.x, nb, ncol, ncx, gz, npb, false, bpre, coord, slots, perm, sorted,
                  cl_info, cl_col, cl_z, zbin, qpart, qstats);
}

__global__ void __launch_bounds__(256) k_bin_local_batch(const BatchTable* __restrict__ tab,
                                                         const BoxDesc* __restrict__ desc) {
    batch_for(tab, BK_BINLOCAL, [&](int i, int item) {
        const BoxDesc& d = desc[tab->slot[i]];
        bin_local_body(d.bin, item, d.xyz, d.q, d.coord, d.slots, d.bpre, d.qpart);
    });
}

__global__ void __launch_bounds__(256) k_colbuild_batch(const BatchTable* __restrict__ tab,
                                                        const BoxDesc* __restrict__ desc) {
    batch_for(tab, BK_COLBUILD, [&](int i, int item) {
        const BoxDesc& d = desc[tab->slot[i]];
        colbuild_body(item, d.nq, d.ncol, d.bin.nc[0], d.grid.g[2], d.npb, item == 0, d.bpre,
                      d.coord, d.slots, d.perm, d.sorted, d.cl_info, d.cl_col, d.cl_z, d.zbin,
                      d.qpart, d.qstats);
    });
}

hipError_t launch_bin_local_batch(const BatchTable* tab, const BoxDesc* desc, int grid,
                                  hipStream_t st) {
    hipLaunchKernelGGL(k_bin_local_batch, dim3(grid), dim3(256), 0, st, tab, desc);
    return hipGetLastError();
}

hipError_t launch_colbuild_batch(const BatchTable* tab, const BoxDesc* desc, int grid,
                                 hipStream_t st) {
    hipLaunchKernelGGL(k_colbuild_batch, dim3(grid), dim3(256), 0, st, tab, desc);
    return hipGetLastError();
}

hipError_t launch_bin_local(const BinArgs& a, const float* xyz, const float* q, uint4* coord,
                            int* slots, int* bpre, double* qpart, hipStream_t st) {
    const int nb = (a.n + 255) / 256;
    if (nb > 0)
        hipLaunchKernelGGL(k_bin_local, dim3(nb), dim3(256), 0, st, xyz, q, coord, slots, bpre,
                           qpart, a);
    return hipGetLastError();
}

hipError_t launch_colbuild(int n, int ncol, int ncx, int gz, int npb, const int* bpre,
                           const uint4* coord, const int* slots, int* perm, uint4* sorted,
                           int2* cl_info, int* cl_col, uint2* cl_z, int* zbin,
                           const double* qpart, double* qstats, hipStream_t st) {
    const int nb = (n + 255) / 256;
    hipLaunchKernelGGL(k_colbuild, dim3(ncol + 1), dim3(256), 0, st, nb, ncol, ncx, gz, npb, bpre,
                       coord, slots, perm, sorted, cl_info, cl_col, cl_z, zbin, qpart, qstats);
    return hipGetLastError();
}

hipError_t launch_encode(const BinArgs& a, const float* xyz, const float* q, uint4* coord,
                         int* col_count, double* qpart, int nqpart, hipStream_t st) {
    if (a.n > 0)
        hipLaunchKernelGGL(k_encode, dim3(nqpart), dim3(256), 0, st, xyz, q, coord, col_count,
                           qpart, a);
    return hipGetLastError();
}

hipError_t launch_scan(int ncol, int* col_count, int* col_start, int* clus_start,
                       int* col_fill, const double* qpart, int nqpart, double* qstats,
                       hipStream_t st) {
    hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, st, ncol, col_count, col_start, clus_start,
                       col_fill, qpart, nqpart, qstats);
    return hipGetLastError();
}

bool scan_fused(int n, int ncol) {
    const long long nb = (n + 255) / 256;
    return ncol <= kHistCols && nb * ncol <= (1ll << 22);
}

hipError_t launch_scatter(const BinArgs& a, const uint4* coord, uint4* sorted, const int* col_count,
                          int* col_start, int* clus_start, int* col_fill, int* slots,
                          const double* qpart, int nqpart, double* qstats, hipStream_t st) {
    const int n = a.n, ncol = a.nc[0] * a.nc[1];
    const int fused = scan_fused(n, ncol) ? 1 : 0;
    // with no charges the fused prefix still has to run once (all columns empty)
    const int nb = std::max(1, (n + 255) / 256);
    if (n > 0 || fused)
        hipLaunchKernelGGL(k_scatter, dim3(nb), dim3(256), 0, st, fused, nqpart, coord, col_count,
                           sorted, col_start, clus_start, col_fill, slots, qpart, qstats, a);
    return hipGetLastError();
}

hipError_t launch_colsort(int ncol, int ncx, const int* col_start, const int* clus_start,
                          const int* slots, const uint4* coord, int* perm, uint4* sorted,
                          int2* cl_info, int* cl_col, uint2* cl_z, int gz, int* zbin,
                          int* col_count, int* col_fill, int npb, hipStream_t st) {
    hipLaunchKernelGGL(k_colsort, dim3(ncol), dim3(256), 0, st, col_start, clus_start, slots,
                       coord, perm, sorted, cl_info, cl_col, ncx, cl_z, gz, zbin, col_count,
                       col_fill, npb);
    return hipGetLastError();
}

hipError_t launch_encode_batch(const BatchTable* tab, const BoxDesc* desc, int grid, hipStream_t st) {
    hipLaunchKernelGGL(k_encode_batch, dim3(grid), dim3(256), 0, st, tab, desc);
    return hipGetLastError();
}

hipError_t launch_scan_batch(const BatchTable* tab, const BoxDesc* desc, int grid, hipStream_t st) {
    hipLaunchKernelGGL(k_scan_batch, dim3(grid), dim3(1024), 0, st, tab, desc);
    return hipGetLastError();
}

hipError_t launch_scatter_batch(const BatchTable* tab, const BoxDesc* desc, int grid,
                                hipStream_t st) {
    hipLaunchKernelGGL(k_scatter_batch, dim3(grid), dim3(256), 0, st, tab, desc);
    return hipGetLastError();
}

hipError_t launch_colsort_batch(const BatchTable* tab, const BoxDesc* desc, int grid,
                                hipStream_t st) {
    hipLaunchKernelGGL(k_colsort_batch, dim3(grid), dim3(256), 0, st, tab, desc);
    return hipGetLastError();
}

}  // namespace useries

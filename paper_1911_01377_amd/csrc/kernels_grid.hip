// Spreading and gathering of the far part (Sec. IV.A mesh evaluation, Sec. V
// grid convolution).  Each charge is smeared on the grid by a normalised,
// separable Gaussian of width sigma_s (per axis), sampled on a cube stencil
// of 2P points per axis around it:
//   rho_g = sum_i q_i prod_a W_a(g_a h_a - x_ia),
//   W_a(d) = h_a / (sqrt(2 pi) sigma_s,a) exp(-d^2 / (2 sigma_s,a^2)),
// and potentials and forces are read back with the same weights:
//   phi_i = sum_g phi_g prod_a W_a,   F_i = -q_i grad_i phi_i.
// The mean of rho (its k = 0 mode, the net charge) is removed on the grid.
//
// spread: one block per 8x8x8 brick of the grid.  Candidates come from the
//   x-y columns that can hold a charge touching the brick, each contributing
//   the charges of the brick's z-planes (per-column z-plane index); the block
//   keeps those that touch it, stages their weights in LDS and accumulates the
//   brick in registers by x halves, four wavefronts per half, a lane owning a
//   4-point x row of it; each wavefront takes a share of the charges that
//   touch its half, and the partial sums are added in a fixed order.  No
//   atomics.
// gather: one block per brick with the potential on the brick and its halo in
//   LDS; each charge is evaluated by the block whose brick holds its stencil
//   anchor, 8 or 16 lanes per charge.  One more block forms the energy total.
#include <algorithm>

#include "useries_internal.h"
#include "device_common.h"
#include "energy_total.h"

namespace useries {

namespace {

constexpr int kBrick = 8;
constexpr int kSpreadWaves = 8;                  // wavefronts per brick
constexpr int kSpreadChunk = 64 * kSpreadWaves;  // candidates loaded per pass, one per thread

// columns along axis ax that can hold charges touching grid points
// [X0, X0 + bn): charges whose stencil start lies in [X0 - P, X0 + bn + P - 1)
__device__ __forceinline__ void cell_window(const GridArgs& a, int ax, int X0, int bn, int P,
                                            int* lo, int* cnt) {
    const int g = a.g[ax], nc = a.nc[ax];
    const int l = magic_div((X0 - P + g) * nc, a.mg[ax]) - nc;              // floor
    const int h = magic_div((X0 + bn + P - 1) * nc + g - 1, a.mg[ax]) - 1;  // ceil - 1
    if (h - l + 1 >= nc) {
        *lo = 0;
        *cnt = nc;
    } else {
        *lo = wrap1(l, nc);
        *cnt = h - l + 1;
    }
}

// origin of brick bid (x fastest) of edge B, and its extent on the grid
struct Brick {
    int o[3], n[3];
};
__device__ __forceinline__ Brick brick_at(const GridArgs& a, int bid, int B,
                                          const uint32_t mb[2]) {
    const int nbx = (a.g[0] + B - 1) / B, nby = (a.g[1] + B - 1) / B;
    const int r = nbx > 1 ? magic_div(bid, mb[0]) : bid;
    const int z = nby > 1 ? magic_div(r, mb[1]) : r;
    Brick k;
    k.o[0] = (bid - r * nbx) * B;
    k.o[1] = (r - z * nby) * B;
    k.o[2] = z * B;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) k.n[ax] = min(B, a.g[ax] - k.o[ax]);
    return k;
}

// acc[x] += X_c[x] yz[c] for the four charges c in order, X_c[x] in lane
// 4 c + x of each 16-lane row of xw: the FMA reads it from there (a DPP row
// broadcast as its first operand, which the compiler emits only as a separate
// move).  The two wait states are those a DPP read needs after a vector write
// of its source.
__device__ __forceinline__ void spread_add4(float acc[4], float xw, const float yz[4]) {
#define USERIES_FMAC(X, C, N)                                                                  \
    "v_fmac_f32_dpp %" #X ", %4, %" #C " row_newbcast:" #N " row_mask:0xf bank_mask:0xf\n"
    asm("s_nop 1\n" USERIES_FMAC(0, 5, 0) USERIES_FMAC(1, 5, 1) USERIES_FMAC(2, 5, 2)
            USERIES_FMAC(3, 5, 3) USERIES_FMAC(0, 6, 4) USERIES_FMAC(1, 6, 5)
                USERIES_FMAC(2, 6, 6) USERIES_FMAC(3, 6, 7) USERIES_FMAC(0, 7, 8)
                    USERIES_FMAC(1, 7, 9) USERIES_FMAC(2, 7, 10) USERIES_FMAC(3, 7, 11)
                        USERIES_FMAC(0, 8, 12) USERIES_FMAC(1, 8, 13) USERIES_FMAC(2, 8, 14)
                            USERIES_FMAC(3, 8, 15)
        : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3])
        : "v"(xw), "v"(yz[0]), "v"(yz[1]), "v"(yz[2]), "v"(yz[3]));
#undef USERIES_FMAC
}

}  // namespace

// One block per 8x8x8 brick.  The window of a brick: in x and y the columns
// that can hold a charge whose stencil touches it, in z the grid planes
// [Z0 - P, Z0 + B2 + P - 2] (periodic), read from each column's z-plane index
// as at most two contiguous charge ranges.  The block loads the candidates in
// chunks of one per thread, keeps those whose stencil touches the brick
// (compacted in thread order within three classes: those meeting only the x
// half 0 (x 0..3), both halves, only half 1 -- so the order is deterministic
// and each half's charges are one contiguous run), evaluates their 3 x 8
// weights into LDS (a wavefront takes one axis of 64 charges, a lane the 8
// brick positions of one: no branches, two 16-byte stores), and wavefront
// 4 h + u accumulates every fourth of half h's charges from the u-th into its
// partial half brick (a dense 4 x 8 x 8 product per charge; a charge whose
// stencil ends at brick position d meets both halves only for
// 4 <= d <= 2P + 2, so at P = 3 about 60% of the charges are accumulated by
// one half only); the four partials of each point are summed in a fixed order
// at the end.
//
// Bound: VALU issue (77% of its slots on 90,180 charges, plain: 9,480
// instructions per brick, 38% of them the accumulation, 28% the weights).  It
// was 55.8 us there with 3 LDS reads per charge in the accumulation, branches
// around every stencil point in the weights and 13 integer divisions per
// wavefront, and is 41.1; 26,268 charges 19.1 -> 14.9, BF16X3 10.3 -> 8.4.
__device__ __forceinline__ void spread_body(const GridArgs& a, int bid,
                                            const uint4* __restrict__ sorted,
                                            const int* __restrict__ zbin,
                                            const double* __restrict__ qstats,
                                            float* __restrict__ rho) {
    // staged charges: their records, then their weights [x 8 | y 8 | z 8], each
    // axis's inputs in its own 8 words; rows of 96 B (16-byte stores)
    __shared__ __align__(16) float sw[kSpreadChunk][3 * kBrick];
    static_assert(kSpreadWaves == 8 && kBrick == 8, "four wavefronts per half brick; 8-wide rows");
    // the wavefronts' partial half bricks, summed after the last chunk (reuses
    // sw; rows of 65 so that the 8 partials a thread group reads lie in
    // different banks)
    float (*red)[4][65] = reinterpret_cast<float (*)[4][65]>(&sw[0][0]);
    static_assert(kSpreadWaves * 4 * 65 <= kSpreadChunk * 3 * kBrick, "red fits in sw");
    __shared__ int pbeg[2 * kMaxWindowCols];       // first charge of each non-empty column piece
    __shared__ int poff[2 * kMaxWindowCols + 1];   // prefix sums of the piece lengths
    __shared__ int2 wtot[kSpreadWaves];
    __shared__ int wcat[kSpreadWaves];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // wavefronts 4 h .. 4 h + 3 accumulate the x half h of the brick
    // (x 4 h .. 4 h + 3); lane (y, z) owns the four points of that row,
    // partial sums acc[x - 4 h]
    const int hx = w >> 2, ly = lane & 7, lz = lane >> 3;
    // the grid mean of the charge (removed at the end), loaded first
    const float mean = (float)(qstats[0] * a.inv_ngrid);
    const Brick K = brick_at(a, bid, kBrick, a.mb8);
    const int P = a.P, gz = a.g[2];
    int lo[2], cnt[2];
    cell_window(a, 0, K.o[0], K.n[0], P, &lo[0], &cnt[0]);
    cell_window(a, 1, K.o[1], K.n[1], P, &lo[1], &cnt[1]);
    const int ncw = cnt[0] * cnt[1];
    // z planes of the window: [zs, zs + zl) modulo gz
    const int zl = K.n[2] + 2 * P - 1;
    const int zs = wrap1(K.o[2] - P, gz);
    // candidate charge ranges of window column k = tid: at most two (the
    // second only where the z window wraps)
    static_assert(kMaxWindowCols <= 64 * kSpreadWaves, "one window column per thread");
    int rb0 = 0, n0 = 0, rb1 = 0, n1 = 0;
    if (tid < ncw) {
        const int ky = small_div(tid, __builtin_amdgcn_rcpf((float)cnt[0]));
        const int col = wrap1(lo[1] + ky, a.nc[1]) * a.nc[0] +
                        wrap1(lo[0] + tid - ky * cnt[0], a.nc[0]);
        const int* zr = zbin + (size_t)col * (gz + 1);
        if (zl >= gz) {
            rb0 = zr[0];
            n0 = zr[gz] - rb0;
        } else if (zs + zl <= gz) {
            rb0 = zr[zs];
            n0 = zr[zs + zl] - rb0;
        } else {
            rb0 = zr[zs];
            n0 = zr[gz] - rb0;
            rb1 = zr[0];
            n1 = zr[zs + zl - gz] - rb1;
        }
    }
    // non-empty pieces stored compactly: exclusive scans over the threads of
    // (pieces, charges), then each thread writes its pieces
    int np = 0, total = 0;
    {
        const int m = (n0 > 0) + (n1 > 0), len = n0 + n1;
        const int im = wave_incl_scan(m), il = wave_incl_scan(len);
        if (lane == 63) wtot[w] = make_int2(im, il);
        __syncthreads();
        int M = im - m, O = il - len;
#pragma unroll
        for (int v = 0; v < kSpreadWaves; ++v) {
            const int2 t = wtot[v];
            M += v < w ? t.x : 0;
            O += v < w ? t.y : 0;
            np += t.x;
            total += t.y;
        }
        if (n0 > 0) {
            pbeg[M] = rb0;
            poff[M] = O;
        }
        if (n1 > 0) {
            pbeg[M + (n0 > 0)] = rb1;
            poff[M + (n0 > 0)] = O + n0;
        }
        if (tid == 0) poff[np] = total;
        __syncthreads();
    }
    np = __builtin_amdgcn_readfirstlane(np);
    total = __builtin_amdgcn_readfirstlane(total);

    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};

    // candidate t = base + tid of the window (loads are issued one chunk
    // ahead).  The pieces of the wavefront's first and last candidate by
    // counting the offsets at or below them, then each lane's by bisection
    // between the two (a few pieces)
    auto fetch = [&](int base) {
        const int t0 = base + 64 * w, t = t0 + lane;
        uint4 c = make_uint4(0, 0, 0, 0);
        if (t0 < total) {
            int l = -1, h = 0;
            for (int r0 = 0; r0 < np; r0 += 64) {
                const int o = r0 + lane < np ? poff[r0 + lane] : 0x7fffffff;
                const int cl = __popcll(__builtin_amdgcn_ballot_w64(o <= t0));
                const int ch = __popcll(__builtin_amdgcn_ballot_w64(o <= t0 + 63));
                l += cl;
                h += ch;
            }
            if (t < total) {
                while (h - l > 1) {              // poff[l] <= t < poff[h]
                    const int mid = (l + h) >> 1;
                    if (poff[mid] <= t) l = mid; else h = mid;
                }
                c = sorted[pbeg[l] + (t - poff[l])];
            }
        }
        return c;
    };
    // brick position of a charge's last stencil point: cell + sh modulo the axis
    int sh[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) sh[ax] = wrap1(P - K.o[ax], a.g[ax]);
    uint4 next = fetch(0);
    for (int base = 0; base < total; base += kSpreadChunk) {
        const uint4 c = next;
        if (base + kSpreadChunk < total) next = fetch(base + kSpreadChunk);
        const int d0 = mod_once(cell_coord(c.x, a.g[0]) + sh[0], a.g[0]);
        const int d1 = mod_once(cell_coord(c.y, a.g[1]) + sh[1], a.g[1]);
        const int d2 = mod_once(cell_coord(c.z, a.g[2]) + sh[2], a.g[2]);
        const bool touch = base + tid < total && d0 <= K.n[0] + 2 * P - 2 &&
                           d1 <= K.n[1] + 2 * P - 2 && d2 <= K.n[2] + 2 * P - 2;
        // x halves met: 0 (x 0..3) only, both, 1 (x 4 ..) only; half 1 also
        // from its far side, where the stencil wraps around a narrow axis
        const bool h0 = d0 - 2 * P + 1 <= 3,
                   h1 = (d0 >= 4 || d0 - 2 * P + 1 + a.g[0] < kBrick) && K.n[0] > 4;
        // compaction in thread order within each x-half class, the classes
        // one after the other: half 0's charges are rows [0, n0 + n01), half
        // 1's rows [n0, nst).  The wavefronts' three counts travel in one
        // word, 10 bits each
        const uint64_t mt = __builtin_amdgcn_ballot_w64(touch);
        const uint64_t m0 = __builtin_amdgcn_ballot_w64(h0), m1 = __builtin_amdgcn_ballot_w64(h1);
        const uint64_t mA = mt & m0 & ~m1, mB = mt & m0 & m1, mC = mt & ~m0;
        static_assert(kSpreadChunk < 1024, "10 bits per count");
        if (lane == 0) wcat[w] = __popcll(mA) | __popcll(mB) << 10 | __popcll(mC) << 20;
        __syncthreads();
        int below = 0, all = 0;
#pragma unroll
        for (int v = 0; v < kSpreadWaves; ++v) {
            const int k = wcat[v];
            below += v < w ? k : 0;
            all += k;
        }
        below = __builtin_amdgcn_readfirstlane(below);
        all = __builtin_amdgcn_readfirstlane(all);
        const int nA = all & 1023, nAB = nA + ((all >> 10) & 1023), nst = nAB + (all >> 20);
        // the touching charges' coordinates: x in word 0 of the charge's row,
        // y and the charge in words 8 and 9, z in word 16
        if (touch) {
            const uint64_t mm = !h0 ? mC : h1 ? mB : mA;
            const int first = !h0 ? nAB + (below >> 20)
                                  : h1 ? nA + ((below >> 10) & 1023) : (below & 1023);
            uint32_t* row = reinterpret_cast<uint32_t*>(sw[first + lanes_below(mm)]);
            row[0] = c.x;
            *reinterpret_cast<uint2*>(row + kBrick) = make_uint2(c.y, c.w);
            row[2 * kBrick] = c.z;
        }
        __syncthreads();
        // unit u: axis u % 3 of staged charges 64 (u / 3) + lane.  Brick
        // position b is stencil point k = b + k0 modulo the axis, within
        // the stencil for k < 2P; one subtraction covers the modulus on axes
        // of at least brick + 2P - 1 points, where at most one of b + k0 and
        // b + k0 - g can be a stencil point for the whole brick
        const int nu = 3 * ((nst + 63) >> 6);
        for (int u = w; u < nu; u += kSpreadWaves) {
            const int grp = magic_div(u, 0x55555556u), ax = u - 3 * grp;
            const int s = 64 * grp + lane;
            if (s < nst) {
                float* row = sw[s] + kBrick * ax;
                const int g = ax == 0 ? a.g[0] : ax == 1 ? a.g[1] : a.g[2];
                const int o = ax == 0 ? K.o[0] : ax == 1 ? K.o[1] : K.o[2];
                const float hs = ax == 0 ? a.hs[0] : ax == 1 ? a.hs[1] : a.hs[2];
                const float cw = ax == 0 ? a.cw[0] : ax == 1 ? a.cw[1] : a.cw[2];
                int gi;
                float f;
                grid_coord(__float_as_uint(row[0]), g, &gi, &f);
                const float cf = (float)(P - 1) + f;
                const float sc = ax == 1 ? cw * row[1] : cw;
                const float e2 = -hs * 1.44269504f;   // exp(-t^2 hs) = 2^(t^2 e2)
                const uint32_t k0 = wrap1(o - gi + P - 1, g);
                float wt[kBrick];
                auto eval = [&](auto&& kof) {
#pragma unroll
                    for (int b = 0; b < kBrick; ++b) {
                        const uint32_t k = kof(b);
                        const float t = (float)(int)k - cf;
                        const float v = sc * __builtin_amdgcn_exp2f(t * t * e2);
                        wt[b] = k < (uint32_t)(2 * P) ? v : 0.0f;
                    }
                };
                if (g >= kBrick + 2 * P - 1) {
                    const uint32_t k1 = k0 < (uint32_t)(2 * P) ? k0 : k0 - g;
                    eval([&](int b) { return k1 + b; });
                } else {
                    eval([&](int b) { return min(k0 + b, k0 + b - g); });
                }
                *reinterpret_cast<float4*>(row) = make_float4(wt[0], wt[1], wt[2], wt[3]);
                *reinterpret_cast<float4*>(row + 4) = make_float4(wt[4], wt[5], wt[6], wt[7]);
            }
        }
        __syncthreads();
        // the staged charges of this wavefront's x half, every fourth one, in
        // staged order, four per pass: one 4-byte read gives the four charges'
        // x weights of the half (lane 4 c + x of each 16-lane row: weight x of
        // charge c), which the FMAs take from their lane by a DPP row
        // broadcast; per charge then the lane's y and z weights, one y z
        // product and four FMAs
        const int hend = hx == 0 ? nAB : nst;
        int sidx = (hx == 0 ? 0 : nA) + (w & 3);
        const int xc = (lane >> 2) & 3, xo = 4 * hx + (lane & 3);
        for (; sidx + 12 < hend; sidx += 16) {
            const float* row = sw[sidx];
            const float xw = row[4 * xc * (3 * kBrick) + xo];
            float yz[4];
#pragma unroll
            for (int c = 0; c < 4; ++c)
                yz[c] = row[4 * c * (3 * kBrick) + kBrick + ly] *
                        row[4 * c * (3 * kBrick) + 2 * kBrick + lz];
            spread_add4(acc, xw, yz);
        }
        for (; sidx < hend; sidx += 4) {
            const float* row = sw[sidx];
            const float4 X = *reinterpret_cast<const float4*>(row + 4 * hx);
            const float yz = row[kBrick + ly] * row[2 * kBrick + lz];
            acc[0] = fmaf(X.x, yz, acc[0]);
            acc[1] = fmaf(X.y, yz, acc[1]);
            acc[2] = fmaf(X.z, yz, acc[2]);
            acc[3] = fmaf(X.w, yz, acc[3]);
        }
        __syncthreads();
    }

    // fixed-order sum of the four partials of each point (those of its half's
    // wavefronts, in wavefront order): all partials to LDS, then thread
    // (x, y, z) = (tid % 8, tid / 8 % 8, tid / 64) adds those of its point,
    // lane (y, z)'s partial x % 4 of wavefronts 4 (x / 4) + u
#pragma unroll
    for (int k = 0; k < 4; ++k) red[w][k][lane] = acc[k];
    __syncthreads();
    const int px = tid & 7, py = (tid >> 3) & 7, pz = tid >> 6;
    const int h = px >> 2, k = px & 3, l = py + 8 * pz;
    float v = red[4 * h][k][l];
#pragma unroll
    for (int u = 1; u < 4; ++u) v += red[4 * h + u][k][l];
    if (px < K.n[0] && py < K.n[1] && pz < K.n[2])
        rho[((size_t)(K.o[2] + pz) * a.g[1] + (K.o[1] + py)) * a.g[0] + K.o[0] + px] = v - mean;
}

__global__ void __launch_bounds__(64 * kSpreadWaves) k_spread(int nb,
                                                              const int* __restrict__ zbin,
                                                              const double* __restrict__ qstats,
                                                              const uint4* __restrict__ sorted,
                                                              float* __restrict__ rho, GridArgs a) {
    const int item = xcd_item(blockIdx.x, nb);
    if (item < nb) spread_body(a, item, sorted, zbin, qstats, rho);
}

__global__ void __launch_bounds__(64 * kSpreadWaves) k_spread_batch(
        const BatchTable* __restrict__ tab, const BoxDesc* __restrict__ desc) {
    batch_for(tab, BK_SPREAD, [&](int i, int item) {
        const BoxDesc& d = desc[tab->slot[i]];
        spread_body(d.grid, item, d.sorted, d.zbin, d.qstats, d.rho);
    });
}

// gather: one block per brick of the grid (8^3 for P <= 5, 4^3 beyond).  The
// block stages the potential on the brick and its stencil halo (edge
// brick + 2P - 1) in LDS with coalesced row loads, then takes the charges
// whose stencil anchor (grid cell) lies in the brick: per overlapping column
// the z-plane index gives one contiguous range; candidates are loaded one per
// thread and the owners compacted in thread order.  A wavefront evaluates
// eight owners at a time with 8 lanes each (stencils of up to 8 points per
// axis, compiled for that width) or four with 16: a lane owns stencil rows
// (y, z) and reads the 2P x points of each from LDS; the groups then reduce.
constexpr int kGatherMaxPieces = 256;     // columns overlapping a brick
constexpr int kGatherWaves = 8;           // wavefronts per brick (general stencil)
constexpr int kGatherThreads = 64 * kGatherWaves;
constexpr int kGatherBatch = 8;           // halo loads issued together per thread

__host__ __device__ constexpr int gather_brick(int P) { return P <= 5 ? 8 : 4; }

// stencil half widths with their own code (the two forms' defaults)
__host__ __device__ constexpr bool gather_fixed(int P) { return P == 3 || P == 5; }
// lanes per owner charge
__host__ __device__ constexpr int gather_lanes(int P) { return P == 3 ? 8 : 16; }
// Wavefronts of a block: 16 for the P = 5 stencil while the bricks are at most
// two per CU (4 passes of a wavefront become 2), beyond that 8, with four blocks
// per CU.  At 1 A spacing, 16 against 8: 216 bricks 10.6 and 11.6 us, 343 12.6
// and 13.1, 512 13.0 and 13.6, 729 17.6 and 16.0 (65^3) or 18.7 and 16.0 (72^3),
// 1,000 20.5 and 18.5, 1,331 25.0 and 23.0, 1,728 29.9 and 27.1, 2,197 35.2 and
// 30.8; with fewer charges per brick the line lies lower (11,082 on 64^3 10.3
// and 9.5) and 8 gains more beyond it (26,268 on 81^3 20.5 and 16.5).  P = 3: 8
// (16 wavefronts 7.1 against 6.6 us at 26,268 charges, 36 against 25 at 210,000).
constexpr int kGatherWideBricks = 512;
// owner slots of a block: the candidates of one pass
__host__ __device__ constexpr int gather_slots(int P) {
    return gather_fixed(P) ? 256 : kGatherThreads;
}

// Dynamic LDS of a gather block for stencil half width P (byte offsets): the
// halo of edge brick + 2P - 1 and the per-owner weights are sized by P.
// gather_fix's layout for P = 3 and 5, which has no range tables and fewer
// owner slots, gather_any's for the others.
struct GatherLds {
    int own, ownf, ownp, sphi, sw, rowtab, pbeg, poff, wtot, total;
};
__host__ __device__ constexpr GatherLds gather_lds(int P, int waves) {
    const int E = gather_brick(P) + 2 * P - 1;
    GatherLds L{};
    int o = 0;
    auto take = [&](int bytes) {
        const int r = o;
        o += (bytes + 15) & ~15;
        return r;
    };
    L.own = take(16 * gather_slots(P));                // owner records
    L.ownf = take(16 * gather_slots(P));               // owners' near forces
    L.ownp = take(4 * gather_slots(P));                // owners' input indices
    L.sphi = take(4 * E * E * E);                      // potential on brick + halo
    // weights, derivatives [wave][owner][6][2P]
    L.sw = take(4 * waves * (64 / gather_lanes(P)) * 6 * 2 * P);
    L.rowtab = take(8 * 4 * P * P);                    // stencil rows {offset, ky | kz << 16}
    if (!gather_fixed(P)) {
        L.pbeg = take(4 * kGatherMaxPieces);
        L.poff = take(4 * (kGatherMaxPieces + 1));
    }
    L.wtot = take(4 * waves);
    L.total = o;
    return L;
}

// any stencil half width but those of gather_fix
__device__ __forceinline__ void gather_any(const GridArgs& a, int bid,
                                            const uint4* __restrict__ sorted,
                                            const int* __restrict__ perm,
                                            const int* __restrict__ zbin,
                                            const float* __restrict__ phi,
                                            const float4* __restrict__ fnear,
                                            float* __restrict__ forces, char* lds) {
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    // LPO lanes per owner charge, OPW owners per wavefront pass
    constexpr int LPO = 16, OPW = 64 / LPO;
    const int g = lane / LPO, lg = lane % LPO;
    const int P = a.P, P2 = 2 * P, GB = gather_brick(P);
    constexpr int KMAX = 2 * kMaxStencilHalf;   // x points per stencil row
    const GatherLds LL = gather_lds(P, kGatherWaves);
    uint4* own = reinterpret_cast<uint4*>(lds + LL.own);
    float4* ownf = reinterpret_cast<float4*>(lds + LL.ownf);
    int* ownp = reinterpret_cast<int*>(lds + LL.ownp);
    float* sphi = reinterpret_cast<float*>(lds + LL.sphi);
    float* swb = reinterpret_cast<float*>(lds + LL.sw);
    int2* rowtab = reinterpret_cast<int2*>(lds + LL.rowtab);
    int* pbeg = reinterpret_cast<int*>(lds + LL.pbeg);
    int* poff = reinterpret_cast<int*>(lds + LL.poff);
    int* wtot = reinterpret_cast<int*>(lds + LL.wtot);
    const Brick K = brick_at(a, bid, GB, GB == 8 ? a.mb8 : a.mb4);
    const int X0 = K.o[0], Y0 = K.o[1], Z0 = K.o[2], B0 = K.n[0], B1 = K.n[1], B2 = K.n[2];
    const int E0 = B0 + P2 - 1, E1 = B1 + P2 - 1, E2 = B2 + P2 - 1;
    // potential on the brick and halo: local (hx, hy, hz) = global (X0 - P + 1 + hx, ...)
    // approximate reciprocals: (idx + 1/2) / E stays 1 / (2E) from an integer
    const float inv0 = __builtin_amdgcn_rcpf((float)E0), inv1 = __builtin_amdgcn_rcpf((float)E1);
    const int nh = E0 * E1 * E2;
    // columns overlapping the brick's cells in x and y (at most one per
    // thread): the charge range of the brick's z-planes in each, loaded first
    // so that these loads are in flight with the halo's
    static_assert(kGatherMaxPieces <= kGatherThreads, "one column per thread");
    const int cxl = magic_div(X0 * a.nc[0], a.mg[0]),
              cxh = magic_div((X0 + B0) * a.nc[0] + a.g[0] - 1, a.mg[0]) - 1;
    const int cyl = magic_div(Y0 * a.nc[1], a.mg[1]),
              cyh = magic_div((Y0 + B1) * a.nc[1] + a.g[1] - 1, a.mg[1]) - 1;
    const int cxn = cxh - cxl + 1, np = cxn * (cyh - cyl + 1);
    int zb = 0, ze = 0;
    if (tid < np) {
        const int ky = small_div(tid, __builtin_amdgcn_rcpf((float)cxn));
        const int col = (cyl + ky) * a.nc[0] + cxl + tid - ky * cxn;
        const int* zr = zbin + (size_t)col * (a.g[2] + 1);
        zb = zr[Z0];
        ze = zr[Z0 + B2];
    }
    // the loads of a pass are issued together, then stored
    auto halo_pass = [&](int base) {
        float v[kGatherBatch];
#pragma unroll
        for (int u = 0; u < kGatherBatch; ++u) {
            const int idx = base + kGatherThreads * u;
            const int r = small_div(idx, inv0), hx = idx - r * E0;
            const int hz = small_div(r, inv1), hy = r - hz * E1;
            const int gx = wrap1(X0 - P + 1 + hx, a.g[0]);
            const int gy = wrap1(Y0 - P + 1 + hy, a.g[1]);
            const int gz = wrap1(Z0 - P + 1 + hz, a.g[2]);
            v[u] = idx < nh ? phi[((size_t)gz * a.g[1] + gy) * a.g[0] + gx] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < kGatherBatch; ++u) {
            const int idx = base + kGatherThreads * u;
            if (idx < nh) sphi[idx] = v[u];
        }
    };
    constexpr int kPass = kGatherThreads * kGatherBatch;
    for (int base = tid; base < nh; base += kPass) halo_pass(base);
    // stencil rows (ky, kz) of a charge and their offsets in the halo, once per block
    for (int r = tid; r < P2 * P2; r += kGatherThreads) {
        const int ky = r % P2, kz = r / P2;
        rowtab[r] = make_int2((kz * E1 + ky) * E0, ky | (kz << 16));
    }
    if (tid < np) {
        pbeg[tid] = zb;
        poff[tid + 1] = ze - zb;
    }
    __syncthreads();
    {
        const int v = tid < np ? poff[tid + 1] : 0;
        const int incl = wave_incl_scan(v);
        if (lane == 63) wtot[wave] = incl;
        __syncthreads();
        int wbase = 0;
        for (int w = 0; w < wave; ++w) wbase += wtot[w];
        if (tid < np) poff[tid + 1] = wbase + incl;
        if (tid == 0) poff[0] = 0;
        __syncthreads();
    }
    const int total = poff[np];
    for (int base = 0; base < total; base += kGatherThreads) {
        const int t = base + tid;
        bool mine = false;
        uint4 c = make_uint4(0, 0, 0, 0);
        float4 fn = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        int pj = 0;
        if (t < total) {
            int l = 0, h = np;
            while (h - l > 1) {
                const int mid = (l + h) >> 1;
                if (poff[mid] <= t) l = mid; else h = mid;
            }
            const int j = pbeg[l] + (t - poff[l]);
            // the near force and input index load with the record (most
            // candidates are owners), saving a round trip after the ballot
            c = sorted[j];
            fn = fnear[j];
            pj = perm[j];
            const int gx = cell_coord(c.x, a.g[0]), gy = cell_coord(c.y, a.g[1]);
            mine = gx >= X0 && gx < X0 + B0 && gy >= Y0 && gy < Y0 + B1;
        }
        const uint64_t m = __ballot(mine);
        if (lane == 0) wtot[wave] = __popcll(m);
        __syncthreads();
        int before = 0, nown = 0;
#pragma unroll
        for (int w = 0; w < kGatherWaves; ++w) {
            before += w < wave ? wtot[w] : 0;
            nown += wtot[w];
        }
        if (mine) {
            const int slot = before + __popcll(m & ((1ull << lane) - 1ull));
            own[slot] = c;
            ownf[slot] = fn;
            ownp[slot] = pj;
        }
        __syncthreads();
        // OPW owners per wavefront pass, groups dealt round-robin to the wavefronts
        for (int o0 = wave * OPW; o0 < nown; o0 += OPW * kGatherWaves) {
            const int o = o0 + g;
            const bool valid = o < nown;
            int gi[3] = {0, 0, 0};
            float f[3] = {0.0f, 0.0f, 0.0f};
            float qi = 0.0f;
            if (valid) {
                const uint4 cc = own[o];
                grid_coord(cc.x, a.g[0], &gi[0], &f[0]);
                grid_coord(cc.y, a.g[1], &gi[1], &f[1]);
                grid_coord(cc.z, a.g[2], &gi[2], &f[2]);
                qi = __uint_as_float(cc.w);
                // lane lg < 2P: weights and derivatives of stencil point lg, all axes
                if (lg < P2) {
#pragma unroll
                    for (int ax = 0; ax < 3; ++ax) {
                        const float tt = (float)(lg - P + 1) - f[ax];
                        const float w = a.cw[ax] * __expf(-tt * tt * a.hs[ax]);
                        swb[((wave * OPW + g) * 6 + ax) * P2 + lg] = w;
                        swb[((wave * OPW + g) * 6 + 3 + ax) * P2 + lg] = w * tt * a.dws[ax];
                    }
                }
            }
            wave_sync();
            float px = 0.0f, py = 0.0f, pz = 0.0f;
            if (valid) {
                const float* W = swb + (wave * OPW + g) * 6 * P2;   // [6][2P]
                // stencil point k of the charge is halo point (gi - brick origin) + k
                const int lx = gi[0] - X0, ly = gi[1] - Y0, lz = gi[2] - Z0;
                const float* obase = sphi + (lz * E1 + ly) * E0 + lx;
                for (int r = lg; r < P2 * P2; r += LPO) {
                    const int2 rt = rowtab[r];
                    const int ky = rt.y & 0xffff, kz = rt.y >> 16;
                    const float* rowp = obase + rt.x;
                    float sx = 0.0f, dsx = 0.0f;
#pragma unroll
                    for (int k = 0; k < KMAX; ++k) {
                        if (k < P2) {
                            const float v = rowp[k];
                            sx = fmaf(W[k], v, sx);
                            dsx = fmaf(W[3 * P2 + k], v, dsx);
                        }
                    }
                    const float wy = W[P2 + ky], wz = W[2 * P2 + kz];
                    px = fmaf(wy * wz, dsx, px);
                    py = fmaf(W[4 * P2 + ky] * wz, sx, py);
                    pz = fmaf(wy * W[5 * P2 + kz], sx, pz);
                }
            }
            px = row_sum16(px);
            py = row_sum16(py);
            pz = row_sum16(pz);
            if (valid && lg == 0) {
                const float4 fn = ownf[o];    // near force from the pair kernel
                const int oi = ownp[o];
                forces[3 * oi + 0] = fn.x - qi * px;
                forces[3 * oi + 1] = fn.y - qi * py;
                forces[3 * oi + 2] = fn.z - qi * pz;
            }
            wave_sync();
        }
        __syncthreads();
    }
}

// The two forms' stencils, P compiled in.  A wavefront evaluates OPW owners at
// a time, LPO lanes each: the 3 x 2P weights and derivatives are evaluated by
// the owner's lanes in turn and left in LDS as (weight, derivative) pairs; a
// lane keeps the x pairs in registers and takes every LPO-th of the (2P)^2
// stencil rows: 2P potentials from LDS against them, then three products with
// the row's y and z pairs.
//
// Bound: VALU and LDS about evenly: (2P)^3 potentials read and 2 FMAs on each,
// per charge.  With four weight reads per row, the halo's indices by two
// divisions per value, a bisection per candidate and 56 KB of LDS (two blocks
// per CU at P = 5, now 37 KB), 90,180 charges took 42.5 us plain (now 30.0) and
// 20.3 BF16X3 (14.3); 26,268 charges 14.0 (11.7) and 8.0 (6.7); 210,000 42.2
// (25.6, of which about 12 by the energy total's loads in flight together).
template <int P, int kWaves>
__device__ __forceinline__ void gather_fix(const GridArgs& a, int bid,
                                           const uint4* __restrict__ sorted,
                                           const int* __restrict__ perm,
                                           const int* __restrict__ zbin,
                                           const float* __restrict__ phi,
                                           const float4* __restrict__ fnear,
                                           float* __restrict__ forces, char* lds) {
    constexpr int P2 = 2 * P, GB = gather_brick(P), E = GB + P2 - 1, R = P2 * P2;
    constexpr int kSlots = gather_slots(P), kThreads = 64 * kWaves;
    constexpr int LPO = gather_lanes(P), OPW = 64 / LPO;   // lanes per owner, owners per pass
    constexpr GatherLds LL = gather_lds(P, kWaves);
    static_assert(GB == 8 && kSlots % 64 == 0 && kSlots <= kThreads, "");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float4* own = reinterpret_cast<float4*>(lds + LL.own);     // fractions, halo offset
    float4* ownf = reinterpret_cast<float4*>(lds + LL.ownf);   // near force, charge
    int* ownp = reinterpret_cast<int*>(lds + LL.ownp);
    float* sphi = reinterpret_cast<float*>(lds + LL.sphi);
    int2* rowtab = reinterpret_cast<int2*>(lds + LL.rowtab);
    int* wtot = reinterpret_cast<int*>(lds + LL.wtot);
    const Brick K = brick_at(a, bid, GB, a.mb8);
    // columns overlapping the brick's cells in x and y
    const int cxl = magic_div(K.o[0] * a.nc[0], a.mg[0]),
              cxh = magic_div((K.o[0] + K.n[0]) * a.nc[0] + a.g[0] - 1, a.mg[0]) - 1;
    const int cyl = magic_div(K.o[1] * a.nc[1], a.mg[1]),
              cyh = magic_div((K.o[1] + K.n[1]) * a.nc[1] + a.g[1] - 1, a.mg[1]) - 1;
    const int cxn = cxh - cxl + 1, np = cxn * (cyh - cyl + 1);
    // the charges of the brick's z-planes in columns k0 .. k0 + 63, one per
    // lane (every wavefront holds them all): loaded first, in flight with the
    // halo's loads
    int zb = 0, zn = 0;
    auto ranges = [&](int k0) {
        const int k = k0 + lane;
        zb = zn = 0;
        if (k < np) {
            const int ky = small_div(k, __builtin_amdgcn_rcpf((float)cxn));
            const int* zr = zbin + (size_t)((cyl + ky) * a.nc[0] + cxl + k - ky * cxn) * (a.g[2] + 1);
            zb = zr[K.o[2]];
            zn = zr[K.o[2] + K.n[2]] - zb;
        }
    };
    ranges(0);
    // potential on the brick and halo: local (hx, hy, hz) = global (X0 - P + 1
    // + hx, ...), E^3 in LDS whatever the brick's own extent.  A thread keeps
    // its hx and takes every kRows-th row (hy, hz)
    {
        constexpr int kRows = kThreads / E, kIter = (E * E + kRows - 1) / kRows;
        const int r0 = small_div(tid, 1.0f / (float)E), hx = tid - r0 * E;
        int hz = small_div(r0, 1.0f / (float)E), hy = r0 - hz * E;
        // origin (modulo the axis) + position < g + E - 1 < 3 g, as g >= 2P
        static_assert(E - 2 < 2 * P2, "");
        const int gx = mod_twice(wrap1(K.o[0] - P + 1, a.g[0]) + hx, a.g[0]);
        const int oy = wrap1(K.o[1] - P + 1, a.g[1]), oz = wrap1(K.o[2] - P + 1, a.g[2]);
        const bool in = r0 < kRows && hx < K.n[0] + P2 - 1;
        float v[kIter];
#pragma unroll
        for (int u = 0; u < kIter; ++u) {
            v[u] = 0.0f;
            if (in && hy < K.n[1] + P2 - 1 && hz < K.n[2] + P2 - 1)
                v[u] = phi[(size_t)(mod_twice(oz + hz, a.g[2]) * a.g[1] + mod_twice(oy + hy, a.g[1])) *
                               a.g[0] + gx];
            hy += kRows % E;
            hz += kRows / E;
            if (hy >= E) {
                hy -= E;
                ++hz;
            }
        }
#pragma unroll
        for (int u = 0; u < kIter; ++u)
            if (r0 < kRows && r0 + u * kRows < E * E) sphi[(r0 + u * kRows) * E + hx] = v[u];
    }
    // stencil rows (ky, kz): offset in the halo, and of the weight pairs (bytes)
    for (int r = tid; r < R; r += kThreads) {
        const int kz = small_div(r, 1.0f / (float)P2), ky = r - kz * P2;
        rowtab[r] = make_int2((kz * E + ky) * E, (P2 + ky) * 8 | ((2 * P2 + kz) * 8) << 16);
    }
    // weight evaluations of this lane: values lg, lg + 8, ... of the owner's 6P
    // (axis, point), and what they take from the axis
    constexpr int kEval = (3 * P2 + LPO - 1) / LPO;
    const int g = lane / LPO, lg = lane % LPO;
    int eax[kEval];
    float et[kEval], ehs[kEval], ecw[kEval], edw[kEval];
#pragma unroll
    for (int m = 0; m < kEval; ++m) {
        const int i = lg + LPO * m;
        const int ax = i < P2 ? 0 : i < 2 * P2 ? 1 : 2;
        eax[m] = ax;
        et[m] = (float)(i - ax * P2 - P + 1);
        ehs[m] = ax == 0 ? a.hs[0] : ax == 1 ? a.hs[1] : a.hs[2];
        ecw[m] = ax == 0 ? a.cw[0] : ax == 1 ? a.cw[1] : a.cw[2];
        edw[m] = ax == 0 ? a.dws[0] : ax == 1 ? a.dws[1] : a.dws[2];
    }
    // this group's weight pairs [axis][point]
    float2* W = reinterpret_cast<float2*>(lds + LL.sw) + (wave * OPW + g) * 3 * P2;

    for (int k0 = 0; k0 < np; k0 += 64) {
        if (k0 > 0) ranges(k0);
        const int incl = wave_incl_scan(zn);
        const int off = incl - zn, rel = zb - off;
        const int total = __builtin_amdgcn_readlane(incl, 63);
        for (int base = 0; base < total; base += kSlots) {
            // candidates base + tid of the ranges laid end to end: the last
            // range that starts at or before the wavefront's first, then those
            // that start among them
            const int t0 = base + 64 * wave, t = t0 + lane;
            bool mine = false;
            uint4 c = make_uint4(0, 0, 0, 0);
            float4 fn = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            int pj = 0;
            if (wave < kSlots / 64 && t0 < total) {
                int r = __popcll(__builtin_amdgcn_ballot_w64(off <= t0)) - 1;
                int j = t + __builtin_amdgcn_readlane(rel, r);
                for (++r; r < 64; ++r) {
                    const int o = __builtin_amdgcn_readlane(off, r);
                    if (o > t0 + 63 || o >= total) break;
                    if (t >= o) j = t + __builtin_amdgcn_readlane(rel, r);
                }
                if (t < total) {
                    // the near force and input index load with the record (most
                    // candidates are owners), saving a round trip after the ballot
                    c = sorted[j];
                    fn = fnear[j];
                    pj = perm[j];
                    const int gx = cell_coord(c.x, a.g[0]), gy = cell_coord(c.y, a.g[1]);
                    mine = gx >= K.o[0] && gx < K.o[0] + K.n[0] && gy >= K.o[1] &&
                           gy < K.o[1] + K.n[1];
                }
            }
            const uint64_t m = __builtin_amdgcn_ballot_w64(mine);
            if (lane == 0) wtot[wave] = __popcll(m);
            __syncthreads();
            int before = 0, nown = 0;
#pragma unroll
            for (int w = 0; w < kSlots / 64; ++w) {
                const int n = wtot[w];
                before += w < wave ? n : 0;
                nown += n;
            }
            nown = __builtin_amdgcn_readfirstlane(nown);
            if (mine) {
                const int slot = before + lanes_below(m);
                int gi[3];
                float f[3];
                grid_coord(c.x, a.g[0], &gi[0], &f[0]);
                grid_coord(c.y, a.g[1], &gi[1], &f[1]);
                grid_coord(c.z, a.g[2], &gi[2], &f[2]);
                // stencil point k of the charge is halo point (cell - brick origin) + k
                const int ob = ((gi[2] - K.o[2]) * E + gi[1] - K.o[1]) * E + gi[0] - K.o[0];
                own[slot] = make_float4(f[0], f[1], f[2], __int_as_float(ob));
                ownf[slot] = make_float4(fn.x, fn.y, fn.z, __uint_as_float(c.w));
                ownp[slot] = pj;
            }
            __syncthreads();
            // OPW owners per wavefront pass, groups dealt round-robin to the wavefronts
            for (int o0 = wave * OPW; o0 < nown; o0 += OPW * kWaves) {
                const int o = min(o0 + g, nown - 1);     // a group past the end repeats the last
                const float* of = reinterpret_cast<const float*>(own + o);
#pragma unroll
                for (int v = 0; v < kEval; ++v) {
                    const float tt = et[v] - of[eax[v]];
                    const float w = ecw[v] * __expf(-tt * tt * ehs[v]);
                    if (LPO * (v + 1) <= 3 * P2 || lg + LPO * v < 3 * P2)
                        W[lg + LPO * v] = make_float2(w, w * tt * edw[v]);
                }
                const float* obase = sphi + __float_as_int(of[3]);
                wave_sync();
                float2 wx[P2];
#pragma unroll
                for (int k = 0; k < P2; ++k) wx[k] = W[k];
                float px = 0.0f, py = 0.0f, pz = 0.0f;
#pragma unroll
                for (int it = 0; it < (R + LPO - 1) / LPO; ++it) {
                    if (LPO * (it + 1) <= R || lg + LPO * it < R) {
                        const int2 rt = rowtab[lg + LPO * it];
                        const float* rowp = obase + rt.x;
                        const float2 wy = *reinterpret_cast<const float2*>(
                            reinterpret_cast<const char*>(W) + (rt.y & 0xffff));
                        const float2 wz = *reinterpret_cast<const float2*>(
                            reinterpret_cast<const char*>(W) + (rt.y >> 16));
                        float sx = 0.0f, dsx = 0.0f;
#pragma unroll
                        for (int k = 0; k < P2; ++k) {
                            const float v = rowp[k];
                            sx = fmaf(wx[k].x, v, sx);
                            dsx = fmaf(wx[k].y, v, dsx);
                        }
                        px = fmaf(wy.x * wz.x, dsx, px);
                        py = fmaf(wy.y * wz.x, sx, py);
                        pz = fmaf(wy.x * wz.y, sx, pz);
                    }
                }
                px = LPO == 8 ? sum8(px) : row_sum16(px);
                py = LPO == 8 ? sum8(py) : row_sum16(py);
                pz = LPO == 8 ? sum8(pz) : row_sum16(pz);
                if (lg == 0 && o0 + g < nown) {
                    const float4 fo = ownf[o];    // near force from the pair kernel, charge
                    float* out = forces + 3 * (size_t)ownp[o];
                    out[0] = fo.x - fo.w * px;
                    out[1] = fo.y - fo.w * py;
                    out[2] = fo.z - fo.w * pz;
                }
                wave_sync();
            }
            __syncthreads();
        }
    }
}

// PT = 3 or 5, or 0: a.P, any other (NW = kGatherWaves)
template <int PT, int NW>
__device__ __forceinline__ void gather_body(const GridArgs& a, int bid,
                                            const uint4* __restrict__ sorted,
                                            const int* __restrict__ perm,
                                            const int* __restrict__ zbin,
                                            const float* __restrict__ phi,
                                            const float4* __restrict__ fnear,
                                            float* __restrict__ forces, char* lds) {
    if constexpr (PT > 0)
        gather_fix<PT, NW>(a, bid, sorted, perm, zbin, phi, fnear, forces, lds);
    else
        gather_any(a, bid, sorted, perm, zbin, phi, fnear, forces, lds);
}

// Block 0 forms the energy total: it reads only what earlier launches wrote, so
// it runs beside the bricks (first, as it has the longest chain of loads).
template <int PT, int NW>
__global__ void __launch_bounds__(64 * NW) k_gather(int nb,
                                                const int* __restrict__ zbin,
                                                const float* __restrict__ phi,
                                                const uint4* __restrict__ sorted,
                                                const float4* __restrict__ fnear,
                                                const int* __restrict__ perm,
                                                float* __restrict__ forces,
                                                const double* __restrict__ pair_parts,
                                                const double* __restrict__ far_parts,
                                                const double* __restrict__ qstats,
                                                double* __restrict__ energy,
                                                double* __restrict__ parts, GridArgs a,
                                                FinalArgs fa) {
    extern __shared__ char dyn[];
    if (blockIdx.x == 0) {
        energy_total<kGatherThreads>(fa, pair_parts, far_parts, qstats, energy, parts,
                                     reinterpret_cast<double*>(dyn));
        return;
    }
    const int item = xcd_item(blockIdx.x - 1, nb);
    if (item < nb) gather_body<PT, NW>(a, item, sorted, perm, zbin, phi, fnear, forces, dyn);
}

// every box of the batch has stencil half width PT
template <int PT>
__global__ void __launch_bounds__(kGatherThreads) k_gather_batch(const BatchTable* __restrict__ tab,
                                                      const BoxDesc* __restrict__ desc) {
    extern __shared__ char dyn[];
    batch_for(tab, BK_GATHER, [&](int i, int item) {
        const BoxDesc& d = desc[tab->slot[i]];
        if (item == d.ngb)   // the box's energy total, after its bricks
            energy_total<kGatherThreads>(d.fin, d.pair_parts, d.far_parts, d.qstats,
                                         d.energies + tab->step[i], nullptr,
                                         reinterpret_cast<double*>(dyn));
        else
            gather_body<PT, kGatherWaves>(d.grid, item, d.sorted, d.perm, d.zbin, d.phi, d.fnear, d.forces,
                            dyn);
    });
}

hipError_t launch_spread(const GridArgs& a, const uint4* sorted, const int* zbin,
                         const double* qstats, float* rho, hipStream_t st) {
    const int nb = ((a.g[0] + kBrick - 1) / kBrick) * ((a.g[1] + kBrick - 1) / kBrick) *
                   ((a.g[2] + kBrick - 1) / kBrick);
    hipLaunchKernelGGL(k_spread, dim3(xcd_blocks(nb)), dim3(64 * kSpreadWaves), 0, st, nb, zbin,
                       qstats, sorted, rho, a);
    return hipGetLastError();
}

int gather_blocks(const GridArgs& a) {
    const int GB = gather_brick(a.P);
    return ((a.g[0] + GB - 1) / GB) * ((a.g[1] + GB - 1) / GB) * ((a.g[2] + GB - 1) / GB);
}

hipError_t launch_gather(const GridArgs& a, const uint4* sorted, const int* perm, const int* zbin,
                         const float* phi, const float4* fnear, float* forces,
                         const FinalArgs& fa, const double* pair_parts, const double* far_parts,
                         const double* qstats, double* energy, double* parts, hipStream_t st) {
    const int nb = gather_blocks(a);
    const dim3 grid(xcd_blocks(nb) + 1);
    // the default stencils of the two forms (P = 3, 5) have their own code
#define USERIES_GATHER_LAUNCH(PT, NW)                                                        \
    hipLaunchKernelGGL((k_gather<PT, NW>), grid, dim3(64 * NW),                              \
                       (size_t)gather_lds(a.P, NW).total, st, nb, zbin, phi, sorted, fnear,  \
                       perm, forces, pair_parts, far_parts, qstats, energy, parts, a, fa)
    if (a.P == 3)
        USERIES_GATHER_LAUNCH(3, kGatherWaves);
    else if (a.P == 5 && nb <= kGatherWideBricks)
        USERIES_GATHER_LAUNCH(5, 16);
    else if (a.P == 5)
        USERIES_GATHER_LAUNCH(5, kGatherWaves);
    else
        USERIES_GATHER_LAUNCH(0, kGatherWaves);
#undef USERIES_GATHER_LAUNCH
    return hipGetLastError();
}

hipError_t launch_spread_batch(const BatchTable* tab, const BoxDesc* desc, int grid,
                               hipStream_t st) {
    hipLaunchKernelGGL(k_spread_batch, dim3(grid), dim3(64 * kSpreadWaves), 0, st, tab, desc);
    return hipGetLastError();
}

size_t gather_lds_bytes(int P) { return (size_t)gather_lds(P, kGatherWaves).total; }

hipError_t launch_gather_batch(const BatchTable* tab, const BoxDesc* desc, int P, size_t lds,
                               int grid, hipStream_t st) {
    const dim3 g(grid), b(kGatherThreads);
    if (P == 3)
        hipLaunchKernelGGL(k_gather_batch<3>, g, b, lds, st, tab, desc);
    else if (P == 5)
        hipLaunchKernelGGL(k_gather_batch<5>, g, b, lds, st, tab, desc);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace useries

// fd_step2d.hip -- several leapfrog levels of the 2D acoustic step in one
// launch (the tiling of Section 2.2 and the wave-front tiling of Section
// 2.3.1, done in the registers and LDS of a workgroup).
//
// A one-step launch on a 2D grid is a chain of latencies: 7 us even where
// four workgroups hold the whole grid, and 12.6 us on 2481 x 1281 at so 8,
// where the 51 MB it moves would take 7 us.  Here a workgroup stages a 64 x
// 64 region of u^n, u^{n-1} and p once and advances it `nlev` levels; the
// region shrinks by R points per side and level, so the inner (64 - 2 Hx) x
// (64 - 2 H) points, H = R nlev, are exact at the last one and are written.
// The ring belongs to the neighbours and is recomputed, so no workgroup
// waits for another.  Each level is the one-step kernel's sequence of
// float32 operations (16-bit fields are rounded at every level), so the
// fields are bitwise those of nlev one-step launches.
//
// Split: 512 lanes as 16 float4 columns x 32 blocks of 2 rows.  A lane keeps
// u^n, u^{n-1}, p and 1/(1+s) of its quads in registers for all levels; LDS
// carries only the neighbours' current level (two buffers in turn, one
// barrier per level), and two rows per lane share their column's reads.  The
// row stride of 16 float4 is conflict-free for 16-byte reads (4.4 cycles per
// wave; 8.3 at strides that are not a multiple of 16).  Measured per step,
// float32, nine shapes at every level count (us; one step per launch first):
// 181^2 so 4 7.7, 256 lanes with 4 rows each 1.86, this 1.47, 48 staged rows
// 1.42; 2481 x 1281 so 4 12.5, 5.36, 5.10, 6.16; 4081 x 2081 so 2 26.3, 6.58,
// 6.04, 7.37, so 8 27.8, 19.2, 18.8, 23.1; staging 128 points per row or 96
// rows was slower on every small grid and at most 4 % faster on large ones.
#include "fd_step3d.h"

#include <algorithm>

namespace fd {
namespace {

constexpr int kW4 = 16, kRows = 64, kK = 2;   // staged float4 columns, rows; rows per lane
constexpr int kNT = kW4 * kRows / kK;         // lanes of a workgroup
constexpr int kNodeReach = 15;                // Step2Args::node_reach at most (windowed sinc of half-width 8)
constexpr int kSrcCap = 128;                  // source points of a tile whose values are formed up front

// u^{n+1} .. at the sampled levels of the previous launch
template <Store S>
__device__ void sample_rows(const SampleRows &s, int blk) {
    const int row = blk / s.bpr;
    Sample q{s.npts, s.nc, s.lpp, s.idx, s.w, s.out + row * s.ostride, s.scale};
    sample_block<S, kNT>(q, s.field[row], blk - row * s.bpr);
}

template <Store S>
__global__ __launch_bounds__(kNT) void k_sample_rows(const SampleRows s) {
    sample_rows<S>(s, (int)blockIdx.x);
}

template <int R, Store S, int MODE>
__global__ __launch_bounds__(kNT) void k_step2d_tb(const Step2Args a) {
    using E = Elem<S>;
    using T = typename E::T;
    constexpr int HX4 = (R + 3) / 4;
    // rows above and below and quads before and after the staged region
    // exist only so that every neighbour read stays in the buffer
    constexpr int kBuf = (kRows + 2 * R) * kW4 + 2 * HX4;
    __shared__ float4 lds[2][kBuf];
    __shared__ int s_pos[kSrcCap];
    __shared__ float s_val[kTb2MaxLev * kSrcCap];

    const int ntile = (int)gridDim.x - a.nsamp_blocks;   // tiles first, then sampling
    if ((int)blockIdx.x >= ntile) {
        sample_rows<S>(a.smp, (int)blockIdx.x - ntile);
        return;
    }
    const Layout L = a.L;
    const int nlev = a.nlev;
    const int H = R * nlev, Hx = (H + 3) & ~3;
    const int t0 = xcd_remap((int)blockIdx.x, ntile);
    const int bx = t0 % a.ntx, bz = t0 / a.ntx;
    const int x0 = bx * (4 * kW4 - 2 * Hx) - Hx, z0 = bz * (kRows - 2 * H) - H;   // grid coordinates of staged (0, 0)
    const int lane = (int)threadIdx.x;
    const int c = lane % kW4, row0 = (lane / kW4) * kK;
    const int x = x0 + 4 * c;
    const bool xin = x >= 0 && x < L.nx;
    const long long zcol = L.offset((L.nx + 3) & ~3, 0, 0);   // zero in every field
    const int own = HX4 + (R + row0) * kW4 + c;

    // two register sets take turns as the current and the previous level
    float4 ua[kK], ub[kK], p[kK], al[kK];
    [[maybe_unused]] float4 gp[kK];
    [[maybe_unused]] float sz[kK];
    long long off[kK];
    bool in[kK];
#pragma unroll
    for (int k = 0; k < kK; ++k) {
        const int z = z0 + row0 + k;
        in[k] = xin && z >= 0 && z < L.nz;
        off[k] = in[k] ? L.offset(x, 0, z) : zcol;
        ua[k] = E::ld4((const T *)a.u + off[k]);
        ub[k] = E::ld4((const T *)a.prev + off[k]);
        p[k] = *reinterpret_cast<const float4 *>(a.p + off[k]);
        if constexpr (MODE == kImage) gp[k] = *reinterpret_cast<const float4 *>(a.gpart + off[k]);
    }
    float sx[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) sx[i] = xin ? a.damp[min(x + i, L.nx - 1)] : 0.f;
#pragma unroll
    for (int k = 0; k < kK; ++k) {
        const float s = in[k] ? a.damp[L.nx + L.ny + z0 + row0 + k] : 0.f;
        sz[k] = s;
        al[k] = make_float4(__builtin_amdgcn_rcpf(1.f + (sx[0] + s)), __builtin_amdgcn_rcpf(1.f + (sx[1] + s)),
                            __builtin_amdgcn_rcpf(1.f + (sx[2] + s)), __builtin_amdgcn_rcpf(1.f + (sx[3] + s)));
    }

    // Source points of the staged region: of each 64-point column of the
    // tables that it overlaps the rows it stages.
    constexpr int NC = (4 * kW4 + kTileX - 2) / kTileX + 1;   // columns that a tile can overlap
    int e0[NC], nsum[NC], ns = 0;   // first point of each column, points up to its end
    const int ct0 = max(x0, 0) / kTileX, ct1 = min(x0 + 4 * kW4 - 1, L.nx - 1) / kTileX;
    const int za = max(z0, 0), zb = min(z0 + kRows, L.nz);
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        const int *q = a.inj_pp + (long long)min(ct0 + i, ct1) * (L.nz + 1);
        e0[i] = q[za];
        nsum[i] = q[zb];
    }
    // Whether the tile holds points that are sampled (its intermediate levels
    // are then stored for the next launch's sampling).  The tables leave out
    // nodes of weight zero, which are read all the same (0 times what an
    // earlier run left there may be NaN): every node lies within node_reach of
    // one that the tables have.  (All pointers are loaded before the first is
    // waited for, a column again rather than behind a branch.)
    constexpr int NN = (4 * kW4 + 2 * kNodeReach + kTileX - 2) / kTileX + 1;   // columns in reach, at most
    int nlo[NN], nhi[NN];
    const bool sampled = a.node_pp && nlev > 2;
    if (sampled) {
        const int n = a.node_reach;
        const int xu0 = max(x0 + Hx - n, 0), xu1 = min(x0 + 4 * kW4 - Hx + n, L.nx) - 1;
        const int zu0 = max(z0 + H - n, 0), zu1 = min(z0 + kRows - H + n, L.nz);
#pragma unroll
        for (int i = 0; i < NN; ++i) {
            const int *q = a.node_pp + (long long)min(xu0 / kTileX + i, xu1 / kTileX) * (L.nz + 1);
            nlo[i] = q[zu0];
            nhi[i] = q[zu1];
        }
    }
    bool nodes = false;
#pragma unroll
    for (int i = 0; i < NN; ++i) nodes |= sampled && nlo[i] < nhi[i];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        if (a.vals && ct0 + i <= ct1) ns += nsum[i] - e0[i];
        nsum[i] = ns;
    }
    auto entry = [&](int j) {   // table index of the j-th source point
        int e = e0[0] + j;
#pragma unroll
        for (int i = 1; i < NC; ++i)
            if (j >= nsum[i - 1]) e = e0[i] + j - nsum[i - 1];
        return e;
    };
    // its place in a buffer (in floats, -1: outside the staged columns) and its
    // term at level t
    auto src_pos = [&](int e) {
        const int2 k = *reinterpret_cast<const int2 *>(a.corner + e);
        const int lx = k.x - x0;
        return (unsigned)lx < 4u * kW4 ? 4 * (HX4 + (R + k.y - z0) * kW4) + lx : -1;
    };
    auto src_val = [&](int e, int t) {
        const float *vals = a.vals + t * a.vstride;
        float v = 0.f;
        if (a.one_entry) {   // entry e is point e's only one: no wait for its range
            v = __builtin_fmaf(a.w[e], vals[a.src[e]], v);
        } else {
            const int4 k = a.corner[e];
            for (int i = k.z; i < k.w; ++i) v = __builtin_fmaf(a.w[i], vals[a.src[i]], v);
        }
        return v * a.scale;
    };
    const bool front = ns <= kSrcCap;
    if (ns > 0 && front)
        for (int i = lane; i < ns * nlev; i += kNT) {
            const int t = i / ns, j = i - t * ns;
            const int e = entry(j);
            if (t == 0) s_pos[j] = src_pos(e);
            s_val[t * kSrcCap + j] = src_val(e, t);
        }

    // the lane's quads that are this tile's to write
    bool mine[kK];
#pragma unroll
    for (int k = 0; k < kK; ++k)
        mine[k] = in[k] && c >= Hx / 4 && c < kW4 - Hx / 4 && row0 + k >= H && row0 + k < kRows - H;
    // Tiles at the grid's edge force points outside the grid to zero (the
    // zero extension); p is zero there, but 0 times an overflowed sum is not.
    const bool edge = x0 < 0 || x0 + 4 * kW4 > L.nx || z0 < 0 || z0 + kRows > L.nz;

#pragma unroll
    for (int k = 0; k < kK; ++k) lds[0][own + k * kW4] = ua[k];
    __syncthreads();

    // level t + 1 from cur (level t) and prev, written over prev
    auto level = [&](auto par, int t, const float4 *cur, float4 *prev) __attribute__((always_inline)) {
        constexpr int P = decltype(par)::value;
        const float4 *buf = lds[P];
        float4 *nxt = lds[P ^ 1];
        float4 src[kK];
        if (ns > 0) {   // (uniform) the next level's buffer carries the source terms first
            const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int k = 0; k < kK; ++k) nxt[own + k * kW4] = zero;
            __syncthreads();
            float *f = reinterpret_cast<float *>(nxt);
            for (int j = lane; j < ns; j += kNT) {
                int pos;
                float v;
                if (front) {
                    pos = s_pos[j];
                    v = s_val[t * kSrcCap + j];
                } else {
                    const int e = entry(j);
                    pos = src_pos(e);
                    v = src_val(e, t);
                }
                if (pos >= 0) f[pos] = v;
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kK; ++k) src[k] = nxt[own + k * kW4];
        }
        // rows of this level that a later one or the result needs
        const int need = R * (t + 1);
        const int wrow = __builtin_amdgcn_readfirstlane(row0);   // first row of the wave
        if (wrow + 64 / kW4 * kK > need && wrow < kRows - need) {
            [[maybe_unused]] float4 br[kK];
            if constexpr (MODE == kImage)
#pragma unroll
                for (int k = 0; k < kK; ++k)
                    br[k] = *reinterpret_cast<const float4 *>(a.br_in[t] + (mine[k] ? off[k] : zcol));
            float4 col[kK + 2 * R];   // the lane's column, R rows beyond its own on both sides
#pragma unroll
            for (int j = 0; j < kK + 2 * R; ++j)
                col[j] = j >= R && j < R + kK ? cur[j - R] : buf[own + (j - R) * kW4];
#pragma unroll
            for (int k = 0; k < kK; ++k) {
                float xs[4 * (2 * HX4 + 1)];
#pragma unroll
                for (int q = -HX4; q <= HX4; ++q) {
                    const float4 v = q == 0 ? cur[k] : buf[own + k * kW4 + q];
                    xs[4 * (q + HX4) + 0] = v.x;
                    xs[4 * (q + HX4) + 1] = v.y;
                    xs[4 * (q + HX4) + 2] = v.z;
                    xs[4 * (q + HX4) + 3] = v.w;
                }
                float lap[4];
#pragma unroll
                for (int j = 1; j <= R; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float v = lap_term2(a.wx[j], xs[4 * HX4 + i + j] + xs[4 * HX4 + i - j], a.wz[j],
                                                  comp(col[k + R + j], i) + comp(col[k + R - j], i));
                        lap[i] = j == 1 ? v : lap[i] + v;
                    }
#pragma unroll
                for (int i = 0; i < 4; ++i) lap[i] = __builtin_fmaf(a.w0, xs[4 * HX4 + i], lap[i]);
                if (ns > 0) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) lap[i] += comp(src[k], i);
                }
                const float4 m = prev[k];
                float un[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    un[i] = update_alpha(comp(cur[k], i), comp(m, i), comp(p[k], i), lap[i], comp(al[k], i));
                if (edge) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) un[i] = in[k] && x + i < L.nx ? un[i] : 0.f;
                }
                if constexpr (S != Store::F32) {
                    // round to float32, then to 16 bits, as the stored level is
                    asm volatile("" : "+v"(un[0]), "+v"(un[1]), "+v"(un[2]), "+v"(un[3]));
                    prev[k] = E::cvt(E::raw(make_float4(un[0], un[1], un[2], un[3])));
                } else {
                    prev[k] = make_float4(un[0], un[1], un[2], un[3]);
                }
                if constexpr (MODE == kBracket) {
                    float b[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        b[i] = bracket_point(un[i], comp(cur[k], i), comp(m, i), sx[i] + sz[k]);
                    if (mine[k])
                        *reinterpret_cast<float4 *>(a.br_out[t] + off[k]) = make_float4(b[0], b[1], b[2], b[3]);
                } else if constexpr (MODE == kImage) {
                    gp[k].x = __builtin_fmaf(-un[0], br[k].x, gp[k].x);
                    gp[k].y = __builtin_fmaf(-un[1], br[k].y, gp[k].y);
                    gp[k].z = __builtin_fmaf(-un[2], br[k].z, gp[k].z);
                    gp[k].w = __builtin_fmaf(-un[3], br[k].w, gp[k].w);
                }
                nxt[own + k * kW4] = prev[k];
                if (nodes && t + 2 < nlev && mine[k]) E::st4((T *)a.lev_out[t] + off[k], prev[k]);
            }
        }
        __syncthreads();
    };
    auto finish = [&](const float4 *newest, const float4 *before) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < kK; ++k)
            if (mine[k]) {
                E::st4((T *)a.out + off[k], newest[k]);
                if (nlev > 1) E::st4((T *)a.outp + off[k], before[k]);
                if constexpr (MODE == kImage) *reinterpret_cast<float4 *>(a.gpart + off[k]) = gp[k];
            }
    };
    int t = 0;
    for (; t + 2 <= nlev; t += 2) {
        level(std::integral_constant<int, 0>{}, t, ua, ub);
        level(std::integral_constant<int, 1>{}, t + 1, ub, ua);
    }
    if (t < nlev) {
        level(std::integral_constant<int, 0>{}, t, ua, ub);
        finish(ub, ua);
    } else {
        finish(ua, ub);
    }
}

using Step2Fn = void (*)(const Step2Args);

template <Store S, int MODE, int... Rs>
Step2Fn pick(int r) {
    Step2Fn f = nullptr;
    ((r == Rs ? (f = k_step2d_tb<Rs, S, MODE>, 0) : 0), ...);
    return f;
}

template <Store S, int MODE>
Step2Fn pick_r(int r) {
    return pick<S, MODE, 1, 2, 3, 4, 5, 6, 7, 8>(r);
}

// Tiles of a launch of nlev levels.
void tiles2d(const Layout &L, int nlev, int *ntx, int *ntz) {
    const int H = L.r * nlev, Hx = (H + 3) & ~3;
    const int tx = 4 * kW4 - 2 * Hx, tz = kRows - 2 * H;   // points a tile writes
    *ntx = (L.nx + tx - 1) / tx;
    *ntz = (L.nz + tz - 1) / tz;
}

}  // namespace

// Few tiles: a launch is a fixed latency of about 4 us plus 0.9 us per level
// while every tile has a CU (nearly) to itself, so as many levels as the halo
// allows: 181^2 so 4 at 2 / 4 / 8 levels 3.23 / 2.05 / 1.47 us per step, 1000 x
// 600 (608 tiles at 8) 3.41 / 2.35 / 2.01.
//
// Many tiles: the recomputed ring costs what it adds, so the count is that of
// the lowest time per step by radius, and none (0: one step per launch,
// k_step2d) where an estimate puts it above one step per launch.  The levels
// are bound by their arithmetic and take base + slope x (M points that whole
// tiles cover), 10 % more where the fields exceed the memory-side cache, in any
// storage; one step is bound by its traffic, base + slope x (M points, rows
// rounded up to 64), and moves 10 bytes per point instead of 16 in 16-bit
// storage.  Fitted to float32 and bfloat16 at every order and level count on
// 0.24 to 108 M points and on grids 5, 20, 60 and 130 points thick; on none of
// these 272 the choice is more than 1.5 % above one step per launch.  Measured
// per step (us, levels / one step): 2481 x 1281 so 8 float32 9.5 / 14.4, so 12
// 14.1 / 15.2, bfloat16 14.0 / 12.4; 4081 x 2081 so 10 float32 26.8 / 29.3,
// bfloat16 26.9 / 24.5, so 12 30.2 / 29.6 and 30.4 / 23.8; 7000 x 5000 so 6
// float32 71 / 89, bfloat16 72 / 65; 400000 x 5 so 4 18.6 / 16.4, so 12 50 / 28;
// so 16 at 2481 x 1281 27.7 / 15.8.  At so 8 in float32 three levels beat two
// from 10 M points on: 5600 x 3000 42.2, 48.7, one step 47.2; 7000 x 5000 87.4,
// 99.3, 92.5.
int step2d_levels(const Layout &L, bool f32) {
    constexpr int kFewTiles = 700;
    constexpr int many[kMaxR + 1] = {0, 8, 4, 4, 2, 2, 2, 0, 0};
    constexpr double base[] = {0, 0, 1.5, 1.5, 1.5, 2.0, 2.0}, slope[] = {0, 0, 1.13, 1.95, 2.05, 2.9, 3.4};
    constexpr double kCacheBytes = 256.0 * 1024 * 1024;
    const int most = std::min(kTb2MaxLev, kTb2Halo / L.r);
    int ntx, ntz;
    tiles2d(L, most, &ntx, &ntz);
    if ((long long)ntx * ntz <= kFewTiles) return most;
    const double n = 1e-6 * L.nx * L.nz;
    const int lev = L.r == 4 && f32 && n > 10 ? 3 : many[L.r];
    if (lev == 0 || L.r == 1) return lev;   // (at radius 1 eight levels win everywhere)
    tiles2d(L, lev, &ntx, &ntz);
    const int H = L.r * lev, Hx = (H + 3) & ~3;
    const double covered = 1e-6 * ntx * (4 * kW4 - 2 * Hx) * ntz * (kRows - 2 * H);
    const double rows = 1e-6 * ((L.nx + kTileX - 1) / kTileX * kTileX) * L.nz;
    const bool spills = 1e6 * n * (f32 ? 20 : 12) > kCacheBytes;
    const double levels_us = (base[L.r] + slope[L.r] * covered) * (spills ? 1.1 : 1.0);
    const double one_us = f32 ? (L.r <= 4 ? 5.5 + 2.5 * rows : 6.0 + 2.65 * rows)
                              : (L.r <= 4 ? 5.0 + 1.9 * rows : L.r == 5 ? 5.5 + 2.2 * rows : 4.5 + 2.2 * rows);
    return levels_us <= one_us ? lev : 0;
}

int sample_rows_blocks(int npts, int lpp) { return (npts + kNT / lpp - 1) / (kNT / lpp); }

hipError_t launch_step2d_tb(Step2Args a, Store st, int mode, hipStream_t s) {
    Step2Fn f = nullptr;
    if (mode == kBracket || mode == kImage)
        f = st != Store::F32 ? nullptr
            : mode == kBracket ? pick_r<Store::F32, kBracket>(a.L.r)
                               : pick_r<Store::F32, kImage>(a.L.r);
    else if (mode == kPlain)
        f = st == Store::F32   ? pick_r<Store::F32, kPlain>(a.L.r)
            : st == Store::F16 ? pick_r<Store::F16, kPlain>(a.L.r)
                               : pick_r<Store::BF16, kPlain>(a.L.r);
    if (!f || a.L.ndim != 2 || a.nlev < 1 || a.nlev > kTb2MaxLev || a.nlev * a.L.r > kTb2Halo)
        return hipErrorInvalidValue;
    int ntz;
    tiles2d(a.L, a.nlev, &a.ntx, &ntz);
    hipLaunchKernelGGL(f, dim3(a.ntx * ntz + a.nsamp_blocks), dim3(kNT), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_sample_rows(const SampleRows &smp, Store st, hipStream_t s) {
    const int blocks = smp.nrows * smp.bpr;
    if (blocks <= 0) return hipSuccess;
    switch (st) {
        case Store::F32: hipLaunchKernelGGL(k_sample_rows<Store::F32>, dim3(blocks), dim3(kNT), 0, s, smp); break;
        case Store::F16: hipLaunchKernelGGL(k_sample_rows<Store::F16>, dim3(blocks), dim3(kNT), 0, s, smp); break;
        case Store::BF16: hipLaunchKernelGGL(k_sample_rows<Store::BF16>, dim3(blocks), dim3(kNT), 0, s, smp); break;
    }
    return hipGetLastError();
}

}  // namespace fd

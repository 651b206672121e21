// fd_diffuse2d.hip -- the thesis's benchmark operator (Section 5.1.2): forward
// Euler steps of u_t = nu Lap u in 2D, several levels per launch, by three
// kernels with the same arithmetic (their fields are bitwise equal).
//
// k_diffuse2d_strip, for grids that fill the GPU with strips: one step reads
// and writes each point once (8 B), so beyond a few levels per launch the
// arithmetic is the bound.  A wave works alone: it owns a strip of
// 256 points (a float4 per lane) and marches down a chunk of rows.  Level t
// follows level t - 1 R rows behind: each level keeps its last 2 R + 1 rows in
// registers, takes its z neighbours from there and its x neighbours from the
// lanes beside it (DPP wave shifts, which fold into the additions), so there
// is no LDS, no barrier and no staging.  Recomputed are R T points at either
// end of a strip (rounded to 4) and R T rows at either end of a chunk.
//
// k_diffuse2d_tile, for small and narrow grids, where latency or the lanes of
// a strip are the bound: the scheme of the 2D acoustic levels (fd_step2d.hip),
// a 64 x 64 region staged once and advanced in registers with the neighbours'
// level in LDS.
//
// k_diffuse2d_one, a single level of whole 64 x 64 tiles, where a launch takes
// one level and a strip's halo costs more than it saves: so 16 up to 20 M
// points, single steps of fields beyond the memory-side cache's reach, narrow
// grids at high order.
#include "fd_step3d.h"

#include <algorithm>
#include <utility>

namespace fd {
namespace {

constexpr int kStrip = 256;   // points per wave and row

struct DiffArgs {
    Layout L;
    const float *u;
    float *out;
    float w0;
    float wx[kMaxR + 1];
    float wz[kMaxR + 1];
    int nstrip;       // strips or tiles along x
    int chunk;        // strips: rows per wave
    int nlev;         // levels of this launch
    int out_cached;   // ordinary stores of the new level (small fields), else non-temporal
};

constexpr int kShr1 = 0x138, kShl1 = 0x130;   // DPP: the value of the lane before, after
template <int CTRL>
__device__ inline float shifted(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ inline float4 shifted(const float4 &v) {
    return make_float4(shifted<CTRL>(v.x), shifted<CTRL>(v.y), shifted<CTRL>(v.z), shifted<CTRL>(v.w));
}

// The new level of 4 points: x neighbours xs (the points themselves from
// xs[4 * HQ]), z neighbours zp(j) and zm(j) at distance j.  The order of the
// sums decides the error: a nearly constant field rounds alike everywhere, so
// a step's rounding adds up over the steps.  One chain of fused multiply-adds
// with the centre last (5 instead of 6 operations at radius 1, 34 instead of
// 41 at radius 8) measured 1e-5 against 7e-7 here after 200 steps at so 16.
template <int R, int HQ, typename FP, typename FM>
__device__ inline void diffuse4(const DiffArgs &a, const float *xs, FP zp, FM zm, float un[4]) {
#pragma unroll
    for (int j = 1; j <= R; ++j) {
        const float4 p = zp(j), m = zm(j);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float xsum = xs[4 * HQ + k + j] + xs[4 * HQ + k - j];
            const float acc = __builtin_fmaf(a.wx[j], xsum, a.wz[j] * (comp(p, k) + comp(m, k)));
            un[k] = j == 1 ? __builtin_fmaf(a.w0, xs[4 * HQ + k], acc) : un[k] + acc;
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) un[k] += xs[4 * HQ + k];
}
__device__ inline void put4(float *xs, const float4 &v) {
    xs[0] = v.x;
    xs[1] = v.y;
    xs[2] = v.z;
    xs[3] = v.w;
}

constexpr int kW4 = 16, kRows = 64, kK = 2;   // tile: staged float4 columns, rows; rows per lane
constexpr int kNT = kW4 * kRows / kK;         // lanes of a tile's workgroup

template <int R>
__global__ __launch_bounds__(kNT) void k_diffuse2d_tile(const DiffArgs a) {
    constexpr int HX4 = (R + 3) / 4;
    constexpr int kBuf = (kRows + 2 * R) * kW4 + 2 * HX4;
    __shared__ float4 lds[2][kBuf];
    const Layout L = a.L;
    const int H = R * a.nlev, Hx = (H + 3) & ~3;
    const int t0 = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    const int x0 = (t0 % a.nstrip) * (4 * kW4 - 2 * Hx) - Hx, z0 = (t0 / a.nstrip) * (kRows - 2 * H) - H;
    const int lane = (int)threadIdx.x;
    const int c = lane % kW4, row0 = (lane / kW4) * kK;
    const int x = x0 + 4 * c;
    const int own = HX4 + (R + row0) * kW4 + c;
    const long long zcol = L.offset((L.nx + 3) & ~3, 0, 0);   // zero
    float4 u[kK];
    long long off[kK];
    bool in[kK], mine[kK];
#pragma unroll
    for (int k = 0; k < kK; ++k) {
        const int z = z0 + row0 + k;
        in[k] = x >= 0 && x < L.nx && z >= 0 && z < L.nz;
        off[k] = in[k] ? L.offset(x, 0, z) : zcol;
        u[k] = *reinterpret_cast<const float4 *>(a.u + off[k]);
        mine[k] = in[k] && c >= Hx / 4 && c < kW4 - Hx / 4 && row0 + k >= H && row0 + k < kRows - H;
        lds[0][own + k * kW4] = u[k];
    }
    __syncthreads();
    const bool edge = x0 < 0 || x0 + 4 * kW4 > L.nx || z0 < 0 || z0 + kRows > L.nz;
    const int wrow = __builtin_amdgcn_readfirstlane(row0);   // first row of the wave
    for (int t = 0; t < a.nlev; ++t) {
        const float4 *buf = lds[t & 1];
        float4 *nxt = lds[(t & 1) ^ 1];
        const int need = R * (t + 1);
        if (wrow + 64 / kW4 * kK > need && wrow < kRows - need) {
            float4 col[kK + 2 * R];   // the lane's column, R rows beyond its own on both sides
#pragma unroll
            for (int j = 0; j < kK + 2 * R; ++j)
                col[j] = j >= R && j < R + kK ? u[j - R] : buf[own + (j - R) * kW4];
#pragma unroll
            for (int k = 0; k < kK; ++k) {
                float xs[4 * (2 * HX4 + 1)], un[4];
#pragma unroll
                for (int q = -HX4; q <= HX4; ++q) put4(xs + 4 * (q + HX4), q == 0 ? u[k] : buf[own + k * kW4 + q]);
                diffuse4<R, HX4>(a, xs, [&](int j) { return col[k + R + j]; }, [&](int j) { return col[k + R - j]; },
                                 un);
                if (edge) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) un[i] = in[k] && x + i < L.nx ? un[i] : 0.f;
                }
                u[k] = make_float4(un[0], un[1], un[2], un[3]);
                nxt[own + k * kW4] = u[k];
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kK; ++k)
        if (mine[k]) *reinterpret_cast<float4 *>(a.out + off[k]) = u[k];
}

// One level: a 64 x 64 tile staged with its R halo; each lane updates 4 points
// in each of 4 rows.  Rows are written as whole cache lines, which a strip
// (256 points less its halo) cannot: where one level per launch streams from
// HBM and the arithmetic is short, that decides.
// WAVES bounds the waves per SIMD the compiler plans registers for.
template <int R, int WAVES = 8>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(1, WAVES))) void k_diffuse2d_one(const DiffArgs a) {
    constexpr int HX4 = (R + 3) / 4;
    constexpr int W4 = kTileX / 4 + 2 * HX4;
    constexpr int LH = kTile2Z + 2 * R;
    __shared__ float4 lds[LH * W4];
    const Layout L = a.L;
    const int t = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    const int x0 = (t % a.nstrip) * kTileX, z0 = (t / a.nstrip) * kTile2Z;
    const int lane = (int)threadIdx.x;
    const long long zcol = L.offset((L.nx + 3) & ~3, 0, 0);   // zero
    for (int i = lane; i < LH * W4; i += kBlock) {
        const int lr = i / W4, c = i - lr * W4;
        const int gz = z0 - R + lr, gx = x0 - 4 * HX4 + 4 * c;
        const bool ok = gz >= 0 && gz < L.nz && gx >= 0 && gx < L.nx;
        lds[i] = *reinterpret_cast<const float4 *>(a.u + (ok ? L.offset(gx, 0, gz) : zcol));
    }
    __syncthreads();
    const int tx = lane % (kTileX / 4), tz = lane / (kTileX / 4);
    const int x = x0 + 4 * tx;
    if (x >= L.nx) return;
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
        const int z = z0 + tz * 4 + rr;
        if (z >= L.nz) break;
        const float4 *row = lds + (R + tz * 4 + rr) * W4 + HX4 + tx;
        float xs[4 * (2 * HX4 + 1)], un[4];
#pragma unroll
        for (int c = -HX4; c <= HX4; ++c) put4(xs + 4 * (c + HX4), row[c]);
        diffuse4<R, HX4>(a, xs, [&](int j) { return row[j * W4]; }, [&](int j) { return row[-j * W4]; }, un);
        if (x + 4 > L.nx) {   // (the cells past nx of a row's last group must be zero)
#pragma unroll
            for (int i = 1; i < 4; ++i)
                if (x + i >= L.nx) un[i] = 0.f;
        }
        float *o = a.out + L.offset(x, 0, z);
        const float4 v = make_float4(un[0], un[1], un[2], un[3]);
        if (a.out_cached)
            *reinterpret_cast<float4 *>(o) = v;
        else
            st4nt_f32(o, v);
    }
}

template <int R, int T>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void k_diffuse2d_strip(const DiffArgs a) {
    // Queues do not move: a group of U rows is unrolled, and logical entry k of
    // a queue (0 = oldest of the 2 R + 1 rows) lives in slot (k + I) % NQ at row
    // I of the group.  D rows of level 0 are in flight.
    constexpr int U = R == 1 ? 6 : (2 * R + 3) / 3 * 3;
    constexpr int NQ = R == 1 ? 3 : U;
    constexpr int D = R <= 2 ? 6 : 3;
    constexpr int H = R * T, HX = (H + 3) & ~3;
    static_assert(U % NQ == 0 && U % D == 0, "queues and prefetch must come round with the group");
    const Layout L = a.L;
    const int w = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    const int sx = w % a.nstrip, sz = w / a.nstrip;
    const int x0 = sx * (kStrip - 2 * HX) - HX;
    const int c0 = sz * a.chunk, c1 = min(c0 + a.chunk, L.nz);
    const int zs = c0 - H, nit = c1 - c0 + 2 * H;   // rows of level 0
    const int lane = (int)threadIdx.x;
    const int x = x0 + 4 * lane;
    const int off = 16 * lane;
    const int ld = x >= 0 && x < L.nx ? off : kOob;
    const int st = x < L.nx && 4 * lane >= HX && 4 * lane < kStrip - HX ? off : kOob;
    const float *src = a.u + L.offset(x0, 0, 0);
    float *dst = a.out + L.offset(x0, 0, 0);
    const long long pitch = L.pitch;

    float4 q[T][NQ], pre[D];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int k = 0; k < NQ; ++k) q[t][k] = make_float4(0.f, 0.f, 0.f, 0.f);
    auto load = [&](int i) {   // row zs + i of level 0, zero outside the grid
        const int z = zs + i;
        const bool in = z >= 0 && z < L.nz;
        return bufld4<Store::F32, 0>(src + (in ? z : 0) * pitch, in ? ld : kOob);
    };
#pragma unroll
    for (int i = 0; i < D; ++i) pre[i] = load(i);

    // iteration i = group start + I: row zs + i of level 0 enters, level t
    // computes row zs + i - t R, the last level's row is stored.  CHECK: some
    // levels have no complete neighbourhood yet; EDGE: points outside the grid
    // are forced to zero.
    auto body = [&](auto idx, auto check, auto edge, int i) __attribute__((always_inline)) {
        constexpr int I = decltype(idx)::value;
        float4 nw = pre[I % D];
        pre[I % D] = load(min(i + D, nit - 1));
        bool full = true;
        static_for<1, T + 1>([&](auto tt) __attribute__((always_inline)) {
            constexpr int t = decltype(tt)::value;
            float4 *lv = q[t - 1];
#define LV(k) lv[((k) + I) % NQ]
            if (full) LV(2 * R) = nw;
            if (decltype(check)::value && i < 2 * t * R) full = false;
            if (full) {
                const float4 c = LV(R);
                const float4 l1 = shifted<kShr1>(c), r1 = shifted<kShl1>(c);
                constexpr int HQ = R > 4 ? 2 : 1;
                float xs[4 * (2 * HQ + 1)], un[4];
                if constexpr (HQ == 2) {
                    put4(xs, shifted<kShr1>(l1));
                    put4(xs + 16, shifted<kShl1>(r1));
                }
                put4(xs + 4 * HQ - 4, l1);
                put4(xs + 4 * HQ, c);
                put4(xs + 4 * HQ + 4, r1);
                diffuse4<R, HQ>(a, xs, [&](int j) { return LV(R + j); }, [&](int j) { return LV(R - j); }, un);
                const int z = zs + i - t * R;
                const bool zin = z >= 0 && z < L.nz;
                if constexpr (decltype(edge)::value) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) un[k] = zin && x + k >= 0 && x + k < L.nx ? un[k] : 0.f;
                }
                nw = make_float4(un[0], un[1], un[2], un[3]);
            }
#undef LV
        });
        if (full) {
            float *row = dst + (zs + i - H) * pitch;
            if (a.out_cached)
                bufst4<Store::F32, 0>(row, st, nw);
            else
                bufst4<Store::F32, kNt>(row, st, nw);
        }
        return i + 1 < nit;
    };
    auto group = [&](auto check, auto edge, int i) __attribute__((always_inline)) {
        return all_of_seq(std::make_integer_sequence<int, U>{}, [&](auto I) __attribute__((always_inline)) {
            return body(I, check, edge, i + decltype(I)::value);
        });
    };
    using Yes = std::true_type;
    using No = std::false_type;
    const bool at_edge = x0 < 0 || x0 + kStrip > L.nx || zs < 0 || c1 + H > L.nz;
    int i = 0;
    if (at_edge) {
        while (group(Yes{}, Yes{}, i)) i += U;
    } else {
        bool more = true;
        for (; more && i < 2 * H; i += U) more = group(Yes{}, No{}, i);
        while (more) {
            more = group(No{}, No{}, i);
            i += U;
        }
    }
}

using DiffFn = void (*)(const DiffArgs);

template <int R>
DiffFn pick(int levels) {
    switch (levels) {
        case 1: return k_diffuse2d_strip<R, 1>;
        case 2: return k_diffuse2d_strip<R, 2>;
        case 4:
            if constexpr (4 * R <= kDiffHalo) return k_diffuse2d_strip<R, 4>;
            return nullptr;
        case 8:
            if constexpr (8 * R <= kDiffHalo) return k_diffuse2d_strip<R, 8>;
            return nullptr;
    }
    return nullptr;
}

DiffFn strip_kernel(int r, int levels) {
    switch (r) {
        case 1: return pick<1>(levels);
        case 2: return pick<2>(levels);
        case 3: return pick<3>(levels);
        case 4: return pick<4>(levels);
        case 5: return pick<5>(levels);
        case 6: return pick<6>(levels);
        case 7: return pick<7>(levels);
        case 8: return pick<8>(levels);
    }
    return nullptr;
}

DiffFn tile_kernel(int r) {
    switch (r) {
        case 1: return k_diffuse2d_tile<1>;
        case 2: return k_diffuse2d_tile<2>;
        case 3: return k_diffuse2d_tile<3>;
        case 4: return k_diffuse2d_tile<4>;
        case 5: return k_diffuse2d_tile<5>;
        case 6: return k_diffuse2d_tile<6>;
        case 7: return k_diffuse2d_tile<7>;
        case 8: return k_diffuse2d_tile<8>;
    }
    return nullptr;
}

DiffFn one_kernel(int r, bool cached) {
    switch (r) {
        case 1: return k_diffuse2d_one<1>;
        case 2: return k_diffuse2d_one<2>;
        case 3: return k_diffuse2d_one<3>;
        case 4: return k_diffuse2d_one<4>;
        case 5: return k_diffuse2d_one<5>;
        case 6: return k_diffuse2d_one<6>;
        case 7: return k_diffuse2d_one<7>;
        // (five waves' registers hide the reads of a cached field better, 2500^2 15.9
        // -> 15.3 us, and lose 12 % on 10000^2)
        case 8: return cached ? k_diffuse2d_one<8, 5> : k_diffuse2d_one<8>;
    }
    return nullptr;
}

// Which kernel and how many levels, measured per step at every order, level
// count and kernel on 203 x 141, 500^2, 1000^2, 10000 x 300, 300 x 10000, 2500^2,
// 4000^2 and 10000^2 (float32, us; the former kernels, 64 x 64 tiles in LDS,
// last):
//   tile / strip at their best   so 2          so 4          so 8          so 12
//   500^2                        0.73 / 2.05   0.88 / 2.99   1.47 / 4.60   2.44 / 6.14   (2.5 3.0 4.7 5.9)
//   300 x 10000                  2.02 / 3.01   3.06 / 4.53   5.10 / 6.80   7.78 / 9.26   (4.6 5.3 7.7 9.8)
//   2500^2                       3.28 / 3.75   4.95 / 5.71   8.27 / 8.65   14.1 / 11.4   (7.3 8.4 12.4 15.7)
//   10000^2                      46.4 / 33.6   74.3 / 52.0   128 / 84.8    213 / 110     (85 97 143 174)
// The strips win once they fill the GPU: above 7 M points up to radius 4, 4 M
// at radius 5 and 6, 2 M beyond (where radius 8 takes single levels up to 20 M,
// see use_one); single levels above 4 M up to radius 3, 6.5 M at radius 4
// (2500^2 tiles 13.2, strips 13.4; 2600^2 14.7, 13.9).
bool use_tiles(const Layout &L, int most) {
    const long long n = (long long)L.nx * L.nz;
    if (most == 1 && L.r <= 4) return n <= (L.r <= 3 ? 4000000 : 6500000);
    return n <= (L.r <= 4 ? 7000000 : L.r <= 6 ? 4000000 : 2000000);
}

// Tiles: as many levels as the halo allows while every CU has a few tiles at
// most (a launch is then mostly a fixed latency), else the level count beyond
// which the recomputed ring costs more than the launches saved.
void tile_shape(const Layout &L, int lev, int *ntx, int *ntz) {
    const int H = L.r * lev, Hx = (H + 3) & ~3;
    const int tx = 4 * kW4 - 2 * Hx, tz = kRows - 2 * H;
    *ntx = (L.nx + tx - 1) / tx;
    *ntz = (L.nz + tz - 1) / tz;
}
int tile_levels(const Layout &L) {
    constexpr int kFewTiles = 1100, kMostLevels = 8;
    constexpr int many[kMaxR + 1] = {0, 8, 4, 4, 2, 2, 2, 1, 1};
    const int most = std::min(kMostLevels, kDiffHalo / L.r);
    int ntx, ntz;
    tile_shape(L, most, &ntx, &ntz);
    return (long long)ntx * ntz <= kFewTiles ? most : many[L.r];
}

// Strips: one round of two waves per SIMD (three or four measured no faster on
// the largest grids, up to 30 % slower on 2500^2, as each wave recomputes 2 R T
// rows; but a single level at radius 1 or 2 recomputes little and waits on
// memory: 16384 waves, 4000^2 so 2 / 4 21.3 / 22.5 -> 20.2 / 20.6 us).  With C rows per wave, T levels pay while C is large against that:
// measured, C >= R T for two levels, about (R T)^2 / 6.4 for more; radius 8
// takes two only beyond the memory-side cache's reach (6500^2 68 us a step
// against 79; 4000^2 31.0 against 30.5, 5000^2 44.1 against 41.6).
constexpr int kWaves = 2048, kMinRows = 8;
void strip_shape(const Layout &L, int lev, int *nstrip, int *chunk) {
    const int HX = (L.r * lev + 3) & ~3;
    *nstrip = (L.nx + kStrip - 2 * HX - 1) / (kStrip - 2 * HX);
    const int waves = lev == 1 && L.r <= 2 ? 8 * kWaves : kWaves;
    const int chunks = std::max(1, std::min(waves / *nstrip, L.nz / kMinRows));
    *chunk = (L.nz + chunks - 1) / chunks;
}
int strip_levels(const Layout &L, int most, bool cached) {
    for (int lev = 8; lev > 1; lev /= 2) {
        const long long h = (long long)L.r * lev;
        if (lev > most || h > kDiffHalo || (L.r == 8 && cached)) continue;
        int nstrip, chunk;
        strip_shape(L, lev, &nstrip, &chunk);
        if (lev == 2 ? chunk >= h : 64 * (long long)chunk >= 10 * h * h) return lev;
    }
    return 1;
}

// One level per launch (asked for, the last of a count, or the choice at radius
// 8).  Measured (us):
//                       so 2          so 4          so 8   so 16
//   10000^2, strips       176 (162)     177 (163)     172    177     (16384 waves)
//            this kernel  150           151           158    173
//   5700^2,  strips       55.7          57.8          --     67.3
//            this kernel  54.9          55.9          --     68.4
//   2500^2,  tiles        10.2          10.6          11.6   19.6
//            strips       -- (9.2)      -- (9.6)      --     15.5
//            this kernel  10.0          10.4          11.8   15.3
//   3000^2,  strips       12.5 (12.0)   14.0 (12.3)   15.3   20.4
//            this kernel  13.4          13.8          15.6   18.8
// So: fields beyond the memory-side cache's reach take this kernel, up to
// radius 3 from 31 M points on (at radius 4 5700^2 measured 59.7 against 60.9 on
// one GPU and 50.4 against 47.9 on another), and at radius 8 where the strips' 2 R recomputed rows weigh, up to 20 M points
// (5000^2 41.2 by strips, 43.3).
bool use_one(const Layout &L, bool cached) {
    const long long n = (long long)L.nx * L.nz;
    return !cached || (L.r <= 3 && n > 31000000) || (L.r == 8 && n <= 20000000);
}

// Grids that leave many of a strip's lanes outside take the other kernels
// however many points they have: tiles up to radius 5, single levels of whole
// tiles beyond (there a tile's two levels stage twice what they write), the
// last also below the strips' line on grids of less than a third of a strip.
// Measured (us per step, strips / tiles / single levels): 8 x 1000000 so 2 76 /
// 27 / 63, so 8 165 / 56, so 16 292 / 129 / 110; 64 x 125000 so 4 16.0 / 9.4; 100
// x 160000 so 10 37.6 / 32.5, so 12 43.5 / 40.2 / 35.5; 260 x 61538 so 8 25.5 /
// 21.4, so 12 34.9 / 36.2 / 32.2; 500 x 10000 so 12 13.1 / 12.6 / 12.0; at 300 x
// 26666 so 14 strips win again, 21.8 / 22.5 / 22.1.  Asked for one level, tiles
// beyond the memory-side cache's reach (8 x 1000000 so 2 71.6, single levels
// 62.7) and strips used to less than 0.6 up to radius 4 (300 x 30000 so 8 19.4,
// 18.0) give way to whole tiles as well.
double least_lanes(int r) { return r <= 5 ? 0.52 : r == 6 ? 0.66 : r == 7 ? 0.55 : 0.60; }

}  // namespace

hipError_t launch_diffuse2d(const Layout &L, const float *u, float *out, float w0, const float *wx,
                            const float *wz, int most, int *levels, hipStream_t s) {
    if (L.ndim != 2 || L.r < 1 || L.r > kMaxR || most < 1) return hipErrorInvalidValue;
    DiffArgs a{};
    a.L = L;
    a.u = u;
    a.out = out;
    a.w0 = w0;
    for (int j = 0; j <= kMaxR; ++j) {
        a.wx[j] = wx[j];
        a.wz[j] = wz[j];
    }
    a.out_cached = (size_t)L.elems * sizeof(float) <= kCachedField;
    bool tiles = use_tiles(L, most), one = false;
    a.nlev = strip_levels(L, most, a.out_cached);
    strip_shape(L, a.nlev, &a.nstrip, &a.chunk);
    const double lanes = (double)L.nx / ((double)a.nstrip * kStrip);
    if (lanes < least_lanes(L.r)) {
        if (L.r >= 6) one = !tiles || (lanes < 0.3 && (long long)L.nx * L.nz > 2000000);
        else one = most == 1 && !a.out_cached;
        tiles = !one;
    } else if (!tiles) {
        one = a.nlev == 1 && (use_one(L, a.out_cached) || (L.r <= 4 && lanes < 0.6));
    }
    if (one) {
        a.nlev = 1;
        a.nstrip = (L.nx + kTileX - 1) / kTileX;
        hipLaunchKernelGGL(one_kernel(L.r, a.out_cached), dim3(a.nstrip * ((L.nz + kTile2Z - 1) / kTile2Z)), dim3(kBlock), 0, s, a);
    } else if (tiles) {
        int ntz;
        a.nlev = std::min(most, tile_levels(L));
        tile_shape(L, a.nlev, &a.nstrip, &ntz);
        hipLaunchKernelGGL(tile_kernel(L.r), dim3(a.nstrip * ntz), dim3(kNT), 0, s, a);
    } else {
        hipLaunchKernelGGL(strip_kernel(L.r, a.nlev), dim3(a.nstrip * ((L.nz + a.chunk - 1) / a.chunk)), dim3(64), 0,
                           s, a);
    }
    *levels = a.nlev;
    return hipGetLastError();
}

}  // namespace fd

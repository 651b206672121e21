// fd_kernels.hip -- gfx950 kernels of libfd.
//
// The hot loop is the per-step space loop of an explicit finite-difference
// stepper (the thesis launches one data-parallel loop per time step from a
// host time loop, Section 3.3.3 "Parallel loop invocation"); here one launch
// of k_step3d / k_step2d performs the whole step (several 2D steps per launch
// are in fd_step2d.hip, the diffusion operator is in fd_diffuse2d.hip):
//
//   lap  = w0 u + sum_j wx_j (u_{x+j} + u_{x-j}) + wy_j (..) + wz_j (..)
//   s    = sigma dt / 2                     (per-axis tables, 0 off the layer)
//   unew = (2u - (1 - s) uprev + p (lap + src)) / (1 + s),  p = dt^2 v^2
//
// with the point-source term `src` added by the thread that owns the point
// and the receiver sampling of the centre field done by extra workgroups of
// the same launch.  All weights are precomputed on the host (no division in
// the inner loop: the lesson of the aggressive-DSE kernel of Section 5.1.5).
//
// 3D: 2.5D blocking.  A workgroup owns a 64 x 16 or a 32 x 32 xy tile and
// marches a chunk of z planes.  Each lane keeps 4 consecutive x points and a
// register queue of the 2r+1 z values of its column; the current xy plane (tile + r halo) is
// staged through LDS (double-buffered, one barrier per plane) for the x and y
// neighbours.  Loads of plane z+1 are issued before plane z is computed.
// Arithmetic is FP32 whatever the storage type.  No MFMA: the update is a
// star stencil, not a contraction, and is bound by HBM bandwidth.  The 3D
// step's device code is in fd_step3d.h, its instantiations in the
// fd_step3d_*.hip units (one per storage type and form).
#include "fd_step3d.h"

#include <stdint.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

// Device scratch of the allocation-free diffusion entry point: a fixed
// array in the code object, one copy per GPU, reached from host code only
// through the address hipGetSymbolAddress returns for the current device
// (see fd::static_scratch); the name itself is not a device address there.
static __device__ __align__(256) unsigned char scratch[fd::kStaticScratchBytes];

namespace fd {
namespace {

// ------------------------------------------------------ 3D two-level step
// Temporal blocking of the 2.5D march (the wave-front tiling of Section
// 2.3.1 and the tiling of Section 2.2, done in registers and LDS): from u^n
// and u^{n-1} a workgroup computes level 1, u^{n+1}, on its 64 x 16 tile
// grown by a ring of R points (the ring belongs to the neighbour tiles and
// is recomputed here, so that no workgroup waits for another), and level 2,
// u^{n+2}, on its tile, R planes behind level 1 in the z march.  It writes
// u^{n+1} and u^{n+2} of its tile: per point and two steps HBM carries u^n,
// u^{n-1} and p in and two fields out, 10 bytes per point-step instead of
// 16.  The outputs go to a second pair of fields (u^n and u^{n-1} are read
// as the neighbours' ring until the launch ends).  Each level is the same
// sequence of float32 operations as the one-step kernel's, so two levels
// here give bitwise the fields of two one-step launches.
template <int R>
struct T2Shape {
    static constexpr int TW = 16, TY = 16;                   // tile: 16 float4 columns x 16 rows
    static constexpr int HX4 = (R + 3) / 4;                  // float4 columns of an R-point ring in x
    static constexpr int W1 = TW + 2 * HX4, H1 = TY + 2 * R;    // level-1 region E1 (float4 x rows)
    static constexpr int W2 = W1 + 2 * HX4, H2 = H1 + 2 * R;    // staged u^n plane E2
    static constexpr int N1 = W1 * H1, N2 = W2 * H2;
    static constexpr int NR1 = N1 - TW * TY;                 // ring groups of E1
    static constexpr int NR1L = TY * 2 * HX4;                // ... of which in the tile's rows
    static constexpr int NS = 1 + (NR1 + kBlock - 1) / kBlock;  // level-1 groups per lane (0: own)
    static constexpr int NR2 = N2 - N1;                      // ring groups of E2 (u^n only)
    static constexpr int NR2L = H1 * 2 * HX4;
    static constexpr int HP2 = (NR2 + kBlock - 1) / kBlock;
    static constexpr int NQ = 2 * R + 1;
    static constexpr int kMaxPl = kMaxChunk + 2 * R;         // level-1 planes of a chunk
    // LDS, in float4 (at radius 4 just under the 80 KB that lets two
    // workgroups share a CU); the level-1 source terms of a plane are
    // scattered into the staging buffer the next plane will use, idle then
    static constexpr int kU = 0;                             // [2][N2] staged u^n planes
    static constexpr int kV = kU + 2 * N2;                   // [R + 1][N1] ring of u^{n+1} planes
    static constexpr int kP = kV + (R + 1) * N1;             // [R + 1][NR2] parked E2 ring of u^n
    static constexpr int kS2 = kP + (R + 1) * NR2;           // [kBlock] level-2 source terms
    static constexpr int kDz = kS2 + kBlock;                 // float [kMaxPl] z damping of level-1 planes
    static constexpr int kPp = kDz + kMaxPl / 4;             // int [kMaxPl + 1] source plane pointers
    static constexpr int kSize = kPp + (kMaxPl + 1 + 3) / 4;
};

// Ring group h of a region W x H (float4 x rows) around an inner block of
// IW x IH starting at (HX, RY): the RY rows above (full width), then HX
// columns left and right of each inner row, then the RY rows below.
template <int W, int H, int IW, int IH, int HX, int RY>
__device__ inline void ring_pos(int h, int &cx, int &cy) {
    if (h < RY * W) {
        cy = h / W;
        cx = h - cy * W;
    } else if (h < RY * W + IH * 2 * HX) {
        const int j = h - RY * W;
        const int row = j / (2 * HX), c = j - row * (2 * HX);
        cy = RY + row;
        cx = c < HX ? c : IW + c;
    } else {
        const int j = h - RY * W - IH * 2 * HX;
        cy = RY + IH + j / W;
        cx = j - (j / W) * W;
    }
}

template <int R>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2))) void k_step3d_t2(const StepArgs a) {
    using K = T2Shape<R>;
    constexpr int TW = K::TW, TY = K::TY, HX4 = K::HX4, W1 = K::W1, W2 = K::W2, N1 = K::N1, N2 = K::N2;
    constexpr int NS = K::NS, HP2 = K::HP2, NQ = K::NQ;
    __shared__ float4 smem[K::kSize];
    const int ntile = (int)gridDim.x - a.nsamp_blocks - a.nsamp_blocks2;
    if ((int)blockIdx.x >= ntile) {
        const int b = (int)blockIdx.x - ntile;
        if (b < a.nsamp_blocks)
            sample_block<Store::F32>(a.smp, a.u, b);
        else
            sample_block<Store::F32>(a.smp2, a.prev, b - a.nsamp_blocks);
        return;
    }
    const int t = xcd_remap((int)blockIdx.x, ntile);
    const int tiles = a.ntx * a.nty;
    const int tid = t % tiles, bz = t / tiles;
    const int x0 = (tid % a.ntx) * 4 * TW, y0 = (tid / a.ntx) * TY;
    const Layout L = a.L;
    const int c0 = bz * a.zchunk, c1 = min(c0 + a.zchunk, L.nz);
    const int zl0 = c0 - R;                  // level-1 plane of the first iteration
    const int npl = c1 - c0 + 2 * R;         // iterations: level-1 planes [c0 - R, c1 + R)
    const int lane = (int)threadIdx.x;
    const long long plane = L.plane;
    const long long zcol = L.offset((L.nx + 3) & ~3, 0, 0);   // zero in every row of every plane
    const float *__restrict__ U = (const float *)a.u;
    const float *Pv = (const float *)a.prev;
    const float *__restrict__ Pp = a.p;
    float *O1 = (float *)a.out;
    float *O2 = (float *)a.out2;

    float4 *stg = smem + K::kU;
    float4 *ring = smem + K::kV;
    float4 *park = smem + K::kP;
    float4 *s_src2 = smem + K::kS2;
    float *s_dz = reinterpret_cast<float *>(smem + K::kDz);
    int *s_pp = reinterpret_cast<int *>(smem + K::kPp);
    // per-plane tables of the chunk's level-1 planes (z damping; source plane
    // pointers, which give no sources outside the grid)
    const int *tile_pp = a.inj.plane_ptr + (long long)tid * (L.nz + 1);
    for (int i = lane; i <= npl; i += kBlock) {
        const int z = zl0 + i;
        if (i < npl) s_dz[i] = (z >= 0 && z < L.nz) ? a.damp[L.nx + L.ny + z] : 0.f;
        s_pp[i] = a.inj.vals ? tile_pp[min(max(z, 0), L.nz)] : 0;
    }
    s_src2[lane] = make_float4(0.f, 0.f, 0.f, 0.f);

    // level-1 groups of this lane: slot 0 its own tile group, slots 1.. ring
    // groups of E1; grid coordinates, E1 and E2 indices, validity
    const int tx = lane % TW, ty = lane / TW;
    int e1i[NS], e2i[NS], gxs[NS];
    bool in1[NS];
    long long off[NS];
    float sxy[NS][4];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        int cx = HX4 + tx, cy = R + ty;
        bool used = true;
        if (k > 0) {
            const int h = lane + (k - 1) * kBlock;
            used = h < K::NR1;
            ring_pos<W1, K::H1, TW, TY, HX4, R>(used ? h : 0, cx, cy);
        }
        const int gx = x0 - 4 * HX4 + 4 * cx, gy = y0 - R + cy;
        in1[k] = used && gx >= 0 && gx < L.nx && gy >= 0 && gy < L.ny;
        e1i[k] = used ? cy * W1 + cx : -1;
        e2i[k] = (cy + R) * W2 + cx + HX4;
        gxs[k] = gx;
        off[k] = in1[k] ? L.offset(gx, gy, 0) : zcol;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            sxy[k][i] = in1[k] ? a.damp[min(gx + i, L.nx - 1)] + a.damp[L.nx + gy] : 0.f;
    }
    // the E2 ring of u^n (staged for level 1's x and y neighbours only)
    int h2i[HP2];
    long long hoff[HP2];
#pragma unroll
    for (int k = 0; k < HP2; ++k) {
        const int h = lane + k * kBlock;
        int cx = 0, cy = 0;
        ring_pos<W2, K::H2, W1, K::H1, HX4, R>(h < K::NR2 ? h : 0, cx, cy);
        const int gx = x0 - 8 * HX4 + 4 * cx, gy = y0 - 2 * R + cy;
        const bool ok = h < K::NR2 && gx >= 0 && gx < L.nx && gy >= 0 && gy < L.ny;
        h2i[k] = h < K::NR2 ? cy * W2 + cx : -1;
        hoff[k] = ok ? L.offset(gx, gy, 0) : zcol;
    }
    const bool act = in1[0];                      // the lane's tile group is inside the grid
    const int nvalid = L.nx - gxs[0];

    auto zclamp = [&](int z) { return min(max(z, -R), L.nz + R - 1); };
    // z queues: q[k][j] = u^n of slot k at plane zl - R + j; w[j] = u^{n+1}
    // of slot 0 at plane zl - 2R + j; pq[j] = p of slot 0 at plane zl - R + j
    float4 q[NS][NQ], w[NQ], pq[R + 1];
#pragma unroll
    for (int k = 0; k < NS; ++k)
#pragma unroll
        for (int j = 0; j < 2 * R; ++j) q[k][j] = Elem<Store::F32>::ld4(U + off[k] + (long long)zclamp(c0 - 2 * R + j) * plane);
#pragma unroll
    for (int j = 0; j < NQ; ++j) w[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    // The E2 ring of plane z belongs to neighbour tiles, which fetch plane z
    // as their queue front R planes before this tile stages it; it is loaded
    // with this tile's own fronts (plane zl + R), when the neighbours' fetch
    // can serve it from L2, and parked in LDS slot (iteration + R) mod (R+1)
    // until staged.  The first R planes are parked here.
#pragma unroll
    for (int j = 0; j < R; ++j)
#pragma unroll
        for (int k = 0; k < HP2; ++k)
            if (h2i[k] >= 0)
                park[j * K::NR2 + k * kBlock + lane] = Elem<Store::F32>::ld4(U + hoff[k] + (long long)zclamp(zl0 + j) * plane);
#pragma unroll
    for (int j = 0; j <= R; ++j) pq[j] = make_float4(0.f, 0.f, 0.f, 0.f);

    struct Pre {
        float4 front[NS], mv[NS], pv[NS], h2[HP2];
    };
    // u^{n-1} and p use ordinary loads: the ring's values are read by the
    // neighbour tiles in the same plane step, and their fetch should find
    // the line in L2 (non-temporal loads here doubled the bytes read).
    auto issue = [&](Pre &r, int it) __attribute__((always_inline)) {
        it = min(it, npl - 1);   // past the chunk: a harmless in-bounds reload
        const int zl = zl0 + it;
        const long long fo = (long long)zclamp(zl + R) * plane, zo = (long long)zclamp(zl) * plane;
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            r.front[k] = Elem<Store::F32>::ld4(U + off[k] + fo);
            r.mv[k] = Elem<Store::F32>::ld4(Pv + off[k] + zo);
            r.pv[k] = Elem<Store::F32>::ld4(Pp + off[k] + zo);
        }
#pragma unroll
        for (int k = 0; k < HP2; ++k) r.h2[k] = Elem<Store::F32>::ld4(U + hoff[k] + fo);
    };

    // The Laplacian of one group: x neighbours from an LDS row (the group's
    // own value xc in the middle), y neighbours j rows up and down, z from
    // the queue; the same fused multiply-adds in the same order as the
    // one-step kernel.
    auto laplace = [&](const float4 *row, int rowpitch, const float4 &xc, const float4 *zq, float lap[4])
        __attribute__((always_inline)) {
        float xs[4 * (2 * HX4 + 1)];
#pragma unroll
        for (int c = -HX4; c <= HX4; ++c) {
            const float4 v = (c == 0) ? xc : row[c];
            xs[4 * (c + HX4) + 0] = v.x;
            xs[4 * (c + HX4) + 1] = v.y;
            xs[4 * (c + HX4) + 2] = v.z;
            xs[4 * (c + HX4) + 3] = v.w;
        }
#pragma unroll
        for (int j = 1; j <= R; ++j) {
            const float4 yp = row[j * rowpitch], ym = row[-j * rowpitch];
            const float4 zp = zq[R + j], zm = zq[R - j];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float xsum = xs[4 * HX4 + i + j] + xs[4 * HX4 + i - j];
                lap[i] = j == 1 ? a.wx[1] * xsum : __builtin_fmaf(a.wx[j], xsum, lap[i]);
                lap[i] = __builtin_fmaf(a.wy[j], comp(yp, i) + comp(ym, i), lap[i]);
                lap[i] = __builtin_fmaf(a.wz[j], comp(zp, i) + comp(zm, i), lap[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) lap[i] = __builtin_fmaf(a.w0, xs[4 * HX4 + i], lap[i]);
    };

    auto body = [&](int it, const Pre &cur, Pre &nxt) __attribute__((always_inline)) {
        const int zl = zl0 + it;
        float4 *st = stg + (it & 1) * N2;
        float *s_src1 = reinterpret_cast<float *>(stg + ((it + 1) & 1) * N2);   // idle this plane
        float4 *park_w = park + ((it + R) % (R + 1)) * K::NR2 + lane;
        const float4 *park_r = park + (it % (R + 1)) * K::NR2 + lane;
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            q[k][2 * R] = cur.front[k];
            if (e1i[k] >= 0) st[e2i[k]] = q[k][R];
        }
#pragma unroll
        for (int k = 0; k < HP2; ++k) {
            if (h2i[k] >= 0) {
                park_w[k * kBlock] = cur.h2[k];
                st[h2i[k]] = park_r[k * kBlock];
            }
        }
        issue(nxt, it + 1);
        // sources: level 1 at plane zl (the extended tables, row n), level 2
        // at plane zl - R (the tile's points of the same tables, row n + 1)
        const bool lev2 = it >= 2 * R;
        const int e0 = __builtin_amdgcn_readfirstlane(s_pp[it]);
        const int e1 = __builtin_amdgcn_readfirstlane(s_pp[it + 1]);
        const int f0 = lev2 ? __builtin_amdgcn_readfirstlane(s_pp[it - R]) : 0;
        const int f1 = lev2 ? __builtin_amdgcn_readfirstlane(s_pp[it - R + 1]) : 0;
        if (e0 < e1) {
            // The buffer held the previous plane's staged values: every wave
            // is past reading them, then it is cleared.  (On such a plane
            // the barrier at its end keeps the next plane's staging from
            // overwriting the terms before they are read.)
            __syncthreads();
            for (int i = lane; i < N1; i += kBlock) reinterpret_cast<float4 *>(s_src1)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            __syncthreads();
            for (int e = e0 + lane; e < e1; e += kBlock) {
                const int4 c = a.inj.corner[e];
                float v = 0.f;
                for (int k = c.z; k < c.w; ++k) v = __builtin_fmaf(a.inj.w[k], a.inj.vals[a.inj.src[k]], v);
                s_src1[(c.y - (y0 - R)) * (4 * W1) + (c.x - (x0 - 4 * HX4))] = v * a.inj.scale;
            }
        }
        if (f0 < f1) {
            for (int e = f0 + lane; e < f1; e += kBlock) {
                const int4 c = a.inj.corner[e];
                if (c.x >= x0 && c.x < x0 + 4 * TW && c.y >= y0 && c.y < y0 + TY) {
                    float v = 0.f;
                    for (int k = c.z; k < c.w; ++k) v = __builtin_fmaf(a.inj2.w[k], a.inj2.vals[a.inj2.src[k]], v);
                    reinterpret_cast<float *>(s_src2)[(c.y - y0) * (4 * TW) + (c.x - x0)] = v * a.inj2.scale;
                }
            }
        }
        __syncthreads();
        // level 1 on every slot of the lane, zero outside the grid
        const bool in_z = zl >= 0 && zl < L.nz;
        const float sz1 = s_dz[it];
        float4 *rw = ring + (it % (R + 1)) * N1;
        float4 v1[NS];
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            v1[k] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (k == 0 || e1i[k] >= 0) {
                float lap[4];
                laplace(st + e2i[k], W2, q[k][R], q[k], lap);
                float4 src4 = make_float4(0.f, 0.f, 0.f, 0.f);
                if (e0 < e1 && e1i[k] >= 0) src4 = reinterpret_cast<const float4 *>(s_src1)[e1i[k]];
                const float src[4] = {src4.x, src4.y, src4.z, src4.w};
                float un[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float u1 = update_point(comp(q[k][R], i), comp(cur.mv[k], i), comp(cur.pv[k], i), lap[i],
                                                  src[i], sxy[k][i] + sz1);
                    un[i] = (in_z && in1[k] && gxs[k] + i < L.nx) ? u1 : 0.f;
                }
                asm volatile("" ::"v"(un[0]), "v"(un[1]), "v"(un[2]), "v"(un[3]));
                v1[k] = make_float4(un[0], un[1], un[2], un[3]);
            }
            if (e1i[k] >= 0) rw[e1i[k]] = v1[k];
        }
        w[2 * R] = v1[0];
        pq[R] = cur.pv[0];
        // u^{n+1} of the tile, for the planes of this chunk
        if (act && zl >= c0 && zl < c1) {
            const long long o = off[0] + (long long)zl * plane;
            if (nvalid >= 4) {
                st4nt_f32(O1 + o, v1[0]);
            } else {
                const float rv[3] = {v1[0].x, v1[0].y, v1[0].z};
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    if (i < nvalid) O1[o + i] = rv[i];
            }
        }
        // level 2 at plane zl - R: x and y neighbours from the u^{n+1} plane
        // written R iterations ago, z from the lane's queue, u^n from the
        // bottom of its u^n queue
        if (lev2) {
            float4 src4 = make_float4(0.f, 0.f, 0.f, 0.f);
            if (f0 < f1) {
                src4 = s_src2[lane];
                s_src2[lane] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
            if (act) {
                const float4 *rr = ring + ((it - R) % (R + 1)) * N1 + e1i[0];
                float lap[4];
                laplace(rr, W1, w[R], w, lap);
                const float src[4] = {src4.x, src4.y, src4.z, src4.w};
                const float sz2 = s_dz[it - R];
                float un[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    un[i] = update_point(comp(w[R], i), comp(q[0][0], i), comp(pq[0], i), lap[i], src[i],
                                         sxy[0][i] + sz2);
                asm volatile("" ::"v"(un[0]), "v"(un[1]), "v"(un[2]), "v"(un[3]));
                const long long o = off[0] + (long long)(zl - R) * plane;
                if (nvalid >= 4) {
                    st4nt_f32(O2 + o, make_float4(un[0], un[1], un[2], un[3]));
                } else {
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        if (i < nvalid) O2[o + i] = un[i];
                }
            }
        }
        if (e0 < e1 || f0 < f1) __syncthreads();   // read (and level 2's cleared) before the buffers are reused
#pragma unroll
        for (int k = 0; k < NS; ++k)
#pragma unroll
            for (int j = 0; j < 2 * R; ++j) q[k][j] = q[k][j + 1];
#pragma unroll
        for (int j = 0; j < 2 * R; ++j) w[j] = w[j + 1];
#pragma unroll
        for (int j = 0; j < R; ++j) pq[j] = pq[j + 1];
    };

    __syncthreads();   // staged tables and cleared source buffers, before the first plane
    Pre p0, p1;
    issue(p0, 0);
    int it = 0;
    for (; it + 2 <= npl; it += 2) {
        body(it, p0, p1);
        body(it + 1, p1, p0);
    }
    if (it < npl) body(it, p0, p1);
}

// ------------------------------------------------------------------ 2D step
// Grid axes (x, z); tile 64 x 64 staged whole in LDS with an r halo; each
// lane computes 4 x points in each of 4 rows.  One step per launch, where the
// several-level kernel (fd_step2d.hip) is not taken: time_block 1, served
// shots, fields above 1 GiB, the binomial gradient schedule, and grids on
// which the levels' recomputed ring costs more than they save (step2d_levels).
template <int R, Store S, int MODE>
__global__ __launch_bounds__(kBlock) void k_step2d(const StepArgs a) {
    using E = Elem<S>;
    using T = typename E::T;
    constexpr int HX4 = (R + 3) / 4;
    constexpr int W4 = 16 + 2 * HX4;
    constexpr int LH = kTile2Z + 2 * R;
    __shared__ float4 lds[LH * W4];

    const Layout L = a.L;
    const int ntile = (int)gridDim.x - a.nsamp_blocks;   // tiles first, then sampling
    if ((int)blockIdx.x >= ntile) {
        sample_block<S>(a.smp, a.u, (int)blockIdx.x - ntile);
        return;
    }
    const int t = xcd_remap((int)blockIdx.x, ntile);
    const int bx = t % a.ntx, bz = t / a.ntx;
    const int x0 = bx * kTileX, z0 = bz * kTile2Z;
    const int z1 = min(z0 + kTile2Z, L.nz);
    const int lane = (int)threadIdx.x;
    __shared__ float s_dz[kTile2Z];
    __shared__ int s_pp[kTile2Z + 1];
    const int *tile_pp = a.inj.plane_ptr + (long long)bx * (L.nz + 1);
    for (int i = lane; i <= z1 - z0; i += kBlock) {
        if (i < z1 - z0) s_dz[i] = a.damp[L.nx + L.ny + z0 + i];
        s_pp[i] = a.inj.vals ? tile_pp[z0 + i] : 0;
    }
    const T *U = (const T *)a.u;
    const long long zcol = L.offset((L.nx + 3) & ~3, 0, 0);   // zero in every row

    for (int i = lane; i < LH * W4; i += kBlock) {
        const int lr = i / W4, c = i - lr * W4;
        const int gz = z0 - R + lr, gx = x0 - 4 * HX4 + 4 * c;
        const bool ok = gz >= 0 && gz < L.nz && gx >= 0 && gx < L.nx;
        lds[i] = E::ld4(U + (ok ? L.offset(gx, 0, gz) : zcol));
    }
    __syncthreads();

    const int tx = lane & 15, tz = lane >> 4;
    const int x = x0 + 4 * tx;
    if (x >= L.nx) return;
    const int nvalid = L.nx - x;
    float sx[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) sx[i] = a.damp[min(x + i, L.nx - 1)];
    const T *Pv = (const T *)a.prev;
    T *O = (T *)a.out;
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
        const int z = z0 + tz * 4 + rr;
        if (z >= L.nz) break;
        const float4 *row = lds + (R + tz * 4 + rr) * W4 + HX4 + tx;
        float xs[4 * (2 * HX4 + 1)];
#pragma unroll
        for (int c = -HX4; c <= HX4; ++c) {
            const float4 v = row[c];
            xs[4 * (c + HX4) + 0] = v.x;
            xs[4 * (c + HX4) + 1] = v.y;
            xs[4 * (c + HX4) + 2] = v.z;
            xs[4 * (c + HX4) + 3] = v.w;
        }
        float lap[4];
#pragma unroll
        for (int j = 1; j <= R; ++j) {
            const float4 zp = row[j * W4], zm = row[-j * W4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float t = lap_term2(a.wx[j], xs[4 * HX4 + i + j] + xs[4 * HX4 + i - j], a.wz[j],
                                          comp(zp, i) + comp(zm, i));
                lap[i] = j == 1 ? t : lap[i] + t;
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) lap[i] = __builtin_fmaf(a.w0, xs[4 * HX4 + i], lap[i]);
        float src[4] = {0.f, 0.f, 0.f, 0.f};
        const int e0 = s_pp[z - z0], e1 = s_pp[z - z0 + 1];
        if (e0 < e1) gather_sources(a.inj, e0, e1, x, src[0], src[1], src[2], src[3]);
        const long long off = L.offset(x, 0, z);
        const float4 pc = ld4nt_f32(a.p + off);
        const float4 mc = E::ld4nt(Pv + off);
        const float4 cc = row[0];
        const float sz = s_dz[z - z0];
        float un[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            un[i] = update_point(comp(cc, i), comp(mc, i), comp(pc, i), lap[i], src[i], sx[i] + sz);
        if constexpr (S != Store::F32)   // round to float32, then to 16 bits (no fused conversion)
            asm volatile("" : "+v"(un[0]), "+v"(un[1]), "+v"(un[2]), "+v"(un[3]));
        if (nvalid >= 4) {
            E::st4nt(O + off, make_float4(un[0], un[1], un[2], un[3]));
        } else {
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (i < nvalid) E::st(O + off + i, un[i]);
        }
        if constexpr (MODE != kPlain) {
            float sv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) sv[i] = sx[i] + sz;
            grad_epilogue<MODE>(a.img, off, nvalid, un, cc, mc, sv);
        }
    }
}

template <Store S>
__global__ void k_sample(const Sample s, const void *field) {
    sample_block<S>(s, field, (int)blockIdx.x);
}

// --------------------------------------------------------------- utilities
// Grid-stride walk over the float4 groups of a field's grid rows: a lane
// takes 4 consecutive points at a time (the last group of a row may reach
// past nx), so one index division serves 4 points and the pitched side of
// every access is one 16-byte access per lane.
struct Quads {
    const Layout &L;
    const int g4;          // groups per row
    const long long n, step;
    long long i;
    int gx, y, z;
    __device__ explicit Quads(const Layout &l)
        : L(l), g4((l.nx + 3) / 4), n((long long)((l.nx + 3) / 4) * l.ny * l.nz),
          step((long long)gridDim.x * blockDim.x), i((long long)blockIdx.x * blockDim.x + threadIdx.x) {
        split();
    }
    __device__ void split() {
        if (n < (1LL << 31)) {   // (32-bit division is several times cheaper)
            const unsigned row = (unsigned)i / (unsigned)g4;
            gx = (int)((unsigned)i - row * (unsigned)g4);
            z = (int)(row / (unsigned)L.ny);
            y = (int)(row - (unsigned)z * (unsigned)L.ny);
        } else {
            const long long row = i / g4;
            gx = (int)(i - row * g4);
            z = (int)(row / L.ny);
            y = (int)(row - (long long)z * L.ny);
        }
    }
    __device__ bool more() const { return i < n; }
    __device__ void next() {
        i += step;
        if (i < n) split();
    }
    __device__ int x() const { return 4 * gx; }
    __device__ long long offset() const { return L.offset(4 * gx, y, z); }   // a multiple of 4
    __device__ long long dense() const { return ((long long)z * L.ny + y) * L.nx + 4 * gx; }
};

// Two atomics per workgroup: the lanes' extremes are reduced in the wave and
// then through LDS.  (With two atomics per lane, four million on two
// addresses at most, the kernel took 750 us on any grid of more than 2 M
// points, whatever its size: the atomics were the bound.)
__global__ __launch_bounds__(kBlock) void k_vrange(const Layout L, const float *vel, unsigned *out) {
    float m = 0.f, lo = __uint_as_float(0x7F800000u);
    for (Quads q(L); q.more(); q.next()) {
        const float4 v4 = *reinterpret_cast<const float4 *>(vel + q.offset());
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float v = comp(v4, i);
            if (q.x() + i >= L.nx) break;
            // NaN or non-positive velocities poison the maximum on purpose
            m = (v > 0.f) ? fmaxf(m, v) : __uint_as_float(0x7F800000u);
            lo = (v > 0.f) ? fminf(lo, v) : lo;
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        m = fmaxf(m, __shfl_xor(m, o, 64));
        lo = fminf(lo, __shfl_xor(lo, o, 64));
    }
    __shared__ float s_m[kBlock / 64], s_lo[kBlock / 64];
    if (threadIdx.x % 64 == 0) {
        s_m[threadIdx.x / 64] = m;
        s_lo[threadIdx.x / 64] = lo;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) {
            m = fmaxf(m, s_m[w]);
            lo = fminf(lo, s_lo[w]);
        }
        // positive floats order as their bit patterns
        atomicMax(out, __float_as_uint(m));
        atomicMin(out + 1, __float_as_uint(lo));
    }
}

// Velocity, p and its 16-bit code by float4 groups.  (Point by point, with a
// 64-bit index division each, the three took 121, 97 and 107 us on 336^3; now
// 73, 56 and 50.)  The cells past nx of a row's last group hold zero before
// and after: the velocity is written zero there, which makes p and its code
// zero too.
__global__ __launch_bounds__(kBlock) void k_fill_velocity(const Layout L, const float *vp, int vp_padded, int nbl,
                                                          int px, int py, int pz, float *vel) {
    for (Quads q(L); q.more(); q.next()) {
        const float *row;
        int shift = 0, last = L.nx - 1;
        if (vp_padded) {
            row = vp + ((long long)q.z * L.ny + q.y) * L.nx;
        } else {
            const int iz = min(max(q.z - nbl, 0), pz - 1);
            const int iy = L.ndim == 3 ? min(max(q.y - nbl, 0), py - 1) : 0;
            row = vp + ((long long)iz * (L.ndim == 3 ? py : 1) + iy) * px;
            shift = nbl;
            last = px - 1;
        }
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            v[i] = q.x() + i < L.nx ? row[min(max(q.x() + i - shift, 0), last)] : 0.f;
        *reinterpret_cast<float4 *>(vel + q.offset()) = make_float4(v[0], v[1], v[2], v[3]);
    }
}

__global__ __launch_bounds__(kBlock) void k_make_p(const Layout L, const float *vel, double dt2, float *p) {
    for (Quads q(L); q.more(); q.next()) {
        const float4 v4 = *reinterpret_cast<const float4 *>(vel + q.offset());
        float r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double v = (double)comp(v4, i);
            r[i] = (float)(dt2 * v * v);
        }
        *reinterpret_cast<float4 *>(p + q.offset()) = make_float4(r[0], r[1], r[2], r[3]);
    }
}

// The 16-bit code of p: the nearest integer in [0, 65535] to (p - base) /
// step with p = dt^2 v^2, all in float64 (base and step are the float32
// values the step's decode uses, so the code is the nearest one for that
// decode).  Each operation rounds on its own (no contraction), as the
// definition states.
__global__ __launch_bounds__(kBlock) void k_make_pq(const Layout L, const float *vel, double dt2, double base,
                                                    double step, uint16_t *pq) {
#pragma clang fp contract(off)
    for (Quads q(L); q.more(); q.next()) {
        const float4 v4 = *reinterpret_cast<const float4 *>(vel + q.offset());
        uint32_t code[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double v = (double)comp(v4, i);
            const double p = dt2 * v * v;
            const double c = step > 0.0 ? rint((p - base) / step) : 0.0;
            code[i] = q.x() + i < L.nx ? (uint32_t)(uint16_t)fmin(fmax(c, 0.0), 65535.0) : 0u;
        }
        *reinterpret_cast<uint2 *>(pq + q.offset()) =
            make_uint2(code[0] | code[1] << 16, code[2] | code[3] << 16);
    }
}

// 16-byte stores; n float4 groups.  Then `words` words at each of `nq` places
// `apart` bytes apart from q on.
__global__ __launch_bounds__(kBlock) void k_zero(float4 *f, long long n, char *q, size_t apart, int nq, int words) {
    for (long long i = blockIdx.x * (long long)kBlock + threadIdx.x; i < n; i += (long long)gridDim.x * kBlock)
        f[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < nq * words; i += kBlock)
            reinterpret_cast<uint32_t *>(q + (size_t)(i / words) * apart)[i % words] = 0u;
}

// Zero the cells of a 2D float32 field that hold no grid quad: the pads left
// and right of a row and the halo rows.
__global__ __launch_bounds__(kBlock) void k_zero_rim2d(const Layout L, float *f) {
    const int g4 = (L.nx + 3) / 4, p4 = L.pitch / 4, side = p4 - g4;   // pad quads of a grid row
    const long long rows = (long long)L.nz * side, n = rows + 2LL * L.r * p4;
    float4 *q = reinterpret_cast<float4 *>(f);
    for (long long i = blockIdx.x * (long long)kBlock + threadIdx.x; i < n; i += (long long)gridDim.x * kBlock) {
        long long at;
        if (i < rows) {
            const long long z = i / side;
            const int k = (int)(i - z * side);
            at = (z + L.r) * p4 + (k < kXOff / 4 ? k : k + g4);
        } else {
            const long long h = i - rows;
            at = h < (long long)L.r * p4 ? h : h + (long long)L.nz * p4;
        }
        q[at] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

// 4 points of a dense row from x on (n of them inside the grid); wide: the
// rows start on 16-byte boundaries.
__device__ inline float4 dense_ld4(const float *d, int n, bool wide) {
    if (wide) return *reinterpret_cast<const float4 *>(d);
    return make_float4(d[0], n > 1 ? d[1] : 0.f, n > 2 ? d[2] : 0.f, n > 3 ? d[3] : 0.f);
}
__device__ inline void dense_st4(float *d, const float4 &v, int n, bool wide) {
    if (wide) {
        st4nt_f32(d, v);
        return;
    }
    d[0] = v.x;
    if (n > 1) d[1] = v.y;
    if (n > 2) d[2] = v.z;
    if (n > 3) d[3] = v.w;
}
__device__ inline float4 scale4(const float4 &v, float s) {
    return make_float4(v.x * s, v.y * s, v.z * s, v.w * s);
}
// Store 4 scaled points.  Half precision rounds the exact product once (a
// fused multiply and conversion); a pair conversion of the float32 products
// would round twice where the scale is no power of two.
template <Store S>
__device__ inline void st4_scaled(typename Elem<S>::T *p, const float4 &v, float s) {
    if constexpr (S == Store::F16) {
        auto h = [](float x, float k) { return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)(x * k)); };
        *reinterpret_cast<uint2 *>(p) =
            make_uint2(h(v.x, s) | h(v.y, s) << 16, h(v.z, s) | h(v.w, s) << 16);
    } else {
        Elem<S>::st4(p, scale4(v, s));
    }
}
__device__ inline float4 sub4(const float4 &a, const float4 &b) {
    return make_float4(a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w);
}

// Dense field <-> pitched field, a float4 group per lane.  (Point by point
// with a 64-bit index division each they ran at 3.2 TB/s on 336^3, 94 us.)
// The cells past nx of a row's last group are written zero, as they are.
template <Store S>
__global__ __launch_bounds__(kBlock) void k_dense_to_field(const Layout L, const float *dense, void *f, float scale,
                                                           bool wide) {
    using E = Elem<S>;
    for (Quads q(L); q.more(); q.next())
        st4_scaled<S>((typename E::T *)f + q.offset(), dense_ld4(dense + q.dense(), L.nx - q.x(), wide), scale);
}

template <Store S>
__global__ __launch_bounds__(kBlock) void k_field_to_dense(const Layout L, const void *f, float *dense, float scale,
                                                           bool wide) {
    using E = Elem<S>;
    for (Quads q(L); q.more(); q.next())
        dense_st4(dense + q.dense(), scale4(E::ld4((const typename E::T *)f + q.offset()), scale), L.nx - q.x(), wide);
}

// Difference storage: d = scale * (a - b) rounded once (a, b nullable), and
// dense = scale * (u - d).
template <Store S>
__global__ __launch_bounds__(kBlock) void k_dense_diff_to_field(const Layout L, const float *a, const float *b,
                                                                void *d, float scale, bool wide) {
    using E = Elem<S>;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    for (Quads q(L); q.more(); q.next()) {
        const int n = L.nx - q.x();
        const float4 av = a ? dense_ld4(a + q.dense(), n, wide) : zero;
        const float4 bv = b ? dense_ld4(b + q.dense(), n, wide) : zero;
        st4_scaled<S>((typename E::T *)d + q.offset(), sub4(av, bv), scale);
    }
}

template <Store S>
__global__ __launch_bounds__(kBlock) void k_field_diff_to_dense(const Layout L, const void *u, const void *d,
                                                                float *dense, float scale, bool wide) {
    using E = Elem<S>;
    using T = typename E::T;
    for (Quads q(L); q.more(); q.next()) {
        const float4 v = sub4(E::ld4((const T *)u + q.offset()), E::ld4((const T *)d + q.offset()));
        dense_st4(dense + q.dense(), scale4(v, scale), L.nx - q.x(), wide);
    }
}

// Misfit: residual and per-block FP64 partial sums of r^2/2 (fixed order),
// then a single workgroup folds the partials in index order.
__global__ void k_misfit_partial(const float *rec, const float *obs, long long n, int given,
                                 float *resid, double *partials) {
    __shared__ double sh[kBlock];
    double acc = 0.0;
    for (long long i = blockIdx.x * (long long)kBlock + threadIdx.x; i < n;
         i += (long long)gridDim.x * kBlock) {
        const float r = given ? obs[i] : rec[i] - obs[i];
        if (resid) resid[i] = r;
        acc += 0.5 * (double)r * (double)r;
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) partials[blockIdx.x] = sh[0];
}

__global__ void k_misfit_final(const double *partials, int npart, double *out) {
    __shared__ double sh[kBlock];
    double acc = 0.0;
    for (int i = threadIdx.x; i < npart; i += kBlock) acc += partials[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = sh[0];
}

// ------------------------------------------------------------ dispatch tables
template <Store S, int MODE, int... Rs>
struct Table2 {
    static StepFn get(int r) {
        StepFn f = nullptr;
        ((r == Rs ? (f = k_step2d<Rs, S, MODE>, 0) : 0), ...);
        return f;
    }
};

template <Store S, int MODE>
using Tab2 = Table2<S, MODE, 1, 2, 3, 4, 5, 6, 7, 8>;

// The gradient modes exist for float32 storage and p only, the difference
// storage for 16-bit 3D fields only, the 16-bit p codes in 3D only (kPlain
// and kDiff); the 3D kernels come from the storage type's own unit.
StepFn pick_step(int ndim, int r, Store st, int mode, int tw4, int pf) {
    const bool pq = pf == kPCodes;
    if (ndim == 3) {
        if (pq && mode != kPlain && mode != kDiff) return nullptr;
        if ((mode == kBracket || mode == kImage || mode == kImage3) && st != Store::F32) return nullptr;
        if (mode == kDiff && st == Store::F32) return nullptr;
        if (pf == kPCached && st != Store::F32) {
            StepFn f = st == Store::F16 ? step3d_kernel_f16_cached(r, mode, tw4) : step3d_kernel_bf16_cached(r, mode, tw4);
            if (f) return f;
        }
        switch (st) {
            case Store::F32: return step3d_kernel_f32(r, mode, tw4, pq);
            case Store::F16: return mode == kDiff ? step3d_kernel_f16_diff(r, tw4, pq) : step3d_kernel_f16(r, tw4, pq);
            case Store::BF16:
                return mode == kDiff ? step3d_kernel_bf16_diff(r, tw4, pq) : step3d_kernel_bf16(r, tw4, pq);
        }
        return nullptr;
    }
    if (pq || mode == kDiff || mode == kImage3) return nullptr;
    if (mode == kBracket) return st == Store::F32 ? Tab2<Store::F32, kBracket>::get(r) : nullptr;
    if (mode == kImage) return st == Store::F32 ? Tab2<Store::F32, kImage>::get(r) : nullptr;
    switch (st) {
        case Store::F32: return Tab2<Store::F32, kPlain>::get(r);
        case Store::F16: return Tab2<Store::F16, kPlain>::get(r);
        case Store::BF16: return Tab2<Store::BF16, kPlain>::get(r);
    }
    return nullptr;
}

inline int grid_for(long long n) {
    long long b = (n + kBlock - 1) / kBlock;
    if (b > 8192) b = 8192;
    if (b < 1) b = 1;
    return (int)b;
}

}  // namespace

hipError_t launch_step_t2(const StepArgs &a, hipStream_t s) {
    void (*f)(const StepArgs) = nullptr;
    switch (a.L.r) {
        case 1: f = k_step3d_t2<1>; break;
        case 2: f = k_step3d_t2<2>; break;
        case 3: f = k_step3d_t2<3>; break;
        case 4: f = k_step3d_t2<4>; break;
        default: return hipErrorInvalidValue;
    }
    if (a.L.ndim != 3) return hipErrorInvalidValue;
    const int blocks = a.ntx * a.nty * a.ntz + a.nsamp_blocks + a.nsamp_blocks2;
    if (blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(f, dim3(blocks), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

int step_t2_blocks_per_cu(int r) {
    const void *f = r == 1 ? reinterpret_cast<const void *>(k_step3d_t2<1>)
                    : r == 2 ? reinterpret_cast<const void *>(k_step3d_t2<2>)
                    : r == 3 ? reinterpret_cast<const void *>(k_step3d_t2<3>)
                    : r == 4 ? reinterpret_cast<const void *>(k_step3d_t2<4>)
                             : nullptr;
    if (!f) return 0;
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, kBlock, 0) != hipSuccess) return 0;
    return n;
}

hipError_t launch_step(const StepArgs &a, Store st, int mode, hipStream_t s) {
    const int pf = a.pq ? kPCodes : a.p_cached ? kPCached : kPFloat;
    StepFn f = pick_step(a.L.ndim, a.L.r, st, mode, a.shape3, pf);
    if (!f) return hipErrorInvalidValue;
    const int tiles = (a.ntx * a.nty + (a.L.ndim == 3 ? a.nstrip : 0)) * a.ntz;
    const int blocks = tiles + a.nsamp_blocks;
    if (blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(f, dim3(blocks), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

int step_blocks_per_cu(int ndim, int r, Store st, int mode, int tw4, bool pq) {
    StepFn f = pick_step(ndim, r, st, mode, tw4, pq ? kPCodes : kPFloat);
    if (!f) return 0;
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void *>(f), kBlock, 0) !=
        hipSuccess)
        return 0;
    return n;
}

hipError_t launch_sample(const Sample &smp, const void *field, Store st, hipStream_t s) {
    if (!smp.out || smp.npts <= 0) return hipSuccess;
    const int blocks = sample_blocks(smp);
    switch (st) {
        case Store::F32: hipLaunchKernelGGL(k_sample<Store::F32>, dim3(blocks), dim3(kBlock), 0, s, smp, field); break;
        case Store::F16: hipLaunchKernelGGL(k_sample<Store::F16>, dim3(blocks), dim3(kBlock), 0, s, smp, field); break;
        case Store::BF16: hipLaunchKernelGGL(k_sample<Store::BF16>, dim3(blocks), dim3(kBlock), 0, s, smp, field); break;
    }
    return hipGetLastError();
}

hipError_t launch_fill_velocity(const Layout &L, const float *vp, int vp_padded, int nbl,
                                const int *phys, float *vel, hipStream_t s) {
    const long long quads = (long long)((L.nx + 3) / 4) * L.ny * L.nz;
    hipLaunchKernelGGL(k_fill_velocity, dim3(grid_for(quads)), dim3(kBlock), 0, s, L, vp, vp_padded,
                       nbl, phys[0], phys[1], phys[2], vel);
    return hipGetLastError();
}

hipError_t launch_vrange(const Layout &L, const float *vel, unsigned *out_bits, hipStream_t s) {
    const long long quads = (long long)((L.nx + 3) / 4) * L.ny * L.nz;
    hipLaunchKernelGGL(k_vrange, dim3(std::min(2048, grid_for(quads))), dim3(kBlock), 0, s, L, vel, out_bits);
    return hipGetLastError();
}

hipError_t launch_make_p(const Layout &L, const float *vel, double dt, float *p, hipStream_t s) {
    const long long quads = (long long)((L.nx + 3) / 4) * L.ny * L.nz;
    hipLaunchKernelGGL(k_make_p, dim3(grid_for(quads)), dim3(kBlock), 0, s, L, vel, dt * dt, p);
    return hipGetLastError();
}

hipError_t launch_make_pq(const Layout &L, const float *vel, double dt, double base, double step,
                          uint16_t *pq, hipStream_t s) {
    const long long quads = (long long)((L.nx + 3) / 4) * L.ny * L.nz;
    hipLaunchKernelGGL(k_make_pq, dim3(grid_for(quads)), dim3(kBlock), 0, s, L, vel, dt * dt, base, step, pq);
    return hipGetLastError();
}

hipError_t launch_zero(void *p, size_t bytes, hipStream_t s) {
    return launch_zero_and_quads(p, bytes, nullptr, 0, 0, Store::F32, s);
}

hipError_t launch_zero_and_quads(void *p, size_t bytes, void *quads, size_t apart, int nq, Store st, hipStream_t s) {
    const long long n = (long long)(bytes / sizeof(float4));
    hipLaunchKernelGGL(k_zero, dim3(grid_for(n)), dim3(kBlock), 0, s, (float4 *)p, n, (char *)quads, apart, nq,
                       st == Store::F32 ? 4 : 2);
    return hipGetLastError();
}

hipError_t launch_zero_rim2d(const Layout &L, float *f, hipStream_t s) {
    if (L.ndim != 2) return hipErrorInvalidValue;
    const long long n = (long long)L.nza * (L.pitch / 4) - (long long)L.nz * ((L.nx + 3) / 4);
    hipLaunchKernelGGL(k_zero_rim2d, dim3(grid_for(n)), dim3(kBlock), 0, s, L, f);
    return hipGetLastError();
}

// acc += part, part = 0, over the grid rows of the two pitched fields (x in
// [0, round4(nx)): the cells past nx are zero in both, so they stay zero);
// the zero halo and pad are left alone.
__global__ void k_fold_f64(double *acc, float *part, const Layout L) {
    const int g4 = (L.nx + 3) / 4;   // float4 groups per row
    const long long n = (long long)g4 * L.ny * L.nz;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const long long row = i / g4;
        const int gx = (int)(i - row * g4);
        const long long off = L.offset(4 * gx, (int)(row % L.ny), (int)(row / L.ny));   // a multiple of 4
        const float4 p = *reinterpret_cast<const float4 *>(part + off);
        double2 *a = reinterpret_cast<double2 *>(acc + off);
        double2 a0 = a[0], a1 = a[1];
        a0.x += p.x;
        a0.y += p.y;
        a1.x += p.z;
        a1.y += p.w;
        a[0] = a0;
        a[1] = a1;
        *reinterpret_cast<float4 *>(part + off) = make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

hipError_t launch_fold_f64(const Layout &L, double *acc, float *part, hipStream_t s) {
    const long long n = (long long)((L.nx + 3) / 4) * L.ny * L.nz;
    hipLaunchKernelGGL(k_fold_f64, dim3(grid_for(n)), dim3(kBlock), 0, s, acc, part, L);
    return hipGetLastError();
}

namespace {
inline long long quads(const Layout &L) { return (long long)((L.nx + 3) / 4) * L.ny * L.nz; }
// whether every row of a dense field starts on a 16-byte boundary
inline bool wide_rows(const Layout &L, const void *a, const void *b = nullptr) {
    return L.nx % 4 == 0 && ((uintptr_t)a | (uintptr_t)b) % 16 == 0;
}
}  // namespace

hipError_t launch_dense_to_field(const Layout &L, const float *dense, void *f, Store st,
                                 float scale, hipStream_t s) {
    const dim3 g(grid_for(quads(L))), b(kBlock);
    const bool w = wide_rows(L, dense);
    switch (st) {
        case Store::F32: hipLaunchKernelGGL(k_dense_to_field<Store::F32>, g, b, 0, s, L, dense, f, scale, w); break;
        case Store::F16: hipLaunchKernelGGL(k_dense_to_field<Store::F16>, g, b, 0, s, L, dense, f, scale, w); break;
        case Store::BF16: hipLaunchKernelGGL(k_dense_to_field<Store::BF16>, g, b, 0, s, L, dense, f, scale, w); break;
    }
    return hipGetLastError();
}

hipError_t launch_field_to_dense(const Layout &L, const void *f, float *dense, Store st,
                                 float scale, hipStream_t s) {
    const dim3 g(grid_for(quads(L))), b(kBlock);
    const bool w = wide_rows(L, dense);
    switch (st) {
        case Store::F32: hipLaunchKernelGGL(k_field_to_dense<Store::F32>, g, b, 0, s, L, f, dense, scale, w); break;
        case Store::F16: hipLaunchKernelGGL(k_field_to_dense<Store::F16>, g, b, 0, s, L, f, dense, scale, w); break;
        case Store::BF16: hipLaunchKernelGGL(k_field_to_dense<Store::BF16>, g, b, 0, s, L, f, dense, scale, w); break;
    }
    return hipGetLastError();
}

hipError_t launch_dense_diff_to_field(const Layout &L, const float *a, const float *b, void *d, Store st,
                                      float scale, hipStream_t s) {
    const dim3 g(grid_for(quads(L))), bl(kBlock);
    const bool w = wide_rows(L, a, b);
    if (st == Store::F16)
        hipLaunchKernelGGL(k_dense_diff_to_field<Store::F16>, g, bl, 0, s, L, a, b, d, scale, w);
    else if (st == Store::BF16)
        hipLaunchKernelGGL(k_dense_diff_to_field<Store::BF16>, g, bl, 0, s, L, a, b, d, scale, w);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_field_diff_to_dense(const Layout &L, const void *u, const void *d, float *dense, Store st,
                                      float scale, hipStream_t s) {
    const dim3 g(grid_for(quads(L))), bl(kBlock);
    const bool w = wide_rows(L, dense);
    if (st == Store::F16)
        hipLaunchKernelGGL(k_field_diff_to_dense<Store::F16>, g, bl, 0, s, L, u, d, dense, scale, w);
    else if (st == Store::BF16)
        hipLaunchKernelGGL(k_field_diff_to_dense<Store::BF16>, g, bl, 0, s, L, u, d, dense, scale, w);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

namespace {
// dense = f, or with a velocity field the chain rule from m = 1/v^2 to v:
// dense = f * dm/dv = f * (-2 / v^3), in float64.  (A point per lane: four per
// lane store 32 bytes apart and took 97 us on 280^3 where this takes 74.)
__global__ void k_field_to_dense_f64(const Layout L, const double *f, const float *vel, double *dense) {
    const long long n = (long long)L.nx * L.ny * L.nz;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const int x = (int)(i % L.nx);
        const int y = (int)((i / L.nx) % L.ny);
        const int z = (int)(i / ((long long)L.nx * L.ny));
        const long long o = L.offset(x, y, z);
        double g = f[o];
        if (vel) {
            const double v = (double)vel[o];
            g *= -2.0 / (v * v * v);
        }
        dense[i] = g;
    }
}
}  // namespace

hipError_t launch_field_to_dense_f64(const Layout &L, const double *f, const float *vel, double *dense,
                                     hipStream_t s) {
    const long long n = (long long)L.nx * L.ny * L.nz;
    hipLaunchKernelGGL(k_field_to_dense_f64, dim3(grid_for(n)), dim3(kBlock), 0, s, L, f, vel, dense);
    return hipGetLastError();
}

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices];
}  // namespace

hipError_t static_scratch(int device, void **ptr) {
    if (device < 0 || device >= kMaxDevices || !ptr) return hipErrorInvalidValue;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[device] = p;
    }
    *ptr = g_scratch_ptr[device];
    return hipSuccess;
}

hipError_t launch_misfit(const float *rec, const float *obs, long long n, int residual_given,
                         float *resid, double *partials, int npart, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_misfit_partial, dim3(npart), dim3(kBlock), 0, s, rec, obs, n,
                       residual_given, resid, partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_misfit_final, dim3(1), dim3(kBlock), 0, s, partials, npart, out);
    return hipGetLastError();
}

}  // namespace fd

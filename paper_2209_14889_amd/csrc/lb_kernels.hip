// HIP kernels of liblb for gfx950 (MI355X).
//
//   k_ib_step     immersed-body update (App. A): node Heun step, node forces and force spreading
//                 in one launch, for a step with few patch tiles
//   k_ib_nodes, k_ib_spread   the same in two launches (nodes once per body, then the tiles)
//   k_fused       one pass per step over every lattice site: forces, BGK + Guo collide with pull
//                 streaming, velocity gradient, stiffness, Heun stress and polarization
//   k_tile        the same pass on tiles whose rows are computed at once, for small lattices
//   k_mp_*        the same step as four simple site-parallel kernels (debug / reference path)
//   k_readout     observables at the current time
//   k_sums / k_sums_final, k_body_force   FP64 reductions
//
// The fused kernel walks a strip of columns down its rows like a pipeline.  Iteration j loads the
// polarization of row f = y0 - 4 + j and the stress of row f-1, forms the Ericksen stress at row
// f-1, collides row f-2, predicts row f-3 and corrects row f-4.  Every stage only needs rows that
// earlier stages or earlier iterations produced, so within a work item each value is computed
// once (the items overlap only by the pipeline's halo rows and columns) and row exchanges go
// through small LDS ring buffers.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <hip/hip_fp16.h>

#include "lb_device.h"
#include "lb_launch.h"

namespace lbk {

// ------------------------------------------------------------------------------------------------
// immersed boundary
// ------------------------------------------------------------------------------------------------

// the four x (or y) weights phi(R - i), i = floor(R) - 1 .. floor(R) + 2, of the cosine kernel
// phi(r) = (1 + cos(pi r / 2)) / 4 (App. A).  With f = R - floor(R) in [0, 1) the four distances
// are 1 + f, f, f - 1, f - 2, whose cosines are -sin, cos, sin, -cos of pi f / 2: one sincos
// gives all four (the last weight is 0 at f = 0, where its site leaves the support |r| < 2).
// FP32 is enough for weights of values that are themselves FP32.
__device__ __forceinline__ void phi4(double R, int &i0, float w[4]) {
    const double fl = floor(R);
    i0 = (int)fl - 1;
    const float f = (float)(R - fl);
    float sn, cs;
    sincosf(1.57079632679f * f, &sn, &cs);
    w[0] = 0.25f * (1.0f - sn);
    w[1] = 0.25f * (1.0f + cs);
    w[2] = 0.25f * (1.0f + sn);
    w[3] = 0.25f * (1.0f - cs);
}

// The schedule at time t, by the lanes of one wave: pull = S((t - t_on)/w) - S((t - t_off)/w) with S the
// logistic function (1 for a constant pull); the trap's stiffness k = trap_k [S(u1) - S(u2)] and travelled
// share rho = w / T [sp(u1) - sp(u2)], sp(x) = ln(1 + e^x) (App. A, eqUtrap; App. C).  Lanes 0, 1 take
// the pull's S, 2, 3 the trap's S and 4, 5 its sp, each one exponential.
struct Schedule {
    double pull, k, rho;
};
__device__ __forceinline__ Schedule schedule(const BodyDev &B, double t) {
    Schedule q{1.0, 0.0, 0.0};
    if (B.width <= 0.0 && B.trap_k == 0.0) return q;
    const int lane = threadIdx.x & 63;
    const bool pull = lane < 2, on = (lane & 1) == 0, soft = lane >= 4;
    const double x = pull ? (t - (on ? B.t_on : B.t_off)) / B.width : (t - (on ? B.trap_t1 : B.trap_t2)) / B.trap_w;
    const bool up = soft && !(x > 30.0);
    const double e = exp(up ? x : -x);
    double r;
    if (soft)
        r = x > 30.0 ? x + log1p(e) : log1p(e);
    else
        r = 1.0 / (1.0 + e);
    const double d = r - __shfl_xor(r, 1);   // even lanes: on minus off
    const double T = B.trap_t2 - B.trap_t1;
    if (B.width > 0.0) q.pull = __shfl(d, 0);
    if (B.trap_k != 0.0) {
        q.k = B.trap_k * __shfl(d, 2);
        q.rho = T > 0.0 ? (B.trap_w / T) * __shfl(d, 4) : 0.0;
    }
    return q;
}

typedef float Float4 __attribute__((ext_vector_type(4)));     // 16 bytes each, for loads from global memory
typedef double Double2 __attribute__((ext_vector_type(2)));
// four consecutive floats at any 4-byte boundary (one 16-byte load)
typedef float Row4 __attribute__((ext_vector_type(4), aligned(4)));

// Heun step of one node by a pair of lanes, lane c taking the component c (0: x, 1: y) of the node
// position r: r + (v(R) + v(R + v(R))) / 2 with v interpolated from the body's velocity patch V (side
// ps, origin o[2]; the x plane, then the y plane).  Each lane forms the kernel weights of its own
// coordinate, takes the other's from its partner and sums its own plane's 4 x 4 values.  The second
// position is a small fraction of a site away, so its footprint is nearly always the first one's and
// reuses the values loaded for it.  bad: a footprint outside the patch.
__device__ __forceinline__ double heun_component(const float *V, int ps, int ox, int oy, int c, double r, bool &bad) {
    const float *plane = V + (size_t)c * ps * ps;
    Row4 row[4];
    int at = -1;   // where row[] was loaded from
    double v[2] = {0.0, 0.0};
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
        int i0;
        float w[4], u[4];
        phi4(r + v[0], i0, w);
        const int j0 = __shfl_xor(i0, 1);
#pragma unroll
        for (int k = 0; k < 4; ++k) u[k] = __shfl_xor(w[k], 1);
        const int px0 = (c ? j0 : i0) - ox, py0 = (c ? i0 : j0) - oy;
        const bool out = px0 < 0 || py0 < 0 || px0 + 3 >= ps || py0 + 3 >= ps;
        bad = bad || out;
        double s = 0.0;
        if (!out) {
            const int q = py0 * ps + px0;
            if (q != at)
#pragma unroll
                for (int j = 0; j < 4; ++j) row[j] = *(const LBK_GLOBAL Row4 *)gptr(plane + q + j * ps);
            at = q;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                double a = 0.0;
#pragma unroll
                for (int i = 0; i < 4; ++i) a += (double)(c ? u[i] : w[i]) * (double)row[j][i];
                s += (double)(c ? w[j] : u[j]) * a;
            }
        }
        v[1] = v[0] + s;
        if (pass == 0) v[0] = s;
    }
    return r + 0.5 * v[1];
}

__device__ __forceinline__ double wave_min(double v) {
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ double wave_max(double v) {
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ double wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// centre of mass of the n nodes in LDS, the same in every block: the first 256 threads' sums in node
// order, wave sums, then the four waves in a fixed order
__device__ __forceinline__ double2 block_com(const double2 *sR, int n, double (*sC)[2]) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (tid < 256) {
        double cx = 0.0, cy = 0.0;
        for (int a = tid; a < n; a += 256) {
            cx += sR[a].x;
            cy += sR[a].y;
        }
        cx = wave_sum(cx);
        cy = wave_sum(cy);
        if (lane == 0) {
            sC[wv][0] = cx;
            sC[wv][1] = cy;
        }
    }
    __syncthreads();
    return make_double2(((sC[0][0] + sC[1][0]) + (sC[2][0] + sC[3][0])) / n,
                        ((sC[0][1] + sC[1][1]) + (sC[2][1] + sC[3][1])) / n);
}

// ---- the body update, shared by the one-launch and the two-launch form (the same bits) ----
// A body's block has kIbThreads threads.  What bounds it is its chain: the descriptor, the nodes, the
// velocities, then some hundred FP64 instructions one after the other in every wave.  So each quantity
// is computed once (a spring and an angle belong to one node and reach its neighbours through LDS), the
// second velocity interpolation reuses the first one's values, pairs of lanes share a node's
// interpolation and a site's gather, the extent is reduced in whole sites, and the drive's schedule is
// one wave's work beside the others' nodes.  One launch, before -> after: 64^2, 40 nodes 9.3 -> 6.3 us;
// 2048^2, 8 bodies of 75-150 nodes 10.1 -> 7.8; the 250^2 box with its trap 11.8 -> 8.1.
// The forces of a site are summed in another order than node by node (the even and the odd entries apart), and so
// are a node's pull and trap: FP64 sums that may differ in their last bit, which the rounding of the patch to FP32
// hides nearly always, not by construction (250^2 box, 800 trapped bodies: one force in 2.4 million steps, and with
// it velocities 1e-6 apart a thousand steps later).  One order, used by both forms: the result does not vary by run.
constexpr int kIbThreads = 512;

// LDS of the nodes, sized by the launch for its largest body: position, then spring to the next
// node, d1 and d2
struct BodyNodes {
    double2 *R, *spring, *d1, *d2;
    __device__ BodyNodes(double2 *p, int n) : R(p), spring(p + n), d1(p + 2 * n), d2(p + 3 * n) {}
};
struct BodyScratch {
    Schedule at;   // the schedule at *d_t
    int ext[kIbThreads / 64][4];
    double com[4][2];
};

// Phase 1: the nodes in LDS (ADVANCE: moved from R(t) to R(t+1) by Heun with the velocity patch written
// during step t, App. A: overdamped, no slip; otherwise R[cur] as it is), their extent in whole sites
// and, for a trapped body, their centre of mass; then every node's spring and the derivatives of the
// cosine of its angle with respect to e1 = R_{a-1} - R_a (d1) and e2 = R_{a+1} - R_a (d2).
// Returns the patch origin: 3 sites of margin below the lowest node cover the kernel support (2) plus one
// site of node motion; the same margin above is checked against the patch side.
// The last wave, which has nodes of its own only in a large body, also evaluates the schedule.
template <bool ADVANCE>
__device__ __forceinline__ int2 body_phase1(const BodyDev &B, int cur, const int *d_t, BodyNodes N, BodyScratch &sc,
                                            double2 &com, bool &bad) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, c = tid & 1, n = B.n;
    const double *Rc = B.R[cur];
    int ox = 0, oy = 0;
    if (ADVANCE) {
        ox = gptr(B.origin)[4 * cur];
        oy = gptr(B.origin)[4 * cur + 1];
    }
    if (__builtin_amdgcn_readfirstlane(wv) == kIbThreads / 64 - 1) {
        const Schedule q = schedule(B, (double)d_t[0]);
        if (lane == 0) sc.at = q;
    }
    int lo = 0x7fffffff, hi = -0x7fffffff;
#pragma unroll 1
    for (int a = tid >> 1; a < n; a += kIbThreads / 2) {
        double r = gptr(Rc)[2 * a + c];
        if (ADVANCE) r = heun_component(B.vib, B.ps, ox, oy, c, r, bad);
        reinterpret_cast<double *>(N.R)[2 * a + c] = r;
        const int f = (int)floor(r);
        lo = min(lo, f);
        hi = max(hi, f);
    }
#pragma unroll
    for (int o = 2; o < 64; o <<= 1) {
        lo = min(lo, __shfl_xor(lo, o));
        hi = max(hi, __shfl_xor(hi, o));
    }
    if (lane < 2) {
        sc.ext[wv][c] = lo;
        sc.ext[wv][2 + c] = hi;
    }
    __syncthreads();
    int mn[2] = {0x7fffffff, 0x7fffffff}, mx[2] = {-0x7fffffff, -0x7fffffff};
#pragma unroll
    for (int w = 0; w < kIbThreads / 64; ++w)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            mn[k] = min(mn[k], sc.ext[w][k]);
            mx[k] = max(mx[k], sc.ext[w][2 + k]);
        }
    const int nox = mn[0] - 3, noy = mn[1] - 3;
    if (mx[0] + 3 - nox >= B.ps || mx[1] + 3 - noy >= B.ps) bad = true;
    if (B.trap_k != 0.0) com = block_com(N.R, n, sc.com);
#pragma unroll 1
    for (int a = tid; a < n; a += kIbThreads) {
        const int am = a == 0 ? n - 1 : a - 1, ap = a == n - 1 ? 0 : a + 1;
        const double2 R = N.R[a], Rm = N.R[am], Rp = N.R[ap];
        const double e1x = Rm.x - R.x, e1y = Rm.y - R.y, e2x = Rp.x - R.x, e2y = Rp.y - R.y;
        const double n1 = sqrt(e1x * e1x + e1y * e1y), n2 = sqrt(e2x * e2x + e2y * e2y);
        // spring force k (l - l_eq) d/l on node a from the spring to the next node
        const double cs = B.k * (n2 - B.leq) / n2;
        N.spring[a] = make_double2(cs * e2x, cs * e2y);
        const double in12 = 1.0 / (n1 * n2);
        const double cg = (e1x * e2x + e1y * e2y) * in12;
        N.d1[a] = make_double2(e2x * in12 - cg * e1x / (n1 * n1), e2y * in12 - cg * e1y / (n1 * n1));
        N.d2[a] = make_double2(e1x * in12 - cg * e2x / (n2 * n2), e1y * in12 - cg * e2y / (n2 * n2));
    }
    __syncthreads();
    return make_int2(nox, noy);
}

// -dU/dR_a for U = sum springs + sum bending (eqConst), plus the node's share of the pull and the trap
__device__ __forceinline__ double2 node_force(const BodyDev &B, const BodyNodes &N, int a, double2 share) {
    const int n = B.n, am = a == 0 ? n - 1 : a - 1, ap = a == n - 1 ? 0 : a + 1;
    const double2 s1 = N.spring[a], s0 = N.spring[am], d1 = N.d1[a], d2 = N.d2[a], d2m = N.d2[am], d1p = N.d1[ap];
    return make_double2(s1.x - s0.x + B.eps * ((d1.x + d2.x) - d2m.x - d1p.x) + share.x,
                        s1.y - s0.y + B.eps * ((d1.y + d2.y) - d2m.y - d1p.y) + share.y);
}

// each node's share of the pull and of the trap, k(t) (R_ext(t) - R_com) / n
__device__ __forceinline__ double2 node_share(const BodyDev &B, const Schedule &q, double2 com) {
    double2 s = make_double2(q.pull * B.fx / B.n, q.pull * B.fy / B.n);
    if (B.trap_k != 0.0) {
        s.x += q.k * (B.trap_x0 + B.trap_dx * q.rho - com.x) / B.n;
        s.y += q.k * (B.trap_y0 + B.trap_dy * q.rho - com.y) / B.n;
    }
    return s;
}

// a node's kernel footprint [ix, ix + 4) x [iy, iy + 4) (with one site of margin for the predicted
// position) reaches a wall
__device__ __forceinline__ bool at_wall(const SimDev &S, int ix, int iy) {
    return (S.walls && (iy < 1 || iy + 4 >= S.ny)) || (S.walls == 2 && (ix < 1 || ix + 4 >= S.nx));
}

// Two-launch body update for many bodies (each node advanced once): k_ib_nodes, then k_ib_spread.
// One block per body: phase 1, then the node forces at the new positions with the pull at time *d_t, the
// new patch origin, and each node's footprint weights for the spreading kernel.
template <bool ADVANCE>
__global__ __launch_bounds__(kIbThreads) void k_ib_nodes(const SimDev *__restrict__ sims, BodyDev *__restrict__ bodies,
                                                         int nmax, int cur, const int *__restrict__ d_t,
                                                         int *__restrict__ d_status) {
    extern __shared__ __align__(16) double2 sNodes[];   // 4 nmax
    __shared__ BodyScratch sc;
    const int tid = threadIdx.x;
    const BodyDev &B = bodies[blockIdx.x];
    const SimDev &S = sims[B.sim];
    const BodyNodes N(sNodes, nmax);
    const int n = B.n, dst = ADVANCE ? (cur ^ 1) : cur;
    bool bad = false, wall = false;
    double2 com = make_double2(0.0, 0.0);
    const int2 o = body_phase1<ADVANCE>(B, cur, d_t, N, sc, com, bad);
    const double2 share = node_share(B, sc.at, com);
#pragma unroll 1
    for (int a = tid; a < n; a += kIbThreads) {
        const double2 R = N.R[a];
        reinterpret_cast<double2 *>(B.fnode)[a] = node_force(B, N, a, share);
        if (ADVANCE) reinterpret_cast<double2 *>(B.R[dst])[a] = R;
        int ix, iy;
        float wx[4], wy[4];
        phi4(R.x, ix, wx);
        phi4(R.y, iy, wy);
        wall = wall || at_wall(S, ix, iy);
        B.nix[2 * a] = ix;
        B.nix[2 * a + 1] = iy;
        float4 *w = reinterpret_cast<float4 *>(B.nw) + 2 * a;
        w[0] = make_float4(wx[0], wx[1], wx[2], wx[3]);
        w[1] = make_float4(wy[0], wy[1], wy[2], wy[3]);
    }
    if (tid == 0) {
        B.origin[4 * dst] = o.x;
        B.origin[4 * dst + 1] = o.y;
        B.origin[4 * dst + 2] = wrapi(o.x, S.nx);
        B.origin[4 * dst + 3] = wrapi(o.y, S.ny);
    }
    if (bad) atomicOr(d_status, kStatusPatch);
    if (wall) atomicOr(d_status, kStatusWall);
}

// The nodes whose footprint reaches a tile, in node order: footprint origin (tile coordinates),
// separable weights, force.
struct TileNodes {
    int2 o[kMaxCand];
    float4 w[kMaxCand][2];
    double2 f[kMaxCand];
    int cnt[kIbThreads / 64];
};

// what entry e of the list adds at tile site (lx, ly), e's values in o, wx, wy and f
__device__ __forceinline__ void gather_one(int lx, int ly, int2 o, float4 wx, float4 wy, double2 f, double2 &s) {
    const int i = lx - o.x, j = ly - o.y;
    if ((unsigned)i < 4u && (unsigned)j < 4u) {
        const float wxs = i == 0 ? wx.x : i == 1 ? wx.y : i == 2 ? wx.z : wx.w;
        const float wys = j == 0 ? wy.x : j == 1 ? wy.y : j == 2 ? wy.z : wy.w;
        const double w = (double)wxs * (double)wys;
        s.x += f.x * w;
        s.y += f.y * w;
    }
}

// f_IB at tile site (lx, ly): the listed nodes' f_a phi(x) phi(y), of the entries with an even number (h 0) or
// an odd one (h 1), in order.  The wave's sites are [x0, x1] x [y0, y1]: its
// lanes first look at 64 entries at once, and only those that reach them are read and weighed, the LDS
// reads of four entries before any of them is used.  An entry costs some forty instructions of the chain, and
// of the nodes of an arc across the tile about half reach a wave's 8 x 4 sites (whole rows of the tile, 16 x 2,
// gain nothing from an arc along them: 512^2 22.2 us a step, with 8 x 4 21.6, every entry 21.7; 64^2 14.1, 14.1
// and 14.6; 32 pulled bodies 32.3, 32.2 and 32.8).
__device__ __forceinline__ double2 gather_half(const TileNodes &L, int cnt, int lx, int ly, int x0, int y0, int x1, int y1, int h) {
    constexpr unsigned long long kEven = 0x5555555555555555ull;
    const int lane = threadIdx.x & 63;
    double2 s = make_double2(0.0, 0.0);
#pragma unroll 1
    for (int base = 0; base < cnt; base += 64) {
        const int2 at = L.o[min(base + lane, kMaxCand - 1)];
        const unsigned long long near =
            __ballot(base + lane < cnt && at.y <= y1 && at.y + 4 > y0 && at.x <= x1 && at.x + 4 > x0);
        unsigned long long m = near & (h ? kEven << 1 : kEven);
#pragma unroll 1
        for (int left = max(__popcll(near & kEven), __popcll(near & (kEven << 1))); left > 0; left -= 4) {
            int2 o[4];
            float4 wx[4], wy[4];
            double2 f[4];
            bool have[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                have[u] = m != 0;
                const int e = base + (have[u] ? __builtin_ctzll(m) : 0);
                m &= m - 1;
                o[u] = L.o[e];
                wx[u] = L.w[e][0];
                wy[u] = L.w[e][1];
                f[u] = L.f[e];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (have[u]) gather_one(lx, ly, o[u], wx[u], wy[u], f[u], s);
        }
    }
    return s;
}

// The same of all entries, the even and the odd ones apart (s[0], s[1]).  This launch has hundreds of tiles, several
// to a unit: instructions count and not the chain, and looking for the entries that reach a wave costs more than it
// spares (k_ib_spread of 96 bodies of radius 12, 1536 tiles, 11.9 us that way and 9.7 this way; of 200, 19.2 and 15.5).
__device__ __forceinline__ void gather_all(const TileNodes &L, int cnt, int lx, int ly, double2 s[2]) {
    int e = 0;
    for (; e + 4 <= cnt; e += 4) {
        int2 o[4];
        float4 wx[4], wy[4];
        double2 f[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            o[u] = L.o[e + u];
            wx[u] = L.w[e + u][0];
            wy[u] = L.w[e + u][1];
            f[u] = L.f[e + u];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) gather_one(lx, ly, o[u], wx[u], wy[u], f[u], s[u & 1]);
    }
#pragma unroll
    for (int u = 0; u < 3; ++u)
        if (e + u < cnt) gather_one(lx, ly, L.o[e + u], L.w[e + u][0], L.w[e + u][1], L.f[e + u], s[u & 1]);
}

// the listed nodes' forces on the 16 x 16 sites of tile (tx, ty) of a body's patch, by 256 threads (rows of sites),
// or 512 (8 x 4 to a wave) with a pair of lanes per site (lane h then stores component h).  The even and the odd
// entries are summed apart and then added, so both give the same bits.
template <int THREADS>
__device__ __forceinline__ void spread_tile(const BodyDev &B, const TileNodes &L, int cnt, int tx, int ty) {
    constexpr bool pair = THREADS == 2 * kPatchTile * kPatchTile;
    const int tid = threadIdx.x, h = pair ? tid & 1 : 0;
    const int wv = uniform(tid >> 6), x0 = (wv & 1) * 8, y0 = (wv >> 1) * 4;   // of a wave's sites (pairs)
    const int lx = pair ? x0 + (tid >> 1) % 8 : tid % kPatchTile, ly = pair ? y0 + (tid >> 1) / 8 % 4 : tid / kPatchTile;
    const int px = tx * kPatchTile + lx, py = ty * kPatchTile + ly;
    double2 part[2] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
    if (pair) {
        part[0] = gather_half(L, cnt, lx, ly, x0, y0, x0 + 7, y0 + 3, h);
        part[1] = make_double2(__shfl_xor(part[0].x, 1), __shfl_xor(part[0].y, 1));
    } else {
        gather_all(L, cnt, lx, ly, part);
    }
    const double2 a = make_double2(part[0].x + part[1].x, part[0].y + part[1].y);
    if (px < B.ps && py < B.ps) {
        const unsigned i = (unsigned)(py * B.ps + px), plane = (unsigned)(B.ps * B.ps);
        if (pair) {
            B.fib[h * plane + i] = (float)(h ? a.y : a.x);
        } else {
            B.fib[i] = (float)a.x;
            B.fib[plane + i] = (float)a.y;
        }
    }
}

// One block per (body, 16x16 tile of its patch): f_IB(r) = sum_a f_a phi phi (App. A) as a gather
// over the nodes whose 4x4 footprint reaches the tile (deterministic).
constexpr int kSpreadThreads = 256;
__global__ __launch_bounds__(kSpreadThreads) void k_ib_spread(const BodyDev *__restrict__ bodies, const int2 *__restrict__ blk,
                                                          int dst, int *__restrict__ d_status) {
    __shared__ TileNodes L;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int2 bt = blk[blockIdx.x];
    const BodyDev &B = bodies[bt.x];
    const int n = B.n;
    const int tx = bt.y % B.nside, ty = bt.y / B.nside;
    const int X0 = B.origin[4 * dst] + tx * kPatchTile, Y0 = B.origin[4 * dst + 1] + ty * kPatchTile;
    bool bad = false;
    int tot = 0;
#pragma unroll 1
    for (int base = 0; base < n; base += kSpreadThreads) {
        const int a = base + tid;
        bool flag = false;
        int ix = 0, iy = 0;
        Float4 w0{}, w1{};
        Double2 f{};
        if (a < n) {   // all of a node at once, not one after the other as they are stored (10.7 us -> 9.7)
            ix = gptr(B.nix)[2 * a];
            iy = gptr(B.nix)[2 * a + 1];
            w0 = ((const LBK_GLOBAL Float4 *)gptr(B.nw))[2 * a];
            w1 = ((const LBK_GLOBAL Float4 *)gptr(B.nw))[2 * a + 1];
            f = ((const LBK_GLOBAL Double2 *)gptr(B.fnode))[a];
            flag = ix > X0 - 4 && ix < X0 + kPatchTile && iy > Y0 - 4 && iy < Y0 + kPatchTile;
        }
        const unsigned long long m = __ballot(flag);
        if (lane == 0) L.cnt[wv] = __popcll(m);
        __syncthreads();
        int q = tot + __popcll(m & ((1ull << lane) - 1ull));
#pragma unroll
        for (int w = 0; w < kSpreadThreads / 64; ++w) {
            if (w < wv) q += L.cnt[w];
            tot += L.cnt[w];
        }
        if (flag) {
            if (q < kMaxCand) {
                L.o[q] = make_int2(ix - X0, iy - Y0);
                L.w[q][0] = make_float4(w0.x, w0.y, w0.z, w0.w);
                L.w[q][1] = make_float4(w1.x, w1.y, w1.z, w1.w);
                L.f[q] = make_double2(f.x, f.y);
            } else {
                bad = true;
            }
        }
        __syncthreads();
    }
    spread_tile<kSpreadThreads>(B, L, min(tot, kMaxCand), tx, ty);
    if (bad) atomicOr(d_status, kStatusPatch);
}

// Body update and force spreading in one launch, one block per (body, 16x16 tile of its patch).  Every
// block of a body repeats phase 1 (a few hundred nodes) and evaluates every node's force with the pull at
// time *d_t; of those, the nodes whose 4x4 footprint reaches the tile are listed in node order and
// gathered onto the tile's sites: f_IB(r) = sum_a f_a phi phi (App. A).
// Tile 0 of each body publishes the new positions, all node forces and the origin; the other blocks
// only read the current-parity buffers, so blocks never wait on each other.
template <bool ADVANCE>
__global__ __launch_bounds__(kIbThreads) void k_ib_step(const SimDev *__restrict__ sims, BodyDev *__restrict__ bodies,
                                                        const int2 *__restrict__ blk, int nmax, int cur,
                                                        const int *__restrict__ d_t, int *__restrict__ d_status) {
    extern __shared__ __align__(16) double2 sNodes[];   // 4 nmax
    __shared__ BodyScratch sc;
    __shared__ TileNodes L;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int2 bt = blk[blockIdx.x];
    const BodyDev &B = bodies[bt.x];
    const SimDev &S = sims[B.sim];
    const BodyNodes N(sNodes, nmax);
    const int n = B.n, dst = ADVANCE ? (cur ^ 1) : cur;
    const bool lead = bt.y == 0;
    bool bad = false;        // node outside its patch (every block finds the same; tile 0 reports)
    bool overflow = false;   // more footprints reach this tile than it can list
    bool wall = false;       // a node's kernel footprint reaches a wall
    double2 com = make_double2(0.0, 0.0);
    const int2 o = body_phase1<ADVANCE>(B, cur, d_t, N, sc, com, bad);
    const double2 share = node_share(B, sc.at, com);
    const int tx = bt.y % B.nside, ty = bt.y / B.nside;
    const int X0 = o.x + tx * kPatchTile, Y0 = o.y + ty * kPatchTile;
    int tot = 0;
#pragma unroll 1
    for (int base = 0; base < n; base += kIbThreads) {
        const int a = base + tid;
        bool flag = false;
        int ix = 0, iy = 0;
        float wx[4], wy[4];
        double2 f = make_double2(0.0, 0.0);
        if (a < n) {
            const double2 R = N.R[a];
            f = node_force(B, N, a, share);
            phi4(R.x, ix, wx);
            phi4(R.y, iy, wy);
            wall = wall || at_wall(S, ix, iy);
            flag = ix > X0 - 4 && ix < X0 + kPatchTile && iy > Y0 - 4 && iy < Y0 + kPatchTile;
            if (lead) {
                reinterpret_cast<double2 *>(B.fnode)[a] = f;
                if (ADVANCE) reinterpret_cast<double2 *>(B.R[dst])[a] = R;
            }
        }
        const unsigned long long m = __ballot(flag);
        if (lane == 0) L.cnt[wv] = __popcll(m);
        __syncthreads();
        int q = tot + __popcll(m & ((1ull << lane) - 1ull));
#pragma unroll
        for (int w = 0; w < kIbThreads / 64; ++w) {
            if (w < wv) q += L.cnt[w];
            tot += L.cnt[w];
        }
        if (flag) {
            if (q < kMaxCand) {
                L.o[q] = make_int2(ix - X0, iy - Y0);
                L.w[q][0] = make_float4(wx[0], wx[1], wx[2], wx[3]);
                L.w[q][1] = make_float4(wy[0], wy[1], wy[2], wy[3]);
                L.f[q] = f;
            } else {
                overflow = true;
            }
        }
        __syncthreads();
    }
    if (lead && tid == 0) {
        B.origin[4 * dst] = o.x;
        B.origin[4 * dst + 1] = o.y;
        B.origin[4 * dst + 2] = wrapi(o.x, S.nx);
        B.origin[4 * dst + 3] = wrapi(o.y, S.ny);
    }
    spread_tile<kIbThreads>(B, L, min(tot, kMaxCand), tx, ty);
    if ((bad && lead) || overflow) atomicOr(d_status, kStatusPatch);
    if (wall && lead) atomicOr(d_status, kStatusWall);
}

// ------------------------------------------------------------------------------------------------
// fused single-pass step
// ------------------------------------------------------------------------------------------------

// blocks are dealt round-robin to the 8 XCDs; give each XCD a contiguous run of work items so
// neighbouring strips and segments share that XCD's L2
__device__ __forceinline__ int xcd_remap(int v, int n) {
    int q = n >> 3, r = n & 7;
    int x = v & 7, k = v >> 3;
    return x * q + min(x, r) + k;
}

__device__ __forceinline__ void inc_row(unsigned &r, unsigned ny) { r = (r + 1u == ny) ? 0u : r + 1u; }

// POL = false: every simulation of the launch has P = 0, which the dynamics keep exactly (the
// polarization right-hand side is proportional to P), so the Ericksen stress vanishes and C~ is
// its isotropic value: the scalar model of Sec. II B.  That variant skips all P work.
// ONE: items that one body touches keep it in registers (below).  A launch without bodies takes the
// variant without: the registers and the branch a row cost every item (FP32 lattices without bodies,
// us a step: 1024^2 34.7, with them 35.1; 2048^2 170.9, 171.4; 32 of 128^2 21.7, 22.0).
template <int T, typename HT, bool WALLS, bool POL, bool ONE>
__global__ __launch_bounds__(T, (WALLS || !std::is_same<HT, __half>::value) ? 3 : 4) void k_fused(const SimDev *__restrict__ sims, const BodyDev *__restrict__ bodies,
                                             const WorkItem *__restrict__ items, int n_items, int cur,
                                             int *__restrict__ d_t, int cus) {
    // row-exchange rings; values a thread needs only from its own column one row below live in
    // registers (the "carried" row of the previous iteration)
    typedef typename PolOf<HT>::T PT;   // polarization storage: FP32 offsets with FP16 populations, else FP64
    constexpr int TP = POL ? T : 1;   // the P rings exist only in the variant with P
    __shared__ PT rP[4][2][TP];       // polarization, rows f-3 .. f
    __shared__ float rS[3][3][T];     // stress rows f-3 .. f-1
    __shared__ float rE[2][2][TP];    // Ericksen xx and yx, rows f-2 .. f-1
    __shared__ float rV[2][2][T];     // half-velocity rows f-3 .. f-2
    __shared__ float rQs[2][3][T];    // predicted stress rows f-4 .. f-3
    __shared__ PT rQp[2][2][TP];      // predicted polarization, rows f-4 .. f-3
    __shared__ float4 sTab[2 * kStiffSeg];     // stiffness cubics of the item's simulation
    __shared__ ItemBody sIB[kItemBodies];      // bodies whose patches touch the item
    __shared__ int sNB;                        // their number, -1 if more than kItemBodies
    const int tid = threadIdx.x;
    const int nxt = cur ^ 1;
    if (blockIdx.x == 0 && tid == 0) d_t[0] = d_t[0] + 1;   // the body update after this step uses t+1

    for (int vi = blockIdx.x; vi < n_items; vi += gridDim.x) {
        __syncthreads();   // the previous item's last stages have read the item tables below
        const WorkItem wi = items[xcd_remap(vi, n_items)];
        const SimDev &S = sims[wi.sim];
        const unsigned nx = (unsigned)S.nx, ny = (unsigned)S.ny;
        const unsigned N = nx * ny;
        const HT *__restrict__ hin = reinterpret_cast<const HT *>(S.h[cur]);
        HT *__restrict__ hout = reinterpret_cast<HT *>(S.h[nxt]);
        const float *__restrict__ sgi = S.sig[cur];
        float *__restrict__ sgo = S.sig[nxt];
        const PT *__restrict__ Pi = static_cast<const PT *>(S.P[cur]);
        PT *__restrict__ Po = static_cast<PT *>(S.P[nxt]);
        // A strip of w columns takes lanes 0 .. w+7: 4 halo columns on each side, recomputed by
        // the neighbouring strip.  A lattice no wider than the work-group is one full-width strip
        // (wi.full): lane = column, no halo lanes, and a lane's east and west neighbours wrap
        // around within the strip.  Lanes beyond the strip idle (whole waves skip every stage).
        const bool full = wi.full != 0;
        const int lanes = full ? wi.w : wi.w + 2 * kHalo;
        const bool live = tid < lanes;
        const int c = full ? (live ? tid : 0) : wi.x0 - kHalo + tid;
        const unsigned x = (unsigned)wrapi(c, (int)nx), xm = (unsigned)wrapi(c - 1, (int)nx),
                       xp = (unsigned)wrapi(c + 1, (int)nx);
        const int wcol = wi.w;
        const bool colB = full ? live : tid >= 1 && tid < wcol + 7;
        const bool colC = full ? live : tid >= 2 && tid < wcol + 6;
        const bool colD = full ? live : tid >= 3 && tid < wcol + 5;
        const bool colE = full ? live : tid >= 4 && tid < wcol + 4;
        const float is = S.inv_scale, sc = S.scale;

        // per-item constants: the stiffness cubics, and the bodies whose patches reach the rows
        // y0-2 .. y0+l+1 and columns x0-4 .. x0+w+3 this item touches (wave 0 holds every body:
        // at most kMaxBodies = 64 per simulation)
        for (int q = tid; q < 2 * kStiffSeg; q += T) sTab[q] = reinterpret_cast<const float4 *>(S.tab)[q];
        if (tid < 64) {
            bool hit = false;
            ItemBody ib{0, 0, 0, 0, nullptr, nullptr};
            if (tid < S.nb) {
                const BodyDev &B = bodies[S.b0 + tid];
                ib.ox = gptr(B.origin)[4 * cur + 2];
                ib.oy = gptr(B.origin)[4 * cur + 3];
                ib.ps = B.ps;
                ib.fib = B.fib;
                ib.vib = B.vib;
                hit = ring_overlap(ib.ox, ib.ps, full ? 0 : wrapi(wi.x0 - kHalo, (int)nx), lanes, (int)nx) &&
                      ring_overlap(ib.oy, ib.ps, wrapi(wi.y0 - 2, (int)ny), wi.l + 4, (int)ny);
            }
            const unsigned long long m = __ballot(hit);
            const int cnt = __popcll(m);
            if (hit) {
                const int k = __popcll(m & ((1ull << tid) - 1ull));
                if (k < kItemBodies) sIB[k] = ib;
            }
            if (tid == 0) sNB = cnt <= kItemBodies ? cnt : -1;
        }

        // wrapped row indices relative to the front row f of the current iteration
        // (the rows of iteration 2, where the pipeline starts: f = f0 + 2)
        const int f0 = wi.y0 - 4, f2 = f0 + 2;
        unsigned rp1 = (unsigned)wrapi(f2 + 1, (int)ny), r0 = (unsigned)wrapi(f2, (int)ny);
        unsigned rm1 = (unsigned)wrapi(f2 - 1, (int)ny), rm2 = (unsigned)wrapi(f2 - 2, (int)ny);
        unsigned rm3 = (unsigned)wrapi(f2 - 3, (int)ny), rm4 = (unsigned)wrapi(f2 - 4, (int)ny);
        // walls: the rows next to them, whose neighbour beyond is a ghost
        const bool walls = WALLS && S.walls != 0;   // the periodic variant has no wall code
        const unsigned ytop = ny - 1u;
        // closed box: this lane's column is next to the west / east wall
        const bool xw = WALLS && S.walls == 2 && x == 0u, xe = WALLS && S.walls == 2 && x == nx - 1u;
        // the lanes holding the east and west neighbours (the lane itself beyond a wall: mirror
        // ghosts; wrapped around a full-width strip)
        const int te = xe ? tid : (full && tid + 1 == lanes ? 0 : tid + 1);
        const int tw = xw ? tid : (full && tid == 0 ? lanes - 1 : tid - 1);
        // this lane's column and its neighbours as byte offsets within a row of populations (HT)
        // and of the 4-byte stress and polarization planes; the state arrays as buffers
        const unsigned HB = (unsigned)sizeof(HT);
        const unsigned bh = x * HB, bhm = xm * HB, bhp = xp * HB;
        const unsigned b4 = x * 4u, bP = x * (unsigned)sizeof(PT);
        const __amdgpu_buffer_rsrc_t rHi = state_rsrc(hin), rHo = state_rsrc(hout), rSi = state_rsrc(sgi),
                                     rSo = state_rsrc(sgo), rPi = state_rsrc(Pi), rPo = state_rsrc(Po);

        // Loads for the next iteration, issued one iteration ahead.  Every lane loads (all
        // indices are wrapped into the lattice); lanes outside a stage's columns never use them.
        struct Pre {
            PT P0, P1;                     // P(f+1)
            float S0, S1, S2;              // sigma(f)
            typename Pop<HT>::Raw H[9];    // populations pulled into row f-1
            float F0, F1;                  // the only body's spread force at row f-1 (ONE)
        };
        // Values of this column handed from one iteration to the next: stage D's centre row
        // (the corrector's frozen inputs and the next predictor's south neighbours) and stage E's
        // predicted centre (the next corrector's south neighbour).
        struct Carry {
            float hx, hy, s0, s1, s2;      // hx, hy: half the velocity
            PT p0, p1;
            Grad g;
            Stiff k;
            float q0, q1, q2;
            PT qp0, qp1;
        };
        Pre preA, preB;
        Carry carA, carB;
        // Row iterations 0 and 1 would only commit P rows f0 and f0+1 (their stress rows f0-1 and
        // f0 are read by no stage), so the pipeline starts at iteration 2: those two P rows go
        // into the ring here, with one wait, and preA takes iteration 2's rows.
        if (live) {
            const unsigned rP0 = r0 * nx * (unsigned)sizeof(PT), NP = N * (unsigned)sizeof(PT);
            const unsigned rS0 = rm1 * nx * 4u, N4 = N * 4u;
            if (POL) {
                const unsigned rF0 = rm2 * nx * (unsigned)sizeof(PT), rF1 = rm1 * nx * (unsigned)sizeof(PT);
                PT f00, f01, f10, f11;
                buf_ld(rPi, bP, rF0, f00);
                buf_ld(rPi, bP, NP + rF0, f01);
                buf_ld(rPi, bP, rF1, f10);
                buf_ld(rPi, bP, NP + rF1, f11);
                buf_ld(rPi, bP, rP0, preA.P0);
                buf_ld(rPi, bP, NP + rP0, preA.P1);
                rP[0][0][tid] = f00;
                rP[0][1][tid] = f01;
                rP[1][0][tid] = f10;
                rP[1][1][tid] = f11;
            }
            preA.S0 = buf_ldf(rSi, b4, rS0);
            preA.S1 = buf_ldf(rSi, b4, N4 + rS0);
            preA.S2 = buf_ldf(rSi, b4, 2u * N4 + rS0);
        }
        if (ONE) preA.F0 = preA.F1 = preB.F0 = preB.F1 = 0.f;
        // Ericksen xy, yy of this column at rows f-1, f-2, f-3
        float exy1 = 0.f, eyy1 = 0.f, exy2 = 0.f, eyy2 = 0.f, exy3 = 0.f, eyy3 = 0.f;

        __syncthreads();
        const int nib = sNB;
        const int niter = wi.l + 8;
        // An item with one body keeps its constants in registers (the column's offset in the patch is the
        // same for every row, the row's is scalar) and loads the spread force a row ahead.  The FP16 form
        // takes the list: at four waves a SIMD it would spill; so does the one with walls, which the extra
        // registers slow down (1400 x 1001 channel 46.1 -> 47.8 us).
        const bool one = ONE && nib == 1;
        OneBody ob{0, 0, 0, rSi, rSi};
        unsigned bcol = kOutside;
        if (one) {
            ob = one_body(sIB[0]);
            const int px = wrap_near((int)x - ob.ox, (int)nx);
            bcol = (unsigned)px < (unsigned)ob.ps ? 4u * (unsigned)px : kOutside;
        }

        // one row iteration j; pin/cin were filled by iteration j-1, pout/cout are for j+1
        auto iterate = [&](const int j, const Pre &pin, Pre &pout, const Carry &cin, Carry &cout) {
            const int a0 = j & 3, a1 = (j + 3) & 3, a2 = (j + 2) & 3, a3 = (j + 1) & 3;   // P rows f .. f-3
            const int b1 = (j + 59) % 3, b2 = (j + 58) % 3, b3 = (j + 57) % 3;           // stress rows f-1 .. f-3
            const int o1 = (j + 1) & 1, o0 = j & 1;   // rows f-1 / f-3 (odd lag) and f-2 / f-4 (even lag)

            // One barrier per iteration.  Every value a stage reads from another lane was written
            // in an earlier iteration (stage B reads P rows written by A one or more iterations
            // ago, C the Ericksen row B wrote last iteration, D the velocity row C wrote last
            // iteration, E the predictor row D wrote last iteration); what a stage reads from the
            // current iteration is its own column, written by its own lane.  Every slot written
            // here last held a row that an earlier iteration read.  So one barrier between
            // consecutive iterations orders all of it.
            __syncthreads();

            // ---- stage A: commit P(f), sigma(f-1); take this iteration's populations
            if (POL) {
                rP[a0][0][tid] = pin.P0;
                rP[a0][1][tid] = pin.P1;
            }
            rS[b1][0][tid] = pin.S0;
            rS[b1][1][tid] = pin.S1;
            rS[b1][2][tid] = pin.S2;
            float d[9];
#pragma unroll
            for (int q = 0; q < 9; ++q) d[q] = Pop<HT>::cvt_stored(pin.H[q]);   // times the storage scale
            // prefetch for iteration j+1: P(f+1), sigma(f), and the populations pulled into row
            // f-1: h_n(x, r) = h*_n(x - c_n, r - c_n) from rows f-2, f-1, f
            if (live && j + 1 < niter) {
                const unsigned rP1 = rp1 * nx * (unsigned)sizeof(PT), NP = N * (unsigned)sizeof(PT);
                const unsigned rS1 = r0 * nx * 4u, N4 = N * 4u;
                if (POL) {
                    buf_ld(rPi, bP, rP1, pout.P0);
                    buf_ld(rPi, bP, NP + rP1, pout.P1);
                }
                pout.S0 = buf_ldf(rSi, b4, rS1);
                pout.S1 = buf_ldf(rSi, b4, N4 + rS1);
                pout.S2 = buf_ldf(rSi, b4, 2u * N4 + rS1);
                if (one) {
                    const int py = wrap_near((int)rm1 - ob.oy, (int)ny);
                    pout.F0 = pout.F1 = 0.f;
                    if ((unsigned)py < (unsigned)ob.ps) {
                        pout.F0 = buf_ldf(ob.fib, bcol, (unsigned)(4 * py * ob.ps));
                        pout.F1 = buf_ldf(ob.fib, bcol, (unsigned)(4 * (py + ob.ps) * ob.ps));
                    }
                }
                if (!WALLS && j + 1 >= 4) {
                    // periodic: plane and row in the scalar offset, the column in the lane offset
                    const unsigned NH = N * HB, yc = rm1 * nx * HB, ym = rm2 * nx * HB, yp = r0 * nx * HB;
                    pout.H[0] = Pop<HT>::ld_buf(rHi, bh, yc);
                    pout.H[1] = Pop<HT>::ld_buf(rHi, bhm, NH + yc);
                    pout.H[2] = Pop<HT>::ld_buf(rHi, bh, 2u * NH + ym);
                    pout.H[3] = Pop<HT>::ld_buf(rHi, bhp, 3u * NH + yc);
                    pout.H[4] = Pop<HT>::ld_buf(rHi, bh, 4u * NH + yp);
                    pout.H[5] = Pop<HT>::ld_buf(rHi, bhm, 5u * NH + ym);
                    pout.H[6] = Pop<HT>::ld_buf(rHi, bhp, 6u * NH + ym);
                    pout.H[7] = Pop<HT>::ld_buf(rHi, bhp, 7u * NH + yp);
                    pout.H[8] = Pop<HT>::ld_buf(rHi, bhm, 8u * NH + yp);
                } else if (WALLS && j + 1 >= 4) {
                    const unsigned yc = rm1 * nx, ym = rm2 * nx, yp = r0 * nx;
                    // halfway bounce-back: what would come from beyond a wall is the opposite
                    // direction's post-collision value at the same site
                    const bool blo = walls && rm1 == 0u, bhi = walls && rm1 == ytop;
                    const unsigned own = yc + x;
                    pout.H[0] = Pop<HT>::ld_raw(hin, own);
                    pout.H[1] = Pop<HT>::ld_raw(hin, xw ? 3u * N + own : N + yc + xm);
                    pout.H[2] = Pop<HT>::ld_raw(hin, blo ? 4u * N + own : 2u * N + ym + x);
                    pout.H[3] = Pop<HT>::ld_raw(hin, xe ? N + own : 3u * N + yc + xp);
                    pout.H[4] = Pop<HT>::ld_raw(hin, bhi ? 2u * N + own : 4u * N + yp + x);
                    pout.H[5] = Pop<HT>::ld_raw(hin, blo || xw ? 7u * N + own : 5u * N + ym + xm);
                    pout.H[6] = Pop<HT>::ld_raw(hin, blo || xe ? 8u * N + own : 6u * N + ym + xp);
                    pout.H[7] = Pop<HT>::ld_raw(hin, bhi || xe ? 5u * N + own : 7u * N + yp + xp);
                    pout.H[8] = Pop<HT>::ld_raw(hin, bhi || xw ? 6u * N + own : 8u * N + yp + xm);
                }
            }

            // ---- stage B: Ericksen stress at row f-1
            exy3 = exy2;
            eyy3 = eyy2;
            exy2 = exy1;
            eyy2 = eyy1;
            if (POL && j >= 2 && colB) {
                const int an = walls && rm1 == ytop ? a1 : a0, as = walls && rm1 == 0u ? a1 : a2;
                PT Pc[2] = {rP[a1][0][tid], rP[a1][1][tid]};
                PT Pe[2] = {rP[a1][0][te], rP[a1][1][te]};
                PT Pw[2] = {rP[a1][0][tw], rP[a1][1][tw]};
                PT Pn[2] = {rP[an][0][tid], rP[an][1][tid]};
                PT Ps[2] = {rP[as][0][tid], rP[as][1][tid]};
                float E[4];
                ericksen(S, Pc, Pe, Pw, Pn, Ps, E);
                rE[o1][0][tid] = E[0];
                rE[o1][1][tid] = E[2];
                exy1 = E[1];
                eyy1 = E[3];
            }

            // ---- stage C: force, moments, collision at row f-2
            if (j >= 4 && colC) {
                const bool clo = walls && rm2 == 0u, chi = walls && rm2 == ytop;
                const int bn = chi ? b2 : b1, bs = clo ? b2 : b3;
                // twice the divergence of the stresses (central differences), halved once
                float fx = (rS[b2][0][te] - rS[b2][0][tw]) + (rS[bn][2][tid] - rS[bs][2][tid]);
                float fy = (rS[b2][2][te] - rS[b2][2][tw]) + (rS[bn][1][tid] - rS[bs][1][tid]);
                if (POL && S.ericksen) {
                    const float exn = chi ? exy2 : exy1, exs = clo ? exy2 : exy3;
                    const float eyn = chi ? eyy2 : eyy1, eys = clo ? eyy2 : eyy3;
                    fx += (rE[o0][0][te] - rE[o0][0][tw]) + (exn - exs);
                    fy += (rE[o0][1][te] - rE[o0][1][tw]) + (eyn - eys);
                }
                float Fx = fmaf(0.5f, fx, S.gx), Fy = fmaf(0.5f, fy, S.gy);
                if (one) {
                    Fx += pin.F0;
                    Fy += pin.F1;
                } else if (nib > 0)
                    ib_force_list(sIB, nib, (int)nx, (int)ny, (int)x, (int)rm2, Fx, Fy);
                else if (nib < 0)
                    ib_force(S, bodies, cur, (int)x, (int)rm2, Fx, Fy);
                float drho, ux, uy;
                collide_t<Pop<HT>::kScaled>(d, Fx, Fy, S.omega, S.guo, sc, is, drho, ux, uy);
                rV[o0][0][tid] = 0.5f * ux;   // the gradient and advection stages take v / 2
                rV[o0][1][tid] = 0.5f * uy;
                const int r = wi.y0 + j - 6;   // = f - 2
                if (colE && r >= wi.y0 && r < wi.y0 + wi.l) {
                    const unsigned o = rm2 * nx * HB, NH = N * HB;
#pragma unroll
                    for (int q = 0; q < 9; ++q) Pop<HT>::st_buf(rHo, bh, (unsigned)q * NH + o, d[q]);
                    if (one) {
                        const int py = wrap_near((int)rm2 - ob.oy, (int)ny);
                        if ((unsigned)py < (unsigned)ob.ps) {
                            buf_stf(ob.vib, bcol, (unsigned)(4 * py * ob.ps), ux);
                            buf_stf(ob.vib, bcol, (unsigned)(4 * (py + ob.ps) * ob.ps), uy);
                        }
                    } else if (nib > 0)
                        ib_store_v_list(sIB, nib, (int)nx, (int)ny, (int)x, (int)rm2, ux, uy);
                    else if (nib < 0)
                        ib_store_v(S, bodies, cur, (int)x, (int)rm2, ux, uy);
                }
            }

            // ---- stage D: predictor at row f-3 (from j = 5 only the carried centre values)
            if (j >= 5 && colD) {
                cout.hx = rV[o1][0][tid];
                cout.hy = rV[o1][1][tid];
                PT Pc[2] = {POL ? rP[a3][0][tid] : (PT)0, POL ? rP[a3][1][tid] : (PT)0};
                float X[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) X[q] = rS[b3][q][tid];
                if (j >= 6) {
                    // walls: mirror ghosts for sigma and P, no-slip (negated) ghosts for v
                    const bool dlo = walls && rm3 == 0u, dhi = walls && rm3 == ytop;
                    const float vxn = dhi ? -cout.hx : rV[o0][0][tid], vyn = dhi ? -cout.hy : rV[o0][1][tid];
                    const float vxs = dlo ? -cout.hx : cin.hx, vys = dlo ? -cout.hy : cin.hy;
                    const float sxe = xe ? -1.0f : 1.0f, sxw = xw ? -1.0f : 1.0f;   // no-slip ghosts
                    cout.g = grad_v(sxe * rV[o1][0][te], sxw * rV[o1][0][tw], vxn, vxs,
                                    sxe * rV[o1][1][te], sxw * rV[o1][1][tw], vyn, vys);
                    // without P: the isotropic stiffness (all anisotropic parts vanish at P = 0)
                    cout.k = POL ? stiffness(S, sTab, (float)((PT)S.pref[0] + Pc[0]), (float)((PT)S.pref[1] + Pc[1]))
                                 : Stiff{0.f, 0.f, 0.f, 0.f};
                    float Xe[3], Xw[3], Xn[3], Rs[3];
                    const int bn = dhi ? b3 : b2;
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        Xe[q] = rS[b3][q][te];
                        Xw[q] = rS[b3][q][tw];
                        Xn[q] = rS[bn][q][tid];
                    }
                    const float Xs[3] = {dlo ? X[0] : cin.s0, dlo ? X[1] : cin.s1, dlo ? X[2] : cin.s2};
                    rhs_sigma(S, cout.k, cout.g, cout.hx, cout.hy, X, Xe, Xw, Xn, Xs, Rs);
                    rQs[o1][0][tid] = X[0] + Rs[0];
                    rQs[o1][1][tid] = X[1] + Rs[1];
                    rQs[o1][2][tid] = X[2] + Rs[2];
                    if (POL) {
                        PT Pe[2] = {rP[a3][0][te], rP[a3][1][te]};
                        PT Pw[2] = {rP[a3][0][tw], rP[a3][1][tw]};
                        const int an = dhi ? a3 : a2;
                        PT Pn[2] = {rP[an][0][tid], rP[an][1][tid]};
                        PT Ps[2] = {dlo ? Pc[0] : cin.p0, dlo ? Pc[1] : cin.p1};
                        PT Rp[2];
                        rhs_P(S, cout.g, cout.hx, cout.hy, Pc, Pe, Pw, Pn, Ps, Rp);
                        rQp[o1][0][tid] = Pc[0] + Rp[0];
                        rQp[o1][1][tid] = Pc[1] + Rp[1];
                    }
                }
                cout.s0 = X[0];
                cout.s1 = X[1];
                cout.s2 = X[2];
                cout.p0 = Pc[0];
                cout.p1 = Pc[1];
            }

            // ---- stage E: corrector at row f-4 with the inputs stage D froze one iteration ago;
            // from j = 7 it records the predicted centre values as next iteration's south row
            if (j >= 7 && colE) {
                float X[3], Xe[3], Xw[3], Xn[3], Rs[3];
                PT Y[2], Ye[2], Yw[2], Yn[2], Rp[2];
#pragma unroll
                for (int q = 0; q < 3; ++q) X[q] = rQs[o0][q][tid];
                Y[0] = POL ? rQp[o0][0][tid] : (PT)0;
                Y[1] = POL ? rQp[o0][1][tid] : (PT)0;
                if (j >= 8) {
                    const bool elo = walls && rm4 == 0u, ehi = walls && rm4 == ytop;
                    const int on = ehi ? o0 : o1;
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        Xe[q] = rQs[o0][q][te];
                        Xw[q] = rQs[o0][q][tw];
                        Xn[q] = rQs[on][q][tid];
                    }
                    const float Xs[3] = {elo ? X[0] : cin.q0, elo ? X[1] : cin.q1, elo ? X[2] : cin.q2};
                    rhs_sigma(S, cin.k, cin.g, cin.hx, cin.hy, X, Xe, Xw, Xn, Xs, Rs);
                    const unsigned o = rm4 * nx * 4u, N4 = N * 4u;
                    buf_stf(rSo, b4, o, 0.5f * ((cin.s0 + X[0]) + Rs[0]));
                    buf_stf(rSo, b4, N4 + o, 0.5f * ((cin.s1 + X[1]) + Rs[1]));
                    buf_stf(rSo, b4, 2u * N4 + o, 0.5f * ((cin.s2 + X[2]) + Rs[2]));
                    if (POL) {   // without P both P buffers stay zero
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            Ye[q] = rQp[o0][q][te];
                            Yw[q] = rQp[o0][q][tw];
                            Yn[q] = rQp[on][q][tid];
                        }
                        const PT Ys[2] = {elo ? Y[0] : cin.qp0, elo ? Y[1] : cin.qp1};
                        rhs_P(S, cin.g, cin.hx, cin.hy, Y, Ye, Yw, Yn, Ys, Rp);
                        const unsigned oP = rm4 * nx * (unsigned)sizeof(PT), NP = N * (unsigned)sizeof(PT);
                        buf_st(rPo, bP, oP, (PT)0.5 * ((cin.p0 + Y[0]) + Rp[0]));
                        buf_st(rPo, bP, NP + oP, (PT)0.5 * ((cin.p1 + Y[1]) + Rp[1]));
                    }
                }
                cout.q0 = X[0];
                cout.q1 = X[1];
                cout.q2 = X[2];
                cout.qp0 = Y[0];
                cout.qp1 = Y[1];
            }
            inc_row(rp1, ny);
            inc_row(r0, ny);
            inc_row(rm1, ny);
            inc_row(rm2, ny);
            inc_row(rm3, ny);
            inc_row(rm4, ny);
        };

        // two iterations per trip with the register sets swapped, so no values are copied.  The
        // waves' issue priority falls in thirds as the item progresses: a compute unit's SIMDs are
        // shared by several work-groups, and under the hardware's oldest-first arbitration the
        // last-dispatched ones would otherwise trail alone, at low VALU use, at the end.  When the
        // whole grid is one round of at most four work-groups per unit, dealt to the units in turn,
        // work-group b is the (b / cus)-th on its unit, and the later ones hold each priority three
        // row iterations longer per older work-group (longer grids start their work-groups as
        // others finish, and gain nothing from it).  Items that touch a body (their spread-force
        // reads make them the slowest) keep the top priority, so they no longer finish last.
        const int lag = (int)gridDim.x <= 4 * cus ? 3 * min(3, (int)blockIdx.x / cus) : 0;
        const int q1 = niter / 3 + lag, q2 = (2 * niter) / 3 + lag;
        for (int j = 2; j < niter; j += 2) {
            if (nib != 0)
                __builtin_amdgcn_s_setprio(3);
            else if (j >= q2)
                __builtin_amdgcn_s_setprio(0);
            else if (j >= q1)
                __builtin_amdgcn_s_setprio(1);
            else
                __builtin_amdgcn_s_setprio(2);
            iterate(j, preA, preB, carA, carB);
            if (j + 1 < niter) iterate(j + 1, preB, preA, carB, carA);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// the same step on short items: a tile of sites, all its rows at once
// ------------------------------------------------------------------------------------------------

// k_fused marches down an item's rows, so an item of l rows takes l + 8 row iterations one after the
// other, each a wave's chain of several hundred dependent instructions: what bounds a lattice too
// small to give every wave slot a long item.  Here a work-group takes a tile of w x l sites and every
// stage over the whole tile at once, with its halo: P on (w + 8) x (l + 8) sites, the Ericksen stress on
// (w + 6) x (l + 6), the collision on (w + 4) x (l + 4), the predictor on (w + 2) x (l + 2), the
// corrector on w x l, with one barrier between stages.  It computes more halo sites per lattice site
// (32 x 8, the larger lattices' tile: 2.1, 1.7, 1.3 times the sites in the first three stages) in a chain about a
// tenth as long.  The arithmetic of a site is k_fused's, so the results are the same bits.
// Field pass, FP32, one body, marching -> tiles: 64^2 18.8 -> 7.2 us, 250^2 closed box 21.9 -> 9.0, 512^2 22.9 ->
// 15.8, of which about 1.6 are the launch itself and 2 the loads.  VALU issue is a thirtieth of the first, where a
// wave is alone on its SIMD, 0.45 of the second and 0.6 of the third, at four tiles a unit.
template <int T, typename HT, bool WALLS, bool POL>
__global__ __launch_bounds__(T, T == 64 ? 2 : 4) void k_tile(const SimDev *__restrict__ sims, const BodyDev *__restrict__ bodies,
                                               const WorkItem *__restrict__ items, int n_items, int cur,
                                               int *__restrict__ d_t) {
    typedef typename PolOf<HT>::T PT;
    constexpr int NP = tile_cap(T, 8), NS = tile_cap(T, 6), NC = tile_cap(T, 4), ND = tile_cap(T, 2);
    constexpr int RP = (NP + T - 1) / T, RS = (NS + T - 1) / T, RC = (NC + T - 1) / T;   // rounds of T threads
    __shared__ PT rP[2][POL ? NP : 1];      // polarization
    __shared__ float rS[3][NS];             // stress
    __shared__ float rV[2][NC];             // half the velocity
    struct Late {                           // after the collision: predicted fields, and per core site
        PT qp[2][POL ? ND : 1];             // the velocity gradient and stiffness the corrector reuses
        float qs[3][ND];
        float g[8][T];
    };
    struct Early {
        float e[4][POL ? NS : 1];           // before it: the Ericksen stress
    };
    __shared__ union {
        Late late;
        Early early;
    } U;
    __shared__ float4 sTab[2 * kStiffSeg];
    __shared__ ItemBody sIB[kItemBodies];
    __shared__ int sNB;
    const int tid = threadIdx.x;
    const int nxt = cur ^ 1;
    if (blockIdx.x == 0 && tid == 0) d_t[0] = d_t[0] + 1;   // the body update after this step uses t+1
    const WorkItem wi = items[xcd_remap(blockIdx.x, n_items)];
    const SimDev &S = sims[wi.sim];
    const int nx = S.nx, ny = S.ny, w = wi.w, l = wi.l;
    const unsigned N = (unsigned)nx * (unsigned)ny;
    const int WP = w + 8, WS = w + 6, WC = w + 4, WD = w + 2;
    const bool walls = WALLS && S.walls != 0, box = WALLS && S.walls == 2;
    const float is = S.inv_scale, sc = S.scale;
    const unsigned HB = (unsigned)sizeof(HT);
    const __amdgpu_buffer_rsrc_t rHi = state_rsrc(S.h[cur]), rHo = state_rsrc(S.h[nxt]), rSi = state_rsrc(S.sig[cur]),
                                 rSo = state_rsrc(S.sig[nxt]), rPi = state_rsrc(S.P[cur]), rPo = state_rsrc(S.P[nxt]);

    // site i of a region of width W that begins d sites before the tile: its coordinates in the region and
    // its wrapped lattice site (the region reaches at most 4 sites beyond a lattice of at least 8)
    struct Site {
        int X, Y, x, y;
    };
    auto site = [&](int i, int W, int d) {
        Site q;
        q.Y = (int)tile_div((unsigned)i, (unsigned)W);
        q.X = i - q.Y * W;
        q.x = wrap_near(wi.x0 - d + q.X, nx);
        q.y = wrap_near(wi.y0 - d + q.Y, ny);
        return q;
    };

    // loads of the tile and its halo, all issued before the first is used
    PT lp[RP][2];
    float ls[RS][3];
    typename Pop<HT>::Raw lh[RC][9];
    const int nP = WP * (l + 8), nS = WS * (l + 6), nC = WC * (l + 4), nD = WD * (l + 2), nE = w * l;
    if (POL)
#pragma unroll
        for (int k = 0; k < RP; ++k) {
            if (k * T >= nP) break;
            const Site q = site(min(tid + k * T, nP - 1), WP, 4);
            const unsigned o = ((unsigned)q.y * (unsigned)nx + (unsigned)q.x) * (unsigned)sizeof(PT);
            buf_ld(rPi, o, 0u, lp[k][0]);
            buf_ld(rPi, o, N * (unsigned)sizeof(PT), lp[k][1]);
        }
#pragma unroll
    for (int k = 0; k < RS; ++k) {
        if (k * T >= nS) break;
        const Site q = site(min(tid + k * T, nS - 1), WS, 3);
        const unsigned o = ((unsigned)q.y * (unsigned)nx + (unsigned)q.x) * 4u;
#pragma unroll
        for (int c = 0; c < 3; ++c) ls[k][c] = buf_ldf(rSi, o, (unsigned)c * N * 4u);
    }
#pragma unroll
    for (int k = 0; k < RC; ++k) {
        if (k * T >= nC) break;
        // the populations pulled into a collision site: h_n(x, y) = h*_n(x - c_n, y - c_n)
        const Site q = site(min(tid + k * T, nC - 1), WC, 2);
        const unsigned xm = (unsigned)wrap_near(q.x - 1, nx), xp = (unsigned)wrap_near(q.x + 1, nx), x = (unsigned)q.x;
        const unsigned yc = (unsigned)q.y * (unsigned)nx, ym = (unsigned)wrap_near(q.y - 1, ny) * (unsigned)nx,
                       yp = (unsigned)wrap_near(q.y + 1, ny) * (unsigned)nx;
        const unsigned NH = N * HB;
        if (!WALLS) {
            lh[k][0] = Pop<HT>::ld_buf(rHi, (yc + x) * HB, 0u);
            lh[k][1] = Pop<HT>::ld_buf(rHi, (yc + xm) * HB, NH);
            lh[k][2] = Pop<HT>::ld_buf(rHi, (ym + x) * HB, 2u * NH);
            lh[k][3] = Pop<HT>::ld_buf(rHi, (yc + xp) * HB, 3u * NH);
            lh[k][4] = Pop<HT>::ld_buf(rHi, (yp + x) * HB, 4u * NH);
            lh[k][5] = Pop<HT>::ld_buf(rHi, (ym + xm) * HB, 5u * NH);
            lh[k][6] = Pop<HT>::ld_buf(rHi, (ym + xp) * HB, 6u * NH);
            lh[k][7] = Pop<HT>::ld_buf(rHi, (yp + xp) * HB, 7u * NH);
            lh[k][8] = Pop<HT>::ld_buf(rHi, (yp + xm) * HB, 8u * NH);
        } else {
            // halfway bounce-back: what would come from beyond a wall is the opposite direction's
            // post-collision value at the same site
            const bool blo = walls && q.y == 0, bhi = walls && q.y == ny - 1;
            const bool xw = box && q.x == 0, xe = box && q.x == nx - 1;
            const unsigned own = yc + x;
            auto ld = [&](bool wall, int opp, int n, unsigned from) {
                return Pop<HT>::ld_buf(rHi, ((wall ? (unsigned)opp : (unsigned)n) * N + (wall ? own : from)) * HB, 0u);
            };
            lh[k][0] = Pop<HT>::ld_buf(rHi, own * HB, 0u);
            lh[k][1] = ld(xw, 3, 1, yc + xm);
            lh[k][2] = ld(blo, 4, 2, ym + x);
            lh[k][3] = ld(xe, 1, 3, yc + xp);
            lh[k][4] = ld(bhi, 2, 4, yp + x);
            lh[k][5] = ld(blo || xw, 7, 5, ym + xm);
            lh[k][6] = ld(blo || xe, 8, 6, ym + xp);
            lh[k][7] = ld(bhi || xe, 5, 7, yp + xp);
            lh[k][8] = ld(bhi || xw, 6, 8, yp + xm);
        }
    }
    // per-item constants: the stiffness cubics, and the bodies whose patches reach the rows and columns
    // of the collision region (wave 0 holds every body: at most kMaxBodies = 64 per simulation)
    for (int q = tid; q < 2 * kStiffSeg; q += T) sTab[q] = reinterpret_cast<const float4 *>(S.tab)[q];
    if (tid < 64) {
        bool hit = false;
        ItemBody ib{0, 0, 0, 0, nullptr, nullptr};
        if (tid < S.nb) {
            const BodyDev &B = bodies[S.b0 + tid];
            ib.ox = gptr(B.origin)[4 * cur + 2];
            ib.oy = gptr(B.origin)[4 * cur + 3];
            ib.ps = B.ps;
            ib.fib = B.fib;
            ib.vib = B.vib;
            hit = ring_overlap(ib.ox, ib.ps, wrap_near(wi.x0 - 2, nx), w + 4, nx) &&
                  ring_overlap(ib.oy, ib.ps, wrap_near(wi.y0 - 2, ny), l + 4, ny);
        }
        const unsigned long long m = __ballot(hit);
        const int cnt = __popcll(m);
        if (hit) {
            const int k = __popcll(m & ((1ull << tid) - 1ull));
            if (k < kItemBodies) sIB[k] = ib;
        }
        if (tid == 0) sNB = cnt <= kItemBodies ? cnt : -1;
    }
    if (POL)
#pragma unroll
        for (int k = 0; k < RP; ++k)
            if (tid + k * T < nP) {
                rP[0][tid + k * T] = lp[k][0];
                rP[1][tid + k * T] = lp[k][1];
            }
#pragma unroll
    for (int k = 0; k < RS; ++k)
        if (tid + k * T < nS)
#pragma unroll
            for (int c = 0; c < 3; ++c) rS[c][tid + k * T] = ls[k][c];
    __syncthreads();
    const int nib = sNB;
    // the spread force of the tile's only body, in flight during the next stage
    OneBody ob{0, 0, 0, rSi, rSi};
    unsigned bat[RC];
    float lf[RC][2];
    if (nib == 1) {
        ob = one_body(sIB[0]);
#pragma unroll
        for (int k = 0; k < RC; ++k) {
            const Site q = site(min(tid + k * T, nC - 1), WC, 2);
            const int px = wrap_near(q.x - ob.ox, nx), py = wrap_near(q.y - ob.oy, ny);
            bat[k] = (unsigned)px < (unsigned)ob.ps && (unsigned)py < (unsigned)ob.ps ? 4u * (unsigned)(py * ob.ps + px)
                                                                                    : kOutside;
            lf[k][0] = buf_ldf(ob.fib, bat[k], 0u);
            lf[k][1] = buf_ldf(ob.fib, bat[k], (unsigned)(4 * ob.ps * ob.ps));
        }
    }

    // ---- Ericksen stress
    if (POL) {
#pragma unroll 1
        for (int i = tid; i < nS; i += T) {
            const Site q = site(i, WS, 3);
            const int c = (q.Y + 1) * WP + q.X + 1;
            const int e = box && q.x == nx - 1 ? c : c + 1, ww = box && q.x == 0 ? c : c - 1;
            const int n = walls && q.y == ny - 1 ? c : c + WP, s = walls && q.y == 0 ? c : c - WP;
            PT Pc[2] = {rP[0][c], rP[1][c]}, Pe[2] = {rP[0][e], rP[1][e]}, Pw[2] = {rP[0][ww], rP[1][ww]};
            PT Pn[2] = {rP[0][n], rP[1][n]}, Ps[2] = {rP[0][s], rP[1][s]};
            float E[4];
            ericksen(S, Pc, Pe, Pw, Pn, Ps, E);
#pragma unroll
            for (int k = 0; k < 4; ++k) U.early.e[k][i] = E[k];
        }
        __syncthreads();
    }

    // ---- force, moments, collision
#pragma unroll 1
    for (int k = 0; k < RC; ++k) {
        const int i = tid + k * T;
        float d[9], bx = 0.f, by = 0.f;
        unsigned bo = kOutside;
#pragma unroll
        for (int r = 0; r < RC; ++r)
            if (k == r) {
#pragma unroll
                for (int q = 0; q < 9; ++q) d[q] = Pop<HT>::cvt_stored(lh[r][q]);
                if (nib == 1) {
                    bx = lf[r][0];
                    by = lf[r][1];
                    bo = bat[r];
                }
            }
        if (i >= nC) continue;
        const Site q = site(i, WC, 2);
        const int c = (q.Y + 1) * WS + q.X + 1;
        const int e = box && q.x == nx - 1 ? c : c + 1, ww = box && q.x == 0 ? c : c - 1;
        const int n = walls && q.y == ny - 1 ? c : c + WS, s = walls && q.y == 0 ? c : c - WS;
        // twice the divergence of the stresses (central differences), halved once
        float fx = (rS[0][e] - rS[0][ww]) + (rS[2][n] - rS[2][s]);
        float fy = (rS[2][e] - rS[2][ww]) + (rS[1][n] - rS[1][s]);
        if (POL && S.ericksen) {
            fx += (U.early.e[0][e] - U.early.e[0][ww]) + (U.early.e[1][n] - U.early.e[1][s]);
            fy += (U.early.e[2][e] - U.early.e[2][ww]) + (U.early.e[3][n] - U.early.e[3][s]);
        }
        float Fx = fmaf(0.5f, fx, S.gx), Fy = fmaf(0.5f, fy, S.gy);
        if (nib == 1) {
            Fx += bx;
            Fy += by;
        } else if (nib > 1)
            ib_force_list(sIB, nib, nx, ny, q.x, q.y, Fx, Fy);
        else if (nib < 0)
            ib_force(S, bodies, cur, q.x, q.y, Fx, Fy);
        float r[9], keep, drho, ux, uy;
        collide_terms<Pop<HT>::kScaled>(d, Fx, Fy, S.omega, S.guo, sc, is, r, keep, drho, ux, uy);
        rV[0][i] = 0.5f * ux;   // the gradient and advection stages take v / 2
        rV[1][i] = 0.5f * uy;
        if (q.X >= 2 && q.X < w + 2 && q.Y >= 2 && q.Y < l + 2) {
            const unsigned o = ((unsigned)q.y * (unsigned)nx + (unsigned)q.x) * HB, NH = N * HB;
#pragma unroll
            for (int m = 0; m < 9; ++m) Pop<HT>::st_buf(rHo, o, (unsigned)m * NH, fmaf(keep, d[m], r[m]));
            if (nib == 1) {
                buf_stf(ob.vib, bo, 0u, ux);
                buf_stf(ob.vib, bo, (unsigned)(4 * ob.ps * ob.ps), uy);
            } else if (nib > 1)
                ib_store_v_list(sIB, nib, nx, ny, q.x, q.y, ux, uy);
            else if (nib < 0)
                ib_store_v(S, bodies, cur, q.x, q.y, ux, uy);
        }
    }
    __syncthreads();

    // ---- predictor
#pragma unroll 1
    for (int i = tid; i < nD; i += T) {
        const Site q = site(i, WD, 1);
        const bool xe = box && q.x == nx - 1, xw = box && q.x == 0;
        const bool yhi = walls && q.y == ny - 1, ylo = walls && q.y == 0;
        const int v = (q.Y + 1) * WC + q.X + 1, ve = xe ? v : v + 1, vw = xw ? v : v - 1, vn = yhi ? v : v + WC,
                  vs = ylo ? v : v - WC;
        const float hx = rV[0][v], hy = rV[1][v];
        // walls: no-slip (negated) ghosts for v, mirror ghosts for sigma and P
        const float sxe = xe ? -1.0f : 1.0f, sxw = xw ? -1.0f : 1.0f, syn = yhi ? -1.0f : 1.0f, sys = ylo ? -1.0f : 1.0f;
        const Grad g = grad_v(sxe * rV[0][ve], sxw * rV[0][vw], syn * rV[0][vn], sys * rV[0][vs],
                              sxe * rV[1][ve], sxw * rV[1][vw], syn * rV[1][vn], sys * rV[1][vs]);
        const int p = (q.Y + 3) * WP + q.X + 3;
        PT Pc[2] = {POL ? rP[0][p] : (PT)0, POL ? rP[1][p] : (PT)0};
        const Stiff k = POL ? stiffness(S, sTab, (float)((PT)S.pref[0] + Pc[0]), (float)((PT)S.pref[1] + Pc[1]))
                            : Stiff{0.f, 0.f, 0.f, 0.f};
        const int c = (q.Y + 2) * WS + q.X + 2;
        const int e = xe ? c : c + 1, ww = xw ? c : c - 1, n = yhi ? c : c + WS, s = ylo ? c : c - WS;
        float X[3], Xe[3], Xw[3], Xn[3], Xs[3], Rs[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            X[m] = rS[m][c];
            Xe[m] = rS[m][e];
            Xw[m] = rS[m][ww];
            Xn[m] = rS[m][n];
            Xs[m] = rS[m][s];
        }
        rhs_sigma(S, k, g, hx, hy, X, Xe, Xw, Xn, Xs, Rs);
#pragma unroll
        for (int m = 0; m < 3; ++m) U.late.qs[m][i] = X[m] + Rs[m];
        if (POL) {
            const int pe = xe ? p : p + 1, pw = xw ? p : p - 1, pn = yhi ? p : p + WP, ps = ylo ? p : p - WP;
            PT Pe[2] = {rP[0][pe], rP[1][pe]}, Pw[2] = {rP[0][pw], rP[1][pw]};
            PT Pn[2] = {rP[0][pn], rP[1][pn]}, Ps[2] = {rP[0][ps], rP[1][ps]};
            PT Rp[2];
            rhs_P(S, g, hx, hy, Pc, Pe, Pw, Pn, Ps, Rp);
            U.late.qp[0][i] = Pc[0] + Rp[0];
            U.late.qp[1][i] = Pc[1] + Rp[1];
        }
        if (q.X >= 1 && q.X <= w && q.Y >= 1 && q.Y <= l) {   // the corrector's frozen inputs
            const int j = (q.Y - 1) * w + q.X - 1;
            const float f[8] = {g.psi0, g.psi1, g.psi2, g.om, k.p, k.q, k.r, k.w};
#pragma unroll
            for (int m = 0; m < (POL ? 8 : 4); ++m) U.late.g[m][j] = f[m];
        }
    }
    __syncthreads();

    // ---- corrector (at most one site a thread)
    if (tid < nE) {
        const Site q = site(tid, w, 0);
        const bool xe = box && q.x == nx - 1, xw = box && q.x == 0;
        const bool yhi = walls && q.y == ny - 1, ylo = walls && q.y == 0;
        const int v = (q.Y + 2) * WC + q.X + 2, c = (q.Y + 3) * WS + q.X + 3, p = (q.Y + 4) * WP + q.X + 4;
        const float hx = rV[0][v], hy = rV[1][v];
        const Grad g{U.late.g[0][tid], U.late.g[1][tid], U.late.g[2][tid], U.late.g[3][tid]};
        const Stiff k = POL ? Stiff{U.late.g[4][tid], U.late.g[5][tid], U.late.g[6][tid], U.late.g[7][tid]}
                            : Stiff{0.f, 0.f, 0.f, 0.f};
        const int j = (q.Y + 1) * WD + q.X + 1;
        const int je = xe ? j : j + 1, jw = xw ? j : j - 1, jn = yhi ? j : j + WD, js = ylo ? j : j - WD;
        float X[3], Xe[3], Xw[3], Xn[3], Xs[3], Rs[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            X[m] = U.late.qs[m][j];
            Xe[m] = U.late.qs[m][je];
            Xw[m] = U.late.qs[m][jw];
            Xn[m] = U.late.qs[m][jn];
            Xs[m] = U.late.qs[m][js];
        }
        rhs_sigma(S, k, g, hx, hy, X, Xe, Xw, Xn, Xs, Rs);
        const unsigned at = (unsigned)q.y * (unsigned)nx + (unsigned)q.x;
#pragma unroll
        for (int m = 0; m < 3; ++m) buf_stf(rSo, at * 4u, (unsigned)m * N * 4u, 0.5f * ((rS[m][c] + X[m]) + Rs[m]));
        if (POL) {   // without P both P buffers stay zero
            PT Y[2], Ye[2], Yw[2], Yn[2], Ys[2], Rp[2];
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                Y[m] = U.late.qp[m][j];
                Ye[m] = U.late.qp[m][je];
                Yw[m] = U.late.qp[m][jw];
                Yn[m] = U.late.qp[m][jn];
                Ys[m] = U.late.qp[m][js];
            }
            rhs_P(S, g, hx, hy, Y, Ye, Yw, Yn, Ys, Rp);
            const unsigned SP = (unsigned)sizeof(PT);
            buf_st(rPo, at * SP, 0u, (PT)0.5 * ((rP[0][p] + Y[0]) + Rp[0]));
            buf_st(rPo, at * SP, N * SP, (PT)0.5 * ((rP[1][p] + Y[1]) + Rp[1]));
        }
    }
}

// ------------------------------------------------------------------------------------------------
// multi-pass reference step: one thread per site, intermediate fields in scratch planes
// ------------------------------------------------------------------------------------------------

// site indices of (x, y) and its four neighbours; with walls the row beyond a wall is the mirror
// ghost (the site itself: zero normal derivative), flagged in lo / hi for odd (no-slip) fields
struct Nb {
    size_t c, e, w, n, s;
    bool lo, hi, le, ri;   // the south, north, west, east neighbour is a wall ghost
};
// walls: 1 below row 0 and above row ny-1; 2 also left of column 0 and right of column nx-1
__device__ __forceinline__ Nb nbrs(int x, int y, int nx, int ny, int walls = 0) {
    Nb q;
    size_t row = (size_t)y * nx;
    q.c = row + x;
    q.le = walls == 2 && x == 0;
    q.ri = walls == 2 && x == nx - 1;
    q.e = q.ri ? q.c : row + wrapi(x + 1, nx);
    q.w = q.le ? q.c : row + wrapi(x - 1, nx);
    q.lo = walls && y == 0;
    q.hi = walls && y == ny - 1;
    q.n = q.hi ? q.c : (size_t)wrapi(y + 1, ny) * nx + x;
    q.s = q.lo ? q.c : (size_t)wrapi(y - 1, ny) * nx + x;
    return q;
}

__device__ __forceinline__ bool site_of(const SiteBlock *blk, const SimDev *sims, int &sim, int &x, int &y) {
    SiteBlock b = blk[blockIdx.x];
    const SimDev &S = sims[b.sim];
    int i = b.start + threadIdx.x;
    sim = b.sim;
    if (i >= S.nx * S.ny) return false;
    y = i / S.nx;
    x = i - y * S.nx;
    return true;
}

template <typename PT>
__global__ __launch_bounds__(256) void k_mp_sigE(const SimDev *__restrict__ sims, const SiteBlock *__restrict__ blk,
                                                 int cur, int *__restrict__ d_t) {
    if (d_t && blockIdx.x == 0 && threadIdx.x == 0) d_t[0] = d_t[0] + 1;
    int sim, x, y;
    if (!site_of(blk, sims, sim, x, y)) return;
    const SimDev &S = sims[sim];
    const size_t N = (size_t)S.nx * S.ny;
    const PT *P = static_cast<const PT *>(S.P[cur]);
    Nb q = nbrs(x, y, S.nx, S.ny, S.walls);
    PT Pc[2] = {P[q.c], P[N + q.c]}, Pe[2] = {P[q.e], P[N + q.e]}, Pw[2] = {P[q.w], P[N + q.w]};
    PT Pn[2] = {P[q.n], P[N + q.n]}, Ps[2] = {P[q.s], P[N + q.s]};
    float E[4];
    ericksen(S, Pc, Pe, Pw, Pn, Ps, E);
    for (int k = 0; k < 4; ++k) S.sE[k * N + q.c] = E[k];
}

// force at a site from the stress, the Ericksen scratch planes and the bodies
__device__ __forceinline__ void site_force(const SimDev &S, const BodyDev *bodies, int cur, int x, int y, const Nb &q,
                                           float &Fx, float &Fy, float &fpx, float &fpy) {
    const size_t N = (size_t)S.nx * S.ny;
    const float *sg = S.sig[cur];
    fpx = 0.5f * (sg[q.e] - sg[q.w]) + 0.5f * (sg[2 * N + q.n] - sg[2 * N + q.s]);
    fpy = 0.5f * (sg[2 * N + q.e] - sg[2 * N + q.w]) + 0.5f * (sg[N + q.n] - sg[N + q.s]);
    Fx = fpx + S.gx;
    Fy = fpy + S.gy;
    if (S.ericksen) {
        const float *E = S.sE;
        Fx += 0.5f * (E[q.e] - E[q.w]) + 0.5f * (E[N + q.n] - E[N + q.s]);
        Fy += 0.5f * (E[2 * N + q.e] - E[2 * N + q.w]) + 0.5f * (E[3 * N + q.n] - E[3 * N + q.s]);
    }
    if (S.nb) ib_force(S, bodies, cur, x, y, Fx, Fy);
}

template <typename HT>
__device__ __forceinline__ void pull_pops(const SimDev &S, const HT *hin, int x, int y, float d[9]) {
    const size_t N = (size_t)S.nx * S.ny;
#pragma unroll
    for (int n = 0; n < 9; ++n) {
        const int ys = y - kCY[n], xs = x - kCX[n];
        if ((S.walls && (ys < 0 || ys >= S.ny)) || (S.walls == 2 && (xs < 0 || xs >= S.nx))) {
            // halfway bounce-back: the opposite direction
            d[n] = Pop<HT>::load(hin, kOpp[n] * N + (size_t)y * S.nx + x, S.inv_scale);   // at this site
            continue;
        }
        size_t i = (size_t)wrapi(ys, S.ny) * S.nx + wrapi(xs, S.nx);
        d[n] = Pop<HT>::load(hin, n * N + i, S.inv_scale);
    }
}

template <typename HT>
__global__ __launch_bounds__(256) void k_mp_lb(const SimDev *__restrict__ sims, const BodyDev *__restrict__ bodies,
                                               const SiteBlock *__restrict__ blk, int cur) {
    int sim, x, y;
    if (!site_of(blk, sims, sim, x, y)) return;
    const SimDev &S = sims[sim];
    const size_t N = (size_t)S.nx * S.ny;
    Nb q = nbrs(x, y, S.nx, S.ny, S.walls);
    float Fx, Fy, fpx, fpy;
    site_force(S, bodies, cur, x, y, q, Fx, Fy, fpx, fpy);
    float d[9];
    pull_pops<HT>(S, reinterpret_cast<const HT *>(S.h[cur]), x, y, d);
    float drho, ux, uy;
    collide(d, Fx, Fy, S.omega, S.guo, drho, ux, uy);
    HT *hout = reinterpret_cast<HT *>(S.h[cur ^ 1]);
    for (int n = 0; n < 9; ++n) Pop<HT>::store(hout, n * N + q.c, d[n], S.scale);
    S.v[q.c] = ux;
    S.v[N + q.c] = uy;
    if (S.nb) ib_store_v(S, bodies, cur, x, y, ux, uy);
}

__device__ __forceinline__ Grad grad_at(const SimDev &S, const Nb &q) {
    const size_t N = (size_t)S.nx * S.ny;
    const float *v = S.v;
    // no-slip ghosts beyond a wall: the negated velocity of the wall row
    // (and half of it: grad_v takes v / 2)
    const float sn = q.hi ? -0.5f : 0.5f, ss = q.lo ? -0.5f : 0.5f, se = q.ri ? -0.5f : 0.5f, sw = q.le ? -0.5f : 0.5f;
    return grad_v(se * v[q.e], sw * v[q.w], sn * v[q.n], ss * v[q.s], se * v[N + q.e], sw * v[N + q.w], sn * v[N + q.n],
                  ss * v[N + q.s]);
}

__device__ __forceinline__ void gather3(const float *f, size_t N, const Nb &q, float X[3], float Xe[3], float Xw[3],
                                        float Xn[3], float Xs[3]) {
    for (int k = 0; k < 3; ++k) {
        X[k] = f[k * N + q.c];
        Xe[k] = f[k * N + q.e];
        Xw[k] = f[k * N + q.w];
        Xn[k] = f[k * N + q.n];
        Xs[k] = f[k * N + q.s];
    }
}
template <typename PT>
__device__ __forceinline__ void gather2(const PT *f, size_t N, const Nb &q, PT X[2], PT Xe[2], PT Xw[2], PT Xn[2],
                                        PT Xs[2]) {
    for (int k = 0; k < 2; ++k) {
        X[k] = f[k * N + q.c];
        Xe[k] = f[k * N + q.e];
        Xw[k] = f[k * N + q.w];
        Xn[k] = f[k * N + q.n];
        Xs[k] = f[k * N + q.s];
    }
}

template <typename PT>
__global__ __launch_bounds__(256) void k_mp_pred(const SimDev *__restrict__ sims, const SiteBlock *__restrict__ blk,
                                                 int cur) {
    int sim, x, y;
    if (!site_of(blk, sims, sim, x, y)) return;
    const SimDev &S = sims[sim];
    const size_t N = (size_t)S.nx * S.ny;
    Nb q = nbrs(x, y, S.nx, S.ny, S.walls);
    Grad g = grad_at(S, q);
    float hx = 0.5f * S.v[q.c], hy = 0.5f * S.v[N + q.c];
    float X[3], Xe[3], Xw[3], Xn[3], Xs[3], Rs[3];
    gather3(S.sig[cur], N, q, X, Xe, Xw, Xn, Xs);
    PT Y[2], Ye[2], Yw[2], Yn[2], Ys[2], Rp[2];
    gather2(static_cast<const PT *>(S.P[cur]), N, q, Y, Ye, Yw, Yn, Ys);
    Stiff k = stiffness(S, reinterpret_cast<const float4 *>(S.tab), (float)((PT)S.pref[0] + Y[0]),
                        (float)((PT)S.pref[1] + Y[1]));
    rhs_sigma(S, k, g, hx, hy, X, Xe, Xw, Xn, Xs, Rs);
    rhs_P(S, g, hx, hy, Y, Ye, Yw, Yn, Ys, Rp);
    for (int c = 0; c < 3; ++c) S.sps[c * N + q.c] = X[c] + Rs[c];
    PT *spp = static_cast<PT *>(S.spp);
    for (int c = 0; c < 2; ++c) spp[c * N + q.c] = Y[c] + Rp[c];
}

template <typename PT>
__global__ __launch_bounds__(256) void k_mp_corr(const SimDev *__restrict__ sims, const SiteBlock *__restrict__ blk,
                                                 int cur) {
    int sim, x, y;
    if (!site_of(blk, sims, sim, x, y)) return;
    const SimDev &S = sims[sim];
    const size_t N = (size_t)S.nx * S.ny;
    Nb q = nbrs(x, y, S.nx, S.ny, S.walls);
    Grad g = grad_at(S, q);
    float hx = 0.5f * S.v[q.c], hy = 0.5f * S.v[N + q.c];
    const PT *P = static_cast<const PT *>(S.P[cur]);
    Stiff k = stiffness(S, reinterpret_cast<const float4 *>(S.tab), (float)((PT)S.pref[0] + P[q.c]),
                        (float)((PT)S.pref[1] + P[N + q.c]));
    float X[3], Xe[3], Xw[3], Xn[3], Xs[3], Rs[3];
    gather3(S.sps, N, q, X, Xe, Xw, Xn, Xs);
    PT Y[2], Ye[2], Yw[2], Yn[2], Ys[2], Rp[2];
    gather2(static_cast<const PT *>(S.spp), N, q, Y, Ye, Yw, Yn, Ys);
    rhs_sigma(S, k, g, hx, hy, X, Xe, Xw, Xn, Xs, Rs);
    rhs_P(S, g, hx, hy, Y, Ye, Yw, Yn, Ys, Rp);
    const float *sg = S.sig[cur];
    float *so = S.sig[cur ^ 1];
    PT *Po = static_cast<PT *>(S.P[cur ^ 1]);
    for (int c = 0; c < 3; ++c) so[c * N + q.c] = 0.5f * ((sg[c * N + q.c] + X[c]) + Rs[c]);
    for (int c = 0; c < 2; ++c) Po[c * N + q.c] = (PT)0.5 * ((P[c * N + q.c] + Y[c]) + Rp[c]);
}

// ------------------------------------------------------------------------------------------------
// observables and reductions
// ------------------------------------------------------------------------------------------------

// the planes of `mask` (bits 0 .. 9: drho, vx, vy, sxx, syy, sxy, Px, Py, fpx, fpy) at the current time,
// packed in bit order into `out` (floats).  Only what the mask needs is read: the forces for v and f^p,
// the populations for rho and v.  Bound by memory, and small beside the copy to the host that follows.
template <typename HT>
__global__ __launch_bounds__(256) void k_readout(const SimDev *__restrict__ sims, const BodyDev *__restrict__ bodies,
                                                 const SiteBlock *__restrict__ blk, int cur, unsigned mask,
                                                 float *__restrict__ out) {
    int sim, x, y;
    if (!site_of(blk, sims, sim, x, y)) return;
    const SimDev &S = sims[sim];
    const size_t N = (size_t)S.nx * S.ny;
    Nb q = nbrs(x, y, S.nx, S.ny, S.walls);
    float *o = out + q.c;
    auto put = [&](int bit, float v) {
        if (!((mask >> bit) & 1u)) return;
        *o = v;
        o += N;
    };
    float Fx = 0.f, Fy = 0.f, fpx = 0.f, fpy = 0.f, drho = 0.f, ux = 0.f, uy = 0.f;
    if (mask & kReadForce) site_force(S, bodies, cur, x, y, q, Fx, Fy, fpx, fpy);
    if (mask & kReadPops) {
        float d[9];
        pull_pops<HT>(S, reinterpret_cast<const HT *>(S.h[cur]), x, y, d);
        collide(d, Fx, Fy, S.omega, S.guo, drho, ux, uy);
    }
    typedef typename PolOf<HT>::T PT;
    const float *sg = S.sig[cur];
    const PT *P = static_cast<const PT *>(S.P[cur]);
    put(0, drho);
    put(1, ux);
    put(2, uy);
    for (int k = 0; k < 3; ++k)
        if ((mask >> (3 + k)) & 1u) put(3 + k, sg[k * N + q.c]);
    for (int k = 0; k < 2; ++k)
        if ((mask >> (6 + k)) & 1u) put(6 + k, (float)((PT)S.pref[k] + P[k * N + q.c]));
    put(8, fpx);
    put(9, fpy);
}

// block partial sums (FP64) of drho and sum_n c_n d_n over the stored populations of one sim;
// the stored (post-collision, not yet streamed) populations have the same domain totals
template <typename HT>
__global__ __launch_bounds__(256) void k_sums(const SimDev *__restrict__ sims, int sim, int cur,
                                              double *__restrict__ partial) {
    __shared__ double sh[3][4];
    const SimDev &S = sims[sim];
    const size_t N = (size_t)S.nx * S.ny;
    const HT *h = reinterpret_cast<const HT *>(S.h[cur]);
    double m = 0.0, jx = 0.0, jy = 0.0;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < N; i += (size_t)gridDim.x * 256) {
        float d[9];
#pragma unroll
        for (int n = 0; n < 9; ++n) d[n] = Pop<HT>::load(h, n * N + i, S.inv_scale);
#pragma unroll
        for (int n = 0; n < 9; ++n) {
            m += (double)d[n];
            jx += (double)(kCX[n] * d[n]);
            jy += (double)(kCY[n] * d[n]);
        }
    }
    m = wave_sum(m);
    jx = wave_sum(jx);
    jy = wave_sum(jy);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
        sh[0][wv] = m;
        sh[1][wv] = jx;
        sh[2][wv] = jy;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double s = (sh[threadIdx.x][0] + sh[threadIdx.x][1]) + (sh[threadIdx.x][2] + sh[threadIdx.x][3]);
        partial[3 * blockIdx.x + threadIdx.x] = s;
    }
}

// sum the block partials in a fixed order; out = (sum rho, momentum x, momentum y).  With
// check_mass > 0, raise the watchdog when the mass is not finite or drifts by more than 1e-6.
__global__ __launch_bounds__(64) void k_sums_final(const SimDev *__restrict__ sims, int sim, const double *__restrict__ partial,
                                                   int nblocks, double *__restrict__ out, double check_mass,
                                                   int *__restrict__ d_status) {
    const int lane = threadIdx.x;
    double a[3] = {0.0, 0.0, 0.0};
    for (int b = lane; b < nblocks; b += 64)
        for (int k = 0; k < 3; ++k) a[k] += partial[3 * b + k];
    for (int k = 0; k < 3; ++k) a[k] = wave_sum(a[k]);
    if (lane == 0) {
        const SimDev &S = sims[sim];
        double mass = (double)S.nx * (double)S.ny + a[0];
        out[0] = mass;
        out[1] = a[1];
        out[2] = a[2];
        if (check_mass > 0.0) {
            bool ok = isfinite(mass) && isfinite(a[1]) && isfinite(a[2]) && fabs(mass - check_mass) <= 1e-6 * check_mass;
            if (!ok) atomicOr(d_status, kStatusUnstable);
        }
    }
}

// What one directed edge (xa, ya) -> (xb, yb) of a polygon adds to the site X and the unit cell around it,
// in the row Y: where it crosses the row (NaN if it does not), and the integral along its part within
// [Y - 1/2, Y + 1/2] of g(x) dy with g(x) = clamp(x, x0, x1) - x0.  Summed over a closed polygon the latter
// is, by Green's theorem, the signed area of the polygon inside the cell [x0, x1] x [Y - 1/2, Y + 1/2].  g is
// piecewise linear along the edge, so the midpoint rule on the pieces between its kinks is exact.
struct RowEdge {
    double cross;        // the row is crossed here: sites to the left of it are inside or outside by it
    double xl, dx, inv;  // x at the lower end of the part in the band, its extent, 1 / extent (0 if none)
    double c;            // signed height of the part
};
__device__ __forceinline__ bool touches_row(double ya, double yb, double Y) {
    return fmin(fmax(ya, yb), Y + 0.5) > fmax(fmin(ya, yb), Y - 0.5);   // horizontal edges do not
}
__device__ __forceinline__ RowEdge row_edge(double2 a, double2 b, double Y) {
    const double lo = fmax(fmin(a.y, b.y), Y - 0.5), hi = fmin(fmax(a.y, b.y), Y + 0.5);
    const double s = (b.x - a.x) / (b.y - a.y);
    RowEdge e;
    e.cross = (b.y > Y) != (a.y > Y) ? (a.x - b.x) * (Y - b.y) / (a.y - b.y) + b.x : __builtin_nan("");
    e.xl = a.x + s * (lo - a.y);
    e.dx = (a.x + s * (hi - a.y)) - e.xl;
    e.inv = e.dx != 0.0 ? 1.0 / e.dx : 0.0;
    e.c = (b.y > a.y ? 1.0 : -1.0) * (hi - lo);
    return e;
}
__device__ __forceinline__ double cell_share(const RowEdge &e, double x0, double x1) {
    double ta = fmin(fmax((x0 - e.xl) * e.inv, 0.0), 1.0), tb = fmin(fmax((x1 - e.xl) * e.inv, 0.0), 1.0);
    if (ta > tb) {
        const double u = ta;
        ta = tb;
        tb = u;
    }
    auto g = [&](double t) { return fmin(fmax(e.xl + t * e.dx, x0), x1) - x0; };
    return e.c * (ta * g(0.5 * ta) + (tb - ta) * g(0.5 * (ta + tb)) + (1.0 - tb) * g(0.5 * (tb + 1.0)));
}
__device__ __forceinline__ double lane_value(double v, int lane) {   // the same lane for the whole wave
    const long long q = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readlane((unsigned)q, lane), hi = __builtin_amdgcn_readlane((unsigned)(q >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// body observables, one 1024-thread block per body: restoring force as the sum of div sigma over
// the sites inside the node polygon (even-odd rule), centre of mass, total node force, and the
// area-weighted restoring force: the sum over sites of (area of the site's unit cell inside the
// polygon) * div sigma, which varies continuously with the node positions.
// Bound by the chain of one wave's FP64 instructions.  A wave takes 64 sites of a row at a time; its lanes
// first look at 64 edges at once and work out those few that touch the row, which then go round the wave
// one by one.  (Every site against every edge, with its divisions, in one wave a SIMD: 64 bodies of radius
// 4 to 32 took 542 us, now 27; 32 of radius 4 to 16 took 80, now 15.)  Waves without nodes or without sites skip the
// reductions, which are a small body's time: radius 1.2, 13.7 us with all 16 waves in them, 6.6 without (the start's
// 256 threads 9.5); 300 bodies of radius 4 28.5 and 14.2 (19.1).
constexpr int kForceThreads = 1024;
constexpr double kMaxSide = 16384.0;
__global__ __launch_bounds__(kForceThreads) void k_body_force(const SimDev *__restrict__ sims,
                                                              const BodyDev *__restrict__ bodies, int body0, int cur,
                                                              double *__restrict__ out_all) {
    constexpr int kWaves = kForceThreads / 64;
    __shared__ double2 sR[kMaxNodes];
    __shared__ double sh[9][kWaves];
    const BodyDev &B = bodies[body0 + blockIdx.x];
    double *out = out_all + kBodyOut * blockIdx.x;
    const SimDev &S = sims[B.sim];
    const int n = B.n, tid = threadIdx.x, lane = tid & 63, wv = uniform(tid >> 6);
    const double2 *R = reinterpret_cast<const double2 *>(B.R[cur]);
    const double2 *Fn = reinterpret_cast<const double2 *>(B.fnode);
    double mnx = 1e300, mny = 1e300, mxx = -1e300, mxy = -1e300, cx = 0, cy = 0, fx = 0, fy = 0, ar = 0;
    for (int a = tid; a < n; a += kForceThreads) {
        double2 r = R[a], q = R[a == 0 ? n - 1 : a - 1], f = Fn[a];
        sR[a] = r;
        mnx = fmin(mnx, r.x);
        mny = fmin(mny, r.y);
        mxx = fmax(mxx, r.x);
        mxy = fmax(mxy, r.y);
        cx += r.x;
        cy += r.y;
        fx += f.x;
        fy += f.y;
        ar += q.x * r.y - r.x * q.y;
    }
    const int nodeWaves = min(kWaves, (n + 63) / 64);   // the others have nothing to reduce
    if (wv < nodeWaves) {
        double v9[9] = {wave_min(mnx), wave_min(mny), wave_max(mxx), wave_max(mxy),
                        wave_sum(cx),  wave_sum(cy),  wave_sum(fx),  wave_sum(fy), wave_sum(ar)};
        if (lane == 0)
            for (int k = 0; k < 9; ++k) sh[k][wv] = v9[k];
    }
    __syncthreads();
    double all[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) all[k] = sh[k][0];
#pragma unroll 1
    for (int w = 1; w < nodeWaves; ++w)
#pragma unroll
        for (int k = 0; k < 9; ++k) all[k] = k < 2 ? fmin(all[k], sh[k][w]) : k < 4 ? fmax(all[k], sh[k][w]) : all[k] + sh[k][w];
    mnx = all[0];
    mny = all[1];
    mxx = all[2];
    mxy = all[3];
    const double orient = all[8] < 0.0 ? -1.0 : 1.0;
    __syncthreads();
    const size_t N = (size_t)S.nx * S.ny;
    const float *sg = S.sig[cur];
    // every cell that the bounding box touches; the sites strictly inside it are among them
    const int x0 = (int)floor(mnx + 0.5), x1 = (int)ceil(mxx - 0.5), y0 = (int)floor(mny + 0.5), y1 = (int)ceil(mxy - 0.5);
    const int ix0 = (int)ceil(mnx), ix1 = (int)floor(mxx), iy0 = (int)ceil(mny), iy1 = (int)floor(mxy);
    double ax = 0.0, ay = 0.0, bx = 0.0, by = 0.0;
    // nodes that span more than the largest lattice (or none that are numbers) have no sums: the loops end
    const bool whole = x1 >= x0 && y1 >= y0 && mxx - mnx < kMaxSide && mxy - mny < kMaxSide;
    const int across = whole ? (x1 - x0) / 64 + 1 : 0, units = whole ? across * (y1 - y0 + 1) : 0;
    if (!whole) ax = ay = bx = by = __builtin_nan("");
    for (int u = wv; u < units; u += kWaves) {
        const int Y = y0 + u / across, X = x0 + (u % across) * 64 + lane;
        const Nb q = nbrs(wrapi(min(X, x1), S.nx), wrapi(Y, S.ny), S.nx, S.ny, S.walls);
        const double e0 = sg[q.e], w0 = sg[q.w], n1 = sg[N + q.n], s1 = sg[N + q.s];
        const double e2 = sg[2 * N + q.e], w2 = sg[2 * N + q.w], n2 = sg[2 * N + q.n], s2 = sg[2 * N + q.s];
        bool in = false;
        double w = 0.0;
        for (int a0 = 0; a0 < n; a0 += 64) {
            const int a = a0 + lane;
            const double2 to = sR[min(a, n - 1)], from = sR[a == 0 ? n - 1 : min(a, n) - 1];
            const bool mine = a < n && touches_row(from.y, to.y, Y);
            unsigned long long hit = __ballot(mine);
            if (!hit) continue;
            RowEdge own{};
            if (mine) own = row_edge(from, to, Y);
            for (; hit; hit &= hit - 1) {
                const int k = __builtin_ctzll(hit);
                const RowEdge e{lane_value(own.cross, k), lane_value(own.xl, k), lane_value(own.dx, k),
                                lane_value(own.inv, k), lane_value(own.c, k)};
                in = in != ((double)X < e.cross);
                w += cell_share(e, X - 0.5, X + 0.5);
            }
        }
        if (X > x1) continue;
        const double dx = 0.5 * (e0 - w0) + 0.5 * (n2 - s2), dy = 0.5 * (e2 - w2) + 0.5 * (n1 - s1);
        if (in && X >= ix0 && X <= ix1 && Y >= iy0 && Y <= iy1) {
            ax += dx;
            ay += dy;
        }
        w *= orient;
        if (w != 0.0) {
            bx += w * dx;
            by += w * dy;
        }
    }
    const int unitWaves = min(kWaves, max(units, 1));
    if (wv < unitWaves) {
        double red[4] = {wave_sum(ax), wave_sum(ay), wave_sum(bx), wave_sum(by)};
        if (lane == 0)
            for (int k = 0; k < 4; ++k) sh[k][wv] = red[k];
    }
    __syncthreads();
    if (tid < 4) {
        double v = 0.0;
        for (int w = 0; w < unitWaves; ++w) v += sh[tid][w];
        out[tid < 2 ? tid : tid + 4] = v;
    } else if (tid == 4) {
        out[2] = all[4] / n;
        out[3] = all[5] / n;
        out[4] = all[6];
        out[5] = all[7];
    }
}

// convert host-prepared FP32 population offsets (already un-streamed) to the storage type
template <typename HT>
__global__ __launch_bounds__(256) void k_pack(const float *__restrict__ src, HT *__restrict__ dst, size_t n, float scale) {
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) Pop<HT>::store(dst, i, src[i], scale);
}

// streaming copy of n16 16-byte words, the bandwidth ceiling the field kernel is measured against:
// each thread moves four words per trip, all four loads issued before the stores, and the grid
// strides over the buffer so every compute unit keeps several loads in flight
__global__ __launch_bounds__(256) void k_stream_copy(const uint4 *__restrict__ src, uint4 *__restrict__ dst,
                                                     size_t n16) {
    const size_t stride = (size_t)gridDim.x * 1024;
    for (size_t base = (size_t)blockIdx.x * 1024 + threadIdx.x; base < n16; base += stride) {
        uint4 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (base + 256 * k < n16) v[k] = src[base + 256 * k];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (base + 256 * k < n16) dst[base + 256 * k] = v[k];
    }
}

// ------------------------------------------------------------------------------------------------
// launch wrappers (host)
// ------------------------------------------------------------------------------------------------

hipError_t launch_ib(bool advance, int nbodies, int ntiles, int nmax, hipStream_t st, const SimDev *sims, BodyDev *bodies,
                     const int2 *blk, int cur, const int *d_t, int *d_status) {
    const size_t lds = 4 * (size_t)nmax * sizeof(double2);
    if (nbodies <= 0) return hipSuccess;
    if (ntiles <= kIbOneLaunchTiles) {
        // few tiles: one launch, each block repeats its body's node update
        if (advance)
            k_ib_step<true><<<ntiles, kIbThreads, lds, st>>>(sims, bodies, blk, nmax, cur, d_t, d_status);
        else
            k_ib_step<false><<<ntiles, kIbThreads, lds, st>>>(sims, bodies, blk, nmax, cur, d_t, d_status);
    } else {
        if (advance)
            k_ib_nodes<true><<<nbodies, kIbThreads, lds, st>>>(sims, bodies, nmax, cur, d_t, d_status);
        else
            k_ib_nodes<false><<<nbodies, kIbThreads, lds, st>>>(sims, bodies, nmax, cur, d_t, d_status);
        k_ib_spread<<<ntiles, kSpreadThreads, 0, st>>>(bodies, blk, advance ? (cur ^ 1) : cur, d_status);
    }
    return hipGetLastError();
}

// the kernel for (work-group size, storage type, walls, polarization, any body in the launch)
typedef void (*FusedFn)(const SimDev *, const BodyDev *, const WorkItem *, int, int, int *, int);
template <int T>
static FusedFn fused_fn_t(bool fp16, bool walls, bool pol, bool any_body) {
    if (fp16) {
        if (walls) return pol ? k_fused<T, __half, true, true, false> : k_fused<T, __half, true, false, false>;
        return pol ? k_fused<T, __half, false, true, false> : k_fused<T, __half, false, false, false>;
    }
    if (walls) return pol ? k_fused<T, float, true, true, false> : k_fused<T, float, true, false, false>;
    if (any_body) return pol ? k_fused<T, float, false, true, true> : k_fused<T, float, false, false, true>;
    return pol ? k_fused<T, float, false, true, false> : k_fused<T, float, false, false, false>;
}
static FusedFn fused_fn(int T, bool fp16, bool walls, bool pol, bool any_body) {
    if (T == 64) return fused_fn_t<64>(fp16, walls, pol, any_body);
    if (T == 128) return fused_fn_t<128>(fp16, walls, pol, any_body);
    if (T == 256) return fused_fn_t<256>(fp16, walls, pol, any_body);
    return nullptr;
}

typedef void (*TileFn)(const SimDev *, const BodyDev *, const WorkItem *, int, int, int *);
template <int T, typename HT>
static TileFn tile_fn_t(bool walls, bool pol) {
    if (walls) return pol ? k_tile<T, HT, true, true> : k_tile<T, HT, true, false>;
    return pol ? k_tile<T, HT, false, true> : k_tile<T, HT, false, false>;
}
static TileFn tile_fn(int T, bool fp16, bool walls, bool pol) {
    if (T == 64) return fp16 ? tile_fn_t<64, __half>(walls, pol) : tile_fn_t<64, float>(walls, pol);
    if (T == 128) return fp16 ? tile_fn_t<128, __half>(walls, pol) : tile_fn_t<128, float>(walls, pol);
    if (T == 256) return fp16 ? tile_fn_t<256, __half>(walls, pol) : tile_fn_t<256, float>(walls, pol);
    return nullptr;
}

hipError_t launch_tile(int T, bool fp16, bool walls, bool pol, hipStream_t st, const SimDev *sims, const BodyDev *bodies,
                       const WorkItem *items, int n_items, int cur, int *d_t) {
    TileFn f = tile_fn(T, fp16, walls, pol);
    if (!f) return hipErrorInvalidValue;
    hipLaunchKernelGGL(f, dim3(n_items), dim3(T), 0, st, sims, bodies, items, n_items, cur, d_t);
    return hipGetLastError();
}

hipError_t launch_fused(int T, bool fp16, bool walls, bool pol, bool any_body, int grid, hipStream_t st, const SimDev *sims,
                        const BodyDev *bodies, const WorkItem *items, int n_items, int cur, int *d_t, int cus) {
    FusedFn f = fused_fn(T, fp16, walls, pol, any_body);
    if (!f || cus < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(f, dim3(grid), dim3(T), 0, st, sims, bodies, items, n_items, cur, d_t, cus);
    return hipGetLastError();
}

int fused_blocks_per_cu(int T, bool fp16, bool walls, bool pol, bool any_body) {
    FusedFn f = fused_fn(T, fp16, walls, pol, any_body);
    int n = 0;
    hipFuncAttributes a;
    hipError_t e = f ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, T, 0) : hipErrorInvalidValue;
    if (e == hipSuccess) e = hipFuncGetAttributes(&a, reinterpret_cast<const void *>(f));
    if (e != hipSuccess) return 1;
    // LDS is handed out in units of 1280 bytes, which the count above leaves out: 64 threads in FP32 are 11 by
    // it and 10 in fact (128 lattices of 64^2 in three rows, 11 a unit, take two rounds: 30.2 us, 21.9 in four)
    const int lds = (int)((a.sharedSizeBytes + 1279) / 1280 * 1280);
    if (lds > 0) n = std::min(n, 160 * 1024 / lds);
    return std::max(1, n);
}

hipError_t launch_multipass(bool fp16, int nblocks, hipStream_t st, const SimDev *sims, const BodyDev *bodies,
                            const SiteBlock *blk, int cur, int *d_t) {
    if (fp16) {
        k_mp_sigE<float><<<nblocks, 256, 0, st>>>(sims, blk, cur, d_t);
        k_mp_lb<__half><<<nblocks, 256, 0, st>>>(sims, bodies, blk, cur);
        k_mp_pred<float><<<nblocks, 256, 0, st>>>(sims, blk, cur);
        k_mp_corr<float><<<nblocks, 256, 0, st>>>(sims, blk, cur);
    } else {
        k_mp_sigE<double><<<nblocks, 256, 0, st>>>(sims, blk, cur, d_t);
        k_mp_lb<float><<<nblocks, 256, 0, st>>>(sims, bodies, blk, cur);
        k_mp_pred<double><<<nblocks, 256, 0, st>>>(sims, blk, cur);
        k_mp_corr<double><<<nblocks, 256, 0, st>>>(sims, blk, cur);
    }
    return hipGetLastError();
}

hipError_t launch_readout(bool fp16, int nblocks, int block0, hipStream_t st, const SimDev *sims, const BodyDev *bodies,
                          const SiteBlock *blk, int cur, unsigned mask, float *out) {
    if (mask & kReadForce) {
        if (fp16)
            k_mp_sigE<float><<<nblocks, 256, 0, st>>>(sims, blk + block0, cur, nullptr);
        else
            k_mp_sigE<double><<<nblocks, 256, 0, st>>>(sims, blk + block0, cur, nullptr);
    }
    if (fp16)
        k_readout<__half><<<nblocks, 256, 0, st>>>(sims, bodies, blk + block0, cur, mask, out);
    else
        k_readout<float><<<nblocks, 256, 0, st>>>(sims, bodies, blk + block0, cur, mask, out);
    return hipGetLastError();
}

hipError_t launch_sums(bool fp16, int sim, int nblocks, hipStream_t st, const SimDev *sims, int cur, double *partial,
                       double *out, double check_mass, int *d_status) {
    if (fp16)
        k_sums<__half><<<nblocks, 256, 0, st>>>(sims, sim, cur, partial);
    else
        k_sums<float><<<nblocks, 256, 0, st>>>(sims, sim, cur, partial);
    k_sums_final<<<1, 64, 0, st>>>(sims, sim, partial, nblocks, out, check_mass, d_status);
    return hipGetLastError();
}

hipError_t launch_body_force(hipStream_t st, const SimDev *sims, const BodyDev *bodies, int body0, int nbodies, int cur,
                             double *out) {
    if (nbodies <= 0) return hipSuccess;
    k_body_force<<<nbodies, kForceThreads, 0, st>>>(sims, bodies, body0, cur, out);
    return hipGetLastError();
}

hipError_t launch_stream_copy(hipStream_t st, const void *src, void *dst, size_t bytes) {
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    const size_t blocks = std::min<size_t>((n16 + 1023) / 1024, 256 * 16);
    k_stream_copy<<<(unsigned)blocks, 256, 0, st>>>(static_cast<const uint4 *>(src), static_cast<uint4 *>(dst), n16);
    return hipGetLastError();
}

hipError_t launch_pack(bool fp16, hipStream_t st, const float *src, void *dst, size_t n, float scale) {
    int nb = (int)((n + 255) / 256);
    if (fp16)
        k_pack<__half><<<nb, 256, 0, st>>>(src, reinterpret_cast<__half *>(dst), n, scale);
    else
        k_pack<float><<<nb, 256, 0, st>>>(src, reinterpret_cast<float *>(dst), n, scale);
    return hipGetLastError();
}

}  // namespace lbk

// The fire-mesh time step for small meshes (gfx950): one launch, small tiles.
//
// A mesh of a few hundred cells a side gives the tiled kernel of
// fire_kernels.hip a handful of work-groups whose threads each work through
// several rows; the time is then the latency of that chain, on a few of the
// 256 CUs.  Here a work-group owns a tile of a few atmosphere cells and a
// thread one or two of its nodes: every load of the step is issued at once
// at the start, and each phase is one node's worth of work.
// The step's phases and their arithmetic are those of the tiled kernel, node
// by node the same functions, so the results are the same bits.
//
// Bound by latency: one round trip to memory, then four phases of one node
// each (FP64: two pow calls) between barriers.  A domain's ignition geometry
// comes in the kernel's arguments, formed on the host, so the step is one
// launch.  128^2 FP64 (169 work-groups of 10 x 10 cells) 37 -> 10.5 us per
// step, 500^2 FP64 33.6 -> 23.3, FP32 15.3 -> 10.8; 500^2 FP32 while four lines
// grow 19.7 -> 12.0.  Every active ignition is evaluated at every node: while
// lines grow, psi_g is below psi at nearly all of them, and dropping the others
// per wave by bounds over the frame made such steps slower (500^2 FP64 27.9 ->
// 29.7, 600^2 33.2 -> 36.3: the bounds are a chain before the first barrier).
#include "fire_device.h"

namespace fire {
namespace {

using namespace dev;

#pragma clang fp contract(off)

template <typename T> struct alignas(8) SmallParams {
    StepArgs a;
    IgnTable<T> tab;     // one domain: the ignition geometry of the step
};

template <typename T> struct SmallPtrs {
    const T *psi_in;
    T *psi_out, *tign, *frac;
    const T *u, *v, *gx, *gy;
    const uint8_t *cat;
    T *fsens, *flat;
    int *status;
    T *rec_p0, *rec_b;
    int32_t *mark;
};

// One node of a thread: its place in the frame and in the domain, and what
// the step reads there.
template <typename T> struct Node {
    int f, gx, gy;           // frame index (-1: no node), column and row
    bool in;                 // in the domain
    T u, v, gzx, gzy, ti, fr;
    int cv;
};

// i / w for 0 <= i < 2^16, 1 <= w < 2^12, r = 1 / w in float: (i + 1/2) / w is
// at least 1 / (2 w) away from a whole number, far above the rounding.
__device__ __forceinline__ int quot(int i, float r) { return (int)(((float)i + 0.5f) * r); }

// Fills the ghost nodes of frame array P (pitch w, first node (fx0, fy0)).
template <typename T>
__device__ __forceinline__ void ghosts(T *P, int w, int h, int fx0, int fy0, int nx, int ny,
                                       bool corners, T *Q, T tp) {
    const float rw = 1.0f / (float)w;
    for (int f = threadIdx.x; f < w * h; f += blockDim.x) {
        const int fy = quot(f, rw), fx = f - fy * w;
        const int gx = fx0 + fx, gy = fy0 + fy;
        const bool xin = gx >= 0 && gx < nx, yin = gy >= 0 && gy < ny;
        if (xin && yin) continue;
        const int sx = gx == -1 ? 1 : (gx == nx ? -1 : 0);
        const int sy = (gy == -1 ? 1 : (gy == ny ? -1 : 0)) * w;
        if (yin && sx != 0) {
            P[f] = ghost(P[f + sx], P[f + 2 * sx]);
        } else if (xin && sy != 0) {
            P[f] = ghost(P[f + sy], P[f + 2 * sy]);
        } else if (corners && sx != 0 && sy != 0) {
            const T r1 = ghost(P[f + sy + sx], P[f + 2 * sy + sx]);
            const T r2 = ghost(P[f + sy + 2 * sx], P[f + 2 * sy + 2 * sx]);
            P[f] = ghost(r1, r2);
        }
        if (Q) Q[f] = tp;   // ghost nodes' times are t'
    }
}

// NPT: nodes of the tile and its two inner rings per thread.
template <typename T, bool REC, int NPT>
__device__ __forceinline__ void small_tile(const StepArgs &a, const SmallPtrs<T> &p,
                                           const IgnTable<T> *itab, const T *__restrict__ coef,
                                           int tile, double tnow, T *lds) {
    const int nx = a.nx, ny = a.ny;
    const int tyi = tile / a.tiles_x;
    const int x0 = (tile - tyi * a.tiles_x) * a.tile_x, y0 = tyi * a.tile_y;
    const int w = a.tile_x + 2 * kHalo, h = a.tile_y + 2 * kHalo, F = w * h;
    const int fx0 = x0 - kHalo, fy0 = y0 - kHalo;
    const int nt = blockDim.x, tid = threadIdx.x;
    const float rw = 1.0f / (float)w, rw1 = 1.0f / (float)(w - 2);
    T *A = lds, *B = A + F, *C = B + F, *tab = C + F;   // frames, fuel table
    T *D = tab + a.ncat * kLRow;                        // latent flux of the tile
    int *flag = reinterpret_cast<int *>(D + a.tile_x * a.tile_y);

    Consts<T> c;
    c.rdx = T(a.rdx);
    c.rdy = T(a.rdy);
    c.eps = T(a.eps);
    c.cap = T(a.ros_cap);
    c.visc_mode = a.visc_mode;
    const T dt = T(a.dt), hdt = T(0.5 * a.dt), rdt = T(a.rdt);
    const T t = T(tnow), tp = T(tnow + a.dt);
    const T INF = M<T>::inf();

    // ---- everything the step reads, at once
    constexpr int NF = NPT + 2;   // frame nodes per thread (checked by the launch)
    T pf[NF];
#pragma unroll
    for (int k = 0; k < NF; k++) {
        const int f = tid + k * nt;
        const int fy = quot(f, rw), fx = f - fy * w;
        const int gx = fx0 + fx, gy = fy0 + fy;
        pf[k] = f < F && gx >= 0 && gx < nx && gy >= 0 && gy < ny
                    ? p.psi_in[gy * nx + gx] : T(0);
    }
    Node<T> nd[NPT];
    const int w1 = w - 2, S1 = w1 * (h - 2);
#pragma unroll
    for (int k = 0; k < NPT; k++) {
        const int i = tid + k * nt;
        const int sy = quot(i, rw1), sx = i - sy * w1;
        Node<T> &n = nd[k];
        n.f = i < S1 ? (sy + 1) * w + sx + 1 : -1;
        n.gx = fx0 + 1 + sx;
        n.gy = fy0 + 1 + sy;
        n.in = i < S1 && n.gx >= 0 && n.gx < nx && n.gy >= 0 && n.gy < ny;
        if (n.in) {
            const int o = n.gy * nx + n.gx;   // (small meshes: below 2^31)
            n.cv = p.cat[o];
            n.u = p.u[o];
            n.v = p.v[o];
            n.gzx = p.gx[o];
            n.gzy = p.gy[o];
            if (!REC) {
                n.ti = p.tign[o];
                // a ring cell's F belongs to another work-group, which may be
                // writing it: the tile's first cell in its place (unused)
                const bool mine = (uint32_t)(n.gx - x0) < (uint32_t)a.tile_x &&
                                  (uint32_t)(n.gy - y0) < (uint32_t)a.tile_y;
                n.fr = p.frac[mine ? o : y0 * nx + x0];
            }
        }
    }
    for (int i = tid; i < a.ncat; i += nt) make_row(coef + i * kNCoef, tab + i * kLRow, T(a.ros_cap));
    if (tid == 0) *flag = 0;

    // ---- step 1, ignition (Sect. 4.4), on the frame
#pragma unroll
    for (int k = 0; k < NF; k++) {
        const int f = tid + k * nt;
        if (f >= F) break;
        const int fy = quot(f, rw), fx = f - fy * w;
        T q = pf[k], tig = INF;
        for (int g = 0; g < a.nign; g++) {
            if (!itab->on[g]) continue;
            const IgnGeo<T> geo = itab->g[g];
            const T py = ign_py(geo, fy0 + fy, a.dy);
            ign_apply(geo, ign_px(geo, fx0 + fx, a.dx), py, ign_by(geo, py), q, tig);
        }
        if (!(pf[k] > T(0) && q <= T(0))) tig = INF;
        A[f] = q;
        C[f] = tig;
    }
    __syncthreads();
    const bool interior = fx0 >= 0 && fx0 + w <= nx && fy0 >= 0 && fy0 + h <= ny;
    if (!interior) {
        ghosts(A, w, h, fx0, fy0, nx, ny, false, (T *)nullptr, tp);
        __syncthreads();
    }
    // ---- step 2a: first Heun stage on the tile plus two rings
    const lds_t<T> *tab3 = (const lds_t<T> *)tab;
    const lds_t<T> *row[NPT];
#pragma unroll
    for (int k = 0; k < NPT; k++) {
        const Node<T> &n = nd[k];
        if (!n.in) continue;
        row[k] = tab3 + min(n.cv, a.ncat - 1) * kLRow;
        const T f1 = rhs5(A[n.f], A[n.f - 1], A[n.f + 1], A[n.f - w], A[n.f + w], n.u, n.v, n.gzx,
                          n.gzy, row[k], c);
        B[n.f] = heun1(A[n.f], dt, f1);
    }
    __syncthreads();
    if (!interior) {
        ghosts(B, w, h, fx0, fy0, nx, ny, false, (T *)nullptr, tp);
        __syncthreads();
    }
    // ---- step 2b: second stage on the tile plus one ring; step 3: ignition
    // times (Eq. 14) and node times t^ (Eq. 17)
    int st = 0;
#pragma unroll
    for (int k = 0; k < NPT; k++) {
        const Node<T> &n = nd[k];
        const int rx = n.gx - x0, ry = n.gy - y0;   // place in the tile
        if (!n.in || rx < -1 || rx > a.tile_x || ry < -1 || ry > a.tile_y) continue;
        const bool mine = rx >= 0 && rx < a.tile_x && ry >= 0 && ry < a.tile_y;
        const T pn0 = A[n.f], b0 = B[n.f];
        const T f2 = rhs5(b0, B[n.f - 1], B[n.f + 1], B[n.f - w], B[n.f + w], n.u, n.v, n.gzx,
                          n.gzy, row[k], c);
        const T pn = heun2(pn0, b0, hdt, f2);
        A[n.f] = pn;   // stage-1 reads of A ended at the last barrier
        const int o = n.gy * nx + n.gx;   // (small meshes: below 2^31)
        if (REC) {
            if (mine) {
                p.psi_out[o] = pn;
                p.rec_p0[o] = pn0;
                p.rec_b[o] = b0;
            }
            continue;
        }
        T ti = INF, told = INF;
        const T tig = C[n.f];
        if (pn <= T(0) || tig < INF) {
            told = n.ti;
            ti = told;
            if (is_inf(ti)) ti = tig;
            if (pn0 > T(0) && pn <= T(0) && is_inf(ti)) ti = cross_time(t, pn0, pn, dt);
        }
        C[n.f] = pn >= T(0) ? tp : ti;
        if (mine) {
            p.psi_out[o] = pn;
            if (!(ti == told)) {
                p.tign[o] = ti;
                // the step in which t_i was first set
                if (p.mark && is_inf(told)) p.mark[o] = a.mark_step;
            }
            const int gw = a.guard;
            const bool edge = n.gx < gw || n.gy < gw || n.gx >= nx - gw || n.gy >= ny - gw;
            if (edge && pn < T(0)) st |= kStBoundary;
            if (!__builtin_isfinite(pn)) st |= kStNonfinite;
        }
    }
    if (REC) return;
    __syncthreads();
    if (!interior) {
        ghosts(A, w, h, fx0, fy0, nx, ny, true, C, tp);
        __syncthreads();
    }
    // ---- steps 4-5: fuel fraction and fluxes; B and D take the tile's fluxes
    bool hot = false;
#pragma unroll
    for (int k = 0; k < NPT; k++) {
        const Node<T> &n = nd[k];
        const int rx = n.gx - x0, ry = n.gy - y0;
        if (n.f < 0 || rx < 0 || rx >= a.tile_x || ry < 0 || ry >= a.tile_y) continue;
        T fs = T(0), fl = T(0);
        if (n.in) {
            T pp[3][3], qq[3][3], mn = INF;
#pragma unroll
            for (int j = 0; j < 3; j++)
#pragma unroll
                for (int i = 0; i < 3; i++) {
                    pp[j][i] = A[n.f + (j - 1) * w + i - 1];
                    mn = vmin(mn, pp[j][i]);
                }
            // F^{n+1} = F^n = 1 and no flux unless a stencil node burns or F
            // was already below 1
            if (mn < T(0) || !(n.fr == T(1))) {
                T Fn = T(1);
                if (mn < T(0)) {
#pragma unroll
                    for (int j = 0; j < 3; j++)
#pragma unroll
                        for (int i = 0; i < 3; i++) qq[j][i] = C[n.f + (j - 1) * w + i - 1];
                    Fn = fraction9(pp, qq, tp, row[k][kLTf]);
                }
                const T dF = (n.fr - Fn) * rdt;
                fs = dF * row[k][kLCh];
                fl = dF * row[k][kLCq];
                if (!(Fn == n.fr)) p.frac[n.gy * nx + n.gx] = Fn;
                if (!__builtin_isfinite(Fn)) st |= kStNonfinite;
                hot = true;
            }
        }
        B[ry * a.tile_x + rx] = fs;
        D[ry * a.tile_x + rx] = fl;
    }
    if (st) atomicOr(p.status, st);
    if (hot) *flag = 1;
    __syncthreads();

    // ---- step 6: mean flux over each atmosphere cell of the tile: columns,
    // then the column sums, in order (both zero where no cell has a flux)
    const bool some = *flag != 0;
    const int nI = a.tile_x / a.sr_x, nJ = a.tile_y / a.sr_y;
    if (some) {
        for (int q = tid; q < a.tile_x * nJ; q += nt) {
            const int J = q / a.tile_x, i = q - J * a.tile_x;
            const int o = J * a.sr_y * a.tile_x + i;
            T s1 = T(0), s2 = T(0);
            for (int r = 0; r < a.sr_y; r++) {
                s1 += B[o + r * a.tile_x];
                s2 += D[o + r * a.tile_x];
            }
            B[o] = s1;   // read above by this thread only
            D[o] = s2;
        }
        __syncthreads();
    }
    for (int q = tid; q < nI * nJ; q += nt) {
        const int J = q / nI, I = q - J * nI;
        const int IG = x0 / a.sr_x + I, JG = y0 / a.sr_y + J;
        if (IG >= a.nax || JG >= a.nay) continue;
        T s1 = T(0), s2 = T(0);
        if (some) {
            const int o = J * a.sr_y * a.tile_x + I * a.sr_x;
            for (int i = 0; i < a.sr_x; i++) {
                s1 += B[o + i];
                s2 += D[o + i];
            }
            const T cnt = T(min(nx - IG * a.sr_x, a.sr_x) * min(ny - JG * a.sr_y, a.sr_y));
            s1 = s1 / cnt;
            s2 = s2 / cnt;
        }
        p.fsens[(size_t)JG * a.nax + IG] = s1;
        p.flat[(size_t)JG * a.nax + IG] = s2;
    }
}

template <typename T, bool REC, int NPT>
__global__ void __launch_bounds__(1024)
k_step_small(const SmallParams<T> prm, const SmallPtrs<T> p, const T *__restrict__ coef) {
    extern __shared__ __attribute__((aligned(32))) double dyn_smem[];
    // the geometry table straight from the kernel's arguments (a uniform
    // index, so scalar loads)
    const IgnTable<T> *itab = reinterpret_cast<const IgnTable<T> *>(
        (const char *)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(SmallParams<T>, tab));
    small_tile<T, REC, NPT>(prm.a, p, itab, coef, blockIdx.x, prm.a.t,
                            reinterpret_cast<T *>(dyn_smem));
}

// An ensemble: the work list's tiles, each with its member's arrays; the model
// time and the current psi buffer are on the device.
template <typename T, int NPT>
__global__ void __launch_bounds__(1024)
k_ens_small(const StepArgs common, const SmallPtrs<T> base, const T *__restrict__ coef,
            const EnsDomain *__restrict__ doms, const int32_t *__restrict__ tile_dom,
            const EnsClock *__restrict__ clock, const char *__restrict__ itabs, T *psi_a,
            T *psi_b) {
    extern __shared__ __attribute__((aligned(32))) double dyn_smem[];
    const int g = blockIdx.x;
    const int di = __builtin_amdgcn_readfirstlane(tile_dom[g]);
    const EnsDomain &d = doms[di];
    const double tw = clock->t;
    StepArgs a = common;
    a.nx = d.nx;
    a.ny = d.ny;
    a.tiles_x = d.tiles_x;
    a.nax = d.nax;
    a.nay = d.nay;
    // ignitions only inside the window of their activity (none outside)
    a.nign = (tw >= d.t_ign_lo && tw <= d.t_ign_hi) ? d.nign : 0;
    a.dx = d.dx;
    a.dy = d.dy;
    a.rdx = d.rdx;
    a.rdy = d.rdy;
    const bool flip = clock->cur != 0;
    const int64_t c0 = d.cell_off, a0 = d.atm_off;
    SmallPtrs<T> p = base;
    p.psi_in = (flip ? psi_b : psi_a) + c0;
    p.psi_out = (flip ? psi_a : psi_b) + c0;
    p.tign += c0;
    p.frac += c0;
    p.u += c0;
    p.v += c0;
    p.gx += c0;
    p.gy += c0;
    p.cat += c0;
    p.fsens += a0;
    p.flat += a0;
    p.status += di;
    small_tile<T, false, NPT>(a, p,
                              reinterpret_cast<const IgnTable<T> *>(itabs + (size_t)di * kIgnTableBytes),
                              coef, g - d.tile0, tw, reinterpret_cast<T *>(dyn_smem));
}

template <typename T>
hipError_t launch_t(const StepArgs &a, const StepBuffers &b, const fire_ignition *ign,
                    hipStream_t s) {
    SmallPtrs<T> p;
    p.psi_in = (const T *)b.psi_in;
    p.psi_out = (T *)b.psi_out;
    p.tign = (T *)b.tign;
    p.frac = (T *)b.frac;
    p.u = (const T *)b.u;
    p.v = (const T *)b.v;
    p.gx = (const T *)b.dzdx;
    p.gy = (const T *)b.dzdy;
    p.cat = b.cat;
    p.fsens = (T *)b.fsens;
    p.flat = (T *)b.flat;
    p.status = b.status;
    p.rec_p0 = (T *)b.rec_p0;
    p.rec_b = (T *)b.rec_b;
    p.mark = b.mark;
    const T *coef = (const T *)b.coef;
    int npt, nt;
    small_block(a.tile_x, a.tile_y, &npt, &nt);
    const int F = (a.tile_x + 2 * kHalo) * (a.tile_y + 2 * kHalo);
    const size_t dyn = ((size_t)3 * F + a.ncat * kLRow + a.tile_x * a.tile_y) * sizeof(T) + 16;
    constexpr int kMost = sizeof(T) == 4 ? 2 : 1;   // nodes per thread (step_kind)
    if (npt > kMost || F > (npt + 2) * nt) return hipErrorInvalidValue;
    const dim3 grid(a.ntiles), blk(nt);
    if (b.ens_doms) {
        auto *fn = npt == 1 ? k_ens_small<T, 1> : k_ens_small<T, kMost>;
        hipLaunchKernelGGL(fn, grid, blk, dyn, s, a, p, coef, b.ens_doms, b.ens_tile_dom,
                           b.ens_clock, (const char *)b.ign_tab, (T *)b.psi_in, (T *)b.psi_out);
        return hipGetLastError();
    }
    SmallParams<T> prm;
    prm.a = a;
    for (int g = 0; g < FIRE_MAX_IGNITIONS; g++) {
        IgnGeo<T> geo = {};
        prm.tab.on[g] = g < a.nign && ign_setup<T>(ign[g], a.t, geo) ? 1 : 0;
        prm.tab.g[g] = geo;
    }
    auto *fn = b.rec_p0 ? (npt == 1 ? k_step_small<T, true, 1> : k_step_small<T, true, kMost>)
                        : (npt == 1 ? k_step_small<T, false, 1> : k_step_small<T, false, kMost>);
    hipLaunchKernelGGL(fn, grid, blk, dyn, s, prm, p, coef);
    return hipGetLastError();
}

}  // namespace

// Threads of a small tile: its nodes and those of its two inner rings, one
// per thread up to 1024, then two.
void small_block(int tile_x, int tile_y, int *npt, int *nt) {
    const int s1 = (tile_x + 4) * (tile_y + 4);
    *npt = s1 <= 1024 ? 1 : 2;
    *nt = ((s1 + *npt - 1) / *npt + 63) / 64 * 64;
}

hipError_t launch_step_small(int dtype, const StepArgs &a, const StepBuffers &b,
                             const fire_ignition *ign, hipStream_t s) {
    return dtype == FIRE_F64 ? launch_t<double>(a, b, ign, s) : launch_t<float>(a, b, ign, s);
}

}  // namespace fire

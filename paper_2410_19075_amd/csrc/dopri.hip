// Dormand-Prince 5(4) with step-size control on the device: rings held by one
// workgroup each, and (further below) rings of any size and compressed
// coupling matrices tiled over workgroups.
//
// The paper's default solver is the adaptive embedded pair of Dormand and
// Prince (Sec. III.A).  Every ring of up to 1024 elements is integrated
// by one workgroup from t = 0 to its own t_end: the state and the seven stage
// slopes stay in registers, each stage's window sums come from LDS prefix sums
// of the mapped stage values (as in the resident RK4 kernel), and the step
// control is the usual one (Hairer, Norsett & Wanner, Solving ODEs I, II.4):
//   err = sqrt(mean_i ((y5_i - y4_i) / (atol + rtol max(|y_i|, |y5_i|)))^2),
//   accept when err <= 1, new h = h min(facmax, max(0.2, 0.9 err^(-1/5))),
//   facmax = 10, or 1 right after a rejection; the step that reaches t_end
//   (to within a relative 1e-12 of h) ends on it; rtol <= 0 means fixed steps.
// A controlled run stops as failed when its error estimate is not finite (a
// NaN or Inf in the state or the slopes) or its proposed step falls below 10
// units in the last place of t; the state stays at the last accepted step.
// The fifth-order solution propagates, and the last stage is the first stage
// of the next step.  The error norm is one fixed-order block reduction, so the
// accept/reject decisions are the same in every run.  Each ring decides for
// itself: a batch of rings with different parameters and horizons runs in one
// launch without host round trips.
#include <cmath>

#include "models.h"
#include "carve.h"
#include "runtime.h"

namespace nd {

namespace {
constexpr int kDpBS = 512, kDpEPT = 2, kDpCap = kDpBS * kDpEPT;  // ring capacity 1024
constexpr int kDpStats = 5;  // per ring: t, accepted, rejected, next h, failed

__device__ __constant__ double kDpA[7][6] = {
    {0, 0, 0, 0, 0, 0},
    {1.0 / 5, 0, 0, 0, 0, 0},
    {3.0 / 40, 9.0 / 40, 0, 0, 0, 0},
    {44.0 / 45, -56.0 / 15, 32.0 / 9, 0, 0, 0},
    {19372.0 / 6561, -25360.0 / 2187, 64448.0 / 6561, -212.0 / 729, 0, 0},
    {9017.0 / 3168, -355.0 / 33, 46732.0 / 5247, 49.0 / 176, -5103.0 / 18656, 0},
    {35.0 / 384, 0, 500.0 / 1113, 125.0 / 192, -2187.0 / 6784, 11.0 / 84}};
// fifth- minus fourth-order weights
__device__ __constant__ double kDpE[7] = {71.0 / 57600, 0, -71.0 / 16695, 71.0 / 1920, -17253.0 / 339200,
                                           22.0 / 525, -1.0 / 40};
// continuous extension of order 4 (dense output; Hairer, Norsett & Wanner, Solving ODEs I, II.6)
__device__ __constant__ double kDpD[7] = {-12715105075.0 / 11282082432.0, 0.0, 87487479700.0 / 32700410799.0,
                                           -10690763975.0 / 1880347072.0, 701980252875.0 / 199316789632.0,
                                           -1453857185.0 / 822651844.0, 69997945.0 / 29380423.0};
}  // namespace

// Where the dense output goes: R (and optionally the state) of network b at
// output k is R[b * r_stride + k] (Y[b * y_stride + k * V * n + v * n + i]).
struct DenseOut {
    double t_out;  // output spacing (> 0: outputs at k * t_out, k = 0 .. floor(t_end / t_out))
    double* R;
    int64_t r_stride;
    double* Y;     // may be NULL
    int64_t y_stride;
};

// Bound: FP64 issue, six stages of the resident RK4 kernel's work and 34 coefficient
// FMAs per element and accepted step.  Measured per attempt (rings of 1024, one /
// 512): Kuramoto 8.3 / 19 us, FHN 6.9 / 14.6 us; with four barriers per stage, the
// prefix completed in LDS and branches on the wrap 14.1 / 25.6 and 12.9 / 26.7 us.
template <int MODEL, bool DENSE>
__device__ __forceinline__ void ring_dopri(const NetDesc* __restrict__ D, const double* __restrict__ t_end,
                                           double rtol, double atol, int64_t max_steps, double* __restrict__ stats,
                                           DenseOut out) {
    using M = RingModel<MODEL, double>;
    constexpr int V = M::V, EPT = kDpEPT, NW = kDpBS / kWave;
    // prefix k (sum of the maps before element k), k = 0 .. capacity, at k + k / EPT
    auto px = [](int k) { return (k + k / EPT) * (int)sizeof(double2); };
    __shared__ __align__(16) char pf[(kDpCap + kDpBS + 1) * sizeof(double2)];
    auto pre = [&](int off) -> double2& { return *(double2*)(pf + off); };
    __shared__ double2 wtot[NW];
    __shared__ double lds[2 * NW];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane(tid / kWave);
    const NetDesc& d = D[blockIdx.x];
    const int n = (int)d.n, P = (int)d.P;
    const ModelConst mc(d);
    const bool act = wid * kWave * EPT < n;  // waves without elements only join the barriers
    ND_GLOBAL double* y_g = gp(d.y[d.ypar]);
    double y[EPT][V], k[7][EPT][V];
    // window [i-P, i+P] = prefix(hi) - prefix(lo), plus the ring total where it wraps
    int hi[EPT], lo[EPT];
    bool wrap[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int i = tid * EPT + e;
        int h = i + P + 1, l = i - P;
        wrap[e] = l < 0 || h > n;
        if (l < 0) l += n;
        if (h > n) h -= n;
        hi[e] = px(i < n ? h : 0);
        lo[e] = px(i < n ? l : 0);
    }
    if (tid == 0) pre(0) = make_double2(0.0, 0.0);
    if (!act && lane == 0) wtot[wid] = make_double2(0.0, 0.0);
    const int rtot = px(n);
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int i = tid * EPT + e;
#pragma unroll
        for (int v = 0; v < V; ++v) y[e][v] = i < n ? y_g[(int64_t)v * n + i] : 0.0;
    }
    // slopes of stage value z: map, block prefix sums, window sums, RHS.  Two barriers
    // and one LDS write per element, as in the resident RK4 kernel: the next stage's
    // wave totals are written after this stage's second barrier, its prefixes after
    // the first barrier that follows this stage's reads.  (Elements past n compute
    // slopes nobody reads.)
    auto slopes = [&](const double (&z)[EPT][V], double (&kout)[EPT][V]) {
        double2 x[EPT], in[EPT];
        double2 ex = make_double2(0.0, 0.0);
        if (act) {
            double2 tot = make_double2(0.0, 0.0);
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                x[e] = M::map(z[e]);
                if (tid * EPT + e >= n) x[e] = make_double2(0.0, 0.0);
                tot.x += x[e].x;
                tot.y += x[e].y;
                in[e] = tot;
            }
            const double2 incl = make_double2(wave_incl_scan(tot.x), wave_incl_scan(tot.y));
            if (lane == kWave - 1) wtot[wid] = incl;
            ex = make_double2(wave_shift_up1(incl.x), wave_shift_up1(incl.y));
        }
        lds_barrier();
        if (act) {
            const double2 before = waves_before<NW>(wtot, wid);
            ex.x += before.x;
            ex.y += before.y;
#pragma unroll
            for (int e = 0; e < EPT; ++e)
                pre(px(tid * EPT + e + 1)) = make_double2(ex.x + in[e].x, ex.y + in[e].y);
        }
        lds_barrier();
        if (act) {
            const double2 T = pre(rtot);
            double2 ph[EPT], pl[EPT];
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                ph[e] = pre(hi[e]);
                pl[e] = pre(lo[e]);
            }
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                const double2 t = wrap[e] ? T : make_double2(0.0, 0.0);
                const double2 W = make_double2(ph[e].x + (t.x - pl[e].x) - x[e].x, ph[e].y + (t.y - pl[e].y) - x[e].y);
                M::rhs(mc, z[e], x[e], W, kout[e]);
            }
        }
    };
    // dense output k: the state y + hs sum_q w_q(theta) k_q (theta = 0: y itself), its
    // order parameter by a fixed-order block reduction
    auto emit = [&](int64_t kout, double theta, double hs) {
        double wt[7];
#pragma unroll
        for (int q = 0; q < 7; ++q) {
            const double b = q < 6 ? kDpA[6][q] : 0.0, e1 = q == 0 ? 1.0 : 0.0, e7 = q == 6 ? 1.0 : 0.0;
            wt[q] = theta * (b + (1.0 - theta) * (e1 - b + theta * (2.0 * b - e1 - e7 + (1.0 - theta) * kDpD[q])));
        }
        double s2[2] = {0.0, 0.0};
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int i = tid * EPT + e;
            if (i >= n) continue;
            double yt[V];
#pragma unroll
            for (int v = 0; v < V; ++v) {
                double a = 0.0;
#pragma unroll
                for (int q = 0; q < 7; ++q) a += wt[q] * k[q][e][v];
                yt[v] = theta == 0.0 ? y[e][v] : y[e][v] + hs * a;
                if (out.Y) gp(out.Y)[blockIdx.x * out.y_stride + kout * V * n + (int64_t)v * n + i] = yt[v];
            }
            if constexpr (MODEL == ND_FHN) {
                const double r = sqrt(yt[0] * yt[0] + yt[1] * yt[1]);
                s2[0] += yt[0] / r;
                s2[1] += yt[1] / r;
            } else {
                const double2 x = M::map(yt);
                s2[0] += x.x;
                s2[1] += x.y;
            }
        }
        block_sum<kDpBS, 2>(s2, lds);
        if (tid == 0) gp(out.R)[blockIdx.x * out.r_stride + kout] = sqrt(s2[0] * s2[0] + s2[1] * s2[1]) / (double)n;
    };
    slopes(y, k[0]);
    const double tend = t_end[blockIdx.x];
    double t = 0.0, h = d.dt, facmax = 10.0;
    int64_t acc = 0, rej = 0;
    const int64_t K = DENSE ? (int64_t)floor(tend / out.t_out) : -1;
    int64_t next = 0;
    if (DENSE && K >= 0) {
        emit(0, 0.0, 0.0);
        next = 1;
    }
    // every wave leaves the loop together: t, h, err and the counters are uniform
    bool failed = false;
    while (t < tend && acc + rej < max_steps) {
        if (rtol > 0.0 && h < 10.0 * (nextafter(t, INFINITY) - t)) {  // step below its floor
            failed = true;
            break;
        }
        const bool last = tend - t <= h * (1.0 + 1e-12);
        const double hs = last ? tend - t : h;
        double z[EPT][V];
#pragma unroll
        for (int s = 1; s < 7; ++s) {
#pragma unroll
            for (int e = 0; e < EPT; ++e)
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    double a = 0.0;
#pragma unroll
                    for (int q = 0; q < s; ++q) a = fma(kDpA[s][q], k[q][e][v], a);
                    z[e][v] = fma(hs, a, y[e][v]);
                }
            slopes(z, k[s]);
        }
        // z is the fifth-order solution (stage 7 uses the weights b)
        bool accept = true;
        double f = 1.0;
        if (rtol > 0.0) {
            double sum[1] = {0.0};
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                if (tid * EPT + e >= n) continue;
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    double er = 0.0;
#pragma unroll
                    for (int q = 0; q < 7; ++q) er = fma(kDpE[q], k[q][e][v], er);
                    er *= hs;
                    const double sc = fma(rtol, fmax(fabs(y[e][v]), fabs(z[e][v])), atol);
                    sum[0] += (er / sc) * (er / sc);
                }
            }
            block_sum<kDpBS, 1>(sum, lds);
            const double err = sqrt(sum[0] / (double)(V * n));
            if (!isfinite(err)) {  // a NaN or Inf in the state or the slopes
                failed = true;
                break;
            }
            f = 0.9 * pow(err, -0.2);
            accept = err <= 1.0;
        }
        if (accept) {
            if constexpr (DENSE) {
                // outputs inside (t, t + hs]; the last step takes every one left
                const double tn = last ? tend : t + hs;
                for (; next <= K; ++next) {
                    const double tk = (double)next * out.t_out;
                    if (tk > tn && !last) break;
                    emit(next, fmin((tk - t) / hs, 1.0), hs);
                }
            }
#pragma unroll
            for (int e = 0; e < EPT; ++e)
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    y[e][v] = z[e][v];
                    k[0][e][v] = k[6][e][v];
                }
            t = last ? tend : t + hs;
            ++acc;
            if (rtol > 0.0) h = hs * fmin(facmax, fmax(0.2, f));
            facmax = 10.0;
        } else {
            ++rej;
            h = hs * fmax(0.2, fmin(1.0, f));
            facmax = 1.0;
        }
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int i = tid * EPT + e;
        if (i < n) {
#pragma unroll
            for (int v = 0; v < V; ++v) y_g[(int64_t)v * n + i] = y[e][v];
        }
    }
    if (tid == 0) {
        ND_GLOBAL double* st = gp(stats) + kDpStats * blockIdx.x;
        st[0] = t;
        st[1] = (double)acc;
        st[2] = (double)rej;
        st[3] = h;
        st[4] = failed ? 1.0 : 0.0;
    }
}

template <int MODEL, bool DENSE>
__global__ __launch_bounds__(kDpBS) void k_ring_dopri(const NetDesc* __restrict__ D,
                                                      const double* __restrict__ t_end, double rtol, double atol,
                                                      int64_t max_steps, double* __restrict__ stats, DenseOut out) {
    ring_dopri<MODEL, DENSE>(D, t_end, rtol, atol, max_steps, stats, out);
}

// The Kuramoto ring without dense output fits 128 registers per lane, so two
// rings (workgroups of 8 waves) share a CU and hide each other's barriers.
__global__ __launch_bounds__(kDpBS) __attribute__((amdgpu_waves_per_eu(4))) void k_ring_dopri_kuramoto(
    const NetDesc* __restrict__ D, const double* __restrict__ t_end, double rtol, double atol, int64_t max_steps,
    double* __restrict__ stats, DenseOut out) {
    ring_dopri<ND_KURAMOTO, false>(D, t_end, rtol, atol, max_steps, stats, out);
}


// ------------------------------------------------------------ tiled rings
// Rings larger than one workgroup and compressed coupling matrices: the same method
// and step control over tiles, one launch per stage.  The launch of stage s takes
// the neighbour sums of the stage value z_s from what the launch before it left
// (rings: global prefix sums of the map; matrices: the maps), evaluates the slope
// and, since z_{s+1} needs no slope of another element, goes on to z_{s+1}, its map
// and the tile's prefix sums, double-buffered.  An attempt is the launch that forms
// z_1 (it depends on the controller's step), six stage launches and one controller
// launch that takes the accept / reject decision on the device.  The host replays
// attempts in groups and only reads back whether every network is done.
// Window sums come from global prefix sums of the map: the prefix of element k
// is its tile's offset (fixed-order scan of the tile totals) plus its in-tile
// inclusive prefix.
// Bound: launches and their latency up to some 10^5 elements, HBM beyond, the rows'
// gathers for matrices.  Per attempt, against a map launch and an RHS launch per
// stage: FHN ring of 65,536 90 -> 69 us, of 10^6 361 -> 307 us, four Kuramoto rings of
// 65,536 132 -> 107 us; 60^3 inertia matrix network (33 links a row) with its outputs
// 4.22 -> 2.74 ms a run to t = 50, its tiles of 512 -> 256 and the outputs' slopes read
// once included.
constexpr int kDtBS = 256;
// Elements per thread and tile: matrices take one, which gives twice the workgroups
// to hide the gathers (and needs no prefix); rings two, which halves the tile totals
// every workgroup scans.
template <int TOPO>
struct DtTile {
    static constexpr int EPT = TOPO == ND_LINKS ? 1 : 2, T = kDtBS * EPT;
};
// rings of at most this many tiles get their tile offsets in each RHS workgroup
// (a scan of the tile totals into LDS); longer rings in a launch of their own
constexpr int kDtScanMax = 2048;

// Per-ring control block, advanced by the controller on the device.
struct DtCtl {
    double t, h, hs, facmax;
    int64_t acc, rej;
    int32_t done, last, f, ypar;  // f: physical buffer of k1 (k_q lives at (f + q - 1) mod 7)
    // dense output: outputs [out_lo, out_hi) lie in the step just accepted, which
    // started at t_prev with size hs_prev, state y[ypar_prev] and k1 at f_prev
    int64_t next, out_lo, out_hi;
    double t_prev, hs_prev;
    int32_t f_prev, ypar_prev;
    int32_t failed, pad_;  // failed: non-finite error estimate or step below its floor
};

// Per-ring buffers of one call.
struct DtNet {
    int32_t n, P, G, V;
    double tend;
    double* y[2];     // state, and the fifth-order solution of the attempt
    double* k[7];     // stage slopes (physical buffers)
    double* Z;        // stage value of stages 1 .. 5 (stage 0 is y, stage 6 goes to y[ypar ^ 1])
    // of the stage value of stage s, in buffer s & 1:
    double* M[2];     // matrices: [n] its map, as double2
    double* pre[2];   // rings: [2][n] in-tile inclusive prefix of its map
    double* tot[2];   // rings: [2][G] tile totals, then (after the offsets launch) exclusive offsets
    double* errp;     // [G] error partial sums of the attempt
    DtCtl* ctl;
    int64_t K;        // dense output: last output index (-1: none)
    double* Rpart;    // dense output: [K + 1][G][2] per-tile sums of the order parameter
    double* R;        // dense output: R of outputs 0 .. K (device)
    double* Y;        // dense output: states at the outputs (device, may be NULL)
};

// What a launch leaves for the stage that follows: the maps (matrices) or the tile's
// inclusive prefix sums and totals (rings) of the tile's stage values, in buffer b.
// Element e * kDtBS + tid of the tile belongs to thread tid, so every access of a
// wave is one contiguous run.  lds: 4 * EPT * (kDtBS / 64) doubles.
template <int TOPO>
__device__ __forceinline__ void dt_leave(const DtNet& r, int b, int tile, const double2 (&x)[DtTile<TOPO>::EPT],
                                         double* lds) {
    constexpr int EPT = DtTile<TOPO>::EPT, T = DtTile<TOPO>::T, NE = 2 * EPT;
    const int n = r.n, i0 = tile * T + (int)threadIdx.x;
    if constexpr (TOPO == ND_LINKS) {
#pragma unroll
        for (int e = 0; e < EPT; ++e)
            if (i0 + e * kDtBS < n) ((double2*)r.M[b])[i0 + e * kDtBS] = x[e];
    } else {
        // block sums and thread-exclusive prefixes of each element run
        double bs[NE], ex[NE];
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            bs[2 * e] = ex[2 * e] = x[e].x;
            bs[2 * e + 1] = ex[2 * e + 1] = x[e].y;
        }
        block_sum_and_exscan<kDtBS, NE, NE>(bs, ex, lds);
        double off0 = 0.0, off1 = 0.0;
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int i = i0 + e * kDtBS;
            if (i < n) {
                r.pre[b][i] = off0 + (ex[2 * e] + x[e].x);
                r.pre[b][n + i] = off1 + (ex[2 * e + 1] + x[e].y);
            }
            off0 += bs[2 * e];
            off1 += bs[2 * e + 1];
        }
        if (threadIdx.x == 0) {
            r.tot[b][tile] = off0;
            r.tot[b][r.G + tile] = off1;
        }
    }
}

// The stage value of stage S = 0 (the state, before the first slope) or 1 (z_1 = y +
// h a_10 k_1 of an attempt) and what the stage launch needs of it.
template <int MODEL, int TOPO, int S>
__global__ __launch_bounds__(kDtBS) void k_dt_begin(const DtNet* __restrict__ R, const int2* __restrict__ work,
                                                    int nwork) {
    using M = RingModel<MODEL, double>;
    constexpr int V = M::V, EPT = DtTile<TOPO>::EPT, T = DtTile<TOPO>::T;
    __shared__ double lds[4 * EPT * (kDtBS / kWave)];
    const int w = xcd_work(blockIdx.x, nwork);
    if (w < 0) return;
    const int2 wk = work[w];
    const DtNet& r = R[wk.x];
    const DtCtl c = *r.ctl;
    if (c.done) return;
    const int n = r.n;
    const double* __restrict__ y = r.y[c.ypar];
    const double* __restrict__ k0 = r.k[c.f % 7];
    double2 x[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int i = wk.y * T + e * kDtBS + (int)threadIdx.x;
        x[e] = make_double2(0.0, 0.0);
        if (i < n) {
            double z[V];
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const int64_t o = (int64_t)v * n + i;
                z[v] = S == 0 ? y[o] : fma(c.hs, kDpA[1][0] * k0[o], y[o]);
                if (S > 0) r.Z[o] = z[v];
            }
            x[e] = M::map(z);
        }
    }
    dt_leave<TOPO>(r, S & 1, wk.y, x, lds);
}

// Exclusive offsets of the tiles of buffer b (one workgroup per ring, fixed order).
__global__ __launch_bounds__(kDtBS) void k_dt_offsets(const DtNet* __restrict__ R, int b) {
    const DtNet& r = R[blockIdx.x];
    if (r.ctl->done || r.G <= kDtScanMax) return;
    __shared__ double lds[4 * (kDtBS / kWave)];
    __shared__ double chunk[2];
    double* tot = r.tot[b];
    double carry0 = 0.0, carry1 = 0.0;
    for (int b0 = 0; b0 < r.G; b0 += kDtBS) {
        const int q = b0 + (int)threadIdx.x;
        const double own0 = q < r.G ? tot[q] : 0.0, own1 = q < r.G ? tot[r.G + q] : 0.0;
        double v[2] = {own0, own1};
        block_exscan<kDtBS, 2>(v, lds);  // v: exclusive prefix in this chunk
        if (threadIdx.x == kDtBS - 1) {
            chunk[0] = v[0] + own0;
            chunk[1] = v[1] + own1;
        }
        if (q < r.G) {
            tot[q] = carry0 + v[0];
            tot[r.G + q] = carry1 + v[1];
        }
        __syncthreads();
        carry0 += chunk[0];
        carry1 += chunk[1];
        __syncthreads();
    }
}

// Stage S of an attempt (0: the first slope of the run): neighbour sums of z_S
// (ring: windows from the global prefix; links: the compressed coupling matrix's
// rows, extracted as in the stage kernels of that topology), the RHS into k_{S+1},
// then for S = 1 .. 5 z_{S+1} (the fifth-order solution, S = 5, into y[ypar ^ 1]) and
// what its stage needs, for S = 6 the error terms of the attempt.  The stage is a
// template parameter so the slopes' loads are all issued before the sums that use
// them.
template <int MODEL, int TOPO, int S>
__global__ __launch_bounds__(kDtBS) void k_dt_stage(const DtNet* __restrict__ R, const NetDesc* __restrict__ D,
                                                    const int2* __restrict__ work, int nwork, double rtol,
                                                    double atol) {
    using M = RingModel<MODEL, double>;
    constexpr int V = M::V, EPT = DtTile<TOPO>::EPT, T = DtTile<TOPO>::T, b = S & 1;
    constexpr bool kNext = S >= 1 && S <= 5;
    __shared__ double lds[4 * EPT * (kDtBS / kWave)];
    extern __shared__ double dt_off[];  // [2][G]: exclusive tile offsets (rings of <= kDtScanMax tiles)
    // row tiles that share gathers stay on one XCD (its own L2)
    const int w = xcd_work(blockIdx.x, nwork);
    if (w < 0) return;
    const int2 wk = work[w];
    const DtNet& r = R[wk.x];
    const NetDesc& d = D[wk.x];
    const DtCtl c = *r.ctl;
    if (c.done) return;
    const int n = r.n, P = r.P, t0 = wk.y * T, tid = threadIdx.x;
    const int G = r.G;
    const bool local = TOPO == ND_RING && G <= kDtScanMax;  // uniform over the block
    const double* __restrict__ tot = r.tot[b];
    const double* __restrict__ pre = r.pre[b];
    if (local) {
        // each thread adds a run of consecutive tile totals; the block scans the
        // runs' sums; every workgroup of the ring computes the same offsets
        const int per = (G + kDtBS - 1) / kDtBS, u0 = min(tid * per, G), u1 = min(u0 + per, G);
        double v[2] = {0.0, 0.0};
        for (int u = u0; u < u1; ++u) {
            v[0] += tot[u];
            v[1] += tot[G + u];
        }
        block_exscan<kDtBS, 2>(v, lds);
        for (int u = u0; u < u1; ++u) {
            dt_off[u] = v[0];
            dt_off[G + u] = v[1];
            v[0] += tot[u];
            v[1] += tot[G + u];
        }
        __syncthreads();
    }
    auto prefix = [&](int k, int comp) {  // inclusive global prefix of element k (k = -1: 0)
        if (k < 0) return 0.0;
        const double o = local ? dt_off[comp * G + k / T] : tot[comp * G + k / T];
        return o + pre[comp * n + k];
    };
    const double* y = r.y[c.ypar];
    const double* zs = S == 0 ? y : (S == 6 ? r.y[c.ypar ^ 1] : r.Z);
    double* kq[S + 1];
#pragma unroll
    for (int q = 0; q <= S; ++q) kq[q] = r.k[(c.f + q) % 7];
    double* zo = S == 5 ? r.y[c.ypar ^ 1] : r.Z;
    double es[1] = {0.0};
    double2 xn[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int i = t0 + e * kDtBS + tid;
        xn[e] = make_double2(0.0, 0.0);
        if (i >= n) continue;
        // own operands of the next stage value, in flight during the neighbour sums
        double yv[V], av[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int64_t o = (int64_t)v * n + i;
            yv[v] = kNext || S == 6 ? y[o] : 0.0;
            av[v] = 0.0;
            if constexpr (kNext) {
#pragma unroll
                for (int q = 0; q < S; ++q) av[v] = fma(kDpA[S + 1][q], kq[q][o], av[v]);
            }
            if constexpr (S == 6) {
#pragma unroll
                for (int q = 0; q < S; ++q) av[v] = fma(kDpE[q], kq[q][o], av[v]);
            }
        }
        double z[V];
#pragma unroll
        for (int v = 0; v < V; ++v) z[v] = zs[(int64_t)v * n + i];
        // the element's own map: stored by the launch before where the rows gather
        // maps anyway, else recomputed from the same stage value (same bits)
        const double2 x = TOPO == ND_LINKS ? ((const double2*)r.M[b])[i] : M::map(z);
        double2 W;
        if constexpr (TOPO == ND_RING) {
            const int lo = i - P, hi = i + P;
            double w0, w1;
            if (lo < 0) {
                w0 = prefix(hi, 0) + (prefix(n - 1, 0) - prefix(lo + n - 1, 0));
                w1 = prefix(hi, 1) + (prefix(n - 1, 1) - prefix(lo + n - 1, 1));
            } else if (hi >= n) {
                w0 = (prefix(n - 1, 0) - prefix(lo - 1, 0)) + prefix(hi - n, 0);
                w1 = (prefix(n - 1, 1) - prefix(lo - 1, 1)) + prefix(hi - n, 1);
            } else {
                w0 = prefix(hi, 0) - prefix(lo - 1, 0);
                w1 = prefix(hi, 1) - prefix(lo - 1, 1);
            }
            W = make_double2(w0 - x.x, w1 - x.y);
        } else {
            // row i = (V XOR D[C_i]) shifted by i: V's positions, then the entry's
            // signed positions, divided by the row's link count
            const double2* __restrict__ mp = (const double2*)r.M[b];
            double w0 = 0.0, w1 = 0.0;
#pragma unroll 8
            for (int q = 0; q < d.lnv; ++q) {
                int j = i + d.lvpos[q];
                j -= j >= n ? n : 0;
                const double2 m = mp[j];
                w0 += m.x;
                w1 += m.y;
            }
            const int ke = d.lrow[i];
            for (int e2 = d.ldptr[ke]; e2 < d.ldptr[ke + 1]; ++e2) {
                const int32_t v = d.ldpos[e2];
                int j = i + (v & ~kLinksRemove);
                j -= j >= n ? n : 0;
                const double sg = (v & kLinksRemove) ? -1.0 : 1.0;
                const double2 m = mp[j];
                w0 += sg * m.x;
                w1 += sg * m.y;
            }
            const double inv = d.linv[ke];
            W = inv != 0.0 ? make_double2(w0 * inv, w1 * inv)
                           : (MODEL == ND_FHN ? make_double2(z[0], z[V - 1]) : make_double2(0.0, 0.0));
        }
        double k[V];
        M::rhs(d, z, x, W, k);
        double zn[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int64_t o = (int64_t)v * n + i;
            kq[S][o] = k[v];
            if constexpr (kNext) {
                zn[v] = fma(c.hs, fma(kDpA[S + 1][S], k[v], av[v]), yv[v]);
                zo[o] = zn[v];
            }
            if constexpr (S == 6) {
                if (rtol > 0.0) {
                    const double er = fma(kDpE[6], k[v], av[v]) * c.hs;
                    const double sc = fma(rtol, fmax(fabs(yv[v]), fabs(z[v])), atol);
                    es[0] += (er / sc) * (er / sc);
                }
            }
        }
        if constexpr (kNext) xn[e] = M::map(zn);
    }
    if constexpr (kNext) dt_leave<TOPO>(r, b ^ 1, wk.y, xn, lds);
    if constexpr (S == 6) {
        block_sum<kDtBS, 1>(es, lds);
        if (tid == 0) r.errp[wk.y] = es[0];
    }
}

// The accept / reject decision of the attempt and the next step (one wave per
// ring: lane l adds the error partials of tiles l, l + 64, ... in order, the
// wave adds the lanes' sums in a fixed tree; lane 0 decides).
__global__ __launch_bounds__(kWave) void k_dt_control(const DtNet* __restrict__ R, double rtol, int64_t max_steps,
                                                       double t_out) {
    const DtNet& r = R[blockIdx.x];
    double sum = 0.0;
    if (rtol > 0.0 && !r.ctl->done) {  // uniform over the wave
        for (int q = threadIdx.x; q < r.G; q += kWave) sum += r.errp[q];
        sum = wave_sum(sum);
    }
    if (threadIdx.x != 0) return;
    DtCtl c = *r.ctl;
    if (c.done) {
        if (c.out_hi != c.out_lo) {  // nothing more to emit
            c.out_lo = c.out_hi = 0;
            *r.ctl = c;
        }
        return;
    }
    c.out_lo = c.out_hi = 0;
    bool accept = true;
    double f = 1.0;
    if (rtol > 0.0) {
        const double err = sqrt(sum / ((double)r.V * (double)r.n));
        if (!isfinite(err)) {  // a NaN or Inf in the state or the slopes: stop, state kept
            c.failed = 1;
            c.done = 1;
            *r.ctl = c;
            return;
        }
        f = 0.9 * pow(err, -0.2);
        accept = err <= 1.0;
    }
    if (accept) {
        if (r.K >= 0) {  // outputs inside (t, t + hs]; the last step takes every one left
            const double tn = c.last ? r.tend : c.t + c.hs;
            c.out_lo = c.next;
            while (c.next <= r.K && ((double)c.next * t_out <= tn || c.last)) ++c.next;
            c.out_hi = c.next;
            c.t_prev = c.t;
            c.hs_prev = c.hs;
            c.f_prev = c.f;
            c.ypar_prev = c.ypar;
        }
        c.t = c.last ? r.tend : c.t + c.hs;
        ++c.acc;
        if (rtol > 0.0) c.h = c.hs * fmin(c.facmax, fmax(0.2, f));
        c.facmax = 10.0;
        c.ypar ^= 1;
        c.f = (c.f + 6) % 7;  // k1 of the next step is this step's k7
    } else {
        ++c.rej;
        c.h = c.hs * fmax(0.2, fmin(1.0, f));
        c.facmax = 1.0;
    }
    c.done = !(c.t < r.tend && c.acc + c.rej < max_steps);
    if (!c.done && rtol > 0.0 && c.h < 10.0 * (nextafter(c.t, INFINITY) - c.t)) {  // step below its floor
        c.failed = 1;
        c.done = 1;
    }
    if (!c.done) {
        c.last = r.tend - c.t <= c.h * (1.0 + 1e-12);
        c.hs = c.last ? r.tend - c.t : c.h;
    }
    *r.ctl = c;
}

// Dense output of the step just accepted: the continuous extension on the tile's
// elements at each of its outputs (the state, when requested) and the tile's sums of
// the order parameter's unit vectors.  The slopes are read once for all outputs.
template <int MODEL, int TOPO>
__global__ __launch_bounds__(kDtBS) void k_dt_emit(const DtNet* __restrict__ R, const int2* __restrict__ work,
                                                   double t_out) {
    using M = RingModel<MODEL, double>;
    constexpr int V = M::V, NW = kDtBS / kWave, EPT = DtTile<TOPO>::EPT, T = DtTile<TOPO>::T;
    __shared__ double lds[2 * NW];
    const int2 wk = work[blockIdx.x];
    const DtNet& r = R[wk.x];
    const DtCtl c = *r.ctl;
    if (c.out_hi <= c.out_lo) return;
    const int n = r.n, t0 = wk.y * T, tid = threadIdx.x;
    const double* y = r.y[c.ypar_prev];
    const bool start = c.out_lo == 0;  // output 0 is the initial state (no stage slopes yet)
    double yv[EPT][V], kv[EPT][V][7];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int i = t0 + e * kDtBS + tid;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            yv[e][v] = i < n ? y[(int64_t)v * n + i] : 0.0;
#pragma unroll
            for (int q = 0; q < 7; ++q)
                kv[e][v][q] = i < n && !start ? r.k[(c.f_prev + q) % 7][(int64_t)v * n + i] : 0.0;
        }
    }
    for (int64_t ko = c.out_lo; ko < c.out_hi; ++ko) {
        const double theta = fmin(((double)ko * t_out - c.t_prev) / c.hs_prev, 1.0);
        double wt[7];
#pragma unroll
        for (int q = 0; q < 7; ++q) {
            const double b = q < 6 ? kDpA[6][q] : 0.0, e1 = q == 0 ? 1.0 : 0.0, e7 = q == 6 ? 1.0 : 0.0;
            wt[q] = theta * (b + (1.0 - theta) * (e1 - b + theta * (2.0 * b - e1 - e7 + (1.0 - theta) * kDpD[q])));
        }
        double s2[2] = {0.0, 0.0};
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int i = t0 + e * kDtBS + tid;
            if (i >= n) continue;
            double yt[V];
#pragma unroll
            for (int v = 0; v < V; ++v) {
                yt[v] = yv[e][v];
                if (theta != 0.0) {
                    double a = 0.0;
#pragma unroll
                    for (int q = 0; q < 7; ++q) a += wt[q] * kv[e][v][q];
                    yt[v] += c.hs_prev * a;
                }
                if (r.Y) r.Y[ko * V * n + (int64_t)v * n + i] = yt[v];
            }
            if constexpr (MODEL == ND_FHN) {
                const double rr = sqrt(yt[0] * yt[0] + yt[1] * yt[1]);
                s2[0] += yt[0] / rr;
                s2[1] += yt[1] / rr;
            } else {
                const double2 x = M::map(yt);
                s2[0] += x.x;
                s2[1] += x.y;
            }
        }
        block_sum<kDtBS, 2>(s2, lds);
        if (tid == 0) {
            r.Rpart[(ko * r.G + wk.y) * 2] = s2[0];
            r.Rpart[(ko * r.G + wk.y) * 2 + 1] = s2[1];
        }
    }
}

// R of every emitted output from the tiles' sums: block (ring, y) takes outputs
// y, y + kDtRBlocks, ...; thread l adds tiles l, l + kDtBS, ... in order and
// the block adds the threads' sums in a fixed order.
constexpr int kDtRBlocks = 64;
__global__ __launch_bounds__(kDtBS) void k_dt_reduce_R(const DtNet* __restrict__ R) {
    constexpr int NW = kDtBS / kWave;
    __shared__ double lds[2 * NW];
    const DtNet& r = R[blockIdx.x];
    const int64_t emitted = min(r.ctl->next, r.K + 1);
    for (int64_t ko = blockIdx.y; ko < emitted; ko += kDtRBlocks) {  // uniform over the block
        double s2[2] = {0.0, 0.0};
        for (int q = threadIdx.x; q < r.G; q += kDtBS) {
            s2[0] += r.Rpart[(ko * r.G + q) * 2];
            s2[1] += r.Rpart[(ko * r.G + q) * 2 + 1];
        }
        block_sum<kDtBS, 2>(s2, lds);
        if (threadIdx.x == 0) r.R[ko] = sqrt(s2[0] * s2[0] + s2[1] * s2[1]) / (double)r.n;
    }
}
}  // namespace nd

using namespace nd;

// The tiled kernels of one model and topology.
struct DtKernels {
    void (*begin[2])(const DtNet*, const int2*, int);
    void (*stage[7])(const DtNet*, const NetDesc*, const int2*, int, double, double);
    void (*emit)(const DtNet*, const int2*, double);
    int tile;
};
template <int MODEL, int TOPO>
static DtKernels dt_kernels() {
    return {{k_dt_begin<MODEL, TOPO, 0>, k_dt_begin<MODEL, TOPO, 1>},
            {k_dt_stage<MODEL, TOPO, 0>, k_dt_stage<MODEL, TOPO, 1>, k_dt_stage<MODEL, TOPO, 2>,
             k_dt_stage<MODEL, TOPO, 3>, k_dt_stage<MODEL, TOPO, 4>, k_dt_stage<MODEL, TOPO, 5>,
             k_dt_stage<MODEL, TOPO, 6>},
            k_dt_emit<MODEL, TOPO>,
            DtTile<TOPO>::T};
}
template <int TOPO>
static DtKernels dt_kernels_of(int model) {
    if (model == ND_KURAMOTO) return dt_kernels<ND_KURAMOTO, TOPO>();
    if (model == ND_FHN) return dt_kernels<ND_FHN, TOPO>();
    return dt_kernels<ND_KURAMOTO_INERTIA, TOPO>();
}

// Rings beyond one workgroup: buffers per ring, the stage / controller launches
// replayed in groups of attempts until every ring is done.
static nd_status run_adaptive_tiled(const std::vector<Net*>& nets, int model, int topo, const double* t_end,
                                    const double* dt0, double rtol, double atol, int64_t max_steps,
                                    nd_adaptive_stats* stats, hipStream_t st, double t_out, double* Rh,
                                    int64_t r_stride, double* Yh, int64_t y_stride) {
    const bool dense = t_out > 0.0;
    const DtKernels kern = topo == ND_RING ? dt_kernels_of<ND_RING>(model) : dt_kernels_of<ND_LINKS>(model);
    const int64_t T = kern.tile;
    const int count = (int)nets.size();
    std::vector<DtNet> rs(count);
    std::vector<DtCtl> cs(count);
    std::vector<NetDesc> descs(count);
    std::vector<int2> work;
    for (int b = 0; b < count; ++b) {
        const int64_t G = (nets[b]->prob.n + T - 1) / T;
        for (int64_t t = 0; t < G; ++t) work.push_back(make_int2(b, (int)t));
    }
    const size_t bd = (size_t)count * sizeof(DtNet), bn = (size_t)count * sizeof(NetDesc),
                 bw = work.size() * sizeof(int2);
    const size_t br = dense ? (size_t)count * r_stride * 8 : 0, by = dense && Yh ? (size_t)count * y_stride * 8 : 0;
    DtNet* d_r = nullptr;
    NetDesc* d_desc = nullptr;
    int2* d_work = nullptr;
    double* d_out = nullptr;  // dense output: R, then the states
    auto lay = [&](Carve c) {
        d_r = c.take<DtNet>(count);
        d_desc = c.take<NetDesc>(count);
        d_work = c.take<int2>(work.size());
        for (int b = 0; b < count; ++b) {
            const int64_t n = nets[b]->prob.n, len = nvars_of(nets[b]->prob.model) * n, G = (n + T - 1) / T;
            DtNet& r = rs[b];
            r.y[1] = c.take<double>(len);
            for (int q = 0; q < 7; ++q) r.k[q] = c.take<double>(len);
            r.Z = c.take<double>(len);
            for (int b2 = 0; b2 < 2; ++b2) {  // a network needs the maps or the prefix sums
                double* q = c.take<double>(2 * n);
                r.M[b2] = topo == ND_LINKS ? q : nullptr;
                r.pre[b2] = topo == ND_LINKS ? nullptr : q;
                r.tot[b2] = c.take<double>(2 * G);
            }
            r.errp = c.take<double>(G);
            r.ctl = c.take<DtCtl>(1);
            r.K = dense ? (int64_t)std::floor(t_end[b] / t_out) : -1;
            r.Rpart = dense ? c.take<double>(2 * (r.K + 1) * G) : nullptr;
        }
        d_out = c.take<double>((br + by) / 8);
        return c.bytes();
    };
    char* buf = nullptr;
    hipError_t e = hipMallocAsync((void**)&buf, lay(Carve()), st);
    if (e != hipSuccess) return hip_fail(e, "adaptive scratch");
    lay(Carve(buf));
    for (int b = 0; b < count; ++b) {
        const Net* nt = nets[b];
        const int64_t n = nt->prob.n;
        DtNet& r = rs[b];
        r.n = (int32_t)n;
        r.P = (int32_t)nt->prob.radius;
        r.G = (int32_t)((n + T - 1) / T);
        r.V = nvars_of(nt->prob.model);
        r.tend = t_end[b];
        descs[b] = nt->run_desc(dt0[b], 0);
        r.y[0] = descs[b].y[descs[b].ypar];
        r.R = nullptr;
        r.Y = nullptr;
        DtCtl& c = cs[b];
        c = DtCtl{};
        c.h = dt0[b];
        c.facmax = 10.0;
        c.done = !(0.0 < t_end[b] && max_steps > 0);
        if (!c.done && rtol > 0.0 && c.h < 10.0 * std::nextafter(0.0, INFINITY)) {  // step below its floor
            c.failed = 1;
            c.done = 1;
        }
        c.last = t_end[b] <= c.h * (1.0 + 1e-12);
        c.hs = c.last ? t_end[b] : c.h;
        if (r.K >= 0) {  // output 0 is the initial state (theta = 0)
            c.out_lo = 0;
            c.out_hi = 1;
            c.next = 1;
            c.hs_prev = 1.0;
        }
    }
    double* d_R = dense ? d_out : nullptr;
    double* d_Y = by ? d_out + br / 8 : nullptr;
    for (int b = 0; b < count; ++b) {
        if (d_R) rs[b].R = d_R + (size_t)b * r_stride;
        if (d_Y) rs[b].Y = d_Y + (size_t)b * y_stride;
    }
    const int tiles = (int)work.size();
    // tile offsets: in the RHS launch (LDS) for rings of up to kDtScanMax tiles
    bool long_rings = false;
    int local_g = 0;
    for (const DtNet& r : rs) {
        if (r.G > kDtScanMax) long_rings = true;
        else local_g = std::max(local_g, (int)r.G);
    }
    const size_t off_bytes = topo == ND_RING ? (size_t)2 * local_g * 8 : 0;
    const dim3 grid((tiles + 7) / 8 * 8);
    auto offsets = [&](int b) {
        if (topo == ND_RING && long_rings) hipLaunchKernelGGL(k_dt_offsets, dim3(count), dim3(kDtBS), 0, st, d_r, b);
    };
    auto begin = [&](int s) {
        hipLaunchKernelGGL(kern.begin[s], grid, dim3(kDtBS), 0, st, d_r, d_work, tiles);
        offsets(s);
        return hipGetLastError();
    };
    auto stage = [&](int s) {
        hipLaunchKernelGGL(kern.stage[s], grid, dim3(kDtBS), off_bytes, st, d_r, d_desc, d_work, tiles, rtol, atol);
        if (s >= 1 && s <= 5) offsets((s + 1) & 1);
        return hipGetLastError();
    };
    auto emit = [&]() {
        hipLaunchKernelGGL(kern.emit, dim3(tiles), dim3(kDtBS), 0, st, d_r, d_work, t_out);
        return hipGetLastError();
    };
    // outputs a run does not reach read as NaN (all bits set)
    if (dense) e = hipMemsetAsync(d_R, 0xff, br + by, st);
    // the control blocks live inside the scratch: write them with the descriptors
    for (int b = 0; b < count && e == hipSuccess; ++b)
        e = hipMemcpyAsync(rs[b].ctl, &cs[b], sizeof(DtCtl), hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(d_r, rs.data(), bd, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(d_desc, descs.data(), bn, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(d_work, work.data(), bw, hipMemcpyHostToDevice, st);
    if (e == hipSuccess && dense) e = emit();  // output 0
    if (e == hipSuccess) e = begin(0);
    if (e == hipSuccess) e = stage(0);            // k1 = f(y)
    constexpr int kAttempts = 8;        // attempts launched between checks of the done flags
    while (e == hipSuccess) {
        for (int a = 0; a < kAttempts && e == hipSuccess; ++a) {
            e = begin(1);
            for (int s = 1; s <= 6 && e == hipSuccess; ++s) e = stage(s);
            if (e == hipSuccess) {
                hipLaunchKernelGGL(k_dt_control, dim3(count), dim3(kWave), 0, st, d_r, rtol, max_steps,
                                   t_out);
                e = hipGetLastError();
                if (e == hipSuccess && dense) e = emit();
            }
        }
        for (int b = 0; b < count && e == hipSuccess; ++b)
            e = hipMemcpyAsync(&cs[b], rs[b].ctl, sizeof(DtCtl), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) break;
        bool all = true;
        for (const DtCtl& c : cs) all = all && c.done;
        if (all) break;
    }
    if (e == hipSuccess && dense) {
        hipLaunchKernelGGL(k_dt_reduce_R, dim3(count, kDtRBlocks), dim3(kDtBS), 0, st, d_r);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipMemcpyAsync(Rh, d_R, br, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess && by) e = hipMemcpyAsync(Yh, d_Y, by, hipMemcpyDeviceToHost, st);
    }
    // a state that ended in the scratch buffer goes back to the network
    for (int b = 0; b < count && e == hipSuccess; ++b)
        if (cs[b].ypar)
            e = hipMemcpyAsync(rs[b].y[0], rs[b].y[1], (size_t)rs[b].V * rs[b].n * 8, hipMemcpyDeviceToDevice, st);
    const hipError_t ef = hipFreeAsync(buf, st);
    const hipError_t es = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_fail(e, "adaptive run (tiled)");
    if (ef != hipSuccess) return hip_fail(ef, "adaptive scratch free");
    if (es != hipSuccess) return hip_fail(es, "adaptive run (tiled)");
    int bad = -1;
    for (int b = 0; b < count; ++b) {
        stats[b].t = cs[b].t;
        stats[b].accepted = cs[b].acc;
        stats[b].rejected = cs[b].rej;
        stats[b].h_next = cs[b].h;
        stats[b].failed = cs[b].failed;
        stats[b].reserved = 0;
        if (cs[b].failed && bad < 0) bad = b;
    }
    if (bad >= 0)
        return fail(ND_ERR_NUMERIC, "adaptive run: network %d stopped at t = %.17g (non-finite error estimate or "
                                    "step below its floor)", bad, cs[bad].t);
    return ND_OK;
}

static nd_status run_adaptive(const nd_handle* hs, int32_t count, const double* t_end, const double* dt0,
                              double rtol, double atol, int64_t max_steps, nd_adaptive_stats* stats, void* stream,
                              double t_out, double* R, int64_t r_stride, double* Y, int64_t y_stride) {
    if (!hs || !t_end || !dt0 || !stats || count < 0) return fail(ND_ERR_INVALID_ARG, "bad adaptive-run arguments");
    if (!std::isfinite(rtol) || !std::isfinite(atol) || atol < 0.0 || (rtol > 0.0 && atol == 0.0))
        return fail(ND_ERR_INVALID_ARG, "rtol must be finite; atol finite, and > 0 when rtol > 0");
    if (max_steps < 0) return fail(ND_ERR_INVALID_ARG, "max_steps must be >= 0");
    const bool dense = t_out != 0.0;
    if (dense && (!(t_out > 0.0) || !std::isfinite(t_out) || !R || r_stride < 1))
        return fail(ND_ERR_INVALID_ARG, "dense output needs t_out > 0, R and r_stride >= 1");
    if (count == 0) return ND_OK;
    int model = -1, topo = -1;
    bool tiled = false;
    std::vector<NetDesc> descs(count);
    std::vector<Net*> nets(count);
    for (int i = 0; i < count; ++i) {
        Net* n = reinterpret_cast<Net*>(hs[i]);
        if (!n) return fail(ND_ERR_INVALID_ARG, "NULL handle at %d", i);
        nets[i] = n;
        if ((n->prob.topo != ND_RING && n->prob.topo != ND_LINKS) || n->prob.precision != ND_FP64 ||
            n->prob.model == ND_HH)
            return fail(ND_ERR_UNSUPPORTED, "adaptive stepping runs FP64 rings and compressed coupling matrices");
        if (topo >= 0 && n->prob.topo != topo) return fail(ND_ERR_INVALID_ARG, "one adaptive batch holds one topology");
        topo = n->prob.topo;
        tiled = tiled || n->prob.n > kDpCap || topo == ND_LINKS;
        if (model >= 0 && n->prob.model != model)
            return fail(ND_ERR_INVALID_ARG, "one adaptive batch holds one model");
        model = n->prob.model;
        if (!(t_end[i] >= 0.0) || !std::isfinite(t_end[i]) || !(dt0[i] > 0.0) || !std::isfinite(dt0[i]))
            return fail(ND_ERR_INVALID_ARG, "t_end must be finite and >= 0, dt0 finite and > 0 (network %d)", i);
        if (dense) {
            const int64_t outs = (int64_t)std::floor(t_end[i] / t_out) + 1;
            if (outs > r_stride)
                return fail(ND_ERR_INVALID_ARG, "network %d has %lld outputs, r_stride is %lld", i, (long long)outs,
                            (long long)r_stride);
            if (Y && outs * nvars_of(n->prob.model) * n->prob.n > y_stride)
                return fail(ND_ERR_INVALID_ARG, "network %d needs y_stride >= %lld", i,
                            (long long)(outs * nvars_of(n->prob.model) * n->prob.n));
        }
        descs[i] = n->run_desc(dt0[i], 0);
    }
    if (tiled) {
        return run_adaptive_tiled(nets, model, topo, t_end, dt0, rtol, atol, max_steps, stats, (hipStream_t)stream,
                                  dense ? t_out : 0.0, R, r_stride, Y, y_stride);
    }
    hipStream_t st = (hipStream_t)stream;
    void* buf = nullptr;
    const size_t bd = (size_t)count * sizeof(NetDesc), bt = (size_t)count * 8, bs = (size_t)count * kDpStats * 8;
    const size_t br = dense ? (size_t)count * r_stride * 8 : 0, by = dense && Y ? (size_t)count * y_stride * 8 : 0;
    hipError_t e = hipMallocAsync(&buf, bd + bt + bs + br + by, st);
    if (e != hipSuccess) return hip_fail(e, "adaptive scratch");
    NetDesc* d_desc = (NetDesc*)buf;
    double* d_tend = (double*)((char*)buf + bd);
    double* d_stats = (double*)((char*)buf + bd + bt);
    DenseOut o{dense ? t_out : 0.0, dense ? (double*)((char*)buf + bd + bt + bs) : nullptr, r_stride,
               by ? (double*)((char*)buf + bd + bt + bs + br) : nullptr, y_stride};
    std::vector<double> h_stats((size_t)count * kDpStats);
    // outputs a run does not reach (max_steps) read as NaN (all bits set)
    if (dense) e = hipMemsetAsync(o.R, 0xff, br + by, st);
    if (e == hipSuccess && (e = hipMemcpyAsync(d_desc, descs.data(), bd, hipMemcpyHostToDevice, st)) == hipSuccess &&
        (e = hipMemcpyAsync(d_tend, t_end, bt, hipMemcpyHostToDevice, st)) == hipSuccess) {
        auto launch = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(count), dim3(kDpBS), 0, st, d_desc, d_tend, rtol, atol, max_steps, d_stats, o);
        };
        if (model == ND_KURAMOTO)
            dense ? launch(k_ring_dopri<ND_KURAMOTO, true>) : launch(k_ring_dopri_kuramoto);
        else if (model == ND_FHN)
            dense ? launch(k_ring_dopri<ND_FHN, true>) : launch(k_ring_dopri<ND_FHN, false>);
        else
            dense ? launch(k_ring_dopri<ND_KURAMOTO_INERTIA, true>) : launch(k_ring_dopri<ND_KURAMOTO_INERTIA, false>);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipMemcpyAsync(h_stats.data(), d_stats, bs, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess && dense) e = hipMemcpyAsync(R, o.R, br, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess && by) e = hipMemcpyAsync(Y, o.Y, by, hipMemcpyDeviceToHost, st);
    }
    const hipError_t ef = hipFreeAsync(buf, st);
    const hipError_t es = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_fail(e, "adaptive run");
    if (ef != hipSuccess) return hip_fail(ef, "adaptive scratch free");
    if (es != hipSuccess) return hip_fail(es, "adaptive run");
    int bad = -1;
    for (int i = 0; i < count; ++i) {
        const double* q = h_stats.data() + kDpStats * i;
        stats[i].t = q[0];
        stats[i].accepted = (int64_t)q[1];
        stats[i].rejected = (int64_t)q[2];
        stats[i].h_next = q[3];
        stats[i].failed = q[4] != 0.0;
        stats[i].reserved = 0;
        if (stats[i].failed && bad < 0) bad = i;
    }
    if (bad >= 0)
        return fail(ND_ERR_NUMERIC, "adaptive run: network %d stopped at t = %.17g (non-finite error estimate or "
                                    "step below its floor)", bad, stats[bad].t);
    return ND_OK;
}

extern "C" nd_status nd_run_adaptive(const nd_handle* hs, int32_t count, const double* t_end, const double* dt0,
                                     double rtol, double atol, int64_t max_steps, nd_adaptive_stats* stats,
                                     void* stream) {
    return run_adaptive(hs, count, t_end, dt0, rtol, atol, max_steps, stats, stream, 0.0, nullptr, 0, nullptr, 0);
}

extern "C" nd_status nd_run_adaptive_dense(const nd_handle* hs, int32_t count, const double* t_end,
                                           const double* dt0, double rtol, double atol, int64_t max_steps,
                                           double t_out, double* R, int64_t r_stride, double* Y, int64_t y_stride,
                                           nd_adaptive_stats* stats, void* stream) {
    if (!(t_out > 0.0)) return fail(ND_ERR_INVALID_ARG, "t_out must be > 0");
    return run_adaptive(hs, count, t_end, dt0, rtol, atol, max_steps, stats, stream, t_out, R, r_stride, Y, y_stride);
}

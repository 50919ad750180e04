// Projected Tikhonov problem of RTG-GMRES in float64, one workgroup per
// problem (eqs. (12)-(13), with mu fixed or chosen by the discrepancy
// principle).
//
// The Arnoldi steps already reduced H (the (k+1) x k Hessenberg matrix) by
// Givens rotations to H = Q [R; 0] with Q^T beta e1 = [g_R; gamma], so
//   ||beta e1 - H y||^2 + mu ||y||^2 = ||g_R - R y||^2 + gamma^2 + mu ||y||^2.
// With the SVD R = U diag(s) W^T (one-sided Jacobi, in LDS: plane rotations of
// the columns of R^T until they are orthogonal; rotated along with them, the
// entries of g_R become ghat = U^T g_R, and column i ends as s_i w_i) and ghat,
//   phi(mu) = sum_i (mu / (s_i^2 + mu))^2 ghat_i^2 + gamma^2
// is the projected residual; it increases from gamma^2 to beta^2 and the
// discrepancy principle takes the root of phi(mu) = (eta delta)^2, found by
// multisection in log(mu).  Then y = W diag(s / (s^2 + mu)) ghat, the filter
// form of the stacked least-squares problem (13).  With the GCV rule (Sec. 3,
// parameter selection via GCV) mu minimises
//   GCV(mu) = phi(mu) / (1 + sum_i mu / (s_i^2 + mu))^2
// (the trace of I - H (H^T H + mu I)^{-1} H^T over the k + 1 rows): the best
// of 512 points spread over [log s_min^2 - 10, log s_max^2 + 10], then passes
// of 64 points between the neighbours of the best point so far.  The kernel
// writes the coefficients -y_j of the solution update and the result summary.
#include "rtg_internal.h"

namespace rtg {

// A pair of columns counts as orthogonal once |a_p . a_q| <= tol ||a_p|| ||a_q||;
// below about n * eps the inner product is rounding noise and rotations stop
// making progress.  The process ends after a sweep that rotated nothing, or
// after one whose rotations were all so small that the next would find nothing
// to rotate.  A rotation of (p, q) by the angle t adds t ||a_q|| / ||a_p|| times
// cos(q, r) to cos(p, r), and t ||a_q|| / ||a_p|| is at most
//   u = |cos(p, q)| max(||a_p||^2, ||a_q||^2) / | ||a_p||^2 - ||a_q||^2 |,
// which is no smaller than the cosine itself: columns of close norms turn by
// large angles at tiny cosines and put back what was rotated away before.  With
// every u of a sweep below 2e-8, the 2 (k - 2) <= 188 rotations that a pair meets
// after its own leave at most 188 (2e-8)^2 = 7.5e-14 of it.
constexpr double JACOBI_TOL2 = 1e-26;    // (1e-13)^2
constexpr double JACOBI_LAST2 = 4e-16;   // (2e-8)^2

// Sum over a group of 8 lanes, in every lane (VALU cross-lane moves, no LDS
// round trip): neighbours, then pairs within a quad, then the mirrored quad.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double sum8(double v) {
    v += dpp_f64<0xB1>(v);     // quad_perm [1, 0, 3, 2]
    v += dpp_f64<0x4E>(v);     // quad_perm [2, 3, 0, 1]
    v += dpp_f64<0x141>(v);    // row_half_mirror
    return v;
}

// 1 / sqrt(x) for x in [1/4, 2]: the hardware's estimate and two Newton steps
__device__ __forceinline__ double rsqrt_f64(double x) {
    double y = __builtin_amdgcn_rsq(x);
    y = fma(y * 0.5, fma(-x * y, y, 1.0), y);
    return fma(y * 0.5, fma(-x * y, y, 1.0), y);
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    return v;
}

// phi(mu) evaluated by one wave (k <= 128 terms, two per lane)
__device__ __forceinline__ double proj_res2(const double* sig, const double* gh, int k, double mu,
                                            double gp2, int lane) {
    double s = 0.0;
    for (int i = lane; i < k; i += 64) {
        const double f = mu / (sig[i] * sig[i] + mu);
        s += f * f * gh[i] * gh[i];
    }
    return wave_sum(s) + gp2;
}

// A chain of (sweeps) x (k - 1) rounds, each a barrier: the length of a round
// is what the kernel takes.  The rotations work on R^T with g_R as one more
// row, so no matrix W is accumulated (half the LDS traffic of a round); the
// dot products are reduced by cross-lane moves instead of through LDS; cosine
// and sine come from two reciprocal square roots by the half-angle formulas,
// without a division.  Eight lanes per pair: a problem of k = 50 then has one wave
// per SIMD.  With sixteen it had two, and a round was bound by their float64
// issue (1,750 clocks against 1,520, both with the angle in single precision,
// which saves 3 % of the kernel).  NR: rows per lane, k <= 8 NR (a runtime row
// count cost a scalar branch per row).  One problem, k = 50: 920 -> 347 us;
// k = 20: 178 -> 87 us.
template <int NR>
__global__ void __launch_bounds__(384) k_solve(const Desc* __restrict__ descs) {
    // A lane holds the row pairs 2 gl, 2 gl + 1 (mod 16): 16-byte LDS accesses.
    // Column stride in doubles: 16 mod 32, so that two neighbouring groups,
    // which read neighbouring columns, meet different banks.
    constexpr int LD = (NR <= 2) ? 16 : (NR <= 6 ? 48 : (NR <= 10 ? 80 : 112));
    static_assert(LD >= 8 * NR && NR % 2 == 0 && NR <= 14, "column stride");
    typedef double d2 __attribute__((ext_vector_type(2)));
    __shared__ __attribute__((aligned(16))) double As[8 * NR * LD];
    __shared__ double sig[MMAX], gh[MMAX], fco[MMAX];
    __shared__ int s_big[3];                      // per sweep: a rotation's u was above JACOBI_LAST
    __shared__ int s_cnt[2][8];                  // per wave: its points below the target (two passes in turn)
    __shared__ double s_mu;
    __shared__ int s_flags;

    const Desc& d = descs[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nwave = blockDim.x >> 6;
    const int k = uniform_int(d.state[ST_MEFF]);
    const int m = d.m;
    const double beta = d.scal[SC_BETA];
    const double* gvec = d.gv + 2 * m;

    if (d.state[ST_SKIP]) return;         // a restart cycle this problem sits out
    const int done = d.state[ST_ITERS];   // steps of earlier restart cycles
    if (k == 0) {
        if (tid == 0) {
            d.coef[MMAX + 1] = 1.f;
            rtg_info inf;
            inf.iters = done;
            inf.flags = d.state[ST_FLAGS];
            inf.mu = 0.0;
            inf.beta = beta;
            inf.res_proj = beta;
            inf.res_ls = beta;
            *d.info = inf;
        }
        return;
    }
    // ---- load R^T: column c of As is row c of R (upper triangular, stored
    // column-major with leading dimension m), rows padded with zeros to 8 NR
    for (int r = wave; r < 8 * NR; r += nwave)
        for (int c = lane; c < k; c += 64)
            As[c * LD + r] = (r < k && c <= r) ? *gptr(d.R + (size_t)r * m + c) : 0.0;
    if (tid < k) gh[tid] = gvec[tid];
    if (tid < 3) s_big[tid] = 0;
    const double gam = fabs(gvec[k]);
    __syncthreads();

    // ---- one-sided Jacobi, round-robin (circle) ordering of column pairs.
    // Eight lanes handle one pair, and there is a group for every pair of a round.
    const int nb = k + (k & 1);
    const int grp = tid >> 3, gl = tid & 7;
    // this group's pair of round 0 (position 0 stays, the others step round the circle)
    int qa = grp - 1, qb = nb - 2 - grp;
    for (int sweep = 0; sweep < 60; ++sweep) {
        const int slot = sweep % 3;
        bool big = false;
        int oa = qa, ob = qb;                     // (position - 1 + round) mod (nb - 1)
        for (int rd = 0; rd < nb - 1; ++rd) {
            const int pa = grp == 0 ? 0 : 1 + oa, pb = 1 + ob;
            oa = (oa + 1 >= nb - 1) ? 0 : oa + 1;
            ob = (ob + 1 >= nb - 1) ? 0 : ob + 1;
            if (grp < nb / 2 && pa < k && pb < k) {   // uniform within the group
                d2* ca = (d2*)(As + pa * LD + 2 * gl);
                d2* cb = (d2*)(As + pb * LD + 2 * gl);
                double x[NR], y[NR];
#pragma unroll
                for (int q = 0; q < NR; q += 2) {
                    const d2 u = ca[4 * q], v = cb[4 * q];
                    x[q] = u[0]; x[q + 1] = u[1];
                    y[q] = v[0]; y[q + 1] = v[1];
                }
                const double ga0 = gh[pa], gb0 = gh[pb];
                double al = x[0] * x[0], be = y[0] * y[0], ga = x[0] * y[0];
#pragma unroll
                for (int q = 1; q < NR; ++q) {
                    al = fma(x[q], x[q], al);
                    be = fma(y[q], y[q], be);
                    ga = fma(x[q], y[q], ga);
                }
                al = sum8(al);
                be = sum8(be);
                ga = sum8(ga);
                const double g2 = ga * ga, ab = al * be;
                if (g2 > JACOBI_TOL2 * ab) {
                    // angle t: cos 2t = |df| / hyp, sin 2t = 2 ga / hyp, hyp = sqrt(df^2 + (2 ga)^2)
                    const double df = be - al, g2x = 2.0 * ga;
                    // (both scaled to about 1 first, so that their squares do
                    // not overflow or vanish together)
                    const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(df), fabs(g2x)));
                    const double dfs = __builtin_ldexp(df, ex), gs = __builtin_ldexp(g2x, ex);
                    const double mx = __builtin_ldexp(fmax(al, be), ex);
                    big = big || g2 * (mx * mx) > JACOBI_LAST2 * ab * (dfs * dfs);
                    const double ih = rsqrt_f64(fma(dfs, dfs, gs * gs));      // 1 / hyp
                    const double c2 = fma(0.5 * fabs(dfs), ih, 0.5);          // cos^2 t, in [1/2, 1]
                    const double ic = rsqrt_f64(c2);
                    const double cth = c2 * ic;
                    const double sth = (df < 0.0 ? -0.5 : 0.5) * gs * ih * ic;
#pragma unroll
                    for (int q = 0; q < NR; q += 2) {
                        ca[4 * q] = d2{fma(cth, x[q], -sth * y[q]), fma(cth, x[q + 1], -sth * y[q + 1])};
                        cb[4 * q] = d2{fma(sth, x[q], cth * y[q]), fma(sth, x[q + 1], cth * y[q + 1])};
                    }
                    if (gl == 0) {
                        gh[pa] = fma(cth, ga0, -sth * gb0);
                        gh[pb] = fma(sth, ga0, cth * gb0);
                    }
                }
            }
            if (rd == nb - 2) {
                if (big && gl == 0) s_big[slot] = 1;
                if (tid == 0) s_big[(sweep + 1) % 3] = 0;   // last read two sweeps ago
            }
            __syncthreads();
        }
        if (!s_big[slot]) break;
    }
    // ---- singular values: the norms of the columns (ghat is in gh)
    for (int i = grp; i < k; i += blockDim.x >> 3) {
        double nn = 0.0;
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            const double x = As[i * LD + gl + 8 * q];
            nn = fma(x, x, nn);
        }
        nn = sum8(nn);
        if (gl == 0) sig[i] = sqrt(nn);
    }
    __syncthreads();
    // ---- mu: fixed, by GCV (wave 0), or by the discrepancy principle (every wave)
    const double gp2 = gam * gam;
    if (d.mu_fixed || d.mu_rule == RTG_MU_GCV) {
      if (wave == 0) {
        double mu = d.mu;
        if (!d.mu_fixed) {
            // GCV at log(mu) = x, and the (value, position) minimum over the wave
            auto gcv_at = [&](double x) {
                const double mu_l = exp(x);
                double ph = gp2, tr = 1.0;
                for (int i = 0; i < k; ++i) {
                    const double s2 = sig[i] * sig[i];
                    const double f = mu_l / (s2 + mu_l);
                    ph += f * f * gh[i] * gh[i];
                    tr += s2 > 0.0 ? f : 1.0;
                }
                return ph / (tr * tr);
            };
            auto wave_argmin = [&](double v, int idx, double& vmin, int& imin) {
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) {
                    const double ov = __shfl_xor(v, off, 64);
                    const int oi = __shfl_xor(idx, off, 64);
                    if (ov < v || (ov == v && oi < idx)) { v = ov; idx = oi; }
                }
                vmin = v;
                imin = idx;
            };
            double smax = 0.0, smin = INFINITY;
            for (int i = lane; i < k; i += 64) {
                smax = fmax(smax, sig[i]);
                if (sig[i] > 0.0) smin = fmin(smin, sig[i]);
            }
            smax = wave_max(smax);
            smin = -wave_max(-smin);
            const double smax2 = smax > 0.0 ? smax * smax : 1.0;
            const double smin2 = isfinite(smin) ? fmax(smin * smin, 1e-30 * smax2) : smax2;
            const double glo = log(smin2) - 10.0, ghi = log(smax2) + 10.0;
            // 512 grid points, eight per lane (the same grid as the oracle's)
            double bv = INFINITY;
            int bi = 0;
            for (int q = 0; q < 8; ++q) {
                const int pidx = 8 * lane + q;
                const double v = gcv_at(glo + (ghi - glo) * (double)pidx / 511.0);
                if (v < bv) { bv = v; bi = pidx; }
            }
            double vmin;
            int imin;
            wave_argmin(bv, bi, vmin, imin);
            double lo = glo + (ghi - glo) * (double)max(imin - 1, 0) / 511.0;
            double hi = glo + (ghi - glo) * (double)min(imin + 1, 511) / 511.0;
            double xbest = glo + (ghi - glo) * (double)imin / 511.0;
            for (int it = 0; it < 16; ++it) {
                const double x = lo + (hi - lo) * (double)(lane + 1) / 65.0;
                double v = gcv_at(x);
                if (!(v < vmin)) v = INFINITY;            // keep the best point so far when nothing beats it
                int li;
                double lv;
                wave_argmin(v, lane, lv, li);
                if (!(lv < INFINITY)) {                  // the best point is inside a bracket no lane improves:
                    const double w = (hi - lo) / 65.0;   // shrink around it
                    lo = fmax(lo, xbest - w);
                    hi = fmin(hi, xbest + w);
                } else {
                    vmin = lv;
                    xbest = lo + (hi - lo) * (double)(li + 1) / 65.0;
                    const double w = (hi - lo) / 65.0;
                    lo = xbest - w;
                    hi = xbest + w;
                }
                if (!(hi - lo > 1e-12)) break;
            }
            mu = exp(xbest);
        }
        if (lane == 0) {
            s_mu = mu;
            s_flags = 0;
        }
      }
    } else {
        const double t = d.eta * d.delta;
        const double t2 = t * t;
        double mu;
        int flags = 0;
        if (t2 <= gp2) {
            mu = 0.0;
            flags = RTG_F_DISCREP_UNREACHABLE;
        } else if (t2 >= beta * beta) {
            mu = INFINITY;
            flags = RTG_F_MU_INF;
        } else {
            double smax = 0.0;
            for (int i = lane; i < k; i += 64) smax = fmax(smax, sig[i]);
            smax = wave_max(smax);
            const double smax2 = smax > 0.0 ? smax * smax : 1.0;
            double lo = log(smax2) - 80.0, hi = log(smax2) + 80.0;
            for (int it = 0; it < 40 && proj_res2(sig, gh, k, exp(lo), gp2, lane) > t2; ++it) lo -= 40.0;
            for (int it = 0; it < 40 && proj_res2(sig, gh, k, exp(hi), gp2, lane) < t2; ++it) hi += 40.0;
            // Multisection: every 8-lane group evaluates phi at its interior
            // point of the bracket; phi increases with mu, so the points below
            // the target form a prefix, and with P groups the bracket shrinks
            // P + 1-fold per pass, until it stops shrinking.  In log(mu) while
            // the bracket is wider than a tenth, then in mu itself (a float64
            // exponential is half of a pass).  All waves hold the same
            // bracket: the next one follows from the number of points below.
            const int P = blockDim.x >> 3;
            const double iP = 1.0 / (double)(P + 1), frac = (double)(grp + 1) * iP;
            double sq[NR], gq[NR];
#pragma unroll
            for (int q = 0; q < NR; ++q) {
                const int i = gl + 8 * q;
                sq[q] = i < k ? sig[i] * sig[i] : 1.0;
                gq[q] = i < k ? gh[i] : 0.0;
            }
            bool in_log = true;
            for (int it = 0; it < 40; ++it) {
                if (in_log && hi - lo < 0.1) {
                    in_log = false;
                    lo = exp(lo);
                    hi = exp(hi);
                }
                const double x = lo + (hi - lo) * frac;
                const double mu_l = in_log ? exp(x) : x;
                double ph = 0.0;
#pragma unroll
                for (int q = 0; q < NR; ++q) {
                    const double f = mu_l / (sq[q] + mu_l) * gq[q];
                    ph = fma(f, f, ph);
                }
                ph = sum8(ph) + gp2;
                const unsigned long long below = __ballot(ph < t2);
                if (lane == 0) s_cnt[it & 1][wave] = ((below == ~0ull) ? 64 : __builtin_ctzll(~below)) >> 3;
                __syncthreads();
                int pfx = 0;
                for (int w = 0; w < nwave; ++w) {
                    const int c = s_cnt[it & 1][w];
                    pfx += c;
                    if (c < 8) break;
                }
                const double nlo = pfx > 0 ? lo + (hi - lo) * ((double)pfx * iP) : lo;
                const double nhi = pfx < P ? lo + (hi - lo) * ((double)(pfx + 1) * iP) : hi;
                if (!(nhi - nlo < hi - lo)) break;
                lo = nlo;
                hi = nhi;
            }
            mu = in_log ? exp(0.5 * (lo + hi)) : 0.5 * (lo + hi);
        }
        if (tid == 0) {
            s_mu = mu;
            s_flags = flags;
        }
    }
    __syncthreads();
    const double mu = s_mu;
    if (tid < k) {
        const double s = sig[tid];
        // y = sum_i (s_i / (s_i^2 + mu)) ghat_i w_i, and column i holds s_i w_i
        fco[tid] = isinf(mu) ? 0.0 : (s > 0.0 ? s / (s * s + mu) * gh[tid] / s : 0.0);
    }
    __syncthreads();
    // ---- y; coefficients of X = X0 + sum_j y_j V_j
    bool ok = true;
    if (tid < k) {
        double yv = 0.0;
#pragma unroll 8
        for (int i = 0; i < k; ++i) yv += As[i * LD + tid] * fco[i];
        d.y[tid] = yv;
        // (a V_1 stored unnormalised carries its 1 / beta in its coefficient)
        d.coef[tid] = (float)(-yv * ((d.lazy_v1 && tid == 0) ? 1.0 / beta : 1.0));
        ok = isfinite(yv);
    }
    const int allok = __syncthreads_and(ok ? 1 : 0);
    if (wave == 0) {
        const double rp2 = isinf(mu) ? beta * beta : proj_res2(sig, gh, k, mu, gp2, lane);
        if (lane == 0) {
            int flags = d.state[ST_FLAGS] | s_flags;
            if (!allok) flags |= RTG_F_NONFINITE;
            d.state[ST_FLAGS] = flags;
            d.coef[MMAX + 1] = 1.f;
            d.scal[SC_MU] = mu;
            d.scal[SC_RESPROJ] = sqrt(rp2);
            d.state[ST_ITERS] = done + k;
            rtg_info inf;
            inf.iters = done + k;
            inf.flags = flags;
            inf.mu = mu;
            inf.beta = beta;
            inf.res_proj = sqrt(rp2);
            inf.res_ls = gam;
            *d.info = inf;
        }
    }
}

// cycle 0: a fresh solve.  cycle c > 0 (restarted RTG-GMRES): a new cycle
// from X0 = X; a problem out of restarts, or one that sat out an earlier
// cycle (its residual was below eps), sits this one out too; the others
// keep their step count and flags (but for NOT_CONVERGED, which the cycle
// decides anew).
__global__ void k_init(const Desc* __restrict__ descs, int cycle, int* sched) {
    const Desc& d = descs[blockIdx.x];
    const int tid = threadIdx.x;
    if (sched && blockIdx.x == 0)
        for (int w = tid; w < SCH_WORDS; w += blockDim.x) sched[w] = 0;
    if (cycle > 0) {
        const bool sit_out = cycle > d.restarts || d.state[ST_SKIP] != 0;
        __syncthreads();                      // every thread has read the state
        if (sit_out) {
            if (tid == 0) {
                d.state[ST_SKIP] = 1;
                d.state[ST_ACTIVE] = 0;
            }
            if (tid < NKIND) d.state[ST_DONE + tid] = 0;
            return;
        }
        if (tid < NSTATE) {
            const int v = d.state[tid];
            int nv = 0;
            if (tid == ST_ACTIVE) nv = 1;
            else if (tid == ST_ITERS) nv = v;
            else if (tid == ST_FLAGS) nv = v & ~RTG_F_NOT_CONVERGED;
            d.state[tid] = nv;
        }
    } else if (tid < NSTATE) {
        d.state[tid] = (tid == ST_ACTIVE) ? 1 : ((tid == ST_FLAGS && d.fallback) ? RTG_F_FALLBACK : 0);
    }
    if (tid < NSCAL) d.scal[tid] = 0.0;
    if (tid == 0) d.coef[MMAX + 1] = 1.f;   // the scale of a V_1 formed before the start step
    const int m = d.m;
    for (int e = tid; e < (m + 1) * m; e += blockDim.x) d.H[e] = 0.0;
    for (int e = tid; e < 3 * m + 1; e += blockDim.x) d.gv[e] = 0.0;
}

// Composed sketch matrices: S(Phi(X)) = X x_1 (Om1 A1) x_2 (Om2 A2) x_3 (Om3 B^T)
// (mode products compose; Phi of eq. (2)).  Om1 is the matrix the basis
// sketches use: the bfloat16-rounded one for a bfloat16 basis.  A1 has band
// rows, A1[i', i] = a1[i' (2 r1 + 1) + r1 + i - i'] (read here from the
// transposed copy, so that neighbouring entries read neighbouring words);
// B[k, j] = bb[k (2 rB + 1) + rB + j - k]
// is the weight of input channel k in output channel j.
__global__ void k_compose(const Desc* __restrict__ descs, int nbc) {
    const int p = blockIdx.x / nbc, part = blockIdx.x % nbc;
    const Desc& d = descs[p];
    if (d.st != nullptr) return;          // a general PSF: no banded factors to compose
    const int I1 = d.I1, I2 = d.I2, J = d.J, l1 = d.l1, l2 = d.l2, l3 = d.l3;
    const int r1 = d.r1, r2 = d.r2, rB = d.rB;
    const int wB = 2 * rB + 1;
    // mode 1 over the operand-padded index space: padding entries are
    // written as zeros (the MFMA contractions read whole tiles)
    const int I1p = frag_nkb(I1, FRAG_K_BF16) * FRAG_K_BF16;
    const int E1 = (int)compose_mode1_entries(l1, I1), E2 = l2 * I2, E3 = l3 * J;
    const int nkf = frag_nkb(I1, FRAG_K_F32), nkh = frag_nkb(I1, FRAG_K_BF16);
    const size_t lo_plane = frag_elems(l1, I1, FRAG_K_BF16);
    // one entry per thread; taps read from clamped indices and masked, so
    // that the loads of a thread are independent of each other
    const int e = part * blockDim.x + threadIdx.x;
    if (e < E1) {
        const int a = e / I1p, i = e % I1p;
        const bool real = a < l1 && i < I1;
        const int ac = min(a, l1 - 1);
        float acc = 0.f;
#pragma unroll 5
        for (int dd = -r1; dd <= r1; ++dd) {
            const int ip = i - dd;
            const int ipc = min(max(ip, 0), I1 - 1);
            const float om = d.skbf ? bf2f(*gptr(d.om1h + (size_t)ac * I1 + ipc)) : *gptr(d.om1 + (size_t)ac * I1 + ipc);
            const float w = *gptr(d.a1t + (size_t)(r1 + dd) * I1 + ipc);
            acc = fmaf((ip >= 0 && ip < I1) ? om : 0.f, w, acc);
        }
        acc = real ? acc : 0.f;
        if (i < nkf * FRAG_K_F32) *gptr_w((float*)d.om1t + frag_index(a, i, nkf, FRAG_K_F32)) = acc;
        const bf16_t hi = f2bf(acc);
        const size_t fh = frag_index(a, i, nkh, FRAG_K_BF16);
        *gptr_w((bf16_t*)d.om1th + fh) = hi;
        *gptr_w((bf16_t*)d.om1th + lo_plane + fh) = f2bf(acc - bf2f(hi));
    } else if (e < E1 + E2) {
        const int e2 = e - E1;
        const int b = e2 / I2, i = e2 % I2;
        float acc = 0.f;
#pragma unroll 5
        for (int dd = -r2; dd <= r2; ++dd) {
            const int ip = i - dd;
            const int ipc = min(max(ip, 0), I2 - 1);
            const float om = *gptr(d.om2 + (size_t)b * I2 + ipc);
            const float w = *gptr(d.a2t + (size_t)(r2 + dd) * I2 + ipc);
            acc = fmaf((ip >= 0 && ip < I2) ? om : 0.f, w, acc);
        }
        *gptr_w((float*)d.om2t + e2) = acc;
    } else if (e < E1 + E2 + E3) {
        const int e3 = e - E1 - E2;
        const int c3 = e3 / J, k = e3 % J;
        float acc = 0.f;
        for (int j = max(0, k - rB); j <= min(J - 1, k + rB); ++j) {
            const float o3 = d.has_om3 ? *gptr(d.om3 + (size_t)c3 * J + j) : (c3 == j ? 1.f : 0.f);
            acc = fmaf(o3, *gptr(d.bb + (size_t)k * wB + rB + (j - k)), acc);
        }
        *gptr_w((float*)d.om3t + e3) = acc;
    }
}

__global__ void k_finish_arnoldi(const Desc* __restrict__ descs, double* H, double* beta,
                                 int* m_done, int m) {
    const Desc& d = descs[0];
    for (int e = threadIdx.x; e < (m + 1) * m; e += blockDim.x) H[e] = d.H[e];
    if (threadIdx.x == 0) {
        *beta = d.scal[SC_BETA];
        *m_done = d.state[ST_MEFF];
    }
}

hipError_t launch_solve(const Desc* d, int count, int mmax, hipStream_t s) {
    // eight lanes per Jacobi column pair, and a group for each point of the
    // multisection: a wave per SIMD at least (mmax <= 96: at most 384 threads)
    int threads = 8 * ((mmax + 1) / 2);
    threads = threads < 256 ? 256 : (threads + 63) / 64 * 64;
#define RTG_SOLVE(NRV) hipLaunchKernelGGL(k_solve<NRV>, dim3(count), dim3(threads), 0, s, d)
    if (mmax <= 16) RTG_SOLVE(2);
    else if (mmax <= 32) RTG_SOLVE(4);
    else if (mmax <= 64) RTG_SOLVE(8);
    else if (mmax <= 80) RTG_SOLVE(10);
    else RTG_SOLVE(12);
#undef RTG_SOLVE
    return hipGetLastError();
}

hipError_t launch_init(const Desc* d, int count, hipStream_t s, int cycle, int* sched) {
    hipLaunchKernelGGL(k_init, dim3(count), dim3(256), 0, s, d, cycle, sched);
    return hipGetLastError();
}

hipError_t launch_compose(const Desc* d, int count, int max_entries, hipStream_t s) {
    const int nbc = (max_entries + 255) / 256;
    hipLaunchKernelGGL(k_compose, dim3(count * nbc), dim3(256), 0, s, d, nbc);
    return hipGetLastError();
}

hipError_t launch_finish_arnoldi(const Desc* d, double* H, double* beta, int* m_done, int m,
                                 hipStream_t s) {
    hipLaunchKernelGGL(k_finish_arnoldi, dim3(1), dim3(256), 0, s, d, H, beta, m_done, m);
    return hipGetLastError();
}

}  // namespace rtg

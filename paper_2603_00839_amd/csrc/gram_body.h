#pragma once
// Sketched inner products and the Hessenberg update of one Arnoldi step.
//
// Each workgroup owns a chunk of (a, b) index pairs of the sketch.  It
//  1. finishes the sketch for its chunk: sums the per-tile partials written
//     by k_tile over the i2 tiles, and applies mode 3,
//        s[a,b,c'] = sum_c Om3[c',c] sum_tiles P_(tile,c)[a,b]
//     (Om3 = identity when absent) -- for s = S(Phi(V_j)) and, in a step,
//     for S(V_j), the sketch of the newest stored basis tensor.  In a step
//     the partials of s were taken from V_j with Om1 A1 and Om2 A2, and
//     mode 3 uses Om3 B^T (mode products compose);
//  2. computes its share of the inner products <S(V_i), s> and
//     <S(V_i), S(V_j)> (i <= j) and of ||s||^2 in float64;
//  3. the last workgroup of a problem to finish sums the shares in a fixed
//     order and performs the small, float64 part of the step (Sec. 4.3):
//        h1 = S(V)^T s,  h = h1 + (h1 - G h1)        (classical Gram-Schmidt
//                                                     with one reorthogonal-
//                                                     isation, G = S(V)^T S(V))
//        h_{j+1,j} = ||s - S(V) h|| = sqrt(||s||^2 - 2 h^T h1 + h^T G h)
//     then the breakdown test, the Givens update of the least-squares
//     problem (11S) and the stopping decision.  It writes the coefficients
//     for the next multi-AXPY (k_tile).
// In the start mode it returns beta = ||S(R0)||.
//
// Golub-Kahan mode (Sec. 4.5): the newest tensor X_c of one side (V_c, or
// U_c on the side of Phi^T) was sketched with Omega and with the composed
// matrices of its side's operator, so s = S(Op(X_c)) is finished here as in
// a step, and the next coefficient of the bidiagonal matrix is
//   ||s - cf S(Y)||,  Y the other side's newest tensor, cf its coefficient
// (alpha_c = ||S(Phi^T(U_c)) - beta_c S(V_{c-1})|| on the U side,
//  beta_{c+1} = ||S(Phi(V_c)) - alpha_c S(U_c)|| on the V side),
// summed element by element in float64.  The V side completes column c of
// the bidiagonal matrix and takes the same Givens update and stopping
// decisions as a GMRES step.

#include "rtg_internal.h"

namespace rtg {

// largest step whose stored block of G the finishing workgroup stages in LDS
constexpr int GLDS = 64;

__device__ __forceinline__ double load_coherent(const double* p) {
    return __hip_atomic_load(gptr(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Cross-lane moves of a double (no LDS): lanes without a source, and rows
// outside ROWS, take `old`.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ double dpp_or(double v, double old) {
    const long long b = __builtin_bit_cast(long long, v), o = __builtin_bit_cast(long long, old);
    const int lo = __builtin_amdgcn_update_dpp((int)o, (int)b, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(b >> 32), CTRL, ROWS, 0xf, false);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
constexpr int DPP_SHR = 0x110, DPP_BC15 = 0x142, DPP_BC31 = 0x143;   // row_shr:n, row_bcast:15, row_bcast:31

// Sum over the wave, valid in lane 63: within rows of 16 lanes, then row to row.
__device__ __forceinline__ double wave_sum63(double v) {
    v += dpp_or<DPP_SHR + 1>(v, 0.0);
    v += dpp_or<DPP_SHR + 2>(v, 0.0);
    v += dpp_or<DPP_SHR + 4>(v, 0.0);
    v += dpp_or<DPP_SHR + 8>(v, 0.0);
    v += dpp_or<DPP_BC15, 0xa>(v, 0.0);
    v += dpp_or<DPP_BC31, 0xc>(v, 0.0);
    return v;
}
__device__ __forceinline__ double lane63(double v) {
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)b, 63), hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// The linear recurrence r_{i+1} = A_i r_i + B_i over the lanes (lane i holds
// A_i, B_i): composed prefixes, r_{i+1} = A r_0 + B afterwards.
__device__ __forceinline__ void wave_compose(double& A, double& B) {
#define RTG_COMPOSE(CTRL, ROWS)                                                     \
    {                                                                               \
        const double pa = dpp_or<CTRL, ROWS>(A, 1.0), pb = dpp_or<CTRL, ROWS>(B, 0.0); \
        B = fma(A, pb, B);                                                          \
        A = A * pa;                                                                 \
    }
    RTG_COMPOSE(DPP_SHR + 1, 0xf)
    RTG_COMPOSE(DPP_SHR + 2, 0xf)
    RTG_COMPOSE(DPP_SHR + 4, 0xf)
    RTG_COMPOSE(DPP_SHR + 8, 0xf)
    RTG_COMPOSE(DPP_BC15, 0xa)
    RTG_COMPOSE(DPP_BC31, 0xc)
#undef RTG_COMPOSE
}

// Finished sketch for the pairs [q0, q0 + qn):
//   out[(q - q0) l3 + c'] = sum_c M[c', c] sum_{i2 tiles t of channel c} P[(c, t)][q]
// with M = m3 (l3 x J) or the identity (m3 == nullptr); band >= 0 says that
// M[c', c] = 0 for |c' - c| > band.  NB buffers are finished together.
//
// First the sums over the tiles: a thread takes VW (4, 2 or 1, as the sizes
// allow aligned loads) neighbouring pairs of one channel and buffer, 16 loads
// in flight, and leaves its sums in LDS (Q: FINQ floats; where a workgroup's
// channels do not fit, they are taken in chunks).  Then mode 3 from LDS, four
// finished values of a pair per thread, so that a sum is read once for four
// products.  Every sum runs in a fixed order: tiles ascending, channels
// ascending; with `split` (many channels per pair) the channels in GRAM_SPL
// slices that are added in order.
// (One thread per pair with all of a pair's loads and a 16-wide mode 3 of
// mostly zero weights: 8 us of a 512x512x3 problem's step, 28 us of a
// 64-channel one's.)
constexpr int FINQ = 2 * GLDS * GLDS;   // the G block's LDS, free until the tail

// Sums over the nt2 tiles of rows [0, nrow) (buffer and channel) for the
// pairs [0, qn): Q[row * CH + t].
template <int VW, int U, typename Src>
__device__ __forceinline__ void finish_tiles(int nrow, int qn, int nt2, int L12, int CH, float* Q, Src src) {
    typedef float fv __attribute__((ext_vector_type(VW)));
    constexpr int NI = 16 / U;            // items per thread and turn
    const int tid = block_tid();
    const int nq = qn / VW, n = nrow * nq;
    for (int it0 = tid; it0 < n; it0 += 256 * NI) {
        const float* P[NI];
        fv acc[NI];
#pragma unroll
        for (int k = 0; k < NI; ++k) {
            const int it = min(it0 + 256 * k, n - 1), row = it / nq;
            P[k] = src(row) + VW * (it - row * nq);
#pragma unroll
            for (int i = 0; i < VW; ++i) acc[k][i] = 0.f;
        }
        for (int t0 = 0; t0 < nt2; t0 += U) {
            fv v[NI][U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u < 4 || t0 + (u & ~3) < nt2)
#pragma unroll
                    for (int k = 0; k < NI; ++k) v[k][u] = *gptr((const fv*)(P[k] + (size_t)min(t0 + u, nt2 - 1) * L12));
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (t0 + u < nt2)
#pragma unroll
                    for (int k = 0; k < NI; ++k) acc[k] += v[k][u];
        }
#pragma unroll
        for (int k = 0; k < NI; ++k) {
            const int it = it0 + 256 * k, row = it / nq;
            if (it < n) *(fv*)(Q + row * CH + VW * (it - row * nq)) = acc[k];
        }
    }
}

template <int NB>
__device__ __forceinline__ void finish_sketches(const Desc& d, int q0, int qn, bool split,
                                                const float* __restrict__ P0, const float* __restrict__ m30,
                                                int band0, float* out0, const float* __restrict__ P1,
                                                const float* __restrict__ m31, int band1, float* out1, float* Q) {
    typedef float f4v __attribute__((ext_vector_type(4)));
    const int tid = block_tid();
    const int L12 = d.l1 * d.l2;
    const int J = d.J, nt2 = d.n_i2t * d.nrs, l3 = d.l3;   // (partials of a channel)
    const int l3g = (l3 + 3) >> 2;                       // groups of four finished values
    const int al = L12 | q0 | qn;
    const int CH = (qn + 3) & ~3;                        // row length of Q
    const int cps = (J + GRAM_SPL - 1) / GRAM_SPL;       // channels per slice
    int cmax = FINQ / (NB * CH);                         // channels per chunk
    if (split && cmax >= cps) cmax -= cmax % cps;
    // the mode-3 factors next to the sums, where they fit: W3[c][c'], rows of 4 l3g
    const bool wlds = cmax >= J && NB * J * (CH + 4 * l3g) <= FINQ;
    float* W3 = Q + NB * CH * J;
    if (wlds)
        for (int e = tid; e < NB * 4 * l3g * J; e += 256) {
            const bool second = NB > 1 && e >= 4 * l3g * J;
            const float* m3 = second ? m31 : m30;
            const int e1 = second ? e - 4 * l3g * J : e, c = e1 / (4 * l3g), c3 = e1 - c * 4 * l3g;
            if (m3) W3[e] = c3 < l3 ? *gptr(m3 + (size_t)c3 * J + c) : 0.f;
        }
    for (int clo = 0; clo < J; clo += cmax) {
        const int nc = min(cmax, J - clo);
        if (clo > 0) __syncthreads();                    // the previous chunk has been used
        auto src = [&](int row) {
            const bool second = NB > 1 && row >= nc;
            return (second ? P1 : P0) + (size_t)(clo + (second ? row - nc : row)) * nt2 * L12 + q0;
        };
        if ((al & 3) == 0) {
            if (nt2 > 8) finish_tiles<4, 16>(NB * nc, qn, nt2, L12, CH, Q, src);
            else finish_tiles<4, 8>(NB * nc, qn, nt2, L12, CH, Q, src);
        } else if ((al & 1) == 0) {
            finish_tiles<2, 16>(NB * nc, qn, nt2, L12, CH, Q, src);
        } else {
            finish_tiles<1, 16>(NB * nc, qn, nt2, L12, CH, Q, src);
        }
        __syncthreads();
        // mode 3: values 4 g .. 4 g + 3 of pair t and buffer b, neighbouring
        // threads on neighbouring pairs
        for (int o = tid; o < NB * l3g * qn; o += 256) {
            const int r = o / qn, t = o - r * qn;
            const bool second = NB > 1 && r >= l3g;
            const int g4 = 4 * (second ? r - l3g : r);
            const float* m3 = second ? m31 : m30;
            const int band = second ? band1 : band0;
            const float* q = Q + (second ? nc * CH : 0) + t;
            float* out = (second ? out1 : out0) + t * l3 + g4;
            float a[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = (clo > 0 && g4 + i < l3) ? out[i] : 0.f;
            if (m3 == nullptr) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (g4 + i < l3 && g4 + i >= clo && g4 + i < clo + nc) a[i] = q[(g4 + i - clo) * CH];
            } else {
                // the sum over channels, the four weights of channel c from `w`
                auto sum = [&](auto w) {
                    if (split) {
                        for (int s0 = 0; s0 < nc; s0 += cps) {
                            f4v part = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
                            for (int c = s0; c < min(nc, s0 + cps); ++c) {
                                const f4v wc = w(c);
                                const float qc = q[c * CH];
#pragma unroll
                                for (int i = 0; i < 4; ++i) part[i] = fmaf(wc[i], qc, part[i]);
                            }
#pragma unroll
                            for (int i = 0; i < 4; ++i) a[i] += part[i];
                        }
                    } else {
                        const int c0 = band >= 0 ? max(0, g4 - band - clo) : 0;
                        const int c1 = band >= 0 ? min(nc, g4 + 3 + band + 1 - clo) : nc;
#pragma unroll 4
                        for (int c = c0; c < c1; ++c) {
                            const f4v wc = w(c);
                            const float qc = q[c * CH];
#pragma unroll
                            for (int i = 0; i < 4; ++i) a[i] = fmaf(wc[i], qc, a[i]);
                        }
                    }
                };
                if (wlds) {
                    const float* w = W3 + (second ? 4 * l3g * J : 0) + g4;
                    sum([&](int c) { return *(const f4v*)(w + c * 4 * l3g); });
                } else {
                    sum([&](int c) {
                        f4v v;
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = *gptr(m3 + (size_t)min(g4 + i, l3 - 1) * J + clo + c);
                        return v;
                    });
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (g4 + i < l3) out[i] = a[i];
        }
    }
}

// Sum of 16 values over a wave in 17 shuffles: each of the first four levels
// halves the set a lane keeps (the lane bit of the level's offset picks the
// half), the last two add across neighbours, so that afterwards lanes
// 4k .. 4k + 3 hold the total of value k.
__device__ __forceinline__ void wave_sum16(float (&v)[16], int lane) {
#define RTG_HALVE(H, OFF)                                          \
    {                                                              \
        const bool up = (lane & (OFF)) != 0;                       \
        _Pragma("unroll") for (int k = 0; k < (H); ++k) {          \
            const float send = up ? v[k] : v[k + (H)];             \
            const float keep = up ? v[k + (H)] : v[k];             \
            v[k] = keep + __shfl_xor(send, (OFF), 64);             \
        }                                                          \
    }
    RTG_HALVE(8, 32) RTG_HALVE(4, 16) RTG_HALVE(2, 8) RTG_HALVE(1, 4)
#undef RTG_HALVE
    v[0] += __shfl_xor(v[0], 2, 64);
    v[0] += __shfl_xor(v[0], 1, 64);
}

// FROB_CHUNK elements of a tensor, FROB_PT consecutive ones per thread,
// from a buffer that reads zeros past its end.
constexpr int FROB_PT = FROB_CHUNK / 256;
static_assert(FROB_PT == 16, "two 8-element halves per thread");
__device__ __forceinline__ void frob_load(__amdgpu_buffer_rsrc_t r, bool bf, unsigned e, float (&x)[FROB_PT]) {
    if (bf) {
        typedef unsigned int u4v __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const u4v w = __builtin_amdgcn_raw_buffer_load_b128(r, (e + 8u * h) * 2u, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                x[8 * h + 2 * q] = __uint_as_float(w[q] << 16);
                x[8 * h + 2 * q + 1] = __uint_as_float(w[q] & 0xffff0000u);
            }
        }
    } else {
        typedef float f4v __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const f4v w = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(r, (e + 4u * h) * 4u, 0, 0));
#pragma unroll
            for (int q = 0; q < 4; ++q) x[4 * h + q] = w[q];
        }
    }
}

// LDS of one sketched-Gram workgroup
struct GramSmem {
    double ds[2 * (MMAX + 2)];
    double wds[2 * (MMAX + 2)];   // this workgroup's shares
    double h1s[MMAX], hs[MMAX], gnew[MMAX], Gh1[MMAX], Gh[MMAX], cs_s[MMAX], sn_s[MMAX];
    double sG[GLDS * GLDS];       // stored block of G (symmetric), j <= GLDS
    double g_s;
    float s_s[4096];
    float s_v[4096];
    float red[4][16];
    int s_last;
};

// FROB: the sketch is the identity (unsketched global GMRES): the inner
// products are Frobenius products of the full tensors.  Each workgroup takes
// FROB_CHUNK elements of the problem's tensors and forms its shares of
// <V_i, W> and <V_i, V_j> (i <= j) and ||W||^2, reading every stored basis
// tensor once: the orthogonalisation traffic that a sketch avoids.
template <bool FROB>
__device__ __forceinline__ void gram_task(const Desc* __restrict__ descs, const int* __restrict__ starts,
                                          int count, int mode, int j, int b, GramSmem& sm) {
    float* s_s = sm.s_s;
    float* s_v = sm.s_v;
    double* ds = sm.ds;
    double* wds = sm.wds;
    double *h1s = sm.h1s, *hs = sm.hs, *gnew = sm.gnew, *Gh1 = sm.Gh1, *Gh = sm.Gh, *cs_s = sm.cs_s, *sn_s = sm.sn_s;
    double* sG = sm.sG;
    double& g_s = sm.g_s;
    int& s_last = sm.s_last;

    const TileOf at = find_problem(starts, count, b);
    const Desc& d = descs[at.p];
    const int wgi = at.tile;
    const int nwg = d.ntile[KIND_GRAM];
    if ((mode == GM_STEP || mode == GM_GK) && d.state[ST_ACTIVE] == 0) return;

    const int tid = block_tid(), lane = tid & 63, wave = tid >> 6;
    const int nitems = (mode == GM_STEP) ? j + 1 : 1;
    float* sv_dst = nullptr;             // where this workgroup's part of S(V_j) goes
    int sv_n = 0;
    if constexpr (FROB) {
        // ---- Frobenius shares over elements [wgi FROB_CHUNK, (wgi + 1) FROB_CHUNK)
        float (*red)[16] = sm.red;
        const int es = d.bf16 ? 2 : 4;
        const int nb = (int)(d.n * 4);       // float32 tensors (W, R0); the host keeps n 4 < 2^31
        const unsigned e = (unsigned)wgi * FROB_CHUNK + (unsigned)tid * FROB_PT;
        const float* wsrc = (mode == GM_START) ? (const float*)d.R0src : d.W;
        const auto rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(wsrc), (short)0, nb, 0x00020000);
        float wv[FROB_PT];
        frob_load(rw, false, e, wv);
        float nw = 0.f;
#pragma unroll
        for (int u = 0; u < FROB_PT; ++u) nw = fmaf(wv[u], wv[u], nw);
        if (mode == GM_STEP) {
            auto basis = [&](int i) {
                return __builtin_amdgcn_make_buffer_rsrc((char*)d.V + (size_t)i * d.n * es, (short)0, (int)(d.n * es),
                                                         0x00020000);
            };
            float vj[FROB_PT];
            frob_load(basis(j - 1), d.bf16, e, vj);
            for (int i0 = 0; i0 < j; i0 += 8) {
                float acc[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) acc[k] = 0.f;
                float vb[2][FROB_PT];
                frob_load(basis(min(i0, j - 1)), d.bf16, e, vb[0]);
#pragma unroll
                for (int ii = 0; ii < 8; ++ii) {
                    if (ii + 1 < 8) frob_load(basis(min(i0 + ii + 1, j - 1)), d.bf16, e, vb[(ii + 1) & 1]);
                    __builtin_amdgcn_sched_barrier(0);   // one item ahead, no further
                    const bool live = i0 + ii < j;
#pragma unroll
                    for (int u = 0; u < FROB_PT; ++u) {
                        const float x = live ? vb[ii & 1][u] : 0.f;
                        acc[2 * ii] = fmaf(x, wv[u], acc[2 * ii]);
                        acc[2 * ii + 1] = fmaf(x, vj[u], acc[2 * ii + 1]);
                    }
                }
                wave_sum16(acc, lane);
                if ((lane & 3) == 0) red[wave][(lane >> 2) & 15] = acc[0];
                __syncthreads();
                if (tid < 16 && i0 + tid / 2 < j)
                    wds[2 * (i0 + tid / 2) + (tid & 1)] =
                        ((double)red[0][tid] + (double)red[1][tid]) + ((double)red[2][tid] + (double)red[3][tid]);
                __syncthreads();
            }
        }
        const double nws = wave_sum((double)nw);
        if (lane == 0) ds[wave] = nws;
        __syncthreads();
        if (tid == 0) {
            wds[2 * (nitems - 1)] = (ds[0] + ds[1]) + (ds[2] + ds[3]);
            wds[2 * (nitems - 1) + 1] = 0.0;
        }
    } else {
    const int L12 = d.l1 * d.l2, l3 = d.l3;
    const bool split = gram_split(l3, d.J, d.n_i2t);
    const int CH = (!split && d.gram_ch > 0) ? d.gram_ch : gram_pairs_per_block(l3, d.J, d.n_i2t);
    const int q0 = wgi * CH;
    const int qn = min(CH, L12 - q0);
    const int E = qn * l3;

    // in a step the W partials are those of S(Phi(V_j)) taken with the
    // composed first two matrices, so mode 3 is Om3 B^T
    // (Om3 B^T is banded when Om3 is the identity)
    const float* om3 = d.has_om3 ? d.om3 : nullptr;
    // (a general PSF: the W partials are those of W itself, mode 3 is Om3)
    // (the start step of an unnormalised V_1 reads that tensor's partials)
    const float* p_start = (mode == GM_START && d.lazy_v1) ? d.PV : d.PW;
    if (mode == GM_STEP || mode == GM_GK)
        finish_sketches<2>(d, q0, qn, split, d.PW, d.st ? om3 : d.om3t, (d.st || d.has_om3) ? -1 : d.rB, s_s, d.PV,
                           om3, -1, s_v, (float*)sG);
    else
        finish_sketches<1>(d, q0, qn, split, p_start, om3, -1, s_s, nullptr, nullptr, -1, nullptr, (float*)sG);
    __syncthreads();
    if (mode == GM_STEP && j == 1 && d.lazy_v1) {
        // V_1 is stored unnormalised: S(V_1) and S(Phi(V_1)) scale by 1 / beta
        const float ib = (float)(1.0 / d.scal[SC_BETA]);
        for (int e = tid; e < E; e += 256) {
            s_s[e] *= ib;
            s_v[e] *= ib;
        }
        __syncthreads();
    }

    const size_t Lsz = (size_t)d.L;
    sv_dst = (mode == GM_STEP || mode == GM_GK) ? d.SV + (size_t)(j - 1) * Lsz + (size_t)q0 * l3 : nullptr;
    sv_n = E;
    if (mode == GM_GK) {
        // shares of ||s - cf S(Y)||^2 and ||s||^2; Y is the other side's
        // newest stored tensor (V_{c-1} for the U side, none at c = 1; U_c for
        // the V side) and cf its entry of the bidiagonal matrix (beta_c,
        // alpha_c), both written by earlier launches
        const int c = j, mm = d.m;
        const int prow = (d.gk == 1) ? c - 1 : c - 2;
        const double cf = prow < 0 ? 0.0
                                   : ((d.gk == 1) ? d.H[(size_t)(c - 1) * (mm + 1) + (c - 1)]
                                                  : d.H[(size_t)(c - 2) * (mm + 1) + (c - 1)]);
        const float* pv = d.SVx + (size_t)max(prow, 0) * Lsz + (size_t)q0 * l3;
        double a0 = 0.0, a1 = 0.0;
        for (int e = tid; e < E; e += 256) {
            const double se = s_s[e];
            const double t = se - (prow >= 0 ? cf * (double)pv[e] : 0.0);
            a0 += t * t;
            a1 += se * se;
        }
        a0 = wave_sum63(a0);
        a1 = wave_sum63(a1);
        if (lane == 63) {
            ds[2 * wave] = a0;
            ds[2 * wave + 1] = a1;
        }
        __syncthreads();
        if (tid == 0) {
            wds[0] = (ds[0] + ds[2]) + (ds[4] + ds[6]);
            wds[1] = (ds[1] + ds[3]) + (ds[5] + ds[7]);
        }
    }

    // ---- shares of the inner products (float64): <S(V_i), s> and
    // <S(V_i), S(V_j)> for the stored S(V_i), i < j - 1 (from global memory),
    // then the newest tensor S(V_j) and ||s||^2 from LDS.  Stored item i goes
    // to wave i % 4; a wave takes IG of its items per pass with EU elements
    // of each per lane, all loads in flight together (clamped indices,
    // masked: branch-free).
    const int nglob = (mode == GM_STEP) ? j - 1 : 0;
    if (mode != GM_GK) {
    constexpr int IG = 8, EU = 4;
    for (int it0 = wave; it0 < nglob; it0 += 4 * IG) {
        const float* svb = d.SV + (size_t)q0 * l3;
        double as[IG], av[IG];
#pragma unroll
        for (int u = 0; u < IG; ++u) { as[u] = 0.0; av[u] = 0.0; }
        for (int e0 = lane; e0 < E; e0 += 64 * EU) {
            float xv[IG][EU];
#pragma unroll
            for (int u = 0; u < IG; ++u)
                if (u < 4 || it0 + 4 * (u & ~3) < nglob)
#pragma unroll
                    for (int eu = 0; eu < EU; ++eu)
                        xv[u][eu] = *gptr(svb + (size_t)min(it0 + 4 * u, nglob - 1) * Lsz + min(e0 + 64 * eu, E - 1));
#pragma unroll
            for (int eu = 0; eu < EU; ++eu) {
                const int e = e0 + 64 * eu;
                const bool ok = e < E;
                const double se = ok ? (double)s_s[min(e, E - 1)] : 0.0;
                const double ve = ok ? (double)s_v[min(e, E - 1)] : 0.0;
#pragma unroll
                for (int u = 0; u < IG; ++u) {
                    if (u >= 4 && it0 + 4 * (u & ~3) >= nglob) break;
                    as[u] += (double)xv[u][eu] * se;
                    av[u] += (double)xv[u][eu] * ve;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < IG; ++u) {
            if (u >= 4 && it0 + 4 * (u & ~3) >= nglob) break;
            const double ra = wave_sum63(as[u]);
            const double rv = wave_sum63(av[u]);
            if (lane == 63 && it0 + 4 * u < nglob) {
                wds[(it0 + 4 * u) * 2 + 0] = ra;
                wds[(it0 + 4 * u) * 2 + 1] = rv;
            }
        }
    }
    if (wave == 3) {
        double a0 = 0.0, a1 = 0.0, a2 = 0.0;
        for (int e = lane; e < E; e += 64) {
            const double se = s_s[e], ve = (mode == GM_STEP) ? s_v[e] : 0.f;
            a0 += se * se;
            a1 += ve * se;
            a2 += ve * ve;
        }
        a0 = wave_sum63(a0);
        a1 = wave_sum63(a1);
        a2 = wave_sum63(a2);
        if (lane == 63) {
            wds[(nitems - 1) * 2 + 0] = a0;
            wds[(nitems - 1) * 2 + 1] = 0.0;
            if (mode == GM_STEP) {
                wds[(j - 1) * 2 + 0] = a1;
                wds[(j - 1) * 2 + 1] = a2;
            }
        }
    }
    }   // GMRES shares

    }   // sketched shares

    // ---- the last workgroup of this problem finishes the step.  Wave 0
    // publishes the workgroup's shares: coherent stores (agent scope, written
    // through this XCD's L2), a wait until they are done, then it counts the
    // workgroup in; the last one reads the shares with coherent loads.  Nothing
    // else crosses workgroups here, so neither side needs a fence: a release
    // at agent scope writes back the whole L2 of the XCD, one workgroup after
    // the other (512 workgroups of 64 pairs took longer than 128 of 256).
    // A workgroup's 1,568 bytes are no multiple of a cache line, so two XCDs may
    // write parts of one line: the stores are written through by bytes, and the
    // agent-scope loads do not take the copy of a line that this XCD's L2 may
    // hold from its own stores or from an earlier step.
    __syncthreads();
    if (nwg > 1 && wave == 0) {
        double* dst = d.dots + (size_t)wgi * (MMAX + 2) * 2;
        for (int x = lane; x < 2 * nitems; x += 64)
            __hip_atomic_store(gptr_w(dst + x), wds[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane == 0) {
            const int old = __hip_atomic_fetch_add(d.state + ST_COUNTER, 1, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
            s_last = (old == nwg - 1);
        }
    }
    if (nwg > 1) __syncthreads();
    // (stored only now: no barrier above waits for it)
    for (int e = tid; e < sv_n; e += 256)
        if (sv_dst) *gptr_w(sv_dst + e) = s_v[e];
    if (nwg > 1 && !s_last) return;
    // Everything the rest reads from global memory is requested together:
    // the inner-product shares of all workgroups and, in a step with
    // j <= GLDS, the stored block G[0..j-2][0..j-2] (to LDS), the previous
    // plane rotations and g[j-1].
    const int m = d.m;
    const int ldg = m + 1;
    const int jm = j - 1;              // step: column index, also index of the newest basis tensor
    const bool g_lds = (mode == GM_STEP) && j <= GLDS && jm > 0;
    constexpr int GR = GLDS * GLDS / 256;
    double gblk[GR];
    if (g_lds) {
#pragma unroll
        for (int r = 0; r < GR; ++r) {
            const int e = tid + 256 * r, i = e / GLDS, k = e % GLDS;
            gblk[r] = *gptr(d.G + (size_t)min(i, jm - 1) * ldg + min(k, jm - 1));
        }
    }
    double cs_r = 0.0, sn_r = 0.0, g_r = 0.0;
    if (mode == GM_STEP) {
        cs_r = *gptr(d.gv + min(tid, max(jm - 1, 0)));
        sn_r = *gptr(d.gv + m + min(tid, max(jm - 1, 0)));
        g_r = *gptr(d.gv + 2 * m + jm);
    }
    const double beta1 = (mode == GM_STEP && d.lazy_v1) ? *gptr(d.scal + SC_BETA) : 1.0;
    {
        // sums over the workgroups in a fixed order (deterministic): 2^sh
        // threads share a value, each takes every 2^sh-th workgroup, 16 loads
        // in flight, and neighbouring lanes add their parts (a workgroup
        // alone has its shares in LDS already)
        const int nv = 2 * nitems;
        if (nwg == 1)
            for (int x = tid; x < nv; x += 256) ds[x] = wds[x];
        int sh = 0;
        while (sh < 4 && (nv << (sh + 1)) <= 256 && (1 << sh) < nwg) ++sh;
        const int S = 1 << sh;
        for (int x0 = 0; nwg > 1 && x0 < nv; x0 += 256 >> sh) {
            const int x = x0 + (tid >> sh), seg = tid & (S - 1);
            const double* base = d.dots + min(x, nv - 1);
            double part[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) part[u] = 0.0;
            for (int w0 = seg; w0 < nwg; w0 += 16 * S) {
                double v[16];
#pragma unroll
                for (int u = 0; u < 16; ++u)
                    v[u] = load_coherent(base + (size_t)min(w0 + S * u, nwg - 1) * (MMAX + 2) * 2);
#pragma unroll
                for (int u = 0; u < 16; ++u) part[u] += (w0 + S * u < nwg) ? v[u] : 0.0;
            }
#pragma unroll
            for (int h = 8; h > 0; h >>= 1)
#pragma unroll
                for (int u = 0; u < h; ++u) part[u] += part[u + h];
            double t = part[0];
            for (int o = 1; o < S; o <<= 1) t += __shfl_xor(t, o, 64);
            if (seg == 0 && x < nv) ds[x] = t;
        }
    }
    if (g_lds) {
#pragma unroll
        for (int r = 0; r < GR; ++r) {
            const int e = tid + 256 * r, i = e / GLDS, k = e % GLDS;
            if (i < jm && k < jm) sG[e] = gblk[r];   // row and column jm: below, from the new products
        }
    }
    if (mode == GM_STEP) {
        if (tid < jm) {                  // previous plane rotations, staged for the serial update
            cs_s[tid] = cs_r;
            sn_s[tid] = sn_r;
        }
        if (tid == 0) g_s = g_r;
    }
    __syncthreads();
    int* st = d.state;
    double* sc = d.scal;
    double* gvec = d.gv + 2 * m;       // rotated right-hand side g[0..m]
    if (mode == GM_START) {
        if (tid == 0) {
            st[ST_COUNTER] = 0;
            const double beta = sqrt(ds[0]);
            // a restart cycle (j > 0) starts only while ||R0||_Theta >= eps
            // (the residual test that ends the algorithm of Sec. 4.4)
            if (j > 0 && (st[ST_SKIP] != 0 || (d.stop_res > 0.0 && beta < d.stop_res))) {
                st[ST_SKIP] = 1;
                st[ST_ACTIVE] = 0;
                return;
            }
            sc[SC_BETA] = beta;
            gvec[0] = beta;
            if (!(beta > 0.0) || !isfinite(beta)) {
                st[ST_ACTIVE] = 0;
                st[ST_MEFF] = 0;
                st[ST_FLAGS] |= isfinite(beta) ? RTG_F_BREAKDOWN : RTG_F_NONFINITE;
                d.coef[MMAX + 1] = 0.f;
            } else {
                d.coef[MMAX + 1] = (float)(1.0 / beta);
            }
        }
        return;
    }
    if (mode == GM_GK) {
        if (tid == 0) {
            st[ST_COUNTER] = 0;
            const int c = j;
            const double nrm2 = ds[0];
            const double nrm = sqrt(nrm2 > 0.0 ? nrm2 : 0.0), rho = sqrt(ds[1]);
            const bool finite = isfinite(nrm) && isfinite(rho);
            double* Hc = d.H + (size_t)(c - 1) * (m + 1);
            if (d.gk == 2) {
                // alpha_c, the diagonal entry of column c; V_c = (Phi^T(U_c) - beta_c V_{c-1}) / alpha_c
                Hc[c - 1] = nrm;
                if (c >= 2) d.coef[c - 2] = (float)d.H[(size_t)(c - 2) * (m + 1) + (c - 1)];
                d.coef[MMAX + 1] = nrm > 0.0 ? (float)(1.0 / nrm) : 0.f;
                if (!finite) {
                    st[ST_FLAGS] |= RTG_F_NONFINITE;
                    st[ST_MEFF] = c - 1;
                    st[ST_ACTIVE] = 0;
                } else if (nrm <= d.bd_tol * rho) {
                    st[ST_FLAGS] |= RTG_F_BREAKDOWN;
                    st[ST_MEFF] = c - 1;
                    st[ST_ACTIVE] = 0;
                }
            } else {
                // beta_{c+1} completes column c = (alpha_c, beta_{c+1}) in rows c-1, c;
                // U_{c+1} = (Phi(V_c) - alpha_c U_c) / beta_{c+1}
                const double alpha = Hc[c - 1];
                Hc[c] = nrm;
                // Givens update: of the earlier rotations only the last one
                // meets a nonzero entry of this column
                double* cs = d.gv;
                double* sn = d.gv + m;
                double* Rc = d.R + (size_t)(c - 1) * m;
                for (int i = 0; i + 2 < c; ++i) Rc[i] = 0.0;
                double r_prev = alpha;
                if (c >= 2) {
                    Rc[c - 2] = sn[c - 2] * alpha;
                    r_prev = cs[c - 2] * alpha;
                }
                const double gj = gvec[c - 1];
                if (!finite) {
                    // the solve keeps the c - 1 complete columns: their
                    // rotations and g_1..g_c stay as the last step left them
                    st[ST_FLAGS] |= RTG_F_NONFINITE;
                    st[ST_MEFF] = c - 1;
                    st[ST_ACTIVE] = 0;
                    return;
                }
                const double rr = hypot(r_prev, nrm);
                const double cj = rr > 0.0 ? r_prev / rr : 1.0;
                const double sj = rr > 0.0 ? nrm / rr : 0.0;
                cs[c - 1] = cj;
                sn[c - 1] = sj;
                Rc[c - 1] = rr;
                gvec[c - 1] = cj * gj;
                gvec[c] = -sj * gj;
                const double res_ls = fabs(gvec[c]);
                sc[SC_RESLS] = res_ls;
                d.coef[c - 1] = (float)alpha;
                d.coef[MMAX + 1] = nrm > 0.0 ? (float)(1.0 / nrm) : 0.f;
                if (nrm <= d.bd_tol * rho) {
                    st[ST_FLAGS] |= RTG_F_BREAKDOWN;
                    st[ST_MEFF] = c;
                    st[ST_ACTIVE] = 0;
                } else if (d.stop_res > 0.0 && res_ls <= d.stop_res) {
                    st[ST_MEFF] = c;
                    st[ST_ACTIVE] = 0;
                } else if (c >= m && !d.keep_last) {
                    st[ST_MEFF] = c;
                    st[ST_ACTIVE] = 0;
                    if (d.stop_res > 0.0) st[ST_FLAGS] |= RTG_F_NOT_CONVERGED;
                } else {
                    st[ST_MEFF] = c;
                }
            }
        }
        return;
    }

    // ---- step j: classical Gram-Schmidt + reorthogonalisation in sketch space
    // (this tail runs in one workgroup per problem while the chip waits: its
    // length is a chain of LDS latencies and barriers, so the products with G
    // are split over the waves and everything else is one wave, a column entry
    // per lane)
    if (tid < j) {
        h1s[tid] = ds[2 * tid];
        const double gn = ds[2 * tid + 1];
        gnew[tid] = gn;                  // (to the stored G below: no barrier here waits for the stores)
        if (j <= GLDS) {
            sG[tid * GLDS + jm] = gn;
            sG[jm * GLDS + tid] = gn;
        }
    }
    __syncthreads();
    if (j <= GLDS) {
        // Gh1 = G h1, h = 2 h1 - G h1, then Gh = G h.  Lane i of every wave
        // takes row i (G is symmetric: read as column i, neighbouring lanes on
        // neighbouring words) over the wave's quarter of the columns; the
        // quarters meet in LDS (the finished sketches' space, free by now).
        // Each wave keeps its own copy of h, so one barrier per product is enough.
        double* red = (double*)s_v;                  // [2][4][GLDS]
        double* hw = (double*)s_s + wave * GLDS;
        const int kq = (j + 3) >> 2, k0 = wave * kq, k1 = min(j, k0 + kq);
        double acc = 0.0;
#pragma unroll 4
        for (int k = k0; k < k1; ++k) acc = fma(sG[k * GLDS + lane], h1s[k], acc);
        red[wave * GLDS + lane] = acc;
        __syncthreads();
        const double g1 = (red[lane] + red[GLDS + lane]) + (red[2 * GLDS + lane] + red[3 * GLDS + lane]);
        hw[lane] = 2.0 * h1s[min(lane, j - 1)] - g1;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        acc = 0.0;
#pragma unroll 4
        for (int k = k0; k < k1; ++k) acc = fma(sG[k * GLDS + lane], hw[k], acc);
        red[(4 + wave) * GLDS + lane] = acc;
        if (wave == 0 && lane < j) hs[lane] = hw[lane];
        __syncthreads();
        if (wave == 0 && lane < j)
            Gh[lane] = (red[4 * GLDS + lane] + red[5 * GLDS + lane]) + (red[6 * GLDS + lane] + red[7 * GLDS + lane]);
    } else {
        // each wave takes four rows at a time, lanes run along the row
        // (coalesced), wave reductions
        auto gmatvec = [&](const double* v, double* out, bool make_h) {
            for (int i0 = wave * 4; i0 < j; i0 += 16) {
                double acc4[4] = {0.0, 0.0, 0.0, 0.0};
                double gi[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) gi[u] = gnew[min(i0 + u, j - 1)];
                for (int k = lane; k < j; k += 64) {
                    const double vk = v[k];
                    const double gk = gnew[k];
                    double gl[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) gl[u] = *gptr(d.G + (size_t)min(i0 + u, j - 1) * ldg + k);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        // row / column jm of G are the new entries (held in LDS)
                        const int i = min(i0 + u, j - 1);
                        double gik = (k == jm) ? gi[u] : gl[u];
                        gik = (i == jm) ? gk : gik;
                        acc4[u] += gik * vk;
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = i0 + u;
                    const double r = wave_sum(acc4[u]);
                    if (lane == 0 && i < j) {
                        out[i] = r;
                        if (make_h) hs[i] = 2.0 * h1s[i] - r;
                    }
                }
            }
        };
        gmatvec(h1s, Gh1, true);
        __syncthreads();
        gmatvec(hs, Gh, false);
        __syncthreads();
    }
    if (wave != 0) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // ---- the rest in wave 0: lane i holds column entries i and i + 64
    const double nrm2 = ds[2 * j];
    const double h0 = lane < j ? hs[lane] : 0.0, hx = lane + 64 < j ? hs[min(lane + 64, MMAX - 1)] : 0.0;
    double hth1 = 0.0, hGh = 0.0;
    bool finite = isfinite(h0) && isfinite(hx);
    if (lane < j) {
        hth1 = h0 * h1s[lane];
        hGh = h0 * Gh[lane];
    }
    if (lane + 64 < j) {
        hth1 += hx * h1s[lane + 64];
        hGh += hx * Gh[lane + 64];
    }
    hth1 = lane63(wave_sum63(hth1));
    hGh = lane63(wave_sum63(hGh));
    finite = (__ballot(!finite) == 0ull) && isfinite(nrm2);
    const double hn2 = nrm2 - 2.0 * hth1 + hGh;
    const double hn = sqrt(hn2 > 0.0 ? hn2 : 0.0);
    const double rho = sqrt(nrm2);
    finite = finite && isfinite(hn);
    if (lane == 0) st[ST_COUNTER] = 0;
    if (!finite) {
        // the solve keeps the jm complete columns: the rotations, R and
        // g_1..g_j stay as step jm left them (so gamma_j = g_j is the
        // residual of the jm-step problem)
        if (lane == 0) {
            st[ST_FLAGS] |= RTG_F_NONFINITE;
            st[ST_MEFF] = jm;
            st[ST_ACTIVE] = 0;
        }
        return;
    }
    // coefficients of the orthogonalisation / normalisation (an unnormalised
    // stored V_1 = beta V_1 takes 1 / beta: in the scale at step 1, where it
    // is also the tensor the operator is applied to, and in its own
    // coefficient later)
    const double ib = 1.0 / beta1;
    double* Hc = d.H + (size_t)jm * (m + 1);         // Hessenberg column
    for (int i = lane; i < j; i += 64) {
        const double gn = gnew[i];
        d.G[(size_t)i * ldg + jm] = gn;
        d.G[(size_t)jm * ldg + i] = gn;
    }
    if (lane < j) {
        Hc[lane] = h0;
        d.coef[lane] = (float)(h0 * ((lane == 0 && j >= 2) ? ib : 1.0));
    }
    if (lane + 64 < j) {
        Hc[lane + 64] = hx;
        d.coef[lane + 64] = (float)hx;
    }
    // Givens update of the projected least-squares problem: the earlier
    // rotations on the new column, R[i] = c_i r_i + s_i h_{i+1} with the
    // recurrence r_{i+1} = -s_i r_i + c_i h_{i+1}, r_0 = h_0, as a scan over
    // the lanes (|s_i| <= 1: the composed coefficients do not grow)
    double* Rc = d.R + (size_t)jm * m;
    double r_prev = hs[0];
    for (int i0 = 0; i0 < jm; i0 += 64) {
        const int i = i0 + lane;
        const bool on = i < jm;
        const double ci = on ? cs_s[i] : 0.0, si = on ? sn_s[i] : -1.0, hn1 = on ? hs[i + 1] : 0.0;
        double A = -si, B = ci * hn1;                    // past the end: r stays
        wave_compose(A, B);
        const double r1 = fma(A, r_prev, B);             // r_{i+1}
        double r0 = dpp_or<DPP_SHR + 1>(r1, r_prev);     // r_i: the neighbour's, row by row
        const double r15 = dpp_or<DPP_BC15>(r1, r_prev), r31 = dpp_or<DPP_BC31>(r1, r_prev);
        r0 = (lane & 31) == 16 ? r15 : (lane == 32 ? r31 : r0);
        if (on) Rc[i] = ci * r0 + si * hn1;
        r_prev = lane63(r1);
    }
    if (lane != 0) return;
    Hc[j] = hn;
    const double rr = hypot(r_prev, hn);
    const double cj = rr > 0.0 ? r_prev / rr : 1.0;
    const double sj = rr > 0.0 ? hn / rr : 0.0;
    d.gv[jm] = cj;
    d.gv[m + jm] = sj;
    Rc[jm] = rr;
    const double gj = g_s, gn = -sj * gj;
    gvec[jm] = cj * gj;
    gvec[j] = gn;
    const double res_ls = fabs(gn);
    sc[SC_RESLS] = res_ls;
    d.coef[MMAX + 1] = hn > 0.0 ? (float)((j == 1 ? ib : 1.0) / hn) : 0.f;
    // stopping decisions
    if (hn <= d.bd_tol * rho) {
        st[ST_FLAGS] |= RTG_F_BREAKDOWN;
        st[ST_MEFF] = j;
        st[ST_ACTIVE] = 0;
    } else if (d.stop_res > 0.0 && res_ls <= d.stop_res) {
        st[ST_MEFF] = j;
        st[ST_ACTIVE] = 0;
    } else if (j >= m && !d.keep_last) {
        st[ST_MEFF] = j;
        st[ST_ACTIVE] = 0;
        if (d.stop_res > 0.0) st[ST_FLAGS] |= RTG_F_NOT_CONVERGED;
    } else {
        st[ST_MEFF] = j;
    }
}

}  // namespace rtg

#pragma once
// Fused multi-AXPY, store and mode-wise sketches over one column tile.
//
// A tile is I1 rows x 32 columns (i2) of one channel c, a contiguous block of
// memory in the i1-fastest layout.  Depending on the mode the workgroup
//
//   out = scale * (src - sum_{i<nterms} coef_i V_i)            (multi-AXPY)
//
// which is the orthogonalisation and normalisation of the Arnoldi step
// (Sec. 4.3: W <- W - h_ij V_i, V_{j+1} = W / h_{j+1,j}), a Golub-Kahan
// half-step (Sec. 4.5: one term, U_{k+1} = (Phi(V_k) - alpha_k U_k) / beta_{k+1}
// or V_{k+1} = (Phi^T(U_{k+1}) - beta_{k+1} V_k) / alpha_{k+1}, where the
// composed matrices belong to the operator of the side written) or the
// solution update X = X0 + sum_j y_j V_j (Sec. 4.4), stores it, and/or
// sketches it:
//
//   P[a, b] = sum_{i2 in tile} Om2[b, i2] sum_{i1} Om1[a, i1] out[i1, i2]
//
// (the first two mode products of S(X) = X x_1 Om1 x_2 Om2 x_3 Om3,
// Sec. 3.1).  A new basis tensor is sketched twice in the same pass: with
// (Om1, Om2) for S(V_{j+1}) and with the composed matrices (Om1 A1, Om2 A2)
// for S(Phi(V_{j+1})), because mode products compose and Phi is the mode-wise
// product with (A1, A2, B^T) (eq. (2)).  The next step's sketched inner
// products then need no separate pass over W = Phi(V_{j+1}).
//
// Phase 1 (per block of SBR rows): every lane owns SBR / 8 elements of the
// tile, accumulates the multi-AXPY in float32 registers, stores the result
// (rounded to bfloat16 for a bfloat16 basis) and writes it to LDS, column-
// major.  Terms go in groups, two groups in flight: 16 to 32 KB per workgroup
// (one 512x512x3 problem has 48 workgroups and is bound by their latency:
// 63 -> 45 us per launch against one term in two halves).  Phase 2: the four waves split the (stacked) sketch rows and run the
// mode-1 contraction on MFMA with the tile from LDS as the B operand
// (v_mfma_f32_16x16x4f32 for a float32 basis, v_mfma_f32_16x16x32_bf16 for a
// bfloat16 one; a float32 tile in bfloat16 mode is split into high and low
// bfloat16 planes, and so is the composed matrix Om1 A1).  After the last
// block the mode-2 contraction is a second small MFMA product, and the
// partial P of every tile goes to a buffer that the sketched-Gram kernel
// reduces (applying mode 3).

#include "rtg_internal.h"

namespace rtg {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));
typedef unsigned int u2v __attribute__((ext_vector_type(2)));

// element offset of a chunk outside the tile: its byte offset lies past every
// buffer extent used here (a tile spans 32 x I1 elements of at most 4 bytes)
constexpr unsigned OOB_ELEM = 0x20000000u;
// byte offset past the operand-order sketch matrices (under 1 GiB a plane)
constexpr unsigned OOB_A = 0x80000000u;

// raw buffer resource over [base, base + bytes): loads past the end return
// zero and stores past it are dropped
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, bytes, 0x00020000);
}

template <bool MB, bool SPLIT, int RPW, int SBR>
struct TileSmem {
    static constexpr int TC = TILE_TC;
    static constexpr int CSB = SBR + 8;         // bfloat16 plane column stride (elements)
    static constexpr int CSF = SBR + 4;         // float32 column stride (elements)
    static constexpr int XBYTES = MB ? (SPLIT ? 2 : 1) * TC * CSB * 2 : TC * CSF * 4;
    static constexpr int YP = TC + 1;
    static constexpr int YBYTES = 64 * RPW * YP * 4;   // stacked sketch rows x columns
    static constexpr int BYTES = XBYTES > YBYTES ? XBYTES : YBYTES;
};

// LDS of one tile workgroup
template <bool MB, bool SPLIT, int RPW, int SBR>
struct TileShared {
    float coef_s[MMAX + 2];
    __attribute__((aligned(16))) unsigned char smem[TileSmem<MB, SPLIT, RPW, SBR>::BYTES];
};

// BB: basis stored as bfloat16; MB: the sketch contractions take bfloat16
// MFMA operands (float32 accumulation) -- a bfloat16 basis always does, a
// float32 basis in the mixed form (RTG_F32_BF16) does with its tile rounded
// to bfloat16 for the products; SPLIT: the sketched tile is float32 in
// bfloat16 mode, split into two planes; RPW: sketch row tiles of 16 per wave.
template <bool BB, bool MB, bool SPLIT, int RPW, int SBR>
__device__ __forceinline__ void tile_task(const Desc* __restrict__ descs, const int* __restrict__ starts,
                                          int count, int mode, int nterms_arg, int dst_index, int t0, int b,
                                          TileShared<MB, SPLIT, RPW, SBR>& sh) {
    static_assert(MB || !BB, "a bfloat16 basis uses bfloat16 products");
    using SM = TileSmem<MB, SPLIT, RPW, SBR>;
    constexpr int TC = TILE_TC;
    constexpr int CK = BB ? 8 : 4;             // elements per lane chunk (16 bytes of basis)
    constexpr int NCK = SBR * TC / 256 / CK;   // chunks per lane and term
    constexpr int KBR = MB ? 32 : 16;          // rows per MFMA K-block
    constexpr int NKB = SBR / KBR;             // K-blocks per block
    constexpr int GT = NCK >= (BB ? 4 : 8) ? 1 : (NCK >= (BB ? 2 : 4) ? 2 : 4);   // terms per group, two groups in flight
    constexpr int CSB = SM::CSB, CSF = SM::CSF, YP = SM::YP;

    float* coef_s = sh.coef_s;
    unsigned char* smem = sh.smem;
    bf16_t* Xh = (bf16_t*)smem;                 // high (or only) bfloat16 plane
    bf16_t* Xl = Xh + TC * CSB;                 // low plane (SPLIT)
    float* Xf = (float*)smem;                   // float32 tile
    float* Ys = (float*)smem;                   // mode-1 results (after the last block)

    const TileOf at = find_problem(starts, count, b);
    const Desc& d = descs[at.p];
    const int tile = at.tile;
    const bool newv = (mode == TM_NEWV || mode == TM_GKNEW || mode == TM_NEWV1);
    // V_1 stored by the operator kernel already: sketched from the basis
    const bool v1_stored = (mode == TM_NEWV1) && d.X0 != nullptr;
    if ((newv || mode == TM_SKETCH_W) && d.state[ST_ACTIVE] == 0) return;
    if (mode == TM_ASSEMBLE && d.state[ST_SKIP] != 0) return;   // X stays (restart cycle sat out)

    const int tid = block_tid();
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m16 = lane & 15;        // MFMA row (A) / column (B) index
    const int kq = lane >> 4;         // MFMA K group

    const int I1 = d.I1, I2 = d.I2;
    const int l1 = d.l1, l2 = d.l2;
    // rows [row0, row1) of column tile t2 of channel c: the tile's row part
    const int nrs = d.nrs, ct = tile / nrs;
    const int t2 = ct % d.n_i2t, c = ct / d.n_i2t;
    const int row0 = (tile - ct * nrs) * d.prow, row1 = min(I1, row0 + d.prow);
    const int i20 = t2 * TC;
    const int ncol = min(TC, I2 - i20);
    const size_t tile_off = (size_t)c * I1 * I2 + (size_t)i20 * I1;
    const size_t es = BB ? 2 : 4;

    int nterms = 0;
    if (newv) nterms = nterms_arg;
    else if (mode == TM_ASSEMBLE) nterms = uniform_int(d.state[ST_MEFF]);
    const int first = (mode == TM_GKNEW) ? t0 : 0;   // terms [first, nterms)
    const bool do_store = (newv || mode == TM_ASSEMBLE) && !v1_stored;
    const bool do_sketch = (mode != TM_ASSEMBLE) && !d.unsketched;   // an identity sketch keeps no partials
    const bool dual = newv && d.st == nullptr;   // a general PSF has no composed sketch matrices
    const bool src_is_bf = BB && !SPLIT && (mode == TM_SKETCH_SRC || v1_stored);

    const void* src;
    if (mode == TM_SKETCH_SRC) src = d.R0src;
    else if (mode == TM_SKETCH_W) src = d.W;
    else if (mode == TM_NEWV) src = (nterms == 0) ? d.R0src : (const void*)d.W;
    else if (mode == TM_NEWV1) src = v1_stored ? (const void*)d.V : d.R0src;
    else if (mode == TM_GKNEW) src = d.W;
    else src = d.X0;     // may be null: zero
    src = uniform_ptr(src);

    for (int i = tid; i < nterms; i += 256) coef_s[i] = d.coef[i];
    const float scale = do_store ? d.coef[MMAX + 1] : 1.f;
    __syncthreads();

    const int RT = (l1 + 15) >> 4;
    const int NRT = dual ? 2 * RT : RT;       // stacked row tiles: [Om1 ; Om1 A1]
    // sketch matrices in operand order: Om1, and Om1 A1 (bfloat16: high
    // plane then low plane)
    const int nkbf = frag_nkb(I1, KBR);
    const unsigned fbytes = (unsigned)frag_elems(l1, I1, KBR) * (MB ? 2u : 4u);
    const auto rom1 = make_rsrc(MB ? (const void*)d.om1hf : (const void*)d.om1f, (int)fbytes);
    const auto rom1c = make_rsrc(MB ? (const void*)d.om1th : (const void*)d.om1t, (int)(MB ? 2 * fbytes : fbytes));
    f4 acc[RPW][2];
#pragma unroll
    for (int u = 0; u < RPW; ++u)
#pragma unroll
        for (int g = 0; g < 2; ++g) acc[u][g] = f4{0.f, 0.f, 0.f, 0.f};

    // chunk u of this lane: column col[u], rows row[u] .. row[u] + CK - 1 of the block
    int colu[NCK], rowu[NCK];
#pragma unroll
    for (int u = 0; u < NCK; ++u) {
        const int e = (u * 256 + tid) * CK;
        colu[u] = e / SBR;
        rowu[u] = e % SBR;
    }
    const int tile_elems = ncol * I1;

    for (int r0 = row0; r0 < row1; r0 += SBR) {
        // ---- phase 1: multi-AXPY, store, LDS.
        // Buffer loads and stores with per-lane byte offsets from a uniform
        // base: a chunk outside the tile gets an offset past the buffer's
        // extent, so the hardware returns zeros for its loads and drops its
        // stores -- no branches, no clamping, all loads in flight together.
        unsigned offs[NCK];
#pragma unroll
        for (int u = 0; u < NCK; ++u) {
            const int rg = r0 + rowu[u];
            offs[u] = ((rg < row1) & (colu[u] < ncol)) ? (unsigned)(colu[u] * I1 + rg) : OOB_ELEM;
        }
        // multi-AXPY in groups of GT terms: a group is under way while the
        // one before it is applied
        u4 v[2][GT][NCK];
        const int ngr = (nterms - first + GT - 1) / GT;
        auto load_group = [&](int g, u4 (&vg)[GT][NCK]) {
#pragma unroll
            for (int q = 0; q < GT; ++q) {
                const int i = first + g * GT + q;
                if (i >= nterms) break;
                const auto rv = make_rsrc((const char*)d.V + ((size_t)i * d.n + tile_off) * es, tile_elems * (int)es);
#pragma unroll
                for (int u = 0; u < NCK; ++u)
                    vg[q][u] = __builtin_amdgcn_raw_buffer_load_b128(rv, offs[u] * (unsigned)es, 0, 0);
            }
        };
        float x[NCK][CK];
        auto apply_group = [&](int g, const u4 (&vg)[GT][NCK]) {
#pragma unroll
            for (int q = 0; q < GT; ++q) {
                const int i = first + g * GT + q;
                if (i >= nterms) break;
                const float ci = coef_s[i];
#pragma unroll
                for (int u = 0; u < NCK; ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if constexpr (BB) {
                            x[u][2 * r] = fmaf(-ci, __uint_as_float(vg[q][u][r] << 16), x[u][2 * r]);
                            x[u][2 * r + 1] = fmaf(-ci, __uint_as_float(vg[q][u][r] & 0xffff0000u), x[u][2 * r + 1]);
                        } else {
                            x[u][r] = fmaf(-ci, __uint_as_float(vg[q][u][r]), x[u][r]);
                        }
                    }
            }
        };
        // the source first: the terms are applied to it in order
        u4 xs[NCK][BB ? 2 : 1];
        if (src != nullptr) {
            if (src_is_bf) {
                const auto rs = make_rsrc((const char*)src + tile_off * 2, tile_elems * 2);
#pragma unroll
                for (int u = 0; u < NCK; ++u) xs[u][0] = __builtin_amdgcn_raw_buffer_load_b128(rs, offs[u] * 2u, 0, 0);
            } else {
                const auto rs = make_rsrc((const char*)src + tile_off * 4, tile_elems * 4);
#pragma unroll
                for (int u = 0; u < NCK; ++u)
#pragma unroll
                    for (int q = 0; q < CK / 4; ++q)
                        xs[u][q] = __builtin_amdgcn_raw_buffer_load_b128(rs, offs[u] * 4u + q * 16u, 0, 0);
            }
        }
        if (ngr > 0) load_group(0, v[0]);
        if (ngr > 1) load_group(1, v[1]);
        // A fragments of this block's products in operand order: one
        // contiguous 1 KB read per wave and tile; padding rows and columns
        // are stored zeros, and unused tiles (t >= NRT) read nothing (offset
        // past the buffer range)
        struct AF {
            u4 h, l;     // bfloat16 products: Om1 (h), or Om1 A1 high / low; float32: h as f4 bits
        };
        auto load_a = [&](int kb, AF* A) {
            const int kbg = r0 / KBR + kb;           // (row parts start at multiples of 64)
#pragma unroll
            for (int u = 0; u < RPW; ++u) {
                const int t = wave + 4 * u;
                const bool half = t >= RT;
                const int tl = t - (half ? RT : 0);
                const unsigned off = (t < NRT) ? (unsigned)((tl * nkbf + kbg) * 64 + lane) * 16u : OOB_A;
                const auto& rs = half ? rom1c : rom1;
                A[u].h = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
                if constexpr (MB)
                    A[u].l = half ? __builtin_amdgcn_raw_buffer_load_b128(rs, off + fbytes, 0, 0) : u4{0u, 0u, 0u, 0u};
            }
        };
#pragma unroll
        for (int u = 0; u < NCK; ++u)
#pragma unroll
            for (int q = 0; q < CK / 4; ++q) {
                if (src == nullptr) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) x[u][4 * q + r] = 0.f;
                } else if (src_is_bf) {
                    if constexpr (BB) {
#pragma unroll
                        for (int r = 0; r < 2; ++r) {
                            const unsigned w = xs[u][0][2 * q + r];
                            x[u][4 * q + 2 * r] = __uint_as_float(w << 16);
                            x[u][4 * q + 2 * r + 1] = __uint_as_float(w & 0xffff0000u);
                        }
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) x[u][4 * q + r] = __uint_as_float(xs[u][q][r]);
                }
            }
        for (int g = 0; g < ngr; g += 2) {
            apply_group(g, v[0]);
            if (g + 2 < ngr) load_group(g + 2, v[0]);
            if (g + 1 < ngr) {
                apply_group(g + 1, v[1]);
                if (g + 3 < ngr) load_group(g + 3, v[1]);
            }
        }
        // scale (chunks outside the tile are zero already), round (bfloat16 basis), store
#pragma unroll
        for (int u = 0; u < NCK; ++u)
#pragma unroll
            for (int q = 0; q < CK; ++q) x[u][q] *= scale;
        const int nkb = (min(SBR, row1 - r0) + KBR - 1) / KBR;
        AF A0[RPW], A1[RPW];
        if (do_sketch) {
            load_a(0, A0);
            if (nkb > 1) load_a(1, A1);
        }
        if (newv && BB && do_store) {
            const auto rd = make_rsrc((const char*)d.V + ((size_t)dst_index * d.n + tile_off) * 2, tile_elems * 2);
#pragma unroll
            for (int u = 0; u < NCK; ++u) {
                u4 pk;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    pk[q] = (unsigned)f2bf(x[u][2 * q]) | ((unsigned)f2bf(x[u][2 * q + 1]) << 16);
                __builtin_amdgcn_raw_buffer_store_b128(pk, rd, offs[u] * 2u, 0, 0);
            }
        } else if (do_store) {
            const char* db = newv ? (const char*)d.V + ((size_t)dst_index * d.n + tile_off) * 4
                                               : (const char*)d.X + tile_off * 4;
            const auto rd = make_rsrc(db, tile_elems * 4);
#pragma unroll
            for (int u = 0; u < NCK; ++u)
#pragma unroll
                for (int q = 0; q < CK; q += 4) {
                    const u4 pk = u4{__float_as_uint(x[u][q]), __float_as_uint(x[u][q + 1]),
                                     __float_as_uint(x[u][q + 2]), __float_as_uint(x[u][q + 3])};
                    __builtin_amdgcn_raw_buffer_store_b128(pk, rd, offs[u] * 4u + q * 4u, 0, 0);
                }
        }
        if (!do_sketch) continue;
        if (r0 > row0) __syncthreads();       // the previous block's MFMA reads are done
#pragma unroll
        for (int u = 0; u < NCK; ++u) {
            if constexpr (MB && !BB && !SPLIT) {
                // float32 basis, bfloat16 products: the chunk's four values rounded
                u2v hi;
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    hi[q] = (unsigned)f2bf(x[u][2 * q]) | ((unsigned)f2bf(x[u][2 * q + 1]) << 16);
                *(u2v*)(Xh + colu[u] * CSB + rowu[u]) = hi;
            } else if constexpr (MB && !BB) {
                // float32 source split into high and low planes
                u2v hi, lo;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const bf16_t h0 = f2bf(x[u][2 * q]), h1 = f2bf(x[u][2 * q + 1]);
                    hi[q] = (unsigned)h0 | ((unsigned)h1 << 16);
                    const bf16_t g0 = f2bf(x[u][2 * q] - bf2f(h0)), g1 = f2bf(x[u][2 * q + 1] - bf2f(h1));
                    lo[q] = (unsigned)g0 | ((unsigned)g1 << 16);
                }
                *(u2v*)(Xh + colu[u] * CSB + rowu[u]) = hi;
                *(u2v*)(Xl + colu[u] * CSB + rowu[u]) = lo;
            } else if constexpr (BB) {
                u4 hi, lo;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bf16_t h0 = f2bf(x[u][2 * q]), h1 = f2bf(x[u][2 * q + 1]);
                    hi[q] = (unsigned)h0 | ((unsigned)h1 << 16);
                    if constexpr (SPLIT) {
                        const bf16_t g0 = f2bf(x[u][2 * q] - bf2f(h0)), g1 = f2bf(x[u][2 * q + 1] - bf2f(h1));
                        lo[q] = (unsigned)g0 | ((unsigned)g1 << 16);
                    }
                }
                *(u4*)(Xh + colu[u] * CSB + rowu[u]) = hi;
                if constexpr (SPLIT) *(u4*)(Xl + colu[u] * CSB + rowu[u]) = lo;
            } else {
                *(f4*)(Xf + colu[u] * CSF + rowu[u]) = f4{x[u][0], x[u][1], x[u][2], x[u][3]};
            }
        }
        __syncthreads();

        // ---- phase 2: mode-1 contraction of this block on MFMA.
        // Wave w owns stacked row tiles w, w + 4, ...; rows of tile t are
        // rows of Om1 (t < RT) or of Om1 A1 (RT <= t < 2 RT).
        auto mfma_block = [&](int kb, const AF* A) {
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const int col = 16 * g + m16;
                if constexpr (MB) {
                    const u4 bh = *(const u4*)(Xh + col * CSB + kb * KBR + 8 * kq);
                    u4 bl = u4{0u, 0u, 0u, 0u};
                    if constexpr (SPLIT) bl = *(const u4*)(Xl + col * CSB + kb * KBR + 8 * kq);
#pragma unroll
                    for (int u = 0; u < RPW; ++u) {
                        const int t = wave + 4 * u;
                        if (t >= NRT) break;
                        acc[u][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf8, A[u].h), __builtin_bit_cast(bf8, bh), acc[u][g], 0, 0, 0);
                        if (t >= RT)
                            acc[u][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                __builtin_bit_cast(bf8, A[u].l), __builtin_bit_cast(bf8, bh), acc[u][g], 0, 0, 0);
                        if constexpr (SPLIT)
                            acc[u][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                __builtin_bit_cast(bf8, A[u].h), __builtin_bit_cast(bf8, bl), acc[u][g], 0, 0, 0);
                    }
                } else {
                    const f4 bv = *(const f4*)(Xf + col * CSF + kb * KBR + 4 * kq);
#pragma unroll
                    for (int u = 0; u < RPW; ++u) {
                        const int t = wave + 4 * u;
                        if (t >= NRT) break;
                        const f4 av = __builtin_bit_cast(f4, A[u].h);
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            acc[u][g] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[q], bv[q], acc[u][g], 0, 0, 0);
                    }
                }
            }
        };
        // the fragments of the next K-block are loaded while the current one
        // is multiplied (two named buffers: no dynamically indexed arrays);
        // whole blocks unrolled, the last rows in a loop
        if (nkb == NKB) {
#pragma unroll
            for (int kb = 0; kb < NKB; kb += 2) {
                mfma_block(kb, A0);
                if (kb + 2 < NKB) load_a(kb + 2, A0);
                if (kb + 1 < NKB) {
                    mfma_block(kb + 1, A1);
                    if (kb + 3 < NKB) load_a(kb + 3, A1);
                }
            }
        } else {
            for (int kb = 0; kb < nkb; kb += 2) {
                mfma_block(kb, A0);
                if (kb + 1 < nkb) {
                    if (kb + 2 < nkb) load_a(kb + 2, A0);
                    mfma_block(kb + 1, A1);
                    if (kb + 3 < nkb) load_a(kb + 3, A1);
                }
            }
        }
    }
    if (!do_sketch) return;

    // ---- mode-1 results to LDS: Ys[16 t + r][col]
    float* Pt0 = (newv ? d.PV : d.PW) + (size_t)tile * l1 * l2;
    float* Pt1 = d.PW + (size_t)tile * l1 * l2;
    Mode2Ops<TC> m2;
    mode2_load<TC>(m2, wave, lane, l2, I2, i20, ncol, NRT, RT, d.om2, d.om2t);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < RPW; ++u) {
        const int t = wave + 4 * u;
        if (t >= NRT) break;
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i) Ys[(16 * t + 4 * kq + i) * YP + 16 * g + m16] = acc[u][g][i];
    }
    __syncthreads();

    // ---- mode-2 contraction: P[a][b] = sum_k Ys[a][k] Om2x[b][i20 + k]
    mode2_partials_all<TC, YP>(Ys, m2, wave, lane, NRT, RT, l1, l2, Pt0, Pt1);
}

}  // namespace rtg

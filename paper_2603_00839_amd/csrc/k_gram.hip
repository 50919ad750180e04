// Sketched-Gram kernel (the stage itself is gram_task in gram_body.h) and the
// finish of a stand-alone sketch.
#include "gram_body.h"

namespace rtg {

template <bool FROB>
__global__ void __launch_bounds__(256) k_gram(const Desc* __restrict__ descs,
                                              const int* __restrict__ starts, int count, int mode,
                                              int j) {
    __shared__ GramSmem sm;
    gram_task<FROB>(descs, starts, count, mode, j, blockIdx.x, sm);
}

// A stand-alone sketch: the finished values of each workgroup's pairs, written
// in the column-major order of the C ABI.  A kernel of its own: within the Gram
// step's 57 KB of code every launch was half a microsecond longer.  Where pairs
// carry many column tiles in at most GRAM_SPL channels, a thread takes one pair
// of one channel with 32 loads in flight and the sums meet in LDS once: bound by
// the loads' latency, and with a few dozen workgroups the two passes of
// finish_sketches leave most threads idle (200x994x8 to 33x16x3: 3.9 us, 7.0 in
// two passes; 1000x700x3 to 64x64x3 3.9 and 5.3).  With more channels a thread
// would take several in turn (256x256x64 to 48x48x16: 13 us, 8.1 in two passes).
__global__ void __launch_bounds__(256) k_sketch_out(const Desc* __restrict__ descs, float* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) float Q[FINQ];
    __shared__ float s[4096];
    const Desc& d = descs[0];
    const int l1 = d.l1, l2 = d.l2, l3 = d.l3, J = d.J, nt2 = d.n_i2t;
    const int L12 = l1 * l2, tid = threadIdx.x;
    const bool split = gram_split(l3, J, nt2);
    const int CH = (!split && d.gram_ch > 0) ? d.gram_ch : gram_pairs_per_block(l3, J, nt2);
    const int q0 = blockIdx.x * CH;
    const int qn = min(CH, L12 - q0);
    const float* m3 = d.has_om3 ? d.om3 : nullptr;
    auto put = [&](int t, int c3, float v) {
        const int a = (q0 + t) / l2, b = (q0 + t) - a * l2;
        *gptr_w(out + (size_t)a + (size_t)l1 * (b + (size_t)l2 * c3)) = v;
    };
    if (split && J <= GRAM_SPL) {
        constexpr int U = 32, L3 = 16;                     // (l3 <= 16: gram_split)
        const int t = tid % GRAM_CH_SPLIT, c = tid / GRAM_CH_SPLIT;
        const float* p = d.PW + (size_t)min(c, J - 1) * nt2 * L12 + q0 + min(t, qn - 1);
        float w[L3], sum = 0.f;
#pragma unroll
        for (int i = 0; i < L3; ++i) w[i] = (m3 && i < l3) ? *gptr(m3 + (size_t)i * J + min(c, J - 1)) : 0.f;
        for (int t0 = 0; t0 < nt2; t0 += U) {
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = *gptr(p + (size_t)min(t0 + u, nt2 - 1) * L12);
#pragma unroll
            for (int u = 0; u < U; ++u) sum += t0 + u < nt2 ? v[u] : 0.f;
        }
        if (!m3) {
            if (c < J && t < qn) put(t, c, sum);
            return;
        }
        // channel c's share of value i of pair t: Q[c][i][t], added in the order of the channels
#pragma unroll
        for (int i = 0; i < L3; ++i)
            if (i < l3) Q[(c * L3 + i) * GRAM_CH_SPLIT + t] = w[i] * sum;
        __syncthreads();
        for (int e = tid; e < l3 * GRAM_CH_SPLIT; e += 256) {
            const int te = e % GRAM_CH_SPLIT, i = e / GRAM_CH_SPLIT;
            float v = 0.f;
            for (int k = 0; k < J; ++k) v += Q[(k * L3 + i) * GRAM_CH_SPLIT + te];
            if (te < qn) put(te, i, v);
        }
        return;
    }
    finish_sketches<1>(d, q0, qn, split, d.PW, m3, -1, s, nullptr, nullptr, -1, nullptr, Q);
    __syncthreads();
    for (int e = tid; e < qn * l3; e += 256) put(e / l3, e % l3, s[e]);
}

hipError_t launch_gram(const Desc* d, const int* starts, int count, int total_tiles, int mode, int j, hipStream_t s,
                       int unsketched) {
    if (unsketched)
        hipLaunchKernelGGL(k_gram<true>, dim3(total_tiles), dim3(256), 0, s, d, starts, count, mode, j);
    else
        hipLaunchKernelGGL(k_gram<false>, dim3(total_tiles), dim3(256), 0, s, d, starts, count, mode, j);
    return hipGetLastError();
}

hipError_t launch_sketch_out(const Desc* d, int tiles, float* out, hipStream_t s) {
    hipLaunchKernelGGL(k_sketch_out, dim3(tiles), dim3(256), 0, s, d, out);
    return hipGetLastError();
}

}  // namespace rtg

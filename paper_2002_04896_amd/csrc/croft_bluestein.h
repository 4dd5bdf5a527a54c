// croft_bluestein.h -- lengths with a prime factor above 5 (Bluestein 1970)
// on register groups (included by the kernel translation units only).
//
// With c[j] = exp(-pi i j^2 / n),
//   X[k] = c[k] sum_j (x[j] c[j]) conj(c[k - j]),
// a circular convolution of length m (a power of two >= 2n - 1) done as
// m-point FFTs: forward FFT of the chirped, zero-padded line, product with
// the kernel's DFT (precomputed, divided by m), then the inverse FFT as
// swap(DFT(swap(.))) and the final chirp.  Both FFTs run the grouped stages of
// croft_group.h: the chirp, the padding and the product happen on the
// registers that feed or leave a group, so a line goes through LDS once inside
// each FFT and once between them.
#pragma once

#include "croft_group.h"

namespace croft {
namespace dev {

// LDS: the exchange area and, with TAB, the twiddles of the grouped stages and
// the chirp (n <= M/2 values); the line maxima.
template <class G, bool TAB>
struct BlueLds {
    static constexpr int M = G::plan.n;
    static constexpr size_t kLineBytes = G::groups.K > 1 ? G::kX : 0;
    // between the FFTs the whole line is exchanged, also where one group does each
    static constexpr size_t kCB = G::kCB;
    static constexpr size_t kMid = G::groups.K > 1 ? (size_t)M * G::L * (kCB / (G::kSplit ? 2 : 1)) : 0;
    static constexpr size_t kTw = ((kLineBytes > kMid ? kLineBytes : kMid) + 15) / 16 * 16;
    static constexpr size_t kChirp = kTw + (TAB ? (size_t)G::kTwN * kCB : 0);
    static constexpr size_t kRed = kChirp + (TAB ? (size_t)(M / 2) * kCB : 0);
    static constexpr size_t kBytes = kRed + 4 * (size_t)G::L;
};

template <class Cfg, class St, int KIND, bool TAB>
__global__ void __launch_bounds__(Cfg::kBlock, 2) fft_bluestein(const PassArgs a) {
    using R = typename St::R;
    using Lay = BlueLds<Cfg, TAB>;
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int M = Cfg::plan.n, T = Cfg::T, L = Cfg::L, K = Cfg::groups.K;
    constexpr int G0 = Cfg::size(0), NB0 = M / G0, B0 = (NB0 + T - 1) / T;
    constexpr int GK = Cfg::size(K - 1), NBK = M / GK, BK = (NBK + T - 1) / T;
    static_assert((M & (M - 1)) == 0 && NB0 % T == 0 && NBK % T == 0, "power-of-two groups: no idle threads");
    constexpr int H0 = G0 / 2;  // positions j + m NB0 with m >= G0 / 2 are padding
    const int n = a.n;
    // the twiddles in the stages' order and the chirp, from LDS or (long lines,
    // few to a block: each entry would be copied for one or two uses) from
    // global memory
    const cx<R> *W = reinterpret_cast<const cx<R> *>(a.tw);
    const cx<R> *ch = reinterpret_cast<const cx<R> *>(a.chirp);
    const cx<R> *tws = TAB ? reinterpret_cast<const cx<R> *>(smem + Lay::kTw) : W;
    const cx<R> *chs = TAB ? reinterpret_cast<const cx<R> *>(smem + Lay::kChirp) : ch;
    unsigned *red = reinterpret_cast<unsigned *>(smem + Lay::kRed);
    const cx<R> *bh = reinterpret_cast<const cx<R> *>(a.bhat);
    const bool inv = a.inverse != 0;
    const int tid = threadIdx.x;
    const int l = KIND == kContiguous ? tid / T : tid % L;
    const int t = KIND == kContiguous ? tid % T : tid / L;
    // strided tiles in the XCD-contiguous order: rows narrower than a
    // 128-byte line, or off its boundaries, meet their line in one L2
    const long long tile = KIND == kContiguous ? (long long)blockIdx.x : xcd_tile(blockIdx.x, gridDim.x);
    const long long q = (KIND == kContiguous ? tile : tile % a.ntiles) * L + l;
    const long long w = KIND == kContiguous ? 0 : tile / a.ntiles;
    const bool valid = q < (KIND == kContiguous ? a.nlines : a.es);
    const long long es = KIND == kContiguous ? 1 : a.es;
    const long long base = KIND == kContiguous ? q * n : q + w * a.es * n;
    unsigned ebase = 0;
    if constexpr (St::kHalf) ebase = exp_line_index(a.em, q, w, a.em.a0, a.em.a1, a.em.a2);
    // the line, every load of the thread in flight (past its end: its last element)
    typename St::Raw raw[B0 * H0];
    int ex[St::kHalf ? B0 * H0 : 1];
    if (valid) {
#pragma unroll
        for (int b = 0; b < B0; ++b)
#pragma unroll
            for (int m = 0; m < H0; ++m) {
                const int p = t + b * T + m * NB0;
                const int e = p < n ? p : n - 1;
                raw[b * H0 + m] = St::fetch(a.in, base + es * e);
                if constexpr (St::kHalf) ex[b * H0 + m] = a.in_exp ? (int)a.in_exp[ebase + a.em.a3 * e] : 0;
            }
    }
    if constexpr (TAB) {
        cx<R> *twl = reinterpret_cast<cx<R> *>(smem + Lay::kTw), *chl = reinterpret_cast<cx<R> *>(smem + Lay::kChirp);
        for (int i = tid; i < Cfg::kTwN; i += Cfg::kBlock) twl[i] = W[i];
        for (int i = tid; i < n; i += Cfg::kBlock) chl[i] = ch[i];
    }
    if constexpr (St::kHalf)
        if (tid < L) red[tid] = 0u;
    if constexpr (TAB || St::kHalf) __syncthreads();
    // chirped, zero-padded to M
    cx<R> v[B0 * G0];
#pragma unroll
    for (int b = 0; b < B0; ++b)
#pragma unroll
        for (int m = 0; m < G0; ++m) {
            const int p = t + b * T + m * NB0;
            cx<R> x = {R(0), R(0)};
            if (m < H0) {
                const int i = b * H0 + (m < H0 ? m : 0);
                if (valid && p < n) x = cmul(swap_if(inv, St::decode(raw[i], St::kHalf ? ex[i] : 0)), chs[p]);
            }
            v[b * G0 + m] = x;
            if constexpr (B0 * G0 >= 64) {
                if (m % 8 == 7) __builtin_amdgcn_sched_barrier(0);
            }
        }
    // the longest lines run one block to a CU or two: the kernel's DFT is
    // fetched while the first FFT runs (16 x 4093 x 16: 49.9 -> 43.4 us a call)
    constexpr bool kEarly = M >= 8192;
    cx<R> hat[kEarly ? BK * GK : 1];
    if constexpr (kEarly) {
#pragma unroll
        for (int i = 0; i < BK * GK; ++i) hat[i] = bh[t + (i / GK) * T + (i % GK) * NBK];
    }
    cx<R> y[BK * GK];
    run_groups<Cfg, KIND, 0, R>(smem, tws, l, t, v, y);
    // product with the kernel's DFT, swapped: the next forward FFT then gives
    // the unnormalised inverse once swapped back
#pragma unroll
    for (int b = 0; b < BK; ++b)
#pragma unroll
        for (int m = 0; m < GK; ++m) {
            const cx<R> p = cmul(y[b * GK + m], kEarly ? hat[kEarly ? b * GK + m : 0] : bh[t + b * T + m * NBK]);
            y[b * GK + m] = {p.y, p.x};
            if constexpr (BK * GK >= 64) {
                if ((b * GK + m) % 8 == 7) __builtin_amdgcn_sched_barrier(0);
            }
        }
    if constexpr (K > 1) {
        natural_exchange<Cfg, KIND, R>(smem, l, t, y, v);
    } else {
#pragma unroll
        for (int i = 0; i < B0 * G0; ++i) v[i] = y[i];
    }
    // an opaque zero: the second FFT reads its twiddles and the chirp from LDS
    // again, rather than holding the first one's in registers until here
    const int z = opaque_zero();
    run_groups<Cfg, KIND, 0, R>(smem, tws + z, l, t, v, y);
    // X[k] = c[k] swap(o[k]), k < n <= M/2: outputs t + b T + m NBK with m < GK / 2
    constexpr int HK = GK / 2;
    float mx = 0.0f;
#pragma unroll
    for (int b = 0; b < BK; ++b)
#pragma unroll
        for (int m = 0; m < HK; ++m) {
            const int p = t + b * T + m * NBK;
            cx<R> &o = y[b * GK + m];
            if (p < n) {
                o = cmul(cx<R>{o.y, o.x}, chs[p + z]);
                if constexpr (St::kHalf) mx = fmaxf(mx, fmaxf(fabsf(o.x), fabsf(o.y)));
            }
        }
    int oex = 0;
    if constexpr (St::kHalf) {
        atomicMax(&red[l], __float_as_uint(mx));
        __syncthreads();
        oex = line_exponent(__uint_as_float(red[l]));
        if (valid && t == 0 && a.out_exp)
            a.out_exp[exp_line_index(a.em, q, w, a.em.b0, a.em.b1, a.em.b2)] = (int8_t)oex;
    }
    if (valid) {
#pragma unroll
        for (int b = 0; b < BK; ++b)
#pragma unroll
            for (int m = 0; m < HK; ++m) {
                const int p = t + b * T + m * NBK;
                if (p < n) St::store(a.out, base + es * p, swap_if(inv, y[b * GK + m]), oex);
            }
    }
}

}  // namespace dev
}  // namespace croft

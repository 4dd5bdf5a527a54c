// croft_group.h -- one axis pass with several Stockham stages per register
// group (included by the kernel translation units only).
//
// A run of consecutive stages with radices r_0 .. r_g (product G) and span
// Ns before it takes elements j + m N/G (m < G) to elements
// (j div Ns) Ns G + (j mod Ns) + Ns m, for every j < N/G: the stages of a
// group mix only those G elements, so one thread runs them in registers and
// the line goes through LDS once per group instead of once per stage.
// Inside a group, the stage after radices of product P sees P sub-lines: sub-
// line s has butterfly index j mod Ns + Ns s, and its butterflies read
// m' + q G/(P r), the thread's own registers.  The butterflies, twiddles and
// their order are those of the stage-by-stage kernels (fft_static,
// fft_generic), so the results are the same bits.
#pragma once

#include <vector>

#include "croft_device.h"

namespace croft {
namespace dev {

// How the stages of a length are cut into groups, and the threads per line.
struct GroupPlan {
    int K = 0;                 // groups
    int first[kMaxStages + 1] = {};  // group g runs stages first[g] .. first[g + 1] - 1
    int T = 1;                 // threads per line
    int E = 0;                 // registers (complex) a thread holds at most
};

constexpr int group_size(const RPlan &p, int a, int b) {
    int g = 1;
    for (int i = a; i < b; ++i) g *= p.r[i];
    return g;
}

// The cut with the fewest groups whose threads hold at most emax elements
// (the fewest trips through LDS); among those the cut and thread count with
// the least idle work (threads times butterflies rounded up), then the most
// threads.
constexpr GroupPlan make_groups(const RPlan &p, int emax) {
    GroupPlan best;
    long long best_cost = -1;
    for (int k = 1; k <= p.S && best_cost < 0; ++k) {
        for (int mask = 0; mask < (1 << (p.S - 1)); ++mask) {
            int ones = 0;
            for (int i = 0; i < p.S - 1; ++i) ones += (mask >> i) & 1;
            if (ones != k - 1) continue;
            GroupPlan g;
            g.K = k;
            int at = 0;
            for (int i = 0; i < p.S; ++i)
                if (i == 0 || ((mask >> (i - 1)) & 1)) g.first[at++] = i;
            g.first[k] = p.S;
            // a thread count pays only where it is the least for some group's
            // number of rounds
            for (int c = 0; c < k; ++c) {
                const int sc = group_size(p, g.first[c], g.first[c + 1]);
                for (int rounds = 1; rounds * sc <= emax; ++rounds) {
                    const int t = (p.n / sc + rounds - 1) / rounds;
                    int e = 0;
                    long long cost = 0;
                    for (int i = 0; i < k; ++i) {
                        const int s = group_size(p, g.first[i], g.first[i + 1]);
                        const int held = ((p.n / s + t - 1) / t) * s;
                        e = held > e ? held : e;
                        cost += (long long)held * t;
                    }
                    if (e > emax) continue;
                    if (best_cost < 0 || cost < best_cost || (cost == best_cost && t > best.T)) {
                        best_cost = cost;
                        best = g;
                        best.T = t;
                        best.E = e;
                    }
                }
            }
        }
    }
    return best;
}

// Launch shape: L lines per block, T threads per line, at most EMAX elements
// held by a thread.  One block per tile (the kernel does not loop): several
// small blocks on a CU overlap one tile's loads with another's stages.
template <int N, int KIND, int LREQ, int EMAX, int COMPUTE_BYTES, int SPLIT, int NT = 0, int TREQ = 0>
struct GCfg {
    static constexpr int kCB = COMPUTE_BYTES;
    static constexpr bool kNT = NT != 0;
    static constexpr RPlan plan = make_rplan(N);
    static constexpr GroupPlan groups = make_groups(plan, EMAX);
    static_assert(groups.K >= 1, "the length has a cut");
    static constexpr int T = TREQ > 0 ? TREQ : groups.T;
    static constexpr int L = LREQ;
    static constexpr int kBlock = T * L;
    // lines never straddle a wavefront: exchanges sync per wave, not per block
    static constexpr bool kWaveSync = KIND == kContiguous && T <= 64 && 64 % T == 0;
    static constexpr bool kSplit = SPLIT != 0;   // the real parts, then the imaginary parts, through LDS
    static constexpr int kTwN = tw_offset(plan, plan.S);
    static constexpr int size(int g) { return group_size(plan, groups.first[g], groups.first[g + 1]); }
    // first exchange: a row of padding after every G elements where G, the
    // first group's size, is even: neighbouring threads write G rows apart and
    // would meet in a bank (later groups' writes are consecutive)
    static constexpr int kPad = size(0) % 2 == 0 ? size(0) : 0;
    static constexpr int kLine = groups.K > 1 ? N + (kPad ? N / kPad : 0) : 0;
    static constexpr size_t kX = (size_t)kLine * L * (COMPUTE_BYTES / (kSplit ? 2 : 1));
    static constexpr size_t kTw = (kX + 15) / 16 * 16;
    static constexpr size_t kRed = kTw + (size_t)kTwN * COMPUTE_BYTES;
    static constexpr size_t kLds = kRed + 4 * (size_t)L;
};

template <typename R>
__device__ __forceinline__ cx<R> swap_if(bool inv, cx<R> v) {
    return {inv ? v.y : v.x, inv ? v.x : v.y};
}

// Stages S .. SEND - 1 of a group on v[NSUB][G] (G elements of each of NSUB
// sub-lines): the group's first stage has span NS0, k = j mod NS0.
template <int N, int S, int SEND, int NS0, int NSUB, int G, typename R>
__device__ __forceinline__ void group_stages(cx<R> *v, const cx<R> *tws, int k) {
    if constexpr (S < SEND) {
        constexpr RPlan P = make_rplan(N);
        constexpr int RAD = P.r[S];
        constexpr int H = G / RAD;
        constexpr int Ns = NS0 * NSUB;
        constexpr int kTw = tw_offset(P, S);
        cx<R> w[NSUB * G];
#pragma unroll
        for (int s = 0; s < NSUB; ++s) {
#pragma unroll
            for (int m = 0; m < H; ++m) {
                cx<R> u[RAD];
#pragma unroll
                for (int q = 0; q < RAD; ++q) {
                    u[q] = v[s * G + m + q * H];
                    if constexpr (Ns > 1) {
                        if (q > 0) u[q] = cmul(u[q], tws[kTw + (q - 1) * Ns + NS0 * s + k]);
                    }
                }
                Dft<RAD, R>::run(u);
#pragma unroll
                for (int q = 0; q < RAD; ++q) w[(s + NSUB * q) * H + m] = u[q];
                // keep the next butterflies' twiddle reads below this one:
                // bounds the registers live beside a large group
                if constexpr (NSUB * G >= 64) __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int i = 0; i < NSUB * G; ++i) v[i] = w[i];
        group_stages<N, S + 1, SEND, NS0, NSUB * RAD, H, R>(v, tws, k);
    }
}

template <class Cfg, int KIND>
__device__ __forceinline__ int group_lds(int l, int r) {
    return KIND == kContiguous ? l * Cfg::kLine + r : r * Cfg::L + l;
}

// Exchange after group GI: v[B][G] of group GI into x[BN][GN], the inputs of
// group GI + 1.
template <class Cfg, int KIND, int GI, typename R>
__device__ __forceinline__ void group_exchange(unsigned char *smem, int l, int t, const cx<R> *v, cx<R> *x) {
    constexpr int N = Cfg::plan.n, T = Cfg::T;
    constexpr int G = Cfg::size(GI), NB = N / G, B = (NB + T - 1) / T;
    constexpr int Ns = ns_before(Cfg::plan, Cfg::groups.first[GI]);
    constexpr int GN = Cfg::size(GI + 1), NBN = N / GN, BN = (NBN + T - 1) / T;
    // with padding element e sits at row e + e / G: outputs j G + m at
    // j (G + 1) + m, inputs j + m NBN (NBN a multiple of G) at
    // j + j / G + m (NBN + NBN / G)
    constexpr bool kPadded = GI == 0 && Cfg::kPad > 0;
    constexpr int kStep = kPadded ? NBN + NBN / G : NBN;
    static_assert(!kPadded || (Ns == 1 && NBN % G == 0), "padding follows the first group's outputs");
    constexpr int kParts = Cfg::kSplit ? 2 : 1;
#pragma unroll
    for (int part = 0; part < kParts; ++part) {
        stage_sync<Cfg::kWaveSync>();  // the previous readers of the area are done
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int j = t + b * T;
            if ((NB % T) == 0 || j < NB) {
                const int o = kPadded ? j * (G + 1) : (j / Ns) * Ns * G + j % Ns;
#pragma unroll
                for (int m = 0; m < G; ++m) {
                    const int i = group_lds<Cfg, KIND>(l, o + Ns * m);
                    if constexpr (Cfg::kSplit)
                        reinterpret_cast<R *>(smem)[i] = part ? v[b * G + m].y : v[b * G + m].x;
                    else
                        reinterpret_cast<cx<R> *>(smem)[i] = v[b * G + m];
                }
            }
        }
        stage_sync<Cfg::kWaveSync>();
#pragma unroll
        for (int b = 0; b < BN; ++b) {
            const int j = t + b * T;
            if ((NBN % T) == 0 || j < NBN) {
                const int r = kPadded ? j + j / G : j;
#pragma unroll
                for (int m = 0; m < GN; ++m) {
                    const int i = group_lds<Cfg, KIND>(l, r + m * kStep);
                    if constexpr (Cfg::kSplit) {
                        const R e = reinterpret_cast<const R *>(smem)[i];
                        if (part) x[b * GN + m].y = e;
                        else x[b * GN + m].x = e;
                    } else {
                        x[b * GN + m] = reinterpret_cast<const cx<R> *>(smem)[i];
                    }
                }
            }
        }
    }
}

// Group GI on its inputs v, and the groups after it; the last one's outputs
// (element j + NS m of butterfly j in out[b G + m]) are left in `out`.
template <class Cfg, int KIND, int GI, typename R>
__device__ __forceinline__ void run_groups(unsigned char *smem, const cx<R> *tws, int l, int t, cx<R> *v, cx<R> *out) {
    constexpr int N = Cfg::plan.n, T = Cfg::T;
    constexpr int G = Cfg::size(GI), NB = N / G, B = (NB + T - 1) / T;
    constexpr int NS0 = ns_before(Cfg::plan, Cfg::groups.first[GI]);
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const int j = t + b * T;
        if ((NB % T) == 0 || j < NB)
            group_stages<N, Cfg::groups.first[GI], Cfg::groups.first[GI + 1], NS0, 1, G, R>(v + b * G, tws, NS0 > 1 ? j % NS0 : 0);
    }
    if constexpr (GI + 1 == Cfg::groups.K) {
#pragma unroll
        for (int i = 0; i < B * G; ++i) out[i] = v[i];
    } else {
        constexpr int GN = Cfg::size(GI + 1), BN = (N / GN + T - 1) / T;
        cx<R> x[BN * GN];
        group_exchange<Cfg, KIND, GI, R>(smem, l, t, v, x);
        run_groups<Cfg, KIND, GI + 1, R>(smem, tws, l, t, x, out);
    }
}

// A line in natural order across its threads (element t + b T + m N/GK of the
// last group's outputs in y[b GK + m]) to the inputs of the first group,
// v[b G0 + m] = element t + b T + m N/G0.
template <class Cfg, int KIND, typename R>
__device__ __forceinline__ void natural_exchange(unsigned char *smem, int l, int t, const cx<R> *y, cx<R> *v) {
    constexpr int N = Cfg::plan.n, T = Cfg::T, K = Cfg::groups.K;
    constexpr int G0 = Cfg::size(0), NB0 = N / G0, B0 = (NB0 + T - 1) / T;
    constexpr int GK = Cfg::size(K - 1), NBK = N / GK, BK = (NBK + T - 1) / T;
    constexpr int kParts = Cfg::kSplit ? 2 : 1;
    static_assert(K > 1, "one group holds the whole line");
#pragma unroll
    for (int part = 0; part < kParts; ++part) {
        stage_sync<Cfg::kWaveSync>();
#pragma unroll
        for (int b = 0; b < BK; ++b) {
            if ((NBK % T) == 0 || t + b * T < NBK) {
#pragma unroll
                for (int m = 0; m < GK; ++m) {
                    const int i = group_lds<Cfg, KIND>(l, t + b * T + m * NBK);
                    if constexpr (Cfg::kSplit) reinterpret_cast<R *>(smem)[i] = part ? y[b * GK + m].y : y[b * GK + m].x;
                    else reinterpret_cast<cx<R> *>(smem)[i] = y[b * GK + m];
                }
            }
        }
        stage_sync<Cfg::kWaveSync>();
#pragma unroll
        for (int b = 0; b < B0; ++b) {
            if ((NB0 % T) == 0 || t + b * T < NB0) {
#pragma unroll
                for (int m = 0; m < G0; ++m) {
                    const int i = group_lds<Cfg, KIND>(l, t + b * T + m * NB0);
                    if constexpr (Cfg::kSplit) {
                        const R e = reinterpret_cast<const R *>(smem)[i];
                        if (part) v[b * G0 + m].y = e;
                        else v[b * G0 + m].x = e;
                    } else {
                        v[b * G0 + m] = reinterpret_cast<const cx<R> *>(smem)[i];
                    }
                }
            }
        }
    }
}

// One kernel serves both directions (swap(DFT(swap x)) by a uniform flag: two
// selects per access in a pass that waits for memory).
template <class Cfg, class St, int KIND>
__global__ void __launch_bounds__(Cfg::kBlock) fft_group(const PassArgs a) {
    using R = typename St::R;
    using Raw = typename St::Raw;
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int N = Cfg::plan.n, T = Cfg::T, L = Cfg::L, K = Cfg::groups.K;
    constexpr int G0 = Cfg::size(0), NB0 = N / G0, B0 = (NB0 + T - 1) / T;
    constexpr int GK = Cfg::size(K - 1), NBK = N / GK, BK = (NBK + T - 1) / T;
    cx<R> *tws = reinterpret_cast<cx<R> *>(smem + Cfg::kTw);
    unsigned *red = reinterpret_cast<unsigned *>(smem + Cfg::kRed);
    const bool inv = a.inverse != 0;
    const int tid = threadIdx.x;
    const int l = KIND == kContiguous ? tid / T : tid % L;
    const int t = KIND == kContiguous ? tid % T : tid / L;
    const long long es = KIND == kContiguous ? 1 : a.es;
    const long long tile = a.xcd_order ? xcd_tile(blockIdx.x, gridDim.x) : (long long)blockIdx.x;
    const long long tx = KIND == kContiguous ? tile : tile % a.ntiles;
    const long long w = KIND == kContiguous ? 0 : tile / a.ntiles;
    const long long q = tx * L + l;
    const bool valid = q < (KIND == kContiguous ? a.nlines : a.es);
    const long long tbase = KIND == kContiguous ? tx * L * N : tx * L + w * es * N;
    const unsigned lane = (unsigned)(((KIND == kContiguous ? (long long)l * N : (long long)l) + (long long)t * es) *
                                     (long long)sizeof(Raw));
    // every load of the thread in flight before the first is used
    Raw raw[B0 * G0];
    int ex[(St::kHalf && KIND != kContiguous) ? B0 * G0 : 1];
    int lex = 0;
    if (valid) {
        unsigned elane = 0;
        long long ea3 = 0;
        const int8_t *ep = &kZeroExponent;
        if constexpr (St::kHalf) {
            if (a.in_exp) {
                const ExpMap &m = a.em;
                ep = a.in_exp;
                ea3 = m.a3;
                elane = exp_line_index(m, q, w, m.a0, m.a1, m.a2) + (unsigned)ea3 * (unsigned)t;
            }
        }
        gchar *const ib = uniform_gptr(a.in, tbase * (long long)sizeof(Raw));
        gchar *const eb = uniform_gptr(ep, 0);
        if constexpr (kLineScaled<St, KIND>) lex = *(const __attribute__((address_space(1))) int8_t *)(eb + elane);
#pragma unroll
        for (int b = 0; b < B0; ++b) {
            if ((NB0 % T) == 0 || t + b * T < NB0) {
                const unsigned lr = lane_reg(lane);
#pragma unroll
                for (int m = 0; m < G0; ++m) {
                    const long long pos = b * T + m * NB0;  // uniform part of the position
                    raw[b * G0 + m] = fetch_at<St, Cfg::kNT, false>(ib, pos * es, lr);
                    if constexpr (St::kHalf && KIND != kContiguous)
                        ex[b * G0 + m] = *(const __attribute__((address_space(1))) int8_t *)(eb + ea3 * pos + elane);
                }
            }
        }
    }
    if constexpr (Cfg::kTwN > 0) {
        const cx<R> *W = reinterpret_cast<const cx<R> *>(a.tw);
        for (int i = tid; i < Cfg::kTwN; i += Cfg::kBlock) tws[i] = W[i];
    }
    if constexpr (St::kHalf && T > 1) {
        if (tid < L) red[tid] = 0u;
    }
    if constexpr (Cfg::kTwN > 0 || (St::kHalf && T > 1)) __syncthreads();
    cx<R> v[B0 * G0];
#pragma unroll
    for (int i = 0; i < B0 * G0; ++i) {
        if constexpr (kLineScaled<St, KIND>) v[i] = swap_if(inv, St::decode_raw(raw[i]));
        else v[i] = swap_if(inv, St::decode(raw[i], St::kHalf ? ex[i] : 0));
    }
    cx<R> y[BK * GK];
    run_groups<Cfg, KIND, 0, R>(smem, tws, l, t, v, y);
    int oex = 0;
    if constexpr (St::kHalf) {
        float mx = 0.0f;
#pragma unroll
        for (int b = 0; b < BK; ++b)
            if ((NBK % T) == 0 || t + b * T < NBK) {
#pragma unroll
                for (int m = 0; m < GK; ++m) mx = fmaxf(mx, fmaxf(fabsf(y[b * GK + m].x), fabsf(y[b * GK + m].y)));
            }
        if constexpr (T > 1) {
            atomicMax(&red[l], __float_as_uint(mx));
            __syncthreads();
            mx = __uint_as_float(red[l]);
        }
        oex = kLineScaled<St, KIND> ? line_exponent_scaled(mx, lex) : line_exponent(mx);
        if (valid && t == 0 && a.out_exp) {
            const ExpMap &m = a.em;
            a.out_exp[exp_line_index(m, q, w, m.b0, m.b1, m.b2)] = (int8_t)oex;
        }
        if constexpr (kLineScaled<St, KIND>) oex -= lex;
    }
    if (valid) {
        gchar *const ob = uniform_gptr(a.out, tbase * (long long)sizeof(Raw));
#pragma unroll
        for (int b = 0; b < BK; ++b) {
            if ((NBK % T) == 0 || t + b * T < NBK) {
                const unsigned lr = lane_reg(lane);
#pragma unroll
                for (int m = 0; m < GK; ++m)
                    store_at<St, Cfg::kNT, false>(ob, (long long)(b * T + m * NBK) * es, lr,
                                               swap_if(inv, y[b * GK + m]), oex);
            }
        }
    }
}

// The fused forward FFT / multiply / inverse FFT pass of a convolution plan
// (fft_conv_z: the same product, weights and energy terms) on the grouped
// stages: the product happens on the registers the forward FFT leaves, which
// one exchange brings to the inverse FFT's first group.  One block per tile,
// one energy partial per block, summed over the block in a fixed order.
template <class Cfg, class St>
__global__ void __launch_bounds__(Cfg::kBlock) fft_group_conv(const PassArgs a) {
    using R = typename St::R;
    using Raw = typename St::Raw;
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int N = Cfg::plan.n, T = Cfg::T, L = Cfg::L, K = Cfg::groups.K;
    constexpr int G0 = Cfg::size(0), NB0 = N / G0, B0 = (NB0 + T - 1) / T;
    constexpr int GK = Cfg::size(K - 1), NBK = N / GK, BK = (NBK + T - 1) / T;
    cx<R> *tws = reinterpret_cast<cx<R> *>(smem + Cfg::kTw);
    const int tid = threadIdx.x;
    const int l = tid % L;
    const int t = tid / L;
    const long long es = a.es;
    const long long tile = a.xcd_order ? xcd_tile(blockIdx.x, gridDim.x) : (long long)blockIdx.x;
    const long long tx = tile % a.ntiles, w = tile / a.ntiles;
    const long long q = tx * L + l;
    const bool valid = q < es;
    const long long tbase = tx * L + w * es * N;
    const unsigned lane = (unsigned)(((long long)l + (long long)t * es) * (long long)sizeof(Raw));
    const unsigned glane = lane / 2;  // the multiplier: one real per element
    // the line and its multiplier, every load of the thread in flight
    Raw raw[B0 * G0];
    R g[BK * GK];
    if (valid) {
        gchar *const ib = uniform_gptr(a.in, tbase * (long long)sizeof(Raw));
        gchar *const gb = uniform_gptr(a.mul, tbase * (long long)sizeof(R));
#pragma unroll
        for (int b = 0; b < B0; ++b) {
            if ((NB0 % T) == 0 || t + b * T < NB0) {
                const unsigned lr = lane_reg(lane);
#pragma unroll
                for (int m = 0; m < G0; ++m)
                    raw[b * G0 + m] = fetch_at<St, false, false>(ib, (long long)(b * T + m * NB0) * es, lr);
            }
        }
#pragma unroll
        for (int b = 0; b < BK; ++b) {
            if ((NBK % T) == 0 || t + b * T < NBK) {
                const unsigned lr = lane_reg(glane);
#pragma unroll
                for (int m = 0; m < GK; ++m)
                    g[b * GK + m] = *(const __attribute__((address_space(1))) R *)(
                        gb + (long long)(b * T + m * NBK) * es * (long long)sizeof(R) + lr);
            }
        }
    }
    {
        const cx<R> *W = reinterpret_cast<const cx<R> *>(a.tw);
        for (int i = tid; i < Cfg::kTwN; i += Cfg::kBlock) tws[i] = W[i];
        __syncthreads();
    }
    cx<R> v[B0 * G0], y[BK * GK];
#pragma unroll
    for (int i = 0; i < B0 * G0; ++i) v[i] = St::decode(raw[i], 0);
    run_groups<Cfg, kStrided, 0, R>(smem, tws, l, t, v, y);
    double acc = 0.0;
    if (valid) {
        const long long kx = q % a.hx;
        const double wgt = (kx == 0 || kx == a.hx - 1) ? 1.0 : 2.0;
#pragma unroll
        for (int b = 0; b < BK; ++b) {
            if ((NBK % T) == 0 || t + b * T < NBK) {
#pragma unroll
                for (int m = 0; m < GK; ++m) {
                    cx<R> &o = y[b * GK + m];
                    const R gv = g[b * GK + m];
                    const double m2 = (double)o.x * o.x + (double)o.y * o.y;
                    acc = fma(wgt * (double)gv, m2, acc);
                    o = cx<R>{o.y * gv, o.x * gv};  // the product, swapped for the inverse
                }
            }
        }
    }
    natural_exchange<Cfg, kStrided, R>(smem, l, t, y, v);
    run_groups<Cfg, kStrided, 0, R>(smem, tws + opaque_zero(), l, t, v, y);
    if (valid) {
        gchar *const ob = uniform_gptr(a.out, tbase * (long long)sizeof(Raw));
#pragma unroll
        for (int b = 0; b < BK; ++b) {
            if ((NBK % T) == 0 || t + b * T < NBK) {
                const unsigned lr = lane_reg(lane);
#pragma unroll
                for (int m = 0; m < GK; ++m)
                    store_at<St, false, false>(ob, (long long)(b * T + m * NBK) * es, lr,
                                               cx<R>{y[b * GK + m].y, y[b * GK + m].x}, 0);
            }
        }
    }
    // the block's sum: a butterfly over each wavefront, then its wavefronts in
    // order.  A block need not be whole wavefronts (40 threads at 75 points
    // complex128): what a shuffle returns from a lane past its end is undefined
    // and stays out of the sum.
#pragma unroll
    for (int h = 32; h > 0; h /= 2) {
        const double peer = __shfl_xor(acc, h, 64);
        if (butterfly_peer_exists(Cfg::kBlock, tid, h)) acc += peer;
    }
    double *sum = reinterpret_cast<double *>(smem);
    __syncthreads();  // the exchange area is free
    if ((tid & 63) == 0) sum[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) {
        double s = sum[0];
        for (int i = 1; i < (Cfg::kBlock + 63) / 64; ++i) s += sum[i];
        a.partial[blockIdx.x] = s;
    }
}

// Elements a thread holds at short lengths (FP32 and FP64): 10, or the largest
// radix, or 16 where that saves a trip through LDS.  Few registers let more
// blocks share a CU (complex64 fused pass at 150 points, 16 / 10 elements:
// 28 / 25 us, 200 39 / 34; 180, where 16 saves a trip, 27 / 32).
constexpr int short_elements(int n) {
    const RPlan p = make_rplan(n);
    const int e = p.rmax > 10 ? p.rmax : 10;
    return e < 16 && make_groups(p, 16).K < make_groups(p, e).K ? 16 : e;
}

// The shape of a pass by length and storage.  What bounds these passes is how
// many loads a CU keeps in flight and the LDS trips between them, so the rule
// takes rows of one 128-byte line (64 bytes for 16-bit storage above 480,
// where wider tiles leave one block per CU), few registers, and the exchange
// in two halves (kSplit) where a tile would take more than 48 KiB of LDS.
// Strided, 0.8 GB moved (rows of 360 elements / of 36000; us, the
// stage-by-stage tile before, on its best grid): complex64 360 166/129
// (196/146), 480 172/116 (196/136), 576 188/148 (197/168), 720 171/89
// (258/145), 864 172/107 (239/162), 1000 217/145 (218/171); complex128 576
// 153/138 (236/219), 720 164/182 (258/298), 864 167/211 (229/307); FP16 40
// 149/151 (229/155), 144 178/162 (407/350), 256 181/161 (263/209), 480
// 176/150, 720 221/164 (506/414), 768 281/211 (304/249).
template <int N, int KIND, int STORE_BYTES, int COMPUTE_BYTES>
struct GroupShape {
    static constexpr bool kStridedPass = KIND != kContiguous;
    static constexpr int L = kStridedPass ? (STORE_BYTES == 16 ? 8 : STORE_BYTES == 8 ? 16 : N <= 64 ? 64 : N <= 480 ? 32 : 16)
                                          : (STORE_BYTES == 4 ? (N <= 256 ? 16 : 8) : 4);
    // strided complex64: 48 elements where 32 would cost a third trip through LDS and
    // 48 does not idle most of the block (720 and 810 do: 45 x 16, 45 x 18);
    // 64 at 960 (15 x 64: 202/137 us against 230/154 with three trips)
    // contiguous 16-bit storage above 256: 32 elements where that takes two
    // trips (400 205 -> 182 us), else 16 (960 284 -> 198)
    static constexpr int E = !kStridedPass ? (STORE_BYTES == 4 && N > 256 && make_groups(make_rplan(N), 32).K <= 2 ? 32 : 16)
                             : STORE_BYTES == 4  ? (N <= 180 ? 16 : 32)
                             : N <= 256          ? short_elements(N)
                             : STORE_BYTES == 16 ? 20
                             : N == 960          ? 64
                             : (N == 576 || N == 640 || N >= 900) ? 48
                                                                  : 32;
    static constexpr int kSplit = (long long)N * L * COMPUTE_BYTES > 48 * 1024 ? 1 : 0;
};

template <int N, class St, int SB, int DT, int KIND, int NT = 0>
Entry make_group_entry(int cand) {
    constexpr int CB = (int)sizeof(cx<typename St::R>);
    using S = GroupShape<N, KIND, SB, CB>;
    using Cfg = GCfg<N, KIND, S::L, S::E, CB, S::kSplit, NT>;
    static_assert(Cfg::kBlock <= 1024, "block too large");
    static_assert(Cfg::kLds <= 160 * 1024, "LDS beyond the 160 KiB of a gfx950 workgroup");
    Entry e;
    e.n = N;
    e.kind = KIND;
    e.dtype = DT;
    e.cand = cand;
    e.func[0] = e.func[1] = reinterpret_cast<const void *>(&fft_group<Cfg, St, KIND>);
    e.T = Cfg::T;
    e.L = Cfg::L;
    e.block = Cfg::kBlock;
    e.lds = Cfg::kLds;
    e.plan = Cfg::plan;
    e.one_tile = true;
    return e;
}

// The fused multiply pass of length N in tiles of L lines, at most E elements
// held by a thread.
template <int N, class St, int SB, int DT, int L, int E>
Entry make_group_conv_entry(int cand) {
    constexpr int CB = (int)sizeof(cx<typename St::R>);
    using Cfg = GCfg<N, kStrided, L, E, CB, ((long long)N * L * CB > 48 * 1024 ? 1 : 0)>;
    static_assert(Cfg::kBlock <= 1024, "block too large");
    static_assert(Cfg::kLds <= 160 * 1024, "LDS beyond the 160 KiB of a gfx950 workgroup");
    static_assert(Cfg::kX >= 16 * sizeof(double), "wavefront sums fit the exchange area");
    Entry e;
    e.n = N;
    e.kind = kConvZ;
    e.dtype = DT;
    e.cand = cand;
    e.func[0] = e.func[1] = reinterpret_cast<const void *>(&fft_group_conv<Cfg, St>);
    e.T = Cfg::T;
    e.L = Cfg::L;
    e.block = Cfg::kBlock;
    e.lds = Cfg::kLds;
    e.plan = Cfg::plan;
    e.one_tile = true;
    return e;
}

// The 2^a 3^b 5^c lengths up to 1024 that fft_group runs as strided passes,
// for every storage (long lines), and for 16-bit storage also the short ones.
// FP32 and FP64 storage keep fft_static there where rows are whole 128-byte
// lines (complex64, 150 points, rows of 360 and 36000: 151/149 us against
// 173/159) and take fft_group, in its tile order, where they are not
// (CROFT_GROUP_PARTIAL: 97 elements a row, 25 MB: 162 points 18.6 -> 10.3 us,
// 240 22.8 -> 13.7; complex128 180 28.4 -> 17.9).
#define CROFT_GROUP_LONG(X)                                                                                        \
    X(243) X(250) X(270) X(288) X(300) X(320) X(324) X(360) X(375) X(400) X(405) X(432) X(450) X(480) X(486) X(500) \
    X(540) X(576) X(600) X(625) X(640) X(648) X(675) X(720) X(729) X(750) X(768) X(800) X(810) X(864) X(900) X(960) \
    X(972) X(1000)
#define CROFT_GROUP_SHORT(X)                                                                                       \
    X(18) X(20) X(24) X(25) X(27) X(30) X(36) X(40) X(45) X(50) X(54) X(75) X(81) X(90) X(108) X(125) X(135)         \
    X(144) X(150) X(162) X(180) X(216) X(225)

#define CROFT_GROUP_PARTIAL(X)                                                                                     \
    X(48) X(54) X(60) X(64) X(72) X(75) X(80) X(81) X(90) X(96) X(100) X(108) X(120) X(125) X(135) X(144) X(150)     \
    X(160) X(162) X(180) X(192) X(200) X(216) X(225) X(240)

}  // namespace dev
}  // namespace croft

// semi_walk.hip -- the semi-Markov CRF by walks over the segment potentials themselves.  The
// vector holds the K*C states s = r*C + c of the expanded chain (c the label of the segment in
// progress, r the steps it still has to run; semimarkov.hip), but a step reads only the K*C^2
// segment potentials that start there, not the (K*C)^2 entries of the expanded edge:
//   a_{t+1}[(j, r)] = sum_i a_t[(i, 0)] exp(sp[t, r, i, j]) + a_t[(j, r + 1)],
// where a segment that would run past the end is left out, and the same in the max semiring.
// One workgroup walks a whole sequence in one direction.
//
// Log semiring: k_semi_walk walks linear float32 vectors both ways (the range and the scaling of
// recur.h); k_semi_wide walks the sequences that leave that range again, in float64 logarithms;
// k_semi_form forms the marginals from either.  Max semiring: float64 scores, backpointers in
// LDS, and the path decoded by the same workgroup.
//
// Bound: E dependent steps of two barriers each, about 0.5 us up to 16 labels, 0.8 up to 32, 2 up
// to 64 and 3 above (the max semiring 0.8, 1 and 4.5); the potentials, read once per direction,
// stay far below the rate of HBM.  B = 32, N = 25, K = 5, C = 20, against the recursions over the
// expanded chain (30 MB of expanded edges written, read and gathered, 100 x 100 tiles of which 80
// rows hold one entry each): log Z 24 us (58), marginals 35 (94), Viterbi 28 (58).  With every
// sequence outside the linear range: log Z 99 (281 to 988), marginals 112 (375 to 1045).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device.h"
#include "internal.h"
#include "recur.h"

namespace tsc {
namespace {

constexpr int kMaxStates = 256;

struct SemiArgs {
    const float* sp;
    const int32_t* lengths;
    int64_t B, N;
    int K, C;
    // log semiring
    SemiWalk w;
    float* logZ;        // [B] or nullptr
    float* marg;        // [B, E, K, C, C] or nullptr: log Z only
    // max semiring
    int32_t* path;      // [B, N]
    int32_t* seglen;    // [B, E]
    float* score;       // [B]
};

// Layout of a step over NW waves: wave w takes the rows (previous labels) i = w + NW q, q < R,
// and its lane l the columns (states) s = l + 64 m, m < CP.  Rows and columns past the end read
// the last ones and are given no weight.  kDepth steps' potentials are in flight.
template <int CP, int R, int NW>
struct Step {
    static constexpr int kCP = CP, kR = R, kNW = NW, kT = NW * 64;
    static constexpr int kDepth = NW == 16 ? 1 : R * CP <= 8 ? 4 : R * CP <= 16 ? 2 : 1;
    const float* base;
    int C, NS, w, lane;
    int off[CP], row[R];
    __device__ Step(const SemiArgs& a, int b) {
        C = a.C;
        NS = a.K * C;
        w = uniform((int)(threadIdx.x >> 6));
        lane = threadIdx.x & 63;
        base = a.sp + (size_t)b * (a.N - 1) * NS * C;
#pragma unroll
        for (int m = 0; m < CP; ++m) {
            const int s = min(lane + 64 * m, NS - 1);
            off[m] = s / C * C * C + s % C;
        }
#pragma unroll
        for (int q = 0; q < R; ++q) row[q] = min(w + NW * q, C - 1) * C;
    }
    __device__ bool has_row(int q) const { return w + NW * q < C; }
    __device__ void load(float (&x)[R][CP], int t) const {
        const float* e = base + (size_t)t * NS * C;
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
            for (int m = 0; m < CP; ++m) x[q][m] = (e + row[q])[off[m]];
    }
    // Whether a segment may start at step t in the state of column m: the state exists, and the
    // segment, of s / C + 1 steps, ends inside the sequence
    __device__ bool open(int m, int t, int Eb) const {
        const int s = lane + 64 * m;
        return s < NS && s < (Eb - t) * C;
    }
    // Calls step(x, u) for u = 0 .. Eb - 1 with the potentials of step at(u), loaded kDepth
    // steps before
    template <class At, class Fn>
    __device__ void walk(int Eb, At&& at, Fn&& step) const {
        float x[kDepth][R][CP];
#pragma unroll
        for (int d = 0; d < kDepth; ++d) load(x[d], at(min(d, Eb - 1)));
        int u = 0;
        for (; u + kDepth <= Eb; u += kDepth) {
#pragma unroll
            for (int d = 0; d < kDepth; ++d) {
                step(x[d], u + d);
                load(x[d], at(min(u + d + kDepth, Eb - 1)));
            }
        }
#pragma unroll
        for (int d = 0; d < kDepth; ++d)
            if (u + d < Eb) step(x[d], u + d);
    }
};

__device__ __forceinline__ bool out_of_range(float v) {
    return v != 0.f && !(v >= kRecLow && v <= 0x1p60f);
}

// Workgroups [0, B) walk forward, the others (marginals only) backward
template <class F>
__global__ __launch_bounds__(F::kT) void k_semi_walk(SemiArgs a) {
    __shared__ float vec[2][kMaxStates], part[F::kNW][kMaxStates], tops[2][4];
    constexpr int CP = F::kCP, R = F::kR, NW = F::kNW;
    const bool back = blockIdx.x >= (unsigned)a.B;
    const int b = (int)blockIdx.x - (back ? (int)a.B : 0), tid = threadIdx.x;
    const int Eb = uniform((int)clamp_len(a.lengths, b, a.N)) - 1;
    if (Eb == 0) {
        if (tid == 0) a.w.bad[blockIdx.x] = 0;
        if (tid == 0 && !back && a.logZ) a.logZ[b] = logf((float)a.C);
        return;
    }
    const F st(a, b);
    const int C = st.C, NS = st.NS;
    unsigned big = 0;
    bool bad = false;
    if (!back) {
        float* al = a.marg ? a.w.alpha + (size_t)b * a.N * NS : nullptr;
        int32_t* cx = a.marg ? a.w.cx + (size_t)b * a.N : nullptr;
        // no segment is in progress at the start
        if (tid < NS) {
            vec[0][tid] = tid < C ? 1.f : 0.f;
            if (al) al[tid] = tid < C ? 1.f : 0.f;
        }
        if (tid < 4) tops[0][tid] = 1.f;
        if (tid == 0 && cx) cx[0] = 0;
        int c = 0;
        __syncthreads();
        st.walk(Eb, [](int u) { return u; }, [&](const float (&x)[R][CP], int t) {
            const int cur = t & 1, nxt = cur ^ 1;
            float acc[CP] = {};
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const float v = st.has_row(q) ? vec[cur][st.w + NW * q] : 0.f;
#pragma unroll
                for (int m = 0; m < CP; ++m) {
                    const float y = st.open(m, t, Eb) ? x[q][m] : -INFINITY;
                    big = max(big, fin_bits(y));
                    acc[m] = fmaf(v, edge_exp(y), acc[m]);
                }
            }
#pragma unroll
            for (int m = 0; m < CP; ++m) part[st.w][st.lane + 64 * m] = acc[m];
            const int ex = exponent_of(fmaxf(fmaxf(tops[cur][0], tops[cur][1]), fmaxf(tops[cur][2], tops[cur][3])));
            c += ex;
            __syncthreads();
            float v = 0.f;
            if (tid < NS) {
                float s = tid + C < NS ? vec[cur][tid + C] : 0.f;   // the segments that run on
#pragma unroll
                for (int g = 0; g < NW; ++g) s += part[g][tid];
                v = ldexpf(s, -ex);
                bad |= out_of_range(v);
                vec[nxt][tid] = v;
                if (al) al[(size_t)(t + 1) * NS + tid] = v;
            }
            if (tid < kMaxStates) {
                const float top = wave_max_fast(v);
                if (st.lane == 0) tops[nxt][st.w] = top;
            }
            if (tid == 0 && cx) cx[t + 1] = c;
            __syncthreads();
        });
        bad = __syncthreads_or(bad || big > kRecPotBits);
        if (tid >= 64) return;
        double s = 0.0;
        for (int i = tid; i < C; i += 64) s += vec[Eb & 1][i];
        s = wave_sum_d(s);
        if (tid == 0) {
            a.w.bad[b] = bad;
            if (a.logZ) a.logZ[b] = (float)((log2(s) + c) * 0.6931471805599453);
        }
        return;
    }
    float* be = a.w.beta + (size_t)b * a.N * NS;
    // no segment is in progress after the last step (columns past NS stay 0)
    if (tid < kMaxStates) {
        vec[0][tid] = tid < C ? 1.f : 0.f;
        vec[1][tid] = 0.f;
    }
    if (tid < NS) be[(size_t)Eb * NS + tid] = tid < C ? 1.f : 0.f;
    __syncthreads();
    st.walk(Eb, [&](int u) { return Eb - 1 - u; }, [&](const float (&x)[R][CP], int u) {
        const int t = Eb - 1 - u, cur = u & 1, nxt = cur ^ 1;
        float bv[CP], top = 0.f;
#pragma unroll
        for (int m = 0; m < CP; ++m) {
            bv[m] = vec[cur][st.lane + 64 * m];
            top = fmaxf(top, bv[m]);
        }
        const int ex = exponent_of(wave_max_fast(top));
        float sum[R] = {};
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
            for (int m = 0; m < CP; ++m) {
                const float y = st.open(m, t, Eb) ? x[q][m] : -INFINITY;
                big = max(big, fin_bits(y));
                sum[q] = fmaf(ldexpf(bv[m], -ex), edge_exp(y), sum[q]);
            }
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const float v = wave_sum_fast(sum[q]);
            if (st.has_row(q)) {
                bad |= out_of_range(v);
                if (st.lane == 0) {
                    vec[nxt][st.w + NW * q] = v;
                    be[(size_t)t * NS + st.w + NW * q] = v;
                }
            }
        }
        if (tid >= C && tid < NS) {   // the segments that run on
            const float v = ldexpf(vec[cur][tid - C], -ex);
            bad |= out_of_range(v);
            vec[nxt][tid] = v;
            be[(size_t)t * NS + tid] = v;
        }
        __syncthreads();
    });
    bad = __syncthreads_or(bad || big > kRecPotBits);
    if (tid == 0) a.w.bad[blockIdx.x] = bad;
}

__device__ __forceinline__ bool left_over(const SemiArgs& a, int b) {
    return uniform((a.w.bad[b] | (a.marg ? a.w.bad[a.B + b] : 0)) != 0);
}

// The walks of the sequences that left k_semi_walk's range, in float64 logarithms.  Rare, so
// simple: four threads share a column going forward, a wave takes a row going backward.
__global__ __launch_bounds__(1024) void k_semi_wide(SemiArgs a) {
    __shared__ double vec[2][kMaxStates], pm[4][kMaxStates], ps[4][kMaxStates];
    const bool back = blockIdx.x >= (unsigned)a.B;
    const int b = (int)blockIdx.x - (back ? (int)a.B : 0), tid = threadIdx.x;
    if (!left_over(a, b)) return;
    const int Eb = (int)clamp_len(a.lengths, b, a.N) - 1, C = a.C, NS = a.K * C;
    const float* base = a.sp + (size_t)b * (a.N - 1) * NS * C;
    double* out = back ? a.w.beta64 : a.w.alpha64;
    if (out) out += (size_t)b * a.N * NS;
    if (tid < NS) {
        vec[0][tid] = tid < C ? 0.0 : -INFINITY;
        if (out) out[(size_t)(back ? Eb : 0) * NS + tid] = vec[0][tid];
    }
    __syncthreads();
    for (int u = 0; u < Eb; ++u) {
        const int t = back ? Eb - 1 - u : u, cur = u & 1, nxt = cur ^ 1;
        const float* e = base + (size_t)t * NS * C;
        const int lim = min(NS, (Eb - t) * C);   // the states in which a segment may start
        if (back) {
            for (int i = tid >> 6; i < C; i += 16) {
                double m = -INFINITY, s = 0.0, y[kMaxStates / 64];
#pragma unroll
                for (int q = 0; q < kMaxStates / 64; ++q) {
                    const int st = (tid & 63) + 64 * q;
                    y[q] = st < lim ? vec[cur][st] + (double)e[(st / C * C + i) * C + st % C] : -INFINITY;
                    m = fmax(m, y[q]);
                }
                m = safe_shift_d(wave_max_d(m));
#pragma unroll
                for (int q = 0; q < kMaxStates / 64; ++q) s += exp(y[q] - m);
                s = wave_sum_d(s);
                if ((tid & 63) == 0) vec[nxt][i] = m + log(s);
            }
            if (tid >= C && tid < NS) vec[nxt][tid] = vec[cur][tid - C];
        } else {
            const int st = tid & (kMaxStates - 1), g = tid / kMaxStates;
            double m = -INFINITY, s = 0.0;
            if (st < lim) {
                const float* col = e + st / C * C * C + st % C;
                for (int i = g; i < C; i += 4) m = fmax(m, vec[cur][i] + (double)col[i * C]);
                m = safe_shift_d(m);
                for (int i = g; i < C; i += 4) s += exp(vec[cur][i] + (double)col[i * C] - m);
            }
            pm[g][st] = s > 0.0 ? m : -INFINITY;
            ps[g][st] = s;
            __syncthreads();
            if (tid < NS) {
                const double on = tid + C < NS ? vec[cur][tid + C] : -INFINITY;
                const double top = safe_shift_d(
                    fmax(fmax(fmax(pm[0][tid], pm[1][tid]), fmax(pm[2][tid], pm[3][tid])), on));
                double v = exp(on - top);
#pragma unroll
                for (int h = 0; h < 4; ++h) v += ps[h][tid] * exp(pm[h][tid] - top);
                vec[nxt][tid] = top + log(v);
            }
        }
        __syncthreads();
        if (out && tid < NS) out[(size_t)(back ? t : t + 1) * NS + tid] = vec[nxt][tid];
    }
    if (back || tid >= 64) return;
    double m = -INFINITY, s = 0.0;
    for (int i = tid; i < C; i += 64) m = fmax(m, vec[Eb & 1][i]);
    m = safe_shift_d(wave_max_d(m));
    for (int i = tid; i < C; i += 64) s += exp(vec[Eb & 1][i] - m);
    s = wave_sum_d(s);
    if (tid == 0) {
        if (a.logZ) a.logZ[b] = (float)(m + log(s));
        if (a.marg) a.w.lz[b] = m + log(s);
    }
}

// The marginals of one step per workgroup.  magic: 2^32 / C rounded up (quotients of numbers
// below K C^2 <= 2^15 come out exactly).
__global__ __launch_bounds__(256) void k_semi_form(SemiArgs a, unsigned magic) {
    const int E = (int)a.N - 1, C = a.C, NS = a.K * C, n = NS * C, tid = threadIdx.x, lane = tid & 63;
    const int b = (int)(blockIdx.x / (unsigned)E), t = (int)blockIdx.x - b * E;
    const int Eb = (int)clamp_len(a.lengths, b, a.N) - 1;
    const float* sp = a.sp + (size_t)blockIdx.x * n;
    float* out = a.marg + (size_t)blockIdx.x * n;
    if (t >= Eb) {
        for (int e = tid; e < n; e += 256) out[e] = 0.f;
        return;
    }
    const size_t at = ((size_t)b * a.N + t) * NS;
    const int lim = (Eb - t) * C;   // states past it: a segment that would run past the end
    if (left_over(a, b)) {
        const double lz = a.w.lz[b];
        const double* a0 = a.w.alpha64 + at;
        const double* b1 = a.w.beta64 + at + NS;
        for (int e = tid; e < n; e += 256) {
            const int ki = e / C, s = ki / C * C + (e - ki * C);
            // (log Z = -inf: no segmentation is allowed, and every marginal is 0)
            const double y = a0[ki % C] + (double)sp[e] + b1[s] - lz;
            out[e] = s < lim && lz != -INFINITY ? (float)exp(y) : 0.f;
        }
        return;
    }
    __shared__ float al[kMaxStates], be[kMaxStates];
    const float* a0 = a.w.alpha + at;
    const float* a1 = a0 + NS;
    const float* b1 = a.w.beta + at + NS;
    // a_{t+1} carries dc binary places more than a_t; both are weighed against their product
    // with b_{t+1}, scaled by its largest entry, which every wave forms for itself
    const int dc = a.w.cx[(size_t)b * a.N + t + 1] - a.w.cx[(size_t)b * a.N + t];
    float y[4], z[4], m = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int s = lane + 64 * u;
        y[u] = s < NS ? a1[s] : 0.f;
        z[u] = s < NS ? b1[s] : 0.f;
        m = fmaxf(m, z[u]);
    }
    const int ex = exponent_of(wave_max_fast(m));
    float d = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        z[u] = ldexpf(z[u], -ex);
        d = fmaf(y[u], z[u], d);
    }
    d = wave_sum_fast(d);
    const float inv = d > 0.f ? ldexpf(1.f / d, -dc) : 0.f;
    if (tid < 64) {
#pragma unroll
        for (int u = 0; u < 4; ++u) be[lane + 64 * u] = lane + 64 * u < lim ? z[u] : 0.f;
    }
    if (tid < C) al[tid] = a0[tid] * inv;
    __syncthreads();
    for (int e = tid; e < n; e += 256) {   // e = (k C + i) C + j
        const int ki = C > 1 ? (int)__umulhi((unsigned)e, magic) : e, j = e - ki * C;
        const int k = C > 1 ? (int)__umulhi((unsigned)ki, magic) : ki, i = ki - k * C;
        const float w = be[k * C + j];
        // (a state without weight may hold any potential, also one past the exponential's range)
        out[e] = w == 0.f ? 0.f : edge_exp(sp[e]) * w * al[i];
    }
}

// Max semiring: forward scores, then the path, its segment lengths and its score
template <class F>
__global__ __launch_bounds__(F::kT) void k_semi_max(SemiArgs a) {
    __shared__ double vec[2][kMaxStates], part[F::kNW][kMaxStates];
    __shared__ uint8_t arg[F::kNW][kMaxStates];
    extern __shared__ uint8_t bp[];   // [Eb][NS], then the states of the path [Eb + 1]
    constexpr int CP = F::kCP, R = F::kR, NW = F::kNW;
    const int b = (int)blockIdx.x, tid = threadIdx.x, C = a.C, NS = a.K * C, E = (int)a.N - 1;
    const int Eb = uniform((int)clamp_len(a.lengths, b, a.N)) - 1;
    int32_t* path = a.path + (size_t)b * a.N;
    int32_t* seglen = a.seglen + (size_t)b * E;
    for (int n = tid; n <= E; n += F::kT)
        if (n > Eb) {
            path[n] = -1;
            seglen[n - 1] = -1;
        }
    if (Eb == 0) {
        if (tid == 0) {
            path[0] = 0;
            a.score[b] = 0.f;
        }
        return;
    }
    const F st(a, b);
    if (tid < kMaxStates) vec[0][tid] = tid < C ? 0.0 : -INFINITY;
    __syncthreads();
    st.walk(Eb, [](int u) { return u; }, [&](const float (&x)[R][CP], int t) {
        const int cur = t & 1, nxt = cur ^ 1;
        double best[CP];
        int from[CP];
#pragma unroll
        for (int m = 0; m < CP; ++m) { best[m] = -INFINITY; from[m] = st.w; }
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const double v = st.has_row(q) ? vec[cur][st.w + NW * q] : -INFINITY;
#pragma unroll
            for (int m = 0; m < CP; ++m) {
                const double y = v + (double)x[q][m];
                const bool up = y > best[m];   // ties keep the lower row
                best[m] = up ? y : best[m];
                from[m] = up ? st.w + NW * q : from[m];
            }
        }
#pragma unroll
        for (int m = 0; m < CP; ++m) {
            part[st.w][st.lane + 64 * m] = best[m];
            arg[st.w][st.lane + 64 * m] = (uint8_t)from[m];
        }
        __syncthreads();
        if (tid < NS) {
            // the best segment that starts here (the lowest previous label among equals, label
            // 0 where none is allowed), or the one in progress where that is better
            double v = -INFINITY;
            int i = 0;
            if (tid < (Eb - t) * C) {
#pragma unroll
                for (int g = 0; g < NW; ++g) {
                    const double o = part[g][tid];
                    const int oi = arg[g][tid];
                    const bool up = o > v || (o == v && o != -INFINITY && oi < i);
                    v = up ? o : v;
                    i = up ? oi : i;
                }
            }
            const double on = tid + C < NS ? vec[cur][tid + C] : -INFINITY;
            const bool runs = on > v;
            vec[nxt][tid] = runs ? on : v;
            bp[t * NS + tid] = (uint8_t)(runs ? tid + C : i);
        }
        __syncthreads();
    });
    if (tid < 64) {
        // the lowest of the best last labels (no segment is in progress there)
        double best = -INFINITY;
        int z = C;
        for (int i = tid; i < C; i += 64)
            if (vec[Eb & 1][i] > best || z == C) { best = vec[Eb & 1][i]; z = i; }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double ov = __shfl_xor(best, o, kWave);
            const int oi = __shfl_xor(z, o, kWave);
            if (oi < C && (z == C || ov > best || (ov == best && oi < z))) { best = ov; z = oi; }
        }
        if (tid == 0) {
            a.score[b] = (float)best;
            uint8_t* states = bp + Eb * NS;
            int s = z;
            states[Eb] = (uint8_t)s;
            for (int t = Eb - 1; t >= 0; --t) {
                s = bp[t * NS + s];
                states[t] = (uint8_t)s;
            }
        }
    }
    __syncthreads();
    const uint8_t* states = bp + Eb * NS;
    for (int n = tid; n <= Eb; n += F::kT) {
        const int s = states[n];
        path[n] = s % C;
        if (n < Eb) seglen[n] = s < C ? states[n + 1] / C + 1 : 0;
    }
}

template <class T>
struct Type { using type = T; };

// Calls fn with the layout for C labels and K C states: eight waves of up to 8 rows, sixteen
// above 64 labels
template <class Fn>
hipError_t with_step(int K, int C, Fn&& fn) {
    auto rows = [&](auto cp) {
        constexpr int CP = decltype(cp)::value;
        if (C <= 16) return fn(Type<Step<CP, 2, 8>>{});
        if (C <= 32) return fn(Type<Step<CP, 4, 8>>{});
        if (C <= 64) return fn(Type<Step<CP, 8, 8>>{});
        return fn(Type<Step<CP, 8, 16>>{});
    };
    switch ((K * C + 63) / 64) {
        case 1: return rows(std::integral_constant<int, 1>{});
        case 2: return rows(std::integral_constant<int, 2>{});
        case 3: return rows(std::integral_constant<int, 3>{});
        default: return rows(std::integral_constant<int, 4>{});
    }
}

}  // namespace

size_t semi_walk_bytes(int64_t B, int64_t N, int64_t KC, void* base, SemiWalk* w) {
    char* p = static_cast<char*>(base);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char* at = p ? p + off : nullptr;
        off += (bytes + 255) / 256 * 256;
        return at;
    };
    const size_t n = (size_t)B * N * KC;
    w->bad = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * 2 * B));
    w->lz = reinterpret_cast<double*>(take(sizeof(double) * B));
    w->cx = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * B * N));
    w->alpha = reinterpret_cast<float*>(take(sizeof(float) * n));
    w->beta = reinterpret_cast<float*>(take(sizeof(float) * n));
    w->alpha64 = reinterpret_cast<double*>(take(sizeof(double) * n));
    w->beta64 = reinterpret_cast<double*>(take(sizeof(double) * n));
    return off;
}

hipError_t launch_semi_walk(const SemiWalk& w, const float* sp, const int32_t* lengths, int64_t B,
                            int64_t N, int64_t K, int64_t C, float* logZ, float* marg,
                            hipStream_t s) {
    SemiArgs a{};
    a.sp = sp; a.lengths = lengths; a.B = B; a.N = N; a.K = (int)K; a.C = (int)C;
    a.w = w; a.logZ = logZ; a.marg = marg;
    if (!marg) a.w.alpha64 = a.w.beta64 = nullptr;
    const dim3 grid((unsigned)(marg ? 2 * B : B));
    hipError_t e = with_step(a.K, a.C, [&](auto f) {
        using F = typename decltype(f)::type;
        hipLaunchKernelGGL((k_semi_walk<F>), grid, dim3(F::kT), 0, s, a);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_semi_wide, grid, dim3(1024), 0, s, a);
    e = hipGetLastError();
    if (e != hipSuccess || !marg) return e;
    const unsigned magic = (unsigned)((((uint64_t)1 << 32) + C - 1) / C);
    hipLaunchKernelGGL(k_semi_form, dim3((unsigned)(B * (N - 1))), dim3(256), 0, s, a, magic);
    return hipGetLastError();
}

hipError_t launch_semi_max(const float* sp, const int32_t* lengths, int64_t B, int64_t N, int64_t K,
                           int64_t C, int32_t* path, int32_t* seglen, float* score, hipStream_t s) {
    SemiArgs a{};
    a.sp = sp; a.lengths = lengths; a.B = B; a.N = N; a.K = (int)K; a.C = (int)C;
    a.path = path; a.seglen = seglen; a.score = score;
    const size_t lds = (size_t)(N - 1) * K * C + N;
    return with_step(a.K, a.C, [&](auto f) {
        using F = typename decltype(f)::type;
        hipLaunchKernelGGL((k_semi_max<F>), dim3((unsigned)B), dim3(F::kT), lds, s, a);
        return hipGetLastError();
    });
}

}  // namespace tsc

// recur_max.hip -- Viterbi by chunked vector recursions in the max semiring (recur.h): the
// forward scores delta_{t+1}(j) = max_i delta_t(i) + l[t,i,j] in float64, with the
// backpointers of every step, C^2 work per edge (paper Sec. 5.2; the max semiring of Table 2).
#include <hip/hip_runtime.h>

#include "device.h"
#include "internal.h"
#include "recur.h"

#include <type_traits>

namespace tsc {
namespace {

struct RecMaxArgs {
    const float* pot;
    const int32_t* lengths;
    int64_t B, N;
    int C, S, K, round;
    double* delta;      // [B, E, C] scores before each edge, relative to the chunk's start
    double* vend;       // [kRecRounds + 2][B, K, C] scores after the chunk's last edge
    int32_t* chg;       // [kRecRounds][B, K]
    double* shift;      // [B, K] the start vector's maximum plus what the stored scores lack
                        // of the walk from it
    int32_t* last;      // [B, K] last position that the chunk's latest walk has rewritten
    uint8_t* bp;        // [B, E, C]
    int32_t* zlast;     // [B]
    float* score;       // [B]
    int32_t* gate;      // [B] sequences left to the tree, or nullptr: none are
    int limit;          // chunks walked in order before a sequence is left to the tree
};

// What two walks' scores of one label may differ by, beyond their offset, of the larger one's
// magnitude: each sum rounds at 2^-53 of it (float32 potentials mostly add exactly), and walks
// that have met share all but their last few sums.
constexpr double kMaxTol = 0x1p-50;

// Scores past this magnitude lose the potentials' low bits (2^-25 and below), so they depend on
// what they are relative to; such sequences are scored from their start, as one walk does.
constexpr double kMaxScore = 0x1p28;

template <class F>
struct MaxLds {
    double v[2][F::kNG][F::kCols];      // the row groups' partial maxima, by step parity
    double off[2][2][16];               // each wave's bounds of the offset
    uint8_t arg[2][F::kNG][F::kCols];   // the rows (within their group) of the maxima
};

struct WalkEnd {
    bool agreed;    // the scores met the stored ones
    int last;       // up to this position they were rewritten
    double off;     // new minus stored, at and past the meeting
};

// Walks the edges [s, e) of sequence b from the scores d (label j of the lane, see RecCfg) and
// leaves the last ones in d.  kAgain: stops where the scores agree with the stored ones past
// position `last` (or, at e, with old_end), up to one offset.
//
// Bound: one read of the edges from HBM, 4 C^2 bytes each (C = 256: 732 us for 4.29 GB, 5.9
// TB/s); the arithmetic (convert, add, maximum, compare, select per entry) takes about a third
// of that time.  The edge's tile is held in registers (64 floats per lane at C = 256), each
// reloaded with the entry of the edge kDepthMax further on as soon as it has been used: kDepthMax
// whole edges per workgroup are in flight (a step at C = 64 is shorter than the memory latency).
template <class F, bool kAgain>
__device__ WalkEnd walk(const RecMaxArgs& a, MaxLds<F>& sm, int64_t b, int s, int e, double& d,
                        const double* old_end, int last) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, C = a.C, CC = C * C;
    const int c = lane & 15, q = lane >> 4, gl = lane / F::kLPR;
    const int j = w * F::kRPW + c;                 // the label this lane merges
    const bool own = c < F::kRPW && j < C;
    const int64_t row = b * (a.N - 1) + s;
    double* dl = a.delta + (size_t)row * C + (own ? j : 0);
    uint8_t* bp = a.bp + (size_t)row * C + (own ? j : 0);
    if (own && q == 0) *dl = d;

    const unsigned voff = tile_offset<F>(C);
    const float* edge = a.pot + (size_t)row * CC;
    Tile<F> ring[F::kDepthMax];
#pragma unroll
    for (int i = 0; i < F::kDepthMax; ++i) {
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(uniform(edge), uniform(s + i < e ? CC : 0));
#pragma unroll
        for (int r = 0; r < F::kRG; ++r) {
            tile_load_row<F>(ring[i].x[r], rs, voff, r, C);
            __builtin_amdgcn_sched_barrier(0);     // in the order of use
        }
        edge += CC;
    }
    double dlo = 0.0, dhi = 0.0;                   // this wave's bounds at position t
    auto publish = [&](int buf) {
        if (lane == 0) { sm.off[buf][0][w] = dlo; sm.off[buf][1][w] = dhi; }
    };
    // Whether every wave's labels have one offset (after the barrier that follows publish).  Each
    // label bounds it by its own two scores, which are known to kMaxTol of their magnitude, and
    // the walks have met when all bounds share a point: labels that carry a large finite mask
    // say nothing about the others, and the offset is as exact as the smallest scores.
    auto agree = [&](int buf, double& off) {
        const int i = c < F::kNW ? c : 0;
        const double lo = row_max_d(sm.off[buf][0][i]), hi = -row_max_d(-sm.off[buf][1][i]);
        off = hi == INFINITY ? 0.0 : 0.5 * (lo + hi);   // (no label has a finite score)
        return uniform(lo <= hi);
    };
    double off = 0.0;
    // One step, edge t in x: returns whether the walk ends at position t (if asked to look)
    auto step = [&](Tile<F>& x, int t, auto look) {
        constexpr bool kLook = kAgain && decltype(look)::value;
        const int buf = t & 1;
        double was = 0.0;                          // the stored scores of position t + 1
        if (kAgain) was = t + 1 < e ? dl[C] : old_end[own ? j : 0];
        double dw = d;                             // lane r of each 16: row r of the lane's group
        if constexpr (F::kG > 1) dw = __shfl(d, (gl * F::kRG + c) & 15, kWave);
        // past the chunk's last edge nothing is read: a descriptor of no entries
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(uniform(edge), uniform(t + F::kDepthMax < e ? CC : 0));
        edge += CC;
        double best[F::kCB];
        int arg[F::kCB];
#pragma unroll
        for (int v = 0; v < F::kCB; ++v) { best[v] = -INFINITY; arg[v] = 0; }
#pragma unroll
        for (int r = 0; r < F::kRG; ++r) {
            double dr;
            if constexpr (F::kLPR >= 16) dr = row_bcast(dw, r);
            else dr = __shfl(d, gl * F::kRG + r, kWave);
#pragma unroll
            for (int v = 0; v < F::kCB; ++v) {
                asm volatile("" : "+v"(x.x[r][v]));   // converted here, not where it is loaded
                const double y = dr + (double)x.x[r][v];
                const bool up = y > best[v];       // ties keep the lower row
                best[v] = up ? y : best[v];
                arg[v] = up ? r : arg[v];
            }
            tile_load_row<F>(x.x[r], rs, voff, r, C);
            __builtin_amdgcn_sched_barrier(0);     // rows in order, so that one row's registers
                                                   // are free before the next is converted
        }
#pragma unroll
        for (int cp = 0; cp < F::kCP; ++cp) {
            const int col = (cp * F::kLPR + lane % F::kLPR) * F::kVec;
            double* o = &sm.v[buf][w * F::kG + gl][col];
            uint8_t* oa = &sm.arg[buf][w * F::kG + gl][col];
            if constexpr (F::kVec == 4) {
                ((double2*)o)[0] = make_double2(best[cp * 4], best[cp * 4 + 1]);
                ((double2*)o)[1] = make_double2(best[cp * 4 + 2], best[cp * 4 + 3]);
#pragma unroll
                for (int v = 0; v < 4; ++v) asm("" : "+v"(arg[cp * 4 + v]));   // packed here only
                *(uint32_t*)oa = (uint32_t)arg[cp * 4] | (uint32_t)arg[cp * 4 + 1] << 8 |
                                 (uint32_t)arg[cp * 4 + 2] << 16 | (uint32_t)arg[cp * 4 + 3] << 24;
            } else {
                *o = best[cp];
                *oa = (uint8_t)arg[cp];
            }
        }
        if (kLook) publish(buf);
        __syncthreads();
        // position t agrees: the rest of the chunk stands as it is
        if (kLook && t > last && agree(buf, off)) return true;
        // merge the groups' partial maxima of label j: ascending groups, ties to the lower
        constexpr int kPer = F::kNG / 4;
        double y[kPer];
        int ya[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            y[u] = sm.v[buf][q * kPer + u][own ? j : 0];
            ya[u] = sm.arg[buf][q * kPer + u][own ? j : 0] + (q * kPer + u) * F::kRG;
        }
        double m = y[0];
        int mi = ya[0];
#pragma unroll
        for (int u = 1; u < kPer; ++u) {
            const bool up = y[u] > m;
            m = up ? y[u] : m;
            mi = up ? ya[u] : mi;
        }
        const PairD p16 = pair16_d(m);
        const Pair i16 = pair16((unsigned)mi);
        bool up = p16.b > p16.a;
        m = up ? p16.b : p16.a;
        mi = (int)(up ? i16.b : i16.a);
        const PairD p32 = pair32_d(m);
        const Pair i32 = pair32((unsigned)mi);
        up = p32.b > p32.a;
        m = up ? p32.b : p32.a;
        mi = (int)(up ? i32.b : i32.a);
        d = own ? m : -INFINITY;
        dl += C;
        if (own && q == 0) {
            *bp = (uint8_t)mi;
            if (t + 1 < e) *dl = d;
        }
        bp += C;
        if (kAgain) {
            // one finite and one infinite score never agree
            const bool fin = own && d != -INFINITY && was != -INFINITY;
            const bool odd = own && (d != -INFINITY) != (was != -INFINITY);
            const double df = d - was, tol = kMaxTol * fmax(fabs(d), fabs(was));
            dlo = row_max_d(odd ? INFINITY : fin ? df - tol : -INFINITY);
            dhi = -row_max_d(odd ? INFINITY : fin ? -df - tol : -INFINITY);
        }
        return false;
    };
    // (whole groups of kDepthMax steps, so that the loads in flight are counted exactly across the
    // loop; agreement is looked for once per group)
    int t = s;
    for (; t + F::kDepthMax <= e; t += F::kDepthMax) {
        if (step(ring[0], t, std::true_type{})) return {true, t, off};
#pragma unroll
        for (int i = 1; i < F::kDepthMax; ++i) step(ring[i], t + i, std::false_type{});
    }
#pragma unroll
    for (int i = 0; i + 1 < F::kDepthMax; ++i)
        if (uniform(t + i < e)) step(ring[i], t + i, std::false_type{});
    if (!kAgain) return {false, s, 0.0};
    publish(e & 1);
    __syncthreads();
    if (agree(e & 1, off)) return {true, e - 1, off};
    return {false, s, 0.0};
}

// Last label and score of sequence b from its final scores v[C] and the chunks' offsets
__device__ void finish_sequence(const RecMaxArgs& a, int64_t b, int n, const double* v) {
    if (threadIdx.x >= 64) return;
    const int lane = threadIdx.x;
    double sum = 0.0;
    for (int k = 1 + lane; k < n; k += 64) sum += a.shift[b * a.K + k];
    sum = wave_sum_d(sum);
    double best = -INFINITY;
    int arg = 0x7fffffff;
    for (int i = lane; i < a.C; i += 64)
        if (v[i] > best || arg == 0x7fffffff) { best = v[i]; arg = i; }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double ov = __shfl_xor(best, o, kWave);
        const int oi = __shfl_xor(arg, o, kWave);
        if (ov > best || (ov == best && oi < arg)) { best = ov; arg = oi; }
    }
    if (lane == 0) {
        a.zlast[b] = arg;
        a.score[b] = (float)(best + sum);
    }
}

// The first walk of every chunk: from zeros (the true start of chunk 0, a guess elsewhere).
// Consecutive workgroups take the same chunk of consecutive sequences.
template <class F>
__global__ __launch_bounds__(F::kT, F::kNW >= 8 ? 4 : 2) void k_rec_max(RecMaxArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    MaxLds<F>& sm = *(MaxLds<F>*)smem;
    const int k = uniform((int)(blockIdx.x / (unsigned)a.B)), b = (int)blockIdx.x - k * (int)a.B;
    const int Eb = uniform((int)clamp_len(a.lengths, b, a.N)) - 1;
    const int s = k * a.S, e = uniform(min(s + a.S, Eb));
    if (s >= Eb) {
        if (Eb == 0 && k == 0 && threadIdx.x == 0) { a.zlast[b] = 0; a.score[b] = 0.f; }
        return;
    }
    const int c = threadIdx.x & 15, j = (threadIdx.x >> 6) * F::kRPW + c;
    const bool own = c < F::kRPW && j < a.C;
    double d = own ? 0.0 : -INFINITY;
    walk<F, false>(a, sm, b, s, e, d, nullptr, s);
    const int64_t bk = (int64_t)b * a.K + k;
    if (own && (threadIdx.x & 48) == 0) a.vend[(size_t)bk * a.C + j] = d;
    if (threadIdx.x == 0) { a.shift[bk] = 0.0; a.last[bk] = s; }
    if (a.K > 1) return;
    __syncthreads();
    finish_sequence(a, b, 1, a.vend + (size_t)bk * a.C);
}

// Walks chunk k of sequence b again from its predecessor's end scores `start`, and writes its
// own as version `ver` if they change: whether they did
template <class F>
__device__ bool walk_again(const RecMaxArgs& a, MaxLds<F>& sm, int b, int k, int Eb,
                           const double* start, const double* old_end, int ver) {
    const int64_t nbk = a.B * a.K, bk = (int64_t)b * a.K + k;
    const int lane = threadIdx.x & 63, c = lane & 15, j = (threadIdx.x >> 6) * F::kRPW + c;
    const bool own = c < F::kRPW && j < a.C;
    // relative to their maximum, so that a chunk's scores stay small
    double m = -INFINITY;
    for (int i = lane; i < a.C; i += 64) m = fmax(m, start[i]);
    m = wave_max_d(m);
    double d = own ? start[j] - safe_shift_d(m) : -INFINITY;
    const int s = k * a.S, e = uniform(min(s + a.S, Eb));
    const WalkEnd r = walk<F, true>(a, sm, b, s, e, d, old_end, a.last[bk]);
    if (!r.agreed && own && lane < 16) a.vend[((size_t)ver * nbk + bk) * a.C + j] = d;
    __syncthreads();   // (every lane has read a.last[bk])
    if (threadIdx.x == 0) {
        a.shift[bk] = m + r.off;
        // positions past `last` keep an older walk's scores; none do once the whole chunk has
        // been walked again
        a.last[bk] = r.last;
    }
    return !r.agreed;
}

// Round `round` (1 .. kRecRounds): every chunk whose predecessor's end scores are new (in round
// 1 all but the first) is walked again
template <class F>
__global__ __launch_bounds__(F::kT, F::kNW == 16 ? 4 : 2) void k_rec_max_again(RecMaxArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int k = uniform((int)(blockIdx.x / (unsigned)a.B)), b = (int)blockIdx.x - k * (int)a.B;
    const int Eb = uniform((int)clamp_len(a.lengths, b, a.N)) - 1;
    if (k * a.S >= Eb) return;
    const int64_t nbk = a.B * a.K, bk = (int64_t)b * a.K + k;
    const int ver = a.round - 1;   // the predecessor's version, if it is new
    bool changed = false;
    if (k > 0 && (ver == 0 || a.chg[(size_t)(ver - 1) * nbk + bk - 1]))
        changed = walk_again<F>(a, *(MaxLds<F>*)smem, b, k, Eb,
                                a.vend + ((size_t)ver * nbk + bk - 1) * a.C,
                                a.vend + ((size_t)latest_version(a.chg, nbk, bk, ver) * nbk + bk) * a.C,
                                a.round);
    if (threadIdx.x == 0) a.chg[(size_t)ver * nbk + bk] = changed;
}

// One workgroup per sequence: what the rounds have left is walked in order, each chunk from
// its predecessor's final end scores, or marked for the tree where that is more than a few chunks
// and the tree is faster (a.gate); then the last label and
// the score.  Usually nothing is left; a sequence whose walks never meet, or whose scores pass
// kMaxScore (masks that no path avoids), is walked whole here.
template <class F>
__global__ __launch_bounds__(F::kT, F::kNW == 16 ? 4 : 2) void k_rec_max_finish(RecMaxArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int b = blockIdx.x;
    const int Eb = uniform((int)clamp_len(a.lengths, b, a.N)) - 1;
    if (Eb == 0) {
        if (a.gate && threadIdx.x == 0) a.gate[b] = 0;
        return;
    }
    const int64_t nbk = a.B * a.K;
    const int n = (Eb + a.S - 1) / a.S;
    bool changed = false, any = false;
    int pending = 0, walked = 0;
    auto late_at = [&](int k) {
        return k < n && a.chg[(size_t)(kRecRounds - 1) * nbk + (int64_t)b * a.K + k - 1] != 0;
    };
    for (int k = 1 + threadIdx.x; k < n; k += F::kT) any |= late_at(k);
    if (__syncthreads_or(any))   // (rarely)
        for (int k0 = 1; k0 < n; k0 += F::kT) pending += __syncthreads_count(late_at(k0 + (int)threadIdx.x));
    for (int k = 1; pending > 0 && k < n; ++k) {
        const int64_t bk = (int64_t)b * a.K + k;
        const bool late = late_at(k);
        if (!uniform(changed || late)) continue;
        // (the tree writes the last label and the score, too)
        if (a.gate && (pending > a.limit || walked++ == 2 * a.limit)) {
            if (threadIdx.x == 0) a.gate[b] = 1;
            return;
        }
        changed = walk_again<F>(a, *(MaxLds<F>*)smem, b, k, Eb,
                                a.vend + ((size_t)(kRecRounds + changed) * nbk + bk - 1) * a.C,
                                a.vend + ((size_t)latest_version(a.chg, nbk, bk, kRecRounds) * nbk + bk) * a.C,
                                kRecRounds + 1);
        changed = uniform(changed);
    }
    if (a.gate && threadIdx.x == 0) a.gate[b] = 0;
    __syncthreads();
    const int64_t bk = (int64_t)b * a.K + n - 1;
    const int ver = changed ? kRecRounds + 1 : latest_version(a.chg, nbk, bk, kRecRounds);
    const double* v = a.vend + ((size_t)ver * nbk + bk) * a.C;
    auto past = [](double x) { return x != -INFINITY && fabs(x) > kMaxScore; };
    bool large = false;
    for (int k = 1 + threadIdx.x; k < n; k += F::kT) large |= past(a.shift[(int64_t)b * a.K + k]);
    double best = -INFINITY;
    for (int i = threadIdx.x & 63; i < a.C; i += 64) best = fmax(best, v[i]);
    large |= past(wave_max_d(best));
    if (!__syncthreads_or(large) || n == 1) {   // (one chunk is walked from the start anyway)
        finish_sequence(a, b, n, v);
        return;
    }
    if (a.gate) {
        if (threadIdx.x == 0) a.gate[b] = 1;
        return;
    }
    const int c = threadIdx.x & 15, j = (threadIdx.x >> 6) * F::kRPW + c;
    const bool own = c < F::kRPW && j < a.C;
    double d = own ? a.vend[(size_t)b * a.K * a.C + j] : -INFINITY;   // chunk 0's end
    walk<F, false>(a, *(MaxLds<F>*)smem, b, a.S, Eb, d, nullptr, 0);
    double* end = a.vend + (size_t)bk * a.C;
    if (own && (threadIdx.x & 48) == 0) end[j] = d;
    __syncthreads();
    finish_sequence(a, b, 1, end);
}

template <class Kernel>
hipError_t launch_walk(Kernel* kernel, size_t lds, int64_t blocks, int threads,
                       const RecMaxArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3((unsigned)threads), lds, s, a);
    return hipGetLastError();
}

template <class F>
hipError_t launch(RecMaxArgs a, hipStream_t s) {
    constexpr size_t lds = sizeof(MaxLds<F>);
    static AllowLds allow;
    hipError_t e = allow(lds, k_rec_max<F>, k_rec_max_again<F>, k_rec_max_finish<F>);
    if (e != hipSuccess) return e;
    e = launch_walk(k_rec_max<F>, lds, a.B * a.K, F::kT, a, s);
    if (a.K == 1) return e;
    for (a.round = 1; e == hipSuccess && a.round <= kRecRounds; ++a.round)
        e = launch_walk(k_rec_max_again<F>, lds, a.B * a.K, F::kT, a, s);
    return e == hipSuccess ? launch_walk(k_rec_max_finish<F>, lds, a.B, F::kT, a, s) : e;
}

}  // namespace

int rec_threads(int64_t C) {
    int threads = 0;
    (void)with_rec_cfg(C, [&](auto f) {
        threads = decltype(f)::kT;
        return hipSuccess;
    });
    return threads;
}

hipError_t launch_rec_max(const Plan& p, const float* pot, const int32_t* lengths, float* score,
                          hipStream_t s) {
    RecMaxArgs a{};
    a.pot = pot; a.lengths = lengths; a.B = p.B; a.N = p.N; a.C = (int)p.C;
    a.S = (int)p.rec_S; a.K = (int)p.rec_K;
    a.delta = p.rec_delta; a.vend = p.rec_vendd; a.chg = p.rec_chg; a.shift = p.rec_shift;
    a.last = p.rec_last; a.bp = p.bp; a.zlast = p.zlast; a.score = score; a.gate = p.gate;
    a.limit = rec_limit(p.rec_S, p.rec_K);
    return with_rec_cfg(p.C, [&](auto f) { return launch<decltype(f)>(a, s); });
}

}  // namespace tsc

// recur_log.hip -- log Z and edge marginals by chunked vector recursions in the log semiring
// (recur.h), C^2 work per edge (paper Sec. 5.1-5.2: the forward algorithm and its reverse).
//
// Messages are kept in the linear domain: alpha_t[i] = a_t[i] 2^c_t with a in float32 and the
// exponent c an exact integer, so an entry's relative precision does not depend on its size
// and no logarithm is taken before log Z.  The forward walk forms a_{t+1} = a_t E_t with
// E_t[i][j] = exp(l[t,i,j]); the backward walk b_t = E_t b_{t+1} and, from the same
// exponentials, the marginals mu_t[i][j] = a_t[i] E_t[i][j] b_{t+1}[j] / n_t, whose normaliser
// n_t = sum_ij a_t E_t b_{t+1} = 2^(c_{t+1} - c_t) a_{t+1} . b_{t+1} is known before the edge
// is read.
//
// The range this needs is checked, not assumed.  While every finite potential is at most 24
// (kRecPotBits) in magnitude and no entry that is not 0 falls below kRecLow (of a vector scaled
// by the power of two of the one before it), no product and no sum underflows or overflows:
// a 0 is then exactly a -inf log message.  A sequence that leaves this range is left to the
// tree, as is one whose walks do not meet where the tree is much faster than walking it in
// order (Plan::gate).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device.h"
#include "internal.h"
#include "recur.h"

namespace tsc {
namespace {

// Both directions walk side by side and the marginals are formed afterwards while the edges
// are few enough to be read mostly from the caches the second and third time; larger batches
// form the marginals on the backward walk, two reads in all.
constexpr size_t kRecBothBytes = (size_t)320 << 20;

struct RecLogArgs {
    const float* pot;
    float* epot;        // [B, E, C, C] the edges' exponentials, formed beforehand, or nullptr
    const int32_t* lengths;
    int64_t B, N;
    int C, S, K, round;
    // forward
    float* alpha;       // [B, E, C] a before each edge
    int32_t* cx;        // [B, E] its exponent, relative to the chunk's start
    float* vend;        // [kRecRounds + 2][B, K, C] a after the chunk's last edge
    int32_t* xend;      // [kRecRounds + 2][B, K] its exponent
    int32_t* chg;       // [kRecRounds + 1][B, K]
    double* shift;      // [B, K] what the exponents past `last` lack, to float's precision
    double* ratio;      // [B, K] the ratio whose log2 shift holds
    int32_t* last;      // [B, K] last position that the chunk's latest walk has rewritten
    int32_t* bad;       // [2][B, K] the chunk has left the range: its first walk, a later one
    // backward
    float* beta;        // [B, E, C] b before each edge (inside chunks)
    float* vbeg;        // [kRecRounds + 2][B, K, C] b before the chunk's first edge
    int32_t* chgb;      // [kRecRounds + 1][B, K]
    int32_t* badb;      // [2][B, K]
    int32_t* gateb;     // [B] what the backward walks beside the forward ones leave to the tree
    float* marg;
    float* logZ;        // [B] or nullptr
    int32_t* gate;      // [B]
    bool tree_pending;  // walks that do not meet are left to the tree, too
    int limit;          // unless they are at most this many chunks
    bool meet;          // log Z of one chunk: the two directions meet in its middle
    int32_t* xbeg;      // [B, K] exponent of the backward walk
    // log Z once more (k_rec_refine); fine is nullptr where no sequence is long enough
    int32_t* fine;      // [B] which sequences
    int32_t* count;     // [B] their chunks that are done
    double* part;       // [B, K] log2 of the chunks' growth
};

// log Z of long chains with potentials of log Z near 0 (row-normalised ones, say): each edge's float32
// arithmetic is off by up to 1e-8 on average (the hardware exponential; C = 8: 2e-9, C = 200: 1e-8),
// which adds up over the edges and passes 1e-5 of max(|log Z|, 1) past this many.
constexpr int kRefineEdges = 1000;

template <bool kPre>
__device__ __forceinline__ float exp_of(float x) {
    return kPre ? x : edge_exp(x);
}

// Edges [s, e) of chunk k of a sequence with Eb edges; with a.meet the direction's half
__device__ __forceinline__ void chunk_edges(const RecLogArgs& a, int k, int Eb, bool back, int& s, int& e) {
    s = k * a.S;
    e = uniform(min(s + a.S, Eb));
    if (a.meet && back) s = uniform(Eb / 2);
    else if (a.meet) e = uniform(Eb / 2);
}

template <class F>
struct FwdLds {
    float v[2][F::kNG][F::kCols];   // the row groups' partial sums, by step parity
    float top[2][16];               // each wave's largest entry
    float ratio[2][2][16];          // and smallest and largest ratio to the stored entries
    double sum[2][16];              // sums of its entries and of the stored ones, where they meet
};
template <class F>
struct BwdLds {
    float b[2][F::kCols];
    float top[2][16];
    float ratio[2][2][16];
};

struct WalkEnd {
    bool agreed;    // the vector met the stored one
    int last;       // up to this position it was rewritten
    int off;        // new over stored, past it: the exponents' difference and the vectors' ratio
    double ratio;
};

// Ratios of new to stored entries over a wave's labels; 0 against not 0 never agrees
struct Ratio {
    float lo = INFINITY, hi = 0.f;
};
__device__ __forceinline__ Ratio ratio_of(bool use, float now, float was) {
    Ratio r;
    if (use && (now > 0.f || was > 0.f)) {
        const bool both = now > 0.f && was > 0.f;
        const float q = now * __builtin_amdgcn_rcpf(was);
        r.lo = both ? q : 0.f;
        r.hi = both ? q : INFINITY;
    }
    return r;
}
// Whether two walks have met: their vectors differ by the rounding of their sums, some 1e-7 per
// entry, and a remainder of the guessed start within 2^-20 over all labels is no longer told from
// it.  It cannot grow (the recursions do not expand the ratio of two vectors), so a
// vector's entries are within 2^-20 of the true ones' proportions, and a marginal within twice that
// (measured against float64 for slowly and quickly mixing chains, C = 8 to 200: 4e-8 to 2e-7 in the
// 2-norm).
__device__ __forceinline__ bool same_ratio(const float (&ratio)[2][16], int c, int nw) {
    const int i = c < nw ? c : 0;
    const float lo = -row_max(-ratio[0][i]), hi = row_max(ratio[1][i]);
    return uniform(lo > hi || hi <= lo * (1.f + 0x1p-20f));   // (lo > hi: no label has an entry)
}
// The ratio of two vectors that have met, whose log2 their chunk adds to log Z: that of their sums,
// in which roundings and what remains of the guessed start cancel for the most part (in exact
// arithmetic the remainders of one constant transition matrix with 4 added to its diagonal, C = 8,
// added up to 1.5e-8 per chunk, those of independent potentials to 1e-9; the smallest or largest
// ratio would add one-sided errors of up to 2^-20).
template <class F>
__device__ __forceinline__ double sum_ratio(FwdLds<F>& sm, float now, float was) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, c = lane & 15;
    const double n = row_sum_d(now), o = row_sum_d(was);
    if (lane == 0) { sm.sum[0][w] = n; sm.sum[1][w] = o; }
    __syncthreads();
    const double sn = row_sum_d(c < F::kNW ? sm.sum[0][c] : 0.0), so = row_sum_d(c < F::kNW ? sm.sum[1][c] : 0.0);
    return sn > 0.0 && so > 0.0 ? sn / so : 1.0;
}

// ---- forward

// Walks the edges [s, e) of sequence b from the vector v (label j of the lane, see RecCfg) and
// leaves the last one in v and its exponent in x.  kAgain: stops where it agrees with the
// stored one, past position `last` (or, at e, with old_end), up to a factor.  The first walk
// looks at the potentials' magnitudes and stops early where they leave the range.
//
// Bound: one read of the edges from HBM; per entry about ten issue slots (four of them the
// exponential).  Loads as in the max semiring's walk: a tile register is reloaded with the
// entry of the edge kDepth further on once it has been used.
template <class F, bool kAgain, bool kPre>
__device__ WalkEnd walk_fwd(const RecLogArgs& a, FwdLds<F>& sm, int b, int s, int e, float& v,
                            int& x, bool& bad, const float* old_end, int old_x, int last) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, C = a.C, CC = C * C;
    const int c = lane & 15, q = lane >> 4, gl = lane / F::kLPR;
    const int j = w * F::kRPW + c;
    const bool own = c < F::kRPW && j < C;
    const int64_t row = (int64_t)b * (a.N - 1) + s;
    float* al = a.alpha + (size_t)row * C + (own ? j : 0);
    int32_t* cx = a.cx + row;
    x = 0;
    if (own && q == 0) *al = v;
    if (threadIdx.x == 0) *cx = 0;

    const unsigned voff = tile_offset<F>(C);
    const float* edge = (kPre ? a.epot : a.pot) + (size_t)row * CC;
    Tile<F> ring[F::kDepth];
#pragma unroll
    for (int i = 0; i < F::kDepth; ++i) {
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(uniform(edge), uniform(s + i < e ? CC : 0));
#pragma unroll
        for (int r = 0; r < F::kRG; ++r) {
            tile_load_row<F>(ring[i].x[r], rs, voff, r, C);
            __builtin_amdgcn_sched_barrier(0);     // in the order of use
        }
        edge += CC;
    }
    constexpr bool kRange = !kAgain && !kPre;
    unsigned big = 0;                              // largest finite magnitude read
    Ratio ra;                                      // at position t
    float vs = 0.f;                                // and the stored entry and exponent there
    int xw = 0;
    auto publish = [&](int buf) {
        if (lane == 0) { sm.ratio[buf][0][w] = ra.lo; sm.ratio[buf][1][w] = ra.hi; }
    };
    // One step, edge t in tile: returns whether the walk ends at position t (if asked to look);
    // whether position t + 1 is looked at
    auto step = [&](Tile<F>& tile, int t, auto look, auto next) {
        constexpr bool kLook = kAgain && decltype(look)::value, kNext = kAgain && decltype(next)::value;
        const int buf = t & 1;
        float was = 0.f;                           // the stored entry of position t + 1
        int xn = 0;
        if (kNext) {
            was = t + 1 < e ? al[C] : old_end[own ? j : 0];
            xn = t + 1 < e ? cx[1] : old_x;
        }
        float vw = v;                              // lane r of each 16: row r of the lane's group
        if constexpr (F::kG > 1) vw = __shfl(v, (gl * F::kRG + c) & 15, kWave);
        const float top = row_max(v);
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(uniform(edge), uniform(t + F::kDepth < e ? CC : 0));
        edge += CC;
        float acc[F::kCB];
#pragma unroll
        for (int i = 0; i < F::kCB; ++i) acc[i] = 0.f;
#pragma unroll
        for (int r = 0; r < F::kRG; ++r) {
            float vr;
            if constexpr (F::kLPR >= 16) vr = row_bcast(vw, r);
            else vr = __shfl(v, gl * F::kRG + r, kWave);
#pragma unroll
            for (int i = 0; i < F::kCB; ++i) {
                asm volatile("" : "+v"(tile.x[r][i]));   // used here, not where it is loaded
                if (kRange) big = max(big, fin_bits(tile.x[r][i]));
                acc[i] = fmaf(vr, exp_of<kPre>(tile.x[r][i]), acc[i]);
            }
            if (kRange) asm volatile("" : "+v"(big));   // (its chain of maxima kept in row order)
            tile_load_row<F>(tile.x[r], rs, voff, r, C);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int cp = 0; cp < F::kCP; ++cp) {
            float* o = &sm.v[buf][w * F::kG + gl][(cp * F::kLPR + lane % F::kLPR) * F::kVec];
            if constexpr (F::kVec == 4)
                *(float4*)o = make_float4(acc[cp * 4], acc[cp * 4 + 1], acc[cp * 4 + 2], acc[cp * 4 + 3]);
            else
                *o = acc[cp];
        }
        // (an infinite top stops every wave: the chunk has left the range)
        const bool out = !kAgain && __any(kPre ? bad : big > kRecPotBits);
        if (lane == 0) sm.top[buf][w] = out ? INFINITY : top;
        if (kLook) publish(buf);
        __syncthreads();
        if (kLook && t > last && same_ratio(sm.ratio[buf], c, F::kNW)) return true;
        const int ex = uniform(exponent_of(row_max(sm.top[buf][c < F::kNW ? c : 0])));
        if (!kAgain && ex > 127) return true;
        constexpr int kPer = F::kNG / 4;
        float y[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) y[u] = sm.v[buf][q * kPer + u][own ? j : 0];
        float m = y[0];
#pragma unroll
        for (int u = 1; u < kPer; ++u) m += y[u];
        const Pair p16 = pair16(__float_as_uint(m));
        m = __uint_as_float(p16.a) + __uint_as_float(p16.b);
        const Pair p32 = pair32(__float_as_uint(m));
        m = __uint_as_float(p32.a) + __uint_as_float(p32.b);
        v = own ? ldexpf(m, -ex) : 0.f;
        x += ex;
        bad |= v != 0.f && !(v >= kRecLow && v <= 0x1p60f);
        al += C;
        ++cx;
        if (t + 1 < e) {
            if (own && q == 0) *al = v;
            if (threadIdx.x == 0) *cx = x;
        }
        if (kNext) {
            ra = ratio_of(own, v, was);
            ra.lo = -row_max(-ra.lo);
            ra.hi = row_max(ra.hi);
            vs = was;
            xw = xn;
        }
        return false;
    };
    // (whole groups of kDepth steps, so that the loads in flight are counted exactly across the
    // loop; agreement is looked for once per group)
    int t = s, met = -1;
    for (; t + F::kDepth <= e; t += F::kDepth) {
        if (step(ring[0], t, std::true_type{}, std::bool_constant<F::kDepth == 1>{})) {
            met = t;
            if constexpr (kAgain) break;
            bad = true;
            return {true, t, 0, 1.0};
        }
#pragma unroll
        for (int i = 1; i + 1 < F::kDepth; ++i) step(ring[i], t + i, std::false_type{}, std::false_type{});
        if constexpr (F::kDepth > 1)
            step(ring[F::kDepth - 1], t + F::kDepth - 1, std::false_type{}, std::true_type{});
    }
    if (met < 0) {
#pragma unroll
        for (int i = 0; i + 1 < F::kDepth; ++i)
            if (uniform(t + i < e)) step(ring[i], t + i, std::false_type{}, std::true_type{});
        bad |= kRange && big > kRecPotBits;
        if (kAgain) {
            publish(e & 1);
            __syncthreads();
            if (same_ratio(sm.ratio[e & 1], c, F::kNW)) met = e - 1;
        }
    }
    if (!kAgain || met < 0) return {false, s, 0, 1.0};
    return {true, met, x - xw, sum_ratio(sm, v, own ? vs : 0.f)};
}

// Stores log Z (lz its log2) and marks it for k_rec_refine
__device__ __forceinline__ void set_log_z(const RecLogArgs& a, int64_t b, double lz, bool left) {
    if (!a.logZ) return;
    const double z = lz * 0.6931471805599453;
    a.logZ[b] = (float)z;
    if (!a.fine) return;
    const double edges = (double)clamp_len(a.lengths, b, a.N) - 1.0;
    a.fine[b] = !left && edges > kRefineEdges * fmax(fabs(z), 1.0);
    a.count[b] = 0;
}

// log Z of sequence b from its final vector v[C] and the chunks' exponents, and whether the
// tree has to compute it
__device__ void finish_fwd(const RecLogArgs& a, int64_t b, int n, const float* v, int ver_last,
                           bool left) {
    if (threadIdx.x >= 64) return;
    const int lane = threadIdx.x;
    const int64_t nbk = a.B * a.K;
    double sum = 0.0, tot = 0.0;
    for (int k = lane; k < n; k += 64) {
        const int64_t bk = b * a.K + k;
        const int ver = k == n - 1 ? ver_last
                        : a.K == 1 ? 0
                                   : latest_version(a.chg, nbk, bk, kRecRounds + 1);
        const double ratio = a.ratio[bk];
        sum += a.xend[(size_t)ver * nbk + bk] + (a.shift[bk] - (double)__builtin_amdgcn_logf((float)ratio)) + log2(ratio);
        left |= (a.bad[bk] | a.bad[nbk + bk]) != 0;
    }
    for (int i = lane; i < a.C; i += 64) tot += v[i];
    sum = wave_sum_d(sum);
    tot = wave_sum_d(tot);
    left = __any(left);
    if (lane == 0) {
        a.gate[b] = left;
        set_log_z(a, b, sum + log2(tot), left);
    }
}

// The first walk of a chunk: from ones (the true start of chunk 0, a guess elsewhere)
template <class F>
__device__ void first_fwd(const RecLogArgs& a, FwdLds<F>& sm, int b, int k) {
    const int Eb = uniform((int)clamp_len(a.lengths, b, a.N)) - 1;
    int s, e;
    chunk_edges(a, k, Eb, false, s, e);
    if (s >= Eb) {
        if (Eb == 0 && k == 0 && threadIdx.x == 0) {
            a.gate[b] = 0;
            if (a.logZ) a.logZ[b] = logf((float)a.C);
            if (a.fine) a.fine[b] = 0;
        }
        return;
    }
    const int c = threadIdx.x & 15, j = (threadIdx.x >> 6) * F::kRPW + c;
    const bool own = c < F::kRPW && j < a.C;
    float v = own ? 1.f : 0.f;
    int x = 0;
    bool bad = false;
    if (F::kPre && a.epot) {
        if (s < e) walk_fwd<F, false, F::kPre>(a, sm, b, s, e, v, x, bad, nullptr, 0, s);
    } else {
        if (s < e) walk_fwd<F, false, false>(a, sm, b, s, e, v, x, bad, nullptr, 0, s);
    }
    const int64_t bk = (int64_t)b * a.K + k;
    if (own && (threadIdx.x & 48) == 0) a.vend[(size_t)bk * a.C + j] = v;
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) {
        a.xend[bk] = x;
        a.shift[bk] = 0.0;
        a.ratio[bk] = 1.0;
        a.last[bk] = s;
        a.bad[bk] = bad;
        a.bad[a.B * a.K + bk] = 0;
    }
    if (a.K > 1 || a.meet) return;
    __syncthreads();
    finish_fwd(a, b, 1, a.vend + (size_t)bk * a.C, 0, false);
}

// Walks chunk k again from its predecessor's end vector `start`, and writes its own as version
// `ver` if it changes: whether it did
template <class F>
__device__ bool again_fwd(const RecLogArgs& a, FwdLds<F>& sm, int b, int k, int Eb,
                          const float* start, int old, int ver) {
    const int64_t nbk = a.B * a.K, bk = (int64_t)b * a.K + k;
    const int c = threadIdx.x & 15, j = (threadIdx.x >> 6) * F::kRPW + c;
    const bool own = c < F::kRPW && j < a.C;
    float v = own ? start[j] : 0.f;
    int x;
    bool bad = false;
    const int s = k * a.S, e = uniform(min(s + a.S, Eb));
    const size_t oi = (size_t)old * nbk + bk;
    const float* old_end = a.vend + oi * a.C;
    const WalkEnd r =
        F::kPre && a.epot ? walk_fwd<F, true, F::kPre>(a, sm, b, s, e, v, x, bad, old_end, a.xend[oi], a.last[bk])
                          : walk_fwd<F, true, false>(a, sm, b, s, e, v, x, bad, old_end, a.xend[oi], a.last[bk]);
    if (!r.agreed && own && (threadIdx.x & 48) == 0) a.vend[((size_t)ver * nbk + bk) * a.C + j] = v;
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) {
        if (!r.agreed) a.xend[(size_t)ver * nbk + bk] = x;
        a.shift[bk] = r.off + (double)__builtin_amdgcn_logf((float)r.ratio);
        a.ratio[bk] = r.ratio;
        // exponents past `last` are an older walk's; none are once the whole chunk has been
        // walked again
        a.last[bk] = r.last;
        if (bad) a.bad[nbk + bk] = 1;
    }
    return !r.agreed;
}

// Round `round` (1 .. kRecRounds): every chunk whose predecessor's end vector is new is walked
// again
template <class F>
__device__ void round_fwd(const RecLogArgs& a, FwdLds<F>& sm, int b, int k) {
    const int Eb = uniform((int)clamp_len(a.lengths, b, a.N)) - 1;
    if (k * a.S >= Eb) return;
    const int64_t nbk = a.B * a.K, bk = (int64_t)b * a.K + k;
    const int ver = a.round - 1;   // the predecessor's version, if it is new
    bool changed = false;
    // (the first walks' marks: the predecessor's workgroup may be marking a later one now)
    if (k > 0 && (ver == 0 || a.chg[(size_t)(ver - 1) * nbk + bk - 1]) && !(a.bad[bk] | a.bad[bk - 1]))
        changed = again_fwd<F>(a, sm, b, k, Eb, a.vend + ((size_t)ver * nbk + bk - 1) * a.C,
                               latest_version(a.chg, nbk, bk, ver), a.round);
    if (threadIdx.x == 0) a.chg[(size_t)ver * nbk + bk] = changed;
}

// One workgroup per sequence: what the rounds have left is walked in order (or left to the
// tree); then log Z
template <class F>
__device__ void last_fwd(const RecLogArgs& a, FwdLds<F>& sm, int b) {
    const int Eb = uniform((int)clamp_len(a.lengths, b, a.N)) - 1;
    if (Eb == 0) return;
    const int64_t nbk = a.B * a.K, b0 = (int64_t)b * a.K;
    const int n = (Eb + a.S - 1) / a.S;
    int32_t* const chg = a.chg + (size_t)kRecRounds * nbk + b0;   // this walk's own changes
    bool left = false, any = false;
    auto late_at = [&](int k) { return k > 0 && a.chg[(size_t)(kRecRounds - 1) * nbk + b0 + k - 1] != 0; };
    for (int k = threadIdx.x; k < n; k += F::kT) {
        left |= (a.bad[b0 + k] | a.bad[nbk + b0 + k]) != 0;
        any |= late_at(k);
        chg[k] = 0;
    }
    int pending = 0, walked = 0;
    if (__syncthreads_or(left || any)) {   // (rarely)
        for (int k0 = 0; k0 < n; k0 += F::kT) {
            const int k = k0 + (int)threadIdx.x;
            pending += __syncthreads_count(k < n && late_at(k));
        }
        left = __syncthreads_or(left) || (a.tree_pending && pending > a.limit);
    }
    bool changed = false;
    for (int k = 1; pending > 0 && !left && k < n; ++k) {
        const bool late = late_at(k);
        if (!uniform(changed || late)) continue;
        if (a.tree_pending && walked++ == 2 * a.limit) {
            left = true;
            break;
        }
        changed = again_fwd<F>(a, sm, b, k, Eb,
                               a.vend + ((size_t)(kRecRounds + changed) * nbk + b0 + k - 1) * a.C,
                               latest_version(a.chg, nbk, b0 + k, kRecRounds), kRecRounds + 1);
        changed = uniform(changed);
        if (threadIdx.x == 0) chg[k] = changed;
    }
    __syncthreads();
    const int ver = latest_version(a.chg, nbk, b0 + n - 1, kRecRounds + 1);
    finish_fwd(a, b, n, a.vend + ((size_t)ver * nbk + b0 + n - 1) * a.C, ver, left);
}

// ---- backward and marginals

// Sums over the kLPR lanes of a row, for the kRG rows of the lane's group: halving steps leave
// each lane with one row, `which` of its group; lanes that differ in the bits below kLow hold
// the same row
template <class F>
struct RowSums {
    static constexpr int kN = F::kRG <= 1 ? 1 : F::kRG <= 2 ? 2 : F::kRG <= 4 ? 4 : F::kRG <= 8 ? 8 : 16;
    static constexpr int kStages = kN == 1 ? 0 : kN == 2 ? 1 : kN == 4 ? 2 : kN == 8 ? 3 : 4;
    static constexpr int kTop = F::kLPR == 64 ? 5 : F::kLPR == 32 ? 4 : F::kLPR == 16 ? 3 : 2;
    static constexpr int kLow = 1 << (kTop + 1 - kStages);
    static __device__ __forceinline__ int which(int lane) {
        int r = 0;
#pragma unroll
        for (int i = 0; i < kStages; ++i) r |= ((lane >> (kTop - i)) & 1) << (kStages - 1 - i);
        return r;
    }
    // a of the lanes with bit `bit` clear plus b of those with it set, across that bit
    template <int bit>
    static __device__ __forceinline__ float merge(float a, float b, int lane) {
        if constexpr (bit == 5) {
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
            return __uint_as_float(r[0]) + __uint_as_float(r[1]);
        } else if constexpr (bit == 4) {
            const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
            return __uint_as_float(r[0]) + __uint_as_float(r[1]);
        } else {
            const bool hi = (lane >> bit) & 1;
            const float keep = hi ? b : a, send = hi ? a : b;
            return keep + shift<bit>(send);
        }
    }
    // the value of a lane across the bit (bit 2: the mirror within 8 lanes, whose lower bits
    // are summed over afterwards)
    template <int bit>
    static __device__ __forceinline__ float shift(float x) {
        const int v = __float_as_int(x);
        constexpr int ctrl = bit == 3 ? 0x128 : bit == 2 ? 0x141 : bit == 1 ? 0x4E : 0xB1;
        return __int_as_float(__builtin_amdgcn_update_dpp(v, v, ctrl, 0xF, 0xF, false));
    }
    template <int bit, int n>
    static __device__ __forceinline__ float run(float (&x)[kN], int lane) {
        if constexpr (bit < 0) {
            return x[0];
        } else if constexpr (n > 1) {
#pragma unroll
            for (int i = 0; i < n / 2; ++i) x[i] = merge<bit>(x[i], x[i + n / 2], lane);
            return run<bit - 1, n / 2>(x, lane);
        } else {
            x[0] = bit >= 4 ? merge<bit>(x[0], x[0], lane) : x[0] + shift<bit>(x[0]);
            return run<bit - 1, 1>(x, lane);
        }
    }
    static __device__ __forceinline__ float sum(const float (&rs)[F::kRG], int lane) {
        float x[kN];
#pragma unroll
        for (int i = 0; i < kN; ++i) x[i] = i < F::kRG ? rs[i] : 0.f;
        return run<kTop, kN>(x, lane);
    }
};

// What a lane needs to form marginals of chunk k of sequence b: the forward vectors at its
// columns and at the rows of its group (lane r of each 16 lanes, or of each 8 for rows of 8
// lanes), the normaliser and the store offsets
template <class F>
struct FormAt {
    const RecLogArgs& a;
    int64_t row0, bk;
    int C, lane, g0, ver;
    bool row_ok;
    double shift;
    int flast;
    __device__ FormAt(const RecLogArgs& a_, int b, int k, int C_) : a(a_), C(C_) {
        lane = threadIdx.x & 63;
        g0 = ((threadIdx.x >> 6) * F::kG + lane / F::kLPR) * F::kRG;
        row0 = (int64_t)b * (a.N - 1);
        bk = (int64_t)b * a.K + k;
        const int gr = lane & (F::kLPR >= 16 ? 15 : 7);
        row_ok = gr < F::kRG && g0 + gr < C;
        ver = a.K == 1 ? 0 : latest_version(a.chg, a.B * a.K, bk, kRecRounds + 1);
        shift = a.shift[bk];
        flast = a.last[bk];
    }
    __device__ int col(int cp) const { return (cp * F::kLPR + lane % F::kLPR) * F::kVec; }
    __device__ void load_cols(float (&o)[F::kCB], const float* from) const {
#pragma unroll
        for (int cp = 0; cp < F::kCP; ++cp) {
            const float* f = from + (col(cp) < C ? col(cp) : 0);
            if constexpr (F::kVec == 4) {
                const float4 y = *(const float4*)f;
                o[cp * 4] = y.x; o[cp * 4 + 1] = y.y; o[cp * 4 + 2] = y.z; o[cp * 4 + 3] = y.w;
            } else {
                o[cp] = *f;
            }
        }
    }
    __device__ float load_row(const float* vec, int t) const {
        const int gr = lane & (F::kLPR >= 16 ? 15 : 7);
        return row_ok ? vec[(size_t)(row0 + t) * C + g0 + gr] : 0.f;
    }
    __device__ const float* end_vector() const { return a.vend + ((size_t)ver * a.B * a.K + bk) * C; }
    __device__ double end_exponent() const { return a.xend[(size_t)ver * a.B * a.K + bk] + shift; }
    __device__ double exponent(int t) const { return a.cx[row0 + t] + (t > flast ? shift : 0.0); }
    // Lane r's weight of its group's row r: a_t over the normaliser 2^dc a_{t+1} . b_{t+1}
    __device__ float row_weight(const float (&an)[F::kCB], const float (&bv)[F::kCB], float ar,
                                double dc, bool& bad) const {
        using R = RowSums<F>;
        float n = 0.f;
#pragma unroll
        for (int v = 0; v < F::kCB; ++v) n = fmaf(an[v], bv[v], n);
        // over the row's lanes (every row of lanes holds all columns)
        n += R::template shift<0>(n);
        n += R::template shift<1>(n);
        n += R::template shift<2>(n);
        if constexpr (F::kLPR >= 16) n += R::template shift<3>(n);
        if constexpr (F::kLPR >= 32) n = R::template merge<4>(n, n, lane);
        if constexpr (F::kLPR >= 64) n = R::template merge<5>(n, n, lane);
        const float norm = n * exp2f((float)dc);
        bad |= n > 0.f && !(norm >= 0x1p-100f && norm <= 0x1p100f);
        return n > 0.f ? ar / norm : 0.f;
    }
    __device__ float row_of(float w, int r) const {
        if constexpr (F::kLPR >= 16) return row_bcast(w, r);
        else return __shfl(w, (lane & ~7) + r, kWave);
    }
    // The marginals are not read again here, so they leave the caches to the edges (mid-sized
    // batches: 192 to 180 us; C = 256, 4.3 GB: 2.79 to 2.74 ms).
    static constexpr int kNt = 2;
    // Offsets of the lane's columns; rows and columns past C go past the descriptor's end, which
    // drops them
    static constexpr unsigned kNowhere = 0x40000000u;
    __device__ void store_offsets(unsigned (&o)[F::kCP]) const {
#pragma unroll
        for (int cp = 0; cp < F::kCP; ++cp) o[cp] = col(cp) < C ? 4u * (unsigned)(g0 * C + col(cp)) : kNowhere;
    }
    __device__ void store_row(const float (&y)[F::kCB], __amdgpu_buffer_rsrc_t ro,
                              const unsigned (&o)[F::kCP], int r) const {
#pragma unroll
        for (int cp = 0; cp < F::kCP; ++cp) {
            const unsigned at = g0 + r < C ? o[cp] : kNowhere;
            if constexpr (F::kVec == 4)
                buffer_store4<kNt>(make_float4(y[cp * 4], y[cp * 4 + 1], y[cp * 4 + 2], y[cp * 4 + 3]), ro, at, 4 * r * C);
            else
                buffer_store1<kNt>(y[cp], ro, at, 4 * r * C);
        }
    }
};

// Walks the edges [s, e) of sequence b backwards from the vector in sm.b[e & 1] (its largest
// entries per wave in sm.top[e & 1]) and, with kForm, writes their marginals; the vector of position s is
// left in sm.b[s & 1], and the exponent it lacks in x.  kAgain: stops where the vector agrees with the stored one (at s with
// old_beg) up to a factor, and returns whether it did; the marginals of the edges before that
// position do not depend on the factor.
//
// Bound: one read and one write of the edges (8 C^2 bytes each).  A row's exponentials serve
// its sum and its marginals at once, so a tile register is stored and reloaded row by row.
template <class F, bool kAgain, bool kForm, bool kPre>
__device__ bool walk_bwd(const RecLogArgs& a, BwdLds<F>& sm, int b, int k, int s, int e, int& x, bool& bad,
                         const float* old_beg) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, C = a.C, CC = C * C;
    const int gl = lane / F::kLPR, c = lane & 15;
    const int64_t E = a.N - 1, row0 = (int64_t)b * E;
    // the row whose sum this lane holds, and the rows of its group
    const int g0 = (w * F::kG + gl) * F::kRG;
    const int rw = RowSums<F>::which(lane);
    const int i = g0 + rw;
    const bool own = rw < F::kRG && i < C && (lane & (RowSums<F>::kLow - 1)) == 0;
    const unsigned voff = tile_offset<F>(C);
    const FormAt<F> at(a, b, k, C);
    unsigned soff[F::kCP];
    at.store_offsets(soff);
    const float* edge = (kPre ? a.epot : a.pot) + (size_t)(row0 + e - 1) * CC;
    float* out = a.marg + (size_t)(row0 + e - 1) * CC;
    Tile<F> ring[F::kDepth];
#pragma unroll
    for (int d = 0; d < F::kDepth; ++d) {
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(uniform(edge), uniform(e - 1 - d >= s ? CC : 0));
#pragma unroll
        for (int r = 0; r < F::kRG; ++r) {
            tile_load_row<F>(ring[d].x[r], rs, voff, r, C);
            __builtin_amdgcn_sched_barrier(0);
        }
        edge -= CC;
    }
    float an[F::kCB] = {}, ar = 0.f;       // a_{t+1} at the columns, a_t at the rows
    double c1 = 0.0, c0 = 0.0;             // their exponents
    if (kForm) {
        at.load_cols(an, at.end_vector());
        ar = at.load_row(a.alpha, e - 1);
        c1 = at.end_exponent();
        c0 = at.exponent(e - 1);
    }
    constexpr bool kFirst = !kAgain && !kForm;   // (with kForm the forward walks have checked)
    constexpr bool kRange = kFirst && !kPre;
    x = 0;
    unsigned big = 0;
    // One step, edge t in tile: returns whether the walk ends at position t
    auto step = [&](Tile<F>& tile, int t, auto look) {
        constexpr bool kLook = kAgain && decltype(look)::value;
        const int from = (t + 1) & 1, to = t & 1;
        // b_{t+1}, scaled by its exponent
        const int ex = uniform(exponent_of(row_max(sm.top[from][c < F::kNW ? c : 0])));
        if (kFirst && ex > 127) return true;
        x += ex;
        float bv[F::kCB];
#pragma unroll
        for (int cp = 0; cp < F::kCP; ++cp) {
            const float* o = &sm.b[from][(cp * F::kLPR + lane % F::kLPR) * F::kVec];
            if constexpr (F::kVec == 4) {
                const float4 y = *(const float4*)o;
                bv[cp * 4] = y.x; bv[cp * 4 + 1] = y.y; bv[cp * 4 + 2] = y.z; bv[cp * 4 + 3] = y.w;
            } else {
                bv[cp] = *o;
            }
        }
#pragma unroll
        for (int v = 0; v < F::kCB; ++v) bv[v] = ldexpf(bv[v], -ex);
        const bool more = t > s;
        float wr0 = 0.f;
        if (kForm) {
            wr0 = at.row_weight(an, bv, ar, c1 - c0, bad);
            // the next step's vectors
            c1 = c0;
            if (more) {
                at.load_cols(an, a.alpha + (size_t)(row0 + t) * C);
                ar = at.load_row(a.alpha, t - 1);
                c0 = at.exponent(t - 1);
            }
        }
        float was = 0.f;
        if (kLook && own) was = more ? a.beta[(size_t)(row0 + t) * C + i] : old_beg[i];
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(uniform(edge), uniform(t - F::kDepth >= s ? CC : 0));
        const __amdgpu_buffer_rsrc_t ro = make_rsrc(uniform(out), CC);
        edge -= CC;
        out -= CC;
        float sums[F::kRG];
#pragma unroll
        for (int r = 0; r < F::kRG; ++r) {
            const float wr = kForm ? at.row_of(wr0, r) : 0.f;
            float y[F::kCB], sum = 0.f;
#pragma unroll
            for (int v = 0; v < F::kCB; ++v) {
                asm volatile("" : "+v"(tile.x[r][v]));
                if (kRange) big = max(big, fin_bits(tile.x[r][v]));
                const float p = exp_of<kPre>(tile.x[r][v]) * bv[v];
                sum += p;
                y[v] = p * wr;
            }
            if (kRange) asm volatile("" : "+v"(big));
            sums[r] = sum;
            if (kForm) at.store_row(y, ro, soff, r);
            tile_load_row<F>(tile.x[r], rs, voff, r, C);
            __builtin_amdgcn_sched_barrier(0);
        }
        const float v = RowSums<F>::sum(sums, lane);
        const float mine = own ? v : 0.f;
        bad |= mine != 0.f && !(mine >= kRecLow && mine <= 0x1p60f);
        if (own) {
            sm.b[to][i] = v;
            if (more && a.beta) a.beta[(size_t)(row0 + t) * C + i] = v;
        }
        float top = row_max(mine);
        {
            const Pair p16 = pair16(__float_as_uint(top));
            top = fmaxf(__uint_as_float(p16.a), __uint_as_float(p16.b));
            const Pair p32 = pair32(__float_as_uint(top));
            top = fmaxf(__uint_as_float(p32.a), __uint_as_float(p32.b));
        }
        const bool out = kFirst && __any(kPre ? bad : big > kRecPotBits);
        if (lane == 0) sm.top[to][w] = out ? INFINITY : top;
        if (kLook) {
            Ratio ra = ratio_of(own, v, was);
            ra.lo = row_max(-ra.lo);
            ra.hi = row_max(ra.hi);
            const Pair l16 = pair16(__float_as_uint(ra.lo)), h16 = pair16(__float_as_uint(ra.hi));
            ra.lo = fmaxf(__uint_as_float(l16.a), __uint_as_float(l16.b));
            ra.hi = fmaxf(__uint_as_float(h16.a), __uint_as_float(h16.b));
            const Pair l32 = pair32(__float_as_uint(ra.lo)), h32 = pair32(__float_as_uint(ra.hi));
            ra.lo = -fmaxf(__uint_as_float(l32.a), __uint_as_float(l32.b));
            ra.hi = fmaxf(__uint_as_float(h32.a), __uint_as_float(h32.b));
            if (lane == 0) { sm.ratio[to][0][w] = ra.lo; sm.ratio[to][1][w] = ra.hi; }
        }
        __syncthreads();
        return kLook && same_ratio(sm.ratio[to], c, F::kNW);
    };
    int t = e - 1;
    for (; t - F::kDepth + 1 >= s; t -= F::kDepth) {
#pragma unroll
        for (int d = 0; d + 1 < F::kDepth; ++d) step(ring[d], t - d, std::false_type{});
        if (step(ring[F::kDepth - 1], t - F::kDepth + 1, std::true_type{})) {
            bad |= kFirst;
            return true;
        }
    }
    bool agreed = false;
#pragma unroll
    for (int d = 0; d + 1 < F::kDepth; ++d)
        if (uniform(t - d >= s)) agreed = step(ring[d], t - d, std::true_type{});
    bad |= kRange && big > kRecPotBits;
    return agreed;
}

// Puts the start vector of a backward walk into LDS: `start`, or ones
template <class F>
__device__ void start_bwd(const RecLogArgs& a, BwdLds<F>& sm, int e, const float* start) {
    __syncthreads();   // (an earlier walk's readers)
    for (int i = threadIdx.x; i < F::kCols; i += F::kT) {
        sm.b[e & 1][i] = i < a.C ? (start ? start[i] : 1.f) : 0.f;
        sm.b[(e & 1) ^ 1][i] = 0.f;   // (columns past C stay 0)
    }
    if (threadIdx.x < 64) {
        float m = 0.f;
        for (int i = threadIdx.x; i < a.C; i += 64) m = fmaxf(m, start ? start[i] : 1.f);
        m = wave_max(m);
        if (threadIdx.x < 16) sm.top[e & 1][threadIdx.x] = m;
    }
    __syncthreads();
}

template <class F>
__device__ void end_bwd(const RecLogArgs& a, BwdLds<F>& sm, int s, int64_t bk, int ver) {
    for (int i = threadIdx.x; i < a.C; i += F::kT)
        a.vbeg[((size_t)ver * a.B * a.K + bk) * a.C + i] = sm.b[s & 1][i];
}

__device__ void zero_edges(float* p, int64_t n) {
    // (p is 16-byte aligned when C is a multiple of 4, and n a multiple of 4 then)
    if (((uintptr_t)p & 15) == 0 && (n & 3) == 0) {
        float4* q = (float4*)p;
        for (int64_t i = threadIdx.x; i < n / 4; i += blockDim.x) q[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
        for (int64_t i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0.f;
    }
}

// The first backward walk of a chunk: from ones (the true end of the last chunk, a guess
// elsewhere); with kForm, also zeros for the padding edges
template <class F, bool kForm>
__device__ void first_bwd(const RecLogArgs& a, BwdLds<F>& sm, int b, int k) {
    const int E = (int)a.N - 1, Eb = uniform((int)clamp_len(a.lengths, b, a.N)) - 1;
    int s, e;
    chunk_edges(a, k, Eb, true, s, e);
    if (kForm) {
        if (uniform(a.gate[b] != 0)) return;
        const int CC = a.C * a.C, z = max(s, Eb), ze = min(s + a.S, E);
        if (z < ze) zero_edges(a.marg + (size_t)((int64_t)b * E + z) * CC, (int64_t)(ze - z) * CC);
    } else if (Eb == 0 && k == 0 && threadIdx.x == 0) {
        a.gateb[b] = 0;
    }
    if (s >= Eb) return;
    start_bwd<F>(a, sm, e, nullptr);
    int x;
    bool bad = false;
    if (!kForm && F::kPre && a.epot) walk_bwd<F, false, kForm, !kForm && F::kPre>(a, sm, b, k, s, e, x, bad, nullptr);
    else walk_bwd<F, false, kForm, false>(a, sm, b, k, s, e, x, bad, nullptr);
    const int64_t bk = (int64_t)b * a.K + k;
    end_bwd<F>(a, sm, s, bk, 0);
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) {
        a.badb[bk] = bad;
        a.badb[a.B * a.K + bk] = 0;
        a.xbeg[bk] = x;
        if (a.K == 1) (kForm ? a.gate : a.gateb)[b] = bad;
    }
}

template <class F, bool kForm>
__device__ bool again_bwd(const RecLogArgs& a, BwdLds<F>& sm, int b, int k, int Eb,
                          const float* start, int old, int ver) {
    const int64_t nbk = a.B * a.K, bk = (int64_t)b * a.K + k;
    const int s = k * a.S, e = uniform(min(s + a.S, Eb));
    start_bwd<F>(a, sm, e, start);
    int x;
    bool bad = false;
    const float* old_beg = a.vbeg + ((size_t)old * nbk + bk) * a.C;
    const bool agreed =
        !kForm && F::kPre && a.epot
            ? walk_bwd<F, true, kForm, !kForm && F::kPre>(a, sm, b, k, s, e, x, bad, old_beg)
            : walk_bwd<F, true, kForm, false>(a, sm, b, k, s, e, x, bad, old_beg);
    if (!agreed) end_bwd<F>(a, sm, s, bk, ver);
    bad = __syncthreads_or(bad);
    if (bad && threadIdx.x == 0) a.badb[nbk + bk] = 1;
    return !agreed;
}

template <class F, bool kForm>
__device__ void round_bwd(const RecLogArgs& a, BwdLds<F>& sm, int b, int k) {
    if (kForm && uniform(a.gate[b] != 0)) return;
    const int Eb = uniform((int)clamp_len(a.lengths, b, a.N)) - 1;
    if (k * a.S >= Eb) return;
    const int64_t nbk = a.B * a.K, bk = (int64_t)b * a.K + k;
    const int ver = a.round - 1;
    bool changed = false;
    if ((k + 1) * a.S < Eb && (ver == 0 || a.chgb[(size_t)(ver - 1) * nbk + bk + 1]) &&
        (kForm || !(a.badb[bk] | a.badb[bk + 1])))
        changed = again_bwd<F, kForm>(a, sm, b, k, Eb, a.vbeg + ((size_t)ver * nbk + bk + 1) * a.C,
                                      latest_version(a.chgb, nbk, bk, ver), a.round);
    if (threadIdx.x == 0) a.chgb[(size_t)ver * nbk + bk] = changed;
}

template <class F, bool kForm>
__device__ void last_bwd(const RecLogArgs& a, BwdLds<F>& sm, int b) {
    const int Eb = uniform((int)clamp_len(a.lengths, b, a.N)) - 1;
    if (Eb == 0 || (kForm && uniform(a.gate[b] != 0))) return;
    const int64_t nbk = a.B * a.K, b0 = (int64_t)b * a.K;
    const int n = (Eb + a.S - 1) / a.S;
    int32_t* const chg = a.chgb + (size_t)kRecRounds * nbk + b0;
    bool left = false, any = false;
    auto late_at = [&](int k) { return k + 1 < n && a.chgb[(size_t)(kRecRounds - 1) * nbk + b0 + k + 1] != 0; };
    for (int k = threadIdx.x; k < n; k += F::kT) {
        left |= (a.badb[b0 + k] | a.badb[nbk + b0 + k] | a.bad[b0 + k]) != 0;
        any |= late_at(k);
        chg[k] = 0;
    }
    int pending = 0, walked = 0;
    if (__syncthreads_or(left || any)) {
        for (int k0 = 0; k0 < n; k0 += F::kT) pending += __syncthreads_count(late_at(k0 + (int)threadIdx.x));
        left = __syncthreads_or(left) || (a.tree_pending && pending > a.limit);
    }
    bool changed = false;
    for (int k = n - 2; pending > 0 && !left && k >= 0; --k) {
        const bool late = late_at(k);
        if (!uniform(changed || late)) continue;
        if (a.tree_pending && walked++ == 2 * a.limit) {
            left = true;
            break;
        }
        changed = again_bwd<F, kForm>(a, sm, b, k, Eb,
                                      a.vbeg + ((size_t)(kRecRounds + changed) * nbk + b0 + k + 1) * a.C,
                                      latest_version(a.chgb, nbk, b0 + k, kRecRounds), kRecRounds + 1);
        changed = uniform(changed);
        if (threadIdx.x == 0) chg[k] = changed;
        __syncthreads();
        left |= uniform(a.badb[nbk + b0 + k] != 0);
    }
    if (threadIdx.x == 0) (kForm ? a.gate : a.gateb)[b] = left;
}

// ---- kernels

// The walks of one launch: forward, both directions side by side (the first half of the grid
// forward), or backward with the marginals formed on the way
enum Dir { kFwd, kBoth, kBwdForm };

template <class F>
union Lds {
    FwdLds<F> f;
    BwdLds<F> b;
};

// kFirst, kRound: one workgroup per chunk, consecutive ones the same chunk of consecutive
// sequences; kLast: one per sequence
enum Part { kFirst, kRound, kLast };

template <class F, Dir dir, Part part>
__global__ __launch_bounds__(F::kT, F::kNW == 16 ? 4 : 2) void k_rec_log(RecLogArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    Lds<F>& sm = *(Lds<F>*)smem;
    const unsigned half = (unsigned)(part == kLast ? a.B : a.B * a.K);
    const bool back = dir == kBwdForm || (dir == kBoth && blockIdx.x >= half);
    const unsigned i = blockIdx.x - (dir == kBoth && back ? half : 0u);
    const int k = part == kLast ? 0 : uniform((int)(i / (unsigned)a.B)), b = (int)i - k * (int)a.B;
    if (dir != kBwdForm && !back) {
        if constexpr (part == kFirst) first_fwd<F>(a, sm.f, b, k);
        else if constexpr (part == kRound) round_fwd<F>(a, sm.f, b, k);
        else last_fwd<F>(a, sm.f, b);
    }
    if (dir != kFwd && back) {
        if constexpr (part == kFirst) first_bwd<F, dir == kBwdForm>(a, sm.b, b, k);
        else if constexpr (part == kRound) round_bwd<F, dir == kBwdForm>(a, sm.b, b, k);
        else last_bwd<F, dir == kBwdForm>(a, sm.b, b);
    }
}

// The marginals of one edge per workgroup from the vectors of both directions (after kBoth)
template <class F>
__global__ __launch_bounds__(F::kT, F::kNW == 16 ? 4 : 2) void k_rec_form(RecLogArgs a) {
    const int E = (int)a.N - 1, C = a.C, CC = C * C;
    const int b = uniform((int)(blockIdx.x / (unsigned)E)), t = (int)blockIdx.x - b * E;
    if (uniform((a.gate[b] | a.gateb[b]) != 0)) {
        if (t == 0 && threadIdx.x == 0) a.gate[b] = 1;
        return;
    }
    const int Eb = uniform((int)clamp_len(a.lengths, b, a.N)) - 1;
    float* out = a.marg + ((size_t)b * E + t) * CC;
    if (t >= Eb) {
        zero_edges(out, CC);
        return;
    }
    Tile<F> x;
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(uniform((a.epot ? a.epot : a.pot) + ((size_t)b * E + t) * CC), CC);
    const unsigned voff = tile_offset<F>(C);
#pragma unroll
    for (int r = 0; r < F::kRG; ++r) tile_load_row<F>(x.x[r], rs, voff, r, C);
    const int k = uniform(t / a.S), e = uniform(min((k + 1) * a.S, Eb));
    const FormAt<F> at(a, b, k, C);
    const bool end = t + 1 == e;
    float an[F::kCB], bv[F::kCB];
    at.load_cols(an, end ? at.end_vector() : a.alpha + (size_t)(at.row0 + t + 1) * C);
    if (end && e == Eb) {
#pragma unroll
        for (int v = 0; v < F::kCB; ++v) bv[v] = 1.f;
    } else {
        const int64_t nbk = a.B * a.K;
        at.load_cols(bv, end ? a.vbeg + ((size_t)latest_version(a.chgb, nbk, at.bk + 1, kRecRounds + 1) * nbk + at.bk + 1) * C
                             : a.beta + (size_t)(at.row0 + t + 1) * C);
    }
    const float ar = at.load_row(a.alpha, t);
    const double dc = (end ? at.end_exponent() : at.exponent(t + 1)) - at.exponent(t);
    // scaled as the walks scale it; columns past C weigh nothing
    float m = 0.f;
#pragma unroll
    for (int cp = 0; cp < F::kCP; ++cp)
#pragma unroll
        for (int v = 0; v < F::kVec; ++v) {
            float& y = bv[cp * F::kVec + v];
            if (at.col(cp) >= C) y = 0.f;
            m = fmaxf(m, y);
        }
    m = wave_max_fast(m);
    const int ex = exponent_of(m);
#pragma unroll
    for (int v = 0; v < F::kCB; ++v) bv[v] = ldexpf(bv[v], -ex);
    bool bad = false;
    const float w = at.row_weight(an, bv, ar, dc, bad);
    if (bad) a.gate[b] = 1;   // (the tree then computes the sequence)
    unsigned soff[F::kCP];
    at.store_offsets(soff);
    const __amdgpu_buffer_rsrc_t ro = make_rsrc(uniform(out), CC);
#pragma unroll
    for (int r = 0; r < F::kRG; ++r) {
        const float wr = at.row_of(w, r);
        float y[F::kCB];
#pragma unroll
        for (int v = 0; v < F::kCB; ++v) {
            const float e1 = F::kPre && a.epot ? x.x[r][v] : edge_exp(x.x[r][v]);
            y[v] = e1 * bv[v] * wr;
        }
        at.store_row(y, ro, soff, r);
    }
}

// The exponentials of every edge, one workgroup each; an entry outside the range becomes an
// infinity, which the walks notice
__global__ __launch_bounds__(256) void k_rec_exp(RecLogArgs a) {
    const int E = (int)a.N - 1, CC = a.C * a.C;
    const int b = (int)(blockIdx.x / (unsigned)E), t = (int)blockIdx.x - b * E;
    if (t >= (int)clamp_len(a.lengths, b, a.N) - 1) return;
    const size_t at = ((size_t)b * E + t) * CC;
    const float* from = a.pot + at;
    float* to = a.epot + at;
    auto f = [](float x) { return fin_bits(x) > kRecPotBits ? INFINITY : edge_exp(x); };
    if (CC % 4 == 0) {   // (16-byte aligned edges; eight loads in flight per thread)
        const int n = CC / 4;
        for (int i = threadIdx.x; i < n; i += 8 * 256) {
            float4 x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = ((const float4*)from)[min(i + 256 * u, n - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i + 256 * u < n) ((float4*)to)[i + 256 * u] = make_float4(f(x[u].x), f(x[u].y), f(x[u].z), f(x[u].w));
        }
    } else {
        for (int i = threadIdx.x; i < CC; i += 256) to[i] = f(from[i]);
    }
}

// log Z where the two halves of a one-chunk sequence meet: sum_j a_m[j] b_m[j]
__global__ __launch_bounds__(64) void k_rec_meet(RecLogArgs a) {
    const int64_t b = blockIdx.x;
    if (clamp_len(a.lengths, b, a.N) == 1) return;
    const int lane = threadIdx.x;
    double tot = 0.0;
    for (int i = lane; i < a.C; i += 64) tot += (double)a.vend[(size_t)b * a.C + i] * (double)a.vbeg[(size_t)b * a.C + i];
    tot = wave_sum_d(tot);
    if (lane != 0) return;
    const bool left = (a.bad[b] | a.badb[b]) != 0;
    a.gate[b] = left;
    set_log_z(a, b, log2(tot) + a.xend[b] + a.xbeg[b], left);
}

// log Z of the marked sequences in float64: one workgroup per chunk walks it from its
// predecessor's end vector and takes its growth against its own end vector, whose directions are
// known to some 1e-7, an error of about 1e-8 per chunk (row-normalised, C = 8, N = 65536: 1.4e-4
// before this, see the tests).  Rare, so simple: four threads share a column.
__global__ __launch_bounds__(1024) void k_rec_refine(RecLogArgs a) {
    __shared__ double vec[kMaxLabels], part[4][kMaxLabels];
    __shared__ bool done;
    const int k = (int)(blockIdx.x / (unsigned)a.B), b = (int)(blockIdx.x - k * (unsigned)a.B);
    if (!a.fine[b]) return;
    const int Eb = (int)clamp_len(a.lengths, b, a.N) - 1, C = a.C, tid = threadIdx.x;
    const int s = k * a.S, e = min(s + a.S, Eb);
    if (s >= Eb) return;
    const int n = (Eb + a.S - 1) / a.S, j = tid % kMaxLabels, g = tid / kMaxLabels;
    const int64_t nbk = a.B * a.K, bk = (int64_t)b * a.K + k;
    auto end_of = [&](int64_t at) {
        return a.vend + ((size_t)latest_version(a.chg, nbk, at, kRecRounds + 1) * nbk + at) * C;
    };
    if (tid < C) vec[tid] = k == 0 ? 1.0 : (double)end_of(bk - 1)[tid];
    __syncthreads();
    int x = 0;
    const float* edge = a.pot + ((size_t)b * (a.N - 1) + s) * C * C;
    for (int t = s; t < e; ++t, edge += (size_t)C * C) {
        if ((t - s) % 8 == 7) {   // (a step changes the largest entry by less than 2^43)
            double m = 0.0;
            for (int i = tid & 63; i < C; i += 64) m = fmax(m, vec[i]);
            const int ex = (int)((__double_as_longlong(wave_max_d(m)) >> 52) & 0x7ff) - 1023;
            __syncthreads();
            if (tid < C) vec[tid] = ldexp(vec[tid], -ex);
            x += ex;
            __syncthreads();
        }
        double acc = 0.0;
        if (j < C)
            for (int i = g; i < C; i += 4) acc = fma(vec[i], exp((double)edge[(size_t)i * C + j]), acc);
        part[g][j] = acc;
        __syncthreads();
        if (tid < C) vec[tid] = (part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]);
        __syncthreads();
    }
    if (tid < 64) {
        double now = 0.0, was = 0.0;
        for (int i = tid; i < C; i += 64) {
            now += vec[i];
            was += k + 1 < n ? (double)end_of(bk)[i] : 0.0;
        }
        now = wave_sum_d(now);
        was = wave_sum_d(was);
        if (tid == 0) {
            a.part[bk] = x + log2(now) - (k + 1 < n ? log2(was) : 0.0);
            // the last chunk to end adds them up, in order
            done = __hip_atomic_fetch_add(a.count + b, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
        }
    }
    __syncthreads();
    if (!done || tid >= 64) return;
    double sum = 0.0;
    for (int i = tid; i < n; i += 64) sum += a.part[(int64_t)b * a.K + i];
    sum = wave_sum_d(sum);
    if (tid == 0) a.logZ[b] = (float)(sum * 0.6931471805599453);
}

template <class F, Dir dir>
hipError_t launch_walks(RecLogArgs a, hipStream_t s) {
    constexpr size_t lds = sizeof(Lds<F>);
    static_assert(lds <= 65536, "no LDS attribute needed");
    const int64_t sides = dir == kBoth ? 2 : 1;
    const dim3 chunks((unsigned)(sides * a.B * a.K)), seqs((unsigned)(sides * a.B)), threads(F::kT);
    hipLaunchKernelGGL((k_rec_log<F, dir, kFirst>), chunks, threads, lds, s, a);
    hipError_t e = hipGetLastError();
    if (a.K == 1) return e;
    for (a.round = 1; e == hipSuccess && a.round <= kRecRounds; ++a.round) {
        hipLaunchKernelGGL((k_rec_log<F, dir, kRound>), chunks, threads, lds, s, a);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_rec_log<F, dir, kLast>), seqs, threads, lds, s, a);
    return hipGetLastError();
}

hipError_t refine(const RecLogArgs& a, hipStream_t s) {
    if (!a.fine) return hipSuccess;
    hipLaunchKernelGGL(k_rec_refine, dim3((unsigned)(a.B * a.K)), dim3(1024), 0, s, a);
    return hipGetLastError();
}

template <class F>
hipError_t launch(RecLogArgs a, bool both, hipStream_t s) {
    if (!F::kPre) a.epot = nullptr;
    if (a.epot) {
        hipLaunchKernelGGL(k_rec_exp, dim3((unsigned)(a.B * (a.N - 1))), dim3(256), 0, s, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (a.meet) {
        const hipError_t e = launch_walks<F, kBoth>(a, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_rec_meet, dim3((unsigned)a.B), dim3(64), 0, s, a);
        const hipError_t em = hipGetLastError();
        return em == hipSuccess ? refine(a, s) : em;
    }
    if (!a.marg || !both) {
        hipError_t e = launch_walks<F, kFwd>(a, s);
        if (e == hipSuccess) e = refine(a, s);
        return e == hipSuccess && a.marg ? launch_walks<F, kBwdForm>(a, s) : e;
    }
    hipError_t e = launch_walks<F, kBoth>(a, s);
    if (e == hipSuccess) e = refine(a, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_rec_form<F>, dim3((unsigned)(a.B * (a.N - 1))), dim3(F::kT), 0, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_rec_log(const Plan& p, const float* pot, const int32_t* lengths, float* logZ,
                          float* marg, hipStream_t s) {
    RecLogArgs a{};
    a.pot = pot; a.lengths = lengths; a.B = p.B; a.N = p.N; a.C = (int)p.C;
    a.S = (int)p.rec_S; a.K = (int)p.rec_K;
    a.alpha = p.rec_alpha; a.cx = p.rec_cx; a.vend = p.rec_vend; a.xend = p.rec_xend;
    a.chg = p.rec_chg; a.shift = p.rec_shift; a.ratio = p.rec_ratio; a.last = p.rec_last; a.bad = p.rec_bad;
    a.beta = p.rec_beta; a.vbeg = p.rec_vbeg; a.chgb = p.rec_chgb; a.badb = p.rec_badb;
    a.marg = marg; a.logZ = logZ; a.gate = p.gate; a.gateb = p.rec_gateb; a.tree_pending = p.rec_tree;
    a.limit = rec_limit(p.rec_S, p.rec_K);
    a.xbeg = p.rec_xbeg; a.epot = p.rec_exp;
    if (logZ && p.E > kRefineEdges) { a.fine = p.rec_fine; a.count = p.rec_count; a.part = p.rec_part; }
    a.meet = !marg && logZ && p.rec_K == 1 && p.E >= 4;
    const bool both = (size_t)p.B * p.E * p.C * p.C * sizeof(float) <= kRecBothBytes &&
                      grid_fits(p.B * p.E, rec_threads(p.C));   // (k_rec_form)
    return with_rec_cfg(p.C, [&](auto f) { return launch<decltype(f)>(a, both, s); });
}

}  // namespace tsc

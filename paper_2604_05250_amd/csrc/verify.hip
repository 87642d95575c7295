// Verification pass over the vocabulary (Sec. 3.2): one streaming read of the verifier
// logits (and, in the KL modes, the drafter logits) produces per position the verifier
// confidence c_V = max_x p_V(x) (Eq. 7), its argmax, and KL(p_D || p_V) (Eq. 5); a small
// finishing kernel applies the remask rule (Eq. 4, the KL / confidence thresholds, Eq. 6,
// and the 1 - c_V rule).
//
// HBM-bound design: every logit is loaded exactly once with 16-byte coalesced loads.
// A row is split over `S` workgroups.  Each wave keeps wave-uniform references (the
// running verifier and drafter maxima) so the per-element work
// is one fma + one exp2 + one add per logit, and the argmax / rescale logic runs only
// when some lane of the wave sees a new maximum (a few times per row).  Partial states
//     (ref_D, sum e^{l_D-ref_D}, sum e^{l_D-ref_D}(l_D-l_V), max l_V, sum e^{l_V-max}, argmax)
// are merged in a fixed order (lanes -> waves -> splits), so results are run-to-run
// identical; the last merge and the log / divide are done in fp64.
#include "dd_internal.h"

#include <algorithm>
#include <limits.h>
#include <math.h>

#include <type_traits>

namespace dd {
namespace {

constexpr int kThreads = 256;
constexpr int kUnroll = 4;   // independent 16-byte loads per matrix in flight per lane
constexpr float kLog2e = 1.44269504088896340736f;
constexpr float kNegInf = -INFINITY;
// The drafter reference is raised when a logit exceeds it by more than this.  Zero keeps it
// equal to the running maximum, exactly as on the verifier side, so identical drafter and
// verifier rows go through identical arithmetic and give KL = 0 exactly.
constexpr float kLazyMargin = 0.0f;

struct __align__(32) VerifyPartial {
    float ref_d, s_d, a;   // drafter reference, sum e^{l_D-ref}, sum e^{l_D-ref} (l_D - l_V)
    float best_v, s_v;     // verifier maximum, sum e^{l_V-best}
    int idx;               // lowest index attaining best_v
    int idx_d;             // lowest index attaining ref_d (the drafter's most likely token)
    int pad1;
};

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// streaming 16-byte load: every logit is read once, so it need not displace cached lines
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 stream_load16(const uint4 *p)
{
    const u32x4 w = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
    return make_uint4(w.x, w.y, w.z, w.w);
}

// Reductions over the 64 lanes of a wave, every lane with the result (the same bits: a + b == b + a): neighbours, pairs of
// two, halves of eight and of sixteen lanes by DPP, the rest by the two lane-half exchanges.  Shuffles through the LDS
// crossbar cost their latency six times per reduction, and a short call is a chain of such reductions.
// (All lanes take part and every lane named exists, so the exchange needs no second operand: it becomes part of the operation.)
template <int CTRL> __device__ __forceinline__ unsigned dpp(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
template <typename F> __device__ __forceinline__ unsigned wave_reduce(unsigned v, F &&f)
{
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    v = f(v, dpp<0xB1>(v));                                  // quad_perm [1,0,3,2]
    v = f(v, dpp<0x4E>(v));                                  // quad_perm [2,3,0,1]
    v = f(v, dpp<0x141>(v));                                 // row_half_mirror
    v = f(v, dpp<0x140>(v));                                 // row_mirror
    const u32x2 h = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = f(h.x, h.y);
    const u32x2 w = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return f(w.x, w.y);
}
// The steps of a reduction over aligned groups of sixteen lanes: the value of a lane of the group's other part (neighbours, pairs of two,
// halves of eight and of sixteen; the lanes of a part agree after the steps before).
template <int STEP> __device__ __forceinline__ unsigned other16(unsigned v)
{
    return dpp<STEP == 0 ? 0xB1 : STEP == 1 ? 0x4E : STEP == 2 ? 0x141 : 0x140>(v);
}
template <int STEP> __device__ __forceinline__ float other16(float v) { return __uint_as_float(other16<STEP>(__float_as_uint(v))); }
template <int STEP> __device__ __forceinline__ int other16(int v) { return (int)other16<STEP>((unsigned)v); }
template <int STEP> __device__ __forceinline__ double other16(double v)
{
    return __hiloint2double((int)other16<STEP>((unsigned)__double2hiint(v)), (int)other16<STEP>((unsigned)__double2loint(v)));
}
template <int N, typename F> __device__ __forceinline__ void for_steps(F &&f)
{
    if constexpr (N > 0) {
        for_steps<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}
__device__ __forceinline__ float wave_max(float v)
{
    return __uint_as_float(wave_reduce(__float_as_uint(v), [](unsigned x, unsigned y) {
        return __float_as_uint(fmaxf(__uint_as_float(x), __uint_as_float(y))); }));
}
__device__ __forceinline__ int wave_min(int v)
{
    return (int)wave_reduce((unsigned)v, [](unsigned x, unsigned y) { return (unsigned)min((int)x, (int)y); });
}
__device__ __forceinline__ float wave_sum(float v)
{
    return __uint_as_float(wave_reduce(__float_as_uint(v), [](unsigned x, unsigned y) {
        return __float_as_uint(__uint_as_float(x) + __uint_as_float(y)); }));
}

// Four reductions in little more than the work of one: lanes 4 i + p carry on with value p alone once neighbours and pairs have
// exchanged.  Lane l returns the result of value l % 4, summed in wave_reduce's order (the same bits).
template <typename F> __device__ __forceinline__ unsigned wave_reduce4(const unsigned (&v)[4], int lane, F &&f)
{
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const bool b0 = (lane & 1) != 0, b1 = (lane & 2) != 0;
    const unsigned x = f(b0 ? v[1] : v[0], dpp<0xB1>(b0 ? v[0] : v[1])), y = f(b0 ? v[3] : v[2], dpp<0xB1>(b0 ? v[2] : v[3]));
    unsigned z = f(b1 ? y : x, dpp<0x4E>(b1 ? x : y));
    z = f(z, dpp<0x141>(dpp<0x1B>(z)));                      // quad_perm [3,2,1,0], row_half_mirror: the lane four away
    z = f(z, dpp<0x128>(z));                                 // row_ror:8
    const u32x2 h = __builtin_amdgcn_permlane16_swap(z, z, false, false);
    z = f(h.x, h.y);
    const u32x2 w = __builtin_amdgcn_permlane32_swap(z, z, false, false);
    return f(w.x, w.y);
}
__device__ __forceinline__ void wave_max4(float (&v)[4], int lane)            // every lane with all four
{
    const unsigned u[4] = {__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
    const unsigned r = wave_reduce4(u, lane, [](unsigned x, unsigned y) {
        return __float_as_uint(fmaxf(__uint_as_float(x), __uint_as_float(y))); });
#pragma unroll
    for (int p = 0; p < 4; ++p) v[p] = __uint_as_float(__builtin_amdgcn_readlane(r, p));
}
__device__ __forceinline__ float wave_sum4(const float (&v)[4], int lane)     // lane l: sum l % 4
{
    const unsigned u[4] = {__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
    return __uint_as_float(wave_reduce4(u, lane, [](unsigned x, unsigned y) {
        return __float_as_uint(__uint_as_float(x) + __uint_as_float(y)); }));
}

// e^{ref - m} with the convention that an empty state (ref = -inf) weighs nothing
__device__ __forceinline__ float rescale_factor(float ref, float m)
{
    return ref == kNegInf ? 0.0f : fast_exp2((ref - m) * kLog2e);
}

template <bool BF16> struct VecTraits;
template <> struct VecTraits<true> {
    static constexpr int kElems = 8;
    static __device__ __forceinline__ void unpack(const uint4 &r, float (&x)[8])
    {
        const unsigned w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[2 * i] = __uint_as_float(w[i] << 16);
            x[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
    }
};
template <> struct VecTraits<false> {
    static constexpr int kElems = 4;
    static __device__ __forceinline__ void unpack(const uint4 &r, float (&x)[4])
    {
        x[0] = __uint_as_float(r.x); x[1] = __uint_as_float(r.y);
        x[2] = __uint_as_float(r.z); x[3] = __uint_as_float(r.w);
    }
};

struct LaneState {
    float ref_d = kNegInf, s_d = 0.f, a = 0.f;   // ref_d is wave-uniform
    float best_v = kNegInf, s_v = 0.f;           // best_v, idx_v are wave-uniform
    int idx_v = INT_MAX, idx_d = INT_MAX;        // idx_d: where the drafter reference was found (wave-uniform)
};

// Fold one 16-byte vector of verifier logits (and the matching drafter vector) into the state.
// Must be called by all lanes of a wave together; `valid` masks lanes past the row chunk's end.
// TRACKD: also keep the index of the drafter's maximum (only the all-scores entry point asks for it)
template <bool BF16, bool KL, bool TRACKD>
__device__ __forceinline__ void consume(const uint4 &rv, const uint4 &rd, bool valid, int elem_base, LaneState &st)
{
    constexpr int E = VecTraits<BF16>::kElems;
    float xv[E], xd[E];
    VecTraits<BF16>::unpack(rv, xv);
    float bmax = xv[0];
#pragma unroll
    for (int e = 1; e < E; ++e) bmax = fmaxf(bmax, xv[e]);
    if (!valid) bmax = kNegInf;

    if (__any(bmax > st.best_v)) {
        // rare: a new verifier maximum appears in this wave
        const float wmax = wave_max(bmax);
        int cand = INT_MAX;
        if (valid && bmax == wmax) {
#pragma unroll
            for (int e = E - 1; e >= 0; --e)
                if (xv[e] == wmax) cand = elem_base + e;
        }
        const int widx = wave_min(cand);
        st.s_v *= rescale_factor(st.best_v, wmax);
        st.best_v = wmax;
        st.idx_v = widx;
    }
    if (KL) {
        VecTraits<BF16>::unpack(rd, xd);
        float dmax = xd[0];
#pragma unroll
        for (int e = 1; e < E; ++e) dmax = fmaxf(dmax, xd[e]);
        if (!valid) dmax = kNegInf;
        if (__any(dmax > st.ref_d + kLazyMargin)) {
            const float wmax = wave_max(dmax);
            if (TRACKD) {
                int cand = INT_MAX;
                if (valid && dmax == wmax) {
#pragma unroll
                    for (int e = E - 1; e >= 0; --e)
                        if (xd[e] == wmax) cand = elem_base + e;
                }
                st.idx_d = wave_min(cand);
            }
            const float c = rescale_factor(st.ref_d, wmax);
            st.s_d *= c;
            st.a *= c;
            st.ref_d = wmax;
        }
    }
    if (valid) {
        const float mv = st.best_v * kLog2e;
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) acc += fast_exp2(fmaf(xv[e], kLog2e, -mv));
        st.s_v += acc;
        if (KL) {
            const float md = st.ref_d * kLog2e;
            float accs = 0.f, acca = 0.f;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const float ed = fast_exp2(fmaf(xd[e], kLog2e, -md));
                accs += ed;
                acca = fmaf(ed, xd[e] - xv[e], acca);
            }
            st.s_d += accs;
            st.a += acca;
        }
    }
}

struct WaveState {
    float ref_d, s_d, a, best_v, s_v;
    int idx, idx_d;
};

// associative merge of two partial states (b comes after a in index order)
__device__ __forceinline__ WaveState merge(const WaveState &x, const WaveState &y)
{
    WaveState r;
    const float mv = fmaxf(x.best_v, y.best_v);
    r.s_v = x.s_v * rescale_factor(x.best_v, mv) + y.s_v * rescale_factor(y.best_v, mv);
    const bool take_y = (y.best_v > x.best_v) || (y.best_v == x.best_v && y.idx < x.idx);
    r.best_v = mv;
    r.idx = take_y ? y.idx : x.idx;
    const float md = fmaxf(x.ref_d, y.ref_d);
    const float cx = rescale_factor(x.ref_d, md), cy = rescale_factor(y.ref_d, md);
    r.idx_d = ((y.ref_d > x.ref_d) || (y.ref_d == x.ref_d && y.idx_d < x.idx_d)) ? y.idx_d : x.idx_d;
    r.ref_d = md;
    r.s_d = x.s_d * cx + y.s_d * cy;
    r.a = x.a * cx + y.a * cy;
    return r;
}

// Reduce vectors [vbeg, vend) of one row with a workgroup of THREADS lanes.  Returns true on thread 0,
// whose `out` then holds the merged state of the range (lanes -> waves -> workgroup, fixed order).
template <bool BF16, bool KL, int THREADS, bool TRACKD>
__device__ __forceinline__ bool reduce_range(const uint4 *__restrict__ pv, const uint4 *__restrict__ pd,
                                             int vbeg, int vend, WaveState &out)
{
    constexpr int E = VecTraits<BF16>::kElems;
    constexpr int NW = THREADS / 64;
    const int tid = threadIdx.x;
    LaneState st;
    int base = vbeg;
    // full iterations: kUnroll independent 16-byte loads per matrix in flight per lane
    for (; base + THREADS * kUnroll <= vend; base += THREADS * kUnroll) {
        uint4 rv[kUnroll], rd[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int idx = base + u * THREADS + tid;
            rv[u] = stream_load16(pv + idx);
            if (KL) rd[u] = stream_load16(pd + idx);
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u)
            consume<BF16, KL, TRACKD>(rv[u], rd[u], true, (base + u * THREADS + tid) * E, st);
    }
    // Ragged remainder of the range: the vectors that some lane of the wave has are asked for together (past the end the last vector), and
    // folded after that.  With loads under a lane's own condition the round was four round trips: 512 x 32000 KL 17.8 us, now 17.2;
    // 128 x 32000 11.0 / 10.5; 1024 x 50264 confidence 21.9 / 21.1; 64 x 1024 fp32 KL 4.15 / 4.02.  With every load issued, also of vectors
    // that no lane of the wave has, short rows were slower (fp32 KL 1122 x 816 8.5 / 9.1, 910 x 1424 8.6 / 9.1).
    if (base < vend) {
        uint4 rv[kUnroll], rd[kUnroll];
        const int wave_base = base + (__builtin_amdgcn_readfirstlane(tid) & ~63);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            if (wave_base + u * THREADS >= vend) break;
            const int at = min(base + u * THREADS + tid, vend - 1);
            rv[u] = stream_load16(pv + at);
            if (KL) rd[u] = stream_load16(pd + at);
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            if (wave_base + u * THREADS >= vend) break;
            const int idx = base + u * THREADS + tid;
            consume<BF16, KL, TRACKD>(rv[u], rd[u], idx < vend, idx * E, st);
        }
    }

    // lanes -> wave (references are already wave-uniform), waves -> workgroup
    __shared__ WaveState ws[NW];
    WaveState w;
    w.ref_d = st.ref_d;
    w.s_d = KL ? wave_sum(st.s_d) : 0.f;
    w.a = KL ? wave_sum(st.a) : 0.f;
    w.best_v = st.best_v;
    w.s_v = wave_sum(st.s_v);
    w.idx = st.idx_v;
    w.idx_d = st.idx_d;
    if ((tid & 63) == 0) ws[tid >> 6] = w;
    __syncthreads();
    if (tid != 0) return false;
    WaveState r = ws[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) r = merge(r, ws[i]);
    out = r;
    return true;
}

// grid: P * S workgroups; workgroup (row, split) reduces vectors [split*chunk, (split+1)*chunk) of its row
template <bool BF16, bool KL, bool TRACKD = false>
__global__ __launch_bounds__(kThreads) void verify_partial_kernel(const uint4 *__restrict__ logits_d,
                                                                  const uint4 *__restrict__ logits_v,
                                                                  int nvec, int S, int chunk,
                                                                  VerifyPartial *__restrict__ part)
{
    const int row = blockIdx.x / S;
    const int split = blockIdx.x - row * S;
    const size_t rbase = (size_t)row * (size_t)nvec;
    const int vbeg = split * chunk;
    const int vend = min(nvec, vbeg + chunk);
    WaveState r;
    if (reduce_range<BF16, KL, kThreads, TRACKD>(logits_v + rbase, KL ? logits_d + rbase : nullptr, vbeg, vend, r)) {
        VerifyPartial p;
        p.ref_d = r.ref_d; p.s_d = r.s_d; p.a = r.a;
        p.best_v = r.best_v; p.s_v = r.s_v; p.idx = r.idx;
        p.idx_d = r.idx_d; p.pad1 = 0;
        part[(size_t)row * S + split] = p;
    }
}

// Philox-4x32 with ten rounds (Salmon et al., SC'11): counter-based, so the uniform of a
// row depends only on (seed, row index) and not on the launch geometry.
__device__ __forceinline__ unsigned philox_word0(uint64_t seed, uint64_t row)
{
    unsigned c0 = (unsigned)row, c1 = (unsigned)(row >> 32), c2 = 0u, c3 = 0u;
    unsigned k0 = (unsigned)seed, k1 = (unsigned)(seed >> 32);
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const unsigned hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
        const unsigned hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
        const unsigned n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c0;
}
__device__ __forceinline__ double row_uniform(uint64_t seed, uint64_t row)
{
    return (double)(philox_word0(seed, row) >> 8) * (1.0 / 16777216.0);
}

// Finish one row from its merged sums (fp64): score, token, remask rule.
//   KL = E_D[l_D - l_V] - lse_D + lse_V = a/s_D - (m_D + ln s_D) + (m_V + ln s_V);   c_V = e^{max - lse_V} = 1/s_V
__device__ __forceinline__ void finish_row(int row, double md, double sd, double a, double mv, double sv, int idx,
                                           const uint8_t *__restrict__ mask, int mode, float threshold, uint64_t seed,
                                           int kl_mode, uint8_t *__restrict__ out_mask,
                                           int32_t *__restrict__ out_tokens, float *__restrict__ out_scores,
                                           int idx_d = 0, const VerifyExtra ex = VerifyExtra{}, float *keep_score = nullptr,
                                           int *keep_token = nullptr)
{
    const double score = kl_mode ? a / sd - (md + log(sd)) + (mv + log(sv)) : 1.0 / sv;
    const float s32 = (float)score;
    out_scores[row] = s32;
    out_tokens[row] = idx;
    if (keep_score != nullptr) {                 // a per-sequence rule follows in this workgroup (it decides out_mask)
        *keep_score = s32;
        *keep_token = idx;
        return;
    }
    if (mode == kModeScores) {                   // every per-position quantity, no rule: c = e^{max - lse} = 1 / sum
        ex.conf_v[row] = (float)(1.0 / sv);
        if (ex.conf_d) ex.conf_d[row] = (float)(1.0 / sd);
        if (ex.tok_d) ex.tok_d[row] = idx_d;
        return;
    }
    const uint8_t m = mask[row];
    bool remask = false;
    switch (mode) {
    case 1: remask = s32 > threshold; break;                                // KL threshold
    case 2: remask = s32 < threshold; break;                                // confidence threshold
    case 4: remask = row_uniform(seed, (uint64_t)row) < 1.0 - (double)s32; break;
    default: break;                                                         // trust; per-sequence rules decided later
    }
    out_mask[row] = (uint8_t)((m != 0) || remask);
}

// (Through LDS shuffles, KL's sums carried along in every mode, an unmasking call on 32 x 126464 took 9.7 us in a stream of them, now 8.6,
// a confidence rule 8.2 and 7.8.)
// Sixteen lanes per row (S <= 16): lane s takes the partial state of split s, the group merges them in fp64
// by DPP exchanges (every lane ends with the same totals: a + b == b + a exactly), lane 0 finishes the row.
constexpr int kFinalizeLanes = 16;
// Called by whole groups of sixteen consecutive lanes (lane sp of the group takes split sp of `row`); `row_ok`
// false for a group without a row: it still takes part in the shuffles.
__device__ __forceinline__ void merge_splits_and_finish(const VerifyPartial *__restrict__ part, int S, long row,
                                                        bool row_ok, int sp, const uint8_t *__restrict__ mask,
                                                        int mode, float threshold, uint64_t seed, int kl_mode,
                                                        uint8_t *__restrict__ out_mask,
                                                        int32_t *__restrict__ out_tokens,
                                                        float *__restrict__ out_scores, const VerifyExtra &ex,
                                                        float *keep_score = nullptr, int *keep_token = nullptr)
{
    const bool have = row_ok && sp < S;                    // no early exit: the shuffles below need every lane
    VerifyPartial p;
    p.ref_d = kNegInf; p.s_d = 0.f; p.a = 0.f; p.best_v = kNegInf; p.s_v = 0.f; p.idx = INT_MAX; p.idx_d = INT_MAX;
    if (have) p = part[(size_t)row * S + sp];
    float mv = p.best_v, md = kNegInf;
    int idx = p.idx, idx_d = p.idx_d;
    double sv = 0.0, sd = 0.0, a = 0.0;
    // (KL's exchanges beside the verifier's, not after them: a sequence of 63 rows keeps sixteen waves busy with them, Eq. 6 on 3 x 63 rows
    // of 256 fp32 logits 10.7 us through LDS shuffles, 11.3 one after the other, 10.7 side by side; 3 x 48 rows 9.9, 9.9, 9.2)
    if (kl_mode) {                                         // uniform
        md = p.ref_d;
        for_steps<4>([&](auto step) __attribute__((always_inline)) {
            constexpr int STEP = decltype(step)::value;
            const float ov = other16<STEP>(mv), od = other16<STEP>(md);
            const int oi = other16<STEP>(idx), oid = other16<STEP>(idx_d);
            if (ov > mv || (ov == mv && oi < idx)) { mv = ov; idx = oi; }
            if (od > md || (od == md && oid < idx_d)) { md = od; idx_d = oid; }
        });
        if (p.best_v != kNegInf) sv = (double)p.s_v * exp((double)p.best_v - (double)mv);
        if (p.ref_d != kNegInf) {
            const double c = exp((double)p.ref_d - (double)md);
            sd = (double)p.s_d * c;
            a = (double)p.a * c;
        }
        for_steps<4>([&](auto step) __attribute__((always_inline)) {
            constexpr int STEP = decltype(step)::value;
            sv += other16<STEP>(sv);
            sd += other16<STEP>(sd);
            a += other16<STEP>(a);
        });
    } else {
        for_steps<4>([&](auto step) __attribute__((always_inline)) {
            constexpr int STEP = decltype(step)::value;
            const float ov = other16<STEP>(mv);
            const int oi = other16<STEP>(idx);
            if (ov > mv || (ov == mv && oi < idx)) { mv = ov; idx = oi; }
        });
        if (p.best_v != kNegInf) sv = (double)p.s_v * exp((double)p.best_v - (double)mv);
        for_steps<4>([&](auto step) __attribute__((always_inline)) { sv += other16<decltype(step)::value>(sv); });
    }
    if (sp == 0 && row_ok)
        finish_row((int)row, md, sd, a, mv, sv, idx, mask, mode, threshold, seed, kl_mode, out_mask, out_tokens,
                   out_scores, idx_d, ex, keep_score, keep_token);
}

__global__ __launch_bounds__(256) void verify_finalize_kernel(const VerifyPartial *__restrict__ part, int S, int P,
                                                              const uint8_t *__restrict__ mask, int mode,
                                                              float threshold, uint64_t seed, int kl_mode,
                                                              uint8_t *__restrict__ out_mask,
                                                              int32_t *__restrict__ out_tokens,
                                                              float *__restrict__ out_scores, VerifyExtra ex)
{
    const int gid = blockIdx.x * 256 + threadIdx.x;
    const int row = gid / kFinalizeLanes;
    merge_splits_and_finish(part, S, row, row < P, gid % kFinalizeLanes, mask, mode, threshold, seed, kl_mode, out_mask,
                            out_tokens, out_scores, ex);
}

// The state of a row that is finished where it is reduced, as the merge of split rows reads one: without a reference (no logit
// above -inf) its sums count as zero, so that a confidence is 1 / 0 and ranks, and is not a NaN that every rank ignores.
__device__ __forceinline__ WaveState as_merged(WaveState r)
{
    if (r.best_v == kNegInf) r.s_v = 0.f;
    if (r.ref_d == kNegInf) r.s_d = r.a = 0.f;
    return r;
}

// One workgroup per row: stream the whole row and finish it in the same kernel (no partial states,
// no second launch).  Used whenever there are enough rows to fill the chip with such workgroups, and (UNSPLIT) for fewer rows
// that are too short to split.
template <bool BF16, bool KL, int THREADS, bool TRACKD = false, bool UNSPLIT = false>
__global__ __launch_bounds__(THREADS) void verify_row_kernel(const uint4 *__restrict__ logits_d,
                                                             const uint4 *__restrict__ logits_v, int nvec,
                                                             const uint8_t *__restrict__ mask, int mode,
                                                             float threshold, uint64_t seed,
                                                             uint8_t *__restrict__ out_mask,
                                                             int32_t *__restrict__ out_tokens,
                                                             float *__restrict__ out_scores, VerifyExtra ex)
{
    const int row = blockIdx.x;
    const size_t rbase = (size_t)row * (size_t)nvec;
    WaveState r;
    if (reduce_range<BF16, KL, THREADS, TRACKD>(logits_v + rbase, KL ? logits_d + rbase : nullptr, 0, nvec, r)) {
        if (UNSPLIT) r = as_merged(r);
        finish_row(row, (double)r.ref_d, (double)r.s_d, (double)r.a, (double)r.best_v, (double)r.s_v, r.idx,
                   mask, mode, threshold, seed, KL ? 1 : 0, out_mask, out_tokens, out_scores, r.idx_d, ex);
    }
}

// Eq. 6: one workgroup per sequence sums the divergences of its eligible rows, then draws
template <int THREADS>
__device__ __forceinline__ void klprob_sequence(const float *__restrict__ scores, const uint8_t *__restrict__ mask,
                                                size_t base, int G, uint64_t seed, uint8_t *__restrict__ out_mask,
                                                double *red)
{
    const int tid = threadIdx.x;
    double local = 0.0;
    for (int g = tid; g < G; g += THREADS) {
        const float s = scores[base + g];
        if (mask[base + g] == 0 && s > 0.0f) local += (double)s;
    }
    red[tid] = local;
    __syncthreads();
    for (int o = THREADS / 2; o > 0; o >>= 1) {
        if (tid < o) red[tid] += red[tid + o];
        __syncthreads();
    }
    const double total = red[0];
    for (int g = tid; g < G; g += THREADS) {
        const size_t i = base + g;
        const float s = scores[i];
        const double k = s > 0.0f ? (double)s : 0.0;
        const double p = total > 0.0 ? k / total : 0.0;
        const bool remask = mask[i] == 0 && row_uniform(seed, (uint64_t)i) < p;
        out_mask[i] = (uint8_t)(mask[i] != 0 || remask);
    }
}

__global__ __launch_bounds__(256) void verify_klprob_kernel(const float *__restrict__ scores,
                                                            const uint8_t *__restrict__ mask, int G, uint64_t seed,
                                                            uint8_t *__restrict__ out_mask)
{
    __shared__ double red[256];
    klprob_sequence<256>(scores, mask, (size_t)blockIdx.x * G, G, seed, out_mask, red);
}

// Budgeted remasking: rank the eligible rows of a sequence by badness (KL: larger score, confidence: smaller
// score; equal scores: lower row first) and remask those of rank < k.  The rank of a row is the number of
// eligible rows of its sequence that are worse.  One workgroup takes 64 rows of one sequence, four lanes per
// row, each lane a quarter of the comparisons; the sequence's scores pass through LDS in chunks and are
// read back 16 bytes at a time (a scalar loop here is bound by the LDS latency of every single read).
constexpr int kTopkRows = 64, kTopkChunk = 2048;
// Rank of row g among the rows of its sequence whose mask byte equals `want` (the candidates), ordered by
// sign * score descending, equal values by row; -1 for a row that is no candidate.  Called by all THREADS lanes
// of a workgroup (it contains barriers); lanes 4r..4r+3 hold row r of the workgroup's THREADS / 4 and all four
// return its rank.
template <int THREADS>
__device__ __forceinline__ int sequence_rank(const float *__restrict__ scores, const uint8_t *__restrict__ mask,
                                             size_t base, int G, int g, uint8_t want, float sign, float *bad_sh)
{
    const int tid = threadIdx.x, sub = tid % 4;
    const bool candidate = g < G && mask[base + g] == want;
    const float bad = candidate ? sign * scores[base + g] : 0.0f;
    int rank = 0;
    for (int c0 = 0; c0 < G; c0 += kTopkChunk) {             // uniform trip count: every lane reaches the barriers
        const int n = min(kTopkChunk, G - c0), n16 = (n + 15) & ~15;
        __syncthreads();
        for (int j = tid; j < n16; j += THREADS)             // -inf marks a row that is no candidate
            bad_sh[j] = (j < n && mask[base + c0 + j] == want) ? sign * scores[base + c0 + j] : kNegInf;
        __syncthreads();
        if (candidate) {
#pragma unroll 4
            for (int j = 4 * sub; j < n16; j += 16) {
                const float4 o = *reinterpret_cast<const float4 *>(&bad_sh[j]);
                const int i = c0 + j;
                rank += (o.x > bad || (o.x == bad && i < g)) ? 1 : 0;
                rank += (o.y > bad || (o.y == bad && i + 1 < g)) ? 1 : 0;
                rank += (o.z > bad || (o.z == bad && i + 2 < g)) ? 1 : 0;
                rank += (o.w > bad || (o.w == bad && i + 3 < g)) ? 1 : 0;
            }
        }
    }
    rank += __shfl_xor(rank, 1);
    rank += __shfl_xor(rank, 2);
    return candidate ? rank : -1;
}

// rows [slab * THREADS / 4, + THREADS / 4) of the sequence at `base`; called by all lanes of a workgroup
template <int THREADS>
__device__ __forceinline__ void topk_slab(const float *__restrict__ scores, const uint8_t *__restrict__ mask,
                                          size_t base, int G, int slab, int kl_mode, float budget,
                                          uint8_t *__restrict__ out_mask, float *bad_sh)
{
    const int tid = threadIdx.x;
    const int g = slab * (THREADS / 4) + tid / 4;
    const int rank = sequence_rank<THREADS>(scores, mask, base, G, g, 0, kl_mode ? 1.0f : -1.0f, bad_sh);
    if (g < G && tid % 4 == 0) out_mask[base + g] = (uint8_t)(mask[base + g] != 0 || (rank >= 0 && (float)rank < budget));
}

__global__ __launch_bounds__(256) void verify_topk_kernel(const float *__restrict__ scores,
                                                          const uint8_t *__restrict__ mask, int G, int kl_mode,
                                                          float budget, uint8_t *__restrict__ out_mask)
{
    __shared__ __attribute__((aligned(16))) float bad_sh[kTopkChunk];
    const int slabs = (G + kTopkRows - 1) / kTopkRows;        // workgroups per sequence
    topk_slab<256>(scores, mask, (size_t)(blockIdx.x / slabs) * G, G, blockIdx.x % slabs, kl_mode, budget, out_mask, bad_sh);
}

// Drafter unmasking (Alg. 1, drafting phase): of the positions that still hold [MASK], those selected by
// confidence are decoded to the drafter's most likely token.  mode 0: confidence above the threshold, and
// always the most confident one of the sequence; mode 1: the k most confident ones.
template <int THREADS>
__device__ __forceinline__ void unmask_slab(const float *__restrict__ conf, const uint8_t *__restrict__ mask,
                                            const int32_t *__restrict__ tokens, size_t base, int G, int slab, int mode,
                                            float threshold, uint8_t *__restrict__ out_mask, int32_t *__restrict__ x,
                                            float *bad_sh)
{
    const int tid = threadIdx.x;
    const int g = slab * (THREADS / 4) + tid / 4;
    const int rank = sequence_rank<THREADS>(conf, mask, base, G, g, 1, 1.0f, bad_sh);
    if (g < G && tid % 4 == 0) {
        const bool take = rank >= 0 && (mode == 0 ? (rank == 0 || conf[base + g] > threshold) : (float)rank < threshold);
        out_mask[base + g] = (uint8_t)(mask[base + g] != 0 && !take);
        if (take && x) x[base + g] = tokens[base + g];
    }
}

__global__ __launch_bounds__(256) void unmask_select_kernel(const float *__restrict__ conf,
                                                            const uint8_t *__restrict__ mask,
                                                            const int32_t *__restrict__ tokens, int G, int mode,
                                                            float threshold, uint8_t *__restrict__ out_mask,
                                                            int32_t *__restrict__ x)
{
    __shared__ __attribute__((aligned(16))) float bad_sh[kTopkChunk];
    const int slabs = (G + kTopkRows - 1) / kTopkRows;
    unmask_slab<256>(conf, mask, tokens, (size_t)(blockIdx.x / slabs) * G, G, blockIdx.x % slabs, mode, threshold, out_mask,
                     x, bad_sh);
}

// Split path with a per-sequence rule (Eq. 6, the budgeted rules, the unmasking step): one workgroup per
// sequence first finishes the rows of its sequence from their partial states, then applies the rule to them
// - the second and third launch of such a call in one.  The split path has fewer than kFusedMinRows rows, so a sequence's scores,
// tokens and mask bytes stay in LDS between the two: reading them back from memory was a third of this kernel's time.
constexpr int kFusedMinRows = 192;            // calls of fewer rows split them over several workgroups each
constexpr int kSeqThreads = 1024, kSeqMaxRows = kFusedMinRows;
static_assert(kSeqMaxRows % 64 == 0 && kSeqMaxRows <= 2 * (kSeqThreads / 8), "whole waves of rows, ranked in two passes at most");
struct SequenceShared {
    __attribute__((aligned(16))) float score[kSeqMaxRows], bad[kSeqMaxRows];
    double red[kSeqThreads / 64];
    int token[kSeqMaxRows];
    uint8_t mask[kSeqMaxRows];
};

// The rule of one sequence, rows [base, base + G), whose scores and tokens are in `sh` (a barrier after they were written is part of
// this); lane g holds row g's mask byte.  Called by all lanes of the workgroup.
__device__ __forceinline__ void apply_sequence_rule(SequenceShared &sh, uint8_t mbyte, size_t base, int G, int mode, float threshold,
                                                    uint64_t seed, int kl_mode, uint8_t *__restrict__ out_mask,
                                                    int32_t *__restrict__ x_tokens)
{
    const int tid = threadIdx.x;
    if (tid < G) sh.mask[tid] = mbyte;
    __syncthreads();
    if (mode == 3) {                                         // Eq. 6: sum of the eligible rows' divergences, then the draws
        const float s = tid < G ? sh.score[tid] : 0.f;
        const double k = s > 0.0f ? (double)s : 0.0;
        double local = mbyte == 0 ? k : 0.0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) local += __shfl_xor(local, o);
        if ((tid & 63) == 0) sh.red[tid >> 6] = local;
        __syncthreads();
        double total = 0.0;
        for (int w = 0; w < kSeqMaxRows / 64; ++w) total += sh.red[w];       // (later waves hold no row)
        if (tid < G) {
            const double p = total > 0.0 ? k / total : 0.0;
            const bool remask = mbyte == 0 && row_uniform(seed, (uint64_t)(base + tid)) < p;
            out_mask[base + tid] = (uint8_t)(mbyte != 0 || remask);
        }
        return;
    }
    // the other rules rank the candidates of the sequence (see sequence_rank): rows still masked (unmasking) or decoded
    const bool unmasking = mode == kModeUnmaskThresh || mode == kModeUnmaskTopk;
    const bool candidate = tid < G && (mbyte != 0) == unmasking && (!unmasking || mbyte == 1);
    const float sign = unmasking || kl_mode ? 1.0f : -1.0f;
    const int n16 = (G + 15) & ~15;
    if (tid < n16) sh.bad[tid] = candidate ? sign * sh.score[tid] : kNegInf;
    __syncthreads();
    // eight lanes per row, each a part of the comparisons: passes of 128 rows
    const float budget = mode == kModeUnmaskThresh ? 0.f : floorf(threshold);
    for (int g0 = 0; g0 < G; g0 += kSeqThreads / 8) {
        const int g = g0 + tid / 8, sub = tid % 8;
        const float bad = g < G ? sh.bad[g] : kNegInf;
        int rank = 0;
        for (int j = 4 * sub; j < n16; j += 32) {
            const float4 o = *reinterpret_cast<const float4 *>(&sh.bad[j]);
            rank += (o.x > bad || (o.x == bad && j < g)) ? 1 : 0;
            rank += (o.y > bad || (o.y == bad && j + 1 < g)) ? 1 : 0;
            rank += (o.z > bad || (o.z == bad && j + 2 < g)) ? 1 : 0;
            rank += (o.w > bad || (o.w == bad && j + 3 < g)) ? 1 : 0;
        }
        rank += other16<0>(rank);
        rank += other16<1>(rank);
        rank += other16<2>(rank);
        if (g < G && sub == 0) {
            const uint8_t m = sh.mask[g];
            const bool is = unmasking ? m == 1 : m == 0;
            if (unmasking) {
                const bool take = is && (mode == kModeUnmaskThresh ? (rank == 0 || sh.score[g] > threshold) : (float)rank < budget);
                out_mask[base + g] = (uint8_t)(m != 0 && !take);
                if (take && x_tokens) x_tokens[base + g] = sh.token[g];
            } else {
                out_mask[base + g] = (uint8_t)(m != 0 || (is && (float)rank < budget));
            }
        }
    }
}

__global__ __launch_bounds__(kSeqThreads) void verify_finalize_seq_kernel(const VerifyPartial *__restrict__ part, int S, int G,
                                                                  const uint8_t *__restrict__ mask, int mode,
                                                                  float threshold, uint64_t seed, int kl_mode,
                                                                  uint8_t *__restrict__ out_mask,
                                                                  int32_t *__restrict__ out_tokens,
                                                                  float *__restrict__ out_scores,
                                                                  int32_t *__restrict__ x_tokens)
{
    __shared__ SequenceShared sh;
    const int tid = threadIdx.x;
    const size_t base = (size_t)blockIdx.x * G;
    const uint8_t mbyte = tid < G ? mask[base + tid] : 0;    // (requested with the states)
    constexpr int kRowsPerPass = kSeqThreads / kFinalizeLanes;
    for (int g0 = 0; g0 < G; g0 += kRowsPerPass) {           // uniform trip count
        const int g = g0 + tid / kFinalizeLanes;
        merge_splits_and_finish(part, S, (long)base + g, g < G, tid % kFinalizeLanes, mask, mode, threshold, seed, kl_mode,
                                out_mask, out_tokens, out_scores, VerifyExtra{}, &sh.score[min(g, G - 1)], &sh.token[min(g, G - 1)]);
    }
    apply_sequence_rule(sh, mbyte, base, G, mode, threshold, seed, kl_mode, out_mask, x_tokens);
}

// One row on one wave, in the arithmetic of the kThreads-lane workgroup that reduces it elsewhere (reduce_range), so that a score is
// the same number, bit for bit, whichever rule asks for it: what wave p reads there - the vectors 64 p .. of every kThreads - is
// part p here, with a reference and sums of its own, and lane p writes its state (idx: the whole row's).
constexpr int kParts = kThreads / 64;
static_assert(kParts == 4, "reductions of four values");
template <bool BF16, bool KL>
__device__ __forceinline__ void reduce_row_on_wave(const uint4 *__restrict__ pv, const uint4 *__restrict__ pd, int nvec, int lane,
                                                   WaveState *parts)
{
#pragma clang fp contract(off)                               // (a product rescaled by consume() is rounded before it is added to)
    constexpr int E = VecTraits<BF16>::kElems;
    float best_v[kParts], s_v[kParts], ref_d[kParts], s_d[kParts], a[kParts];
#pragma unroll
    for (int p = 0; p < kParts; ++p) {
        best_v[p] = ref_d[p] = kNegInf;
        s_v[p] = s_d[p] = a[p] = 0.f;
    }
    float top = kNegInf;                                     // this lane's largest verifier logit, the vector that has it first
    uint4 top_vec = make_uint4(0, 0, 0, 0);
    int top_at = 0;
    for (int v0 = 0; v0 < nvec; v0 += kThreads) {
        uint4 rv[kParts], rd[kParts];
        bool ok[kParts];
#pragma unroll
        for (int p = 0; p < kParts; ++p) {
            const int idx = v0 + p * 64 + lane;
            ok[p] = idx < nvec;
            rv[p] = rd[p] = make_uint4(0, 0, 0, 0);
            if (ok[p]) {
                rv[p] = stream_load16(pv + idx);
                if (KL) rd[p] = stream_load16(pd + idx);
            }
        }
        float mv[kParts], md[kParts];
#pragma unroll
        for (int p = 0; p < kParts; ++p) {
            float x[E];
            VecTraits<BF16>::unpack(rv[p], x);
            float m = x[0];
#pragma unroll
            for (int e = 1; e < E; ++e) m = fmaxf(m, x[e]);
            mv[p] = ok[p] ? m : kNegInf;
            if (mv[p] > top) {
                top = mv[p];
                top_vec = rv[p];
                top_at = v0 + p * 64 + lane;
            }
            if (KL) {
                VecTraits<BF16>::unpack(rd[p], x);
                m = x[0];
#pragma unroll
                for (int e = 1; e < E; ++e) m = fmaxf(m, x[e]);
                md[p] = ok[p] ? m : kNegInf;
            }
        }
        wave_max4(mv, lane);
        if (KL) wave_max4(md, lane);
#pragma unroll
        for (int p = 0; p < kParts; ++p) {
            if (v0 > 0) s_v[p] *= rescale_factor(best_v[p], fmaxf(best_v[p], mv[p]));         // (one where the reference stays)
            best_v[p] = fmaxf(best_v[p], mv[p]);
            if (KL) {
                if (v0 > 0) {
                    const float c = rescale_factor(ref_d[p], fmaxf(ref_d[p], md[p]));
                    s_d[p] *= c;
                    a[p] *= c;
                }
                ref_d[p] = fmaxf(ref_d[p], md[p]);
            }
            if (ok[p]) {
                float xv[E], xd[E];
                VecTraits<BF16>::unpack(rv[p], xv);
                const float m = best_v[p] * kLog2e;
                float acc = 0.f;
#pragma unroll
                for (int e = 0; e < E; ++e) acc += fast_exp2(fmaf(xv[e], kLog2e, -m));
                s_v[p] += acc;
                if (KL) {
                    VecTraits<BF16>::unpack(rd[p], xd);
                    const float n = ref_d[p] * kLog2e;
                    float accs = 0.f, acca = 0.f;
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        const float ed = fast_exp2(fmaf(xd[e], kLog2e, -n));
                        accs += ed;
                        acca = fmaf(ed, xd[e] - xv[e], acca);
                    }
                    s_d[p] += accs;
                    a[p] += acca;
                }
            }
        }
    }
    float all = best_v[0];
#pragma unroll
    for (int p = 1; p < kParts; ++p) all = fmaxf(all, best_v[p]);
    int cand = INT_MAX;
    if (top == all && all != kNegInf) {
        float x[E];
        VecTraits<BF16>::unpack(top_vec, x);
#pragma unroll
        for (int e = E - 1; e >= 0; --e)
            if (x[e] == all) cand = top_at * E + e;
    }
    const int idx = wave_min(cand);
    WaveState w;
    w.s_v = wave_sum4(s_v, lane);
    w.s_d = KL ? wave_sum4(s_d, lane) : 0.f;
    w.a = KL ? wave_sum4(a, lane) : 0.f;
    w.idx = idx;
    w.idx_d = INT_MAX;
    w.best_v = best_v[0];
    w.ref_d = ref_d[0];
#pragma unroll
    for (int p = 1; p < kParts; ++p)
        if (lane == p) {
            w.best_v = best_v[p];
            w.ref_d = ref_d[p];
        }
    if (lane < kParts) parts[lane] = w;
}

// A per-sequence rule on few short rows, in one launch: a workgroup per sequence whose sixteen waves take whole rows and then
// apply the rule.  Such a call is launches and round trips; seq_rounds says where it wins.
template <bool BF16, bool KL>
__global__ __launch_bounds__(kSeqThreads) void verify_seq_kernel(const uint4 *__restrict__ logits_d, const uint4 *__restrict__ logits_v,
                                                                 int nvec, int G, const uint8_t *__restrict__ mask, int mode,
                                                                 float threshold, uint64_t seed, uint8_t *__restrict__ out_mask,
                                                                 int32_t *__restrict__ out_tokens, float *__restrict__ out_scores,
                                                                 int32_t *__restrict__ x_tokens)
{
    __shared__ SequenceShared sh;
    __shared__ WaveState rows_sh[kSeqMaxRows][kParts];
    const int tid = threadIdx.x, lane = tid & 63;
    const size_t base = (size_t)blockIdx.x * G;
    const uint8_t mbyte = tid < G ? mask[base + tid] : 0;
    for (int g = tid >> 6; g < G; g += kSeqThreads / 64)
        reduce_row_on_wave<BF16, KL>(logits_v + (base + g) * nvec, KL ? logits_d + (base + g) * nvec : nullptr, nvec, lane, rows_sh[g]);
    __syncthreads();
    if (tid < G) {                                           // G <= kSeqMaxRows: a lane per row
        WaveState r = rows_sh[tid][0];
        if (nvec > 64) {                                     // uniform (a part without a vector adds nothing)
#pragma unroll
            for (int p = 1; p < kParts; ++p) r = merge(r, rows_sh[tid][p]);
        }
        r = as_merged(r);
        finish_row((int)base + tid, (double)r.ref_d, (double)r.s_d, (double)r.a, (double)r.best_v, (double)r.s_v, r.idx, mask, mode,
                   threshold, seed, KL ? 1 : 0, out_mask, out_tokens, out_scores, 0, VerifyExtra{}, &sh.score[tid], &sh.token[tid]);
    }
    apply_sequence_rule(sh, mbyte, base, G, mode, threshold, seed, KL ? 1 : 0, out_mask, x_tokens);
}

}  // namespace

// Rows are handled by one workgroup each (fused finish) once there are enough of them to occupy the
// chip; the workgroup grows as the row count shrinks so that the bytes in flight stay about constant.
int verify_fused_threads(int P)
{
    if (P < kFusedMinRows) return 0;               // too few rows: split them over several workgroups instead
    return P >= 2048 ? 256 : 512;        // measured: 512 lanes per row stream best for 256..1024 rows
}

// A row's splits.  Where sixteen splits of every row still leave each workgroup a compute unit of its own, a split is as short as kThreads
// vectors allow: what a workgroup folds (a ragged load round, or full ones and a ragged one) is then the call.  us per call, KL: 4 x 32000
// 7.1 -> 5.7, 16 x 16384 7.9 -> 6.5, 20 x 20000 7.9 -> 6.7; unmasking 4 x 32000 6.4 -> 5.6.  Past a workgroup per unit it turns: KL
// 20 x 152064 (300 workgroups for 200) 9.8 -> 10.6, 32 x 65536 (512 for 256) 8.6 -> 8.8.
// Otherwise a split is a whole number of full load rounds (kThreads * kUnroll vectors), so that only the last of a row is ragged: every
// round of a workgroup is a dependent memory round trip, and with few rows those round trips are the call.  These are also what a call
// takes whose workspace does not hold the states of shorter ones.  A row of one such round is not split.
constexpr int kRowWorkgroups = 2048, kMaxRowSplits = 16, kFineWorkgroups = 256;      // (about 2048 workgroups in all)
struct RowSplits { int count, chunk; };              // of a row; vectors in each
static RowSplits row_splits(int P, int V, int elem_bytes, size_t workspace_bytes)
{
    const long nvec = (long)V * elem_bytes / 16, iter = (long)kThreads * kUnroll;
    if (nvec <= iter) return RowSplits{1, (int)iter};
    long s = (kRowWorkgroups + P - 1) / P;
    if (s > kMaxRowSplits) s = kMaxRowSplits;
    if (s < 1) s = 1;
    const long shortest = (nvec + s - 1) / s;
    auto of = [&](long multiple) {
        const long chunk = (shortest + multiple - 1) / multiple * multiple;
        return RowSplits{(int)((nvec + chunk - 1) / chunk), (int)chunk};
    };
    const RowSplits fine = of(kThreads);
    const long states = (long)P * fine.count;
    return states <= tune("DD_TUNE_VERIFY_FINE", kFineWorkgroups) && states * sizeof(VerifyPartial) <= workspace_bytes ? fine : of(iter);
}

// Dependent load rounds of verify_seq_kernel (sixteen rows of kThreads vectors each), and up to how many it is taken: a round costs
// its one workgroup 2 us (KL 4), the launch that it saves 3.  us per call in a stream of them, two launches -> one, fp32:
// unmasking 16 x 1024 7.1 -> 4.7, 16 x 2048 or 32 x 1024 (two rounds) 7.4 -> 6.4 - 6.8; Eq. 6 16 x 1024 8.0 -> 7.7.
static int seq_rounds(int G, int nvec)
{
    return (G + kSeqThreads / 64 - 1) / (kSeqThreads / 64) * ((nvec + kThreads - 1) / kThreads);
}
constexpr int kSeqMaxRounds = 2, kSeqMaxRoundsKl = 1;
// A bf16 vector is eight logits, so full rounds of them take longer: above 5120 vectors per sequence (KL 2560) two launches are as
// fast or faster - unmasking 29 x 1744 8.1 against 8.7, 32 x 1480 7.7 / 8.2, KL 13 x 1552 7.9 / 8.3, 13 x 1832 8.1 / 8.6.
static bool seq_in_one_launch(int G, int nvec, bool bf16, bool kl)
{
    const int forced = tune("DD_TUNE_SEQ_ROUNDS", -1), rounds = seq_rounds(G, nvec);
    if (forced >= 0) return rounds <= forced;
    return rounds <= (kl ? kSeqMaxRoundsKl : kSeqMaxRounds) && (!bf16 || (long)G * nvec <= (kl ? 2560 : 5120));
}

// The most states that any count of rows up to P has, so that a size queried for P rows, up to 191, serves fewer: where one more row lowers
// the splits, its states can be half of what one row less has (126464 bf16 logits, 136 rows 16 splits, 137 rows 8).
size_t verify_workspace_bytes(int P, int V, int elem_bytes)
{
    if (P <= 0 || verify_fused_threads(P) != 0) return 0;
    const long nvec = (long)V * elem_bytes / 16;
    long most = (long)P * row_splits(P, V, elem_bytes, SIZE_MAX).count;
    if (nvec > (long)kThreads * kUnroll) {
        const long fine = P * row_splits(1, V, elem_bytes, SIZE_MAX).count;
        most = std::max(most, std::min(fine, (long)kFineWorkgroups));
        for (int s = kMaxRowSplits; s > 1; --s) {
            const int last = (kRowWorkgroups + s - 2) / (s - 1) - 1;             // the most rows that are split s times
            if (last >= P) break;
            most = std::max(most, (long)last * row_splits(last, V, elem_bytes, 0).count);
        }
    }
    return (size_t)most * sizeof(VerifyPartial);
}

size_t verify_least_workspace_bytes(int P, int V, int elem_bytes)
{
    if (P <= 0 || verify_fused_threads(P) != 0) return 0;
    return (size_t)P * (size_t)row_splits(P, V, elem_bytes, 0).count * sizeof(VerifyPartial);
}

template <bool BF16, bool KL, bool TRACKD = false>
static hipError_t launch_row_kernel(int threads, dim3 grid, hipStream_t stream, const uint4 *ld, const uint4 *lv,
                                    int nvec, const uint8_t *mask, int mode, float threshold, uint64_t seed,
                                    uint8_t *out_mask, int32_t *out_tokens, float *out_scores, VerifyExtra ex)
{
    if (threads == 256)
        return launch(verify_row_kernel<BF16, KL, 256, TRACKD>, grid, dim3(256), stream, ld, lv, nvec, mask, mode,
                      threshold, seed, out_mask, out_tokens, out_scores, ex);
    return launch(verify_row_kernel<BF16, KL, 512, TRACKD>, grid, dim3(512), stream, ld, lv, nvec, mask, mode,
                  threshold, seed, out_mask, out_tokens, out_scores, ex);
}

hipError_t launch_verify(const void *logits_d, const void *logits_v, const uint8_t *mask,
                         int mode, float threshold, uint64_t seed,
                         uint8_t *out_mask, int32_t *out_tokens, float *out_scores,
                         int B, int G, int V, int logit_is_bf16, void *workspace, size_t workspace_bytes, hipStream_t stream,
                         int32_t *x_tokens, const VerifyExtra *extra)
{
    const int P = B * G;
    if (P == 0) return hipSuccess;
    const int eb = logit_is_bf16 ? 2 : 4;
    const int nvec = (int)((long)V * eb / 16);
    const bool kl = (mode == 1 || mode == 3 || mode == 5 || mode == kModeScores);
    const VerifyExtra ex = extra ? *extra : VerifyExtra{};
    const uint4 *ld = static_cast<const uint4 *>(logits_d);
    const uint4 *lv = static_cast<const uint4 *>(logits_v);
    hipError_t e;
    const int fused = verify_fused_threads(P);
    const bool track_d = mode == kModeScores && ex.tok_d != nullptr;     // the drafter's argmax is wanted as well
    if (fused != 0 && track_d) {
        const dim3 grid((unsigned)P);
        e = logit_is_bf16 ? launch_row_kernel<true, true, true>(fused, grid, stream, ld, lv, nvec, mask, mode, threshold, seed, out_mask, out_tokens, out_scores, ex)
                          : launch_row_kernel<false, true, true>(fused, grid, stream, ld, lv, nvec, mask, mode, threshold, seed, out_mask, out_tokens, out_scores, ex);
    } else if (fused != 0) {
        const dim3 grid((unsigned)P);
        if (logit_is_bf16)
            e = kl ? launch_row_kernel<true, true>(fused, grid, stream, ld, lv, nvec, mask, mode, threshold, seed, out_mask, out_tokens, out_scores, ex)
                   : launch_row_kernel<true, false>(fused, grid, stream, ld, lv, nvec, mask, mode, threshold, seed, out_mask, out_tokens, out_scores, ex);
        else
            e = kl ? launch_row_kernel<false, true>(fused, grid, stream, ld, lv, nvec, mask, mode, threshold, seed, out_mask, out_tokens, out_scores, ex)
                   : launch_row_kernel<false, false>(fused, grid, stream, ld, lv, nvec, mask, mode, threshold, seed, out_mask, out_tokens, out_scores, ex);
    } else {
        const RowSplits split = row_splits(P, V, eb, workspace_bytes);
        const int S = split.count, chunk = split.chunk;
        VerifyPartial *part = static_cast<VerifyPartial *>(workspace);
        const dim3 grid((unsigned)((long)P * S)), block(kThreads);
        const bool per_sequence = mode == 3 || mode == 5 || mode == 6 || mode == kModeUnmaskThresh || mode == kModeUnmaskTopk;
        // Rows that are not split leave nothing to merge: rules of one row finish it in the launch that streams it, ...
        if (S == 1 && !per_sequence && !track_d) {
            const dim3 rows((unsigned)P), lanes(kThreads);
            if (logit_is_bf16)
                return kl ? launch(verify_row_kernel<true, true, kThreads, false, true>, rows, lanes, stream, ld, lv, nvec, mask, mode, threshold, seed, out_mask, out_tokens, out_scores, ex)
                          : launch(verify_row_kernel<true, false, kThreads, false, true>, rows, lanes, stream, ld, lv, nvec, mask, mode, threshold, seed, out_mask, out_tokens, out_scores, ex);
            return kl ? launch(verify_row_kernel<false, true, kThreads, false, true>, rows, lanes, stream, ld, lv, nvec, mask, mode, threshold, seed, out_mask, out_tokens, out_scores, ex)
                      : launch(verify_row_kernel<false, false, kThreads, false, true>, rows, lanes, stream, ld, lv, nvec, mask, mode, threshold, seed, out_mask, out_tokens, out_scores, ex);
        }
        // ... rules of a sequence stream its rows in the workgroup that applies the rule, as long as that is a few round trips
        if (S == 1 && per_sequence && seq_in_one_launch(G, nvec, logit_is_bf16 != 0, kl)) {
            const dim3 seqs((unsigned)B), lanes(kSeqThreads);
            if (logit_is_bf16)
                return kl ? launch(verify_seq_kernel<true, true>, seqs, lanes, stream, ld, lv, nvec, G, mask, mode, threshold, seed, out_mask, out_tokens, out_scores, x_tokens)
                          : launch(verify_seq_kernel<true, false>, seqs, lanes, stream, ld, lv, nvec, G, mask, mode, threshold, seed, out_mask, out_tokens, out_scores, x_tokens);
            return kl ? launch(verify_seq_kernel<false, true>, seqs, lanes, stream, ld, lv, nvec, G, mask, mode, threshold, seed, out_mask, out_tokens, out_scores, x_tokens)
                      : launch(verify_seq_kernel<false, false>, seqs, lanes, stream, ld, lv, nvec, G, mask, mode, threshold, seed, out_mask, out_tokens, out_scores, x_tokens);
        }
        if (track_d) {
            e = logit_is_bf16 ? launch(verify_partial_kernel<true, true, true>, grid, block, stream, ld, lv, nvec, S, chunk, part)
                              : launch(verify_partial_kernel<false, true, true>, grid, block, stream, ld, lv, nvec, S, chunk, part);
        } else if (logit_is_bf16) {
            if (kl) e = launch(verify_partial_kernel<true, true>, grid, block, stream, ld, lv, nvec, S, chunk, part);
            else    e = launch(verify_partial_kernel<true, false>, grid, block, stream, ld, lv, nvec, S, chunk, part);
        } else {
            if (kl) e = launch(verify_partial_kernel<false, true>, grid, block, stream, ld, lv, nvec, S, chunk, part);
            else    e = launch(verify_partial_kernel<false, false>, grid, block, stream, ld, lv, nvec, S, chunk, part);
        }
        if (e != hipSuccess) return e;
        if (per_sequence)
            return launch(verify_finalize_seq_kernel, dim3((unsigned)B), dim3(kSeqThreads), stream, (const VerifyPartial *)part, S,
                          G, mask, mode, threshold, seed, kl ? 1 : 0, out_mask, out_tokens, out_scores, x_tokens);
        e = launch(verify_finalize_kernel, dim3((unsigned)(((long)P * kFinalizeLanes + 255) / 256)), dim3(256), stream,
                   (const VerifyPartial *)part, S, P, mask, mode, threshold, seed, kl ? 1 : 0, out_mask, out_tokens, out_scores,
                   ex);
    }
    if (e != hipSuccess) return e;
    if (mode == 3)
        e = launch(verify_klprob_kernel, dim3(B), dim3(256), stream, (const float *)out_scores, mask, G, seed, out_mask);
    if (mode == kModeUnmaskThresh || mode == kModeUnmaskTopk)
        // the pass above ran as for the Trust rule on the drafter's logits: confidence and argmax of every row
        return launch(unmask_select_kernel, dim3((unsigned)((long)((G + kTopkRows - 1) / kTopkRows) * B)), dim3(256),
                      stream, (const float *)out_scores, mask, (const int32_t *)out_tokens, G, mode - kModeUnmaskThresh,
                      mode == kModeUnmaskTopk ? floorf(threshold) : threshold, out_mask, x_tokens);
    if (mode == 5 || mode == 6)
        e = launch(verify_topk_kernel, dim3((unsigned)((long)((G + kTopkRows - 1) / kTopkRows) * B)), dim3(256), stream,
                   (const float *)out_scores, mask, G, kl ? 1 : 0, floorf(threshold), out_mask);
    return e;
}

}  // namespace dd

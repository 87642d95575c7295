// Attention of few query rows whose waves stream keys of their own: the drafter's call where workgroups of 32 rows are few or key
// streams short (Sec. 2.3) and small verifier calls (Sec. 2.2), bf16 or fp8 Q/K, bf16 or (with fp8 Q/K) e4m3 V.
//     O = softmax(Q K^T / sqrt(d_k)) V   (Eq. 3)
// One workgroup = four or eight waves on one or two blocks of 32 query rows; wave w takes every fourth (eighth) 32-key unit of the key
// range with a state (reference, sum, O) of its own, and the states are merged through LDS at the end, the waves sharing out the head dims.
//   - No K/V row is used by two waves, so none waits for another: a wave has one K and one V buffer in LDS, filled by
//     global_load_lds_dwordx4, waits for its own loads only, and asks for the next unit's K as soon as the fragments of this
//     one's are in registers, V likewise: all buffers are on their way nearly all the time.
//   - A block of 32 rows leaves no wave idle (the 64-row workgroups of attention_stream.hip halve there), and 64 rows are two
//     workgroups that share K/V through an XCD's L2.
//   - The head dims of V and O may be divided over 2 or 4 workgroups ("parts"), each with the whole of K: S is computed by all of
//     them, but there is no merge between them, and a call of few heads spreads over more compute units.
// What bounds it: some 4 us of launch, first loads and merge, then per unit a chain (K fragments, S, weights, V fragments, O) of
// 0.45 - 0.75 us that nothing else on the SIMD covers while a workgroup is four waves, and the 64 B/clk of a compute unit's path to LDS (100
// GB/s at most, measured).  Parts shorten a unit and the merge; a second wave per SIMD (eight waves) fills the chain's gaps where streams
// are long, for 0.3 - 0.8 us more of launch and merge; two row blocks share a unit's loads.  A form is named by its digits (row blocks, parts,
// waves).  us per call in a stream of them, 114 -> the form that the rule picks: 1 x 32 heads, 32 rows, 512 keys bf16 7.5 -> 5.9 (148), 1024
// keys bf16 9.6 -> 8.0, fp8 8.8 -> 6.7, e4m3 V 9.3 -> 6.9 (148); 4 x 32/8, 16 rows, 2048 keys fp8 10.4 -> 9.4 (124); 2 x 32, 48 rows, 800 keys
// e4m3 V 11.8 -> 8.1 (128); 11 x 32/8, 64 rows, 1237 keys e4m3 V 15.1 -> 12.3 (228), fp8 114 itself (11.45, 228 11.54).
// What the first loads need arrives in registers, as leading scalar arguments, and no hidden argument is asked for (the grid's size
// costs a launch 256 bytes more): with the arguments in a struct 1 x 32, 512 keys on 144 takes 6.8, so 6.2 us, 11 x 32/8 fp8 11.6 -> 11.2.
// Tried and not kept: a second unit on its way per wave (bf16 8.0 -> 9.4, 4 parts 6.8 -> 7.6: the first units' loads queue behind it); two
// blocks with all dims (12.3, one wave's registers); eight waves on all dims for bf16 (8.6).
#include "attention_common.h"
#include "dd_internal.h"

#include <type_traits>

namespace dd {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef int intx8 __attribute__((ext_vector_type(8)));
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

[[maybe_unused]] constexpr float kSoloMargin = 7.0f;     // a reference is set this far above a unit's maximum (log2 units)

__device__ __forceinline__ float solo_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ unsigned solo_pack(float lo, float hi)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    floatx2 f = {lo, hi};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2));
}
__device__ __forceinline__ u32x2 solo_swap(unsigned a, unsigned b)       // {a.lo, b.lo}, {a.hi, b.hi} by lane halves
{
    return __builtin_amdgcn_permlane32_swap(a, b, false, false);
}
__device__ __forceinline__ const uint8_t *solo_scalar(const uint8_t *p)          // a uniform address, in scalar registers
{
    const unsigned long long v = reinterpret_cast<unsigned long long>(p);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return reinterpret_cast<const uint8_t *>(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ uint4 solo_decode(unsigned w0, unsigned w1)           // eight e4m3 codes to bf16, exactly
{
    return make_uint4(__builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w0, 1.0f, false)),
                      __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w0, 1.0f, true)),
                      __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w1, 1.0f, false)),
                      __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w1, 1.0f, true)));
}
template <int I, int N, typename F> __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// V8: V is stored as e4m3 codes.  They travel to LDS as they are and the wave decodes its own 4 KB into its V buffer, exactly, when
// they arrive (32 conversions of two elements per lane and unit); v_scale multiplies the result once.
// RB row blocks per workgroup, VP parts of the head dims, NW waves.
template <int D, bool FP8, bool V8, int RB, int VP, int NW>
__device__ __forceinline__ void attn_solo(const AttnHead &h, const AttnTail &a)
{
    // (device pass only: the host pass needs the kernels' handles, not assembly it cannot check)
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int U = 32;               // keys per unit
    constexpr int DV = D / VP;                       // head dims of V / O that this workgroup handles
    constexpr int CH = DV / 8;                       // 16-byte chunks per V row in LDS
    constexpr int DC = DV / 32;                      // 32-wide chunks of its head dims
    constexpr int ROWB = DV * 2;                     // bytes per V row in LDS
    constexpr int KROWB = FP8 ? D : D * 2, KCH = KROWB / 16;   // Q / K as stored: bytes and chunks per row
    constexpr int KF = KROWB / 32;                   // 16-byte K fragments per lane and unit
    constexpr int KB = U * KROWB, VB = U * ROWB;     // bytes of a wave's K / V buffer
    constexpr int VPITCH = V8 ? D : D * 2;           // bytes between V rows in memory
    constexpr int VSROWB = V8 ? DV : ROWB, VSCH = VSROWB / 16, VSB = V8 ? U * VSROWB : 0;   // V as stored; its own buffer if decoded
    constexpr int NK = KB / 1024, NV = U * VSROWB / 1024;                    // wave-wide loads per buffer (1 KB each)
    constexpr int VDMA_ROWS = 1024 / VSROWB, KDMA_ROWS = 1024 / KROWB;       // rows per load
    constexpr int GB = DC * 4, GP = RB * GB >= NW ? RB * GB / NW : 1;   // groups of four O registers per lane and row block, ... that a wave finishes
    static_assert((!FP8 && !V8) || (FP8 && D == 128), "fp8 rows are 128 bytes");
    static_assert(RB == 1 || RB == 2, "a wave finishes groups of one row block");
    static_assert(NV >= 1 && GP >= 1, "not too many parts");
    static_assert(NK <= 8 && NV <= 8, "a buffer is within the loads' immediate offsets");
    constexpr int SLOTB = KB + VB + VSB;
    constexpr int NF = RB * GB < NW ? RB * GB : NW;  // waves that finish groups
    constexpr int PARKB = NW * (NF - 1 + (NF < NW)) * GP * 1024;             // the parked states share the buffers' memory
    constexpr int LDSB = (NW * SLOTB > PARKB ? NW * SLOTB : PARKB);
    // per wave: K [key][chunk ^ (key & 7)], then V [key][chunk ^ ((key % (CH/4)) << 2)]
    __shared__ __attribute__((aligned(1024))) uint4 KV[LDSB / 16];
    __shared__ __attribute__((aligned(1024))) uint4 QS[RB * KB / 16];        // the query rows, as K
    __shared__ float qs_sh[64];                      // the scales of the query rows
    __shared__ float ml_sh[NW][2][32 * RB];          // per wave: (reference, sum) of the query rows

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hh = lane >> 5;

    // ---- which (batch, kv head, row tile, key split); same XCD for workgroups that share K/V
    unsigned bid = blockIdx.x;
    {
        const unsigned total = h.wgs, per = total >> 3, rem = total & 7;
        const unsigned xcd = bid & 7, slot = bid >> 3;
        bid = xcd * per + min(xcd, rem) + slot;
    }
    const int part = bid % VP; bid /= VP;
    int rt, sp;
    place_of(bid, h.row_tiles, rt);
    place_of(bid, h.splits, sp);
    const size_t kv_head = bid;                      // batch and kv head
    const int rows_total = h.rows_total;             // query rows of this (batch, kv head): contiguous in memory
    const int v_first = rt * 32 * RB;
    const size_t row_base = kv_head * rows_total;
    auto lds_addr = [&](const void *p) __attribute__((always_inline)) { return (unsigned)(size_t)(__attribute__((address_space(3))) const void *)p; };
    const int krow0 = lane / KCH;
    auto kchunk = [&](int i) __attribute__((always_inline)) { return (unsigned)(((lane % KCH) ^ ((i * KDMA_ROWS + krow0) & 7)) * 16); };

    // ---- the query rows, shared out over the waves: first, as they need nothing that is still on its way
    for (int i = wave; i < RB * NK; i += NW) {
        const int r = min(v_first + i * KDMA_ROWS + krow0, rows_total - 1);
        const uint8_t *const src = h.Q + (row_base + r) * KROWB + kchunk(i);
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr(QS) + i * 1024), "v"(src) : "memory", "m0");
    }

    const int kbeg = sp * h.keys_per_split;
    const int kend = min(h.N, kbeg + h.keys_per_split);
    // (any value is safe: rows are chosen by range test)
    const int bstart = a.block_starts ? uniform_load(a.block_starts + (unsigned)kv_head / (unsigned)a.Hkv) : h.block_start;
    const int blen = h.block_len;
    const int nunits = (kend - kbeg + U - 1) / U;
    const int whole = (kend - kbeg) / U;             // units [0, whole) hold 32 rows of the range

    const uint8_t *const kc = h.K + kv_head * h.kv_stride * (size_t)KROWB;
    const uint8_t *const vc = h.V + kv_head * h.kv_stride * (size_t)VPITCH + part * VSROWB;
    const uint8_t *const kb_ = blen ? static_cast<const uint8_t *>(a.Kblk) + kv_head * blen * (size_t)KROWB : nullptr;
    const uint8_t *const vb_ = blen ? static_cast<const uint8_t *>(a.Vblk) + kv_head * blen * (size_t)VPITCH + part * VSROWB : nullptr;
    char *const kbuf = reinterpret_cast<char *>(KV) + wave * SLOTB, *const vbuf = kbuf + KB, *const vstored = vbuf + VB;
    const unsigned kdst = lds_addr(KV) + wave * SLOTB, vdst = kdst + KB + (V8 ? VB : 0);
    // load i of a buffer fills its rows i * DMA_ROWS ..; lane l lands at chunk position l % CH of row l / CH and fetches the
    // chunk the swizzle maps there (with 256-byte rows K's depends on whether i is odd)
    const int vrow0 = lane / VSCH;
    const unsigned vchunk = V8 ? lane % VSCH * 16 : ((lane % CH) ^ ((vrow0 & (CH / 4 - 1)) << 2)) * 16;   // (codes lie as in memory)
    const unsigned koff[2] = {krow0 * KROWB + kchunk(0), krow0 * KROWB + kchunk(1)}, voff = vrow0 * VPITCH + vchunk;
    int blk0 = 0, blk1 = 0;                          // units outside [blk0, blk1) hold rows of the cache only
    if (blen) {
        const long s0 = min(max((long)bstart, (long)kbeg), (long)kend), s1 = min(max((long)bstart + blen, (long)kbeg), (long)kend);
        if (s1 > s0) {
            blk0 = (int)(s0 - kbeg) / U;
            blk1 = ((int)(s1 - kbeg) + U - 1) / U;
        }
    }
    // One buffer's loads.  A unit of whole cache rows is contiguous in memory as in LDS: one scalar base and the instruction's
    // immediate, which counts on both sides.  Otherwise every lane chooses its row, and rows past the end of the range repeat
    // its last one (finite stand-ins, masked or zeroed below).
    auto load_rows = [&](auto is_k, int u) __attribute__((always_inline)) {
        constexpr bool K = decltype(is_k)::value;
        constexpr int NL = K ? NK : NV, BIAS = NL > 4 ? 4096 : 0, PITCH = K ? KROWB : VPITCH;
        constexpr bool PARTIAL = !K && VP > 1;       // part of a row: what lies together in LDS does not in memory
        const unsigned dst = (K ? kdst : vdst) + BIAS;
        const int k0 = kbeg + u * U;
        if (u < whole && (unsigned)(u - blk0) >= (unsigned)(blk1 - blk0)) {
            const uint8_t *const src = solo_scalar((K ? kc : vc) + (size_t)k0 * PITCH + BIAS);
            static_for<0, NL>([&](auto i) __attribute__((always_inline)) {
                constexpr int I = decltype(i)::value, IMM = I * 1024 - BIAS;
                const unsigned d = dst, o = K ? koff[I & 1] : voff;
                const uint8_t *const sbase = src;
                if constexpr (PARTIAL) {
                    const uint8_t *const at = sbase - BIAS + I * VDMA_ROWS * PITCH;
                    const unsigned di = d - BIAS + I * 1024;
                    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(di), "v"(o), "s"(at) : "memory", "m0");
                } else if constexpr (IMM >= 0)
                    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3" ::"s"(d), "v"(o), "s"(sbase), "n"(IMM) : "memory", "m0");
                else
                    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2 offset:-%3" ::"s"(d), "v"(o), "s"(sbase), "n"(-IMM) : "memory", "m0");
            });
        } else {
            static_for<0, NL>([&](auto i) __attribute__((always_inline)) {
                constexpr int I = decltype(i)::value;
                const int j = min(k0 + I * (K ? KDMA_ROWS : VDMA_ROWS) + (K ? krow0 : vrow0), kend - 1);
                const bool in_blk = (unsigned)j - (unsigned)bstart < (unsigned)blen;
                const uint8_t *const src = (K ? (in_blk ? kb_ : kc) : (in_blk ? vb_ : vc)) +
                                           (size_t)(in_blk ? j - bstart : j) * PITCH + (K ? kchunk(I) : vchunk);
                const unsigned d = dst - BIAS + I * 1024;
                asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(d), "v"(src) : "memory", "m0");
            });
        }
    };
    const std::true_type of_k;
    const std::false_type of_v;

    // ---- the rest of the prologue: the query rows' scales, this wave's first unit
    const float k_scale = a.k_scale ? uniform_load(a.k_scale + kv_head) : 1.0f;
    // (through LDS like the rows: the compiler's own wait for a load of its own would wait for every load after it as well)
    if (a.q_scale && wave == 0) {
        const float *const src = a.q_scale + kv_head * a.group + min(v_first + (RB == 2 ? lane : l32), rows_total - 1) / a.Nq;
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_addr(qs_sh)), "v"(src) : "memory", "m0");
    }
    if (wave < nunits) {
        load_rows(of_k, wave);
        load_rows(of_v, wave);
    }

    // operand addresses inside a unit's rows (bytes)
    int k_off[KF], v_off[DC];
#pragma unroll
    for (int f = 0; f < KF; ++f) k_off[f] = (l32 * KCH + ((2 * f + hh) ^ (l32 & 7))) * 16;
    {
        const int t = lane & 15, gq = l32 >> 4, row = 4 * hh + (t >> 2);
#pragma unroll
        for (int i = 0; i < DC; ++i) {
            const int chunk = 4 * i + 2 * gq + ((t & 3) >> 1);
            v_off[i] = (row * CH + (chunk ^ ((row & (CH / 4 - 1)) << 2))) * 16 + (t & 1) * 8;
        }
    }
    // (a wave without a unit has no later loads to leave outstanding)
    if (wave < nunits) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NK + NV) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile("s_barrier" ::: "memory");
    // Q fragments (B operand of S^T = K Q^T): lane (query l32, half hh) holds 16-byte chunk 2 f + hh of its row
    intx4 qf[RB][KF];
    float c[RB];                                     // scores are exponentiated as 2^(s*c)
    floatx16 acc[RB][DC];                            // O^T, unnormalised
#pragma unroll
    for (int q = 0; q < RB; ++q) {
#pragma unroll
        for (int f = 0; f < KF; ++f) qf[q][f] = *reinterpret_cast<const intx4 *>(reinterpret_cast<const char *>(QS) + q * KB + k_off[f]);
        c[q] = a.scale_log2 * k_scale;
        if (a.q_scale) c[q] *= qs_sh[32 * q + l32];
#pragma unroll
        for (int i = 0; i < DC; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[q][i][r] = 0.f;
    }
    // Row sums of the weights as multiplied (rounded to bf16), by the matrix instruction of sixteen 4 x 4 blocks: lane l is
    // column l % 4 of block l / 4 with four values of k, so with an A operand of ones every lane gets the sum of its own
    // weights; the lane halves hold different keys of a row and are added at the end.
    floatx4 acc_l[RB];
    const short4v ones = {0x3F80, 0x3F80, 0x3F80, 0x3F80};
    // The reference m of the weights p = 2^(s c - m), as -m (log2 units), equal in both lane halves.  It only has to be near the
    // running maximum (any common factor 2^-m cancels): the first unit sets it to its maximum + 7; a later one first takes its
    // weights with the one in use, and only if some weight reached 2 - one bit of its bf16 pattern, the packed weights are or-ed
    // together - it is raised to the unit's maximum + 7, the sums are scaled and the weights taken again.
    float nm[RB];
#pragma unroll
    for (int q = 0; q < RB; ++q) {
        acc_l[q] = floatx4{0.f, 0.f, 0.f, 0.f};
        nm[q] = INFINITY;
    }

    // ---- this wave's units.  Its loads complete in order: K and V of the unit, then the next unit's K, asked for when this one's
    // K is in registers, and its V, when this one's V is.
    for (int u = wave; u < nunits; u += NW) {
        const bool more = u + NW < nunits;           // uniform
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NV) : "memory");
        intx4 kf[KF];
#pragma unroll
        for (int f = 0; f < KF; ++f) kf[f] = *reinterpret_cast<const intx4 *>(kbuf + k_off[f]);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (more) load_rows(of_k, u + NW);
        floatx16 s[RB];
#pragma unroll
        for (int q = 0; q < RB; ++q)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[q][r] = 0.f;
        if constexpr (FP8) {
#pragma unroll
            for (int j = 0; j < KF / 2; ++j) {
                const intx8 kx = __builtin_shufflevector(kf[2 * j], kf[2 * j + 1], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                for (int q = 0; q < RB; ++q) {
                    const intx8 qx = __builtin_shufflevector(qf[q][2 * j], qf[q][2 * j + 1], 0, 1, 2, 3, 4, 5, 6, 7);
                    s[q] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(kx, qx, s[q], 0, 0, 0, 0x7F7F7F7F, 0, 0x7F7F7F7F);
                }
            }
        } else {
#pragma unroll
            for (int f = 0; f < KF; ++f)
#pragma unroll
                for (int q = 0; q < RB; ++q)
                    s[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[f]), __builtin_bit_cast(bf16x8, qf[q][f]), s[q], 0, 0, 0);
        }
        if (u == whole) {                            // (a unit with rows past the end of the range)
            // score register r is key key0 + 8 (r / 4) + 4 hh + (r % 4) for query row l32
            const int key0 = kbeg + u * U;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (key0 + 8 * (r >> 2) + 4 * hh + (r & 3) >= kend)
#pragma unroll
                    for (int q = 0; q < RB; ++q) s[q][r] = -INFINITY;
        }
        if (more) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NK) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if constexpr (V8) {
            // 16 codes of a row per load and lane, two 16-byte chunks of the row's bf16 form; rows past the end are zero (a weight of
            // zero times an infinity is a NaN)
            uint4 codes[NV];
#pragma unroll
            for (int i = 0; i < NV; ++i) codes[i] = *reinterpret_cast<const uint4 *>(vstored + i * 1024 + lane * 16);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (more) load_rows(of_v, u + NW);
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int row = i * VDMA_ROWS + vrow0, chunk = lane % VSCH * 2;
                const bool ok = u != whole || kbeg + u * U + row < kend;
                const uint4 lo = ok ? solo_decode(codes[i].x, codes[i].y) : make_uint4(0u, 0u, 0u, 0u);
                const uint4 hi = ok ? solo_decode(codes[i].z, codes[i].w) : make_uint4(0u, 0u, 0u, 0u);
                const int swz = (row & (CH / 4 - 1)) << 2;
                *reinterpret_cast<uint4 *>(vbuf + (row * CH + (chunk ^ swz)) * 16) = lo;
                *reinterpret_cast<uint4 *>(vbuf + (row * CH + ((chunk + 1) ^ swz)) * 16) = hi;
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        } else if (u == whole) {
            // V rows past the end have weight zero, but zero times an infinity is a NaN: zeroed by the lanes that loaded them
#pragma unroll
            for (int i = 0; i < NV; ++i)
                if (kbeg + u * U + i * VDMA_ROWS + vrow0 >= kend) *reinterpret_cast<uint4 *>(vbuf + i * 1024 + lane * 16) = make_uint4(0u, 0u, 0u, 0u);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
        // V^T fragments: dims 32 i + l32, keys 16 st + 4 hh + {0..3, 8..11} of the unit
        bf16x8 vf[2][DC];
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int i = 0; i < DC; ++i) {
                const char *p = vbuf + 16 * st * ROWB + v_off[i];
                const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v *)(p));
                const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v *)(p + 8 * ROWB));
                const short8v w = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                vf[st][i] = __builtin_bit_cast(bf16x8, w);
            }
        unsigned pk[RB][2][4], seen[RB];             // P^T as the B operand of O^T += V^T P^T
#pragma unroll
        for (int q = 0; q < RB; ++q) seen[q] = 0u;
        if (u != wave) {
#pragma unroll
            for (int q = 0; q < RB; ++q) {
#pragma unroll
                for (int r = 0; r < 16; r += 2)
                    pk[q][r >> 3][(r & 7) >> 1] = solo_pack(solo_exp2(fmaf(s[q][r], c[q], nm[q])), solo_exp2(fmaf(s[q][r + 1], c[q], nm[q])));
#pragma unroll
                for (int k = 0; k < 8; ++k) seen[q] |= pk[q][k >> 2][k & 3];
            }
        }
        // A row block at a time.  (With one test for both, peaked scores made two-block calls slower than one-block workgroups: 8 heads, 1679
        // keys, e4m3 V 24.5 us on those; here 21.9 with scores of deviation 1, 26.2 with 3, which take 24.2 a block at a time.)
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            if (u != wave && !__any((seen[q] & 0x40004000u) != 0u)) continue;        // uniform
            const u32x2 both = solo_swap(seen[q], seen[q]);
            const bool raise = u == wave || ((both.x | both.y) & 0x40004000u) != 0u;
            float mx = s[q][0];
#pragma unroll
            for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[q][r]);
            const u32x2 mm = solo_swap(__float_as_uint(mx), __float_as_uint(mx));
            mx = fmaxf(__uint_as_float(mm.x), __uint_as_float(mm.y)) * c[q] + kSoloMargin;
            const float m_old = -nm[q], m_new = raise ? fmaxf(m_old, mx) : m_old;
            const float corr = m_new == m_old ? 1.0f : solo_exp2(m_old - m_new);     // first unit: 2^(-inf) = 0
            const float use = m_new == -INFINITY ? 0.f : -m_new;                     // every score so far is -inf: weights 0
            nm[q] = -m_new;
            if (u != wave) {                         // (the first unit's sums are zero)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc_l[q][r] *= corr;
#pragma unroll
                for (int i = 0; i < DC; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[q][i][r] *= corr;
            }
#pragma unroll
            for (int r = 0; r < 16; r += 2)
                pk[q][r >> 3][(r & 7) >> 1] = solo_pack(solo_exp2(fmaf(s[q][r], c[q], use)), solo_exp2(fmaf(s[q][r + 1], c[q], use)));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (!V8 && more) load_rows(of_v, u + NW);
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int q = 0; q < RB; ++q) {
                const uint4 pw = make_uint4(pk[q][st][0], pk[q][st][1], pk[q][st][2], pk[q][st][3]);
#pragma unroll
                for (int i = 0; i < DC; ++i)
                    acc[q][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[st][i], __builtin_bit_cast(bf16x8, pw), acc[q][i], 0, 0, 0);
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const u32x2 half = {pk[q][st][2 * k], pk[q][st][2 * k + 1]};
                    acc_l[q] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones, __builtin_bit_cast(short4v, half), acc_l[q], 0, 0, 0);
                }
            }
    }

    // ---- merge the waves' states through LDS: a wave parks the groups of O registers that others finish
    __syncthreads();                                 // every wave is done with its buffers (and has no load outstanding)
    float4 *park = reinterpret_cast<float4 *>(KV);
    auto park_at = [&](int from, int to, int g) __attribute__((always_inline)) {
        return ((from * (NF - 1 + (NF < NW)) + (NF < NW || to < from ? to : to - 1)) * GP + g) * 64 + lane;
    };
#pragma unroll
    for (int q = 0; q < RB; ++q) {
        const u32x2 ls = solo_swap(__float_as_uint(acc_l[q][0]), __float_as_uint(acc_l[q][0]));
        ml_sh[wave][0][32 * q + l32] = -nm[q];
        ml_sh[wave][1][32 * q + l32] = __uint_as_float(ls.x) + __uint_as_float(ls.y);
    }
#pragma unroll
    for (int to = 0; to < NF; ++to)
        if (to != wave) {
#pragma unroll
            for (int g = 0; g < GP; ++g) {
                const int q = (to * GP + g) / GB, i = (to * GP + g) % GB / 4, r = 4 * ((to * GP + g) % 4);
                park[park_at(wave, to, g)] = make_float4(acc[q][i][r], acc[q][i][r + 1], acc[q][i][r + 2], acc[q][i][r + 3]);
            }
        }
    __syncthreads();
    if (NF < NW && wave >= NF) return;               // (uniform; no barrier follows)
    const int mine = wave * GP / GB;                 // the row block whose groups this wave finishes
    float m_all = -INFINITY, wgt[NW], l_tot = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) m_all = fmaxf(m_all, ml_sh[w][0][32 * mine + l32]);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float m = ml_sh[w][0][32 * mine + l32];
        wgt[w] = m == -INFINITY ? 0.f : solo_exp2(m - m_all);                // a wave that saw no key weighs nothing
        l_tot += ml_sh[w][1][32 * mine + l32] * wgt[w];
    }
    float o[GP][4], w_own = wgt[0];
#pragma unroll
    for (int w = 0; w < NF; ++w)
        if (w == wave) {
            w_own = wgt[w];
#pragma unroll
            for (int g = 0; g < GP; ++g)
#pragma unroll
                for (int k = 0; k < 4; ++k) o[g][k] = acc[(w * GP + g) / GB][(w * GP + g) % GB / 4][4 * ((w * GP + g) % 4) + k];
        }
#pragma unroll
    for (int g = 0; g < GP; ++g)
#pragma unroll
        for (int k = 0; k < 4; ++k) o[g][k] *= w_own;
#pragma unroll
    for (int w = 0; w < NW; ++w)
        if (w != wave) {
#pragma unroll
            for (int g = 0; g < GP; ++g) {
                const float4 x = park[park_at(w, wave, g)];
                o[g][0] += x.x * wgt[w]; o[g][1] += x.y * wgt[w]; o[g][2] += x.z * wgt[w]; o[g][3] += x.w * wgt[w];
            }
        }
    if constexpr (V8) {
        const float vs = uniform_load(a.v_scale + kv_head);         // the decoded values times this are the real ones
#pragma unroll
        for (int g = 0; g < GP; ++g)
#pragma unroll
            for (int k = 0; k < 4; ++k) o[g][k] *= vs;
    }
    // ---- output: group g of this wave is dims 8 (first + g) + 4 hh .. + 3 of query row l32 of its row block
    const int v = v_first + 32 * mine + l32, first = part * GB + wave * GP % GB;
    const bool row_ok = v < rows_total;
    const size_t orow = row_base + v;
    if (h.splits == 1) {
        const float inv = 1.0f / l_tot;
        uint16_t *out = static_cast<uint16_t *>(a.O) + orow * D;
        if constexpr (GP == 1) {
            if (row_ok)
                *reinterpret_cast<uint2 *>(out + 8 * first + 4 * hh) =
                    make_uint2(solo_pack(o[0][0] * inv, o[0][1] * inv), solo_pack(o[0][2] * inv, o[0][3] * inv));
        } else {
#pragma unroll
            for (int g = 0; g + 1 < GP; g += 2) {
                // the halves exchange words so that each lane stores eight consecutive dims
                const u32x2 x0 = solo_swap(solo_pack(o[g][0] * inv, o[g][1] * inv), solo_pack(o[g + 1][0] * inv, o[g + 1][1] * inv));
                const u32x2 x1 = solo_swap(solo_pack(o[g][2] * inv, o[g][3] * inv), solo_pack(o[g + 1][2] * inv, o[g + 1][3] * inv));
                if (row_ok) *reinterpret_cast<uint4 *>(out + 8 * (first + g + hh)) = make_uint4(x0.x, x1.x, x0.y, x1.y);
            }
        }
    } else if (row_ok) {
        float *po = a.part_o + (orow * h.splits + sp) * D;
#pragma unroll
        for (int g = 0; g < GP; ++g) *reinterpret_cast<float4 *>(po + 8 * (first + g) + 4 * hh) = make_float4(o[g][0], o[g][1], o[g][2], o[g][3]);
        if (hh == 0 && first == 0) {
            float *ml = a.part_ml + (orow * h.splits + sp) * 2;
            ml[0] = m_all;
            ml[1] = l_tot;
        }
    }
#endif
}

template <int D, bool FP8, bool V8, int RB, int VP, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_solo_kernel(DD_ATTN_HEAD, const AttnTail a)
{
    attn_solo<D, FP8, V8, RB, VP, NW>(DD_ATTN_HEAD_ARGS, a);
}

// The same launch with the block-completion copy on the workgroups past the attending ones: for a call without key splits, which has no
// merge launch to take it along.
template <int D, bool FP8, bool V8, int RB, int VP, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_solo_refresh_kernel(DD_ATTN_HEAD, const AttnTail a, const RefreshArgs r)
{
    if ((int)blockIdx.x >= wgs) {                            // uniform: these only copy
        refresh_cache_rows<64 * NW>(r);
        return;
    }
    attn_solo<D, FP8, V8, RB, VP, NW>(DD_ATTN_HEAD_ARGS, a);
}

template <int D, bool FP8, bool V8, int RB, int VP, int NW> hipError_t launch_solo(const AttnArgs &a, hipStream_t stream)
{
    AttnKernelArgs k;
    fill_kernel_args(a, k, 32 * RB, 32);
    k.wgs = (int)((long)a.B * a.Hkv * k.row_tiles * k.splits * VP);
    const dim3 block(64 * NW);
    RefreshArgs r{};
    const long copy_wgs = k.splits == 1 ? fill_refresh(a, r, kCopyWgs) : 0;
    if (copy_wgs > 0) {
        r.first_wg = k.wgs;
        return launch_headed(attn_solo_refresh_kernel<D, FP8, V8, RB, VP, NW>, dim3((unsigned)(k.wgs + copy_wgs)), block, stream, k, r);
    }
    const hipError_t e = launch_headed(attn_solo_kernel<D, FP8, V8, RB, VP, NW>, dim3((unsigned)k.wgs), block, stream, k);
    return e != hipSuccess ? e : finish_attention(a, k.splits, stream);
}
// `form`: row blocks, parts, waves as decimal digits.  (Each storage type has the forms that win somewhere for it: kSoloCosts.)
template <int D, bool FP8, bool V8> hipError_t launch_form(const AttnArgs &a, int form, hipStream_t stream)
{
    switch (form) {
    case 114: return launch_solo<D, FP8, V8, 1, 1, 4>(a, stream);
    case 124: return launch_solo<D, FP8, V8, 1, 2, 4>(a, stream);
    case 128: return launch_solo<D, FP8, V8, 1, 2, 8>(a, stream);
    case 118: if constexpr (D == 64) return launch_solo<D, FP8, V8, 1, 1, 8>(a, stream); break;
    case 144: if constexpr (D == 128) return launch_solo<D, FP8, V8, 1, 4, 4>(a, stream); break;
    case 148: if constexpr (D == 128) return launch_solo<D, FP8, V8, 1, 4, 8>(a, stream); break;
    case 224: if constexpr (D == 128 && FP8 == V8) return launch_solo<D, FP8, V8, 2, 2, 4>(a, stream); break;
    case 228: if constexpr (FP8) return launch_solo<D, FP8, V8, 2, 2, 8>(a, stream); break;
    }
    return hipErrorInvalidValue;
}

}  // namespace

bool attn_solo_serves(const AttnArgs &a)
{
    if (a.q_mx != nullptr) return false;
    if (a.qk_dtype == 1) return a.v_dtype == 1;
    return a.qk_dtype == 2 && a.d == 128 && (a.v_dtype == 1 || a.v_dtype == 2);
}

// What a form costs, in hundredths of a microsecond: a workgroup, that again per 100 workgroups beside it, a round (every wave of the
// workgroup one unit), a round past the fourth on top, and, in tenths, a megabyte of K and V, and one of those past 80; `pair` is the same
// past 256 workgroups, two to a compute unit (four waves only, up to 512 workgroups; divided head dims with the cache refresh, whose workgroups
// then come on top, to 480: 256 heads, 32 rows, 33 keys 7.4 on 124, 6.1 on 114).
// Fitted per storage type and form to the times of 4000 drawn drafter calls on three sets of inputs in turn, which the last-level cache
// holds up to 80 MB (1 - 16 x 8 head counts, 1 - 64 rows per head, 20 - 4200 keys, 1 - 16 splits, some 30000 timings; rms of the fits 2 - 7 %).  `late`
// and the constants of 118 were then searched over 7700 drawn calls timed on such inputs and on 650 MB of them in turn, from memory, as a
// model's layers find them: eight waves that stream many units each are fast from the cache alone (fp8 32 heads, 64 rows, 3643 keys on 148
// 13.6 us, from memory 20.5; on 114 in four key splits 13.2 and 16.2).  The mean of the two counts, and a loss of 2 % or more against the
// kernels that served a call before these forms weighs six times.  Over 8500 other drawn calls the picks take 0.79 - 0.90 of those kernels' time
// by type, from the cache and from memory; half a percent takes more than 1.06 from memory (up to 1.15), most of it 0.8 - 0.9 from the cache.
namespace {
struct SoloTerms { int fixed, beside, round, late, mb, cold; };
struct SoloCost { int form; SoloTerms one, pair; };
constexpr SoloCost kSoloBf16[] = {{114, {491, 13, 69, 0, 44, 110}, {494, 15, 107, 0, 91, 47}}, {124, {430, 10, 64, 0, 31, 103}, {406, 14, 92, 0, 66, 76}},
                                  {128, {473, 10, 86, 11, 60, 110}, {}}, {144, {402, 10, 62, 0, 24, 117}, {400, 8, 86, 0, 50, 157}},
                                  {148, {411, 10, 82, 26, 60, 153}, {}}, {224, {483, 15, 92, 0, 16, 55}, {469, 25, 134, 0, 63, 39}}};
constexpr SoloCost kSoloFp8[] = {{114, {459, 10, 61, 0, 43, 111}, {485, 14, 82, 0, 79, 76}}, {124, {407, 5, 50, 0, 40, 134}, {429, 10, 62, 0, 55, 102}},
                                 {128, {483, 5, 57, 0, 55, 158}, {}}, {144, {386, 3, 44, 0, 51, 243}, {411, 7, 58, 0, 33, 244}},
                                 {148, {416, 8, 52, 15, 50, 228}, {}}, {228, {665, 11, 82, 0, 42, 105}, {}}};
constexpr SoloCost kSoloV8[] = {{114, {437, 11, 102, 0, 33, 0}, {449, 18, 135, 0, 63, 2}}, {124, {398, 6, 70, 0, 39, 0}, {402, 11, 99, 15, 24, 73}},
                                {128, {457, 10, 88, 1, 43, 0}, {}}, {144, {380, 5, 53, 0, 50, 0}, {390, 9, 73, 0, 15, 267}},
                                {148, {402, 9, 63, 14, 51, 0}, {}}, {224, {467, 9, 91, 0, 22, 37}, {469, 22, 121, 0, 34, 30}},
                                {228, {539, 13, 111, 0, 40, 131}, {}}};
constexpr SoloCost kSoloD64[] = {{114, {376, 0, 51, 0, 34, 123}, {440, 5, 61, 0, 66, 81}}, {118, {440, 1, 70, 2, 51, 140}, {}},
                                 {124, {372, 0, 45, 0, 39, 273}, {386, 9, 60, 0, 46, 124}}, {128, {403, 0, 52, 0, 56, 236}, {}}};
// A merge launch of key splits, and what it adds per 1000 rows of partial states (64 dims: half the bytes).
constexpr int kMerge = 200, kMergeRows = 27, kMergeRowsD64 = 14;
// The streaming kernel's cost likewise (64 rows, a round = a tile of 64 keys; `more`: per tile and round of 256 workgroups past the first).
struct StreamTerms { int fixed, beside, round, more, mb, cold; };
constexpr StreamTerms kStreamBf16 = {429, 40, 90, 138, 36, 0}, kStreamFp8 = {394, 26, 72, 38, 21, 32};

long megabytes(int mb, int cold, long kb)                                    // hundredths
{
    return (mb * kb + cold * (kb > 80000 ? kb - 80000 : 0)) / 10000;
}
struct SoloPick { int form, splits; long cost; };                            // form 0: none
template <size_t FORMS>
SoloPick cheapest(const SoloCost (&forms)[FORMS], int only, long rows, long heads, int N, long kb, int merge_rows, int most_splits, bool refresh)
{
    SoloPick best{0, 1, 0};
    for (const SoloCost &f : forms) {
        const int blocks = f.form / 100, parts = f.form / 10 % 10, waves = f.form % 10;
        if (only != 0 ? f.form != only : blocks == 2 && rows <= 32) continue;
        const long w1 = heads * ((rows + 32 * blocks - 1) / (32 * blocks)) * parts;
        if (w1 > (waves == 8 ? 256 : refresh && parts > 1 ? 480 : 512) && only == 0) continue;
        int last = 0;
        for (int s = 1; s <= most_splits && (s == 1 || w1 * s <= 256); ++s) {
            const int keys = ((N + s - 1) / s + 31) / 32 * 32, rounds = (keys + 32 * waves - 1) / (32 * waves);
            if (rounds == last) continue;                // more splits for nothing
            last = rounds;
            const SoloTerms &t = w1 * s > 256 && waves == 4 ? f.pair : f.one;
            long cost = t.fixed + t.beside * w1 * s / 100 + (long)t.round * rounds + (long)t.late * (rounds > 4 ? rounds - 4 : 0) + megabytes(t.mb, t.cold, kb);
            if (s > 1) cost += kMerge + merge_rows * heads * rows * s / 1000;
            if (best.form == 0 || cost < best.cost) best = SoloPick{f.form, s, cost};
        }
    }
    return best;
}
SoloPick solo_pick(long rows, long heads, int N, int d, bool fp8, bool v8, int most_splits, bool refresh)
{
    const int only = tune("DD_TUNE_SOLO_FORM", 0);
    const long kb = heads * (long)N * (d == 64 || v8 ? 256 : fp8 ? 384 : 512) / 1000;
    return d == 64 ? cheapest(kSoloD64, only, rows, heads, N, kb, kMergeRowsD64, most_splits, refresh)
         : v8      ? cheapest(kSoloV8, only, rows, heads, N, kb, kMergeRows, most_splits, refresh)
         : fp8     ? cheapest(kSoloFp8, only, rows, heads, N, kb, kMergeRows, most_splits, refresh)
                   : cheapest(kSoloBf16, only, rows, heads, N, kb, kMergeRows, most_splits, refresh);
}
long stream_cost(const StreamTerms &t, long rows, long heads, int N, long kb, bool refresh, int splits)
{
    const int keys = ((N + splits - 1) / splits + 63) / 64 * 64;
    const long s = (N + keys - 1) / keys, wgs = heads * s, tiles = keys / 64;
    return t.fixed + t.beside * wgs / 100 + t.round * tiles + t.more * tiles * ((wgs + 255) / 256 - 1) + megabytes(t.mb, t.cold, kb) +
           (s > 1 ? kMerge + kMergeRows * heads * rows * s / 1000 : refresh ? kMerge : 0);          // (a refresh is a launch like a merge)
}
}  // namespace

// Drafter calls: the cheapest form and key splits (as many as leave every workgroup a compute unit), where that beats the other kernels.
// `fresh`: keys that come from the block's own rows (N: all of them, nothing is read from the cache); `wide_wgs`, `wide_rows`: the wide
// kernel's workgroups, 0 where it cannot serve, and the rows of one.
//
// At most 64 keys are one tile of the other kernels, and nothing for waves to stream.  Few rows stay off this kernel there, unless
//   - its parts spread the call, up to 96 workgroups of 32 rows (bf16 5.05 -> 4.6, fp8 and e4m3 V 4.6 -> 4.35; with 240 5.36 / 5.65 and
//     4.66 / 5.3 the other way; 64 head dims never: 4.05 / 4.25), and bf16 reads some row from the cache (80 heads, 8 keys, all of them the
//     block's 3.98 / 4.42), or
//   - the call has the cache refresh, a launch of its own on the others.
// So do more than 512 workgroups where a head's rows are two (d = 64, 272 heads, 48 rows, 48 keys 5.3 / 7.6).  Up to 256 workgroups of more rows
// run here (bf16 120 heads, 64 rows, 48 keys 5.95 -> 5.1, 64 keys 5.85 -> 4.7, fp8 64 keys 4.95 -> 4.45), but by their cost where the last unit is
// not full and holds the block's keys: bf16 of fewer than 56 rows (40 rows, 33 keys 5.3 / 5.5) or of the block's keys alone (60 rows, 15 keys 4.96 /
// 5.4), fp8 where keys of both kinds meet (56 rows, 33 keys 4.92 / 5.17).
//
// More than 64 rows (against the two-waves-per-SIMD, the wide and the MFMA kernel; thousands of drawn calls, from the cache and from memory):
//   - up to 256 workgroups 0.46 - 0.9 of the time.  bf16 past twelve rounds of 128 keys loses from 2048 keys on, on at most 128 workgroups from
//     3072 on (8 heads, 256 rows, 1708 keys 15.0 -> 11.1; 32 x 112, 4083 keys 24.8 / 28.1; 48 x 96, 2946 keys 25.2 / 30.9), fp8 past 95 MB where
//     no eight-wave form fits (80 x 96, 3600 keys 31.0 / 36.9, 4200 34.2 / 41.4; 3000 even).
//   - up to 512, bf16 and fp8: 0.75 - 0.97 from 65 to 1536 keys (d = 64 to 2560), longer ones up to 1.2 (88 heads, 120 rows, 3084 keys
//     fp8 36.9 / 45.0).  bf16 past 70 MB loses too, where the two-waves-per-SIMD kernel takes 64-row workgroups (120 x 80, 1536 keys 26.5 / 29.6;
//     128 x 128, 1000 keys, 66 MB, 16.9 / 16.1 the other way), past 95 MB where it does not (168 x 96, 1200 keys 26.3 / 28.3).  From memory the
//     last third of the range is up to 1.1 the other way, fp8 to 1.15.
//   - up to 512, e4m3 V: 0.45 - 0.93 at any length, 64 keys and fewer included (48 heads x 256 rows, 64 keys 10.8 -> 6.1) down to 25 with two workgroups
//     per compute unit (96 x 72, 33 keys 6.05 -> 5.7, 24 keys 5.4 / 5.7), except long streams
//     that the wide kernel can serve, in four waves here: up to 320 workgroups where it fills four fifths of the compute units, past 2600 keys (80 x
//     80, 2900 keys 26.5 / 29.4; 64 x 96, eight waves, 25.4 / 20.1 the other way) or, with its 128-row tiles nearly full, 2200 (72 x 112, 2600 keys
//     27.0 / 30.3); up to 512 past 3328 where full tiles are 180 compute units' worth or more (20 x 448, 3800 keys 33.4 / 39.8, 64 x 256, 4050 keys
//     47.3 / 54.9; 72 x 160, 3900 keys, 135 of them, 67.8 / 45.0 the other way).  Where it cannot serve: 72 x 128, 4200 keys 48 -> 46, 80 x 168, 3500 keys
//     69 -> 43.
//   - past 512 1.06 - 1.3.
//
// Up to 64 rows:
//   - d = 64: throughout.
//   - e4m3 V, against the MFMA kernel: up to 512 workgroups of 32 rows; then where a head's rows are one workgroup, or streams are longer
//     than three rounds of 128 keys (up to 768) or four (11 x 32, 63 rows, 90 keys 9.3 there / 10.5).
//   - bf16 and fp8, against the streaming kernel: by its cost (0.91 and 0.87 of the time of one form by rule).  Calls from memory must win by a
//     twentieth (128 heads, 11 rows, 2423 keys fp8 24.3 streamed / 26.4, predicted 24.8 / 23.2), and fp8 rows of one workgroup, two workgroups
//     to a compute unit, stay streamed past 100 MB (288 heads, 32 rows, 1500 keys 39.5 / 41.8, 320 x 32, 892 keys 24.5 / 26.0).
SoloPlan attn_solo_plan(long rows, long heads, int N, int d, bool fp8, bool v8, bool refresh, int fresh, long wide_wgs, int wide_rows,
                        int stream_splits)
{
    const int forced = tune("DD_TUNE_SOLO", -1), forced_splits = tune("DD_TUNE_BLOCK_SPLITS", 0);
    const SoloPlan no{false, 0, 1};
    if (forced == 0) return no;
    const long row_tiles = (rows + 31) / 32, wgs = heads * row_tiles;
    SoloPick pick = solo_pick(rows, heads, N, d, fp8, v8, stream_splits, refresh);
    const bool four_waves = pick.form % 10 != 8;
    if (pick.form == 0) pick.form = v8 && row_tiles == 2 ? 224 : 114;        // (more workgroups than the costs know)
    const SoloPlan plan{true, pick.form, forced_splits >= 1 ? stream_splits : pick.splits};
    if (forced == 1) return plan;
    if (forced_splits >= 1) return no;
    const long rounds = (N + 127) / 128, kb = heads * (long)N * (d == 64 || v8 ? 256 : fp8 ? 384 : 512) / 1000;
    if (rows <= 64 && N <= 64) {
        if (wgs > 512 && row_tiles == 2) return no;
        const bool few = wgs <= 512 && !refresh && heads <= 256 && rows <= (d == 64 || fp8 ? 48 : 32);
        if (few && (d == 64 || wgs > 96 || (!fp8 && fresh == N))) return no;
        const bool plain = N % 32 == 0 || fresh == 0 || (fp8 ? fresh == N : fresh < N && rows >= 56);
        if (!few && row_tiles == 2 && wgs <= 256 && plain) return plan;
    }
    if (rows > 64) {
        if (wgs > 512) return no;
        if (v8 && wide_wgs > 0 && wgs > 192 && four_waves) {
            const long tile_rows = (rows + wide_rows - 1) / wide_rows * wide_rows;
            if (wgs <= 320 && 5 * wide_wgs > 4 * 256 && N > (wgs > 256 && wide_rows == 128 && rows >= 112 ? 2200 : 2600)) return no;
            if (wgs > 256 && 8 * rows >= 7 * tile_rows && rows * wide_wgs > 180 * tile_rows && N > 3328) return no;
        }
        if (v8) return wgs > 256 && N <= 24 ? no : plan;
        if (wgs > 256 && (N <= 64 || N > (d == 64 ? 2560 : 1536))) return no;
        if (d == 64) return plan;
        if (fp8 && wgs > 192 && wgs <= 256 && four_waves && kb > 95000) return no;
        if (!fp8 && wgs > 256 && kb > (heads * ((rows + 63) / 64) <= 256 ? 70000 : 95000)) return no;
        if (!fp8 && wgs <= 256 && (N / pick.splits + 127) / 128 > 12 && N >= (wgs <= 128 ? 3072 : 2048)) return no;
        return plan;
    }
    if (d == 64) return plan;
    if (v8) return wgs <= 512 || (wgs <= 768 && (row_tiles == 1 || rounds > 3)) || rounds > 4 ? plan : no;
    if (fp8 && wgs > 256 && row_tiles == 1 && kb > 100000) return no;
    const long streamed = stream_cost(fp8 ? kStreamFp8 : kStreamBf16, rows, heads, N, kb, refresh, stream_splits);
    return pick.cost != 0 && pick.cost * (kb > 80000 ? 20 : 19) <= 19 * streamed ? plan : no;
}

// Verifier calls: the form alone.
int attn_solo_form(long rows, long heads, int N, int d, bool fp8, bool v8)
{
    const int form = solo_pick(rows, heads, N, d, fp8, v8, 1, false).form;
    return form != 0 ? form : 114;
}

hipError_t launch_attention_solo(const AttnArgs &a, int form, hipStream_t stream)
{
    if (a.v_dtype == 2) return launch_form<128, true, true>(a, form, stream);
    if (a.qk_dtype == 2) return launch_form<128, true, false>(a, form, stream);
    return a.d == 128 ? launch_form<128, false, false>(a, form, stream) : launch_form<64, false, false>(a, form, stream);
}

}  // namespace dd

// Attention of few query rows whose waves stream keys of their own: the drafter's call where workgroups of 32 rows are few or key
// streams short (Sec. 2.3) and small verifier calls (Sec. 2.2), bf16 or fp8 Q/K, bf16 or (with fp8 Q/K) e4m3 V.
//     O = softmax(Q K^T / sqrt(d_k)) V   (Eq. 3)
// One workgroup = four waves on one block of 32 query rows; wave w takes every fourth 32-key unit of the key range with a state
// (reference, sum, O) of its own, and the states are merged through LDS at the end, every wave finishing a quarter of the head dims.
//   - No K/V row is used by two waves, so none waits for another: a wave has one K and one V buffer in LDS, filled by
//     global_load_lds_dwordx4, waits for its own loads only, and asks for the next unit's K as soon as the fragments of this
//     one's are in registers, V likewise: 64 KB (fp8 48 KB) per workgroup are on their way nearly all the time.
//   - A block of 32 rows leaves no wave idle (the 64-row workgroups of attention_stream.hip halve there), and 64 rows are two
//     workgroups that share K/V through an XCD's L2.  Two workgroups fit a compute unit.
// What bounds it: some 4 us of launch, first loads and merge, then 1.1 us (fp8 0.9) per 128 keys while a compute unit has one
// workgroup - 60 GB/s, the same with eight waves and twice the bytes on their way, so what a unit draws from beyond its L2.
// us per call in a stream of them, attention_stream.hip -> here: 11 x 32/8 heads, 16 rows, 1237 keys fp8 20.5 -> 16.3, bf16
// 23.8 -> 20.8; 1 x 32, 512 keys, 32 rows bf16 9.7 -> 8.0, 64 rows 11.9 -> 8.4; 1 x 32, 300 keys, 16 rows 9.5 -> 7.2; 4 x 32/8, 16 rows,
// 2048 keys 17.7 -> 14.6 (4 splits).  Tried and not kept: eight waves per workgroup (bf16 11 x 32/8 19.9 where four took 19.3, 1 x 32 9.9 /
// 9.1, 4 x 32/8 15.1 / 14.3).
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

constexpr int kSoloWaves = 4;

// V8: V is stored as e4m3 codes.  They travel to LDS as they are and the wave decodes its own 4 KB into its V buffer, exactly, when
// they arrive (32 conversions of two elements per lane and unit); v_scale multiplies the result once.
// `wgs`: the launch's attending workgroups.
template <int D, bool FP8, bool V8>
__device__ __forceinline__ void attn_solo(const AttnKernelArgs &a, const int wgs)
{
    // (device pass only: the host pass needs the kernels' handles, not assembly it cannot check)
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int NW = kSoloWaves, U = 32;           // keys per unit
    constexpr int CH = D / 8;                        // 16-byte chunks per V / O row
    constexpr int DC = D / 32;                       // 32-wide chunks of the head dim
    constexpr int ROWB = D * 2;                      // bytes per V / O row
    constexpr int KROWB = FP8 ? D : ROWB, KCH = KROWB / 16;   // Q / K as stored: bytes and chunks per row
    constexpr int KF = KROWB / 32;                   // 16-byte K fragments per lane and unit
    constexpr int KB = U * KROWB, VB = U * ROWB;     // bytes of a wave's K / V buffer
    constexpr int VSROWB = V8 ? D : ROWB, VSCH = VSROWB / 16, VSB = V8 ? U * VSROWB : 0;   // V as stored; its own buffer if decoded
    constexpr int NK = KB / 1024, NV = U * VSROWB / 1024;                    // wave-wide loads per buffer (1 KB each)
    constexpr int VDMA_ROWS = 1024 / VSROWB, KDMA_ROWS = 1024 / KROWB;       // rows per load
    constexpr int G = DC * 4, GP = G / NW;           // groups of four O registers per lane, ... that a wave finishes
    static_assert((!FP8 && !V8) || (FP8 && D == 128), "fp8 rows are 128 bytes");
    static_assert(GP % 2 == 0, "groups are stored in pairs");
    static_assert(NK <= 8 && NV <= 8, "a buffer is within the loads' immediate offsets");
    constexpr int SLOTB = KB + VB + VSB;
    constexpr int PARKB = NW * (NW - 1) * GP * 1024; // the parked states share the buffers' memory
    constexpr int LDSB = (NW * SLOTB > PARKB ? NW * SLOTB : PARKB);
    // per wave: K [key][chunk ^ (key & 7)], then V [key][chunk ^ ((key % (CH/4)) << 2)]
    __shared__ __attribute__((aligned(1024))) uint4 KV[LDSB / 16];
    __shared__ __attribute__((aligned(1024))) uint4 QS[KB / 16];             // the query rows, as K
    __shared__ float qs_sh[64];                      // the scales of the query rows
    __shared__ float ml_sh[NW][2][32];               // per wave: (reference, sum) of the query rows

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hh = lane >> 5;

    // ---- which (batch, kv head, row tile, key split); same XCD for workgroups that share K/V
    int bid = blockIdx.x;
    {
        const int total = wgs, per = total >> 3, rem = total & 7;
        const int xcd = bid & 7, slot = bid >> 3;
        bid = xcd * per + min(xcd, rem) + slot;
    }
    const int rt = bid % a.row_tiles; bid /= a.row_tiles;
    const int sp = bid % a.splits; bid /= a.splits;
    const int kvh = bid % a.Hkv;
    const int b = bid / a.Hkv;
    const int rows_total = a.group * a.Nq;           // query rows of this (batch, kv head): contiguous in memory
    const int v_first = rt * 32;
    const size_t row_base = ((size_t)b * a.H + (size_t)kvh * a.group) * a.Nq;
    const int kbeg = sp * a.keys_per_split;
    const int kend = min(a.N, kbeg + a.keys_per_split);
    const int bstart = a.block_starts ? a.block_starts[b] : a.block_start;   // any value is safe: rows are chosen by range test
    const int blen = a.block_len;
    const int nunits = (kend - kbeg + U - 1) / U;
    const int whole = (kend - kbeg) / U;             // units [0, whole) hold 32 rows of the range

    const size_t kv_head = (size_t)b * a.Hkv + kvh;
    const uint8_t *const kc = static_cast<const uint8_t *>(a.K) + kv_head * a.kv_stride * (size_t)KROWB;
    const uint8_t *const vc = static_cast<const uint8_t *>(a.V) + kv_head * a.kv_stride * (size_t)VSROWB;
    const uint8_t *const kb_ = blen ? static_cast<const uint8_t *>(a.Kblk) + kv_head * blen * (size_t)KROWB : nullptr;
    const uint8_t *const vb_ = blen ? static_cast<const uint8_t *>(a.Vblk) + kv_head * blen * (size_t)VSROWB : nullptr;
    auto lds_addr = [&](const void *p) __attribute__((always_inline)) { return (unsigned)(size_t)(__attribute__((address_space(3))) const void *)p; };
    char *const kbuf = reinterpret_cast<char *>(KV) + wave * SLOTB, *const vbuf = kbuf + KB, *const vstored = vbuf + VB;
    const unsigned kdst = lds_addr(KV) + wave * SLOTB, vdst = kdst + KB + (V8 ? VB : 0);
    // load i of a buffer fills its rows i * DMA_ROWS ..; lane l lands at chunk position l % CH of row l / CH and fetches the
    // chunk the swizzle maps there (with 256-byte rows K's depends on whether i is odd)
    const int vrow0 = lane / VSCH, krow0 = lane / KCH;
    auto kchunk = [&](int i) __attribute__((always_inline)) { return (unsigned)(((lane % KCH) ^ ((i * KDMA_ROWS + krow0) & 7)) * 16); };
    const unsigned vchunk = V8 ? lane % VSCH * 16 : ((lane % CH) ^ ((vrow0 & (CH / 4 - 1)) << 2)) * 16;   // (codes lie as in memory)
    const unsigned koff[2] = {krow0 * KROWB + kchunk(0), krow0 * KROWB + kchunk(1)}, voff = vrow0 * VSROWB + vchunk;
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
        constexpr int NL = K ? NK : NV, BIAS = NL > 4 ? 4096 : 0, PITCH = K ? KROWB : VSROWB;
        const unsigned dst = (K ? kdst : vdst) + BIAS;
        const int k0 = kbeg + u * U;
        if (u < whole && (unsigned)(u - blk0) >= (unsigned)(blk1 - blk0)) {
            const uint8_t *const src = solo_scalar((K ? kc : vc) + (size_t)k0 * PITCH + BIAS);
            static_for<0, NL>([&](auto i) __attribute__((always_inline)) {
                constexpr int I = decltype(i)::value, IMM = I * 1024 - BIAS;
                const unsigned d = dst, o = K ? koff[I & 1] : voff;
                const uint8_t *const sbase = src;
                if constexpr (IMM >= 0)
                    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3" ::"s"(d), "v"(o), "s"(sbase), "n"(IMM) : "memory", "m0");
                else
                    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2 offset:-%3" ::"s"(d), "v"(o), "s"(sbase), "n"(-IMM) : "memory", "m0");
            });
        } else {
            static_for<0, NL>([&](auto i) __attribute__((always_inline)) {
                constexpr int I = decltype(i)::value;
                const int j = min(k0 + I * (K ? KDMA_ROWS : VDMA_ROWS) + (K ? krow0 : vrow0), kend - 1);
                const bool in_blk = (unsigned)j - (unsigned)bstart < (unsigned)blen;
                const uint8_t *const src = (K ? (in_blk ? kb_ : kc) : (in_blk ? vb_ : vc)) + (size_t)(in_blk ? j - bstart : j) * PITCH + (K ? kchunk(I) : vchunk);
                const unsigned d = dst - BIAS + I * 1024;
                asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(d), "v"(src) : "memory", "m0");
            });
        }
    };
    const std::true_type of_k;
    const std::false_type of_v;

    // ---- prologue: the query rows, shared out over the waves, then this wave's first unit
    const int v = v_first + l32;
    const bool row_ok = v < rows_total;
    const float k_scale = a.k_scale ? a.k_scale[kv_head] : 1.0f;
    // (through LDS like the rows: the compiler's own wait for a load of its own would wait for every load after it as well)
    if (a.q_scale && wave == 0) {
        const float *const src = a.q_scale + b * a.H + kvh * a.group + min(v, rows_total - 1) / a.Nq;
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_addr(qs_sh)), "v"(src) : "memory", "m0");
    }
    for (int i = wave; i < NK; i += NW) {
        const int r = min(v_first + i * KDMA_ROWS + krow0, rows_total - 1);
        const uint8_t *const src = static_cast<const uint8_t *>(a.Q) + (row_base + r) * KROWB + kchunk(i);
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr(QS) + i * 1024), "v"(src) : "memory", "m0");
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
    intx4 qf[KF];
#pragma unroll
    for (int f = 0; f < KF; ++f) qf[f] = *reinterpret_cast<const intx4 *>(reinterpret_cast<const char *>(QS) + k_off[f]);

    float c = a.scale_log2 * k_scale;                // scores are exponentiated as 2^(s*c)
    if (a.q_scale) c *= qs_sh[lane];

    floatx16 acc[DC];                                // O^T, unnormalised
#pragma unroll
    for (int i = 0; i < DC; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
    // Row sums of the weights as multiplied (rounded to bf16), by the matrix instruction of sixteen 4 x 4 blocks: lane l is
    // column l % 4 of block l / 4 with four values of k, so with an A operand of ones every lane gets the sum of its own
    // weights; the lane halves hold different keys of a row and are added at the end.
    floatx4 acc_l = {0.f, 0.f, 0.f, 0.f};
    const short4v ones = {0x3F80, 0x3F80, 0x3F80, 0x3F80};
    // The reference m of the weights p = 2^(s c - m), as -m (log2 units), equal in both lane halves.  It only has to be near the
    // running maximum (any common factor 2^-m cancels): the first unit sets it to its maximum + 7; a later one first takes its
    // weights with the one in use, and only if some weight reached 2 - one bit of its bf16 pattern, the packed weights are or-ed
    // together - it is raised to the unit's maximum + 7, the sums are scaled and the weights taken again.
    float nm = INFINITY;

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
        floatx16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
        if constexpr (FP8) {
#pragma unroll
            for (int j = 0; j < KF / 2; ++j) {
                const intx8 kx = __builtin_shufflevector(kf[2 * j], kf[2 * j + 1], 0, 1, 2, 3, 4, 5, 6, 7);
                const intx8 qx = __builtin_shufflevector(qf[2 * j], qf[2 * j + 1], 0, 1, 2, 3, 4, 5, 6, 7);
                s = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(kx, qx, s, 0, 0, 0, 0x7F7F7F7F, 0, 0x7F7F7F7F);
            }
        } else {
#pragma unroll
            for (int f = 0; f < KF; ++f)
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[f]), __builtin_bit_cast(bf16x8, qf[f]), s, 0, 0, 0);
        }
        if (u == whole) {                            // (a unit with rows past the end of the range)
            // score register r is key key0 + 8 (r / 4) + 4 hh + (r % 4) for query row l32
            const int key0 = kbeg + u * U;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (key0 + 8 * (r >> 2) + 4 * hh + (r & 3) >= kend) s[r] = -INFINITY;
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
        unsigned pk[2][4], seen = 0u;                // P^T as the B operand of O^T += V^T P^T
        bool raise_any = true;                       // uniform
        if (u != wave) {
#pragma unroll
            for (int r = 0; r < 16; r += 2)
                pk[r >> 3][(r & 7) >> 1] = solo_pack(solo_exp2(fmaf(s[r], c, nm)), solo_exp2(fmaf(s[r + 1], c, nm)));
#pragma unroll
            for (int k = 0; k < 8; ++k) seen |= pk[k >> 2][k & 3];
            raise_any = __any((seen & 0x40004000u) != 0u);
        }
        if (raise_any) {
            const u32x2 both = solo_swap(seen, seen);
            const bool raise = u == wave || ((both.x | both.y) & 0x40004000u) != 0u;
            float mx = s[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
            const u32x2 mm = solo_swap(__float_as_uint(mx), __float_as_uint(mx));
            mx = fmaxf(__uint_as_float(mm.x), __uint_as_float(mm.y)) * c + kSoloMargin;
            const float m_old = -nm, m_new = raise ? fmaxf(m_old, mx) : m_old;
            const float corr = m_new == m_old ? 1.0f : solo_exp2(m_old - m_new);         // first unit: 2^(-inf) = 0
            const float use = m_new == -INFINITY ? 0.f : -m_new;                         // every score so far is -inf: weights 0
            nm = -m_new;
            if (u != wave) {                         // (the first unit's sums are zero)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc_l[r] *= corr;
#pragma unroll
                for (int i = 0; i < DC; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[i][r] *= corr;
            }
#pragma unroll
            for (int r = 0; r < 16; r += 2)
                pk[r >> 3][(r & 7) >> 1] = solo_pack(solo_exp2(fmaf(s[r], c, use)), solo_exp2(fmaf(s[r + 1], c, use)));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (!V8 && more) load_rows(of_v, u + NW);
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            const uint4 pw = make_uint4(pk[st][0], pk[st][1], pk[st][2], pk[st][3]);
#pragma unroll
            for (int i = 0; i < DC; ++i)
                acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[st][i], __builtin_bit_cast(bf16x8, pw), acc[i], 0, 0, 0);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const u32x2 half = {pk[st][2 * k], pk[st][2 * k + 1]};
                acc_l = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones, __builtin_bit_cast(short4v, half), acc_l, 0, 0, 0);
            }
        }
    }

    // ---- merge the waves' states through LDS: a wave parks the groups of O registers that others finish
    const float mc = -nm;
    const u32x2 ls = solo_swap(__float_as_uint(acc_l[0]), __float_as_uint(acc_l[0]));
    const float l_own = __uint_as_float(ls.x) + __uint_as_float(ls.y);
    __syncthreads();                                 // every wave is done with its buffers (and has no load outstanding)
    float4 *park = reinterpret_cast<float4 *>(KV);
    auto park_at = [&](int from, int to, int g) __attribute__((always_inline)) {
        return ((from * (NW - 1) + (to < from ? to : to - 1)) * GP + g) * 64 + lane;
    };
    ml_sh[wave][0][l32] = mc;
    ml_sh[wave][1][l32] = l_own;
#pragma unroll
    for (int to = 0; to < NW; ++to)
        if (to != wave) {
#pragma unroll
            for (int g = 0; g < GP; ++g) {
                const int i = (to * GP + g) / 4, r = 4 * ((to * GP + g) % 4);
                park[park_at(wave, to, g)] = make_float4(acc[i][r], acc[i][r + 1], acc[i][r + 2], acc[i][r + 3]);
            }
        }
    __syncthreads();
    float m_all = -INFINITY, wgt[NW], l_tot = 0.f;
#pragma unroll
    for (int q = 0; q < NW; ++q) m_all = fmaxf(m_all, ml_sh[q][0][l32]);
#pragma unroll
    for (int q = 0; q < NW; ++q) {
        const float m = ml_sh[q][0][l32];
        wgt[q] = m == -INFINITY ? 0.f : solo_exp2(m - m_all);                // a wave that saw no key weighs nothing
        l_tot += ml_sh[q][1][l32] * wgt[q];
    }
    float o[GP][4], w_own = wgt[0];
#pragma unroll
    for (int q = 0; q < NW; ++q)
        if (q == wave) {
            w_own = wgt[q];
#pragma unroll
            for (int g = 0; g < GP; ++g)
#pragma unroll
                for (int k = 0; k < 4; ++k) o[g][k] = acc[(q * GP + g) / 4][4 * ((q * GP + g) % 4) + k];
        }
#pragma unroll
    for (int g = 0; g < GP; ++g)
#pragma unroll
        for (int k = 0; k < 4; ++k) o[g][k] *= w_own;
#pragma unroll
    for (int q = 0; q < NW; ++q)
        if (q != wave) {
#pragma unroll
            for (int g = 0; g < GP; ++g) {
                const float4 x = park[park_at(q, wave, g)];
                o[g][0] += x.x * wgt[q]; o[g][1] += x.y * wgt[q]; o[g][2] += x.z * wgt[q]; o[g][3] += x.w * wgt[q];
            }
        }
    if constexpr (V8) {
        const float vs = a.v_scale[kv_head];         // the decoded values times this are the real ones
#pragma unroll
        for (int g = 0; g < GP; ++g)
#pragma unroll
            for (int k = 0; k < 4; ++k) o[g][k] *= vs;
    }
    // ---- output: group g of this wave is dims 8 (wave GP + g) + 4 hh .. + 3 of query row l32
    const size_t orow = row_base + v;
    if (a.splits == 1) {
        const float inv = 1.0f / l_tot;
        uint16_t *out = static_cast<uint16_t *>(a.O) + orow * D;
#pragma unroll
        for (int g = 0; g < GP; g += 2) {
            // the halves exchange words so that each lane stores eight consecutive dims
            const u32x2 x0 = solo_swap(solo_pack(o[g][0] * inv, o[g][1] * inv), solo_pack(o[g + 1][0] * inv, o[g + 1][1] * inv));
            const u32x2 x1 = solo_swap(solo_pack(o[g][2] * inv, o[g][3] * inv), solo_pack(o[g + 1][2] * inv, o[g + 1][3] * inv));
            if (row_ok) *reinterpret_cast<uint4 *>(out + 8 * (wave * GP + g + hh)) = make_uint4(x0.x, x1.x, x0.y, x1.y);
        }
    } else if (row_ok) {
        float *po = a.part_o + (orow * a.splits + sp) * D;
#pragma unroll
        for (int g = 0; g < GP; ++g) *reinterpret_cast<float4 *>(po + 8 * (wave * GP + g) + 4 * hh) = make_float4(o[g][0], o[g][1], o[g][2], o[g][3]);
        if (hh == 0 && wave == 0) {
            float *ml = a.part_ml + (orow * a.splits + sp) * 2;
            ml[0] = m_all;
            ml[1] = l_tot;
        }
    }
#endif
}

template <int D, bool FP8, bool V8>
__global__ __launch_bounds__(64 * kSoloWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_solo_kernel(const AttnKernelArgs a)
{
    attn_solo<D, FP8, V8>(a, gridDim.x);
}

// The same launch with the block-completion copy on the workgroups past the attending ones: for a call without key splits, which has no
// merge launch to take it along.  (A kernel of its own: the look at where the copying workgroups start costs a plain call 0.4 us.)
template <int D, bool FP8, bool V8>
__global__ __launch_bounds__(64 * kSoloWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_solo_refresh_kernel(const AttnKernelArgs a, const RefreshArgs r)
{
    if ((int)blockIdx.x >= r.first_wg) {             // uniform: these only copy
        refresh_cache_rows(r);
        return;
    }
    attn_solo<D, FP8, V8>(a, r.first_wg);
}

template <int D, bool FP8, bool V8> hipError_t launch_solo(const AttnArgs &a, hipStream_t stream)
{
    AttnKernelArgs k;
    fill_kernel_args(a, k, 32, 32);
    const long wgs = (long)a.B * a.Hkv * k.row_tiles * k.splits;
    const dim3 block(64 * kSoloWaves);
    RefreshArgs r{};
    const long copy_wgs = k.splits == 1 ? fill_refresh(a, r, kCopyWgs) : 0;
    if (copy_wgs > 0) {
        r.first_wg = (int)wgs;
        return launch(attn_solo_refresh_kernel<D, FP8, V8>, dim3((unsigned)(wgs + copy_wgs)), block, stream, k, r);
    }
    const hipError_t e = launch(attn_solo_kernel<D, FP8, V8>, dim3((unsigned)wgs), block, stream, k);
    return e != hipSuccess ? e : finish_attention(a, k.splits, stream);
}

}  // namespace

bool attn_solo_serves(const AttnArgs &a)
{
    if (a.q_mx != nullptr) return false;
    if (a.qk_dtype == 1) return a.v_dtype == 1;
    return a.qk_dtype == 2 && a.d == 128 && (a.v_dtype == 1 || a.v_dtype == 2);
}

// Drafter calls.  Key splits: those of least cost while every workgroup has a compute unit, in hundredths of a microsecond, fitted per
// storage type to some 35000 timings of 19500 calls at one to sixteen splits: a workgroup, its rounds of 128 keys, both again by
// the workgroups beside it (the caches' share), a merge launch, that again by its workgroups up to 48 and by the rows of the
// partial states.  (The split picked is 0.1 % off the best one on average.  Decoded e4m3 values cost a round more and share less, so they split earlier: 1 x 32 heads, block 8,
// 801 keys 12.0 unsplit, 9.3 with four splits, 11.1 on the MFMA kernel; bf16 5 x 8 heads, 7 rows, 724 keys 11.3 unsplit, 9.8 with four.)
namespace {
struct SoloCost { long fixed, fixed_beside, round, round_beside, merge, merge_beside, krows; };     // (beside: per 100 workgroups; merge: 48)
constexpr SoloCost kSoloBf16 = {441, 23, 80, 28, 214, 57, 4}, kSoloFp8 = {412, 20, 70, 20, 214, 43, 12}, kSoloD64 = {351, 17, 54, 16, 206, 48, 1},
                   kSoloV8 = {388, 37, 108, 4, 202, 46, 16};
}  // namespace
// Against the streaming kernel (8300 calls of 1 - 16 x 32/32, 32/8, 28/4 and 16/16 heads, 8 - 64 rows, 200 - 4096 keys): with one
// workgroup per compute unit and at most 7 rounds of 128 keys each (8 unsplit) it takes 0.83 of the time (bf16) and 0.87 (fp8), up to 3 %
// more on one call in a hundred.  Longer streams are bound by memory bandwidth, which that kernel's larger workgroups draw better - 8 x 32, 32
// rows, 3992 keys fp8 63.6 / 71.8 - unless they leave it a third of its compute units idle: 11 x 32/8, 1237 keys above (264 of its
// workgroups).  Past 256 workgroups: bf16 of at most 32 rows 0.85 up to 512, the others lose (64 rows bf16 1.03, fp8 1.01).  d = 64: 0.79
// throughout.  e4m3 values, against the MFMA kernel (746 such calls): 0.78, 9 x 32, 48 rows, 3774 keys 125 -> 85, 11 x 32/8, 16 rows, 1360 keys
// 23.2 -> 18.3.  Slower, up to 1.13, where a kv head's rows are two workgroups, more than 512 in all, and few keys leave both launches their
// ramps: 11 x 32, 63 rows, 90 keys 9.3 / 10.5; from a fourth round on and with one workgroup per head it is not.
// At most 64 keys are one tile of the kernels before, and nothing for waves to stream: few rows of up to 256 heads are faster there, fp8 8
// rows, 37 - 62 keys 4.2 against 4.9 here, bf16 4.5 - 4.8 / 4.9 - 5.3, as is anything past 512 workgroups where a head's rows are two
// (d = 64 272 heads, 48 rows, 48 keys 5.3 / 7.6); with the cache refresh, a launch of its own there, 7.2 / 5.1, with 64 rows 6.1 / 5.1 (fp8).
// More than 64 rows (900 calls of 32/8, 28/4, 32/16 and 16/2 heads, 16 - 64 rows per head, 300 - 4096 keys; before: the two-waves-per-SIMD,
// the wide or the MFMA kernel): up to 256 workgroups with at most 12 rounds each 0.78 of the time (bf16), 0.75 (fp8), 0.65 (e4m3 V, these up
// to 512), on none more than 1.00; 256 - 384 workgroups and longer streams up to 1.3.
SoloPlan attn_solo_plan(long rows, long heads, int N, int d, bool fp8, bool v8, bool refresh, int stream_splits)
{
    const int forced = tune("DD_TUNE_SOLO", -1);
    if (forced == 0) return SoloPlan{false, 1};
    if (tune("DD_TUNE_BLOCK_SPLITS", 0) >= 1) return SoloPlan{forced == 1, stream_splits};
    const long row_tiles = (rows + 31) / 32, wgs = heads * row_tiles;
    const SoloCost &c = d == 64 ? kSoloD64 : v8 ? kSoloV8 : fp8 ? kSoloFp8 : kSoloBf16;
    const long most = wgs >= 256 ? 1 : 256 / wgs < stream_splits ? 256 / wgs : stream_splits;
    long splits = 1, rounds = 0, best = 0;
    for (long s = 1; s <= most; ++s) {
        const long r = ((N + s - 1) / s + 127) / 128, w = wgs * s;
        long cost = c.fixed + c.round * r + (c.fixed_beside + c.round_beside * r) * w / 100;
        if (s > 1) cost += c.merge + c.merge_beside * (w < 48 ? w : 48) / 48 + c.krows * heads * rows * s / 1000;
        if (best == 0 || cost < best) {
            splits = s;
            rounds = r;
            best = cost;
        }
    }
    if (forced == 1) return SoloPlan{true, (int)splits};
    if (rows <= 64 && N <= 64 && (wgs > 512 ? row_tiles == 2 : !refresh && heads <= 256 && rows <= (d == 64 || fp8 ? 48 : 32)))
        return SoloPlan{false, 1};
    if (rows > 64) return SoloPlan{wgs <= (v8 ? 512 : 256) && rounds <= 12, (int)splits};
    if (d == 64) return SoloPlan{true, (int)splits};
    if (v8) return SoloPlan{wgs <= 512 || (wgs <= 768 && (row_tiles == 1 || rounds > 3)) || rounds > 4, (int)splits};
    const long stream_wgs = heads * stream_splits, stream_slots = (stream_wgs + 255) / 256 * 256;
    const bool fits = wgs <= 256 || (!fp8 && row_tiles == 1 && wgs <= 512);
    const bool idle = 10 * stream_wgs < (fp8 ? 6 : 7) * stream_slots;
    return SoloPlan{fits && (rounds <= (splits == 1 ? 8 : 7) || idle), (int)splits};
}

hipError_t launch_attention_solo(const AttnArgs &a, hipStream_t stream)
{
    if (a.v_dtype == 2) return launch_solo<128, true, true>(a, stream);
    if (a.qk_dtype == 2) return launch_solo<128, true, false>(a, stream);
    return a.d == 128 ? launch_solo<128, false, false>(a, stream) : launch_solo<64, false, false>(a, stream);
}

}  // namespace dd

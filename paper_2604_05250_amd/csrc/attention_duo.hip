// Attention with two waves per SIMD on the same query rows: the drafter's call with more than 64 rows per kv head, which
// grouped heads make compute bound (Sec. 2.3), and long verifier calls of 449 to 512 workgroups of 32 rows (bf16 past 1344 keys, fp8 past 3072; Sec. 2.2).
//     O = softmax(Q K^T / sqrt(d_k)) V   (Eq. 3)
// One workgroup = 8 waves = R blocks of 32 query rows x P = 8 / R key phases: wave w owns row block w % R and takes every
// P-th 32-key unit of the key stream, with a state (reference, sum, O) of its own; the P states of a row block are merged
// through LDS at the end, every wave finishing 1 / P of the head dims.
//   - A wave runs S = K Q^T, the softmax and O += V P of a unit one after the other and the other wave of its SIMD fills the
//     gaps of that chain.  The two phases halve (R = 4) or quarter (R = 2) the chain of a workgroup without another workgroup's
//     partial state and a merge launch.
//   - K/V tiles (32 P keys) go from global memory straight into an LDS ring (global_load_lds_dwordx4, written as assembly:
//     the compiler knows nothing of them and every wait for them is explicit).
//   - Key row j comes from the block tensors inside the block and from the cache elsewhere, whatever the block's position: a
//     tile that lies in the cache has scalar addresses, any other is gathered row by row.
// K is XOR-swizzled for its 16-byte operand reads; V stays row-major (swizzled in 64-byte granules) and its transposed
// operand comes from ds_read_b64_tr_b16.
// What bounds it (16 x 32/8 heads, 64 rows, 2048 keys, fp8, R = 4): no unit by itself.  MfmaUtil 25 %, VALUBusy 29 %, LdsUtil 16 % (0.32
// conflict cycles per access); a wave waits 35 % of its 80 k cycles for memory, LDS or a barrier and 31 % for its turn to issue.  Per
// 64 keys and 128 rows that is some 2500 cycles, 830 of them matrix time of a SIMD, for 96 KB of LDS reads and 24 KB of tile loads.
// us per call in a stream of them, both sides in turn,
// before (128- or 256-row tiles of attention_wide.hip, or attention_mfma.hip where a block is shorter than a tile) -> here: 16 x 32/8
// heads, 64 rows, 2048 keys fp8 46.2 -> 45.2 (among other calls 42.2 -> 40.4), bf16 54.6 -> 49.3; 32 rows fp8 41.0 -> 31.1, bf16 45.0 ->
// 40.4; 8 x 28/4, 48 rows, 1111 keys bf16 30.1 -> 20.6, fp8 29.6 -> 16.9; 10 x 32/8, 48 rows, 700 keys fp8 28.2 -> 14.9.  Tried on R = 4 and
// not kept (fp8, then 41.5): scores of unit u + 1, weights of u and product of u - 1 in one step (41.5); the
// waves of a SIMD taking turns between matrix and vector steps, two barriers per tile (39.7, bf16 46.4: 2-3 % for a second
// loop); 64 rows per wave, four phases (40.4).
#include "attention_common.h"
#include "dd_internal.h"

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

constexpr int kDuoThreads = 512, kDuoWaves = 8;
[[maybe_unused]] constexpr float kDuoMargin = 7.0f;      // a reference is set this far above a unit's maximum (log2 units)

__device__ __forceinline__ float duo_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ unsigned duo_pack(float lo, float hi)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    floatx2 f = {lo, hi};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2));
}
__device__ __forceinline__ u32x2 duo_swap(unsigned a, unsigned b)        // {a.lo, b.lo}, {a.hi, b.hi} by lane halves
{
    return __builtin_amdgcn_permlane32_swap(a, b, false, false);
}
constexpr int duo_waitcnt_vm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

// R: row blocks per workgroup, RING: tile buffers
template <int D, bool FP8, int R, int RING>
__global__ __launch_bounds__(kDuoThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_duo_kernel(DD_ATTN_HEAD, const AttnTail a)
{
    // (device pass only: the host pass needs the handle, not assembly it cannot check)
#if defined(__HIP_DEVICE_COMPILE__)
    const AttnHead h = DD_ATTN_HEAD_ARGS;
    constexpr int P = kDuoWaves / R;                 // key phases
    constexpr int TK = 32 * P;                       // keys per tile
    constexpr int CH = D / 8;                        // 16-byte chunks per V / O row
    constexpr int DC = D / 32;                       // 32-wide chunks of the head dim
    constexpr int ROWB = D * 2;                      // bytes per V / O row
    constexpr int KROWB = FP8 ? D : ROWB, KCH = KROWB / 16;   // Q / K as stored: bytes and chunks per row
    constexpr int KF = KROWB / 32;                   // 16-byte K fragments per lane and unit
    constexpr int VDMA_ROWS = 1024 / ROWB, KDMA_ROWS = 1024 / KROWB;         // rows per wave-wide load
    constexpr int NV = TK / VDMA_ROWS / kDuoWaves, NK = TK / KDMA_ROWS / kDuoWaves, NLOADS = NV + NK;   // loads per wave and tile
    constexpr int NQ = R * 32 / KDMA_ROWS / kDuoWaves;                       // ... and for its share of the Q rows
    constexpr int TILEB = TK * ROWB, KTILEB = TK * KROWB;                    // bytes of one V / K tile
    constexpr int SLOTB = KTILEB + TILEB;            // a ring slot: the K tile [key][chunk ^ (key & 7)], then the V tile
                                                     // [key][chunk ^ ((key % (CH/4)) << 2)]
    constexpr int G = DC * 4, GP = G / P;            // groups of four O registers per lane, ... that a wave finishes
    static_assert(NV >= 1 && NK >= 1 && NQ >= 1, "every wave loads its share");
    static_assert((kDuoWaves * VDMA_ROWS) % 8 == 0 && (kDuoWaves * KDMA_ROWS) % 8 == 0, "swizzle phase must not depend on the load index");
    static_assert(!FP8 || D == 128, "fp8 rows are 128 bytes");
    static_assert(RING >= 2, "one tile in use, one on its way");
    static_assert(NV % 2 == 0 || NV == 1, "V loads are issued in two parts");
    static_assert(R * 32 * KROWB <= SLOTB, "the Q rows fit the ring slot they pass through");
    static_assert(kDuoWaves * (P - 1) * GP * 1024 <= RING * SLOTB, "the parked states fit the ring");
    __shared__ __attribute__((aligned(1024))) uint4 KV[RING * SLOTB / 16];
    __shared__ float ml_sh[kDuoWaves][2][32];        // per wave: (max, sum) of its query rows
    __shared__ float qs_sh[kDuoWaves][64];           // per wave: the scales of its query rows

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hh = lane >> 5;
    const int rg = wave % R, ph = wave / R;          // row block, key phase

    // ---- which (batch, kv head, row tile, key split); same XCD for workgroups that share K/V
    unsigned bid = blockIdx.x;
    {
        const unsigned total = h.wgs, per = total >> 3, rem = total & 7;
        const unsigned xcd = bid & 7, slot = bid >> 3;
        bid = xcd * per + min(xcd, rem) + slot;
    }
    int sp, rt;
    place_of(bid, h.splits, sp);
    place_of(bid, h.row_tiles, rt);
    const size_t kv_head = bid;                      // batch and kv head; its query rows are contiguous in memory
    const int v_tile = rt * (32 * R), v_first = v_tile + rg * 32;
    const bool wave_active = v_first < rows_total;   // uniform
    const size_t row_base = kv_head * rows_total;
    const int kbeg = sp * h.keys_per_split;
    const int kend = min(h.N, kbeg + h.keys_per_split);
    // (any value is safe: rows are chosen by range test)
    const int bstart = a.block_starts ? uniform_load(a.block_starts + (unsigned)kv_head / (unsigned)a.Hkv) : h.block_start;
    const int blen = h.block_len;
    const int ntiles = (kend - kbeg + TK - 1) / TK;

    // ---- staging by LDS DMA: load i of this wave moves rows (8 i + wave) * DMA_ROWS .. of a tile; lane l lands at chunk
    // position l % CH of row l / CH and therefore fetches the chunk the swizzle maps there
    const int vrow0 = wave * VDMA_ROWS + lane / CH, krow0 = wave * KDMA_ROWS + lane / KCH;
    const unsigned vchunk = ((lane % CH) ^ ((vrow0 & (CH / 4 - 1)) << 2)) * 16;
    const unsigned kchunk = ((lane % KCH) ^ (krow0 & 7)) * 16;
    const unsigned voff = vrow0 * ROWB + vchunk, koff = krow0 * KROWB + kchunk;
    const uint8_t *const kc = h.K + kv_head * h.kv_stride * (size_t)KROWB;
    const uint8_t *const vc = h.V + kv_head * h.kv_stride * (size_t)ROWB;
    const uint8_t *const kb_ = blen ? static_cast<const uint8_t *>(a.Kblk) + kv_head * blen * (size_t)KROWB : nullptr;
    const uint8_t *const vb_ = blen ? static_cast<const uint8_t *>(a.Vblk) + kv_head * blen * (size_t)ROWB : nullptr;
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void *)KV;
    auto load_at = [&](unsigned dst, const uint8_t *src) __attribute__((always_inline)) {                    // per-lane address
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(dst), "v"(src) : "memory", "m0");
    };
    auto load4_at = [&](unsigned dst, const void *src) __attribute__((always_inline)) {                      // four bytes per lane
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off" ::"s"(dst), "v"(src) : "memory", "m0");
    };
    const int whole = (kend - kbeg) / TK;            // tiles [0, whole) hold TK rows of the range, ...
    int blk0 = 0, blk1 = 0;                          // ... those outside [blk0, blk1) among them rows of the cache only
    if (blen) {
        const long s0 = min(max((long)bstart, (long)kbeg), (long)kend), s1 = min(max((long)bstart + blen, (long)kbeg), (long)kend);
        if (s1 > s0) {
            blk0 = (int)(s0 - kbeg) / TK;
            blk1 = ((int)(s1 - kbeg) + TK - 1) / TK;
        }
    }
    // Where this lane's loads of a tile come from: scalar addresses plus the lane's offset where the tile lies in the cache,
    // otherwise every lane chooses, and rows at or past the end of the range (all of them in a stand-in tile past it) repeat
    // its last row (finite stand-ins, masked or zeroed below).
    struct Source { const uint8_t *k[NK], *v[NV]; };
    auto source_of = [&](int tile) __attribute__((always_inline)) {
        Source r;
        const int k0 = kbeg + tile * TK;
        if (tile < whole && (unsigned)(tile - blk0) >= (unsigned)(blk1 - blk0)) {
#pragma unroll
            for (int i = 0; i < NK; ++i) r.k[i] = kc + (ptrdiff_t)k0 * KROWB + i * kDuoWaves * 1024 + koff;
#pragma unroll
            for (int i = 0; i < NV; ++i) r.v[i] = vc + (ptrdiff_t)k0 * ROWB + i * kDuoWaves * 1024 + voff;
        } else {
#pragma unroll
            for (int i = 0; i < NK; ++i) {
                const int j = min(k0 + i * kDuoWaves * KDMA_ROWS + krow0, kend - 1);
                const bool in_blk = (unsigned)j - (unsigned)bstart < (unsigned)blen;
                r.k[i] = (in_blk ? kb_ : kc) + (size_t)(in_blk ? j - bstart : j) * KROWB + kchunk;
            }
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int j = min(k0 + i * kDuoWaves * VDMA_ROWS + vrow0, kend - 1);
                const bool in_blk = (unsigned)j - (unsigned)bstart < (unsigned)blen;
                r.v[i] = (in_blk ? vb_ : vc) + (size_t)(in_blk ? j - bstart : j) * ROWB + vchunk;
            }
        }
        return r;
    };
    auto load_k = [&](const Source &src, int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NK; ++i) load_at(lds0 + slot * SLOTB + (i * kDuoWaves + wave) * 1024, src.k[i]);
    };
    auto load_v = [&](const Source &src, int slot, int first, int last) __attribute__((always_inline)) {
#pragma unroll
        for (int i = first; i < last; ++i) load_at(lds0 + slot * SLOTB + KTILEB + (i * kDuoWaves + wave) * 1024, src.v[i]);
    };
    const int v = v_first + l32;
    const bool row_ok = v < rows_total;
    // ---- prologue: this wave's scales and the workgroup's Q rows (these pass through the last ring slot), then RING - 1 tiles
    if (a.q_scale)
        load4_at((unsigned)(size_t)(__attribute__((address_space(3))) void *)qs_sh + wave * 256, a.q_scale + kv_head * a.group + min(v, rows_total - 1) / a.Nq);
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const int r = min(v_tile + i * kDuoWaves * KDMA_ROWS + krow0, rows_total - 1);
        load_at(lds0 + (RING - 1) * SLOTB + (i * kDuoWaves + wave) * 1024, h.Q + (row_base + r) * KROWB + kchunk);
    }
#pragma unroll
    for (int t = 0; t < RING - 1; ++t) {
        const Source src = source_of(t);
        load_k(src, t);
        load_v(src, t, 0, NV);
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
    const char *const lds = reinterpret_cast<const char *>(KV);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((RING - 1) * NLOADS) : "memory");
    // Q fragments (B operand of S^T = K Q^T): lane (query l32, half hh) holds 16-byte chunk 2 f + hh of its row
    intx4 qf[KF];
#pragma unroll
    for (int f = 0; f < KF; ++f)
        qf[f] = *reinterpret_cast<const intx4 *>(lds + (RING - 1) * SLOTB + rg * 32 * KROWB + k_off[f]);
    float c = a.scale_log2;                          // scores are exponentiated as 2^(s*c)
    if (a.q_scale) c *= qs_sh[wave][lane];
    if (a.k_scale) c *= uniform_load(a.k_scale + kv_head);

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
    // running maximum (any common factor 2^-m cancels): a unit first takes its weights with the one in use, and only if some
    // weight reached 2 - one bit of its bf16 pattern, the packed weights are or-ed together - it is raised to the unit's maximum
    // + 7, the sums are scaled and the weights taken again.  The first unit always does.
    float nm = INFINITY;
    // One 32-key unit (tile `tile`, in slot `slot`); the loads of `next` are dealt out over it: issued together they queue at
    // the compute unit's memory path.
    auto unit = [&](int tile, int slot, const Source &next, int next_slot) __attribute__((always_inline)) {
        const char *const kt = lds + slot * SLOTB + ph * 32 * KROWB, *const vt = lds + slot * SLOTB + KTILEB + ph * 32 * ROWB;
        intx4 kf[KF];
#pragma unroll
        for (int f = 0; f < KF; ++f) kf[f] = *reinterpret_cast<const intx4 *>(kt + k_off[f]);
        load_k(next, next_slot);
        // The scores are a chain: every instruction waits for the one before.  V^T fragments (dims 32 i + l32, keys 16 st + 4 hh +
        // {0..3, 8..11} of the unit) are read between its links.
        floatx16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
        constexpr int NS = FP8 ? KF / 2 : KF, VPS = 2 * DC / NS;             // links; fragments per link
        static_assert(VPS * NS == 2 * DC, "whole fragments per link");
        bf16x8 vf[2][DC];
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            if constexpr (FP8) {
                const intx8 kx = __builtin_shufflevector(kf[2 * j], kf[2 * j + 1], 0, 1, 2, 3, 4, 5, 6, 7);
                const intx8 qx = __builtin_shufflevector(qf[2 * j], qf[2 * j + 1], 0, 1, 2, 3, 4, 5, 6, 7);
                s = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(kx, qx, s, 0, 0, 0, 0x7F7F7F7F, 0, 0x7F7F7F7F);
            } else {
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[j]), __builtin_bit_cast(bf16x8, qf[j]), s, 0, 0, 0);
            }
#pragma unroll
            for (int n = j * VPS; n < (j + 1) * VPS; ++n) {
                const int st = n / DC, i = n % DC;
                const char *p = vt + 16 * st * ROWB + v_off[i];
                const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v *)(p));
                const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v *)(p + 8 * ROWB));
                const short8v w = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                vf[st][i] = __builtin_bit_cast(bf16x8, w);
            }
            if (j == NS / 2 - 1) load_v(next, next_slot, 0, NV / 2);
        }
        load_v(next, next_slot, NV / 2, NV);
        if (tile == whole) {                                 // (a tile with rows past the end of the range)
            // score register r is key key0 + 8 (r / 4) + 4 hh + (r % 4) for query row l32
            const int key0 = kbeg + tile * TK + 32 * ph;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (key0 + 8 * (r >> 2) + 4 * hh + (r & 3) >= kend) s[r] = -INFINITY;
        }
        unsigned pk[2][4], seen = 0u;                        // P^T as the B operand of O^T += V^T P^T
#pragma unroll
        for (int r = 0; r < 16; r += 2)
            pk[r >> 3][(r & 7) >> 1] = duo_pack(duo_exp2(fmaf(s[r], c, nm)), duo_exp2(fmaf(s[r + 1], c, nm)));
#pragma unroll
        for (int k = 0; k < 8; ++k) seen |= pk[k >> 2][k & 3];
        if (__any((seen & 0x40004000u) != 0u)) {
            const u32x2 both = duo_swap(seen, seen);
            const bool raise = ((both.x | both.y) & 0x40004000u) != 0u;
            float mx = s[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
            const u32x2 mm = duo_swap(__float_as_uint(mx), __float_as_uint(mx));
            mx = fmaxf(__uint_as_float(mm.x), __uint_as_float(mm.y)) * c + kDuoMargin;
            const float m_old = -nm, m_new = raise ? fmaxf(m_old, mx) : m_old;
            const float corr = m_new == m_old ? 1.0f : duo_exp2(m_old - m_new);          // first unit: 2^(-inf) = 0
            const float use = m_new == -INFINITY ? 0.f : -m_new;                         // every score so far is -inf: weights 0
            nm = -m_new;
#pragma unroll
            for (int r = 0; r < 4; ++r) acc_l[r] *= corr;
#pragma unroll
            for (int i = 0; i < DC; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][r] *= corr;
#pragma unroll
            for (int r = 0; r < 16; r += 2)
                pk[r >> 3][(r & 7) >> 1] = duo_pack(duo_exp2(fmaf(s[r], c, use)), duo_exp2(fmaf(s[r + 1], c, use)));
        }
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
    };

    // ---- tiles.  The barrier of tile t waits until this wave's loads of the RING - 2 newer tiles are the only ones outstanding,
    // i.e. tile t has landed, and tells that every wave is done with tile t - 1 (its LDS reads included), whose slot then receives
    // tile t + RING - 1 (past the end: a stand-in, so that the counts stay the same).
    int slot = 0;
    for (int t = 0; t < ntiles; ++t) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((RING - 2) * NLOADS) : "memory");
        const int k0 = kbeg + t * TK;
        if (t == whole) {
            // V rows past the end have weight zero, but zero times an infinity is a NaN: zeroed by the lanes that loaded them
#pragma unroll
            for (int i = 0; i < NV; ++i)
                if (k0 + i * kDuoWaves * VDMA_ROWS + vrow0 >= kend)
                    KV[(slot * SLOTB + KTILEB + (i * kDuoWaves + wave) * 1024) / 16 + lane] = make_uint4(0u, 0u, 0u, 0u);
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        const Source next = source_of(t + RING - 1);
        const int next_slot = slot == 0 ? RING - 1 : slot - 1;
        if (wave_active && k0 + 32 * ph < kend) unit(t, slot, next, next_slot);
        else {
            load_k(next, next_slot);
            load_v(next, next_slot, 0, NV);
        }
        slot = slot + 1 == RING ? 0 : slot + 1;
    }
    const float mc = -nm;

    // ---- merge the P states of a row block through LDS: a wave parks the groups of O registers that others finish
    const u32x2 ls = duo_swap(__float_as_uint(acc_l[0]), __float_as_uint(acc_l[0]));
    const float l_own = __uint_as_float(ls.x) + __uint_as_float(ls.y);
    __builtin_amdgcn_s_waitcnt(duo_waitcnt_vm(0));           // stand-ins may still be on their way
    __syncthreads();
    float4 *park = reinterpret_cast<float4 *>(KV);
    auto park_at = [&](int w, int from_ph, int to_ph, int g) __attribute__((always_inline)) {
        return ((w * (P - 1) + (to_ph < from_ph ? to_ph : to_ph - 1)) * GP + g) * 64 + lane;
    };
    if (wave_active) {
        ml_sh[wave][0][l32] = mc;
        ml_sh[wave][1][l32] = l_own;
#pragma unroll
        for (int to = 0; to < P; ++to)
            if (to != ph) {
#pragma unroll
                for (int g = 0; g < GP; ++g) {
                    const int i = (to * GP + g) / 4, r = 4 * ((to * GP + g) % 4);
                    park[park_at(wave, ph, to, g)] = make_float4(acc[i][r], acc[i][r + 1], acc[i][r + 2], acc[i][r + 3]);
                }
            }
    }
    __syncthreads();
    if (!wave_active) return;
    float m_all = -INFINITY, wgt[P], l_tot = 0.f;
#pragma unroll
    for (int q = 0; q < P; ++q) m_all = fmaxf(m_all, ml_sh[q * R + rg][0][l32]);
#pragma unroll
    for (int q = 0; q < P; ++q) {
        const float m = ml_sh[q * R + rg][0][l32];
        wgt[q] = m == -INFINITY ? 0.f : duo_exp2(m - m_all);                 // a phase that saw no key weighs nothing
        l_tot += ml_sh[q * R + rg][1][l32] * wgt[q];
    }
    float o[GP][4];
#pragma unroll
    for (int to = 0; to < P; ++to)
        if (to == ph) {
#pragma unroll
            for (int g = 0; g < GP; ++g)
#pragma unroll
                for (int k = 0; k < 4; ++k) o[g][k] = acc[(to * GP + g) / 4][4 * ((to * GP + g) % 4) + k];
        }
    float w_own = wgt[0];
#pragma unroll
    for (int q = 1; q < P; ++q) w_own = ph == q ? wgt[q] : w_own;
#pragma unroll
    for (int g = 0; g < GP; ++g)
#pragma unroll
        for (int k = 0; k < 4; ++k) o[g][k] *= w_own;
#pragma unroll
    for (int q = 0; q < P; ++q)
        if (q != ph) {
#pragma unroll
            for (int g = 0; g < GP; ++g) {
                const float4 x = park[park_at(q * R + rg, q, ph, g)];
                o[g][0] += x.x * wgt[q]; o[g][1] += x.y * wgt[q]; o[g][2] += x.z * wgt[q]; o[g][3] += x.w * wgt[q];
            }
        }
    // ---- output: group g of this wave is dims 8 (ph GP + g) + 4 hh .. + 3 of query row l32
    const size_t orow = row_base + v;
    if (h.splits == 1) {
        const float inv = 1.0f / l_tot;
        uint16_t *out = static_cast<uint16_t *>(a.O) + orow * D;
        static_assert(GP % 2 == 0, "groups are stored in pairs");
#pragma unroll
        for (int g = 0; g < GP; g += 2) {
            // the halves exchange words so that each lane stores eight consecutive dims
            const u32x2 x0 = duo_swap(duo_pack(o[g][0] * inv, o[g][1] * inv), duo_pack(o[g + 1][0] * inv, o[g + 1][1] * inv));
            const u32x2 x1 = duo_swap(duo_pack(o[g][2] * inv, o[g][3] * inv), duo_pack(o[g + 1][2] * inv, o[g + 1][3] * inv));
            if (row_ok) *reinterpret_cast<uint4 *>(out + 8 * (ph * GP + g + hh)) = make_uint4(x0.x, x1.x, x0.y, x1.y);
        }
    } else if (row_ok) {
        float *po = a.part_o + (orow * h.splits + sp) * D;
#pragma unroll
        for (int g = 0; g < GP; ++g) *reinterpret_cast<float4 *>(po + 8 * (ph * GP + g) + 4 * hh) = make_float4(o[g][0], o[g][1], o[g][2], o[g][3]);
        if (hh == 0 && ph == 0) {
            float *ml = a.part_ml + (orow * h.splits + sp) * 2;
            ml[0] = m_all;
            ml[1] = l_tot;
        }
    }
#endif
}

template <int R, int RING8, int RING16>
hipError_t launch_duo(const AttnArgs &a, hipStream_t stream)
{
    AttnKernelArgs k;
    fill_kernel_args(a, k, 32 * R, 32 * (kDuoWaves / R));
    k.wgs = (int)((long)a.B * a.Hkv * k.row_tiles * k.splits);
    const dim3 grid((unsigned)k.wgs), block(kDuoThreads);
    hipError_t e;
    if (a.qk_dtype == 2) e = launch_headed(attn_duo_kernel<128, true, R, RING8>, grid, block, stream, k);
    else if (a.d == 128) e = launch_headed(attn_duo_kernel<128, false, R, RING16>, grid, block, stream, k);
    else                 e = launch_headed(attn_duo_kernel<64, false, R, 4>, grid, block, stream, k);
    return e != hipSuccess ? e : finish_attention(a, k.splits, stream);
}

}  // namespace

bool attn_duo_serves(const AttnArgs &a)
{
    return a.v_dtype == 1 && a.q_mx == nullptr && (a.qk_dtype == 1 || (a.qk_dtype == 2 && a.d == 128));
}

// Drafter calls.  One workgroup occupies a compute unit, so what counts is the time of one: its tiles, and the merge if the key
// range is split until the 256 compute units are taken.  Tenths of a microsecond, fitted to measured calls: 128 keys cost
// 18 on two row blocks and 24 on four (fp8 keys or 64 head dims: 12.5 and 21), `s` splits 60 + 6 s.  us per call on two / four
// blocks: 8 x 28/4 heads, 48 rows, 1111 keys bf16 20.5 / 24.5, fp8 16.9 / 22.7; 7 x 32/8, 48 rows, 2900 keys bf16 47.1 / 37.2 (2
// splits); 9 x 32/8, 24 rows, 3000 keys fp8 33.4 / 29.2 (3 splits); 4 x 32/8, 32 rows, 4096 keys fp8 22.7 (4 splits) / 24.9 (8), unsplit
// 39.9; four blocks unsplit / split: 5 x 32/8, 64 rows, 1500 keys bf16 30.0 / 25.1 (3 splits), fp8 27.8 / 24.9 (20.2 on two).
// More than one round of 64-row workgroups: 128 rows.  More than one of these: nothing here (see the caller).
DuoPlan attn_duo_plan(long rows, long heads, int N, bool light)
{
    const int forced = tune("DD_TUNE_DUO", -1), forced_splits = tune("DD_TUNE_BLOCK_SPLITS", 0);
    const long tiles = (N + 127) / 128;
    DuoPlan best{0, 1};
    long best_cost = 0;
    for (int blocks = 2; blocks <= 4; blocks += 2) {
        const long wgs = heads * ((rows + 32 * blocks - 1) / (32 * blocks));
        if (forced >= 0 ? forced != blocks : wgs > 256) continue;
        const long per_tile = blocks == 2 ? (light ? 125 : 180) : (light ? 210 : 240);
        long most = forced_splits >= 1 ? forced_splits : 256 / (wgs < 256 ? wgs : 256);
        if (most > tiles / 2) most = tiles / 2;
        if (most > 16) most = 16;
        for (int i = 0; i < 2; ++i) {                // not split, or as far as it goes
            const long s = i == 0 ? 1 : most;
            if (i == 1 && s <= 1) break;
            const long cost = (tiles + s - 1) / s * per_tile + (s > 1 ? 600 + 60 * s : 0);
            if (best.blocks == 0 || cost < best_cost || (i == 1 && forced_splits > 1)) {
                best = DuoPlan{blocks, (int)s};
                best_cost = cost;
            }
        }
    }
    return best;
}

hipError_t launch_attention_duo(const AttnArgs &a, int blocks, hipStream_t stream)
{
    return blocks == 4 ? launch_duo<4, 4, 4>(a, stream) : launch_duo<2, 3, 2>(a, stream);
}

}  // namespace dd

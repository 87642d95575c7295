// Drafter attention over the cached K/V (Sec. 2.3), streaming form (bf16, or fp8 Q/K with 128 head dims):
//     O = softmax(Q_blk K^T / sqrt(d_k)) V     for the block_len queries of the active block (Eq. 3),
// key/value row j coming from the block tensors inside the block and from the cache elsewhere.
//
// With a few dozen query rows per head this call is bound by reading K and V once, so the kernel is
// built around the memory pipeline, not the matrix cores:
//   - K/V tiles of 64 keys go from global memory straight into LDS (global_load_lds_dwordx4, no
//     staging registers) through a ring of four tile buffers (fp8: three): three tiles (96 KB per compute unit; fp8: two
//     of 24 KB, twice per compute unit) are always in flight while another is consumed.  The barrier that opens a tile only
//     waits until the newest two (fp8: the newest) are the only loads outstanding (memory operations complete in order).  The
//     compiler would wait for every outstanding LDS load before any read of such a buffer, so the
//     operand reads of the tiles are written as inline assembly with their own wait;
//   - one workgroup = 4 waves (one per SIMD) owns up to 64 query rows of one (batch, kv head): wave w holds
//     the 32-row block w % 2 and takes unit w / 2 of every tile (two key phases), so all four waves work on
//     every tile; the two phases of a row block merge their (max, sum, O) states through LDS at the end.
//     Calls with more than 64 rows per kv head stay with the MFMA kernel of attention_mfma.hip;
//   - per unit a wave simply runs S = K Q^T, the online softmax and O += V P back to back.
// K is XOR-swizzled for its 16-byte operand reads; V stays row-major (swizzled in 64-byte granules) and
// its transposed operand comes from ds_read_b64_tr_b16.
// The key range can also be split over workgroups; their partial states go to the workspace and are
// merged by the combine kernel of attention_mfma.hip.
#include "attention_common.h"
#include "dd_internal.h"

#include <type_traits>

namespace dd {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef int intx8 __attribute__((ext_vector_type(8)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));

constexpr int TKS = 64;                 // keys per tile
constexpr int QBS = 1;                  // 32-row query blocks per wave
constexpr int kRowsWaveS = 32 * QBS;
constexpr float kSlackS = 8.0f;         // the maximum in use is raised when exceeded by 2^8

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ unsigned pack2_bf16(float lo, float hi)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    floatx2 f = {lo, hi};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2));
}
__device__ __forceinline__ float swap_max(float x)
{
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
}
__device__ __forceinline__ float swap_sum(float x)
{
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r.x) + __uint_as_float(r.y);
}

// s_waitcnt immediate: wait until at most n vector-memory operations are outstanding, nothing else
constexpr int waitcnt_vm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

// NT: the K/V tiles are loaded with the non-temporal hint (see the launcher).
// FP8: Q and K are e4m3 codes with per-head scales (in the exponent's factor), V bf16.  K tiles stay as stored, 128-byte
// rows; S = K Q^T is two 64-deep fp8 matrix instructions per unit (the block-scaled one with the neutral scale code 127:
// of a lane's 32 operand bytes the first 16 are dims 16 hh .. of the 64, the last 16 dims 32 + 16 hh ..).  A tile is 24 KB
// instead of 32 and what bounds a workgroup is its chain of dependent steps per tile, some 1.3 us however many bytes: three
// tile buffers and half the registers let two workgroups share a compute unit and work in each other's gaps (with four
// buffers, alone on it: 24.0 us for the first call below).  us per call against the MFMA kernel, which transposes V through
// registers: 11 x 32 / 8 heads, 16 rows, 1237 keys 21.2 -> 18.6; 1 x 32, 512 keys 12.8 -> 9.2; 8 x 32, 64 rows, 1024 keys 29.5
// -> 21.6 (4.9 TB/s); 16 x 32, 64 rows, 4096 keys 164.9 -> 149.7 (5.4 TB/s).
template <int D, bool NT, bool FP8>
__global__ __launch_bounds__(kAttnThreads) __attribute__((amdgpu_waves_per_eu(FP8 ? 2 : 1, FP8 ? 2 : 1)))
void attn_stream_kernel(DD_ATTN_HEAD, const AttnTail a)
{
    const AttnHead h = DD_ATTN_HEAD_ARGS;
    constexpr int CH = D / 8;                        // 16-byte chunks (8 bf16) per row
    constexpr int KS = D / 16;                       // MFMA k-steps over the head dim
    constexpr int DC = D / 32;                       // 32-wide chunks of the head dim
    constexpr int ROWB = D * 2;                      // bytes per K / V row
    constexpr int DMA_ROWS = 1024 / ROWB;            // rows moved by one wave-wide 16-byte-per-lane load
    constexpr int NDMA = TKS / DMA_ROWS / 4;         // such loads per wave per K or V tile
    static_assert((4 * DMA_ROWS) % 8 == 0, "swizzle phase must not depend on the load index");
    static_assert(!FP8 || D == 128, "fp8 K rows are 128 bytes");
    constexpr int KROWB = FP8 ? D : ROWB, KCH = KROWB / 16;   // K as stored: bytes and chunks per row, ...
    constexpr int KDMA_ROWS = 1024 / KROWB, KDMA = TKS / KDMA_ROWS / 4;      // ... rows per load, loads per wave and tile
    constexpr int NLOADS = KDMA + NDMA;              // loads per wave and tile
    constexpr int KF = KROWB / 32;                   // 16-byte K fragments per lane and unit

    constexpr int kRing = FP8 ? 3 : 4;               // tile buffers
    constexpr int TILEB = TKS * ROWB, KTILEB = TKS * KROWB;   // bytes of one V / K tile
    constexpr int STATE = QBS * DC * 16 * 64;        // floats of a wave's O state
    static_assert(4 * STATE * 4 <= kRing * (TILEB + KTILEB), "the waves' O states must fit the ring");
    __shared__ __attribute__((aligned(1024))) uint4 KV[kRing * TKS * (KCH + CH)];   // K ring [key][chunk ^ (key & 7)], then
                                                     // V ring [key][chunk ^ ((key % (CH/4)) << 2)]
    __shared__ float ml_sh[4][2][64];                // per wave: (max, sum) of its query block, for the phase merge

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hh = lane >> 5;
    const int rg = wave & 1, ph = wave >> 1;         // row block, key phase

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
    const int v_first = rt * 2 * kRowsWaveS + rg * kRowsWaveS;
    const bool wave_active = v_first < rows_total;
    const size_t row_base = kv_head * rows_total;
    const int kbeg = sp * h.keys_per_split;
    const int kend = min(h.N, kbeg + h.keys_per_split);
    // (any value is safe: rows are chosen by range test)
    const int bstart = a.block_starts ? uniform_load(a.block_starts + (unsigned)kv_head / (unsigned)a.Hkv) : h.block_start;
    const int ntiles = (kend - kbeg + TKS - 1) / TKS;

    // ---- staging by LDS DMA: load i of this wave moves rows (4i + wave) * DMA_ROWS .. of a tile; lane l
    // lands at chunk position l % CH of row l / CH and therefore fetches the chunk the swizzle maps there.
    const int dma_row = lane / CH, dma_pos = lane % CH;
    const int dma_row0 = wave * DMA_ROWS + dma_row;
    const int kdma_row0 = wave * KDMA_ROWS + lane / KCH;
    const unsigned dma_koff = (lane % KCH ^ (kdma_row0 & 7)) * 16;
    const unsigned dma_voff = (dma_pos ^ ((dma_row0 & (CH / 4 - 1)) << 2)) * 16;
    const uint8_t *const kc = h.K + kv_head * h.kv_stride * (size_t)KROWB;
    const uint8_t *const vc = h.V + kv_head * h.kv_stride * (size_t)ROWB;
    const uint8_t *const kb_ = h.block_len ? static_cast<const uint8_t *>(a.Kblk) + kv_head * h.block_len * (size_t)KROWB : nullptr;
    const uint8_t *const vb_ = h.block_len ? static_cast<const uint8_t *>(a.Vblk) + kv_head * h.block_len * (size_t)ROWB : nullptr;
    // rows of the last tile at or past the end of the key range repeat its last row (finite stand-ins, masked later)
    auto dma_tile = [&](int tile) __attribute__((always_inline)) {
        uint4 *kd = KV + (tile % kRing) * (TKS * KCH), *vd = KV + kRing * TKS * KCH + (tile % kRing) * (TKS * CH);
#pragma unroll
        for (int i = 0; i < NDMA; ++i) {
            if (i < KDMA) {
                const int j = min(kbeg + tile * TKS + i * 4 * KDMA_ROWS + kdma_row0, kend - 1);
                const bool in_blk = (unsigned)j - (unsigned)bstart < (unsigned)h.block_len;
                const uint8_t *ks = (in_blk ? kb_ : kc) + (size_t)(in_blk ? j - bstart : j) * KROWB + dma_koff;
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)ks,
                                                 (__attribute__((address_space(3))) void *)(kd + (i * 4 + wave) * 64), 16, 0, NT ? 2 : 0);
            }
            const int j = min(kbeg + tile * TKS + i * 4 * DMA_ROWS + dma_row0, kend - 1);
            const bool in_blk = (unsigned)j - (unsigned)bstart < (unsigned)h.block_len;
            const uint8_t *vs = (in_blk ? vb_ : vc) + (size_t)(in_blk ? j - bstart : j) * ROWB + dma_voff;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)vs,
                                             (__attribute__((address_space(3))) void *)(vd + (i * 4 + wave) * 64), 16, 0, NT ? 2 : 0);
        }
    };

    // ---- Q fragments (B operand of S^T = K Q^T): lane (query l32, half hh) holds dims 16 ks + 8 hh .. +7
    bool row_ok[QBS];
    float c[QBS];                                    // scores are exponentiated as 2^(s*c)
    bf16x8 qf[QBS][FP8 ? 1 : KS];
    intx8 qx[QBS][FP8 ? D / 64 : 1];
#pragma unroll
    for (int q = 0; q < QBS; ++q) {
        const int v = v_first + q * 32 + l32;
        row_ok[q] = v < rows_total;
        const int vv = row_ok[q] ? v : rows_total - 1;
        if constexpr (FP8) {
            const uint8_t *qrow = h.Q + (row_base + vv) * D + 16 * hh;
#pragma unroll
            for (int j = 0; j < D / 64; ++j) {
                const uint4 lo = *reinterpret_cast<const uint4 *>(qrow + 64 * j), hi = *reinterpret_cast<const uint4 *>(qrow + 64 * j + 32);
                qx[q][j] = intx8{(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
            }
        } else {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                qf[q][ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(
                                reinterpret_cast<const uint16_t *>(h.Q) + (row_base + vv) * D + ks * 16 + hh * 8));
        }
        c[q] = 1.0f;
        if (a.q_scale) c[q] = a.q_scale[kv_head * a.group + vv / a.Nq];
    }
    float k_scale = 1.0f;
    if (a.k_scale) k_scale = uniform_load(a.k_scale + kv_head);
    __builtin_amdgcn_sched_barrier(0);               // these loads are requested before the first tiles ...
    // (a tile past the range repeats its last row)
#pragma unroll
    for (int t0 = 0; t0 < kRing - 1; ++t0) dma_tile(t0);
    // ... and waited for here while the tiles are still on their way: the compiler, left to place this wait, waits for
    // the tiles as well, and the memory pipeline runs empty before the first tile is even looked at
    __builtin_amdgcn_s_waitcnt(waitcnt_vm((kRing - 1) * NLOADS));
#pragma unroll
    for (int q = 0; q < QBS; ++q) c[q] = a.scale_log2 * c[q] * k_scale;

    floatx16 acc[QBS][DC];                           // O^T, unnormalised
#pragma unroll
    for (int q = 0; q < QBS; ++q)
#pragma unroll
        for (int i = 0; i < DC; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[q][i][r] = 0.f;
    float mc[QBS] = {-INFINITY};                     // maximum in use (log2 units), equal in both lane halves
    float l_run[QBS] = {0.f};                        // this lane half's share of the running sums

    // operand addresses inside a tile buffer (bytes), without the unit offset
    int k_off[KF], v_off[DC];
#pragma unroll
    for (int ks = 0; ks < KF; ++ks) k_off[ks] = (l32 * KCH + ((2 * ks + hh) ^ (l32 & 7))) * 16;
    {
        const int t = lane & 15, gq = l32 >> 4, row = 4 * hh + (t >> 2);
#pragma unroll
        for (int i = 0; i < DC; ++i) {
            const int chunk = 4 * i + 2 * gq + ((t & 3) >> 1);
            v_off[i] = (row * CH + (chunk ^ ((row & (CH / 4 - 1)) << 2))) * 16 + (t & 1) * 8;
        }
    }

    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void *)KV;   // LDS byte address of the ring
    // One 32-key unit: S = K Q^T, online softmax, O += V P.  kaddr / vaddr = LDS byte addresses of the
    // unit's first K / V row, key0 = global index of its first key.
    auto unit = [&](unsigned kaddr, unsigned vaddr, int key0) __attribute__((always_inline)) {
        // ---- all K fragments of the unit (keys l32, 16-byte chunks 2 ks + hh of the stored row) in one go, with their wait
        uint4 kf[KF];
        if constexpr (KF == 8) {
            asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
                         "ds_read_b128 %4, %12\n\tds_read_b128 %5, %13\n\tds_read_b128 %6, %14\n\tds_read_b128 %7, %15\n\t"
                         "s_waitcnt lgkmcnt(0)"
                         : "=&v"(kf[0]), "=&v"(kf[1]), "=&v"(kf[2]), "=&v"(kf[3]), "=&v"(kf[4]), "=&v"(kf[5]), "=&v"(kf[6]), "=&v"(kf[7])
                         : "v"(kaddr + k_off[0]), "v"(kaddr + k_off[1]), "v"(kaddr + k_off[2]), "v"(kaddr + k_off[3]),
                           "v"(kaddr + k_off[4]), "v"(kaddr + k_off[5]), "v"(kaddr + k_off[6]), "v"(kaddr + k_off[7])
                         : "memory");
        } else {
            asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\t"
                         "s_waitcnt lgkmcnt(0)"
                         : "=&v"(kf[0]), "=&v"(kf[1]), "=&v"(kf[2]), "=&v"(kf[3])
                         : "v"(kaddr + k_off[0]), "v"(kaddr + k_off[1]), "v"(kaddr + k_off[2]), "v"(kaddr + k_off[3])
                         : "memory");
        }
        floatx16 s[QBS];
#pragma unroll
        for (int q = 0; q < QBS; ++q)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[q][r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < (FP8 ? 0 : KF); ++ks)
#pragma unroll
            for (int q = 0; q < QBS; ++q)
                s[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[ks]), qf[q][ks], s[q], 0, 0, 0);
        if constexpr (FP8) {
#pragma unroll
            for (int j = 0; j < D / 64; ++j) {
                const uint4 lo = kf[2 * j], hi = kf[2 * j + 1];
                const intx8 kx = {(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
#pragma unroll
                for (int q = 0; q < QBS; ++q)
                    s[q] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(kx, qx[q][j], s[q], 0, 0, 0, 0x7F7F7F7F, 0, 0x7F7F7F7F);
            }
        }
        // score register r of a block is key key0 + 8 (r / 4) + 4 hh + (r % 4) for query row l32
        if (key0 + 32 > kend) {
#pragma unroll
            for (int q = 0; q < QBS; ++q)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (key0 + 8 * (r >> 2) + 4 * hh + (r & 3) >= kend) s[q][r] = -INFINITY;
        }
        float tm[QBS];
        bool need = false;
#pragma unroll
        for (int q = 0; q < QBS; ++q) {
            float t = s[q][0];
#pragma unroll
            for (int r = 1; r < 16; ++r) t = fmaxf(t, s[q][r]);
            tm[q] = swap_max(t) * c[q];
            need = need || (tm[q] > mc[q] + kSlackS);
        }
        if (__any(need)) {                                   // rare after the first units: raise the maxima in use
#pragma unroll
            for (int q = 0; q < QBS; ++q) {
                const float mn = fmaxf(mc[q], tm[q]);
                const float corr = exp2_fast(mc[q] - mn);    // first unit: 2^(-inf) = 0
                mc[q] = mn;
                l_run[q] *= corr;
#pragma unroll
                for (int i = 0; i < DC; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[q][i][r] *= corr;
            }
        }
        unsigned pk[QBS][2][4];                              // P^T as the B operand of O^T += V^T P^T
#pragma unroll
        for (int q = 0; q < QBS; ++q) {
            float lsum = 0.f;
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const float p0 = exp2_fast(fmaf(s[q][r], c[q], -mc[q]));
                const float p1 = exp2_fast(fmaf(s[q][r + 1], c[q], -mc[q]));
                lsum += p0 + p1;
                pk[q][r >> 3][(r & 7) >> 1] = pack2_bf16(p0, p1);
            }
            l_run[q] += lsum;
        }
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            // V^T fragments of 16 keys: dims 32 i + l32, keys 16 st + 4 hh + {0..3, 8..11} of the unit
            uint2 lo[DC], hi[DC];
            const unsigned va = vaddr + 16 * st * ROWB;
            if constexpr (DC == 4) {
                asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:%12\n\t"
                             "ds_read_b64_tr_b16 %2, %9\n\tds_read_b64_tr_b16 %3, %9 offset:%12\n\t"
                             "ds_read_b64_tr_b16 %4, %10\n\tds_read_b64_tr_b16 %5, %10 offset:%12\n\t"
                             "ds_read_b64_tr_b16 %6, %11\n\tds_read_b64_tr_b16 %7, %11 offset:%12\n\t"
                             "s_waitcnt lgkmcnt(0)"
                             : "=&v"(lo[0]), "=&v"(hi[0]), "=&v"(lo[1]), "=&v"(hi[1]), "=&v"(lo[2]), "=&v"(hi[2]), "=&v"(lo[3]), "=&v"(hi[3])
                             : "v"(va + v_off[0]), "v"(va + v_off[1]), "v"(va + v_off[2]), "v"(va + v_off[3]), "n"(8 * ROWB)
                             : "memory");
            } else {
                asm volatile("ds_read_b64_tr_b16 %0, %4\n\tds_read_b64_tr_b16 %1, %4 offset:%6\n\t"
                             "ds_read_b64_tr_b16 %2, %5\n\tds_read_b64_tr_b16 %3, %5 offset:%6\n\t"
                             "s_waitcnt lgkmcnt(0)"
                             : "=&v"(lo[0]), "=&v"(hi[0]), "=&v"(lo[1]), "=&v"(hi[1])
                             : "v"(va + v_off[0]), "v"(va + v_off[1]), "n"(8 * ROWB)
                             : "memory");
            }
#pragma unroll
            for (int i = 0; i < DC; ++i) {
                const uint4 w = make_uint4(lo[i].x, lo[i].y, hi[i].x, hi[i].y);
#pragma unroll
                for (int q = 0; q < QBS; ++q) {
                    const uint4 pw = make_uint4(pk[q][st][0], pk[q][st][1], pk[q][st][2], pk[q][st][3]);
                    acc[q][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, pw),
                                                                        acc[q][i], 0, 0, 0);
                }
            }
        }
    };

    // ---- tiles.  Tile t sits in ring slot t % kRing.  Its barrier waits until this wave's loads of the (up to
    // kRing - 2) newer tiles are the only ones outstanding - i.e. tile t has landed - and tells that every wave is
    // done with tile t-1, whose slot then receives tile t + kRing - 1.  A wave takes the unit of its key phase.
    for (int t = 0; t < ntiles; ++t) {
        const int newer = ntiles - 1 - t;                    // tiles after t (all requested up to t + kRing - 2)
        if (newer >= kRing - 2 || t == 0) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((kRing - 2) * NLOADS) : "memory");
        else if (newer >= 1) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(NLOADS) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        if (t + kRing - 1 < ntiles) dma_tile(t + kRing - 1);
        if (wave_active) {
            const unsigned slot = (unsigned)(t % kRing);
            const int key0 = kbeg + t * TKS + 32 * ph;
            if (key0 < kend) unit(lds0 + slot * KTILEB + ph * 32 * KROWB, lds0 + kRing * KTILEB + slot * TILEB + ph * 32 * ROWB, key0);
        }
    }

    float l_tot[QBS];
#pragma unroll
    for (int q = 0; q < QBS; ++q) l_tot[q] = swap_sum(l_run[q]);

    // ---- merge the two key phases of a row block through LDS: phase 1 parks its state in slot `wave`
    // of the ring's memory (register r of chunk i at [i 16 + r][lane]), phase 0 adds it to its own
    // (with a single tile the stand-ins behind it may still be on their way, and a barrier by itself waits for nobody's loads)
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __syncthreads();                                         // all waves are done with the ring; its loads have landed
    float *region = reinterpret_cast<float *>(KV) + wave * STATE;
    if (ph != 0 && wave_active) {
#pragma unroll
        for (int i = 0; i < DC; ++i)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4)
                *reinterpret_cast<float4 *>(region + ((i * 4 + r4) * 64 + lane) * 4) =
                    make_float4(acc[0][i][4 * r4], acc[0][i][4 * r4 + 1], acc[0][i][4 * r4 + 2], acc[0][i][4 * r4 + 3]);
        ml_sh[wave][0][lane] = mc[0];
        ml_sh[wave][1][lane] = l_tot[0];
    }
    __syncthreads();
    if (ph == 0 && wave_active) {
        const int w = wave + 2;
        const float *src = reinterpret_cast<const float *>(KV) + w * STATE;
        const float mo = ml_sh[w][0][lane], lo = ml_sh[w][1][lane];
        const float mn = fmaxf(mc[0], mo);
        // a phase that saw no key at all has max -inf and weighs nothing
        const float ws = mc[0] == -INFINITY ? 0.f : exp2_fast(mc[0] - mn);
        const float wo = mo == -INFINITY ? 0.f : exp2_fast(mo - mn);
        l_tot[0] = l_tot[0] * ws + lo * wo;
        mc[0] = mn;
#pragma unroll
        for (int i = 0; i < DC; ++i)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const float4 o = *reinterpret_cast<const float4 *>(src + ((i * 4 + r4) * 64 + lane) * 4);
                acc[0][i][4 * r4] = acc[0][i][4 * r4] * ws + o.x * wo;
                acc[0][i][4 * r4 + 1] = acc[0][i][4 * r4 + 1] * ws + o.y * wo;
                acc[0][i][4 * r4 + 2] = acc[0][i][4 * r4 + 2] * ws + o.z * wo;
                acc[0][i][4 * r4 + 3] = acc[0][i][4 * r4 + 3] * ws + o.w * wo;
            }
    }
    if (ph != 0 || !wave_active) return;

    // ---- output: O^T register r of chunk i holds dim 32 i + 8 (r / 4) + 4 hh + (r % 4) of query row l32
#pragma unroll
    for (int q = 0; q < QBS; ++q) {
        if (!row_ok[q]) continue;
        const size_t orow = row_base + v_first + q * 32 + l32;
        if (h.splits == 1) {
            const float inv = 1.0f / l_tot[q];
            uint16_t *o = static_cast<uint16_t *>(a.O) + orow * D;
#pragma unroll
            for (int i = 0; i < DC; ++i)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const uint2 w = make_uint2(pack2_bf16(acc[q][i][4 * q4] * inv, acc[q][i][4 * q4 + 1] * inv),
                                               pack2_bf16(acc[q][i][4 * q4 + 2] * inv, acc[q][i][4 * q4 + 3] * inv));
                    *reinterpret_cast<uint2 *>(o + i * 32 + q4 * 8 + hh * 4) = w;
                }
        } else {
            float *po = a.part_o + (orow * h.splits + sp) * D;
#pragma unroll
            for (int i = 0; i < DC; ++i)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    *reinterpret_cast<float4 *>(po + i * 32 + q4 * 8 + hh * 4) =
                        make_float4(acc[q][i][4 * q4], acc[q][i][4 * q4 + 1], acc[q][i][4 * q4 + 2], acc[q][i][4 * q4 + 3]);
            if (hh == 0) {
                float *ml = a.part_ml + (orow * h.splits + sp) * 2;
                ml[0] = mc[q];
                ml[1] = l_tot[q];
            }
        }
    }
}

}  // namespace

// The streaming kernel serves calls with at most this many query rows per (batch, kv head).
bool attn_stream_fits(const AttnArgs &a) { return (long)(a.H / a.Hkv) * a.Nq <= 2 * kRowsWaveS; }

constexpr double kStreamPastCacheBytes = 100.0e6;

hipError_t launch_attention_stream(const AttnArgs &a, hipStream_t stream)
{
    AttnKernelArgs k;
    fill_kernel_args(a, k, 2 * kRowsWaveS, TKS);
    k.wgs = (int)((long)a.B * a.Hkv * k.row_tiles * k.splits);
    const dim3 grid((unsigned)k.wgs), block(kAttnThreads);
    // A model's layers take their turns, each with a cache of its own, so a large one has left the 256 MB last-level cache
    // when it is read again: above 100 MB it is streamed past it.  us per call with plain loads -> with the hint, four
    // copies in turn (two of the largest): 67 MB 20.7 -> 22.0, 101 MB 24.9 -> 23.6, 134 MB 29.2 -> 26.6, 252 MB 54.4 -> 50.8,
    // 537 MB 110 -> 101; fp8 101 MB 21.8 -> 20.4, 201 MB 40.9 -> 38.3.  A caller that reads one and the same copy again and
    // again gives up what the cache would have kept of it: 134 MB 24.8 -> 25.3, 252 MB 47.4 -> 50.3, fp8 201 MB 34.7 -> 36.4
    // (537 MB: 117 -> 109).  The verifier's rows share K/V between workgroups: never for them.
    const bool fp8 = a.qk_dtype == 2;
    const bool nt = tune("DD_TUNE_STREAM_NT", a.Nq != a.N && (fp8 ? 3.0 : 4.0) * a.B * a.Hkv * a.N * a.d > kStreamPastCacheBytes) != 0;
    hipError_t e;
    if (fp8)             e = nt ? launch_headed(attn_stream_kernel<128, true, true>, grid, block, stream, k) : launch_headed(attn_stream_kernel<128, false, true>, grid, block, stream, k);
    else if (a.d == 128) e = nt ? launch_headed(attn_stream_kernel<128, true, false>, grid, block, stream, k) : launch_headed(attn_stream_kernel<128, false, false>, grid, block, stream, k);
    else                 e = nt ? launch_headed(attn_stream_kernel<64, true, false>, grid, block, stream, k) : launch_headed(attn_stream_kernel<64, false, false>, grid, block, stream, k);
    return e != hipSuccess ? e : finish_attention(a, k.splits, stream);
}

}  // namespace dd

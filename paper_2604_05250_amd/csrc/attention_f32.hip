// fp32 attention, softmax(Q K^T / sqrt(d_k)) V (Eq. 3) over all key positions (Sec. 2.2), in fp32 throughout, on the
// fp32 matrix instruction (v_mfma_f32_16x16x4_f32: fp32 products and sums).  It serves fp32 inputs (the small
// CPU-checkable configuration) for both the verifier's full attention and the drafter's
// block attention over the cached K/V (Sec. 2.3); the bf16 / fp8 workloads run on the kernels of the other files.
//
// Such calls are small (a few heads, a few hundred keys), so what counts is the length of the dependent chain, not a
// rate: one workgroup takes 16 (or 32) query rows of one (batch, kv head), its eight waves take 16-key units in turn,
// and nothing passes through LDS before the waves' states are merged at the end.  K and V go from memory straight into
// the instruction's operand registers in 16-byte loads; which head dim or key an operand element stands for is free as
// long as both operands agree:
//   S^T = K Q^T   k index g of step (j, e) is head dim 16 j + 4 g + e: lane (key l % 16, g = l / 16) loads
//                 K[key][16 j + 4 g ..+3], the Q fragment likewise.  The result holds, per lane, query l % 16 and keys
//                 4 g + r: the softmax row reductions are in-register plus two lane exchanges;
//   O^T += V^T P^T  k index g of step r is key 4 g + r, so the weights are the B operand as they stand; row m of chunk
//                 (h, e) is head dim 64 h + 4 m + e: lane (m, g) loads V[key][64 h + 4 m ..+3] and its four elements
//                 are the operands of four instructions.
// The next unit's K and V are requested before the current one is worked on.  Measured against the vector-ALU kernel before
// it (one lane per 32 dims of a query row, keys in turn, K/V broadcast from LDS), us per call: the smallest workload (4
// heads, 128 keys, d = 64) 43.2 -> 5.2 (drafter) and 43.8 -> 5.3 (verifier), of which some 4 are any launch; 1 x 32 heads x 512
// keys, d = 128 194 -> 72; 2 x 32 x 1024, d = 64 360 -> 198 (87 TFLOP/s of the instruction's 157).
#include "attention_common.h"
#include "dd_internal.h"

namespace dd {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kThreadsF = 512;
constexpr int kWavesF = kThreadsF / 64;
constexpr int kUnitF = 16;                          // keys per unit
constexpr int kSplitKeys = 256;                     // keys per key split, at least

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// RB: 16-row query blocks per workgroup
template <int D, int RB>
__device__ __forceinline__ void attn_f32(const AttnHead &h, const AttnTail &a)
{
    constexpr int NJ = D / 16;                      // 16-byte fragments of a Q / K row per lane
    constexpr int NH = D / 64;                      // ... of a V row
    // Partial sums of a score, 16 or 32 products each: one chain of d products rounds d times, against fp64 1.0e-6 of the
    // result (d = 128, Q three times N(0, 1), 8 / 2 heads x 16 rows x 700 keys) where four give 4.2e-7 and the vector-ALU
    // kernel, whose lanes summed 32 products each, gave 4.6e-7.  (Two on the 32-row form: 200 us against 203.)
    constexpr int NS = RB == 2 ? 2 : 4;
    constexpr int NO = NH * 4;                      // 16-byte pieces of an O row per lane
    __shared__ floatx4 states[kWavesF * RB * NO * 64];
    __shared__ float ml[kWavesF][RB][2][16];        // per wave: (max in use, sum) of its query rows

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    unsigned bid = blockIdx.x;
    int sp, rt;
    place_of(bid, h.splits, sp);
    place_of(bid, h.row_tiles, rt);
    const size_t kv_head = bid;                     // batch and kv head; its query rows are contiguous in memory
    const int rows_total = h.rows_total;
    const size_t row_base = kv_head * rows_total;

    const int k_begin = sp * h.keys_per_split;
    const int k_end = min(h.N, k_begin + h.keys_per_split);
    // (any value is safe: rows are chosen by range test)
    const int bstart = a.block_starts ? uniform_load(a.block_starts + (unsigned)kv_head / (unsigned)a.Hkv) : h.block_start;
    const float *const kc = reinterpret_cast<const float *>(h.K) + kv_head * h.kv_stride * D;
    const float *const vc = reinterpret_cast<const float *>(h.V) + kv_head * h.kv_stride * D;
    const float *const kb = h.block_len ? static_cast<const float *>(a.Kblk) + kv_head * h.block_len * D : nullptr;       // (length 0: no block)
    const float *const vb = h.block_len ? static_cast<const float *>(a.Vblk) + kv_head * h.block_len * D : nullptr;

    floatx4 qf[RB][NJ], acc[RB][NO], kf[2][NJ], vf[2][4][NH];
    float c[RB], m_run[RB], l_run[RB];
    // rows past the end of the range repeat its last one (their scores are masked, their values zeroed before use)
    auto load_unit = [&](int u, floatx4 (&k)[NJ], floatx4 (&v)[4][NH]) __attribute__((always_inline)) {
        const int j0 = k_begin + u * kUnitF;
        {
            const int j = min(j0 + l16, k_end - 1);
            const bool in_blk = (unsigned)j - (unsigned)bstart < (unsigned)h.block_len;
            const float *p = (in_blk ? kb + (size_t)(j - bstart) * D : kc + (size_t)j * D) + 4 * g;
#pragma unroll
            for (int i = 0; i < NJ; ++i) k[i] = *reinterpret_cast<const floatx4 *>(p + 16 * i);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = min(j0 + 4 * g + r, k_end - 1);
            const bool in_blk = (unsigned)j - (unsigned)bstart < (unsigned)h.block_len;
            const float *p = (in_blk ? vb + (size_t)(j - bstart) * D : vc + (size_t)j * D) + 4 * l16;
#pragma unroll
            for (int h = 0; h < NH; ++h) v[r][h] = *reinterpret_cast<const floatx4 *>(p + 64 * h);
        }
    };
    const int units = (k_end - k_begin + kUnitF - 1) / kUnitF;
    if (wave < units) load_unit(wave, kf[0], vf[0]);
#pragma unroll
    for (int q = 0; q < RB; ++q) {
        const int v = min((rt * RB + q) * 16 + l16, rows_total - 1);
        const float *p = reinterpret_cast<const float *>(h.Q) + (row_base + v) * D + 4 * g;
#pragma unroll
        for (int i = 0; i < NJ; ++i) qf[q][i] = *reinterpret_cast<const floatx4 *>(p + 16 * i);
        c[q] = a.scale_log2;
        if (a.q_scale) c[q] *= a.q_scale[kv_head * a.group + v / a.Nq];
        if (a.k_scale) c[q] *= a.k_scale[kv_head];
        m_run[q] = -INFINITY;
        l_run[q] = 0.f;
#pragma unroll
        for (int i = 0; i < NO; ++i) acc[q][i] = floatx4{0.f, 0.f, 0.f, 0.f};
    }

    auto unit = [&](int u, const floatx4 (&k)[NJ], floatx4 (&v)[4][NH]) __attribute__((always_inline)) {
        const int j0 = k_begin + u * kUnitF;
        if (j0 + kUnitF > k_end) {                           // (zero times an infinite value would be a NaN)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (j0 + 4 * g + r >= k_end)
#pragma unroll
                    for (int h = 0; h < NH; ++h) v[r][h] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            floatx4 part[NS];
#pragma unroll
            for (int e = 0; e < NS; ++e) part[e] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < NJ; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) part[e % NS] = __builtin_amdgcn_mfma_f32_16x16x4f32(k[i][e], qf[q][i][e], part[e % NS], 0, 0, 0);
            floatx4 s = part[0] + part[1];
            if constexpr (NS == 4) s += part[2] + part[3];
            if (j0 + kUnitF > k_end) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (j0 + 4 * g + r >= k_end) s[r] = -INFINITY;
            }
            float t = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
            t = fmaxf(t, __shfl_xor(t, 16));
            t = fmaxf(t, __shfl_xor(t, 32));
            const float m_new = fmaxf(m_run[q], t);
            // (a unit whose scores are all -inf before any finite one: weights 0, not 2^(-inf + inf))
            const float m_ref = m_new == -INFINITY ? 0.f : m_new;
            const float corr = fast_exp2((m_run[q] - m_ref) * c[q]), mc = m_ref * c[q];
            m_run[q] = m_new;
            float p[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) p[r] = fast_exp2(fmaf(s[r], c[q], -mc));
            l_run[q] = l_run[q] * corr + ((p[0] + p[1]) + (p[2] + p[3]));
#pragma unroll
            for (int i = 0; i < NO; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[q][i][r] *= corr;
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int h = 0; h < NH; ++h)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[q][h * 4 + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[r][h][e], p[r], acc[q][h * 4 + e], 0, 0, 0);
        }
    };
    for (int u = wave; u < units; u += 2 * kWavesF) {        // wave-uniform
        if (u + kWavesF < units) load_unit(u + kWavesF, kf[1], vf[1]);
        unit(u, kf[0], vf[0]);
        if (u + kWavesF < units) {
            if (u + 2 * kWavesF < units) load_unit(u + 2 * kWavesF, kf[0], vf[0]);
            unit(u + kWavesF, kf[1], vf[1]);
        }
    }

    // ---- merge the waves' states.  Register r of chunk (h, e) is head dim 64 h + 4 (4 g + r) + e of query row l16: piece
    // (h, r) is four consecutive dims.
#pragma unroll
    for (int q = 0; q < RB; ++q) {
        float l = l_run[q];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        if (g == 0) {
            ml[wave][q][0][l16] = m_run[q] * c[q];           // log2 units (a wave without keys: -inf)
            ml[wave][q][1][l16] = l;
        }
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                states[((wave * RB + q) * NO + h * 4 + r) * 64 + lane] =
                    floatx4{acc[q][h * 4][r], acc[q][h * 4 + 1][r], acc[q][h * 4 + 2][r], acc[q][h * 4 + 3][r]};
    }
    __syncthreads();
    for (int i = tid; i < RB * NO * 64; i += kThreadsF) {
        const int q = i / (NO * 64), piece = (i / 64) % NO, ln = i & 63;
        const int row = (rt * RB + q) * 16 + (ln & 15);
        if (row >= rows_total) continue;
        float m = -INFINITY, l = 0.f;
#pragma unroll
        for (int w = 0; w < kWavesF; ++w) m = fmaxf(m, ml[w][q][0][ln & 15]);
        floatx4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kWavesF; ++w) {
            const float x = fast_exp2(ml[w][q][0][ln & 15] - m);
            const floatx4 s = states[((w * RB + q) * NO + piece) * 64 + ln];
            l += x * ml[w][q][1][ln & 15];
#pragma unroll
            for (int r = 0; r < 4; ++r) o[r] += x * s[r];
        }
        const size_t orow = row_base + row;
        const int dim = (piece / 4) * 64 + (ln >> 4) * 16 + (piece & 3) * 4;
        if (h.splits == 1) {
            const float inv = 1.0f / l;
#pragma unroll
            for (int r = 0; r < 4; ++r) o[r] *= inv;
            *reinterpret_cast<floatx4 *>(static_cast<float *>(a.O) + orow * D + dim) = o;
        } else {
            *reinterpret_cast<floatx4 *>(a.part_o + (orow * h.splits + sp) * D + dim) = o;
            if (dim == 0) {
                a.part_ml[(orow * h.splits + sp) * 2] = m;
                a.part_ml[(orow * h.splits + sp) * 2 + 1] = l;
            }
        }
    }
}

template <int D, int RB>
__global__ __launch_bounds__(kThreadsF) void attn_f32_kernel(DD_ATTN_HEAD, const AttnTail a)
{
    attn_f32<D, RB>(DD_ATTN_HEAD_ARGS, a);
}

// The same launch with the block-completion copy on the workgroups past the attending ones: for a call without key splits, which has no
// merge launch to take it along (a launch of its own for it: 61.8 us per cycle of 4 heads and 128 keys, here 58.5).
template <int D, int RB>
__global__ __launch_bounds__(kThreadsF) void attn_f32_refresh_kernel(DD_ATTN_HEAD, const AttnTail a, const RefreshArgs r)
{
    if ((int)blockIdx.x >= wgs) {            // uniform: these only copy
        refresh_cache_rows<kThreadsF>(r);
        return;
    }
    attn_f32<D, RB>(DD_ATTN_HEAD_ARGS, a);
}

}  // namespace

hipError_t launch_attention_f32(const AttnArgs &a, hipStream_t stream)
{
    AttnKernelArgs k;
    // 32 rows per workgroup (d = 64; at d = 128 they do not fit the registers) halve the K/V reads per row; taken once
    // such workgroups alone fill the chip
    const long heads = (long)a.B * a.Hkv, rows = (long)(a.H / a.Hkv) * a.Nq;
    const bool two = a.d == 64 && heads * ((rows + 31) / 32) >= 512;
    AttnArgs s = a;
    // A workgroup's eight waves split the keys already: splitting them over workgroups as well (a merge launch) is for
    // key ranges that leave every wave several units, and only until there is a workgroup per compute unit.
    const int rows_per_wg = two ? 32 : 16;
    const long wgs = heads * ((rows + rows_per_wg - 1) / rows_per_wg);
    const long most = a.N / kSplitKeys < 256 / wgs ? a.N / kSplitKeys : 256 / wgs;
    if (s.splits > most) s.splits = most > 1 ? (int)most : 1;
    fill_kernel_args(s, k, rows_per_wg, kUnitF);
    k.wgs = (int)(heads * k.row_tiles * k.splits);
    const dim3 block(kThreadsF);
    RefreshArgs r{};
    const long copy_wgs = k.splits == 1 ? fill_refresh(s, r, kCopyWgs) : 0;
    if (copy_wgs > 0) {
        r.first_wg = k.wgs;
        const dim3 grid((unsigned)(k.wgs + copy_wgs));
        return a.d == 128 ? launch_headed(attn_f32_refresh_kernel<128, 1>, grid, block, stream, k, r)
             : two ? launch_headed(attn_f32_refresh_kernel<64, 2>, grid, block, stream, k, r) : launch_headed(attn_f32_refresh_kernel<64, 1>, grid, block, stream, k, r);
    }
    const dim3 grid((unsigned)k.wgs);
    const hipError_t e = a.d == 128 ? launch_headed(attn_f32_kernel<128, 1>, grid, block, stream, k)
                       : two ? launch_headed(attn_f32_kernel<64, 2>, grid, block, stream, k) : launch_headed(attn_f32_kernel<64, 1>, grid, block, stream, k);
    return e != hipSuccess ? e : finish_attention(s, k.splits, stream);
}

}  // namespace dd

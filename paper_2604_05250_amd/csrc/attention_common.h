// Device-side argument block and work decomposition shared by the attention kernels.
//
// Both the verifier's full bidirectional attention (Sec. 2.2) and the drafter's block
// attention over a cached K/V (Sec. 2.3) are softmax(Q K^T / sqrt(d_k)) V (Eq. 3) over
// every key position; they differ only in which query rows exist and where a key row is
// read from.  The kernels therefore work on "virtual rows": for one (batch, kv head) the
// query rows of the `group` query heads that share it, v = (head - kvh*group) * Nq + i.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dd_internal.h"

namespace dd {

// Block-completion refresh of the cache (Sec. 2.3: the cache is brought up to date when a block is done):
// the block's K and V rows, dense in [B*Hkv, block_len, d], replace rows block_start.. of every (batch, kv head)
// of the cache.  Everything in 16-byte chunks; workgroups `first_wg`.. of a launch do the copying: the one that merges
// partial states, or, where the key range is not split, the attention's own (no workgroup of it uses the rows that are written).
struct RefreshArgs {
    const uint4 *src[2];       // Kblk, Vblk
    uint4 *dst[2];             // Kc, Vc at row 0 of (batch 0, kv head 0)
    int per_bh[2];             // chunks of the block per (batch, kv head)
    long bh_stride[2];         // chunks between consecutive (batch, kv head) in the cache
    long offset[2];            // chunks from a cache (batch, kv head) base to row block_start
    int wgs_per_bh;            // copying workgroups per (batch, kv head)
    int first_wg;              // workgroups below this one attend / merge partial states
};

struct AttnKernelArgs {
    const void *Q, *K, *V, *Kblk, *Vblk;
    void *O;                   // final output (splits == 1)
    float *part_o;             // [rows][splits][d] unnormalised partial outputs (splits > 1)
    float *part_ml;            // [rows][splits][2] (running max in log2 units, partial sum)
    const float *q_scale, *k_scale;
    const float *v_scale;      // [B*Hkv] or nullptr: multiplier of the decoded V values (fp8 V)
    const uint8_t *q_mx, *k_mx, *v_mx;   // block-scaled inputs: E8M0 scales [rows][d / 32] of Q, K, V; nullptr otherwise
    int B, H, Hkv, Nq, N;
    int kv_stride;             // rows between consecutive (batch, kv head) in K and V (N unless the call sees a window)
    int group;                 // H / Hkv
    int rows_per_wg;           // query rows per workgroup (a multiple of a wave's rows)
    int row_tiles;             // ceil(group * Nq / rows_per_wg)
    int splits;                // key-range splits
    int keys_per_split;        // multiple of the key tile
    int wgs;                   // attending workgroups of the launch.  (Asking for the grid's size adds 256 bytes of hidden arguments to
                               // every launch, which the host writes, 3.9 us for one where 184 bytes take 3.4, and the kernel fetches.)
    int block_start, block_len;
    const int32_t *block_starts;   // [B] or nullptr: the block's first row per batch entry (overrides block_start)
    float scale_log2;          // log2(e) / sqrt(d)
};

template <int THREADS> __device__ __forceinline__ void refresh_cache_rows(const RefreshArgs &r)
{
    const int cw = (int)blockIdx.x - r.first_wg;
    const int bh = cw / r.wgs_per_bh;
    const int first = (cw - bh * r.wgs_per_bh) * THREADS + (int)threadIdx.x;
    const int step = r.wgs_per_bh * THREADS;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const uint4 *src = r.src[w] + (long)bh * r.per_bh[w];
        uint4 *dst = r.dst[w] + (long)bh * r.bh_stride[w] + r.offset[w];
        for (int in = first; in < r.per_bh[w]; in += step) dst[in] = src[in];
    }
}

// What the kernels of short calls take instead: their first loads need the head only, fourteen words that the hardware has put in
// registers when a wave starts (the build asks for it; it works for leading scalar arguments), and the tail arrives while those
// loads are on their way.  us per call: 1 x 32 heads, 512 keys, 32 rows 6.6 -> 6.2, the verifier's on them 11.5 -> 11.1.
struct AttnHead {
    const uint8_t *Q, *K, *V;
    int rows_total;            // query rows of a (batch, kv head): contiguous in memory
    int N, kv_stride, keys_per_split, wgs, row_tiles, splits, block_start, block_len;
};
struct AttnTail {
    const void *Kblk, *Vblk;
    void *O;
    float *part_o, *part_ml;
    const float *q_scale, *k_scale, *v_scale;
    const int32_t *block_starts;
    int Hkv, Nq, group;
    float scale_log2;
};
#define DD_ATTN_HEAD const uint8_t *Q, const uint8_t *K, const uint8_t *V, int rows_total, int N, int kv_stride, int keys_per_split, int wgs, \
                     unsigned tiles_splits, int block_start, int block_len
#define DD_ATTN_HEAD_ARGS ::dd::AttnHead{Q, K, V, rows_total, N, kv_stride, keys_per_split, wgs, (int)(tiles_splits >> 4), (int)(tiles_splits & 15) + 1, block_start, block_len}
template <typename... Params, typename... Rest>
hipError_t launch_headed(void (*kernel)(Params...), dim3 grid, dim3 block, hipStream_t stream, const AttnKernelArgs &k, Rest... rest)
{
    return launch(kernel, grid, block, stream, static_cast<const uint8_t *>(k.Q), static_cast<const uint8_t *>(k.K), static_cast<const uint8_t *>(k.V),
                  k.group * k.Nq, k.N, k.kv_stride, k.keys_per_split, k.wgs, (unsigned)k.row_tiles << 4 | (unsigned)(k.splits - 1),   // (at most 16 splits)
                  k.block_start, k.block_len,
                  AttnTail{k.Kblk, k.Vblk, k.O, k.part_o, k.part_ml, k.q_scale, k.k_scale, k.v_scale, k.block_starts, k.Hkv, k.Nq, k.group,
                           k.scale_log2}, rest...);
}
// This workgroup's place, from its number: of `row_tiles` and `splits` (a division is some 150 cycles before the first load).
__device__ __forceinline__ void place_of(unsigned &bid, int count, int &at)
{
    at = 0;
    if (count > 1) { at = bid % (unsigned)count; bid /= (unsigned)count; }
}
// A value at a uniform address that no workgroup writes, by a scalar load.  (After a statement that may write memory the compiler takes a
// vector load instead, and waits for every load before it.)
template <typename T> __device__ __forceinline__ T uniform_load(const T *p)
{
    return *(__attribute__((address_space(4))) const T *)(unsigned long long)p;
}

constexpr int kAttnThreads = 256;

struct AttnArgs;
// Host side: derive the launch decomposition (row tiles, key splits, partial buffers).
void fill_kernel_args(const AttnArgs &a, AttnKernelArgs &k, int rows_per_wg, int key_tile);
// Host side: where the block-completion copy of a call goes from and to, by at most about `most_wgs` workgroups; returns how many (0:
// nothing to copy).
long fill_refresh(const AttnArgs &a, RefreshArgs &r, long most_wgs);
// An attending workgroup's LDS is set aside for a copying one of its launch too: about one of these per compute unit.
constexpr long kCopyWgs = 256;

}  // namespace dd

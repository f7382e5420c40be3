// Tier-2 ring append (Sec. 2.5: the window keeps the W most recent tokens so
// the cache stays bounded by K + W + |q| while generating), and the Tier-1
// gather that copies the selected memory rows' K/V into a contiguous block
// once per question.
//
// Appended row t of kv head h goes to slot (count + t) mod W, then count +=
// T_new.  A few rows (a decode step) are moved by one workgroup per sequence,
// which also owns count[b]; a prefill's rows are spread over the whole chip
// and count is advanced by a second launch, after every workgroup of the
// first has read it (no counters: the caller gives no workspace).  Rows move
// as 16-byte vectors.
#include <algorithm>

#include "device_common.hpp"
#include "kernels.hpp"

namespace cmc {

namespace {

// Slot of appended row t: T_new <= W, so it wraps at most once.
__device__ __forceinline__ int append_slot(int slot0, int t, int W) {
    const int room = W - slot0;
    return t < room ? slot0 + t : t - room;
}

// One workgroup per sequence.  Bound by latency up to one trip of its loop,
// then by what one CU can move; a trip requests kAppendVecs vectors of K and
// of V per thread before it stores the first.  One row of 8 heads for 64
// sequences: 8.0 us with ordinary stores, 2.7 us with non-temporal ones.
constexpr int kAppendVecs = 4;
template <int NT>
__global__ __launch_bounds__(NT) void window_append_kernel(AppendParams p, unsigned row_shift) {
    const int b = blockIdx.x;
    const int count = p.win_count[b] < 0 ? 0 : p.win_count[b];  // count >= 0 is a precondition
    const int slot0 = count % p.W;
    const unsigned total = ((unsigned)p.Hkv * (unsigned)p.T_new) << row_shift;  // small: see kAppendOneWg
    const size_t src0 = (size_t)b * total, dst0 = ((size_t)b * p.Hkv * p.W) << row_shift;
    const uint4 *nk = static_cast<const uint4 *>(p.new_k) + src0;
    const uint4 *nv = static_cast<const uint4 *>(p.new_v) + src0;
    uint4 *wk = static_cast<uint4 *>(p.win_k) + dst0;
    uint4 *wv = static_cast<uint4 *>(p.win_v) + dst0;
    for (unsigned i0 = threadIdx.x; i0 < total; i0 += NT * kAppendVecs) {
        uint4 k[kAppendVecs], v[kAppendVecs];
#pragma unroll
        for (int u = 0; u < kAppendVecs; ++u) {
            const unsigned i = min(i0 + u * NT, total - 1);  // past the end: loaded, not stored
            k[u] = nk[i];
            v[u] = nv[i];
        }
#pragma unroll
        for (int u = 0; u < kAppendVecs; ++u) {
            const unsigned i = i0 + u * NT;
            if (i < total) {
                const unsigned r = i >> row_shift, h = r / (unsigned)p.T_new, t = r % (unsigned)p.T_new;
                const size_t row = (size_t)h * p.W + append_slot(slot0, (int)t, p.W);
                const size_t dst = (row << row_shift) + (i & ((1u << row_shift) - 1));
                st16_nt(&wk[dst], k[u]);
                st16_nt(&wv[dst], v[u]);
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) p.win_count[b] = count + p.T_new;
}

// The same copy by the whole chip.  Bound by memory: every byte is read once
// and written once.  A workgroup moves a run of kAppendVecs * 256 vectors of
// one (sequence, kv head), each thread's K and V loads requested before its
// first store; the rows' places come from 32-bit arithmetic and one ring
// wrap.  8 sequences x 8 heads x 1024 rows of 256 bytes (67 MB moved): 362 us
// by one workgroup per sequence with ordinary stores, 10.2 us here (6.6 TB/s,
// served partly by the last-level cache); 64 sequences (537 MB): 543 -> 77 us
// (7.0 TB/s).  With ordinary stores this kernel took 23 and 116 us (see
// st16_nt).
__global__ __launch_bounds__(256) void window_copy_kernel(AppendParams p, unsigned row_shift, size_t groups,
                                                          size_t head_vecs) {
    const int b = blockIdx.y;
    const int count = p.win_count[b] < 0 ? 0 : p.win_count[b];
    const int slot0 = count % p.W;
    // One (kv head, run of vectors) per trip: one trip, unless there are more
    // of them than workgroups (see launch_window_append).
    for (size_t w = blockIdx.x; w < groups * p.Hkv; w += gridDim.x) {  // uniform
        const size_t head = (size_t)b * p.Hkv + w / groups;
        const uint4 *nk = static_cast<const uint4 *>(p.new_k) + head * head_vecs;
        const uint4 *nv = static_cast<const uint4 *>(p.new_v) + head * head_vecs;
        uint4 *wk = static_cast<uint4 *>(p.win_k) + ((head * p.W) << row_shift);
        uint4 *wv = static_cast<uint4 *>(p.win_v) + ((head * p.W) << row_shift);
        const size_t first = (w % groups) * (256 * kAppendVecs) + threadIdx.x;
        uint4 k[kAppendVecs], v[kAppendVecs];
#pragma unroll
        for (int u = 0; u < kAppendVecs; ++u) {
            const size_t i = min(first + 256 * u, head_vecs - 1);  // past the end: loaded, not stored
            k[u] = nk[i];
            v[u] = nv[i];
        }
#pragma unroll
        for (int u = 0; u < kAppendVecs; ++u) {
            const size_t i = first + 256 * u;
            if (i < head_vecs) {
                const int slot = append_slot(slot0, (int)(i >> row_shift), p.W);
                const size_t dst = ((size_t)slot << row_shift) + (i & ((1u << row_shift) - 1));
                st16_nt(&wk[dst], k[u]);
                st16_nt(&wv[dst], v[u]);
            }
        }
    }
}

__global__ __launch_bounds__(256) void window_count_kernel(int32_t *win_count, int B, int T_new) {
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b < B) win_count[b] = (win_count[b] < 0 ? 0 : win_count[b]) + T_new;
}

// Tier-1 gather: out[b][h][j] = pool[b][h][idx[b][j]] (clamped into the
// pool) for j < k_b, 16-byte vectors, one thread per vector: consecutive
// threads copy consecutive vectors of a row, so every row moves as whole
// 64-byte segments.  Rows j >= k_b are left untouched.  Bound by memory (read
// once, written once); with the stores non-temporal the selection and gather of
// 64 sequences take 168.4 us instead of 175.6 (225 MB gathered).
__global__ __launch_bounds__(256) void gather_kernel(GatherParams p) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t per_seq = (size_t)p.Hkv * p.k * p.row_vecs;
    const int b = (int)(i / per_seq);
    if (b >= p.B) return;
    const size_t r = i % per_seq;
    const int v = (int)(r % p.row_vecs);
    const int j = (int)((r / p.row_vecs) % p.k);
    const int h = (int)(r / ((size_t)p.row_vecs * p.k));
    int kb = p.k;
    if (p.k_len) {
        const int x = p.k_len[b];
        kb = x < 0 ? 0 : (x > p.k ? p.k : x);
    }
    if (j >= kb) return;
    int src = p.idx ? p.idx[(size_t)b * p.idx_stride + j] : j;
    src = src < 0 ? 0 : (src > p.N - 1 ? p.N - 1 : src);
    const size_t head = (size_t)b * p.Hkv + h;
    const size_t s_off = (head * p.N + src) * p.row_vecs + v;
    const size_t d_off = (head * p.k + j) * p.row_vecs + v;
    st16_nt(static_cast<uint4 *>(p.out_k) + d_off, static_cast<const uint4 *>(p.cme_k)[s_off]);
    st16_nt(static_cast<uint4 *>(p.out_v) + d_off, static_cast<const uint4 *>(p.cme_v)[s_off]);
}

}  // namespace

hipError_t launch_gather(const GatherParams &p, hipStream_t stream) {
    const size_t total = (size_t)p.B * p.Hkv * p.k * p.row_vecs;
    if (total == 0) return hipSuccess;
    gather_kernel<<<(unsigned)((total + 255) / 256), 256, 0, stream>>>(p);
    return hipGetLastError();
}

// Most 16-byte vectors (of K, and as many of V) per sequence that one
// workgroup moves.  Kernel times, one workgroup per sequence / whole chip and
// count (two launches, which cost the host 2.6 us more): 4096 vectors 3.5 /
// 4.4 us (1 sequence), 5.0 / 5.4 us (64); 8192 vectors 5.6 / 4.7 us (1), 6.9
// / 6.8 us (64); 16384 vectors 9.7 / 4.7 us (1); 131072 vectors 79 / 11.5 us
// (8), 101 / 82 us (64).
#ifndef CMC_APPEND_ONE_WG
#define CMC_APPEND_ONE_WG 8192
#endif
constexpr size_t kAppendOneWg = CMC_APPEND_ONE_WG;

hipError_t launch_window_append(const AppendParams &p, hipStream_t stream) {
    if (p.B == 0 || p.W == 0) return hipSuccess;
    const size_t head_vecs = (size_t)p.T_new * p.row_vecs;
    const unsigned row_shift = (unsigned)__builtin_ctz((unsigned)p.row_vecs);  // Dh and the element size are powers of two
    if (head_vecs * p.Hkv <= kAppendOneWg) {
        if (head_vecs * p.Hkv <= 256 * kAppendVecs) window_append_kernel<256><<<p.B, 256, 0, stream>>>(p, row_shift);
        else window_append_kernel<1024><<<p.B, 1024, 0, stream>>>(p, row_shift);
        return hipGetLastError();
    }
    const size_t groups = (head_vecs + 256 * kAppendVecs - 1) / (256 * kAppendVecs);
    const unsigned grid = (unsigned)std::min(groups * p.Hkv, (size_t)1 << 20);
    window_copy_kernel<<<dim3(grid, p.B), 256, 0, stream>>>(p, row_shift, groups, head_vecs);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    window_count_kernel<<<(p.B + 255) / 256, 256, 0, stream>>>(p.win_count, p.B, p.T_new);
    return hipGetLastError();
}

}  // namespace cmc

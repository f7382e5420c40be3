// Two-tier decode attention (Sec. 2.5, KV cache assembly): one decode step of
// softmax attention over the key list [Tier-1 pool rows idx[0..k-1]] ++
// [Tier-2 ring slots 0..min(count,W)-1], optionally fused with the ring append
// of this step's new rows, in ONE launch.
//
// Grid (S, Hkv, B), 4 or 8 waves per workgroup (chosen by the split plan).  Workgroup s owns keys
// [s*chunk, (s+1)*chunk) of sequence b's virtual key list and all G = Hq/Hkv
// query heads sharing kv head h, so each K/V byte is read from HBM once per
// step and reused G times on chip.
//
// Fused append: with T_new > 0, the rows appended this step go to slots
// (count + t) mod W.  The workgroup owning such a slot reads the row from
// new_k/new_v instead of the ring and writes it into the ring; count is
// advanced once every (sequence, kv head) pair has been completed, i.e.
// after every workgroup of the sequence has read it.  The result equals
// cmc_window_append followed by the decode.
//
// Main loop: a wave takes 16 keys per block.  S = Q K^T on MFMA, the 16
// A-rows holding the G query heads repeated (row m = head m % G), so every lane
// ends with the scores of key (lane % 16) for all heads (G <= 4) or for four
// of the eight (G = 8: heads 4 ((lane / 16) % 2) .. + 3).
//   bf16 K/V: one v_mfma_f32_16x16x32_bf16 chain per Dh/32 slice, q split into
//     bf16 parts (hi + lo, two MFMAs per slice, for G <= 4; three parts, the
//     whole fp32 significand, for G = 8), which keeps the logit error at the
//     level of fp32 accumulation.
//   fp32 K/V: v_mfma_f32_16x16x4_f32, or the VALU where the heads are few (see
//     QOperand<float>), fp32 products and sums throughout.
// P V runs on the VALU in fp32 in four quarters of 4 keys: lane l owns key
// (l & 3) of each quarter and Dh/16 dims; the p values reach that layout
// through 16 x G floats of LDS private to the wave.  V rows are loaded
// non-temporally, K rows with ordinary loads (see ld16).  Each wave keeps an
// online softmax (running max in log2 units, q pre-scaled by scale*log2 e),
// then the waves are combined through LDS.
// Measured, with this loop in place of one that loaded 4 - 16 rows at a time
// and reduced their dot products across lanes, waiting for each load: 24
// ragged sequences of 64/8 heads (bf16, Dh = 128, G = 8) 155 -> 36 us; fp32, 30
// sequences of 32/8 heads, Dh = 128, 1000 keys 74.6 -> 48.8 us.
//
// Latency (one launch of a single layer at batch 1 is a chain of memory round
// trips, not a stream): the first K/V loads depend only on kernel arguments
// that arrive preloaded in SGPRs.  The ring count is fetched with a vector
// load and read where the masks need it, q is loaded and split after the
// first K/V loads are issued, and where the key list is split often enough
// the rows appended in this call get a split of their own, so no workgroup runs
// two dependent phases (see plan_decode).  Measured, the step is bound by that chain and by memory:
// with P V taken out entirely a step got only 2-3% faster.
//
// Split merge, inside the same launch: with S == 1 the workgroup writes the
// output directly.  With S > 1 every workgroup publishes (m, l, acc[Dh]) per
// head to the workspace and arrives on a per-(b, kv head) counter; the last
// to arrive merges the S partials in fixed split order (so results are
// bit-identical run to run), writes the output and re-arms the counter.
// Publication uses agent-coherent relaxed atomics plus a store-completion
// wait instead of device-scope fences (see coherent_store2).  A head whose key
// list is empty gets zeros.
#include <float.h>
#include <limits.h>

#include <type_traits>

#include "device_common.hpp"
#include "kernels.hpp"

namespace cmc {

namespace {

// Build-time tuning knob: widest K/V row, in bytes, that is double-buffered
// (wider rows' second register set would cost a wave per SIMD).
#ifndef CMC_DOUBLE_BUFFER_MAX_ROW
#define CMC_DOUBLE_BUFFER_MAX_ROW 256
#endif

constexpr float kLog2e = 1.4426950408889634f;

// A running max before any key.  Finite, so that a key whose score is -inf
// weighs exp2(-inf) = 0 also where no other key came before it (from -inf
// the difference would be NaN, and with it the whole head).
constexpr float kNoMax = -FLT_MAX;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// Orders this wave's LDS writes before its following LDS reads (and reads
// before later writes).  LDS operations of one wave execute in order, so only
// the compiler must be kept from moving memory accesses across this point; a
// fence would also wait for every outstanding global load, including the
// next block's prefetch.
__device__ __forceinline__ void wave_lds_sync() { asm volatile("" ::: "memory"); }

// 2^x with the hardware instruction alone: results below 2^-126 are 0 (see
// kSmallWeights; the waves' and splits' weights at the merge always take it).
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// d[e] += q[e] of lane I .. I + 3 of this lane's 16-lane row times element e of
// k0 .. k3, in that order, each a multiply-add with a DPP row broadcast (the
// compiler makes a move and a multiply-add of it).  The s_nop covers the two
// wait states between a VALU write of q and its DPP read, which the compiler
// cannot see in here.  (The five after a VALU write of EXEC are not needed:
// EXEC is written by the scalar unit alone.)  All lanes must be active.
template <int I>
__device__ __forceinline__ void row_fma(float (&d)[4], const float4 &q, const uint4 &k0, const uint4 &k1, const uint4 &k2,
                                        const uint4 &k3) {
    asm("s_nop 1\n"
        "v_fmac_f32_dpp %[d0], %[q0], %[a0] row_newbcast:%[i0] row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %[d1], %[q1], %[a1] row_newbcast:%[i0] row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %[d2], %[q2], %[a2] row_newbcast:%[i0] row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %[d3], %[q3], %[a3] row_newbcast:%[i0] row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %[d0], %[q0], %[b0] row_newbcast:%[i1] row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %[d1], %[q1], %[b1] row_newbcast:%[i1] row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %[d2], %[q2], %[b2] row_newbcast:%[i1] row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %[d3], %[q3], %[b3] row_newbcast:%[i1] row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %[d0], %[q0], %[c0] row_newbcast:%[i2] row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %[d1], %[q1], %[c1] row_newbcast:%[i2] row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %[d2], %[q2], %[c2] row_newbcast:%[i2] row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %[d3], %[q3], %[c3] row_newbcast:%[i2] row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %[d0], %[q0], %[e0] row_newbcast:%[i3] row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %[d1], %[q1], %[e1] row_newbcast:%[i3] row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %[d2], %[q2], %[e2] row_newbcast:%[i3] row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %[d3], %[q3], %[e3] row_newbcast:%[i3] row_mask:0xf bank_mask:0xf"
        : [d0] "+&v"(d[0]), [d1] "+&v"(d[1]), [d2] "+&v"(d[2]), [d3] "+&v"(d[3])
        : [q0] "v"(q.x), [q1] "v"(q.y), [q2] "v"(q.z), [q3] "v"(q.w), [a0] "v"(k0.x), [a1] "v"(k0.y), [a2] "v"(k0.z),
          [a3] "v"(k0.w), [b0] "v"(k1.x), [b1] "v"(k1.y), [b2] "v"(k1.z), [b3] "v"(k1.w), [c0] "v"(k2.x), [c1] "v"(k2.y),
          [c2] "v"(k2.z), [c3] "v"(k2.w), [e0] "v"(k3.x), [e1] "v"(k3.y), [e2] "v"(k3.z), [e3] "v"(k3.w), [i0] "n"(I),
          [i1] "n"(I + 1), [i2] "n"(I + 2), [i3] "n"(I + 3));
}

// Whether softmax weights below 2^-126 are kept (as the library's exp2f gives
// them; times a large value they count) instead of taken as 0.  A lane that
// holds one takes a branch.  24 ragged sequences of 64/8 heads 35.1 -> 35.8
// us; an fp32 step is as before.
template <typename T, int G>
constexpr bool kSmallWeights = sizeof(T) == 4 || G > 4;

// 16-byte load; NT marks it non-temporal.  The MFMA path loads its V rows
// that way and its K rows with ordinary loads.  Launch times, with the
// Mistral-shaped batch rotated over 8 copies so that nothing is reused from
// the last-level cache (ordinary / V non-temporal / K and V / K only):
// 74.7 / 66.1 / 66.7 / 70.1 us; the 32-layer stack 38.4 / 36.3 / 36.3 /
// 36.7 us; the Dh = 256 layer 136.5 / 128.4 / 139.6 / 127.8 us.
template <bool NT = false>
__device__ __forceinline__ uint4 ld16(const void *p) {
    if constexpr (NT) {
        const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
        return make_uint4(v.x, v.y, v.z, v.w);
    } else {
        return *reinterpret_cast<const uint4 *>(p);
    }
}
__device__ __forceinline__ void st16(void *p, const uint4 &v) { *reinterpret_cast<uint4 *>(p) = v; }

// Query heads whose scores one lane holds (C rows per lane of the MFMA tile).
template <int G>
constexpr int kLaneHeads = G < 4 ? G : 4;

// Per-wave online-softmax state for G heads and VEC output dims per lane.
// Every lane holds all G running maxima; the denominators are those of the
// lane's own heads (all of them for G <= 4).
template <int G, int VEC>
struct WaveState {
    float m[G], l[kLaneHeads<G>], acc[G][VEC];
    __device__ __forceinline__ void init() {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            m[g] = kNoMax;
            if (g < kLaneHeads<G>) l[g] = 0.f;
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[g][i] = 0.f;
        }
    }
};

// The ring count, fetched by a wave with a vector load issued after its
// first K/V loads (nothing waits for it before they are in flight) and read
// where a mask or a ring slot needs it, and at the end of the walk (stored
// into LDS before the arrival).
struct RingCount {
    int raw;
    bool loaded;  // wave-uniform
    __device__ __forceinline__ void load(const int32_t *win_count, int b) {
        if (!loaded) {
            raw = win_count ? __hip_atomic_load(win_count + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
            loaded = true;
        }
    }
    __device__ __forceinline__ int value() const {  // clamped at 0, wave-uniform
        const int c = __builtin_amdgcn_readfirstlane(raw);
        return c < 0 ? 0 : c;
    }
};

// One arrival on a counter (relaxed, agent scope) that returns the previous
// value.  The address goes through a VGPR so that the compiler keeps it a
// single returning atomic: its atomic optimizer would otherwise turn it into
// a wave-wide scan that reads the result at once, and since loads and atomics
// complete in order, that wait would also cover every load issued before.
// As it is, the result is waited for only where it is used.
__device__ __forceinline__ unsigned arrive_once(unsigned *ctrs, int i, unsigned one) {
    int iv;
    asm volatile("v_mov_b32 %0, %1" : "=v"(iv) : "s"(i));
    return __hip_atomic_fetch_add(ctrs + iv, one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// --------------------------------------------------------------- MFMA loop
//
// The key list is walked in three phases, each a contiguous run of rows
// addressed from one uniform base with 32-bit offsets:
//   pool  rows [0, kb):          pool row idx[row] (clamped into the pool);
//   ring  rows [kb, kb + W):     ring slot row - kb, masked unless it holds a
//                                token that survives this call's append
//                                (slot < min(count, W), not one of the slots
//                                (count + t) mod W, t < T_new);
//   new   rows [kb + W, L):      the T_new rows appended in this call, read
//                                from new_k/new_v and written to ring slots
//                                (count + t) mod W.
// That is the same key set as [pool rows] ++ [ring slots after the append];
// softmax attention does not depend on key order.  No address and no phase
// boundary depends on the ring count, so the first K/V loads are issued
// without waiting for it; the count only enters the masks and the slots the
// new rows are written to.  (A masked slot that is being overwritten in the
// same launch may be read before or after the write: its value is unused.)

// IX: rows through the index list (else the pool is the gathered block and
// row r is pool row r; the list pointer is then never read).
template <bool IX>
struct PoolRows {
    const int32_t *idx;  // index list base (IX)
    size_t off;          // this sequence's first entry
    int nmax;
    static constexpr bool kMasked = false;
    __device__ __forceinline__ int key(int row) const {
        if constexpr (IX) return idx[off + row];
        else return row;
    }
    __device__ __forceinline__ int slot(int, int key) const { return key < 0 ? 0 : (key > nmax ? nmax : key); }
    __device__ __forceinline__ bool valid(int) const { return true; }
    __device__ __forceinline__ bool all_valid(int, int) const { return true; }
    __device__ __forceinline__ void resolve(const RingCount &) {}
    __device__ __forceinline__ int limit(int r1) const { return r1; }
};
// The ring in physical slot order: row `first` is slot 0.  Addresses do not
// depend on the count; a slot holds a key of this step when it is filled
// (slot < min(count, W)) and not overwritten by this step's append (slots
// (count + t) mod W, t < T_new) -- a mask applied at compute time.
struct RingRows {
    int first, T_new, W;
    int nvalid = 0, cnt_mod = 0;  // set by resolve(), before the first mask
    static constexpr bool kMasked = true;
    __device__ __forceinline__ void resolve(const RingCount &cnt) {
        const int c = cnt.value();
        nvalid = min(c, W);
        cnt_mod = c % W;
    }
    // Slots past the filled ones hold no key: once the count is known the
    // phase ends there (a ring that has not wrapped yet is not read whole).
    __device__ __forceinline__ int limit(int r1) const { return min(r1, first + nvalid); }
    __device__ __forceinline__ int key(int row) const { return row; }
    __device__ __forceinline__ int slot(int row, int) const { return row - first; }
    __device__ __forceinline__ bool valid(int row) const {
        const int s = row - first;
        int d = s - cnt_mod;
        d += d < 0 ? W : 0;
        return s < nvalid && d >= T_new;
    }
    // Whether every row of [r0, r1) is valid (wave-uniform; in steady state
    // only the T_new slots being overwritten are masked).
    __device__ __forceinline__ bool all_valid(int r0, int r1) const {
        const int s0 = r0 - first, s1 = r1 - first;
        if (s1 > nvalid) return false;
        // the overwritten slots are [cnt_mod, cnt_mod + T_new) mod W
        const int e = cnt_mod + T_new;
        return !(s0 < e && s1 > cnt_mod) && s0 >= e - W;
    }
};
struct NewRows {
    int first, W;  // row `first` is appended row 0, bound for ring slot count mod W
    int slot0 = 0;  // set by resolve()
    static constexpr bool kMasked = false;
    __device__ __forceinline__ void resolve(const RingCount &cnt) { slot0 = cnt.value() % W; }
    __device__ __forceinline__ int limit(int r1) const { return r1; }
    __device__ __forceinline__ int key(int row) const { return row; }
    __device__ __forceinline__ int slot(int row, int) const { return row - first; }
    __device__ __forceinline__ bool valid(int) const { return true; }
    __device__ __forceinline__ bool all_valid(int, int) const { return true; }
    __device__ __forceinline__ int ring_slot(int row) const {
        const int sl = slot0 + (row - first);
        return sl >= W ? sl - W : sl;
    }
};

// q's A operand (this lane's dims of query head (lane % 16) % G, pre-scaled),
// filled by the first phase that has a block for the wave, after that
// block's K/V loads are issued (both round trips overlap), and the scores of
// a 16-key block from it.  The lane's K elements of key lane % 16 are the
// 16-byte chunks 4 i + lane / 16 of the row; the dims of a chunk are the k
// indices of one MFMA (bf16) or of four (fp32), in the same order for q.
//
// Eight heads of bf16 (three parts, beside 8 DH/16 accumulators per lane)
// keep the operand in LDS of the wave's own instead, where its registers would
// cost the second wave per SIMD, and read it back for every block: 16 bytes per
// lane and MFMA, one copy per head.
template <typename T, int DH, int G>
struct QOperand;

template <int DH, int G>
struct QOperand<uint16_t, DH, G> {
    static constexpr int kChunks = DH / 32;
    static constexpr bool kLds = G > 4;
    // bf16 parts of q: hi + lo carry 16 bits of its significand; the third
    // completes fp32's 24.  (Two parts: output error 2.6e-6 against 64 bits;
    // three: 2e-7, what an fp32 dot product gives.)
    static constexpr int kParts = G > 4 ? 3 : 2;
    static constexpr int kLdsWords = kLds ? kChunks * kParts * 4 * G : 1;  // 16-byte words per wave
    bf16x8 part[kLds ? 1 : kParts][kLds ? 1 : kChunks];
    uint4 *lds;
    bool ready;
    __device__ __forceinline__ void load(const DecodeParams &p, int b, int kvh) {
        const int lane = threadIdx.x & 63;
        const int r16 = lane & 15, q4 = lane >> 4;
        const float *qp = p.q + ((size_t)b * p.Hq + (size_t)kvh * G + (r16 % G)) * DH + 8 * q4;
#pragma unroll
        for (int i = 0; i < kChunks; ++i) {
            const float4 x0 = *reinterpret_cast<const float4 *>(qp + 32 * i);
            const float4 x1 = *reinterpret_cast<const float4 *>(qp + 32 * i + 4);
            const float xs[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
            bf16x8 h[kParts];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float v = xs[e] * p.qscale;
#pragma unroll
                for (int t = 0; t < kParts; ++t) {
                    h[t][e] = (__bf16)v;
                    v -= (float)h[t][e];  // exact
                }
            }
#pragma unroll
            for (int t = 0; t < kParts; ++t) {
                if constexpr (kLds) {
                    if (r16 < G) lds[((i * kParts + t) * 4 + q4) * G + r16] = __builtin_bit_cast(uint4, h[t]);
                } else {
                    part[t][i] = h[t];
                }
            }
        }
        if constexpr (kLds) wave_lds_sync();
    }
    __device__ __forceinline__ floatx4 scores(const uint4 (&kr)[kChunks]) const {
        // Three parts: the small ones summed apart, the large ones in runs of
        // two slices, so that no partial sum is rounded often.
        floatx4 c = {0.f, 0.f, 0.f, 0.f}, rest = c, sum = c;
#pragma unroll
        for (int i = 0; i < kChunks; ++i) {
            const bf16x8 kbf = __builtin_bit_cast(bf16x8, kr[i]);
#pragma unroll
            for (int t = 0; t < kParts; ++t) {
                bf16x8 a;
                if constexpr (kLds) {
                    const int lane = threadIdx.x & 63;
                    a = __builtin_bit_cast(bf16x8, lds[((i * kParts + t) * 4 + lane / 16) * G + lane % G]);
                } else {
                    a = part[t][i];
                }
                if constexpr (kParts > 2) {
                    if (t > 0) rest = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, kbf, rest, 0, 0, 0);
                    else c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, kbf, c, 0, 0, 0);
                } else {
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, kbf, c, 0, 0, 0);
                }
            }
            if constexpr (kParts > 2) {
                if (i % 2 == 1) {
                    sum = sum + c;
                    c = floatx4{0.f, 0.f, 0.f, 0.f};
                }
            }
        }
        if constexpr (kParts > 2) {
            // An infinite key element: the large parts have q's signs and give
            // the score; the small ones may differ in sign, so their sum is
            // held finite (also where it is NaN).
#pragma unroll
            for (int e = 0; e < 4; ++e) c[e] = sum[e] + __builtin_amdgcn_fmed3f(rest[e], -FLT_MAX, FLT_MAX);
        }
        return c;
    }
};

template <int DH, int G>
struct QOperand<float, DH, G> {
    static constexpr int kChunks = DH / 16;
    // Few heads, and rows of 256: the dot products on the VALU.  An fp32 MFMA
    // step takes 32 cycles however few of its 16 rows are distinct heads: DH/4
    // of them per block against G (DH/4 + 6) VALU instructions of 4 cycles.
    // One or two heads keep the lane's chunks of q in registers.  Two to eight
    // of 256 keep chunk i of every head in lane i of each 16-lane row, and the
    // multiply takes it from there (a DPP row broadcast): G registers of four
    // floats instead of LDS reads, whose 16 G per block and wave took as long
    // as the products.  Four heads of 256, MFMA in one run of 16 chunks / q
    // read from LDS / so: 24 pairs of 768 keys 22.4 / 22.5 / 19.4 us, 136 of
    // 120 keys 23.1 / 27.0 / 20.6, 184 of 3072 keys 244 / 248 / 202; output
    // error against 64 bits 2.3e-7 / 1.7e-7 / 1.7e-7 (13 registers spill so, 48
    // did with shorter MFMA runs).  Eight heads, MFMA / so: 104 pairs of 3072
    // keys 159 / 137, 264 pairs of 120 keys 59 / 54.  Two heads, q from LDS /
    // so: 24 pairs of 768 keys 18.0 / 15.7.
    static constexpr bool kRow = DH == 256 && G >= 2;
    static constexpr bool kDot = kRow || (G * DH <= 256 && G <= 2);
    static constexpr int kLdsWords = 1;  // none needed
    float4 x[kRow ? G : kDot ? G * kChunks : kChunks];
    uint4 *lds;
    bool ready;
    __device__ __forceinline__ void load(const DecodeParams &p, int b, int kvh) {
        const int lane = threadIdx.x & 63;
        const int r16 = lane & 15, q4 = lane >> 4;
        const float *q0 = p.q + ((size_t)b * p.Hq + (size_t)kvh * G) * DH + 4 * q4;
        constexpr int kRows = kDot ? G : 1;
        constexpr int kLoads = kRow ? 1 : kChunks;
#pragma unroll
        for (int g = 0; g < kRows; ++g) {
            const float *qp = q0 + (kDot ? g : r16 % G) * DH + (kRow ? 16 * r16 : 0);
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                const float4 t = *reinterpret_cast<const float4 *>(qp + 16 * i);
                const float4 u = make_float4(t.x * p.qscale, t.y * p.qscale, t.z * p.qscale, t.w * p.qscale);
                x[g * kLoads + i] = u;
            }
        }
    }
    __device__ __forceinline__ floatx4 scores(const uint4 (&kr)[kChunks]) const {
        floatx4 c = {0.f, 0.f, 0.f, 0.f}, c1 = c, c2 = c, c3 = c, sum = c;
        if constexpr (kDot) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float d[4] = {0.f, 0.f, 0.f, 0.f};  // short chains: less rounding, more in flight
                if constexpr (kRow) {
                    static_assert(!kRow || kChunks == 16, "a chunk per lane of a row");
                    row_fma<0>(d, x[g], kr[0], kr[1], kr[2], kr[3]);
                    row_fma<4>(d, x[g], kr[4], kr[5], kr[6], kr[7]);
                    row_fma<8>(d, x[g], kr[8], kr[9], kr[10], kr[11]);
                    row_fma<12>(d, x[g], kr[12], kr[13], kr[14], kr[15]);
                } else {
#pragma unroll
                    for (int i = 0; i < kChunks; ++i) {
                        const float4 a = x[g * kChunks + i];
                        d[0] = fmaf(a.x, __uint_as_float(kr[i].x), d[0]);
                        d[1] = fmaf(a.y, __uint_as_float(kr[i].y), d[1]);
                        d[2] = fmaf(a.z, __uint_as_float(kr[i].z), d[2]);
                        d[3] = fmaf(a.w, __uint_as_float(kr[i].w), d[3]);
                    }
                }
                const float t = lane_reduce<OpSum, 16, kWave>((d[0] + d[1]) + (d[2] + d[3]));
                if constexpr (G > 4) {  // the odd lane rows hold heads 4 .. 7
                    const bool mine = (g >= 4) == (((threadIdx.x & 63) / 16) % 2 != 0);
                    c[g % 4] = mine ? t : c[g % 4];
                } else {
                    c[g] = t;
                }
            }
            return c;
        }
#pragma unroll
        for (int i = 0; i < kChunks; ++i) {
            const float4 a = x[kDot ? 0 : i];
            c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, __uint_as_float(kr[i].x), c, 0, 0, 0);
            c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, __uint_as_float(kr[i].y), c1, 0, 0, 0);
            c2 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, __uint_as_float(kr[i].z), c2, 0, 0, 0);
            c3 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, __uint_as_float(kr[i].w), c3, 0, 0, 0);
            // Short runs, so that no partial sum is rounded often.  Output
            // error against 64 bits (140 pairs, 300 keys) with runs of four
            // chunks / two: Dh = 64, G = 4 1.66e-7 / 1.61e-7, G = 8 1.67e-7 /
            // 1.60e-7; Dh = 128, G = 8 1.72e-7 / 1.66e-7, at the same times
            // (the lane sums that this walk replaced: 1.52e-7, 1.52e-7,
            // 1.63e-7).
            constexpr int kRun = 2;
            if (i % kRun == kRun - 1) {
                sum = sum + ((c + c1) + (c2 + c3));
                c = c1 = c2 = c3 = floatx4{0.f, 0.f, 0.f, 0.f};
            }
        }
        return sum;
    }
};

// Byte offsets from a (sequence, kv head)'s pool or ring base: 32 bits for
// bf16 (the host checks that they suffice), 64 for fp32.
template <typename T>
using row_off_t = std::conditional_t<sizeof(T) == 2, uint32_t, size_t>;

// One phase: rows [r0, r1) from bases kbase/vbase (bytes).  A wave takes 16
// rows per block.  K: the lane's row blk + (lane % 16) in the MFMA B layout
// (its 16-byte chunks 4i + lane/16).  V: four quarters of 4 rows; in quarter qq
// the lane owns row blk + 4qq + (lane % 4) and DH/16 dims of it, the 16-byte
// words lane/4, lane/4 + 16, ... of the row, so that every load takes whole
// 256-byte runs of four rows (DH/16 consecutive dims, two to four words at a
// 32- or 64-byte stride, had each load touch every line of the rows and the
// non-temporal lines fetched again: bf16 Dh = 256 step 133.0 -> 127.2 us, fp32
// Dh = 256 of 400 pairs 157 -> 110 us), and accumulates those output dims per
// head.  The p values travel from the score layout (lane r holds key r's G weights) to
// the V layout through a 16 x G slot of LDS private to the wave.  Keys
// (index-list entries) are fetched one block ahead of the K/V rows, and the
// K/V rows one block ahead of their use.
template <int NW, typename T, int DH, int G, class Rows, bool RING_WRITE>
__device__ __forceinline__ void mfma_phase(const DecodeParams &p, int b, int kvh, int r0, int r1, Rows rows,
                                           const char *kbase, const char *vbase, char *ringK, char *ringV,
                                           QOperand<T, DH, G> &qo, RingCount &cnt, float *s_p,
                                           WaveState<G, DH / 16> &st) {
    using off_t = row_off_t<T>;
    constexpr int RB = DH * (int)sizeof(T);    // bytes of a row
    constexpr int SL = RB / 64, VD = DH / 16;  // 16-byte words of K per lane; output dims per lane
    constexpr int VE = Vec16<T>::N;            // elements per 16-byte word
    constexpr int VB = VD * (int)sizeof(T);    // bytes of V per lane per quarter: 8 to 64
    constexpr int NH = kLaneHeads<G>;
    constexpr int VW = VB >= 16 ? VB / 16 : 1; // 16-byte words (or one 8-byte word)
    constexpr int BSTRIDE = NW * 16;
    // The next block's rows in a second register set while this block is
    // computed, where both fit 256 registers (two waves per SIMD); else the
    // other waves' loads cover a block's compute.
    constexpr bool kDoubleBuffer = RB <= CMC_DOUBLE_BUFFER_MAX_ROW && !(sizeof(T) == 2 && G > 4 && RB > 128);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r16 = lane & 15, q4 = lane >> 4, kq = lane & 3, dg = lane >> 2;
    const uint32_t koff = 16u * q4;  // + 64 * i for chunk i
    const uint32_t voff = (uint32_t)(VB < 16 ? VB : 16) * dg;  // + 256 * j for word j
    const bool upper = (q4 & 1) != 0;  // G = 8: this lane's heads are 4 .. 7

    int blk = r0 + wave * 16;
    if (blk >= r1) return;  // wave-uniform

    // Rows past the phase end are clamped to its last row and loaded anyway
    // (branch-free loads keep the compiler's wait counts exact, so a block's
    // prefetch is never waited for early); their scores are masked to -inf,
    // so they contribute p = 0.
#define CMC_KEYS(B0_, K_, V_)                                               \
    do {                                                                   \
        K_ = rows.key(min((B0_) + r16, r1 - 1));                           \
        _Pragma("unroll") for (int qq = 0; qq < 4; ++qq)                   \
            V_[qq] = rows.key(min((B0_) + 4 * qq + kq, r1 - 1));           \
    } while (0)
#define CMC_LOAD(B0_, K_, V_, KR_, VR_)                                                                \
    do {                                                                                             \
        {                                                                                            \
            const off_t o = (off_t)rows.slot(min((B0_) + r16, r1 - 1), K_) * RB + koff;             \
            _Pragma("unroll") for (int i = 0; i < SL; ++i) KR_[i] = ld16(kbase + o + 64 * i);        \
        }                                                                                            \
        _Pragma("unroll") for (int qq = 0; qq < 4; ++qq) {                                           \
            const off_t o = (off_t)rows.slot(min((B0_) + 4 * qq + kq, r1 - 1), V_[qq]) * RB + voff;  \
            if constexpr (VB >= 16) {                                                                \
                _Pragma("unroll") for (int j = 0; j < VW; ++j) VR_[qq][j] = ld16<true>(vbase + o + 256 * j);  \
            } else {                                                                                 \
                const uint2 t = *reinterpret_cast<const uint2 *>(vbase + o);                         \
                VR_[qq][0] = make_uint4(t.x, t.y, 0, 0);                                             \
            }                                                                                        \
        }                                                                                            \
    } while (0)
    // A phase without masks ends in copies of its last row: their values are
    // zeroed, since an infinite one times p = 0 is NaN.
#define CMC_TAIL(B0_, VR_)                                                                            \
    do {                                                                                             \
        if constexpr (!Rows::kMasked && (sizeof(T) == 4 || G > 4)) {                                 \
            if ((B0_) + 16 > r1) {                                                                   \
                _Pragma("unroll") for (int qq = 0; qq < 4; ++qq)                                     \
                    if ((B0_) + 4 * qq + kq >= r1)                                                   \
                        _Pragma("unroll") for (int j = 0; j < VW; ++j) VR_[qq][j] = make_uint4(0, 0, 0, 0); \
            }                                                                                        \
        }                                                                                            \
    } while (0)
    // S = Q K^T by MFMA; online softmax rescaling the accumulators only when
    // a head's running max grows (wave-uniform: every lane row holds the same
    // scores); P V on the VALU.
#define CMC_COMPUTE(B0_, KR_, VR_)                                                                     \
    do {                                                                                             \
        /* uniform; a block reaching past r1 is never "full": its rows past the */                    \
        /* phase end may have been loaded before r1 was limited by the count */                     \
        const bool bfull = (B0_) + 16 <= r1 && rows.all_valid((B0_), (B0_) + 16);                   \
        const bool kval = (B0_) + r16 < r1 && (bfull || rows.valid((B0_) + r16));                    \
        const floatx4 c = qo.scores(KR_);                                                            \
        float pk[NH], mbs[G];                                                                        \
        /* the lane's heads' maxima first, in straight-line code, so their chains interleave; */     \
        /* with eight heads the other four come from the neighbouring lane row */                    \
        _Pragma("unroll") for (int g = 0; g < NH; ++g) {                                             \
            const float mx = lane_max16(kval ? c[g] : -INFINITY);                                    \
            if constexpr (G > 4) pair_rows16(mx, mbs[g], mbs[(g + 4) % G]);                          \
            else mbs[g] = mx;                                                                        \
        }                                                                                            \
        _Pragma("unroll") for (int g = 0; g < G; ++g) {                                              \
            const float mb = mbs[g];                                                                 \
            if (mb > st.m[g]) {                                                                      \
                if (st.m[g] != kNoMax) { /* before the first valid key l and acc are 0 */            \
                    const float d = st.m[g] - mb;                                                    \
                    const float alpha = kSmallWeights<T, G> ? exp2f(d) : fast_exp2(d);               \
                    if constexpr (G > 4) st.l[g % NH] *= (g >= 4) == upper ? alpha : 1.f;            \
                    else st.l[g] *= alpha;                                                           \
                    _Pragma("unroll") for (int i = 0; i < VD; ++i) st.acc[g][i] *= alpha;            \
                }                                                                                    \
                st.m[g] = mb;                                                                        \
            }                                                                                        \
        }                                                                                            \
        float xs[NH], least = 0.f;                                                                   \
        _Pragma("unroll") for (int g = 0; g < NH; ++g) {                                             \
            const float ma = st.m[g], mb = st.m[(g + 4) % G];                                        \
            const float m = G > 4 && upper ? mb : ma;                                                \
            xs[g] = c[g] - m;                                                                        \
            /* a masked key weighs 0 */                                                              \
            pk[g] = kval ? fast_exp2(xs[g]) : 0.f;                                                   \
            if constexpr (kSmallWeights<T, G>) least = fminf(least, xs[g]);                          \
        }                                                                                            \
        if constexpr (kSmallWeights<T, G>) {                                                         \
            if (kval && least < -126.f) { /* rare */                                                 \
                _Pragma("unroll") for (int g = 0; g < NH; ++g) pk[g] = exp2f(xs[g]);                 \
            }                                                                                        \
        }                                                                                            \
        _Pragma("unroll") for (int g = 0; g < NH; ++g) st.l[g] += pk[g];                             \
        if (q4 < G / NH) {                                                                           \
            _Pragma("unroll") for (int g = 0; g < NH; ++g) s_p[r16 * G + q4 * NH + g] = pk[g];      \
        }                                                                                            \
        wave_lds_sync();                                                                             \
        _Pragma("unroll") for (int qq = 0; qq < 4; ++qq) {                                           \
            if constexpr (Rows::kMasked) {                                                           \
                /* masked ring slots (and unfilled slots past r1) may hold anything, */              \
                /* NaN included: zero their values, since 0 * NaN is NaN (p is 0) */                  \
                const int vrow = (B0_) + 4 * qq + kq;                                                \
                if (!bfull && !(vrow < r1 && rows.valid(vrow))) {                                    \
                    _Pragma("unroll") for (int j = 0; j < VW; ++j) VR_[qq][j] = make_uint4(0, 0, 0, 0); \
                }                                                                                    \
            }                                                                                        \
            float pv[G];                                                                             \
            _Pragma("unroll") for (int g = 0; g < G; ++g) pv[g] = s_p[(4 * qq + kq) * G + g];         \
            _Pragma("unroll") for (int j = 0; j < VW; ++j) {                                         \
                float vf[VE];                                                                        \
                Vec16<T>::widen(VR_[qq][j], vf);                                                     \
                _Pragma("unroll") for (int g = 0; g < G; ++g)                                        \
                    _Pragma("unroll") for (int e = 0; e < (VD < VE ? VD : VE); ++e)                  \
                        st.acc[g][VE * j + e] = fmaf(pv[g], vf[e], st.acc[g][VE * j + e]);           \
            }                                                                                        \
        }                                                                                            \
        wave_lds_sync();                                                                             \
        if constexpr (RING_WRITE) {                                                                  \
            if ((B0_) + r16 < r1) {                                                                  \
                const off_t o = (off_t)rows.ring_slot((B0_) + r16) * RB + koff;                      \
                _Pragma("unroll") for (int i = 0; i < SL; ++i) st16(ringK + o + 64 * i, KR_[i]);     \
            }                                                                                        \
            _Pragma("unroll") for (int qq = 0; qq < 4; ++qq) {                                       \
                const int vrow = (B0_) + 4 * qq + kq;                                                \
                if (vrow < r1) {                                                                     \
                    const off_t o = (off_t)rows.ring_slot(vrow) * RB + voff;                         \
                    if constexpr (VB >= 16) {                                                        \
                        _Pragma("unroll") for (int j = 0; j < VW; ++j) st16(ringV + o + 256 * j, VR_[qq][j]);\
                    } else {                                                                         \
                        *reinterpret_cast<uint2 *>(ringV + o) = make_uint2(VR_[qq][0].x, VR_[qq][0].y); \
                    }                                                                                \
                }                                                                                    \
            }                                                                                        \
        }                                                                                            \
    } while (0)

    // Once the wave's first K/V loads are in flight: fetch the ring count
    // and q, split q (both round trips overlap the K/V loads'), then read the
    // count into the masks and end the phase at the last filled ring slot
    // (a phase without masks does not wait for the count).
#define CMC_AFTER_FIRST_LOAD()                    \
    do {                                          \
        if (!qo.ready) {                          \
            cnt.load(p.win_count, b);             \
            qo.load(p, b, kvh);                   \
            qo.ready = true;                      \
        }                                         \
        rows.resolve(cnt);                        \
        r1 = rows.limit(r1);                      \
    } while (0)

    // Two register sets used in turn: the next block's K/V loads are in
    // flight while this block computes (the loop is unrolled by two so no
    // registers are copied).  Index-list entries are fetched two blocks
    // ahead and issued before the next block's K/V loads: loads retire in
    // issue order, so waiting for the entries then never waits for the
    // prefetched K/V rows.  The wave's last block prefetches nothing (loads
    // past the end would be drained by the barrier after the loop).
    int kc, kvc[4], kn, kvn[4];
    if constexpr (!kDoubleBuffer) {
        uint4 kr[SL], vr[4][VW];
        CMC_KEYS(blk, kc, kvc);
#pragma unroll 1
        for (; blk < r1; blk += BSTRIDE) {
            CMC_LOAD(blk, kc, kvc, kr, vr);
            CMC_AFTER_FIRST_LOAD();
            CMC_KEYS(blk + BSTRIDE, kc, kvc);
            CMC_TAIL(blk, vr);
            CMC_COMPUTE(blk, kr, vr);
        }
        return;
    }
    uint4 kA[SL], vA[4][VW], kB[SL], vB[4][VW];
    CMC_KEYS(blk, kc, kvc);
    CMC_LOAD(blk, kc, kvc, kA, vA);
    CMC_AFTER_FIRST_LOAD();
    CMC_KEYS(blk + BSTRIDE, kc, kvc);
#pragma unroll 1
    while (true) {
        int nb = blk + BSTRIDE;
        if (nb >= r1) {  // wave-uniform
            CMC_TAIL(blk, vA);
            CMC_COMPUTE(blk, kA, vA);
            break;
        }
        CMC_KEYS(nb + BSTRIDE, kn, kvn);
        CMC_LOAD(nb, kc, kvc, kB, vB);
        kc = kn;
#pragma unroll
        for (int i = 0; i < 4; ++i) kvc[i] = kvn[i];
        __builtin_amdgcn_sched_barrier(0);  // keep the prefetch above this block's compute
        CMC_COMPUTE(blk, kA, vA);
        blk = nb;
        nb = blk + BSTRIDE;
        if (nb >= r1) {
            CMC_TAIL(blk, vB);
            CMC_COMPUTE(blk, kB, vB);
            break;
        }
        CMC_KEYS(nb + BSTRIDE, kn, kvn);
        CMC_LOAD(nb, kc, kvc, kA, vA);
        kc = kn;
#pragma unroll
        for (int i = 0; i < 4; ++i) kvc[i] = kvn[i];
        __builtin_amdgcn_sched_barrier(0);
        CMC_COMPUTE(blk, kB, vB);
        blk = nb;
    }
#undef CMC_KEYS
#undef CMC_LOAD
#undef CMC_TAIL
#undef CMC_COMPUTE
#undef CMC_AFTER_FIRST_LOAD
}

template <int NW, typename T, int DH, int G, bool IX>
__device__ __forceinline__ void mfma_loop(const DecodeParams &p, int b, int kvh, int kb, int c0, int c1,
                                          RingCount &cnt, float *s_p, uint4 *s_q, WaveState<G, DH / 16> &st) {
    QOperand<T, DH, G> qo;
    qo.lds = s_q;
    qo.ready = false;
    constexpr size_t RB = DH * sizeof(T);
    const size_t head = (size_t)b * p.Hkv + kvh;
    const int T_new = p.W > 0 ? p.T_new : 0;
    const int pool_end = kb, ring_end = kb + p.W;

    // pool rows
    {
        const PoolRows<IX> rows{p.idx, (size_t)b * p.k, p.N > 0 ? p.N - 1 : 0};
        const char *kb = static_cast<const char *>(p.cme_k) + head * (size_t)p.N * RB;
        const char *vb = static_cast<const char *>(p.cme_v) + head * (size_t)p.N * RB;
        mfma_phase<NW, T, DH, G, PoolRows<IX>, false>(p, b, kvh, c0, min(c1, pool_end), rows, kb, vb, nullptr, nullptr,
                                                  qo, cnt, s_p, st);
    }
    if (p.W > 0) {
        char *wk = static_cast<char *>(p.win_k) + head * (size_t)p.W * RB;
        char *wv = static_cast<char *>(p.win_v) + head * (size_t)p.W * RB;
        // the W ring slots in physical order, masked by the count
        const RingRows rr{pool_end, T_new, p.W};
        mfma_phase<NW, T, DH, G, RingRows, false>(p, b, kvh, max(c0, pool_end), min(c1, ring_end), rr, wk, wv, nullptr,
                                                  nullptr, qo, cnt, s_p, st);
        // rows appended in this call
        if (T_new > 0) {
            const NewRows nr{ring_end, p.W};
            const char *nk = static_cast<const char *>(p.new_k) + head * (size_t)T_new * RB;
            const char *nv = static_cast<const char *>(p.new_v) + head * (size_t)T_new * RB;
            mfma_phase<NW, T, DH, G, NewRows, true>(p, b, kvh, max(c0, ring_end), c1, nr, nk, nv, wk, wv, qo, cnt, s_p,
                                                    st);
        }
    }
    // Wave totals: l over the 16 keys of one lane row (rows hold copies),
    // acc over the 4 keys sharing a dim group.
#pragma unroll
    for (int g = 0; g < G; ++g) {
        if (g < kLaneHeads<G>) st.l[g] = lane_reduce<OpSum, 1, 16>(st.l[g]);
#pragma unroll
        for (int i = 0; i < DH / 16; ++i) st.acc[g][i] = lane_reduce<OpSum, 1, 4>(st.acc[g][i]);
    }
}

// ------------------------------------------------------------------ kernel

// Cross-workgroup publication without device-scope fences.  The partials are
// written and read with relaxed agent-scope atomic accesses (coherent across
// the XCDs' L2 caches, unlike plain accesses), the writer waits until its
// stores have completed (s_waitcnt) before arriving on the counter, and the
// reader issues its loads only after the arrival count has returned.  An
// agent-scope fence would instead write back and invalidate the whole L2 of
// the XCD for every workgroup, which costs microseconds each.
// Two adjacent floats (8-byte aligned) as one 64-bit coherent access.
__device__ __forceinline__ void coherent_store2(float *p, float a, float b) {
    const uint64_t v = (uint64_t)__float_as_uint(a) | ((uint64_t)__float_as_uint(b) << 32);
    __hip_atomic_store(reinterpret_cast<uint64_t *>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 coherent_load2(const float *p) {
    const uint64_t v = __hip_atomic_load(reinterpret_cast<const uint64_t *>(p), __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
}

// Combine the waves' (m, l, acc) of head g, dim d; returns the joint max.
template <int NW, int G, int DH>
__device__ __forceinline__ float combine_waves(const float (&sm)[NW][G], const float (&sl)[NW][G],
                                               const float (&sa)[NW][G][DH], int g, int d, float &num,
                                               float &den) {
    // Every LDS read issued before the first wait, and no branch on M: with
    // no valid key in any wave (M = kNoMax) the weights are 1 against zeros, so
    // num = den = 0.
    float mw[NW], lw[NW], aw[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        mw[w] = sm[w][g];
        lw[w] = sl[w][g];
        aw[w] = sa[w][g][d];
    }
    float M = mw[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, mw[w]);
    num = 0.f;
    den = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float f = fast_exp2(mw[w] - M);
        num = fmaf(f, aw[w], num);
        den = fmaf(f, lw[w], den);
    }
    return M;
}

// Waves per SIMD the compiler must leave registers for, where its own choice
// would be fewer: one for eight heads (but not of 256, whose accumulators
// alone take half of the registers) and 256-wide fp32 rows, and two for the
// 4-wave kernel of eight heads of 128 in bf16, which keeps one block of rows
// in flight per wave and so lives on its waves (264 pairs, 6144 keys: 221 us
// with two, 172 us with three).
template <int NW, typename T, int DH, int G>
constexpr int kMinWaves = NW == 4 && sizeof(T) == 2 && DH == 128 && G == 8 ? 3
                          : G * DH <= 1024 && (G > 4 || sizeof(T) * DH > 512) ? 2 : 1;

// The leading arguments are the fields the first K/V loads need (info packs
// S, new_split, whether k_len is given, and T_new); they arrive in
// SGPRs at wave launch (kernel-argument preloading, 14 dwords), so those
// loads never wait for the kernel-argument segment.  The rest of the
// parameters come from `pm`.
template <int NW, typename T, int DH, int G, bool IX>
__global__ __launch_bounds__(NW * kWave, (kMinWaves<NW, T, DH, G>)) void decode_kernel(const void *cme_k, const void *cme_v, void *win_k,
                                                            void *win_v, int k, int W, int N, int Hkv, int chunk,
                                                            int info, DecodeParams pm) {
    DecodeParams p = pm;
    p.cme_k = cme_k;
    p.cme_v = cme_v;
    p.win_k = win_k;
    p.win_v = win_v;
    p.k = k;
    p.W = W;
    p.N = N;
    p.Hkv = Hkv;
    p.chunk = chunk;
    p.S = info & 0xFF;
    p.new_split = (info >> 8) & 1;
    const bool has_klen = (info >> 10) & 1;
    p.T_new = (int)((unsigned)info >> 16);
    constexpr int kThreads = NW * kWave;
    constexpr int VEC = DH / 16;  // output dims a lane accumulates
    constexpr int NH = kLaneHeads<G>;
    const int s = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;

    // Fetched by each wave after its first K/V loads, so they never wait for it.
    RingCount cnt{0, false};
    int kb = p.k;  // pool rows of this sequence
    if (has_klen) {
        const int v = p.k_len[b];
        kb = v < 0 ? 0 : (v > p.k ? p.k : v);
    }
    // Key list: kb pool rows, the W ring slots, the T_new appended rows (see
    // the phases above); its length does not depend on the ring count.  The
    // split plan covers k + W rows in chunks; the appended rows go to the last
    // split, or to a split of their own (the last) when p.new_split is set.
    const int Lkw = kb + p.W;
    const int L = kb + (p.W > 0 ? p.W + p.T_new : 0);
    int c0, c1;
    if (p.new_split) {
        const bool own = s == p.S - 1;
        c0 = own ? Lkw : s * p.chunk;
        c1 = own ? L : (s == p.S - 2 ? Lkw : min(c0 + p.chunk, Lkw));
    } else {
        c0 = s * p.chunk;
        c1 = s == p.S - 1 ? L : min(c0 + p.chunk, L);
    }

    // Ring count.  It may be advanced only after every wave of the
    // sequence's workgroups has read it.  Each wave stores the count it read
    // into LDS before the barrier that ends its walk (a store of the loaded
    // value, so the read has returned by then); after that barrier one
    // arrival per (sequence, kv head) pair goes to the sequence's counter:
    //   S == 1: thread 0 of the workgroup, right after the barrier;
    //   S > 1: each split arrives on its pair counter after that barrier, and
    //     the merging workgroup (the last split of the pair) then arrives for
    //     the pair, overlapping its merge loads.
    // The last of the Hkv arrivals writes the advanced count and re-arms the
    // counter, at its workgroup's end (the arrival's value is waited for only
    // there).  No data is published through the counter, so no fence is
    // needed.
    const bool bump = p.T_new > 0 && p.W > 0;
    unsigned prev = ~0u;  // the sequence counter before this workgroup's arrival (one lane)

    WaveState<G, VEC> st;
    st.init();
    __shared__ __attribute__((aligned(16))) float s_pw[NW][16 * G];
    __shared__ uint4 s_q[NW][QOperand<T, DH, G>::kLdsWords];
    mfma_loop<NW, T, DH, G, IX>(p, b, kvh, kb, c0, c1, cnt, s_pw[threadIdx.x >> 6], s_q[threadIdx.x >> 6], st);
    if (p.W > 0) cnt.load(p.win_count, b);  // a wave without K/V rows
    const int cnt_now = cnt.value();
#define CMC_BUMP()                                                                         \
    do {                                                                                 \
        if (bump && prev == (unsigned)(p.Hkv - 1)) { /* one lane per sequence */       \
            p.win_count[b] = cnt_now + p.T_new;                                          \
            __hip_atomic_store(&p.seq_counter[b], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); \
        }                                                                                \
    } while (0)

    // One lane of each dim group holds it after the wave reduction.
    const bool holder = (lane & 3) == 0;
    constexpr int VL = VEC < Vec16<T>::N ? VEC : Vec16<T>::N;  // consecutive dims a lane holds: of word j, dims
                                                                // 16 VL j + VL (lane / 4) .. + VL - 1

    __shared__ float s_acc[NW][G][DH];
    __shared__ float s_m[NW][G], s_l[NW][G];
    if (holder) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int i = 0; i < VEC; ++i) s_acc[wave][g][(i / VL) * 16 * VL + (lane >> 2) * VL + i % VL] = st.acc[g][i];
    }
    if ((lane & 15) == 0 && lane / 16 < G / NH) {  // lanes 0 (and, G = 8, 16): the heads they hold
#pragma unroll
        for (int g = 0; g < NH; ++g) {
            const float ma = st.m[g], mb = st.m[(g + 4) % G];
            s_m[wave][(lane / 16) * NH + g] = G > 4 && lane != 0 ? mb : ma;
            s_l[wave][(lane / 16) * NH + g] = st.l[g];
        }
    }
    __shared__ int s_cnt[NW];
    if (bump && lane == 0) s_cnt[wave] = cnt.raw;  // stored once the wave's count read has returned
    __syncthreads();

    const size_t head = (size_t)b * p.Hkv + kvh;
    float *outp = p.out + ((size_t)b * p.Hq + (size_t)kvh * G) * DH;
    __shared__ int s_last;
    if (p.S == 1) {
        // every wave's count read returned before the barrier above
        if (bump && threadIdx.x == 0) prev = arrive_once(p.seq_counter, b, (unsigned)(s_cnt[NW - 1] != INT_MIN));
        for (int t = threadIdx.x; t < G * DH; t += kThreads) {
            const int g = t / DH, d = t % DH;
            float num, den;
            combine_waves<NW, G, DH>(s_m, s_l, s_acc, g, d, num, den);
            outp[t] = den > 0.f ? num * __builtin_amdgcn_rcpf(den) : 0.f;
        }
        CMC_BUMP();
    } else {
        // Publish this split's partial with agent-coherent 64-bit stores (two
        // dims per thread), wait for them to complete, then arrive on the
        // (b, kv head) counter.
        const size_t part = (head * p.S + s) * G;
        for (int t = threadIdx.x; t < G * DH / 2; t += kThreads) {
            const int g = (2 * t) / DH, d = (2 * t) % DH;
            float n0, n1, den;
            const float M = combine_waves<NW, G, DH>(s_m, s_l, s_acc, g, d, n0, den);
            combine_waves<NW, G, DH>(s_m, s_l, s_acc, g, d + 1, n1, den);
            coherent_store2(&p.part_acc[(part + g) * DH + d], n0, n1);
            if (d == 0) coherent_store2(&p.part_ml[(part + g) * 2], M, den);
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned prev = __hip_atomic_fetch_add(&p.pair_counter[head], 1u, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
            s_last = prev == (unsigned)(p.S - 1);
        }
        __syncthreads();
        if (!s_last) return;  // workgroup-uniform
        // The last split merges all S partials in fixed split order.  Its
        // first batch of acc partials (up to kMB splits per dim pair) and all
        // (m, l) pairs are requested together, so the merge costs one round
        // trip when S <= kMB; the (m, l) pairs are staged in LDS.  The
        // batch's loads are issued unconditionally (splits past S - 1 reload
        // split S - 1 and are never used): as atomic loads they cannot be
        // speculated, and a branch around each cost about a dozen
        // instructions between the arrival and the merge's data.
        constexpr int kPairs = (G * DH / 2 + kThreads - 1) / kThreads;  // dim pairs per thread
        constexpr int kMB = kPairs >= 4 ? 8 : 16;
        const float *ml = p.part_ml + head * p.S * G * 2;
        const float *ac = p.part_acc + head * p.S * G * DH;
        float *s_ml = &s_acc[0][0][0];  // reuse: S*G*2 <= NW*G*DH floats (S <= 2*DH)
        // The (m, l) pairs are requested first (loads complete in issue
        // order, and the max and the weights need only them), and the barrier
        // that publishes them in LDS waits for LDS alone: the acc partials
        // may still be in flight while the weights are computed, and their
        // first use waits for them.
        const bool ml_first = threadIdx.x < p.S * G;  // the first kThreads pairs
        float2 mlv = make_float2(0.f, 0.f);
        if (ml_first) mlv = coherent_load2(&ml[2 * threadIdx.x]);
        float2 a[kPairs][kMB];
#pragma unroll
        for (int pr = 0; pr < kPairs; ++pr) {
            const int t = threadIdx.x + pr * kThreads;
            const int g = (2 * min(t, G * DH / 2 - 1)) / DH, d = (2 * min(t, G * DH / 2 - 1)) % DH;
#pragma unroll
            for (int j = 0; j < kMB; ++j) a[pr][j] = coherent_load2(&ac[(min(j, p.S - 1) * G + g) * DH + d]);
        }
        if (ml_first) {
            s_ml[2 * threadIdx.x] = mlv.x;
            s_ml[2 * threadIdx.x + 1] = mlv.y;
        }
        for (int t = threadIdx.x + kThreads; t < p.S * G; t += kThreads) {
            const float2 v = coherent_load2(&ml[2 * t]);
            s_ml[2 * t] = v.x;
            s_ml[2 * t + 1] = v.y;
        }
        // this workgroup completes the pair; the arrival overlaps the merge loads
        if (bump && threadIdx.x == 0) prev = arrive_once(p.seq_counter, b, (unsigned)(s_cnt[NW - 1] != INT_MIN));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0) only: vmcnt and expcnt at their maxima
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int pr = 0; pr < kPairs; ++pr) {
            const int t = threadIdx.x + pr * kThreads;
            if (t >= G * DH / 2) continue;
            const int g = (2 * t) / DH, d = (2 * t) % DH;
            // The first batch's (m, l) pairs read together (splits past S - 1
            // read split S - 1 again), and its terms masked by selects rather
            // than branches: no LDS round trip waits for another.  The max
            // is unchanged by the repeats, and the sums take the splits in
            // order as before.
            float mj[kMB], lj[kMB];
#pragma unroll
            for (int j = 0; j < kMB; ++j) {
                const float2 v = *reinterpret_cast<const float2 *>(&s_ml[(min(j, p.S - 1) * G + g) * 2]);
                mj[j] = v.x;
                lj[j] = v.y;
            }
            float M = kNoMax;
#pragma unroll
            for (int j = 0; j < kMB; ++j) M = fmaxf(M, mj[j]);
            for (int q = kMB; q < p.S; ++q) M = fmaxf(M, s_ml[(q * G + g) * 2]);
            float n0 = 0.f, n1 = 0.f, den = 0.f;
            if (M != kNoMax) {
#pragma unroll
                for (int j = 0; j < kMB; ++j) {
                    const bool in = j < p.S;
                    const float f = fast_exp2(mj[j] - M);
                    den = in ? fmaf(f, lj[j], den) : den;
                    n0 = in ? fmaf(f, a[pr][j].x, n0) : n0;
                    n1 = in ? fmaf(f, a[pr][j].y, n1) : n1;
                }
                for (int q0 = kMB; q0 < p.S; q0 += kMB) {
                    float2 x[kMB];
#pragma unroll
                    for (int j = 0; j < kMB; ++j)
                        x[j] = q0 + j < p.S ? coherent_load2(&ac[((q0 + j) * G + g) * DH + d])
                                            : make_float2(0.f, 0.f);
#pragma unroll
                    for (int j = 0; j < kMB; ++j) {
                        if (q0 + j < p.S) {
                            const int q = q0 + j;
                            const float f = fast_exp2(s_ml[(q * G + g) * 2] - M);
                            den = fmaf(f, s_ml[(q * G + g) * 2 + 1], den);
                            n0 = fmaf(f, x[j].x, n0);
                            n1 = fmaf(f, x[j].y, n1);
                        }
                    }
                }
            }
            const float inv = den > 0.f ? __builtin_amdgcn_rcpf(den) : 0.f;  // within 1 ulp
            *reinterpret_cast<float2 *>(&outp[g * DH + d]) = make_float2(n0 * inv, n1 * inv);
        }
        if (threadIdx.x == 0)
            __hip_atomic_store(&p.pair_counter[head], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        CMC_BUMP();
    }
#undef CMC_BUMP

}

template <typename T, int DH, int G>
hipError_t launch3(const DecodeParams &p, hipStream_t stream) {
    dim3 grid(p.S, p.Hkv, p.B);
    if (p.S < 1 || p.S > 0xFF || p.T_new < 0 || p.T_new > kMaxAppendRows) return hipErrorInvalidValue;
    const int info = p.S | (p.new_split << 8) | ((p.k_len != nullptr) << 10) | (p.T_new << 16);
    const bool ix = p.idx != nullptr;
#define CMC_LAUNCH(NW_, IX_)                                                                                     \
    decode_kernel<NW_, T, DH, G, IX_><<<grid, NW_ * kWave, 0, stream>>>(p.cme_k, p.cme_v, p.win_k, p.win_v, \
                                                                             p.k, p.W, p.N, p.Hkv, p.chunk, info, p)
    if (p.waves == 4) {
        if (ix) CMC_LAUNCH(4, true);
        else CMC_LAUNCH(4, false);
    } else if constexpr (decode_waves_ok(8, G, DH)) {
        if (p.waves != 8) return hipErrorInvalidValue;
        if (ix) CMC_LAUNCH(8, true);
        else CMC_LAUNCH(8, false);
    } else {
        return hipErrorInvalidValue;
    }
#undef CMC_LAUNCH
    return hipGetLastError();
}

template <typename T, int DH>
hipError_t launch_g(const DecodeParams &p, int G, hipStream_t stream) {
    switch (G) {
        case 1: return launch3<T, DH, 1>(p, stream);
        case 2: return launch3<T, DH, 2>(p, stream);
        case 4: return launch3<T, DH, 4>(p, stream);
        case 8: return launch3<T, DH, 8>(p, stream);
    }
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_dh(const DecodeParams &p, int G, int Dh, hipStream_t stream) {
    switch (Dh) {
        case 64: return launch_g<T, 64>(p, G, stream);
        case 128: return launch_g<T, 128>(p, G, stream);
        case 256: return launch_g<T, 256>(p, G, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_two_tier_decode(const DecodeParams &p, bool bf16, int G, int Dh, hipStream_t stream) {
    if (p.B == 0) return hipSuccess;
    return bf16 ? launch_dh<uint16_t>(p, G, Dh, stream) : launch_dh<float>(p, G, Dh, stream);
}

float decode_qscale(float scale) { return scale * kLog2e; }

}  // namespace cmc

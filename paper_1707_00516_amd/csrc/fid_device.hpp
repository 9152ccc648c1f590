// Device helpers shared by the libfastid kernels: lane and wave utilities,
// the per-wave top-k list primitives and the workgroup top-k selection.
#pragma once

#include "fid_common.hpp"

namespace fid {

// Scalar (constant address space) view of a wave-uniform pointer: loads
// through it become s_load_dwordxN into SGPRs.
typedef const __attribute__((address_space(4))) uint32_t* kptr_u32;
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
typedef const __attribute__((address_space(4))) u32x16* kptr_u32x16;

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63u); }

// acc + popcount(x) as one v_bcnt_u32_b32 with its accumulator operand.  The
// compiler would otherwise rebalance a long run of these sums into trees of
// popcounts and three-way adds (2.5 VALU per word instead of 2).
__device__ __forceinline__ uint32_t popc_acc(uint32_t x, uint32_t acc)
{
    __asm__("v_bcnt_u32_b32 %0, %1, %2" : "=v"(acc) : "v"(x), "v"(acc));
    return acc;
}

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Largest key of a k-slot list and its position (ties: the last position).
template <typename ListPtr>
__device__ __forceinline__ void list_max(ListPtr list, int k, uint64_t& mx, int& mpos)
{
    const int lane = lane_id();
    uint64_t v = 0;
    int pos = -1;
    for (int i = lane; i < k; i += 64) {
        const uint64_t x = list[i];
        if (pos < 0 || x > v) {
            v = x;
            pos = i;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint64_t ov = __shfl_xor(v, off);
        const int op = __shfl_xor(pos, off);
        if (ov > v || (ov == v && op > pos)) {
            v = ov;
            pos = op;
        }
    }
    mx = v;
    mpos = pos;
}

// Per-wave top-k list of one query, k slots in global memory or LDS.  A worker
// scans its references in increasing index order, so a new candidate whose
// count equals the list's worst count has a larger index and is never better:
// once the list is full the filter is "count < worst count".  Entry i of a
// list is only ever read or written by lane (i & 63) of the owning wave, so
// program order makes every update visible to the next scan.

__device__ __forceinline__ void topk_insert(uint64_t* __restrict__ list, int k, int64_t rbase,
                                            uint32_t acc, uint64_t m, uint32_t* lthr_q,
                                            uint32_t* lfill_q)
{
    const int lane = lane_id();
    uint32_t t = *lthr_q;
    uint32_t fill = *lfill_q;
    while (m) {
        const int src = __builtin_ctzll(m);
        m &= m - 1;
        const uint32_t c = (uint32_t)__shfl((int)acc, src);
        if (c >= t) continue;
        const uint64_t key = ((uint64_t)c << kIdxBits) | (uint64_t)(rbase + src);
        uint64_t mx;
        int mpos;
        if (fill < (uint32_t)k) {
            if (lane == (int)(fill & 63u)) list[fill] = key;
            ++fill;
            if (fill < (uint32_t)k) continue;
            list_max(list, k, mx, mpos);
        } else {
            list_max(list, k, mx, mpos);
            if (key >= mx) continue;
            if (lane == (mpos & 63)) list[mpos] = key;
            list_max(list, k, mx, mpos);
        }
        const uint32_t worst = (uint32_t)(mx >> kIdxBits);
        if (worst < t) t = worst;
    }
    if (lane == 0) {
        *lthr_q = t;
        *lfill_q = fill;
    }
}

// Ascending bitonic sort of the first p2 (a power of two) keys of s.
template <int NT>
__device__ __forceinline__ void bitonic_sort(uint64_t* s, int p2)
{
    for (int size = 2; size <= p2; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int t = (int)threadIdx.x; t < p2 / 2; t += NT) {
                const int i = 2 * t - (t & (stride - 1));
                const int j = i + stride;
                const bool asc = (i & size) == 0;
                const uint64_t a = s[i], b = s[j];
                if ((a > b) == asc) {
                    s[i] = b;
                    s[j] = a;
                }
            }
            __syncthreads();
        }
    }
}

// Exact k smallest of n_in keys (k <= kSelectSlots / 2).  On return s[0..k)
// holds them ascending (kSentinel where fewer than k keys exist).  Keys below
// the current k-th best (and below `below`, which the caller guarantees every
// member of the answer is) are gathered in s[half..) and merged by a full
// sort whenever some arrived, so the work tracks the number of improving keys.
template <int NT = kSelectThreads, class Load>
__device__ void wg_topk(Load load, int64_t n_in, int k, uint64_t* s, int* nb, uint64_t below = kSentinel)
{
    constexpr int half = kSelectSlots / 2;
    for (int i = (int)threadIdx.x; i < kSelectSlots; i += NT) s[i] = kSentinel;
    if (threadIdx.x == 0) *nb = 0;
    __syncthreads();
    for (int64_t base = 0; base < n_in; base += half) {
        const uint64_t kth = s[k - 1] < below ? s[k - 1] : below;
        for (int j = 0; j < half / NT; ++j) {
            const int64_t i = base + j * NT + threadIdx.x;
            if (i < n_in) {
                const uint64_t key = load(i);
                if (key < kth) s[half + atomicAdd(nb, 1)] = key;
            }
        }
        __syncthreads();
        const int n = *nb;
        __syncthreads();
        if (n > 0) {
            bitonic_sort<NT>(s, kSelectSlots);
            for (int i = (int)threadIdx.x; i < half; i += NT) s[half + i] = kSentinel;
            if (threadIdx.x == 0) *nb = 0;
            __syncthreads();
        }
    }
}

template <int NT = kSelectThreads>
__device__ __forceinline__ void write_topk(const uint64_t* s, int k, int32_t* cnt, int64_t* idx)
{
    for (int j = (int)threadIdx.x; j < k; j += NT) {
        const uint64_t key = s[j];
        cnt[j] = key == kSentinel ? INT32_MAX : (int32_t)(key >> kIdxBits);
        idx[j] = key == kSentinel ? -1 : (int64_t)(key & kIdxMask);
    }
}

// Sum of v over the threads before this one in the workgroup (part: NT / 64
// words of LDS; contains a barrier before part is read and one after).
template <int NT>
__device__ __forceinline__ uint32_t wg_exclusive_sum(uint32_t v, uint32_t* part)
{
    const int lane = lane_id(), wv = (int)threadIdx.x >> 6;
    uint32_t run = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = (uint32_t)__shfl_up((int)run, o);
        if (lane >= o) run += u;
    }
    if (lane == 63) part[wv] = run;
    __syncthreads();
    uint32_t before = run - v;
    for (int i = 0; i < wv; ++i) before += part[i];
    __syncthreads();
    return before;
}

// The bin where the running count of hist[0 .. nbins) first reaches target,
// and that running count; untouched when the total is smaller.  Called by all
// threads, between barriers; bin and cum are in LDS.
template <int NT>
__device__ __forceinline__ void wg_crossing(const uint32_t* hist, int nbins, uint32_t target, uint32_t* part,
                                            uint32_t* bin, uint32_t* cum)
{
    const int tid = (int)threadIdx.x;
    const int seg = (nbins + NT - 1) / NT;
    const int lo = min(nbins, tid * seg), hi = min(nbins, (tid + 1) * seg);
    uint32_t sum = 0;
    for (int i = lo; i < hi; ++i) sum += hist[i];
    uint32_t run = wg_exclusive_sum<NT>(sum, part);
    if (run < target && run + sum >= target) {
        for (int i = lo; i < hi; ++i) {
            run += hist[i];
            if (run >= target) {
                *bin = (uint32_t)i;
                *cum = run;
                break;
            }
        }
    }
    __syncthreads();
}

// f(i, row[i]) for i in [i0, n) by the threads of a workgroup.  A row of
// counts is long (up to 262,144) and a query has one workgroup, so what counts
// is the bytes in flight: 16-byte loads (a row may start at any multiple of 4
// bytes), eight of them per thread.
template <int NT, class F>
__device__ __forceinline__ void wg_for_each_count(const int32_t* __restrict__ row, int64_t i0, int64_t n, F f)
{
    typedef int i32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
    constexpr int kUnroll = 8;
    const int tid = (int)threadIdx.x;
    int64_t b0 = i0;
    for (; b0 + 4 * kUnroll * NT <= n; b0 += 4 * kUnroll * NT) {
        i32x4_a4 v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u)
            v[u] = *reinterpret_cast<const i32x4_a4*>(row + b0 + 4 * (u * NT + tid));
#pragma unroll
        for (int u = 0; u < kUnroll; ++u)
#pragma unroll
            for (int h = 0; h < 4; ++h) f(b0 + 4 * (u * NT + tid) + h, (uint32_t)v[u][h]);
    }
    for (; b0 < n; b0 += kUnroll * NT) {
        uint32_t v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int64_t i = b0 + u * NT + tid;
            v[u] = i < n ? (uint32_t)row[i] : 0u;
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int64_t i = b0 + u * NT + tid;
            if (i < n) f(i, v[u]);
        }
    }
}

// Histogram of the counts row[0 .. n) in bins of 2^shift counts, complete up to
// the bin of the k-th smallest count: a first stretch is counted in full, and
// of the rest only what does not lie above that stretch's own k-th smallest
// (counts crowd around the mean, so counting all of them is mostly the same
// few LDS words).  hist must be zero; ends with a barrier.  part, bin, cum as
// in wg_crossing.
template <int NT>
__device__ __forceinline__ void wg_low_histogram(const int32_t* __restrict__ row, int64_t n, int32_t k, int shift,
                                                 int nbins, uint32_t* hist, uint32_t* part, uint32_t* bin,
                                                 uint32_t* cum)
{
    const int tid = (int)threadIdx.x;
    const int64_t n1 = min(n, (int64_t)max(4096, 8 * k));
    if (tid == 0) *bin = (uint32_t)nbins;
    wg_for_each_count<NT>(row, 0, n1, [&](int64_t, uint32_t v) { atomicAdd(&hist[v >> shift], 1u); });
    __syncthreads();
    if (n1 == n) return;
    wg_crossing<NT>(hist, nbins, (uint32_t)k, part, bin, cum);
    const uint32_t top = *bin;
    wg_for_each_count<NT>(row, n1, n, [&](int64_t, uint32_t v) {
        if (v >> shift <= top) atomicAdd(&hist[v >> shift], 1u);
    });
    __syncthreads();
}

// The k smallest of the n <= kSelectSlots unique keys in s (LDS), ascending.  Up
// to one key per thread, each key's place is the number of smaller ones (n
// broadcast reads and no barrier, where the sort of 2048 slots took 66); more
// are sorted.  Called by all threads after a barrier.
template <int NT>
__device__ __forceinline__ void wg_write_smallest(uint64_t* s, int n, int k, int32_t* __restrict__ cnt,
                                                  int64_t* __restrict__ idx)
{
    const int tid = (int)threadIdx.x;
    if (n > NT) {
        int p2 = 2;
        while (p2 < n) p2 <<= 1;
        for (int i = n + tid; i < p2; i += NT) s[i] = kSentinel;
        __syncthreads();
        bitonic_sort<NT>(s, p2);
        for (int j = tid; j < min(n, k); j += NT) {
            cnt[j] = (int32_t)(s[j] >> kIdxBits);
            idx[j] = (int64_t)(s[j] & kIdxMask);
        }
    } else if (tid < n) {
        const uint64_t key = s[tid];
        int place = 0;
#pragma unroll 4
        for (int j = 0; j < n; ++j) place += s[j] < key ? 1 : 0;
        if (place < k) {
            cnt[place] = (int32_t)(key >> kIdxBits);
            idx[place] = (int64_t)(key & kIdxMask);
        }
    }
    for (int j = n + tid; j < k; j += NT) {
        cnt[j] = INT32_MAX;
        idx[j] = -1;
    }
}

// LDS of a workgroup selection (one query): the bins of the histogram and the
// slots of the selected keys share their space.
template <int NT>
struct SelectLds {
    uint64_t s[kSelectSlots];
    uint32_t part[NT / 64];
    uint32_t bin, cum;
    int nb;
};
constexpr int kSelectBins = 2 * kSelectSlots;

__device__ __forceinline__ int select_shift(int32_t n_loci)
{
    int shift = 0;
    while ((n_loci >> shift) + 1 > kSelectBins) ++shift;
    return shift;
}

// Exact top-k of one row of counts; the key of column i is (row[i], idx_base +
// i).  The histogram gives the bin of the k-th smallest count; the keys up to
// it (little more than k) are gathered and put in order.
template <int NT>
__device__ inline void select_row(const int32_t* __restrict__ row, int64_t n, int32_t k, int32_t n_loci,
                                  int64_t idx_base, int32_t* __restrict__ cnt, int64_t* __restrict__ idx,
                                  SelectLds<NT>& L)
{
    const int tid = (int)threadIdx.x;
    const int shift = select_shift(n_loci), nbins = (n_loci >> shift) + 1;
    auto key_of = [&](int64_t i) { return ((uint64_t)(uint32_t)row[i] << kIdxBits) | (uint64_t)(idx_base + i); };
    uint32_t* hist = reinterpret_cast<uint32_t*>(L.s);
    uint32_t edge = (uint32_t)nbins, kept = (uint32_t)min(n, (int64_t)INT32_MAX);
    if (n > k) {
        for (int i = tid; i < nbins; i += NT) hist[i] = 0u;
        __syncthreads();
        wg_low_histogram<NT>(row, n, k, shift, nbins, hist, L.part, &L.bin, &L.cum);
        wg_crossing<NT>(hist, nbins, (uint32_t)k, L.part, &L.bin, &L.cum);
        edge = L.bin;
        kept = L.cum;
        __syncthreads();
    }
    if (kept > (uint32_t)kSelectSlots) {  // a bin of many equal counts
        wg_topk<NT>(key_of, n, k, L.s, &L.nb, (uint64_t)(edge + 1u) << (shift + kIdxBits));
        write_topk<NT>(L.s, k, cnt, idx);
        return;
    }
    if (tid == 0) L.nb = 0;
    __syncthreads();
    wg_for_each_count<NT>(row, 0, n, [&](int64_t i, uint32_t v) {
        if (v >> shift <= edge) L.s[atomicAdd(&L.nb, 1)] = ((uint64_t)v << kIdxBits) | (uint64_t)(idx_base + i);
    });
    __syncthreads();
    wg_write_smallest<NT>(L.s, (int)kept, k, cnt, idx);
}

// Exact top-k of one query from n_rsplit lists of k slots, of which only the
// first fills[w] of list w are valid.  Densely filled lists are streamed slot
// by slot with coalesced loads (unfilled slots skipped), sparse ones list by
// list, a thread each.  A histogram of the counts (bins of 2^shift counts)
// first gives the bin holding the k-th smallest count; only keys up to it can
// be in the answer, so little more than k keys are gathered and ordered.
// Called by all NT threads of a workgroup.  Bound: latency (a few hundred keys
// a query); the 2048-slot sort and two log-step prefix sums it replaces took
// 319 us for 2048 queries x 256 lists and 43 us for 131 x 2048.
template <int NT = kSelectThreads>
__device__ inline void merge_query_lists(const uint64_t* __restrict__ lists_in,
                                         const uint32_t* __restrict__ fills, int32_t n_rsplit,
                                         int32_t k, int32_t n_loci, int32_t* __restrict__ cnt,
                                         int64_t* __restrict__ idx, SelectLds<NT>& L)
{
    typedef const __attribute__((address_space(1))) uint64_t* gptr_u64;
    const gptr_u64 lists = (gptr_u64)lists_in;  // global: never aliases the LDS below
    const int tid = (int)threadIdx.x;
    uint32_t sum = 0;
    for (int w = tid; w < n_rsplit; w += NT) sum += fills[w];
    if (tid == 0) {
        L.cum = 0;
        L.nb = 0;
    }
    __syncthreads();
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += (uint32_t)__shfl_xor((int)sum, o);
    if (lane_id() == 0) atomicAdd(&L.cum, sum);
    __syncthreads();
    const int64_t total = L.cum;
    __syncthreads();
    const int64_t n_slots = (int64_t)n_rsplit * k;  // < 2^31 (n_rsplit <= 8192, k <= 1024)
    const bool dense = total * 4 >= n_slots;
    constexpr int kUnroll = 4;  // independent loads in flight per thread
    auto load_slot = [&](int64_t i) -> uint64_t {
        const int32_t w = (int32_t)i / k;
        return (uint32_t)((int32_t)i - w * k) < fills[w] ? lists[i] : kSentinel;
    };
    auto for_each_key = [&](auto take) {
        if (dense) {
            for (int64_t b0 = 0; b0 < n_slots; b0 += kUnroll * NT) {
                uint64_t key[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    const int64_t i = b0 + u * NT + tid;
                    key[u] = i < n_slots ? load_slot(i) : kSentinel;
                }
#pragma unroll
                for (int u = 0; u < kUnroll; ++u)
                    if (key[u] != kSentinel) take(key[u]);
            }
        } else {
            for (int w = tid; w < n_rsplit; w += NT) {
                const uint32_t f = fills[w];
                const gptr_u64 list = lists + (size_t)w * k;
                for (uint32_t e = 0; e < f; ++e) take(list[e]);
            }
        }
    };
    const int shift = select_shift(n_loci), nbins = (n_loci >> shift) + 1;
    uint32_t edge = 0xFFFFFFFFu;
    int64_t kept = total;
    if (total > k) {
        uint32_t* hist = reinterpret_cast<uint32_t*>(L.s);
        for (int i = tid; i < nbins; i += NT) hist[i] = 0u;
        __syncthreads();
        for_each_key([&](uint64_t key) {
            atomicAdd(&hist[min((uint32_t)(key >> kIdxBits) >> shift, (uint32_t)(nbins - 1))], 1u);
        });
        __syncthreads();
        wg_crossing<NT>(hist, nbins, (uint32_t)k, L.part, &L.bin, &L.cum);
        edge = L.bin;
        kept = L.cum;
        __syncthreads();
    }
    if (kept > kSelectSlots) {  // a bin of many equal counts
        wg_topk<NT>(load_slot, n_slots, k, L.s, &L.nb, (uint64_t)(edge + 1u) << (shift + kIdxBits));
        write_topk<NT>(L.s, k, cnt, idx);
        return;
    }
    for_each_key([&](uint64_t key) {
        if ((uint32_t)(key >> kIdxBits) >> shift <= edge) L.s[atomicAdd(&L.nb, 1)] = key;
    });
    __syncthreads();
    wg_write_smallest<NT>(L.s, (int)kept, k, cnt, idx);
}

}  // namespace fid

// libfastid: the int8 matrix-core formulation of the overloaded product.
//
// For 0/1 profiles the Eq. 1 count has a closed form in the ordinary dot
// product D[q][r] = sum_k Q_k R_k (an exact int32 sum of 0/1 int8 products):
//   mixture : popcount(R & ~Q) = popcount(R) - D
//   identity: popcount(R ^ Q)  = popcount(R) + popcount(Q) - 2 D
// so the all-pairs comparison becomes a dense int8 GEMM on the MFMA units
// (v_mfma_i32_32x32x32_i8), with the reference bits expanded to bytes in
// registers and the query tile held as bytes in LDS.
//
// Workgroup = 8 waves (2 per SIMD) sharing one 64-query tile held in LDS as
// bytes for the kernel's whole lifetime (rows padded by 16 bytes so the 32
// rows a wave reads at one column hit distinct banks); each wave streams its
// own 128 references (4 MFMA column blocks) against both 32-query row
// blocks: 8 accumulators of 32x32 int32 per wave.  Per 32-locus step a lane
// expands 4 x 16 reference bits (3 VALU ops per 4 loci) and issues 8 MFMAs;
// the next 128-locus unit of reference bits is prefetched.
#include <type_traits>

#include "fid_device.hpp"

namespace fid {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

namespace {

constexpr int kWavesM = 8;
constexpr int kWGM = kWavesM * kWave;
constexpr int kQB = 64;                 // queries per workgroup tile
constexpr int kNBW = 4;                 // 32-reference column blocks per wave
constexpr int kRefsPerWave = 32 * kNBW;
constexpr int kRefsPerWG = kRefsPerWave * kWavesM;
static_assert(kDbTileRefs % kRefsPerWG == 0, "tiles must not cross the database padding granule");
constexpr int kMaxKpad = 2304;          // 64 x (2304 + 16) B of query tile fits the 160 KiB LDS

// 16 bits of w starting at bit sh -> 16 bytes of 0/1: a nibble x times
// 0x204081 puts bit i at bit 8i of the product (the four shifted copies do not
// overlap, so there are no carries).  3 VALU ops per 4 loci.
__device__ __forceinline__ v4i expand16(uint32_t w, uint32_t sh)
{
    v4i r;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        r[j] = (int)((__builtin_amdgcn_ubfe(w, sh + 4u * j, 4u) * 0x204081u) & 0x01010101u);
    return r;
}

// Workgroups are dealt to the 8 XCDs round-robin; renumber them so that the
// workgroups resident on one XCD at a time are consecutive, i.e. share a
// reference range and hit in that XCD's L2.
__device__ __forceinline__ int xcd_local_index(int wg, int n_wg)
{
    const int x = wg & 7, s = wg >> 3;
    const int per = n_wg >> 3, rem = n_wg & 7;
    return x < rem ? x * (per + 1) + s : rem * (per + 1) + (x - rem) * per + s;
}

typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef __attribute__((address_space(1))) uint64_t glb_u64;
typedef __attribute__((address_space(1))) uint32_t glb_u32;

// Insert the candidates of one ballot into the wave's lists (entry i of a
// list is only touched by lane i & 63).  Candidates arrive in no particular
// index order, so the decision compares full (count, index) keys, and the
// filter bound of a full list is its worst count plus one (an equal count
// may still win on index).  The address spaces are explicit: this out-of-line
// helper would otherwise reach the LDS bounds and the global lists through
// flat accesses.
__device__ __noinline__ void mfma_insert(uint64_t mask, uint32_t c, int64_t r, int m,
                                         glb_u64* __restrict__ lists, int64_t qstride, int k,
                                         lds_u32* lthr, lds_u32* lfill)
{
    const int lane = lane_id();
    while (mask) {
        // src is wave-uniform: the candidate's fields are read straight from its lane
        const int src = __builtin_ctzll(mask);
        mask &= mask - 1;
        const int ms = __builtin_amdgcn_readlane(m, src);
        const uint32_t cs = (uint32_t)__builtin_amdgcn_readlane((int)c, src);
        const uint32_t rlo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)r, src);
        const uint32_t rhi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)r >> 32), src);
        uint32_t t = lthr[ms];
        if (cs >= t) continue;
        const uint64_t key = ((uint64_t)cs << kIdxBits) | ((uint64_t)rhi << 32) | rlo;
        glb_u64* list = lists + (size_t)ms * qstride;
        uint32_t fill = lfill[ms];
        uint64_t mx;
        int mpos;
        bool changed = false;
        if (fill < (uint32_t)k) {
            if (lane == (int)(fill & 63u)) list[fill] = key;
            ++fill;
            changed = fill == (uint32_t)k;
        } else {
            list_max(list, k, mx, mpos);
            if (key < mx) {
                if (lane == (mpos & 63)) list[mpos] = key;
                changed = true;
            }
        }
        if (changed) {
            list_max(list, k, mx, mpos);
            const uint32_t bound = (uint32_t)(mx >> kIdxBits) + 1u;
            if (bound < t) t = bound;
        }
        if (lane == 0) {
            lthr[ms] = t;
            lfill[ms] = fill;
        }
        wave_lds_sync();
    }
}

__device__ __noinline__ void mfma_append_hits(uint64_t mask, bool hit, int32_t c, int64_t r, int q,
                                              unsigned long long* __restrict__ hit_count,
                                              uint64_t* __restrict__ hit_keys,
                                              int32_t* __restrict__ hit_cnt, int64_t cap)
{
    const int lane = lane_id();
    const int first = __builtin_ctzll(mask);
    unsigned long long base = 0;
    if (lane == first) base = atomicAdd(hit_count, (unsigned long long)__popcll(mask));
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)base, first);
    const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(base >> 32), first);
    base = ((unsigned long long)hi << 32) | lo;
    if (hit) {
        const unsigned long long pos =
            base + (unsigned long long)__popcll(mask & ((1ull << lane) - 1ull));
        if (pos < (unsigned long long)cap) {
            hit_keys[pos] = ((uint64_t)q << kIdxBits) | (uint64_t)r;
            hit_cnt[pos] = c;
        }
    }
}

// Candidates of one fp4 tile epilogue wait in a per-wave LDS queue of
// kCandQ4 entries.  An entry packs tile query m (7 bits), reference 0..63 of
// the wave's block (6 bits) and the count (at most 65535, 16 bits):
// m | ref << 7 | c << 13.
constexpr int kCandQ4 = 64;

// Drain the queue of n <= 64 entries into the wave's top-k lists.  Every lane
// takes one entry, so the bound, fill and witness lookups of all candidates
// happen at once.  The entries of one query below its bound are appended at
// the next free slots, all queries at once; a list that fills takes its entries
// one by one, since its new bound needs the list's worst key.  Witness counts
// (every queued candidate, under the lowest level that it is below: each is a
// distinct reference of its query, as the scan meets a pair once) go to the
// workgroup's LDS counters wloc, which the waves add to the global ones now
// and then.  Inlined where nothing of the
// tile but the candidate test's operands is live: an out-of-line call waits
// for every memory operation of the wave on entry and on return, the next
// tile's prefetch and its own list stores included.
__device__ __forceinline__ void fp4_drain_lists(const lds_u32* cq, int n, int64_t rbase,
                                                glb_u64* __restrict__ lists, int64_t qstride, int k, lds_u32* lthr,
                                                lds_u32* lfill, const lds_u32* tlvl, lds_u32* wloc)
{
    const int lane = lane_id();
    const bool act = lane < n;
    const uint32_t v = act ? cq[lane] : 0u;
    const int m = (int)(v & 127u);
    const uint32_t c = v >> 13;
    const uint64_t key = ((uint64_t)c << kIdxBits) | (uint64_t)(rbase + ((v >> 7) & 63u));
    const uint32_t t0 = act ? lthr[m] : 0u;
    const uint32_t f0 = act ? lfill[m] : 0u;
    if (wloc && act) {
        // the levels fall, so the count is below the first `under` of them;
        // the lowest of these is worth a count while it would lower the bound
        int under = 0;
        uint32_t lowest = t0;
#pragma unroll
        for (int l = 0; l < kWitLevels; ++l) {
            const uint32_t level = tlvl[kWitLevels * m + l];
            under += c < level;
            lowest = c < level ? level : lowest;
        }
        if (lowest < t0)
            __hip_atomic_fetch_add(wloc + kWitLevels * m + under - 1, 1u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    const bool keep = act && c < t0;
    // no list can fill up: every entry takes its query's next slot
    if (!__builtin_amdgcn_ballot_w64(keep && f0 + (uint32_t)n >= (uint32_t)k)) {
        if (keep) {
            const uint32_t slot =
                __hip_atomic_fetch_add(lfill + m, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            lists[(int64_t)m * qstride + slot] = key;
        }
        wave_lds_sync();
        return;
    }
    uint64_t rem = __builtin_amdgcn_ballot_w64(keep);
    while (rem) {
        const int lead = __builtin_ctzll(rem);
        const int ms = __builtin_amdgcn_readlane(m, lead);
        const bool mine = keep && m == ms;
        uint64_t sel = __builtin_amdgcn_ballot_w64(mine);
        rem &= ~sel;
        const uint32_t nsel = (uint32_t)__popcll(sel);
        uint32_t t = (uint32_t)__builtin_amdgcn_readlane((int)t0, lead);
        uint32_t fill = (uint32_t)__builtin_amdgcn_readlane((int)f0, lead);
        glb_u64* list = lists + (size_t)ms * qstride;
        if (fill + nsel < (uint32_t)k) {
            // appends only: every entry is below the bound, which stays put
            if (mine)
                list[fill + (uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(sel >> 32),
                                                                __builtin_amdgcn_mbcnt_lo((uint32_t)sel, 0u))] = key;
            fill += nsel;
        } else {
            while (sel) {
                const int src = __builtin_ctzll(sel);
                sel &= sel - 1;
                const uint32_t cs = (uint32_t)__builtin_amdgcn_readlane((int)c, src);
                if (cs >= t) continue;
                const uint64_t ks =
                    ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(key >> 32), src) << 32) |
                    (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)key, src);
                uint64_t mx;
                int mpos;
                uint32_t at = fill;
                if (fill == (uint32_t)k) {
                    wave_lds_sync();  // (orders this wave's list stores before its loads)
                    list_max(list, k, mx, mpos);
                    if (ks >= mx) continue;
                    at = (uint32_t)mpos;
                } else {
                    ++fill;
                }
                if (lane == (int)(at & 63u)) list[at] = ks;
                if (fill == (uint32_t)k) {
                    wave_lds_sync();
                    list_max(list, k, mx, mpos);
                    const uint32_t bound = (uint32_t)(mx >> kIdxBits) + 1u;
                    if (bound < t) t = bound;
                }
            }
        }
        if (lane == 0) {
            lthr[ms] = t;
            lfill[ms] = fill;
        }
    }
    wave_lds_sync();
}

// Append the queued references whose count is below the threshold + 1 (tthr)
// of their query to the threshold hits: one atomic per drain.
__device__ __forceinline__ void fp4_drain_hits(const lds_u32* cq, int n, int64_t rbase, int q0, const lds_u32* tthr,
                                               unsigned long long* __restrict__ hit_count,
                                               uint64_t* __restrict__ hit_keys, int32_t* __restrict__ hit_cnt,
                                               int64_t cap)
{
    const int lane = lane_id();
    const bool act = lane < n;
    const uint32_t v = act ? cq[lane] : 0u;
    const int m = (int)(v & 127u);
    const uint32_t c = v >> 13;
    const bool hit = act && c < tthr[m];
    const uint64_t hm = __builtin_amdgcn_ballot_w64(hit);
    if (!hm) return;
    unsigned long long first = 0;
    if (lane == 0) first = atomicAdd(hit_count, (unsigned long long)__popcll(hm));
    first = ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(first >> 32)) << 32) |
            (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)first);
    const unsigned long long pos = first + (unsigned long long)__popcll(hm & ((1ull << lane) - 1ull));
    if (hit && pos < (unsigned long long)cap) {
        hit_keys[pos] = ((uint64_t)(q0 + m) << kIdxBits) | (uint64_t)(rbase + ((v >> 7) & 63u));
        hit_cnt[pos] = (int32_t)c;
    }
}

}  // namespace

// LDS layout: [query tile 64 x (kpad + 16)] [per-wave bound 8 x 64] [per-wave
// fill 8 x 64] [tile query popcounts 64] [tile thresholds 64].
template <int MODE, int EPI>
__global__ __launch_bounds__(kWGM) void mfma_scan_kernel(
    const ScanParams p, const uint8_t* __restrict__ qx, int32_t kpad,
    const int32_t* __restrict__ pcq, int32_t* __restrict__ out, uint64_t* __restrict__ lists,
    uint32_t* __restrict__ fills, const uint32_t* __restrict__ thr_init,
    const int32_t* __restrict__ thr, unsigned long long* __restrict__ hit_count,
    uint64_t* __restrict__ hit_keys, int32_t* __restrict__ hit_cnt)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int row_bytes = kpad + 16;
    uint8_t* qt = smem;
    uint32_t* lthr_all = reinterpret_cast<uint32_t*>(smem + kQB * row_bytes);
    uint32_t* lfill_all = lthr_all + kWavesM * kQB;
    int32_t* tpcq = reinterpret_cast<int32_t*>(lfill_all + kWavesM * kQB);
    int32_t* tthr = tpcq + kQB;

    const int lane = lane_id();
    const int tid = (int)threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int g = lane >> 5;       // MFMA k half
    const int n32 = lane & 31;     // MFMA row / column within a 32-block

    // Workgroup -> (query tile, reference range).
    const int n_qtiles = (p.q_hi - p.q_lo + kQB - 1) / kQB;
    const int wg = xcd_local_index((int)blockIdx.x, (int)gridDim.x);
    const int qt_idx = wg % n_qtiles;
    const int wr_g = wg / n_qtiles;
    const int q0 = p.q_lo + qt_idx * kQB;
    const int nq_tile = min(kQB, p.q_hi - q0);
    const int64_t base = (p.r_lo / kDbTileRefs) * kDbTileRefs;
    const int64_t ntiles = (p.r_hi - base + kRefsPerWG - 1) / kRefsPerWG;
    const int64_t tb = (ntiles * wr_g) / p.n_rsplit;
    const int64_t te = (ntiles * (wr_g + 1)) / p.n_rsplit;
    const int worker = wr_g * kWavesM + wv;  // list owner along references
    const int n_workers_r = p.n_rsplit * kWavesM;

    // Resident query tile (bytes) and per-query side data.
    const int vec_per_row = kpad / 16;
    for (int i = tid; i < kQB * vec_per_row; i += kWGM) {
        const int row = i / vec_per_row;
        const int col = (i - row * vec_per_row) * 16;
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (row < nq_tile) v = *reinterpret_cast<const uint4*>(qx + (size_t)(q0 + row) * kpad + col);
        *reinterpret_cast<uint4*>(qt + row * row_bytes + col) = v;
    }
    if (tid < kQB) {
        tpcq[tid] = (MODE == FID_MODE_IDENTITY && tid < nq_tile) ? pcq[q0 + tid] : 0;
        tthr[tid] = (EPI == EPI_THRESH && tid < nq_tile) ? thr[q0 + tid] : -1;
    }
    uint32_t* lthr = lthr_all + wv * kQB;
    uint32_t* lfill = lfill_all + wv * kQB;
    if constexpr (EPI == EPI_TOPK) {
        for (int i = lane; i < kQB; i += 64) {
            lthr[i] = i < nq_tile ? thr_init[q0 + i] : 0u;
            lfill[i] = 0u;
        }
    }
    __syncthreads();

    const int nunits = kpad / 128;
    const int w4 = p.db.w4;
    const uint8_t* arow0 = qt + n32 * row_bytes + g * 16;
    const uint8_t* arow1 = qt + (32 + n32) * row_bytes + g * 16;
    for (int64_t tile = tb; tile < te; ++tile) {
        const int64_t rbase = base + tile * kRefsPerWG + (int64_t)wv * kRefsPerWave;
        // Reference words: one uniform base per tile plus a 32-bit lane
        // offset; the database is padded to whole tiles, so every load is
        // unconditional (references past r_hi are never read by the epilogue).
        const char* tbase = reinterpret_cast<const char*>(p.db.words) + (size_t)(rbase >> 6) * w4 * 1024;
        const uint32_t loff = (uint32_t)n32 * 16u;
        auto load_unit = [&](uint4 (&dst)[kNBW], int u) {
#pragma unroll
            for (int j = 0; j < kNBW; ++j)
                dst[j] = *reinterpret_cast<const uint4*>(
                    tbase + ((size_t)(j >> 1) * w4 * 64 + 32 * (j & 1)) * 16 + (size_t)u * 1024 + loff);
        };
        v16i acc[2][kNBW];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int j = 0; j < kNBW; ++j) acc[a][j] = v16i{0};

        // One 16-byte unit (128 loci) of each reference feeds 4 MFMA steps.
        auto step_unit = [&](const uint4 (&bits)[kNBW], int u) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int kofs = u * 128 + s * 32;
                const v4i a0 = *reinterpret_cast<const v4i*>(arow0 + kofs);
                const v4i a1 = *reinterpret_cast<const v4i*>(arow1 + kofs);
#pragma unroll
                for (int j = 0; j < kNBW; ++j) {
                    const uint32_t w = s == 0 ? bits[j].x : s == 1 ? bits[j].y : s == 2 ? bits[j].z : bits[j].w;
                    const v4i b = expand16(w, 16u * (uint32_t)g);
                    acc[0][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a0, b, acc[0][j], 0, 0, 0);
                    acc[1][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1, b, acc[1][j], 0, 0, 0);
                }
            }
        };
        uint4 ba[kNBW], bb[kNBW];
        load_unit(ba, 0);
#pragma unroll 1
        for (int u = 0; u < nunits; u += 2) {
            load_unit(bb, u + 1);
            step_unit(ba, u);
            load_unit(ba, u + 2);  // last pass: up to two units past the row, never used
            step_unit(bb, u + 1);
        }

        // ---- epilogue: lane holds reference rbase + 32 j + n32 and, in
        // register i of block a, tile query m = 32 a + (i & 3) + 8 (i >> 2) + 4 g.
#pragma unroll
        for (int j = 0; j < kNBW; ++j) {
            const int64_t r = rbase + 32 * j + n32;
            const bool rin = r >= p.r_lo && r < p.r_hi;
            const int32_t pr = rin ? p.db.pc[r] : 0;
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                int32_t cv[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int m = 32 * a + (i & 3) + 8 * (i >> 2) + 4 * g;
                    const int32_t d = acc[a][j][i];
                    cv[i] = MODE == FID_MODE_MIXTURE ? pr - d : pr + tpcq[m] - 2 * d;
                }
                if constexpr (EPI == EPI_FULL) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int m = 32 * a + (i & 3) + 8 * (i >> 2) + 4 * g;
                        if (rin && m < nq_tile)
                            out[(size_t)(q0 + m - p.out_q_base) * p.ld + (r - p.out_r_base)] = cv[i];
                    }
                } else if constexpr (EPI == EPI_TOPK) {
                    bool any = false;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int m = 32 * a + (i & 3) + 8 * (i >> 2) + 4 * g;
                        any |= (uint32_t)cv[i] < lthr[m];
                    }
                    if (__builtin_amdgcn_ballot_w64(any && rin)) {
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            const int m = 32 * a + (i & 3) + 8 * (i >> 2) + 4 * g;
                            const bool cand = rin && (uint32_t)cv[i] < lthr[m];
                            const uint64_t bm = __builtin_amdgcn_ballot_w64(cand);
                            if (bm)
                                mfma_insert(bm, (uint32_t)cv[i], r, m,
                                            (glb_u64*)(lists + ((size_t)q0 * n_workers_r + worker) * p.k),
                                            (int64_t)n_workers_r * p.k, p.k, (lds_u32*)lthr, (lds_u32*)lfill);
                        }
                    }
                } else {
                    bool any = false;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int m = 32 * a + (i & 3) + 8 * (i >> 2) + 4 * g;
                        any |= cv[i] <= tthr[m];
                    }
                    if (__builtin_amdgcn_ballot_w64(any && rin)) {
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            const int m = 32 * a + (i & 3) + 8 * (i >> 2) + 4 * g;
                            const bool hit = rin && cv[i] <= tthr[m];
                            const uint64_t bm = __builtin_amdgcn_ballot_w64(hit);
                            if (bm)
                                mfma_append_hits(bm, hit, cv[i], r, q0 + m, hit_count, hit_keys,
                                                 hit_cnt, p.hit_cap);
                        }
                    }
                }
            }
        }
    }
    if constexpr (EPI == EPI_TOPK) {
        wave_lds_sync();
        for (int i = lane; i < nq_tile; i += 64)
            fills[(size_t)(q0 + i) * n_workers_r + worker] = lfill[i];
    }
}

// Expanded queries for the matrix-core path: byte k of row q = locus k of
// query q (0/1), zero padded to kpad; plus popcount(Q_q) for identity mode.
__global__ void expand_queries_kernel(const uint64_t* __restrict__ q, int32_t n_q,
                                      int32_t row_words, int32_t n_loci, uint8_t* __restrict__ qx,
                                      int32_t kpad, int32_t* __restrict__ pcq)
{
    const int64_t total = (int64_t)n_q * (kpad / 4);
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = t / (kpad / 4);
        const int32_t k0 = (int32_t)(t - i * (kpad / 4)) * 4;
        uint32_t v = 0;
        if (k0 < n_loci) {
            const uint64_t w = q[i * row_words + (k0 >> 6)];
            uint32_t nib = (uint32_t)(w >> (k0 & 63)) & 0xFu;
            if (k0 + 4 > n_loci) nib &= (1u << (n_loci - k0)) - 1u;
            v = (nib * 0x204081u) & 0x01010101u;
        }
        reinterpret_cast<uint32_t*>(qx + i * kpad)[k0 >> 2] = v;
    }
    // popcounts: one thread per query
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_q;
         i += (int64_t)gridDim.x * blockDim.x) {
        int32_t s = 0;
        const int32_t full = n_loci >> 6;
        for (int32_t w = 0; w < full; ++w) s += __popcll(q[i * row_words + w]);
        if (n_loci & 63) s += __popcll(q[i * row_words + full] & ((1ull << (n_loci & 63)) - 1ull));
        pcq[i] = s;
    }
}

hipError_t launch_expand_queries(const uint64_t* q, int32_t n_q, int32_t row_words,
                                 int32_t n_loci, uint8_t* qx, int32_t kpad, int32_t* pcq,
                                 hipStream_t s)
{
    const int64_t total = (int64_t)n_q * (kpad / 4);
    int64_t blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(expand_queries_kernel, dim3((unsigned)blocks), dim3(256), 0, s, q, n_q,
                       row_words, n_loci, qx, kpad, pcq);
    return hipGetLastError();
}

// Loci padded to whole pairs of 128-locus units (the unit loop is unrolled by
// two); the padding is zero on the query side, so whatever the reference
// side holds there adds nothing.
int mfma_kpad(int32_t n_loci) { return ((n_loci + 255) / 256) * 256; }
int mfma_max_loci() { return kMaxKpad; }
int mfma_refs_per_wg() { return kRefsPerWG; }
int mfma_queries_per_wg() { return kQB; }
int mfma_waves_per_wg() { return kWavesM; }

static size_t mfma_lds_bytes(int32_t kpad)
{
    return (size_t)kQB * (kpad + 16) + 2 * (size_t)kWavesM * kQB * 4 + 2 * (size_t)kQB * 4;
}

template <int MODE, int EPI>
static hipError_t launch_mfma_t(const ScanParams& p, const MfmaBuffers& b, hipStream_t s)
{
    if (b.kpad > kMaxKpad) return hipErrorInvalidValue;
    const int n_qtiles = (p.q_hi - p.q_lo + kQB - 1) / kQB;
    const int64_t blocks = (int64_t)n_qtiles * p.n_rsplit;
    const size_t lds = mfma_lds_bytes(b.kpad);
    const hipError_t e = lds_opt_in<&mfma_scan_kernel<MODE, EPI>>((int)mfma_lds_bytes(kMaxKpad));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((mfma_scan_kernel<MODE, EPI>), dim3((unsigned)blocks), dim3(kWGM), lds, s,
                       p, b.qx, b.kpad, b.pcq, b.out, b.lists, b.fills, b.thr_init, b.thr,
                       b.hit_count, b.hit_keys, b.hit_cnt);
    return hipGetLastError();
}

hipError_t launch_mfma_scan(int mode, int epi, const ScanParams& p, const MfmaBuffers& b,
                            hipStream_t s)
{
    if (p.n_rsplit <= 0) return hipSuccess;
    if (mode == kModePerQuery) return hipErrorInvalidValue;  // per-query modes: fp4 or popcount
    if (mode == FID_MODE_MIXTURE) {
        if (epi == EPI_FULL) return launch_mfma_t<FID_MODE_MIXTURE, EPI_FULL>(p, b, s);
        if (epi == EPI_TOPK) return launch_mfma_t<FID_MODE_MIXTURE, EPI_TOPK>(p, b, s);
        return launch_mfma_t<FID_MODE_MIXTURE, EPI_THRESH>(p, b, s);
    }
    if (epi == EPI_FULL) return launch_mfma_t<FID_MODE_IDENTITY, EPI_FULL>(p, b, s);
    if (epi == EPI_TOPK) return launch_mfma_t<FID_MODE_IDENTITY, EPI_TOPK>(p, b, s);
    return launch_mfma_t<FID_MODE_IDENTITY, EPI_THRESH>(p, b, s);
}

// ======================================================================
// fp4 (e2m1) matrix-core variant: v_mfma_f32_16x16x128_f8f6f4 with both
// operands in e2m1 and the fp32 accumulation of at most 65536 products of 1
// (or of 2), which is exact.  It runs at twice the MAC rate of the int8 kernel.
//
// With identity queries' codes doubled (mul = 2, else 1), the accumulators
// start at -|R| and a sum x = mul D - |R| = tpcq - count, with tpcq = |Q| for
// identity queries and 0 for mixtures.  "count < bound" is x > tpcq - bound: one
// starting value per reference and one cut per query, and every instance
// serves both modes, one or per query.  (Products of -1 would count without
// the starting value, from codes that are -1 where Q is 0; but the sums of
// negative products cost so much power that the clock falls from 2.3 to
// 2.05 GHz: 2048 x 20M x 2048 25.3 ms against 22 ms.)
//
// Element order and values: a dot product does not depend on the order of k
// as long as both operands use the same one.  Each 32-locus word w of a
// reference is spread into 4 dwords, dword d holding locus 4j + d in nibble
// j.  A set bit need not be 1.0 on both sides, only the product of the two
// codes must be: the reference keeps loci 4j, 4j+1, 4j+2 where they are (e2m1
// 0x1 = 0.5, 0x2 = 1.0, 0x4 = 2.0: dword d = w & (0x11111111 << d)) and moves
// locus 4j+3 down one bit (2.0), 5 VALU ops per 32 loci; the queries, staged
// once, carry the reciprocals (2.0, 1.0, 0.5, 0.5) or twice those.  The k
// index of an MFMA is permuted further so that each lane loads whole 16-byte
// units: within a group of 4 units (512 loci), lane group kg (k quarter of
// the MFMA operand) holds unit 4g + kg and feeds its word t to step t, so one
// dwordx4 load per lane and 16-reference block covers 4 MFMA steps.
//
// Workgroup = 8 waves sharing a query tile of NA 16-query blocks (NA <= 8) in
// LDS.  Each wave computes them against its own 64-reference database block:
// NA x 4 blocks of 16 x 16 accumulators with the references along the rows,
// so a lane holds 4 consecutive references of one query per block (16-byte
// stores of full counts, one bound per lane and query block).
namespace {

constexpr int kQB4 = 128;               // most queries per workgroup (and per wave)
constexpr int kNB4 = 4;                 // 16-reference blocks per wave
constexpr int kRefsPerWave4 = 16 * kNB4;
constexpr int kRefsPerWG4 = kRefsPerWave4 * kWavesM;
constexpr int kUnitsPerGroup4 = 4;      // 16-byte units per load group
constexpr int kHalfLoci4 = 1024;        // loci of the query tile in one of the two LDS halves
constexpr int kHalfRow4 = kHalfLoci4 / 2;           // staged bytes of a row in a half
constexpr int kPlane4 = kQB4 * kHalfRow4 / 4;       // one k quarter of a half: 128 rows x 128 bytes
constexpr int kHalfBytes4 = 4 * kPlane4;            // 64 KiB
constexpr int kMaxKpad4 = 65536;
constexpr int kRing4 = 2;               // query blocks read from LDS ahead of their MFMAs
constexpr int kWaitVm0 = 0x0F70;        // s_waitcnt vmcnt(0), other counters untouched
constexpr int kWaitVm4 = 0x0F74;        // s_waitcnt vmcnt(4): all but the newest four
static_assert(kUnitsPerGroup4 % kRing4 == 0, "the ring of query blocks restarts with every group");
static_assert(kNB4 == 4, "kWaitVm4 leaves one group's loads in flight");
static_assert(kRefsPerWave4 == 64, "a wave covers exactly one database block");
static_assert(kDbTileRefs % kRefsPerWG4 == 0, "tiles must not cross the database padding granule");

typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
// four counts of a row at any 4-byte aligned address
typedef int v4i_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef __attribute__((address_space(3))) v4u lds_v4u;

__device__ __forceinline__ v8i spread_fp4(uint32_t w)
{
    v8i r;
    r[0] = (int)(w & 0x11111111u);          // locus 4j     -> 0.5
    r[1] = (int)(w & 0x22222222u);          // locus 4j + 1 -> 1.0
    r[2] = (int)(w & 0x44444444u);          // locus 4j + 2 -> 2.0
    r[3] = (int)((w >> 1) & 0x44444444u);   // locus 4j + 3 -> 2.0
    r[4] = 0;
    r[5] = 0;
    r[6] = 0;
    r[7] = 0;
    return r;
}

__device__ __forceinline__ uint32_t word_of(const uint4& v, int t)
{
    return t == 0 ? v.x : t == 1 ? v.y : t == 2 ? v.z : v.w;
}

// Query tiles: the 16-query blocks of [0, n_q) dealt evenly to a launch's
// tiles (ceil(n_q / 128) of them, more over a short range), so that 131 queries
// run as tiles of 5 and 4 blocks and not as 8 and 1 (whose references are read,
// spread and checked for 3 queries).
__host__ __device__ inline int fp4_tile_blocks(int n_q) { return (n_q + 15) / 16; }
__host__ __device__ inline int fp4_tile_begin(int n_q, int n_tiles, int t)
{
    return 16 * (int)((int64_t)fp4_tile_blocks(n_q) * t / n_tiles);
}

}  // namespace

// One work item of the fp4 scan (see fp4_work).
struct Fp4Work {
    DbView db;
    int64_t r_lo, r_hi;            // the query set's reference range (others are masked)
    int64_t base;                  // r_lo rounded down to a database tile
    int64_t tb, te;                // 512-reference tiles [tb, te) from base
    const uint8_t* qx;             // staged queries of the set, row q at qx + q * kpad / 2
    int32_t kpad;
    const int32_t* pcq;            // |Q| per query of the set
    int mode;                      // fid_mode of every query, or kModePerQuery
    const int32_t* qmode;          // per-query fid_mode (kModePerQuery)
    int32_t q0, nq_tile;           // query tile of the set
    int32_t slot, n_slots;         // this item's reference range among the set's ranges
    int32_t k;
    int32_t* out;                  // EPI_FULL: out[(q - out_q_base) * ld + (r - out_r_base)]
    int64_t ld;
    int32_t out_q_base;
    int64_t out_r_base;
    uint64_t* lists;               // top-k lists [q][n_slots * waves][k], fills [q][n_slots * waves]
    uint32_t* fills;
    const uint32_t* thr_init;      // per-query starting bound, witness levels and counters
    const uint32_t* level;
    uint32_t* wit;
    const int32_t* thr;            // threshold hits
    unsigned long long* hit_count;
    uint64_t* hit_keys;
    int32_t* hit_cnt;
    int64_t hit_cap;
};

// A wave-uniform value in scalar registers (the persistent kernel reads its
// items between assembly that may write memory, so its loads are vector loads).
__device__ __forceinline__ int32_t uni(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uni(int64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
template <class T>
__device__ __forceinline__ T* uni(T* p)
{
    return reinterpret_cast<T*>(uni((int64_t)reinterpret_cast<uintptr_t>(p)));
}

// A wave's DMA instruction: 64 lanes x `16 bytes` (or 4) from base + off into
// LDS at the wave-uniform byte address lds.  Written as assembly because the
// compiler makes every LDS read that follows the builtin wait for all loads
// in flight; here the LDS halves alternate, and the wait (vmcnt 0, before the
// workgroup barrier that hands a half over) is the caller's.  No vector
// register is written, and a wait the compiler places for its own loads can
// only get stricter by loads it does not know of.  The s_nop stands for two
// hazards that the hardware leaves to the program, and that the compiler does
// not look for inside assembly: one wait state from the write of m0 to a load
// into LDS, and five from a VALU write of a scalar register (the base comes
// from v_readfirstlane) to a vector memory instruction that reads it.
__device__ __forceinline__ void dma16(uint32_t lds, const void* base, uint32_t off)
{
    __asm__ volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2"
                     :
                     : "s"(uni((int32_t)lds)), "v"(off), "s"(uni(base))
                     : "memory");
}
__device__ __forceinline__ void dma4(uint32_t lds, const void* base, uint32_t off)
{
    __asm__ volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dword %1, %2"
                     :
                     : "s"(uni((int32_t)lds)), "v"(off), "s"(uni(base))
                     : "memory");
}

// Stage half row hh (loci [1024 hh, 1024 hh + 1024)) of the tile's 16 NA rows
// into the LDS half at byte address half: NA instructions per wave.  A half
// is four planes, one per k quarter, of 128-byte rows whose eight 16-byte
// words (two groups x four steps) are permuted by the row (word c at c ^
// (row / 2 mod 8)): the 16 lanes that an LDS read serves at a time then meet
// all 64 banks.  Rows past the tile's queries repeat its last query; their
// bounds admit nothing.
template <int NA>
__device__ __forceinline__ void fp4_stage_half(const Fp4Work& w, int wv, int lane, int hh, uint32_t half)
{
    const int qrow = w.kpad / 2;
    const uint8_t* base = w.qx + (size_t)w.q0 * qrow + (size_t)hh * kHalfRow4;
    // opaque: the addresses are recomputed (four ops each), not held or
    // spilled across the scan loop
    int l = lane;
    __asm__ volatile("" : "+v"(l));
    const int row0 = l >> 3;
    const uint32_t word0 = (uint32_t)((l & 7) ^ (l >> 4)) * 16u;
#pragma unroll
    for (int s = 0; s < NA; ++s) {
        const int idx = wv * NA + s;          // (plane, 8-row block)
        const int kg = idx / (2 * NA), rb = idx % (2 * NA);
        const uint32_t row = (uint32_t)min(rb * 8 + row0, w.nq_tile - 1);
        dma16(half + (uint32_t)(kg * kPlane4 + rb * 1024), base + kg * 128,
              __umul24(row, (uint32_t)qrow) + (word0 ^ ((uint32_t)(rb & 1) << 6)));
    }
}

// Witness counts gathered in LDS since the last flush go to the global
// counters: wave wv takes an eighth of the tile's (query, level) counters,
// swapping each with zero (other waves may be adding to it meanwhile).
__device__ __forceinline__ void fp4_flush_witness(uint32_t* wloc, uint32_t* __restrict__ wit_tile, int n, int wv,
                                                  int lane)
{
    constexpr int kPer = kWitLevels * kQB4 / kWavesM;
#pragma unroll
    for (int h = 0; h < (kPer + 63) / 64; ++h) {
        const int i = kPer * wv + 64 * h + lane;
        if (64 * h + lane < kPer && i < n) {
            const uint32_t cnt = __hip_atomic_exchange((lds_u32*)(wloc + i), 0u, __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            if (cnt) __hip_atomic_fetch_add(wit_tile + i, cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// LDS: [query tile: 2 halves] [bound 8 x 128] [fill 8 x 128]
// [reference popcounts of this and the next tile 8 x 2 x 64] [tile popcounts 128]
// [tile thresholds 128] [witness levels 128 x kWitLevels]
// [staged witness counts 128 x kWitLevels, shared by the waves]
// [candidate queues 8 x kCandQ4]
// [witness counts not yet flushed 128 x kWitLevels].
constexpr size_t kLdsFp4 = 2 * (size_t)kHalfBytes4 + 3 * (size_t)kWavesM * kQB4 * 4 + 2 * (size_t)kQB4 * 4 +
                           3 * (size_t)kWitLevels * kQB4 * 4 + (size_t)kWavesM * kCandQ4 * 4;
// (the persistent batch kernel adds 16 bytes for its work queue)
static_assert(kLdsFp4 + 16 <= 163840, "fp4 query tile and epilogue state must fit the 160 KiB LDS");

// One work item of the fp4 scan: query tile [q0, q0 + nq_tile), at most 16 NA
// queries, of a query set against tiles [tb, te) of a reference range (the
// kernels below take their items from the launch geometry or from a queue).
// Every wave of the workgroup calls it with the same item.
//
// Bound: the matrix cores and, once they are kept busy, the card's power (the
// clock falls from 2.4 to 2.28 GHz).  The 128 queries x 64 references of
// accumulators leave two waves per SIMD, so the order of a wave's own
// instructions decides: each block of four MFMAs is pinned together with the
// LDS read of the query block two ahead and its share of the next step's
// spread (scheduling barriers; left to itself the compiler waits for an LDS
// read before every four MFMAs), the LDS words are permuted so that no read
// meets a bank twice, and the next half of a long row is copied by the DMA
// engine under the current one.  Measured at 2048 x 20M x 2048, top-32 (the
// scan alone): 23.1 ms before, 21.9 with these, MFMA pipes busy 0.73 -> 0.80 of
// the time, 20.8 with fewer and cheaper visits to the selection; 256 x 2M x
// 32768 5.53 -> 4.95 ms; 2048 x 1M x 2048 full counts 3.75 -> 2.68 ms (16-byte
// stores); 131 x 20M x 2048 3.17 -> 2.0 ms (tiles of 5 and 4 blocks).
template <int EPI, bool KCHUNKS, int NA>
__device__ __forceinline__ void fp4_work(const Fp4Work& w)
{
    // (aligned so that the read addresses' permutation bits are the tile's own)
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem4[];
    constexpr bool kLists = EPI == EPI_TOPK || EPI == EPI_BOTH;    // top-k lists
    constexpr bool kHits = EPI == EPI_THRESH || EPI == EPI_BOTH;   // threshold hits
    const int32_t* __restrict__ pcq = w.pcq;
    int32_t* __restrict__ out = w.out;
    uint64_t* __restrict__ lists = w.lists;
    uint32_t* __restrict__ fills = w.fills;
    const uint32_t* __restrict__ thr_init = w.thr_init;
    const uint32_t* __restrict__ level = w.level;
    uint32_t* __restrict__ wit = w.wit;
    const int32_t* __restrict__ thr = w.thr;
    const int q0 = w.q0;
    const int nq_tile = w.nq_tile;
    const int64_t base = w.base;
    const int64_t tb = w.tb;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int worker = w.slot * kWavesM + wv;
    const int n_workers_r = w.n_slots * kWavesM;
    uint32_t* lthr_all = reinterpret_cast<uint32_t*>(smem4 + 2 * kHalfBytes4);
    uint32_t* lfill_all = lthr_all + kWavesM * kQB4;
    int32_t* pcst_all = reinterpret_cast<int32_t*>(lfill_all + kWavesM * kQB4);
    int32_t* tpcq = pcst_all + kWavesM * 2 * kRefsPerWave4;
    int32_t* tthr = tpcq + kQB4;
    uint32_t* tlvl = reinterpret_cast<uint32_t*>(tthr + kQB4);
    uint32_t* wst = tlvl + kWitLevels * kQB4;
    uint32_t* cq_all = wst + kWitLevels * kQB4;
    uint32_t* wloc = cq_all + kWavesM * kCandQ4;  // witness counts not yet in global memory
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)smem4;

    const int lane = lane_id();
    const int tid = (int)threadIdx.x;
    const int kg = lane >> 4;      // MFMA k quarter = output row group
    const int n16 = lane & 15;

    // groups of 512 loci, and the half rows that hold them; rows of more than
    // two halves are staged half by half while the tile is scanned
    const int ngroups = (w.db.n_loci + 511) / 512;
    const int nhalves = (ngroups + 1) / 2;
    const bool multi = KCHUNKS && nhalves > 2;
    fp4_stage_half<NA>(w, wv, lane, 0, lds0);
    if (!multi && nhalves > 1) fp4_stage_half<NA>(w, wv, lane, 1, lds0 + kHalfBytes4);
    // the popcounts of the wave's 64 references of a tile: two buffers, the
    // next tile's copied while this one is scanned (the database popcounts
    // are padded like its words, so every reference of a tile is readable)
    const uint32_t pcst = (uint32_t)(uintptr_t)(lds_u32*)(uint32_t*)(pcst_all + wv * 2 * kRefsPerWave4);
    const int32_t* wpc = w.db.pc + base + tb * kRefsPerWG4 + wv * kRefsPerWave4;
    if (w.te > tb) dma4(pcst, wpc, (uint32_t)lane * 4u);
    if (tid < kQB4) {
        // |Q| of identity queries, 0 for mixtures; rows past the tile's
        // queries get a value that no sum exceeds
        const int md = w.mode != kModePerQuery ? w.mode : (tid < nq_tile ? w.qmode[q0 + tid] : FID_MODE_MIXTURE);
        tpcq[tid] = tid >= nq_tile ? 1 << 24 : md == FID_MODE_IDENTITY ? pcq[q0 + tid] : 0;
        // threshold hit "count <= thr" is "count < thr + 1"; thr is clamped to
        // [-1, L] first (counts lie in [0, L]), which keeps every fp32 value exact
        int32_t tq = (kHits && tid < nq_tile) ? thr[q0 + tid] : -1;
        tq = tq < -1 ? -1 : (tq > w.db.n_loci ? w.db.n_loci : tq);
        tthr[tid] = tq + 1;
        for (int l = 0; l < kWitLevels; ++l) {
            tlvl[kWitLevels * tid + l] =
                (kLists && wit && tid < nq_tile) ? level[(size_t)kWitLevels * (q0 + tid) + l] : 0u;
            // staged witness counts start at zero for every item: a wave may
            // read rows whose staging another wave issues
            wst[kWitLevels * tid + l] = 0u;
            wloc[kWitLevels * tid + l] = 0u;
        }
    }
    uint32_t* lthr = lthr_all + wv * kQB4;
    uint32_t* lfill = lfill_all + wv * kQB4;
    lds_u32* cq = (lds_u32*)(cq_all + wv * kCandQ4);   // the wave's candidate queue
    const bool witness = kLists && wit != nullptr;
    if constexpr (kLists) {
        // rows past the tile's queries get bound 0: no count is below it.
        // A caller's bound may be anything up to 0xFFFFFFFF ("no bound yet");
        // counts never exceed L, so min(bound, L + 1) filters exactly the
        // same and keeps every compared value an integer below 2^25, exact
        // in fp32.
        const uint32_t cap = (uint32_t)w.db.n_loci + 1u;
        for (int i = lane; i < kQB4; i += 64) {
            lthr[i] = i < nq_tile ? min(thr_init[q0 + i], cap) : 0u;
            lfill[i] = 0u;
        }
    }
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __syncthreads();

    // Unit group g of reference tile t for this wave: its database block is
    // (base + 512 t + 64 wv) / 64; lane (kg, n16) loads unit 4 g + kg of
    // reference 16 j + n16 of that block.  Groups past the row (it may end up
    // to 3 units into its last group) read the next block or the database's
    // slack: the matching query loci are zero.
    const int w4 = w.db.w4;
    const char* words = reinterpret_cast<const char*>(w.db.words);
    const uint32_t loff = (uint32_t)kg * 1024u + (uint32_t)n16 * 16u;
    // Byte offsets of the wave's group g of tile t: wave-uniform, so a load
    // is a scalar base plus the lane's 32-bit offset.
    const char* wbase = words + ((base >> 6) + wv) * w4 * 1024;
    const int64_t tile_bytes = (int64_t)kWavesM * w4 * 1024;
    auto load_at = [&](uint4 (&dst)[kNB4], int64_t off) {
        const char* gp = wbase + off;
#pragma unroll
        for (int j = 0; j < kNB4; ++j)
            dst[j] = *reinterpret_cast<const uint4*>(gp + (loff + (uint32_t)j * 256u));
    };
    // Query block a of step t in the group at x: row 16 a + n16 of plane kg,
    // word (group parity, t) at its permuted place.
    auto lds_a = [&](uint32_t x, int t, int a) -> v4u {
        return *(const lds_v4u*)(uintptr_t)((x ^ (uint32_t)(t * 16)) + (uint32_t)(a * 16 * 128));
    };
    const uint32_t x_first = lds0 + (uint32_t)(kg * kPlane4 + n16 * 128 + ((n16 >> 1) & 7) * 16);

    uint4 cur[kNB4], nxt[kNB4];
    // tiles are counted from the range start in 32 bits (a range is far
    // shorter than 2^31 tiles), which keeps the loop state in scalar registers
    const int nt = (int)(w.te - tb);
    if (nt > 0) load_at(cur, tb * tile_bytes);
    int64_t toff = tb * tile_bytes;
    uint32_t half = 0;             // byte offset of the LDS half in use
    v4u ring[kRing4];
#pragma unroll
    for (int a = 0; a < kRing4; ++a) ring[a] = lds_a(x_first, 0, a);
    v4f acc[NA][kNB4];
    int refresh = 0;               // the tile at which the bounds are renewed
    const int gap = min(max(w.n_slots >> 6, 1), 4);
    for (int it = 0; it < nt; ++it, toff += tile_bytes) {
        const int64_t tile = tb + it;
        const int64_t rbase = base + tile * kRefsPerWG4 + (int64_t)wv * kRefsPerWave4;
        const uint32_t pcs = pcst + (uint32_t)(it & 1) * (kRefsPerWave4 * 4);
        if (it + 1 < nt)
            dma4(pcst + (uint32_t)(~it & 1) * (kRefsPerWave4 * 4), wpc + (int64_t)(it + 1) * kRefsPerWG4,
                 (uint32_t)lane * 4u);
        // now and then the query tile's witness counts, read by the
        // epilogue; the workgroup's waves share them, each staging an eighth
        // (any value read is a count some time during the scan, and counts
        // only grow; rows past the tile's queries repeat its last query).
        // The k-th smallest count falls with the share of the database seen, so
        // the renewals thin out: after each quarter more tiles, at most 16
        // apart, and at least a tile per 64 workgroups that count into the same
        // few lines of memory (64 queries x 2M x 300 loci, 256 workgroups: 248
        // us with a renewal each tile, 130 with one every fourth).
        if (witness && it == refresh) {
            constexpr int kPer = kWitLevels * kQB4 / kWavesM;
#pragma unroll
            for (int h = 0; h < (kPer + 63) / 64; ++h) {
                const int o = kPer * wv + 64 * h;
                if (64 * h + lane < kPer)
                    dma4((uint32_t)(uintptr_t)(lds_u32*)(wst + o), wit + (size_t)kWitLevels * q0,
                         (uint32_t)min(o + lane, kWitLevels * nq_tile - 1) * 4u);
            }
        }
        // One group: prefetch the next (tile, group) into dst while the
        // MFMAs consume src.  Groups alternate between the two register sets,
        // so nothing is copied between them.  The ring of query blocks runs
        // on into the group at xn.
        const int64_t next_tile_off = it + 1 < nt ? toff + tile_bytes : toff;  // the last re-reads itself
        auto group = [&](auto first, const uint4 (&src)[kNB4], uint4 (&dst)[kNB4], int g, uint32_t x, uint32_t xn,
                         auto after_step0) {
            load_at(dst, g + 1 < ngroups ? toff + (int64_t)(g + 1) * (kUnitsPerGroup4 * 1024) : next_tile_off);
            // keep the prefetch ahead of this group's MFMAs (the scheduler
            // would otherwise sink it to its use to save registers)
            __builtin_amdgcn_sched_barrier(0);
            v8i b[2][kNB4];
            v4f start[kNB4];   // -|R| of the lane's references
#pragma unroll
            for (int j = 0; j < kNB4; ++j) {
                b[0][j] = spread_fp4(word_of(src[j], 0));
                if constexpr (decltype(first)::value) {
                    const v4u pr = *(const lds_v4u*)(uintptr_t)(pcs + (uint32_t)(16 * j + 4 * kg) * 4u);
#pragma unroll
                    for (int i = 0; i < 4; ++i) start[j][i] = -(float)(int32_t)pr[i];
                }
            }
#pragma unroll
            for (int t = 0; t < kUnitsPerGroup4; ++t) {
#pragma unroll
                for (int a = 0; a < NA; ++a) {
                    const int slot = (t * NA + a) % kRing4;  // (a group takes a whole number of rounds)
                    const v4u q = ring[slot];
                    const v8i qv = v8i{(int)q[0], (int)q[1], (int)q[2], (int)q[3], 0, 0, 0, 0};
#pragma unroll
                    for (int j = 0; j < kNB4; ++j) {
                        const v4f c = decltype(first)::value && t == 0 ? start[j] : acc[a][j];
                        acc[a][j] =
                            __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b[t & 1][j], qv, c, 4, 4, 0, 0, 0, 0);
                    }
                    const int an = (a + kRing4) % NA, tn = t + (a + kRing4) / NA;
                    ring[slot] = tn < kUnitsPerGroup4 ? lds_a(x, tn, an) : lds_a(xn, tn - kUnitsPerGroup4, an);
                    if (t + 1 < kUnitsPerGroup4) {
#pragma unroll
                        for (int j = kNB4 * a / NA; j < kNB4 * (a + 1) / NA; ++j)
                            b[(t + 1) & 1][j] = spread_fp4(word_of(src[j], t + 1));
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (t == 0) after_step0();
            }
        };
        // One half row: its two groups (one at the end of a row with an odd
        // number of groups); a row of more than two halves has the next half
        // copied into the other LDS half meanwhile (the barrier at the end
        // of the previous half has freed it).
        auto half_row = [&](auto first, int g) {
            // opaque: the permuted addresses are cheaper recomputed (one op a
            // step) than held in registers across the loop
            uint32_t x = x_first + half;
            __asm__ volatile("" : "+v"(x));
            const uint32_t xo = x + kHalfBytes4 - 2 * half;
            const bool two = g + 1 < ngroups;
            const uint32_t x_next = multi || nhalves == 1 ? x : xo;  // where the next half will be read
            auto copy_next = [&]() {
                if constexpr (KCHUNKS) {
                    if (multi && (g + 2 < ngroups || it + 1 < nt))
                        fp4_stage_half<NA>(w, wv, lane, g + 2 < ngroups ? (g >> 1) + 1 : 0,
                                           lds0 + (half ^ kHalfBytes4));
                }
            };
            group(first, cur, nxt, g, x, two ? x ^ 64u : x_next, copy_next);
            if (two) {
                group(std::false_type{}, nxt, cur, g + 1, x ^ 64u, x_next, [] {});
            } else {
#pragma unroll
                for (int j = 0; j < kNB4; ++j) cur[j] = nxt[j];
            }
            if (nhalves > 1) half ^= kHalfBytes4;
            if constexpr (KCHUNKS) {
                // (every wave reaches these barriers equally often: the tile
                // range is the workgroup's)
                if (multi) {
                    __builtin_amdgcn_s_waitcnt(kWaitVm0);
                    __syncthreads();
#pragma unroll
                    for (int a = 0; a < kRing4; ++a) ring[a] = lds_a(x_first + half, 0, a);
                }
            }
        };
        // a wave in its scan loop outranks one in its epilogue, so the
        // matrix-core pipe keeps being fed while the other wave selects
        __builtin_amdgcn_s_setprio(1);
        half_row(std::true_type{}, 0);
#pragma unroll 1
        for (int g = 2; g < ngroups; g += 2) half_row(std::false_type{}, g);
        if (!multi) half = 0;
        __builtin_amdgcn_s_setprio(0);

        // ---- epilogue: element i of block (a, j) holds x of reference
        // rbase + 16 j + 4 kg + i and tile query 16 a + n16.  The lane
        // coordinates are re-derived here, so that values computed from them
        // stay local to the epilogue instead of living (or spilling) across
        // the scan loop.
        int lane_e = lane;
        __asm__ volatile("" : "+v"(lane_e));
        const int kg_e = lane_e >> 4;
        const int n16_e = lane_e & 15;
        const bool inside = rbase >= w.r_lo && rbase + kRefsPerWave4 <= w.r_hi;  // wave-uniform
        // The next tile's popcounts and the witness counts copied at this
        // tile's start have landed: loads complete in order, and only the
        // four of the next tile's first group may still be in flight.
        __builtin_amdgcn_s_waitcnt(kWaitVm4);
        __asm__ volatile("" ::: "memory");
        if constexpr (EPI == EPI_FULL) {
#pragma unroll
            for (int a = 0; a < NA; ++a) {
                const int m = 16 * a + n16_e;
                const int32_t pq = tpcq[m];
                if (m < nq_tile) {
                    int32_t* row = out + (size_t)(q0 + m - w.out_q_base) * w.ld + (rbase + 4 * kg_e - w.out_r_base);
#pragma unroll
                    for (int j = 0; j < kNB4; ++j) {
                        if (inside) {
                            v4i_a4 c;
#pragma unroll
                            for (int i = 0; i < 4; ++i) c[i] = pq - (int32_t)acc[a][j][i];
                            *reinterpret_cast<v4i_a4*>(row + 16 * j) = c;
                        } else {
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const int64_t r = rbase + 16 * j + 4 * kg_e + i;
                                if (r >= w.r_lo && r < w.r_hi) row[16 * j + i] = pq - (int32_t)acc[a][j][i];
                            }
                        }
                    }
                }
            }
        } else {
            // x > tpcq - bound is a candidate (bound: the top-k bound, the
            // threshold + 1, or the larger of the two); every operand is an
            // integer below 2^25, so the comparison is exact in fp32
            float cut[NA], top[NA];
            bool any = false;
#pragma unroll
            for (int a = 0; a < NA; ++a) {
                const int m = 16 * a + n16_e;
                const uint32_t bound = EPI == EPI_TOPK     ? lthr[m]
                                       : EPI == EPI_THRESH ? (uint32_t)tthr[m]
                                                           : max(lthr[m], (uint32_t)tthr[m]);
                cut[a] = (float)(tpcq[m] - (int32_t)bound);
                top[a] = acc[a][0][0];
#pragma unroll
                for (int j = 0; j < kNB4; ++j)
#pragma unroll
                    for (int i = (j == 0 ? 1 : 0); i < 4; ++i) top[a] = fmaxf(top[a], acc[a][j][i]);
                any |= top[a] > cut[a];
            }
            // (the stated probability is for the register allocator: what does not
            // fit is to be spilled around the selection, never in the scan loop)
            if (__builtin_expect_with_probability(__builtin_amdgcn_ballot_w64(any) != 0, 0, 0.99999)) {
                // Queue the candidates of each block that holds one and drain
                // the queue.  A third of the tiles of a short row's scan come
                // here, so few operations matter: a block with a candidate,
                // then four elements with one, then the element, each a test
                // that the whole wave takes alike (512 queries x 10M x 512
                // loci, cycles a visit: 7400 with a test per element, 2600 so;
                // draining its 3.3 candidates 2600 list by list, 1200 with all
                // appended at once; the call 1250 us and 990).  Should it fill up, the elements from `resume` on
                // are queued in another pass (an element has at most 64
                // candidates, one per lane, so every pass gets on); their
                // bounds have tightened meanwhile, which the drain looks up.
                int resume = 0;
                // the block's references inside the range: [in_lo, in_lo + in_n), none of a
                // block of padding
                const int in_lo = (int)min(max(w.r_lo - rbase, (int64_t)0), (int64_t)kRefsPerWave4);
                const int in_hi = (int)min(max(w.r_hi - rbase, (int64_t)0), (int64_t)kRefsPerWave4);
                const uint32_t in_n = (uint32_t)max(in_hi - in_lo, 0);
                do {
                    int stop = 16 * NA, qn = 0;  // (wave-uniform)
                    // opaque values, so that nothing of an element is
                    // computed ahead of this loop and held (or spilled)
                    float zero = 0.f;
                    int row0 = 4 * kg_e;
                    __asm__ volatile("" : "+v"(zero), "+v"(row0));
#pragma unroll
                    for (int a = 0; a < NA; ++a) {
                        if (16 * a + 15 < resume || 16 * a >= stop) continue;
                        float ca = cut[a];
                        __asm__ volatile("" : "+v"(ca));
                        if (!__builtin_amdgcn_ballot_w64(top[a] > ca)) continue;
                        const int m = 16 * a + n16_e;
                        const int32_t pq = tpcq[m];
#pragma unroll
                        for (int j = 0; j < kNB4; ++j) {
                            float x0 = acc[a][j][0];
                            __asm__ volatile("" : "+v"(x0));  // (not computed ahead for all blocks)
                            const float top4 = fmaxf(fmaxf(fmaxf(x0, acc[a][j][1]), acc[a][j][2]), acc[a][j][3]);
                            if (!__builtin_amdgcn_ballot_w64(top4 > ca)) continue;
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const int e = 16 * a + 4 * j + i;
                                const float x = acc[a][j][i];
                                if (!__builtin_amdgcn_ballot_w64(x > ca)) continue;
                                const int ref = 16 * j + i + row0;
                                const bool cand = x > ca && (uint32_t)(ref - in_lo) < in_n;
                                const uint64_t cm = __builtin_amdgcn_ballot_w64(cand);
                                if (!cm || e < resume || e >= stop) continue;
                                const int nb = __popcll(cm);
                                if (qn + nb > kCandQ4) {
                                    stop = e;
                                    continue;
                                }
                                if (cand) {
                                    const int pos = qn + (int)__builtin_amdgcn_mbcnt_hi(
                                                             (uint32_t)(cm >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((uint32_t)cm, 0u));
                                    cq[pos] = (uint32_t)m | ((uint32_t)ref << 7) | ((uint32_t)(pq - (int32_t)(x + zero)) << 13);
                                }
                                qn += nb;
                            }
                        }
                    }
                    if (qn > 0) {
                        wave_lds_sync();
                        if constexpr (kHits)
                            fp4_drain_hits(cq, qn, rbase, q0, (const lds_u32*)(uint32_t*)tthr, w.hit_count,
                                           w.hit_keys, w.hit_cnt, w.hit_cap);
                        if constexpr (kLists)
                            fp4_drain_lists(cq, qn, rbase,
                                            (glb_u64*)(lists + ((size_t)q0 * n_workers_r + worker) * w.k),
                                            (int64_t)n_workers_r * w.k, w.k, (lds_u32*)lthr, (lds_u32*)lfill,
                                            (const lds_u32*)tlvl, witness ? (lds_u32*)wloc : nullptr);
                        wave_lds_sync();
                    }
                    resume = stop;
                } while (resume < 16 * NA);
            }
            if (witness && it == refresh) {
                refresh += min(max(it >> 2, gap), 16);
                fp4_flush_witness(wloc, wit + kWitLevels * q0, kWitLevels * nq_tile, wv, lane_e);
                // k distinct references below one of a query's witness
                // levels make that level a bound (a counter holds those below
                // its level but not below the next lower one)
#pragma unroll
                for (int h = 0; h < kQB4 / 64; ++h) {
                    const int i = lane_e + 64 * h;
                    uint32_t b = lthr[i], below = 0;
#pragma unroll
                    for (int l = kWitLevels - 1; l >= 0; --l) {
                        below += wst[kWitLevels * i + l];
                        if (below >= (uint32_t)w.k) b = min(b, tlvl[kWitLevels * i + l]);
                    }
                    lthr[i] = b;
                }
                wave_lds_sync();
            }
        }
    }
    if constexpr (kLists) {
        wave_lds_sync();
        for (int i = lane; i < nq_tile; i += 64)
            fills[(size_t)(q0 + i) * n_workers_r + worker] = lfill[i];
        if (witness) fp4_flush_witness(wloc, wit + kWitLevels * q0, kWitLevels * nq_tile, wv, lane);
    }
}

template <int EPI, bool KCHUNKS, int NA>
__global__ __launch_bounds__(kWGM) void fp4_scan_kernel(
    const ScanParams p, int mode, const uint8_t* __restrict__ qx, int32_t kpad,
    const int32_t* __restrict__ pcq, int32_t* __restrict__ out, uint64_t* __restrict__ lists,
    uint32_t* __restrict__ fills, const uint32_t* __restrict__ thr_init,
    const uint32_t* __restrict__ level, uint32_t* __restrict__ wit,
    const int32_t* __restrict__ thr, unsigned long long* __restrict__ hit_count,
    uint64_t* __restrict__ hit_keys, int32_t* __restrict__ hit_cnt)
{
    const int n_q = p.q_hi - p.q_lo;
    const int n_qtiles = p.n_qtiles;
    const int wg = xcd_local_index((int)blockIdx.x, (int)gridDim.x);
    const int qt_idx = wg % n_qtiles;
    const int wr_g = wg / n_qtiles;
    Fp4Work w;
    w.db = p.db;
    w.r_lo = p.r_lo;
    w.r_hi = p.r_hi;
    w.base = (p.r_lo / kDbTileRefs) * kDbTileRefs;
    const int64_t ntiles = (p.r_hi - w.base + kRefsPerWG4 - 1) / kRefsPerWG4;
    w.tb = (ntiles * wr_g) / p.n_rsplit;
    w.te = (ntiles * (wr_g + 1)) / p.n_rsplit;
    w.qx = qx;
    w.kpad = kpad;
    w.pcq = pcq;
    w.mode = mode;
    w.qmode = p.qmode;
    const int t0 = fp4_tile_begin(n_q, n_qtiles, qt_idx);
    w.q0 = p.q_lo + t0;
    w.nq_tile = min(fp4_tile_begin(n_q, n_qtiles, qt_idx + 1), n_q) - t0;
    w.slot = wr_g;
    w.n_slots = p.n_rsplit;
    w.k = p.k;
    w.out = out;
    w.ld = p.ld;
    w.out_q_base = p.out_q_base;
    w.out_r_base = p.out_r_base;
    w.lists = lists;
    w.fills = fills;
    w.thr_init = thr_init;
    w.level = level;
    w.wit = wit;
    w.thr = thr;
    w.hit_count = hit_count;
    w.hit_keys = hit_keys;
    w.hit_cnt = hit_cnt;
    w.hit_cap = p.hit_cap;
    fp4_work<EPI, KCHUNKS, NA>(w);
}

// The staged codes of one 32-locus query word: the reciprocals of the
// reference values, so that every product is 1; doubled for identity
// queries (products 2).  (e2m1 codes: 0x1 = 0.5, 0x2 = 1.0, 0x4 = 2.0,
// 0x6 = 4.0; a code times a 0/1 nibble is that code or 0.)
__device__ __forceinline__ uint4 fp4_query_codes(uint32_t w, bool dbl)
{
    uint4 v;
    v.x = (w & 0x11111111u) * (dbl ? 0x6u : 0x4u);          // 2.0 (4.0)
    v.y = ((w >> 1) & 0x11111111u) * (dbl ? 0x4u : 0x2u);   // 1.0 (2.0)
    v.z = ((w >> 2) & 0x11111111u) * (dbl ? 0x2u : 0x1u);   // 0.5 (1.0)
    v.w = ((w >> 3) & 0x11111111u) * (dbl ? 0x2u : 0x1u);   // 0.5 (1.0)
    return v;
}

// One wave stages one query row and counts its bits.  Word wi = 16 g + 4 kg + t
// of the row goes to the place the scan's LDS copy reads: half g / 2, k quarter
// kg, group parity, step t.
__device__ __forceinline__ void fp4_expand_row(const uint64_t* __restrict__ q, int32_t n_loci, bool identity,
                                               int32_t kpad, uint8_t* __restrict__ qx, int32_t* __restrict__ pcq)
{
    const int lane = lane_id();
    const int32_t words = kpad / 32;
    int32_t bits = 0;
    for (int32_t wi = lane; wi < words; wi += 64) {
        const int32_t left = n_loci - wi * 32;
        uint32_t v = 0;
        if (left > 0) {
            v = reinterpret_cast<const uint32_t*>(q)[wi];
            if (left < 32) v &= (1u << left) - 1u;
        }
        bits += __popc(v);
        const int32_t g = wi >> 4, at = (g >> 1) * 32 + ((wi >> 2) & 3) * 8 + (g & 1) * 4 + (wi & 3);
        reinterpret_cast<uint4*>(qx)[at] = fp4_query_codes(v, identity);
    }
    for (int o = 32; o > 0; o >>= 1) bits += __shfl_xor(bits, o);
    if (lane == 0) *pcq = bits;
}

constexpr int kExpandWaves = 4;

// Staged queries for the fp4 kernel: for every 32-locus word, 4 dwords in the
// element order above (zero past the row), plus popcount(Q_q).
__global__ __launch_bounds__(64 * kExpandWaves) void expand_queries_fp4_kernel(
    const uint64_t* __restrict__ q, int32_t n_q, int32_t row_words, int32_t n_loci, int mode,
    const int32_t* __restrict__ qmode, uint8_t* __restrict__ qx, int32_t kpad, int32_t* __restrict__ pcq,
    uint64_t* __restrict__ clear)
{
    if (clear && blockIdx.x == 0 && threadIdx.x == 0) *clear = 0ull;
    const int64_t i = (int64_t)blockIdx.x * kExpandWaves + (threadIdx.x >> 6);
    if (i >= n_q) return;
    const int md = mode == kModePerQuery ? qmode[i] : mode;
    fp4_expand_row(q + i * row_words, n_loci, md == FID_MODE_IDENTITY, kpad, qx + i * (kpad / 2), pcq + i);
}

hipError_t launch_expand_queries_fp4(const uint64_t* q, int32_t n_q, int32_t row_words,
                                     int32_t n_loci, int mode, const int32_t* qmode, uint8_t* qx,
                                     int32_t kpad, int32_t* pcq, hipStream_t s, uint64_t* clear)
{
    const unsigned blocks = (unsigned)((n_q + kExpandWaves - 1) / kExpandWaves);
    hipLaunchKernelGGL(expand_queries_fp4_kernel, dim3(blocks), dim3(64 * kExpandWaves), 0, s, q, n_q,
                       row_words, n_loci, mode, qmode, qx, kpad, pcq, clear);
    return hipGetLastError();
}

// ---------------------------------------------------------- batched passes

// Persistent fp4 pass: every workgroup takes work items from the queue of
// its own XCD (workgroups are dealt to the 8 XCDs round-robin, so those of
// one XCD -- and the items of one queue, which the planner fills range by
// range -- share that XCD's L2), then from the other queues, until all are
// empty.  An item is one query tile of one job against a run of reference
// tiles; the job's queries carry their own modes.
template <int EPI>
__global__ __launch_bounds__(kWGM) void fp4_batch_kernel(const Fp4BatchSet* __restrict__ sets,
                                                         const Fp4BatchItem* __restrict__ items,
                                                         const int32_t* __restrict__ queue_off,
                                                         unsigned int* __restrict__ counters)
{
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem4[];
    int& s_item = *reinterpret_cast<int*>(smem4 + kLdsFp4);
    const int home = (int)(blockIdx.x & 7u);
    for (int h = 0; h < 8; ++h) {
        const int qi = (home + h) & 7;
        const int32_t first = queue_off[qi];
        const uint32_t n_in = (uint32_t)(queue_off[qi + 1] - first);
        for (;;) {
            if (threadIdx.x == 0) {
                const uint32_t t = atomicAdd(counters + qi, 1u);
                s_item = t < n_in ? first + (int)t : -1;
            }
            __syncthreads();
            const int it = __builtin_amdgcn_readfirstlane(s_item);
            __syncthreads();  // every wave has read s_item before the next item overwrites it
            if (it < 0) break;
            const Fp4BatchItem& I = items[it];
            const Fp4BatchSet& S = sets[uni(I.set)];
            Fp4Work w;
            w.db.words = uni(S.db.words);
            w.db.pc = uni(S.db.pc);
            w.db.n_refs = 0;
            w.db.nblk = 0;
            w.db.n_loci = uni(S.db.n_loci);
            w.db.w4 = uni(S.db.w4);
            w.r_lo = uni(S.r_lo);
            w.r_hi = uni(S.r_hi);
            w.base = (w.r_lo / kDbTileRefs) * kDbTileRefs;
            w.tb = uni(I.tb);
            w.te = uni(I.te);
            w.qx = uni(S.qx);
            w.kpad = uni(S.kpad);
            w.pcq = uni(S.pcq);
            w.mode = kModePerQuery;
            w.qmode = uni(S.qmode);
            const int n_q = uni(S.n_q), n_qtiles = (n_q + kQB4 - 1) / kQB4, qtile = uni(I.qtile);
            w.q0 = fp4_tile_begin(n_q, n_qtiles, qtile);
            w.nq_tile = min(fp4_tile_begin(n_q, n_qtiles, qtile + 1), n_q) - w.q0;
            w.slot = uni(I.slot);
            w.n_slots = uni(S.n_slots);
            w.k = uni(S.k);
            w.out = uni(S.out);
            w.ld = uni(S.ld);
            w.out_q_base = 0;
            w.out_r_base = uni(S.out_r_base);
            w.lists = uni(S.lists);
            w.fills = uni(S.fills);
            w.thr_init = uni(S.thr_init);
            w.level = uni(S.level);
            w.wit = uni(S.wit);
            w.thr = nullptr;
            w.hit_count = nullptr;
            w.hit_keys = nullptr;
            w.hit_cnt = nullptr;
            w.hit_cap = 0;
            switch (fp4_tile_blocks(w.nq_tile)) {
                case 1:
                case 2: fp4_work<EPI, true, 2>(w); break;
                case 3:
                case 4: fp4_work<EPI, true, 4>(w); break;
                case 5: fp4_work<EPI, true, 5>(w); break;
                case 6: fp4_work<EPI, true, 6>(w); break;
                case 7: fp4_work<EPI, true, 7>(w); break;
                default: fp4_work<EPI, true, 8>(w); break;
            }
            __syncthreads();  // the next item restages the LDS tile
        }
    }
}

template <int EPI>
static hipError_t launch_fp4_batch_t(const Fp4BatchSet* sets, const Fp4BatchItem* items, const int32_t* queue_off,
                                     unsigned int* counters, int32_t grid, hipStream_t s)
{
    const hipError_t e = lds_opt_in<&fp4_batch_kernel<EPI>>((int)kLdsFp4 + 16);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fp4_batch_kernel<EPI>, dim3((unsigned)grid), dim3(kWGM), kLdsFp4 + 16, s, sets, items, queue_off,
                       counters);
    return hipGetLastError();
}

hipError_t launch_fp4_batch(int epi, const Fp4BatchSet* sets, const Fp4BatchItem* items, const int32_t* queue_off,
                            unsigned int* counters, int32_t grid, hipStream_t s)
{
    if (grid <= 0) return hipSuccess;
    if (epi == EPI_FULL) return launch_fp4_batch_t<EPI_FULL>(sets, items, queue_off, counters, grid, s);
    if (epi == EPI_TOPK) return launch_fp4_batch_t<EPI_TOPK>(sets, items, queue_off, counters, grid, s);
    return hipErrorInvalidValue;
}

// One wave per query of any job.
__global__ __launch_bounds__(64 * kExpandWaves) void expand_batch_fp4_kernel(const Fp4ExpandJob* __restrict__ jobs,
                                                                             int32_t n_jobs, int64_t total_q,
                                                                             const int32_t* __restrict__ qmode,
                                                                             int32_t* __restrict__ pcq)
{
    const int64_t g = (int64_t)blockIdx.x * kExpandWaves + (threadIdx.x >> 6);
    if (g >= total_q) return;
    int a = 0, b = n_jobs;  // the last job with q_off <= g
    while (b - a > 1) {
        const int m = (a + b) >> 1;
        if (jobs[m].q_off <= g) a = m;
        else b = m;
    }
    const Fp4ExpandJob& J = jobs[a];
    const int64_t i = g - J.q_off;
    fp4_expand_row(J.q + i * J.row_words, J.n_loci, qmode[g] == FID_MODE_IDENTITY, J.kpad, J.qx + i * (J.kpad / 2),
                   pcq + g);
}

hipError_t launch_expand_batch_fp4(const Fp4ExpandJob* jobs, int32_t n_jobs, int64_t total_q, const int32_t* qmode,
                                   int32_t* pcq, hipStream_t s)
{
    if (n_jobs <= 0) return hipSuccess;
    const unsigned blocks = (unsigned)((total_q + kExpandWaves - 1) / kExpandWaves);
    hipLaunchKernelGGL(expand_batch_fp4_kernel, dim3(blocks), dim3(64 * kExpandWaves), 0, s, jobs, n_jobs, total_q,
                       qmode, pcq);
    return hipGetLastError();
}

// Loci padded to whole LDS halves (1024 loci); zero on the query side.
int fp4_kpad(int32_t n_loci) { return ((n_loci + kHalfLoci4 - 1) / kHalfLoci4) * kHalfLoci4; }
int fp4_max_kpad() { return kMaxKpad4; }
int fp4_refs_per_wg() { return kRefsPerWG4; }
int fp4_queries_per_wg() { return kQB4; }
int fp4_list_workers_per_wg() { return kWavesM; }

template <int EPI, bool KCHUNKS, int NA>
static hipError_t launch_fp4_t(int mode, const ScanParams& p, const MfmaBuffers& b, hipStream_t s)
{
    const int64_t blocks = (int64_t)p.n_qtiles * p.n_rsplit;
    const hipError_t e = lds_opt_in<&fp4_scan_kernel<EPI, KCHUNKS, NA>>((int)kLdsFp4);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((fp4_scan_kernel<EPI, KCHUNKS, NA>), dim3((unsigned)blocks), dim3(kWGM), kLdsFp4, s, p, mode,
                       b.qx, b.kpad, b.pcq, b.out, b.lists, b.fills, b.thr_init, b.level, b.wit, b.thr, b.hit_count,
                       b.hit_keys, b.hit_cnt);
    return hipGetLastError();
}

// The instance for the largest of the launch's (even) query tiles.
template <int EPI, bool KCHUNKS>
static hipError_t launch_fp4_na(int mode, const ScanParams& p, const MfmaBuffers& b, hipStream_t s)
{
    switch ((fp4_tile_blocks(p.q_hi - p.q_lo) + p.n_qtiles - 1) / p.n_qtiles) {
        case 1:
        case 2: return launch_fp4_t<EPI, KCHUNKS, 2>(mode, p, b, s);
        case 3:
        case 4: return launch_fp4_t<EPI, KCHUNKS, 4>(mode, p, b, s);
        case 5: return launch_fp4_t<EPI, KCHUNKS, 5>(mode, p, b, s);
        case 6: return launch_fp4_t<EPI, KCHUNKS, 6>(mode, p, b, s);
        case 7: return launch_fp4_t<EPI, KCHUNKS, 7>(mode, p, b, s);
        default: return launch_fp4_t<EPI, KCHUNKS, 8>(mode, p, b, s);
    }
}

template <bool KCHUNKS>
static hipError_t launch_fp4_k(int mode, int epi, const ScanParams& p, const MfmaBuffers& b, hipStream_t s)
{
    switch (epi) {
        case EPI_FULL: return launch_fp4_na<EPI_FULL, KCHUNKS>(mode, p, b, s);
        case EPI_TOPK: return launch_fp4_na<EPI_TOPK, KCHUNKS>(mode, p, b, s);
        case EPI_BOTH: return launch_fp4_na<EPI_BOTH, KCHUNKS>(mode, p, b, s);
        default: return launch_fp4_na<EPI_THRESH, KCHUNKS>(mode, p, b, s);
    }
}

hipError_t launch_fp4_scan(int mode, int epi, const ScanParams& p, const MfmaBuffers& b,
                           hipStream_t s)
{
    if (p.n_rsplit <= 0) return hipSuccess;
    // (no tile of more queries than it holds, none without)
    if (p.n_qtiles < (p.q_hi - p.q_lo + kQB4 - 1) / kQB4 || p.n_qtiles > fp4_tile_blocks(p.q_hi - p.q_lo))
        return hipErrorInvalidValue;
    if (b.kpad > kMaxKpad4 || b.kpad != fp4_kpad(p.db.n_loci)) return hipErrorInvalidValue;
    if (b.kpad > 2 * kHalfLoci4) return launch_fp4_k<true>(mode, epi, p, b, s);
    return launch_fp4_k<false>(mode, epi, p, b, s);
}

}  // namespace fid

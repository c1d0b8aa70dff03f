// gfx950 kernels of the page-based RaaS decode path (arXiv 2502.11147,
// Algorithm 1 and Sections 3.2-3.3).
//
// Pool layout in HBM, per unit (sequence, layer, KV head): a contiguous run of
// Lcap = roundup(S * page_size, 32) token rows for K and for V. Token t of
// slot s sits at row s * page_size + t. Rows are grouped in blocks of 32; in a
// bf16 pool each block is stored in the order the attention MFMA operands
// are loaded, so that every 16-byte-per-lane load of a wavefront reads 1 KiB
// of consecutive bytes:
//   K block: [2 row tiles][D/32 k-steps][4 lane groups][16 rows][8 channels],
//            tile q, row i holding token 8*(i/4) + 4*q + i%4, lane group a
//            channels 32*ks + 8*a .. +8;
//   V block: [D/16 channel tiles][4 token octets][16 channels][8 tokens],
//            V transposed so a lane reads 8 consecutive tokens of one channel.
// An fp32 pool keeps plain [row][channel] order.
//
// One decode step is one launch of a step kernel (attention over the
// resident pages with the new token substituted in registers, the append of
// that token, the page scores, the top-r refresh, the eviction, the next
// target slot, the state out). When a unit is split over several workgroups,
// or units decide together, the last of these workgroups to end merges,
// decides and writes the state.
#include <math.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "raas_internal.h"

namespace raas {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(uint16_t x) { return __uint_as_float((uint32_t)x << 16); }

// round to nearest even; inputs are finite
__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t b = __float_as_uint(f);
    b += 0x7FFFu + ((b >> 16) & 1u);
    return (uint16_t)(b >> 16);
}

template <typename T>
__device__ __forceinline__ float to_f(T x);
template <>
__device__ __forceinline__ float to_f<float>(float x) { return x; }
template <>
__device__ __forceinline__ float to_f<uint16_t>(uint16_t x) { return bf2f(x); }

template <typename T>
__device__ __forceinline__ T from_f(float x);
template <>
__device__ __forceinline__ float from_f<float>(float x) { return x; }
template <>
__device__ __forceinline__ uint16_t from_f<uint16_t>(float x) { return f2bf(x); }

// element offset of (token row t, channel c) inside a unit's bf16 K run
template <int D>
__device__ __forceinline__ size_t k_off(int t, int c) {
    const int b = t >> 5, tt = t & 31;
    const int i = 4 * (tt >> 3) + (tt & 3), qq = (tt >> 2) & 1;
    const int ks = c >> 5, a = (c >> 3) & 3, e = c & 7;
    return (size_t)b * 32 * D + (size_t)(qq * (D / 32) + ks) * 512 + (16 * a + i) * 8 + e;
}

// element offset of (token row t, channel c) inside a unit's bf16 V run
template <int D>
__device__ __forceinline__ size_t v_off(int t, int c) {
    const int b = t >> 5, tt = t & 31;
    const int nb = c >> 4, i = c & 15, a = tt >> 3, j = tt & 7;
    return (size_t)b * 32 * D + (size_t)nb * 512 + (16 * a + i) * 8 + j;
}

__device__ __forceinline__ u32x4 ld4(const void* p) { return *reinterpret_cast<const u32x4*>(p); }
// The same from a caller's tensor, which is aligned to its element type only
// (the hardware takes any address for a 16-byte global load).
typedef uint32_t u32x4_at2 __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x4_at4 __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ u32x4 ld4_in(const uint16_t* p) { return *reinterpret_cast<const u32x4_at2*>(p); }
__device__ __forceinline__ u32x4 ld4_in(const float* p) { return *reinterpret_cast<const u32x4_at4*>(p); }
__device__ __forceinline__ void st4(void* p, u32x4 x) { *reinterpret_cast<u32x4*>(p) = x; }

__device__ __forceinline__ uint16_t u16_at(const u32x4& x, int e) {
    return (uint16_t)((x[e >> 1] >> ((e & 1) * 16)) & 0xFFFFu);
}

// element e of a 16-byte vector of T, as fp32
template <typename T>
__device__ __forceinline__ float vec_elem(const u32x4& x, int e);
template <>
__device__ __forceinline__ float vec_elem<uint16_t>(const u32x4& x, int e) { return bf2f(u16_at(x, e)); }
template <>
__device__ __forceinline__ float vec_elem<float>(const u32x4& x, int e) { return __uint_as_float(x[e]); }

// Makes this wavefront's LDS writes visible to its own later LDS reads (the
// lanes of one wavefront exchanging data through LDS; no workgroup barrier).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// Prefill (the prefill stage of Algorithm 1's cache store): a unit's first
// tokens go to pages 0, 1, ..., which are marked pinned; at most S-1 pages
// are kept (the first ones), so one slot stays for decode pages. Lengths are
// per sequence or uniform; sequences that are not selected keep their state.
// The input holds in.stride rows per unit.

// Prefill length of unit u, or -1 when its sequence is not selected.
__device__ __forceinline__ int unit_prefill_len(const LayerView& L, const PrefillIn& in, int u) {
    const int seq = u / L.nkv;
    return in.P >= 0 ? in.P : in.lens != nullptr ? in.lens[seq] : in.arg_lens[seq];
}

// pages kept of a prefill of P tokens: the first min(ceil(P/ps), pcap)
// (pcap = S-1, or the prompt region's slots)
__device__ __forceinline__ int kept_pages(const LayerView& L, int P) {
    return min((P + L.ps - 1) / L.ps, L.pcap);
}

// Slot and unit records of a unit just prefilled with P tokens.
__device__ __forceinline__ void prefill_records(const LayerView& L, int u, int P) {
    const int keep_pages = kept_pages(L, P);
    const size_t base = (size_t)u * L.S;
    for (int s = threadIdx.x; s < L.S; s += blockDim.x) {
        const bool pin = s < keep_pages;
        L.state[base + s] = pin ? kPinned : kFree;
        L.lid[base + s] = pin ? s : -1;
        L.ts[base + s] = -1;
        L.fill[base + s] = pin ? min(L.ps, P - s * L.ps) : 0;
    }
    if (threadIdx.x == 0) {
        int32_t* U4 = L.unit + (size_t)u * kUnitFields;
        U4[kTail] = -1;
        U4[kNextLid] = (P + L.ps - 1) / L.ps;
        U4[kClock] = P;
        U4[kEvicted] = -1;
        U4[kNextSlot] = max(keep_pages, L.dbase);  // lowest free decode slot; decode starts a fresh page
        U4[kNextFill] = 0;
        U4[kPinnedPages] = keep_pages;
    }
}

// Wavefronts of a prefill workgroup.
constexpr int kPrefillWaves = 4;
// Tokens of a wavefront's tile: eight per lane, a row of D channels over D /
// (16 bytes of T) lanes; 8 KB of keys and of values either way.
template <typename T, int D>
constexpr int prefill_tile() {
    return 8 * 64 * 16 / (D * (int)sizeof(T));
}

// The prefill store, in one launch: keys, values, slot records and (REP, pools
// that rank or select prompt pages) the kept pages' representative keys. A
// wavefront takes `tiles` consecutive tiles (more than one only where a page
// is longer than a tile, so that its representative key stays with one
// wavefront): a lane reads 16 bytes of each of eight rows, all 16 reads of a
// tile's keys and values in flight together, whole rows side by side. fp32
// pools store them as they are. bf16 pools store blocks in operand order: a
// lane's 8x8 values turn in registers (32 byte permutes), then keys and values
// pass through LDS in 16-byte pieces, so that every store writes 1 KiB of
// consecutive bytes. Bound by HBM: one read and one write of the prompt. (The
// form before read values two bytes at a time and stored keys in 64-byte runs,
// 3.9 TB/s at 256 units of 1024 tokens, then read every key again for the
// representative keys, two bytes at a time, 0.4 TB/s.)
// Tokens past a unit's kept ones are skipped (the rest of the last octet of
// values is zero).
template <typename T, int D, bool REP>
__global__ __launch_bounds__(kPrefillWaves * 64) void k_prefill(LayerView L, const T* __restrict__ k,
                                                                const T* __restrict__ v, PrefillIn in, int chunks,
                                                                int tiles) {
    constexpr bool BF = sizeof(T) == 2;
    constexpr int V = 16 / sizeof(T), LC = D / V, NO = 64 / LC, TT = 8 * NO;
    static_assert(TT == prefill_tile<T, D>(), "");
    __shared__ __align__(16) u32x4 s_piece[BF ? kPrefillWaves : 1][BF ? 512 : 1];
    const int u = blockIdx.x / chunks, chunk = blockIdx.x - u * chunks;
    const int P = unit_prefill_len(L, in, u);
    if (P < 0) return;  // not selected
    if (chunk == 0) prefill_records(L, u, P);
    const int keep = min(P, kept_pages(L, P) * L.ps);
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, oct = lane / LC, ch = lane % LC;
    T* K = (T*)L.K + (size_t)u * L.Lcap * D;
    T* Vp = (T*)L.V + (size_t)u * L.Lcap * D;
    const T* ku = k + (size_t)u * in.stride * D + V * ch;
    const T* vu = v + (size_t)u * in.stride * D + V * ch;
    const T inf = from_f<T>(INFINITY), ninf = from_f<T>(-INFINITY);
    T hi[V], lo[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        hi[e] = ninf;
        lo[e] = inf;
    }
    for (int it = 0; it < tiles; ++it) {
        const int t_tile = ((chunk * kPrefillWaves + w) * tiles + it) * TT;
        if (t_tile >= keep) break;
        const int t0 = t_tile + 8 * oct, n = min(max(keep - t0, 0), 8);  // this lane's tokens
        u32x4 kr[8], vr[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) kr[r] = r < n ? ld4_in(ku + (size_t)(t0 + r) * D) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int r = 0; r < 8; ++r) vr[r] = r < n ? ld4_in(vu + (size_t)(t0 + r) * D) : u32x4{0u, 0u, 0u, 0u};
        if constexpr (REP) {  // per-channel min and max, the first of equals
#pragma unroll
            for (int r = 0; r < 8; ++r)
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const float x = vec_elem<T>(kr[r], e);
                    if (r < n && x > to_f(hi[e])) hi[e] = from_f<T>(x);
                    if (r < n && x < to_f(lo[e])) lo[e] = from_f<T>(x);
                }
        }
        if constexpr (!BF) {
#pragma unroll
            for (int r = 0; r < 8; ++r)
                if (r < n) {
                    st4(K + (size_t)(t0 + r) * D + V * ch, kr[r]);
                    st4(Vp + (size_t)(t0 + r) * D + V * ch, vr[r]);
                }
        } else {
            // 16-byte piece p of the tile lies at LDS slot p with its low three
            // bits turned by the next three: the lanes of a write, eight pieces
            // apart, fall on different banks, and a read still covers 128-byte runs
            constexpr int BP = 4 * D;  // pieces of a block
            u32x4* sp = s_piece[w];
            auto slot = [](int p) { return p ^ ((p >> 3) & 7); };
            const int blk = oct >> 2, a = oct & 3;
#pragma unroll
            for (int r = 0; r < 8; ++r)  // token 8a + r of the block: see k_off
                sp[slot(blk * BP + ((r >> 2) * (D / 32) + (ch >> 2)) * 64 + 16 * (ch & 3) + 4 * a + (r & 3))] = kr[r];
            wave_lds_sync();
            const size_t out = (size_t)(t_tile >> 5) * 32 * D;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int p = 64 * j + lane, q = p % BP, i = q & 15;
                const int t = 32 * (p / BP) + 8 * (i >> 2) + 4 * (q / (2 * D)) + (i & 3);
                if (t_tile + t < keep) st4(K + out + (size_t)p * 8, sp[slot(p)]);
            }
            wave_lds_sync();
            // values: channel e of this lane's eight, its eight tokens side by side
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                u32x4 x;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    x[j] = __builtin_amdgcn_perm(vr[2 * j + 1][e >> 1], vr[2 * j][e >> 1],
                                                 (e & 1) ? 0x07060302u : 0x05040100u);
                const int c = 8 * ch + e;  // see v_off
                sp[slot(blk * BP + (c >> 4) * 64 + 16 * a + (c & 15))] = x;
            }
            wave_lds_sync();
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int p = 64 * j + lane;
                const int t = 32 * (p / BP) + 8 * ((p >> 4) & 3);
                if (t_tile + t < keep) st4(Vp + out + (size_t)p * 8, sp[slot(p)]);
            }
            wave_lds_sync();
        }
        if constexpr (REP) {
            // a page's octets combine (the earlier one's value kept between
            // equals on the lowest lanes, which store) when the page ends
            const int po = min(L.ps >> 3, NO);  // octets of a page in a tile
            const int t_last = t_tile + TT;
            if ((t_last & (L.ps - 1)) == 0 || L.ps <= TT || t_last >= keep) {
                for (int d = 1; d < po; d <<= 1)
#pragma unroll
                    for (int e = 0; e < V; ++e) {
                        const float h = __shfl_xor(to_f(hi[e]), d * LC), l = __shfl_xor(to_f(lo[e]), d * LC);
                        if (h > to_f(hi[e])) hi[e] = from_f<T>(h);
                        if (l < to_f(lo[e])) lo[e] = from_f<T>(l);
                    }
                if ((oct & (po - 1)) == 0 && t0 < keep) {
                    const size_t o = ((size_t)u * L.S + t0 / L.ps) * D + V * ch;
                    u32x4 x, y;
                    __builtin_memcpy(&x, hi, 16);
                    __builtin_memcpy(&y, lo, 16);
                    st4((T*)L.kmax + o, x);
                    st4((T*)L.kmin + o, y);
                }
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    hi[e] = ninf;
                    lo[e] = inf;
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// The retention rules of a step, for one unit; retention_wave (one workgroup per
// unit) and retention_block (the last workgroup of a split one) apply them. Slot
// state is in LDS with the page the step opened already marked evictable;
// s_score holds the score of every ranked page.
//  - Top-r refresh (Algorithm 1; Section 3.2): with n evictable pages and
//    k = floor(r*n), page p gets ts = clock when at least n-k evictable
//    pages score strictly less, i.e. exactly the pages above the (n-k)-th
//    smallest score.
//  - Eviction (Algorithm 1, the eviction branch of the decode-stage store):
//    when the tail page is full and no slot is free, the evictable page
//    with the smallest (timestamp, logical id) is freed.
//  - The next token's target: the tail page if it has room, else the lowest
//    free slot (a fresh page).

// The unit record as read once at the start of a step.
struct UnitRec {
    int ns, nf, clock, next_lid;
    __device__ bool opened() const { return nf == 0; }
};

// Slots that take part in the top-r order statistic: the evictable pages,
// and the pinned ones when the pool ranks them.
__device__ __forceinline__ bool ranked(const LayerView& L, int st) {
    return st == kEvictable || (L.rank_pinned && st == kPinned);
}

__device__ __forceinline__ UnitRec read_unit(const LayerView& L, int u) {
    const int32_t* U4 = L.unit + (size_t)u * kUnitFields;
    return UnitRec{U4[kNextSlot], U4[kNextFill], U4[kClock], U4[kNextLid]};
}

// Stages slot s (state, timestamp, logical id as read from the pool) in LDS,
// with the page the step opens already marked evictable.
__device__ __forceinline__ void stage_slot(const UnitRec& ur, int s, int st, int t, int id, double* s_score,
                                           int* s_state, int* s_ts, int* s_lid) {
    if (s == ur.ns && ur.opened()) {
        st = kEvictable;
        t = ur.clock;
        id = ur.next_lid;
    }
    s_state[s] = st;
    s_ts[s] = t;
    s_lid[s] = id;
    s_score[s] = INFINITY;  // scored below when evictable; never ranks under a real score
}

__device__ __forceinline__ void load_slots(const LayerView& L, int u, const UnitRec& ur, double* s_score, int* s_state,
                           int* s_ts, int* s_lid, int first = 0) {
    const int S = L.S;
    const size_t base = (size_t)u * S;
    for (int s = threadIdx.x + first; s < S; s += blockDim.x)
        stage_slot(ur, s, L.state[base + s], L.ts[base + s], L.lid[base + s], s_score, s_state, s_ts, s_lid);
}

// ---------------------------------------------------------------------------
// Results handed from one workgroup to another inside a launch. The L2s of
// the XCDs are not coherent with each other, and an agent-scope release
// writes back a whole L2 (6 to 9 us per step with hundreds of workgroups
// doing so). So the few kilobytes that cross workgroups are written with
// agent-scope (write-through) stores and read with agent-scope loads, which
// miss the L2: once a wavefront's stores have been acknowledged (vmcnt 0)
// they are where every XCD reads them, and nothing needs to be written back.
template <typename T>
__device__ __forceinline__ void publish(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T published(const T* p) {
    return __hip_atomic_load(const_cast<T*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// True on the last of `total` workgroups to call it for this counter, once
// everything that all of them published before is readable. The counter goes
// back to zero for the next launch. No workgroup waits for another. Every
// thread of the workgroup calls it; s_last: one LDS int.
__device__ __forceinline__ bool arrive_last(int32_t* counter, int total, int* s_last) {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);  // this wavefront's stores are acknowledged
    __syncthreads();
    if (threadIdx.x == 0) {
        const int before = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (before == total - 1) publish(counter, 0);
        *s_last = before == total - 1;
    }
    __syncthreads();
    return *s_last != 0;
}

// ---------------------------------------------------------------------------
// Page scores (Section 3.3, Quest's representative keys): for each evictable
// page, max over the G query heads of sum_c max(q_c*kmax_c, q_c*kmin_c),
// summed in fp64. bf16 pools: a product of two bf16 values has at most 16 significant
// bits, so both products are formed exactly in fp32 (q and the keys are
// staged as fp32), the larger is widened and added in fp64: each add rounds
// exactly as the fp64 sum of the exact product (products below fp32's normal
// range, under 1e-38 in magnitude, would be the exception). Eight
// lanes per page: lane part p sums D/8 consecutive channels in two chains
// (even and odd channels), the eight parts combine through a fixed xor tree,
// so equal pages score equal. A wavefront scores 8 pages per pass; its passes
// are interleaved with its attention blocks, each pass's keys loading while
// the previous block computes. The page the step writes to has its min/max
// widened by the new key and stored back.

// Cross-lane moves that stay in the VALU (no LDS round trip). dpp_f64<CTRL>:
// a DPP move of both halves of a double; 0xB1 and 0x4E (quad_perm
// [1,0,3,2] and [2,3,0,1]) give lane ^ 1 and lane ^ 2, 0x141 (row_half_mirror)
// gives lane 7 - i within each group of 8. max_xor16_32: the max over lanes
// i, i ^ 16, i ^ 32 and i ^ 48 through the two permlane swaps (a swap of a
// value with itself leaves both 16-lane or 32-lane halves side by side).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xF, 0xF, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// lanes i ^ 16 and i ^ 32 of a double (each half by a permlane swap; swap16
// and swap32 return both sides, which the caller combines)
__device__ __forceinline__ double2 swap16_f64(double x) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    return make_double2(__builtin_bit_cast(double, ((unsigned long long)(unsigned)hi[0] << 32) | (unsigned)lo[0]),
                        __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi[1] << 32) | (unsigned)lo[1]));
}
__device__ __forceinline__ double2 swap32_f64(double x) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    return make_double2(__builtin_bit_cast(double, ((unsigned long long)(unsigned)hi[0] << 32) | (unsigned)lo[0]),
                        __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi[1] << 32) | (unsigned)lo[1]));
}
// Whole-wavefront maximum and sum of a double, the result on every lane, in
// the same order on each: quads (xor 1, xor 2), the mirrors within 8 and 16
// lanes (the lanes of a quad, then of a half, hold equal values by then), and
// the two swaps.
__device__ __forceinline__ double wave_max_f64(double x) {
    x = fmax(x, dpp_f64<0xB1>(x));
    x = fmax(x, dpp_f64<0x4E>(x));
    x = fmax(x, dpp_f64<0x141>(x));
    x = fmax(x, dpp_f64<0x140>(x));
    const double2 a = swap16_f64(x);
    const double2 b = swap32_f64(fmax(a.x, a.y));
    return fmax(b.x, b.y);
}
__device__ __forceinline__ double wave_sum_f64(double x) {
    x += dpp_f64<0xB1>(x);
    x += dpp_f64<0x4E>(x);
    x += dpp_f64<0x141>(x);
    x += dpp_f64<0x140>(x);
    const double2 a = swap16_f64(x);
    const double2 b = swap32_f64(a.x + a.y);
    return b.x + b.y;
}
__device__ __forceinline__ float max_xor16_32(float x) {
    const unsigned u = __builtin_bit_cast(unsigned, x);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const float m = fmaxf(__builtin_bit_cast(float, (unsigned)a[0]), __builtin_bit_cast(float, (unsigned)a[1]));
    const unsigned v = __builtin_bit_cast(unsigned, m);
    const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return fmaxf(__builtin_bit_cast(float, (unsigned)b[0]), __builtin_bit_cast(float, (unsigned)b[1]));
}
// DPP move of a float; 0x124 and 0x128 (row_ror 4 and 8) turn the 16 lanes of
// a row, so that two steps with each reach the lanes equal in lane & 3.
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float sum_ror4_8(float x) {
    x += dpp_f32<0x124>(x);
    return x + dpp_f32<0x128>(x);
}
// sum over lanes i, i ^ 16, i ^ 32 and i ^ 48, in the same order on each
__device__ __forceinline__ float sum_xor16_32(float x) {
    const unsigned u = __builtin_bit_cast(unsigned, x);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    x = __builtin_bit_cast(float, (unsigned)a[0]) + __builtin_bit_cast(float, (unsigned)a[1]);
    const unsigned v = __builtin_bit_cast(unsigned, x);
    const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return __builtin_bit_cast(float, (unsigned)b[0]) + __builtin_bit_cast(float, (unsigned)b[1]);
}

// LDS slot of element i = head * D + channel of the fp32 query array: a
// 16-byte pad after each D/8 channels, so that the eight lanes scoring a
// page, which read channels D/8 apart, fall on different LDS banks and every
// group of four stays 16-byte aligned.
constexpr int qpad_row(int D) { return D + 32; }
template <int D>
__device__ __forceinline__ int qpad_index(int i) {
    const int h = i / D, c = i - (i / D) * D;
    return h * qpad_row(D) + c + 4 * (c / (D / 8));
}

template <typename T, int D>
struct ScoreFrag {
    static constexpr int SV = D * (int)sizeof(T) / 128;  // 16-byte vectors per array per lane (D/8 channels)
    u32x4 kx[SV], kn[SV];
};

template <typename T, int D>
__device__ __forceinline__ void score_issue(const LayerView& L, int u, int p, int part, bool load,
                                            ScoreFrag<T, D>& f) {
    constexpr int V = 16 / sizeof(T);
    const size_t off = ((size_t)u * L.S + p) * D + part * (D / 8);
    const T* kx = (const T*)L.kmax + off;
    const T* kn = (const T*)L.kmin + off;
#pragma unroll
    for (int i = 0; i < ScoreFrag<T, D>::SV; ++i) {
        f.kx[i] = load ? ld4(kx + V * i) : u32x4{0u, 0u, 0u, 0u};
        f.kn[i] = load ? ld4(kn + V * i) : u32x4{0u, 0u, 0u, 0u};
    }
}

template <typename T, int D>
__device__ __forceinline__ double score_finish(const LayerView& L, int u, int p, int part, bool act,
                                               ScoreFrag<T, D>& f, bool is_tail, bool opened,
                                               const T* k_new, const float* qf, double* hb) {
    constexpr int SV = ScoreFrag<T, D>::SV, V = 16 / sizeof(T);
    const int G = L.G;
    if (act && is_tail) {
#pragma unroll
        for (int i = 0; i < SV; ++i) {
            const u32x4 x = ld4(k_new + part * (D / 8) + V * i);
            if (opened) {
                f.kx[i] = x;
                f.kn[i] = x;
            } else if constexpr (sizeof(T) == 4) {
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    const float xv = __uint_as_float(x[h]);
                    f.kx[i][h] = xv > __uint_as_float(f.kx[i][h]) ? x[h] : f.kx[i][h];
                    f.kn[i][h] = xv < __uint_as_float(f.kn[i][h]) ? x[h] : f.kn[i][h];
                }
            } else {
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    uint32_t a = 0, b = 0;
#pragma unroll
                    for (int half = 0; half < 2; ++half) {
                        const uint16_t xv = (uint16_t)(x[h] >> (16 * half));
                        const uint16_t hv = (uint16_t)(f.kx[i][h] >> (16 * half));
                        const uint16_t lv = (uint16_t)(f.kn[i][h] >> (16 * half));
                        a |= (uint32_t)(bf2f(xv) > bf2f(hv) ? xv : hv) << (16 * half);
                        b |= (uint32_t)(bf2f(xv) < bf2f(lv) ? xv : lv) << (16 * half);
                    }
                    f.kx[i][h] = a;
                    f.kn[i][h] = b;
                }
            }
            const size_t off = ((size_t)u * L.S + p) * D + part * (D / 8) + V * i;
            st4((T*)L.kmax + off, f.kx[i]);
            st4((T*)L.kmin + off, f.kn[i]);
        }
    }
    const int c0 = part * (D / 8);
    // the keys widened to fp32 once for all heads (exact for bf16)
    float kxf[D / 8], knf[D / 8];
#pragma unroll
    for (int i = 0; i < SV; ++i)
#pragma unroll
        for (int e = 0; e < V; ++e) {
            kxf[V * i + e] = vec_elem<T>(f.kx[i], e);
            knf[V * i + e] = vec_elem<T>(f.kn[i], e);
        }
    double best = -INFINITY;
#pragma unroll 1
    for (int j = 0; j < G; ++j) {
        const float* qj = qf + (size_t)j * qpad_row(D) + c0 + 4 * part;  // see qpad_index
        double a;
        if constexpr (sizeof(T) == 4) {
            // products of two fp32 values are exact in fp64: the larger of the
            // two is the one that q's sign picks, and each fused multiply-add
            // rounds as the sum of the exact product
            a = 0.0;
#pragma unroll
            for (int c = 0; c < D / 8; c += 4) {
                const float4 qq = *reinterpret_cast<const float4*>(qj + c);
                a = fma((double)qq.x, (double)(qq.x >= 0.0f ? kxf[c] : knf[c]), a);
                a = fma((double)qq.y, (double)(qq.y >= 0.0f ? kxf[c + 1] : knf[c + 1]), a);
                a = fma((double)qq.z, (double)(qq.z >= 0.0f ? kxf[c + 2] : knf[c + 2]), a);
                a = fma((double)qq.w, (double)(qq.w >= 0.0f ? kxf[c + 3] : knf[c + 3]), a);
            }
        } else {
            double a0 = 0.0, a1 = 0.0;  // even and odd channels
#pragma unroll
            for (int c = 0; c < D / 8; c += 4) {
                const float4 qq = *reinterpret_cast<const float4*>(qj + c);
                a0 += (double)fmaxf(qq.x * kxf[c], qq.x * knf[c]);
                a1 += (double)fmaxf(qq.y * kxf[c + 1], qq.y * knf[c + 1]);
                a0 += (double)fmaxf(qq.z * kxf[c + 2], qq.z * knf[c + 2]);
                a1 += (double)fmaxf(qq.w * kxf[c + 3], qq.w * knf[c + 3]);
            }
            a = a0 + a1;
        }
        // the eight parts: pairs, then quads, then the two quads (the lanes of
        // a quad hold equal sums by then, so the mirror partner gives lane ^ 4's)
        a += dpp_f64<0xB1>(a);
        a += dpp_f64<0x4E>(a);
        a += dpp_f64<0x141>(a);
        best = a > best ? a : best;
        if (hb != nullptr && part == 0) publish(hb + j, a);  // per-head bounds, for the softmax aggregation
    }
    return best;
}

// Order-preserving map of a float onto an int (for an LDS atomic minimum), and back.
__device__ __forceinline__ int float_order(float x) {
    const int i = __builtin_bit_cast(int, x);
    return i >= 0 ? i : i ^ 0x7FFFFFFF;
}
__device__ __forceinline__ float order_float(int i) { return __builtin_bit_cast(float, i >= 0 ? i : i ^ 0x7FFFFFFF); }

// Order-preserving unsigned key of a float (unsigned order = numeric order,
// -0 just below +0), and back.
__device__ __forceinline__ unsigned ukey_f32(float x) {
    const unsigned b = __float_as_uint(x);
    return (b >> 31) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float from_ukey_f32(unsigned k) { return __uint_as_float((k >> 31) ? (k & 0x7FFFFFFFu) : ~k); }

// Wavefront 0's part of a pass of a radix select from the top: hist[0 .. 255]
// holds the counts of one digit among the keys still in play; finds the bin
// holding the want-th largest of them (1-based) and the rank within that bin,
// into hist[256] and hist[257]. Lane l scans bins 255-4l .. 252-4l.
__device__ __forceinline__ void radix_pick_top(int* hist, int want, int lane) {
    const int c0 = hist[255 - 4 * lane], c1 = hist[254 - 4 * lane], c2 = hist[253 - 4 * lane],
              c3 = hist[252 - 4 * lane];
    const int sum = c0 + c1 + c2 + c3;
    int incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
    }
    const int excl = incl - sum;
    if (excl < want && want <= incl) {
        int r = want - excl, b = 255 - 4 * lane;
        if (r > c0) {
            r -= c0;
            --b;
            if (r > c1) {
                r -= c1;
                --b;
                if (r > c2) {
                    r -= c2;
                    --b;
                }
            }
        }
        hist[256] = b;
        hist[257] = r;
    }
}

// Per bf16 half: the magnitude, at least the smallest normal (2^-126).
__device__ __forceinline__ uint32_t mag_floor(uint32_t x) {
    uint32_t lo = x & 0x7FFFu, hi = (x >> 16) & 0x7FFFu;
    lo = lo < 0x80u ? 0x80u : lo;
    hi = hi < 0x80u ? 0x80u : hi;
    return lo | (hi << 16);
}

// Quest bounds of the pages in slots 0 .. npages-1 (max over the heads of
// sum_c max(q_c kmax_c, q_c kmin_c), Section 4.2 with Quest's page
// representatives), as intervals, on the MFMA. With q+ and q- the positive
// and negative parts of q, a channel's term is q+ kmax + q- kmin, so per
// tile of 16 pages the bounds of every head are the product of [kmax | kmin]
// (pages x 2D) with [q+ ; q-] (2D x heads). The fp32 sum B of those 2D exact
// products lies within 2D 2^-23 E of the exact one whichever way each
// addition rounds, E the sum of their magnitudes; a product flushed for a
// subnormal factor or result loses at most what the same product of
// magnitudes floored at 2^-126 keeps, or 2^-126. So, with E taken over the
// floored magnitudes (one more product on the MFMA), the exact bound lies in
// B -+ (2^-13 E + 1e-30) at D up to 128, with room for E's own rounding.
// Written to lo/hi, with (-inf, inf) where a sum is not finite. Each
// wavefront takes tiles w, w + NW, ..., TPW of them loaded at once. q_ops:
// this lane's query operands (heads as columns). issue: the caller's loads,
// issued behind the last round of tiles on every wavefront. The keys are read
// with ordinary loads whatever the step's blocks are read with: a lane takes 16
// bytes of a row at a time, and every step reads the same keys (us per step
// among pools of 0.8 GB, non-temporal / ordinary: 64 units, 256 pages, 8 decode
// blocks 28.1 / 26.4; 128 units, 512 pages, 32 blocks, three pools in turn 45.9 /
// 42.6; 256 units, 256 pages, 8 blocks, the other way, 31.9 / 32.7).
template <int D, int NW, class Issue>
__device__ __forceinline__ void prompt_bounds(const LayerView& L, size_t base, int npages, const bf16x8 (&q_ops)[D / 32],
                                              float* lo, float* hi, Issue&& issue) {
    constexpr int KS = D / 32, TPW = D >= 128 ? 2 : 4;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, grp = lane >> 4, col = lane & 15;
    u32x4 qpos[KS], qneg[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const u32x4 x = __builtin_bit_cast(u32x4, q_ops[ks]);
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const uint32_t neg = ((x[h] >> 15) & 0x00010001u) * 0xFFFFu;  // halves with the sign set
            qneg[ks][h] = x[h] & neg;
            qpos[ks][h] = x[h] & ~neg;
        }
    }
    auto mfma = [](u32x4 a, u32x4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                       0, 0, 0);
    };
    auto floored = [](u32x4 x) { return u32x4{mag_floor(x[0]), mag_floor(x[1]), mag_floor(x[2]), mag_floor(x[3])}; };
    const int ntile = (npages + 15) / 16;
    constexpr int RT = TPW * NW;  // tiles per round of the workgroup
    const int nround = w < ntile ? (ntile - w + RT - 1) / RT : 0;  // rounds of this wavefront
    // lane (grp, col) supplies page 16t + col's channels 32ks + 8grp .. +7
    // (rows past npages, and tiles past the last, repeat the last page and
    // are not written)
    auto load = [&](int t0, u32x4 (&ax)[TPW][KS], u32x4 (&an)[TPW][KS]) {
#pragma unroll
        for (int h = 0; h < TPW; ++h) {
            const int t = min(t0 + h * NW, ntile - 1);
            const size_t off = (base + min(16 * t + col, npages - 1)) * D + 8 * grp;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const uint16_t* px = (const uint16_t*)L.kmax + off + 32 * ks;
                const uint16_t* pn = (const uint16_t*)L.kmin + off + 32 * ks;
                ax[h][ks] = ld4(px);
                an[h][ks] = ld4(pn);
            }
        }
    };
    auto bound = [&](int t0, const u32x4 (&ax)[TPW][KS], const u32x4 (&an)[TPW][KS]) {
#pragma unroll
        for (int h = 0; h < TPW; ++h) {
            const int t = t0 + h * NW;  // (a tile past the last is computed and not written)
            f32x4 sb = {0.f, 0.f, 0.f, 0.f}, se = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                sb = mfma(ax[h][ks], qpos[ks], sb);
                sb = mfma(an[h][ks], qneg[ks], sb);
                se = mfma(floored(ax[h][ks]), floored(qpos[ks]), se);
                se = mfma(floored(an[h][ks]), floored(qneg[ks]), se);
            }
            // lane (grp, col) holds head col of pages 16t + 4grp + i: the max over the heads
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float bm = col < L.G ? sb[i] : -INFINITY, em = col < L.G ? se[i] : 0.0f;
#pragma unroll
                for (int o = 8; o >= 1; o >>= 1) {
                    bm = fmaxf(bm, __shfl_xor(bm, o));
                    em = fmaxf(em, __shfl_xor(em, o));
                }
                const int p = 16 * t + 4 * grp + i;
                if (col == 0 && p < npages) {
                    const float err = em * 1.220703125e-04f + 1e-30f;  // 2^-13 E + 1e-30
                    const bool fin = __builtin_isfinite(bm) && __builtin_isfinite(err);
                    lo[p] = fin ? bm - err : -INFINITY;
                    hi[p] = fin ? bm + err : INFINITY;
                }
            }
        }
    };
    for (int r = 0; r + 1 < nround; ++r) {
        u32x4 ax[TPW][KS], an[TPW][KS];
        load(w + r * RT, ax, an);
        bound(w + r * RT, ax, an);
    }
    // the last round: its tiles, then the caller's loads, which the wait for
    // the tiles leaves in flight (loads complete in issue order); a wavefront
    // with no tile loads the last one and writes nothing
    const int tl = w + max(nround - 1, 0) * RT;
    u32x4 ax[TPW][KS], an[TPW][KS];
    load(tl, ax, an);
    __builtin_amdgcn_sched_barrier(0);  // (the caller's loads stay behind the tiles')
    issue();
    __builtin_amdgcn_sched_barrier(0);
    bound(tl, ax, an);
}

// Results of the retention policy for one step, computed by the retention
// wavefront and applied to the pool once the attention has read it.
struct RetShared {
    int victim, evicted, next_slot, next_fill, tail_after, errs;
};

// Page scores of the softmax aggregation, by a whole workgroup (every
// thread calls it): for each query head, a softmax over the ranked pages of
// the head's bounds b (scale c = 1/sqrt(D), shifted by the head's largest
// bound M), summed over the heads in head order: score(p) = sum_hj
// exp(c (b_hj(p) - M_hj)) / Z_hj. The heads are the G of each of nu units
// deciding together; hb[((h*S) + p)*G + j] holds head j of unit h's bound of
// page p for every ranked page p. First one wavefront per head finds M and Z
// (into s_mz), then one thread per page sums its terms; s_score is visible
// to the whole workgroup on return. The fp64 exponentials are the cost: with
// the bounds in LDS (PUB false) each replaces its bound, so that it is taken
// once; bounds too many for that are read as published (PUB) and take it
// twice.
template <bool PUB>
__device__ __forceinline__ void softmax_sum_block(const LayerView& L, double* hb, int nu, const int* s_state,
                                                  double* s_score, double* s_mz, int tid, int nthreads) {
    auto bound = [](const double* p) {
        if constexpr (PUB) return published(p);
        else return *p;
    };
    const int S = L.S, G = L.G, H = nu * G, lane = tid & 63, nw = nthreads >> 6;
    const double c = 1.0 / sqrt((double)L.D);
    for (int hj = tid >> 6; hj < H; hj += nw) {
        const int h = hj / G, j = hj - (hj / G) * G;
        double* hbj = hb + (size_t)h * S * G + j;
        double mx = -INFINITY;
        for (int p = lane; p < S; p += 64)
            if (ranked(L, s_state[p])) mx = fmax(mx, bound(hbj + (size_t)p * G));
        mx = wave_max_f64(mx);
        double z = 0.0;
        for (int p = lane; p < S; p += 64)
            if (ranked(L, s_state[p])) {
                const double e = exp(c * (bound(hbj + (size_t)p * G) - mx));
                if (!PUB) hbj[(size_t)p * G] = e;
                z += e;
            }
        z = wave_sum_f64(z);
        if (lane == 0) {
            s_mz[2 * hj] = mx;
            s_mz[2 * hj + 1] = z;
        }
    }
    __syncthreads();
    for (int p = tid; p < S; p += nthreads) {
        if (!ranked(L, s_state[p])) continue;
        double acc = 0.0;
#pragma unroll 4
        for (int hj = 0; hj < H; ++hj) {
            const int h = hj / G, j = hj - (hj / G) * G;
            const double b = bound(hb + ((size_t)h * S + p) * G + j);
            acc += (PUB ? exp(c * (b - s_mz[2 * hj])) : b) / s_mz[2 * hj + 1];
        }
        s_score[p] = acc;
    }
    __syncthreads();
}

// Retention policy of one unit, run by one wavefront (Algorithm 1, the
// decode-stage cache store; Sections 3.2-3.3) on the slot state in LDS, the opened page
// already marked evictable and s_score holding every ranked page's score
// (+inf elsewhere):
//  - top-r refresh: with n ranked pages and k = floor(r*n), an evictable
//    page p gets ts = clock when at least n-k ranked pages score strictly
//    less, i.e. exactly the pages above the (n-k)-th smallest score (the
//    ranked pages are the evictable ones, plus the pinned ones when the pool
//    ranks them; pinned pages never take a timestamp);
//  - eviction (Algorithm 1, the eviction branch of the decode-stage store):
//    when the tail page is full and no slot is free, the evictable page with
//    the smallest (timestamp, logical id) is freed;
//  - the next token's target: the tail page if it has room, else the lowest
//    free slot (a fresh page).
__device__ __forceinline__ void evict_wave(const LayerView& L, const UnitRec& ur, int* s_state, int* s_ts, const int* s_lid,
                           RetShared& out);

// lo: where the rank count starts, at most the first slot that a ranked
// page can occupy (slots below the decode base, and below the unit's pinned
// pages unless the pool ranks them, hold none).
template <bool F32>
__device__ __forceinline__ void retention_wave(const LayerView& L, const UnitRec& ur, double r, const double* s_score,
                               int* s_state, int* s_ts, const int* s_lid, RetShared& out, int lo) {
    const int S = L.S, lane = threadIdx.x & 63, s_lo = lo;
    int n = 0;
    for (int s0 = s_lo; s0 < S; s0 += 64) {
        const int s = s0 + lane;
        const int st = s < S ? s_state[s] : -1;
        n += __popcll(__ballot(st >= 0 && ranked(L, st)));
    }
    const int k = (int)floor(r * (double)n);
    if (k > 0) {
        // two scores per LDS read (s_score is 16-byte aligned; slots below lo
        // hold +inf), and the last of an odd S. The adds are one chain per
        // counter, hence two; unrolled by 8 (one counter) 64 slots took as long
        // as one score per read (8 units, 64 slots, us per step: one per read
        // 13.23, two with one counter 13.30, so 13.14; 1 unit, 48 slots 12.18,
        // 12.01, 11.94; 1 unit, 112 slots 17.56, 16.31, 15.70). fp32 pools, with
        // fewer slots to a block, by 8 (1 unit, 16 slots: 9.31 us with one
        // counter, 9.36 by 4, 9.29 so)
        const double2* sc2 = reinterpret_cast<const double2*>(s_score);
        const double last = (S & 1) ? s_score[S - 1] : INFINITY;
        for (int s0 = s_lo; s0 < S; s0 += 64) {
            const int p = s0 + lane;
            if (p < S && s_state[p] == kEvictable) {
                const double sp = s_score[p];
                int less = !F32 && last < sp ? 1 : 0, less1 = 0;
#pragma unroll(F32 ? 8 : 4)
                for (int o = s_lo >> 1; o < S >> 1; ++o) {
                    const double2 x = sc2[o];
                    less += x.x < sp ? 1 : 0;
                    less1 += x.y < sp ? 1 : 0;
                }
                if (F32 && (S & 1) && last < sp) ++less;
                if (less + less1 >= n - k) s_ts[p] = ur.clock;
            }
        }
    }
    evict_wave(L, ur, s_state, s_ts, s_lid, out);
}

// Eviction and the next token's target, by one wavefront, once the refresh
// has set the timestamps.
__device__ __forceinline__ void evict_wave(const LayerView& L, const UnitRec& ur, int* s_state, int* s_ts, const int* s_lid,
                           RetShared& out) {
    const int S = L.S, ps = L.ps, lane = threadIdx.x & 63;
    int nfree = 0;  // free decode slots
    for (int s0 = L.dbase; s0 < S; s0 += 64) {
        const int s = s0 + lane;
        nfree += __popcll(__ballot(s < S && s_state[s] == kFree));
    }
    const int fill_tail = ur.nf + 1;
    const bool full = fill_tail == ps && nfree == 0;
    int victim = -1;
    if (full) {
        unsigned long long best = ~0ull;
        for (int s0 = L.dbase; s0 < S; s0 += 64) {  // no decode page lies below the decode base
            const int s = s0 + lane;
            if (s < S && s_state[s] == kEvictable) {
                const unsigned long long key = ((unsigned long long)(uint32_t)s_ts[s] << 32) | (uint32_t)s_lid[s];
                best = key < best ? key : best;
            }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const unsigned long long o = __shfl_xor(best, off);
            best = o < best ? o : best;
        }
        for (int s0 = L.dbase; s0 < S; s0 += 64) {
            const int s = s0 + lane;
            const bool hit = s < S && s_state[s] == kEvictable &&
                             (uint32_t)s_lid[s] == (uint32_t)(best & 0xFFFFFFFFull);
            const unsigned long long m = __ballot(hit);
            if (m) {
                victim = s0 + __builtin_ctzll(m);
                break;
            }
        }
    }
    const bool tail_gone = victim == ur.ns;
    const int tail_fill = tail_gone ? 0 : fill_tail;
    const bool need_free = tail_gone || tail_fill == ps;
    int next_slot = ur.ns;
    if (need_free) {
        next_slot = S;
        for (int s0 = L.dbase; s0 < S; s0 += 64) {
            const int s = s0 + lane;
            const unsigned long long m = __ballot(s < S && (s_state[s] == kFree || s == victim));
            if (m) {
                next_slot = s0 + __builtin_ctzll(m);
                break;
            }
        }
    }
    if (lane == 0) {
        out.victim = victim;
        out.evicted = victim >= 0 ? s_lid[victim] : -1;
        out.next_slot = next_slot < S ? next_slot : 0;
        out.next_fill = need_free ? 0 : tail_fill;
        out.tail_after = tail_gone ? -1 : ur.ns;
        out.errs = (full && victim < 0 ? 2 : 0) | (need_free && next_slot >= S ? 4 : 0);
    }
    if (victim >= 0 && lane == 0) {
        s_state[victim] = kFree;
        s_ts[victim] = -1;
    }
}

// Order-preserving 64-bit key of a finite double (unsigned order = numeric
// order, with -0 just below +0), and back.
__device__ __forceinline__ unsigned long long order_key(double x) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    return (b >> 63) ? ~b : (b | (1ull << 63));
}
__device__ __forceinline__ double from_order_key(unsigned long long k) {
    return __longlong_as_double((long long)((k >> 63) ? (k & ~(1ull << 63)) : ~k));
}

// kth_largest_wg for doubles: eight 8-bit digits of order_key (-0 counted as
// +0, which it equals), by a workgroup of nth threads. hist: 258 ints.
__device__ double kth_largest_f64_wg(const double* x, int n, int k, int* hist, int tid, int nth) {
    const int lane = tid & 63;
    unsigned long long prefix = 0;
    int want = k;
    for (int shift = 56; shift >= 0; shift -= 8) {
        for (int b = tid; b < 256; b += nth) hist[b] = 0;
        __syncthreads();
        const unsigned long long high = shift == 56 ? 0ull : ~0ull << (shift + 8);
        for (int p = tid; p < n; p += nth) {
            const unsigned long long key = order_key(x[p] + 0.0);
            if ((key & high) == prefix) atomicAdd(&hist[(int)((key >> shift) & 255ull)], 1);
        }
        __syncthreads();
        if (tid < 64) radix_pick_top(hist, want, lane);
        __syncthreads();
        prefix |= (unsigned long long)hist[256] << shift;
        want = hist[257];
    }
    return from_order_key(prefix);
}

// The number of ranked slots among those this thread staged, added up over the
// workgroup into *s_n (zero before, complete after the caller's next barrier).
__device__ __forceinline__ void count_ranked(bool mine, int* s_n) {
    const unsigned long long m = __ballot(mine);
    if ((threadIdx.x & 63) == 0 && m) atomicAdd(s_n, __popcll(m));
}

// Top-r refresh and eviction by a whole workgroup (every thread calls it; the
// version of the rules in retention_wave for split units): with n ranked pages and k = floor(r*n), an evictable page is
// refreshed when at least n-k ranked pages score strictly less. meanwhile():
// the caller's own work, done by the other wavefronts while wavefront 0
// evicts. Slots below first hold no ranked page (the prompt region's, and
// pinned pages that are not ranked), so no loop starts before it: a long
// pinned prompt costs nothing here.
// Up to 64 slots wavefront 0 counts the lower scores (two per LDS read); up to
// 256 every thread, a slot's count spread over as many as there are (into
// s_less, zero before). Beyond, the workgroup finds theta, the (n-k)-th
// smallest ranked score, by a radix select over order_key (8-bit digits, most
// significant first, a 256-bin histogram each) and refreshes the evictable
// pages scoring above theta: the same pages, since fewer than n-k ranked scores
// lie below theta and at least n-k lie at or below it. It stops at the digit
// that leaves theta alone in its bin (the third, mostly), when a larger prefix
// means a larger score. s_score: 16-byte aligned, [S] and one more slot when S
// is odd; s_less: [S] ints; s_aux: 261 ints. The caller's barrier comes before
// and after.
template <class F>
__device__ __forceinline__ void retention_block(const LayerView& L, const UnitRec& ur, double r, int n,
                                                const double* s_score, int* s_state, int* s_ts, const int* s_lid,
                                                int* s_less, int* s_aux, RetShared& out, int tid, int nthreads,
                                                int first, F&& meanwhile) {
    const int S = L.S, lane = tid & 63, nsl = S - first;
    const int k = (int)floor(r * (double)n);
    const double2* sc2 = reinterpret_cast<const double2*>(s_score);
    const int pair0 = first >> 1, pair1 = (S + 1) >> 1;  // (slots below first and the one past S hold +inf)
    if (k > 0 && k < n && nsl <= 64) {
        if (tid < 64 && first + tid < S && s_state[first + tid] == kEvictable) {
            const double sp = s_score[first + tid];
            int less = 0;
#pragma unroll 8
            for (int o = pair0; o < pair1; ++o) {
                const double2 x = sc2[o];
                less += (x.x < sp ? 1 : 0) + (x.y < sp ? 1 : 0);
            }
            if (less >= n - k) s_ts[first + tid] = ur.clock;
        }
    } else if (k > 0 && k < n && nsl <= 256) {
        // slot first + i % wide, the pairs of scores share, share + shares, ...
        const int log_wide = nsl <= 128 ? 7 : 8, shares = max(1, nthreads >> log_wide);
        for (int i = tid; i < shares << log_wide; i += nthreads) {
            const int share = i >> log_wide, p = first + i - (share << log_wide);
            if (p >= S || s_state[p] != kEvictable) continue;
            const double sp = s_score[p];
            int less = 0;
#pragma unroll 8
            for (int o = pair0 + share; o < pair1; o += shares) {
                const double2 x = sc2[o];
                less += (x.x < sp ? 1 : 0) + (x.y < sp ? 1 : 0);
            }
            if (less) atomicAdd(&s_less[p], less);
        }
        __syncthreads();
        if (tid < 64) {
            for (int p = first + tid; p < S; p += 64)
                if (s_state[p] == kEvictable && s_less[p] >= n - k) s_ts[p] = ur.clock;
        }
    } else if (k > 0) {
        unsigned long long prefix = 0, mask = 0;
        int want = n - k - 1;  // 0-based rank of theta among the ranked scores that match prefix
        for (int shift = 56; shift >= 0 && k < n; shift -= 8) {
            for (int b = tid; b < 256; b += nthreads) s_aux[b] = 0;
            __syncthreads();
            for (int p = first + tid; p < S; p += nthreads) {
                if (!ranked(L, s_state[p])) continue;
                const unsigned long long key = order_key(s_score[p] + 0.0);  // (-0 counts as +0)
                if ((key & mask) == prefix) atomicAdd(&s_aux[(int)((key >> shift) & 255ull)], 1);
            }
            __syncthreads();
            if (tid < 64) {  // wavefront 0 scans the bins: lane l holds bins 4l .. 4l+3
                const int c0 = s_aux[4 * lane], c1 = s_aux[4 * lane + 1], c2 = s_aux[4 * lane + 2],
                          c3 = s_aux[4 * lane + 3];
                const int sum = c0 + c1 + c2 + c3;
                int incl = sum;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const int v = __shfl_up(incl, off);
                    if (lane >= off) incl += v;
                }
                const int excl = incl - sum;
                if (excl <= want && want < incl) {
                    int w = want - excl, b = 4 * lane, c = c0;
                    if (w >= c0) {
                        w -= c0;
                        ++b;
                        c = c1;
                        if (w >= c1) {
                            w -= c1;
                            ++b;
                            c = c2;
                            if (w >= c2) {
                                w -= c2;
                                ++b;
                                c = c3;
                            }
                        }
                    }
                    s_aux[257] = b;
                    s_aux[258] = w;
                    s_aux[259] = c;
                }
            }
            __syncthreads();
            prefix |= (unsigned long long)s_aux[257] << shift;
            mask |= 255ull << shift;
            want = s_aux[258];
            if (s_aux[259] == 1) break;
        }
        // (k == n: no digit was taken, and every page is refreshed)
        for (int p = first + tid; p < S; p += nthreads)
            if (s_state[p] == kEvictable && (k == n || (order_key(s_score[p] + 0.0) & mask) > prefix))
                s_ts[p] = ur.clock;
        __syncthreads();
    }
    if (tid < 64) {
        wave_lds_sync();
        evict_wave(L, ur, s_state, s_ts, s_lid, out);
    }
    meanwhile();
}

// Writes the step's retention results to the pool and the optional outputs.
__device__ __forceinline__ void retention_store(const LayerView& L, const StepIO& io, int u, const UnitRec& ur,
                                const int* s_state, const int* s_ts, const int* s_lid, const RetShared& rs,
                                int first, int stride) {
    const int S = L.S;
    const size_t base = (size_t)u * S;
    for (int s = first; s < S; s += stride) {
        const bool gone = s == rs.victim;
        const int st = s_state[s];
        const int id = gone ? -1 : s_lid[s];
        if (st == kEvictable || gone) L.ts[base + s] = s_ts[s];
        if (s == ur.ns || gone) {
            L.state[base + s] = st;
            L.lid[base + s] = id;
            L.fill[base + s] = gone ? 0 : ur.nf + 1;
        }
        if (io.page_table_out) io.page_table_out[base + s] = (st == kFree) ? -1 : id;
        if (io.timestamps_out) io.timestamps_out[base + s] = (st == kEvictable) ? s_ts[s] : -1;
    }
    if (first == 0) {
        int32_t* U4 = L.unit + (size_t)u * kUnitFields;
        U4[kTail] = rs.tail_after;
        U4[kNextLid] = ur.next_lid + (ur.opened() ? 1 : 0);
        U4[kClock] = ur.clock + 1;
        U4[kEvicted] = rs.evicted;
        U4[kNextSlot] = rs.next_slot;
        U4[kNextFill] = rs.next_fill;
        if (io.evicted_out) io.evicted_out[u] = rs.evicted;
        if (rs.errs) atomicOr(L.err, rs.errs);
    }
}

// Waits for every vector-memory load in flight (vmcnt(0); expcnt and lgkmcnt left at their maxima).
__device__ __forceinline__ void vm_drain() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Workgroup barrier that waits for this wavefront's LDS traffic only: loads
// already issued to global memory stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0); vmcnt and expcnt left at their maxima
    __builtin_amdgcn_s_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// The k-th largest of x[0 .. n-1] (1 <= k <= n, counted with multiplicity),
// by a whole workgroup of NT threads (every thread calls it and gets the
// value): a radix select over ukey_f32, four 8-bit digits from the most
// significant, a 256-bin histogram of the keys that match the digits found
// so far in each pass; wavefront 0 scans the bins from the top for the one
// holding the k-th key. hist: 258 ints of LDS.
template <int NT>
__device__ float kth_largest_wg(const float* x, int n, int k, int* hist, int tid) {
    const int lane = tid & 63;
    unsigned prefix = 0;
    int want = k;  // rank from the top among the keys that match prefix, 1-based
    for (int shift = 24; shift >= 0; shift -= 8) {
        for (int b = tid; b < 256; b += NT) hist[b] = 0;
        lds_barrier();
        const unsigned high = shift == 24 ? 0u : ~0u << (shift + 8);
        for (int p = tid; p < n; p += NT) {
            const unsigned key = ukey_f32(x[p]);
            if ((key & high) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1);
        }
        lds_barrier();
        if (tid < 64) radix_pick_top(hist, want, lane);
        lds_barrier();
        prefix |= (unsigned)hist[256] << shift;
        want = hist[257];
    }
    return from_ukey_f32(prefix);
}

// Merge of unit u's splits (out = sum_s 2^(M_s - M) O_s / sum_s 2^(M_s - M)
// L_s) from their published partials, by a whole workgroup, in two parts, so
// that every read of the first part is in flight together with the caller's
// own: kMergeAhead splits of this thread's first output, and item tid of the
// splits' maxima and sums. s_ml: [nsplit][G][2] floats of LDS.
constexpr int kMergeAhead = 16;
struct MergeFirst {
    float m, l, o[kMergeAhead];
};
__device__ __forceinline__ MergeFirst merge_first(const LayerView& L, int u, int tid) {
    const int G = L.G, D = L.D, nsplit = L.nsplit;
    const float* pu = L.part + (size_t)u * nsplit * G * (D + 2);
    MergeFirst f;
    const float* pm = pu + (size_t)min(tid, nsplit * G - 1) * (D + 2) + D;
    f.m = published(pm);
    f.l = published(pm + 1);
    const int idx = min(tid, G * D - 1), h = idx / D, c = idx - (idx / D) * D;
#pragma unroll
    for (int s = 0; s < kMergeAhead; ++s) f.o[s] = published(pu + ((size_t)min(s, nsplit - 1) * G + h) * (D + 2) + c);
    return f;
}
// every split's running max and sum into s_ml (visible after the caller's barrier)
__device__ __forceinline__ void merge_stage(const LayerView& L, int u, const MergeFirst& f, float* s_ml, int tid,
                                            int nth) {
    const int G = L.G, D = L.D, nsplit = L.nsplit;
    const float* pu = L.part + (size_t)u * nsplit * G * (D + 2);
    if (tid < nsplit * G) {
        s_ml[2 * tid] = f.m;
        s_ml[2 * tid + 1] = f.l;
    }
    for (int i = tid + nth; i < nsplit * G; i += nth) {
        s_ml[2 * i] = published(pu + (size_t)i * (D + 2) + D);
        s_ml[2 * i + 1] = published(pu + (size_t)i * (D + 2) + D + 1);
    }
}
template <typename T>
__device__ __forceinline__ void merge_out(const LayerView& L, const StepIO& io, int u, const MergeFirst& f,
                                          const float* s_ml, int tid, int nth) {
    const int G = L.G, D = L.D, nsplit = L.nsplit;
    const float* pu = L.part + (size_t)u * nsplit * G * (D + 2);
    for (int idx = tid; idx < G * D; idx += nth) {
        const int h = idx / D, c = idx - (idx / D) * D;
        float M = -INFINITY;
        for (int s = 0; s < nsplit; ++s) M = fmaxf(M, s_ml[2 * (s * G + h)]);
        float O = 0.0f, Ls = 0.0f;
        for (int s0 = 0; s0 < nsplit; s0 += kMergeAhead) {
            float o[kMergeAhead];
            if (idx == tid && s0 == 0) {
#pragma unroll
                for (int e = 0; e < kMergeAhead; ++e) o[e] = f.o[e];
            } else {
#pragma unroll
                for (int e = 0; e < kMergeAhead; ++e)
                    o[e] = published(pu + ((size_t)min(s0 + e, nsplit - 1) * G + h) * (D + 2) + c);
            }
#pragma unroll
            for (int e = 0; e < kMergeAhead; ++e) {
                if (s0 + e >= nsplit) break;
                const float ms = s_ml[2 * ((s0 + e) * G + h)];
                const float wt = (ms == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(ms - M);
                O += wt * o[e];
                Ls += wt * s_ml[2 * ((s0 + e) * G + h) + 1];
            }
        }
        ((T*)io.out)[((size_t)u * G + h) * D + c] = from_f<T>(O / Ls);
    }
}

// LDS bytes of finish_units: scores, slot records and counts, the softmax
// aggregation's M and Z and (where they fit kMaxStagedBounds) its bounds, the
// splits' maxima and sums
constexpr size_t kMaxStagedBounds = 64 * 1024;
__host__ __device__ constexpr size_t staged_bounds(int G, int S, int agg, int nu) {
    const size_t b = agg ? (size_t)nu * S * G * 8 : 0;
    return b <= kMaxStagedBounds ? b : 0;
}
__host__ __device__ constexpr size_t finish_lds(int G, int S, int nsplit, int agg, int nu) {
    return (size_t)(S + (S & 1)) * 8 + staged_bounds(G, S, agg, nu) + (agg ? (size_t)nu * G * 16 : 0) +
           (size_t)S * 16 + (size_t)2 * nsplit * G * 4;
}

// What is left of a step once the splits of every unit of a decision have
// published their page scores (and, with merge, their partial attention): the
// retention policy, the merge, and the state out, by one workgroup (every
// thread calls it). A decision covers units u0 .. u0+nu-1: one unit, or the KV
// heads of a sequence when they share one page table (whose slot states are
// then identical), a page's score aggregating the bounds of all their heads;
// merge (of unit u0) goes with nu 1. This is one chain of latencies, so its
// reads (scores, slot records, partials) all go out together, and wavefront 0
// evicts while the others merge. smem: finish_lds bytes of LDS, 16-byte
// aligned; s_aux: 261 ints.
template <typename T>
__device__ __forceinline__ void finish_units(const LayerView& L, const StepIO& io, double r, int u0, int nu,
                                             bool merge, unsigned char* smem, int* s_aux, RetShared& ret, int tid,
                                             int nth) {
    const int S = L.S, G = L.G;
    const size_t nhb = staged_bounds(G, S, L.agg, nu) / 8;
    double* s_score = reinterpret_cast<double*>(smem);
    double* s_hb = s_score + S + (S & 1);  // [nu][S][G], softmax aggregation only
    double* s_mz = s_hb + nhb;             // [nu*G][2], likewise
    int* s_state = reinterpret_cast<int*>(s_mz + (L.agg ? 2 * (size_t)nu * G : 0));
    int* s_ts = s_state + S;
    int* s_lid = s_ts + S;
    int* s_less = s_lid + S;
    float* s_ml = reinterpret_cast<float*>(s_less + S);
    const size_t base = (size_t)u0 * S;
    MergeFirst mf;
    if (merge) mf = merge_first(L, u0, tid);
    const UnitRec ur = read_unit(L, u0);
    const int first = L.rank_pinned ? L.dbase : max(L.dbase, L.unit[(size_t)u0 * kUnitFields + kPinnedPages]);
    if (tid == 0) {
        s_aux[256] = 0;
        if (S & 1) s_score[S] = INFINITY;
    }
    lds_barrier();  // (the count's zero; the reads stay in flight)
    for (int s = tid; s < S; s += nth) {
        double sc = INFINITY;
        if (!L.agg) {  // max over the units; read whether or not the page turns out to be ranked
            sc = published(L.score + base + s);
#pragma unroll 8
            for (int h = 1; h < nu; ++h) sc = fmax(sc, published(L.score + base + (size_t)h * S + s));
        }
        stage_slot(ur, s, L.state[base + s], L.ts[base + s], L.lid[base + s], s_score, s_state, s_ts, s_lid);
        s_less[s] = 0;
        const bool rk = ranked(L, s_state[s]);
        if (rk && !L.agg) s_score[s] = sc;
        count_ranked(rk, &s_aux[256]);
    }
    if (nhb > 0) {
        // no page below first is ranked, so no bound there is read (64 units, 1664
        // prompt pages, 40 blocks: 61.2 us with them, 57.7 without)
        const int row = S * G, skip = first * G, len = row - skip;
        for (int i = tid; i < nu * len; i += nth) {
            const int h = nu == 1 ? 0 : i / len, at = h * row + skip + i - h * len;
            s_hb[at] = published(L.score + base * G + at);
        }
    }
    if (merge) merge_stage(L, u0, mf, s_ml, tid, nth);
    __syncthreads();
    if (L.agg) {
        if (nhb > 0) softmax_sum_block<false>(L, s_hb, nu, s_state, s_score, s_mz, tid, nth);
        else softmax_sum_block<true>(L, L.score + base * G, nu, s_state, s_score, s_mz, tid, nth);
    }
    retention_block(L, ur, r, s_aux[256], s_score, s_state, s_ts, s_lid, s_less, s_aux, ret, tid, nth, first, [&] {
        if (merge) merge_out<T>(L, io, u0, mf, s_ml, tid, nth);
    });
    __syncthreads();
    // the units side by side, each by an equal share of the threads
    int per = nth, share = 0, shares = 1;
    if (nu > 1) {
        per = max(1, nth / nu);
        share = tid / per;
        shares = nth / per;
    }
    for (int uh = share; uh < nu && share < shares; uh += shares)
        retention_store(L, io, u0 + uh, ur, s_state, s_ts, s_lid, ret, tid - share * per, per);
}

// One 32-token block of attention for the GQA group held by this wavefront:
// QK^T as two 16x16x32 bf16 MFMA tiles per 32 channels (rows = tokens,
// columns = query heads), online softmax in base 2 with one cross-lane max,
// PV as D/16 MFMAs of V^T times P^T. nv: valid rows among this lane's eight.
template <int D>
__device__ __forceinline__ void attend_block(const u32x4 (&kr)[D / 16], const u32x4 (&vr)[D / 16], int nv,
                                             const bf16x8 (&qv)[D / 32], float scale_log2, float& m_run,
                                             float& l_run, f32x4 (&acc)[D / 16]) {
    constexpr int KS = D / 32, NB = D / 16;
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kr[ks]), qv[ks], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kr[KS + ks]), qv[ks], s1, 0, 0, 0);
    }
    // x[j]: scaled logit of token 8*grp + j for head `col` (base 2)
    float x[8];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        x[v] = (v < nv) ? s0[v] * scale_log2 : -INFINITY;
        x[4 + v] = (4 + v < nv) ? s1[v] * scale_log2 : -INFINITY;
    }
    float mb = x[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) mb = fmaxf(mb, x[j]);
    mb = max_xor16_32(mb);
    const float m_new = fmaxf(m_run, mb);
    if (__ballot(m_new > m_run) != 0ull) {
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        l_run *= alpha;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[nb] *= alpha;
        m_run = m_new;
    }
    float psum = 0.0f;
    bf16x8 pb;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float pj = __builtin_amdgcn_exp2f(x[j] - m_run);
        psum += pj;
        pb[j] = (__bf16)pj;
    }
    l_run += psum;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
        acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vr[nb]), pb, acc[nb], 0, 0, 0);
}

// The same for fp32 pools, on 16 tokens: the products are fp32 and so are
// their sums. A lane's 16-byte load of a key row holds channels 16j + 4grp ..
// +3 of token `col`, whichever way the matrix cores then take it; the queries
// come from LDS in the same order (s_q: this lane's head and channel group).
// nv: valid rows among the four tokens whose probabilities this lane holds.
//
// G > 4 (v_mfma_f32_16x16x4_f32): element e is the left operand of step (j,
// e), whose four channels are 16j + 4grp + e over the lane groups. The
// probabilities leave that product as tokens 4grp + i of head `col`, which is
// the right operand of the second one when its step tt takes the tokens 4grp +
// tt: a lane loads values of those four rows, channels 64h + 4col .. +3, and
// row i of the result's tile (h, e) is channel 64h + 16grp + 4i + e.
//
// G <= 4 (g4, v_mfma_f32_4x4x1_16b_f32, sixteen 4x4 products side by side): 16
// columns would idle at a cost of 64 steps of 32 cycles per block, 6.8 us of
// the 21.8 us that a step of 512 tokens took; 64 steps of 8 cycles do the
// same. Block (grp, tg), tg = (lane >> 2) & 3, multiplies tokens 4tg .. +3
// with the channels of its grp, head lane & 3; the four grp then add up, so
// every one of them holds the same logits of tokens 4tg + i. In the second
// product block (grp, tg) takes the tokens of its tg, channels 64h + 16grp +
// 4i + e as row i, so the values are loaded at rows 4tg + tt, channels 64h +
// 16grp + 4(lane & 3); the tg add up once, after the last block.
template <int D, bool g4>
__device__ __forceinline__ void attend_block_f32(const u32x4 (&kr)[D / 16], u32x4 (&vr)[D / 16], int nv,
                                                 const float* s_q, int grp, float scale_log2, float& m_run,
                                                 float& l_run, f32x4 (&acc)[D / 16]) {
    constexpr int NS = g4 ? 4 : 2;  // sums side by side (the 4x4 products are short)
    f32x4 s[NS];
#pragma unroll
    for (int e = 0; e < NS; ++e) s[e] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto logits = [&](auto mfma) {
#pragma unroll
        for (int j = 0; j < D / 16; ++j) {
            const int c = 16 * j + 4 * grp;
            const f32x4 q = *reinterpret_cast<const f32x4*>(s_q + c + 4 * (c / (D / 8)));  // see qpad_index
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e % NS] = mfma(__uint_as_float(kr[j][e]), q[e], s[e % NS]);
        }
    };
    auto mfma4 = [](float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0); };
    auto mfma16 = [](float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); };
    if constexpr (g4) logits(mfma4);
    else logits(mfma16);
    float x[4], mb = -INFINITY;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        x[v] = s[0][v] + s[1][v];
        if constexpr (NS == 4) x[v] += s[2][v] + s[3][v];
        if (g4) x[v] = sum_xor16_32(x[v]);
        x[v] = (v < nv) ? x[v] * scale_log2 : -INFINITY;
        mb = fmaxf(mb, x[v]);
    }
    if (g4) {
        mb = fmaxf(mb, dpp_f32<0x124>(mb));
        mb = fmaxf(mb, dpp_f32<0x128>(mb));
    } else {
        mb = max_xor16_32(mb);
    }
    const float m_new = fmaxf(m_run, mb);
    if (__ballot(m_new > m_run) != 0ull) {
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        l_run *= alpha;
#pragma unroll
        for (int nb = 0; nb < D / 16; ++nb) acc[nb] *= alpha;
        m_run = m_new;
    }
    float pj[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        pj[v] = __builtin_amdgcn_exp2f(x[v] - m_run);
        l_run += pj[v];
    }
    if (__ballot(nv < 4) != 0ull) {  // rows that hold no token weigh 0 whatever is stored there
#pragma unroll
        for (int tt = 0; tt < 4; ++tt)
#pragma unroll
            for (int h = 0; h < D / 64; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) vr[tt * (D / 64) + h][e] = tt < nv ? vr[tt * (D / 64) + h][e] : 0u;
    }
    auto values = [&](auto mfma) {
#pragma unroll
        for (int tt = 0; tt < 4; ++tt)
#pragma unroll
            for (int h = 0; h < D / 64; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc[4 * h + e] = mfma(__uint_as_float(vr[tt * (D / 64) + h][e]), pj[tt], acc[4 * h + e]);
    };
    if constexpr (g4) values(mfma4);
    else values(mfma16);
}

// ---------------------------------------------------------------------------
// Step kernel. One workgroup of NW wavefronts per (unit, split). Described for
// bf16 pools; fp32 pools run the same on blocks of 16 tokens, 16 KB either way
// at head_dim 128.
//
// Attention (Algorithm 1, attention(Q, K_old::K_new, V_old::V_new)) over
// every resident token, split-K over 32-token blocks. Each wavefront holds
// the unit's whole GQA query group; it takes one block statically, then
// claims further blocks from a counter in LDS, so the wavefronts that the
// memory system serves faster take more blocks. The next block loads while
// the current one computes. Per block: QK^T as two 16x16x32 bf16 MFMA tiles
// per 32 channels (rows = tokens, columns = query heads, G <= 16 of the 16
// used), online softmax in base 2 with one cross-lane max per block, and PV
// as D/16 MFMAs of V^T (rows = channels) times P^T (columns = heads). A lane
// owns one head (its column) in both products, so no data moves between
// lanes except the block max. The new token is not in the pool when the
// block is read: its K/V come from the step's inputs, substituted in
// registers, and the wavefront holding that block stores it.
//
// Page-score passes ride along with the first blocks. Once every wavefront
// has finished its passes (a workgroup barrier), wavefront 0 runs the
// retention policy when one workgroup covers the unit (fused), then goes on
// claiming blocks. The state reaches the pool only after the attention has
// read it; the wavefronts' partial outputs merge at the end, into the output
// when one workgroup covers the unit, else into the split's partial.

// AGG: the softmax aggregation of the page scores (a separate instance, so
// that the default one carries none of its registers).
// LM, pools with a prompt region (Quest on the prompt): 1, the blocks come
// from the unit's block list (the prompt blocks the selection kernel chose,
// then the decode region's); 2, the workgroup covers the unit and selects the
// prompt pages itself before its block loop (bounds on the MFMA, exact ones
// for the pages near the cut), then claims the decode blocks and the chosen
// prompt blocks from one list. 0: no prompt region.
// NT: K/V blocks are read with non-temporal loads (too little of the layer is
// left in the memory-side cache: non_temporal_loads).
// SPLIT: the unit is spread over several workgroups, or decides with others,
// and the last workgroup to end finishes the step (instances of their own:
// in one kernel with the fused ones, that code cost the block loop spills).
// The step of work item wi = unit * nsplit + split, by one workgroup (the
// arguments by value: as kernel arguments, they leave the registers of the
// block loop alone).
template <typename T, int D, int NW, bool AGG, int LM, bool NT, bool SPLIT, bool G4>
__device__ __forceinline__ void step_item(LayerView L, StepIO io, float scale_log2, double r, const int wi) {
    constexpr bool fused = !SPLIT;
    constexpr bool F32 = sizeof(T) == 4;
    constexpr int KS = D / 32, NB = D / 16;  // 16-byte vectors per lane: NB of a block's keys and of its values
    constexpr int BT = F32 ? 16 : 32, BLK = BT * D;  // tokens and elements of a block
    constexpr int BPB = 32 / BT;                     // blocks in the 32 tokens that the plan and the lists count in
    constexpr int TPL = BT / 4;                      // tokens whose probabilities a lane holds
    constexpr int VE = 16 / sizeof(T);               // elements of a 16-byte vector
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ float s_m[NW][16];
    __shared__ float s_l[NW][16];
    __shared__ RetShared ret;
    __shared__ int s_next;  // next unclaimed block index
    __shared__ int s_nsel;  // LM 2: prompt blocks chosen
    __shared__ int s_lo;    // LM 2: the topk-th largest lower end of a prompt bound (ordered bits)
    __shared__ int s_ncand; // LM 2: candidate prompt pages
    __shared__ __align__(16) T s_kn[D];  // the new token's key and value, staged so that
    __shared__ __align__(16) T s_vn[D];  // no read in the block loop waits on memory

    const int G = L.G, S = L.S, ps = L.ps;
    float* s_qf = reinterpret_cast<float*>(smem);  // [G][D+32] q in fp32, padded: qpad_index
    float* s_o = s_qf + (size_t)G * qpad_row(D);   // [NW][G][D+4]
    double* s_score = reinterpret_cast<double*>(s_o + (size_t)NW * G * (D + 4));  // [S], fused only, 16-byte aligned
    double* s_hb = s_score + S;  // [S][G] per-head bounds, fused softmax aggregation only
    double* s_mz = s_hb + (AGG ? (size_t)S * G : 0);  // [G][2] each head's M and Z, likewise
    int* s_state = reinterpret_cast<int*>(s_mz + (AGG ? 2 * G : 0));  // [S], fused only
    int* s_ts = s_state + S;
    int* s_lid = s_ts + S;
    int* s_list = fused ? s_lid + S : reinterpret_cast<int*>(s_score);  // LM 1: this workgroup's blocks
    // LM 2: the prompt pages' bound intervals and attended fills, the chosen
    // prompt blocks, the candidate pages and their exact bounds
    float* s_plo = reinterpret_cast<float*>(  // [dbase] lower ends, 16-byte aligned (the smem base is)
        reinterpret_cast<int*>(smem) + ((s_lid + S - reinterpret_cast<int*>(smem) + 3) & ~3));
    float* s_phi = s_plo + L.dbase;                                // [dbase] upper ends
    int* s_fatt = reinterpret_cast<int*>(s_phi + L.dbase);         // [dbase]
    int* s_plist = s_fatt + L.dbase;                               // [dbase * ps / 32]
    int* s_cand = s_plist + L.dbase * ps / 32;                     // [dbase]
    double* s_ex = reinterpret_cast<double*>(                      // [dbase], 8-byte aligned
        reinterpret_cast<int*>(smem) + ((s_cand + L.dbase - reinterpret_cast<int*>(smem) + 1) & ~1));

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int grp = lane >> 4, col = lane & 15;
    // tg: which of the block's TPL-token runs this lane's probabilities are of
    constexpr bool g4 = G4;
    const int tg = g4 ? (lane >> 2) & 3 : grp;
    const int vcol = g4 ? 16 * grp + 4 * (lane & 3) : 4 * col;  // fp32: channel of a value load
    const int nsplit = L.nsplit;
    const unsigned uwi = (unsigned)wi;  // (unsigned arithmetic, as on blockIdx.x)
    const int u = uwi / nsplit, split = uwi - (uwi / nsplit) * nsplit;
    if (io.active != nullptr && io.active[u / L.nkv] == 0) return;  // the sequence sits this step out
    const size_t base = (size_t)u * S;
    // this workgroup's claims lo .. hi-1: blocks of the unit (a range), or
    // (LIST) entries of its block list; pages scored here: those whose first
    // row lies in blocks sb0 .. sb1-1
    int lo, hi, sb0, sb1;
    const int nbp = LM ? L.dbase * ps / 32 : 0;  // LM: the decode region starts at this block
    if constexpr (LM == 2) {
        lo = 0;
        hi = L.nblk - nbp;  // decode blocks, claimed first; claims beyond are the chosen prompt blocks
        sb0 = nbp;          // score passes: the decode pages
        sb1 = L.nblk;
    } else if constexpr (LM == 1) {
        const int nsel = L.bcnt[2 * u], ntot = L.bcnt[2 * u + 1];
        const int per = (ntot + nsplit - 1) / nsplit;
        lo = min(ntot, split * per);
        hi = min(ntot, lo + per);
        sb0 = nbp + max(lo, nsel) - nsel;
        sb1 = nbp + max(hi, nsel) - nsel;
        for (int i = tid; i < hi - lo; i += NW * 64) s_list[i] = L.blist[(size_t)u * L.lcap_blk + lo + i];
        __syncthreads();
    } else {
        sb0 = split * L.bps;
        sb1 = max(sb0, min(L.nblk, sb0 + L.bps));
        lo = sb0 * BPB;
        hi = sb1 * BPB;
    }
    const int nown = LM ? (hi - lo) * BPB : hi - lo;  // claims of this workgroup
    const int bend = LM ? 0x40000000 : hi;     // no block: every block index lies below
    auto real = [&](int x) { return x < bend; };
    const T* qg = (const T*)io.q + (size_t)u * G * D;
    const T* kn_g = (const T*)io.k_new + (size_t)u * D;
    const T* vn_g = (const T*)io.v_new + (size_t)u * D;
    const T* Ku = (const T*)L.K + (size_t)u * L.Lcap * D;
    const T* Vu = (const T*)L.V + (size_t)u * L.Lcap * D;
    // fills the attention sees (the plain fill pointer where they are the
    // same: read through it, the first block's fill arrives sooner)
    const int32_t* fu = (LM == 1 ? L.fill_att : L.fill) + base;
    auto ldb = [&](const T* p) {
        if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
        else return ld4(p);
    };
    auto load_block = [&](int b, u32x4 (&kr)[NB], u32x4 (&vr)[NB]) {
        if constexpr (F32) {
            const T* Kb = Ku + (size_t)b * BLK + col * D + 4 * grp;
            const T* Vb = Vu + (size_t)b * BLK + 4 * tg * D + vcol;
#pragma unroll
            for (int j = 0; j < NB; ++j) kr[j] = ldb(Kb + 16 * j);
#pragma unroll
            for (int tt = 0; tt < 4; ++tt)
#pragma unroll
                for (int h = 0; h < D / 64; ++h) vr[tt * (D / 64) + h] = ldb(Vb + tt * D + 64 * h);
        } else {
            const T* Kb = Ku + (size_t)b * BLK + lane * 8;
            const T* Vb = Vu + (size_t)b * BLK + lane * 8;
#pragma unroll
            for (int i = 0; i < NB; ++i) kr[i] = ldb(Kb + i * 512);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) vr[nb] = ldb(Vb + nb * 512);
        }
    };

    // Loads complete in issue order, so the small reads go out first: the
    // unit record, this thread's staging elements and slot, the first
    // block's fill and the queries; then the first block (its index w is
    // static), which the staging below no longer waits for (LM 2: the
    // staging, then the bound tiles, then the first block).
    const int32_t* U4 = L.unit + (size_t)u * kUnitFields;
    const UnitRec ur{U4[kNextSlot], U4[kNextFill], U4[kClock], U4[kNextLid]};
    const int pinned = U4[kPinnedPages];
    // claim index i of the own blocks, ascending or (L.rev) descending
    auto blk_of = [&](int i) {
        const int j = L.rev ? nown - 1 - i : i;
        if constexpr (LM == 1) return s_list[j / BPB] * BPB + j % BPB;
        else if constexpr (LM == 2) return nbp + j;
        else return lo + j;
    };
    int b = (w < nown) ? blk_of(w) : bend;  // (LM 2: a prompt block, once they are chosen)
    const int slot_first = (BT * b + TPL * tg) / ps;
    const int fill_first = (real(b) && slot_first < S) ? fu[slot_first] : 0;
    // unconditional (clamped) reads: a read under a branch draws its first
    // use into the branch, with a wait for it ahead of the block loads
    const T q_first = qg[tid < G * D ? tid : 0];
    const int t_new = tid < D / VE ? tid : 0;
    const u32x4 kn_first = ld4_in(kn_g + VE * t_new), vn_first = ld4_in(vn_g + VE * t_new);
    const int s_first = tid < S ? tid : 0;
    const int st_first = L.state[base + s_first], ts_first = L.ts[base + s_first], lid_first = L.lid[base + s_first];
    const int pf_first = LM == 2 ? fu[tid < L.dbase ? tid : 0] : 0;  // LM 2: a prompt page's fill
    // LM 2: a second slot and prompt page per thread, with the reads above
    const int sl_sec = tid + NW * 64 < S ? tid + NW * 64 : 0, pg_sec = tid + NW * 64 < L.dbase ? tid + NW * 64 : 0;
    int st_sec = 0, ts_sec = 0, lid_sec = 0, pf_sec = 0;
    if constexpr (LM == 2) {
        st_sec = L.state[base + sl_sec];
        ts_sec = L.ts[base + sl_sec];
        lid_sec = L.lid[base + sl_sec];
        pf_sec = fu[pg_sec];
    }
    bf16x8 qv[F32 ? 1 : KS];  // bf16: the queries as MFMA operands (fp32 reads them from LDS)
    if constexpr (!F32) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const u32x4 x = (col < G) ? ld4_in(qg + (size_t)col * D + 32 * ks + 8 * grp) : u32x4{0u, 0u, 0u, 0u};
            qv[ks] = __builtin_bit_cast(bf16x8, x);
        }
    }
    u32x4 kr_next[NB], vr_next[NB];
    int f_first = 0;  // LM 2: the first block's fill
    if constexpr (LM == 2) {
        // The staging first (the other instances stage below, behind the first
        // block's loads), so that none of its reads waits behind the bound
        // tiles or the block: they go out about when the tiles would, which
        // wait for the queries anyway.
        if (tid < L.dbase) s_fatt[tid] = tid < pinned ? pf_first : 0;  // the kept prompt pages' fills
        if (tid + NW * 64 < L.dbase) s_fatt[tid + NW * 64] = tid + NW * 64 < pinned ? pf_sec : 0;
        for (int p = tid + 2 * NW * 64; p < L.dbase; p += NW * 64) s_fatt[p] = p < pinned ? fu[p] : 0;
        // q in fp32 from the query operands: lane (grp, col < G) holds head
        // col's channels 32 ks + 8 grp .. +7, one padded row segment; the
        // wavefronts take turns over ks
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks % NW == w && col < G) {
                const u32x4 x = __builtin_bit_cast(u32x4, qv[ks]);
                float* d = s_qf + qpad_index<D>(col * D + 32 * ks + 8 * grp);
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    d[2 * h] = __uint_as_float(x[h] << 16);
                    d[2 * h + 1] = __uint_as_float(x[h] & 0xFFFF0000u);
                }
            }
        }
        if (tid < D / 8) {
            st4(&s_kn[8 * tid], kn_first);
            st4(&s_vn[8 * tid], vn_first);
        }
        {
            if (tid < S) stage_slot(ur, tid, st_first, ts_first, lid_first, s_score, s_state, s_ts, s_lid);
            if (tid + NW * 64 < S) stage_slot(ur, tid + NW * 64, st_sec, ts_sec, lid_sec, s_score, s_state, s_ts, s_lid);
            load_slots(L, u, ur, s_score, s_state, s_ts, s_lid, 2 * NW * 64);
        }
        if (tid == 0) {
            s_next = 2 * NW;  // claims start after the two static blocks of every wavefront
            s_lo = 0x7FFFFFFF;
            s_ncand = 0;
        }
        if (w < nown) f_first = slot_first < S ? (slot_first == ur.ns ? ur.nf + 1 : fill_first) : 0;
        // nothing else is in flight yet: every read has landed from here on,
        // also to the compiler, which loses count of loads issued in loops
        vm_drain();
        // the prompt region's bound intervals (the selection reads those of the
        // kept pages), and behind their last loads the first block, which
        // streams during the selection; a wavefront with no decode block reads
        // block 0 and drops it (loads on every path keep the waits for the
        // tiles short of the block)
        auto first = [&]() { load_block(real(b) ? b : 0, kr_next, vr_next); };
        if (L.dbase > L.topk) prompt_bounds<D, NW>(L, base, L.dbase, qv, s_plo, s_phi, first);
        else first();
    } else {
        if (real(b)) load_block(b, kr_next, vr_next);
    }

    const int ns = ur.ns, nf = ur.nf;
    const bool opened = ur.opened();
    const int row_new = ns * ps + nf, b_new = row_new / BT, tt_new = row_new % BT;
    bool decided = false;  // this wavefront has passed the score barrier
    // the block of claim index i, or bend when none is left (LM 2: the decode
    // blocks, then the chosen prompt blocks)
    auto take = [&](int i) {
        if constexpr (LM == 2) {
            if (i < nown) return blk_of(i);
            return i - nown < s_nsel ? s_plist[i - nown] : bend;
        } else {
            return i < nown ? blk_of(i) : bend;
        }
    };
    // pages scored here: those whose first row lies in this workgroup's blocks, pinned ones
    // excepted unless they are ranked
    const int sl0 = max(L.rank_pinned ? 0 : pinned, min(S, (32 * sb0 + ps - 1) / ps));
    const int sl1 = min(S, (32 * sb1 + ps - 1) / ps);

    // fill of the page holding this lane's TPL rows of block b (page_size % 8 == 0)
    auto row_fill = [&](int b) {
        const int slot = (BT * b + TPL * tg) / ps;
        if constexpr (LM == 2)
            if (slot < L.dbase) return s_fatt[slot];  // read only once the prompt pages are chosen
        return (slot < S) ? (slot == ns ? nf + 1 : fu[slot]) : 0;
    };
    auto valid_rows = [&](int b, int f) {
        const int t0 = BT * b + TPL * tg;
        return min(max(f - (t0 - (t0 / ps) * ps), 0), TPL);
    };
    int f_next = f_first;
    if constexpr (LM != 2) {
        if (real(b)) f_next = (w < nown) ? (slot_first < S ? (slot_first == ns ? nf + 1 : fill_first) : 0) : row_fill(b);

        // staging for the scores and the retention
        if (tid < G * D) s_qf[qpad_index<D>(tid)] = to_f(q_first);
        for (int i = tid + NW * 64; i < G * D; i += NW * 64) s_qf[qpad_index<D>(i)] = to_f(qg[i]);
        if (tid < D / VE) {
            st4(&s_kn[VE * tid], kn_first);
            st4(&s_vn[VE * tid], vn_first);
        }
        if (fused) {
            if (tid < S) stage_slot(ur, tid, st_first, ts_first, lid_first, s_score, s_state, s_ts, s_lid);
            load_slots(L, u, ur, s_score, s_state, s_ts, s_lid, NW * 64);
        }
        if (tid == 0) s_next = 2 * NW;  // claims start after the two static blocks of every wavefront
    }
    // the staging is visible: the first block is still in flight, and every
    // wavefront reaches this point after the same short reads
    lds_barrier();

    if constexpr (LM == 2) {
        // the topk kept prompt pages of largest bound, ties to the lower slot
        // (Quest on the prompt): the others' fills are cleared. Each page's
        // exact bound lies in [s_plo, s_phi]; with lo the topk-th largest lower
        // end, at least topk pages have bounds >= lo, so a page whose upper end
        // is below lo ranks below all of them: the top k are among the
        // candidates with upper end >= lo, and rank among them as among all
        // kept pages.
        if (pinned > L.topk && L.topk > 0) {
            float lo_cut;
            if (pinned > 2 * NW * 64) {
                // many kept pages: lo by a radix select (the count below is
                // quadratic in them); s_ex is free until the candidates' bounds
                lo_cut = kth_largest_wg<NW * 64>(s_plo, pinned, L.topk, reinterpret_cast<int*>(s_ex), tid);
            } else {
                const int pin4 = pinned & ~3;
                for (int p = tid; p < pinned; p += NW * 64) {
                    // lower ends above p's: four per 16-byte read, then the last few
                    const float lp = s_plo[p];
                    int above = 0;
#pragma unroll 4
                    for (int o = 0; o < pin4; o += 4) {
                        const float4 x = *reinterpret_cast<const float4*>(s_plo + o);
                        above += (x.x > lp ? 1 : 0) + (x.y > lp ? 1 : 0) + (x.z > lp ? 1 : 0) + (x.w > lp ? 1 : 0);
                    }
                    for (int o = pin4; o < pinned; ++o) above += s_plo[o] > lp ? 1 : 0;
                    if (above < L.topk) atomicMin(&s_lo, float_order(lp));
                }
                lds_barrier();
                lo_cut = order_float(s_lo);
            }
            for (int p = tid; p < pinned; p += NW * 64) {
                if (s_phi[p] >= lo_cut) s_cand[atomicAdd(&s_ncand, 1)] = p;
                else s_fatt[p] = 0;
            }
            lds_barrier();
            // exactly topk candidates: they are the top k; more: the candidates'
            // bounds in fp64, eight lanes per page as the decode pages' scores
            const int nc = s_ncand;
            if (nc > L.topk) {
                for (int c0 = 8 * w; c0 < nc; c0 += 8 * NW) {
                    const int c = c0 + (lane >> 3);
                    const bool act = c < nc;
                    const int p = act ? s_cand[c] : 0;
                    ScoreFrag<T, D> f;
                    score_issue<T, D>(L, u, p, lane & 7, act, f);
                    const double sc = score_finish<T, D>(L, u, p, lane & 7, act, f, false, false, s_kn, s_qf, nullptr);
                    if (act && (lane & 7) == 0) s_ex[c] = sc;
                }
                lds_barrier();
                for (int c = tid; c < nc; c += NW * 64) {
                    const int p = s_cand[c];
                    const double e = s_ex[c];
                    int above = 0;
                    for (int o = 0; o < nc; ++o) {
                        const double x = s_ex[o];
                        above += (x > e || (x == e && s_cand[o] < p)) ? 1 : 0;
                    }
                    if (above >= L.topk) s_fatt[p] = 0;
                }
            }
        }
        lds_barrier();
        if (w == 0) {  // the prompt blocks holding a chosen page, ascending
            int cnt = 0;
            for (int c0 = 0; c0 < nbp; c0 += 64) {
                const int bb = c0 + lane;
                bool any = false;
                if (bb < nbp)
                    for (int sl = 32 * bb / ps; sl <= (32 * bb + 31) / ps; ++sl) any = any || s_fatt[sl] > 0;
                const unsigned long long m = __ballot(any);
                if (any) s_plist[cnt + __popcll(m & ((1ull << lane) - 1ull))] = bb;
                cnt += __popcll(m);
            }
            if (lane == 0) s_nsel = cnt;
        }
        lds_barrier();
        if (w >= nown) {  // no decode block for this wavefront: its first claim is a prompt block
            b = take(w);
            if (b < bend) {
                f_next = row_fill(b);
                load_block(b, kr_next, vr_next);
            }
        }
    }

    float m_run = -INFINITY, l_run = 0.0f;
    f32x4 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};

    // score passes of this wavefront: 8 pages each, page = first + (lane >> 3)
    const int part = lane & 7;
    const int ngroups = (sl1 - sl0 + 7) / 8;  // 8-page groups, in the step's direction
    auto pass_page = [&](int pass) {
        const int g = pass * NW + w;
        return sl0 + 8 * (L.rev ? ngroups - 1 - g : g) + (lane >> 3);
    };
    auto pass_act = [&](int p) { return p < sl1 && (p == ns || ranked(L, L.state[base + p])); };
    const int npass = (sl1 - sl0 - 8 * w > 0) ? (sl1 - sl0 - 8 * w + 8 * NW - 1) / (8 * NW) : 0;
    const int npass_all = (sl1 - sl0 + 8 * NW - 1) / (8 * NW);  // passes of wavefront 0, the most
    int pass = 0;
    ScoreFrag<T, D> frag;
    bool act_cur = false;
    auto score_step = [&]() {
        const int p = pass_page(pass);
        double* hb = (AGG && act_cur) ? (fused ? s_hb : L.score + base * G) + (size_t)p * G : nullptr;
        const double sc = score_finish<T, D>(L, u, p, part, act_cur, frag, p == ns, opened, s_kn, s_qf, hb);
        if (act_cur && part == 0 && !AGG) {
            if (fused) s_score[p] = sc;
            else publish(L.score + base + p, sc);
        }
        ++pass;
        if (pass < npass) {
            const int pn = pass_page(pass);
            act_cur = pass_act(pn);
            score_issue<T, D>(L, u, pn, part, act_cur && !(pn == ns && opened), frag);
        }
    };
    // retention policy once every wavefront's scores are in LDS
    auto scores_done = [&]() {
        lds_barrier();
        if (AGG && fused) softmax_sum_block<false>(L, s_hb, 1, s_state, s_score, s_mz, tid, NW * 64);
        // (after the block loop, as with the softmax aggregation, the retention
        // is on the critical path: its count skips the pinned pages; mid-loop
        // it overlaps the streaming, and the narrower count measured no faster)
        if (fused && w == 0)
            retention_wave<F32>(L, ur, r, s_score, s_state, s_ts, s_lid, ret,
                           AGG && !L.rank_pinned ? max(L.dbase, pinned) : L.dbase);
        decided = true;
    };

    // after the first block: the first pass's keys start loading
    auto staged = [&]() {
        if (npass > 0) {
            const int p = pass_page(0);
            act_cur = pass_act(p);
            score_issue<T, D>(L, u, p, part, act_cur && !(p == ns && opened), frag);
        }
    };
    // the first score pass's loads go out now, behind the first blocks' (L.early),
    // or once the first block has been attended and its registers are free
    const int early = L.early;
    if (early) staged();
    int it = 0;
    while (b < bend) {
        const int f_cur = f_next;
        u32x4 kr[NB], vr[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) kr[i] = kr_next[i];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) vr[nb] = vr_next[nb];
        // one claim per wavefront: from the LDS counter, or (L.det) a fixed
        // interleave, whose partial sums are reproducible
        int bn = bend;
        if (lane == 0) bn = take(L.det ? w + (it + 1) * NW : (it == 0 ? w + NW : atomicAdd(&s_next, 1)));
        bn = __builtin_amdgcn_readfirstlane(bn);
        if (bn < bend) {
            f_next = row_fill(bn);
            load_block(bn, kr_next, vr_next);
        }
        const int nv = valid_rows(b, f_cur);
        if (__ballot(nv > 0) != 0ull) {
            if (b == b_new) {  // the new token: K/V from the inputs
                if constexpr (F32) {
                    if (col == tt_new) {
#pragma unroll
                        for (int j = 0; j < NB; ++j) kr[j] = ld4(&s_kn[16 * j + 4 * grp]);
                    }
                    if (tg == (tt_new >> 2)) {
#pragma unroll
                        for (int tt = 0; tt < 4; ++tt)
                            if (tt == (tt_new & 3)) {
#pragma unroll
                                for (int h = 0; h < D / 64; ++h) vr[tt * (D / 64) + h] = ld4(&s_vn[64 * h + vcol]);
                            }
                    }
                    // append: the new token joins the pool (Algorithm 1, decode-stage store)
                    T* Kw = (T*)L.K + ((size_t)u * L.Lcap + row_new) * D;
                    T* Vw = (T*)L.V + ((size_t)u * L.Lcap + row_new) * D;
                    if (lane < D / 4) {
                        st4(Kw + 4 * lane, ld4(&s_kn[4 * lane]));
                        st4(Vw + 4 * lane, ld4(&s_vn[4 * lane]));
                    }
                } else {
                    const int i_new = 4 * (tt_new >> 3) + (tt_new & 3), q_new = (tt_new >> 2) & 1;
                    if (col == i_new) {
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks) {
                            const u32x4 x = ld4(&s_kn[32 * ks + 8 * grp]);
                            if (q_new == 0) kr[ks] = x; else kr[KS + ks] = x;
                        }
                    }
                    if (grp == (tt_new >> 3)) {
                        const int j_new = tt_new & 7;
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) {
                            const uint32_t val = s_vn[16 * nb + col];
#pragma unroll
                            for (int h = 0; h < 4; ++h) {
                                if ((j_new >> 1) == h) {
                                    const int sh = (j_new & 1) * 16;
                                    vr[nb][h] = (vr[nb][h] & ~(0xFFFFu << sh)) | (val << sh);
                                }
                            }
                        }
                    }
                    // append: the new token joins the pool (Algorithm 1, decode-stage store)
                    T* Kw = (T*)L.K + (size_t)u * L.Lcap * D;
                    T* Vw = (T*)L.V + (size_t)u * L.Lcap * D;
                    if (lane < D / 8) st4(Kw + k_off<D>(row_new, lane * 8), ld4(&s_kn[lane * 8]));
                    for (int c = lane; c < D; c += 64) Vw[v_off<D>(row_new, c)] = s_vn[c];
                }
            }

            if constexpr (F32)
                attend_block_f32<D, g4>(kr, vr, nv, s_qf + min(g4 ? lane & 3 : col, G - 1) * qpad_row(D), grp, scale_log2, m_run, l_run,
                                    acc);
            else
                attend_block<D>(kr, vr, nv, qv, scale_log2, m_run, l_run, acc);
        }
        // this block's registers are free again
        if (it == 0 && !early) {
            staged();
        } else if (pass < npass) {
            score_step();
        }
        // (the softmax aggregation waits for the end of the loop: mid-loop, its
        // arithmetic would compete with the prefetched block for registers;
        // wavefront 0, which has the most passes, has finished them here)
        if (!AGG && it == npass_all - early) scores_done();
        ++it;
        b = bn;
    }
    if (it == 0 && !early) staged();
    while (pass < npass) score_step();  // passes left when the wavefront ran out of blocks
    if (!decided) scores_done();

    // park this wavefront's partial attention in LDS
    const int head = g4 ? lane & 3 : col;
    if (g4) {
        l_run = sum_ror4_8(l_run);
    } else {
        l_run += __shfl_xor(l_run, 16);
        l_run += __shfl_xor(l_run, 32);
    }
    if (g4 ? lane < 4 : grp == 0) {
        s_m[w][head] = m_run;
        s_l[w][head] = l_run;
    }
    float* o = &s_o[((size_t)w * G + head) * (D + 4)];
    if constexpr (F32) {  // tile (h, e), row i: channel 64h + 16grp + 4i + e
        if (g4) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[nb][i] = sum_ror4_8(acc[nb][i]);
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int h = nb >> 2, i = nb & 3;
            if (head < G && (!g4 || tg == i))
                *reinterpret_cast<f32x4*>(o + 64 * h + 16 * grp + 4 * i) =
                    f32x4{acc[4 * h][i], acc[4 * h + 1][i], acc[4 * h + 2][i], acc[4 * h + 3][i]};
        }
    } else if (col < G) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) *reinterpret_cast<f32x4*>(o + 16 * nb + 4 * grp) = acc[nb];
    }
    lds_barrier();  // partials parked, retention decided
    // the state goes out first (every block has been read), its stores
    // draining while the partials merge
    if (fused) retention_store(L, io, u, ur, s_state, s_ts, s_lid, ret, tid, NW * 64);

    // merge the wavefronts' partial outputs
    for (int idx = tid; idx < G * D; idx += NW * 64) {
        const int h = idx / D, c = idx - (idx / D) * D;
        float M = -INFINITY;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) M = fmaxf(M, s_m[ww][h]);
        float O = 0.0f, Ls = 0.0f;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) {
            const float mw = s_m[ww][h];
            const float wt = (mw == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(mw - M);
            O += wt * s_o[((size_t)ww * G + h) * (D + 4) + c];
            Ls += wt * s_l[ww][h];
        }
        if (nsplit == 1) {  // the whole unit: the output itself
            ((T*)io.out)[((size_t)u * G + h) * D + c] = from_f<T>(O / Ls);
        } else {
            float* pp = L.part + (((size_t)u * nsplit + split) * G + h) * (D + 2);
            publish(pp + c, O);
            if (c == 0) {
                publish(pp + D, M);
                publish(pp + D + 1, Ls);
            }
        }
    }
    if constexpr (SPLIT) {
        // The last workgroup of the unit to get here finishes its step; with
        // one decision per sequence it merges the unit, and the last unit of
        // the sequence decides.
        __shared__ int s_last, s_aux[261];
        const int nu = L.hgrp;
        if ((nsplit > 1 || nu == 1) && !arrive_last(L.arrived + u, nsplit, &s_last)) return;
        if (nu > 1 && nsplit > 1) {
            const MergeFirst mf = merge_first(L, u, tid);
            merge_stage(L, u, mf, reinterpret_cast<float*>(smem), tid, NW * 64);
            __syncthreads();
            merge_out<T>(L, io, u, mf, reinterpret_cast<float*>(smem), tid, NW * 64);
        }
        if (nu > 1 && !arrive_last(L.arrived + L.U + u / nu, nu, &s_last)) return;
        finish_units<T>(L, io, r, u / nu * nu, nu, nu == 1 && nsplit > 1, smem, s_aux, ret, tid, NW * 64);
    }
}

// The step kernel of bf16 pools, work item blockIdx.x.
template <int D, int NW, bool AGG, int LM, bool NT, bool SPLIT>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_step_bf16(
    LayerView L, StepIO io, float scale_log2, double r) {
    step_item<uint16_t, D, NW, AGG, LM, NT, SPLIT, false>(L, io, scale_log2, r, blockIdx.x);
}

// fp32 pools; G4: groups of up to 4 heads (attend_block_f32)
template <int D, int NW, bool AGG, int LM, bool NT, bool SPLIT, bool G4>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_step_f32(
    LayerView L, StepIO io, float scale_log2, double r) {
    step_item<float, D, NW, AGG, LM, NT, SPLIT, G4>(L, io, scale_log2, r, blockIdx.x);
}

// Quest on the prompt pages (pools with a prompt region): for one unit, each
// kept prompt page's representative bound against the step's queries, max
// over the G heads of sum_c max(q_c kmax_c, q_c kmin_c) in fp64, channels
// summed in order; the topk pages of largest bound, ties to the lower slot,
// are attended. One thread per page reads the page's kmin/kmax rows with
// 16-byte loads and widens each key once for all heads; with q split into
// q+ = max(q, 0) and q- = min(q, 0), a channel's term is
// fma(q+, kmax, fma(q-, kmin, acc)): one of the two products is zero, which
// adds exactly, and the other is exact in fp64, so each bound rounds as the
// sequential sum does. Writes the fills the attention sees (0 for the other
// prompt pages) and the unit's block list: the prompt blocks holding a
// chosen page, ascending, then every block of the decode region. One
// workgroup per unit: 256 threads, 1024 when there are fewer units than CUs.
// GQ: the query group size G, a compile-time constant so that the head loop
// unrolls into straight-line fused multiply-adds.

template <typename T, int GQ>
__global__ __launch_bounds__(1024) void k_prompt_select(LayerView L, StepIO io) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int u = blockIdx.x, tid = threadIdx.x, lane = tid & 63, nth = blockDim.x;
    if (io.active != nullptr && io.active[u / L.nkv] == 0) return;
    constexpr int G = GQ;
    const int S = L.S, D = L.D, ps = L.ps, npr = L.dbase;
    const size_t base = (size_t)u * S;
    constexpr int V = 16 / sizeof(T);  // channels per 16-byte load
    double2* s_qpm = reinterpret_cast<double2*>(smem);                 // [G][D] (q+, q-)
    double* s_b = reinterpret_cast<double*>(s_qpm + (size_t)G * D);    // [npr] bounds
    int* s_sel = reinterpret_cast<int*>(s_b + npr);                    // [npr] chosen
    int* s_hist = s_sel + npr;  // [276] radix histogram, its pick, the count above theta, per-wavefront counts
    const int kp = L.unit[(size_t)u * kUnitFields + kPinnedPages];
    const T* qg = (const T*)io.q + (size_t)u * G * D;
    for (int i = tid; i < G * D; i += nth) {
        const double q = (double)to_f(qg[i]);
        s_qpm[i] = make_double2(q > 0.0 ? q : 0.0, q < 0.0 ? q : 0.0);
    }
    __syncthreads();
    const bool all = kp <= L.topk;
    for (int p = tid; p < kp && !all; p += nth) {
        const T* kx = (const T*)L.kmax + (base + p) * D;
        const T* kn = (const T*)L.kmin + (base + p) * D;
        double acc[G];
#pragma unroll
        for (int j = 0; j < G; ++j) acc[j] = 0.0;
#pragma unroll 4
        for (int c = 0; c < D; c += V) {
            const u32x4 xv = ld4(kx + c), nv = ld4(kn + c);
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const double hi = (double)vec_elem<T>(xv, e), lo = (double)vec_elem<T>(nv, e);
#pragma unroll
                for (int j = 0; j < G; ++j) {
                    const double2 qpm = s_qpm[j * D + c + e];
                    acc[j] = fma(qpm.x, hi, fma(qpm.y, lo, acc[j]));
                }
            }
        }
        double best = -INFINITY;
#pragma unroll
        for (int j = 0; j < G; ++j) best = fmax(best, acc[j]);
        s_b[p] = best;
    }
    __syncthreads();
    // the topk pages of largest bound, ties to the lower slot. Up to 256
    // pages, each page is ranked against all others; beyond (the count is
    // quadratic in the pages), theta, the topk-th largest bound (counted with
    // multiplicity), by a radix select, then every page above it and, of
    // those equal to it, the lowest slots, as many as are left (a prefix
    // count in slot order): the same pages.
    if (all || kp <= 256) {
        for (int p = tid; p < npr; p += nth) {
            bool sel = p < kp;
            if (sel && !all) {
                const double bp = s_b[p];
                int above = 0;
                for (int o = 0; o < kp; ++o) above += (s_b[o] > bp || (s_b[o] == bp && o < p)) ? 1 : 0;
                sel = above < L.topk;
            }
            s_sel[p] = sel ? 1 : 0;
        }
    } else {
        const double theta = kth_largest_f64_wg(s_b, kp, L.topk, s_hist, tid, nth);
        if (tid == 0) s_hist[258] = 0;
        __syncthreads();
        int gt = 0;
        for (int p = tid; p < kp; p += nth) gt += s_b[p] > theta ? 1 : 0;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) gt += __shfl_xor(gt, off);
        if (lane == 0 && gt) atomicAdd(&s_hist[258], gt);
        __syncthreads();
        const int need = L.topk - s_hist[258], w = tid >> 6, nw = nth >> 6;
        int run = 0;  // tied pages in the slots before this chunk
        for (int c0 = 0; c0 < kp; c0 += nth) {
            const int p = c0 + tid;
            const bool eq = p < kp && s_b[p] == theta;
            const unsigned long long m = __ballot(eq);
            if (lane == 0) s_hist[259 + w] = __popcll(m);
            __syncthreads();
            int before = run + __popcll(m & ((1ull << lane) - 1ull)), tot = 0;
            for (int ww = 0; ww < nw; ++ww) {
                const int cw = s_hist[259 + ww];
                tot += cw;
                before += ww < w ? cw : 0;
            }
            if (p < kp) s_sel[p] = (s_b[p] > theta || (eq && before < need)) ? 1 : 0;
            run += tot;
            __syncthreads();
        }
        for (int p = kp + tid; p < npr; p += nth) s_sel[p] = 0;
    }
    __syncthreads();
    for (int p = tid; p < npr; p += nth) L.fill_att[base + p] = s_sel[p] ? L.fill[base + p] : 0;
    for (int s = npr + tid; s < S; s += nth) L.fill_att[base + s] = L.fill[base + s];
    __syncthreads();
    if (tid < 64) {
        const int nbp = npr * ps / 32;  // prompt blocks (the region is a whole number of blocks)
        int32_t* bl = L.blist + (size_t)u * L.lcap_blk;
        int cnt = 0;
        for (int c0 = 0; c0 < nbp; c0 += 64) {
            const int b = c0 + lane;
            bool any = false;
            if (b < nbp)
                for (int s = 32 * b / ps; s <= (32 * b + 31) / ps; ++s) any = any || s_sel[s] != 0;
            const unsigned long long m = __ballot(any);
            if (any) bl[cnt + __popcll(m & ((1ull << lane) - 1ull))] = b;
            cnt += __popcll(m);
        }
        for (int b = nbp + lane; b < L.nblk; b += 64) bl[cnt + b - nbp] = b;
        if (lane == 0) {
            L.bcnt[2 * u] = cnt;
            L.bcnt[2 * u + 1] = cnt + max(0, L.nblk - nbp);
        }
    }
}

// The kept prompt pages' bound intervals (prompt_bounds) into L.pivl, for
// units too few to fill the chip: one wavefront per L.pchunk pages of a
// unit, so that the pages' representative keys stream through many CUs;
// nothing for units with no more kept pages than topk.
template <int D>
__global__ __launch_bounds__(64) void k_prompt_intervals(LayerView L, StepIO io) {
    constexpr int KS = D / 32;
    const int nch = (L.dbase + L.pchunk - 1) / L.pchunk;
    const int u = blockIdx.x / nch, ch = blockIdx.x - u * nch;
    if (io.active != nullptr && io.active[u / L.nkv] == 0) return;
    const int kp = L.unit[(size_t)u * kUnitFields + kPinnedPages], p0 = ch * L.pchunk;
    if (kp <= L.topk || p0 >= kp) return;
    const int n = min(L.pchunk, kp - p0), lane = threadIdx.x, grp = lane >> 4, col = lane & 15;
    const uint16_t* qg = (const uint16_t*)io.q + (size_t)u * L.G * D;
    bf16x8 qv[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const u32x4 x = (col < L.G) ? ld4_in(qg + (size_t)col * D + 32 * ks + 8 * grp) : u32x4{0u, 0u, 0u, 0u};
        qv[ks] = __builtin_bit_cast(bf16x8, x);
    }
    float* lo = L.pivl + (size_t)u * L.dbase + p0;
    prompt_bounds<D, 1>(L, (size_t)u * L.S + p0, n, qv, lo, lo + (size_t)L.U * L.dbase, [] {});
}

// The same selection for bf16 pools, on the MFMA: each kept prompt page's
// bound as an interval (prompt_bounds), lo_cut the topk-th largest lower end,
// and the candidates, the pages whose upper end reaches lo_cut; at least
// topk pages have bounds >= lo_cut, so every other page ranks below all of
// them. Only the candidates' bounds are taken exactly (fp64, as the decode
// pages' scores), and the topk among them, ties to the lower slot, are the
// chosen pages. Then the fills and the block list, as above, the list's
// positions by a prefix count over the whole workgroup. One workgroup of
// NW wavefronts per unit. With L.pchunk > 0 the intervals come from
// k_prompt_intervals, launched just before.
template <int D, int NW>
__global__ __launch_bounds__(NW * 64) void k_prompt_select_mfma(LayerView L, StepIO io) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_lo, s_ncand, s_wc[NW];
    constexpr int KS = D / 32, NT = NW * 64;
    const int u = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6, grp = lane >> 4, col = lane & 15;
    if (io.active != nullptr && io.active[u / L.nkv] == 0) return;
    const int G = L.G, S = L.S, ps = L.ps, npr = L.dbase;
    const size_t base = (size_t)u * S;
    float* s_qf = reinterpret_cast<float*>(smem);     // [G][qpad_row(D)] q in fp32 (a multiple of 16 bytes)
    float* s_plo = s_qf + (size_t)G * qpad_row(D);    // [npr] bound intervals (16-byte reads of s_plo)
    float* s_phi = s_plo + npr;
    double* s_ex = reinterpret_cast<double*>(s_phi + npr);  // [npr] candidates' exact bounds
    int* s_cand = reinterpret_cast<int*>(s_ex + npr);       // [npr] candidates
    int* s_sel = s_cand + npr;                          // [npr] chosen
    int* s_hist = s_sel + npr;                          // [258] radix histogram and its pick
    const int kp = L.unit[(size_t)u * kUnitFields + kPinnedPages];
    const bool all = kp <= L.topk;
    // lane (grp, col < G): head col's channels 32 ks + 8 grp .. +7, the MFMA's query operands
    const uint16_t* qg = (const uint16_t*)io.q + (size_t)u * G * D;
    bf16x8 qv[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const u32x4 x = (col < G) ? ld4_in(qg + (size_t)col * D + 32 * ks + 8 * grp) : u32x4{0u, 0u, 0u, 0u};
        qv[ks] = __builtin_bit_cast(bf16x8, x);
    }
    for (int p = tid; p < npr; p += NT) s_sel[p] = p < kp ? 1 : 0;
    if (tid == 0) {
        s_lo = 0x7FFFFFFF;
        s_ncand = 0;
    }
    if (!all) {
        // q in fp32 for the exact bounds, the wavefronts taking turns over ks
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks % NW == w && col < G) {
                const u32x4 x = __builtin_bit_cast(u32x4, qv[ks]);
                float* d = s_qf + qpad_index<D>(col * D + 32 * ks + 8 * grp);
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    d[2 * h] = __uint_as_float(x[h] << 16);
                    d[2 * h + 1] = __uint_as_float(x[h] & 0xFFFF0000u);
                }
            }
        }
        if (L.pchunk > 0) {
            const float* glo = L.pivl + (size_t)u * npr;
            const float* ghi = glo + (size_t)L.U * npr;
            for (int p = tid; p < kp; p += NT) {
                s_plo[p] = glo[p];
                s_phi[p] = ghi[p];
            }
        } else {
            prompt_bounds<D, NW>(L, base, kp, qv, s_plo, s_phi, [] {});
        }
    }
    __syncthreads();
    if (!all) {
        float lo_cut;
        if (kp > 256) {  // (the count is quadratic in the pages)
            lo_cut = kth_largest_wg<NT>(s_plo, kp, L.topk, s_hist, tid);
        } else {
            const int kp4 = kp & ~3;
            for (int p = tid; p < kp; p += NT) {
                const float lp = s_plo[p];
                int above = 0;  // lower ends above p's: four per 16-byte read, then the last few
#pragma unroll 4
                for (int o = 0; o < kp4; o += 4) {
                    const float4 x = *reinterpret_cast<const float4*>(s_plo + o);
                    above += (x.x > lp ? 1 : 0) + (x.y > lp ? 1 : 0) + (x.z > lp ? 1 : 0) + (x.w > lp ? 1 : 0);
                }
                for (int o = kp4; o < kp; ++o) above += s_plo[o] > lp ? 1 : 0;
                if (above < L.topk) atomicMin(&s_lo, float_order(lp));
            }
            __syncthreads();
            lo_cut = order_float(s_lo);
        }
        for (int p = tid; p < kp; p += NT) {
            if (s_phi[p] >= lo_cut) s_cand[atomicAdd(&s_ncand, 1)] = p;
            else s_sel[p] = 0;
        }
        __syncthreads();
        // exactly topk candidates: they are the top k; more: their bounds in
        // fp64, eight lanes per page, and the topk of those
        const int nc = s_ncand;
        if (nc > L.topk) {
            for (int c0 = 8 * w; c0 < nc; c0 += 8 * NW) {
                const int c = c0 + (lane >> 3);
                const bool act = c < nc;
                const int p = act ? s_cand[c] : 0;
                ScoreFrag<uint16_t, D> f;
                score_issue<uint16_t, D>(L, u, p, lane & 7, act, f);
                const double sc = score_finish<uint16_t, D>(L, u, p, lane & 7, act, f, false, false, nullptr, s_qf, nullptr);
                if (act && (lane & 7) == 0) s_ex[c] = sc;
            }
            __syncthreads();
            for (int c = tid; c < nc; c += NT) {
                const int p = s_cand[c];
                const double e = s_ex[c];
                int above = 0;
                for (int o = 0; o < nc; ++o) {
                    const double x = s_ex[o];
                    above += (x > e || (x == e && s_cand[o] < p)) ? 1 : 0;
                }
                if (above >= L.topk) s_sel[p] = 0;
            }
        }
    }
    __syncthreads();
    for (int p = tid; p < npr; p += NT) L.fill_att[base + p] = s_sel[p] ? L.fill[base + p] : 0;
    for (int sl = npr + tid; sl < S; sl += NT) L.fill_att[base + sl] = L.fill[base + sl];
    // the prompt blocks holding a chosen page, ascending (a block's place: the
    // chosen blocks before it, in its wavefront and in the ones before), then
    // every block of the decode region
    const int nbp = npr * ps / 32;
    int32_t* bl = L.blist + (size_t)u * L.lcap_blk;
    int run = 0;
    for (int c0 = 0; c0 < nbp; c0 += NT) {
        const int bb = c0 + tid;
        bool any = false;
        if (bb < nbp)
            for (int sl = 32 * bb / ps; sl <= (32 * bb + 31) / ps; ++sl) any = any || s_sel[sl] != 0;
        const unsigned long long m = __ballot(any);
        if (lane == 0) s_wc[w] = __popcll(m);
        __syncthreads();
        int before = run + __popcll(m & ((1ull << lane) - 1ull)), tot = 0;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) {
            tot += s_wc[ww];
            before += ww < w ? s_wc[ww] : 0;
        }
        if (any) bl[before] = bb;
        run += tot;
        __syncthreads();
    }
    for (int b = nbp + tid; b < L.nblk; b += NT) bl[run + b - nbp] = b;
    if (tid == 0) {
        L.bcnt[2 * u] = run;
        L.bcnt[2 * u + 1] = run + max(0, L.nblk - nbp);
    }
}

// LDS of the step kernel: the queries in fp32, the attention wavefronts'
// partial outputs, the fused retention's slot arrays (with the per-head
// bounds of the softmax aggregation), and a block list
size_t step_lds(int G, int D, int S, int NW, bool fused, int agg, int list_ints) {
    size_t b = (size_t)4 * G * qpad_row(D) + (size_t)NW * G * (D + 4) * 4;
    if (fused) b += (size_t)S * 20 + (agg ? (size_t)S * G * 8 + (size_t)G * 16 : 0);
    return b + (size_t)list_ints * 4;
}

// Every instance of the step kernel for one type, head_dim and workgroup size.
// f(pointer) is called for the one that the layer and plan ask for, or (all)
// for each. Workgroups of 2 wavefronts always cover their unit (plan_step: from
// kSmallWorkUnits on), so they have no split instances.
template <typename T, int D, int NW, bool G4, class F>
void each_step(bool all, bool agg, int lm, bool nt, bool split, F&& f) {
    auto one = [&](auto A, auto M, auto N, auto P) {
        if (all || (agg == A.value && lm == M.value && nt == N.value && split == P.value)) {
            if constexpr (sizeof(T) == 2) f(k_step_bf16<D, NW, A.value, M.value, N.value, P.value>);
            else f(k_step_f32<D, NW, A.value, M.value, N.value, P.value, G4>);
        }
    };
    auto nts = [&](auto A, auto M, auto P) {
        if constexpr (NW > 2 || !P.value) {
            one(A, M, std::false_type{}, P);
            one(A, M, std::true_type{}, P);
        }
    };
    const std::integral_constant<int, 0> m0{};
    const std::integral_constant<int, 1> m1{};
    const std::integral_constant<int, 2> m2{};
    const std::true_type yes{};
    const std::false_type no{};
    nts(no, m0, no);
    nts(no, m0, yes);
    nts(no, m1, yes);
    if constexpr (sizeof(T) == 2) nts(no, m2, no);  // (a fused bf16 plan without the softmax aggregation selects in the step)
    else nts(no, m1, no);
    nts(yes, m0, no);
    nts(yes, m0, yes);
    nts(yes, m1, no);
    nts(yes, m1, yes);
}

}  // namespace

template <typename T, int D, int NW, bool G4>
hipError_t launch_step_inst(const LayerView& L, const StepIO& io, const StepPlan& pl, float sl2, double r,
                            hipStream_t s) {
    const int lm = pl.select_in_step ? 2 : L.topk >= 0 ? 1 : 0;
    bool found = false;
    each_step<T, D, NW, G4>(false, L.agg != 0, lm, L.nt != 0, !pl.fused, [&](auto* kernel) {
        found = true;
        hipLaunchKernelGGL(kernel, dim3((unsigned)(L.U * pl.nsplit)), dim3(NW * 64), pl.lds, s, L, io, sl2, r);
    });
    return found ? hipGetLastError() : hipErrorInvalidDeviceFunction;
}

template <typename T, int D, int NW, bool G4>
hipError_t allow_lds_all(int bytes) {
    hipError_t e = hipSuccess;
    each_step<T, D, NW, G4>(true, false, 0, false, false, [&](auto* kernel) {
        hipError_t r = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (r != hipSuccess) e = r;
    });
    return e;
}

// This file is compiled once for each RAAS_PART (in parallel): parts 1 and up
// hold the instances of the step kernel, part 0 everything else.
#if RAAS_PART == 0
#define RAAS_STEP(T, D, NW, G4)                                                                                 \
    extern template hipError_t launch_step_inst<T, D, NW, G4>(const LayerView&, const StepIO&, const StepPlan&, \
                                                              float, double, hipStream_t);                      \
    extern template hipError_t allow_lds_all<T, D, NW, G4>(int);
#else
#define RAAS_STEP(T, D, NW, G4)                                                                                   \
    template hipError_t launch_step_inst<T, D, NW, G4>(const LayerView&, const StepIO&, const StepPlan&, float,   \
                                                       double, hipStream_t);                                      \
    template hipError_t allow_lds_all<T, D, NW, G4>(int);
#endif
#if RAAS_PART == 0 || RAAS_PART == 1
RAAS_STEP(uint16_t, 128, 8, false)
#endif
#if RAAS_PART == 0 || RAAS_PART == 2
RAAS_STEP(uint16_t, 128, 4, false)
#endif
#if RAAS_PART == 0 || RAAS_PART == 3
RAAS_STEP(uint16_t, 128, 2, false)
#endif
#if RAAS_PART == 0 || RAAS_PART == 4
RAAS_STEP(uint16_t, 64, 8, false)
#endif
#if RAAS_PART == 0 || RAAS_PART == 5
RAAS_STEP(uint16_t, 64, 4, false)
#endif
#if RAAS_PART == 0 || RAAS_PART == 6
RAAS_STEP(uint16_t, 64, 2, false)
#endif
#if RAAS_PART == 0 || RAAS_PART == 7
RAAS_STEP(float, 128, 8, false)
#endif
#if RAAS_PART == 0 || RAAS_PART == 8
RAAS_STEP(float, 128, 8, true)
#endif
#if RAAS_PART == 0 || RAAS_PART == 9
RAAS_STEP(float, 128, 4, false)
#endif
#if RAAS_PART == 0 || RAAS_PART == 10
RAAS_STEP(float, 128, 4, true)
#endif
#if RAAS_PART == 0 || RAAS_PART == 11
RAAS_STEP(float, 64, 8, false)
#endif
#if RAAS_PART == 0 || RAAS_PART == 12
RAAS_STEP(float, 64, 8, true)
#endif
#if RAAS_PART == 0 || RAAS_PART == 13
RAAS_STEP(float, 64, 4, false)
#endif
#if RAAS_PART == 0 || RAAS_PART == 14
RAAS_STEP(float, 64, 4, true)
#endif

#if RAAS_PART == 0
// ---------------------------------------------------------------------------

// One fused workgroup per unit, or the unit's blocks split over several
// workgroups, the last of which finishes the step. A split workgroup pays for
// its start and for publishing (about 8 us, of which the last one's finish is
// 4), so splits pay only where they put idle CUs to work, in one round:
// 256 / U workgroups per unit at most, and none from 129 units on (fused / in
// two, cold: 129 units, 64 blocks 30.6 / 49.8, 256 blocks 95.3 / 129.8; 160
// units, 128 blocks 55.6 / 79.8; 192 units, L 8192: 118 against 137 to 163 at
// any split). Below, a unit is split when it has more blocks than
// fused_limit: kFusedBlocks where idle CUs stream what one would have to, more
// where the publishing, which grows with G, or head_dim 64's shorter blocks
// leave less to gain, and more again for many units that are still cached.
// us per step, fused / split, page 16, one pool alone (cached) and 0.8 GB of
// pools in turn (cold):
//   G 4    8 units, 40 blocks  14.7 / 14.0 cached, 15.9 / 14.5 cold
//         32 units, 48 blocks  16.2 / 15.5, 22.3 / 17.1
//         48 units, 33 blocks  14.5 / 14.5, 18.6 / 17.1
//         64 units, 40 blocks  15.3 / 15.8, 21.1 / 18.9
//         64 units, 48 blocks  16.4 / 16.3 (three in turn, still cached, 17.4 / 18.9), 23.4 / 19.9
//        112 units, 48 blocks  18.5 / 20.5, 25.1 / 24.6
//   G 8    8 units, 40 blocks  16.3 / 16.7, 17.4 / 17.1
//         64 units, 48 blocks  18.0 / 19.4, 24.8 / 22.3
//   G 16   8 units, 48 blocks  20.2 / 22.5, 21.5 / 22.9
//         32 units, 48 blocks  20.7 / 23.7, 26.7 / 25.3
//   G 7, head_dim 64: 8 units, 48 blocks 12.7 / 13.3, 12.9 / 13.3; 64 units 13.0 / 14.4, 15.6 / 16.3
// Two workgroups per unit still fit the chip's 256 CUs up to 128 units, but
// from kHalfUnits on the first of them no longer gains enough when cold for what
// it loses when cached, up to kFusedBlocksHalf blocks (G 4, fused / split: 112
// units, 64 blocks 22.4 / 24.3 cached, 32.1 / 29.4 cold; 120 units 23.2 / 25.2,
// 33.2 / 30.7; 124 units 24.0 / 26.3, 31.8 / 31.0; 128 units 24.2 / 26.4, 30.6
// / 32.1; 120 units, 56 blocks 21.1 / 23.1, 28.2 / 27.9; 116 units, 49 blocks
// 19.2 / 21.0, 25.6 / 25.3; 128 units, 256 blocks 95.4 / 91.1 cold). More than
// kSplits splits, or fewer than 8 blocks in one, no longer help (8 units: 64
// blocks 15.1 in 8 and 15.3 in 16; 256 blocks 26.1 in 4, 21.3 in 8, 19.2 in 16,
// 21.0 in 32). An fp32 block costs more arithmetic, so fp32 units split at half
// as many (8 units, 32 blocks 18.9 / 14.2; 64 units 22.0 / 18.8; 128 units, 32
// blocks 25.5 / 27.0, 64 blocks 38.6 / 37.5).
constexpr int kFusedBlocks = 32;
constexpr int kHalfUnits = 113;
constexpr int kFusedBlocksHalf = 64;
constexpr int kSplits = 16;
// Up to this many blocks per wavefront (in pools of at most kFewSlots slots,
// kFewSlotsBlocksPerWave) raas_decode_step_static leaves its fixed array alone:
// such a unit's split keeps its scratch in the pool's buffers, so that these
// steps may overlap other pools' as they may in one workgroup.
constexpr int kSmallBlocksPerWave = 6;
constexpr int kFewSlotsBlocksPerWave = 8;
constexpr int kFewSlots = 64;
// With a prompt region and fewer units than CUs, fused up to this many
// attended blocks per wavefront and prompt pages. us per step, page 16, the
// decode blocks and 8 chosen ones, fused / split (intervals, selection, step),
// cached:
//     8 units, 128 pages  20.8 / 25.7 at 16 blocks, 25.1 / 26.8 at 40, 31.9 / 27.8 at 72
//     8 units, 512 pages  30.8 / 29.0, 35.1 / 30.1, 41.5 / 30.9
//     8 units, 640 pages  41.5 / 30.0, 46.2 / 30.6, 52.8 / 31.7
//    64 units, 256 pages  24.7 / 30.6, 29.4 / 33.9, 36.5 / 38.4
//    64 units, 512 pages  31.8 / 32.9, 36.6 / 37.5, 43.7 / 41.6
//    64 units, 640 pages  43.6 / 35.4, 48.5 / 39.9, 56.0 / 44.3
//   128 units, 512 pages  32.5 / 39.0, 38.4 / 44.8, 50.5 / 54.6
// The pages' line lies between 512 and 640 for all of them. The blocks' line was
// drawn against a split step of two kernels; now that it is one, 8 units would be
// faster split from about 60 attended blocks on (the static entry point's
// selection, without the interval kernel, is slower than these figures from 257
// pages on), and it stands where it was.
constexpr int kFusedPromptBlocksPerWave = 12;
constexpr int kFusedPromptPages = 512;

// Workgroups of 2 wavefronts, four per CU, from this many units on when a
// unit's step attends at most kSmallWorkBlocks blocks (same box, batch 128,
// page 32: L 512 45.1 -> 42.7 us, L 512 plus the top 8 prompt pages 114.4 ->
// 101.8 us; L 2048, 64 blocks, 170.1 -> 173.4 us, so longer pools keep 4).
constexpr int kSmallWorkUnits = 1024;
constexpr int kSmallWorkBlocks = 32;

// Most blocks that one workgroup attends for a unit (the measurements are at
// kFusedBlocks). long_prompt: a prompt region of more than kFusedPromptPages,
// whose slots the last workgroup of a split unit would all read again (64
// units, 40 blocks: 1536 pages 52.5 us fused; 1664 pages, which no longer fit
// one workgroup's LDS with the softmax aggregation's bounds, 56.5 split).
int fused_limit(int U, int G, int D, int S, bool bf16, bool long_prompt, bool cold) {
    if (!bf16) return (U < kHalfUnits ? kFusedBlocks : kFusedBlocksHalf) / 2;
    if (U >= kHalfUnits) return kFusedBlocksHalf;
    const int most = S <= kFewSlots ? 64 : 48;
    if (long_prompt) return most;
    if (D == 64) return G <= 8 && U <= (cold ? 64 : 16) ? 48 : most;
    if (cold) return G <= 8 ? (U <= 48 ? kFusedBlocks : 39) : U <= 64 ? 47 : most;
    if (G <= 4) return U <= 32 ? kFusedBlocks : U <= 48 ? 48 : most;
    return U <= 16 ? (G <= 8 ? 40 : std::min(56, most)) : most;
}

StepPlan plan_step(int U, int G, int D, int S, int Lcap, int work_blocks, bool bf16, int agg,
                   bool grouped, int list_ints, int split_override, int npr, int nkv, bool cold) {
    StepPlan pl{};
    const int nblk = Lcap / kBlockTokens;
    // blocks of 16 KB (head_dim 128): 32 tokens in bf16, 16 in fp32
    const int blocks = bf16 ? nblk : 2 * nblk, work = bf16 ? work_blocks : 2 * work_blocks;
    int want;
    pl.waves = bf16 ? 2 : 4;
    for (int nw : {8, 4}) {
        if (step_lds(G, D, S, nw, false, agg, list_ints) <= kMaxLds) {
            pl.waves = nw;
            break;
        }
    }
    // more units than CUs: workgroups of 4 wavefronts, two per CU, so that
    // one unit's serial phases (staging, selection, retention) overlap
    // another's streaming, and up to 512 units run in one round (288 units,
    // L 1024: 45.4 -> 39.0 us; 352 units, L 8192: 254 -> 242; 504 units,
    // L 2048: 90.5 -> 87.5)
    if (split_override <= 0 && U > 256 && pl.waves == 8 &&
        2 * step_lds(G, D, S, 4, !grouped, agg, list_ints) <= kMaxLds)
        pl.waves = 4;
    // four or more units per CU, each with little to stream: four
    // workgroups per CU overlap more units' serial phases
    if (split_override <= 0 && bf16 && !grouped && U >= kSmallWorkUnits && work <= kSmallWorkBlocks &&
        pl.waves == 4 && 4 * step_lds(G, D, S, 2, true, agg, list_ints) <= kMaxLds)
        pl.waves = 2;
    const bool fits = !grouped && step_lds(G, D, S, pl.waves, true, agg, list_ints) <= kMaxLds;
    const bool many_prompt_slots = list_ints > 0 && npr > kFusedPromptPages;
    const int fused_blocks = fused_limit(U, G, D, S, bf16, many_prompt_slots, cold);
    if (split_override > 0) {
        want = split_override;
    } else if (fits && bf16 && list_ints > 0 && !agg && U < 256 && npr <= kFusedPromptPages &&
               work <= kFusedPromptBlocksPerWave * pl.waves) {
        // a short prompt region: the fused workgroup chooses its prompt
        // pages itself and attends the chosen blocks and the decode ones,
        // which saves the selection kernel's launch as well
        want = 1;
    } else if (fits && work <= fused_blocks && (!many_prompt_slots || agg || !bf16)) {
        want = 1;
    } else {
        want = std::min(std::min(std::max(256 / U, 1), kSplits), (work + 7) / 8);
    }
    want = want < 1 ? 1 : want;
    want = want > kMaxSplits ? kMaxSplits : want;
    want = want > nblk ? nblk : want;
    pl.bps = (nblk + want - 1) / want;
    pl.nsplit = (nblk + pl.bps - 1) / pl.bps;
    // (fused, a bf16 step with fewer units than CUs would bound a long prompt
    // region on one CU per unit: the selection kernels do that faster)
    const bool long_prompt = bf16 && list_ints > 0 && !agg && U < 256 && npr > kFusedPromptPages;
    pl.fused = !grouped && !long_prompt && pl.nsplit == 1 &&
               step_lds(G, D, S, pl.waves, true, agg, list_ints) <= kMaxLds;
    pl.pool_scratch = fits && split_override <= 0 &&
                      (blocks <= kSmallBlocksPerWave * pl.waves ||
                       (S <= kFewSlots && blocks <= kFewSlotsBlocksPerWave * pl.waves));
    pl.lds = step_lds(G, D, S, pl.waves, pl.fused, agg, list_ints);
    // (the workgroup that finishes a split unit reuses the step's LDS)
    if (!pl.fused) pl.lds = std::max(pl.lds, finish_lds(G, S, pl.nsplit, agg, grouped ? nkv : 1));
    // a fused workgroup covers its unit, so it can choose the prompt pages
    // itself (the softmax aggregation keeps the selection kernel)
    pl.select_in_step = bf16 && pl.fused && list_ints > 0 && !agg;
    return pl;
}

hipError_t allow_large_lds(bool bf16, int D, int G) {
    const int bytes = (int)kMaxLds;
    if (bf16) {
        hipError_t e = hipSuccess;
        for (hipError_t r : {D == 128 ? allow_lds_all<uint16_t, 128, 8, false>(bytes) : allow_lds_all<uint16_t, 64, 8, false>(bytes),
                             D == 128 ? allow_lds_all<uint16_t, 128, 4, false>(bytes) : allow_lds_all<uint16_t, 64, 4, false>(bytes),
                             D == 128 ? allow_lds_all<uint16_t, 128, 2, false>(bytes) : allow_lds_all<uint16_t, 64, 2, false>(bytes)})
            if (r != hipSuccess) e = r;
        return e;
    }
    auto f32 = [&](auto d, auto g4) {
        constexpr int DD = decltype(d)::value;
        constexpr bool G4 = decltype(g4)::value;
        const hipError_t r = allow_lds_all<float, DD, 8, G4>(bytes), q = allow_lds_all<float, DD, 4, G4>(bytes);
        return r != hipSuccess ? r : q;
    };
    const std::integral_constant<int, 128> d128{};
    const std::integral_constant<int, 64> d64{};
    const std::true_type yes{};
    const std::false_type no{};
    if (G <= 4) return D == 128 ? f32(d128, yes) : f32(d64, yes);
    return D == 128 ? f32(d128, no) : f32(d64, no);
}

template <typename T, int GQ>
void launch_select_g(const LayerView& L, const StepIO& io, size_t shm, hipStream_t stream) {
    // fewer units than CUs: a unit's pages over more threads
    hipLaunchKernelGGL((k_prompt_select<T, GQ>), dim3(L.U), dim3(L.U < 256 ? 1024 : 256), shm, stream, L, io);
}

template <typename T, int... GS>
void launch_select_t(const LayerView& L, const StepIO& io, size_t shm, hipStream_t stream,
                     std::integer_sequence<int, GS...>) {
    ((L.G == GS + 1 ? launch_select_g<T, GS + 1>(L, io, shm, stream) : void()), ...);
}

template <int D>
void launch_select_mfma(const LayerView& L, const StepIO& io, hipStream_t stream) {
    // q in fp32 (padded rows), per prompt slot the interval, the exact bound,
    // the candidate and the chosen flag, and the radix histogram
    const size_t shm = (size_t)L.G * qpad_row(D) * 4 + (size_t)L.dbase * 24 + 258 * 4;
    if (L.pchunk > 0) {
        const int nch = (L.dbase + L.pchunk - 1) / L.pchunk;
        hipLaunchKernelGGL((k_prompt_intervals<D>), dim3(L.U * nch), dim3(64), 0, stream, L, io);
    }
    // fewer units than CUs: 8 wavefronts per unit; four units per CU and
    // more: 2, so that more units are resident at once
    if (L.U < 256)
        hipLaunchKernelGGL((k_prompt_select_mfma<D, 8>), dim3(L.U), dim3(512), shm, stream, L, io);
    else if (L.U < 1024)
        hipLaunchKernelGGL((k_prompt_select_mfma<D, 4>), dim3(L.U), dim3(256), shm, stream, L, io);
    else
        hipLaunchKernelGGL((k_prompt_select_mfma<D, 2>), dim3(L.U), dim3(128), shm, stream, L, io);
}

hipError_t launch_prompt_select(const LayerView& L, const StepIO& io, hipStream_t stream) {
    if (L.bf16) {
        if (L.D == 128)
            launch_select_mfma<128>(L, io, stream);
        else
            launch_select_mfma<64>(L, io, stream);
        return hipGetLastError();
    }
    // q split in two (16 B per element), the bounds and the chosen flags, the
    // radix histogram and its counts
    const size_t shm = (size_t)L.G * L.D * 16 + (size_t)L.dbase * 12 + 276 * 4;
    launch_select_t<float>(L, io, shm, stream, std::make_integer_sequence<int, 16>{});
    return hipGetLastError();
}

template <typename T, int D>
void launch_prefill_t(const LayerView& L, const void* k, const void* v, const PrefillIn& in, int max_tok,
                      hipStream_t stream) {
    const bool reps = L.rank_pinned || L.topk >= 0;
    const int tile = prefill_tile<T, D>(), tiles = reps ? std::max(1, L.ps / tile) : 1;
    const int per = kPrefillWaves * tiles * tile;  // tokens of a workgroup
    const int chunks = std::max(1, (max_tok + per - 1) / per);
    const dim3 grid((unsigned)((size_t)L.U * chunks)), block(kPrefillWaves * 64);
    if (reps)
        hipLaunchKernelGGL((k_prefill<T, D, true>), grid, block, 0, stream, L, (const T*)k, (const T*)v, in, chunks, tiles);
    else
        hipLaunchKernelGGL((k_prefill<T, D, false>), grid, block, 0, stream, L, (const T*)k, (const T*)v, in, chunks, tiles);
}

hipError_t launch_prefill(const LayerView& L, const void* k, const void* v, const PrefillIn& in, int max_tok,
                          hipStream_t stream) {
    if (L.bf16 && L.D == 128) launch_prefill_t<uint16_t, 128>(L, k, v, in, max_tok, stream);
    else if (L.bf16) launch_prefill_t<uint16_t, 64>(L, k, v, in, max_tok, stream);
    else if (L.D == 128) launch_prefill_t<float, 128>(L, k, v, in, max_tok, stream);
    else launch_prefill_t<float, 64>(L, k, v, in, max_tok, stream);
    return hipGetLastError();
}

hipError_t launch_step(const LayerView& L, const StepIO& io, const StepPlan& plan, double r, hipStream_t s) {
    const float sl2 = (float)(1.4426950408889634 / sqrt((double)L.D));
    auto waves = [&](auto d, auto t, auto g4) {
        using T = decltype(t);
        constexpr int D = decltype(d)::value;
        constexpr bool G4 = decltype(g4)::value;
        if (plan.waves == 8) return launch_step_inst<T, D, 8, G4>(L, io, plan, sl2, r, s);
        if constexpr (sizeof(T) == 2)
            if (plan.waves == 2) return launch_step_inst<T, D, 2, G4>(L, io, plan, sl2, r, s);
        return launch_step_inst<T, D, 4, G4>(L, io, plan, sl2, r, s);
    };
    const std::integral_constant<int, 128> d128{};
    const std::integral_constant<int, 64> d64{};
    const std::true_type yes{};
    const std::false_type no{};
    if (L.bf16) return L.D == 128 ? waves(d128, uint16_t{}, no) : waves(d64, uint16_t{}, no);
    if (L.G <= 4) return L.D == 128 ? waves(d128, float{}, yes) : waves(d64, float{}, yes);
    return L.D == 128 ? waves(d128, float{}, no) : waves(d64, float{}, no);
}

#endif  // RAAS_PART == 0

}  // namespace raas

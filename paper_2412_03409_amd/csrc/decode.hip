// Stage 4b: one decode step over the ragged compressed cache (Sec. 3.1: the newest token's query
// interacts with the cached KV vectors of every layer).  ONE kernel per step (two for bf16 caches whose
// KV heads serve several query heads: decode_gqa_kernel and decode_gqa_merge_kernel, further down):
//
//  decode_attn_kernel   a unit is one (sequence, layer, kv head), or a sub-group of G of its query heads.  One to
//                       eight wavefronts work on a unit (see the launcher) and take its row blocks round-robin.  A
//                       wavefront requests the K and V rows of its first block together (16 B per lane, whole rows, fully
//                       coalesced) and those of the next one as this one's are used up; it does the dot products, a
//                       block softmax and the weighted V sum in registers
//                       for every query head of the group, so each cached byte is read from HBM once per group.
//                       The wavefronts' (max, sum, weighted V) are merged through LDS and the output is
//                       written directly: no partial results ever go to HBM.
//
// Append: the new token's k/v are taken from k_new/v_new in place of the slot they are written to, so
// no wavefront reads a slot that is written in the same launch.
//
// lens is advanced inside the launch of decode_attn_kernel without a second kernel: every wavefront reads the old
// length of its segment when it starts, and every unit, once its wavefronts have, is counted in the
// bits above kLenBits of lens[b,l] (by itself, or by the first of its workgroup).  The one that finds all others of
// the segment already counted stores the new plain length, which also clears the count.  Between launches lens holds plain
// lengths (< 2^20).  The ranking of the segments goes by capacity, which no launch changes.
#include "pkv_common.hpp"
#include "decode_rows.hpp"

#include <type_traits>

namespace pkv {

static int pick_group(int grp) { return grp % 8 == 0 ? 8 : grp % 4 == 0 ? 4 : grp % 2 == 0 ? 2 : 1; }

constexpr int kLenBits = 20;
constexpr int kLenMask = (1 << kLenBits) - 1;

struct DecodeParams {
    int B, L, l0, nl, H, Hkv, D, grp, append;
    const unsigned char* q;       // [B,L,H,D]
    const unsigned char* k_new;   // [B,L,Hkv,D]
    const unsigned char* v_new;
    const float* scale;           // [L]
    unsigned char* kc;
    unsigned char* vc;
    const int64_t* seg_off;       // [B,L]
    const int32_t* caps;          // [B,L]
    int32_t* lens;                // [B,L]
    unsigned char* out;           // [B,L,H,D]
    // pruning at a fixed distance (EV = true only)
    int N, t, d;                  // prompt length, 1-based decode step, distance
    int slot_new, slot_due;       // ring slots of the token stored in this step and of the one decided in it
    const int32_t* base_lens;     // [B,L] entries kept after prefill
    int32_t* kept_pos;            // one int per slot, may be null
    int n_seg;
    // grouped-query kernels: wavefronts, workspace
    int waves;
    int* ws;
    RankedShape rank;   // ranked launches of decode_attn_kernel
    int turn;                // grouped launches: grouped_turn
    FastDiv by_nl, by_seg;   // nl, n_seg
};

constexpr int kRankRegs = 8;      // capacities per lane of a ranked launch: groups of up to 512 segments

// Cache rows are read once per decode step and never reused by the same launch: stream them past the
// caches (nontemporal) so that they do not evict each other on the way in.
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_t;
__device__ __forceinline__ uint4 load_stream16(const unsigned char* p) {
    const u32x4_t t = __builtin_nontemporal_load((const u32x4_t*)p);
    return make_uint4(t.x, t.y, t.z, t.w);
}

__device__ __forceinline__ int64_t uniform64(int64_t x) {   // a value that is the same in all lanes, in scalar registers
    return ((int64_t)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

template <bool BF16>
__device__ __forceinline__ void unpack16(const uint4& r, float* f) {
    if constexpr (BF16) {
        f[0] = __uint_as_float(r.x << 16); f[1] = __uint_as_float(r.x & 0xffff0000u);
        f[2] = __uint_as_float(r.y << 16); f[3] = __uint_as_float(r.y & 0xffff0000u);
        f[4] = __uint_as_float(r.z << 16); f[5] = __uint_as_float(r.z & 0xffff0000u);
        f[6] = __uint_as_float(r.w << 16); f[7] = __uint_as_float(r.w & 0xffff0000u);
    } else {
        f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y);
        f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
    }
}

// The other lanes' values come by DPP and lane swaps, not through LDS: a step of a shuffle by ds_bpermute is a round trip of
// some hundred cycles, and a block of rows needs six in a row (32 units, one layer of the 7B shape 5.63 -> 5.36 us per launch,
// 768 units of 1200 rows 88.5 -> 84.3).  Same sums in the same order.
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xF, 0xF, true));
}
template <class F> __device__ __forceinline__ float with_xor16(float x, F f) {
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return f(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
template <class F> __device__ __forceinline__ float with_xor32(float x, F f) {
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return f(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
// Sum over the LPR lanes of a row, in all of them.  Once the lanes of a quad (of a half of 16) agree, the mirrored lane has what
// the lane at distance 4 (8) has.
template <int LPR>
__device__ __forceinline__ float row_sum(float x) {
    static_assert(LPR == 8 || LPR == 16 || LPR == 32, "16 bytes per lane, D 64 or 128");
    x += dpp<0xB1>(x);                                     // quad_perm [1,0,3,2]
    x += dpp<0x4E>(x);                                     // quad_perm [2,3,0,1]
    x += dpp<0x141>(x);                                    // row_half_mirror
    if constexpr (LPR >= 16) x += dpp<0x140>(x);           // row_mirror
    if constexpr (LPR >= 32) x = with_xor16(x, [](float a, float b) { return a + b; });
    return x;
}
// f over the row groups: lanes at distances LPR, 2 LPR ... 32.
template <int LPR, class F>
__device__ __forceinline__ float over_groups(float x, F f) {
    if constexpr (LPR <= 8) x = f(x, dpp<0x128>(x));       // row_ror:8
    if constexpr (LPR <= 16) x = with_xor16(x, f);
    return with_xor32(x, f);
}

// One query head group and one block of NI * 64/LPR rows (LPR lanes cover a row with 16 bytes each, a lane has NI rows).
// Scores from the K rows, summed over the lanes of a row.
template <bool BF16, int LPR, int G, int NI>
__device__ __forceinline__ void block_scores(const uint4 (&kr)[NI], const float (&qf)[G][BF16 ? 8 : 4], float (&s)[G][NI]) {
    constexpr int EPL = BF16 ? 8 : 4;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        float kf[EPL];
        unpack16<BF16>(kr[i], kf);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float d = 0.f;
#pragma unroll
            for (int x = 0; x < EPL; ++x) d = fmaf(qf[g][x], kf[x], d);
            s[g][i] = d;
        }
    }
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int g = 0; g < G; ++g) s[g][i] = row_sum<LPR>(s[g][i]);
}
// Online-softmax update of (mrun, srun, o) with the block.
template <bool BF16, int LPR, int G, int NI>
__device__ __forceinline__ void block_values(const float (&s)[G][NI], const uint4 (&vr)[NI], float (&o)[G][BF16 ? 8 : 4],
                                             float (&mrun)[G], float (&srun)[G]) {
    constexpr int EPL = BF16 ? 8 : 4;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        float mx = s[g][0];
#pragma unroll
        for (int i = 1; i < NI; ++i) mx = fmaxf(mx, s[g][i]);
        mx = over_groups<LPR>(mx, [](float a, float b) { return fmaxf(a, b); });
        // no score above -inf so far: all keys of the wavefront's blocks are that far off, or the only row of the first
        // one is pruned in this step
        const float mnew = fmaxf(mrun[g], mx);
        const float mref = mnew == -INFINITY ? 0.f : mnew;
        const float corr = __builtin_amdgcn_exp2f(mrun[g] - mref);  // 0 on the first block
        mrun[g] = mnew;
        // the block's own sums first, so that a long segment adds one value per block to the running ones and not one per row
        float sum = 0.f, ob[EPL];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const float pr = __builtin_amdgcn_exp2f(s[g][i] - mref);
            sum += pr;
            float vf[EPL];
            unpack16<BF16>(vr[i], vf);
#pragma unroll
            for (int x = 0; x < EPL; ++x) ob[x] = i == 0 ? pr * vf[x] : fmaf(pr, vf[x], ob[x]);
        }
        srun[g] = fmaf(srun[g], corr, sum);   // per row group; the groups are merged at the end
#pragma unroll
        for (int x = 0; x < EPL; ++x) o[g][x] = fmaf(o[g][x], corr, ob[x]);
    }
}
__device__ __forceinline__ uint4 select16(bool first, const uint4& a, const uint4& b) {
    return make_uint4(first ? a.x : b.x, first ? a.y : b.y, first ? a.z : b.z, first ? a.w : b.w);
}

// Maximum over the wavefront.
__device__ __forceinline__ int wave_max(int x) {
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, true));    // quad_perm [1,0,3,2]
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, true));    // quad_perm [2,3,0,1]
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x124, 0xF, 0xF, true));   // row_ror:4
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x128, 0xF, 0xF, true));   // row_ror:8
    const auto h = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = max((int)h[0], (int)h[1]);
    const auto w = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return __builtin_amdgcn_readfirstlane(max((int)w[0], (int)w[1]));
}

// The segment of rank `r` when the n segments are ordered by length class, longest first, and by index inside a class:
// found by every wavefront for itself.  A class is a quarter octave of capacity below the largest one, the last of sixteen
// holds everything shorter than a thirteenth of it: enough to start the long segments early, at four ballots per 64
// segments.  (The exact order takes a ballot for every bit of the capacities: 1 ... 2 us at the start of every unit, which
// short units do not earn back.)  n <= 64 * PER.
template <int PER>
__device__ __forceinline__ int ranked_segment(const int32_t* __restrict__ caps, int n, int nl, int L, int l0, int first, int r, int lane) {
    int c[PER];
    int top = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = u * kWave + lane;
        c[u] = 0;
        if (i < n) { const int j = first + i; c[u] = caps[nl == L ? j : (j / nl) * L + l0 + j % nl] & kLenMask; }
        top = max(top, c[u]);
    }
    top = wave_max(top);
#pragma unroll
    for (int u = 0; u < PER; ++u) c[u] = u * kWave + lane < n ? length_class(c[u], top) : kLengthClasses;
    int cls = 0, left = r;                  // the class found so far (high bits), rank among those that share it
#pragma unroll
    for (int half = kLengthClasses / 2; half >= 1; half >>= 1) {
        int cnt = 0;
#pragma unroll
        for (int u = 0; u < PER; ++u) cnt += __builtin_popcountll(__builtin_amdgcn_ballot_w64((c[u] & -half) == cls));
        if (left >= cnt) { left -= cnt; cls |= half; }
    }
    int found = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const unsigned long long m = __builtin_amdgcn_ballot_w64(c[u] == cls);
        const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
        const unsigned long long hit = __builtin_amdgcn_ballot_w64(c[u] == cls && before == left);
        if (hit) found = u * kWave + __builtin_ctzll(hit);
        left -= __builtin_popcountll(m);
    }
    return found;
}

// W wavefronts per workgroup; OCC = wavefronts per SIMD the register allocation must allow.  RANK = 0: all W are for one unit, -1: and it
// is counted in before its rows.  kGrouped: W, W/2 ... or one, by the segment's rows.  RANK > 0: units of the longest segments first,
// with W, W/2 or W/4 wavefronts per unit (see the launcher).
constexpr int kGrouped = -2;
template <bool BF16, int LPR, int G, int NI, int W, int OCC, bool EV, int RANK>
__global__ void __launch_bounds__(W * kWave, OCC)
decode_attn_kernel(DecodeParams p) {
    constexpr int EPL = BF16 ? 8 : 4;            // elements per lane (16 bytes)
    constexpr int RPI = kWave / LPR;             // rows per wavefront-wide load instruction
    constexpr int BR = NI * RPI;                 // rows per block
    constexpr int D = LPR * EPL, ROWB = LPR * 16;
    __shared__ float s_num[W][G][D];
    __shared__ float2 s_md[W][G];                // maximum and denominator

    const int HU = p.H / G;                     // units per segment
    const int lane = threadIdx.x & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    int UW = W, hu, b, l;
    bool live = true;
    if constexpr (RANK > 0) {
        static_assert(W == 4, "a workgroup holds one, two or four units");
        const RankedUnit x = ranked_unit(blockIdx.x, wv, p.rank, HU, p.n_seg);
        UW = x.UW; hu = x.hu; live = x.live;
        if (!live && UW != 2) return;                      // one wavefront each: the barrier below is for those that go on; four: none of the workgroup has a unit
        int i_seg = 0;
        if (live) i_seg = x.first + (p.rank.by_length ? ranked_segment<RANK>(p.caps, x.n, p.nl, p.L, p.l0, x.first, x.rank, lane) : x.rank);
        b = i_seg / p.nl; l = p.l0 + i_seg % p.nl;
    } else if constexpr (RANK == kGrouped) {
        // the segment; how many wavefronts its units have, and so which are this workgroup's, when the capacity is there (below)
        const int seg = __builtin_amdgcn_readfirstlane(grouped_segment((int)blockIdx.x, (int)blockIdx.y, p.turn, p.by_seg));
        const DivMod bl = uniform_div_mod(seg, p.by_nl);
        b = bl.q; l = p.l0 + bl.r; hu = 0;
    } else {
        hu = blockIdx.x; l = p.l0 + blockIdx.y; b = blockIdx.z;
    }
    const int sl = b * p.L + l;
    const int sub = lane % LPR, rg = lane / LPR;

    // What the first rows wait for, in one round trip to memory (left to itself the compiler waits for the length before it
    // requests the capacity, and for that before the offset and the queries): the words of the segment and the other arguments.
    int len_raw = __hip_atomic_load(p.lens + sl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);   // from the caches: the length is the same in every value of this launch
    int cap = uniform_load(p.caps + sl);
    int64_t off = uniform_load(p.seg_off + sl);
    int base = EV ? uniform_load(p.base_lens + sl) : 0;
    uint4 qr[G];
    auto load_q = [&]() {
#pragma unroll
        for (int g = 0; g < G; ++g) qr[g] = *(const uint4*)(p.q + ((int64_t)sl * p.H + hu * G + g) * ROWB + sub * 16);
    };
    constexpr bool kOne = RANK == 0 || RANK == -1;           // one unit per workgroup
    if constexpr (kOne) load_q();
    asm volatile("" : "+v"(len_raw), "+s"(cap), "+s"(off), "+s"(base)
                 : "s"(p.kc), "s"(p.vc), "s"(p.k_new), "s"(p.v_new), "s"(p.out), "s"(p.scale), "s"(p.Hkv), "s"(p.grp), "s"(p.append) : "memory");
    const float scale = uniform_load(p.scale + l);
    const int len_old = __builtin_amdgcn_readfirstlane(len_raw) & kLenMask;
    cap = __builtin_amdgcn_readfirstlane(cap);
    off = uniform64(off);
    if constexpr (RANK == kGrouped) {
        // By what no workgroup changes: the capacity or, under pruning, the entries kept after prefill.  The grid is for one unit
        // per workgroup, and those that are not needed end here, all their wavefronts and ahead of any barrier.
        const int rows = EV ? base + (p.t < p.d + 1 ? p.t : p.d + 1) : cap;
        UW = __builtin_amdgcn_readfirstlane(active_waves(row_blocks(rows, BR), HU, W));
        if ((int)blockIdx.y >= grouped_blocks(HU, UW, W)) return;
        const GroupedUnit x = grouped_unit((int)blockIdx.y, wv, UW, W, HU);
        hu = x.hu; live = x.live;
    }
    const int uw = wv & (UW - 1);
    // The unit is counted in once every wavefront of it has read lens.  The smallest launches: here, so that the round trip of the
    // atomic passes under the rows; it is the last wavefront's, which has the fewest.  (32 units 5.36 -> 4.94 us per launch.  Where
    // units start while others count in, their reads of lens wait for the atomics: 256 units 5 ... 20 % slower, 512 by up to half.)
    constexpr bool kEarly = RANK == -1;
    const bool counter = live && uw == (kEarly ? UW - 1 : 0) && lane == 0;
    int counted = 0, count = 1;
    if (kEarly || (!kOne && UW == 1)) {
        asm volatile("" : : : "memory");                     // nothing but lens is behind this barrier, and its value has arrived
        __builtin_amdgcn_s_barrier();
        asm volatile("" : : : "memory");
    }
    // The first of the workgroup's units of a segment counts all of them in, behind a barrier that they have
    // passed with lens read.  The atomics on the few cache lines of lens were what launches of short rows took, about 8 ns each: 2048 units
    // of 26 rows 18.5 ... 34 us in the same shape, now 17 ... 26, 12 800 of 136 rows 172 -> 160.
    if constexpr (!kOne) count = counted_units(wv >> __builtin_ctz(UW), W >> __builtin_ctz(UW), hu, HU);
    // The result is wanted at the end only; of an address that it knows to be uniform the compiler makes a sum over the lanes first
    // and waits for the atomic on the spot.
    int zero = 0;
    asm volatile("" : "+v"(zero));
    auto count_in = [&]() { counted = atomicAdd(p.lens + sl + zero, count << kLenBits); };
    if (kEarly && counter) count_in();
    // plain step: append at slot len_old.  Pruning step: len_old counts the permanent entries, the new
    // token goes to ring slot (t-1) mod (d+1), and the token stored d steps ago (ring slot t mod (d+1))
    // either becomes permanent entry len_old or is left out from now on.
    const StepRows step = step_rows<EV>(len_old, cap, base, p.append, p.t, p.d);   // under pruning nothing if the capacity cannot hold the ring
    const bool app = step.app;
    const int len = step.rows;
    int len_next = len, ring0 = 0;
    RingMap ring = {0, -1, -1};
    bool grad = false, decide = false;
    if constexpr (EV) {
        ring0 = cap - (p.d + 1);
        decide = app && p.t > p.d;
        grad = decide && len_old < ring0 && within_target(len_old + p.d + 1, base, p.N, p.t);
        ring.shift = ring0 - len_old;
        ring.r_new = len_old + p.slot_new;
        ring.r_mask = (decide && !grad) ? len_old + p.slot_due : -1;
        len_next = len_old + (grad ? 1 : 0);
    }
    const int nb = live ? (len + BR - 1) / BR : 0, nfull = len_old / BR;
    const int kvh = p.grp == G ? hu : (hu * G) / p.grp;
    const bool writer = app && live && (p.grp == G || (hu * G) % p.grp == 0);
    const int64_t segbase = uniform64((off * p.Hkv + (int64_t)kvh * cap) * ROWB);
    const int64_t newrow = ((int64_t)sl * p.Hkv + kvh) * ROWB;
    unsigned char* kseg = p.kc + segbase;
    unsigned char* vseg = p.vc + segbase;

    // The new row: the wavefront that has its block takes it from k_new / v_new, requested ahead of the cached rows, and stores it
    // behind them.  Under pruning the same one moves the surviving token from its ring slot to the next permanent slot (attention
    // reads it from the ring slot; nobody reads the permanent slot in this launch).
    const int r_new = EV ? ring.r_new : len_old;
    const bool own = app && live && ((r_new / BR) & (UW - 1)) == uw;
    uint4 nk = make_uint4(0, 0, 0, 0), nv = nk, gk = nk, gv = nk;
    if constexpr (!kOne) load_q();                           // ahead of the new row: what is requested late waits behind the counts
    if (own) {
        nk = *(const uint4*)(p.k_new + newrow + sub * 16);
        nv = *(const uint4*)(p.v_new + newrow + sub * 16);
        if (EV && grad) {
            gk = *(const uint4*)(kseg + (size_t)(ring0 + p.slot_due) * ROWB + sub * 16);
            gv = *(const uint4*)(vseg + (size_t)(ring0 + p.slot_due) * ROWB + sub * 16);
        }
    }
    float o[G][EPL], mrun[G], srun[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        mrun[g] = -INFINITY; srun[g] = 0.f;
#pragma unroll
        for (int x = 0; x < EPL; ++x) o[g][x] = 0.f;
    }
    if (uw < nb) {
        // a segment with no row but the new one: k_new / v_new stand in for its slots
        const bool lone = app && len == 1;
        const unsigned char *kload = lone ? p.k_new + newrow : kseg, *vload = lone ? p.v_new + newrow : vseg;
        float qf[G][EPL] = {};
        auto scale_q = [&]() {                               // while the first rows are on their way, not ahead of them
            float qs = scale;
            asm volatile("" : "+s"(qs));
            qs *= 1.4426950408889634f;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                uint4 t = qr[g];
                asm volatile("" : "+v"(t.x), "+v"(t.y), "+v"(t.z), "+v"(t.w));
                unpack16<BF16>(t, qf[g]);
#pragma unroll
                for (int x = 0; x < EPL; ++x) qf[g][x] *= qs;
            }
        };
        uint4 kr[NI], vr[NI];
        float s[G][NI];
        int blk = uw;
        // Blocks of stored rows.  The next block's K rows are requested when this one's are used up, its V rows likewise: no register
        // more, and the wavefronts of the longest units, with which a launch ends, wait less (13B, batch 8:
        // 158.8 -> 154.6 us a step).  In launches of one round the compiler may request V rows as their registers come free (512 units of
        // 1200 rows, lengths within a factor 30, 62.8 -> 61.5 us; 480 of 204 14.1 -> 13.8; 0.997 ... 1.00 of the time of others); in ranked ones of
        // short rows that is 2 ... 10 % slower.
        if (blk < nfull) {
            const unsigned char *ka = kseg + (size_t)blk * (NI * 1024), *va = vseg + (size_t)blk * (NI * 1024);
            const uint32_t lane_off = (uint32_t)lane * 16u;
            auto load_k = [&]() {
#pragma unroll
                for (int i = 0; i < NI; ++i) kr[i] = load_stream16(ka + i * 1024 + lane_off);
            };
            auto load_v = [&]() {
#pragma unroll
                for (int i = 0; i < NI; ++i) vr[i] = load_stream16(va + i * 1024 + lane_off);
            };
            load_k();
            load_v();
            scale_q();
            for (; blk + UW < nfull; blk += UW) {
                block_scores<BF16, LPR, G, NI>(kr, qf, s);
                ka += (size_t)UW * (NI * 1024);
                va += (size_t)UW * (NI * 1024);
                load_k();
                __builtin_amdgcn_sched_barrier(0);
                block_values<BF16, LPR, G, NI>(s, vr, o, mrun, srun);
                if constexpr (RANK > 0) __builtin_amdgcn_sched_barrier(0);
                load_v();
            }
            block_scores<BF16, LPR, G, NI>(kr, qf, s);
            block_values<BF16, LPR, G, NI>(s, vr, o, mrun, srun);
            blk += UW;
        }
        // Blocks with the new row, ring rows or rows that take no part.
        for (; blk < nb; blk += UW) {
            const int r0 = blk * BR + rg;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const uint32_t at = (lone ? 0 : (uint32_t)row_slot<EV>(r0 + i * RPI, blk * BR, len, len_old, app ? r_new : -1, ring) * (uint32_t)ROWB) + sub * 16;
                kr[i] = load_stream16(kload + at);
                vr[i] = load_stream16(vload + at);
            }
            if (blk == uw) scale_q();
            if (own) {
#pragma unroll
                for (int i = 0; i < NI; ++i) kr[i] = select16(r0 + i * RPI == r_new, nk, kr[i]);
            }
            block_scores<BF16, LPR, G, NI>(kr, qf, s);
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int r = r0 + i * RPI;
                const bool valid = r < len && (!EV || r != ring.r_mask);
#pragma unroll
                for (int g = 0; g < G; ++g) s[g][i] = valid ? s[g][i] : -INFINITY;
                vr[i] = select16(valid, select16(own && r == r_new, nv, vr[i]), make_uint4(0, 0, 0, 0));   // 0 * (what is there) could be NaN
            }
            block_values<BF16, LPR, G, NI>(s, vr, o, mrun, srun);
        }
        // merge the RPI row groups of the wavefront (they share mrun)
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const auto add = [](float a, float b) { return a + b; };
            srun[g] = over_groups<LPR>(srun[g], add);
#pragma unroll
            for (int x = 0; x < EPL; ++x) o[g][x] = over_groups<LPR>(o[g][x], add);
        }
    }
    if (own && writer && rg == 0) {
        const size_t slot = (size_t)(EV ? ring0 + p.slot_new : len_old) * ROWB + sub * 16;
        *(uint4*)(kseg + slot) = nk;
        *(uint4*)(vseg + slot) = nv;
        if (EV && grad) {
            *(uint4*)(kseg + (size_t)len_old * ROWB + sub * 16) = gk;
            *(uint4*)(vseg + (size_t)len_old * ROWB + sub * 16) = gv;
        }
    }
    if constexpr (EV) {
        if (p.kept_pos && app && live && hu == 0 && uw == 0 && lane == 0) {
            int32_t* kp = p.kept_pos + off;
            kp[ring0 + p.slot_new] = p.N + p.t - 1;
            if (decide) {
                if (grad) kp[len_old] = p.N + p.t - p.d - 1;
                kp[ring0 + p.slot_due] = -1;
            }
        }
    }
    // The other launches count the unit in here (UW > 1: behind the barrier below); the round trip of the atomic passes while the
    // output is written.
    if (!kOne && UW == 1) {
        if (counter && count > 0) count_in();
        if (live && rg == 0) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const size_t oi = ((size_t)sl * p.H + hu * G + g) * D + sub * EPL;
                float r[EPL];
#pragma unroll
                for (int x = 0; x < EPL; ++x) r[x] = srun[g] > 0.f ? o[g][x] / srun[g] : 0.f;   // an empty segment gives zeros
                if constexpr (BF16) {
                    uint32_t w[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x) w[x] = pack_bf16(r[2 * x], r[2 * x + 1]);
                    *(uint4*)((bf16_t*)p.out + oi) = make_uint4(w[0], w[1], w[2], w[3]);
                } else {
                    *(float4*)((float*)p.out + oi) = make_float4(r[0], r[1], r[2], r[3]);
                }
            }
        }
    } else {
        if (rg == 0) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float* dst = s_num[wv][g] + sub * EPL;
#pragma unroll
                for (int x = 0; x < EPL; x += 4) *(float4*)(dst + x) = make_float4(o[g][x], o[g][x + 1], o[g][x + 2], o[g][x + 3]);
                if (sub == 0) s_md[wv][g] = make_float2(mrun[g], srun[g]);
            }
        }
        __syncthreads();
        if (!kEarly && counter && count > 0) count_in();
        // merge the wavefronts of a unit: thread (g, d); all its values are requested together
        const int w0 = wv & ~(UW - 1);
        for (int i = uw * kWave + lane; live && i < G * D; i += UW * kWave) {
            const int g = i / D, d = i % D;
            float2 md[W];
            float num_w[W];
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const int at = !kOne ? w0 + (w & (UW - 1)) : w;
                md[w] = s_md[at][g];
                num_w[w] = s_num[at][g][d];
            }
            float M = md[0].x;
#pragma unroll
            for (int w = 1; w < W; ++w) M = fmaxf(M, md[w].x);
            const float ref = M == -INFINITY ? 0.f : M;
            float num = 0.f, den = 0.f;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                if (!kOne && w >= UW) break;
                const float wgt = __builtin_amdgcn_exp2f(md[w].x - ref);
                num = fmaf(wgt, num_w[w], num);
                den = fmaf(wgt, md[w].y, den);
            }
            const float r = den > 0.f ? num / den : 0.f;   // an empty segment gives zeros
            const size_t oi = ((size_t)sl * p.H + hu * G + g) * D + d;
            if constexpr (BF16) ((bf16_t*)p.out)[oi] = (bf16_t)pack_bf16(r, r); else ((float*)p.out)[oi] = r;
        }
    }
    // the last unit of the segment to be counted in stores the new length
    if (counter && count > 0) {
        asm volatile("" : "+v"(counted));
        if ((int)((unsigned)counted >> kLenBits) + count == HU)
            __hip_atomic_store(p.lens + sl, len_next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// ---------------------------------------------------------------------------------------------------
// Grouped-query variant on the matrix cores (bf16 storage, G = 2, 4 or 8 query heads per KV head).
//
// The rows of a launch are one stream: the units (segment by segment, its head groups one after the other) cut into blocks of
// BR rows, and every wavefront takes the same number of consecutive blocks (gqa_share), wherever the units' borders lie.  So
// the work is even whatever the lengths (they differ by up to two orders of magnitude), and the next two blocks, of this unit
// or of later ones, are on their way to LDS while a wavefront works on one: it does not wait between units.  What it has of a
// unit that other wavefronts share goes to the workspace as (numerators, max, denominator); decode_gqa_merge_kernel adds
// those up in block order and advances lens, so nothing counts arrivals and the result does not depend on timing.
//
// Long caches are bound by the rate at which a compute unit's reads are served (6.6 TB/s while all wavefronts are at work; at
// B4 H32/8 N8192 10 % they ended between 59 and 84 us of a launch, between 63 and 80 since they give way as they get on, and
// larger first shares with smaller ones dispatched behind them cost more in starts than they even out: 84 -> 90 us), short ones
// by the chain lengths -> block counts -> first block and by the two launches.  Against the kernel before, which claimed pieces of
// 1024 rows from a planned list, one workgroup each, and handed a split segment to the last arriver (7 us per piece between the
// streams of rows), us per step, lengths within a factor 30, D 128 (D 64):
//   B4 H32/8 N8192 10 % 96 -> 81 (61 -> 45), equal lengths 84 -> 75 (54 -> 43), the whole cache 725 -> 665 (382 -> 337); B64 N680 10 %
//   279 -> 193 (227 -> 135), B8 N680 20 % 57 -> 42, B1 N2000 35 -> 21, N500 18 -> 13 (15 -> 10); with pruning B4 N2000 62 -> 47; H32/4 B32
//   N2000 10 % 136 -> 119, B1 N2000 20 % 42 -> 20; one layer a call: B1 N2000 20 % 16.5 -> 9.4, a single layer kept whole N500 15.9 ->
//   9.7 (12.5 -> 8.8), N8192 34 -> 20.
// The running numerators take one addition per row: 256 of them are off by 2e-7 (fp64), 4096 by 1.3e-6.  The block's own sums first
// halves that, far below the bf16 output's 2e-3, and costs up to 9 % (H32/4, D 64, B4 260 MB 54 -> 59 us).
//   scores^T[16 rows x 16 head columns] = K[16 rows x D] . Q^T with v_mfma_f32_16x16x32_bf16 (A = cache rows from LDS, B = the
//   queries, head lane%16, columns >= G are zero): a lane holds four rows of one head, and softmax runs in that layout.  The
//   weighted sum stays on the vector ALU with fp32 probabilities: a group of 16 lanes takes the V rows whose probabilities
//   it holds, so that they reach it as row broadcasts (DPP), without LDS.
// K and V go to LDS by the 16-byte copies: the matrix operand wants a row per lane, and 16 bytes per lane at row distance
// take 64 cycles of the compute unit's address unit, whole rows 16.
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((address_space(3))) void lds_void_t;

// State of one segment for this step, computed identically by every wavefront that touches it.
struct SegState {
    int len_old;   // occupied slots before the step (under pruning: permanent entries)
    int cap;
    int len;       // rows to attend to in this step (virtual rows under pruning)
    int len_next;  // value of lens after the step
    int ring0, cs; // pruning: first ring slot, ring slot of the token decided in this step
    bool app, grad, decide;
    RingMap ring;
    int64_t off;
};

template <bool EV>
__device__ __forceinline__ SegState seg_state(const DecodeParams& p, int len_old, int cap, int64_t off, int base) {
    SegState s;
    s.len_old = len_old; s.cap = cap; s.off = off;
    const StepRows r = step_rows<EV>(len_old, cap, base, p.append, p.t, p.d);
    s.app = r.app;
    s.len = s.len_next = r.rows;
    s.ring = {0, s.app ? s.len_old : -1, -1};
    s.ring0 = 0; s.cs = 0; s.grad = false; s.decide = false;
    if constexpr (EV) {
        s.ring0 = s.cap - (p.d + 1);
        s.decide = s.app && p.t > p.d;
        s.cs = p.slot_due;
        s.grad = s.decide && s.len_old < s.ring0 && within_target(s.len_old + p.d + 1, base, p.N, p.t);
        s.ring.shift = s.ring0 - s.len_old;
        s.ring.r_new = s.app ? s.len_old + p.slot_new : -1;
        s.ring.r_mask = (s.decide && !s.grad) ? s.len_old + s.cs : -1;
        s.len_next = s.len_old + (s.grad ? 1 : 0);
    }
    return s;
}


__device__ __forceinline__ int seg_slot(const DecodeParams& p, int i) { return (i / p.nl) * p.L + p.l0 + i % p.nl; }

// inclusive sum over the lanes, by DPP: every wavefront waits for it before its first rows
__device__ __forceinline__ int wave_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast:15, to the odd rows of 16
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast:31, to the upper half
    return v;
}

// 16 bytes per lane from global memory to LDS[dst + 16 * lane] (nothing else here uses m0); ONCE: without a place in the caches
template <bool ONCE>
__device__ __forceinline__ void copy16(const unsigned char* base, uint32_t off, uint32_t dst) {
    if constexpr (ONCE) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" :: "s"(dst), "v"(off), "s"(base) : "memory");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(dst), "v"(off), "s"(base) : "memory");
}
__device__ __forceinline__ void copy16_any(const unsigned char* src, uint32_t dst) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(dst), "v"(src) : "memory");
}

__device__ __forceinline__ float swap_add16(float a, float b) {   // lanes with bit 4 clear: a of both rows of 16, set: b
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ __forceinline__ float swap_add32(float a, float b) {   // lower half: a of both halves, upper: b
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
// value of lane `g` of the own 16 lanes
template <int g>
__device__ __forceinline__ float row_bcast(float x) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), 0x150 + g, 0xF, 0xF, true));
}
template <int G, class F> __device__ __forceinline__ void for_heads(F f) {
    f(std::integral_constant<int, 0>{}); f(std::integral_constant<int, 1>{});
    if constexpr (G > 2) { f(std::integral_constant<int, 2>{}); f(std::integral_constant<int, 3>{}); }
    if constexpr (G > 4) {
        f(std::integral_constant<int, 4>{}); f(std::integral_constant<int, 5>{});
        f(std::integral_constant<int, 6>{}); f(std::integral_constant<int, 7>{});
    }
}

// wavefronts of a workgroup, of a launch at most (8 on each of 256 compute units); block counts per lane that are held between the
// passes
constexpr int kGqaWaves = 4, kGqaWavesMax = 2048, kGqaHeld = 4;

// Rows of up to so many bytes are read through the caches: the last level holds 256 MiB, and the next step reads them again.
// Beyond that a pass evicts what the next one looks for, and rows that do not enter are faster.  us per step, through the caches
// / past them, H 32/8, D 128, B4: equal lengths, 180 MB 40.6 / 41.0, 260 55.0 / 56.1, 340 75.5 / 66.9, 420 91.7 / 79.1, 4.3 GB 737 /
// 661; within a factor 30, 230 49.1 / 51.7, 300 60.0 / 62.4, 340 67.8 / 68.2, 380 76.0 / 74.6, 700 135 / 123.
constexpr long long kGqaCached = 320ll << 20;

template <int D, int G, bool EV>
__global__ void __launch_bounds__(kGqaWaves * kWave, 2)
decode_gqa_kernel(DecodeParams p) {
    constexpr int ROWB = D * 2, LPR = D / 8, RPI = kWave / LPR;   // bytes of a row, lanes and rows of a copy instruction
    constexpr int NT = 128 / D;                   // 16-row tiles of a block
    constexpr int BR = 16 * NT;
    constexpr int NJ = D / 32;                    // MFMAs per tile
    constexpr int NI = BR / RPI;                  // copy instructions per tensor: 4
    constexpr int TB = BR * ROWB;                 // bytes of a block of K: 4096
    static_assert(NI == 4 && TB == 4096, "block of 4 KB per tensor");
    constexpr int QB = G * ROWB;                  // bytes of a unit's queries
    __shared__ __attribute__((aligned(1024))) unsigned char s_ring[kGqaWaves][2][2 * TB];   // [wavefront][stage][K, V]
    __shared__ __attribute__((aligned(1024))) unsigned char s_q[kGqaWaves][2][QB < 1024 ? 1024 : QB];   // the queries of two units

    const int HU = p.H / G, n = p.n_seg;
    const int lane = threadIdx.x & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int gid = blockIdx.x * kGqaWaves + wv;
    const int kr = lane & 15, kq = lane >> 4;            // K / score layout: row (or head) kr, quad kq
    const int sub = lane % LPR, rg = lane / LPR;         // V layout

    // ---- where this wavefront's blocks are: block counts of all segments, their sum, the segment of the first block
    struct Words { int len, cap, base; int64_t off; };   // of a segment, as they lie in memory
    auto read = [&](int i) {
        Words w = {0, 0, 0, 0};
        if (i < n) {
            const int sl = seg_slot(p, i);
            w.len = p.lens[sl] & kLenMask; w.cap = p.caps[sl]; w.off = p.seg_off[sl];
            if (EV) w.base = p.base_lens[sl];
        }
        return w;
    };
    auto blocks_of = [&](int i, const Words& w) {
        return i < n ? row_blocks(step_rows<EV>(w.len, w.cap, w.base, p.append, p.t, p.d).rows, BR) : 0;
    };
    Words held[kGqaHeld];
    int sum = 0;
#pragma unroll
    for (int u = 0; u < kGqaHeld; ++u) { held[u] = read(u * kWave + lane); sum += blocks_of(u * kWave + lane, held[u]); }
    for (int i = kGqaHeld * kWave; i < n; i += kWave) sum += blocks_of(i + lane, read(i + lane));
    const int total = __builtin_amdgcn_readlane(wave_scan(sum), kWave - 1);   // of one head group
    const int all = total * HU;
    const int share = gqa_share(all, p.waves, gqa_least(all, p.waves, n * HU, G * D));
    if (gid == 0 && lane == 0) { p.ws[0] = share; p.ws[kGqaHdr + n] = total; }
    const bool once = (long long)total * p.Hkv * (2 * TB) > kGqaCached;
    const int x0 = gid * share, x1 = x0 + share < all ? x0 + share : all;
    if (x0 >= all) return;
    const int y0 = x0 / HU;
    int seg = 0, first = 0, before = 0;                  // the segment of block x0, first block of it (per head group)
    Words mine = {0, 0, 0, 0};                           // its words
    auto look = [&](int u, const Words& w) {
        const int nb = blocks_of(u * kWave + lane, w);
        const int incl = before + wave_scan(nb), excl = incl - nb;
        if (gid == 0 && u * kWave + lane < n) p.ws[kGqaHdr + u * kWave + lane] = excl;
        const unsigned long long m = __builtin_amdgcn_ballot_w64(nb > 0 && excl <= y0);
        if (m) {
            const int at = 63 - __builtin_clzll(m);
            seg = u * kWave + at;
            first = __builtin_amdgcn_readlane(excl, at);
            mine.len = __builtin_amdgcn_readlane(w.len, at);
            mine.cap = __builtin_amdgcn_readlane(w.cap, at);
            mine.base = __builtin_amdgcn_readlane(w.base, at);
            mine.off = ((int64_t)__builtin_amdgcn_readlane((int)(w.off >> 32), at) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)w.off, at);
        }
        before = __builtin_amdgcn_readlane(incl, kWave - 1);
    };
#pragma unroll
    for (int u = 0; u < kGqaHeld; ++u)
        if (u * kWave < n && (before <= y0 || gid == 0)) look(u, held[u]);
    for (int u = kGqaHeld; u * kWave < n && (before <= y0 || gid == 0); ++u) look(u, read(u * kWave + lane));
    seg = __builtin_amdgcn_readfirstlane(seg);

    // ---- the unit under way
    struct Unit {
        SegState ss;
        int sl, hu, nb;
        unsigned char *k, *v;                            // its rows in the cache
        int64_t fresh;                                   // byte offset of its row in k_new / v_new
    };
    auto set_segment = [&](Unit& u, const Words& w) {
        u.ss = seg_state<EV>(p, w.len, w.cap, w.off, w.base);
        u.nb = row_blocks(u.ss.len, BR);
    };
    auto enter_segment = [&](Unit& u, int i) {
        u.sl = __builtin_amdgcn_readfirstlane(seg_slot(p, i));
        set_segment(u, {uniform_load(p.lens + u.sl) & kLenMask, uniform_load(p.caps + u.sl), EV ? uniform_load(p.base_lens + u.sl) : 0, uniform_load(p.seg_off + u.sl)});
    };
    auto enter_head = [&](Unit& u, int hu) {
        const int kvh = (hu * G) / p.grp;
        u.hu = hu;
        int64_t at = (u.ss.off * p.Hkv + (int64_t)kvh * u.ss.cap) * ROWB;
        at = ((int64_t)__builtin_amdgcn_readfirstlane((int)(at >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
        u.k = p.kc + at; u.v = p.vc + at;
        u.fresh = ((int64_t)u.sl * p.Hkv + kvh) * ROWB;
    };
    // two cursors: the block that is worked on and, two blocks ahead, the one that is requested
    Unit cur;
    cur.sl = __builtin_amdgcn_readfirstlane(seg_slot(p, seg));
    set_segment(cur, mine);
    int blk;
    {
        const GqaPlace at = gqa_place(x0, first, cur.nb, HU);
        blk = at.blk;
        enter_head(cur, at.hu);
    }
    auto advance = [&](Unit& u, int& b, int& i) {          // true: a new unit
        int hu = u.hu;
        const GqaNext next = gqa_next(b, hu, i, u.nb, HU);
        if (next == GqaNext::segment) enter_segment(u, i);
        if (next != GqaNext::block) enter_head(u, hu);
        return next != GqaNext::block;
    };
    // copies of a block; K's chunks swizzled so that 16 rows at one chunk lie in different banks
    auto kpos = [](int row) { return LPR == 16 ? row & 15 : (row >> 1) & 7; };
    const uint32_t ring = (uint32_t)(uintptr_t)(lds_void_t*)&s_ring[wv][0][0];
    uint32_t koff[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) koff[i] = (uint32_t)(rg * ROWB + ((sub ^ kpos(i * RPI + rg)) * 16));
    // K or V of a block into its half of a stage; how many instructions that were
    auto issue = [&](const Unit& u, int b, int stage, auto is_v) {
        constexpr bool V = decltype(is_v)::value;
        const int r0 = b * BR;
        const uint32_t dst = __builtin_amdgcn_readfirstlane(ring + stage * 2 * TB + (V ? TB : 0));
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // what was there has been read
        if (r0 + BR <= u.ss.len_old) {
            const unsigned char* base = (V ? u.v : u.k) + (size_t)r0 * ROWB;
            if (once) {
#pragma unroll
                for (int i = 0; i < NI; ++i) copy16<true>(base + i * 1024, V ? (uint32_t)lane * 16u : koff[i], dst + i * 1024);
                return NI;
            }
#pragma unroll
            for (int i = 0; i < NI; ++i) copy16<false>(base + i * 1024, V ? (uint32_t)lane * 16u : koff[i], dst + i * 1024);
        } else if (r0 < u.ss.len) {
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int r = i * RPI + rg;
                const RowSource src = row_source<EV>(r0 + r, r0, u.ss.len, u.ss.len_old, u.ss.app, u.ss.ring);
                const unsigned char* from = src.from_new ? (V ? p.v_new : p.k_new) + u.fresh : (V ? u.v : u.k) + (int64_t)src.slot * ROWB;
                copy16_any(from + (V ? sub : sub ^ kpos(r)) * 16, dst + i * 1024);
            }
        } else {
            return 0;
        }
        return NI;
    };
    const uint32_t ldsq = (uint32_t)(uintptr_t)(lds_void_t*)&s_q[wv][0][0];
    int q_put = 0, q_get = 0;                             // the slots take turns
    auto issue_q = [&](const Unit& u) {
        const unsigned char* src = p.q + ((int64_t)u.sl * p.H + u.hu * G) * ROWB;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        const uint32_t dst = __builtin_amdgcn_readfirstlane(ldsq + q_put * (QB < 1024 ? 1024 : QB));
#pragma unroll
        for (int i = 0; i < (QB + 1023) / 1024; ++i) copy16_any(src + i * 1024 + (lane * 16) % (QB < 1024 ? QB : 1024), dst + i * 1024);
        q_put ^= 1;
    };
    constexpr std::false_type of_k{};
    constexpr std::true_type of_v{};
    Unit ahead = cur;
    int a_blk = blk, a_seg = seg;
    issue_q(ahead);
    issue(ahead, a_blk, 0, of_k);
    issue(ahead, a_blk, 0, of_v);
    int flying = 0;                                       // copies of the block after the next to work on
    if (x0 + 1 < x1) {
        if (advance(ahead, a_blk, a_seg)) issue_q(ahead);
        flying = issue(ahead, a_blk, 1, of_k);
        flying += issue(ahead, a_blk, 1, of_v);
    }
    bf16x8_t qb[NJ];

    // The older wavefronts of a SIMD are served first and are done (at 59 of 84 us) when the younger, too few to keep the
    // memory busy, have a fifth of their blocks left.  So every wavefront gives way as it gets on (then 63 and 69 of 80).
    const int quarter = (x1 - x0 + 3) / 4;
    int next_prio = x0 + quarter;
    __builtin_amdgcn_s_setprio(3);
    float o[G * 8], m_run = -INFINITY, l_run = 0.f, qs = 0.f;
    bool fresh_unit = true;
    int begun = x0 - blk;                                // flat number of the unit's first block
    for (int x = x0;; ++x) {
        const int stage = (x - x0) & 1;
        // the block and, with it, the queries of a new unit are here; the block after it may be on its way
        if (flying) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (fresh_unit) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                uint4 t = *(const uint4*)(&s_q[wv][q_get][0] + (kr < G ? kr : 0) * ROWB + (4 * j + kq) * 16);
                if (kr >= G) t = make_uint4(0, 0, 0, 0);
                qb[j] = __builtin_bit_cast(bf16x8_t, t);
            }
            q_get ^= 1;
            qs = uniform_load(p.scale + cur.sl % p.L) * 1.4426950408889634f;
            m_run = -INFINITY; l_run = 0.f;
#pragma unroll
            for (int e = 0; e < G * 8; ++e) o[e] = 0.f;
            fresh_unit = false;
        }
        const bool more = x + 1 < x1, ends = blk + 1 == cur.nb;
        if (x >= next_prio) {
            const int k = (x - x0) / quarter;
            if (k == 1) __builtin_amdgcn_s_setprio(2); else if (k == 2) __builtin_amdgcn_s_setprio(1); else __builtin_amdgcn_s_setprio(0);
            next_prio += quarter;
        }
        const int r0 = blk * BR;
        const unsigned char *sk = &s_ring[wv][stage][0], *sv = sk + TB;
        const SegState& ss = cur.ss;
        f32x4_t acc[NT];
        const bool some = r0 < ss.len, full = r0 + BR <= ss.len_old;
        if (some) {
            // the appended row goes to its slot out of the stage (only the first head group of a KV head writes)
            const int rn = ss.ring.r_new - r0;
            if (rn >= 0 && rn < BR && ss.app && (cur.hu * G) % p.grp == 0 && lane < 2 * LPR) {
                const bool is_v = lane >= LPR;
                const uint4 t = *(const uint4*)(is_v ? sv + rn * ROWB + sub * 16 : sk + rn * ROWB + ((sub ^ kpos(rn)) * 16));
                const size_t slot = (size_t)(ss.ring.r_new + (EV ? ss.ring.shift : 0));
                *(uint4*)((is_v ? cur.v : cur.k) + slot * ROWB + sub * 16) = t;
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                acc[t] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const int row = 16 * t + kr;
                    const bf16x8_t kf = __builtin_bit_cast(bf16x8_t, *(const uint4*)(sk + row * ROWB + (((4 * j + kq) ^ kpos(row)) * 16)));
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qb[j], acc[t], 0, 0, 0);
                }
            }
        }
        // the block after the next takes the place of this one, K now and V below
        const bool request = x + 2 < x1;
        flying = 0;
        if (request) {
            if (advance(ahead, a_blk, a_seg)) issue_q(ahead);
            flying = issue(ahead, a_blk, stage, of_k);
        }
        if (some) {
            float mx = -INFINITY;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float sc = acc[t][r] * qs;
                    if (!full) {
                        const int row = r0 + 16 * t + 4 * kq + r;
                        sc = (row < ss.len && row != ss.ring.r_mask) ? sc : -INFINITY;
                    }
                    acc[t][r] = sc;
                    mx = fmaxf(mx, sc);
                }
            {
                auto s2 = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
                mx = fmaxf(__uint_as_float(s2[0]), __uint_as_float(s2[1]));
                s2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
                mx = fmaxf(__uint_as_float(s2[0]), __uint_as_float(s2[1]));
            }
            const float mnew = fmaxf(m_run, mx), mref = mnew == -INFINITY ? 0.f : mnew;
            const float corr = __builtin_amdgcn_exp2f(m_run - mref);
            m_run = mnew;
            float psum = 0.f;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    acc[t][r] = __builtin_amdgcn_exp2f(acc[t][r] - mref);
                    psum += acc[t][r];
                }
            l_run = fmaf(l_run, corr, psum);
            if (__builtin_amdgcn_ballot_w64(kr < G && corr != 1.f)) {
                for_heads<G>([&](auto g) {
                    const float cg = row_bcast<g.value>(corr);
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[8 * g.value + e] *= cg;
                });
            }
            // the rows whose probabilities the own 16 lanes hold: 4 * kq + i, of the tile that the lane's half of them takes
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int row = NT == 1 ? 4 * kq + i : 16 * (rg & 1) + 4 * kq + i;
                uint4 vr = *(const uint4*)(sv + row * ROWB + sub * 16);
                if (!full) {
                    const bool valid = r0 + row < ss.len && r0 + row != ss.ring.r_mask;
                    vr.x = valid ? vr.x : 0; vr.y = valid ? vr.y : 0; vr.z = valid ? vr.z : 0; vr.w = valid ? vr.w : 0;
                }
                float vf[8];
                unpack16<true>(vr, vf);
                for_heads<G>([&](auto g) {
                    float pg = row_bcast<g.value>(acc[0][i]);
                    if constexpr (NT == 2) {
                        const float other = row_bcast<g.value>(acc[NT - 1][i]);   // by all lanes, also those that do not want it
                        pg = (rg & 1) ? other : pg;
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[8 * g.value + e] = fmaf(pg, vf[e], o[8 * g.value + e]);
                });
            }
        }
        if (request) issue(ahead, a_blk, stage, of_v);
        if constexpr (EV) {
            // the surviving token moves from its ring slot to the next permanent slot, which nobody reads in this launch
            if (blk == 0 && ss.app) {
                const int ring0 = ss.ring0, cs = ss.cs;
                if (ss.grad && (cur.hu * G) % p.grp == 0 && lane < 2 * LPR) {
                    unsigned char* base = lane >= LPR ? cur.v : cur.k;
                    *(uint4*)(base + (size_t)ss.len_old * ROWB + sub * 16) = *(const uint4*)(base + (size_t)(ring0 + cs) * ROWB + sub * 16);
                }
                if (p.kept_pos && cur.hu == 0 && lane == 0) {
                    int32_t* kp = p.kept_pos + ss.off;
                    kp[ring0 + p.slot_new] = p.N + p.t - 1;
                    if (ss.decide) {
                        if (ss.grad) kp[ss.len_old] = p.N + p.t - p.d - 1;
                        kp[ring0 + cs] = -1;
                    }
                }
            }
        }
        if (ends || !more) {
            // the row groups meet: afterwards register e is value e + 4 G (upper half) + 2 G (odd 16 lanes) of the G * 8
            float l = swap_add16(l_run, l_run);
            l = swap_add32(l, l);
            float f[G * 4], r[G * 2];
#pragma unroll
            for (int e = 0; e < G * 4; ++e) f[e] = swap_add32(o[e], o[e + G * 4]);
#pragma unroll
            for (int e = 0; e < G * 2; ++e) {
                r[e] = swap_add16(f[e], f[e + G * 2]);
                if constexpr (LPR == 8) r[e] += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(r[e]), 0x128, 0xF, 0xF, true));
            }
            const int E0 = (lane >> 5) * G * 4 + ((lane >> 4) & 1) * G * 2;
            const bool whole = ends && begun >= x0;
            const bool writes = LPR == 16 || (lane & 8) == 0;
            float* part = (float*)p.ws + gqa_partial_word(n) + (size_t)gqa_slot(gid, seg, cur.hu, HU) * (G * (D + 2));
#pragma unroll
            for (int e = 0; e < G * 2; e += 4) {
                const int g = (E0 + e) / 8, col = sub * 8 + (E0 + e) % 8;
                if (whole) {
                    const float den = __shfl(l, g, kWave), inv = den > 0.f ? 1.f : 0.f;     // an empty segment gives zeros
                    float y[4];
#pragma unroll
                    for (int z = 0; z < 4; ++z) y[z] = inv > 0.f ? r[e + z] / den : 0.f;
                    if (writes)
                        *(uint2*)((bf16_t*)p.out + ((size_t)cur.sl * p.H + cur.hu * G + g) * D + col) =
                            make_uint2(pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3]));
                } else if (writes) {
                    *(float4*)(part + g * D + col) = make_float4(r[e], r[e + 1], r[e + 2], r[e + 3]);
                }
            }
            if (!whole && lane < G) *(float2*)(part + G * D + 2 * lane) = make_float2(m_run, l);
            if (!more) break;
            begun = x + 1;
            fresh_unit = true;
        }
        advance(cur, blk, seg);
    }
}

// Adds up the partial results of every unit that several wavefronts shared, in groups of consecutive pieces, each in block
// order, and stores the new lengths.  One workgroup per unit: a unit of a long segment can have as many pieces as there are
// wavefronts, and in one wavefront their loads would follow each other (B2 H32/4 N8192, 73 pieces: 36 us).  Bound by its chain of
// memory round trips, so a group takes its own maximum from the pieces it adds up; with a pass over all maxima and a barrier
// ahead of that, one layer of 500 positions, H 32/8, D 128, kept whole took 11.7 us per call in both kernels, now 10.4, B4 N8192 10 %
// 82.6, now 81.0.  Four pieces in flight: the third workgroup of a compute unit costs more registers than eight are worth.
constexpr int kMergeThreads = 512;
template <int D, int G, bool EV>
__global__ void __launch_bounds__(kMergeThreads)
decode_gqa_merge_kernel(DecodeParams p) {
    constexpr int NE = G * D / 4, PG = kMergeThreads / NE, PST = G * (D + 2);   // float4 elements, groups of pieces
    constexpr int NP = 4;                                // pieces whose loads are in flight together
    __shared__ float s_m[PG][G], s_d[PG][G];
    __shared__ __attribute__((aligned(16))) float s_num[PG][G * D];
    const int HU = p.H / G, tid = threadIdx.x;
    const int i = blockIdx.x / HU, hu = blockIdx.x - i * HU, sl = seg_slot(p, i);
    const int share = uniform_load(p.ws);
    const int first = uniform_load(p.ws + kGqaHdr + i), nb = uniform_load(p.ws + kGqaHdr + i + 1) - first;
    if (hu == 0 && tid == 0)
        p.lens[sl] = seg_state<EV>(p, p.lens[sl] & kLenMask, p.caps[sl], p.seg_off[sl], EV ? p.base_lens[sl] : 0).len_next;
    const GqaPieces pieces = gqa_pieces(first, nb, hu, HU, share);
    const int np = pieces.n;
    if (np == 1) return;                                 // one wavefront had it all and wrote the output
    const float* ws = (const float*)p.ws + gqa_partial_word(p.n_seg) + (size_t)gqa_slot(pieces.wave, i, hu, HU) * PST;
    const int e = tid % NE, pg = tid / NE, g = e * 4 / D;
    const int per = (np + PG - 1) / PG, k0 = pg * per, k1 = k0 + per < np ? k0 + per : np;
    // numerators, denominator and the maximum they refer to of the group's pieces, in one pass over them
    float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
    float den = 0.f, m = -INFINITY;
    for (int k = k0; k < k1; k += NP) {
        float2 md[NP];
        float4 v[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            md[j] = make_float2(-INFINITY, 0.f);
            v[j] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (k + j < k1) {
                const float* piece = ws + (size_t)(k + j) * PST;
                md[j] = *(const float2*)(piece + G * D + 2 * g);
                v[j] = *(const float4*)(piece + 4 * e);
            }
        }
        float mn = m;
#pragma unroll
        for (int j = 0; j < NP; ++j) mn = fmaxf(mn, md[j].x);
        const float ref = mn == -INFINITY ? 0.f : mn, corr = __builtin_amdgcn_exp2f(m - ref);
        m = mn;
        num.x *= corr; num.y *= corr; num.z *= corr; num.w *= corr;
        den *= corr;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const float wgt = __builtin_amdgcn_exp2f(md[j].x - ref);
            num.x = fmaf(wgt, v[j].x, num.x); num.y = fmaf(wgt, v[j].y, num.y);
            num.z = fmaf(wgt, v[j].z, num.z); num.w = fmaf(wgt, v[j].w, num.w);
            den = fmaf(wgt, md[j].y, den);
        }
    }
    if constexpr (PG > 1) {
        *(float4*)&s_num[pg][4 * e] = num;
        if (4 * e % D == 0) { s_m[pg][g] = m; s_d[pg][g] = den; }
        __syncthreads();
        if (pg != 0) return;
        float M = m;
#pragma unroll
        for (int k = 1; k < PG; ++k) M = fmaxf(M, s_m[k][g]);
        const float ref = M == -INFINITY ? 0.f : M, own = __builtin_amdgcn_exp2f(m - ref);
        num.x *= own; num.y *= own; num.z *= own; num.w *= own;
        den *= own;
#pragma unroll
        for (int k = 1; k < PG; ++k) {
            const float4 v = *(const float4*)&s_num[k][4 * e];
            const float wgt = __builtin_amdgcn_exp2f(s_m[k][g] - ref);
            num.x = fmaf(wgt, v.x, num.x); num.y = fmaf(wgt, v.y, num.y);
            num.z = fmaf(wgt, v.z, num.z); num.w = fmaf(wgt, v.w, num.w);
            den = fmaf(wgt, s_d[k][g], den);
        }
    }
    const bool some = den > 0.f;                         // an empty segment gives zeros
    const float y0 = some ? num.x / den : 0.f, y1 = some ? num.y / den : 0.f, y2 = some ? num.z / den : 0.f, y3 = some ? num.w / den : 0.f;
    *(uint2*)((bf16_t*)p.out + ((size_t)sl * p.H + hu * G) * D + 4 * e) =
        make_uint2(pack_bf16(y0, y1), pack_bf16(y2, y3));
}

// Number of compute units of the current device (queried once per device).
int compute_units() {
    static int cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cached[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
        cached[dev] = n;
    }
    return cached[dev];
}

// Launch shapes of decode_attn_kernel.  A unit is one head group of one segment; its rows are dealt to its
// wavefronts in blocks of NI * 64/LPR rows.  What decides is how many wavefronts a launch has: 16 per compute unit are
// resident (4 per SIMD; 20 of a ranked launch of the plain bf16 step), and each start costs (12 800 units of 26 rows, one
// wavefront each: 42 us, of 136 rows 160, for rows that stream in 30 and 150).  Hence
//   up to 1.75 units per compute unit: 8 wavefronts per unit (32 units, one layer of the 7B shape: 8.6 -> 6.1 us; 16 wavefronts
//       per unit 6.2; 512 units with 4 against 8: N300 10.8 / 12.5 us, N680 11.5 / 12.4, 384 of N680 11.4 / 10.9), of short prompts,
//       keys of up to 50 KB per head, 4 if a unit is one head (96 units of 24 rows 5.5 / 5.8, 192 6.6 / 6.9, 416 9.4 / 9.6; of 80 rows 5.8 / 5.8, 6.8 / 7.0,
//       10.3 / 10.6; kept at 50 %, one layer of eight sequences, 100 rows 6.5 / 6.1; four fp32 heads, 128 units of 20 rows 7.4 / 7.1);
//   up to 4: 4 wavefronts per unit, which fill the chip (7B, batch 1, lengths within a factor 30: 21.3 -> 18.7 us; equal: 21.7
//       -> 21.0; equal lengths of 2048 rows and more are 1 ... 10 % slower than with two wavefronts and 16 loads in flight
//       each, 164.1 -> 169.6 us at 1024 units); of short prompts several units may share a workgroup (units_grouped);
//   beyond: one, two or four wavefronts per unit, the longest segments first (see ranked_shape).  The lengths differ by up
//       to two orders of magnitude, and in index order the launch ends with a few long segments on a chip that is
//       otherwise empty.
// Four row loads of K and of V in flight per wavefront; the next block's go into the registers of those that are used up.
template <bool BF16, int LPR, int G, bool EV>
static hipError_t launch_decode_s(DecodeParams p, int nblk, hipStream_t st) {
    constexpr int NI = 4;
    constexpr int OCC = G >= 4 ? 2 : 4, RES = BF16 && !EV ? kRankedResident : 16, ROCC = RES > 16 ? RES / 4 : OCC;   // (the pruning step spills at five wavefronts per SIMD)
    const int HU = p.H / G, cus = compute_units();
    p.n_seg = nblk / HU;
    if (4 * nblk <= cus) {
        hipLaunchKernelGGL((decode_attn_kernel<BF16, LPR, G, NI, 8, OCC, EV, -1>), dim3(HU, p.nl, p.B), dim3(8 * kWave), 0, st, p);
        return hipGetLastError();
    }
    const int row_bytes = p.D * (BF16 ? 2 : 4);
    if (units_grouped(p.n_seg, HU, p.nl, p.L, cus, p.N, row_bytes)) {
        p.turn = grouped_turn(p.n_seg);
        p.by_nl = fast_div(p.nl);
        p.by_seg = fast_div(p.n_seg);
        hipLaunchKernelGGL((decode_attn_kernel<BF16, LPR, G, NI, 4, OCC, EV, kGrouped>), dim3(p.n_seg, HU), dim3(4 * kWave), 0, st, p);
        return hipGetLastError();
    }
    if (4 * nblk <= 7 * cus && (G > 1 || p.N * row_bytes > 50 << 10)) {
        hipLaunchKernelGGL((decode_attn_kernel<BF16, LPR, G, NI, 8, OCC, EV, 0>), dim3(HU, p.nl, p.B), dim3(8 * kWave), 0, st, p);
        return hipGetLastError();
    }
    if (nblk <= 4 * cus) {
        hipLaunchKernelGGL((decode_attn_kernel<BF16, LPR, G, NI, 4, OCC, EV, 0>), dim3(HU, p.nl, p.B), dim3(4 * kWave), 0, st, p);
        return hipGetLastError();
    }
    const int ngrp = (p.n_seg + kRankRegs * kWave - 1) / (kRankRegs * kWave);
    p.rank.gsz = (p.n_seg + ngrp - 1) / ngrp;
    ranked_shape(p.rank, nblk, cus, p.N, row_bytes, RES);
    const dim3 grid(ranked_blocks(p.rank, HU) * ngrp), block(4 * kWave);
    const int lds = BF16 ? ranked_lds(p.rank, 4ll * grid.x, cus) : 0;
    if (p.rank.gsz <= kWave) hipLaunchKernelGGL((decode_attn_kernel<BF16, LPR, G, NI, 4, ROCC, EV, 1>), grid, block, lds, st, p);
    else hipLaunchKernelGGL((decode_attn_kernel<BF16, LPR, G, NI, 4, ROCC, EV, kRankRegs>), grid, block, lds, st, p);
    return hipGetLastError();
}

template <bool BF16, int LPR, bool EV>
static hipError_t launch_decode_g(const DecodeParams& p, int G, int nblk, hipStream_t st) {
    if constexpr (!BF16) {   // bf16 caches with several query heads per KV head use decode_gqa_kernel instead
        switch (G) {
            case 8: return launch_decode_s<BF16, LPR, 8, EV>(p, nblk, st);
            case 4: return launch_decode_s<BF16, LPR, 4, EV>(p, nblk, st);
            case 2: return launch_decode_s<BF16, LPR, 2, EV>(p, nblk, st);
            default: break;
        }
    }
    return launch_decode_s<BF16, LPR, 1, EV>(p, nblk, st);
}

// Workspace of a grouped-query launch in words: a slot for each unit and each wavefront of the largest launch, whatever N and the
// layer range (see gqa_partial_word; 4.3 MB with four heads of D 128 at up to 256 units).  A size that followed the prompt's length
// bounded the wavefronts instead: one layer a call, H 32/8, D 128, kept whole: N 500 8 wavefronts and 42 us, now 11.7; N 1000
// 44 -> 11.8; B1 L32 N500 50 %, all layers a launch, 33 -> 16.5, H32/4 40 -> 17.5.
static size_t gqa_ws_words(int n_seg, int H, int G, int D) {
    return gqa_partial_word(n_seg) + ((size_t)kGqaWavesMax + (size_t)n_seg * (H / G)) * G * (D + 2);
}

size_t decode_ws_bytes(const pkv_shape& s) {
    const int G = pick_group(s.H / s.Hkv);
    if (s.dtype != PKV_BF16 || G < 2) return 0;
    return gqa_ws_words(s.B * s.L, s.H, G, s.D) * 4 + kGqaWsAlign;
}

// Grouped-query bf16 launches: one resident round of wavefronts over the stream of blocks, then the partial results.
template <int D, int G, bool EV>
static hipError_t launch_gqa_s(DecodeParams p, const pkv_shape& s, void* ws, hipStream_t st) {
    p.n_seg = s.B * p.nl;
    p.ws = (int*)gqa_ws_base((uintptr_t)ws);
    const long long units = (long long)p.n_seg * (s.H / G);
    p.waves = compute_units() * 8;                         // two wavefronts per SIMD
    if (p.waves > kGqaWavesMax) p.waves = kGqaWavesMax;
    hipLaunchKernelGGL((decode_gqa_kernel<D, G, EV>), dim3((unsigned)((p.waves + kGqaWaves - 1) / kGqaWaves)), dim3(kGqaWaves * kWave), 0, st, p);
    hipLaunchKernelGGL((decode_gqa_merge_kernel<D, G, EV>), dim3((unsigned)units), dim3(kMergeThreads), 0, st, p);
    return hipGetLastError();
}

template <int D, bool EV>
static hipError_t launch_gqa(const DecodeParams& p, const pkv_shape& s, int G, void* ws, hipStream_t st) {
    switch (G) {
        case 8: return launch_gqa_s<D, 8, EV>(p, s, ws, st);
        case 4: return launch_gqa_s<D, 4, EV>(p, s, ws, st);
        default: return launch_gqa_s<D, 2, EV>(p, s, ws, st);
    }
}

template <bool EV>
static hipError_t launch_decode_any(const pkv_shape& s, const DecodeParams& p, void* ws, hipStream_t st) {
    const int G = pick_group(p.grp);
    const int nblk = s.B * p.nl * (s.H / G);
    const bool bf16 = s.dtype == PKV_BF16;
    if (bf16 && G >= 2)     // several query heads share the cached rows: scores on the matrix cores
        return s.D == 128 ? launch_gqa<128, EV>(p, s, G, ws, st) : launch_gqa<64, EV>(p, s, G, ws, st);
    const int lpr = s.D * (bf16 ? 2 : 4) / 16;
    if (bf16) {
        if (lpr == 8) return launch_decode_g<true, 8, EV>(p, G, nblk, st);
        return launch_decode_g<true, 16, EV>(p, G, nblk, st);
    }
    if (lpr == 16) return launch_decode_g<false, 16, EV>(p, G, nblk, st);
    return launch_decode_g<false, 32, EV>(p, G, nblk, st);
}

static DecodeParams make_params(const pkv_shape& s, int l0, int l1, const void* q, const void* k_new,
                                const void* v_new, const float* scale, void* kc, void* vc,
                                const int64_t* seg_off, const int32_t* caps, int32_t* lens, void* out) {
    DecodeParams p;
    p.B = s.B; p.L = s.L; p.l0 = l0; p.nl = l1 - l0; p.H = s.H; p.Hkv = s.Hkv; p.D = s.D;
    p.grp = s.H / s.Hkv; p.append = k_new != nullptr;
    p.q = (const unsigned char*)q; p.k_new = (const unsigned char*)k_new;
    p.v_new = (const unsigned char*)v_new; p.scale = scale;
    p.kc = (unsigned char*)kc; p.vc = (unsigned char*)vc; p.seg_off = seg_off; p.caps = caps;
    p.lens = lens; p.out = (unsigned char*)out;
    p.N = s.N; p.t = 0; p.d = 0; p.slot_new = 0; p.slot_due = 0; p.base_lens = nullptr; p.kept_pos = nullptr;
    p.n_seg = 0; p.waves = 0; p.ws = nullptr;
    p.rank = RankedShape{0, 0, 0, false};
    p.turn = 0; p.by_nl = p.by_seg = FastDiv{1, 0};
    return p;
}

hipError_t launch_decode(const pkv_shape& s, int l0, int l1, const void* q, const void* k_new,
                         const void* v_new, const float* scale, void* kc, void* vc,
                         const int64_t* seg_off, const int32_t* caps, int32_t* lens, void* out, void* ws,
                         hipStream_t st) {
    const DecodeParams p = make_params(s, l0, l1, q, k_new, v_new, scale, kc, vc, seg_off, caps, lens, out);
    return launch_decode_any<false>(s, p, ws, st);
}

hipError_t launch_decode_evict(const pkv_shape& s, int l0, int l1, const void* q, const void* k_new,
                               const void* v_new, const float* scale, void* kc, void* vc,
                               const int64_t* seg_off, const int32_t* caps, const int32_t* base_lens,
                               int32_t* lens, int32_t* kept_pos, int t, int d, void* out, void* ws,
                               hipStream_t st) {
    DecodeParams p = make_params(s, l0, l1, q, k_new, v_new, scale, kc, vc, seg_off, caps, lens, out);
    p.t = t; p.d = d; p.slot_new = (t - 1) % (d + 1); p.slot_due = t % (d + 1); p.base_lens = base_lens; p.kept_pos = kept_pos;
    return launch_decode_any<true>(s, p, ws, st);
}

}  // namespace pkv

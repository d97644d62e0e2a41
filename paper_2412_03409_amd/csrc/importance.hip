// Stage 1: KV importance (Sec. 3.2) -- column sums of the causal softmax, averaged over heads.
//
// bf16 inputs run on the matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulate), in one of two forms:
//   importance_stream_kernel, one sweep over the score matrix per launch: the log-sum-exp of the rows (queries
//       stationary in registers, keys stream through LDS), unless the caller has it, then the column sums (keys
//       stationary, queries stream).  The stationary row of a lane never changes, so its running maximum and sum, or
//       its column sum, is one register.
//   importance_fused_kernel, both sweeps in one launch that reads the queries and the keys of a head from HBM once:
//       for prompts of up to 768 positions without a given log-sum-exp, when the heads fill the chip.
//
// The head mean is another, tiny kernel: four quarters of the heads, each in head order, then their four sums, so the result
// is bitwise reproducible.  fp32 inputs (small validation shapes) have kernels of their own.
#include "pkv_common.hpp"
#include "block_order.hpp"

#include <type_traits>

namespace pkv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr int kStage = 128;   // streamed rows per LDS stage

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// Accumulator register r of lane `lane` holds row 8*(r/4) + 4*(lane/32) + r%4, column lane%32 of
// the 32x32 product.
__device__ __forceinline__ int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// ---- staging of a streamed kStage-row tile: global memory -> LDS without passing through registers ------
// gfx950's 16-byte global-to-LDS load writes lane i's 16 bytes to LDS[base + 16*i] (base is uniform per
// wavefront), i.e. one instruction fills 1 KB of consecutive LDS; each lane may fetch any global address.
// The tile is stored unpadded, rows of D bf16, with the 16-byte chunks of a row XOR-swizzled by the row
// index so that the MFMA fragment reads (32 rows x one chunk) hit all banks evenly:
//   chunk c of row r lives at chunk position c ^ ((r / RPB) & (CPR-1)),  RPB = rows per 256 bytes.
typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) const void glb_void_t;

template <int D, int WV = 4> struct Stage {
    static constexpr int CPR = D / 8;                 // 16-byte chunks per row
    static constexpr int ROWB = D * 2;                // bytes per row
    static constexpr int RPB = 256 / ROWB;            // rows per 256 bytes (one pass over the 64 banks)
    static constexpr int BYTES = kStage * ROWB;
    static constexpr int PIECES = BYTES / 1024;       // 1 KB pieces of the tile, dealt to the wavefronts in turn
    static constexpr int INSTS = (PIECES + WV - 1) / WV;
    // Issue the asynchronous copy of rows [row0, row0 + kStage) (clamped to N-1) into `lds`.
    static __device__ __forceinline__ void issue(const bf16_t* base, int64_t ld, int row0, int N,
                                                 unsigned char* lds, int wv, int lane) {
        // the per-lane address pieces are recomputed at every call (a few integer operations per stage): kept
        // across a long loop they would occupy two dozen registers
        asm volatile("" : "+v"(lane));
#pragma unroll
        for (int i = 0; i < INSTS; ++i) {
            const int inst = i * WV + wv;             // which 1 KB piece of the tile
            if (PIECES % WV != 0 && inst >= PIECES) break;
            const int L = inst * 64 + lane;           // linear chunk index in LDS
            const int row = L / CPR, pos = L % CPR;
            const int c = pos ^ ((row / RPB) & (CPR - 1));
            int grow = row0 + row;
            grow = grow < N ? grow : N - 1;
            // 32-bit element offset from the uniform base of this head (N * ld < 2^31, checked by the launcher)
            const bf16_t* g = base + ((uint32_t)grow * (uint32_t)ld + (uint32_t)(c * 8));
            __builtin_amdgcn_global_load_lds((glb_void_t*)g, (lds_void_t*)(lds + inst * 1024), 16, 0, 0);
        }
    }
    // MFMA operand fragment for k-step kk of the 32 rows starting at row0 (a multiple of 32)
    static __device__ __forceinline__ bf16x8 frag(const unsigned char* lds, int row0, int kk, int lane) {
        const int r = lane & 31;
        const int pos = (2 * kk + (lane >> 5)) ^ ((r / RPB) & (CPR - 1));
        return as_bf16x8(*(const uint4*)(lds + (row0 + r) * ROWB + pos * 16));
    }
};
// wait until this wavefront's global-to-LDS copies have landed (vmcnt = 0; other counters untouched)
__device__ __forceinline__ void wait_async_copies() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// The wavefront's stationary operand: two tiles of 32 rows (starting at row0 and row1), straight from global memory into the MFMA
// register layout.  flip = the rows are negated (exact in bf16) so that the logit scale is positive.
template <int D>
__device__ __forceinline__ void load_stationary(bf16x8 (&f)[2][D / 16], const bf16_t* base, int64_t ld, int row0,
                                                int row1, int N, int lane, bool flip) {
    const uint32_t sgn = flip ? 0x80008000u : 0u;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        int row = (a == 0 ? row0 : row1) + (lane & 31);
        row = row < N ? row : N - 1;
#pragma unroll
        for (int kk = 0; kk < D / 16; ++kk) {
            uint4 v = *(const uint4*)(base + (int64_t)row * ld + 16 * kk + 8 * (lane >> 5));
            v.x ^= sgn; v.y ^= sgn; v.z ^= sgn; v.w ^= sgn;
            f[a][kk] = as_bf16x8(v);
        }
    }
}

__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// All k-step fragments of a staged 32-row sub-tile into distinct registers: the reads are issued together
// and the MFMAs run back to back, instead of one LDS round trip per k-step.
template <int D>
__device__ __forceinline__ void load_frags(bf16x8 (&fr)[D / 16], const unsigned char* lds, int row0, int lane) {
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) fr[kk] = Stage<D>::frag(lds, row0, kk, lane);
}
// acc = A.B over all k-steps; STREAM_IS_A: the streamed fragment is the A (row) operand.
template <int KS, bool STREAM_IS_A>
__device__ __forceinline__ f32x16 mma_tile(const bf16x8 (&stat)[KS], const bf16x8 (&fr)[KS]) {
    f32x16 acc = {0};
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
        acc = STREAM_IS_A ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[kk], stat[kk], acc, 0, 0, 0)
                          : __builtin_amdgcn_mfma_f32_32x32x16_bf16(stat[kk], fr[kk], acc, 0, 0, 0);
    return acc;
}
// ---- fused kernel: Q and K are read from HBM once -------------------------------------------------------
// One workgroup of WV = 12 wavefronts owns one (sequence, layer, head) of up to 768 positions (one workgroup per CU,
// three wavefronts per SIMD: their MFMA chains and softmax phases overlap each other).  Its 32-query tiles are taken
// in PAIRS: tile i with tile T-1-i, so that every pair -- and therefore every wavefront -- has the same amount of
// causal work (T+1 tile products per sweep).
// The wavefront keeps its two query tiles in registers for the whole
// kernel and the keys stream through LDS (128-row stages, asynchronous copies, double-buffered) twice:
//   sweep 1:  S^T = K.Q^T (a lane holds one query): online max / sum -> lse of the wavefront's 64 rows
//   sweep 2:  S   = Q.K^T (a lane holds one key):   exp2(c*s - lse) summed over the lane's 32 query rows;
//             the keys come back from L2 / the last-level cache.
// Swapping the MFMA operands transposes the product, so the same stationary fragments serve both sweeps.  The
// column sums of one 128-key stage leave the workgroup once per stage: the wavefronts' values meet in LDS
// behind the barrier the stage needs anyway and are added in a fixed order (no atomics, bitwise reproducible).
struct FusedParams {
    int N;
    int T;                     // 32-row tiles: ceil(N / 32)
    int npairs;                // ceil(T / 2), at most the wavefronts of a workgroup
    int nheads;                // B*L*H
    int chunk;                 // heads per XCD
    FastDiv by_h, by_l, by_grp;   // H, L, H / Hkv
    const bf16_t* q; Strides qs;
    const bf16_t* k; Strides ks;
    const float* scale;        // [L]
    float* partial;            // [B*L*H][N] column sums
};

// barrier that orders LDS traffic only: loads from global memory that are still in flight stay in flight
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
// one wavefront copies a whole stage (rolled loop: a few address registers)
template <int D>
__device__ __forceinline__ void copy_stage(const bf16_t* base, int64_t ld, int row0, int N, unsigned char* lds, int lane) {
    using S1 = Stage<D, 1>;
#pragma unroll 2
    for (int inst = 0; inst < S1::PIECES; ++inst) {
        const int L = inst * 64 + lane;
        const int row = L / S1::CPR, pos = L % S1::CPR;
        const int c = pos ^ ((row / S1::RPB) & (S1::CPR - 1));
        int grow = row0 + row;
        grow = grow < N ? grow : N - 1;
        const bf16_t* g = base + ((uint32_t)grow * (uint32_t)ld + (uint32_t)(c * 8));
        __builtin_amdgcn_global_load_lds((glb_void_t*)g, (lds_void_t*)(lds + inst * 1024), 16, 0, 0);
    }
}
template <int D>
__device__ __forceinline__ void load_stationary_one(bf16x8 (&f)[D / 16], const bf16_t* base, int64_t ld, int row0,
                                                    int N, int lane, bool flip) {
    const uint32_t sgn = flip ? 0x80008000u : 0u;
    int row = row0 + (lane & 31);
    row = row < N ? row : N - 1;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
        uint4 v = *(const uint4*)(base + (int64_t)row * ld + 16 * kk + 8 * (lane >> 5));
        v.x ^= sgn; v.y ^= sgn; v.z ^= sgn; v.w ^= sgn;
        f[kk] = as_bf16x8(v);
    }
}

// WV wavefronts per workgroup; OCC wavefronts per SIMD the register allocation must allow.
// SPREAD (last wavefront without tiles): see the start of the kernel.
template <int D, int WV, int OCC, bool SPREAD>
__global__ void __launch_bounds__(WV * kWave, OCC)
importance_fused_kernel(FusedParams p) {
    constexpr int KS = D / 16;
    constexpr int NSUB = kStage / 32;
    using St = Stage<D, WV>;
    __shared__ __attribute__((aligned(16))) unsigned char s_tile0[St::BYTES];   // even steps
    __shared__ __attribute__((aligned(16))) unsigned char s_tile1[St::BYTES];   // odd steps
    __shared__ float s_red[2][WV][NSUB][32];              // column sums of a wavefront's rows:
                                                          // [parity][wavefront][sub-tile][key]
    __shared__ __attribute__((aligned(16))) float s_nl2[WV][2][32];   // -lse (log2 units) of a wavefront's two
                                                          // tiles by row; -inf for rows that do not exist
    // the wavefront index as a scalar: everything derived from it (which tiles exist, which sub-tiles are
    // needed) is then known to be uniform and branches on it are scalar branches
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int head = (int)(blockIdx.x % kXcds) * p.chunk + (int)(blockIdx.x / kXcds);
    if (head >= p.nheads) return;
    const DivMod bl_h = uniform_div_mod(head, p.by_h), b_l = uniform_div_mod(bl_h.q, p.by_l);
    const int h = bl_h.r, l = b_l.r, b = b_l.q;
    const bf16_t* qb = p.q + p.qs.b * b + p.qs.l * l + p.qs.h * h;
    const bf16_t* kb = p.k + p.ks.b * b + p.ks.l * l + p.ks.h * uniform_div_mod(h, p.by_grp).q;
    float* part = p.partial + (size_t)head * p.N;
    float c = uniform_load(p.scale + l) * kLog2e;
    const bool flip = c < 0.f;
    c = fmaxf(fabsf(c), 1e-30f);                           // > 0, so that c * (-inf) of a masked entry stays -inf

    // this wavefront's pair: the early tile tE and the late tile tL (only tL for the middle tile of an odd T)
    int tE = wv < p.npairs ? wv : -1, tL = wv < p.npairs ? p.T - 1 - wv : -1;
    if (tE == tL) tE = -1;
    const int qlo0 = 32 * tE, qlo1 = 32 * tL;             // negative: tile absent
    const int S = (p.N + kStage - 1) / kStage;            // key stages per sweep
    // Steps t = 0 .. 2S-1: step t works on key stage t mod S, sweep 1 for t < S and sweep 2 from S on, out of
    // s_tile{t & 1}; the stage of step t+1 is copied into the other buffer meanwhile.

    // SPREAD: the first sweep walks the key stages downwards: the late tiles are needed first (the last stage by
    // the two latest tiles only), the early tiles not before the low stages, so the queries are requested late
    // tile first and arrive while the first stages are worked on, instead of all before the first product.
    // For that the key copies are issued by the last wavefront alone -- the launcher picks this form only when
    // that wavefront has no tiles (fewer pairs than wavefronts) -- and the barriers order LDS traffic only: a
    // wavefront's query loads then stay in flight across barriers.  (Measured: -2..3 % at 680 positions.)
    const bool copier = wv == WV - 1;
    bf16x8 bq[2][KS];
    if constexpr (SPREAD) {
        if (copier) copy_stage<D>(kb, p.ks.n, (S - 1) * kStage, p.N, s_tile0, lane);
        else {
            if (tL >= 0) load_stationary_one<D>(bq[1], qb, p.qs.n, qlo1, p.N, lane, flip);
            if (tE >= 0) load_stationary_one<D>(bq[0], qb, p.qs.n, qlo0, p.N, lane, flip);
        }
    } else {
        St::issue(kb, p.ks.n, 0, p.N, s_tile0, wv, lane);
        load_stationary<D>(bq, qb, p.qs.n, tE < 0 ? 0 : qlo0, tL < 0 ? 0 : qlo1, p.N, lane, flip);
    }
    float mrun[2] = {-INFINITY, -INFINITY}, srun[2] = {0.f, 0.f};
    if constexpr (SPREAD) {
        if (copier) wait_async_copies();
        lds_barrier();
    } else {
        wait_async_copies();
        __syncthreads();
    }
    int par = 0;

    // sweep 1, one key stage: S^T = K.Q^T, a lane holds one query and 16 keys
    auto stage1 = [&](const unsigned char* cur, int s) {
#pragma unroll
        for (int j = 0; j < NSUB; ++j) {
            const int n0 = s * kStage + 32 * j;            // first key of the sub-tile
            const bool need0 = tE >= 0 && n0 <= qlo0 + 31;
            const bool need1 = tL >= 0 && n0 <= qlo1 + 31;
            if (!need1) continue;                          // tE < tL: need0 implies need1
            // the two products of the sub-tile one after the other (16 accumulator registers live at a time: the
            // other wavefronts of the SIMD fill the gaps of the single MFMA chain)
            bf16x8 fr[KS];
            load_frags<D>(fr, cur, 32 * j, lane);
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                if (a == 0 && !need0) continue;
                const f32x16 acc = mma_tile<KS, true>(bq[a], fr);
                const int qlo = a == 0 ? qlo0 : qlo1;
                float mnew, msafe, ps = 0.f;
                if (n0 + 31 <= qlo) {                      // every key of the sub-tile is visible to every query
                    float mx = max3(acc[0], acc[1], acc[2]);
#pragma unroll
                    for (int r = 3; r < 15; r += 2) mx = max3(mx, acc[r], acc[r + 1]);
                    mx = fmaxf(mx, acc[15]);
                    mnew = fmaxf(mrun[a], mx * c);
                    msafe = mnew;
#pragma unroll
                    for (int r = 0; r < 16; ++r) ps += __builtin_amdgcn_exp2f(fmaf(acc[r], c, -msafe));
                } else {                                   // the diagonal sub-tile: mask key > query
                    int q = lane & 31;
                    asm volatile("" : "+v"(q));            // keeps the compares out of loop-invariant registers
                    float mx = -INFINITY;
#pragma unroll
                    for (int r = 0; r < 16; ++r) mx = acc_row(r, lane) <= q ? fmaxf(mx, acc[r]) : mx;
                    mnew = fmaxf(mrun[a], mx * c);
                    msafe = mnew == -INFINITY ? 0.f : mnew;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const float e = __builtin_amdgcn_exp2f(fmaf(acc[r], c, -msafe));
                        ps += acc_row(r, lane) <= q ? e : 0.f;
                    }
                }
                srun[a] = srun[a] * __builtin_amdgcn_exp2f(mrun[a] - msafe) + ps;
                mrun[a] = mnew;
            }
        }
    };
    // lse of the wavefront's rows: lanes l and l^32 hold the two key halves of the same query; sweep 2 reads
    // the result by accumulator row from a wavefront-private LDS row
    auto finish_lse = [&]() {
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const float mo = __shfl_xor(mrun[a], 32, kWave), so = __shfl_xor(srun[a], 32, kWave);
            const float M = fmaxf(mrun[a], mo);
            const float Ssum = srun[a] * __builtin_amdgcn_exp2f(mrun[a] - M) + so * __builtin_amdgcn_exp2f(mo - M);
            const int t = a == 0 ? tE : tL;
            if (lane < 32) s_nl2[wv][a][lane] = (t >= 0 && 32 * t + lane < p.N) ? -(M + __log2f(Ssum)) : -INFINITY;
        }
    };
    // sweep 2, one key stage: S = Q.K^T, a lane holds one key and 16 queries; the column sums of each product
    // go to the product's own LDS slot
    auto stage2 = [&](const unsigned char* cur, int s) {
#pragma unroll
        for (int j = 0; j < NSUB; ++j) {
            const int n0 = s * kStage + 32 * j;
            const bool need0 = tE >= 0 && n0 <= qlo0 + 31;
            const bool need1 = tL >= 0 && n0 <= qlo1 + 31;
            float ps0 = 0.f, ps1 = 0.f;
            if (need1) {
                bf16x8 fr[KS];
                load_frags<D>(fr, cur, 32 * j, lane);
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    if (a == 0 && !need0) continue;
                    // -lse of accumulator rows 8q + 4*(lane/32) + 0..3: requested before the MFMA chain, so that
                    // the LDS round trip is over when the chain is
                    const float4* src = (const float4*)&s_nl2[wv][a][4 * (lane >> 5)];
                    float nl[16];
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        const float4 x = src[2 * q4];
                        nl[4 * q4] = x.x; nl[4 * q4 + 1] = x.y; nl[4 * q4 + 2] = x.z; nl[4 * q4 + 3] = x.w;
                    }
                    const f32x16 acc = mma_tile<KS, false>(bq[a], fr);
                    const int qlo = a == 0 ? qlo0 : qlo1;
                    float ps = 0.f;
                    if (n0 + 31 <= qlo) {                  // every key of the sub-tile is visible to every query
#pragma unroll
                        for (int r = 0; r < 16; ++r) ps += __builtin_amdgcn_exp2f(fmaf(acc[r], c, nl[r]));
                    } else {                               // the diagonal sub-tile: mask key > query
                        int key = lane & 31;
                        asm volatile("" : "+v"(key));      // keeps the compares out of loop-invariant registers
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const float pr = __builtin_amdgcn_exp2f(fmaf(acc[r], c, nl[r]));
                            ps += key <= acc_row(r, lane) ? pr : 0.f;
                        }
                    }
                    if (a == 0) ps0 = ps; else ps1 = ps;
                }
            }
            // lanes l and l+32 hold the two query halves of the same key
            const float ps = ps0 + ps1;
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(ps), __float_as_uint(ps), false, false);
            if (lane < 32) s_red[par][wv][j][lane] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
        }
    };
    auto step = [&](const unsigned char* cur, unsigned char* nxt, int t) {
        if (t + 1 < 2 * S) St::issue(kb, p.ks.n, ((t + 1) % S) * kStage, p.N, nxt, wv, lane);
        const int s = t >= S ? t - S : t;
        if (t < S) {
            stage1(cur, s);
            if (t == S - 1) finish_lse();
            wait_async_copies();
            __syncthreads();
        } else {
            stage2(cur, s);
            wait_async_copies();
            __syncthreads();
            if (threadIdx.x < kStage) {
                const int sub = threadIdx.x >> 5, c32 = threadIdx.x & 31;
                float sum = 0.f;
#pragma unroll
                for (int w = 0; w < WV; ++w) sum += s_red[par][w][sub][c32];
                const int n = s * kStage + threadIdx.x;
                if (n < p.N) part[n] = sum;
            }
            par ^= 1;
        }
    };
    if constexpr (!SPREAD) {
        for (int t = 0; t < 2 * S; t += 2) {
            step(s_tile0, s_tile1, t);
            if (t + 1 < 2 * S) step(s_tile1, s_tile0, t + 1);
        }
    } else {
        // step u of sweep 1 works on stage S-1-u, step u of sweep 2 on stage u; buffers alternate throughout
        auto flush = [&](int s) {
            if (threadIdx.x < kStage) {
                const int sub = threadIdx.x >> 5, c32 = threadIdx.x & 31;
                float sum = 0.f;
#pragma unroll
                for (int w = 0; w < WV; ++w) sum += s_red[par][w][sub][c32];
                const int n = s * kStage + threadIdx.x;
                if (n < p.N) part[n] = sum;
            }
            par ^= 1;
        };
        auto step1 = [&](const unsigned char* cur, unsigned char* nxt, int u) {
            if (copier) copy_stage<D>(kb, p.ks.n, (u + 1 < S ? S - 2 - u : 0) * kStage, p.N, nxt, lane);
            stage1(cur, S - 1 - u);
            if (u == S - 1) finish_lse();
            if (copier) wait_async_copies();
            lds_barrier();
        };
        auto step2 = [&](const unsigned char* cur, unsigned char* nxt, int u) {
            if (copier && u + 1 < S) copy_stage<D>(kb, p.ks.n, (u + 1) * kStage, p.N, nxt, lane);
            stage2(cur, u);
            if (copier) wait_async_copies();
            lds_barrier();
            flush(u);
        };
        int sel = 0;
        for (int u = 0; u < S; ++u, sel ^= 1) {
            if (sel == 0) step1(s_tile0, s_tile1, u); else step1(s_tile1, s_tile0, u);
        }
        // every query load has been consumed by now; saying so keeps the second sweep free of waits for them
        __builtin_amdgcn_s_waitcnt(0x0F70);
        for (int u = 0; u < S; ++u, sel ^= 1) {
            if (sel == 0) step2(s_tile0, s_tile1, u); else step2(s_tile1, s_tile0, u);
        }
    }
}

struct StreamParams {
    int N;
    int nheads;                // B*L*H
    int heads_per_xcd;
    FastDiv nblk;              // blocks of stationary rows per head
    FastDiv tail;              // heads of an XCD whose blocks run longest first
    FastDiv by_h, by_l, by_grp;   // H, L, H / Hkv
    const bf16_t* q; Strides qs;
    const bf16_t* k; Strides ks;
    const float* scale;        // [L]
    const float* lse_in;       // column sums: [B,L,H,N], times nl_scale the negative log-sum-exp in log2 units
    float nl_scale;
    float* out;                // [B,L,H,N]: column sums, or the negative log-sum-exp in log2 units
};
constexpr int kStWaves = 4, kStStage = 64;   // wavefronts that share a stage, streamed rows per stage
constexpr int kStTailBlocks = 256;

// ---- streamed kernels: one sweep each ------------------------------------------------------------------
// COLS = true: a wavefront owns NK tiles of 32 keys as the B operand of the product and the queries that see them
// stream through LDS as the A operand: a lane holds one key and 16 queries of each product, and the column sum of a
// key is one register from the first query to the last -- nothing meets in LDS, one store per key at the end.
// COLS = false: the same with 32 * NK queries stationary and the keys streaming: running maximum and sum per lane,
// the row log-sum-exp at the end.
// Bound by the vector ALU (fma, exp2, add per score: 276 cycles per 32x32 product) with the matrix cores next to it
// (256); no form spills (NK = 2 at D = 128: 156 and 162 registers of the 170 of three wavefronts per SIMD).  NK = 2: a
// fragment read from LDS feeds two products; from two rounds of workgroups on (B4 H32/8 N8192, column sums: 1105 us = 995
// TFLOP/s, NK = 1 1230), below NK = 1 fills the chip better (B2 H32 N2048: 58 against 71 us).
// GS = 2: two groups of four wavefronts share a block and take its stages in turn, for launches of about one
// workgroup per CU, whose time is the longest block's (one layer, H32 N680: 17 against 19 us with the head mean).
// Against the fused kernel with a given log-sum-exp, which kept the queries stationary, let the wavefronts' column
// sums meet in LDS at every stage and had one workgroup per head: 31 -> 17 us there, 115 -> 77 us at B8 H40 N1021,
// 1264 -> 1104 us at B4 H32/8 N8192.
template <int D, int NK, int GS, bool COLS>
__global__ void __launch_bounds__(GS * kStWaves * kWave, 3)
importance_stream_kernel(StreamParams p) {
    constexpr int KS = D / 16;
    constexpr int ROWB = D * 2, CPR = D / 8, RPB = 256 / ROWB;
    constexpr int BLK = kStWaves * 32 * NK;               // stationary rows per workgroup
    constexpr int INSTS = kStStage * ROWB / 1024 / kStWaves;
    __shared__ __attribute__((aligned(1024))) unsigned char s_a[GS][kStStage * ROWB];
    __shared__ __attribute__((aligned(1024))) unsigned char s_b[GS][kStStage * ROWB];
    __shared__ __attribute__((aligned(16))) float s_nl[2][GS][kStStage];
    __shared__ float s_part[2][kStWaves][kWave];           // GS > 1: one group's shares at a time
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wv = wave % kStWaves, gs = wave / kStWaves;  // the groups of four wavefronts take the stages in turn
    const int ln = lane & 31, hf = lane >> 5;
    // blocks of a head next to each other on one XCD, the XCD's last p.tail heads longest block first
    // (all arguments in one round trip to memory: left to itself the compiler asks for them as it comes to them)
    asm volatile("" : : "s"(p.q), "s"(p.k), "s"(p.qs.b), "s"(p.qs.l), "s"(p.qs.h), "s"(p.qs.n), "s"(p.ks.b), "s"(p.ks.l), "s"(p.ks.h), "s"(p.ks.n), "s"(p.scale));
    const int j = (int)(blockIdx.x / kXcds);
    HeadBlock hb = head_block(j, p.heads_per_xcd, p.nblk, p.tail);
    hb.head = __builtin_amdgcn_readfirstlane(hb.head); hb.rank = __builtin_amdgcn_readfirstlane(hb.rank);
    const int head = (int)(blockIdx.x % kXcds) * p.heads_per_xcd + hb.head;
    if (head >= p.nheads) return;
    const int blk = COLS ? hb.rank : (int)p.nblk.d - 1 - hb.rank;
    const DivMod bl_h = uniform_div_mod(head, p.by_h), b_l = uniform_div_mod(bl_h.q, p.by_l);
    const int h = bl_h.r, l = b_l.r, b = b_l.q;
    const bf16_t* qb = p.q + p.qs.b * b + p.qs.l * l + p.qs.h * h;
    const bf16_t* kb = p.k + p.ks.b * b + p.ks.l * l + p.ks.h * uniform_div_mod(h, p.by_grp).q;
    const bf16_t* st_base = COLS ? kb : qb;
    const bf16_t* sm_base = COLS ? qb : kb;
    const int64_t st_ld = COLS ? p.ks.n : p.qs.n;
    const uint32_t sm_ld = (uint32_t)(COLS ? p.qs.n : p.ks.n);    // N * stride < 2^31, checked by the launcher
    float c = uniform_load(p.scale + l) * kLog2e;
    const bool flip = c < 0.f;
    c = fmaxf(fabsf(c), 1e-30f);
    // The earlier tiles of a block (COLS = false: the later ones) have up to 4 * NK products more than the others, and wavefront w
    // of every workgroup runs on the same SIMD.  So a wavefront takes tiles w and 7 - w; with one tile each, the order differs
    // between the two groups and between the workgroups of a compute unit.  (With products in the future left out one by one
    // instead of a wavefront's stage at a time: attention and importance of B8 H40 N1021 208 -> 204 us, both sweeps of B1 L8
    // H32/8 N2000 314 -> 303, of H32/4 N8192 602 -> 596.)
    const int x0 = blk * BLK;                             // first stationary row of the workgroup
    const int tw = NK == 2 ? wv : GS > 1 ? (gs == 0 ? wv : kStWaves - 1 - wv) : (wv + j / 32) % kStWaves;
    auto tile = [&](int t) { return x0 + 32 * (t == 0 ? tw : 2 * kStWaves - 1 - tw); };   // first row of the wavefront's tile t
    const int xw = tile(0), xl = tile(NK - 1);            // of its earliest and its latest one
    const int first = COLS ? x0 : 0;                      // first streamed row
    const int nst = COLS ? (p.N - x0 + kStStage - 1) / kStStage : (min(p.N, x0 + BLK) + kStStage - 1) / kStStage;

    int cp_row[INSTS], cp_col[INSTS];
#pragma unroll
    for (int i = 0; i < INSTS; ++i) {
        const int idx = (wv * INSTS + i) * kWave + lane;
        const int r = idx / CPR, pos = idx % CPR;
        cp_row[i] = r;
        cp_col[i] = 8 * (pos ^ ((r / RPB) & (CPR - 1)));
    }
    float nl_next = 0.f;                                  // of row nl_row, as it lies in memory
    int nl_row = 0;
    auto issue = [&](int st, unsigned char* dst) {
#pragma unroll
        for (int i = 0; i < INSTS; ++i) {
            int row = first + st * kStStage + cp_row[i];
            row = row < p.N ? row : p.N - 1;
            __builtin_amdgcn_global_load_lds((glb_void_t*)(sm_base + ((uint32_t)row * sm_ld + (uint32_t)cp_col[i])),
                                             (lds_void_t*)(dst + (wv * INSTS + i) * 1024), 16, 0, 0);
        }
        // Without a branch, and as an atomic load so that the compiler neither waits for it here (with the product behind a condition
        // it waited for the whole stage) nor moves it behind the work on the stage before: one wavefront did, and with it all at
        // the next barrier.
        if constexpr (COLS) {
            nl_row = first + st * kStStage + lane;
            nl_next = __hip_atomic_load(p.lse_in + (size_t)head * p.N + (nl_row < p.N ? nl_row : p.N - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        }
    };
    if (gs < nst) issue(gs, s_a[gs]);
    bf16x8 f[NK][KS];
#pragma unroll
    for (int t = 0; t < NK; ++t) {
        int row = tile(t) + ln;
        row = row < p.N ? row : p.N - 1;
        const uint32_t sgn = flip ? 0x80008000u : 0u;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            uint4 v = *(const uint4*)(st_base + (int64_t)row * st_ld + 16 * kk + 8 * hf);
            v.x ^= sgn; v.y ^= sgn; v.z ^= sgn; v.w ^= sgn;
            f[t][kk] = as_bf16x8(v);
        }
    }
    uint32_t aoff[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
        aoff[kk] = (uint32_t)(ln * ROWB + (((2 * kk + hf) ^ ((ln / RPB) & (CPR - 1))) * 16));
        asm volatile("" : "+v"(aoff[kk]));
    }
    float mrun[NK], srun[NK];
#pragma unroll
    for (int t = 0; t < NK; ++t) { mrun[t] = -INFINITY; srun[t] = 0.f; }

    // one stage; DIAG: it holds rows in the future of some of the wavefront's tiles.  There a product wholly in the future is left
    // out and only the one on the diagonal is masked.
    auto attend = [&](auto diag_tag, int st, const unsigned char* buf, int par) {
        constexpr bool DIAG = decltype(diag_tag)::value;
        const int r0 = first + st * kStStage;
#pragma unroll
        for (int u = 0; u < kStStage / 32; ++u) {
            const int ru = r0 + 32 * u;
            if (DIAG && (COLS ? ru < xw : ru > xl)) continue;
            bf16x8 fr[KS];
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) fr[kk] = as_bf16x8(*(const uint4*)(buf + u * 32 * ROWB + aoff[kk]));
            float nl[16];
            if constexpr (COLS) {
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const float4 x = *(const float4*)&s_nl[par][gs][32 * u + 8 * q4 + 4 * hf];
                    nl[4 * q4] = x.x; nl[4 * q4 + 1] = x.y; nl[4 * q4 + 2] = x.z; nl[4 * q4 + 3] = x.w;
                }
            }
#pragma unroll
            for (int t = 0; t < NK; ++t) {
                const int xt = tile(t);
                if (DIAG && (COLS ? ru < xt : ru > xt || xt >= p.N)) continue;
                f32x16 acc = {0};
#pragma unroll
                for (int kk = 0; kk < KS; ++kk) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[kk], f[t][kk], acc, 0, 0, 0);
                // register r holds streamed row ru + 4*hf + 8*(r/4) + r%4
                const int d = xt + ln - (ru + 4 * hf);
                if constexpr (COLS) {
                    float ps = 0.f;
                    if (DIAG && ru == xt) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const float e = __builtin_amdgcn_exp2f(fmaf(acc[r], c, nl[r]));
                            ps += 8 * (r >> 2) + (r & 3) >= d ? e : 0.f;
                        }
                    } else {
#pragma unroll
                        for (int r = 0; r < 16; ++r) ps += __builtin_amdgcn_exp2f(fmaf(acc[r], c, nl[r]));
                    }
                    srun[t] += ps;
                } else {
                    if (DIAG && ru == xt) {
                        const int lim = min(d, p.N - 1 - (ru + 4 * hf));
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[r] = 8 * (r >> 2) + (r & 3) <= lim ? acc[r] : -INFINITY;
                    }
                    float mx = max3(acc[0], acc[1], acc[2]);
#pragma unroll
                    for (int r = 3; r < 15; r += 2) mx = max3(mx, acc[r], acc[r + 1]);
                    mx = fmaxf(mx, acc[15]) * c;
                    const float mnew = fmaxf(mrun[t], mx);
                    const float mref = mnew == -INFINITY ? 0.f : mnew;
                    float ps = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; ++r) ps += __builtin_amdgcn_exp2f(fmaf(acc[r], c, -mref));
                    srun[t] = srun[t] * __builtin_amdgcn_exp2f(mrun[t] - mref) + ps;
                    mrun[t] = mnew;
                }
            }
        }
    };
    constexpr std::true_type diag{};
    constexpr std::false_type plain{};
    auto sync = [&](int par) {
        if (COLS && wv == 0) s_nl[par][gs][lane] = nl_row < p.N ? p.nl_scale * nl_next : -INFINITY;   // rows past the end weigh 0
        wait_async_copies();
        __syncthreads();
    };
    // a stage in the future of, across or past the wavefront's tiles
    auto step = [&](int st, const unsigned char* buf, int par) {
        const int r0 = first + st * kStStage, r1 = r0 + kStStage - 1;
        if (xw >= p.N || st >= nst || (COLS ? r1 < xw : r0 > xl + 31)) return;
        if (xl < p.N && (COLS ? r0 > xl : r1 < xw)) attend(plain, st, buf, par); else attend(diag, st, buf, par);
    };
    for (int i = 0; i < nst; i += 2 * GS) {
        const int st = i + gs;
        sync(0);
        if (st + GS < nst) issue(st + GS, s_b[gs]);
        step(st, s_a[gs], 0);
        if (i + GS >= nst) break;
        sync(1);
        if (st + 2 * GS < nst) issue(st + 2 * GS, s_a[gs]);
        step(st + GS, s_b[gs], 1);
    }
    // the groups' shares of a stationary row, in group order
    if constexpr (GS > 1) {
        static_assert(NK == 1, "one stationary tile per wavefront");
        for (int g = 1; g < GS; ++g) {
            __syncthreads();
            if (gs == g) {
                // lane -> slot of the wavefront with the same tile in group 0
                s_part[0][tw][lane] = srun[0];
                if (!COLS) s_part[1][tw][lane] = mrun[0];
            }
            __syncthreads();
            if (gs == 0) {
                const float so = s_part[0][tw][lane];
                if constexpr (COLS) srun[0] += so;
                else {
                    const float mo = s_part[1][tw][lane], M = fmaxf(mrun[0], mo), ref = M == -INFINITY ? 0.f : M;
                    srun[0] = srun[0] * __builtin_amdgcn_exp2f(mrun[0] - ref) + so * __builtin_amdgcn_exp2f(mo - ref);
                    mrun[0] = M;
                }
            }
        }
        if (gs != 0) return;
    }
    // the two halves of a stationary row
#pragma unroll
    for (int t = 0; t < NK; ++t) {
        const int row = tile(t) + ln;
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(srun[t]), __float_as_uint(srun[t]), false, false);
        const float s0 = __uint_as_float(sw[0]), s1 = __uint_as_float(sw[1]);
        float res = s0 + s1;
        if constexpr (!COLS) {
            const auto mw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mrun[t]), __float_as_uint(mrun[t]), false, false);
            const float m0 = __uint_as_float(mw[0]), m1 = __uint_as_float(mw[1]);
            const float M = fmaxf(m0, m1);
            res = -(M + __log2f(s0 * __builtin_amdgcn_exp2f(m0 - M) + s1 * __builtin_amdgcn_exp2f(m1 - M)));
        }
        if (hf == 0 && row < p.N) p.out[(size_t)head * p.N + row] = res;
    }
}

// importance[b,l,n] = (1/H) * sum_h partial[b,l,h,n].
// A workgroup takes 64 consecutive keys; its four wavefronts each add a quarter of the heads in order
// (several loads in flight: the sum is bound by memory latency, not by bytes) and the four sums are added in
// wavefront order, so the result does not depend on timing.
// The heads past a quarter's last eight are requested together like the others (one after the other before),
// with the arguments and the divisions by N at the kernel's start this took the whole importance of 4 x 12 heads
// x 500 keys of 64 from 17.1 to 16.5 us, of 40 layers x 24 heads x 300 from 57.8 to 56.6.
constexpr int kMeanKeys = 64, kMeanParts = 4;
__global__ void __launch_bounds__(kMeanKeys * kMeanParts)
head_mean_parts_kernel(int H, int N, FastDiv by_n, long long total, const float* __restrict__ partial,
                       float* __restrict__ importance) {
    __shared__ float s_acc[kMeanParts][kMeanKeys];
    asm volatile("" : : "s"(partial), "s"(importance), "s"(by_n.d), "s"(by_n.mul), "s"(total), "s"(N), "s"(H));   // the arguments at once
    const int lane = threadIdx.x % kMeanKeys, part = threadIdx.x / kMeanKeys;
    const long long i = ((long long)blockIdx.y * gridDim.x + blockIdx.x) * kMeanKeys + lane;
    const bool live = i < total;
    long long bl = 0;
    int n = 0;
    if (total <= 0x7fffffff) {                            // (the whole grid: a 64-bit division takes over a hundred instructions)
        const DivMod x = div_mod(live ? (int)i : 0, by_n);
        bl = x.q; n = x.r;
    } else if (live) {
        bl = i / N; n = (int)(i % N);
    }
    const int per = (H + kMeanParts - 1) / kMeanParts;
    const int h0 = part * per, h1 = min(H, h0 + per);
    const float* src = partial + (size_t)bl * H * N + n;
    float acc = 0.f;
    if (live) {
        for (int h = h0; h < h1; h += 8) {                // (the heads past a quarter's last: its last once more, not added)
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = src[(size_t)min(h + j, h1 - 1) * N];
#pragma unroll
            for (int j = 0; j < 8; ++j) acc = h + j < h1 ? acc + v[j] : acc;
        }
    }
    s_acc[part][lane] = acc;
    __syncthreads();
    if (part == 0 && live) {
        float sum = s_acc[0][lane];
#pragma unroll
        for (int q = 1; q < kMeanParts; ++q) sum += s_acc[q][lane];
        importance[i] = sum / (float)H;
    }
}

// ---- fp32 storage --------------------------------------------------------------------------------------
// Both products on v_mfma_f32_16x16x4_f32 (fp32 operands, so nothing is rounded that one-thread-per-row loops would
// keep).  A workgroup owns 16 rows of one head -- queries for the log-sum-exp, keys for the column sums -- as the
// B operand in registers; its wavefronts take the 16-row tiles of the other tensor in turn as the A operand, so
// that a lane holds one stationary row (lane % 16) and four streamed ones.  The four quarters of a row's columns are
// the four k-slots of the MFMA: lane quarter kq loads columns kq*D/4 ... of its row with 16-byte loads, the same for
// both operands, and no data goes through LDS.  Bound: latency at the small shapes that fp32 storage is used with
// (B1 L4 H2 N128 D64: one row per thread on 8 workgroups took 637 + 831 us, these take 6.6 + 4.9), else the fp32 matrix
// rate.
typedef __attribute__((ext_vector_type(4))) float f32x4;

struct F32Params {
    int B, L, H, Hkv, N;
    const float* q; Strides qs;
    const float* k; Strides ks;
    const float* scale;
    const float* lse_in;       // column sums
    float* out;                // log-sum-exp (natural log) or column sums, [B,L,H,N]
};

constexpr int kF32Waves = 4;

template <int D>
__device__ __forceinline__ void load_f32_rows(f32x4 (&f)[D / 16], const float* base, int64_t ld, int row0, int N, int lane) {
    int row = row0 + (lane & 15);
    row = row < N ? row : N - 1;
    const float* src = base + (int64_t)row * ld + (lane >> 4) * (D / 4);
#pragma unroll
    for (int i = 0; i < D / 16; ++i) f[i] = *(const f32x4*)(src + 4 * i);
}

// LSE: 16 queries against the keys they see.  Otherwise: 16 keys against the queries that see them.
template <int D, bool LSE>
__global__ void __launch_bounds__(kF32Waves * kWave)
importance_f32_kernel(F32Params p) {
    constexpr int KF = D / 16;
    __shared__ float s_m[kF32Waves][16], s_s[kF32Waves][16];
    const int T = (p.N + 15) / 16;
    const long long id = (long long)blockIdx.y * gridDim.x + blockIdx.x;
    const int t = (int)(id % T);
    const long long head = id / T;
    if (head >= (long long)p.B * p.L * p.H) return;
    const int h = (int)(head % p.H), l = (int)((head / p.H) % p.L), b = (int)(head / ((long long)p.H * p.L));
    const float* qb = p.q + p.qs.b * b + p.qs.l * l + p.qs.h * h;
    const float* kb = p.k + p.ks.b * b + p.ks.l * l + p.ks.h * (h / (p.H / p.Hkv));
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int col = lane & 15, rq = lane >> 4;            // stationary row, streamed rows 4*rq .. 4*rq + 3
    const float c = uniform_load(p.scale + l) * kLog2e;
    const float* sb = LSE ? kb : qb;
    const int64_t sld = LSE ? p.ks.n : p.qs.n;
    const int first = LSE ? 0 : t, last = LSE ? t : T - 1;
    f32x4 st[KF], cur[KF], nxt[KF];
    load_f32_rows<D>(st, LSE ? qb : kb, LSE ? p.qs.n : p.ks.n, 16 * t, p.N, lane);
    float mrun = -INFINITY, srun = 0.f;
    const int mine = 16 * t + col;
    if (first + wv <= last) load_f32_rows<D>(cur, sb, sld, 16 * (first + wv), p.N, lane);
    for (int u = first + wv; u <= last; u += kF32Waves) {
        const bool more = u + kF32Waves <= last;
        if (more) load_f32_rows<D>(nxt, sb, sld, 16 * (u + kF32Waves), p.N, lane);
        float nl[4];
        if constexpr (!LSE) {
            const float* lse = p.lse_in + (size_t)head * p.N;
#pragma unroll
            for (int r = 0; r < 4; ++r) nl[r] = lse[min(16 * u + 4 * rq + r, p.N - 1)] * -kLog2e;
        }
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < KF; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(cur[i][e], st[i][e], acc, 0, 0, 0);
        float x[4];
        bool see[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int other = 16 * u + 4 * rq + r;         // key (LSE) or query
            see[r] = other < p.N && (LSE ? other <= mine : other >= mine);
            x[r] = acc[r] * c;
        }
        if constexpr (LSE) {
            float mnew = mrun;
#pragma unroll
            for (int r = 0; r < 4; ++r) mnew = see[r] ? fmaxf(mnew, x[r]) : mnew;
            const float mref = mnew == -INFINITY ? 0.f : mnew;
            float ps = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) ps += see[r] ? __builtin_amdgcn_exp2f(x[r] - mref) : 0.f;
            srun = srun * __builtin_amdgcn_exp2f(mrun - mref) + ps;
            mrun = mnew;
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) srun += see[r] ? __builtin_amdgcn_exp2f(x[r] + nl[r]) : 0.f;
        }
        if (more) {
#pragma unroll
            for (int i = 0; i < KF; ++i) cur[i] = nxt[i];
        }
    }
    // the four lanes of a stationary row, then the wavefronts, in a fixed order
    auto merge = [](float& m, float& sum, float mo, float so) {
        const float M = fmaxf(m, mo), ref = M == -INFINITY ? 0.f : M;
        sum = sum * __builtin_amdgcn_exp2f(m - ref) + so * __builtin_amdgcn_exp2f(mo - ref);
        m = M;
    };
#pragma unroll
    for (int sh = 16; sh < kWave; sh <<= 1) {
        const float so = __shfl_xor(srun, sh, kWave);
        if constexpr (LSE) { const float mo = __shfl_xor(mrun, sh, kWave); merge(mrun, srun, mo, so); }
        else srun += so;
    }
    if (rq == 0) { s_m[wv][col] = mrun; s_s[wv][col] = srun; }
    __syncthreads();
    if (threadIdx.x < 16 && mine < p.N) {
        float m = s_m[0][col], sum = s_s[0][col];
#pragma unroll
        for (int w = 1; w < kF32Waves; ++w) {
            if constexpr (LSE) merge(m, sum, s_m[w][col], s_s[w][col]);
            else sum += s_s[w][col];
        }
        p.out[(size_t)head * p.N + mine] = LSE ? (m + __log2f(sum)) * kLn2 : sum;
    }
}

constexpr long long kMaxGridX = 1 << 23;   // workgroups of 256 threads: fewer than 2^32 threads in a grid's row

template <bool LSE>
static hipError_t launch_importance_f32(const pkv_shape& s, const F32Params& p, hipStream_t st) {
    const long long nblk = (long long)s.B * s.L * s.H * ((s.N + 15) / 16);
    const long long gx = nblk < kMaxGridX ? nblk : kMaxGridX, gy = (nblk + gx - 1) / gx;
    if (gy > 65535) return hipErrorInvalidValue;
    const dim3 grid((unsigned)gx, (unsigned)gy), block(kF32Waves * kWave);
    if (s.D == 128) hipLaunchKernelGGL((importance_f32_kernel<128, LSE>), grid, block, 0, st, p);
    else hipLaunchKernelGGL((importance_f32_kernel<64, LSE>), grid, block, 0, st, p);
    return hipGetLastError();
}

static size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// wavefronts per workgroup of the fused kernel: 12 (one workgroup per CU, three wavefronts per SIMD), a pair of
// 32-query tiles each: heads of up to 768 positions
constexpr int kFusedWaves = 12;
constexpr int kFusedOcc = 1;
constexpr int kFusedMaxN = 64 * kFusedWaves;

// Whether a call without a given log-sum-exp runs on the fused kernel.  It takes one head per CU and round and reads Q
// and K once; the stream kernels share the chip evenly but read both twice, in two launches.  N = 680, streams against
// fused: 64 heads 32 / 48 us, 192: 54 / 53, 256: 67 / 58, 320: 81 / 100, 384: 97 / 101, 640: 145 / 149, 768: 170 / 157,
// 1024: 240 / 213 -- fused when its rounds are nearly full.  Up to 256 positions one round of it is never slower
// (64 heads of 100: 15.1 / 13.3 us, 256 of 200: 22.1 / 20.2).
static bool fused_fits(const pkv_shape& s, long long cus) {
    if (s.N > kFusedMaxN) return false;
    const long long heads = (long long)s.B * s.L * s.H;
    const long long rounds = (heads + cus - 1) / cus;
    return rounds == 1 ? s.N <= 256 || heads * 4 >= cus * 3 : heads * 8 >= rounds * cus * 7;
}

// Rows of N floats per head that the kernels use: the column sums and, without a given log-sum-exp, the call's own behind
// them.  Only the fused kernel keeps that to itself: a short bf16 prompt without room for it runs there.
static size_t ws_rows_bytes(const pkv_shape& s, int rows) {
    return align_up(rows * (size_t)s.B * s.L * s.H * s.N * sizeof(float), 256);
}
static size_t stream_ws_bytes(const pkv_shape& s) { return ws_rows_bytes(s, 2); }
// What a call accepts at least.
size_t importance_ws_min_bytes(const pkv_shape& s, bool has_lse) {
    if (s.dtype == PKV_F32) return ws_rows_bytes(s, 1) * (has_lse ? 1 : 2);
    return has_lse || s.N <= kFusedMaxN ? ws_rows_bytes(s, 1) : stream_ws_bytes(s);
}
// What the size query returns: for bf16 one row per 768 positions, what earlier versions of the kernels used and callers
// have sized by, or the stream kernels' two where they are the faster form for a short prompt.  The query knows no device:
// it asks for the 256 compute units of the MI355X, and the launcher decides by those there are.
size_t importance_ws_bytes(const pkv_shape& s, bool has_lse) {
    if (s.dtype == PKV_F32) return importance_ws_min_bytes(s, has_lse);
    if (s.N <= kFusedMaxN && !has_lse && !fused_fits(s, 256)) return stream_ws_bytes(s);
    return ws_rows_bytes(s, (s.N + kFusedMaxN - 1) / kFusedMaxN);
}

template <int NK, int GS, bool COLS>
static void launch_stream_d(const pkv_shape& s, const StreamParams& p, dim3 grid, hipStream_t st) {
    const dim3 block(GS * kStWaves * kWave);
    if (s.D == 128) hipLaunchKernelGGL((importance_stream_kernel<128, NK, GS, COLS>), grid, block, 0, st, p);
    else hipLaunchKernelGGL((importance_stream_kernel<64, NK, GS, COLS>), grid, block, 0, st, p);
}
template <bool COLS>
static hipError_t launch_stream(const pkv_shape& s, StreamParams p, hipStream_t st) {
    const long long cus = compute_units(), hx = ((long long)p.nheads + kXcds - 1) / kXcds;   // heads per XCD
    // 64 stationary rows per wavefront from two rounds of workgroups on, unless that pads the blocks further (1024
    // heads of 100 positions: 47 against 32 us); for the column sums of D = 128 with three to six blocks per head also
    // where these just fill one round of three workgroups per CU (256 heads of 680: 36.3 against 39.2 us, of 768: 40.3
    // against 43.7; 192 of 768: 37.1 against 36.3; six blocks, 128 heads of 1500: 61.6 against 62.5; 96 of 2048 with eight:
    // 83.0 against 79.9)
    const long long nb2 = (s.N + 255) / 256, nb1 = (s.N + 127) / 128, blocks = p.nheads * nb2;
    const bool wide = (blocks >= 4 * cus && (2 * nb2 == nb1 || nb2 > 2)) ||
                      (COLS && s.D == 128 && nb2 >= 3 && nb2 <= 6 && 2 * blocks >= 5 * cus && blocks <= 3 * cus);
    const long long nblk = wide ? nb2 : nb1, tail = (kStTailBlocks + nblk - 1) / nblk;
    if (hx * kXcds * nblk > 0x7fffffffll) return hipErrorInvalidValue;
    p.nblk = fast_div(nblk);
    p.tail = fast_div(tail < hx ? tail : hx);
    p.heads_per_xcd = (int)hx;
    const dim3 grid((unsigned)(hx * kXcds * nblk));
    if (wide) launch_stream_d<2, 1, COLS>(s, p, grid, st);
    else if (p.nheads * nblk * 4 <= 5 * cus) launch_stream_d<1, 2, COLS>(s, p, grid, st);
    else launch_stream_d<1, 1, COLS>(s, p, grid, st);
    return hipGetLastError();
}

hipError_t launch_importance(const pkv_shape& s, const void* q, Strides qs, const void* k, Strides ks,
                             const float* scale, const float* lse, float* importance, void* ws, size_t ws_bytes,
                             hipStream_t st) {
    float* partial = (float*)ws;
    float* lse_ws = partial + (size_t)s.B * s.L * s.H * s.N;
    const long long total = (long long)s.B * s.L * s.N, heads = (long long)s.B * s.L * s.H;
    if (s.dtype != PKV_F32 && !heads_fit(heads, kXcds)) return hipErrorInvalidValue;
    hipError_t e;
    if (s.dtype == PKV_F32) {
        F32Params p{s.B, s.L, s.H, s.Hkv, s.N, (const float*)q, qs, (const float*)k, ks, scale, nullptr, lse_ws};
        if (!lse && (e = launch_importance_f32<true>(s, p, st)) != hipSuccess) return e;
        p.lse_in = lse ? lse : lse_ws; p.out = partial;
        if ((e = launch_importance_f32<false>(s, p, st)) != hipSuccess) return e;
    } else if (lse || (!fused_fits(s, compute_units()) && ws_bytes >= stream_ws_bytes(s))) {
        StreamParams p;
        p.N = s.N; p.nheads = (int)heads; p.by_h = fast_div(s.H); p.by_l = fast_div(s.L); p.by_grp = fast_div(s.H / s.Hkv);
        p.q = (const bf16_t*)q; p.qs = qs; p.k = (const bf16_t*)k; p.ks = ks; p.scale = scale;
        p.lse_in = nullptr; p.nl_scale = lse ? -kLog2e : 1.f; p.out = lse_ws;
        if (!lse && (e = launch_stream<false>(s, p, st)) != hipSuccess) return e;
        p.lse_in = lse ? lse : lse_ws; p.out = partial;
        if ((e = launch_stream<true>(s, p, st)) != hipSuccess) return e;
    } else {
        FusedParams p;
        p.N = s.N;
        p.T = (s.N + 31) / 32;
        p.npairs = (p.T + 1) / 2;
        p.nheads = (int)heads;
        p.chunk = (int)((heads + kXcds - 1) / kXcds);
        p.by_h = fast_div(s.H); p.by_l = fast_div(s.L); p.by_grp = fast_div(s.H / s.Hkv);
        p.q = (const bf16_t*)q; p.qs = qs; p.k = (const bf16_t*)k; p.ks = ks; p.scale = scale;
        p.partial = partial;
        if (p.npairs > kFusedWaves) return hipErrorInvalidValue;
        const dim3 grid((unsigned)p.chunk * kXcds), block(kFusedWaves * kWave);
        const bool spread = p.npairs < kFusedWaves;       // the last wavefront only copies
        if (spread) {
            if (s.D == 128) hipLaunchKernelGGL((importance_fused_kernel<128, kFusedWaves, kFusedOcc, true>), grid, block, 0, st, p);
            else hipLaunchKernelGGL((importance_fused_kernel<64, kFusedWaves, kFusedOcc, true>), grid, block, 0, st, p);
        } else {
            if (s.D == 128) hipLaunchKernelGGL((importance_fused_kernel<128, kFusedWaves, kFusedOcc, false>), grid, block, 0, st, p);
            else hipLaunchKernelGGL((importance_fused_kernel<64, kFusedWaves, kFusedOcc, false>), grid, block, 0, st, p);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const long long nblk = (total + kMeanKeys - 1) / kMeanKeys;
    const long long gx = nblk < kMaxGridX ? nblk : kMaxGridX, gy = (nblk + gx - 1) / gx;
    if (gy > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(head_mean_parts_kernel, dim3((unsigned)gx, (unsigned)gy), dim3(kMeanKeys * kMeanParts), 0, st, s.H,
                       s.N, fast_div(s.N), total, partial, importance);
    return hipGetLastError();
}

}  // namespace pkv

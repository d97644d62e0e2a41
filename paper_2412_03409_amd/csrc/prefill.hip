// Causal prefill attention that also emits the log-sum-exp of every row (Sec. 3.1: the prefill phase
// attends over the whole prompt; Sec. 3.2 builds the importance from the same score matrix).  With the
// row lse handed over, the importance stage needs one pass over Q K^T instead of two.
//
//  prefill_attn_kernel  one workgroup = 128 queries of one (sequence, layer, head); a wavefront owns 32 of
//                       them.  Keys and values stream through LDS 64 rows at a time (asynchronous
//                       global-to-LDS copies, double-buffered).  Both products run on the matrix cores with
//                       v_mfma_f32_32x32x16_bf16:
//                         S^T[32 keys x 32 queries] = K[32 x D] . Q^T            (A = K rows from LDS)
//                         O^T[32 d    x 32 queries] += V^T[32 d x 16 keys] . P^T (B = the probabilities,
//                                                       straight from the accumulators of S^T)
//                       In the accumulator layout a lane holds one query and 16 keys, so the softmax state
//                       is per lane and P^T needs no data movement: the 8 keys a lane contributes to a
//                       16-key product are 8 consecutive accumulator registers.  V^T in that same key
//                       order comes from LDS with gfx950's transposing 64-bit read: 16 lanes point at
//                       4 keys x 16 columns of row-major V and each receives 4 keys of one column.
#include "pkv_common.hpp"
#include "fast_div.hpp"

#include <type_traits>

namespace pkv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef short v4i16_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16_t lds_v4i16_t;

struct PrefillParams {
    int N;
    int heads, heads_per_xcd;      // B*L*H
    FastDiv nqb;                   // query blocks of a head
    FastDiv tail;                  // heads of an XCD whose blocks run longest first (see the kernel)
    FastDiv by_h, by_l, by_grp;    // H, L, H / Hkv
    const bf16_t* q; Strides qs;
    const bf16_t* k; Strides ks;
    const bf16_t* v; Strides vs;
    const float* scale;   // [L]
    bf16_t* out;          // [B,L,H,N,D]
    float* lse;           // [B,L,H,N] natural log
};

constexpr int kPfQueries = 128;   // queries per workgroup (4 wavefronts x 2 tiles x 16)
constexpr int kPfStage = 64;      // keys per LDS stage
constexpr int kPfTailBlocks = 256;   // workgroups of an XCD at the end of a launch that run longest first (4 per slot)

// 4 keys of one column of row-major V: lane r of a 16-lane group points at 4 consecutive columns of key
// r/4 (columns 4*(r%4) ...); lane i receives column i of keys 0..3.
__device__ __forceinline__ v4i16_t lds_read_tr(const unsigned char* p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)p);
}

// Chunk swizzle of the staged rows: chunk c of row r sits at position c ^ swz(r).  The fragment reads of K
// touch 16 consecutive rows at one chunk, the transposing reads of V touch 4 consecutive rows at 4
// consecutive chunks; swapping the two low bit pairs of the row index sends both patterns to distinct banks.
template <int CPR>
__device__ __forceinline__ int swz(int r) {
    if constexpr (CPR == 16) return ((r & 3) << 2) | ((r >> 2) & 3);
    else return ((r & 1) << 2) | ((r >> 1) & 3);
}

template <int D>
__global__ void __launch_bounds__(256, 2)   // two wavefronts per SIMD: at most 256 registers, accumulators included
prefill_attn_kernel(PrefillParams p) {
    constexpr int ROWB = D * 2;
    constexpr int CPR = D / 8;            // 16-byte chunks per row
    constexpr int NJ = D / 16;            // MFMAs per S^T tile
    constexpr int NDT = D / 32;           // 32-column tiles of the output
    constexpr int NKT = kPfStage / 32;
    constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;
    // rows are stored unpadded, their 16-byte chunks swizzled (see swz).
    // Two statically separate buffer pairs: while one is read, the asynchronous copy of the next stage
    // fills the other, and the compiler can see that the two do not alias
    __shared__ __attribute__((aligned(1024))) unsigned char sKa[kPfStage * ROWB];
    __shared__ __attribute__((aligned(1024))) unsigned char sVa[kPfStage * ROWB];
    __shared__ __attribute__((aligned(1024))) unsigned char sKb[kPfStage * ROWB];
    __shared__ __attribute__((aligned(1024))) unsigned char sVb[kPfStage * ROWB];

    // (all arguments in one round trip to memory: left to itself the compiler asks for them as it comes to them)
    asm volatile("" : : "s"(p.q), "s"(p.k), "s"(p.v), "s"(p.qs.b), "s"(p.qs.l), "s"(p.qs.h), "s"(p.qs.n), "s"(p.ks.b), "s"(p.ks.l), "s"(p.ks.h),
                 "s"(p.ks.n), "s"(p.vs.b), "s"(p.vs.l), "s"(p.vs.h), "s"(p.vs.n), "s"(p.scale));
    const int nqb = (int)p.nqb.d;
    // The query blocks of one head run next to each other on one XCD (the hardware deals consecutive workgroups
    // out to the eight XCDs in turn) and share the head's K and V through that XCD's L2, as do the query heads
    // of one KV head; within a head the long (late) query blocks start first.  The last p.tail heads of an XCD are
    // taken together, all their longest blocks first: in head order the launch would end on a few long blocks
    // (64 heads of 2048 positions: 107 -> 86 us; 320 heads of 1021: 164 -> 154; all heads that way loses the
    // sharing: 1024 heads of 680 positions 253 -> 309 us).
    const int j = (int)(blockIdx.x / kXcds);              // index inside the XCD
    const int hx = p.heads_per_xcd, lead = hx - (int)p.tail.d;   // the XCD's heads; the last p.tail of them longest block first
    int qb, hl;
    if (j < lead * nqb) { const DivMod x = uniform_div_mod(j, p.nqb); hl = x.q; qb = nqb - 1 - x.r; }
    else { const DivMod x = uniform_div_mod(j - lead * nqb, p.tail); qb = nqb - 1 - x.q; hl = lead + x.r; }
    const int hh = (int)(blockIdx.x % kXcds) * hx + hl;
    if (hh >= p.heads) return;
    const DivMod bl_h = uniform_div_mod(hh, p.by_h), b_l = uniform_div_mod(bl_h.q, p.by_l);
    const int h = bl_h.r, l = b_l.r, b = b_l.q;
    const int kvh = uniform_div_mod(h, p.by_grp).q;
    const bf16_t* qbase = p.q + p.qs.b * b + p.qs.l * l + p.qs.h * h;
    const bf16_t* kbase = p.k + p.ks.b * b + p.ks.l * l + p.ks.h * kvh;
    const bf16_t* vbase = p.v + p.vs.b * b + p.vs.l * l + p.vs.h * kvh;
    const int lane = threadIdx.x & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int ln = lane & 31, hf = lane >> 5;               // MFMA operand row / column, and k-half
    const int q0 = qb * kPfQueries + wv * 32;               // first query of this wavefront
    const int query = q0 + ln;
    float sc_l = uniform_load(p.scale + l);
    const int last_q = min(p.N, (qb + 1) * kPfQueries) - 1;  // last query of the workgroup
    const int nst = last_q / kPfStage + 1;                   // stages that hold a key <= last_q

    // asynchronous copy of one stage (keys and values) into a buffer pair: gfx950's 16-byte global-to-LDS
    // load writes lane i's bytes to LDS[base + 16*i], so one instruction fills 1 KB of consecutive LDS and
    // the swizzle is applied on the global side
    constexpr int kInst = kPfStage * ROWB / 1024 / 4;        // copy instructions per wavefront and tensor
    int cp_row[kInst], cp_col[kInst];                        // row within the stage and first element of the chunk
#pragma unroll
    for (int i = 0; i < kInst; ++i) {
        const int idx = (wv * kInst + i) * 64 + lane;
        const int r = idx / CPR, pos = idx % CPR;
        cp_row[i] = r;
        cp_col[i] = 8 * (pos ^ swz<CPR>(r));
    }
    const uint32_t ksn = (uint32_t)p.ks.n, vsn = (uint32_t)p.vs.n;   // N * stride < 2^31, checked by the launcher
    auto issue = [&](int st, unsigned char* dK, unsigned char* dV) {
#pragma unroll
        for (int i = 0; i < kInst; ++i) {
            int row = st * kPfStage + cp_row[i];
            row = row < p.N ? row : p.N - 1;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(kbase + ((uint32_t)row * ksn + (uint32_t)cp_col[i])),
                                             (__attribute__((address_space(3))) void*)(dK + (wv * kInst + i) * 1024), 16, 0, 0);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(vbase + ((uint32_t)row * vsn + (uint32_t)cp_col[i])),
                                             (__attribute__((address_space(3))) void*)(dV + (wv * kInst + i) * 1024), 16, 0, 0);
        }
    };
    // The first stage is requested ahead of the queries: the two round trips to memory pass together (one layer of
    // H32 N680, attention and importance, with the arithmetic at the start 34.6 -> 33.0 us).
    issue(0, sKa, sVa);
    // a negative logit scale is moved into the queries (negation is exact in bf16), so that the running
    // maximum can be taken on the raw products
    asm volatile("" : "+s"(sc_l));                          // first looked at here
    const float qs0 = fabsf(sc_l) * kLog2e;
    const float qs = qs0 < 1e-30f ? 1e-30f : qs0;           // > 0, so that a masked -inf stays one; NaN stays NaN
    const uint32_t sgn = sc_l < 0.f ? 0x80008000u : 0u;

    // the queries: B operand of the score products, one fragment per 16 columns of the head dimension
    bf16x8_t qf[NJ];
    {
        const int row = query < p.N ? query : p.N - 1;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            uint4 t = *(const uint4*)(qbase + p.qs.n * row + 16 * j + 8 * hf);
            t.x ^= sgn; t.y ^= sgn; t.z ^= sgn; t.w ^= sgn;
            qf[j] = __builtin_bit_cast(bf16x8_t, t);
        }
    }
    f32x16_t o[NDT];
    float m_run = -INFINITY, l_run = 0.f;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;

    // byte offsets of this lane's fragment reads inside a staged tile: computed once (a 16-row step of the swizzled
    // layout is a plain offset)
    uint32_t koff[NJ], voff[NDT][2];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        koff[j] = (uint32_t)(ln * ROWB + (((2 * j + hf) ^ swz<CPR>(ln)) * 16));
        asm volatile("" : "+v"(koff[j]));
    }
    {
        // the 16 lanes of a group point at 4 consecutive keys x 16 columns and each receives the 4 keys of its column
        const int g2 = (lane >> 4) & 1, i16 = lane & 15;
        const int vrow = 4 * hf + (i16 >> 2);
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const int chunk = 4 * dt + 2 * g2 + ((i16 & 3) >> 1), r = vrow + 8 * x;
                voff[dt][x] = (uint32_t)(r * ROWB + ((chunk ^ swz<CPR>(r)) * 16) + (i16 & 1) * 8);
                asm volatile("" : "+v"(voff[dt][x]));
            }
    }
    // One stage of kPfStage keys for this wavefront, both 32-key tiles at once: one look at the reference,
    // and the second tile's products cover the latency of the first.  MASKED: the stage holds keys some of its
    // queries must not see; a plain stage costs no compare (the masks cost 70 vector instructions per tile when
    // one body served both).  Measured against 32 keys at a time, in turn on one card:
    // 202 -> 145 us at B8 H40 N1021, 2660 -> 2385 us at B4 H32/8 N8192 (922 TFLOP/s), 26.6 -> 22.5 us at H32 N680.
    // Forcing the exponentials between the matrix instructions (scheduling groups) changed nothing.
    auto attend = [&](auto masked_tag, int key0, const unsigned char* sK, const unsigned char* sV) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        // The second tile of the wavefront's own stage may lie wholly in its queries' future.  It is left out, so that no
        // value in it -- infinite or NaN -- is multiplied by a probability of zero.
        const bool second = !MASKED || key0 + 32 <= q0;
        // scores S^T[64 keys x 32 queries] = K . Q^T, two 32-key products
        f32x16_t s[NKT];
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt) {
#pragma unroll
            for (int r = 0; r < 16; ++r) s[kt][r] = 0.f;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const bf16x8_t kf = __builtin_bit_cast(bf16x8_t, *(const uint4*)(sK + kt * 32 * ROWB + koff[j]));
                s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[j], s[kt], 0, 0, 0);
            }
        }
        if constexpr (MASKED) {
            const int lim = min(query, p.N - 1) - key0 - 4 * hf;     // register r holds key 8*(r/4) + r%4 + 4*hf
#pragma unroll
            for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r) s[kt][r] = 32 * kt + 8 * (r >> 2) + (r & 3) <= lim ? s[kt][r] : -INFINITY;
        }
        // The reference of a tile's probabilities is the maximum over the keys up to the end of that 32-key tile: they are
        // rounded to bf16, and against the maximum over both tiles the largest of the first would not be exactly 1.
        // (One reference for both is 2 ... 8 % faster -- 142 and 2310 us at the sizes above, 20.8 at H32 N680 -- but its
        // error against fp64 was larger for each of 15 inputs, 1.4687e-3 -> 1.4718e-3 at N680, 1.6439e-3 -> 1.6492e-3 at
        // N200.  Letting the maximum grow by 2^8 first: 1.5e-3 -> 1.7e-3.)
        // Most stages of a long prompt move no query's maximum: that takes one look, before the two halves of a query
        // exchange theirs.  Otherwise the output is rescaled in front of each tile that moves it.
        float mx[NKT];
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt) {
            mx[kt] = s[kt][0];
#pragma unroll
            for (int r = 1; r + 1 < 16; r += 2) mx[kt] = fmaxf(fmaxf(mx[kt], s[kt][r]), s[kt][r + 1]);
            mx[kt] = fmaxf(mx[kt], s[kt][15]);
        }
        float mref[NKT], corr[NKT];
        bool later = false;                                  // the second tile moves it
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt) { mref[kt] = m_run; corr[kt] = 1.f; }
        if (__builtin_amdgcn_ballot_w64(fmaxf(mx[0], mx[1]) * qs > m_run)) {
#pragma unroll
            for (int kt = 0; kt < NKT; ++kt) {
                const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx[kt]), __float_as_uint(mx[kt]), false, false);
                mref[kt] = fmaxf(m_run, fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * qs);
                corr[kt] = mref[kt] == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run - mref[kt]);
                if (kt == 1) later = __builtin_amdgcn_ballot_w64(mref[kt] > m_run) != 0;
                m_run = mref[kt];
            }
            if (__builtin_amdgcn_ballot_w64(corr[0] != 1.f)) {
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[dt][r] *= corr[0];
            }
        }
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt) {
            if (kt == 1 && !second) break;
            const float ref = mref[kt] == -INFINITY ? 0.f : mref[kt];      // no finite score so far
            bf16x8_t pf[2];
            float psum = 0.f;
#pragma unroll
            for (int sl = 0; sl < 2; ++sl) {
                uint32_t pk[4];
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    const float p0 = __builtin_amdgcn_exp2f(fmaf(s[kt][8 * sl + e], qs, -ref));
                    const float p1 = __builtin_amdgcn_exp2f(fmaf(s[kt][8 * sl + e + 1], qs, -ref));
                    psum += p0 + p1;
                    pk[e / 2] = pack_bf16(p0, p1);
                }
                pf[sl] = __builtin_bit_cast(bf16x8_t, make_uint4(pk[0], pk[1], pk[2], pk[3]));
            }
            l_run = fmaf(l_run, corr[kt], psum);
            if (kt == 1 && later) {
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[dt][r] *= corr[kt];
            }
#pragma unroll
            for (int sl = 0; sl < 2; ++sl)
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt) {
                    const unsigned char* sVs = sV + (32 * kt + 16 * sl) * ROWB;
                    const v4i16_t a0 = lds_read_tr(sVs + voff[dt][0]), a1 = lds_read_tr(sVs + voff[dt][1]);
                    const bf16x8_t vf = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7));
                    o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[sl], o[dt], 0, 0, 0);
                }
        }
    };
    // Stages 0 .. 2*qb - 1 lie wholly in the past of every query of the workgroup; the last one or two hold the
    // diagonal.
    auto sync = [&]() {
        __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0): this wavefront's part of the stage has landed
        __syncthreads();                                     // ... and everybody's; the other pair is free again
    };
    constexpr std::true_type masked{};
    constexpr std::false_type plain{};
    for (int st = 0; st < 2 * qb; st += 2) {
        sync();
        issue(st + 1, sKb, sVb);
        attend(plain, st * kPfStage, sKa, sVa);
        sync();
        issue(st + 2, sKa, sVa);
        attend(plain, (st + 1) * kPfStage, sKb, sVb);
    }
    sync();
    if (2 * qb + 1 < nst) issue(2 * qb + 1, sKb, sVb);
    if (q0 < p.N) attend(masked, 2 * qb * kPfStage, sKa, sVa);
    if (2 * qb + 1 < nst) {
        sync();
        if (wv >= 2 && q0 < p.N) attend(masked, (2 * qb + 1) * kPfStage, sKb, sVb);
    }

    // epilogue: the two halves of a query column hold partial row sums; the output tile is transposed:
    // register r of o[dt] is column 32*dt + 8*(r/4) + 4*hf + r%4 of this lane's query
    float lt = l_run;
    lt += __shfl_xor(lt, 32, kWave);
    if (query < p.N) {
        const float inv = 1.f / lt;
        const size_t row = (size_t)hh * p.N + query;
        if (hf == 0) p.lse[row] = kLn2 * (m_run + __builtin_amdgcn_logf(lt));
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
            for (int g = 0; g < 4; g += 2) {
                // the two halves of a query swap, so that a lane stores 16 bytes: lane half hf gets columns 8*(g + hf) ...
                uint32_t w[2][2];
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    w[x][0] = pack_bf16(o[dt][4 * (g + x)] * inv, o[dt][4 * (g + x) + 1] * inv);
                    w[x][1] = pack_bf16(o[dt][4 * (g + x) + 2] * inv, o[dt][4 * (g + x) + 3] * inv);
                }
                const auto s0 = __builtin_amdgcn_permlane32_swap(w[0][0], w[1][0], false, false);
                const auto s1 = __builtin_amdgcn_permlane32_swap(w[0][1], w[1][1], false, false);
                *(uint4*)(p.out + row * D + 32 * dt + 8 * (g + hf)) = make_uint4(s0[0], s1[0], s0[1], s1[1]);
            }
    }
}

hipError_t launch_prefill_attn(const pkv_shape& s, const void* q, Strides qs, const void* k, Strides ks,
                               const void* v, Strides vs, const float* scale, void* out, float* lse,
                               hipStream_t st) {
    PrefillParams p;
    p.N = s.N;
    p.q = (const bf16_t*)q; p.qs = qs; p.k = (const bf16_t*)k; p.ks = ks; p.v = (const bf16_t*)v; p.vs = vs;
    p.scale = scale; p.out = (bf16_t*)out; p.lse = lse;
    const long long heads = (long long)s.B * s.L * s.H;
    const long long nqb = (s.N + kPfQueries - 1) / kPfQueries;
    const long long nblk = (heads + kXcds - 1) / kXcds * nqb * kXcds;   // whole heads per XCD
    if (nblk > 0x7fffffffll) return hipErrorInvalidValue;
    const long long hx = (heads + kXcds - 1) / kXcds, tail = (kPfTailBlocks + nqb - 1) / nqb;
    p.heads = (int)heads; p.heads_per_xcd = (int)hx;
    p.nqb = fast_div(nqb); p.tail = fast_div(tail < hx ? tail : hx);
    p.by_h = fast_div(s.H); p.by_l = fast_div(s.L); p.by_grp = fast_div(s.H / s.Hkv);
    const dim3 grid((unsigned)nblk);
    if (s.D == 128) hipLaunchKernelGGL(prefill_attn_kernel<128>, grid, dim3(256), 0, st, p);
    else hipLaunchKernelGGL(prefill_attn_kernel<64>, grid, dim3(256), 0, st, p);
    return hipGetLastError();
}

}  // namespace pkv

// Small-tile attention for gfx950: the decode-like case where every request
// has only a few new tokens (GreenCache §2.1-2.2: a cached context followed by
// token-by-token generation still attends over the whole stored KV).
//
// Computes exactly what the prefill path computes (causal scaled-dot-product
// attention of the new tokens over cached prefix plus new tokens, GQA), for
// query tiles of 16 rows (the g query heads of one KV head over 16/g new
// tokens) and key tiles of 32 keys (two pool pages). Such work is bound by
// reading K and V, so each wavefront owns one work item and streams its K and V
// pages through its own LDS ring (direct copies, no barriers), and takes the
// matrix-core operands from there:
//   S^T (32 keys x 16 rows)  = K . Q^T     two 16x16 blocks, MFMA 16x16x32 bf16
//   O^T (D x 16 rows)       += V^T . P^T   D/16 blocks,     MFMA 16x16x32 bf16
// The key rows fed to the first product are permuted so that a lane's score
// accumulators are eight adjacent slots of one page: they are already laid out
// as the P^T operand, and the V^T operand is one LDS read.
// With 8-bit pools (E4M3 codes times one scale per pool) the same fragments are
// copied at half the width and widened to bf16 in registers (exact: every E4M3
// value is a bf16 value); the key scale is folded into the softmax scale and the
// value scale into the final normalisation, so the loop is otherwise unchanged.
#include "gc_internal.h"

namespace gc {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(4))) int32_t* scalar_i32p;

constexpr float kLn2 = 0.69314718055994530942f;

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const bf16x2 p = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, p);
}

// x combined with the value of lane l ^ 16 (max or sum), then with lane l ^ 32
__device__ __forceinline__ float row_max4(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float row_sum4(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Four E4M3 codes (one 32-bit word) as four bf16 values (two 32-bit words).
__device__ __forceinline__ u32x2 widen_e4m3x4(uint32_t w) {
    const bf16x2 lo = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, false);
    const bf16x2 hi = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, true);
    return u32x2{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
}

// Direct global->LDS copies of N KiB (one page): 16 bytes per lane and KiB, from
// base + off[e] + 1024 e to lds + 1024 e + 16 lane (the instruction's offset applies to
// both sides). Inline assembly, so the compiler does not track the copies: every wait
// for them is explicit (wait_copies).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int N>
__device__ __forceinline__ void copy_page(const unsigned char* base, const uint32_t (&off)[N], uint32_t lds) {
    static_assert(N == 1 || N == 2 || N == 4, "page size");
    if constexpr (N == 4)
        asm volatile("s_mov_b32 m0, %5\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %4\n\t"
                     "global_load_lds_dwordx4 %1, %4 offset:1024\n\tglobal_load_lds_dwordx4 %2, %4 offset:2048\n\t"
                     "global_load_lds_dwordx4 %3, %4 offset:3072"
                     :: "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base), "s"(lds) : "memory", "m0");
    else if constexpr (N == 2)
        asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2\n\t"
                     "global_load_lds_dwordx4 %1, %2 offset:1024"
                     :: "v"(off[0]), "v"(off[1]), "s"(base), "s"(lds) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                     :: "v"(off[0]), "s"(base), "s"(lds) : "memory", "m0");
}
#pragma clang diagnostic pop

// Wait until at most N of this wavefront's vector-memory operations are outstanding
// (s_waitcnt: vmcnt in bits 3:0 and 15:14, the other counters at their maxima).
template <int N>
__device__ __forceinline__ void wait_copies() {
    static_assert(N >= 0 && N < 64, "vmcnt field");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
    asm volatile("" ::: "memory");  // no LDS read moves above the wait
}
// Wait for this wavefront's LDS reads; later copies may then overwrite what they read.
__device__ __forceinline__ void wait_lds_reads() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt 0
    asm volatile("" ::: "memory");
}

// What bounds it: HBM, so everything serves the copies.
//   - Whole pages are copied in 1 KiB instructions. Reading the operands straight into
//     registers (16 rows x 64 bytes of K, 8 or 4 bytes per lane of V) took as many
//     address cycles for 8-bit pools as for bf16 ones and held a compute unit to about
//     47 bytes per ns; the copies reach 6.0 TB/s on scattered 2 and 4 KiB pages.
//   - One wavefront per workgroup, a ring of R tiles in LDS. A tile's operands are read
//     into registers at once, so its slot is refilled (tile kt + R) before the products
//     and R tiles stay in flight while a tile is computed.
//   - The exponent offset of a row is its exact running maximum: the heaviest key's
//     weight is then 1, which bf16 holds exactly (error against 64 bits 14 % lower than
//     with the first tile's maximum kept as the offset), and the time is the same.
// Measured against that register form (attention and merge, with the split policy of
// each): 32 requests of 791 MB 145 us (174), of 396 MB of codes 81 us (117); one request
// of 16.8 MB 15.9 us (43.8).
template <int D, bool FP8>
__global__ __launch_bounds__(64, 2) void attention_small_kernel(const AttnArgs a) {
    constexpr int KS = D / 32;                    // k-steps of QK^T
    constexpr int DB = D / 16;                    // 16-row blocks of O^T
    static_assert(kDecM == 16 && kDecN == 32 && kPage == 16, "tile shape");
    constexpr int EB = FP8 ? 1 : 2;               // bytes per pool element
    constexpr int kRow = D * EB;                  // bytes of a key row
    constexpr int kPageBytes = kPage * kRow;
    constexpr int kTileBytes = 4 * kPageBytes;    // K pages 0 and 1, V pages 0 and 1
    constexpr int N = kPageBytes / 1024;          // copies per page
    constexpr int R = 2;                          // tiles in the ring
    constexpr int kCopies = 4 * N;                // per tile
    __shared__ __align__(1024) unsigned char ring[R * kTileBytes];

    const int lane = threadIdx.x & 63;
    const int kvh = (int)(blockIdx.x % (unsigned)a.num_kv_heads);
    const WorkItem it = a.items[blockIdx.x / (unsigned)a.num_kv_heads];
    if (it.r < 0 || it.kt_begin >= it.kt_end) return;

    // (the planner repeats the request's lengths in the item)
    const int r = it.r;
    const int P = it.P;
    const int cu = it.cu;
    const int n = it.n;
    const int L = P + n;
    const int ntok = min(a.tq, n - it.q0);

    const int g4 = lane >> 4;
    const int j = lane & 15;    // query row of the tile: token t, head kvh * g + hl
    const int t = (int)((unsigned)j / (unsigned)a.group);
    const int hl = j - t * a.group;
    const bool row_ok = t < ntok;
    const int lim = P + it.q0 + (row_ok ? t : 0);  // last key this row may see
    const int64_t qrow = (int64_t)(cu + it.q0 + t) * a.num_q_heads + kvh * a.group + hl;

    // Lane group G of the score accumulators holds the keys 8 half(G) .. + 7 of page
    // page(G) of the tile: accumulator v of block b is slot 8 half + 4 b + v. Pages
    // alternate with G over bf16 pools and halves over 8-bit pools, whichever keeps the
    // V reads below free of bank conflicts.
    auto page_of = [](int G) { return FP8 ? G >> 1 : G & 1; };
    auto half_of = [](int G) { return FP8 ? G & 1 : G >> 1; };
    const int key_lane = kPage * page_of(g4) + 8 * half_of(g4);  // this lane's first key of a tile
    // 16-byte chunk c of key row `slot` of page p lies at chunk c ^ swz(p, slot) of the
    // row: the 16 rows that a read takes (one per lane of a group) fall into different banks.
    auto swz = [](int p, int slot) {
        const int half = slot >> 3, G = FP8 ? 2 * p + half : p + 2 * half;
        return kRow == 256 ? slot ^ (4 * p) : kRow == 128 ? ((slot >> 1) & 1) | (G << 1) : G;
    };
    // K^T operand of block b, k-step (pair) s: lane j = 4 G + v reads chunk 4 s + g4 of its row
    uint32_t k_at[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int G = j >> 2, p = page_of(G), slot = 8 * half_of(G) + 4 * b + (j & 3);
        k_at[b] = (uint32_t)(p * kPageBytes + slot * kRow + (g4 ^ swz(p, slot)) * 16);  // ^ 64 s
    }
    // V^T operand of block db: value row 16 db + j, this lane's eight slots (over bf16
    // pools the two halves of a row are swapped in every other group of eight rows)
    const uint32_t v_at = (uint32_t)((2 + page_of(g4)) * kPageBytes + j * kPage * EB +
                                     (FP8 ? 8 * half_of(g4) : 16 * (half_of(g4) ^ (j >> 3))));
    // where each lane of a copy reads (relative to the page and the copy's 1 KiB)
    uint32_t k_src[2][N], v_src[N];
#pragma unroll
    for (int e = 0; e < N; ++e) {
        constexpr int C = kRow / 16;  // chunks per row
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int row = lane / C;
            k_src[p][e] = (uint32_t)(row * kRow + ((lane % C) ^ swz(p, e * (1024 / kRow) + row)) * 16);
        }
        v_src[e] = FP8 ? 16u * lane : (uint32_t)((lane >> 1) * 32 + ((lane & 1) ^ ((lane >> 4) & 1)) * 16);
    }

    const scalar_i32p table = (scalar_i32p)(a.block_tables + (int64_t)r * a.max_blocks);
    const int64_t block_bytes = (int64_t)a.num_kv_heads * kPageBytes;
    const unsigned char* kbase = reinterpret_cast<const unsigned char*>(a.k_pool) + (int64_t)kvh * kPageBytes;
    const unsigned char* vbase = reinterpret_cast<const unsigned char*>(a.v_pool) + (int64_t)kvh * kPageBytes;
    const uint32_t ring_at = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)ring);
    const int kt_end = it.kt_end;

    // Block ids of a tile's two pages (scalar loads, fetched a tile ahead of their use).
    // A page past the table row or the sequence, or with an id outside the pool, is
    // copied from block 0 (its keys are masked, its values zeroed).
    struct Ids {
        int b0, b1;
    };
    auto fetch_ids = [&](int kt) -> Ids {
        return Ids{table[min(kt * 2, a.max_blocks - 1)], table[min(kt * 2 + 1, a.max_blocks - 1)]};
    };
    auto copy_tile = [&](int kt, int slot, const Ids& ids) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int lp = kt * 2 + p, blk = p ? ids.b1 : ids.b0;
            const bool ok = (lp < a.max_blocks) & (lp * kPage < L) & (blk >= 0) & (blk < a.num_blocks);
            const int64_t off = (int64_t)(ok ? blk : 0) * block_bytes;
            const uint32_t at = ring_at + slot * kTileBytes + p * kPageBytes;
            copy_page<N>(kbase + off, k_src[p], at);
            copy_page<N>(vbase + off, v_src, at + 2 * kPageBytes);
        }
    };

    f32x4 o[DB];
    float m_run;  // running maximum of the row (score * scale * log2(e) units)
    float l_run;  // this lane's share of the row sum of the bf16 weights
    const float c = a.scale_log2;
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    bf16x8 qf[KS];

    Ids ids = fetch_ids(it.kt_begin);
#pragma unroll
    for (int i = 0; i < R; ++i) {
        if (it.kt_begin + i < kt_end) copy_tile(it.kt_begin + i, i, ids);
        ids = fetch_ids(it.kt_begin + i + 1);
    }
    // Q^T operand of k-step s: lane holds q[row j][32 s + 8 g4 .. +7]. Over 8-bit
    // pools the head dimension is taken in another order (the sum over d does not
    // depend on it): k-steps 2p and 2p + 1 cover d = 64 p + 16 g4 .. +15 of lane
    // group g4, so one 16-byte read brings a lane's K codes for both steps.
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int d0 = FP8 ? 64 * (s >> 1) + 16 * g4 + 8 * (s & 1) : 32 * s + 8 * g4;
        qf[s] = row_ok ? *reinterpret_cast<const bf16x8*>(a.q + qrow * D + d0)
                       : __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
    }
    // arrived before the loop: a wait in the loop would wait for the copies too
#pragma unroll
    for (int s = 0; s < KS; ++s) asm volatile("" : "+v"(qf[s]));
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    m_run = -INFINITY;
    l_run = 0.f;
    int slot = 0;
    for (int kt = it.kt_begin; kt < kt_end; ++kt) {
        // tile kt has landed when only the next tile's copies are outstanding
        static_assert(R == 2, "the wait");
        if (kt + 1 < kt_end) wait_copies<kCopies>();
        else wait_copies<0>();

        const unsigned char* tile = ring + slot * kTileBytes;
        u32x4 kw[2][FP8 ? KS / 2 : KS];
        u32x4 vw[DB];  // 8-bit pools: two words each
#pragma unroll
        for (int s = 0; s < (FP8 ? KS / 2 : KS); ++s)
#pragma unroll
            for (int b = 0; b < 2; ++b) kw[b][s] = *reinterpret_cast<const u32x4*>(tile + (k_at[b] ^ (64u * s)));
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const unsigned char* at = tile + v_at + db * 16 * kPage * EB;
            if constexpr (FP8) {
                const u32x2 w = *reinterpret_cast<const u32x2*>(at);
                vw[db][0] = w[0];
                vw[db][1] = w[1];
            } else {
                vw[db] = *reinterpret_cast<const u32x4*>(at);
            }
        }
        wait_lds_reads();
        if (kt + R < kt_end) {
            copy_tile(kt + R, slot, ids);
            ids = fetch_ids(kt + R + 1);
        }
        slot = slot + 1 == R ? 0 : slot + 1;

        f32x4 s[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                bf16x8 kf;
                if constexpr (FP8) {
                    const u32x4 w = kw[b][ks >> 1];
                    const u32x2 x = widen_e4m3x4(w[2 * (ks & 1)]), y = widen_e4m3x4(w[2 * (ks & 1) + 1]);
                    kf = __builtin_bit_cast(bf16x8, u32x4{x[0], x[1], y[0], y[1]});
                } else {
                    kf = __builtin_bit_cast(bf16x8, kw[b][ks]);
                }
                s[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[ks], s[b], 0, 0, 0);
            }
        // s[b][v] is the score of tile key key_lane + 4 b + v
        const int key0 = kt * kDecN;
        if (key0 + kDecN - 1 > P + it.q0) {
            const int rel = lim - key0 - key_lane;
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) s[b][v] = (4 * b + v > rel) ? -INFINITY : s[b][v];
            // values past the sequence end become 0 (weight 0 times a stale value)
            const int bad = L - key0 - key_lane;  // first of this lane's slots at or past the end
            if (bad < 8) {
                u32x4 keep;
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    keep[x] = (2 * x < bad ? 0xFFFFu : 0u) | (2 * x + 1 < bad ? 0xFFFF0000u : 0u);
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    if constexpr (FP8) {
#pragma unroll
                        for (int x = 0; x < 2; ++x)
                            vw[db][x] &= (keep[2 * x] & 0xFFu) | ((keep[2 * x] >> 16) & 0xFF00u) |
                                         ((keep[2 * x + 1] & 0xFFu) << 16) | (keep[2 * x + 1] & 0xFF000000u);
                    } else {
                        vw[db] &= keep;
                    }
                }
            }
        }
        const float mx = fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])),
                               fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3])));
        const float m_new = fmaxf(m_run, row_max4(mx) * c);
        if (__any(m_new > m_run)) {
            // rows that have seen no visible key yet keep o = l = 0 with any finite alpha
            const float alpha = m_new == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db) o[db] *= alpha;
        }
        const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
        u32x4 pw;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(s[x >> 1][2 * (x & 1)], c, -m_use));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(s[x >> 1][2 * (x & 1) + 1], c, -m_use));
            const bf16x2 pair = {(__bf16)p0, (__bf16)p1};
            l_run = __builtin_amdgcn_fdot2_f32_bf16(pair, ones, l_run, false);
            pw[x] = __builtin_bit_cast(uint32_t, pair);
        }
        const bf16x8 pf = __builtin_bit_cast(bf16x8, pw);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            bf16x8 vf;
            if constexpr (FP8) {
                const u32x2 x = widen_e4m3x4(vw[db][0]), y = widen_e4m3x4(vw[db][1]);
                vf = __builtin_bit_cast(bf16x8, u32x4{x[0], x[1], y[0], y[1]});
            } else {
                vf = __builtin_bit_cast(bf16x8, vw[db]);
            }
            o[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf, o[db], 0, 0, 0);
        }
    }

    const float l_tot = row_sum4(l_run);
    const float inv = l_tot > 0.f ? a.v_scale / l_tot : 0.f;  // v_scale is 1 for bf16 pools
    // (a split item passes a NaN sum on to the merge)
    const float lse_v = l_tot > 0.f ? (m_run + log2f(l_tot)) * kLn2 : (it.part >= 0 && l_tot != l_tot ? l_tot : -INFINITY);
    // o[db][v] is element d = 16 db + 4 g4 + v of row j
    if (it.part < 0) {
        if (row_ok) {
            uint16_t* op = a.out + qrow * D + 4 * g4;
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                u32x2 w;
                w[0] = pack_bf16x2(o[db][0] * inv, o[db][1] * inv);
                w[1] = pack_bf16x2(o[db][2] * inv, o[db][3] * inv);
                *reinterpret_cast<u32x2*>(op + 16 * db) = w;
            }
            if (a.lse != nullptr && g4 == 0) a.lse[qrow] = lse_v;
        }
    } else {
        const int64_t prow = ((int64_t)it.part * a.num_kv_heads + kvh) * kDecM + j;
        if (row_ok) {  // (the merge reads no other rows)
            float* po = a.part_o + prow * D + 4 * g4;
#pragma unroll
            for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4*>(po + 16 * db) = o[db] * inv;
            if (g4 == 0) a.part_lse[prow] = lse_v;
        }
    }
}

}  // namespace

hipError_t launch_attention_small(const AttnArgs& a, int head_dim, int64_t num_items, bool fp8,
                                  hipStream_t s) {
    const dim3 grid((unsigned)(num_items * a.num_kv_heads));
    if (fp8) {
        if (head_dim == 128)
            attention_small_kernel<128, true><<<grid, 64, 0, s>>>(a);
        else
            attention_small_kernel<64, true><<<grid, 64, 0, s>>>(a);
    } else {
        if (head_dim == 128)
            attention_small_kernel<128, false><<<grid, 64, 0, s>>>(a);
        else
            attention_small_kernel<64, false><<<grid, 64, 0, s>>>(a);
    }
    return hipGetLastError();
}

}  // namespace gc

// Prefix-cached prefill attention and split-KV merge for gfx950 (CDNA4).
//
// Computes, for every new token of every request and every query head, causal
// scaled-dot-product attention over the request's cached prefix keys plus the
// new keys up to and including the token itself (GreenCache §2.2, Fig. 1a:
// cached and new KV processed together; §2.1 prefill). Keys are gathered from
// the paged pool through the block table.
//
// Work decomposition. A workgroup (4 wavefronts, or 8 for the wide tiling) owns
// one work item: 128 (256) query rows = the g query heads of one KV head stacked
// over consecutive new tokens of one request, against a range of 64-key tiles.
// Each wavefront owns 32 of the rows, as two blocks of 16. Per key tile:
//   S^T (64 keys x 32 rows)  = K_tile . Q^T        4 x 2 blocks of 16x16, MFMA 16x16x32 bf16
//   online softmax on S^T in registers               fp32, base-2 exponent
//   O^T (D x 32 rows)       += V_tile^T . P^T       D/16 x 2 blocks, MFMA 16x16x32 bf16
// Every K and V fragment read from LDS serves both row blocks. Computing the transposed
// products puts the scores of one query row in four lanes (l, l + 16, l + 32, l + 48), so
// row maxima and sums are in-lane plus two exchanges, and the QK^T accumulators double as
// the PV operand once the key rows fed to the first product are permuted.
// The 16x16x32 products are taken because these tiles run against the card's power limit
// on real data (zero inputs: 370 us instead of 503 for the 32k reuse batch, at the same
// instructions): a register loop of products on normal data sustains 2070 TFLOP/s with
// 16x16x32 and 1800 with 32x32x16 (2460 with either on zeros). Kernel against kernel, 32k
// reuse 483 -> 458 us, mixed 70B batch 2206 -> 2107, one request of 512 tokens on 8000
// 137 -> 127.
// K and V tiles are staged through LDS, double buffered: the next tile's
// global loads are in flight while the current tile is computed. Value pages
// are stored transposed in the pool ([D][16]), so both LDS tiles are read with
// 16-byte loads; XOR swizzles keep those reads free of bank conflicts.
// The tile copies go straight from global memory to LDS; they are issued as
// inline assembly with explicit waits, so the compiler's own LDS waits count
// only LDS reads and can keep several fragment reads in flight per MFMA
// (scheduling fences hold that order).
// 8-bit pools (E4M3 codes times one scale per pool): the next tile's codes are
// loaded into registers instead, widened to bf16 (exact) and written to the same
// LDS layout after the current tile's products, so the compute loop is shared;
// the key scale is folded into the softmax scale, the value scale into the
// final normalisation.
#pragma once
#include "gc_internal.h"

namespace gc {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr float kLn2 = 0.69314718055994530942f;

// Position of 16-byte chunk `chunk` inside key row `row` of a tile in LDS. A fragment
// read takes, per 16 lanes, the rows 16 p + 8 h + 4 b + v (p, h = 0, 1, v = 0 .. 3) of one
// block b at one chunk: the swizzle sends them to different banks.
template <int D>
__device__ __forceinline__ int swz_k(int chunk, int row) {
    const int p = (row >> 4) & 1, h = (row >> 3) & 1;
    if constexpr (D == 128) return chunk ^ (row & 15) ^ (4 * p);             // 256-byte rows
    else return chunk ^ (((row >> 1) & 1) | (2 * p) | (4 * h));               // 128-byte rows
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    __bf16 a = (__bf16)lo;
    __bf16 b = (__bf16)hi;
    return (uint32_t)__builtin_bit_cast(uint16_t, a) | ((uint32_t)__builtin_bit_cast(uint16_t, b) << 16);
}


// A direct global->LDS copy of 16 bytes per lane, from base + off (a wave-uniform base in
// scalar registers, a 32-bit lane offset): lane i's bytes land at lds + 16 i (a wave-uniform
// LDS byte address). Issued as inline assembly so the compiler does not track it: every
// wait for these copies is explicit (wait_vmem). The compiler emits no other use of m0 in
// these kernels; the clobber keeps it that way. The four copies of a tile and wavefront cost
// no vector instruction besides themselves, where 64-bit lane addresses took an addition
// each between the QK^T products (mixed 70B batch 2223 -> 2206 us with the offset and the
// first-tile test kept out of the tile loop, 32k reuse 489 -> 483, 8B chat 132.7 -> 128.6).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16(const unsigned char* base, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(off), "s"(base), "s"(lds) : "memory", "m0");
}
#pragma clang diagnostic pop

__device__ __forceinline__ uint32_t lds_address(const unsigned char* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)p;
}

// Wait until at most N vector-memory operations of this wave are outstanding
// (s_waitcnt immediate: vmcnt in bits 3:0, expcnt 6:4 and lgkmcnt 11:8 left at
// their maxima). A real wait instruction, so the compiler also knows it.
template <int N>
__device__ __forceinline__ void wait_vmem() {
    static_assert(N >= 0 && N < 16, "vmcnt field");
    __builtin_amdgcn_s_waitcnt(0x0F70 | N);
    asm volatile("" ::: "memory");  // no LDS access moves above the wait
}

// The lanes of one wavefront exchange data through LDS: a release and an acquire at
// wavefront scope between the writes and the reads, so the compiler neither reuses
// values a lane loaded earlier nor moves the reads across the writes of other lanes
// (the hardware runs one wavefront's LDS operations in order).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sixteen E4M3 codes (four words) as sixteen bf16 values (eight words).
__device__ __forceinline__ void widen_e4m3x16(const u32x4 c, u32x4& lo, u32x4& hi) {
    uint32_t w[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        w[2 * i] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c[i], 1.0f, false));
        w[2 * i + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c[i], 1.0f, true));
    }
    lo = u32x4{w[0], w[1], w[2], w[3]};
    hi = u32x4{w[4], w[5], w[6], w[7]};
}

// One work item (a workgroup of WAVES wavefronts): the item of launch index bid (blockIdx.x
// in the regular launch), i.e. work item bid / Hkv for KV head bid % Hkv.
template <int D, int WAVES, bool FP8, int WGS = 8 / WAVES>
__device__ __forceinline__ void attention_body(const AttnArgs& a, const unsigned bid) {
    constexpr int kBlockRows = WAVES * kRowsPerWave;  // query rows of a work item
    constexpr int KS = D / 32;                      // k-steps of QK^T
    constexpr int DB = D / 16;                      // 16-row blocks of O^T
    constexpr int RB = kRowsPerWave / 16;           // 16-row query blocks per wavefront
    static_assert(RB == 2, "row blocks");
    constexpr int kPageBytes = kPage * D * 2;       // one (block, KV head) page of K or V
    constexpr int kTileBytes = kBlockN * D * 2;     // four pages
    constexpr int kKbPerPage = kPageBytes / 1024;   // 1 KiB pieces per page
    constexpr int NI = kTileBytes / (WAVES * 1024);  // direct loads per wave per tensor per tile
    constexpr int kTileLog2Thresh = 8;              // rescale only when the max grows by > 2^8

    // K tile: [64 keys][D], row-major, 16-byte chunks XOR-swizzled by row.
    // V tile: 4 pages of [D][16 keys], the two 16-byte halves of a row swapped on odd 8-row groups.
    // Two separate buffers of each (distinct objects, so the compiler can tell that
    // reads of one do not wait for the asynchronous loads into the other).
    __shared__ __align__(16) unsigned char k_lds0[kTileBytes];
    __shared__ __align__(16) unsigned char v_lds0[kTileBytes];
    __shared__ __align__(16) unsigned char k_lds1[kTileBytes];
    __shared__ __align__(16) unsigned char v_lds1[kTileBytes];

    // (opaque to the compiler, so that the lane constants derived from it are computed per
    // work item: hoisted out of the resident launch's item loop they would be held, or
    // spilled, across the tile loop)
    int tid_opaque = (int)threadIdx.x;
    asm volatile("" : "+v"(tid_opaque));
    const int tid = tid_opaque;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // One of a SIMD's two wavefronts is preferred throughout (the older half of a wide
    // workgroup; over d = 128 every other round of a workgroup per compute unit, which of the
    // two the host says: two 128-row workgroups share a unit): the preferred one's products
    // run while the other computes weights and the other way round, where equal ones take turns
    // product by product and then wait for the vector unit together. Mixed 70B batch 2107 ->
    // 2052 us, 70B chat 434 -> 422, 8B chat 125.7 -> 121.5, over 8-bit pools 173.6 -> 154.8; at
    // d = 64, where three 128-row workgroups share a compute unit, 2 % slower, so not there.
    // (Before the item's loads: between them and their uses the branch cost 1-3 % of short launches.)
    if (WAVES == kWideWaves ? wave < WAVES / 2 : D == 128 && (bid / a.prefer_span & 1) == a.prefer_odd)
        __builtin_amdgcn_s_setprio(2);
    const int g4 = lane >> 4;
    const int j16 = lane & 15;
    const int kvh = (int)(bid % (unsigned)a.num_kv_heads);
    const WorkItem it = a.items[bid / (unsigned)a.num_kv_heads];
    // all eight fields in one load (else the fields the test below needs are loaded
    // first and the rest after it, a second dependent round trip)
    asm volatile("" ::"s"(it.r), "s"(it.q0), "s"(it.kt_begin), "s"(it.kt_end), "s"(it.part), "s"(it.P),
                 "s"(it.cu), "s"(it.n));
    if (it.r < 0 || it.kt_begin >= it.kt_end) return;
    // (the planner repeats the request's lengths in the item: one load for all of them)
    const int r = it.r;
    const int P = it.P;
    const int cu = it.cu;
    const int n = it.n;
    const int L = P + n;
    const int ntok = min(a.tq, n - it.q0);

    // this lane's query rows, 16 rb + j16 of the wavefront's 32: token t of the tile, query
    // head kvh * g + hl
    bool row_ok[RB];
    int lim[RB];  // last key the row may see
    int64_t qrow[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int m = wave * kRowsPerWave + 16 * rb + j16;
        const int t = (int)((unsigned)m / (unsigned)a.group);
        row_ok[rb] = t < ntok;
        lim[rb] = P + it.q0 + (row_ok[rb] ? t : 0);
        qrow[rb] = (int64_t)(cu + it.q0 + t) * a.num_q_heads + kvh * a.group + (m - t * a.group);
    }

    // block-table entries of the first key tile, loaded before Q: loads return in
    // order, so the first tile's copies then wait for these entries only and go out
    // while Q is still in flight (entry p in lanes with lane % 4 == p; clamped into
    // the row, checked at use)
    int ids = a.block_tables[(int64_t)r * a.max_blocks + min(it.kt_begin * 4 + (lane & 3), a.max_blocks - 1)];

    // Q^T operands: lane holds q[row 16 rb + j16][32 ks + 8 g4 .. +7]
    bf16x8 qf[RB][KS];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        if (row_ok[rb]) {
            const uint16_t* qp = a.q + qrow[rb] * D + g4 * 8;
#pragma unroll
            for (int k = 0; k < KS; ++k) qf[rb][k] = *reinterpret_cast<const bf16x8*>(qp + 32 * k);
        } else {
#pragma unroll
            for (int k = 0; k < KS; ++k) qf[rb][k] = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
        }
    }

    // Direct global->LDS loads: instruction e of a wave moves 1 KiB piece 4e + wave of
    // a tile tensor, i.e. piece `sub` of page `page_of(e)`; lane i lands at byte 16 i.
    const int sub = wave % kKbPerPage;
    static_assert(WAVES % kKbPerPage == 0, "piece layout");
    auto page_of = [&](int e) -> int { return (WAVES / kKbPerPage) * e + (wave & (WAVES - 1)) / kKbPerPage; };
    const int k_row = sub * (1024 / (2 * D)) + lane / (D / 8);         // key slot in the page
    // source chunk of the row, by the parity of the page in the tile (that of e where the
    // pieces of one instruction cover one page, else the wavefront's own)
    auto parity = [&](int e) { return (WAVES / kKbPerPage) % 2 == 1 ? e & 1 : (wave / kKbPerPage) & 1; };
    auto k_chunk = [&](int e) -> uint32_t { return swz_k<D>(lane % (D / 8), 16 * parity(e) + k_row) * 16; };
    uint32_t k_src[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) k_src[e] = k_row * (2 * D) + k_chunk(e);
    const int v_d = sub * 32 + (lane >> 1);                            // value row (d) in the page
    const int v_half = (lane & 1) ^ ((v_d >> 3) & 1);                  // logical half held by the lane
    const uint32_t v_src = v_d * 32 + v_half * 16;
    const int32_t* table = a.block_tables + (int64_t)r * a.max_blocks;
    const int64_t head_off = (int64_t)kvh * kPageBytes;
    const int64_t block_stride = (int64_t)a.num_kv_heads * kPageBytes;
    // raw table entries of tile kt (indices clamped into the row; checked at use)
    // (a vector load: lane p of every 4 holds entry p; it completes with the tile loads,
    // and no scalar load is left in flight to force full LDS waits in the compute phase)
    auto fetch_ids = [&](int kt, int& ids) {
        ids = table[(uint32_t)min(kt * 4 + (lane & 3), a.max_blocks - 1)];
    };
    // Copies of piece e of tile kt (one page of K and of V for this wave). A page past the
    // table, past the sequence or with a block id outside the pool is copied from block 0
    // instead (its keys are masked and its values zeroed after the copy), so the copy needs
    // no branch and can be issued between the products of the tile before.
    // (blk: the raw table entry of the page, read from the lanes of `ids` beforehand)
    // (the destination: buffer 0 or 1 of the tiles)
    const uint32_t lds_piece = __builtin_amdgcn_readfirstlane(sub * 1024);
    const unsigned char* kpool = reinterpret_cast<const unsigned char*>(a.k_pool);
    const unsigned char* vpool = reinterpret_cast<const unsigned char*>(a.v_pool);
    auto issue_page = [&](int buf, int kt, const int blk, int e) {
        const int pg = page_of(e);
        const int lp = kt * 4 + pg;
        const bool ok = lp < a.max_blocks && lp * kPage < L && blk >= 0 && blk < a.num_blocks;
        const int64_t off = (int64_t)(ok ? blk : 0) * block_stride + head_off;
        const uint32_t at = pg * kPageBytes + lds_piece;
        dma16(kpool + off, k_src[e & 1], lds_address(buf ? k_lds1 : k_lds0) + at);
        dma16(vpool + off, v_src, lds_address(buf ? v_lds1 : v_lds0) + at);
    };
    auto page_ids = [&](const int ids, int (&blk)[NI]) {
#pragma unroll
        for (int e = 0; e < NI; ++e) blk[e] = __builtin_amdgcn_readlane(ids, page_of(e));
    };
    auto issue_tile = [&](int buf, int kt, const int ids) {
        int blk[NI];
        page_ids(ids, blk);
#pragma unroll
        for (int e = 0; e < NI; ++e) issue_page(buf, kt, blk[e], e);
    };
    // After this wave's loads of tile kt landed: value slots at or past the sequence
    // end become 0 (masked keys get weight 0, and 0 * NaN would poison the product).
    auto zero_tail = [&](unsigned char* vdst, int kt) {
        const int first_bad = L - kt * kBlockN;  // tile-relative key index
        if (first_bad >= kBlockN) return;
#pragma unroll
        for (int e = 0; e < NI; ++e) {
            const int pg = page_of(e);
            const int key0 = pg * kPage + v_half * 8;
            uint16_t* dst = reinterpret_cast<uint16_t*>(vdst + pg * kPageBytes + sub * 1024 + lane * 16);
#pragma unroll
            for (int x = 0; x < 8; ++x)
                if (key0 + x >= first_bad) dst[x] = 0;
        }
    };

    f32x4 o[RB][DB];
    float m_run[RB];   // exponent offset (score * scale * log2(e) units)
    float neg_off[RB]; // -m_run, 0 while the row has none
    bool need_max;     // some row has no offset yet, or the exact pass
    float l_run[RB];   // this lane's share of the row sum of the bf16 weights
    // Exponent offset: a row takes the maximum of its first tile with a visible key and
    // keeps it; the weights of later tiles are exp2 of up to ~100 and fp32 holds their
    // products and sums. If some row's sum leaves that range (a score jump of more than
    // ~100 in log2 units), the work item is run again with the exact running maximum of
    // every tile (rescaled lazily, when it grows by more than 2^8). The final
    // normalisation uses the same offset, so the result does not depend on it.
    bool exact = false;
    const float c = a.scale_log2;
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};

    // Lane group G of the score accumulators holds keys 16 (G % 2) + 8 (G / 2) .. + 7 of
    // each 32-key half of a tile: accumulator v of block b is the (4 b + v)-th of them. The
    // K rows are fed to the products in that order, so that the accumulators are already
    // the P^T operand and the V^T operand is eight adjacent slots of one page.
    const int key_lane = kPage * (g4 & 1) + 8 * (g4 >> 1);
    // K^T operand of (half hb, block b, k-step ks): lane j16 = 4 G + v reads chunk
    // 4 ks + g4 of its row; block 1's rows are 4 further (for d = 128 with the chunk
    // swizzled by 4 more), a half's 32 further.
    constexpr int kRow = 2 * D;
    uint32_t k_at[KS];
    {
        const int r0 = kPage * ((j16 >> 2) & 1) + 8 * (j16 >> 3) + (j16 & 3);
#pragma unroll
        for (int x = 0; x < KS; ++x) k_at[x] = (uint32_t)(r0 * kRow + swz_k<D>(g4, r0) * 16) ^ (64u * x);
    }
    // V^T operand of (half hb, block db): value row 16 db + j16, this lane's eight slots
    const uint32_t v_at = (uint32_t)((g4 & 1) * kPageBytes + j16 * 32 + 16 * ((g4 >> 1) ^ (j16 >> 3)));

    // LDS fragment reads kept in flight ahead of their products (three and five within 1 %,
    // eight 1-10 % slower; two for three 128-row workgroups per compute unit over 8-bit pools, whose
    // 168 registers then spill 12 instead of 16: 1 % faster)
    constexpr int kAhead = FP8 && WGS * WAVES == 12 ? 2 : 4;
    // hook(i) runs after the products of the i-th K fragment are issued (the next tile's copies go there)
    auto compute_tile = [&](const unsigned char* kb, const unsigned char* vb, int kt, auto&& hook) {
        // S^T = K_tile . Q^T: fragment i is (half i / 2 KS, k-step, block i % 2), used for
        // both row blocks. Every group below is fenced so the fragment reads stay kAhead
        // fragments ahead.
        constexpr int NK = 4 * KS;
        bf16x8 kf[NK];
        auto kread = [&](int i) {
            const int hb = i / (2 * KS), ks = (i >> 1) % KS, b = i & 1;
            const int x = D == 128 ? ks ^ b : ks;
            kf[i] = *reinterpret_cast<const bf16x8*>(kb + (32 * hb + 4 * b) * kRow + k_at[x]);
        };
        f32x4 s[RB][2][2];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int hb = 0; hb < 2; ++hb)
#pragma unroll
                for (int b = 0; b < 2; ++b) s[rb][hb][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < kAhead; ++i) kread(i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NK; ++i) {
            const int hb = i / (2 * KS), ks = (i >> 1) % KS, b = i & 1;
            if (i + kAhead < NK) kread(i + kAhead);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                s[rb][hb][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[i], qf[rb][ks], s[rb][hb][b], 0, 0, 0);
            hook(i);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the first V fragments go out now; they land during the softmax
        bf16x8 vf[2 * DB];
        auto vread = [&](int i) {
            vf[i] = *reinterpret_cast<const bf16x8*>(vb + (i / DB) * 2 * kPageBytes + (i % DB) * 512 + v_at);
        };
#pragma unroll
        for (int i = 0; i < kAhead; ++i) vread(i);
        __builtin_amdgcn_sched_barrier(0);

        // s[rb][hb][b][v] is the score of row 16 rb + j16 and tile key 32 hb + key_lane + 4 b + v
        const int key0 = kt * kBlockN;
        if (key0 + kBlockN - 1 > P + it.q0) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const int rel = lim[rb] - key0 - key_lane;
#pragma unroll
                for (int hb = 0; hb < 2; ++hb)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            s[rb][hb][b][v] = (32 * hb + 4 * b + v > rel) ? -INFINITY : s[rb][hb][b][v];
            }
        }
        // row maximum: NaN-propagating maxima need no operand canonicalisation and
        // fold three operands per instruction
        if (need_max) {
            need_max = exact;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                float mx = s[rb][0][0][0];
#pragma unroll
                for (int e = 1; e < 16; ++e)
                    mx = __builtin_elementwise_maximum(mx, s[rb][e >> 3][(e >> 2) & 1][e & 3]);
                {
                    const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
                    mx = __builtin_elementwise_maximum(__uint_as_float(x[0]), __uint_as_float(x[1]));
                    const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
                    mx = __builtin_elementwise_maximum(__uint_as_float(y[0]), __uint_as_float(y[1]));
                }
                const float m_tile = mx * c;
                if (__any(m_tile > m_run[rb] + kTileLog2Thresh)) {
                    const float m_new = fmaxf(m_run[rb], m_tile);
                    // rows that have seen no visible key yet (all -inf; possible in a key chunk
                    // that starts past them) hold o = l = 0: any finite alpha keeps them so
                    const float alpha = m_new == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run[rb] - m_new);
                    m_run[rb] = m_new;
                    l_run[rb] *= alpha;
#pragma unroll
                    for (int db = 0; db < DB; ++db) o[rb][db] *= alpha;
                }
                need_max |= __any(m_run[rb] == -INFINITY);
                neg_off[rb] = m_run[rb] == -INFINITY ? 0.f : -m_run[rb];
            }
        }
        __builtin_amdgcn_sched_barrier(0);

        // O^T += V^T . P^T
        bf16x8 pf[RB][2];
        // pair q of a half's eight weights of a row, as bf16, and its part of the row sum
        auto w_pair = [&](int rb, int hb, int q) {
            const float x0 = s[rb][hb][q >> 1][2 * (q & 1)], x1 = s[rb][hb][q >> 1][2 * (q & 1) + 1];
            const bf16x2 pq = {(__bf16)__builtin_amdgcn_exp2f(fmaf(x0, c, neg_off[rb])),
                               (__bf16)__builtin_amdgcn_exp2f(fmaf(x1, c, neg_off[rb]))};
            pf[rb][hb][2 * q] = pq[0];
            pf[rb][hb][2 * q + 1] = pq[1];
            l_run[rb] = __builtin_amdgcn_fdot2_f32_bf16(pq, ones, l_run[rb], false);
            // keep the sums here, beside the products (not sunk to the end of the tile)
            asm volatile("" : "+v"(l_run[rb]));
        };
        // The weights are computed in blocks, not between single products: a wavefront's
        // vector instructions and its own 16-cycle products hardly overlap (about one per
        // product does), those of the SIMD's other wavefront do. All of a tile's weights
        // first on the 8-wavefront tiles; on the 4-wavefront ones the first half's, then a
        // quarter of the second half's after every quarter of the first half's products
        // (a pair after every fragment: 2 % slower on wide tiles, 10 % on the 8B chat batch).
        constexpr bool kAllFirst = WAVES == kWideWaves;
#pragma unroll
        for (int hb = 0; hb < (kAllFirst ? 2 : 1); ++hb)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) w_pair(rb, hb, q);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2 * DB; ++i) {
            const int hb = i / DB, db = i % DB;
            if (i + kAhead < 2 * DB) vread(i + kAhead);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                o[rb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[i], pf[rb][hb], o[rb][db], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (!kAllFirst && hb == 0 && db % (DB / 4) == DB / 4 - 1) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) w_pair(rb, 1, db / (DB / 4));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    // 8-bit pools: 16-byte chunks of codes. Chunk c of the K tile is key row
    // c / (D/16), codes 16 (c % (D/16)) ..; chunk c of the V tile is value row c % D
    // of page c / D (16 keys). Lane chunk e is c = 64 (WAVES e + wave) + lane, so a
    // wave's chunks of one e lie in one page.
    constexpr int kChunks = 4 * D;                                   // per tensor and tile
    constexpr int NC = (kChunks + WAVES * 64 - 1) / (WAVES * 64);   // per lane
    const int64_t page_codes = (int64_t)kPage * D;                   // bytes of an 8-bit page
    const int64_t block_codes = (int64_t)a.num_kv_heads * page_codes;
    u32x4 kc8[NC], vc8[NC];
    auto load8 = [&](int kt, const int ids) {
#pragma unroll
        for (int e = 0; e < NC; ++e) {
            const int c0 = 64 * (WAVES * e + wave);  // the wave's first chunk
            const int c = c0 + lane;
            if (c0 < kChunks) {
                const int kpg = (c0 / (D / 16)) / kPage;
                const int vpg = c0 / D;
                int kb = __builtin_amdgcn_readlane(ids, kpg), vb = __builtin_amdgcn_readlane(ids, vpg);
                // pages past the table, past the sequence or with a bad id read block 0
                // (their keys are masked and their values zeroed below)
                const bool kok = kt * 4 + kpg < a.max_blocks && (kt * 4 + kpg) * kPage < L &&
                                 kb >= 0 && kb < a.num_blocks;
                const bool vok = kt * 4 + vpg < a.max_blocks && (kt * 4 + vpg) * kPage < L &&
                                 vb >= 0 && vb < a.num_blocks;
                kb = kok ? kb : 0;
                vb = vok ? vb : 0;
                const uint8_t* kp = reinterpret_cast<const uint8_t*>(a.k_pool) + kb * block_codes +
                                    kvh * page_codes + (c / (D / 16)) % kPage * D + (c % (D / 16)) * 16;
                const uint8_t* vp = reinterpret_cast<const uint8_t*>(a.v_pool) + vb * block_codes +
                                    kvh * page_codes + (c % D) * kPage;
                kc8[e] = *reinterpret_cast<const u32x4*>(kp);
                vc8[e] = *reinterpret_cast<const u32x4*>(vp);
            }
        }
    };
    auto store8 = [&](unsigned char* kdst, unsigned char* vdst, int kt) {
        const int first_bad = L - kt * kBlockN;  // tile-relative key index
#pragma unroll
        for (int e = 0; e < NC; ++e) {
            const int c = 64 * (WAVES * e + wave) + lane;
            if (c < kChunks) {
                u32x4 lo, hi;
                widen_e4m3x16(kc8[e], lo, hi);
                const int kr = c / (D / 16), c8 = c % (D / 16);
                *reinterpret_cast<u32x4*>(kdst + kr * (2 * D) + swz_k<D>(2 * c8, kr) * 16) = lo;
                *reinterpret_cast<u32x4*>(kdst + kr * (2 * D) + swz_k<D>(2 * c8 + 1, kr) * 16) = hi;
                widen_e4m3x16(vc8[e], lo, hi);
                const int pg = c / D, d = c % D;
                const int key0 = pg * kPage;
                if (key0 + kPage > first_bad) {
#pragma unroll
                    for (int x = 0; x < 8; ++x) {
                        const uint32_t keep = (key0 + x < first_bad ? 0xFFFFu : 0u);
                        const uint32_t keep8 = (key0 + 8 + x < first_bad ? 0xFFFFu : 0u);
                        if (x % 2 == 0) {
                            lo[x / 2] &= keep | 0xFFFF0000u;
                            hi[x / 2] &= keep8 | 0xFFFF0000u;
                        } else {
                            lo[x / 2] &= (keep << 16) | 0xFFFFu;
                            hi[x / 2] &= (keep8 << 16) | 0xFFFFu;
                        }
                    }
                }
                unsigned char* vrow = vdst + pg * kPageBytes + d * 32;
                const int sw = (d >> 3) & 1;
                *reinterpret_cast<u32x4*>(vrow + sw * 16) = lo;
                *reinterpret_cast<u32x4*>(vrow + (sw ^ 1) * 16) = hi;
            }
        }
    };

    // One pipeline step: start the next tile's loads into the other buffers, compute
    // this tile, make the next tile visible.
    // (ids: block-table entries of the next tile to copy, entry p in lanes with lane % 4 == p)
    int kt = it.kt_begin;
    auto step = [&](const int cur) {  // (cur: the buffer that holds tile kt)
        unsigned char* const kc = cur ? k_lds1 : k_lds0;
        unsigned char* const vc = cur ? v_lds1 : v_lds0;
        unsigned char* const kn = cur ? k_lds0 : k_lds1;
        unsigned char* const vn = cur ? v_lds0 : v_lds1;
        const bool more = kt + 1 < it.kt_end;
        // the next tile's block ids, read before any copy of this step is in flight (the
        // compiler waits for every outstanding load before reading `ids`)
        int nb[NI];
        page_ids(ids, nb);
        if (more) {
            if constexpr (FP8) {
                load8(kt + 1, ids);
                if (kt + 2 < it.kt_end) fetch_ids(kt + 2, ids);
            }
        }
        // bf16 pools: the next tile's copies are issued between the first products of
        // this one (piece e after those of K fragment 3e + 2), then the table
        // entries of the tile after
        static_assert(3 * NI < 4 * KS, "copies fit between the QK^T products");
        constexpr int kCopyAt = 2;
        compute_tile(kc, vc, kt, [&](int i) {
            if constexpr (!FP8) {
                if (i % 3 == kCopyAt && i / 3 < NI) {
                    if (more) issue_page(1 - cur, kt + 1, nb[i / 3], i / 3);
                } else if (i == 3 * NI) {
                    if (kt + 2 < it.kt_end) fetch_ids(kt + 2, ids);
                }
            }
        });
        if (more) {
            if constexpr (FP8) {
                store8(kn, vn, kt + 1);
            } else {
                wait_vmem<0>();
                zero_tail(vn, kt + 1);
            }
        }
        __syncthreads();
    };

    for (;;) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
        for (int db = 0; db < DB; ++db) o[rb][db] = f32x4{0.f, 0.f, 0.f, 0.f};
        m_run[rb] = -INFINITY;
        neg_off[rb] = 0.f;
        l_run[rb] = 0.f;
    }
    need_max = true;
    kt = it.kt_begin;
    if (exact) fetch_ids(kt, ids);  // the first pass has them from the start
    if constexpr (FP8) {
        load8(kt, ids);
        if (kt + 1 < it.kt_end) fetch_ids(kt + 1, ids);
        store8(k_lds0, v_lds0, kt);
    } else {
        issue_tile(0, kt, ids);
        if (kt + 1 < it.kt_end) fetch_ids(kt + 1, ids);
        wait_vmem<0>();
        zero_tail(v_lds0, kt);
    }
    __syncthreads();
    while (true) {
        step(0);
        if (++kt >= it.kt_end) break;
        step(1);
        if (++kt >= it.kt_end) break;
    }
    if (exact || !__syncthreads_or(!(l_run[0] <= 0x1p100f) || !(l_run[1] <= 0x1p100f))) break;
    exact = true;
    }

    float inv[RB], lse_v[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        float l = l_run[rb];
        const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(l), __float_as_uint(l), false, false);
        l = __uint_as_float(x[0]) + __uint_as_float(x[1]);
        const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l), false, false);
        l = __uint_as_float(y[0]) + __uint_as_float(y[1]);
        inv[rb] = l > 0.f ? a.v_scale / l : 0.f;  // v_scale is 1 for bf16 pools
        // (a split item passes a NaN sum on to the merge)
        lse_v[rb] = l > 0.f ? (m_run[rb] + log2f(l)) * kLn2 : (it.part >= 0 && l != l ? l : -INFINITY);
    }
    // o[rb][db][v] is element d = 16 db + 4 g4 + v of row 16 rb + j16
    if (it.part < 0) {
        // Output rows go through LDS so that every store writes whole rows: a lane's own
        // values cover 16 bytes of each of 32 rows, 256 bytes apart. The tiles are no
        // longer read (the last barrier above), so each wavefront takes 8 KiB (4 KiB for
        // d = 64) of the tile buffers: its 32 rows, 16-byte chunks XOR-swizzled by row.
        // Each store then covers 256 (128) contiguous bytes of 4 (8) rows, and the rows
        // of one token's query heads are adjacent in the output.
        constexpr int kOutRow = 2 * D;                  // bytes per row
        constexpr int CH = kOutRow / 16;                // 16-byte chunks per row
        constexpr int kStage = kRowsPerWave * kOutRow;  // bytes per wavefront
        constexpr int kPerBuf = kTileBytes / kStage;    // wavefronts per tile buffer
        static_assert(kPerBuf * 4 >= WAVES && kPerBuf * kStage == kTileBytes, "stage layout");
        const int sb = wave / kPerBuf;
        unsigned char* stage = (sb == 0 ? k_lds0 : sb == 1 ? v_lds0 : sb == 2 ? k_lds1 : v_lds1) +
                               (wave % kPerBuf) * kStage;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int row = 16 * rb + j16;
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                u32x2 w;
                w[0] = pack_bf16x2(o[rb][db][0] * inv[rb], o[rb][db][1] * inv[rb]);
                w[1] = pack_bf16x2(o[rb][db][2] * inv[rb], o[rb][db][3] * inv[rb]);
                *reinterpret_cast<u32x2*>(stage + row * kOutRow + ((2 * db + (g4 >> 1)) ^ (row & (CH - 1))) * 16 +
                                          8 * (g4 & 1)) = w;
            }
            if (row_ok[rb] && a.lse != nullptr && g4 == 0) a.lse[qrow[rb]] = lse_v[rb];
        }
        wave_lds_sync();
        constexpr int kRowsPerStore = 64 / CH;
#pragma unroll
        for (int i = 0; i < kRowsPerWave / kRowsPerStore; ++i) {
            const int rr = i * kRowsPerStore + lane / CH, ch = lane % CH;
            const u32x4 v = *reinterpret_cast<const u32x4*>(stage + rr * kOutRow + (ch ^ (rr & (CH - 1))) * 16);
            const int mr = wave * kRowsPerWave + rr;  // the stored row's token and head
            const int tr = mr / a.group;
            if (tr < ntok) {
                const int64_t qr = (int64_t)(cu + it.q0 + tr) * a.num_q_heads + kvh * a.group + (mr - tr * a.group);
                *reinterpret_cast<u32x4*>(a.out + qr * D + ch * 8) = v;
            }
        }
    } else {
        // Partial rows (fp32) of a split item, through the same stage: the wavefront's 32
        // rows are contiguous in the partial buffer, so each store covers whole rows; rows
        // larger than the stage go in rounds of kRows.
        constexpr int kOutRow = 4 * D;                        // bytes per fp32 row
        constexpr int CH = kOutRow / 16;                      // 16-byte chunks per row
        constexpr int kStage = 4 * kTileBytes / WAVES;        // stage bytes per wavefront
        constexpr int kRows = kStage / kOutRow < kRowsPerWave ? kStage / kOutRow : kRowsPerWave;
        static_assert(kRows >= 2 && kRowsPerWave % kRows == 0 && (kRows * CH) % 64 == 0, "partial stage");
        constexpr int kPerBuf = kTileBytes / kStage;
        const int sb = wave / kPerBuf;
        unsigned char* stage = (sb == 0 ? k_lds0 : sb == 1 ? v_lds0 : sb == 2 ? k_lds1 : v_lds1) +
                               (wave % kPerBuf) * kStage;
        const int64_t prow0 = ((int64_t)it.part * a.num_kv_heads + kvh) * kBlockRows + wave * kRowsPerWave;
        constexpr int kSw = CH < 16 ? CH : 16;                // chunk swizzle span
#pragma unroll
        for (int r0 = 0; r0 < kRowsPerWave; r0 += kRows) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const int sr = 16 * rb + j16 - r0;
                if (sr < 0 || sr >= kRows) continue;
#pragma unroll
                for (int db = 0; db < DB; ++db)
                    *reinterpret_cast<f32x4*>(stage + sr * kOutRow + ((4 * db + g4) ^ (sr & (kSw - 1))) * 16) =
                        o[rb][db] * inv[rb];
            }
            wave_lds_sync();
#pragma unroll
            for (int i = 0; i < kRows * CH / 64; ++i) {
                const int c = i * 64 + lane, sr = c / CH, ch = c % CH;
                const f32x4 v = *reinterpret_cast<const f32x4*>(stage + sr * kOutRow + (ch ^ (sr & (kSw - 1))) * 16);
                *reinterpret_cast<f32x4*>(a.part_o + (prow0 + r0 + sr) * D + ch * 4) = v;
            }
            wave_lds_sync();  // the next round overwrites the stage
        }
        if (g4 == 0) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) a.part_lse[prow0 + 16 * rb + j16] = lse_v[rb];
        }
    }
}

// WGS: workgroups per compute unit to compile for. Two wavefronts per SIMD, or three: the 128-row tiles
// at d = 64 take 164 registers over bf16 pools, and 189 over 8-bit ones, whose third workgroup costs 12
// spilled registers (the launcher's rule says when it pays).
template <int D, int WAVES, bool FP8, int WGS = 8 / WAVES>
__global__ __launch_bounds__(WAVES * 64, WGS) void attention_kernel(const AttnArgs a) {
    attention_body<D, WAVES, FP8, WGS>(a, blockIdx.x);
}

// Resident launch (wide tiles): one workgroup per compute unit, each
// taking work items until none is left. Queue x holds the regular launch's indices
// x, x + 8, x + 16, ...: the hardware deals workgroups to the eight XCDs in turn, so
// workgroup b serves queue b % 8 and each XCD runs the items (and KV heads) it runs in
// the regular launch, keeping their K/V in its L2. A workgroup whose queue is empty
// takes items from the other queues, so XCDs that run slower do not hold up the end of
// the launch; and a freed compute unit starts its next item without waiting for the
// dispatcher, which hands out new workgroups in index order across the XCDs. Tickets
// are agent-scope atomics on the workspace's counters; the last workgroup to leave
// sets them back to zero for the next launch (the ticket atomics of every other
// workgroup returned before it counted itself out).
template <int D, bool FP8>
__global__ __launch_bounds__(kWideWaves * 64, 1) void attention_resident_kernel(const AttnArgs a, int total) {
    __shared__ int s_tk, s_empty;
    const int x = (int)(blockIdx.x % (unsigned)kQueues);
    if (threadIdx.x == 0) s_empty = 0;
    for (;;) {
        if (threadIdx.x == 0) {
            int b = -1, empty = s_empty;
            for (int j = 0; j < kQueues && b < 0; ++j) {
                const int y = (x + j) % kQueues;
                if (empty & (1 << y)) continue;
                const int k = __hip_atomic_fetch_add(&a.queues[y], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if ((int64_t)k * kQueues + y < total) b = k * kQueues + y;
                else empty |= 1 << y;
            }
            s_empty = empty;
            s_tk = b;
        }
        __syncthreads();
        const int b = s_tk;
        __syncthreads();  // every wavefront has read the ticket before the next one is written
        if (b < 0) break;
        attention_body<D, kWideWaves, FP8>(a, (unsigned)b);
    }
    if (threadIdx.x == 0) {
        const int out = __hip_atomic_fetch_add(&a.queues[kQueues], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (out == (int)gridDim.x - 1)
            for (int y = 0; y <= kQueues; ++y)
                __hip_atomic_store(&a.queues[y], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Merge the key chunks of one split query tile: with m = max_s lse_s,
// lse = m + log sum_s exp(lse_s - m) and o = sum_s exp(lse_s - m) o_s / sum_s exp(lse_s - m),
// in a fixed order (deterministic). A thread owns four consecutive
// output elements of one row, so the partial rows are read with coalesced 16-byte loads.
// What bounds it is the round trips of dependent loads, not the bytes: chunks and their
// log-sum-exps are read kBatch at a time in one pass with a running maximum, and with
// S > 1 a row's chunks are dealt to S groups of threads (chunk s to group s % S) whose
// results are joined through LDS in group order.
template <int D, int S>
__global__ __launch_bounds__(kCombineThreads) void combine_kernel(const CombineArgs a) {
    constexpr int CPR = D / 4;                          // float4 chunks per row
    constexpr int kRows = kCombineThreads / (CPR * S);  // rows per workgroup
    __shared__ f32x4 s_acc[S > 1 ? kCombineThreads : 1];
    __shared__ float s_max[S > 1 ? kCombineThreads / CPR : 1], s_tot[S > 1 ? kCombineThreads / CPR : 1];
    const int groups = ceil_div(a.block_m, kRows);
    const unsigned tile = blockIdx.x / (unsigned)groups;
    const int lane_row = (int)threadIdx.x / CPR;        // (row, group) of this thread
    const int sub = lane_row % S;
    const int m = (int)(blockIdx.x % (unsigned)groups) * kRows + lane_row / S;
    const int c4 = (int)threadIdx.x % CPR;
    const int kvh = (int)(tile % (unsigned)a.num_kv_heads);
    const CombineItem ci = a.combines[tile / (unsigned)a.num_kv_heads];
    if (ci.ns <= 0 || ci.r < 0 || ci.r >= a.batch || ci.q0 < 0 || ci.part_base < 0 ||
        ci.part_base + ci.ns > a.num_partials)
        return;
    const int cu = a.cu_new_lens[ci.r];
    const int n = a.cu_new_lens[ci.r + 1] - cu;
    if (ci.q0 >= n) return;
    const int ntok = min(a.tq, n - ci.q0);
    const int t = (int)((unsigned)m / (unsigned)a.group), hl = m - t * a.group;
    const bool row_ok = m < a.block_m && t < ntok;
    if (S == 1 && !row_ok) return;
    float mx = -INFINITY, tot = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if (row_ok) {
        const int64_t row0 = ((int64_t)ci.part_base * a.num_kv_heads + kvh) * a.block_m + m;
        const int64_t split_stride = (int64_t)a.num_kv_heads * a.block_m;  // rows between chunks
        constexpr int kBatch = S > 1 ? 4 : 8;
        for (int s0 = sub; s0 < ci.ns; s0 += kBatch * S) {
            float l[kBatch];
            f32x4 v[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const bool ok = s0 + u * S < ci.ns;
                const int64_t pr = row0 + (int64_t)(s0 + u * S) * split_stride;
                l[u] = ok ? a.part_lse[pr] : -INFINITY;
                // (a padding entry adds weight 0 times 0, never times a row that may hold
                // infinities; zeroing a row read in its place took 0.6 us of 84 on 16 document
                // questions, skipping the read takes nothing)
                v[u] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (ok) v[u] = *reinterpret_cast<const f32x4*>(a.part_o + pr * D + 4 * c4);
            }
            float mn = mx;
#pragma unroll
            for (int u = 0; u < kBatch; ++u) mn = fmaxf(mn, l[u]);
            const float off = mn == -INFINITY ? 0.f : mn;  // (chunks in which the row sees no key)
            const float alpha = expf(mx - off);
            tot *= alpha;
            acc *= alpha;
            mx = mn;
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const float w = expf(l[u] - off);  // 0 for the padding entries
                tot += w;
                acc += w * v[u];
            }
        }
    }
    if constexpr (S > 1) {
        s_acc[threadIdx.x] = acc;
        if (c4 == 0) {
            s_max[lane_row] = mx;
            s_tot[lane_row] = tot;
        }
        __syncthreads();
        if (sub != 0 || !row_ok) return;
        const float mx0 = mx;
#pragma unroll
        for (int g = 1; g < S; ++g) mx = fmaxf(mx, s_max[lane_row + g]);
        const float off = mx == -INFINITY ? 0.f : mx;
        const float w0 = expf(mx0 - off);
        tot *= w0;
        acc *= w0;
#pragma unroll
        for (int g = 1; g < S; ++g) {
            const float w = expf(s_max[lane_row + g] - off);
            tot += w * s_tot[lane_row + g];
            acc += w * s_acc[threadIdx.x + g * CPR];
        }
    }
    // as in an unsplit item: a row whose weights are all 0 gives 0, one whose sum is NaN
    // gives NaN (already in acc), both with the log-sum-exp -inf
    const float lse_tot = tot > 0.f ? mx + logf(tot) : -INFINITY;
    acc *= tot > 0.f ? 1.f / tot : 0.f;
    const int64_t qrow = (int64_t)(cu + ci.q0 + t) * a.num_q_heads + kvh * a.group + hl;
    u32x2 w2;
    w2[0] = pack_bf16x2(acc[0], acc[1]);
    w2[1] = pack_bf16x2(acc[2], acc[3]);
    *reinterpret_cast<u32x2*>(a.out + qrow * D + 4 * c4) = w2;
    if (a.lse != nullptr && c4 == 0) a.lse[qrow] = lse_tot;
}

}  // namespace
}  // namespace gc

// fp32 attention over one key partition on the gfx950 matrix cores, for fp32 inputs.  Same online-softmax
// recurrence, same partial format and the same transposed mapping as the bf16 kernel (Section 3 of the
// paper: softmax(scale * Q K^T) V; window keys masked with j <= i).
//
// Products.  A bf16 matrix instruction does sixteen times the work of an fp32 one, and an fp32 number is the
// sum of three bf16 numbers without a remainder (8 + 8 + 8 bits of significand, the exponents have the same
// range).  Every operand (Q, K, V and the weights) is split that way, and a product is the six bf16 products of
// parts whose indices add up to at most two, exact in the fp32 accumulator; the three that are left out are
// below 2^-23 of the product, of either sign, 2^-26 as a rule (the middle part is rounded to nearest).  The bf16 matrix
// instruction rounds its sums towards minus infinity (an offset of 1e-9 of the values per key, measured; the fp32
// one rounds to nearest), which adds up over a history: every other tile's weights are negated and its product
// subtracted, so that the offsets cancel.  Measured against 64 bits, 2-norm, fp32 matrix instructions -> this kernel
// (without the change of sign): 40 rows x 64 over 20000 rows 1.77e-7 -> 1.47e-7 (1.97e-7), over 10^5 1.85e-7 ->
// 1.62e-7 (3.33e-7), over 10^6 2.48e-7 -> 2.33e-7 (1.03e-6).
//   32 heads x 128, 512 rows over 32768 history rows: 2451 -> 1298 us (215 TFLOP/s, 1.29 PFLOP/s of bf16
//   products; the library's bf16 matrix product reaches 1.33 on this card, the power limit), 32 heads x 36, 64
//   rows over 32768: 170 -> 116, causal, 16 heads x 128, 4096 rows: 1032 -> 379.
//
// Mapping (wave64; a wave owns 32 query rows; operand layouts as in attn_bf16_pipe_body):
//   * Tiles of 32 keys.  A lane loads its share of a tile into registers (the tile after the next step's), splits
//     it and writes three planes of bf16 rows to LDS, in the layout and swizzle of the bf16 kernels' K and V
//     tiles: 48 KB of planes at D = 128.  The split costs 5.5 vector instructions per element, once per workgroup.
//   * Two barriers per tile and a single buffer: while the score products read K(t), V(t) is split and written;
//     while the value products read V(t), K(t+1) is.  The smaller workgroups share a compute unit, and one's
//     softmax and barriers are hidden by the others' products.
//   * Registers at D = 128: parts 0 and 1 of the queries 64, accumulator 64, scores 32 (leading and other
//     products apart); part 2 of the queries, in one product of six, sits in LDS.
//   * Tensors with a head dimension a.D below the kernel's D: see DP.  a.D is a multiple of 4, so 16-byte pieces of
//     a row are whole or absent; absent ones lie beyond the tile descriptor's size (zeros, no memory request).
#pragma once
#include "attn_bf16.h"

namespace tlin {

// x = p[0] + p[1] + p[2] exactly, each part four bf16 values: the leading 8 bits as they stand, the next 8 rounded
// to nearest (so that what lies below them carries no common sign), and the rest.  Not for infinities, whose p[1] is
// NaN: see the end of attn_f32_body.
__device__ __forceinline__ void split4(f32x4 x, u32x2 (&p)[3])
{
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const float x0 = x[2 * e], x1 = x[2 * e + 1];
        const unsigned u0 = __builtin_bit_cast(unsigned, x0), u1 = __builtin_bit_cast(unsigned, x1);
        p[0][e] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);
        const float r0 = x0 - __builtin_bit_cast(float, u0 & 0xffff0000u), r1 = x1 - __builtin_bit_cast(float, u1 & 0xffff0000u);
        const bf16x2 b = {(__bf16)r0, (__bf16)r1};
        unsigned ub = __builtin_bit_cast(unsigned, b);
        asm("" : "+v"(ub));                    // (or both are converted once more for their remainders)
        p[1][e] = ub;
        const bf16x2 c = {(__bf16)(r0 - __builtin_bit_cast(float, ub << 16)), (__bf16)(r1 - __builtin_bit_cast(float, ub & 0xffff0000u))};
        p[2][e] = __builtin_bit_cast(unsigned, c);
    }
}

// The smallest magnitude among values that are not zero, as an ordered number (the bits without the sign, doubled,
// less one: zeros come out last).
__device__ __forceinline__ unsigned least_nonzero(unsigned least, float x)
{
    return min(least, (__builtin_bit_cast(unsigned, x) << 1) - 1u);
}

// Order of a region's instructions: M products, with the next region's R operand reads and V vector instructions
// spread over them.  (Left to itself the compiler requests operands right before their product and lumps the
// splits together between the products: 32 heads x 128, 512 rows over 32768 7 % faster with this order, 16
// heads x 128, 1000 causal rows 98 -> 82 us; 96 columns with eight waves 1.5 % slower.)
template <int R, int M, int V, int ID>
__device__ __forceinline__ void interleave()
{
    constexpr int AHEAD = 2;               // reads behind the first product, then one behind each
    static_for<M>([](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value, nv = (V * (i + 1)) / M - (V * i) / M, ri = AHEAD + i;
        constexpr int nr = (i == 0 ? AHEAD : 0) + (ri < R ? 1 : 0) + (i == M - 1 && ri + 1 < R ? R - ri - 1 : 0);
        __builtin_amdgcn_sched_group_barrier(SG_MFMA, 1, ID);
        if (nr > 0) __builtin_amdgcn_sched_group_barrier(SG_DSR, nr, ID);
        if (nv > 0) __builtin_amdgcn_sched_group_barrier(SG_VALU, nv, ID);
    });
    __builtin_amdgcn_sched_barrier(0);
}

// The work of one workgroup; `bid` of `nblocks` is its index among the blocks of this problem set.
// DP: 0 where the tensors' head dimension a.D is the kernel's D.  Where it is smaller, the columns that are
// computed: at least a.D, a multiple of 16; rows keep the kernel's D elements in LDS.
// REMAP: bid is a hardware block index (mapped to a logical one here); otherwise it is the logical index.
template <int D, int NW, bool CAUSAL, int DP, bool REMAP = true>
__device__ __forceinline__ void attn_f32_body(const AttnArgs &a, int bid, int nblocks)
{
    constexpr int BN = 32;                 // keys per tile
    constexpr int BM = NW * 32;            // query rows per workgroup
    constexpr int ROWB = D * 2;            // bytes per row of a plane
    constexpr int PLANE_B = BN * ROWB;
    constexpr int DU = DP ? DP : D;        // columns computed
    constexpr int DS = DU / 16;            // contraction steps of Q K^T
    constexpr int DB = (DU + 31) / 32;     // 32-row blocks of O^T
    constexpr int CPR = D / 4;             // 16-byte pieces of a row in memory
    constexpr int NLD = BN * CPR / (NW * 64);   // pieces of a tile of K (and of V) that a lane loads and splits
    constexpr int LROWS = NW * 64 / CPR;   // tile rows covered by one load of the workgroup
    static_assert(NLD >= 1 && BN % LROWS == 0, "tile does not divide over the threads");

    char *const Ks = tlin_smem;
    char *const Vs = Ks + 3 * PLANE_B;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 31, h = lane >> 5;
    char *const Q2 = Vs + 3 * PLANE_B + wave * (DS * 1024);

    const int L = REMAP ? xcd_remap(bid, nblocks) : bid;
    const Problem pr = decode_problem<BM, BN, CAUSAL>(a, L, a.nqb);
    if (pr.skip) return;                   // uniform over the workgroup
    const int qb = pr.qb, split = pr.split, bh = pr.bh;
    const int b = bh / a.H, hd = bh % a.H;
    const int Wq = pr.W, NK = pr.NK;       // query and key rows of this problem

    int t0 = 0, t1 = (min(NK, qb * BM + BM) + BN - 1) / BN;
    if (!CAUSAL) partition_tiles<BM, BN, 4>(a, pr, t0, t1);

    const int64_t k_rb = a.k_sr * 4, v_rb = a.v_sr * 4;
    const float *Qg = (const float *)a.Q + (int64_t)b * a.q_sb + (int64_t)hd * a.q_sh + pr.qrow_off * a.q_sr;
    const char *Kg = (const char *)((const float *)a.K + (int64_t)b * a.k_sb + (int64_t)hd * a.k_sh) + pr.krow_off * k_rb;
    const char *Vg = (const char *)((const float *)a.V + (int64_t)b * a.v_sb + (int64_t)hd * a.v_sh) + pr.krow_off * v_rb;

    // ---- Q^T fragments (B operand of the score product): lane holds query j, columns 16 s + 8 h .. + 7.  Parts
    // 0 and 1 stay in registers, part 2 (one product in six) in LDS, each wave its own.
    const int qrow0 = qb * BM + wave * 32;
    bf16x8 q0[DS], q1[DS];
    uint64_t far;                          // lanes whose queries leave 2^-100 .. 2^100 (see below)
    {
        float q_most[2] = {0.f, 0.f};
        unsigned q_least[2] = {0xffffffffu, 0xffffffffu};
        const float *const qp = Qg + (int64_t)min(qrow0 + j, Wq - 1) * a.q_sr + 8 * h;
#pragma unroll
        for (int s = 0; s < DS; ++s) {
            u32x2 p[2][3];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const f32x4 x = 16 * s + 8 * h + 4 * e < a.D ? *(const f32x4 *)(qp + 16 * s + 4 * e) : f32x4{0.f, 0.f, 0.f, 0.f};
                split4(x, p[e]);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    q_most[e] = fmaxf(q_most[e], fabsf(x[v]));
                    q_least[e] = least_nonzero(q_least[e], x[v]);
                }
            }
            q0[s] = __builtin_bit_cast(bf16x8, u32x4{p[0][0][0], p[0][0][1], p[1][0][0], p[1][0][1]});
            q1[s] = __builtin_bit_cast(bf16x8, u32x4{p[0][1][0], p[0][1][1], p[1][1][0], p[1][1][1]});
            *(u32x4 *)(Q2 + s * 1024 + lane * 16) = u32x4{p[0][2][0], p[0][2][1], p[1][2][0], p[1][2][1]};
        }
        far = __builtin_amdgcn_ballot_w64(fmaxf(q_most[0], q_most[1]) > 0x1p100f || min(q_least[0], q_least[1]) < least_nonzero(0xffffffffu, 0x1p-100f));
        asm volatile("" : "+s"(far));          // here, where the queries are at hand
    }

    // ---- tile loads: load i of this lane is piece `lc` of tile row i * LROWS + lr, in memory and in LDS
    const int lr = tid / CPR, lc = tid % CPR;
    // pieces beyond the rows' end: an offset beyond every tile descriptor (a tile is below 2^30 bytes), zeros
    const unsigned koff = 4 * lc < a.D ? (unsigned)(lr * k_rb) + 16 * lc : 0x80000000u;
    const unsigned voff = 4 * lc < a.D ? (unsigned)(lr * v_rb) + 16 * lc : 0x80000000u;
    const unsigned krow_step = (unsigned)(LROWS * k_rb), vrow_step = (unsigned)(LROWS * v_rb);
    auto load_tile = [&](f32x4 (&x)[NLD], const char *base, int64_t rb, unsigned off, unsigned step, int t) __attribute__((always_inline)) {
        const int key0 = t * BN, rows = min(BN, NK - key0);      // rows past the end of the tensor arrive as zeros
        auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(base + key0 * rb), 0, (int)(rows * rb), 0x00020000);
#pragma unroll
        for (int i = 0; i < NLD; ++i)
            x[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off + i * step, 0, 0));
    };
    auto store_piece = [&](f32x4 x, char *planes, int row, int swz) __attribute__((always_inline)) {
        u32x2 p[3];
        split4(x, p);
        char *dst = planes + row * ROWB + (((lc >> 1) ^ swz) << 4) + 8 * (lc & 1);
#pragma unroll
        for (int k = 0; k < 3; ++k) *(u32x2 *)(dst + k * PLANE_B) = p[k];
    };
    f32x4 kx[NLD], vx[NLD];
    auto load_k = [&](int t) __attribute__((always_inline)) { load_tile(kx, Kg, k_rb, koff, krow_step, t); };
    auto load_v = [&](int t) __attribute__((always_inline)) { load_tile(vx, Vg, v_rb, voff, vrow_step, t); };
    auto put_k = [&](int i) __attribute__((always_inline)) { store_piece(kx[i], Ks, i * LROWS + lr, Swz<D>::k(i * LROWS + lr)); };
    auto put_v = [&](int i) __attribute__((always_inline)) { store_piece(vx[i], Vs, i * LROWS + lr, Swz<D>::v(i * LROWS + lr)); };
    // this wave's LDS writes are done, then every wave's are (and every wave is past its reads)
    auto meet = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // ---- state: running maximum (raw logit units), running sum, O^T accumulator
    float m = -INFINITY, l = 0.f;
    f32x16 oacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[db][v] = 0.f;
    // The running maximum only moves when a tile maximum exceeds it by more than 2^8 in the
    // exponent: weights stay <= 256 and the accumulator is rescaled rarely.  Any reference point
    // gives the same normalised result.
    const float thr = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, 8.0f / a.c)));

    // LDS addresses: K fragment of step s, key j, columns 16 s + 8 h .. + 7; V operand of column block db, see
    // attn_bf16_pipe_body
    typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
    const int i16 = lane & 15, blk1 = (lane >> 4) & 1;
    unsigned kaddr[DS], vaddr[DB];
#pragma unroll
    for (int s = 0; s < DS; ++s) kaddr[s] = lds_offset(Ks) + j * ROWB + (((2 * s + h) ^ Swz<D>::k(j)) << 4);
    {
        const int r0 = 4 * h + (i16 >> 2);
        const int sw = Swz<D>::v(r0) << 4;           // the same for rows r0 + 8 k
#pragma unroll
        for (int db = 0; db < DB; ++db) vaddr[db] = lds_offset(Vs) + r0 * ROWB + ((64 * db + 32 * blk1 + 8 * (i16 & 3)) ^ sw);
    }
    const unsigned q2addr = lds_offset(Q2) + lane * 16;
    auto k_read = [&](int s, int plane) __attribute__((always_inline)) { return *(lds_bf16x8 *)(uintptr_t)(kaddr[s] + plane * PLANE_B); };
    auto v_read = [&](int db, int t2, int plane) __attribute__((always_inline)) {
        const unsigned ad = vaddr[db] + plane * PLANE_B + t2 * (16 * ROWB);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(uintptr_t)ad);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(uintptr_t)(ad + 8 * ROWB));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto mma = [](bf16x8 x, bf16x8 y, f32x16 c) __attribute__((always_inline)) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, c, 0, 0, 0); };

    // ---- mask of a tile's scores (keys past the end of the tensor, and (causal) keys after the query row) and its
    // maximum, and the reference point's move to it
    auto mask_and_reference = [&](f32x16 &s, int key0, int j, int h) __attribute__((always_inline)) {
        const int row = qrow0 + j;
        if (key0 + BN > NK || (CAUSAL && key0 + BN - 1 > qrow0)) {
            const int lim = CAUSAL ? min(row, NK - 1) : NK - 1;   // last visible key
            const int rel = lim - key0 - 4 * h;                    // the same, counted from this lane's first key
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (8 * (v >> 2) + (v & 3) > rel) s[v] = -INFINITY;
        }

        float mx = s[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
        mx = xhalf_max(mx);
        if (__builtin_amdgcn_ballot_w64(mx > m + thr) != 0) {
            const float mn = fmaxf(m, mx);
            const float alpha = (mn == -INFINITY) ? 1.f : fast_exp2((m - mn) * a.c);
            l *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) oacc[db][v] *= alpha;
            m = mn;
        }
    };

    // Tiles after every row this wave owns (causal), and all tiles where the window ends before its first
    // row, are not computed by it, but the wave still loads and splits its share of them for the others and meets
    // them at the barriers: the waves that have rows get the matrix cores for themselves.
    const int t1w = qrow0 >= Wq ? t0 : CAUSAL ? min(t1, (qrow0 + 31) / BN + 1) : t1;

    // ---- The same over the partition by fp32 matrix instructions, a wave for itself, its operands straight from memory.
    // A 32x32x2 product contracts over two indices, one per half-wave; which two is free as long as both operands agree:
    //   scores  step (t, e) pairs columns 8 t + e (h = 0) and 8 t + 4 + e (h = 1): a lane needs K[key j][8 t + 4 h ..
    //           + 3], one 16-byte load per four products, and its query's same columns, which it keeps in registers.
    //   values  step (g, e) pairs keys 8 g + e and 8 g + 4 + e: the weight operand is the score accumulator's register
    //           4 g + e as it stands, the other V[key 8 g + 4 h + e][32 db + j].
    // Sums over columns run as chains of 32 terms, a tile's value product on its own: short chains round less.
    auto fp32_pass = [&]() __attribute__((always_inline)) {
        // (what depends on the lane is computed again instead of being kept through the first pass)
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        const int j = lane & 31, h = lane >> 5;
        const float *const qp = Qg + (int64_t)min(qrow0 + j, Wq - 1) * a.q_sr + 4 * h;
        f32x4 qf[4 * DB];
#pragma unroll
        for (int t8 = 0; t8 < 4 * DB; ++t8) qf[t8] = 8 * t8 + 4 * h < a.D ? *(const f32x4 *)(qp + 8 * t8) : f32x4{0.f, 0.f, 0.f, 0.f};
        m = -INFINITY;
        l = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) oacc[db][v] = 0.f;
        for (int t = t0; t < t1w; ++t) {
            const int key0 = t * BN, rows = min(BN, NK - key0);      // as in load_tile
            auto kr = __builtin_amdgcn_make_buffer_rsrc((void *)(Kg + key0 * k_rb), 0, (int)(rows * k_rb), 0x00020000);
            auto vr = __builtin_amdgcn_make_buffer_rsrc((void *)(Vg + key0 * v_rb), 0, (int)(rows * v_rb), 0x00020000);
            const unsigned ko = (unsigned)(j * k_rb) + 16 * h, vo = (unsigned)(4 * h * v_rb) + 4 * j;
            f32x16 s;
#pragma unroll
            for (int c = 0; c < DB; ++c) {
                f32x16 part;
#pragma unroll
                for (int v = 0; v < 16; ++v) part[v] = 0.f;
#pragma unroll
                for (int t8 = 4 * c; t8 < 4 * c + 4; ++t8) {
                    const f32x4 kf = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(kr, 8 * t8 + 4 * h < a.D ? ko + 32 * t8 : 0x80000000u, 0, 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e) part = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[e], qf[t8][e], part, 0, 0, 0);
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) s[v] = c == 0 ? part[v] : s[v] + part[v];
            }
            mask_and_reference(s, key0, j, h);
            const float mref = (m == -INFINITY) ? 0.f : m;
            float ls = 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                s[v] = fast_exp2((s[v] - mref) * a.c);
                ls += s[v];
            }
            l += ls;
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                f32x16 pv;
#pragma unroll
                for (int v = 0; v < 16; ++v) pv[v] = 0.f;
#pragma unroll
                for (int g = 0; g < 4; ++g)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const unsigned off = 32 * db + j < a.D ? vo + (unsigned)((8 * g + e) * v_rb) + 128 * db : 0x80000000u;
                        const float vf = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(vr, off, 0, 0));
                        pv = __builtin_amdgcn_mfma_f32_32x32x2f32(vf, s[4 * g + e], pv, 0, 0, 0);
                    }
#pragma unroll
                for (int v = 0; v < 16; ++v) oacc[db][v] += pv[v];
                __builtin_amdgcn_sched_barrier(0);     // keeps the next block's loads (registers) behind this block
            }
        }
    };

    if (t0 < t1) {
        load_k(t0);
#pragma unroll
        for (int i = 0; i < NLD; ++i) put_k(i);
        load_v(t0);
        meet();
    }
    int t = t0;
    for (; t < t1w; ++t) {
        const int tn = min(t + 1, t1 - 1);     // behind the last tile it is loaded once more, and nobody reads it
        const int key0 = t * BN;
        // ---- scores S^T = K Q^T, the tile's values split and written meanwhile.  The products of the leading
        // parts and the others are summed apart: the latter are 2^-8 of the former and cost no accuracy.
        load_k(tn);
        f32x16 s, lo;
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = lo[v] = 0.f;
        bf16x8 kf[2][4];                       // operands of a step: three parts of K, part 2 of Q; requested a step ahead
        auto read_step = [&](int c) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < 3; ++k) kf[c & 1][k] = k_read(c, k);
            kf[c & 1][3] = *(lds_bf16x8 *)(uintptr_t)(q2addr + c * 1024);
        };
        read_step(0);
        static_for<DS>([&](auto cc) __attribute__((always_inline)) {
            constexpr int c = decltype(cc)::value;
            if (c + 1 < DS) read_step(c + 1);
            const bf16x8 (&f)[4] = kf[c & 1];
            lo = mma(f[0], q1[c], lo);
            s = mma(f[0], q0[c], s);
            lo = mma(f[1], q0[c], lo);
            lo = mma(f[1], q1[c], lo);
            lo = mma(f[0], f[3], lo);
            lo = mma(f[2], q0[c], lo);
            constexpr int p0 = c * NLD / DS, p1 = (c + 1) * NLD / DS;
#pragma unroll
            for (int i = p0; i < p1; ++i) put_v(i);
            interleave<4, 6, (p1 - p0) * 27, 0>();
        });
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] += lo[v];

        mask_and_reference(s, key0, j, h);

        // ---- weights.
        // (every other tile's negated: see the value product)
        const unsigned flip = (unsigned)t << 31;
        const float sign = __builtin_bit_cast(float, 0x3f800000u ^ flip);
        // (s - m) * c rather than fma(s, c, -m*c): the key that holds the maximum gets weight exactly 1
        const float mref = (m == -INFINITY) ? 0.f : m;
        float ls = 0.f;
        bf16x8 pw[2][3];      // weights, B-operand order, split
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2) {
            u32x2 p[2][3];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                f32x4 w;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float p = fast_exp2((s[8 * t2 + 4 * e + v] - mref) * a.c);
                    ls += p;
                    w[v] = __builtin_bit_cast(float, __builtin_bit_cast(unsigned, p) ^ flip);
                }
                split4(w, p[e]);
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) pw[t2][k] = __builtin_bit_cast(bf16x8, u32x4{p[0][k][0], p[0][k][1], p[1][k][0], p[1][k][1]});
        }
        l += ls;
        __builtin_amdgcn_sched_barrier(0);
        meet();
        __builtin_amdgcn_sched_barrier(0);

        // ---- O^T += V^T P^T, the next tile's keys split and written meanwhile.  The tile's product is summed on
        // its own, small parts first, and then added to the running accumulator: short summation chains round
        // less than one long one.
        load_v(tn);
        bf16x8 vf[2][3], v0a;                  // operands of a step: three parts of V
        f32x16 pv;
        auto read_v = [&](int i) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 2; k >= 0; --k) vf[i & 1][k] = v_read(i >> 1, i & 1, k);
        };
        read_v(0);
        static_for<2 * DB>([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value, db = i >> 1, t2 = i & 1;
            if (i + 1 < 2 * DB) read_v(i + 1);
            const bf16x8 (&f)[3] = vf[i & 1];
            if (t2 == 0)
#pragma unroll
                for (int v = 0; v < 16; ++v) pv[v] = 0.f;
            pv = mma(f[2], pw[t2][0], pv);
            pv = mma(f[1], pw[t2][1], pv);
            pv = mma(f[0], pw[t2][2], pv);
            pv = mma(f[1], pw[t2][0], pv);
            pv = mma(f[0], pw[t2][1], pv);
            if (t2 == 0) v0a = f[0];
            else {
                pv = mma(v0a, pw[0][0], pv);
                pv = mma(f[0], pw[1][0], pv);
            }
            constexpr int p0 = i * NLD / (2 * DB), p1 = (i + 1) * NLD / (2 * DB);
#pragma unroll
            for (int n = p0; n < p1; ++n) put_k(n);
            if (t2 == 1)
#pragma unroll
                for (int v = 0; v < 16; ++v) oacc[db][v] = fmaf(pv[v], sign, oacc[db][v]);
            interleave<6, 5 + 2 * t2, (p1 - p0) * 27, 1>();
        });
        meet();
    }
    // the remaining tiles of a wave that does not compute on them
    for (; t < t1; ++t) {
        const int tn = min(t + 1, t1 - 1);
        load_k(tn);
#pragma unroll
        for (int i = 0; i < NLD; ++i) put_v(i);
        meet();
        load_v(tn);
#pragma unroll
        for (int i = 0; i < NLD; ++i) put_k(i);
        meet();
    }


    // ---- inputs that three bf16 parts cannot hold.  Infinities (and NaN) in Q, K or V and products that overflow leave
    // something that is not finite in a row's sum or accumulator.  Parts below bf16's range are lost: an element of Q, K
    // or V keeps an absolute precision of 2^-134, which matters only where it meets something very large or where a
    // column is as small throughout: queries beyond 2^100 or (not zero) below 2^-100, outputs (not zero) below 2^-110
    // in several rows (in one it is sums that cancel; a wave of fewer than four rows: below 2^-116).  The wave then goes
    // over its partition again with fp32 matrix instructions.
    if (t0 < t1w) {
        float nan[4] = {l * 0.f, 0.f, 0.f, 0.f};        // stay 0 unless something is not finite (four: short chains)
        unsigned least[4] = {0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu};
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                nan[v & 3] = fmaf(oacc[db][v], 0.f, nan[v & 3]);
                least[v & 3] = least_nonzero(least[v & 3], oacc[db][v]);
            }
        const uint64_t odd = far | __builtin_amdgcn_ballot_w64(!((nan[0] + nan[1]) + (nan[2] + nan[3]) == 0.f));
        const bool few = Wq - qrow0 < 4;
        const unsigned limit = least_nonzero(0xffffffffu, xhalf_sum(l) * (few ? 0x1p-116f : 0x1p-110f));
        const uint64_t small = __builtin_amdgcn_ballot_w64(qrow0 + j < Wq && min(min(least[0], least[1]), min(least[2], least[3])) < limit);
        if (odd != 0 || __builtin_popcountll(small) >= (few ? 1 : 4)) fp32_pass();
    }

    // ---- epilogue.  Accumulator register v of block db is d = 32*db + 8*(v/4) + 4*h + v%4.
    const float lt = xhalf_sum(l);
    int lane_e = threadIdx.x & 63;             // (computed again, as in fp32_pass)
    asm volatile("" : "+v"(lane_e));
    const int row = qrow0 + (lane_e & 31), half = lane_e >> 5;
    if (row >= Wq) return;
    if (a.direct) {
        const float inv = 1.0f / lt;
        const int64_t off = (int64_t)b * a.o_sb + (int64_t)hd * a.o_sh + (pr.qrow_off + row) * a.o_sr;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int d = 32 * db + 8 * g + 4 * half;
                if (DP && d >= a.D) continue;      // column beyond the tensors' head dimension
                f32x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = oacc[db][4 * g + e] * inv;
                if (a.out_bf16) {
                    bf16x4 ob;
#pragma unroll
                    for (int e = 0; e < 4; ++e) ob[e] = (__bf16)o[e];
                    *(bf16x4 *)((__bf16 *)a.O + off + d) = ob;
                } else {
                    *(f32x4 *)((float *)a.O + off + d) = o;
                }
            }
        if (a.lse && half == 0) a.lse[(int64_t)bh * a.W + row] = m * a.scale + logf(lt);
    } else {
        const int64_t slot = pr.slot + a.part0 + (CAUSAL ? 0 : split);
        float *op = a.Opart + (slot * a.W + row) * D;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f32x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = oacc[db][4 * g + e];
                *(f32x4 *)(op + 32 * db + 8 * g + 4 * half) = o;
            }
        if (half == 0) {
            a.Mpart[slot * a.W + row] = m * a.c;
            a.Lpart[slot * a.W + row] = lt;
        }
    }
}

// Waves per SIMD that the registers are cut for: at head dimension 128 the LDS of a two-wave workgroup allows no
// more than one, and the others' 512 threads two; at 64 three, two in the two-wave shape, whose lanes hold more of a tile.
constexpr int f32_waves_per_simd(int D, int NW) { return D == 128 ? (NW == 2 ? 1 : 2) : (NW == 4 ? 3 : 2); }

template <int D, int NW, bool CAUSAL, int DP>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(f32_waves_per_simd(D, NW), 8)))
void attn_f32_kernel(const AttnArgs a)
{
    attn_f32_body<D, NW, CAUSAL, DP>(a, blockIdx.x, gridDim.x);
}

// History partition blocks and window causal blocks of one call in a single launch.
template <int D, int NW, int DP>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(f32_waves_per_simd(D, NW), 8)))
void attn_f32_pair_kernel(const PairArgs f)
{
    // logical index of the window block this workgroup computes, or -1
    int win_block = (int)blockIdx.x < f.n_hist_blocks ? -1 : xcd_remap(blockIdx.x - f.n_hist_blocks, f.n_win_blocks);
    if ((int)blockIdx.x < f.n_hist_blocks) {
        attn_f32_body<D, NW, false, DP>(f.hist, blockIdx.x, f.n_hist_blocks);
        if (f.hist.fuse_window) {
            // the workgroup of partition 0 goes on to the window's causal block of the same rows
            // (causal blocks are numbered from the last query block down)
            const Problem pr = decode_problem<NW * 32, 32, false>(f.hist, xcd_remap(blockIdx.x, f.n_hist_blocks), f.hist.nqb);
            if (pr.split == 0) {
                win_block = pr.bh * f.win.nqb + (f.win.nqb - 1 - pr.qb);
                __syncthreads();      // every wave is done with the history tiles in LDS
            }
        }
    }
    if (win_block >= 0) attn_f32_body<D, NW, true, DP, false>(f.win, win_block, 0);
}

}  // namespace tlin

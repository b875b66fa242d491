// rowsum.hip -- row-sum diagnostics of MXFP4-quantized attention
// probabilities for gfx950 (Sec. 5.5, "Validation of Pre-Normalization
// Quantization", Fig. pnq_rowsum).
//
// The paper measures what direct MXFP4 quantization does to the mass of each
// row of a materialized probability matrix P = softmax(Q K^T / sqrt(d)).  Two
// kernels:
//
//   attn_rows_kernel    S^T on the bf16 matrix cores (V_MFMA_F32_32X32X16_BF16,
//                       fp32 accumulation), then two passes over the keys: the
//                       first for each row's maximum and normalizer, the
//                       second forming p = 2^(t - m) / L in fp32 and either
//                       storing it (a materialized tile of P) or quantizing it
//                       in 32-key blocks in registers (a lane holds a whole
//                       block) and accumulating the row statistics below, so
//                       that whole tensors are diagnosed without writing P;
//   rowsum_diag_kernel  the statistics of a given fp32 P: each row quantized
//                       in 32-entry blocks (optionally pre-scaled by gamma),
//                       reduced to the quantized mass, the unquantized mass,
//                       the contributions Q(x)/gamma - p of zeroed,
//                       saturated, rounded-down, rounded-up and exact
//                       entries, and the entropy -sum p ln p.
//
// Both quantize and sum with the same arithmetic per block (BlockDiag), so on
// the same p they classify every entry identically and their fp64 sums differ
// only in the order of additions.
//
// Row sums.  Each of a row's two lanes walks its share of the keys (every other
// four) with an online maximum and one chain of fp32 additions, and the two are
// merged at the end (row_max).  The order is part of the result: the quantized
// statistics jump where an entry's block maximum crosses 7.25/8 of a power of
// two, so another association of L (4e-5 at 32760 keys, where the chain rounds
// small terms away) moves whole entries of P^, and a row by up to 0.3.  L is
// therefore not divided over workgroups.  p given m and L is: a launch with few
// row tiles of long rows, which would leave most of the chip idle, forms m and L in
// one workgroup per row tile (rows_norm_kernel) and p in one per 8 key tiles
// (rows_write_kernel).  Both ways form m, L and p from the same operations in
// the same order, bit for bit.
//
// What bounds them (one MI355X): the fused diagnostic vector issue (91 % of the
// cycles, 33 vector instructions per entry over the two passes: 40 heads x 4096^2
// entries in 0.73 ms; with every class summed per entry in fp64 behind compares and
// selects 2.55 ms); the materialized rows of 40 x 128 x 32760 entries the
// normalizer in 40 workgroups, one wave per SIMD (0.39 ms, see rows_norm_kernel),
// then the stores of P (0.24 ms, 4.2 TB/s with the keys read; both passes in one
// workgroup per row tile 1.35 ms), and their diagnostic vector issue and its own
// chains (0.19 ms = 3.4 TB/s of P, vector issue in 67 % of the cycles).
#include <cmath>

#include "device_common.h"
#include "launch.h"

namespace mxattn {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kRowsPerWg = 128;  // query rows per workgroup (4 waves x 32)
constexpr int kKeyTile = 128;    // keys staged in LDS per step (32 KiB)
constexpr int kRunTiles = 8;     // key tiles per workgroup of rows_write_kernel
constexpr float kNegBig = -3.0e38f;

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// Copies keys [tile * 128, tile * 128 + 128) of one head straight into LDS
// (buffer loads to LDS; the buffer's range check reads zeros past Nkv).  LDS
// row 64 c + 32 j + r holds, with kBlocks, key 64 c + 32 ((r >> 2) & 1) + 16 j +
// 4 (r >> 3) + (r & 3), so that lane (query, h) finds keys 32 h .. 32 h + 31 of
// the chunk c in the accumulators of its two score products, and otherwise key
// 64 c + 32 j + r.  The 16-byte slot of a row is XOR-ed with the row, so 16
// consecutive rows read at one slot hit 16 bank groups.
template <bool kBlocks>
struct KeyStage {
    const uint8_t* kh;
    int Nkv, wave;
    uint32_t off;  // lane offset of the wave's first row

    __device__ __forceinline__ KeyStage(const uint16_t* k, int64_t bh, int nkv, int wave_, int lane)
        : kh(reinterpret_cast<const uint8_t*>(k) + bh * (int64_t)nkv * 256), Nkv(nkv), wave(wave_) {
        const int x = lane >> 4;  // row of a load's four
        off = (uint32_t)((64 * (wave >> 1) + (kBlocks ? 16 : 32) * (wave & 1) + x) * 256 + ((lane & 15) ^ x) * 16);
    }

    // wave w copies LDS rows 32 w .. 32 w + 31 (A-rows of product (c, j) = (w >> 1, w & 1)), four per
    // load: row 4 i + x is key 32 (i & 1) + 4 (i >> 1) + x or 4 i + x further on, its slots XOR-ed by 4 (i & 3) + x
    __device__ __forceinline__ void load(uint8_t* lds, int tile_) const {
        const int tile = __builtin_amdgcn_readfirstlane(tile_);
        const int64_t left = ((int64_t)Nkv - (int64_t)tile * kKeyTile) * 256;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(kh + (int64_t)tile * kKeyTile * 256), 0, (int)(left < kKeyTile * 256 ? left : kKeyTile * 256),
            0x00020000);
        uint32_t base = off;
        asm volatile("" : "+v"(base));  // the eight offsets are formed here, not kept in registers
#pragma unroll
        for (int i = 0; i < 8; i++)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs, (lds_ptr_t)(lds + wave * 8192 + i * 1024), 16,
                (int)((base ^ (64 * (i & 3))) + (kBlocks ? 32 * (i & 1) + 4 * (i >> 1) : 4 * i) * 256), 0, 0, 0);
    }
};

// S^T of LDS rows 32 j .. 32 j + 31 (as A rows) x this wave's 32 queries (as B
// columns): lane (col, h) supplies row 32 j + col and query col, each with
// channels 16 s + 8 h .. + 7 per 16-channel step s.
__device__ __forceinline__ v16f scores_t(const bf16x8* qb, const uint8_t* lds, int j, int col, int h) {
    v16f acc;
#pragma unroll
    for (int i = 0; i < 16; i++) acc[i] = 0.f;
    const uint8_t* row = lds + (32 * j + col) * 256;
#pragma unroll
    for (int s = 0; s < 8; s++) {
        const bf16x8 ka =
            __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(row + (((2 * s + h) ^ (col & 15)) * 16)));
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qb[s], acc, 0, 0, 0);
    }
    return acc;
}

// The scores of a tile: sv[c][j][i] is key 64 c + 32 h + 16 j + i with kBlocks,
// otherwise 64 c + 32 j + 8 (i >> 2) + 4 h + (i & 3).
typedef v16f TileScores[2][2];

// -inf past the end of the sequence: per score the sign of (last - its key)
// selects the bits of -inf, so that the compares are not hoisted and held as 64
// condition masks in scalar registers, which spilled (P of 26 rows over 7 keys 8.3
// us with them, 7.0 so).
template <bool kBlocks>
__device__ __forceinline__ void mask_tail(int t, int Nkv, int h, TileScores& sv) {
    if ((t + 1) * kKeyTile > Nkv) {
        const int last = Nkv - t * kKeyTile - (kBlocks ? 32 : 4) * h - 1;
#pragma unroll
        for (int c = 0; c < 2; c++)
#pragma unroll
            for (int j = 0; j < 2; j++)
#pragma unroll
                for (int i = 0; i < 16; i++) {
                    const int past = (last - (64 * c + (kBlocks ? 16 * j + i : 32 * j + 8 * (i >> 2) + (i & 3)))) >> 31;
                    const float s = sv[c][j][i];  // (a bit cast of a vector's element takes element 0)
                    const int b = __builtin_bit_cast(int, s);
                    sv[c][j][i] = __builtin_bit_cast(float, (past & (int)0xFF800000u) | (~past & b));
                }
    }
}

template <bool kBlocks>
__device__ __forceinline__ void tile_scores(const bf16x8* qb, const uint8_t* lds, int t, int Nkv, int col, int h,
                                            TileScores& sv) {
#pragma unroll
    for (int c = 0; c < 2; c++)
#pragma unroll
        for (int j = 0; j < 2; j++) sv[c][j] = scores_t(qb, lds, 2 * c + j, col, h);
    mask_tail<kBlocks>(t, Nkv, h, sv);
}

// Calls work(t, scores, landed) for the tiles t0 .. t1 - 1.  The next tile is
// copied into LDS while the work runs on this one's scores, which by then are
// in registers; the work calls landed() once, where the copy should be through
// (vmcnt counts stores too: before its stores, so that they are not waited for
// at the next tile).
template <bool kBlocks, typename Work>
__device__ __forceinline__ void for_tiles(const bf16x8* qb, const KeyStage<kBlocks>& ks, uint8_t* lds, int t0, int t1, int col,
                                          int h, const Work& work) {
    auto landed = [] { __builtin_amdgcn_s_waitcnt(0); };
    ks.load(lds, t0);
    landed();
    for (int t = t0; t < t1; t++) {
        __syncthreads();  // tile t landed everywhere
        TileScores sv;
        tile_scores<kBlocks>(qb, lds, t, ks.Nkv, col, h, sv);
        __syncthreads();  // and was read everywhere
        if (t + 1 < t1) ks.load(lds, t + 1);
        work(t, sv, landed);
    }
}

// Query operand (B columns) of local query row lr (clamped to the last row).
__device__ __forceinline__ void load_queries(const SoftmaxRowsArgs& a, int64_t bh, int lr, int h, bf16x8 (&qb)[8]) {
    const uint4* qrow = reinterpret_cast<const uint4*>(a.q) + (bh * a.Nq + a.row0 + min(lr, a.rows - 1)) * 16;
#pragma unroll
    for (int s = 0; s < 8; s++) qb[s] = __builtin_bit_cast(bf16x8, qrow[2 * s + h]);
}

// Scores are never NaN: the NaN-propagating maximum fuses into the 3-input form.
__device__ __forceinline__ float max2f(float a, float b) { return __builtin_elementwise_maximum(a, b); }

// A row's maximum m of t = c s, and 1 / L of its two lanes, which merge their
// sums each with its own first: entry (key >> 2) & 1 belongs to that lane's keys.
struct RowNorm {
    float m, inv[2];
};

// fp32(s c), not fused into a later addition.
__device__ __forceinline__ float rounded_product(float s, float c) {
#pragma clang fp contract(off)
    return s * c;
}

// A lane's running maximum and sum.  A tile updates the maximum (grow) and then
// adds its 64 entries in key order (add).
struct LaneNorm {
    float m = kNegBig, l = 0.f;

    __device__ __forceinline__ void grow(const TileScores& sv, float c) {
        float tm = sv[0][0][0];
#pragma unroll
        for (int i = 1; i < 63; i += 2)
            tm = max2f(max2f(tm, sv[i >> 5][(i >> 4) & 1][i & 15]), sv[(i + 1) >> 5][((i + 1) >> 4) & 1][(i + 1) & 15]);
        tm = max2f(tm, sv[1][1][15]);
        // (a lane whose keys are all past the end keeps m: c tm = -inf)
        const float mn = max2f(m, rounded_product(tm, c));
        l = l * __builtin_amdgcn_exp2f(m - mn);
        m = mn;
    }
    __device__ __forceinline__ void add(float s, float c) {
        l += __builtin_amdgcn_exp2f(rounded_product(s, c) - m);
    }
    __device__ __forceinline__ RowNorm row(int h) const {
        const float mo = __shfl_xor(m, 32);
        const float lo = __shfl_xor(l, 32);
        const float mn = max2f(m, mo);
        const float inv = 1.0f / (l * __builtin_amdgcn_exp2f(m - mn) + lo * __builtin_amdgcn_exp2f(mo - mn));
        const float other = __shfl_xor(inv, 32);
        return {mn, {h == 0 ? inv : other, h == 0 ? other : inv}};
    }
};

__device__ __forceinline__ RowNorm row_norm(const SoftmaxRowsArgs& a, int64_t bh, const bf16x8* qb, uint8_t* lds,
                                            int wave, int lane, int col, int h) {
    const KeyStage<false> ks(a.k, bh, a.Nkv, wave, lane);
    LaneNorm n;
    for_tiles<false>(qb, ks, lds, 0, (a.Nkv + kKeyTile - 1) / kKeyTile, col, h, [&](int, TileScores& sv, auto landed) {
        n.grow(sv, a.c);
#pragma unroll
        for (int i = 0; i < 64; i++) n.add(sv[i >> 5][(i >> 4) & 1][i & 15], a.c);
        landed();
    });
    return n.row(h);
}

// log2 of a positive fp32.  The hardware logarithm takes what is below the normal
// range as zero: a subnormal is scaled by 2^32 into it first.  Zero gives a finite
// value, so p log2 p is 0 for p = 0.
constexpr float kMinNormal = 1.17549435e-38f;
__device__ __forceinline__ float log2_normal(float p) {
    // (of bit patterns: the maximum of floats would quiet its operand first)
    return __builtin_amdgcn_logf(__builtin_bit_cast(
        float, max(__builtin_bit_cast(uint32_t, p), __builtin_bit_cast(uint32_t, kMinNormal))));
}
__device__ __forceinline__ float log2_full(float p) {
    return p < kMinNormal ? log2_normal(p * 4294967296.0f) - 32.0f : log2_normal(p);
}

// sum += p log2 p of entries i .. i + 3, p >= 0.  Scaling every entry costs the whole
// diagnostic 5 to 8 %; so one class test per entry and a branch per four, which
// costs 40 heads x 4096 tokens nothing with or without outlier channels (704 us),
// and where every wave has subnormals in most fours (scores of a standard
// deviation of 36 bits) 5 %.
template <int kN>
__device__ __forceinline__ void add_plog(double& sum, const float (&p)[kN], int i) {
    constexpr int kSubnormal = 0x80;  // class mask of positive subnormals
    bool low = false;
#pragma unroll
    for (int e = 0; e < 4; e++) low |= __builtin_amdgcn_classf(p[i + e], kSubnormal);
    if (__any(low)) {
#pragma unroll
        for (int e = 0; e < 4; e++) sum += (double)(p[i + e] * log2_full(p[i + e]));
    } else {
#pragma unroll
        for (int e = 0; e < 4; e++) sum += (double)(p[i + e] * log2_normal(p[i + e]));
    }
}

// Shared-scale exponent of a block from the bits of its largest magnitude.
template <int kRule>
__device__ __forceinline__ int block_exponent_f32(uint32_t mb) {
    return mb == 0 ? 0 : scale_exponent_f32<kRule>(mb);
}

// fp32 to unsigned, fractions dropped and negatives 0 (the conversion clamps).
__device__ __forceinline__ uint32_t cvt_u32(float x) {
    uint32_t r;
    asm("v_cvt_u32_f32_e32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}
__device__ __forceinline__ uint32_t cvt_u32_neg(float x) {
    uint32_t r;
    asm("v_cvt_u32_f32_e64 %0, -%1" : "=v"(r) : "v"(x));
    return r;
}

// Row statistics of a lane, added up block by block (see mxattn.h).
//
// kGamma = kGammaOne, kGammaPow2: gamma is 1, the usual one, or a power of two
// up to 2^16, so that x = gamma p is exact.  Then an entry's contribution is (r - x / sigma) sigma /
// gamma exactly, r its E2M1 value, and with r > 0 (so x / sigma >= 1/4) the
// difference is a multiple of 2^-25 of at most 2: the up, down and saturated
// entries of a block add up exactly in 32-bit integers (at most 32 * 2 * 2^25),
// one fp64 product and sum per block each; only zeroed entries and the entropy
// take an fp64 sum per entry.  Otherwise every entry's terms are formed and
// added in fp64, as they are where an entry is not a finite number >= 0
// (add_unusual).
enum Gamma { kGammaOne = 0, kGammaPow2 = 1, kGammaAny = 2 };
template <int kGamma>
struct RowStats {
    static constexpr bool kPow2 = kGamma != kGammaAny;
    // kPow2: sum Q, up, down, saturated (the last two positive), zeroed p, p log2 p;
    // otherwise the eight statistics, the last as sum p log2 p
    static constexpr int kSums = kPow2 ? 6 : 8, kEntropy = kSums - 1;
    double v[kSums];
    bool nan = false;  // kPow2: a p is NaN (the mass and the exact entries' sum are, then)
};

// Adds this lane's kN entries of a block whose largest x has the bits mb.
// (x is formed again from p where it is needed: registers.)
template <int kRule, int kGamma, int kN>
__device__ __forceinline__ void add_block(RowStats<kGamma>& st, const float (&p)[kN], float gamma, uint32_t mb,
                                          double g) {
    if constexpr (kGamma == kGammaOne) gamma = 1.0f;
    const int ex = block_exponent_f32<kRule>(mb);
    const float sf = e8m0_as_f32((uint32_t)(ex + 127));
    if constexpr (kGamma != kGammaAny) {
        constexpr float k25 = 33554432.0f;  // 2^25
        uint32_t up = 0, down = 0, sat = 0;
        float rsum = 0.f;  // multiples of 2^24 below 2^33: exact
#pragma unroll
        for (int i = 0; i < kN; i += 2) {
            // (forms the sums entry by entry, no instruction emitted: with the
            // work of the whole block interleaved it spills)
            if (i % 4 == 0) {
                asm volatile("" : "+v"(up), "+v"(down), "+v"(sat), "+v"(rsum), "+v"(st.v[4]), "+v"(st.v[5]));
                __builtin_amdgcn_sched_barrier(0);
            }
            const float x[2] = {gamma * p[i], gamma * p[i + 1]};
            const uint32_t c = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, x[0], x[1], sf, 0);
            const auto r = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c, k25, 0);
            rsum += r[0] + r[1];
#pragma unroll
            for (int e = 0; e < 2; e++) {
                const float xs = __builtin_ldexpf(x[e], 25 - ex);
                const float d = r[e] - xs;
                const bool zero = r[e] == 0.f;
                up += cvt_u32(d);
                // (the operand is selected: a conversion under a condition is a branch)
                down += cvt_u32_neg(zero ? 0.f : d);
                sat += cvt_u32(xs - 6.0f * k25);
                st.v[4] += (double)(zero ? p[i + e] : 0.f);
            }
            if (i % 4 == 2) add_plog(st.v[5], p, i - 2);
        }
        // sigma / gamma 2^-25
        const double s = __builtin_bit_cast(double, (uint64_t)(ex + 1023 - 25) << 52) * g;
        st.v[0] += s * (double)rsum;
        st.v[1] += s * (double)up;
        st.v[2] += s * (double)(down - sat);
        st.v[3] += s * (double)sat;
    } else {
        const float inv = __builtin_bit_cast(float, (uint32_t)(127 - ex) << 23);  // 2^-ex, normal
        const double sig = __builtin_bit_cast(double, (uint64_t)(ex + 1023) << 52);
#pragma unroll
        for (int i = 0; i < kN; i += 2) {
            if (i % 8 == 0) __builtin_amdgcn_sched_barrier(0);
            const float x[2] = {gamma * p[i], gamma * p[i + 1]};
            const uint32_t c = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, x[0], x[1], sf, 0);
            const auto r = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c, 1.0f, 0);
#pragma unroll
            for (int e = 0; e < 2; e++) {
                const float xs = x[e] * inv;  // exact
                const double pd = (double)p[i + e];
                const double qv = (double)r[e] * sig * g;
                const double cj = qv - pd;
                const bool zer = p[i + e] > 0.f && r[e] == 0.f;
                const bool sat = !zer && xs > 6.0f;
                const bool dn = !zer && !sat && r[e] < xs;
                const bool up = !zer && !sat && r[e] > xs;
                const bool eq = !zer && !sat && !dn && !up;
                st.v[0] += qv;
                st.v[1] += pd;
                st.v[2] += zer ? cj : 0.0;
                st.v[3] += sat ? cj : 0.0;
                st.v[4] += dn ? cj : 0.0;
                st.v[5] += up ? cj : 0.0;
                st.v[6] += eq ? cj : 0.0;
            }
            if (i % 4 == 2) add_plog(st.v[7], p, i - 2);
        }
    }
}

// The same for one entry of any block, also of one with an entry that is infinite
// (x may be although p is not), NaN or negative: its terms from their definition.
template <int kRule, int kGamma>
__device__ __forceinline__ void add_unusual(RowStats<kGamma>& st, float p, float gamma, uint32_t mb, double g) {
    const int ex = block_exponent_f32<kRule>(mb);
    const float sf = e8m0_as_f32((uint32_t)(ex + 127));
    const float inv = __builtin_bit_cast(float, (uint32_t)(127 - ex) << 23);
    const double sig = __builtin_bit_cast(double, (uint64_t)(ex + 1023) << 52);
    const uint32_t c = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, gamma * p, 0.f, sf, 0);
    const float r = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c, 1.0f, 0)[0];
    const float xs = gamma * p * inv;
    const double qv = (double)r * sig * g;
    const double cj = qv - (double)p;
    const bool zer = p > 0.f && r == 0.f;
    const bool sat = !zer && xs > 6.0f;
    const bool dn = !zer && !sat && r < xs;
    const bool up = !zer && !sat && r > xs;
    const bool eq = !zer && !sat && !dn && !up;
    const double plog = p > 0.f ? (double)(p * log2_full(p)) : 0.0;
    st.v[0] += qv;
    if constexpr (kGamma != kGammaAny) {
        st.v[1] += up ? cj : 0.0;
        st.v[2] -= dn ? cj : 0.0;
        st.v[3] -= sat ? cj : 0.0;
        st.v[4] -= zer ? cj : 0.0;
        st.v[5] += plog;
        st.nan |= p != p;
    } else {
        st.v[1] += (double)p;
        st.v[2] += zer ? cj : 0.0;
        st.v[3] += sat ? cj : 0.0;
        st.v[4] += dn ? cj : 0.0;
        st.v[5] += up ? cj : 0.0;
        st.v[6] += eq ? cj : 0.0;
        st.v[7] += plog;
    }
}

// The eight statistics of a row from its sums over all lanes.
template <int kGamma>
__device__ __forceinline__ void write_stats(double* dst, const RowStats<kGamma>& st) {
    constexpr double kMinusLn2 = -0.6931471805599453;  // -sum p ln p = -ln 2 sum p log2 p
    if constexpr (kGamma != kGammaAny) {
        const double R = st.v[0], up = st.v[1], down = st.v[2], sat = st.v[3], z = st.v[4];
        const double eq = st.nan ? __builtin_nan("") : 0.0;
        dst[0] = R;
        dst[1] = R + z + ((down + sat) - up) - eq;  // the mass: what was quantized less what it gained
        dst[2] = 0.0 - z;
        dst[3] = 0.0 - sat;
        dst[4] = 0.0 - down;
        dst[5] = up;
        dst[6] = eq;
        dst[7] = kMinusLn2 * st.v[5];
    } else {
#pragma unroll
        for (int i = 0; i < 7; i++) dst[i] = st.v[i];
        dst[7] = kMinusLn2 * st.v[7];
    }
}

// A wave's place: its 32 query rows of a row tile.
struct RowPlace {
    int64_t bh;
    int qt, wave, lane, col, h, lr;
    bool ok;
    __device__ __forceinline__ RowPlace(const SoftmaxRowsArgs& a, int64_t tile) {
        bh = tile / a.qtiles;
        qt = (int)(tile - bh * a.qtiles);
        wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        lane = threadIdx.x & 63;
        col = lane & 31;
        h = lane >> 5;
        lr = qt * kRowsPerWg + 32 * wave + col;  // this lane's local query row
        ok = lr < a.rows;
    }
    __device__ __forceinline__ float* prow(const SoftmaxRowsArgs& a) const {
        return a.p + (bh * a.rows + lr) * (int64_t)a.ld;
    }
};

// p of the staged tile's entries: stored (kOut = kRowsStoreP) or diagnosed.
// A lane holds 32 consecutive entries of one row, so stored straight from
// registers every store instruction would touch 64 cache lines 16 bytes each
// (2.2 TB/s written); 16 rows x 64 entries at a time go through the wave's
// 4 KiB of `out` (slots of a row XOR-ed by the row) and leave as four 256-byte
// row pieces per instruction.
constexpr int kOutBytes = 4096;  // per wave
template <int kOut, int kGamma, typename Landed>
__device__ __forceinline__ void emit_tile(const SoftmaxRowsArgs& a, const RowPlace& w, TileScores& sv, uint8_t* out,
                                          int t, const RowNorm& r, RowStats<kGamma>& st, const Landed& landed) {
    if constexpr (kOut == kRowsStoreP) {
#pragma unroll
        for (int c = 0; c < 2; c++)
#pragma unroll
            for (int j = 0; j < 2; j++)
#pragma unroll
                for (int i = 0; i < 16; i++)
                    sv[c][j][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[c][j][i], a.c, -r.m)) * r.inv[(i >> 2) & 1];
        landed();
        const int row0 = w.qt * kRowsPerWg + 32 * w.wave;
#pragma unroll
        for (int c = 0; c < 2; c++)
#pragma unroll
            for (int pass = 0; pass < 2; pass++) {
                if (row0 + 16 * pass >= a.rows || t * kKeyTile + 64 * c >= a.Nkv) continue;  // nothing to store
                if ((w.col >> 4) == pass) {
                    const int row = w.col & 15;
#pragma unroll
                    for (int n = 0; n < 32; n += 4) {
                        const v16f& p = sv[c][n >> 4];
                        *reinterpret_cast<float4*>(out + row * 256 + (((8 * w.h + n / 4) ^ row) * 16)) =
                            make_float4(p[n & 15], p[(n & 15) + 1], p[(n & 15) + 2], p[(n & 15) + 3]);
                    }
                }
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const int row = 4 * k + (w.lane >> 4), slot = w.lane & 15;
                    const float4 v = *reinterpret_cast<const float4*>(out + row * 256 + ((slot ^ row) * 16));
                    const int lr = row0 + 16 * pass + row, key = t * kKeyTile + 64 * c + 4 * slot;
                    if (lr < a.rows && key < a.Nkv)
                        *reinterpret_cast<float4*>(a.p + (w.bh * a.rows + lr) * (int64_t)a.ld + key) = v;
                }
                __builtin_amdgcn_wave_barrier();
            }
    } else {
        constexpr int kRule = kOut == kRowsDiagUos ? kRuleUos : kRuleOcp;
#pragma unroll
        for (int c = 0; c < 2; c++) {
            float p[32], mx = 0.f;  // gamma > 0: the largest x is gamma times the largest p
#pragma unroll
            for (int n = 0; n < 32; n++)
                p[n] = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[c][n >> 4][n & 15], a.c, -r.m)) * r.inv[(n >> 2) & 1];
#pragma unroll
            for (int n = 0; n < 32; n += 2) mx = max2f(max2f(mx, p[n]), p[n + 1]);
            add_block<kRule, kGamma, 32>(st, p, a.gamma, __builtin_bit_cast(uint32_t, a.gamma * __builtin_fabsf(mx)),
                                         a.g);
        }
        landed();
    }
}

// The entries between the last key and the next multiple of 4 are 0, since the
// score of a key past the end is -inf; but NaN in a row whose maximum or normalizer
// is not finite, where 0 is stored over them.
__device__ __forceinline__ void clear_past_end(const SoftmaxRowsArgs& a, const RowPlace& w, const RowNorm& r) {
    if ((a.Nkv & 3) == 0 || r.inv[0] < INFINITY || !w.ok || w.h != 0) return;
    __builtin_amdgcn_s_waitcnt(0);  // the wave's stores to the same entries
    for (int64_t j = a.Nkv; (j & 3) != 0; j++) w.prow(a)[j] = 0.f;
}

// Rows of attention probabilities, one workgroup per 128 query rows: pass 1
// the row maximum m and normalizer L, pass 2 p.
template <int kOut, int kGamma>
__global__ __launch_bounds__(256, 3) void attn_rows_kernel(SoftmaxRowsArgs a) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[kKeyTile * 256];
    __shared__ __attribute__((aligned(16))) uint8_t out[kOut == kRowsStoreP ? 4 * kOutBytes : 16];
    const RowPlace w(a, blockIdx.x);
    bf16x8 qb[8];
    load_queries(a, w.bh, w.lr, w.h, qb);
    const RowNorm r = row_norm(a, w.bh, qb, lds, w.wave, w.lane, w.col, w.h);

    const KeyStage<true> ks(a.k, w.bh, a.Nkv, w.wave, w.lane);
    const int tiles = (a.Nkv + kKeyTile - 1) / kKeyTile;
    RowStats<kGamma> st;
#pragma unroll
    for (int i = 0; i < RowStats<kGamma>::kSums; i++) st.v[i] = 0.0;
    for_tiles<true>(qb, ks, lds, 0, tiles, w.col, w.h, [&](int t, TileScores& sv, auto landed) {
        emit_tile<kOut, kGamma>(a, w, sv, out + (kOut == kRowsStoreP ? w.wave * kOutBytes : 0), t, r, st, landed);
    });
    if constexpr (kOut == kRowsStoreP) {
        clear_past_end(a, w, r);
    } else {
#pragma unroll
        for (int i = 0; i < RowStats<kGamma>::kSums; i++) st.v[i] += __shfl_xor(st.v[i], 32);
        // p is at most 1, or NaN in the whole row: a NaN is quantized to +-6 at the
        // scale 2^126, is in no class but "exact" and has no entropy
        if (!(r.inv[0] < INFINITY)) {
            st.v[0] = __builtin_copysign((double)a.Nkv * (6.0 * 0x1p126 * a.g), st.v[0]);
            st.v[RowStats<kGamma>::kEntropy] = 0.0;
            st.nan = true;
        }
        if (w.ok && w.h == 0) write_stats(a.stats + (w.bh * a.Nq + a.row0 + w.lr) * 8, st);
    }
}

// Few row tiles: m and L in one workgroup per row tile, p in one per (row tile,
// run of kRunTiles key tiles).  Every run's (m, 1 / L) goes to the first three
// of the run's own entries of the row (p has room for at least four there); a
// workgroup of rows_write_kernel reads those of its own run before it overwrites
// them, so no other workspace is needed.
//
// One wave per SIMD: rows_norm_kernel keeps two tiles in LDS and the next in
// flight.  40 heads x 128 rows x 32760 keys 390 us; with one tile in LDS 475 us.
// The loop below issues a product of tile t + 1 after every two entries of tile t,
// but the compiler moves the exponentials and additions behind the branch of the
// ragged tile, so a tile's 32 products (1030 cycles), 65 exponentials and 64
// additions still follow one another: 3780 cycles per tile, 1890 of them vector
// issue.
__global__ __launch_bounds__(256) void rows_norm_kernel(SoftmaxRowsArgs a) {
    // (two arrays: reads of one do not wait for copies into the other)
    __shared__ __attribute__((aligned(16))) uint8_t lds0[kKeyTile * 256];
    __shared__ __attribute__((aligned(16))) uint8_t lds1[kKeyTile * 256];
    const RowPlace w(a, blockIdx.x);
    bf16x8 qb[8];
    load_queries(a, w.bh, w.lr, w.h, qb);
    const KeyStage<false> ks(a.k, w.bh, a.Nkv, w.wave, w.lane);
    const int tiles = (a.Nkv + kKeyTile - 1) / kKeyTile;
    LaneNorm n;

    // tile t, its scores in sv and its keys in cur; leaves tile t + 1's scores, from nxt
    auto step = [&](int t, uint8_t* cur, const uint8_t* nxt, TileScores& sv, TileScores& next) {
        __syncthreads();  // tile t was read everywhere, tile t + 1 landed everywhere
        if (t + 2 < tiles) ks.load(cur, t + 2);
        n.grow(sv, a.c);
#pragma unroll
        for (int p = 0; p < 4; p++)
#pragma unroll
            for (int i = 0; i < 16; i++) next[p >> 1][p & 1][i] = 0.f;
        auto operand = [&](int k) {  // key rows 32 (k & 3) + col, channels of step k >> 2
            return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(
                nxt + (32 * (k & 3) + w.col) * 256 + (((2 * (k >> 2) + w.h) ^ (w.col & 15)) * 16)));
        };
        bf16x8 ka[4];
#pragma unroll
        for (int k = 0; k < 4; k++) ka[k] = operand(k);
#pragma unroll
        for (int k = 0; k < 32; k++) {
            v16f& acc = next[(k >> 1) & 1][k & 1];
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[k & 3], qb[k >> 2], acc, 0, 0, 0);
            if (k + 4 < 32) ka[k & 3] = operand(k + 4);
#pragma unroll
            for (int e = 2 * k; e < 2 * k + 2; e++) n.add(sv[e >> 5][(e >> 4) & 1][e & 15], a.c);
            __builtin_amdgcn_sched_barrier(0);
        }
        mask_tail<false>(t + 1, a.Nkv, w.h, next);
        __builtin_amdgcn_s_waitcnt(0);
    };
    ks.load(lds0, 0);
    if (tiles > 1) ks.load(lds1, 1);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    TileScores s0, s1;
    tile_scores<false>(qb, lds0, 0, a.Nkv, w.col, w.h, s0);
    // (after the last tile the scores of whatever is staged are formed and dropped)
    for (int t = 0; t < tiles; t += 2) {
        step(t, lds0, lds1, s0, s1);
        if (t + 1 < tiles) step(t + 1, lds1, lds0, s1, s0);
    }
    const RowNorm r = n.row(w.h);
    if (w.ok)
        for (int run = w.h; run < a.runs; run += 2)
            *reinterpret_cast<float4*>(w.prow(a) + (int64_t)run * (kRunTiles * kKeyTile)) =
                make_float4(r.m, r.inv[0], r.inv[1], 0.f);
}

__global__ __launch_bounds__(256, 3) void rows_write_kernel(SoftmaxRowsArgs a) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[kKeyTile * 256];
    __shared__ __attribute__((aligned(16))) uint8_t out[4 * kOutBytes];
    const RowPlace w(a, blockIdx.x / a.runs);
    const int run = blockIdx.x % a.runs;
    bf16x8 qb[8];
    load_queries(a, w.bh, w.lr, w.h, qb);
    const KeyStage<true> ks(a.k, w.bh, a.Nkv, w.wave, w.lane);
    RowNorm r = {0.f, {0.f, 0.f}};
    if (w.ok) {
        const float4 v = *reinterpret_cast<const float4*>(w.prow(a) + (int64_t)run * (kRunTiles * kKeyTile));
        r = {v.x, {v.y, v.z}};
    }
    RowStats<kGammaOne> st;
    const int t1 = min((a.Nkv + kKeyTile - 1) / kKeyTile, (run + 1) * kRunTiles);
    // (the wait for the first tile is also one for the row's values)
    for_tiles<true>(qb, ks, lds, run * kRunTiles, t1, w.col, w.h, [&](int t, TileScores& sv, auto landed) {
        emit_tile<kRowsStoreP, kGammaOne>(a, w, sv, out + w.wave * kOutBytes, t, r, st, landed);
    });
    if (run == a.runs - 1) clear_past_end(a, w, r);
}

// One workgroup per row; 4 lanes per 32-entry block, 8 entries per lane.
template <int kRule, int kGamma>
__global__ __launch_bounds__(256) void rowsum_diag_kernel(RowsumDiagArgs a) {
    constexpr int kSums = RowStats<kGamma>::kSums;
    __shared__ double red[4][kSums];
    __shared__ int flags[4];
    const int64_t r = blockIdx.x;
    const float* prow = a.p + r * a.ld;
    RowStats<kGamma> st;
#pragma unroll
    for (int i = 0; i < kSums; i++) st.v[i] = 0.0;
    const float gamma = kGamma == kGammaOne ? 1.0f : a.gamma;

    auto quad_max = [](uint32_t mb) {
        mb = max(mb, (uint32_t)__builtin_amdgcn_mov_dpp((int)mb, 0xB1, 0xF, 0xF, false));  // lane ^ 1
        return max(mb, (uint32_t)__builtin_amdgcn_mov_dpp((int)mb, 0x4E, 0xF, 0xF, false));  // lane ^ 2
    };
    uint32_t worst = 0;
    auto block = [&](const float (&p)[8]) {
        // as unsigned numbers, the bits of finite x >= 0 lie below those of all others
        uint32_t mb = 0;
#pragma unroll
        for (int e = 0; e < 8; e++) mb = max(mb, __builtin_bit_cast(uint32_t, gamma * p[e]));
        mb = quad_max(mb);
        worst = max(worst, mb);
        add_block<kRule, kGamma, 8>(st, p, a.gamma, mb, a.g);
    };
    // entries 8 t .. 8 t + 7 of each whole step of 2048, the next step's
    // fetched before a step is worked on
    const int64_t whole = a.N / 2048 * 2048;
    const float4* src = reinterpret_cast<const float4*>(prow) + 2 * threadIdx.x;
    float4 n0 = make_float4(0.f, 0.f, 0.f, 0.f), n1 = n0;
    if (whole > 0) {
        n0 = src[0];
        n1 = src[1];
    }
    for (int64_t base = 0; base < whole; base += 2048) {
        const float p[8] = {n0.x, n0.y, n0.z, n0.w, n1.x, n1.y, n1.z, n1.w};
        const int64_t nb = base + 2048 < whole ? base + 2048 : base;  // the last step reads itself again
        n0 = src[nb / 4];
        n1 = src[nb / 4 + 1];
        block(p);
    }
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (whole + 512 * wave < a.N) {  // the rest of the row, zeros past its end, in the waves that it reaches
        const int64_t j = whole + 8 * threadIdx.x;
        float p[8];
#pragma unroll
        for (int e = 0; e < 8; e += 4) {
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (j + e < a.N) v = *reinterpret_cast<const float4*>(prow + j + e);  // ld % 4 == 0
            p[e] = v.x;
            p[e + 1] = j + e + 1 < a.N ? v.y : 0.f;
            p[e + 2] = j + e + 2 < a.N ? v.z : 0.f;
            p[e + 3] = j + e + 3 < a.N ? v.w : 0.f;
        }
        block(p);
    }
    auto reduce = [&](bool flag) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
            for (int i = 0; i < kSums; i++) st.v[i] += __shfl_xor(st.v[i], off);
        flag = __any(flag);
        if ((threadIdx.x & 63) == 0) {
#pragma unroll
            for (int i = 0; i < kSums; i++) red[wave][i] = st.v[i];
            flags[wave] = flag;
        }
        __syncthreads();
        return (flags[0] | flags[1] | flags[2] | flags[3]) != 0;
    };
    // a row with an entry that is not a finite x >= 0 is formed again from the
    // definitions, 8 entries of a lane one at a time
    if (reduce(worst >= 0x7F800000u)) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kSums; i++) st.v[i] = 0.0;
        for (int64_t base = 0; base < a.N; base += 2048) {
            const int64_t j = base + 8 * threadIdx.x;
            uint32_t mb = 0;
#pragma unroll 1
            for (int64_t i = j; i < j + 8 && i < a.N; i++)
                mb = max(mb, __builtin_bit_cast(uint32_t, gamma * prow[i]) & 0x7FFFFFFFu);
            mb = quad_max(mb);
#pragma unroll 1
            for (int64_t i = j; i < j + 8 && i < a.N; i++) add_unusual<kRule, kGamma>(st, prow[i], a.gamma, mb, a.g);
        }
        st.nan = reduce(st.nan);
    }
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < kSums; i++) st.v[i] = (red[0][i] + red[1][i]) + (red[2][i] + red[3][i]);
        const int64_t head = r / a.rows_per_head, lr = r % a.rows_per_head;
        write_stats(a.stats + ((head * a.out_rows_per_head) + a.out_row0 + lr) * 8, st);
    }
}

// The arithmetic that gamma allows (RowStats).
int gamma_kind(float gamma) {
    int e;
    if (gamma == 1.0f) return kGammaOne;
    return gamma > 1.0f && gamma <= 65536.0f && std::frexp(gamma, &e) == 0.5f ? kGammaPow2 : kGammaAny;
}

}  // namespace

template <int kGamma>
static void launch_attn_diag(const SoftmaxRowsArgs& a, int out, dim3 grid, hipStream_t stream) {
    if (out == kRowsDiagUos)
        attn_rows_kernel<kRowsDiagUos, kGamma><<<grid, 256, 0, stream>>>(a);
    else
        attn_rows_kernel<kRowsDiagOcp, kGamma><<<grid, 256, 0, stream>>>(a);
}

// Whether m and L are formed apart from p (rows_norm_kernel, rows_write_kernel)
// or in one launch (attn_rows_kernel, three workgroups per CU).  A CU holds one
// workgroup of rows_norm_kernel (316 VGPRs), so beyond 256 row tiles it takes a
// second round and two launches never gain; with fewer, what the second launch and
// the second read of the keys cost is repaid by p on the whole chip the sooner the
// fewer tiles there are and the longer the rows.  Measured, one launch against
// two, us:
//   tiles   keys 1300      1600       2048       3000       4096       8192       32760
//     40     54 |  52   63 |  54   77 |  58  114 |  71  149 |  83  292 | 139  1348 |  660
//    128     57 |  56   66 |  59   79 |  63  116 |  95  156 | 139  338 | 254  1590 | 1146
//    160     58 |  63   67 |  66   80 |  74  119 | 107  167 | 157  378 | 294  1759 | 1352
//    200     60 |  68   68 |  68   82 |  80  144 | 136  185 | 191  410 | 348  1961 | 1582
//    256     65 |  76   72 |  73   90 |  91  167 | 181  211 | 204  436 | 407  2180 | 1872
//    280     83 | 109   88 | 108  114 | 148  200 | 238  237 | 268  491 | 514  2417 | 2388
//    400     97 | 133  106 | 139  136 | 190  253 | 301  279 | 350  577 | 662  2867 | 3098
// and from 512 tiles on two launches are 10 to 50 % slower at every length.
static bool apart(int64_t tiles, int Nkv) {
    if (tiles <= 128) return Nkv >= 1280;
    if (tiles <= 192) return Nkv >= 2048;
    return tiles <= 256 && Nkv >= 4096;
}

hipError_t launch_attn_rows(const SoftmaxRowsArgs& args, int64_t BH, int out, hipStream_t stream) {
    SoftmaxRowsArgs a = args;
    a.qtiles = (a.rows + kRowsPerWg - 1) / kRowsPerWg;
    a.c = 0.12751743082459868f;  // fp32(log2(e) / sqrt(128))
    a.runs = (a.Nkv + kRunTiles * kKeyTile - 1) / (kRunTiles * kKeyTile);
    const int64_t tiles = BH * a.qtiles;
    if (out != kRowsStoreP) {
        switch (gamma_kind(a.gamma)) {
            case kGammaOne: launch_attn_diag<kGammaOne>(a, out, dim3((unsigned)tiles), stream); break;
            case kGammaPow2: launch_attn_diag<kGammaPow2>(a, out, dim3((unsigned)tiles), stream); break;
            default: launch_attn_diag<kGammaAny>(a, out, dim3((unsigned)tiles), stream); break;
        }
        return hipGetLastError();
    }
    if (!apart(tiles, a.Nkv)) {
        attn_rows_kernel<kRowsStoreP, kGammaOne><<<dim3((unsigned)tiles), 256, 0, stream>>>(a);
        return hipGetLastError();
    }
    rows_norm_kernel<<<dim3((unsigned)tiles), 256, 0, stream>>>(a);
    if (hipError_t e = hipGetLastError()) return e;
    rows_write_kernel<<<dim3((unsigned)(tiles * a.runs)), 256, 0, stream>>>(a);
    return hipGetLastError();
}

template <int kGamma>
static void launch_diag(const RowsumDiagArgs& a, int64_t rows, int rule, hipStream_t stream) {
    if (rule == kRuleUos)
        rowsum_diag_kernel<kRuleUos, kGamma><<<dim3((unsigned)rows), 256, 0, stream>>>(a);
    else
        rowsum_diag_kernel<kRuleOcp, kGamma><<<dim3((unsigned)rows), 256, 0, stream>>>(a);
}

hipError_t launch_rowsum_diag(const RowsumDiagArgs& a, int64_t rows, int rule, hipStream_t stream) {
    if (rows == 0) return hipSuccess;
    switch (gamma_kind(a.gamma)) {
        case kGammaOne: launch_diag<kGammaOne>(a, rows, rule, stream); break;
        case kGammaPow2: launch_diag<kGammaPow2>(a, rows, rule, stream); break;
        default: launch_diag<kGammaAny>(a, rows, rule, stream); break;
    }
    return hipGetLastError();
}

}  // namespace mxattn
